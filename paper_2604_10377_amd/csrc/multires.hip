// Two uses of the solve beyond one square map per pair (Eq. (1), Sec. 3.1):
//
// 1. Several spectral resolutions from one projection.  Multi-resolution
//    pipelines project the features once onto the first k_max eigenfunctions
//    and compute maps at several smaller resolutions.  Resolution (k_x', k_y')
//    is the solve of Eqs. (4)-(7) restricted to the first k_x' source and k_y'
//    target eigenpairs: the leading k_x' rows of A, the leading k_y' rows of B,
//    the eigenvalues truncated alike (the mask, and the resolvent normaliser,
//    are those of the truncated spectra).  Its normal products are the leading
//    blocks of those of a larger resolution, entry by entry the same sums, so
//    where one resolution covers the others the products are formed once for
//    it, and the others' blocks are gathered from them.  Otherwise the leading
//    rows of A and B are gathered per resolution and the batched solve runs as
//    for a plain call.
//
// 2. The projector given directly.  Eq. (1) writes A = Phi^+ F with the
//    pseudo-inverse; a caller holding Phi^+ (k x n) passes its transpose P
//    [n][k] (the same array read column-major), and A = P^T F, dF = P dA are
//    the projection kernels with unit vertex weights (a weight array of ones
//    written into the workspace by a fill kernel, multiplication by 1 being
//    exact).
#include "../../include/fmap.h"

#include <algorithm>
#include <vector>

#include "fmap_launch.h"

namespace fmap {

namespace {

struct RowCopy {              // dst[p][r][c] = src[p][r][c] for r < rows, c < cols, pairs p; dst dense
    const float *src;
    float *dst;
    int64_t src_pair_stride;  // floats between pairs in src
    int src_row_stride;       // and between rows
    int rows, cols;
};

// Up to 8 resolutions of four arrays (1.3 KB of kernel arguments)
constexpr int MAX_COPIES = 32;
struct RowCopies {
    RowCopy job[MAX_COPIES];
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct ResLayout {
    size_t A, B, ex, ey, info, solve, total;
};

ResLayout res_layout(int64_t P, int64_t kx, int64_t ky, int64_t d)
{
    ResLayout L;
    size_t off = 0;
    L.A = off;
    off += align256((size_t)P * kx * d * sizeof(float));
    L.B = off;
    off += align256((size_t)P * ky * d * sizeof(float));
    L.ex = off;
    off += align256((size_t)P * kx * sizeof(float));
    L.ey = off;
    off += align256((size_t)P * ky * sizeof(float));
    L.info = off;
    off += align256((size_t)P * ky * sizeof(int32_t));
    L.solve = off;
    off += solve_workspace_layout(P, kx, ky, d).total;
    L.total = off;
    return L;
}

}  // namespace

// One wave per row: the row's pair and place are split once, in scalar registers, and the lanes walk the columns
// (an element-wise copy divided two 64-bit indices per float: 6 us for 5 MB, bound by that).
__global__ __launch_bounds__(256) void copy_rows_kernel(RowCopies js, int64_t P)
{
    const RowCopy &j = js.job[blockIdx.y];
    const int64_t rows = P * j.rows;
    for (int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); w < rows;
         w += (int64_t)gridDim.x * 4) {
        const int64_t p = w / j.rows, r = w - p * j.rows;
        const float *src = j.src + p * j.src_pair_stride + r * j.src_row_stride;
        float *dst = j.dst + w * j.cols;
        for (int c = threadIdx.x & 63; c < j.cols; c += 64) dst[c] = src[c];
    }
}

__global__ __launch_bounds__(256) void fill_ones_kernel(float *__restrict__ x, int64_t n)
{
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) x[e] = 1.f;
}

static unsigned blocks_for(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096)); }

size_t resolutions_workspace_bytes(int64_t P, int64_t kx, int64_t ky, int64_t d, int nres, const int32_t *kxs,
                                   const int32_t *kys)
{
    size_t mx = 0;
    for (int r = 0; r < nres; ++r) mx = std::max(mx, res_layout(P, kxs[r], kys[r], d).total);
    (void)kx;
    (void)ky;
    return mx;
}

static void launch_copies(const RowCopies &js, int n, int64_t P, hipStream_t st)
{
    int64_t rows = 1;
    for (int i = 0; i < n; ++i) rows = std::max<int64_t>(rows, P * js.job[i].rows);
    hipLaunchKernelGGL(copy_rows_kernel, dim3((unsigned)std::min<int64_t>((rows + 3) / 4, 4096), n), dim3(256), 0, st,
                       js, P);
}

hipError_t launch_solve_resolutions(const float *A, const float *B, const float *ex, const float *ey, const float *lam,
                                    int mask_kind, float gamma, int64_t P, int64_t kx, int64_t ky, int64_t d, int nres,
                                    const int32_t *kxs, const int32_t *kys, float *const *C, int32_t *const *info,
                                    void *ws, hipStream_t st)
{
    char *base = (char *)ws;
    // the resolution that covers all others, if there is one
    const int64_t mx = *std::max_element(kxs, kxs + nres), my = *std::max_element(kys, kys + nres);
    int top = -1;
    for (int r = 0; r < nres; ++r)
        if (kxs[r] == mx && kys[r] == my) top = r;
    const bool in_place = mx == kx && my == ky;
    // A and B in place take the products' 16-byte loads only if aligned; gathered rows always do
    const bool aligned = !in_place || d % 4 != 0 || ((((uintptr_t)A) | ((uintptr_t)B)) & 15) == 0;
    if (nres > 1 && top >= 0 && aligned) {
        const ResLayout L = res_layout(P, mx, my, d);
        const SolveWs S = solve_workspace_layout(P, mx, my, d);
        char *sb = base + L.solve;
        float *K = (float *)(sb + S.K), *R = (float *)(sb + S.R), *tiles = (float *)(sb + S.tiles);
        const float *At = A, *Bt = B;
        if (!in_place) {
            RowCopies js{};
            js.job[0] = RowCopy{A, (float *)(base + L.A), kx * d, (int)d, (int)mx, (int)d};
            js.job[1] = RowCopy{B, (float *)(base + L.B), ky * d, (int)d, (int)my, (int)d};
            launch_copies(js, 2, P, st);
            At = js.job[0].dst;
            Bt = js.job[1].dst;
        }
        launch_gram(At, Bt, P, mx, my, d, true, K, R, st);
        // The blocks of the others and their spectra go where a refinement would keep its float64 products: room for
        // any one resolution, mostly for all, gathered by one launch for as many as fit.
        float *room = (float *)(sb + S.K64);
        const size_t cap = (S.dlam - S.K64) / sizeof(float);
        for (int r0 = 0; r0 < nres;) {
            RowCopies js{};
            int n = 0, r1 = r0;
            size_t used = 0;
            for (; r1 < nres && n + 4 <= MAX_COPIES; ++r1) {
                if (kxs[r1] == mx && kys[r1] == my && in_place) continue;
                const size_t x = kxs[r1], y = kys[r1], need = (size_t)P * (x * x + y * x + x + y);
                if (used + need > cap) break;
                float *o = room + used;
                js.job[n++] = RowCopy{K, o, mx * mx, (int)mx, (int)x, (int)x};
                js.job[n++] = RowCopy{R, o + P * x * x, my * mx, (int)mx, (int)y, (int)x};
                js.job[n++] = RowCopy{ex, o + P * (x * x + y * x), kx, (int)kx, 1, (int)x};
                js.job[n++] = RowCopy{ey, o + P * (x * x + y * x + x), ky, (int)ky, 1, (int)y};
                used += need;
            }
            if (n > 0) launch_copies(js, n, P, st);
            n = 0;
            for (; r0 < r1; ++r0) {
                const bool whole = kxs[r0] == mx && kys[r0] == my && in_place;
                int32_t *inf = (info && info[r0]) ? info[r0] : (int32_t *)(base + L.info);
                const RowCopy *j = js.job + n;
                launch_solve_products(whole ? K : j[0].dst, whole ? R : j[1].dst, whole ? ex : j[2].dst,
                                      whole ? ey : j[3].dst, lam, mask_kind, gamma, P, kxs[r0], kys[r0], C[r0], inf,
                                      tiles, st);
                n += whole ? 0 : 4;
            }
        }
        return hipGetLastError();
    }
    for (int r = 0; r < nres; ++r) {
        const int64_t kxr = kxs[r], kyr = kys[r];
        const ResLayout L = res_layout(P, kxr, kyr, d);
        int32_t *inf = (info && info[r]) ? info[r] : (int32_t *)(base + L.info);
        const float *Ar = A, *Br = B, *exr = ex, *eyr = ey;
        if (kxr != kx || kyr != ky) {
            RowCopies js{};
            js.job[0] = RowCopy{A, (float *)(base + L.A), kx * d, (int)d, (int)kxr, (int)d};
            js.job[1] = RowCopy{B, (float *)(base + L.B), ky * d, (int)d, (int)kyr, (int)d};
            js.job[2] = RowCopy{ex, (float *)(base + L.ex), kx, (int)kx, 1, (int)kxr};
            js.job[3] = RowCopy{ey, (float *)(base + L.ey), ky, (int)ky, 1, (int)kyr};
            launch_copies(js, 4, P, st);
            Ar = js.job[0].dst;
            Br = js.job[1].dst;
            exr = js.job[2].dst;
            eyr = js.job[3].dst;
        }
        hipError_t e = launch_solve(Ar, Br, exr, eyr, lam, mask_kind, gamma, P, kxr, kyr, d, 0, 0.f, C[r], nullptr, inf,
                                    nullptr, base + L.solve, st);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

size_t project_pinv_workspace_bytes(int64_t batch, int64_t n, int64_t k, int64_t d, int32_t dtype)
{
    return align256((size_t)batch * n * sizeof(float)) + project_workspace_bytes(batch, n, k, d, dtype);
}

hipError_t launch_project_pinv(const void *P, const void *feat, int32_t dtype, int64_t batch, int64_t n, int64_t k,
                               int64_t d, float *A, void *ws, hipStream_t st)
{
    float *ones = (float *)ws;
    hipLaunchKernelGGL(fill_ones_kernel, dim3(blocks_for(batch * n)), dim3(256), 0, st, ones, batch * n);
    void *rest = (char *)ws + align256((size_t)batch * n * sizeof(float));
    return launch_project(P, ones, feat, dtype, batch, n, k, d, A, rest, st);
}

hipError_t launch_project_pinv_backward(const void *P, int32_t dtype, const float *dA, int64_t batch, int64_t n,
                                        int64_t k, int64_t d, float *dF, void *ws, hipStream_t st)
{
    float *ones = (float *)ws;
    hipLaunchKernelGGL(fill_ones_kernel, dim3(blocks_for(batch * n)), dim3(256), 0, st, ones, batch * n);
    return launch_project_backward(P, ones, dtype, dA, batch, n, k, d, dF, st);
}

}  // namespace fmap

namespace {

bool dims_ok(int64_t v) { return v >= 1 && v < ((int64_t)1 << 30); }

fmap_status res_args_ok(int64_t kx, int64_t ky, int32_t nres, const int32_t *kxs, const int32_t *kys)
{
    if (nres < 1 || nres > 64) return FMAP_ERR_SHAPE;
    if (!kxs || !kys) return FMAP_ERR_NULL;
    for (int r = 0; r < nres; ++r)
        if (kxs[r] < 1 || kys[r] < 1 || kxs[r] > kx || kys[r] > ky) return FMAP_ERR_SHAPE;
    return FMAP_OK;
}

}  // namespace

extern "C" {

size_t fmap_solve_resolutions_workspace_bytes(int64_t pairs, int64_t kx, int64_t ky, int64_t d, int32_t nres,
                                              const int32_t *kxs, const int32_t *kys)
{
    if (!dims_ok(pairs) || !dims_ok(kx) || !dims_ok(ky) || !dims_ok(d)) return 0;
    if (res_args_ok(kx, ky, nres, kxs, kys) != FMAP_OK) return 0;
    return fmap::resolutions_workspace_bytes(pairs, kx, ky, d, nres, kxs, kys);
}

fmap_status fmap_solve_resolutions(const float *A, const float *B, const float *evals_x, const float *evals_y,
                                   const float *lambda, int32_t mask_kind, float gamma, int64_t pairs, int64_t kx,
                                   int64_t ky, int64_t d, int32_t nres, const int32_t *kxs, const int32_t *kys,
                                   float *const *C, int32_t *const *info, void *workspace, size_t workspace_bytes,
                                   void *stream)
{
    if (!A || !B || !evals_x || !evals_y || !lambda || !C) return FMAP_ERR_NULL;
    if (!dims_ok(pairs) || !dims_ok(kx) || !dims_ok(ky) || !dims_ok(d)) return FMAP_ERR_SHAPE;
    if (mask_kind != FMAP_MASK_LAPLACIAN && mask_kind != FMAP_MASK_RESOLVENT) return FMAP_ERR_VALUE;
    if (mask_kind == FMAP_MASK_RESOLVENT && !(gamma > 0.f && gamma < 1e30f)) return FMAP_ERR_VALUE;
    if (kx > fmap_max_k() || ky > fmap_max_k()) return FMAP_ERR_UNSUPPORTED;
    if (pairs * ky > ((int64_t)1 << 30) || pairs * kx * d > ((int64_t)1 << 40)) return FMAP_ERR_SHAPE;
    const fmap_status a = res_args_ok(kx, ky, nres, kxs, kys);
    if (a != FMAP_OK) return a;
    for (int r = 0; r < nres; ++r)
        if (!C[r]) return FMAP_ERR_NULL;
    const size_t need = fmap::resolutions_workspace_bytes(pairs, kx, ky, d, nres, kxs, kys);
    if (!workspace || workspace_bytes < need) return FMAP_ERR_WORKSPACE;
    return fmap::launch_solve_resolutions(A, B, evals_x, evals_y, lambda, mask_kind, gamma, pairs, kx, ky, d, nres,
                                          kxs, kys, C, info, workspace, (hipStream_t)stream) == hipSuccess
               ? FMAP_OK
               : FMAP_ERR_HIP;
}

size_t fmap_project_pinv_workspace_bytes(int64_t batch, int64_t n, int64_t k, int64_t d, int32_t in_dtype)
{
    if (!dims_ok(batch) || !dims_ok(n) || !dims_ok(k) || !dims_ok(d)) return 0;
    return fmap::project_pinv_workspace_bytes(batch, n, k, d, in_dtype);
}

fmap_status fmap_project_pinv(const void *pinv_t, const void *feat, int32_t in_dtype, int64_t batch, int64_t n,
                              int64_t k, int64_t d, float *A, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!pinv_t || !feat || !A) return FMAP_ERR_NULL;
    if (in_dtype != FMAP_F32 && in_dtype != FMAP_BF16) return FMAP_ERR_DTYPE;
    if (!dims_ok(batch) || !dims_ok(n) || !dims_ok(k) || !dims_ok(d)) return FMAP_ERR_SHAPE;
    if (n * k > ((int64_t)1 << 31) || n * d > ((int64_t)1 << 31) || batch * n > ((int64_t)1 << 34))
        return FMAP_ERR_SHAPE;
    if (!workspace || workspace_bytes < fmap::project_pinv_workspace_bytes(batch, n, k, d, in_dtype))
        return FMAP_ERR_WORKSPACE;
    return fmap::launch_project_pinv(pinv_t, feat, in_dtype, batch, n, k, d, A, workspace, (hipStream_t)stream) ==
                   hipSuccess
               ? FMAP_OK
               : FMAP_ERR_HIP;
}

fmap_status fmap_project_pinv_backward(const void *pinv_t, int32_t pinv_dtype, const float *dA, int64_t batch,
                                       int64_t n, int64_t k, int64_t d, float *dF, void *workspace,
                                       size_t workspace_bytes, void *stream)
{
    if (!pinv_t || !dA || !dF) return FMAP_ERR_NULL;
    if (pinv_dtype != FMAP_F32 && pinv_dtype != FMAP_BF16) return FMAP_ERR_DTYPE;
    if (!dims_ok(batch) || !dims_ok(n) || !dims_ok(k) || !dims_ok(d)) return FMAP_ERR_SHAPE;
    if (n * k > ((int64_t)1 << 31) || n * d > ((int64_t)1 << 31) || batch * n > ((int64_t)1 << 34))
        return FMAP_ERR_SHAPE;
    if (!workspace || workspace_bytes < (size_t)batch * n * sizeof(float)) return FMAP_ERR_WORKSPACE;
    return fmap::launch_project_pinv_backward(pinv_t, pinv_dtype, dA, batch, n, k, d, dF, workspace,
                                              (hipStream_t)stream) == hipSuccess
               ? FMAP_OK
               : FMAP_ERR_HIP;
}

}  // extern "C"
