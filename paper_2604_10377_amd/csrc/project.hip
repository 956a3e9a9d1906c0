// Spectral projection, Eq. (1) read as the mass-weighted pseudo-inverse:
//     A[b] = Phi[b]^T diag(M[b]) F[b]          (forward)
//     dF[b] = diag(M[b]) Phi[b] dA[b]           (its adjoint)
//
// Both are tall-skinny contractions over vertex-major (n-major) arrays.  This
// file holds the general kernels, on the float32 matrix cores
// (v_mfma_f32_32x32x2f32) for any size, type and alignment, the sums of the
// forward's chunks, and the dispatch: most float32 calls run on the split
// kernels (project_short.hip, project_tall.hip, project_back.hip; the sliced one
// and the bf16 ones in project_mc.hip).
//
// Forward: the reduction over n is split into `nsplit` chunks.  A workgroup
// (4 waves) owns one (shape, chunk, k-block, d-block); each wave owns an
// MT*32 x NT*32 accumulator tile.  Per matrix-core step a lane reads one basis
// value and one feature value of vertex v0 + lane/32: 32 consecutive floats of
// a vertex row per half-wave, so every Phi and F byte is read from HBM once.
// Partial sums go to a workspace and a second kernel adds the chunks in a fixed
// order (deterministic, and chunked accumulation keeps the float32 error of a
// 1e5-term sum small).
//
// Backward: rows of dF are vertices; a wave owns 32 vertices x NT*32 feature
// columns and contracts over k.  The two lane halves take the two halves of
// the k range, so a lane walks along its own basis row.
#include <algorithm>

#include "fmap_device.h"
#include "fmap_launch.h"
#include "fmap_lds.h"
#include "proj_general.h"

namespace fmap {

template <typename T, int MT, int NT, int U>
__global__ __launch_bounds__(256) void proj_fwd_kernel(const T *__restrict__ phi, const float *__restrict__ mass,
                                                       const T *__restrict__ feat, int n, int k, int d, int nsplit,
                                                       int chunk, int kblocks, int dblocks,
                                                       float *__restrict__ out)
{
    int bid = blockIdx.x;
    const int db = bid % dblocks;
    bid /= dblocks;
    const int kb = bid % kblocks;
    bid /= kblocks;
    const int split = bid % nsplit;
    const int s = bid / nsplit;
    const int v0 = split * chunk;
    const int v1 = min(n, v0 + chunk);
    proj_fwd_tile<T, MT, NT, U>(phi + (size_t)s * n * k, mass + (size_t)s * n, feat + (size_t)s * n * d, k, d, v0, v1,
                                kb * (MT * 32), (db * 4 + (threadIdx.x >> 6)) * (NT * 32),
                                out + ((size_t)s * nsplit + split) * (size_t)k * d);
}

// Persistent forward over a table of work items (uneven shapes): each workgroup
// takes items blockIdx.x, blockIdx.x + gridDim.x, ...
template <int MT, int NT, int U>
__global__ __launch_bounds__(256) void proj_fwd_items_kernel(const FwdItem *__restrict__ items, int nitems)
{
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const FwdItem w = items[it];
        proj_fwd_tile<float, MT, NT, U>(global_ptr(w.phi), global_ptr(w.mass), global_ptr(w.feat), w.k, w.d, w.v0, w.v1,
                                        w.kbase, w.dbase + (threadIdx.x >> 6) * (NT * 32), global_ptr(w.out));
    }
}

// A[s] = sum over chunks (in chunk order) of part[s][chunk].  Four consecutive
// elements per thread (k*d % 4 == 0, 16-byte aligned buffers); the chunks are
// read in groups of RG, all loads of a group in flight before the adds.
constexpr int RG = 8;

__global__ __launch_bounds__(256) void proj_reduce_kernel(const float *__restrict__ part, int nsplit, int64_t kd,
                                                          int64_t total, float *__restrict__ A)
{
    const int64_t q4 = kd / 4, tq = total / 4;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < tq; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t s = e / q4, r = e - s * q4;
        const f32x4 *p = reinterpret_cast<const f32x4 *>(part + (size_t)s * nsplit * kd) + r;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        for (int c0 = 0; c0 < nsplit; c0 += RG) {
            f32x4 v[RG];
#pragma unroll
            for (int u = 0; u < RG; ++u) v[u] = p[(size_t)min(c0 + u, nsplit - 1) * q4];
#pragma unroll
            for (int u = 0; u < RG; ++u)
                if (c0 + u < nsplit) acc += v[u];
        }
        reinterpret_cast<f32x4 *>(A)[e] = acc;
    }
}

// The same sum where few elements have many chunks: wave w of a workgroup takes the w-th quarter of the chunks, and the
// four sums are added in that order.  One wave alone is a chain of memory round trips, 0.7 us per RG chunks.  The call, us:
// 1 shape of n = 20000, k = 4, d = 512 27.5, 18.9 so; 4 of n = 49998, k = 4, d = 16 38.1, 33.1.  Taken up to one workgroup per
// CU (with two 0.98 to 1.04 of the time of the call) and above 64 chunks: with 9 to 64 the call alone gains 4% to 11%, but a
// map of one pair, bound by its launches, does not (37.2, 37.6 us).  For k <= 64 alone: with more, C can hang on the last bits
// of A.
__global__ __launch_bounds__(256) void proj_reduce_parts_kernel(const float *__restrict__ part, int nsplit, int64_t kd,
                                                                int64_t total, float *__restrict__ A)
{
    __shared__ f32x4 s_sum[3][64];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t q4 = kd / 4, tq = total / 4, e = (int64_t)blockIdx.x * 64 + lane;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (e < tq) {
        const int64_t s = e / q4, r = e - s * q4;
        const f32x4 *p = reinterpret_cast<const f32x4 *>(part + (size_t)s * nsplit * kd) + r;
        const int end = (int)((int64_t)nsplit * (w + 1) / 4);
        for (int c0 = (int)((int64_t)nsplit * w / 4); c0 < end; c0 += RG) {
            f32x4 v[RG];
#pragma unroll
            for (int u = 0; u < RG; ++u) v[u] = p[(size_t)min(c0 + u, end - 1) * q4];
#pragma unroll
            for (int u = 0; u < RG; ++u)
                if (c0 + u < end) acc += v[u];
        }
    }
    if (w > 0) s_sum[w - 1][lane] = acc;
    __syncthreads();
    if (w == 0 && e < tq)
        reinterpret_cast<f32x4 *>(A)[e] = acc + s_sum[0][lane] + s_sum[1][lane] + s_sum[2][lane];
}

// The same sum, one element per thread, for any k*d and alignment.
__global__ __launch_bounds__(256) void proj_reduce1_kernel(const float *__restrict__ part, int nsplit, int64_t kd,
                                                           int64_t total, float *__restrict__ A)
{
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t s = e / kd, r = e - s * kd;
        const float *p = part + (size_t)s * nsplit * kd + r;
        float acc = 0.f;
        for (int c = 0; c < nsplit; ++c) acc += p[(size_t)c * kd];
        A[e] = acc;
    }
}

// Backward: one workgroup owns a column block of NT*32 feature columns and RB
// consecutive blocks of 128 vertices of one shape (32 per wave).  The rows
// [j0, j0+KC) of dA restricted to the column block are staged in LDS once per
// chunk (once per workgroup when k <= KC); matrix-core step t consumes basis
// columns j0 + 2t + half, so the two lane halves read adjacent LDS rows, which
// the padded row stride puts on disjoint banks.  Each lane's basis values are
// loaded for the whole chunk before the multiplies.
constexpr int BWD_KC = 64;

__host__ __device__ constexpr int bwd_stride(int nt) { return (nt * 32) % 64 == 32 ? nt * 32 : nt * 32 + 32; }

// RB consecutive blocks of 128 vertices starting at vertex r0 of one shape, for
// the column block [dbase, dbase + NT*32).  Must be called by all 256 threads.
template <typename T, int NT>
__device__ __forceinline__ void proj_bwd_rows(float *sG, const T *__restrict__ P, const float *__restrict__ Mv,
                                              const float *__restrict__ G, float *__restrict__ O, int n, int k, int d,
                                              int r0, int RB, int dbase)
{
    constexpr int LD = bwd_stride(NT);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    int cols[NT];
    bool cok[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        cols[nt] = dbase + nt * 32 + l32;
        cok[nt] = cols[nt] < d;
    }
    const int nchunks = (k + BWD_KC - 1) / BWD_KC;
    auto stage = [&](int j0, int kc) {
        const int kc2 = (kc + 1) & ~1;
        batched_for<8>(
            threadIdx.x, kc2 * NT * 32, 256,
            [&](int e) {
                const int jj = e / (NT * 32), cc = e - jj * (NT * 32);
                return G[(size_t)(j0 + min(jj, kc - 1)) * d + min(dbase + cc, d - 1)];
            },
            [&](int e, float g) {
                const int jj = e / (NT * 32), cc = e - jj * (NT * 32);
                sG[jj * LD + cc] = (jj < kc && dbase + cc < d) ? g : 0.f;
            });
    };
    __syncthreads();  // sG may still be read by a previous call
    if (nchunks == 1) {
        stage(0, k);
        __syncthreads();
    }
    for (int rb = 0; rb < RB; ++rb) {
        const int row0 = r0 + (rb * 4 + wave) * 32;
        const int row = row0 + l32;
        const bool rok = row < n;
        const float m = rok ? Mv[row] : 0.f;
        f32x16 acc[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[nt] = zero16();
        for (int ch = 0; ch < nchunks; ++ch) {
            const int j0 = ch * BWD_KC;
            const int kc = min(BWD_KC, k - j0);
            if (nchunks > 1) {
                __syncthreads();
                stage(j0, kc);
                __syncthreads();
            }
            float a[BWD_KC / 2];
#pragma unroll
            for (int t = 0; t < BWD_KC / 2; ++t) {
                const int jj = 2 * t + half;
                a[t] = (rok && jj < kc) ? load_elem(P, (size_t)row * k + j0 + jj) * m : 0.f;
            }
            const int steps = (kc + 1) >> 1;
#pragma unroll
            for (int t = 0; t < BWD_KC / 2; ++t) {
                if (t < steps) {
                    const float *g = sG + (2 * t + half) * LD;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[nt] = mfma32x32x2(a[t], g[nt * 32 + l32], acc[nt]);
                }
            }
        }
        if (row0 < n) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int rr = row0 + acc32_row(r, lane);
                    if (rr < n && cok[nt]) O[(size_t)rr * d + cols[nt]] = acc[nt][r];
                }
        }
    }
}

template <typename T, int NT>
__global__ __launch_bounds__(256) void proj_bwd_kernel(const T *__restrict__ phi, const float *__restrict__ mass,
                                                       const float *__restrict__ dA, int n, int k, int d,
                                                       int rgroups, int RB, int dblocks, float *__restrict__ dF)
{
    extern __shared__ float sG[];  // [min(k,KC) rounded to even][bwd_stride(NT)]
    int bid = blockIdx.x;
    const int db = bid % dblocks;
    bid /= dblocks;
    const int rg = bid % rgroups;
    const int s = bid / rgroups;
    proj_bwd_rows<T, NT>(sG, phi + (size_t)s * n * k, mass + (size_t)s * n, dA + (size_t)s * k * d,
                         dF + (size_t)s * n * d, n, k, d, rg * RB * 128, RB, db * (NT * 32));
}

// Persistent backward over a table of work items (uneven shapes).
template <int NT>
__global__ __launch_bounds__(256) void proj_bwd_items_kernel(const BwdItem *__restrict__ items, int nitems)
{
    extern __shared__ float sG[];
    for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
        const BwdItem w = items[it];
        proj_bwd_rows<float, NT>(sG, global_ptr(w.phi), global_ptr(w.mass), global_ptr(w.dA), global_ptr(w.dF), w.n, w.k, w.d, w.r0, w.rb, w.dbase);
    }
}

// ---------------------------------------------------------------------------
// Host-side launch planning
// ---------------------------------------------------------------------------

static int device_cu_count()
{
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cus[dev] == 0) {
        int c = 0;
        if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0) c = 256;
        cus[dev] = c;
    }
    return cus[dev];
}

ProjPlan plan_project(int64_t batch, int64_t n, int64_t k, int64_t d, int32_t dtype)
{
    ProjPlan p;
    p.MT = k <= 32 ? 1 : 2;
    p.kblocks = (int)((k + 32 * p.MT - 1) / (32 * p.MT));
    // 4 waves per workgroup along d; NT 32-column tiles per wave.
    p.NT = d <= 128 ? 1 : 2;
    p.dblocks = (int)((d + 128 * p.NT - 1) / (128 * p.NT));
    // Split the vertex sum so that the grid has ~2 workgroups per CU, chunks of >= 512 vertices.
    const int64_t tiles = batch * p.kblocks * p.dblocks;
    int64_t want = (2 * device_cu_count() + tiles - 1) / tiles;
    int64_t maxsplit = (n + 511) / 512;
    int64_t ns = want < maxsplit ? want : maxsplit;
    if (ns < 1) ns = 1;
    int64_t chunk = (n + ns - 1) / ns;
    chunk = (chunk + 15) & ~(int64_t)15;
    ns = (n + chunk - 1) / chunk;
    p.nsplit = (int)ns;
    p.chunk = (int)chunk;
    (void)dtype;
    return p;
}

static bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }

// The chunk budget that workspaces are sized for: the chunks of the general and bf16 kernels and, for d % 4 == 0 and
// n % 4 == 0, two workgroups per CU over 64-row slices and 256-column blocks (one for odd k <= 64).  The sizes it gives
// decide which calls the built-in scratch array takes, so they stay as they are.
static int64_t budget_nsplit(int64_t batch, int64_t n, int64_t k, int64_t d, int32_t dtype)
{
    int64_t ns = plan_project(batch, n, k, d, dtype).nsplit;
    if (dtype == 1 && bf16_fwd_shape_ok(n, k, d) && n % 4 == 0)
        ns = std::max<int64_t>(ns, bf16_fwd_nsplit(batch, n, k, d));
    if (dtype == 0 && k <= kMaxK && d % 4 == 0 && n % 4 == 0 && n >= 128) {
        const int64_t blocks = batch * ((d + 255) / 256), quarter = (n + 31) / 32 / 4, cus = device_cu_count();
        if (k <= 64) ns = std::max(ns, std::min((cus + blocks - 1) / blocks, quarter));
        if (k > 64 ? k % 4 == 0 : k >= 4 && k % 2 == 0)
            ns = std::max(ns, std::min(2 * cus / (blocks * ((k + 63) / 64)), quarter));
    }
    return ns;
}

// Chunks of the split kernels: within that budget, or more while the partial sums fit the built-in scratch array (a few
// shapes of any n then still spread over the chip, and no call outgrows the array).
static int64_t split_cap(int64_t batch, int64_t n, int64_t k, int64_t d, int32_t dtype)
{
    const int64_t fit = (int64_t)(32u << 20) / (batch * k * d * (int64_t)sizeof(float));
    return std::max(fit, budget_nsplit(batch, n, k, d, dtype));
}
static int bf16_chunks(int64_t batch, int64_t n, int64_t k, int64_t d)
{
    return (int)std::min<int64_t>(bf16_fwd_nsplit(batch, n, k, d), split_cap(batch, n, k, d, 1));
}
static int tall_chunks(int64_t batch, int64_t n, int64_t k, int64_t d)
{
    return tall_nsplit(batch, n, k, d, split_cap(batch, n, k, d, 0));
}
static int short_chunks(int64_t batch, int64_t n, int64_t k, int64_t d)
{
    return (int)std::min<int64_t>(short_nsplit(batch, n, k, d), split_cap(batch, n, k, d, 0));
}

size_t project_workspace_bytes(int64_t batch, int64_t n, int64_t k, int64_t d, int32_t dtype)
{
    int64_t ns = budget_nsplit(batch, n, k, d, dtype);
    if (dtype == 0 && tall_shape_ok(n, k, d)) ns = std::max<int64_t>(ns, tall_chunks(batch, n, k, d));
    if (dtype == 0 && short_shape_ok(n, k, d)) ns = std::max<int64_t>(ns, short_chunks(batch, n, k, d));
    if (dtype == 1 && bf16_fwd_shape_ok(n, k, d)) ns = std::max<int64_t>(ns, bf16_chunks(batch, n, k, d));
    if (ns <= 1) return 0;
    return (size_t)batch * ns * k * d * sizeof(float);
}

template <typename T, int MT, int NT>
static void launch_fwd_t(const void *phi, const float *mass, const void *feat, int64_t batch, int64_t n, int64_t k,
                         int64_t d, const ProjPlan &p, float *out, hipStream_t st)
{
    const unsigned grid = (unsigned)(batch * p.nsplit * p.kblocks * p.dblocks);
    hipLaunchKernelGGL((proj_fwd_kernel<T, MT, NT, 8>), dim3(grid), dim3(256), 0, st, (const T *)phi, mass,
                       (const T *)feat, (int)n, (int)k, (int)d, p.nsplit, p.chunk, p.kblocks, p.dblocks, out);
}

template <typename T>
static void launch_fwd_dt(const void *phi, const float *mass, const void *feat, int64_t batch, int64_t n, int64_t k,
                          int64_t d, const ProjPlan &p, float *out, hipStream_t st)
{
    if (p.MT == 1 && p.NT == 1) launch_fwd_t<T, 1, 1>(phi, mass, feat, batch, n, k, d, p, out, st);
    else if (p.MT == 1) launch_fwd_t<T, 1, 2>(phi, mass, feat, batch, n, k, d, p, out, st);
    else if (p.NT == 1) launch_fwd_t<T, 2, 1>(phi, mass, feat, batch, n, k, d, p, out, st);
    else launch_fwd_t<T, 2, 2>(phi, mass, feat, batch, n, k, d, p, out, st);
}

// Per-shape reduction of partial slots (uneven shapes), fixed chunk order.  Four elements per thread and the chunks in
// groups of RG, all loads of a group in flight before the adds: one element per thread and one load at a time, the
// kernel was a chain of memory round trips, one per chunk (32 shapes of 2000 to 20000 vertices, k = 30 to 120,
// d = 256: 38.6 us before, 11.9 us now).
__global__ __launch_bounds__(256) void reduce_items_kernel(const RedItem *__restrict__ items, int nitems)
{
    for (int it = blockIdx.y; it < nitems; it += gridDim.y) {
        const RedItem w = items[it];
        const float *part = global_ptr(w.part);
        float *A = global_ptr(w.A), *U = global_ptr(w.A_user);
        if (w.kd % 4 == 0 && ((uintptr_t)part & 15) == 0 && ((uintptr_t)A & 15) == 0 && ((uintptr_t)U & 15) == 0) {
            const int q4 = w.kd / 4;
            for (int e = blockIdx.x * 256 + threadIdx.x; e < q4; e += gridDim.x * 256) {
                const f32x4 *p = reinterpret_cast<const f32x4 *>(part) + e;
                f32x4 acc = {0.f, 0.f, 0.f, 0.f};
                for (int c0 = 0; c0 < w.nchunks; c0 += RG) {
                    f32x4 v[RG];
#pragma unroll
                    for (int u = 0; u < RG; ++u) v[u] = p[(size_t)min(c0 + u, w.nchunks - 1) * q4];
#pragma unroll
                    for (int u = 0; u < RG; ++u)
                        if (c0 + u < w.nchunks) acc += v[u];
                }
                reinterpret_cast<f32x4 *>(A)[e] = acc;
                if (U) reinterpret_cast<f32x4 *>(U)[e] = acc;
            }
            continue;
        }
        for (int e = blockIdx.x * 256 + threadIdx.x; e < w.kd; e += gridDim.x * 256) {
            float acc = 0.f;
            for (int c = 0; c < w.nchunks; ++c) acc += part[(size_t)c * w.kd + e];
            A[e] = acc;
            if (U) U[e] = acc;
        }
    }
}

int device_cus() { return device_cu_count(); }

hipError_t launch_fwd_items(const FwdItem *items, int nitems, int kmax, int grid, hipStream_t st)
{
    grid = std::min(grid, nitems);
    if (kmax <= 32)
        hipLaunchKernelGGL((proj_fwd_items_kernel<1, 2, 8>), dim3(grid), dim3(256), 0, st, items, nitems);
    else
        hipLaunchKernelGGL((proj_fwd_items_kernel<2, 2, 8>), dim3(grid), dim3(256), 0, st, items, nitems);
    return hipGetLastError();
}

hipError_t launch_bwd_items(const BwdItem *items, int nitems, int kmax, int grid, hipStream_t st)
{
    grid = std::min(grid, nitems);
    const int kc = kmax < BWD_KC ? kmax : BWD_KC;
    const size_t lds = (size_t)((kc + 1) & ~1) * bwd_stride(8) * sizeof(float);
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)proj_bwd_items_kernel<8>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)(BWD_KC * bwd_stride(8) * sizeof(float)));
        attr_set = true;
    }
    hipLaunchKernelGGL((proj_bwd_items_kernel<8>), dim3(grid), dim3(256), lds, st, items, nitems);
    return hipGetLastError();
}

hipError_t launch_reduce_items(const RedItem *items, int nitems, hipStream_t st)
{
    hipLaunchKernelGGL(reduce_items_kernel, dim3(16, (unsigned)(nitems < 65535 ? nitems : 65535)), dim3(256), 0, st,
                       items, nitems);
    return hipGetLastError();
}

hipError_t launch_reduce(const float *part, int nsplit, int64_t batch, int64_t k, int64_t d, float *A,
                         bool parts, hipStream_t st)
{
    const int64_t total = batch * k * d;
    const bool vec = (k * d) % 4 == 0 && aligned16(part) && aligned16(A);
    if (parts && vec && nsplit > 8 * RG && total <= 256 * (int64_t)device_cus()) {
        hipLaunchKernelGGL(proj_reduce_parts_kernel, dim3((unsigned)((total / 4 + 63) / 64)), dim3(256), 0, st, part,
                           nsplit, (int64_t)(k * d), total, A);
        return hipGetLastError();
    }
    int64_t blocks = ((vec ? total / 4 : total) + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(vec ? proj_reduce_kernel : proj_reduce1_kernel, dim3((unsigned)blocks), dim3(256), 0, st, part,
                       nsplit, (int64_t)(k * d), total, A);
    return hipGetLastError();
}

hipError_t launch_project(const void *phi, const float *mass, const void *feat, int32_t dtype, int64_t batch, int64_t n,
                          int64_t k, int64_t d, float *A, void *ws, hipStream_t st)
{
    if (dtype == 0 && sliced_fwd_shape_ok(n, k, d) && (near_square(k, d) || tall_too_small(batch, n, k, d)) &&
        aligned16(phi) && aligned16(mass) && aligned16(feat))
        return launch_project_sliced((const float *)phi, mass, (const float *)feat, batch, n, k, d, A, ws, st);
    if (dtype == 0 && tall_shape_ok(n, k, d) && aligned16(feat) && aligned16(A) && aligned16(ws))
        return launch_project_tall((const float *)phi, mass, (const float *)feat, batch, n, k, d,
                                   tall_chunks(batch, n, k, d), A, ws, st);
    if (dtype == 0 && short_shape_ok(n, k, d) && aligned16(feat) && aligned16(A) && aligned16(ws))
        return launch_project_short((const float *)phi, mass, (const float *)feat, batch, n, k, d,
                                    short_chunks(batch, n, k, d), A, ws, st);
    if (dtype == 1 && bf16_fwd_shape_ok(n, k, d) && aligned16(phi) && aligned16(feat))
        return launch_project_bf16((const uint16_t *)phi, mass, (const uint16_t *)feat, batch, n, k, d,
                                   bf16_chunks(batch, n, k, d), A, ws, st);
    ProjPlan p = plan_project(batch, n, k, d, dtype);
    float *out = p.nsplit > 1 ? (float *)ws : A;
    if (dtype == 0) launch_fwd_dt<float>(phi, mass, feat, batch, n, k, d, p, out, st);
    else launch_fwd_dt<uint16_t>(phi, mass, feat, batch, n, k, d, p, out, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.nsplit <= 1) return e;
    return launch_reduce((const float *)ws, p.nsplit, batch, k, d, A, false, st);
}

template <typename T, int NT>
static void launch_bwd_t(const void *phi, const float *mass, const float *dA, int64_t batch, int64_t n, int64_t k,
                         int64_t d, float *dF, hipStream_t st)
{
    const int rblocks = (int)((n + 127) / 128);
    const int dblocks = (int)((d + NT * 32 - 1) / (NT * 32));
    // ~4 row blocks per workgroup, but keep >= ~1024 workgroups when the problem allows
    int RB = 4;
    while (RB > 1 && batch * dblocks * ((rblocks + RB - 1) / RB) < 1024) RB >>= 1;
    const int rgroups = (rblocks + RB - 1) / RB;
    const unsigned grid = (unsigned)(batch * rgroups * dblocks);
    const int kc = (int)(k < BWD_KC ? k : BWD_KC);
    const size_t lds = (size_t)((kc + 1) & ~1) * bwd_stride(NT) * sizeof(float);
    static bool attr_set = false;  // up to 64 x 288 floats (72 KB) for NT = 8
    if (!attr_set) {
        (void)hipFuncSetAttribute((const void *)proj_bwd_kernel<T, NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)(BWD_KC * bwd_stride(NT) * sizeof(float)));
        attr_set = true;
    }
    hipLaunchKernelGGL((proj_bwd_kernel<T, NT>), dim3(grid), dim3(256), lds, st, (const T *)phi, mass, dA, (int)n,
                       (int)k, (int)d, rgroups, RB, dblocks, dF);
}

// Backward for k = 1, 2, 3 in float32: a stream of dF with a few multiply-adds an entry.  A thread keeps its V columns of
// dA and walks down the vertices; the rows a workgroup writes at a time are adjacent, so its stores are one run of
// memory whatever d is.  Bound by the writes (5.4 to 6.2 TB/s).  On the general kernel, whose matrix tiles are made for 32
// columns of the basis and more, and here: 16 shapes of n = 5000, k = 3, d = 256 25.7 -> 15.1 us; k = 2, d = 300 42 -> 17 us; 4
// of n = 49998, k = 2, d = 16 18.5 -> 4.9 us.  Ordinary stores: non-temporal ones write the lines that two rows share twice
// (d = 300 24 us).
constexpr int FEW_U = 4;  // rows whose basis values and masses are in flight together

template <int K, int V>
__global__ __launch_bounds__(256) void proj_bwd_few_kernel(const float *__restrict__ phi, const float *__restrict__ mass,
                                                           const float *__restrict__ dA, int n, int d, int per, int cblocks,
                                                           int chunks, int steps, float *__restrict__ dF)
{
    typedef float vec __attribute__((ext_vector_type(V)));
    const int cb = blockIdx.x % cblocks, q = blockIdx.x / cblocks;
    const int chunk = q % chunks, s = q / chunks;
    const int R = 256 / per, r = threadIdx.x / per, c = V * (cb * 256 + (int)threadIdx.x - r * per);
    if (r >= R || c >= d) return;
    const float *P = phi + (size_t)s * n * K, *M = mass + (size_t)s * n, *G = dA + (size_t)s * K * d + c;
    float *O = dF + (size_t)s * n * d + c;
    vec g[K];
#pragma unroll
    for (int j = 0; j < K; ++j) g[j] = *reinterpret_cast<const vec *>(G + (size_t)j * d);
    const int v0 = chunk * steps * R + r, v1 = min(n, (chunk + 1) * steps * R);
    for (int v = v0; v < v1; v += FEW_U * R) {
        float m[FEW_U], a[FEW_U][K];
#pragma unroll
        for (int u = 0; u < FEW_U; ++u) {
            const int row = min(v + u * R, n - 1);
            m[u] = M[row];
#pragma unroll
            for (int j = 0; j < K; ++j) a[u][j] = P[(size_t)row * K + j];
        }
#pragma unroll
        for (int u = 0; u < FEW_U; ++u) {
            vec o = a[u][0] * m[u] * g[0];
#pragma unroll
            for (int j = 1; j < K; ++j) o += a[u][j] * m[u] * g[j];
            if (v + u * R < v1) *reinterpret_cast<vec *>(O + (size_t)(v + u * R) * d) = o;
        }
    }
}

template <int V>
static void launch_bwd_few(const float *phi, const float *mass, const float *dA, int64_t batch, int64_t n, int64_t k,
                           int64_t d, float *dF, hipStream_t st)
{
    const int64_t groups = (d + V - 1) / V, per = std::min<int64_t>(groups, 256), cblocks = (groups + 255) / 256;
    const int64_t R = 256 / per, rows = (n + R - 1) / R;  // rows: of R vertices
    // eight workgroups per CU where that leaves them 4 to 32 rows
    const int64_t fair = batch * cblocks * rows / (8 * (int64_t)device_cus()) / FEW_U * FEW_U;
    const int64_t steps = std::min<int64_t>(std::max<int64_t>(fair, FEW_U), 32), chunks = (rows + steps - 1) / steps;
    const dim3 grid((unsigned)(batch * cblocks * chunks));
#define FMAP_FEW(K)                                                                                                   \
    hipLaunchKernelGGL((proj_bwd_few_kernel<K, V>), grid, dim3(256), 0, st, phi, mass, dA, (int)n, (int)d, (int)per,    \
                       (int)cblocks, (int)chunks, (int)steps, dF)
    if (k == 1) FMAP_FEW(1);
    else if (k == 2) FMAP_FEW(2);
    else FMAP_FEW(3);
#undef FMAP_FEW
}

hipError_t launch_project_backward(const void *phi, const float *mass, int32_t dtype, const float *dA, int64_t batch,
                                   int64_t n, int64_t k, int64_t d, float *dF, hipStream_t st)
{
    if (dtype == 0 && back_shape_ok(k, d))
        return launch_project_back((const float *)phi, mass, dA, batch, n, k, d, dF, st);
    if (dtype == 1 && bf16_bwd_shape_ok(n, k, d) && aligned16(phi) && aligned16(dF))
        return launch_project_backward_bf16((const uint16_t *)phi, mass, dA, batch, n, k, d, dF, st);
    if (dtype == 0 && k < 4) {
        if (d % 4 == 0 && aligned16(dA) && aligned16(dF)) launch_bwd_few<4>((const float *)phi, mass, dA, batch, n, k, d, dF, st);
        else launch_bwd_few<1>((const float *)phi, mass, dA, batch, n, k, d, dF, st);
        return hipGetLastError();
    }
    if (dtype == 0) {
        if (d <= 128) launch_bwd_t<float, 4>(phi, mass, dA, batch, n, k, d, dF, st);
        else launch_bwd_t<float, 8>(phi, mass, dA, batch, n, k, d, dF, st);
    } else {
        if (d <= 128) launch_bwd_t<uint16_t, 4>(phi, mass, dA, batch, n, k, d, dF, st);
        else launch_bwd_t<uint16_t, 8>(phi, mass, dA, batch, n, k, d, dF, st);
    }
    return hipGetLastError();
}

}  // namespace fmap
