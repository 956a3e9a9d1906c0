// Forward projection A = Phi^T diag(M) F (Eq. (1)) in float32 for k <= 64, any n and k, d % 4 == 0, on the float16
// matrix cores (fmap_split.h: both operands as two float16 parts, three products).
//
// Workgroup = 4 waves over a 256-column block and all (at most 64) basis rows; wave w owns block columns 64w .. 64w + 63
// (column 4m + t of the wave is column m of tile t).  Stages of 32 vertices, one matrix-core K step.  Each lane loads
// its 4 feature columns of 8 vertices straight into registers (eight 16-byte loads), two stages ahead, so the feature
// stream -- nearly all of the bytes -- needs no LDS, no barrier and no LDS round trip.  The small basis tile
// (32 x k floats) and the masses arrive by direct global->LDS loads in a ring of 3, four bytes per lane, so rows of
// any k and shapes at any offset are taken (16-byte windows needed n % 4 == 0 and k even).  Per stage wave w splits
// the basis x mass values of row tile w (rows 4R + w) and stores the parts in LDS as matrix-core operands; after a
// barrier every wave reads all four tiles.  The column blocks of one vertex chunk take consecutive ids on one XCD, so
// the basis tile they all read comes from HBM once and from that XCD's L2 afterwards.
//
// Scales (powers of two): each basis row and feature column takes one from the first stage of the chunk (a column from
// its vertices of nonzero mass), with room for values 64 times as large; one that is all zeros there borrows that of the
// wave's largest one.  The largest magnitudes are followed in registers; a chunk where one does not fit (or is infinite),
// or lies too low on a borrowed scale to keep its bits, is computed again by the general float32 routine, and so is one
// with borrowed scales and massless vertices, whose values would hide that.  (Lowering the scales and the sums inside the
// stage loop, or leaving the loop to restart it, made the register allocator spill.)
//
// What bounds it: the feature stream (5.3 TB/s with the reduction at d = 256; loads and barriers alone take 64 of the
// 69 us of 64 shapes of n = 5000, k = 50).  Measured with the reduction, against three-part bf16 operands (six
// products; the general or an LDS kernel where n % 4 != 0 or k is odd): 64 shapes of n = 5000, k = 50, d = 256
// 77 -> 74 us; of n = 5003, k = 64 152 -> 78 us; 64 of n = 5000, k = 30, d = 128 68 -> 55 us; 16 of n = 7001, k = 49,
// d = 128 57 -> 32 us; 2 of n = 4999, k = 50 65 -> 20 us.  Error against float64 4.1e-7 -> 2.9e-7 at the first shape.
#include <algorithm>

#include "fmap_lds.h"
#include "fmap_launch.h"
#include "fmap_split.h"
#include "proj_general.h"

namespace fmap {

constexpr int HS = 32;                      // vertices per stage
constexpr int HNST = 3;                     // basis stages in the LDS ring
constexpr int HFF = 8;                      // feature loads per lane per stage
constexpr int HSTAGE = 8 * 1024 + 256;      // basis tile (32 x k floats, k <= 64) + masses
constexpr int HPARTS = 2 * 4 * 64 * 16;     // split basis tile: [part][row tile][lane] of 16 bytes
constexpr size_t h2_lds() { return (size_t)HNST * HSTAGE + HPARTS + 64 * sizeof(int) + 16; }  // (+ row shifts, flags)

// BW: basis windows of 64 floats per wave and stage, 4 BW >= k / 2
template <int BW>
__device__ __forceinline__ void h2_block(const float *__restrict__ P, const float *__restrict__ Mv,
                                         const float *__restrict__ F, int k, int d, int vbeg, int vend, int dbase,
                                         float *__restrict__ O)
{
    extern __shared__ __align__(16) float smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m16 = lane & 15, g4 = lane >> 4;
    const int nst = (vend - vbeg + HS - 1) / HS;
    if (nst <= 0) return;

    char *ring = reinterpret_cast<char *>(smem);
    u32x4_t *parts = reinterpret_cast<u32x4_t *>(ring + HNST * HSTAGE);
    int *s_sh = reinterpret_cast<int *>(parts + 2 * 4 * 64);  // [64] row shifts (row 4 R + a at 16 a + R), [2] flags

    // feature role: columns fc .. fc + 3 (clamped into d; d % 4 == 0) of vertices 8 g4 .. + 7
    const int cw = wave * 64 + 4 * m16;
    const int fc = min(dbase + cw, d - 4);
    const int nw = (HS * k + 63) >> 6;  // windows of the basis tile
    auto issue = [&](int t, f32x4 (&fr)[HFF]) {
        char *S = ring + (t % HNST) * HSTAGE;
        const int v = vbeg + t * HS;
        const int rows = min(HS, vend - v);
        const float *Pv = P + (size_t)v * k;
        const int pv = rows * k - 1;  // values past the stage's rows repeat the last one (their masses are zero)
#pragma unroll
        for (int i = 0; i < BW; ++i) {
            const int w = min(4 * i + wave, nw - 1);
            __builtin_amdgcn_global_load_lds((glb_void_t *)(Pv + min(64 * w + lane, pv)), (lds_void_t *)(S + 256 * w), 4,
                                             0, 0);
        }
        __builtin_amdgcn_global_load_lds((glb_void_t *)(Mv + v + min(lane & 31, rows - 1)),
                                         (lds_void_t *)(S + 8 * 1024), 4, 0, 0);
#pragma unroll
        for (int i = 0; i < HFF; ++i)
            fr[i] = __builtin_nontemporal_load(
                reinterpret_cast<const f32x4 *>(F + (size_t)(v + min(8 * g4 + i, rows - 1)) * d + fc));
    };

    f32x4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[a][t] = f32x4{0, 0, 0, 0};
    // split role: row tile a = wave, operand lane = lane: basis row 4 m16 + wave, vertices 8 g4 .. + 7
    const int srow = 4 * m16 + wave;
    const bool srow_ok = srow < k;
    const int srow_c = min(srow, k - 1);
    float rsc = 0.f, csc[4];  // the row's and the columns' scales

    auto basis = [&](int t, float (&x)[8], float (&mv)[8]) {  // basis x mass of the split role, and the masses
        const char *S = ring + (t % HNST) * HSTAGE;
        const float *Ps = reinterpret_cast<const float *>(S);
        const float *Ms = reinterpret_cast<const float *>(S + 8 * 1024);
        const int vrem = vend - (vbeg + t * HS);
        const f32x4 m0 = *reinterpret_cast<const f32x4 *>(Ms + 8 * g4);
        const f32x4 m1 = *reinterpret_cast<const f32x4 *>(Ms + 8 * g4 + 4);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            mv[i] = i < 4 ? m0[i] : m1[i - 4];
            // past the last vertex the tile repeats its last value, which may be a NaN: the product is masked (its bits,
            // so that the LDS reads stay unconditional and are issued together)
            const uint32_t keep = (srow_ok && 8 * g4 + i < vrem) ? ~0u : 0u;
            x[i] = __uint_as_float(__float_as_uint(Ps[(8 * g4 + i) * k + srow_c] * mv[i]) & keep);
        }
    };
    auto magnitude = [](const float (&x)[8]) {
        float mx = 0.f;
#pragma unroll
        for (int i = 0; i < 8; ++i) mx = fmaxf(mx, fabsf(x[i]));
        return mx;
    };
    auto magnitude_of = [](const f32x4 (&fr)[HFF], int tt) {
        float mx = 0.f;
#pragma unroll
        for (int i = 0; i < HFF; ++i) mx = fmaxf(mx, fabsf(fr[i][tt]));
        return mx;
    };
    auto over_groups = [](float mx) {
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        return fmaxf(mx, __shfl_xor(mx, 32, 64));
    };
    // Scales from the values of stage t.  The four vertex groups of a row or column agree; one that is all zeros borrows
    // that of the wave's largest one (sparse features: its first values are likely to be as large as the others').
    // lanes whose column tt [0..3] or row [4] borrowed its scale, and whether any of the wave did
    uint64_t borrowed[5], any = 0;
    auto take_scales = [&](int t, const f32x4 (&fr)[HFF]) {
        float x[8], mv[8];
        basis(t, x, mv);
        float mx = over_groups(magnitude(x)), top = wave_max(mx);
        const int sh = split_shift<9>(__float_as_uint(mx > 0.f ? mx : top));
        rsc = split_scale(sh);
        if (g4 == 0) s_sh[16 * wave + m16] = sh;
        borrowed[4] = __ballot(mx == 0.f && srow_ok);
        any |= borrowed[4];
        float cm[4];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) cm[tt] = magnitude_of(fr, tt);
        bool massless = false;
#pragma unroll
        for (int i = 0; i < HFF; ++i) massless = massless || mv[i] == 0.f;
        if (__ballot(massless) != 0) {
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) {
                cm[tt] = 0.f;
#pragma unroll
                for (int i = 0; i < HFF; ++i) cm[tt] = fmaxf(cm[tt], mv[i] != 0.f ? fabsf(fr[i][tt]) : 0.f);
            }
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            cm[tt] = over_groups(cm[tt]);
            borrowed[tt] = __ballot(cm[tt] == 0.f);
            any |= borrowed[tt];
        }
        top = wave_max(fmaxf(fmaxf(cm[0], cm[1]), fmaxf(cm[2], cm[3])));
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) csc[tt] = split_scale(split_shift<9>(__float_as_uint(cm[tt] > 0.f ? cm[tt] : top)));
    };
    float rmx = 0.f, cmx[4] = {0.f, 0.f, 0.f, 0.f};  // largest magnitudes so far of the row and the columns
    auto stage = [&](int t, const f32x4 (&fr)[HFF]) {
        {
            float x[8], mv[8];
            basis(t, x, mv);
            u32x4_t h, l;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                uint32_t hh, ll;
                split_pair(x[2 * jj], x[2 * jj + 1], rsc, hh, ll);
                h[jj] = hh;
                l[jj] = ll;
            }
            parts[wave * 64 + lane] = h;
            parts[(4 + wave) * 64 + lane] = l;
            rmx = fmaxf(rmx, magnitude(x));
        }
        lds_barrier();
        u32x4_t A[4][2];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int p = 0; p < 2; ++p) A[a][p] = parts[(p * 4 + a) * 64 + lane];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            u32x4_t h, l;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                uint32_t hh, ll;
                split_pair(fr[2 * jj][tt], fr[2 * jj + 1][tt], csc[tt], hh, ll);
                h[jj] = hh;
                l[jj] = ll;
            }
            cmx[tt] = fmaxf(cmx[tt], magnitude_of(fr, tt));
#pragma unroll
            for (int a = 0; a < 4; ++a) acc[a][tt] = mfma16x16x32f16(A[a][1], h, acc[a][tt]);
#pragma unroll
            for (int a = 0; a < 4; ++a) acc[a][tt] = mfma16x16x32f16(A[a][0], l, acc[a][tt]);
#pragma unroll
            for (int a = 0; a < 4; ++a) acc[a][tt] = mfma16x16x32f16(A[a][0], h, acc[a][tt]);
        }
    };

    // Per stage t: wait for stage t (stage t + 1 may stay in flight), barrier (stage t visible; every wave done with
    // stage t - 1, so its ring slot, the split buffer and its feature registers are free), issue stage t + 2 into
    // them, split, barrier, products.  The three feature buffers rotate by unrolling; prefetches past the chunk reload
    // its last stage (the same bytes into the same places), and every load has landed before the workgroup ends (its
    // LDS is then reused).  The loop runs whole triples and has no early exit, the last one or two stages follow it: an
    // exit edge back into the loop header, or prologue loads reordered across the two stages, leaves the compiler's
    // wait analysis unable to tell which loads stage t needs, and it then waits for all of them, the stage t + 2
    // prefetch included.
    f32x4 f0[HFF], f1[HFF], f2[HFF];
    constexpr int VPS = BW + 1 + HFF;  // vector-memory operations per stage
    if (tid < 2) s_sh[64 + tid] = 0;
    issue(0, f0);
    __builtin_amdgcn_sched_barrier(0);
    issue(min(1, nst - 1), f1);
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<VPS>();
    lds_barrier();
    take_scales(0, f0);
    const int nfull = nst - nst % 3;
    for (int t = 0; t < nfull; t += 3) {
        wait_vmcnt<VPS>();
        lds_barrier();
        issue(min(t + 2, nst - 1), f2);
        stage(t, f0);
        wait_vmcnt<VPS>();
        lds_barrier();
        issue(min(t + 3, nst - 1), f0);
        stage(t + 1, f1);
        wait_vmcnt<VPS>();
        lds_barrier();
        issue(min(t + 4, nst - 1), f1);
        stage(t + 2, f2);
    }
    if (nst % 3 != 0) {  // stages nfull (in f0) and nfull + 1 (in f1) are issued
        wait_vmcnt<VPS>();
        lds_barrier();
        stage(nfull, f0);
        if (nst % 3 == 2) {
            wait_vmcnt<0>();
            lds_barrier();
            stage(nfull + 1, f1);
        }
    }
    wait_vmcnt<0>();
    float big = rmx * rsc;
#pragma unroll
    for (int tt = 0; tt < 4; ++tt) big = fmaxf(big, cmx[tt] * csc[tt]);
    if (!(big < kSplitLimit)) s_sh[64] = 1;
    if (any != 0) {
        auto low = [&](float mx, float sc, uint64_t of, bool &foreign) {
            mx = over_groups(mx);
            foreign = mx > 0.f && (of >> lane & 1) != 0;
            return foreign && mx * sc < kSplitLeast;
        };
        bool foreign;
        if (low(rmx, rsc, borrowed[4], foreign)) s_sh[64] = 1;
#pragma unroll
        for (int tt = 0; tt < 4; ++tt) {
            if (low(cmx[tt], csc[tt], borrowed[tt], foreign)) s_sh[64] = 1;
            if (foreign) s_sh[65] = 1;
        }
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(s_sh[65]) != 0) {
        for (int v = vbeg + tid; v < vend; v += 256)
            if (Mv[v] == 0.f) s_sh[64] = 1;
        __syncthreads();
    }
    if (__builtin_amdgcn_readfirstlane(s_sh[64]) != 0) {
        proj_fwd_tile<float, 2, 2, 2>(P, Mv, F, k, d, vbeg, vend, 0, dbase + 64 * wave, O);
        return;
    }

    // Lane (m16, g4), register r: matrix-core row 4 g4 + r -> basis row 4 (4 g4 + r) + a; column m16 of tile tt -> block
    // column 64 wave + 4 m16 + tt
    const int col = dbase + cw;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const int row = 16 * g4 + 4 * r + a;
            if (row >= k || col >= d) continue;
            const int rs = s_sh[16 * a + 4 * g4 + r];
            f32x4 v;
#pragma unroll
            for (int tt = 0; tt < 4; ++tt)
                v[tt] = __builtin_amdgcn_ldexpf(acc[a][tt][r], 127 - rs - (int)(__float_as_uint(csc[tt]) >> 23));
            *reinterpret_cast<f32x4 *>(O + (size_t)row * d + col) = v;  // d % 4 == 0: all 4 columns exist
        }
}

template <int BW>
__global__ __launch_bounds__(256, 2) void proj_fwd_h2_kernel(const float *__restrict__ phi,
                                                            const float *__restrict__ mass,
                                                            const float *__restrict__ feat, int n, int k, int d,
                                                            int nsplit, int dblocks, int ntiles,
                                                            float *__restrict__ out)
{
    const int bid = blockIdx.x;
    const int xs = bid & 7, q = bid >> 3;
    const int db = q % dblocks;
    const int j = (q / dblocks) * 8 + xs;
    if (j >= ntiles) return;  // whole workgroup, before any barrier
    const int split = j % nsplit, s = j / nsplit;
    const int nst_all = (n + HS - 1) / HS;
    const int st0 = (int)(((long)split * nst_all) / nsplit), st1 = (int)(((long)(split + 1) * nst_all) / nsplit);
    h2_block<BW>(phi + (size_t)s * n * k, mass + (size_t)s * n, feat + (size_t)s * n * d, k, d, st0 * HS,
                 min(n, st1 * HS), db * 256, out + (size_t)j * k * d);
}

// Uneven batches: one workgroup per work item.
__global__ __launch_bounds__(256, 2) void proj_fwd_h2_items_kernel(const FwdItem *__restrict__ items)
{
    const FwdItem w = items[blockIdx.x];
    if (w.v0 >= w.v1) return;  // empty slot of the table (whole workgroup, before any barrier)
    h2_block<8>(global_ptr(w.phi), global_ptr(w.mass), global_ptr(w.feat), w.k, w.d, w.v0, w.v1, w.dbase,
                global_ptr(w.out));
}

bool short_shape_ok(int64_t n, int64_t k, int64_t d)
{
    return k >= 1 && k <= kSmallK && d >= 4 && d % 4 == 0 && n >= 4 * HS;
}

int short_nsplit(int64_t batch, int64_t n, int64_t k, int64_t d)
{
    const int64_t blocks = (d + 255) / 256;
    const int64_t stages = (n + HS - 1) / HS;
    int64_t ns = (2 * device_cus()) / (batch * blocks);  // two workgroups per CU
    if (ns > stages / 4) ns = stages / 4;                // keep >= 4 stages per chunk
    if (ns < 1) ns = 1;
    return (int)ns;
}

hipError_t launch_project_short(const float *phi, const float *mass, const float *feat, int64_t batch, int64_t n,
                                int64_t k, int64_t d, int ns, float *A, void *ws, hipStream_t st)
{
    float *out = ns > 1 ? (float *)ws : A;
    const int dblocks = (int)((d + 255) / 256);
    const int ntiles = (int)(batch * ns);
    const unsigned grid = (unsigned)(8 * dblocks * ((ntiles + 7) / 8));
#define FMAP_H2(BW)                                                                                                  \
    hipLaunchKernelGGL((proj_fwd_h2_kernel<BW>), dim3(grid), dim3(256), h2_lds(), st, phi, mass, feat, (int)n, (int)k, \
                       (int)d, ns, dblocks, ntiles, out)
    if (k <= 32) FMAP_H2(4);
    else if (k <= 56) FMAP_H2(7);
    else FMAP_H2(8);
#undef FMAP_H2
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || ns <= 1) return e;
    return launch_reduce(out, ns, batch, k, d, A, true, st);
}

hipError_t launch_fwd_short_items(const FwdItem *items, int nitems, hipStream_t st)
{
    if (nitems <= 0) return hipSuccess;
    hipLaunchKernelGGL(proj_fwd_h2_items_kernel, dim3((unsigned)nitems), dim3(256), h2_lds(), st, items);
    return hipGetLastError();
}

}  // namespace fmap
