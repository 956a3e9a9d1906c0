// Backward projection dF = diag(M) Phi dA (the adjoint of Eq. (1)) in float32 for 4 <= k <= kMaxK, any n, k and d, on
// the float16 matrix cores (fmap_split.h: both operands as two float16 parts, three products).
//
// The upstream gradient stays in registers: a wave holds the parts of dA for 32 columns and every k as matrix-core
// operands with one scale per column (8 registers per 16 k, at most 160), and CW waves along the columns times VW along
// the vertices make a workgroup of 8, so the basis is read and split once per 256 (128) columns.  A tile of basis rows
// goes through LDS: a wave loads whole rows, 8 consecutive values per lane, scales each row by its largest value, and
// writes the parts as operand slots, permuted so that the lanes of a row hit different bank groups.  Two tiles are in
// LDS (one barrier per tile) and a third one's loads are in flight.  The result tile has the vertices along registers
// and the columns along lanes, so every store instruction writes whole 128-byte lines of two vertices; stores are
// non-temporal (the output is written once and not read here).  The column blocks of one vertex range share an XCD, so
// the basis rows they all read come from HBM once and from that XCD's L2 afterwards.
// With k > 192 the weights of 32 columns would leave no registers: two waves split k, and each adds the other's half of
// the result registers through LDS before it stores its own half of the rows.
//
// What bounds it: the writes of dF for k <= 96 (5.0 to 5.3 TB/s of the kernel's bytes), then the chain of a tile (LDS,
// barrier and memory latency at two waves per SIMD).  Measured against three-part bf16 operands with dA in LDS (odd k on
// the LDS or general kernels): 64 shapes of n = 5000, d = 256: k = 50 77 -> 75 us, k = 120 141 -> 100 us; 32 of
// n = 11000, k = 80 127 -> 92 us; 16 of n = 20000, k = 160, d = 384 335 -> 205 us; 8 of n = 9998, k = 200 69 -> 53 us;
// 16 of n = 100000, k = 300, d = 512 3090 -> 2247 us; 16 of n = 7001, k = 49, d = 128 45 -> 19 us.  Error against
// float64 1.4e-7 -> 1.2e-7 at k = 50, 2.8e-7 -> 1.6e-7 at k = 300.
#include <algorithm>

#include "fmap_lds.h"
#include "fmap_launch.h"
#include "fmap_split.h"

namespace fmap {

namespace {

typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // rows of any k: 4-byte aligned

__device__ __forceinline__ f32x16 mfma32x32x16f16(u32x4_t a, u32x4_t b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0,
                                                   0, 0);
}

// KS: K steps of 32 (k <= 32 KS); CW: waves along the columns
template <int KS, int CW>
struct Back {
    static constexpr int KW = KS >= 7 ? 2 : 1;          // waves along k
    static constexpr int VW = 8 / (CW * KW);            // waves along the vertices
    static_assert(VW >= 1, "eight waves");
    // (the last pass alone is clamped into the row: the others end below the least k of the instance)
    static constexpr int least_k() { return KS == 1 ? 4 : (KS == 6 ? 129 : (KS == 10 ? 257 : 32 * KS - 31)); }
    static constexpr int STEPS = 2 * KS / KW;           // matrix-core steps of 16 k per wave
    static constexpr int VT = KS <= 2 && CW > 2 ? 2 : 1;  // vertex tiles of 32 per wave
    static constexpr int VERTS = 32 * VT * VW;          // vertices per tile of the workgroup
    static constexpr int COLS = 32 * CW;                // columns per workgroup
    static constexpr int RPW = VERTS / 8;               // rows a wave loads
    static constexpr int LR = 64 / RPW;                 // lanes per row
    static constexpr int PASS = (4 * KS + LR - 1) / LR; // 8-value pieces per lane
    static_assert(8 * LR * (PASS - 1) < least_k(), "passes below the row's end");
    static constexpr int BUF = VERTS * KS * 8;          // 16-byte slots per tile (two float16 parts per value)
    static constexpr int XCH = KW > 1 ? 8 * 8 * 64 : 0; // floats that the waves along k exchange
    static constexpr size_t LDS = (size_t)2 * BUF * 16 + (2 * VERTS * 2 + XCH) * sizeof(float);
    static constexpr int PER_CU = KS <= 2 ? 2 : 1;      // resident workgroups (registers)
};

// Tiles [t0, t1) of one shape (basis P, masses Mv, G = dA, O = dF) for the columns [dbase, dbase + COLS).
template <int KS, int CW>
__device__ __forceinline__ void back_block(const float *__restrict__ P, const float *__restrict__ Mv,
                                           const float *__restrict__ G, float *__restrict__ O, int n, int k, int d,
                                           int t0, int t1, int dbase)
{
    using C = Back<KS, CW>;
    constexpr int S16 = 2 * KS;  // matrix-core steps of 16 k
    extern __shared__ __align__(16) float smem[];
    u32x4_t *buf = reinterpret_cast<u32x4_t *>(smem);     // two tiles [vertex tile][step][part][64 slots]
    int *s_sh = reinterpret_cast<int *>(buf + 2 * C::BUF);  // [2][VERTS] row shifts
    float *s_m = reinterpret_cast<float *>(s_sh + 2 * C::VERTS);  // [2][VERTS] masses
    float *s_x = s_m + 2 * C::VERTS;                               // [wave][8][64] partial sums
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int cw = wave % CW, kw = wave / CW % C::KW, vw = wave / (CW * C::KW);
    if (t0 >= t1) return;

    // loading role: 8-value pieces lr, lr + LR, ... of row `row` of the tile.  Loads are clamped into the row; the last
    // pass holds the row's end, and its values past k are zeroed
    const int row = wave * C::RPW + lane / C::LR, lr = lane % C::LR;
    struct Rows {
        f32x4 x[C::PASS][2];
        float m;
    };
    auto issue = [&](int t, Rows &r) {
        const int v = min(t * C::VERTS + row, n - 1);
        const float *pr = P + (size_t)v * k;
#pragma unroll
        for (int q = 0; q < C::PASS; ++q)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const int j0 = 8 * (q * C::LR + lr) + 4 * c;
                r.x[q][c] = *reinterpret_cast<const f32x4u *>(pr + (q + 1 < C::PASS ? j0 : min(j0, k - 4)));
            }
        r.m = Mv[v];
    };
    auto split = [&](int b, Rows &r) {
        constexpr int Q = C::PASS - 1;
        const int cut = k & 3;  // a chunk that straddles k was loaded 4 - cut values early
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int j0 = 8 * (Q * C::LR + lr) + 4 * c;
            f32x4 y = r.x[Q][c];
            if (cut != 0) {
                const bool straddles = j0 == (k & ~3);
                const f32x4 w = cut == 1 ? f32x4{y[3], 0, 0, 0} : (cut == 2 ? f32x4{y[2], y[3], 0, 0} : f32x4{y[1], y[2], y[3], 0});
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = straddles ? w[e] : y[e];
            }
            const bool in = j0 < k;
#pragma unroll
            for (int e = 0; e < 4; ++e) r.x[Q][c][e] = in ? y[e] : 0.f;
        }
        float mx = 0.f;
#pragma unroll
        for (int q = 0; q < C::PASS; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = fmaxf(mx, fmaxf(fabsf(r.x[q][0][e]), fabsf(r.x[q][1][e])));
#pragma unroll
        for (int o = 1; o < C::LR; o *= 2) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        const int sh = split_shift(__float_as_uint(mx));
        const float sc = split_scale(sh);
        if (lr == 0) {
            s_sh[b * C::VERTS + row] = sh;
            s_m[b * C::VERTS + row] = r.m;
        }
        u32x4_t *B = buf + b * C::BUF + (row >> 5) * S16 * 128;
#pragma unroll
        for (int q = 0; q < C::PASS; ++q) {
            const int piece = q * C::LR + lr;
            u32x4_t h, l;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                uint32_t hh, ll;
                split_pair(r.x[q][jj >> 1][2 * (jj & 1)], r.x[q][jj >> 1][2 * (jj & 1) + 1], sc, hh, ll);
                h[jj] = hh;
                l[jj] = ll;
            }
            u32x4_t *o = B + (piece >> 1) * 128 + ((row & 31) ^ (piece & 15)) + 32 * (piece & 1);
            if (4 * KS % C::LR == 0 || piece < 4 * KS) {
                o[0] = h;
                o[64] = l;
            }
        }
    };

    Rows x;
    issue(t0, x);
    // this wave's columns of dA (and, with two waves along k, its half of the steps): lane (l32, half) holds column l32,
    // k 16 s + 8 half .. + 7 of step s
    const int c0 = dbase + 32 * cw;
    u32x4_t wh[C::STEPS], wl[C::STEPS];
    int csh;
    {
        const int c = min(c0 + l32, d - 1);
        const int k0 = 16 * C::STEPS * kw;
        auto load = [&](int s, float (&g)[8]) {
#pragma unroll
            for (int i = 0; i < 8; ++i) g[i] = G[(unsigned)(min(k0 + 16 * s + 8 * half + i, k - 1) * d + c)];
#pragma unroll
            for (int i = 0; i < 8; ++i)  // (the bit mask keeps the loads unconditional)
                g[i] = __uint_as_float(__float_as_uint(g[i]) & (k0 + 16 * s + 8 * half + i < k ? ~0u : 0u));
        };
        auto parts = [&](int s, const float (&g)[8], float sc) {
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                uint32_t h, l;
                split_pair(g[2 * jj], g[2 * jj + 1], sc, h, l);
                wh[s][jj] = h;
                wl[s][jj] = l;
            }
        };
        auto magnitude = [](const float (&g)[8], float mx) {
#pragma unroll
            for (int i = 0; i < 8; ++i) mx = fmaxf(mx, fabsf(g[i]));
            return mx;
        };
        float mx = 0.f;
        float g[C::STEPS][8];
#pragma unroll
        for (int s = 0; s < C::STEPS; ++s) load(s, g[s]);
#pragma unroll
        for (int s = 0; s < C::STEPS; ++s) mx = magnitude(g[s], mx);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        if constexpr (C::KW > 1) {  // both halves of k take one scale
            if (half == 0) s_x[wave * 32 + l32] = mx;
            __syncthreads();
            mx = fmaxf(mx, s_x[((wave + CW) % (2 * CW)) * 32 + l32]);
            __syncthreads();
        }
        csh = split_shift(__float_as_uint(mx));
#pragma unroll
        for (int s = 0; s < C::STEPS; ++s) parts(s, g[s], split_scale(csh));
    }
    split(0, x);
    issue(min(t0 + 1, t1 - 1), x);
    lds_barrier();

    const unsigned ocol = c0 + l32 < d ? 4u * (unsigned)(4 * half * d + c0 + l32) : 0x80000000u;  // dropped past d
    for (int t = t0; t < t1; ++t) {
        const int b = (t - t0) & 1;
        f32x16 acc[C::VT];
#pragma unroll
        for (int v = 0; v < C::VT; ++v) {
            acc[v] = zero16();
            int ln = lane;  // (opaque: the slots of all steps would be kept in registers)
            asm volatile("" : "+v"(ln));
            const int l32 = ln & 31, half = ln >> 5;
            const int s0 = kw * C::STEPS;
            const u32x4_t *B = buf + b * C::BUF + ((vw * C::VT + v) * S16 + s0) * 128 + 32 * half;
#pragma unroll
            for (int s = 0; s < C::STEPS; ++s) {
                const int sl = l32 ^ ((2 * (s0 + s) + half) & 15);
                const u32x4_t ph = B[s * 128 + sl], pl = B[s * 128 + 64 + sl];
                acc[v] = mfma32x32x16f16(pl, wh[s], acc[v]);
                acc[v] = mfma32x32x16f16(ph, wl[s], acc[v]);
                acc[v] = mfma32x32x16f16(ph, wh[s], acc[v]);
            }
        }
        // with two waves along k, each keeps half of the result registers and gives the other half away
        if constexpr (C::KW > 1) {
            static_assert(C::VT == 1, "one tile per wave");
#pragma unroll
            for (int r = 0; r < 8; ++r) s_x[(wave * 8 + r) * 64 + lane] = kw == 0 ? acc[0][8 + r] : acc[0][r];
        }
        split(b ^ 1, x);  // tile t + 1 (past the last one: the last one again, never read)
        issue(min(t + 2, t1 - 1), x);
        if constexpr (C::KW > 1) {
            lds_barrier();
            const int other = wave + (kw == 0 ? CW : -CW);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const float y = s_x[(other * 8 + r) * 64 + lane];
                // (the first wave's part first, in both halves)
                acc[0][r] = kw == 0 ? acc[0][r] + y : y + acc[0][8 + r];
            }
        }
        // register r of lane (l32, half): vertex 8 (r / 4) + 4 half + r % 4, column l32
#pragma unroll
        for (int v = 0; v < C::VT; ++v) {
            const int lv = (vw * C::VT + v) * 32, v0 = t * C::VERTS + lv;
            if (v0 >= n) continue;
            const bool whole = v0 + 32 <= n;
            const __amdgpu_buffer_rsrc_t out =
                __builtin_amdgcn_make_buffer_rsrc(O + (size_t)v0 * d, 0, 0x7fffffff, 0x00020000);
#pragma unroll
            for (int i4 = 0; i4 < 4 / C::KW; ++i4) {
                const int r4 = i4 + 2 * kw;  // (kw > 0: its half of the rows, in registers 0..7)
                const int base = b * C::VERTS + lv + 8 * r4 + 4 * half;
                const int4 sh = *reinterpret_cast<const int4 *>(&s_sh[base]);
                const f32x4 m = *reinterpret_cast<const f32x4 *>(&s_m[base]);
                const int shr[4] = {sh.x, sh.y, sh.z, sh.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float val = __builtin_amdgcn_ldexpf(acc[v][4 * i4 + e], -(shr[e] + csh)) * m[e];
                    const unsigned off = whole || v0 + 8 * r4 + 4 * half + e < n ? ocol : 0x80000000u;
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val), out, off, 4 * (8 * r4 + e) * d, 2);
                }
            }
        }
        lds_barrier();
    }
}

}  // namespace

template <int KS, int CW>
__global__ __launch_bounds__(512, KS <= 2 ? 4 : 2) void proj_bwd_split_kernel(const float *__restrict__ phi,
                                                                             const float *__restrict__ mass,
                                                                             const float *__restrict__ dA, int n, int k,
                                                                             int d, int vsplit, int dblocks, int ntasks,
                                                                             float *__restrict__ dF)
{
    using C = Back<KS, CW>;
    const int bid = blockIdx.x;
    const int xs = bid & 7, q = bid >> 3;
    const int db = q % dblocks;
    const int j = (q / dblocks) * 8 + xs;
    if (j >= ntasks) return;  // whole workgroup, before any barrier
    const int vs = j % vsplit, s = j / vsplit;
    const int ntile = (n + C::VERTS - 1) / C::VERTS;
    const int t0 = (int)(((long)vs * ntile) / vsplit), t1 = (int)(((long)(vs + 1) * ntile) / vsplit);
    back_block<KS, CW>(phi + (size_t)s * n * k, mass + (size_t)s * n, dA + (size_t)s * k * d, dF + (size_t)s * n * d, n, k,
                       d, t0, t1, db * C::COLS);
}

// Uneven batches: one workgroup per work item (vertices in units of 32 rows: [t0, t1) tiles of VERTS).
template <int KS, int CW>
__global__ __launch_bounds__(512, KS <= 2 ? 4 : 2) void proj_bwd_split_items_kernel(const McItem *__restrict__ items)
{
    const McItem w = items[blockIdx.x];
    if (w.t0 >= w.t1) return;  // empty slot of the table (whole workgroup, before any barrier)
    back_block<KS, CW>(global_ptr(w.phi), global_ptr(w.mass), global_ptr(w.dA), global_ptr(w.dF), w.n, w.k, w.d, w.t0,
                       w.t1, w.dbase);
}

bool back_shape_ok(int64_t k, int64_t d) { return k >= 4 && k <= kMaxK && d >= 1 && d <= (1 << 20); }

// 256 columns per workgroup, or 128 where that leaves fewer idle columns or the weights need two waves along k.  Up to 64
// columns (coordinates, a few signals) two waves along the columns and four along the vertices, where the larger tile
// fits LDS: 64 shapes of n = 2001, four waves along the columns and two, us: k = 30, d = 16 10.9, 8.7; k = 100, d = 3 23.0,
// 18.4; k = 200, d = 16 37.4, 27.1.
static int back_cw(int64_t k, int64_t d)
{
    if (d <= 64 && (k <= 128 || (k > 192 && k <= 256))) return 2;
    return k > 192 || (d + 127) / 128 * 128 < (d + 255) / 256 * 256 ? 4 : 8;
}
int back_cols(int64_t k, int64_t d) { return 32 * back_cw(k, d); }
int back_slots(int64_t k) { return device_cus() * (k <= 64 ? 2 : 1); }
int back_verts(int64_t k, int64_t d)
{
    const int cw = back_cw(k, d);
    return 32 * (k <= 64 && cw > 2 ? 2 : 1) * (8 / cw / (k > 192 ? 2 : 1));
}

// Vertex ranges per (shape, column block), at most one range per tile.
// One workgroup per CU (k > 64): the fewest ranges that take the least time, counted as rounds of resident workgroups
// times the tiles of the longest range plus three for what a workgroup does first (its columns of dA, 3 to 5 us).  (The
// fewest that keep 95% of the last round busy took a third round of one tile each where one round of four was 94% full:
// 2 shapes of n = 5000, k = 100, d = 600 25.0 us, 15.4 now.)
// Two per CU (k <= 64): one's start hides behind the other's tiles, and more, shorter ranges even out the rounds: the
// fewest that keep 95% of the last round busy (32 shapes of n = 2992, k = 38, d = 300 54 us, counted as above 65; 16 of
// n = 5000, k = 30, d = 128 10.7 and 12.6).
static int back_vsplit(int64_t batch, int64_t dblocks, int64_t ntile, int64_t slots, int per_cu)
{
    const int64_t base = batch * dblocks;
    int64_t best = 1, least = INT64_MAX;
    double best_e = 0.0;
    for (int64_t v = 1; v <= ntile && (v == 1 || base * v <= 4 * slots); ++v) {
        if (per_cu > 1) {
            const int64_t tot = base * v, rounds = (tot + slots - 1) / slots;
            const double e = (double)tot / (double)(rounds * slots);
            if (e >= 0.95) return (int)v;
            if (e > best_e + 1e-9) {
                best_e = e;
                best = v;
            }
        } else {
            const int64_t time = xcd_rounds(batch * v, dblocks, slots) * ((ntile + v - 1) / v + 3);
            if (time < least) {
                least = time;
                best = v;
            }
        }
    }
    return (int)best;
}

template <int KS, int CW>
static hipError_t dispatch_back(const float *phi, const float *mass, const float *dA, int64_t batch, int64_t n, int64_t k,
                                int64_t d, float *dF, hipStream_t st)
{
    using C = Back<KS, CW>;
    static bool set = false;
    if (!set) {
        (void)hipFuncSetAttribute((const void *)proj_bwd_split_kernel<KS, CW>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)C::LDS);
        set = true;
    }
    const int dblocks = (int)((d + C::COLS - 1) / C::COLS);
    const int64_t ntile = (n + C::VERTS - 1) / C::VERTS;
    const int vsplit = back_vsplit(batch, dblocks, ntile, (int64_t)device_cus() * C::PER_CU, C::PER_CU);
    const int ntasks = (int)(batch * vsplit);
    const unsigned grid = (unsigned)(8 * dblocks * ((ntasks + 7) / 8));
    hipLaunchKernelGGL((proj_bwd_split_kernel<KS, CW>), dim3(grid), dim3(512), C::LDS, st, phi, mass, dA, (int)n, (int)k,
                       (int)d, vsplit, dblocks, ntasks, dF);
    return hipGetLastError();
}

template <int KS, int CW>
static hipError_t dispatch_back_items(const McItem *items, int nitems, hipStream_t st)
{
    const size_t lds = Back<KS, CW>::LDS;
    static bool set = false;
    if (!set) {
        (void)hipFuncSetAttribute((const void *)proj_bwd_split_items_kernel<KS, CW>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        set = true;
    }
    hipLaunchKernelGGL((proj_bwd_split_items_kernel<KS, CW>), dim3((unsigned)nitems), dim3(512), lds, st, items);
    return hipGetLastError();
}

#define FMAP_BACK_CW(FN, KS, ...)                                                                                     \
    return cw == 8 ? FN<KS, 8>(__VA_ARGS__) : (cw == 4 ? FN<KS, 4>(__VA_ARGS__) : FN<KS, 2>(__VA_ARGS__))
#define FMAP_BACK(FN, ...)                                                     \
    const int cw = back_cw(k, d);                                              \
    switch ((k + 31) / 32) {                                                   \
    case 1: FMAP_BACK_CW(FN, 1, __VA_ARGS__);                                  \
    case 2: FMAP_BACK_CW(FN, 2, __VA_ARGS__);                                  \
    case 3: FMAP_BACK_CW(FN, 3, __VA_ARGS__);                                  \
    case 4: FMAP_BACK_CW(FN, 4, __VA_ARGS__);                                  \
    case 5:                                                                    \
    case 6: return cw == 8 ? FN<6, 8>(__VA_ARGS__) : FN<6, 4>(__VA_ARGS__);    \
    case 7: return cw == 4 ? FN<7, 4>(__VA_ARGS__) : FN<7, 2>(__VA_ARGS__);    \
    case 8: return cw == 4 ? FN<8, 4>(__VA_ARGS__) : FN<8, 2>(__VA_ARGS__);    \
    default: return FN<10, 4>(__VA_ARGS__);                                    \
    }

hipError_t launch_project_back(const float *phi, const float *mass, const float *dA, int64_t batch, int64_t n, int64_t k,
                               int64_t d, float *dF, hipStream_t st)
{
    FMAP_BACK(dispatch_back, phi, mass, dA, batch, n, k, d, dF, st)
}

hipError_t launch_bwd_split_items(const McItem *items, int nitems, int64_t k, int64_t d, hipStream_t st)
{
    if (nitems <= 0) return hipSuccess;
    FMAP_BACK(dispatch_back_items, items, nitems, st)
}

}  // namespace fmap
