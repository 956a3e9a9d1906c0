// Forward projection A = Phi^T diag(M) F (Eq. (1)) in float32 for 64 < k <= kMaxK, 5 k / 4 <= d, any n and k, d % 4 == 0, on the
// float16 matrix cores (fmap_split.h: both operands as two float16 parts, three products).
//
// A workgroup of 8 waves owns every basis row of one vertex chunk and a block of columns, so the features are read
// and split once; the 64-row slices used before read and split them once per slice (five times at k = 300).  Stages of
// 32 vertices, one matrix-core K step.  Each thread loads 4 consecutive entries of 8 consecutive vertices straight
// into registers (the last waves of the features, the first of the basis), two stages ahead, splits them a stage
// later and writes them to LDS as matrix-core operands: its 8 vertices are the 8 K slots of one lane, so the
// transposition costs nothing.  The operands are double-buffered, with one barrier per stage.  Rows of LDS tiles are
// written 4 apart; the slots are permuted per tile so that 16 consecutive lanes hit 16 different bank groups.
//
// Each basis row and each feature column has its own power-of-two scale in LDS, taken from the first stage; a value
// that does not fit raises a flag that the whole workgroup sees at the next stage, where the scales and the sums are
// lowered together and the stage is split again.  A row or column that is all zeros so far has no value to take a scale
// from and borrows that of the largest one; its largest value is known at the end of the chunk, and where that lies
// too low on the borrowed scale to keep its bits, or where a value is infinite, the general float32 routine computes
// the chunk again.  Loads go through one buffer descriptor per vertex row, whose range ends with the chunk: vertices
// past its end read as zeros.
//
// Instances by k: 4 x 64 columns for k <= 128 (RG = 2 row groups of RT = 4 tiles; d <= 128: RG = 4, RT = 2), 2 x 64 above
// (RG = 4, RT = 3, 4, 5).
// What bounds it: at 100000 vertices, k = 300, d = 512 the matrix cores and the vector units together (taking out the
// products or the splitting alone saves a quarter and an eighth of the time), at k <= 200 the chain of one stage
// (latencies of LDS and memory at two waves per SIMD).  Alternating products and splitting within a wave gave 3% to 6%
// for RT <= 4; at RT = 5 it spills.  Measured against the sliced kernel with six bf16 products, projection and
// reduction: 16 shapes of n = 100000, k = 300, d = 512 3043 -> 1879 us; 64 of n = 5000, k = 120, d = 256 141 -> 114 us;
// 8 of n = 9998, k = 200, d = 256 (the general kernel took n % 4 != 0) 137 -> 55 us.  The error against float64 falls
// with the number of roundings (three products instead of six): 3.7e-6 -> 2.1e-6, 5.7e-7 -> 4.0e-7, 4.6e-7 -> 3.0e-7.
#include <algorithm>

#include "fmap_lds.h"
#include "fmap_launch.h"
#include "fmap_split.h"
#include "proj_general.h"

namespace fmap {

constexpr int TS = 32;        // vertices per stage (one matrix-core K step)
constexpr int TT = 512;       // threads per workgroup
constexpr int kIdle = 0x7ffffe00;  // a byte offset past every descriptor's range: the load returns zeros
constexpr int TILE = 64;      // 16-byte slots of one operand tile (16 rows x 32 vertices of one part)

template <int RG, int RT>
struct Tall {
    static constexpr int CG = 8 / RG;            // column groups of 64
    static constexpr int COLS = 64 * CG;         // columns per workgroup
    static constexpr int ROWS = 16 * RG * RT;    // basis rows per workgroup (k <= ROWS)
    static_assert(ROWS % 64 == 0 && COLS % 64 == 0, "whole waves of scales");
    static constexpr int AT = RG * RT, BT = 4 * CG;
    // 16-byte slots: the two buffers of basis tiles, the two of feature tiles, slots that idle threads write
    static constexpr int ABUF = AT * 2 * TILE, BBUF = BT * 2 * TILE, IDLE = 2 * (ABUF + BBUF);
    static constexpr size_t LDS = (size_t)(IDLE + 2 * TILE) * 16 + (ROWS + COLS) * 12 + 32;
};

template <int RG, int RT>
__device__ __forceinline__ void tall_block(const float *__restrict__ P, const float *__restrict__ Mv,
                                           const float *__restrict__ F, int k, int d, int vbeg, int vend, int dbase,
                                           float *__restrict__ O)
{
    using C = Tall<RG, RT>;
    extern __shared__ __align__(16) float smem[];
    u32x4_t *buf = reinterpret_cast<u32x4_t *>(smem);
    uint32_t *s_mx = reinterpret_cast<uint32_t *>(buf + C::IDLE + 2 * TILE);  // [ROWS + COLS] largest magnitude so far
    int *s_sh = reinterpret_cast<int *>(s_mx + C::ROWS + C::COLS);      // scale shifts
    int *s_dl = s_sh + C::ROWS + C::COLS;                               // their last changes
    uint32_t *s_top = reinterpret_cast<uint32_t *>(s_dl + C::ROWS + C::COLS);  // [2] basis, features: largest
    // [2] of stages t % 2: bit 0, a value does not fit; bit 1 (in both), a scale was borrowed.  [1] the chunk goes to the
    // general routine
    int *s_flag = reinterpret_cast<int *>(s_top + 2);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m16 = lane & 15, g4 = lane >> 4;
    const int rg = wave % RG, cg = wave / RG;
    const int nst = (vend - vbeg + TS - 1) / TS;
    if (nst <= 0) return;

    // loading role: 4 consecutive entries of 8 consecutive vertices.  The last waves take the feature block,
    // the first threads the basis rows (chunks of 4 entries; the last chunk overlaps its neighbour when
    // k % 4 != 0 and writes the same values again).
    const bool isF = wave >= (TT - C::COLS) / 64;
    const int kc = (k + 3) >> 2;
    const int task = isF ? tid - (TT - C::COLS) : tid;
    const int per = isF ? C::COLS / 4 : kc;
    const bool active = isF || task < 4 * kc;
    const int tg = active ? task / per : 0, ch = active ? task - tg * per : 0;
    const int ld = isF ? d : k;
    const int e0 = isF ? min(dbase + 4 * ch, d - 4) : min(4 * ch, k - 4);
    const int sidx = (isF ? C::ROWS + 4 * ch : e0);  // scale index of the first entry
    uint32_t slots[2];                               // operand slots (buffer 0) of the 4 entries, 16 bits each
    {
        int sl[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (isF) {
                // column 4 N + t of a 64-column group is column N of its tile t
                sl[t] = 2 * C::ABUF + (4 * (ch >> 4) + t) * 2 * TILE + (ch & 15) + 16 * tg;
            } else {
                const int j = e0 + t, tile = j >> 4;
                sl[t] = tile * 2 * TILE + (((j & 15) + 16 * tg) ^ (tile % RT & 3));
            }
            if (!active) sl[t] = C::IDLE + lane;
        }
        slots[0] = (uint32_t)(sl[0] | sl[1] << 16);
        slots[1] = (uint32_t)(sl[2] | sl[3] << 16);
    }
    const int bstep = !active ? 0 : (isF ? C::BBUF : C::ABUF);  // from buffer 0 to buffer 1
    // byte offset of the task's first row within a stage; an idle thread's is past every descriptor's range
    const int vo = active ? 4 * (8 * tg * ld + e0) : kIdle;
    const float *base = (isF ? F : P) + (size_t)vbeg * ld;

    struct Raw {
        f32x4 x[8];
        float m;
    };
    auto issue = [&](int t, Raw &r) {
        const int v = vbeg + t * TS, rows = min(TS, vend - v);
        // one descriptor per row i: rows past the end of the chunk are past its range and read as zeros
        const float *row = base + (size_t)t * TS * ld;
        int64_t left = (int64_t)rows * ld * 4;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc((void *)row, 0, (int)(left > 0 ? left : 0), 0x00020000);
            r.x[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, vo, 0, 0));
            row += ld;
            left -= (int64_t)ld * 4;
        }
        r.m = Mv[v + min(lane & 31, rows - 1)];
    };
    // masses onto the features (zero past the end of the chunk; 1 for the basis, so that no branch splits the
    // stage)
    auto weigh = [&](int t, Raw &r) {
        if (RT > 4 && !isF) return;
        const float m = isF ? ((lane & 31) < vend - (vbeg + t * TS) ? r.m : 0.f) : 1.f;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            r.x[i] *= __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (8 * tg + i), __float_as_int(m)));
    };
    float sc[4];
    // entry e of the task's 8 (weighed) values to its operand slots
    auto split1 = [&](int t, int e, const Raw &r, float &big) {
        u32x4_t h, l;
        float mx = 0.f;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            uint32_t hh, ll;
            split_pair(r.x[2 * jj][e], r.x[2 * jj + 1][e], sc[e], hh, ll);
            mx = fmaxf(mx, fmaxf(fabsf(r.x[2 * jj][e]), fabsf(r.x[2 * jj + 1][e])));
            h[jj] = hh;
            l[jj] = ll;
        }
        big = fmaxf(big, mx * sc[e]);
        u32x4_t *B = buf + ((slots[e >> 1] >> (16 * (e & 1))) & 0xffff) + ((t & 1) ? bstep : 0);
        B[0] = h;
        B[TILE] = l;
    };
    auto split = [&](int t, const Raw &r) {
        float big = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) split1(t, e, r, big);
        if (big >= kSplitLimit) atomicOr(&s_flag[t & 1], 1);
    };

    f32x4 acc[RT][4];
#pragma unroll
    for (int a = 0; a < RT; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = f32x4{0, 0, 0, 0};

    // Follows the largest magnitudes of the (still unweighed) values of stage t, once a row or column has borrowed a scale
    auto follow = [&](int t, const Raw &r) {
        const float m = isF ? ((lane & 31) < vend - (vbeg + t * TS) ? r.m : 0.f) : 1.f;
        float mx[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float mi = __int_as_float(__builtin_amdgcn_ds_bpermute(4 * (8 * tg + i), __float_as_int(m)));
#pragma unroll
            for (int e = 0; e < 4; ++e) mx[e] = fmaxf(mx[e], fabsf(r.x[i][e] * mi));
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (active) atomicMax(&s_mx[sidx + e], __float_as_uint(mx[e]));
    };
    // Lowers the scales so that the (weighed) values r fit, and the sums with them.  Every thread of the workgroup
    // comes here together.  A row or column that is all zeros so far borrows the scale of the largest one (sparse
    // features: its first values are likely to be as large as the others').
    auto rescale = [&](const Raw &r) {
        if (active) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float mx = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) mx = fmaxf(mx, fabsf(r.x[i][e]));
                atomicMax(&s_mx[sidx + e], __float_as_uint(mx));
            }
        }
        __syncthreads();
        for (int e = tid; e < C::ROWS + C::COLS; e += TT) {  // (64 entries of one kind per wave)
            const float top = wave_max(__uint_as_float(s_mx[e]));
            if (lane == 0) atomicMax(&s_top[e >= C::ROWS], __float_as_uint(top));
        }
        __syncthreads();
        for (int e = tid; e < C::ROWS + C::COLS; e += TT) {
            const uint32_t mx = s_mx[e];
            const int old = s_sh[e], now = min(old, split_shift(mx ? mx : s_top[e >= C::ROWS]));
            s_sh[e] = now;
            s_dl[e] = now - old;
            if (mx == 0x7f800000u) s_flag[2] = 1;
            if (mx == 0 && (e < k || e >= C::ROWS)) {
                atomicOr(&s_flag[0], 2);
                atomicOr(&s_flag[1], 2);
            }
        }
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int dc = s_dl[C::ROWS + cg * 64 + 4 * m16 + c];
#pragma unroll
            for (int a = 0; a < RT; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[a][c][q] = __builtin_amdgcn_ldexpf(acc[a][c][q], dc + s_dl[(rg * RT + a) * 16 + 4 * g4 + q]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) sc[e] = active ? split_scale(s_sh[sidx + e]) : 0.f;
    };
    u32x4_t bh[4], bl[4];
    auto load_b = [&](int t) {
        const u32x4_t *B = buf + 2 * C::ABUF + (t & 1) * C::BBUF + 4 * cg * 2 * TILE + lane;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            bh[c] = B[c * 2 * TILE];
            bl[c] = B[c * 2 * TILE + TILE];
        }
    };
    auto load_a = [&](int t, int a, u32x4_t &ah, u32x4_t &al) {
        const u32x4_t *A = buf + (t & 1) * C::ABUF + rg * RT * 2 * TILE + a * 2 * TILE + (lane ^ (a & 3));
        ah = A[0];
        al = A[TILE];
    };

    Raw x, y;
    issue(0, x);
    for (int e = tid; e < C::ROWS + C::COLS; e += TT) {
        s_mx[e] = 0;
        s_sh[e] = 126;
    }
    if (tid < 2) s_flag[tid] = s_top[tid] = 0;
    if (tid == 0) s_flag[2] = 0;
    __syncthreads();
    weigh(0, x);
    rescale(x);
    split(0, x);
    issue(min(1, nst - 1), y);
    lds_barrier();
    // Stage t: its operands are in buffer t % 2; `next` holds the values of stage t + 1 (arriving).  The products
    // of one row tile alternate with a quarter of the next stage's splitting, so that the matrix cores and the
    // vector units of a SIMD work at the same time.
    auto stage = [&](int t, Raw &free, Raw &next) {
        const int flag = s_flag[t & 1];
        if (RT <= 4) load_b(t);
        if (const int bits = __builtin_amdgcn_readfirstlane(flag)) {
            if (bits & 2) follow(t + 1, next);
            if (bits & 1) {
                issue(t, free);
                weigh(t, free);
                rescale(free);
                split(t, free);
                __syncthreads();
                if (tid == 0) atomicAnd(&s_flag[t & 1], ~1);
            }
            if (RT <= 4) load_b(t);
        }
        issue(min(t + 2, nst - 1), free);
        if (RT > 4) load_b(t);
        float big = 0.f;
        u32x4_t ah, al, nh, nl;
        if (RT <= 4) {
            load_a(t, 0, ah, al);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int a = 0; a < RT; ++a) {
            if (RT > 4) load_a(t, a, ah, al);
            if (RT <= 4 && a + 1 < RT) load_a(t, a + 1, nh, nl);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[a][c] = mfma16x16x32f16(al, bh[c], acc[a][c]);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[a][c] = mfma16x16x32f16(ah, bl[c], acc[a][c]);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[a][c] = mfma16x16x32f16(ah, bh[c], acc[a][c]);
            if (a == (RT <= 4 ? 0 : RT - 1)) weigh(t + 1, next);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((RT <= 4 ? e * RT / 4 : RT - 1) == a) split1(t + 1, e, next, big);
            if (RT <= 4) {
                ah = nh;
                al = nl;
            }
            if (RT <= 4) __builtin_amdgcn_sched_barrier(0);
        }
        if (big >= kSplitLimit) atomicOr(&s_flag[(t + 1) & 1], 1);
        lds_barrier();
    };
    for (int t = 0; t < nst; t += 2) {
        stage(t, x, y);
        if (t + 1 < nst) stage(t + 1, y, x);
    }

    if (__builtin_amdgcn_readfirstlane(s_flag[0]) & 2) {  // (s_mx is complete since the last stage's barrier)
        for (int e = tid; e < C::ROWS + C::COLS; e += TT) {
            const float mx = __uint_as_float(s_mx[e]);
            if (mx > 0.f && mx * split_scale(s_sh[e]) < kSplitLeast) s_flag[2] = 1;
        }
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(s_flag[2]) != 0) {
#pragma unroll 1
        for (int kb = 64 * (wave / C::CG); kb < k; kb += 64 * (8 / C::CG))
            proj_fwd_tile<float, 2, 2, 2>(P, Mv, F, k, d, vbeg, vend, kb, dbase + 64 * (wave % C::CG), O);
        return;
    }

    const int col = dbase + cg * 64 + 4 * m16;
    if (col < d) {
#pragma unroll
        for (int a = 0; a < RT; ++a)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int rl = (rg * RT + a) * 16 + 4 * g4 + q;
                if (rl >= k) continue;
                f32x4 v;
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    v[c] = __builtin_amdgcn_ldexpf(acc[a][c][q], -(s_sh[rl] + s_sh[C::ROWS + cg * 64 + 4 * m16 + c]));
                *reinterpret_cast<f32x4 *>(O + (size_t)rl * d + col) = v;  // d % 4 == 0: all 4 columns exist
            }
    }
}

template <int RG, int RT>
__global__ __launch_bounds__(TT, 2) void proj_fwd_tall_kernel(const float *__restrict__ phi,
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
    const int nst_all = (n + TS - 1) / TS;
    const int st0 = (int)(((long)split * nst_all) / nsplit), st1 = (int)(((long)(split + 1) * nst_all) / nsplit);
    tall_block<RG, RT>(phi + (size_t)s * n * k, mass + (size_t)s * n, feat + (size_t)s * n * d, k, d, st0 * TS,
                       min(n, st1 * TS), db * Tall<RG, RT>::COLS, out + (size_t)j * k * d);
}

// Uneven batches: one workgroup per work item.
template <int RG, int RT>
__global__ __launch_bounds__(TT, 2) void proj_fwd_tall_items_kernel(const FwdItem *__restrict__ items)
{
    const FwdItem w = items[blockIdx.x];
    if (w.v0 >= w.v1) return;  // empty slot of the table (whole workgroup, before any barrier)
    tall_block<RG, RT>(global_ptr(w.phi), global_ptr(w.mass), global_ptr(w.feat), w.k, w.d, w.v0, w.v1, w.dbase,
                       global_ptr(w.out));
}

// Instances by k (rows in blocks of 16 RG RT); up to k = 128 with 256 columns per workgroup, or 128 where d fits those.
// (Wider d take 256 also where the last block is half idle: blocks of 128 split the basis once each.  k = 100, blocks of
// 128 and of 256, us: 8 shapes of n = 5000, d = 300 43.5, 32.9; 32 of n = 5000, d = 352 127, 97; 4 of n = 20000, d = 640
// 96, 75.)
int tall_class(int64_t k, int64_t d)
{
    if (k <= 128) return d <= 128 ? 1 : 0;
    return k <= 192 ? 2 : (k <= 256 ? 3 : 4);
}
int tall_cols(int64_t k, int64_t d) { return tall_class(k, d) == 0 ? Tall<2, 4>::COLS : Tall<4, 4>::COLS; }

// Calls too small for this kernel: a workgroup needs 2 us before its first stage and 1.8 us a stage, so with few stages
// per CU the sliced kernel's smaller workgroups are done sooner, where it takes the shape.  Sliced against tall, by stages
// per CU: k <= 128 and wide d (256 columns a workgroup) 0.5 to 1 1 / 1.36, 2 to 2.5 1 / 1.13, 4.5 to 5 1 / 1.02, 5 to 6
// 1.01, 8 to 10 1.06; k <= 128, d <= 128 1 to 1.5 1 / 1.21, 2.5 to 3 1.01; k > 128 2 to 2.5 1 / 1.15, 4 to 4.5 1.00, 5 to
// 6 1.02 to 1.07 (2 shapes of n = 1000, k = 100, d = 256 12.5 us against 20.7; 4 of n = 5000 23.1 against 24.6; 16 of
// n = 5000 38.3 against 35.8).  Error against float64 at n = 1000 2.0e-7 sliced, 1.7e-7 tall.
bool tall_too_small(int64_t batch, int64_t n, int64_t k, int64_t d)
{
    const int64_t cols = tall_cols(k, d), stages = batch * ((n + TS - 1) / TS) * ((d + cols - 1) / cols);
    return 2 * stages < (k > 128 ? 8 : (d > 128 ? 10 : 5)) * (int64_t)device_cus();
}

bool tall_shape_ok(int64_t n, int64_t k, int64_t d)
{
    return k > 64 && k <= kMaxK && !near_square(k, d) && d >= 4 && d % 4 == 0 && d <= (1 << 20) && n >= 4 * TS;
}

int tall_nsplit(int64_t batch, int64_t n, int64_t k, int64_t d, int64_t cap)
{
    const int64_t dblocks = (d + tall_cols(k, d) - 1) / tall_cols(k, d), base = batch * dblocks;
    const int64_t stages = (n + TS - 1) / TS;
    const int64_t slots = device_cus();  // one workgroup per CU (LDS)
    int64_t most = std::min<int64_t>(stages / 4, cap);  // at least 4 stages per chunk
    int64_t ns = 1;
    double best = 0.0;
    for (int64_t v = 1; v <= most && v * base <= 2 * slots; ++v) {
        const double e = (double)(base * v) / (double)(xcd_rounds(batch * v, dblocks, slots) * slots);
        if (e > best + 0.02) {
            best = e;
            ns = v;
        }
    }
    return (int)ns;
}

template <int RG, int RT>
static hipError_t dispatch_tall(const float *phi, const float *mass, const float *feat, int64_t batch, int64_t n,
                                int64_t k, int64_t d, int ns, float *out, hipStream_t st)
{
    using C = Tall<RG, RT>;
    static bool set = false;
    if (!set) {
        (void)hipFuncSetAttribute((const void *)proj_fwd_tall_kernel<RG, RT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)C::LDS);
        set = true;
    }
    const int dblocks = (int)((d + C::COLS - 1) / C::COLS);
    const int ntiles = (int)(batch * ns);
    const unsigned grid = (unsigned)(8 * dblocks * ((ntiles + 7) / 8));
    hipLaunchKernelGGL((proj_fwd_tall_kernel<RG, RT>), dim3(grid), dim3(TT), C::LDS, st, phi, mass, feat, (int)n, (int)k,
                       (int)d, ns, dblocks, ntiles, out);
    return hipGetLastError();
}

hipError_t launch_project_tall(const float *phi, const float *mass, const float *feat, int64_t batch, int64_t n,
                               int64_t k, int64_t d, int ns, float *A, void *ws, hipStream_t st)
{
    float *out = ns > 1 ? (float *)ws : A;
    hipError_t e;
    switch (tall_class(k, d)) {
    case 0: e = dispatch_tall<2, 4>(phi, mass, feat, batch, n, k, d, ns, out, st); break;
    case 1: e = dispatch_tall<4, 2>(phi, mass, feat, batch, n, k, d, ns, out, st); break;
    case 2: e = dispatch_tall<4, 3>(phi, mass, feat, batch, n, k, d, ns, out, st); break;
    case 3: e = dispatch_tall<4, 4>(phi, mass, feat, batch, n, k, d, ns, out, st); break;
    default: e = dispatch_tall<4, 5>(phi, mass, feat, batch, n, k, d, ns, out, st); break;
    }
    if (e != hipSuccess || ns <= 1) return e;
    return launch_reduce(out, ns, batch, k, d, A, false, st);
}

template <int RG, int RT>
static hipError_t dispatch_tall_items(const FwdItem *items, int nitems, hipStream_t st)
{
    const size_t lds = Tall<RG, RT>::LDS;
    static bool set = false;
    if (!set) {
        (void)hipFuncSetAttribute((const void *)proj_fwd_tall_items_kernel<RG, RT>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        set = true;
    }
    hipLaunchKernelGGL((proj_fwd_tall_items_kernel<RG, RT>), dim3((unsigned)nitems), dim3(TT), lds, st, items);
    return hipGetLastError();
}

hipError_t launch_fwd_tall_items(const FwdItem *items, int nitems, int cls, hipStream_t st)
{
    if (nitems <= 0) return hipSuccess;
    switch (cls) {
    case 0: return dispatch_tall_items<2, 4>(items, nitems, st);
    case 1: return dispatch_tall_items<4, 2>(items, nitems, st);
    case 2: return dispatch_tall_items<4, 3>(items, nitems, st);
    case 3: return dispatch_tall_items<4, 4>(items, nitems, st);
    default: return dispatch_tall_items<4, 5>(items, nitems, st);
    }
}

}  // namespace fmap
