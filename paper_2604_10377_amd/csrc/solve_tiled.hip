// Row systems of order 64 < k_x <= 319 (Eqs. (5)-(7) at large spectral
// resolution), and the adjoint products for any k.
//
// A blocked left-looking Cholesky: the lower triangle of S_i = K + lambda diag(D_i)
// is cut into 32x32 tiles, and the right-hand side is appended as one extra row
// (index k_x), so the factorisation performs the forward substitution L y = r
// on the fly.  A workgroup of 4 or 8 waves keeps the active block column in LDS and the
// finished tiles in its slot of the workspace, and several systems share a CU
// (rowsolve_ll_kernel, described below).

#include <algorithm>

#include "fmap_device.h"
#include "fmap_launch.h"

namespace fmap {

namespace {

constexpr int TLD = 33;                 // row stride of a stored tile (odd: conflict-free columns)
constexpr int TSZ = 32 * TLD;           // floats per tile

__device__ __forceinline__ int packed_col_t(int c, int m) { return c * m - (c * (c - 1)) / 2; }
__device__ __forceinline__ float uniform_f(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
// index of tile (I, J), I >= J, in column-major order of the lower triangle with TR tile rows
__device__ __forceinline__ int tile_index(int I, int J, int TR) { return J * TR - (J * (J - 1)) / 2 + (I - J); }

// LDS scratch of the diagonal-tile routine below (floats, 16-byte aligned)
constexpr int DIAG_LR = 16 * 16;

// Wait states.  The compiler keeps the distances that the hardware asks for between its own instructions, but does not
// see inside the inline assembly here, neither its writes nor its reads.  After a vector instruction that writes a
// register, two must pass before a DPP operand or a permlane swap reads it, and one before a lane read does.  So
//   * the DPP operand x of row_fnma: an s_nop 1 tied to the column's own broadcast (xn); used for the columns after it,
//     it is older;
//   * both registers of each permlane swap, written by moves in assembly (left to the compiler, the two copies are
//     one): swap_pad, where fewer than two instructions of diag_rest stand between;
//   * the next pivot, read from the result of a row_fnma: an s_nop 0 tied to it.
// diag_rest ends with a scheduling barrier, so what stands before it in the source stays before it.  A CPU test counts
// the distances in the compiled code.

// acc -= x_Q y, where x_Q is lane Q of the own row of 16 lanes (a DPP row broadcast in the
// multiply-add; left to the compiler each becomes a move of its own, all held in registers).
template <int Q>
__device__ __forceinline__ void row_fnma(float &acc, float x, float y)
{
    asm volatile("v_fmac_f32_dpp %0, %1, -%2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
                 : "+v"(acc) : "v"(x), "v"(y), "n"(Q));
}
// The subtractions of column P that the next pivot does not need: item I of diag_rest_count(P), in the order in
// which the following columns need them (x: the column's entries, y: the lane's factor).
constexpr int diag_rest_count(int P) { return P < 0 ? 0 : (P < 16 ? 15 : (P < 30 ? 30 - P : 0)); }
template <int P, int I, int END>
__device__ __forceinline__ void diag_rest(float (&s)[16], float x, float y)
{
    if constexpr (I < END && I < diag_rest_count(P)) {
        row_fnma<(P + 2 + I) & 15>(s[(P + 2 + I) & 15], x, y);
        diag_rest<P, I + 1, END>(s, x, y);
    } else {
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Before a permlane swap of a and b, written by assembly with items I .. END - 1 of diag_rest<P> after it
template <int P, int I, int END>
__device__ __forceinline__ void swap_pad(float &a, float &b)
{
    constexpr int between = (diag_rest_count(P) < END ? diag_rest_count(P) : END) - I;
    if constexpr (between < 2) asm volatile("s_nop %2" : "+v"(a), "+v"(b) : "n"(between == 1 ? 0 : 1));
}

// Column C of the factor and column C % 16 of its diagonal block's inverse; see diag_factor_inverse.  pv: the
// pivot.  Dcol: where the own row of the factor goes, Mcol: the own column of the inverse; other lanes have
// addresses there whose contents are not needed.  From pivot to pivot this is a chain of dependent instructions;
// what column P leaves to do (x, y: its values) goes into its gaps.
template <int C, int P>
__device__ __forceinline__ void diag_column(float (&s)[16], float *Dcol, float *Mcol, int row16, float &pv, float &x,
                                            float &y)
{
    constexpr int J = C & 15, N = (C + 1) & 15;
    const float r = __builtin_amdgcn_rsqf(pv);
    diag_rest<P, 0, 3>(s, x, y);
    float l = s[J] * r, l2, xn;
    asm volatile("v_mov_b32 %0, %1" : "=v"(l2) : "v"(l));
    float ri = __builtin_amdgcn_rcpf(pv * r);  // of the diagonal entry of L: scales the inverse
    diag_rest<P, 3, 6>(s, x, y);
    if constexpr (C < 16) {
        swap_pad<P, 3, 6>(l, l2);
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l), __float_as_uint(l2), false, false);
        l = __uint_as_float(sw[0]);
        float l3;
        asm volatile("v_mov_b32 %0, %2\n\tv_mov_b32 %1, %2" : "=&v"(l2), "=&v"(l3) : "v"(l));
        diag_rest<P, 6, 9>(s, x, y);
        swap_pad<P, 6, 9>(l2, l3);
        const auto rw = __builtin_amdgcn_permlane16_swap(__float_as_uint(l2), __float_as_uint(l3), false, false);
        xn = __uint_as_float(row16 == 3 ? rw[1] : rw[0]);
    } else {
        float l3;
        asm volatile("v_mov_b32 %0, %1" : "=v"(l3) : "v"(l));
        diag_rest<P, 6, 9>(s, x, y);
        swap_pad<P, 6, 9>(l2, l3);
        xn = __uint_as_float(__builtin_amdgcn_permlane16_swap(__float_as_uint(l2), __float_as_uint(l3), false, false)[1]);
    }
    const float yn = row16 == 2 ? s[J] * ri : l;
    Dcol[C] = l;
    Mcol[J * TLD] = yn;
    diag_rest<P, 9, 11>(s, x, y);
    asm volatile("s_nop 1" : "+v"(xn));  // a DPP operand next
    if constexpr (C < 31) {
        row_fnma<N>(s[N], xn, yn);  // the next pivot's column
        diag_rest<P, 11, 12>(s, x, y);
        asm volatile("s_nop 0" : "+v"(s[N]));  // a lane read next
        pv = uniform_f(readlane(s[N], C < 15 ? C + 1 : 33 + C));
    }
    diag_rest<P, C < 31 ? 12 : 11, 16>(s, x, y);
    x = xn;
    y = yn;
}

// Columns C0 .. C0 + 15
template <int C0, int I = 0>
__device__ __forceinline__ void diag_columns(float (&s)[16], float *Dcol, float *Mcol, int row16, float &pv, float &x,
                                             float &y)
{
    if constexpr (I < 16) {
        diag_column<C0 + I, I == 0 ? -1 : C0 + I - 1>(s, Dcol, Mcol, row16, pv, x, y);
        diag_columns<C0, I + 1>(s, Dcol, Mcol, row16, pv, x, y);
    } else {
        diag_rest<C0 + 15, 0, 16>(s, x, y);
    }
}

// One wave (64 lanes): Cholesky factor of the 32 x 32 diagonal tile Dt (rows at stride TLD, lower part, the
// first kxl columns; rows past kxl, e.g. the appended right-hand side row, are eliminated with them), and the
// inverse of the factor, Minv[q][c] at q * TLD + c (rows and columns past kxl zero).  Returns 0, or 1 + the
// first column whose pivot is not positive and finite (then Dt and Minv hold garbage).
//   * lane (i, g), i = lane % 16 of row g of lanes, holds 16 entries in registers, and step c subtracts from each a
//     DPP row broadcast times a value of the lane: 16 instructions for all of the following.  While c < 16, rows 0
//     and 1 of lanes hold columns 0..15 of tile rows i and 16 + i, row 3 holds columns 16..31 of tile row 16 + i,
//     and row 2 column i of the inverse of the upper diagonal block, which starts as a column of the identity and
//     takes the same broadcasts.  From c = 16 on, row 3 goes on with tile row 16 + i and row 2 starts on the lower
//     block's inverse.  Column c is scaled where it is held and spread to the other rows of lanes by permlane
//     swaps.  Finished columns go to LDS at once; their registers hold garbage from then on.  Columns past kxl are
//     eliminated as well and come out as garbage, which reaches neither the columns before them nor Minv;
//   * then the lower-left block M21 = -M22 L21 M11 as two 16 x 16 x 16 products on the float32 matrix cores.
// Bound by the instructions of the one wave, some 30 per column at five cycles each (8-byte encodings), and what
// stands around the columns: 8200 cycles alone on its SIMD; 14400 when each entry L_qc was a lane read and the
// inverse followed the factor.
// Lr (16 x 16) is scratch for the product L21 M11.
__device__ __forceinline__ int diag_factor_inverse(float *Dt, float *Lr, float *Minv, int kxl, int lane)
{
    // the lane index made opaque, so its masks are formed where used, not hoisted into registers
    asm volatile("" : "+v"(lane));
    const int l32 = lane & 31, i16 = lane & 15, k4 = lane >> 4;
    float s[16];
    {
        const float *D = Dt + l32 * TLD + (lane < 32 ? 0 : 16);
#pragma unroll
        for (int q = 0; q < 16; ++q) s[q] = D[q];
        // all loaded before any is replaced (else a branch around each load)
        asm volatile(""
                     : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]), "+v"(s[4]), "+v"(s[5]), "+v"(s[6]), "+v"(s[7]),
                       "+v"(s[8]), "+v"(s[9]), "+v"(s[10]), "+v"(s[11]), "+v"(s[12]), "+v"(s[13]), "+v"(s[14]),
                       "+v"(s[15]));
#pragma unroll
        for (int q = 0; q < 16; ++q) s[q] = k4 == 2 ? (q == i16 ? 1.f : 0.f) : s[q];
    }
    float pv = uniform_f(readlane(s[0], 0)), x = 0.f, y = 0.f;
    // rows 2 and 3 of lanes write copies of rows 0 and 1 of Dt; all but row 2 write to the rows of Minv filled later
    diag_columns<0>(s, Dt + l32 * TLD, Minv + (k4 == 2 ? 0 : 16 * TLD) + i16, k4, pv, x, y);
#pragma unroll
    for (int q = 0; q < 16; ++q) s[q] = k4 == 2 ? (q == i16 ? 1.f : 0.f) : s[q];
    // row 3 writes Dt, the others the scratch; row 2 writes the lower block of Minv, the others the block on its left
    diag_columns<16>(s, k4 == 3 ? Dt + l32 * TLD : Lr + i16, Minv + 16 * TLD + (k4 == 2 ? 16 : 0) + i16, k4, pv, x, y);
    // a pivot that is zero, negative, infinite or NaN times its reciprocal root is NaN, and so are the later ones
    const float dg = Dt[l32 * TLD + l32];
    const unsigned bad = (unsigned)__ballot(lane < kxl && dg != dg);  // kxl <= 32
    if (bad != 0u) return __ffs((int)bad);
    // the block right of M11 is zero, and so are rows and columns past kxl (the last tile's)
    if (lane < 16) {
#pragma unroll
        for (int q = 0; q < 16; ++q) Minv[q * TLD + 16 + lane] = 0.f;
    }
    if (kxl < 32) {
        for (int q = min(kxl, 32); q < 32; ++q)
            if (lane < 32) Minv[q * TLD + lane] = 0.f;
    }
    __builtin_amdgcn_wave_barrier();
    {
        // 16 x 16 x 4 float32 matrix-core steps: lane (i, k) = (lane % 16, lane / 16) supplies A[i][k] and
        // B[k][i]; the result row 4 (lane / 16) + r, column lane % 16 is register r
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < 4; ++st)  // T = L21 M11
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(Dt[(16 + i16) * TLD + 4 * st + k4],
                                                       Minv[(4 * st + k4) * TLD + i16], acc, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) Lr[(4 * k4 + r) * 16 + i16] = acc[r];
        __builtin_amdgcn_wave_barrier();
        f32x4 acc2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int st = 0; st < 4; ++st)  // M21 = -M22 T
            acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(Minv[(16 + i16) * TLD + 16 + 4 * st + k4],
                                                        Lr[(4 * st + k4) * 16 + i16], acc2, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) Minv[(16 + 4 * k4 + r) * TLD + i16] = 16 + 4 * k4 + r < kxl ? -acc2[r] : 0.f;
    }
    __builtin_amdgcn_wave_barrier();
    return 0;
}

}  // namespace

enum { RT_FWD = 0, RT_BWD_RECOMPUTE = 2 };

// ---------------------------------------------------------------------------
// The left-looking kernel, 64 < k_x <= 319: several row systems per CU.
//
// Keeping every tile of a system in LDS (118 KB at k_x = 200) would hold a CU
// to one system, idle while one wave factorises a diagonal tile.  Here a
// workgroup of 4 (8) waves keeps only the active block column in LDS (37 KB in all
// at k_x = 200) and writes each finished tile L_Ip, and the inverse of each
// diagonal tile, to its own slot of the workspace (32 x 32 row-major tiles in
// the lower-triangle order of the tile grid; the diagonal positions hold the
// inverses).  Two to four systems then share a CU and hide each other's serial
// diagonal steps.  Step p:
//   1. each wave loads its own tiles of block column p of
//      S = K + lambda diag(D_i) (the right-hand side as the appended row)
//      straight into its accumulators, with no barrier before step 2;
//   2. left-looking update S_Ip -= sum_{q < p} L_Iq L_pq^T on the float32
//      matrix cores, the L tiles read from the slot straight into the operand
//      registers: lane (m, h) supplies row m, columns 16 h .. 16 h + 15, with
//      the K order of the matrix-core steps permuted alike for both operands.
//      One wave updates the diagonal tile and goes on to step 3 at once, while
//      the others update the tiles below it, and the next diagonal tile as far as
//      it goes, so that the serial wave of the next step starts one product short
//      of done; the updated tiles go to LDS;
//   3. that wave factorises the diagonal tile and forms its inverse
//      (diag_factor_inverse);
//   4. the panel L_Ip = S_Ip L_pp^{-T} on the matrix cores, stored to the slot.
// The appended row carries the forward substitution, so its tile row yields
// y.  The back substitution runs block by block from the last: the finished
// blocks' contribution L_Ip^T c_I as matrix-vector products over the slot's
// tiles, then c_p = L_pp^{-T} v as one product with the stored inverse.
// ---------------------------------------------------------------------------
// Waves per workgroup: where two workgroups fill a CU's workspace slots (k_x >= 224), eight waves each; four where
// four do.  Eight shorten the serial path of one system, and the registers allow 16 waves per CU either way.
// k = 256, one system per CU: the factorisation took 218000 cycles with four waves, 187000 with eight.
constexpr int ll_waves(int TRM) { return TRM == 10 ? 8 : 4; }
constexpr int LTS = 32 * 32;    // floats per tile in the workspace slot

constexpr int ll_lds_floats(int TRM) { return TRM * TSZ + TSZ + DIAG_LR + 2 * TRM * 32 + ll_waves(TRM) + 4; }

__device__ __forceinline__ f32x4 ldg4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }

// STORE: the factor is written to Lout (forward mode with stored factors).
template <int TMAX, int MODE, bool STORE>
__global__ __launch_bounds__(64 * ll_waves(TMAX)) __attribute__((amdgpu_waves_per_eu(4))) void rowsolve_ll_kernel(
    const float *__restrict__ K, const float *__restrict__ rhs, const float *__restrict__ ex,
    const float *__restrict__ ey, const float *__restrict__ lam, int mask_kind, float gamma, int kx, int ky, int nsys,
    float *out, float *__restrict__ Lout, int *__restrict__ info, const float *__restrict__ Cfwd,
    float *__restrict__ dlam_part, float *__restrict__ Lws, int cus, const int *__restrict__ only)
{
    constexpr int TRM = TMAX;
    constexpr int NW = ll_waves(TMAX), NTHR = 64 * NW;
    constexpr int NTL = TMAX * (TMAX + 1) / 2;
    extern __shared__ __align__(16) float smem[];
    float *bc = smem;                    // tile j: rows 32 (p + j) .. 32 (p + j) + 31 of block column p
    float *s_minv = bc + TRM * TSZ;      // inverse of the diagonal tile, Minv[q][c] at q * TLD + c
    float *s_lr = s_minv + TSZ;          // scratch of the diagonal-tile routine
    float *s_dval = s_lr + DIAG_LR;      // mask row D_i
    float *s_vec = s_dval + TRM * 32;    // y, then c
    float *s_red = s_vec + TRM * 32;     // [NW]
    int *s_fail = reinterpret_cast<int *>(s_red + NW);
    float *Ls = Lws + (size_t)blockIdx.x * NTL * LTS;

    const int tid = threadIdx.x, wave = tid >> 6;
    // the wave that runs the serial diagonal steps: different for the workgroups that share a CU (ids one grid
    // round of CUs apart), so that their diagonal chains do not all land on the same SIMD
    const int dwave = (blockIdx.x / cus) % NW;
    const int T = (kx + 31) >> 5;   // column tiles
    const int TR = (kx + 32) >> 5;  // tile rows (row kx is the right-hand side)
    const int AR = kx >> 5, ar = kx & 31;

    for (int sys = blockIdx.x; sys < nsys; sys += gridDim.x) {
        const int p = sys / ky, i = sys % ky;
        if (only && __builtin_amdgcn_readfirstlane(only[p]) == 0) continue;  // uniform: before any barrier
        int tid = threadIdx.x;  // opaque per system, as in the steps below
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63;
        // ---- lambda, mask row, normaliser -----------------------------------------------
        const float lamv = lam[p];
        int fail0 = (!(lamv >= 0.f) || !isfinite(lamv)) ? -1 : 0;
        MaskParams mp;
        mp.kind = mask_kind;
        mp.gamma = gamma;
        mp.inv_scale = 1.f;
        if (mask_kind == 1) {
            float mx = -INFINITY;
            for (int q = tid; q < kx; q += NTHR) mx = fmaxf(mx, ex[(size_t)p * kx + q]);
            for (int q = tid; q < ky; q += NTHR) mx = fmaxf(mx, ey[(size_t)p * ky + q]);
            mx = wave_max(mx);
            if (lane == 0) s_red[wave] = mx;
            __syncthreads();
            mx = s_red[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) mx = fmaxf(mx, s_red[w]);
            if ((!(mx > 0.f) || !isfinite(mx)) && fail0 == 0) fail0 = -2;
            mp.inv_scale = 1.f / mx;
        }
        const float muy = ey[(size_t)p * ky + i];
        for (int q = tid; q < TRM * 32; q += NTHR) {
            const float dv = (q < kx && fail0 != -2) ? mask_entry(muy, ex[(size_t)p * kx + q], mp) : 0.f;
            s_dval[q] = dv;
            s_vec[q] = 0.f;
        }
        if (tid == 0) *s_fail = fail0;
        const float lsh = fail0 == 0 ? lamv : 0.f;  // the diagonal shift is lsh * D_iq
        __syncthreads();

        const float *Kp = K + (size_t)p * kx * kx;
        const float *rp = rhs + ((size_t)p * ky + i) * kx;
        for (int ps = 0; ps < T; ++ps) {
            if (__builtin_amdgcn_readfirstlane(*s_fail) != 0) break;
            // the thread index, made opaque per step: lane-dependent masks and addresses (the identity column
            // of the inverse, the appended row's accumulator slot, the tile offsets of the loads) are then
            // formed where they are used, not hoisted out of every loop into registers (they had taken some 40
            // to 80 registers for the whole kernel)
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            const int lane = tid & 63;
            const int l32 = lane & 31, half = lane >> 5;
            const int nt = TR - ps;                 // tiles of the block column
            const int kxl = min(32, kx - 32 * ps);  // columns of this block
            // ---- 1. block column ps: S_Ip = K_Ip (+ the shift on the diagonal; row k_x is the right-hand
            //         side, rows and columns past it are zero), minus sum_{q < ps} L_Iq L_pq^T ------------
            // Each wave loads its own tiles straight into its accumulators (no barrier between the loads and
            // the update).  The diagonal-tile wave takes the diagonal tile alone and goes straight on to
            // factorise it (step 3, its own LDS writes, no barrier), while the other waves take the tiles
            // below it and, from step 1 on, as tile nt the next diagonal tile less its products of the blocks
            // before ps: the diagonal-tile wave then starts step ps + 1 from that, one product short.  It is
            // passed on in a tile that the shrinking block column no longer uses, the last one and the one before
            // it in turn (the last is free from step 1 on, the other from step 2).
            {
                const int j0 = wave == dwave ? 0 : 1 + (wave - dwave + NW - 1) % NW;
                const int jend = wave == dwave ? 1 : nt + (ps >= 1 && ps + 1 < T ? 1 : 0);
                for (int j = j0; j < jend; j += NW - 1) {
                    const bool ahead = j == nt;           // the next diagonal tile
                    const bool begun = j == 0 && ps >= 2;  // the diagonal tile begun in the step before
                    const int cb = ahead ? ps + 1 : ps;   // block column of the tile
                    const int q0 = begun ? ps - 1 : 0;
                    // lane-derived values formed per tile (kept out of the registers held across the update)
                    int ln = lane;
                    asm volatile("" : "+v"(ln));
                    const int l32 = ln & 31, half = ln >> 5;
                    const int col = 32 * cb + l32;
                    const int colc = min(col, kx - 1);
                    float *X = bc + (ahead ? TRM - 1 - ((ps + 1) & 1) : j) * TSZ;
                    const int I = ahead ? cb : ps + j;
                    const int off = l32 * 32 + 16 * half;
                    // this tile's entries of K (unconditional loads from clamped addresses) and the first
                    // tile pair of the update, all in flight together
                    f32x16 acc;
                    if (begun) {
                        const float *B = bc + (TRM - 1 - (ps & 1)) * TSZ;
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] = B[acc32_row(r, ln) * TLD + l32];
                    } else {
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int rowc = min(32 * I + acc32_row(r, ln), kx);
                            acc[r] = *(rowc == kx ? rp + colc : Kp + (size_t)rowc * kx + colc);
                        }
                    }
                    f32x4 a0[4], b0[4];
                    if (ps > 0) {
                        const float *ap = Ls + (size_t)tile_index(I, q0, TR) * LTS + off;
                        const float *bp = Ls + (size_t)tile_index(cb, q0, TR) * LTS + off;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            a0[u] = ldg4(ap + 4 * u);
                            b0[u] = ldg4(bp + 4 * u);
                        }
                    }
                    if (!begun) {
                        const float dsh = lsh * s_dval[col];  // the shift of this column's diagonal entry
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            const int row = 32 * I + acc32_row(r, ln);
                            const float v = acc[r];
                            float x = 0.f;
                            if (row < kx && col < kx) x = v + (row == col ? dsh : 0.f);
                            else if (row == kx && col < kx) x = v;
                            acc[r] = x;
                        }
                    }
                    // whole tile pairs (16 floats of each operand per lane), the next pair in flight while one is
                    // multiplied
                    for (int q = q0; q < ps; ++q) {
                        const int qn = min(q + 1, ps - 1);
                        const float *ap = Ls + (size_t)tile_index(I, qn, TR) * LTS + off;
                        const float *bp = Ls + (size_t)tile_index(cb, qn, TR) * LTS + off;
                        f32x4 a1[4], b1[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            a1[u] = ldg4(ap + 4 * u);
                            b1[u] = ldg4(bp + 4 * u);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc = mfma32x32x2(-a0[u][e], b0[u][e], acc);
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            a0[u] = a1[u];
                            b0[u] = b1[u];
                        }
                    }
#pragma unroll
                    for (int r = 0; r < 16; ++r) X[acc32_row(r, ln) * TLD + l32] = acc[r];
                }
            }
            // ---- 3. diagonal tile and its inverse (one wave) ----------------------------------
            if (wave == dwave) {
                __builtin_amdgcn_s_setprio(3);  // the one serial step: ahead of the waves that share its SIMD
                const int f = diag_factor_inverse(bc, s_lr, s_minv, kxl, lane);
                __builtin_amdgcn_s_setprio(0);
                if (f != 0) {
                    if (lane == 0) *s_fail = 32 * ps + f;
                } else {
                    // the inverse also into the slot's diagonal position (rows 2 u + half)
                    float *Mi = Ls + (size_t)tile_index(ps, ps, TR) * LTS;
#pragma unroll
                    for (int u = 0; u < 16; ++u) Mi[(2 * u + half) * 32 + l32] = s_minv[(2 * u + half) * TLD + l32];
                }
            }
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(*s_fail) != 0) break;
            if (AR == ps && tid < 32) s_vec[32 * ps + tid] = tid < kxl ? bc[ar * TLD + tid] : 0.f;  // y of this block
            if (STORE) {
                // L_pp into the packed factor, consecutive threads on consecutive rows of a column
                float *Lo = Lout + ((size_t)p * ky + i) * (size_t)(kx * (kx + 1) / 2);
                for (int e = tid; e < 1024; e += NTHR) {
                    const int c = e >> 5, r = e & 31;
                    if (r >= c && r < kxl) Lo[packed_col_t(32 * ps + c, kx) + (r - c)] = bc[r * TLD + c];
                }
            }
            // ---- 4. panel L_Ip = S_Ip Minv^T (I > ps), formed transposed: lane l32 holds row l32 of the tile, register
            //         r column acc32_row(r).  Four columns at a time go to the row-major slot, and whole columns
            //         (consecutive lanes on consecutive rows) to the packed factor, straight from the registers ----
            for (int j = 1 + wave; j < nt; j += NW) {
                const int I = ps + j;
                const float *X = bc + j * TSZ;
                f32x16 nv = zero16();
#pragma unroll
                for (int t = 0; t < 16; ++t)
                    nv = mfma32x32x2(s_minv[l32 * TLD + 2 * t + half], X[l32 * TLD + 2 * t + half], nv);
                float *Lt = Ls + (size_t)tile_index(I, ps, TR) * LTS + l32 * 32;
#pragma unroll
                for (int r = 0; r < 16; r += 4)
                    *reinterpret_cast<f32x4 *>(Lt + acc32_row(r, lane)) = f32x4{nv[r], nv[r + 1], nv[r + 2], nv[r + 3]};
                if (STORE && 32 * I + l32 < kx) {
                    float *Lo = Lout + ((size_t)p * ky + i) * (size_t)(kx * (kx + 1) / 2);
                    int c = 32 * ps + 4 * half;  // a block with rows below it is 32 columns wide
                    unsigned e = (unsigned)(packed_col_t(c, kx) + 32 * I + l32 - c);
                    asm volatile("" : "+v"(c), "+v"(e));  // else sixteen offsets are carried from tile to tile
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        Lo[e] = nv[r];
                        const int step = (r & 3) == 3 ? 5 : 1;  // columns to the next register's
                        e += step * (kx - c - 1) - step * (step - 1) / 2;
                        c += step;
                    }
                }
                if (I == AR && l32 == ar) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) s_vec[32 * ps + acc32_row(r, lane)] = nv[r];
                }
            }
            __syncthreads();
        }
        const int fail = __builtin_amdgcn_readfirstlane(*s_fail);

        // ---- back substitution L^T c = y, column-oriented, from the last block ---------------------------
        // The inverses of the diagonal tiles go to the block-column buffer (free now, T <= TRM tiles).  Step p:
        // c_p = L_pp^{-T} y_p from LDS, then y_q -= L_pq^T c_p for every q < p, wave w taking q = w, w + 4, ...
        // with the tiles' loads issued before c_p is formed.
        if (fail == 0) {
            // lane values formed here, from an opaque thread index (not held from the kernel's start)
            int tb = threadIdx.x;
            asm volatile("" : "+v"(tb));
            const int tid = tb, lane = tb & 63;
            const int l32 = lane & 31, half = lane >> 5;
            for (int e0 = tid; e0 < T * 1024; e0 += 8 * NTHR) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = min(e0 + NTHR * u, T * 1024 - 1);
                    v[u] = Ls[(size_t)tile_index(e >> 10, e >> 10, TR) * LTS + (e & 1023)];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = e0 + NTHR * u;
                    if (e < T * 1024) bc[(e >> 10) * TSZ + ((e >> 5) & 31) * TLD + (e & 31)] = v[u];
                }
            }
            __syncthreads();
            for (int ps = T - 1; ps >= 0; --ps) {
                const int kxl = min(32, kx - 32 * ps);
                // this wave's first tile (ps, q = wave): rows h, h + 2, ... of column l32, in flight while c_ps is
                // formed
                float lv[16];
                {
                    const float *Lt = Ls + (size_t)tile_index(ps, min(wave, max(ps - 1, 0)), TR) * LTS;
#pragma unroll
                    for (int u = 0; u < 16; ++u) lv[u] = Lt[(2 * u + half) * 32 + l32];
                }
                if (wave == dwave && lane < 32) {
                    // c_j = sum_q Minv[q][j] y_q
                    const float *Mi = bc + ps * TSZ;
                    float c = 0.f;
#pragma unroll
                    for (int q = 0; q < 32; ++q) c += Mi[q * TLD + l32] * s_vec[32 * ps + q];
                    s_vec[32 * ps + l32] = l32 < kxl ? c : 0.f;
                }
                __syncthreads();
                if (wave < ps) {
                    float z = 0.f;
#pragma unroll
                    for (int u = 0; u < 16; ++u) z += lv[u] * s_vec[32 * ps + 2 * u + half];
                    z += __shfl_xor(z, 32, 64);
                    if (half == 0) s_vec[32 * wave + l32] -= z;
                }
                for (int q = wave + NW; q < ps; q += NW) {  // further earlier blocks
                    const float *Lt = Ls + (size_t)tile_index(ps, q, TR) * LTS;
#pragma unroll
                    for (int u = 0; u < 16; ++u) lv[u] = Lt[(2 * u + half) * 32 + l32];
                    float z = 0.f;
#pragma unroll
                    for (int u = 0; u < 16; ++u) z += lv[u] * s_vec[32 * ps + 2 * u + half];
                    z += __shfl_xor(z, 32, 64);
                    if (half == 0) s_vec[32 * q + l32] -= z;
                }
                __syncthreads();
            }
        }

        // ---- outputs ----------------------------------------------------------------------
        for (int q = tid; q < kx; q += NTHR) out[((size_t)p * ky + i) * kx + q] = fail == 0 ? s_vec[q] : NAN;
        if (info && tid == 0) info[(size_t)p * ky + i] = fail;
        if (MODE != RT_FWD && dlam_part) {
            float term = 0.f;
            for (int q = tid; q < (tid < 256 ? kx : 0); q += 256)  // by 256 threads whatever the waves: one order
                term += (fail == 0 ? s_vec[q] : NAN) * s_dval[q] * Cfwd[((size_t)p * ky + i) * kx + q];
            term = wave_sum(term);
            if (lane == 0) s_red[wave] = term;
            __syncthreads();
            if (tid == 0) dlam_part[(size_t)p * ky + i] = -((s_red[0] + s_red[1]) + (s_red[2] + s_red[3]));
        }
        __syncthreads();  // LDS and the slot are reused by the next system
    }
}

// ---------------------------------------------------------------------------
// Batched products for the adjoint at any k (operands streamed from global
// memory / L2).  Out[p] (M x N, row-major) = sum over two K-segments s of
// sign_s * X_s Y_s, where X_s is M x K_s read as stored ("N") or as the
// transpose of a K_s x M row-major array ("T"), and Y_s is K_s x N row-major.
// One 4-wave workgroup per 32x32 output tile.  K is cut into batches of 16;
// wave w takes batches w, w + 4, ... of each segment and keeps the loads of the
// next three batches in flight while it multiplies the current one.  The four partial tiles are summed
// through LDS in wave order.
// ---------------------------------------------------------------------------
struct GemmSeg {
    const float *X;
    const float *Y;
    int K;
    int transX;  // 1: X given as K x M row-major
    int ldx, ldy;
    long long strideX, strideY;  // per pair
    float sign;
};

// X load modes: 0 every segment's X transposed; 1 one segment, X as stored with 16-byte aligned rows and
// K % 8 == 0 (two 16-byte loads per lane and batch); 2 any segments and layouts.
struct GemmBatch {
    float a[8], b[8];
};

template <int XM>
__device__ __forceinline__ GemmBatch gemm_batch_load(const float *X, const float *Y, int K, int ldx, int ldy,
                                                     bool transX, int kb, int mc, int nc, int half)
{
    // lane (m, half) supplies k = kb + 8 half + u to matrix step u; every address is clamped into the
    // operand, and entries past K are masked when the operands are formed
    GemmBatch g;
    if constexpr (XM == 1) {
        const int k0 = min(kb + 8 * half, K - 8);
        const f32x4 *px = reinterpret_cast<const f32x4 *>(X + (size_t)mc * ldx + k0);
        const f32x4 v0 = px[0], v1 = px[1];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            g.a[u] = v0[u];
            g.a[4 + u] = v1[u];
        }
    } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int kc = min(kb + 8 * half + u, K - 1);
            const bool tr = XM == 0 || transX;
            g.a[u] = X[tr ? (size_t)kc * ldx + mc : (size_t)mc * ldx + kc];
        }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) g.b[u] = Y[(size_t)min(kb + 8 * half + u, K - 1) * ldy + nc];
    return g;
}

template <int XM>
__global__ __launch_bounds__(256) void batched_gemm_kernel(GemmSeg s0, GemmSeg s1, int nseg, int M, int N,
                                                           int tilesM, int tilesN, float *__restrict__ Out,
                                                           long long strideO)
{
    __shared__ float red[4][16][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int tiles = tilesM * tilesN;
    const int p = blockIdx.x / tiles;
    const int t = blockIdx.x % tiles;
    const int I = t / tilesN, Jt = t % tilesN;
    const int m = I * 32 + l32, n = Jt * 32 + l32;
    const bool mok = m < M, nok = n < N;
    const int mc = min(m, M - 1), nc = min(n, N - 1);
    auto keep = [](float x, bool ok) { return __uint_as_float(__float_as_uint(x) & (ok ? ~0u : 0u)); };
    // this wave's steps: the batches of 16 k starting at 16 (wave + 4 j) of segment 0, then those of
    // segment 1; their count is rounded up to a multiple of 4 for the four-buffer rotation (a step past
    // the last is masked to zero)
    const int nb0 = max(0, ((s0.K + 15) / 16 - wave + 3) / 4);
    const int nb1 = nseg > 1 ? max(0, ((s1.K + 15) / 16 - wave + 3) / 4) : 0;
    const int nsteps = (nb0 + nb1 + 3) & ~3;
    const float *X0 = s0.X + (long long)p * s0.strideX, *Y0 = s0.Y + (long long)p * s0.strideY;
    const float *X1 = s1.X + (long long)p * s1.strideX, *Y1 = s1.Y + (long long)p * s1.strideY;
    auto load = [&](int st) {
        const bool first = st < nb0 || nseg == 1;
        const int kb = 16 * (wave + 4 * (first ? st : st - nb0));
        return first ? gemm_batch_load<XM>(X0, Y0, s0.K, s0.ldx, s0.ldy, s0.transX, kb, mc, nc, half)
                     : gemm_batch_load<XM>(X1, Y1, s1.K, s1.ldx, s1.ldy, s1.transX, kb, mc, nc, half);
    };
    f32x16 acc = zero16();
    auto mma = [&](int st, const GemmBatch &g) {
        const bool first = st < nb0 || nseg == 1;
        const int kb = 16 * (wave + 4 * (first ? st : st - nb0));
        const int K = first ? s0.K : s1.K;
        const float sign = first ? s0.sign : s1.sign;
        const bool live = st < nb0 + nb1;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool kok = live && kb + 8 * half + u < K;
            acc = mfma32x32x2(keep(sign * g.a[u], mok && kok), keep(g.b[u], nok && kok), acc);
        }
    };
    GemmBatch g0 = load(0), g1 = load(1), g2 = load(2), g3;
    for (int st = 0; st < nsteps; st += 4) {
        g3 = load(st + 3);
        mma(st, g0);
        g0 = load(st + 4);
        mma(st + 1, g1);
        g1 = load(st + 5);
        mma(st + 2, g2);
        g2 = load(st + 6);
        mma(st + 3, g3);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[r];
    __syncthreads();
    float *O = Out + (long long)p * strideO;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
        const int r = 4 * wave + rr;
        const float v = ((red[0][r][lane] + red[1][r][lane]) + red[2][r][lane]) + red[3][r][lane];
        const int row = I * 32 + acc32_row(r, lane);
        if (row < M && nok) O[(size_t)row * N + n] = v;
    }
}

// Sum of the per-row dlambda terms of each pair, in row order.
__global__ void dlam_sum_kernel(const float *__restrict__ part, int P, int ky, float *__restrict__ dlam)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= P) return;
    float s = 0.f;
    for (int i = 0; i < ky; ++i) s += part[(size_t)p * ky + i];
    dlam[p] = s;
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------

static int cu_count()
{
    int dev = 0, c = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c <= 0) return 256;
    return c;
}

// Workgroups (and workspace slots) of the left-looking launch: up to four per CU.
static int64_t ll_slots(int64_t nsys)
{
    const int64_t cap = 4 * (int64_t)cu_count();
    return nsys < cap ? nsys : cap;
}

// Tile rows of the instance for k_x (k_x + 1 rows, with the appended right-hand side)
static int ll_tmax(int64_t kx) { return kx < 128 ? 4 : (kx < 224 ? 7 : 10); }

size_t tiled_workspace_bytes(int64_t P, int64_t kx, int64_t ky)
{
    const int64_t tm = ll_tmax(kx);
    return (size_t)ll_slots(P * ky) * (tm * (tm + 1) / 2) * LTS * sizeof(float);
}

template <int TMAX, int MODE, bool STORE>
static void launch_ll(const float *K, const float *rhs, const float *ex, const float *ey, const float *lam,
                      int mask_kind, float gamma, int64_t P, int64_t kx, int64_t ky, float *out, float *Lout, int *info,
                      const float *Cfwd, float *dlam_part, float *ws, hipStream_t st, const int *only)
{
    const size_t lds = (size_t)ll_lds_floats(TMAX) * sizeof(float);
    static bool attr = false;
    if (!attr) {
        (void)hipFuncSetAttribute((const void *)rowsolve_ll_kernel<TMAX, MODE, STORE>,
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        attr = true;
    }
    // one round of resident workgroups (the runtime's occupancy for this instance, at most the four per CU the
    // workspace holds slots for): a persistent grid larger than what fits would leave the surplus workgroups
    // waiting for whole early workgroups, which loop over several systems each.  At TMAX = 10 the
    // registers allow two workgroups of eight waves.
    static int per_cu = 0;
    if (per_cu == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, (const void *)rowsolve_ll_kernel<TMAX, MODE, STORE>,
                                                         64 * ll_waves(TMAX), lds) !=
                hipSuccess ||
            n < 1)
            n = 1;
        const int cap = TMAX == 10 ? 2 : 4;
        per_cu = n < cap ? n : cap;
    }
    const int64_t nsys = P * ky;
    const int64_t grid = std::min<int64_t>(nsys, (int64_t)per_cu * cu_count());
    hipLaunchKernelGGL((rowsolve_ll_kernel<TMAX, MODE, STORE>), dim3((unsigned)grid), dim3(64 * ll_waves(TMAX)), lds, st, K,
                       rhs, ex, ey, lam,
                       mask_kind, gamma, (int)kx, (int)ky, (int)nsys, out, Lout, info, Cfwd, dlam_part, ws, cu_count(),
                       only);
}

void launch_rowsolve_tiled(int mode, const float *K, const float *rhs, const float *ex, const float *ey,
                           const float *lam, int mask_kind, float gamma, int64_t P, int64_t kx, int64_t ky, float *out,
                           float *Lout, int *info, const float *Cfwd, float *dlam_part, float *tws, hipStream_t st,
                           const int *only)
{
    const int tm = ll_tmax(kx);
#define FMAP_LL(TM, MD, SF) launch_ll<TM, MD, SF>(K, rhs, ex, ey, lam, mask_kind, gamma, P, kx, ky, out, Lout, info, \
                                                  Cfwd, dlam_part, tws, st, only)
    if (mode == RT_FWD && Lout) {
        if (tm == 4) FMAP_LL(4, RT_FWD, true);
        else if (tm == 7) FMAP_LL(7, RT_FWD, true);
        else FMAP_LL(10, RT_FWD, true);
    } else if (mode == RT_FWD) {
        if (tm == 4) FMAP_LL(4, RT_FWD, false);
        else if (tm == 7) FMAP_LL(7, RT_FWD, false);
        else FMAP_LL(10, RT_FWD, false);
    } else {
        if (tm == 4) FMAP_LL(4, RT_BWD_RECOMPUTE, false);
        else if (tm == 7) FMAP_LL(7, RT_BWD_RECOMPUTE, false);
        else FMAP_LL(10, RT_BWD_RECOMPUTE, false);
    }
#undef FMAP_LL
}

static void gemm(const GemmSeg &s0, const GemmSeg *s1, int64_t P, int M, int N, float *Out, long long strideO,
                 hipStream_t st)
{
    const int tM = (M + 31) / 32, tN = (N + 31) / 32;
    const unsigned grid = (unsigned)(P * tM * tN);
    GemmSeg z = s0;
    z.K = 0;
    const int nseg = s1 ? 2 : 1;
    const GemmSeg &t1 = s1 ? *s1 : z;
    auto aligned = [](const GemmSeg &g) {
        return g.ldx % 4 == 0 && g.strideX % 4 == 0 && g.K >= 8 && g.K % 8 == 0 && ((uintptr_t)g.X & 15) == 0;
    };
    if (s0.transX && (!s1 || s1->transX))
        hipLaunchKernelGGL(batched_gemm_kernel<0>, dim3(grid), dim3(256), 0, st, s0, t1, nseg, M, N, tM, tN, Out,
                           strideO);
    else if (!s1 && !s0.transX && aligned(s0))
        hipLaunchKernelGGL(batched_gemm_kernel<1>, dim3(grid), dim3(256), 0, st, s0, t1, nseg, M, N, tM, tN, Out,
                           strideO);
    else
        hipLaunchKernelGGL(batched_gemm_kernel<2>, dim3(grid), dim3(256), 0, st, s0, t1, nseg, M, N, tM, tN, Out,
                           strideO);
}

// W = V^T C + C^T V (into Wbuf), dB = V A, dA = V^T B - W A.
void launch_adjoint_general(const float *V, const float *C, const float *A, const float *B, int64_t P, int64_t kx,
                            int64_t ky, int64_t d, float *Wbuf, const float *dlam_part, float *dlam, float *dA,
                            float *dB, hipStream_t st)
{
    const long long skk = kx * ky, sxd = kx * d, syd = ky * d, sww = kx * kx;
    GemmSeg w0{V, C, (int)ky, 1, (int)kx, (int)kx, skk, skk, 1.f};
    GemmSeg w1{C, V, (int)ky, 1, (int)kx, (int)kx, skk, skk, 1.f};
    gemm(w0, &w1, P, (int)kx, (int)kx, Wbuf, sww, st);
    GemmSeg b0{V, A, (int)kx, 0, (int)kx, (int)d, skk, sxd, 1.f};
    gemm(b0, nullptr, P, (int)ky, (int)d, dB, syd, st);
    GemmSeg a0{V, B, (int)ky, 1, (int)kx, (int)d, skk, syd, 1.f};
    GemmSeg a1{Wbuf, A, (int)kx, 1, (int)kx, (int)d, sww, sxd, -1.f};  // W symmetric: W^T = W
    gemm(a0, &a1, P, (int)kx, (int)d, dA, sxd, st);
    if (dlam)
        hipLaunchKernelGGL(dlam_sum_kernel, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, st, dlam_part, (int)P,
                           (int)ky, dlam);
}

}  // namespace fmap
