// DiffusionNet spatial-gradient features (Sec. 3.2), both documented variants.
//
// Per vertex v the D channels carry complex gradients z = x + i y, stored
// interleaved: z[v][2j] = x_j, z[v][2j + 1] = y_j.  With the learned complex
// matrix A = A_re + i A_im ((A z)_c = sum_j A_cj z_j):
//     (A z)_re = A_re x - A_im y
//     (A z)_im = A_re y + A_im x    (variant A)   or   A_re x + A_im y   (variant B)
//     g        = x * (A z)_re + y * (A z)_im
// Read with k over the interleaved z row (length 2D), both transformed parts are
// one product Z [V x 2D] times W^T, where row c of W_re is
// (A_re[c][0], -A_im[c][0], A_re[c][1], -A_im[c][1], ...) and row c of W_im is
// (A_im[c][j], A_re[c][j]) pairs (variant A) or (A_re[c][j], A_im[c][j]) pairs
// (variant B).  That is a dense contraction of 8 D^2 flops per vertex against
// 12 D bytes of traffic (85 flop/B at D = 128), with the elementwise combination
// fused into the epilogue.  On the float32 matrix cores it was bound by them
// (160000 vertices, D = 128: 224 us, 94 TFLOP/s); it runs on the float16 ones with
// both operands split in two (fmap_split.h), three products per float32 one.
//
// The weights stay in registers: a wave holds the parts of W for 16 channels (D = 256: 8), both rows of each, as
// matrix-core operands with one scale per channel, at most 128 registers, and the 8 waves of a workgroup cover all D
// channels (D = 256: 64), so z is read and split once (four times).  A tile of z rows goes through LDS: its loading
// waves take whole rows, 8 consecutive values per lane, scale each row by its largest value, and write the parts as
// operand slots, permuted so that the lanes of a row hit different bank groups.  Two tiles are in LDS (one barrier
// per tile) and a third one's loads are in flight.  The result tile has channels along registers: a lane ends up
// with 4 consecutive channels of one vertex and stores 16 bytes.  With W in LDS instead and the split z rows in
// registers, every wave loaded, split and multiplied in turn, all at the same time: 87 us at 160000 vertices, D = 128.
// Measured (160000 vertices; before: float32 matrix cores): D = 32 32.4 -> 17.1 us, D = 64 64 -> 29 us, D = 128
// 208 -> 69 us (3.6 TB/s of its bytes), 200000 vertices of D = 256 1160 -> 365 us; 5000 of D = 128 42 -> 11.5 us.  The
// error against float64 falls: 2.9e-7 -> 1.9e-7 at D = 128, 4.1e-7 -> 2.5e-7 at D = 256.  Up to D = 128 it is bound by
// memory and its latency (one tile in flight per workgroup); at D = 256 by LDS: a wave's 128 weight registers hold
// one row tile, so every operand read from LDS feeds three products.
#include "../../include/fmap.h"

#include <algorithm>

#include "fmap_launch.h"
#include "fmap_lds.h"
#include "fmap_split.h"

namespace fmap {

namespace {

constexpr int GF_WAVES = 8;
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // g need not be 16-byte aligned

__device__ __forceinline__ f32x4 ld4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }

template <int D>
struct Gf {
    static constexpr int K = 2 * D, KS = K / 32;      // row length, K steps
    static constexpr int CH = D <= 128 ? 16 : 8;      // channels per wave
    static constexpr int NR = D <= 128 ? 2 : 1;       // its W row tiles: re and im, or 8 re + 8 im rows in one
    static constexpr int CW = D <= 128 ? D / CH : 8;  // waves along the channels
    static constexpr int NB = D / (CW * CH);          // channel blocks (workgroups per vertex range)
    static constexpr int VT = 2, VW = GF_WAVES / CW;  // vertex tiles of 16 per wave, waves along the vertices
    static constexpr int VERTS = 16 * VT * VW;        // vertices per tile of the workgroup
    static constexpr int RPW = VERTS / GF_WAVES;      // rows a wave loads
    static constexpr int LR = 64 / RPW;               // lanes per row
    static constexpr int PASS = K / (8 * LR);         // 8-value pieces per lane
    static constexpr int BUF = VERTS * K / 4;         // 16-byte slots per tile (two float16 parts per value)
    static constexpr size_t LDS = (size_t)2 * BUF * 16 + 2 * VERTS * sizeof(int);
    static constexpr int PER_CU = D <= 32 ? 2 : 1;    // resident workgroups (registers, LDS)
};

}  // namespace

// z [V][2D], A_re, A_im [D][D], g [V][D].  grid = vgroups * NB, XCD-ordered.
template <int D>
__global__ __launch_bounds__(64 * GF_WAVES, D <= 32 ? 4 : 2) void gradfeat_mfma_kernel(
    const float *__restrict__ z, const float *__restrict__ Are, const float *__restrict__ Aim, int variant, int V,
    int vgroups, float *__restrict__ g)
{
    using C = Gf<D>;
    constexpr int K = C::K, KS = C::KS;
    extern __shared__ __align__(16) float smem[];
    u32x4_t *buf = reinterpret_cast<u32x4_t *>(smem);       // two tiles [vertex tile][K step][part][64 slots]
    int *s_zs = reinterpret_cast<int *>(buf + 2 * C::BUF);  // [2][VERTS] row shifts
    // XCD-aware decode: ids b, b + 8, b + 16, ... share an XCD; the NB channel blocks of one vertex group are
    // consecutive in that sequence
    const int id = blockIdx.x;
    const int per_xcd = (int)((gridDim.x + 7) / 8);
    const int seq = (id % 8) * per_xcd + id / 8;  // position in the XCD-major order
    if (seq >= vgroups * C::NB) return;
    const int vg = seq / C::NB;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m16 = lane & 15, g4 = lane >> 4;
    const int vw = wave / C::CW;
    const int c0 = (seq % C::NB) * C::CW * C::CH + (wave % C::CW) * C::CH;

    const int tiles = (V + C::VERTS - 1) / C::VERTS;
    const int t0 = (int)((long)vg * tiles / vgroups), t1 = (int)((long)(vg + 1) * tiles / vgroups);
    if (t0 >= t1) return;

    // loading role: 8-value pieces lr, lr + LR, ... of row `row` of the tile
    const int row = wave * C::RPW + lane / C::LR, lr = lane % C::LR;
    f32x4 x[C::PASS][2];
    auto issue = [&](int t) {
        const float *zr = z + (size_t)min(t * C::VERTS + row, V - 1) * K + 8 * lr;
#pragma unroll
        for (int q = 0; q < C::PASS; ++q) {
            x[q][0] = ld4(zr + 8 * C::LR * q);
            x[q][1] = ld4(zr + 8 * C::LR * q + 4);
        }
    };
    // slot of operand lane (m, g) at K step s: the vertex index permuted by the piece number
    auto slot = [](int m, int g, int s) { return (m ^ (4 * (s & 3) + g)) + 16 * g; };
    auto split = [&](int b) {
        float mx = 0.f;
#pragma unroll
        for (int q = 0; q < C::PASS; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = fmaxf(mx, fmaxf(fabsf(x[q][0][e]), fabsf(x[q][1][e])));
#pragma unroll
        for (int o = 1; o < C::LR; o *= 2) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        const int sh = split_shift(__float_as_uint(mx));
        const float sc = split_scale(sh);
        if (lr == 0) s_zs[b * C::VERTS + row] = sh;
        u32x4_t *B = buf + b * C::BUF + (row >> 4) * KS * 128;
#pragma unroll
        for (int q = 0; q < C::PASS; ++q) {
            u32x4_t h, l;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                uint32_t hh, ll;
                split_pair(x[q][jj >> 1][2 * (jj & 1)], x[q][jj >> 1][2 * (jj & 1) + 1], sc, hh, ll);
                h[jj] = hh;
                l[jj] = ll;
            }
            const int piece = q * C::LR + lr, s = piece >> 2;
            u32x4_t *o = B + s * 128 + slot(row & 15, piece & 3, s);
            o[0] = h;
            o[64] = l;
        }
    };

    issue(t0);
    // this wave's weights: lane (m16, g4) holds W row m16, values 32 s + 8 g4 .. + 7 of K step s
    u32x4_t wh[C::NR][KS], wl[C::NR][KS];
    int wshift[4];  // shifts of the rows 4 g4 + r (a channel's two rows hold the same magnitudes)
    {
        const int c = c0 + (C::NR == 2 ? m16 : (m16 & 7));
        f32x4 ar[KS], ai[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            ar[s] = *reinterpret_cast<const f32x4u *>(Are + (size_t)c * D + 16 * s + 4 * g4);
            ai[s] = *reinterpret_cast<const f32x4u *>(Aim + (size_t)c * D + 16 * s + 4 * g4);
        }
        float mx = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) mx = fmaxf(mx, fmaxf(fabsf(ar[s][e]), fabsf(ai[s][e])));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const int sh = split_shift(__float_as_uint(mx));
        const float sc = split_scale(sh);
#pragma unroll
        for (int r = 0; r < 4; ++r) wshift[r] = __shfl(sh, 4 * g4 + r, 64);
#pragma unroll
        for (int n = 0; n < C::NR; ++n) {
            const bool im = C::NR == 2 ? n == 1 : m16 >= 8;
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float a = ar[s][e], b = ai[s][e];
                    uint32_t h, l;
                    split_pair(im && variant == 0 ? b : a, im ? (variant == 0 ? a : b) : -b, sc, h, l);
                    wh[n][s][e] = h;
                    wl[n][s][e] = l;
                }
        }
    }
    split(0);
    issue(min(t0 + 1, t1 - 1));
    lds_barrier();

    for (int t = t0; t < t1; ++t) {
        const int b = (t - t0) & 1;
        const int v0 = t * C::VERTS + vw * 16 * C::VT;  // this wave's vertices
        // the lane's output: 4 channels of one vertex per tile (D = 256: the lanes of the upper half take the second
        // vertex tile, those of the lower half the first); its x and y in flight while the products run
        const int co = c0 + 4 * (C::NR == 2 ? g4 : (g4 & 1));
        constexpr int NO = C::NR == 2 ? C::VT : 1;
        f32x4 xy[NO][2];
        int vo[NO];
#pragma unroll
        for (int n = 0; n < NO; ++n) {
            vo[n] = v0 + 16 * (C::NR == 2 ? n : g4 >> 1) + m16;
            const float *zr = z + (size_t)min(vo[n], V - 1) * K + 2 * co;
            xy[n][0] = ld4(zr);
            xy[n][1] = ld4(zr + 4);
        }
        const u32x4_t *B = buf + b * C::BUF + vw * C::VT * KS * 128;
        f32x4 acc[C::NR][C::VT];
#pragma unroll
        for (int n = 0; n < C::NR; ++n)
#pragma unroll
            for (int v = 0; v < C::VT; ++v) acc[n][v] = f32x4{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            u32x4_t zh[C::VT], zl[C::VT];
#pragma unroll
            for (int v = 0; v < C::VT; ++v) {
                zh[v] = B[v * KS * 128 + s * 128 + slot(m16, g4, s)];
                zl[v] = B[v * KS * 128 + s * 128 + 64 + slot(m16, g4, s)];
            }
#pragma unroll
            for (int n = 0; n < C::NR; ++n)
#pragma unroll
                for (int v = 0; v < C::VT; ++v) acc[n][v] = mfma16x16x32f16(wl[n][s], zh[v], acc[n][v]);
#pragma unroll
            for (int n = 0; n < C::NR; ++n)
#pragma unroll
                for (int v = 0; v < C::VT; ++v) acc[n][v] = mfma16x16x32f16(wh[n][s], zl[v], acc[n][v]);
#pragma unroll
            for (int n = 0; n < C::NR; ++n)
#pragma unroll
                for (int v = 0; v < C::VT; ++v) acc[n][v] = mfma16x16x32f16(wh[n][s], zh[v], acc[n][v]);
        }
        split(b ^ 1);  // tile t + 1 (past the last one: the last one again, never read)
        issue(min(t + 2, t1 - 1));
        // g[v][c] = x_c (A z)_re + y_c (A z)_im; register r of lane (m16, g4): W row 4 g4 + r, vertex m16
#pragma unroll
        for (int n = 0; n < NO; ++n) {
            const f32x4 p = xy[n][0], q = xy[n][1];
            const float xs[4] = {p[0], p[2], q[0], q[2]}, ys[4] = {p[1], p[3], q[1], q[3]};
            const int zs = s_zs[b * C::VERTS + vo[n] - t * C::VERTS];
            f32x4 o;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float re, im;
                if constexpr (C::NR == 2) {
                    re = acc[0][n][r];
                    im = acc[1][n][r];
                } else {
                    const bool up = g4 >= 2;  // holds im rows: keeps those of the second tile, gives the first's away
                    const float got = __shfl_xor(up ? acc[0][0][r] : acc[0][1][r], 32, 64);
                    re = up ? got : acc[0][0][r];
                    im = up ? acc[0][1][r] : got;
                }
                const int sh = -(wshift[r] + zs);
                o[r] = xs[r] * __builtin_amdgcn_ldexpf(re, sh) + ys[r] * __builtin_amdgcn_ldexpf(im, sh);
            }
            if (vo[n] < V) *reinterpret_cast<f32x4u *>(g + (size_t)vo[n] * D + co) = o;
        }
        lds_barrier();
    }
}

// Any D: one thread per output (v, c), plain float32 dot products (the reference path for shapes the
// matrix-core kernel does not take).
__global__ __launch_bounds__(256) void gradfeat_general_kernel(const float *__restrict__ z, const float *__restrict__ Are,
                                                               const float *__restrict__ Aim, int variant, int V, int D,
                                                               float *__restrict__ g)
{
    const int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (o >= (int64_t)V * D) return;
    const int v = (int)(o / D), c = (int)(o % D);
    const float *zv = z + (size_t)v * 2 * D;
    float re = 0.f, im = 0.f;
    for (int j = 0; j < D; ++j) {
        const float x = zv[2 * j], y = zv[2 * j + 1];
        const float ar = Are[(size_t)c * D + j], ai = Aim[(size_t)c * D + j];
        re += ar * x - ai * y;
        im += variant == 0 ? (ar * y + ai * x) : (ar * x + ai * y);
    }
    g[o] = zv[2 * c] * re + zv[2 * c + 1] * im;
}

template <int D>
static void launch_gf(const float *z, const float *Are, const float *Aim, int variant, int64_t V, float *g,
                      hipStream_t st)
{
    using C = Gf<D>;
    static bool attr = false;
    if (!attr) {
        (void)hipFuncSetAttribute((const void *)gradfeat_mfma_kernel<D>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)C::LDS);
        attr = true;
    }
    const int64_t tiles = (V + C::VERTS - 1) / C::VERTS;
    // one round of resident workgroups over all channel blocks, at least one tile each
    const int64_t want = std::max<int64_t>(1, (int64_t)C::PER_CU * device_cus() / C::NB);
    const int64_t vgroups = std::min<int64_t>(want, tiles);
    const int64_t n = vgroups * C::NB;
    const int64_t grid = ((n + 7) / 8) * 8;  // whole rounds of the 8 XCDs; surplus ids exit
    hipLaunchKernelGGL((gradfeat_mfma_kernel<D>), dim3((unsigned)grid), dim3(64 * GF_WAVES), C::LDS, st, z, Are, Aim,
                       variant, (int)V, (int)vgroups, g);
}

hipError_t launch_gradient_features(const float *z, const float *Are, const float *Aim, int variant, int64_t V,
                                    int64_t D, float *g, hipStream_t st)
{
    const bool al = (((uintptr_t)z) & 15) == 0;
    if (al && D == 32) launch_gf<32>(z, Are, Aim, variant, V, g, st);
    else if (al && D == 64) launch_gf<64>(z, Are, Aim, variant, V, g, st);
    else if (al && D == 128) launch_gf<128>(z, Are, Aim, variant, V, g, st);
    else if (al && D == 256) launch_gf<256>(z, Are, Aim, variant, V, g, st);
    else {
        const int64_t n = V * D;
        hipLaunchKernelGGL(gradfeat_general_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, z, Are, Aim,
                           variant, (int)V, (int)D, g);
    }
    return hipGetLastError();
}

}  // namespace fmap

extern "C" fmap_status fmap_gradient_features(const float *z, const float *A_re, const float *A_im, int32_t variant,
                                              int64_t vertices, int64_t channels, float *g, void *stream)
{
    if (!z || !A_re || !A_im || !g) return FMAP_ERR_NULL;
    if (variant != FMAP_GRADFEAT_A && variant != FMAP_GRADFEAT_B) return FMAP_ERR_VALUE;
    if (vertices < 1 || channels < 1 || vertices >= ((int64_t)1 << 31) || channels > 4096 ||
        vertices * channels >= ((int64_t)1 << 31))
        return FMAP_ERR_SHAPE;
    return fmap::launch_gradient_features(z, A_re, A_im, variant, vertices, channels, g, (hipStream_t)stream) ==
                   hipSuccess
               ? FMAP_OK
               : FMAP_ERR_HIP;
}
