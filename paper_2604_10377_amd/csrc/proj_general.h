// The general forward projection of one block on the float32 matrix cores (v_mfma_f32_32x32x2f32): any n, k, d and
// alignment, float32 or bf16 inputs.  The general kernels run it for every block; the split kernels for a chunk whose
// values do not fit their scales.
#pragma once

#include "fmap_device.h"

namespace fmap {

template <typename T>
__device__ __forceinline__ float load_elem(const T *p, size_t i);
template <>
__device__ __forceinline__ float load_elem<float>(const float *p, size_t i) { return p[i]; }
template <>
__device__ __forceinline__ float load_elem<uint16_t>(const uint16_t *p, size_t i) { return bf16_to_f32(p[i]); }

// One (shape, vertex range, k-block, column block) of the forward projection:
// this wave's partial A rows [kbase, kbase + MT*32) x columns [dbase, dbase + NT*32)
// over vertices [v0, v1), written to O (row-major k x d).  No barriers.
template <typename T, int MT, int NT, int U>
__device__ __forceinline__ void proj_fwd_tile(const T *__restrict__ P, const float *__restrict__ Mv,
                                              const T *__restrict__ F, int k, int d, int v0, int v1, int kbase,
                                              int dbase, float *__restrict__ O)
{
    const int lane = threadIdx.x & 63;
    const int half = lane >> 5, l32 = lane & 31;
    if (dbase >= d) return;  // whole wave idle (narrow d)

    int rows[MT], cols[NT];
    bool rok[MT], cok[NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        rows[mt] = kbase + mt * 32 + l32;
        rok[mt] = rows[mt] < k;
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        cols[nt] = dbase + nt * 32 + l32;
        cok[nt] = cols[nt] < d;
    }

    f32x16 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = zero16();

    // Two register stages of U matrix-core steps (2U vertices): the loads of one
    // stage are in flight while the other stage's multiplies run.
    float pa0[U][MT], pb0[U][NT], m0[U], pa1[U][MT], pb1[U][NT], m1[U];
    auto load = [&](float (&pa)[U][MT], float (&pb)[U][NT], float (&mv)[U], int v) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned vv = (unsigned)(v + 2 * u + half);
            mv[u] = Mv[vv];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) pa[u][mt] = rok[mt] ? load_elem(P, vv * (unsigned)k + rows[mt]) : 0.f;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) pb[u][nt] = cok[nt] ? load_elem(F, vv * (unsigned)d + cols[nt]) : 0.f;
        }
    };
    auto mma = [&](float (&pa)[U][MT], float (&pb)[U][NT], float (&mv)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const float a = pa[u][mt] * mv[u];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = mfma32x32x2(a, pb[u][nt], acc[mt][nt]);
            }
    };
    const int S = 2 * U;
    const int nst = (v1 - v0) / S;
    int v = v0;
    if (nst > 0) load(pa0, pb0, m0, v);
    for (int st = 0; st < nst; st += 2) {
        if (st + 1 < nst) load(pa1, pb1, m1, v + S);
        mma(pa0, pb0, m0);
        if (st + 2 < nst) load(pa0, pb0, m0, v + 2 * S);
        if (st + 1 < nst) mma(pa1, pb1, m1);
        v += 2 * S;
    }
    // Tail: guarded single steps.
    for (v = v0 + nst * S; v < v1; v += 2) {
        const int vv = v + half;
        const bool ok = vv < v1;
        const float m = ok ? Mv[vv] : 0.f;
        float a[MT], b[NT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) a[mt] = (ok && rok[mt]) ? load_elem(P, (size_t)vv * k + rows[mt]) * m : 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) b[nt] = (ok && cok[nt]) ? load_elem(F, (size_t)vv * d + cols[nt]) : 0.f;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = mfma32x32x2(a[mt], b[nt], acc[mt][nt]);
    }

#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = kbase + mt * 32 + acc32_row(r, lane);
                if (row < k && cok[nt]) O[(size_t)row * d + cols[nt]] = acc[mt][nt][r];
            }
}

}  // namespace fmap
