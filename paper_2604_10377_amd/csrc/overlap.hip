// Overlap-prediction metrics (Sec. 3.3) over a batch of shapes of uneven size.
//
// Shape s owns vertices [offsets[s], offsets[s+1]) of the concatenated score
// and ground-truth arrays.  A vertex is predicted overlapping when its score is
// strictly greater than the threshold.  Per shape the kernels count the
// confusion matrix (TP, FP, FN, TN) and derive accuracy, precision, recall
// (sensitivity), specificity, IoU, F1 and balanced accuracy, the mean of
// sensitivity and specificity.
//
// The count is one streaming pass (5 bytes per vertex, HBM-bound).
// overlap_shapes_kernel gives each shape to one wave or one workgroup, which
// counts it and writes its counts and metrics at once: nothing to clear, no
// atomics, no second kernel.  Shapes too long for that (one CU would stream
// them alone) get cleared slots there and are counted by overlap_large_kernel,
// whose workgroups take equal slices of all vertices and skip the ordinary
// shapes.
#include "../../include/fmap.h"

#include <algorithm>

#include "fmap_device.h"
#include "fmap_launch.h"

namespace fmap {

namespace {

constexpr int OV_WAVE_MAX = 8192;    // longest shape counted by one wave
constexpr int OV_GROUP_MAX = 65536;  // longest shape counted by one workgroup
constexpr int OV_GROUP = 512;        // threads of a workgroup that counts one shape (or a slice)
constexpr int OV_DEPTH = 4;          // 16-byte score loads in flight per thread

// Largest s in [0, S) with off[s] <= v (off nondecreasing; clamps for any contents), found by the whole
// wave: each round the 64 lanes test 64 evenly spaced candidates (one load each, all in flight together)
// and a ballot narrows the range 64-fold, so 1024 shapes take two rounds of loads.  v is wave-uniform.
__device__ __forceinline__ int wave_shape_of(const int64_t *__restrict__ off, int S, int64_t v, int lane)
{
    int lo = 0, hi = S - 1;  // answer in [lo, hi]
    while (lo < hi) {
        const int span = hi - lo;
        const int step = (span + 63) / 64;
        const int cand = min(lo + 1 + lane * step, hi);  // candidates above lo
        const bool le = off[cand] <= v;
        const unsigned long long m = __ballot(le);
        // candidates increase with the lane index and off is nondecreasing, so the lanes with le form a prefix
        const int cnt = __popcll(m);
        if (cnt == 0) {
            hi = lo;  // even the first candidate is above v: the answer is lo
        } else {
            const int last = min(lo + 1 + (cnt - 1) * step, hi);  // largest candidate with off <= v
            const int next = min(lo + 1 + cnt * step, hi + 1);    // smallest candidate above v (or past hi)
            lo = last;
            hi = next - 1;
        }
    }
    return lo;
}

__device__ __forceinline__ unsigned wave_sum_u32(unsigned v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// What a thread counts: vertices predicted, labelled, and both (the fourth cell follows from the length).
struct OvCount {
    unsigned pos, lab, both;
};

// Counts of vertices [lo, hi) over threads tid of nthr: thread tid takes every nthr-th group of four vertices
// from the group that holds lo (4-aligned, so both arrays are read with one load each; vertices outside the
// range are masked).  VEC: score is 16-byte and truth 4-byte aligned.  Every access lies in [0, total).
template <bool VEC>
__device__ __forceinline__ OvCount count_range(const float *__restrict__ score, const uint8_t *__restrict__ truth,
                                               int64_t lo, int64_t hi, int64_t total, float thr, int tid, int nthr)
{
    OvCount c{0u, 0u, 0u};
    // positions from the aligned base in 32 bits (a range has fewer than 2^31 vertices): one offset per load
    const int64_t base = lo & ~(int64_t)3;
    score += base;
    truth += base;
    const unsigned first = (unsigned)(lo - base), end = (unsigned)(max(hi, base) - base), step = 4u * (unsigned)nthr;
    const unsigned wide = VEC ? (unsigned)min(max(total - base, (int64_t)3) - 3, (int64_t)end) : 0u;
    for (unsigned v = 4u * (unsigned)tid; v < end; v += OV_DEPTH * step) {
        float sc[OV_DEPTH][4];
        uint32_t gt[OV_DEPTH];
#pragma unroll
        for (int u = 0; u < OV_DEPTH; ++u) {
            const unsigned v0 = v + u * step;
            if (v0 < wide) {  // all four vertices exist
                const f32x4 x = *reinterpret_cast<const f32x4 *>(score + v0);
                sc[u][0] = x[0];
                sc[u][1] = x[1];
                sc[u][2] = x[2];
                sc[u][3] = x[3];
                gt[u] = *reinterpret_cast<const uint32_t *>(truth + v0);
            } else {
                gt[u] = 0u;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool in = v0 + e < end;
                    sc[u][e] = in ? score[v0 + e] : 0.f;
                    gt[u] |= in ? (uint32_t)truth[v0 + e] << (8 * e) : 0u;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < OV_DEPTH; ++u) {
            const unsigned v0 = v + u * step;
            uint32_t in = 0x80808080u;  // bit 7 of byte e: vertex v0 + e is in the range
            if (v0 == 0u) in <<= 8 * first;
            if (v0 + 4 > end) in = v0 < end ? in & (0x80808080u >> (8 * (v0 + 4 - end))) : 0u;
            uint32_t p = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) p |= sc[u][e] > thr ? 0x80u << (8 * e) : 0u;
            p &= in;
            const uint32_t l = (((gt[u] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | gt[u]) & in;  // nonzero bytes
            c.pos += __popc(p);
            c.lab += __popc(l);
            c.both += __popc(p & l);
        }
    }
    return c;
}

// The seven metrics of one shape: accuracy, precision, recall, specificity, IoU, F1, balanced accuracy (float64
// arithmetic on the exact counts, rounded once to float32; a ratio with a zero denominator is 0; balanced
// accuracy averages the class recalls that are defined)
__device__ __forceinline__ void write_metrics(double tp, double fp, double fn, double tn, float *__restrict__ m)
{
    auto ratio = [](double a, double b) { return b != 0.0 ? a / b : 0.0; };
    const double sens = ratio(tp, tp + fn), spec = ratio(tn, tn + fp);
    const bool ds = tp + fn != 0.0, dsp = tn + fp != 0.0;
    const double bal = (ds && dsp) ? (sens + spec) / 2.0 : (ds ? sens : (dsp ? spec : 0.0));
    m[0] = (float)ratio(tp + tn, tp + fp + fn + tn);
    m[1] = (float)ratio(tp, tp + fp);
    m[2] = (float)sens;
    m[3] = (float)spec;
    m[4] = (float)ratio(tp, tp + fp + fn);
    m[5] = (float)ratio(2.0 * tp, 2.0 * tp + fp + fn);
    m[6] = (float)bal;
}

}  // namespace

// counts [S][4] = TP, FP, FN, TN and metrics [S][7].  WPS = 1: one wave per shape, four shapes per workgroup;
// WPS = OV_GROUP / 64: one workgroup per shape.  Longer shapes than LIMIT only get their slots cleared.
// Bound by the stream over scores and labels.  58 MB in 1024 shapes of 2000 to 20000 vertices: 16.5 us a call,
// 3.5 TB/s; equal runs of rows per wave with a clear before and a metrics kernel after took 37 us, most of it
// in the vertex-by-vertex atomics of the rows that cross a shape boundary.  At 64 registers four workgroups
// share a CU, so 1024 shapes are in flight at once.
template <bool VEC, int WPS>
__global__ __launch_bounds__(WPS == 1 ? 256 : OV_GROUP, VEC ? 8 : 1) void overlap_shapes_kernel(
    const float *__restrict__ score, const uint8_t *__restrict__ truth, const int64_t *__restrict__ off, int S,
    int64_t total, float thr, int64_t *__restrict__ counts, float *__restrict__ metrics)
{
    constexpr int LIMIT = WPS == 1 ? OV_WAVE_MAX : OV_GROUP_MAX;
    constexpr int PER = WPS == 1 ? 4 : 1;  // shapes per workgroup
    __shared__ unsigned part[3][8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int64_t s = (int64_t)blockIdx.x * PER + (WPS == 1 ? wave : 0); s < S; s += (int64_t)gridDim.x * PER) {
        const int64_t lo = min(max(off[s], (int64_t)0), total), hi = min(max(off[s + 1], lo), total);
        const bool large = hi - lo > LIMIT;
        OvCount c{0u, 0u, 0u};
        if (!large)
            c = count_range<VEC>(score, truth, lo, hi, total, thr, WPS == 1 ? lane : (int)threadIdx.x, 64 * WPS);
        c.pos = wave_sum_u32(c.pos);
        c.lab = wave_sum_u32(c.lab);
        c.both = wave_sum_u32(c.both);
        if (WPS > 1) {
            if (lane == 0) {
                part[0][wave] = c.pos;
                part[1][wave] = c.lab;
                part[2][wave] = c.both;
            }
            __syncthreads();
            c = OvCount{0u, 0u, 0u};
#pragma unroll
            for (int w = 0; w < WPS; ++w) {
                c.pos += part[0][w];
                c.lab += part[1][w];
                c.both += part[2][w];
            }
        }
        if (WPS == 1 ? lane == 0 : threadIdx.x == 0) {
            const unsigned n = large ? 0u : (unsigned)(hi - lo);
            const unsigned tp = c.both, fp = c.pos - c.both, fn = c.lab - c.both, tn = n - c.pos - c.lab + c.both;
            int64_t *cs = counts + 4 * s;
            cs[0] = tp;
            cs[1] = fp;
            cs[2] = fn;
            cs[3] = tn;
            write_metrics(tp, fp, fn, tn, metrics + 7 * s);
        }
        if (WPS > 1) __syncthreads();  // part is written again for the next shape
    }
}

// Shapes of more than limit vertices: workgroup w takes vertices [w slice, (w + 1) slice), finds the shapes
// that reach into them (the first by a 64-way parallel search over the offsets, the others walking forward 64
// at a time), adds its counts of the long ones to their cleared slots, and the last workgroup of a shape to do
// so writes its metrics.  The first word of the shape's metrics, cleared to +0 by the kernel above, counts the
// workgroups that are done.  Integer sums: any order gives the same counts.
template <bool VEC>
__global__ __launch_bounds__(OV_GROUP) void overlap_large_kernel(const float *__restrict__ score,
                                                                 const uint8_t *__restrict__ truth,
                                                                 const int64_t *__restrict__ off, int S,
                                                                 int64_t total, float thr, int64_t limit,
                                                                 int64_t slice, unsigned long long *counts,
                                                                 float *metrics)
{
    const int lane = threadIdx.x & 63;
    __shared__ unsigned sum[3];
    const int64_t b0 = (int64_t)blockIdx.x * slice, b1 = min(b0 + slice, total);
    // every wave walks alike, so the barriers below are reached by all of them
    for (int64_t s0 = wave_shape_of(off, S, b0, lane); s0 < S; s0 += 64) {
        const int64_t s = s0 + lane;
        int64_t lo = total, hi = total;
        if (s < S) {
            lo = min(max(off[s], (int64_t)0), total);
            hi = min(max(off[s + 1], lo), total);
        }
        unsigned long long m = __ballot(hi - lo > limit && lo < b1 && hi > b0);
        while (m) {
            const int src = __ffsll((long long)m) - 1;
            m &= m - 1;
            const int64_t sl = __shfl(lo, src, 64), sh = __shfl(hi, src, 64), ss = s0 + src;
            const OvCount c = count_range<VEC>(score, truth, max(sl, b0), min(sh, b1), total, thr, threadIdx.x, OV_GROUP);
            const unsigned pos = wave_sum_u32(c.pos), lab = wave_sum_u32(c.lab), both = wave_sum_u32(c.both);
            if (threadIdx.x < 3) sum[threadIdx.x] = 0u;
            __syncthreads();
            if (lane == 0) {
                atomicAdd(&sum[0], pos);
                atomicAdd(&sum[1], lab);
                atomicAdd(&sum[2], both);
            }
            __syncthreads();
            if (threadIdx.x == 0) {
                const unsigned tp = sum[2], fp = sum[0] - tp, fn = sum[1] - tp;
                const unsigned n = (unsigned)(min(sh, b1) - max(sl, b0));
                unsigned long long *cs = counts + 4 * ss;
                atomicAdd(&cs[0], (unsigned long long)tp);
                atomicAdd(&cs[1], (unsigned long long)fp);
                atomicAdd(&cs[2], (unsigned long long)fn);
                atomicAdd(&cs[3], (unsigned long long)(n - tp - fp - fn));
                __threadfence();
                const unsigned groups = (unsigned)((sh - 1) / slice - sl / slice + 1);
                if (atomicAdd((unsigned *)(metrics + 7 * ss), 1u) + 1u == groups) {
                    __threadfence();
                    unsigned long long v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        v[q] = __hip_atomic_load(&cs[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    write_metrics((double)v[0], (double)v[1], (double)v[2], (double)v[3], metrics + 7 * ss);
                }
            }
            __syncthreads();
        }
        if (__shfl(lo, 63, 64) >= b1) break;
    }
}

namespace {

template <bool VEC>
void launch_overlap_as(const float *score, const uint8_t *truth, const int64_t *offsets, int64_t S, int64_t total,
                       float thr, int64_t *counts, float *metrics, hipStream_t st)
{
    // One wave per shape up to 4096 vertices on average, one workgroup above.  A workgroup per short shape
    // spends its time starting and reducing (8000 shapes of 2075 vertices: 33.9 us against 19.2 by wave); one
    // wave takes long over a long shape (4000 shapes of 4600: 21.7 us by workgroup, of 4000 by wave 19.3; few
    // shapes of any such length take 12 us either way, the launches).  The grid is capped (the kernel strides).
    const bool by_wave = total <= 4096 * S;
    const int64_t limit = by_wave ? OV_WAVE_MAX : OV_GROUP_MAX;
    if (by_wave)
        hipLaunchKernelGGL((overlap_shapes_kernel<VEC, 1>), dim3((unsigned)std::min<int64_t>((S + 3) / 4, 1 << 20)),
                           dim3(256), 0, st, score, truth, offsets, (int)S, total, thr, counts, metrics);
    else
        hipLaunchKernelGGL((overlap_shapes_kernel<VEC, OV_GROUP / 64>), dim3((unsigned)std::min<int64_t>(S, 1 << 20)),
                           dim3(OV_GROUP), 0, st, score, truth, offsets, (int)S, total, thr, counts, metrics);
    if (total > limit) {  // some shape may be longer than the limit: slices for two workgroups per CU
        // (four, of 8192 vertices at least, took 39 us instead of 17 for one shape of 5M: atomics on one slot)
        const int64_t groups = 2 * (int64_t)device_cus();
        const int64_t slice = std::min<int64_t>(
            std::max<int64_t>(32768, ((total + groups - 1) / groups + 255) / 256 * 256), (int64_t)1 << 30);
        hipLaunchKernelGGL(overlap_large_kernel<VEC>, dim3((unsigned)((total + slice - 1) / slice)), dim3(OV_GROUP), 0,
                           st, score, truth, offsets, (int)S, total, thr, limit, slice,
                           (unsigned long long *)counts, metrics);
    }
}

}  // namespace

hipError_t launch_overlap(const float *score, const uint8_t *truth, const int64_t *offsets, int64_t S, int64_t total,
                          float thr, int64_t *counts, float *metrics, hipStream_t st)
{
    if ((((uintptr_t)score) & 15) == 0 && (((uintptr_t)truth) & 3) == 0)
        launch_overlap_as<true>(score, truth, offsets, S, total, thr, counts, metrics, st);
    else
        launch_overlap_as<false>(score, truth, offsets, S, total, thr, counts, metrics, st);
    return hipGetLastError();
}

}  // namespace fmap

extern "C" fmap_status fmap_overlap_metrics(const float *scores, const uint8_t *truth, const int64_t *offsets,
                                            int64_t shapes, int64_t total, float threshold, int64_t *counts,
                                            float *metrics, void *stream)
{
    if (!offsets || !counts || !metrics) return FMAP_ERR_NULL;
    if (total > 0 && (!scores || !truth)) return FMAP_ERR_NULL;
    if (shapes < 1 || shapes >= ((int64_t)1 << 30) || total < 0 || total >= ((int64_t)1 << 40)) return FMAP_ERR_SHAPE;
    if (threshold != threshold) return FMAP_ERR_VALUE;  // NaN threshold
    return fmap::launch_overlap(scores, truth, offsets, shapes, total, threshold, counts, metrics,
                                (hipStream_t)stream) == hipSuccess
               ? FMAP_OK
               : FMAP_ERR_HIP;
}
