// Host-side launch entry points shared between the kernel files and the C ABI.
#pragma once

#include <algorithm>

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace fmap {

// Largest k_x handled by the register-resident row-solve kernels.
constexpr int kSmallK = 64;
// Largest k_x of the tiled row solve (k_x + 1 rows in at most 10 tile rows of 32).
constexpr int kMaxK = 319;

// Work items of the persistent projections over uneven shapes.
struct FwdItem {                  // partial A rows [kbase, kbase+64) x d-block over vertices [v0, v1)
    const float *phi, *mass, *feat;
    float *out;                   // k x d partial slot
    int n, k, d, v0, v1, kbase, dbase;
};
struct BwdItem {                  // dF rows [r0, r0 + 128*rb) x columns [dbase, dbase + 256)
    const float *phi, *mass, *dA;
    float *dF;
    int n, k, d, r0, rb, dbase;
};
struct McItem {                   // dF tiles [t0, t1) of back_verts vertices x columns [dbase, dbase + back_cols)
    const float *phi, *mass, *dA;
    float *dF;
    int n, k, d, t0, t1, dbase;
};
struct RedItem {                  // A = sum of `nchunks` partial k x d slots
    const float *part;
    float *A, *A_user;
    int nchunks, kd;
};

hipError_t launch_fwd_items(const FwdItem *items, int nitems, int kmax, int grid, hipStream_t st);
hipError_t launch_bwd_items(const BwdItem *items, int nitems, int kmax, int grid, hipStream_t st);
hipError_t launch_reduce_items(const RedItem *items, int nitems, hipStream_t st);
// float32 backward projection for 4 <= k <= kMaxK on the float16 matrix cores, operands split into two parts (any n and
// d, any alignment), and its work-item form for one k: back_cols columns per item, tiles of back_verts vertices,
// back_slots resident workgroups.
bool back_shape_ok(int64_t k, int64_t d);
int back_cols(int64_t k, int64_t d);
int back_verts(int64_t k, int64_t d);
int back_slots(int64_t k);
hipError_t launch_project_back(const float *phi, const float *mass, const float *dA, int64_t batch, int64_t n, int64_t k,
                               int64_t d, float *dF, hipStream_t st);
hipError_t launch_bwd_split_items(const McItem *items, int nitems, int64_t k, int64_t d, hipStream_t st);
// Fixed-order sum of split-K partials [batch][nsplit][k][d] into A [batch][k][d]; `parts`: in four parts where few
// elements have many chunks.
hipError_t launch_reduce(const float *part, int nsplit, int64_t batch, int64_t k, int64_t d, float *A, bool parts,
                         hipStream_t st);
// bf16 forward projection on the bf16 matrix cores (k % 8 == 0, k <= 256, d % 8 == 0, any n).
bool bf16_fwd_shape_ok(int64_t n, int64_t k, int64_t d);
int bf16_fwd_nsplit(int64_t batch, int64_t n, int64_t k, int64_t d);
// bf16-basis backward projection on the bf16 matrix cores (k % 8 == 0, k <= 256).
bool bf16_bwd_shape_ok(int64_t n, int64_t k, int64_t d);
hipError_t launch_project_backward_bf16(const uint16_t *phi, const float *mass, const float *dA, int64_t batch,
                                        int64_t n, int64_t k, int64_t d, float *dF, hipStream_t st);
// float32 forward projection for 64 < k <= kMaxK, operands split into three bf16 parts (k % 4 == 0, d % 4 == 0,
// n % 4 == 0; items of whole 32-vertex stages): small calls, and shapes with d < 5 k / 4 of any size.
bool near_square(int64_t k, int64_t d);
bool sliced_fwd_shape_ok(int64_t n, int64_t k, int64_t d);
hipError_t launch_project_sliced(const float *phi, const float *mass, const float *feat, int64_t batch, int64_t n,
                                 int64_t k, int64_t d, float *A, void *ws, hipStream_t st);
bool sliced_item_shape_ok(int64_t k, int64_t d);
hipError_t launch_fwd_sliced_items(const FwdItem *items, int nitems, hipStream_t st);
// float32 forward projection for 64 < k <= kMaxK and d >= 5 k / 4 on the float16 matrix cores, operands split into two parts
// (d % 4 == 0, 16-byte aligned features, any n and k).
bool tall_shape_ok(int64_t n, int64_t k, int64_t d);
bool tall_too_small(int64_t batch, int64_t n, int64_t k, int64_t d);
// Chunks of the vertex sum, at most `cap`.
int tall_nsplit(int64_t batch, int64_t n, int64_t k, int64_t d, int64_t cap);
hipError_t launch_project_tall(const float *phi, const float *mass, const float *feat, int64_t batch, int64_t n,
                               int64_t k, int64_t d, int ns, float *A, void *ws, hipStream_t st);
// The same for k <= 64.
bool short_shape_ok(int64_t n, int64_t k, int64_t d);
int short_nsplit(int64_t batch, int64_t n, int64_t k, int64_t d);
hipError_t launch_project_short(const float *phi, const float *mass, const float *feat, int64_t batch, int64_t n,
                                int64_t k, int64_t d, int ns, float *A, void *ws, hipStream_t st);
hipError_t launch_fwd_short_items(const FwdItem *items, int nitems, hipStream_t st);
// The tall kernel's work-item form: instances by class of (k, d), tall_cols(k, d) columns per item.
constexpr int kTallClasses = 5;
int tall_class(int64_t k, int64_t d);
int tall_cols(int64_t k, int64_t d);
hipError_t launch_fwd_tall_items(const FwdItem *items, int nitems, int cls, hipStream_t st);
hipError_t launch_project_bf16(const uint16_t *phi, const float *mass, const uint16_t *feat, int64_t batch, int64_t n,
                               int64_t k, int64_t d, int ns, float *A, void *ws, hipStream_t st);
int device_cus();
// Rounds of resident workgroups that `tasks` times `dblocks` column blocks take, when the column blocks of a task run on
// one of the 8 XCDs and the tasks are dealt to them in turn; `slots` workgroups are resident on the whole chip.  The
// XCD with the most tasks decides: 84 tasks of 3 blocks are 252 workgroups, but 33 on four of the XCDs with 32 slots.
inline int64_t xcd_rounds(int64_t tasks, int64_t dblocks, int64_t slots)
{
    const int64_t each = std::max<int64_t>(slots / 8, 1);
    return ((tasks + 7) / 8 * dblocks + each - 1) / each;
}

struct ProjPlan {
    int MT, NT, kblocks, dblocks, nsplit, chunk;
};

ProjPlan plan_project(int64_t batch, int64_t n, int64_t k, int64_t d, int32_t dtype);
size_t project_workspace_bytes(int64_t batch, int64_t n, int64_t k, int64_t d, int32_t dtype);
hipError_t launch_project(const void *phi, const float *mass, const void *feat, int32_t dtype, int64_t batch, int64_t n,
                          int64_t k, int64_t d, float *A, void *ws, hipStream_t st);
hipError_t launch_project_backward(const void *phi, const float *mass, int32_t dtype, const float *dA, int64_t batch,
                                   int64_t n, int64_t k, int64_t d, float *dF, hipStream_t st);

// rs_waves: row systems per workgroup of the register row solve (k_x <= kSmallK): 1, 2 or 4.
// Workspace carve-up of the solver (byte offsets, 256-aligned).
struct SolveWs {
    size_t K, R, V, W, tiles, K64, R64, dlam, flag, total;
};
SolveWs solve_workspace_layout(int64_t pairs, int64_t kx, int64_t ky, int64_t d);

hipError_t launch_solve(const float *A, const float *B, const float *ex, const float *ey, const float *lam,
                        int32_t mask_kind, float gamma, int64_t P, int64_t kx, int64_t ky, int64_t d,
                        int32_t refine_steps, float cond_threshold, float *C, float *factors, int32_t *info,
                        float *cond_est, void *ws, hipStream_t st, int rs_waves = 4);
hipError_t launch_solve_backward(const float *dC, const float *A, const float *B, const float *C, const float *ex,
                                 const float *ey, const float *lam, int32_t mask_kind, float gamma, int64_t P,
                                 int64_t kx, int64_t ky, int64_t d, const float *factors, float *dA, float *dB,
                                 float *dlam, int32_t *info, void *ws, hipStream_t st, int rs_waves = 4);

// Row solves with stored factors (reverse mode, refinement correction) by streaming triangular solves.
void launch_trisolve_stored(const float *Lin, const float *rhs, const float *ex, const float *ey, const float *lam,
                            int mask_kind, float gamma, int64_t P, int64_t kx, int64_t ky, float *out, int *info,
                            const float *Cfwd, float *dlam_part, const float *addend, hipStream_t st,
                            const int *only = nullptr);
// The same for k_x <= 64: one wave per system, both substitutions in registers.
void launch_trisolve_small(const float *Lin, const float *rhs, const float *ex, const float *ey, const float *lam,
                           int mask_kind, float gamma, int64_t P, int64_t kx, int64_t ky, float *out, int *info,
                           const float *Cfwd, float *dlam_part, const float *addend, hipStream_t st);
// Row systems for 64 < k_x <= kMaxK: mode 0 forward (factors to Lout if non-NULL), mode 2 reverse mode with
// refactorisation (V rows, per-row dlambda terms).  tile_ws: tiled_workspace_bytes(P, k_x, k_y) bytes.
// only: if non-NULL, the systems of pairs p with only[p] == 0 are skipped (their outputs left as they are).
void launch_rowsolve_tiled(int mode, const float *K, const float *rhs, const float *ex, const float *ey,
                           const float *lam, int mask_kind, float gamma, int64_t P, int64_t kx, int64_t ky, float *out,
                           float *Lout, int *info, const float *Cfwd, float *dlam_part, float *tile_ws, hipStream_t st,
                           const int *only = nullptr);
size_t tiled_workspace_bytes(int64_t P, int64_t kx, int64_t ky);
void launch_adjoint_general(const float *V, const float *C, const float *A, const float *B, int64_t P, int64_t kx,
                            int64_t ky, int64_t d, float *Wbuf, const float *dlam_part, float *dlam, float *dA,
                            float *dB, hipStream_t st);

// K = A A^T [P][kx][kx] and, with with_R, R = B A^T [P][ky][kx] in float32.
void launch_gram(const float *A, const float *B, int64_t P, int64_t kx, int64_t ky, int64_t d, bool with_R,
                 float *K, float *R, hipStream_t st);
// The row systems of given normal products K [P][kx][kx], R [P][ky][kx], without stored factors.  tiles:
// tiled_workspace_bytes(P, kx, ky) bytes when kx > kSmallK.
void launch_solve_products(const float *K, const float *R, const float *ex, const float *ey, const float *lam,
                           int mask_kind, float gamma, int64_t P, int64_t kx, int64_t ky, float *C, int *info,
                           float *tiles, hipStream_t st);
// One system per pair with a given symmetric matrix: S [P][n][n] (n <= kMaxK), right-hand side g [P][n],
// solution out [P][n], info [P]; ex_zero [P][n] and ey_zero [P] must hold zeros (no mask shift is added) and
// lam [P] only flags an invalid value.  tiles: tiled_workspace_bytes(P, n, 1) bytes when n > kSmallK.
void launch_rowsolve_dense(const float *S, const float *g, const float *ex_zero, const float *ey_zero, const float *lam,
                           int64_t P, int64_t n, float *out, int *info, float *tiles, hipStream_t st);
// The vectorized solve with general commutativity operators (kx ky <= kMaxK).
size_t vectorized_workspace_bytes(int64_t P, int64_t kx, int64_t ky);
hipError_t launch_solve_vectorized(const float *A, const float *B, const float *D1, const float *D2, const float *lam,
                                   int64_t P, int64_t kx, int64_t ky, int64_t d, float *C, int32_t *info, void *ws,
                                   hipStream_t st);

void launch_gram64(const float *A, const float *B, int64_t P, int64_t kx, int64_t ky, int64_t d, double *K64,
                   double *R64, hipStream_t st);
void launch_residual64(const float *C, const double *K64, const double *R64, const float *ex, const float *ey,
                       const float *lam, int mask_kind, float gamma, int64_t P, int64_t kx, int64_t ky, float *rho,
                       hipStream_t st, const int *only = nullptr);
// flag: if non-NULL, flag[p] = 1 where the pair's products were replaced (estimate above threshold), else 0.
void launch_cond(const float *K, int64_t P, int64_t kx, int64_t ky, float threshold, const double *K64,
                 const double *R64, float *Kout, float *Rout, float *cond_est, hipStream_t st, int *flag = nullptr);
// Largest k_x for the condition estimate (its float32 factor lives in LDS).
constexpr int kMaxCondK = 256;

}  // namespace fmap
