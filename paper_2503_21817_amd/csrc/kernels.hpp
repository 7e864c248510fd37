// Host-side launchers of the Skip-FFN kernels.  Every launcher only enqueues
// work on `stream` and returns the hipError_t of the launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "gemm.hpp"

namespace skipffn {

// kernel classes for the built-in event profiler
enum KernelClass : int {
    KC_COMPACT = 0,
    KC_GATHER_RMSNORM,
    KC_GEMM_GATE_UP,
    KC_GEMM_DOWN,
    KC_RESID_SCATTER,
    KC_PASSTHROUGH,
    KC_GATHER_ROWS,
    KC_GEMM_DH_DWDOWN,      // dH + SwiGLU backward and dW_down in one grid
    KC_GEMM_DW_GATE_UP,     // dW_gate and dW_up, batched in one grid
    KC_GEMM_DXN,
    KC_RMSNORM_BWD,
    KC_FILL,
    KC_KV_COMPACT,
    KC_SUMMARY_FWD,
    KC_SUMMARY_BWD,
    KC_SELECT,
    KC_MERGE,
    KC_GEMM_DXN_DW,
    KC_COUNT
};
const char* kernel_class_name(int kc);
void profile_mark_begin(int kc, hipStream_t s);
void profile_mark_end(int kc, hipStream_t s);

// ---- compaction ---------------------------------------------------------------
size_t compact_workspace_bytes(int64_t T);
hipError_t launch_compact(const uint8_t* mask, int64_t T, int32_t* idx, int32_t* num_retained,
                          int32_t* pos, void* ws, hipStream_t s);

// the same with the library's own per-GPU scratch (no workspace, nothing allocated), T <= compact_static_max_tokens()
int64_t compact_static_max_tokens();
hipError_t launch_compact_static(const uint8_t* mask, int64_t T, int32_t* idx, int32_t* num_retained,
                                 int32_t* pos, hipStream_t s);
// status[0] = 0 if idx[0..R) is strictly ascending inside [0, T) else 1; status[1] = first bad position
hipError_t launch_validate_idx(const int32_t* idx, int R, const int32_t* r_dev, int64_t T, int32_t* status,
                               hipStream_t s);

// ---- row kernels ---------------------------------------------------------------
// Rows 0 .. T - 1 of row_chunks 16-byte pieces each; those NOT listed in idx are copied from src to dst (null: none).  A
// job of its own (launch_passthrough), or beside another kernel that reads the same rows.
struct SkippedRows { const void* src; void* dst; int64_t T, row_chunks; const int32_t* idx; };
// x rows (optional copy), normalised rows (scaled = false: as they are, not multiplied) and 1/rms for rows idx[0..R); chunk_major: xn is [C / 8][R][8]
hipError_t launch_gather_rmsnorm(const bf16_t* hidden, const int32_t* idx, int R,
                                 const int32_t* r_dev, int C, float eps, const bf16_t* gain,
                                 bf16_t* xrows, bf16_t* xn, float* rstd, bool chunk_major, bool scaled, const SkippedRows& sk, hipStream_t s);
// How many fp32 partial slabs a reducing kernel adds per output element: `splits` for a plain
// split-K GEMM (sk_nbg == 0), else the per-tile count of the balanced split (streamk_count)
// with sk_nbg workgroups per n-tile group and sk_kt K slabs per tile.
struct PartialLayout { int splits; int sk_nbg; int sk_kt; };
// out[idx[r]] = bf16(res[idx[r]] + sum_z partial[z][r])
hipError_t launch_resid_scatter(const float* partial, PartialLayout pl, int R, const int32_t* r_dev,
                                int C, const int32_t* idx, const bf16_t* res, bf16_t* out,
                                int no_residual, hipStream_t s);
// the same after launch_down_count: the slabs of the plan that the count on the device has (nothing where its K was whole)
hipError_t launch_resid_scatter_count(const float* partial, const RowPlans& plans, int ktiles, int R, int sum_rows, const int32_t* r_dev, int C,
                                      const int32_t* idx, const bf16_t* res, bf16_t* out, int no_residual, hipStream_t s);
// dst[r] = src[idx[r]]  (rows of row_bytes, multiple of 16)
hipError_t launch_gather_rows(const void* src, void* dst, int64_t row_bytes, const int32_t* idx,
                              int R, const int32_t* r_dev, hipStream_t s);
// dst[s][r] = src[s][idx[r]] for n_slabs slabs (slab strides in bytes, multiples of 16)
hipError_t launch_kv_compact(const void* src, void* dst, int64_t n_slabs, int64_t row_bytes,
                             int64_t src_slab_bytes, int64_t dst_slab_bytes, const int32_t* idx,
                             int R, const int32_t* r_dev, hipStream_t s);
// dst[r] = src[idx ? idx[r] : r] (dst optional) and the transposed copy dstT[c][r], leading
// dimension ldT (multiple of 8, >= R bound), columns r >= R zero; one or two copies of the same R rows
struct TransposeJob { const bf16_t* src; int C; const int32_t* idx; bf16_t* dst; bf16_t* dstT; };
hipError_t launch_gather_transpose(const TransposeJob* jobs, int count, int R, const int32_t* r_dev, int ldT, const SkippedRows& sk,
                                   hipStream_t s);
// dG, dU and their transposed copies from `splits` (2 to 4) fp32 slabs of dH, z * R * I apart
struct SwigluBwdArgs {
    const float* partial; int splits;
    const bf16_t *G, *U; bf16_t *dG, *dU, *dGT, *dUT;
    int R; const int32_t* r_dev; int I, ldT;
};
hipError_t launch_swiglu_bwd_reduce(const SwigluBwdArgs& a, hipStream_t s);
hipError_t launch_passthrough(const SkippedRows& sk, int R, const int32_t* r_dev, hipStream_t s);
// dX[idx[r]] = bf16(dY[r] + rmsnorm_bwd(sum_z dxn_partial[z][r], x[r], rstd[r], gain)); with dgain != null
// also dgain[c] (+)= sum_r dxn[r][c] * x[r][c] * rstd[r] (fp32, through gain_partial)
hipError_t launch_rmsnorm_bwd_scatter(const float* dxn_partial, PartialLayout pl, int R,
                                      const int32_t* r_dev, int C, const bf16_t* xrows,
                                      const float* rstd, const bf16_t* gain, const bf16_t* dY,
                                      const int32_t* idx, bf16_t* dX, float* gain_partial,
                                      float* dgain, int accumulate, hipStream_t s);
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);

// ---- adaptive summary layer -------------------------------------------------------------------
constexpr int SUM_CH = 16;        // tokens per workgroup chunk
int64_t summary_max_chunks(int64_t n_tok, int64_t S);      // chunks the launches cover
hipError_t launch_summary_forward(const bf16_t* hidden, int64_t T, int C, const int32_t* tok,
                                  const int32_t* seg, int64_t n_tok, int S, const bf16_t* w,
                                  bf16_t* out, float* scores, float* lse, float* xs_f32,
                                  float* part_acc, float* part_md, hipStream_t s);
hipError_t launch_summary_backward(const bf16_t* hidden, int64_t T, int C, const int32_t* tok,
                                   const int32_t* seg, int64_t n_tok, int S, const bf16_t* w,
                                   const float* xs_f32, const float* scores, const float* lse,
                                   const bf16_t* gout, bf16_t* grad_hidden, float* part_dw, float* dw,
                                   int accumulate, hipStream_t s);

// ---- retained-token selection ---------------------------------------------------------------------
constexpr int SEL_CH = 16;        // tokens per workgroup of the similarity kernel
hipError_t launch_select_retained(const bf16_t* feat, const bf16_t* cls, const int32_t* seq_off,
                                  int64_t n_feat, int B, int Cv, int n_keep, const int32_t* n_keep_dev,
                                  uint8_t* mask, float* sim, const int32_t* token_pos,
                                  uint8_t* skip_mask, int64_t T, hipStream_t s);

// ---- token merge -----------------------------------------------------------------------------------
constexpr int MERGE_MAX_N = 4096;   // tokens per set
constexpr int MERGE_CHUNK = 8;      // rows of a partial sum of normalised rows
hipError_t merge_init();         // raises the dynamic-LDS limits (once per process)
// normalised rows [n_tok][C]; partial sums [n_tok / MERGE_CHUNK + sets + 1][C] and sums [sets][C] of the sets of a group; per token
// 8 bytes and 4 bytes
struct MergeScratch { bf16_t* xn; float* part; float* sum; void* goal; int32_t* dropped; };
hipError_t launch_merge_group(const bf16_t* x, const SegTable& st, int n_max, int C, int k, int set_base, const MergeScratch& ws,
                              float* avg, int32_t* kept_idx, int32_t* assign, bf16_t* out, int ncu, hipStream_t s);
hipError_t launch_merge_bwd_group(const bf16_t* dout, const SegTable& st, int n_max, int C, int k, int set_base,
                                  const int32_t* assign, bf16_t* dx, hipStream_t s);

// ---- measurement aid: register-only MFMA loop -------------------------------------------------------
// out: blocks * 256 floats; clocks: 2 * blocks int64 (shader cycles, 100 MHz wall ticks per workgroup)
hipError_t launch_mfma_probe(int blocks, int iters, int random_operands, float* out, long long* clocks,
                             hipStream_t s);

// A gate/up GEMM that normalises its rows itself reads rows idx of hidden [T][C] and multiplies its sums by 1 / rms
struct RowNorm { const bf16_t* hidden; int64_t T; const int32_t* idx; const bf16_t* gain; float eps; };

// ---- the forward GEMMs of a handful of rows (rows <= 64) -----------------------------------------------
// H = silu(xn Wg^T) * (xn Wu^T); G and U optional.  norm != null: xn is not read (norm_in_gate_up).
// rstd != null: xn holds rows whose products are multiplied by it (scale_in_gate_up).  chunk_major, chunk_major_h: xn, H are [K / 8][rows][8] instead of row-major
hipError_t launch_few_rows_gate_up(const bf16_t* xn, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_gate,
                                   const bf16_t* w_up, bf16_t* H, bf16_t* G, bf16_t* U, bool chunk_major, bool chunk_major_h,
                                   const RowNorm* norm, const float* rstd, hipStream_t s);
// out[idx[r]] = bf16(res[idx[r]] + H[r] Wd^T)
hipError_t launch_few_rows_down(const bf16_t* H, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_down,
                                const int32_t* idx, const bf16_t* res, bf16_t* out, int no_residual, bool chunk_major,
                                hipStream_t s);

// ---- the forward GEMMs of up to 256 rows ------------------------------------------------------------------
hipError_t mid_rows_init();      // raises the dynamic-LDS limit of every instantiation (once per process)
// norm != null: xn is not read, up to kNormInMidRows rows; rstd != null: as above, up to as many rows and splits 1.  cols: gate_up_cols.  chunk_major_h: H is [I / 8][rows][8] instead of row-major; splits > 1: K cut in fp32 partial[splits][rows][2][I]
hipError_t launch_mid_rows_gate_up(const bf16_t* xn, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_gate,
                                   const bf16_t* w_up, bf16_t* H, bf16_t* G, bf16_t* U, bool chunk_major_h, int splits,
                                   int cols, float* partial, const RowNorm* norm, const float* rstd, hipStream_t s);
// fp32 partial[splits][rows][C]
hipError_t launch_mid_rows_down(const bf16_t* H, int rows, const int32_t* r_dev, int C, int I, const bf16_t* w_down,
                                int splits, float* partial, hipStream_t s);

// ---- the forward GEMMs with a row count on the device, below a bound of more than 256 rows (countrows.hip) -----------
hipError_t count_rows_init();    // raises the dynamic-LDS limits (once per process)
// up to 256 rows on tiles of all rows, so neither G and U nor the transposed copy
hipError_t launch_gate_up_count(GemmArgs& args, hipStream_t s);
// partial (for 16 slabs of 256 rows and 8 of the bound) or out0, e0, idx, as the plan of the count wants them
hipError_t launch_down_count(GemmArgs& args, const RowPlans& plans, hipStream_t s);

// ---- GEMMs -----------------------------------------------------------------------
hipError_t gemm_init();   // raises the dynamic-LDS limit of every instantiation (once per process)
// A is K-contiguous; b_kc: B too (stream.hpp), or N-contiguous (gemm.hpp)
hipError_t launch_gemm(bool b_kc, int epi, GemmArgs& args, hipStream_t s);
// two independent GEMMs in one grid, the first dispatched first: SwiGLU backward (dH -> dG, dU), and store (dW_down = dY^T * H)
hipError_t launch_gemm_dh_dw_down(GemmArgs& dh, GemmArgs& dw, hipStream_t s);
// a GEMM with an N-contiguous B operand into fp32 slabs, K cut evenly, and weight gradients in one grid: dXn and dW_gate, dW_up on n0
// and dw_workgroups (plan_dxn); dH and dW_down (dh_splits)
hipError_t launch_gemm_partial_dw(GemmArgs& a, GemmArgs& dw, int n0, int dw_workgroups, hipStream_t s);
hipError_t launch_gemm_dh_partial_dw_down(GemmArgs& dh, GemmArgs& dw, hipStream_t s);
// balanced split-K GEMM into fp32 partial slabs (EPI_PARTIAL): nbg workgroups per n-tile group
hipError_t launch_gemm_streamk(bool b_kc, GemmArgs& args, int nbg, hipStream_t s);

}  // namespace skipffn
