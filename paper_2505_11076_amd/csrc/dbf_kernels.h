// Launchers of the HIP kernels (defined in the .hip files, called from dbf_api.hip).
#ifndef DBF_KERNELS_H
#define DBF_KERNELS_H

#include <hip/hip_runtime.h>

#include "dbf_internal.h"

// Vector-ALU kernel, one stage (B or A): `blocks` workgroups, workgroup i handles work[i]
// (one row tile).  x_base / y_base are the caller's fp16 buffers (only the one the stage
// touches is used).
hipError_t dbf_launch_stage_valu(bool stage_a, const DbfStage* table, const DbfWorkItem* work,
                                 int blocks, const void* x_base, void* y_base, int batch,
                                 hipStream_t stream);

// Matrix-core kernel over items[0..n_items): workgroup i handles items[i].
//   use_sync != 0 (fused launch of B items followed by A items): an A-stage workgroup waits, for at most
//   wait_limit_us microseconds, until the layer's B-stage workgroups of THIS launch have published all their
//   rows (sync, see DbfPlan::d_sync); a workgroup that gives up writes NaN outputs and counts a time-out.
//   use_sync == 0: no waiting and no counters (the caller orders the stages by launches).
// Items with nrt > 1 are allowed only if every item's columns fit one LDS chunk, i.e.
// dbf_mfma_chunk_tiles(batch, max_cols, shared_q) >= dbf_col_tiles(max_cols).
//   pieces != 0: the list may hold column pieces of row tiles (DbfItem::pieces > 1; one row tile per
//   item, batch <= DBF_PIECES_MAX_BATCH); pieces == 0: every item covers all columns of its row tiles.
//   shared_q != 0: the input of the items' stage has been quantised for the whole launch by
//   dbf_launch_quantise_inputs (same stream, earlier); the items copy it instead of quantising it themselves.
//   Only with use_sync == 0 and pieces == 0.
//   one_pass_rows != 0: the caller has checked that every B-stage row of the launch can be read in 16-byte pieces
//   (columns a multiple of 8, 16-byte aligned address at this batch), so that at batch 1 rows of up to
//   dbf_mfma_one_pass_cols() columns all take the one-pass prologue -- which the fp4 x bf6 form of the kernel needs.
hipError_t dbf_launch_items_mfma(const DbfItem* items, int n_items, unsigned long long* sync, int n_layers,
                                 int use_sync, const void* x_base, void* y_base, int batch,
                                 int max_cols, int pieces, int shared_q, int one_pass_rows, int wait_limit_us,
                                 hipStream_t stream);
// Quantises the input of one stage (stage_a = 0: x times b of every layer, 1: the middle activations) of the
// n_layers stages in d_stages for `batch` rows into the stages' q_in buffers.
hipError_t dbf_launch_quantise_inputs(const DbfStage* d_stages, int n_layers, int stage_a, const void* x_base,
                                      int batch, hipStream_t stream);
int dbf_mfma_chunk_tiles(int batch, int max_cols, int shared_q);
// Widest input row (columns) the matrix-core kernel's one-pass prologue takes at batch 1: such rows are
// read once and quantised from registers; wider ones are read twice (scale, then quantisation).
int dbf_mfma_one_pass_cols();
// One-time, per-process set-up of the matrix-core decode kernels (LDS limits); cheap to call again.
hipError_t dbf_mfma_prepare();

// Launches of few workgroups (dbf_gemv_few.hip): one stage of the plan's layers for T (below 65536) tokens or batch rows, every workgroup
// rounding the stage input it needs.  dbf_few_takes: whether the stage is one for it.
// t_over: the middle activations [T][t_stride], or NULL for the layers' own (T <= DBF_MAX_BATCH).
bool dbf_few_takes(const DbfPlan& p, bool stage_a, int T);
// Bytes of DbfPlan::d_few_acc for a stage of n_items row tiles: 8.1 KiB each, 0 if no call cuts its rows.
size_t dbf_few_acc_bytes(int n_items, int max_cols);
hipError_t dbf_launch_few(const DbfPlan& p, bool stage_a, const void* x, void* y, float* t_over, int T, hipStream_t stream);
// Both stages of small layers in one launch, a workgroup per layer and pair of tokens; dbf_small_layer_takes: whether the plan's layers are.
bool dbf_small_layer_takes(const DbfPlan& p, int T);
hipError_t dbf_launch_small_layers(const DbfPlan& p, const void* x, void* y, int T, hipStream_t stream);
// One-time, per-process set-up of those kernels (LDS limits); cheap to call again.
hipError_t dbf_few_prepare();

// Prefill (T tokens): two stages with the middle activations in the caller's workspace; arguments are
// validated by dbf_gemm before this is called.  int8 matrix cores as the adder (masked sign bytes as one
// operand, the activations rounded per token to 16-bit fixed point and split into two int8 planes), exact
// integer sums, middle activations in fp32.
struct dbf_layer;
size_t dbf_gemm_i8_workspace_bytes(const dbf_layer* L, int T);
// One-time, per-process set-up of the prefill kernels (LDS limits); cheap to call again.
hipError_t dbf_gemm_i8_prepare();
hipError_t dbf_gemm_i8_launch(const dbf_layer* L, const void* X_dev, void* Y_dev, int T, void* workspace_dev, hipStream_t stream);

// Middle-channel pruning: fills the sign tiles and vectors of `dst` (a freshly created layer with
// k = n_keep on the same device) from `src` and the kept middle indices keep_dev (device, increasing,
// each < src->k), and zeroes clear_bytes from `clear` on (multiples of 16).  Queued on `stream`.
hipError_t dbf_prune_launch(const dbf_layer* src, dbf_layer* dst, const int* keep_dev, int n_keep, void* clear, size_t clear_bytes, hipStream_t stream);

// What dbf_svid can do with (a launch per round); dbf_svid_workspace_bytes is that or more.
size_t dbf_svid_least_workspace(int rows, int cols);

// For tests: a call of dbf_svid that is one launch (DBF_EINVAL: it is not), whose first `door` workgroups are let in and
// wait `door_spins` polls for all of these and `spins` for each other's sums.
extern "C" int dbf_svid_forced(const void* Z_dev, int rows, int cols, int iters, void* a_dev, void* m_dev, void* bits_dev, void* workspace_dev,
                               size_t workspace_bytes, int door, int door_spins, int spins, void* hip_stream);

// dbf_svid (its arguments checked by the caller) and then the scaled dual of the ADMM update, U = Z - a . Sign(Z) . m^T.
int dbf_svid_dual(const void* Z_dev, int rows, int cols, int iters, void* a_dev, void* m_dev, void* bits_dev, void* workspace_dev, size_t workspace_bytes,
                  float* U_dev, hipStream_t stream);

#endif  // DBF_KERNELS_H
