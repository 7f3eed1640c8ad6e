// Host launchers of the gate-projection products (internal to librecblr.so).
#pragma once

#include <initializer_list>

#include "launch.hpp"

namespace recblr {

// Bytes of the packed-weight scratch that launch_project_forward and
// launch_project_backward_data take (16-byte aligned).
size_t project_pack_workspace(int64_t D, IoType io);

// z_r = x W_r^T + b_r, z_i = x W_i^T + b_i over M = B*L rows (b may be null).
// x, W, b and dx use the I/O type; z and dz are always fp32.  The fast path
// needs zi, dzi after zr, dzr in one allocation (their byte distance is used
// as an offset from zr, dzr).
hipError_t launch_project_forward(const void* x, const void* wr, const void* br, const void* wi,
                                  const void* bi, void* zr, void* zi, int64_t M, int64_t D,
                                  IoType io, void* pack, hipStream_t stream);

// dx += dz_r W_r + dz_i W_i (dx holds the direct term on entry); dx is in the
// I/O type, or fp32 when dx_f32 is set.  With `packed`, pack already holds the
// weights in this product's order (launch_prepare_scan).
hipError_t launch_project_backward_data(const void* dzr, const void* dzi, const void* wr,
                                        const void* wi, void* dx, int64_t M, int64_t D,
                                        IoType io, void* pack, hipStream_t stream,
                                        bool dx_f32 = false, bool packed = false);

// Partial rows of dLoss/dq r ([rows][D]) that still have to be summed to
// dLambda; rows = 0: none.
struct DlambdaRows {
    const float* partial = nullptr;
    int64_t rows = 0;
    const float* lambda = nullptr;
    float* dlambda = nullptr;
};

// dW_r, dW_i = dz^T x and db_r, db_i = column sums of dz; uses
// project_dw_workspace(M, D) bytes of scratch at `ws`.  dl, if it has rows, is
// summed by the same last launch.
hipError_t launch_project_backward_weights(const void* dzr, const void* dzi, const void* x,
                                           float* dwr, float* dbr, float* dwi, float* dbi,
                                           int64_t M, int64_t D, IoType io, void* ws,
                                           hipStream_t stream,
                                           const DlambdaRows& dl = DlambdaRows{});

// The two products above in one pass over dz, where project_backward_both_applies
// (sizes and types at which it is faster, 16-byte aligned operands): dx += dz W, dW,
// db and dl's rows.  x and dx of type x_io, weights of type w_io (fp32 x with bf16
// weights: dx is fp32) packed by launch_prepare_scan with frag; ws:
// project_dw_workspace(M, D) bytes.
bool project_backward_both_applies(int64_t M, int64_t D, IoType x_io, const void* dzr,
                                   const void* dzi, const void* x, const void* dx, const void* ws);
size_t project_backward_both_workspace(int64_t M, int64_t D);
hipError_t launch_project_backward_both(const float* dzr, const float* dzi, const void* x,
                                        const void* pack, void* dx, float* dwr, float* dbr,
                                        float* dwi, float* dbi, int64_t M, int64_t D, IoType x_io,
                                        IoType w_io, void* ws, const DlambdaRows& dl,
                                        hipStream_t stream);
// The last launch of either: split partials [splits][2 D][D] and [splits][2 D] (and
// dl's rows) summed in double in a fixed order.
hipError_t launch_dw_reduce(const float* partial, const float* dbpart, int64_t splits, int64_t D,
                            float* dwr, float* dbr, float* dwi, float* dbi, const DlambdaRows& dl,
                            hipStream_t stream);

// What the scans with the projections fused in need first, in one launch:
// [W_r; W_i] by channel group of 64 (rows 128 g.. : W_r rows of the group's
// channels, then their W_i rows) into `groups`, with dx not null also in the
// order of launch_project_backward_data or (frag) launch_project_backward_both
// (each project_pack_workspace(D, io) bytes of bf16 planes), and the look-back state
// (n words, ticket, status).
hipError_t launch_prepare_scan(const void* wr, const void* wi, int64_t D, IoType io, void* groups,
                               void* dx, bool frag, uint64_t* states, int64_t n, unsigned* ticket,
                               hipStream_t stream);

// Recurrent step with the gate projections fused in (z stays in registers):
// h_next = alpha h_prev + beta x with z = x W^T + b.  Returns false, having
// launched nothing, where the fused path does not apply (D % 8 != 0, x or
// pack not 16-byte aligned, or x too large); else launches and stores the
// launch status in *err.  pack takes step_pack_workspace(D, io) bytes.
size_t step_pack_workspace(int64_t D, IoType io);
bool launch_fused_step(const void* x, const void* wr, const void* br, const void* wi,
                       const void* bi, const float* lambda, const float* h_prev, float* h_next,
                       int64_t B, int64_t D, IoType io, void* pack, hipStream_t stream,
                       hipError_t* err);

// Plain fp32 linear layer Y = X W^T + b, W[N][K] (nn.Linear layout), all
// operands row-major and contiguous, on fp32 matrix-core tiles (fp32
// products): the forward Y[M][N] = X[M][K] W^T + bias (bias may be null;
// act, if given, receives SiLU(Y)), and the data gradient
// dX[M][K] = dY[M][N] W in one of three epilogues: store, accumulate, or
// multiply by SiLU'(aux) with aux[M][K] the SiLU's input.  The data gradient
// first writes W^T into wt (N * K floats).  Preconditions: wgrad_fast_ok for
// the operands and the shape (N and K multiples of 4).
enum class LinearMode { kStore, kAccumulate, kSiluGrad };
hipError_t launch_linear_fwd32(const float* x, const float* w, const float* bias, float* y,
                               float* act, int64_t M, int64_t N, int64_t K, hipStream_t stream);
hipError_t launch_linear_dgrad32(const float* dy, const float* w, float* dx, LinearMode mode,
                                 const float* aux, int64_t M, int64_t N, int64_t K, float* wt,
                                 hipStream_t stream);

// Weight gradient of a plain fp32 linear layer Y = X W^T + b (W[N][K]) on
// the matrix-core tiles (3-term bf16 split of both operands):
// dW[N][K] = dY[M][N]^T X[M][K] and db[N] = column sums of dY (db may be
// null), as split-M partials (wgrad_workspace bytes at ws) summed in a fixed
// order (launch_colsum, colsum_workspace(wgrad_splits, N * K) bytes at
// colsum_ws).  Applies when wgrad_fast_ok holds (row-major contiguous
// operands, N and K multiples of 4, 16-byte alignment, under 2 GiB each).
bool wgrad_fast_ok(std::initializer_list<const void*> ptrs, int64_t M, int64_t N, int64_t K);
int64_t wgrad_splits(int64_t M, int64_t N, int64_t K);
size_t wgrad_workspace(int64_t M, int64_t N, int64_t K);
hipError_t launch_wgrad(const float* dy, const float* x, float* dw, float* db, int64_t M,
                        int64_t N, int64_t K, void* ws, void* colsum_ws, hipStream_t stream);

// The linear sub-layers of the model (fp32) for D = 64 rows: the feed-forward one,
// Q = SiLU(X W1^T + b1) W2^T + b2 with 256 hidden units, and the projections around
// the gated layer, Hx = X Wx^T + bx, Hz = X Wz^T + bz, O = y Wo^T + bo with E = 128
// (sublayers_fused_applies, 16-byte aligned operands), one kernel each way.  The
// feed-forward stores A = X W1^T + b1 for its backward.  Backward: adds to dx (for the
// output projection stores dy) and writes the sub-layer's gradients, contiguous in
// parameter order, at grads; part: sublayers_fused_workspace(M) bytes, summed by
// launch_colsum (colsum_ws: sublayers_fused_colsum(M) bytes).
constexpr int64_t kFfnGrads = 2 * 256 * 64 + 256 + 64;     // dW1, db1, dW2, db2
constexpr int64_t kProjInGrads = 2 * (128 * 64 + 128);     // dWx, dbx, dWz, dbz
constexpr int64_t kProjOutGrads = 128 * 64 + 64;           // dWo, dbo
bool sublayers_fused_applies(int64_t M, int64_t D, std::initializer_list<const void*> ptrs);
size_t sublayers_fused_workspace(int64_t M);
size_t sublayers_fused_colsum(int64_t M);
hipError_t launch_ffn_forward(const float* x, const float* w1, const float* b1, const float* w2,
                              const float* b2, float* a, float* q, int64_t M, hipStream_t stream);
hipError_t launch_ffn_backward(const float* x, const float* dq, const float* a, const float* w1,
                               const float* w2, float* dx, float* grads, int64_t M, float* part,
                               void* colsum_ws, hipStream_t stream);
hipError_t launch_proj_in_forward(const float* x, const float* wx, const float* bx,
                                  const float* wz, const float* bz, float* hx, float* hz,
                                  int64_t M, hipStream_t stream);
hipError_t launch_proj_in_backward(const float* x, const float* dhx, const float* dhz,
                                   const float* wx, const float* wz, float* dx, float* grads,
                                   int64_t M, float* part, void* colsum_ws, hipStream_t stream);
hipError_t launch_proj_out_backward(const float* y, const float* dout, const float* w, float* dy,
                                    float* grads, int64_t M, float* part, void* colsum_ws,
                                    hipStream_t stream);

int64_t project_dw_splits(int64_t M, int64_t D);
size_t project_dw_workspace(int64_t M, int64_t D);

// The prediction head in fp32 (head.hip), D a multiple of 64, at most 512:
// logits = h E^T, dE = dlogits^T h and dh = dlogits E, all stored (not added).  h and
// dh [B][D], E and dE [V][D], logits and dlogits [B][V]; ws: B V floats of scratch.
hipError_t launch_head_logits(const float* h, const float* E, float* logits, int64_t B, int64_t V,
                              int64_t D, hipStream_t stream);
hipError_t launch_head_dE(const float* dlogits, const float* h, float* dE, int64_t B, int64_t V,
                          int64_t D, hipStream_t stream);
hipError_t launch_head_dh(const float* dlogits, const float* E, float* dh, int64_t B, int64_t V,
                          int64_t D, float* ws, hipStream_t stream);

}  // namespace recblr
