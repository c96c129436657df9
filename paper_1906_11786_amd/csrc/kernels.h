// Launchers of the gfx950 kernels, one per device operation.  Arguments are
// validated by the C-ABI layer before these are called; each returns the
// hipGetLastError() of its launches.
//
// Every kernel source is built twice, once per storage dtype (bf16 kernels and
// the fp32 direct-weight step with matrix-core results kept in VGPRs, the other
// fp32 kernels with the compiler's default register assignment; wgrad_wide.hip,
// bf16 only, may keep them in AGPRs); the launchers of each build live in
// ggnn::impl_bf16 / ggnn::impl_f32, and the functions below pick one by dt.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

#include "../../include/ggnn.h"

namespace ggnn {

// Partial-sum reductions that a caller can collect and launch together
// (launch_reduce_multi): out[i] += sum_{s < nsplit} part[s * stride + i].
struct ReduceSeg {
  const float* part;
  float* out;
  int nsplit, count;
  long stride;
};
struct ReduceList {
  static constexpr int kMax = 8;
  ReduceSeg seg[kMax];
  int n = 0;
};
hipError_t launch_reduce_multi(const ReduceList& l, hipStream_t st);
// Appends to *defer (when non-NULL and not full), else launches the reduction.
// Message-transform weight gradient at H = 256 in bf16 with node-major dM
// (csrc/wgrad_wide.hip): per-split partials P [nsplit][E][256][256] and, when
// Pb is not NULL, Pb [nsplit][E][256]; splits of rows_per_split rows.
hipError_t launch_transform_wgrad_nm256(int nsplit, int rows_per_split, long K, int E, const void* X, const void* dM,
                                        long ldk, float* P, float* Pb, hipStream_t st);
// GRU weight gradients at H = 256 in bf16 (csrc/wgrad_wide.hip): partials
// P [nsplit][2][256][768] (dWi, dU) and Pb [nsplit][768]; splits of
// rows_per_split rows (a multiple of 32, as K); prog: nsplit x 8 ints of
// pacing counters (any contents; NULL turns pacing off).
hipError_t launch_gru_wgrad256(int nsplit, int rows_per_split, long K, const float* a, const void* h,
                               const void* saved, const void* ghat, float* P, float* Pb, int* prog, hipStream_t st);
hipError_t reduce_or_defer(const float* part, float* out, int nsplit, int count, long stride, ReduceList* defer,
                           hipStream_t st);

// Supernode share of a fused bit-band step (the first 32 nodes are
// supernodes): the slice bits of the step's direction, [E][n_pad][s/8] (the
// column slice forward, the transposed row slice reverse), and the record
// [P_e (sr x H) | deg_e (sr)], the sums over all nodes that give the first sr
// supernode rows their per-type aggregate (launch_super_long_fused forward,
// launch_super_gather_rev or launch_super_long_fused reverse).
struct SnStep {
  const void* bits;
  const float* rec;
  int s;
  int sr;   // record rows: the supernodes with edges are among the first sr (16 or 32)
};

#define GGNN_DT_LAUNCHERS                                                                                         \
  hipError_t launch_banded_fwd(int n_pad, int B, int H, int E, const void* band, const float* M, float* a,        \
                               hipStream_t st);                                                                   \
  hipError_t launch_banded_bwd(int n_pad, int B, int H, int E, const void* band, const void* da, void* dM,        \
                               long ldm, hipStream_t st);                                                         \
  hipError_t launch_banded_bwd_bits(int n_pad, int B, int H, int E, const void* bits_t, const void* da, void* dM, \
                                    long ldm, hipStream_t st);                                                    \
  hipError_t launch_transpose_weights(int H, int E, const void* W, void* Wt, hipStream_t st);                    \
  hipError_t launch_transform_fwd(int n_pad, int H, int E, const void* X, const void* W, const float* bias,       \
                                  float* M, hipStream_t st);                                                      \
  hipError_t launch_transform_bwd_dx(int n_pad, int H, int E, const void* W, const void* dM, long ld,             \
                                     const float* dX_in, float* dX_out, hipStream_t st);                          \
  hipError_t launch_transform_wgrad(long K, int H, int E, const void* X, const void* dM, long ld, float* dW,      \
                                    float* dbias, void* ws, hipStream_t st);                                      \
  hipError_t launch_transform_wgrad_nm(long K, int H, int E, const void* X, const void* dM, long ldk, float* dW,  \
                                       float* dbias, void* ws, ReduceList* defer, hipStream_t st);                \
  hipError_t launch_gru_fwd(int n_pad, int H, const float* a, const void* h, const void* Wi, const void* U,       \
                            const float* b, void* h_out, void* saved, const void* packed, hipStream_t st);        \
  hipError_t launch_gru_bwd_nodes(int n_pad, int H, const float* dh_out, const void* h, const void* saved,        \
                                  const void* Wi, const void* U, void* da, float* dh, void* ghat,                 \
                                  const void* packed, hipStream_t st);                                            \
  hipError_t launch_gru_pack(int H, const void* Wi, const void* U, void* packed, hipStream_t st);               \
  hipError_t launch_gru_wgrad(long K, int H, const float* a, const void* h, const void* saved, const void* ghat,  \
                              float* dWi, float* dU, float* db, void* ws, ReduceList* defer, hipStream_t st);    \
  hipError_t launch_readout_loss(int H, int n_graphs, const void* X, const float* w_out, const float* b_out,      \
                                 const int32_t* cand_node, const int32_t* cand_ptr, const int32_t* target,       \
                                 float* logits, float* loss, float* dlogit, hipStream_t st);                     \
  hipError_t launch_readout_bwd(int n_pad, int H, int n_cand, const void* X, const float* w_out,                 \
                                const int32_t* cand_node, const float* dlogit, float* dX, float* dw_out,         \
                                float* db_out, void* ws, hipStream_t st);                                        \
  hipError_t launch_sparse_step(int n_pad, int H, int E, const int32_t* row_ptr, const int32_t* col,            \
                                const void* X, const void* Wt, const float* bias, float* a, hipStream_t st);   \
  hipError_t launch_super_fwd(int n_pad, int H, int E, int s, const void* rows, const void* cols, const void* X,  \
                              const void* W, const float* bias, float* a, void* ws, hipStream_t st);            \
  hipError_t launch_super_bwd(int n_pad, int H, int E, int s, const void* rows, const void* rows_t,              \
                              const void* cols_t, const void* X, const void* W, const void* da, float* dX,       \
                              float* dW, float* dbias, void* ws, hipStream_t st);                                \
  bool step_wide_applies(int B, int H);                                                                           \
  hipError_t launch_step_wide(bool rev, int n_pad, int B, int H, int E, const void* bits, const void* V,          \
                              const void* Wsrc, const float* bias, float* out, const float* dX_in, void* dM,      \
                              long ldm, hipStream_t st);                                                          \
  hipError_t launch_step_direct(bool rev, int n_pad, int B, int H, int E, const void* bits, const void* V,        \
                                const void* W, const void* Wt, const float* bias, float* out, const float* dX_in, \
                                void* dM, long ldm, hipStream_t st);

namespace impl_bf16 {
GGNN_DT_LAUNCHERS
// The narrow step kernel (csrc/banded_bits.hip).
hipError_t launch_step_fwd_bits(int n_pad, int B, int H, int E, const void* bits, const void* X, const void* W,
                                const float* bias, float* a, hipStream_t st);
hipError_t launch_step_fwd_bits_gru(int n_pad, int B, int H, int E, const void* bits, const void* X,
                                    const void* W, const void* Wt, const float* bias, float* a, const void* Wi,
                                    const void* U, const float* bg, void* h_out, void* saved, bool* fused,
                                    hipStream_t st);
hipError_t launch_step_bwd_bits_gru(int n_pad, int B, int H, int E, const void* bits_t, const void* da,
                                    const void* W, const float* dX_in, float* dX_out, void* dM, long ldm,
                                    const void* Wi, const void* U, const void* h_prev, const void* saved_prev,
                                    void* da_prev, float* dh_prev, void* ghat_prev, bool* fused,
                                    hipStream_t st);
hipError_t launch_step_bwd_bits(int n_pad, int B, int H, int E, const void* bits_t, const void* da,
                                const void* W, const float* dX_in, float* dX_out, void* dM, long ldm,
                                hipStream_t st);
// Fused supernode steps (bf16, H <= 64, grids small enough for the
// two-group forms): whether both fused steps take the supernode share at
// this size, and the forward step (with its GRU) and reverse step (with the
// previous step's GRU reverse when da_prev is not NULL) carrying it.
bool step_sn_fusable(int n_pad, int B, int H, int E);
// The record of the fused supernode steps: rec = [P_e (sr x H) | deg_e (sr)],
// P_e = bits_e Z over all nodes for the first sr slice rows (zfm: Z
// feature-major), as a gather where Z is node-major (n_pad a multiple of 64),
// else as the long contraction with its per-chunk partials in ws.
hipError_t launch_super_long_fused(int n_pad, int H, int E, int s, int sr, const void* bits, const void* Z, bool zfm,
                                   float* ws, float* rec, hipStream_t st);
// The fused reverse step's supernode record from the step's gate gradients G^ (node-major [n_pad][3H])
// and Wi: (sum over the listed out-edges of G^ rows) Wi^T (bf16, H = 32 or 64).
bool super_gather_rev_applies(int n_pad, int H);
hipError_t launch_super_gather_rev(int n_pad, int H, int E, int s, int sr, const void* bits, const void* ghat,
                                   const void* Wi, float* rec, hipStream_t st);
hipError_t launch_step_fwd_bits_gru_sn(int n_pad, int B, int H, int E, const void* bits, const void* X, const void* W,
                                       const void* Wt, const float* bias, float* a, const void* Wi, const void* U,
                                       const float* bg, void* h_out, void* saved, const SnStep& sn, hipStream_t st);
hipError_t launch_step_bwd_bits_sn(int n_pad, int B, int H, int E, const void* bits_t, const void* da,
                                   const void* W, const float* dX_in, float* dX_out, void* dM, long ldm,
                                   const void* Wi, const void* U, const void* h_prev, const void* saved_prev,
                                   void* da_prev, float* dh_prev, void* ghat_prev, const SnStep& sn, hipStream_t st);
}
namespace impl_f32 {
GGNN_DT_LAUNCHERS
}
#undef GGNN_DT_LAUNCHERS

#define GGNN_DT_PICK(fn, ...) (dt == GGNN_BF16 ? impl_bf16::fn(__VA_ARGS__) : impl_f32::fn(__VA_ARGS__))

// Dense band: transform-first propagation and its reverse.  dM rows have
// length ldm >= n_pad (ldm = T * n_pad when the reverse pass keeps every
// step's message gradient for the weight-gradient products).
inline hipError_t launch_banded_fwd(int dt, int n_pad, int B, int H, int E, const void* band, const float* M,
                                    float* a, hipStream_t st) {
  return GGNN_DT_PICK(launch_banded_fwd, n_pad, B, H, E, band, M, a, st);
}
inline hipError_t launch_banded_bwd(int dt, int n_pad, int B, int H, int E, const void* band, const void* da,
                                    void* dM, long ldm, hipStream_t st) {
  return GGNN_DT_PICK(launch_banded_bwd, n_pad, B, H, E, band, da, dM, ldm, st);
}

// out[i] += sum_s part[s * stride + i], i < count, fixed summation order.
hipError_t launch_reduce_partials(const float* part, float* out, int nsplit, int count, long stride,
                                  hipStream_t st);
hipError_t launch_fill_zero(float* p, size_t count, hipStream_t st);

// Whether a bit-band step runs as the direct-weight kernel (csrc/banded_direct.hip): always in fp32; in bf16
//   where the fused narrow kernel would stream its blocks once per edge type (H = 64 at B >= 256, H = 32 at
//     B = 512): 657 -> 300 us for a pass at H = 64, B = 256 and 100,000 nodes, 515 -> 93 us (T = 2) at 2,000;
//   the reverse up to 128 row tiles of 32 nodes at H = 64, B = 64 or 128 and H = 32, B = 256, where it and the GRU's
//     own launch beat the fused step with its few waves (both directions at T = 4, H = 64, B = 128: 182 -> 163 us at
//     1,000 nodes, 184 -> 177 at 4,000, but 201 -> 223 at 8,000), few types apart (step_fused_small_rev).  Smaller blocks
//     are left to the fused step, in the forward too, though with the types dealt round robin the direct one is ahead at
//     H = 64, B = 32 (2,048 nodes, fused / direct: 4 types forward 9.5 / 9.1, reverse 13.5 / 11.7, 10 types 12.7 / 10.7, 16.2
//     / 13.8) and from about seven types on at H = 32 (B = 128, 4 types 7.4 / 8.2, 8.6 / 8.4, 10 types 10.7 / 9.2, 11.7 / 9.8;
//     B = 32, 10 types 7.1 / 7.5, 7.6 / 8.0).  In the forward of the larger ones it depends on the types (below);
//   at H = 128 up to 1,024 tiles, at H = 256 up to 512, 1,024 at B = 512: with more rows the wide kernel's sharing of
//     every weight between the rows of a block pays.  10 types, wide / direct, forward with its GRU, then reverse, us:
//     H = 128, B = 128: 79 / 24, 71 / 19 at 2,048 nodes, 99 / 70, 76 / 56 at 32,768, 137 / 135, 105 / 128 at 65,536;
//     H = 256, B = 256: 237 / 136, 168 / 121 at 16,384, 252 / 239, 170 / 200 at 24,576; B = 512: 546 / 373, 597 / 296
//     at 32,768, 621 / 731, 614 / 601 at 65,536.
inline bool step_direct(int dt, int n_pad, int B, int H, bool rev) {
  const int tiles = n_pad / 32;
  if (dt == GGNN_F32) return true;
  if (H == 32) return B == 512 || (rev && B == 256 && tiles <= 128);
  if (H == 64) return B >= 256 || (rev && B >= 64 && tiles <= 128);
  return tiles <= (H == 128 || B == 512 ? 1024 : 512);
}
// The reverse step with the GRU reverse after it at these sizes: with few types the launch saved by fusing counts for
// more.  Fused / direct, us: H = 32, B = 256: one type 7.6 / 8.3 at 512 nodes, two 8.2 / 9.4 at 4,096, three 9.4 / 9.2;
// H = 64 with 128 tiles, where the fused step has two waves per workgroup: B = 64 one type 10.9 / 11.9, two 11.5 / 12.1,
// three 12.3 / 12.3; B = 128 one 12.1 / 12.8, two 12.8 / 13.1 (on fewer tiles 15.4 / 12.2 and more apart).
inline bool step_fused_small_rev(int dt, int n_pad, int B, int H, int E) {
  if (dt == GGNN_F32) return false;
  return H == 32 ? B == 256 && E <= 2 : H == 64 && n_pad / 32 == 128 && E * B <= 128;
}
// Without the transposed weights the wide kernel does not apply: at H >= 128 the forward is the direct kernel on every
// grid (the aggregate, B = 128, 4 types, 65,536 nodes: H = 128 108 -> 48 us against the narrow kernel's streamed blocks,
// H = 256 226 -> 175), except where a single type leaves nothing to reuse of what it stages.  Narrow / direct there, us:
// H = 256, B = 64: 21 / 23 at 8,192 nodes, 90 / 96 at 65,536, B = 512 72 / 99, 160 / 236; H = 128, B = 64 17 / 22 at
// 32,768, B = 512 62 / 88 at 65,536; H = 64, B = 512 35 / 45 (26 / 21 at 16,384).
inline bool step_narrow_one_type(int dt, int n_pad, int B, int H, int E) {
  if (dt != GGNN_BF16 || E != 1) return false;
  const int tiles = n_pad / 32;
  if (B == 64) return H == 256 || (H == 128 && tiles > 256);
  return B == 512 && (H == 256 || (H >= 64 && tiles > 1024));
}
inline bool step_direct_no_wt(int dt, int n_pad, int B, int H, int E) {
  return !step_narrow_one_type(dt, n_pad, B, H, E) && (H >= 128 || step_direct(dt, n_pad, B, H, false));
}

// The forward with its GRU on small grids at H <= 64 (with and without transposed weights, the same bits): the fused
// step walks the types one after another, the direct kernel takes up to eight side by side, but the GRU is a launch of its own (4.4 us).
// 8 steps of 1,987 nodes, fused / direct: H = 64, B = 128: 10 types 139 / 121 us, 6 types 114 / 104, 5 types 109 / 102,
// 4 types 100 / 101, 2 types 87 / 97 (10 types at 4,000 nodes: 145 / 124); B = 64: 10 types 119 / 110, 8 types 108 / 99,
// 6 types 97 / 97, 5 types 94 / 96; H = 32, B = 256: 10 types 110 / 95, 8 types 99 / 86, 6 types 87 / 86, 5 types
// 85 / 85.  The line was measured at 1,987 nodes; against the fused step alone the direct one is ahead at every number of
// nodes and types that it is taken for (H = 64, B = 128, 10 types: 512 nodes 17.0 / 13.1, 4,096 18.1 / 13.8).  With
// the types dealt round robin it is level from four types on (B = 64, 2,048 nodes, 4 types 10.8 / 9.7), and the aggregate alone
// (launch_step_fwd_bits), which has no GRU to launch and stays with the fused kernel, would take half the time there (10
// types 13.4 / 7.6).
inline bool step_direct_small_fwd(int n_pad, int B, int H, int E) {
  const bool sizes = H == 64 ? B == 64 || B == 128 : H == 32 && B == 256;
  return sizes && n_pad / 32 <= 128 && E >= (B == 128 ? 5 : 7);
}

// 1-bit band: fused aggregate-first forward and transposed-band reverse.
inline hipError_t launch_step_fwd_bits(int dt, int n_pad, int B, int H, int E, const void* bits, const void* X,
                                       const void* W, const float* bias, float* a, hipStream_t st) {
  if (step_direct_no_wt(dt, n_pad, B, H, E))
    return GGNN_DT_PICK(launch_step_direct, false, n_pad, B, H, E, bits, X, W, nullptr, bias, a, nullptr, nullptr, 0,
                        st);
  return impl_bf16::launch_step_fwd_bits(n_pad, B, H, E, bits, X, W, bias, a, st);
}
inline hipError_t launch_banded_bwd_bits(int dt, int n_pad, int B, int H, int E, const void* bits_t, const void* da,
                                         void* dM, long ldm, hipStream_t st) {
  return GGNN_DT_PICK(launch_banded_bwd_bits, n_pad, B, H, E, bits_t, da, dM, ldm, st);
}
// Forward step with the GRU update fused in where the shape allows (sets
// *fused; otherwise only `a` is written and the caller runs the GRU).
// Wt (W_e^T, optional) lets the direct-weight forms read their weight
// fragments as 16-byte rows instead of 2-byte column gathers.
//
// Wide shapes (bf16, H = 128 or 256, B = 128..512) run the sliced wide step
// kernel instead (forward: only when Wt is given); the GRU then runs in its
// own kernel.
inline bool step_wide(int dt, int B, int H) { return dt == GGNN_BF16 && impl_bf16::step_wide_applies(B, H); }
inline hipError_t launch_step_fwd_bits_gru(int dt, int n_pad, int B, int H, int E, const void* bits, const void* X,
                                           const void* W, const void* Wt, const float* bias, float* a,
                                           const void* Wi, const void* U, const float* bg, void* h_out, void* saved,
                                           bool* fused, hipStream_t st) {
  if (step_direct_small_fwd(n_pad, B, H, E) ||
      (Wt == nullptr ? step_direct_no_wt(dt, n_pad, B, H, E) : step_direct(dt, n_pad, B, H, false))) {
    if (fused) *fused = false;
    return GGNN_DT_PICK(launch_step_direct, false, n_pad, B, H, E, bits, X, W, Wt, bias, a, nullptr, nullptr, 0, st);
  }
  if (Wt != nullptr && step_wide(dt, B, H)) {
    if (fused) *fused = false;
    return impl_bf16::launch_step_wide(false, n_pad, B, H, E, bits, X, Wt, bias, a, nullptr, nullptr, 0, st);
  }
  return impl_bf16::launch_step_fwd_bits_gru(n_pad, B, H, E, bits, X, W, Wt, bias, a, Wi, U, bg, h_out, saved, fused,
                                             st);
}
// Wt[e][o][h] = W[e][h][o].
inline hipError_t launch_transpose_weights(int dt, int H, int E, const void* W, void* Wt, hipStream_t st) {
  return GGNN_DT_PICK(launch_transpose_weights, H, E, W, Wt, st);
}
// Reverse step that continues, where the shape allows (sets *fused), with
// the previous step's GRU reverse on the completed dX: writes da_prev
// (feature-major), dh_prev and ghat_prev; dX_out may then be NULL.  When
// not fused, dX_out is written and the caller runs the GRU reverse.
inline hipError_t launch_step_bwd_bits_gru(int dt, int n_pad, int B, int H, int E, const void* bits_t, const void* da,
                                           const void* W, const float* dX_in, float* dX_out, void* dM, long ldm,
                                           const void* Wi, const void* U, const void* h_prev, const void* saved_prev,
                                           void* da_prev, float* dh_prev, void* ghat_prev, bool* fused,
                                           hipStream_t st) {
  if (dX_out != nullptr && step_direct(dt, n_pad, B, H, true) && !step_fused_small_rev(dt, n_pad, B, H, E)) {
    if (fused) *fused = false;
    return GGNN_DT_PICK(launch_step_direct, true, n_pad, B, H, E, bits_t, da, W, nullptr, nullptr, dX_out, dX_in, dM,
                        ldm, st);
  }
  if (dX_out != nullptr && step_wide(dt, B, H)) {
    if (fused) *fused = false;
    return impl_bf16::launch_step_wide(true, n_pad, B, H, E, bits_t, da, W, nullptr, dX_out, dX_in, dM, ldm, st);
  }
  return impl_bf16::launch_step_bwd_bits_gru(n_pad, B, H, E, bits_t, da, W, dX_in, dX_out, dM, ldm, Wi, U, h_prev,
                                             saved_prev, da_prev, dh_prev, ghat_prev, fused, st);
}
// Fused reverse step: dM_e = A_e^T da stored node-major (rows of type e start
// at row e * ldm of dM), dX_out = dX_in (or 0) + sum_e dM_e W_e^T.
inline hipError_t launch_step_bwd_bits(int dt, int n_pad, int B, int H, int E, const void* bits_t, const void* da,
                                       const void* W, const float* dX_in, float* dX_out, void* dM, long ldm,
                                       hipStream_t st) {
  if (step_direct(dt, n_pad, B, H, true))
    return GGNN_DT_PICK(launch_step_direct, true, n_pad, B, H, E, bits_t, da, W, nullptr, nullptr, dX_out, dX_in, dM,
                        ldm, st);
  if (step_wide(dt, B, H))
    return impl_bf16::launch_step_wide(true, n_pad, B, H, E, bits_t, da, W, nullptr, dX_out, dX_in, dM, ldm, st);
  return impl_bf16::launch_step_bwd_bits(n_pad, B, H, E, bits_t, da, W, dX_in, dX_out, dM, ldm, st);
}

inline hipError_t launch_transform_fwd(int dt, int n_pad, int H, int E, const void* X, const void* W,
                                       const float* bias, float* M, hipStream_t st) {
  return GGNN_DT_PICK(launch_transform_fwd, n_pad, H, E, X, W, bias, M, st);
}
// Input gradient dX_out = dX_in + sum_e dM_e W_e^T (dM rows of length ld).
inline hipError_t launch_transform_bwd_dx(int dt, int n_pad, int H, int E, const void* W, const void* dM, long ld,
                                          const float* dX_in, float* dX_out, hipStream_t st) {
  return GGNN_DT_PICK(launch_transform_bwd_dx, n_pad, H, E, W, dM, ld, dX_in, dX_out, st);
}
// Weight gradients over K rows: dW += X^T dM, dbias += row sums of dM (NULL
// to skip), X = K rows [K][H], dM rows of length ld >= K.  The workspace
// (transform_wgrad_workspace bytes) holds per-split partials, reduced in a
// fixed order.
size_t transform_wgrad_workspace(long K, int H, int E);
inline hipError_t launch_transform_wgrad(int dt, long K, int H, int E, const void* X, const void* dM, long ld,
                                         float* dW, float* dbias, void* ws, hipStream_t st) {
  return GGNN_DT_PICK(launch_transform_wgrad, K, H, E, X, dM, ld, dW, dbias, ws, st);
}
// The same with node-major dM: row k of type e at dM + (e * ldk + k) * H.
// With defer non-NULL the partial-sum reductions are appended to it instead
// of launched (launch_reduce_multi runs them together).
inline hipError_t launch_transform_wgrad_nm(int dt, long K, int H, int E, const void* X, const void* dM, long ldk,
                                            float* dW, float* dbias, void* ws, hipStream_t st,
                                            ReduceList* defer = nullptr) {
  return GGNN_DT_PICK(launch_transform_wgrad_nm, K, H, E, X, dM, ldk, dW, dbias, ws, defer, st);
}

// GRU weights packed in the fragment order of the large-H kernels (bf16,
// H >= 128): gru_pack_bytes is 0 where no kernel reads the packed form, and
// `packed` (NULL allowed) is then ignored by the launchers below.
size_t gru_pack_bytes(int dt, int H);
inline hipError_t launch_gru_pack(int dt, int H, const void* Wi, const void* U, void* packed, hipStream_t st) {
  return GGNN_DT_PICK(launch_gru_pack, H, Wi, U, packed, st);
}
inline hipError_t launch_gru_fwd(int dt, int n_pad, int H, const float* a, const void* h, const void* Wi,
                                 const void* U, const float* b, void* h_out, void* saved, hipStream_t st,
                                 const void* packed = nullptr) {
  return GGNN_DT_PICK(launch_gru_fwd, n_pad, H, a, h, Wi, U, b, h_out, saved, packed, st);
}
// Node pass of the GRU reverse: da, dh and the gate gradients G^ [n_pad][3H].
inline hipError_t launch_gru_bwd_nodes(int dt, int n_pad, int H, const float* dh_out, const void* h,
                                       const void* saved, const void* Wi, const void* U, void* da, float* dh,
                                       void* ghat, hipStream_t st, const void* packed = nullptr) {
  return GGNN_DT_PICK(launch_gru_bwd_nodes, n_pad, H, dh_out, h, saved, Wi, U, da, dh, ghat, packed, st);
}
size_t ghat_bytes(int dt, long rows, int H);
// GRU weight gradients over K rows of (a, h, saved, G^) stacked node-major:
// dWi, dU, db += (partials in ws of gru_wgrad_workspace bytes, fixed order).
size_t gru_wgrad_workspace(long K, int H);
inline hipError_t launch_gru_wgrad(int dt, long K, int H, const float* a, const void* h, const void* saved,
                                   const void* ghat, float* dWi, float* dU, float* db, void* ws, hipStream_t st,
                                   ReduceList* defer = nullptr) {
  return GGNN_DT_PICK(launch_gru_wgrad, K, H, a, h, saved, ghat, dWi, dU, db, ws, defer, st);
}
// One step: node pass with G^ in ws, then the weight gradients over n_pad rows.
size_t gru_bwd_workspace(int dt, int n_pad, int H);
hipError_t launch_gru_bwd(int dt, int n_pad, int H, const float* dh_out, const float* a, const void* h,
                          const void* saved, const void* Wi, const void* U, void* da, float* dh, float* dWi,
                          float* dU, float* db, void* ws, hipStream_t st);

// Readout and loss (candidate logits, per-graph softmax cross-entropy, mean
// over graphs) and their reverse: dX (written whole), dw_out and db_out
// (accumulated; partials in readout_bwd_workspace bytes, fixed order).
inline hipError_t launch_readout_loss(int dt, int H, int n_graphs, const void* X, const float* w_out,
                                      const float* b_out, const int32_t* cand_node, const int32_t* cand_ptr,
                                      const int32_t* target, float* logits, float* loss, float* dlogit,
                                      hipStream_t st) {
  return GGNN_DT_PICK(launch_readout_loss, H, n_graphs, X, w_out, b_out, cand_node, cand_ptr, target, logits, loss,
                      dlogit, st);
}
size_t readout_bwd_workspace(int H, int n_cand);
inline hipError_t launch_readout_bwd(int dt, int n_pad, int H, int n_cand, const void* X, const float* w_out,
                                     const int32_t* cand_node, const float* dlogit, float* dX, float* dw_out,
                                     float* db_out, void* ws, hipStream_t st) {
  return GGNN_DT_PICK(launch_readout_bwd, n_pad, H, n_cand, X, w_out, cand_node, dlogit, dX, dw_out, db_out, ws, st);
}
// Sparse aggregate-first step over receiver-major edge lists (every edge):
// a = sum_e (A_e X) W_e (+ deg_e b_e), W_e given transposed.
inline hipError_t launch_sparse_step(int dt, int n_pad, int H, int E, const int32_t* row_ptr, const int32_t* col,
                                     const void* X, const void* Wt, const float* bias, float* a, hipStream_t st) {
  return GGNN_DT_PICK(launch_sparse_step, n_pad, H, E, row_ptr, col, X, Wt, bias, a, st);
}
// Supernode slices (first s rows and columns), forward (a +=) and reverse
// (dX, dW, dbias +=); workspace of super_workspace bytes.
size_t super_workspace(int n_pad, int H, int E, int s);
// Workspace of the fused supernode steps (bf16, H = 32 or 64): the record
// (super_fused_record_floats floats, room for [P_e (32 x H) | deg_e (32)]),
// then the scratch of launch_super_long_fused (the per-chunk partials).
size_t super_fused_workspace(int n_pad, int H, int E);
size_t super_fused_record_floats(int H, int E);
inline hipError_t launch_super_fwd(int dt, int n_pad, int H, int E, int s, const void* rows, const void* cols,
                                   const void* X, const void* W, const float* bias, float* a, void* ws,
                                   hipStream_t st) {
  return GGNN_DT_PICK(launch_super_fwd, n_pad, H, E, s, rows, cols, X, W, bias, a, ws, st);
}
inline hipError_t launch_super_bwd(int dt, int n_pad, int H, int E, int s, const void* rows, const void* rows_t,
                                   const void* cols_t, const void* X, const void* W, const void* da, float* dX,
                                   float* dW, float* dbias, void* ws, hipStream_t st) {
  return GGNN_DT_PICK(launch_super_bwd, n_pad, H, E, s, rows, rows_t, cols_t, X, W, da, dX, dW, dbias, ws, st);
}
// Momentum update of float32 master parameters (and their compute copy).
hipError_t launch_sgd_momentum(long count, float* theta, float* vel, const float* grad, float lr, float mu, float wd,
                               int nesterov, int copy_dt, void* copy, hipStream_t st);

#undef GGNN_DT_PICK

}  // namespace ggnn
