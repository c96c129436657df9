// GRU node update (Eq. 1's GRU, Cho et al. 2014 form) and its reverse on
// gfx950 matrix cores, with the gate nonlinearities fused into the GEMM
// epilogues.
//
// Layouts: a [n_pad][H] float, h / h_out [n_pad][H] dt, Wi and U [H][3H] dt
// (columns r | z | n), b [3H] float, saved [n_pad][3H] dt (r | z | n),
// da [H][n_pad] dt feature-major, dh [n_pad][H] float.
//
// k order ("accumulator-compatible"): inside a 32-wide feature step kk, lane
// group g holds features 32kk + 4g + {0,1,2,3} and 32kk + 16 + 4g + {0,1,2,3}.
// These are exactly the features a lane holds in the accumulator of the two
// 16-feature output tiles 2kk and 2kk+1 (rows 4g + j), for the same node
// (lane % 16).  So a gate computed in registers is already an operand
// fragment of the next product: (r*h) U_n in the forward and every product of
// the backward chain without any cross-lane exchange.
#include "device_common.h"
#include "gru_wave.h"
#include "kernels.h"

namespace ggnn {
namespace dev {

// Stage the transpose of a 32-column slice of a [H][3H] weight into LDS:
// dst[f * PW + i] = src[i * 3H + col0 + f], f < 32, i < H.
template <typename S, int H, int PW, int NT>
__device__ __forceinline__ void stage_wT(S* dst, const S* src, int col0, int tid) {
  constexpr int V = 16 / sizeof(S);
  constexpr int UPR = 32 / V;  // 16-byte units per row slice
  for (int lin = tid; lin < H * UPR; lin += NT) {
    int i = lin / UPR, f0 = (lin % UPR) * V;
    u32x4 v = *reinterpret_cast<const u32x4*>(src + (size_t)i * 3 * H + col0 + f0);
    const S* pv = reinterpret_cast<const S*>(&v);
#pragma unroll
    for (int x = 0; x < V; ++x) dst[(f0 + x) * PW + i] = pv[x];
  }
}

// ---------------------------------------------------------------------------
// Forward in fp32.  Workgroup: 16*WAVES nodes, wave w: 16 nodes (lane % 16), all
// features.  D[feature][node]: A operand = weight^T rows from LDS, B operand
// = a / h / r*h fragments held in registers.  Phase A computes the reset
// gate for all features (needed in full by (r*h) U_n), phase B the update
// gate, the candidate and the new state, 32 features at a time.
// ---------------------------------------------------------------------------
template <int H, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void gru_fwd_kernel(const float* __restrict__ a, const float* __restrict__ h,
                                                                 const float* __restrict__ Wi, const float* __restrict__ U,
                                                                 const float* __restrict__ b, float* __restrict__ h_out,
                                                                 float* __restrict__ saved, int n_pad) {
  using S = float;
  constexpr int NT = WAVES * kWave;
  constexpr int V = 16 / sizeof(S);
  constexpr int PW = H + V;
  constexpr int KS = H / 32;
  __shared__ __attribute__((aligned(16))) S wt[4][32 * PW];

  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int q = lane % 16, g = lane / 16;
  const int n0 = xcd_swizzle(blockIdx.x, gridDim.x) * (16 * WAVES) + 16 * wave;
  const bool valid = n0 < n_pad;
  const int node = n0 + q;

  frag_t<S> af[KS], hf[KS], rh[KS];
  if (valid) {
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      const float* row = a + (size_t)node * H;
      f32x4 x = *reinterpret_cast<const f32x4*>(row + 32 * kk + 4 * g);
      f32x4 y = *reinterpret_cast<const f32x4*>(row + 32 * kk + 16 + 4 * g);
      const float v[8] = {x[0], x[1], x[2], x[3], y[0], y[1], y[2], y[3]};
      af[kk] = pack8<S>(v);
      hf[kk] = rowfrag<S>(h + (size_t)node * H, kk, g);
    }
  }
  auto afrag = [&](const S* t, int p, int kk) __attribute__((always_inline)) {
    return load4x2(t + (16 * p + q) * PW + 32 * kk + 4 * g, t + (16 * p + q) * PW + 32 * kk + 16 + 4 * g);
  };

  // Phase A: r = sigmoid(a Wi_r + h U_r + b_r); keep r*h as operand fragments.
  for (int c = 0; c < KS; ++c) {
    __syncthreads();
    stage_wT<S, H, PW, NT>(wt[0], Wi, 32 * c, tid);
    stage_wT<S, H, PW, NT>(wt[1], U, 32 * c, tid);
    __syncthreads();
    if (!valid) continue;
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        mma(acc[p], afrag(wt[0], p, kk), af[kk]);
        mma(acc[p], afrag(wt[1], p, kk), hf[kk]);
      }
    float rhv[8];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int f = 32 * c + 16 * p + 4 * g;
      float r[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        r[j] = sigmoidf_(acc[p][j] + b[f + j]);
        rhv[4 * p + j] = r[j] * static_cast<float>(hf[c][4 * p + j]);
      }
      if (saved) store4(saved + (size_t)node * 3 * H + f, r[0], r[1], r[2], r[3]);
    }
    rh[c] = pack8<S>(rhv);
  }
  // Phase B: z, n and the new state, 32 features at a time.
  for (int c = 0; c < KS; ++c) {
    __syncthreads();
    stage_wT<S, H, PW, NT>(wt[0], Wi, H + 32 * c, tid);
    stage_wT<S, H, PW, NT>(wt[1], U, H + 32 * c, tid);
    stage_wT<S, H, PW, NT>(wt[2], Wi, 2 * H + 32 * c, tid);
    stage_wT<S, H, PW, NT>(wt[3], U, 2 * H + 32 * c, tid);
    __syncthreads();
    if (!valid) continue;
    f32x4 az[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    f32x4 an[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        mma(az[p], afrag(wt[0], p, kk), af[kk]);
        mma(an[p], afrag(wt[2], p, kk), af[kk]);
        mma(az[p], afrag(wt[1], p, kk), hf[kk]);
        mma(an[p], afrag(wt[3], p, kk), rh[kk]);
      }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int f = 32 * c + 16 * p + 4 * g;
      float z[4], n[4], o[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        z[j] = sigmoidf_(az[p][j] + b[H + f + j]);
        n[j] = tanhf_(an[p][j] + b[2 * H + f + j]);
        const float hv = static_cast<float>(hf[c][4 * p + j]);
        o[j] = z[j] * hv + (1.f - z[j]) * n[j];
      }
      store4(h_out + (size_t)node * H + f, o[0], o[1], o[2], o[3]);
      if (saved) {
        store4(saved + (size_t)node * 3 * H + H + f, z[0], z[1], z[2], z[3]);
        store4(saved + (size_t)node * 3 * H + 2 * H + f, n[0], n[1], n[2], n[3]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Backward, per node (wave w: 16 nodes, lane % 16 = node): gru_bwd_wave.
// For H <= 64 the weights are staged once per workgroup in LDS (plain
// copies: the reverse products read rows of Wi and U, contiguous in the gate
// dimension); larger H reads their fragments from global memory (cached).
// `dh` may be `gin` (the reverse step that runs the GRU reverse as a launch of
// its own leaves the summed gradient where dh goes): every element is read and
// written by the same lane, and neither pointer is qualified as unaliased.
// ---------------------------------------------------------------------------
template <typename S, int H, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void gru_bwd_kernel(const float* gin, const S* __restrict__ h,
                                                                 const S* __restrict__ saved, const S* __restrict__ Wi,
                                                                 const S* __restrict__ U, S* __restrict__ daT,
                                                                 float* dh, S* __restrict__ ghat, int n_pad) {
  constexpr int MTL = H / 16;
  constexpr int NT = WAVES * kWave;
  constexpr int V = 16 / sizeof(S);
  constexpr bool LDSW = H <= 64;                       // weights fit in LDS
  __shared__ __attribute__((aligned(16))) S wl[LDSW ? 2 * 3 * H * H : 1];   // Wi, U in fragment order

  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int q = lane % 16, g = lane / 16;
  const int n0 = xcd_swizzle(blockIdx.x, gridDim.x) * (16 * WAVES) + 16 * wave;
  const bool valid = n0 < n_pad;
  const int node = n0 + q;

  // The node's inputs are loaded first, so that they are in flight while the
  // weights are staged (all of a thread's weight loads issued before its
  // LDS writes).
  f32x4 gg[MTL];
  GruBwdIn<S, H> in;
  if (valid) {
#pragma unroll
    for (int m = 0; m < MTL; ++m) gg[m] = *reinterpret_cast<const f32x4*>(gin + (size_t)node * H + 16 * m + 4 * g);
    in.load(saved, h, node, g);
  }
  if constexpr (LDSW) {
    constexpr int UNITS = 2 * H * (3 * H / V), ITS = (UNITS + NT - 1) / NT;
    u32x4 w[ITS];
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      const int lin = it * NT + tid;
      if (lin < UNITS) {
        const int mat = lin / (H * (3 * H / V)), rem = lin % (H * (3 * H / V));
        const int r = rem / (3 * H / V), c = (rem % (3 * H / V)) * V;
        w[it] = *reinterpret_cast<const u32x4*>((mat ? U : Wi) + (size_t)r * 3 * H + c);
      }
    }
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
      const int lin = it * NT + tid;
      if (lin < UNITS) {
        const int mat = lin / (H * (3 * H / V)), rem = lin % (H * (3 * H / V));
        const int r = rem / (3 * H / V), c = (rem % (3 * H / V)) * V;
        const S* pw = reinterpret_cast<const S*>(&w[it]);
#pragma unroll
        for (int i = 0; i < V; i += 4)
          put4<S>(wl, gru_rev_idx<S, H>(mat, r / 16, (c + i) / H, ((c + i) % H) / 32), r % 16, (c + i) % H, pw + i);
      }
    }
    __syncthreads();
  }
  if (!valid) return;   // no barrier follows
  if constexpr (LDSW) {
    auto wf = [&](int which, int row, int gate, int kk) __attribute__((always_inline)) {
      return load_fragi<S>(wl, gru_rev_idx<S, H>(which, row / 16, gate, kk), lane);
    };
    gru_bwd_wave<S, H>(gg, n0, q, g, in, wf, daT, n_pad, dh, ghat);
  } else {
    auto wf = [&](int which, int row, int gate, int kk) __attribute__((always_inline)) {
      return rowfrag<S>((which ? U : Wi) + (size_t)row * 3 * H + gate * H, kk, g);
    };
    gru_bwd_wave<S, H>(gg, n0, q, g, in, wf, daT, n_pad, dh, ghat);
  }
}

// ---------------------------------------------------------------------------
// Packed weights of the large-H kernels (H >= 128): lane vectors of eight
// elements (16 bytes) back to back in the order the kernels read them,
//   forward: fragment (feature group fw, matrix c of Wi_r, U_r, Wi_z, U_z,
//     Wi_n, U_n, k step kk, tile i), lane (qq, gg): gate column
//     32 fw + 2 qq + i at input rows 32 kk + 8 gg + {0..7};
//   reverse, after it: fragment (feature group fw, matrix c of U_n, Wi_r,
//     Wi_z, Wi_n, U_r, U_z, k step kk, tile i), lane (qq, gg): input row
//     32 fw + 2 qq + i at gate columns 32 kk + 8 gg + {0..7}.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int gru_pack_units(int H) { return 6 * H * H / 8; }   // per direction

template <typename S, int H>
__device__ __forceinline__ u32x4 gru_fwd_unit(const S* __restrict__ Wi, const S* __restrict__ U, int u) {
  constexpr int KS = H / 32;
  const int l = u % 64, i = (u / 64) % 2, kk = (u / 128) % KS, c = (u / (128 * KS)) % 6, fw = u / (128 * KS * 6);
  const S* src = (c % 2 ? U : Wi) + (size_t)(32 * kk + 8 * (l / 16)) * 3 * H + (c / 2) * H + 32 * fw + 2 * (l % 16) + i;
  u32x4 w;
#pragma unroll
  for (int d = 0; d < 4; ++d)
    w[d] = static_cast<uint32_t>(src[(size_t)(2 * d) * 3 * H]) |
           (static_cast<uint32_t>(src[(size_t)(2 * d + 1) * 3 * H]) << 16);
  return w;
}

template <typename S, int H>
__device__ __forceinline__ u32x4 gru_rev_unit(const S* __restrict__ Wi, const S* __restrict__ U, int u) {
  constexpr int KS = H / 32;
  const int l = u % 64, i = (u / 64) % 2, kk = (u / 128) % KS, c = (u / (128 * KS)) % 6, fw = u / (128 * KS * 6);
  const int gate = c == 0 ? 2 : (c <= 3 ? c - 1 : c - 4);
  const S* src = c >= 1 && c <= 3 ? Wi : U;
  return *reinterpret_cast<const u32x4*>(src + (size_t)(32 * fw + 2 * (l % 16) + i) * 3 * H + gate * H + 32 * kk +
                                         8 * (l / 16));
}

// One thread per unit: forward region, then reverse region.
template <typename S, int H>
__global__ __launch_bounds__(256) void gru_pack_kernel(const S* __restrict__ Wi, const S* __restrict__ U,
                                                       S* __restrict__ out) {
  constexpr int UNITS = gru_pack_units(H);
  const int u = blockIdx.x * 256 + threadIdx.x;
  if (u >= 2 * UNITS) return;
  const u32x4 v = u < UNITS ? gru_fwd_unit<S, H>(Wi, U, u) : gru_rev_unit<S, H>(Wi, U, u - UNITS);
  *reinterpret_cast<u32x4*>(out + (size_t)u * 8) = v;
}


// ---------------------------------------------------------------------------
// Forward in bf16, one wave per 32 state features: a workgroup of H / 32 x NW
// waves holds 16 NTL NW nodes, wave (fw, nw) the three gates' columns of
// features 32 fw .. 32 fw + 31 for the 16 NTL nodes of group nw.  A wave per
// 16 nodes instead (all features, the weights staged in LDS) reads every
// weight from LDS for one or two products and gathers unpacked weights in
// 2-byte pieces.  Here the nodes' operands (a as hi + lo, h, later r*h) sit in
// LDS in fragment order, read by the H / 32 feature waves, and a wave's
// weights come straight from global memory (L2), read once per workgroup, one k step
// ahead of use: a k step reads three fragments per 16 nodes for 16 products
// (r, z and the a part of n together); r*h then adds its share of n in a
// second, short loop.  Measured: 131,072 nodes at H = 256, unpacked weights,
// 298 -> 244 us per launch (packed, 262,144 nodes: 433 -> 410), 65,536 nodes
// at H = 128 46 -> 36 us, 100,096 nodes at H = 64 35 -> 26 us; 2,048 nodes at
// H = 256 58 -> 15 us.  Bound by the phases of a workgroup (staging, products,
// nonlinearities), of which one runs at a time at H = 256, where the operands
// take 131 KB of LDS.
//
// Feature order: the two 16-column tiles of a wave interleave, tile i, row m
// is feature 2 m + i of the wave's 32, so that a weight dword (two consecutive
// columns) holds an element of each tile, and a lane's accumulators of both
// tiles are the eight consecutive features 8 g .. 8 g + 7 of its node: the
// operands of the next product and 16-byte stores without lane exchanges.
// k order: lane group g holds features 32 kk + 8 g + {0..7}.
// ---------------------------------------------------------------------------
// Buffer resource over `elems` 16-bit elements (loads through it take a
// lane offset plus a uniform one, without 64-bit address arithmetic).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const bf16s* p, int elems) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16s*>(p), 0, elems * 2, 0x00027000);
}

template <int H, int NTL, int NW, bool PK>
__global__ __launch_bounds__(H / 32 * NW * kWave) void gru_fwd_cols_kernel(
    const float* __restrict__ a, const bf16s* __restrict__ h, const bf16s* __restrict__ Wi,
    const bf16s* __restrict__ U, const bf16s* __restrict__ pk, const float* __restrict__ b,
    bf16s* __restrict__ h_out, bf16s* __restrict__ saved, int n_pad) {
  constexpr int KS = H / 32, FW = H / 32, TILES = NTL * NW;
  __shared__ __attribute__((aligned(16))) bf16s fr[4][TILES][KS][kWave * 8];   // a hi, a lo, h, r*h
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int q = lane % 16, g = lane / 16;
  const int fw = wave % FW, nw = wave / FW;
  const int n0 = xcd_swizzle(blockIdx.x, gridDim.x) * 16 * TILES;

  // Weights of k step kk, matrix c of (Wi_r, U_r, Wi_z, U_z, Wi_n, U_n): the two tiles' fragments from the packed
  // copy, or eight dwords of gate columns 32 fw + 2 q, + 1 at input features 32 kk + 8 g + {0..7}.
  const auto rp = buffer_of(PK ? pk : Wi, PK ? 6 * H * H : 3 * H * H);
  const auto ru = buffer_of(U, 3 * H * H);
  const int woff = PK ? fw * 6 * KS * 2048 + lane * 16 : (8 * g * 3 * H + 32 * fw + 2 * q) * 2;
  auto load_w = [&](int c, int kk, uint32_t (&w)[8]) __attribute__((always_inline)) {
    if constexpr (PK) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rp, woff, ((c * KS + kk) * 2 + i) * 1024, 0);
#pragma unroll
        for (int d = 0; d < 4; ++d) w[4 * i + d] = v[d];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        w[e] = __builtin_amdgcn_raw_buffer_load_b32(c % 2 ? ru : rp, woff, ((32 * kk + e) * 3 * H + (c / 2) * H) * 2, 0);
    }
  };
  auto frag = [&](const uint32_t (&w)[8], int i) __attribute__((always_inline)) {
    u32x4 v;
#pragma unroll
    for (int d = 0; d < 4; ++d)
      v[d] = PK ? w[4 * i + d] : __builtin_amdgcn_perm(w[2 * d + 1], w[2 * d], i ? 0x07060302u : 0x05040100u);
    return __builtin_bit_cast(bf16x8, v);
  };

  auto state8 = [&](int t, float (&v)[8]) __attribute__((always_inline)) {
    const u32x4 s8 = *reinterpret_cast<const u32x4*>(&fr[2][nw * NTL + t][fw][lane * 8]);
#pragma unroll
    for (int d = 0; d < 4; ++d) v[2 * d] = lo_f(s8[d]), v[2 * d + 1] = hi_f(s8[d]);
  };
  auto frag_of = [&](int arr, int t, int kk) __attribute__((always_inline)) {
    return load8(&fr[arr][nw * NTL + t][kk][lane * 8]);
  };

  // Operand fragments of the nodes, NTL per wave: unit u = node tile u / KS, k step u % KS (a tile past the end
  // repeats the last one; its results are not stored).
  {
    f32x4 x[NTL], y[NTL];
    u32x4 hv[NTL];
#pragma unroll
    for (int j = 0; j < NTL; ++j) {
      const int u = wave * NTL + j, tile = min(n0 + 16 * (u / KS), n_pad - 16);
      const size_t at = (size_t)(tile + q) * H + 32 * (u % KS) + 8 * g;
      x[j] = *reinterpret_cast<const f32x4*>(a + at);
      y[j] = *reinterpret_cast<const f32x4*>(a + at + 4);
      hv[j] = *reinterpret_cast<const u32x4*>(h + at);
    }
#pragma unroll
    for (int j = 0; j < NTL; ++j) {
      const int u = wave * NTL + j, t = u / KS, kk = u % KS;
      const float v[8] = {x[j][0], x[j][1], x[j][2], x[j][3], y[j][0], y[j][1], y[j][2], y[j][3]};
      bf16x8 hi, lo;
      split8(v, hi, lo);
      *reinterpret_cast<bf16x8*>(&fr[0][t][kk][lane * 8]) = hi;
      *reinterpret_cast<bf16x8*>(&fr[1][t][kk][lane * 8]) = lo;
      *reinterpret_cast<u32x4*>(&fr[2][t][kk][lane * 8]) = hv[j];
    }
  }
  uint32_t w[2][5][8], un[2][8];   // of a k step: Wi_r, U_r, Wi_z, U_z, Wi_n; U_n
#pragma unroll
  for (int c = 0; c < 5; ++c) load_w(c, 0, w[0][c]);

  // The lane's eight features: 32 fw + 8 g + e, e = 2 j + i (tile i, accumulator element j).  The sums start from
  // the bias.
  const int fe = 32 * fw + 8 * g;
  f32x4 acc[3][2][NTL];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const f32x4 lo = *reinterpret_cast<const f32x4*>(b + c * H + fe),
                hi = *reinterpret_cast<const f32x4*>(b + c * H + fe + 4);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < NTL; ++t) acc[c][i][t] = f32x4{lo[i], lo[2 + i], hi[i], hi[2 + i]};
  }
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    if (kk + 1 < KS) {
#pragma unroll
      for (int c = 0; c < 5; ++c) load_w(c, kk + 1, w[(kk + 1) & 1][c]);
    } else {
      load_w(5, 0, un[0]);
    }
    bf16x8 f[5][2];
#pragma unroll
    for (int c = 0; c < 5; ++c)
#pragma unroll
      for (int i = 0; i < 2; ++i) f[c][i] = frag(w[kk & 1][c], i);
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      const bf16x8 ah = frag_of(0, t, kk), al = frag_of(1, t, kk), hf = frag_of(2, t, kk);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        mma(acc[0][i][t], f[0][i], ah);
        mma(acc[1][i][t], f[2][i], ah);
        mma(acc[2][i][t], f[4][i], ah);
        mma(acc[0][i][t], f[0][i], al);
        mma(acc[1][i][t], f[2][i], al);
        mma(acc[2][i][t], f[4][i], al);
        mma(acc[0][i][t], f[1][i], hf);
        mma(acc[1][i][t], f[3][i], hf);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    const int tile = n0 + 16 * (nw * NTL + t);
    float hs[8], r[8], rh[8];
    state8(t, hs);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      r[e] = sigmoidf_(acc[0][e & 1][t][e >> 1]);
      rh[e] = r[e] * hs[e];
    }
    *reinterpret_cast<bf16x8*>(&fr[3][nw * NTL + t][fw][lane * 8]) = pack8<bf16s>(rh);
    if (saved && tile < n_pad)
      *reinterpret_cast<bf16x8*>(saved + (size_t)(tile + q) * 3 * H + fe) = pack8<bf16s>(r);
  }
  __syncthreads();
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    if (kk + 1 < KS) load_w(5, kk + 1, un[(kk + 1) & 1]);
    const bf16x8 f0 = frag(un[kk & 1], 0), f1 = frag(un[kk & 1], 1);
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      const bf16x8 rh = frag_of(3, t, kk);
      mma(acc[2][0][t], f0, rh);
      mma(acc[2][1][t], f1, rh);
    }
  }
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    const int tile = n0 + 16 * (nw * NTL + t);
    if (tile >= n_pad) continue;
    float hs[8], z[8], n[8], o[8];
    state8(t, hs);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      z[e] = sigmoidf_(acc[1][e & 1][t][e >> 1]);
      n[e] = tanhf_(acc[2][e & 1][t][e >> 1]);
      o[e] = __builtin_fmaf(z[e], hs[e] - n[e], n[e]);   // z h + (1 - z) n
    }
    const size_t node = tile + q;
    *reinterpret_cast<bf16x8*>(h_out + node * H + fe) = pack8<bf16s>(o);
    if (saved) {
      *reinterpret_cast<bf16x8*>(saved + node * 3 * H + H + fe) = pack8<bf16s>(z);
      *reinterpret_cast<bf16x8*>(saved + node * 3 * H + 2 * H + fe) = pack8<bf16s>(n);
    }
  }
}

// ---------------------------------------------------------------------------
// Reverse in bf16 for H >= 128, the arithmetic of gru_bwd_wave in the form of
// gru_fwd_cols_kernel: one wave per 32 input features for the workgroup's
// 16 NTL nodes, G^ = [r^ z^ n^] of the nodes in LDS in fragment order, read by
// the H / 32 feature waves, the weight rows straight from L2 (16-byte pieces
// of 32 consecutive gate columns; or the packed fragments), each read once per
// workgroup, one k step ahead of use.
//   1: n^, z^ and g' z of the wave's features (the lane's eight);
//   2: q' = n^ U_n^T, hence r^ and the q' r term of dh;
//   3: da = G^ Wi^T as D[node][feature], dh += r^ U_r^T + z^ U_z^T.
// Two consecutive node tiles interleave in fours (tile t, row m is node
// 32 (t / 2) + 8 (m / 4) + 4 (t % 2) + m % 4), so that a lane holds eight
// consecutive nodes of da's feature rows: 16-byte stores.  `dh` may be `gin`
// (every element is read and written by the same lane).  Against one wave per
// 16 nodes with the weights streamed through LDS, per launch: 12,352 nodes at
// H = 128 20 -> 13 us, 65,536 at H = 128 57 -> 51 us, 262,144 at H = 256
// 547 -> 523 us; 24 bytes per node and feature stream in about 320 us there.
// ---------------------------------------------------------------------------
template <int H, int NTL, bool PK>
__global__ __launch_bounds__(H / 32 * kWave) void gru_bwd_cols_kernel(
    const float* gin, const bf16s* __restrict__ h, const bf16s* __restrict__ saved, const bf16s* __restrict__ Wi,
    const bf16s* __restrict__ U, const bf16s* __restrict__ pk, bf16s* __restrict__ daT, float* dh,
    bf16s* __restrict__ ghat, int n_pad) {
  constexpr int KS = H / 32;
  static_assert(NTL % 2 == 0, "node tiles come in pairs");
  __shared__ __attribute__((aligned(16))) bf16s fr[3][NTL][KS][kWave * 8];   // r^, z^, n^
  const int tid = threadIdx.x, fw = tid / kWave, lane = tid % kWave;
  const int q = lane % 16, g = lane / 16;
  const int n0 = xcd_swizzle(blockIdx.x, gridDim.x) * 16 * NTL;
  const int fe = 32 * fw + 8 * g;   // the lane's eight features: element e = 2 j + i (tile i, accumulator element j)

  // Weights of k step kk, matrix c of (U_n, Wi_r, Wi_z, Wi_n, U_r, U_z): rows 32 fw + 2 q + i, gate columns
  // 32 kk + 8 g + {0..7}.
  const auto rp = buffer_of(PK ? pk : Wi, 6 * H * H / (PK ? 1 : 2));
  const auto ru = buffer_of(U, 3 * H * H);
  const int woff = PK ? fw * 6 * KS * 2048 + lane * 16 : ((32 * fw + 2 * q) * 3 * H + 8 * g) * 2;
  auto load_w = [&](int c, int kk, bf16x8 (&w)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      u32x4 v;
      if constexpr (PK) {
        v = __builtin_amdgcn_raw_buffer_load_b128(rp, woff, ((c * KS + kk) * 2 + i) * 1024, 0);
      } else {
        const int gate = c == 0 ? 2 : (c <= 3 ? c - 1 : c - 4);
        v = __builtin_amdgcn_raw_buffer_load_b128(c >= 1 && c <= 3 ? rp : ru, woff,
                                                  (i * 3 * H + gate * H + 32 * kk) * 2, 0);
      }
      w[i] = __builtin_bit_cast(bf16x8, v);
    }
  };
  auto node_of = [&](int t) __attribute__((always_inline)) {
    return n0 + 32 * (t / 2) + 8 * (q / 4) + 4 * (t % 2) + q % 4;
  };
  auto unpack8 = [&](const u32x4& v, float (&o)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int d = 0; d < 4; ++d) o[2 * d] = lo_f(v[d]), o[2 * d + 1] = hi_f(v[d]);
  };

  f32x4 acc[2][NTL];      // dh
  u32x4 rraw[NTL], hraw[NTL];
  bf16x8 w[2][2];
  load_w(0, 0, w[0]);
#pragma unroll
  for (int t = 0; t < NTL; ++t) {
    const int node = min(node_of(t), n_pad - 1);   // past the end: a valid row whose results are not stored
    const f32x4 g0 = *reinterpret_cast<const f32x4*>(gin + (size_t)node * H + fe),
                g1 = *reinterpret_cast<const f32x4*>(gin + (size_t)node * H + fe + 4);
    const bf16s* sv = saved + (size_t)node * 3 * H + fe;
    rraw[t] = *reinterpret_cast<const u32x4*>(sv);
    const u32x4 zr = *reinterpret_cast<const u32x4*>(sv + H), nr = *reinterpret_cast<const u32x4*>(sv + 2 * H);
    hraw[t] = *reinterpret_cast<const u32x4*>(h + (size_t)node * H + fe);
    float z[8], n[8], hv[8], zh[8], nh[8];
    unpack8(zr, z);
    unpack8(nr, n);
    unpack8(hraw[t], hv);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float gg = e < 4 ? g0[e % 4] : g1[e % 4];
      const float dn = gg * (1.f - z[e]), dz = gg * (hv[e] - n[e]);
      acc[e & 1][t][e >> 1] = gg * z[e];
      nh[e] = dn * (1.f - n[e] * n[e]);
      zh[e] = dz * z[e] * (1.f - z[e]);
    }
    const bf16x8 pz = pack8<bf16s>(zh), pn = pack8<bf16s>(nh);
    *reinterpret_cast<bf16x8*>(&fr[1][t][fw][lane * 8]) = pz;
    *reinterpret_cast<bf16x8*>(&fr[2][t][fw][lane * 8]) = pn;
    if (node_of(t) < n_pad) {
      *reinterpret_cast<bf16x8*>(ghat + (size_t)node * 3 * H + H + fe) = pz;
      *reinterpret_cast<bf16x8*>(ghat + (size_t)node * 3 * H + 2 * H + fe) = pn;
    }
  }
  __syncthreads();
  auto frag_of = [&](int arr, int t, int kk) __attribute__((always_inline)) {
    return load8(&fr[arr][t][kk][lane * 8]);
  };
  bf16x8 w3[2][5][2];
  {
    f32x4 qa[2][NTL];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int t = 0; t < NTL; ++t) qa[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      if (kk + 1 < KS) {
        load_w(0, kk + 1, w[(kk + 1) & 1]);
      } else {
#pragma unroll
        for (int c = 0; c < 5; ++c) load_w(1 + c, 0, w3[0][c]);
      }
#pragma unroll
      for (int t = 0; t < NTL; ++t) {
        const bf16x8 f = frag_of(2, t, kk);
#pragma unroll
        for (int i = 0; i < 2; ++i) mma(qa[i][t], w[kk & 1][i], f);
      }
    }
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      float r[8], hv[8], rh[8];
      unpack8(rraw[t], r);
      unpack8(hraw[t], hv);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float qq = qa[e & 1][t][e >> 1];
        rh[e] = qq * hv[e] * r[e] * (1.f - r[e]);
        acc[e & 1][t][e >> 1] += qq * r[e];
      }
      const bf16x8 pr = pack8<bf16s>(rh);
      *reinterpret_cast<bf16x8*>(&fr[0][t][fw][lane * 8]) = pr;
      if (node_of(t) < n_pad) *reinterpret_cast<bf16x8*>(ghat + (size_t)node_of(t) * 3 * H + fe) = pr;
    }
  }
  __syncthreads();
  f32x4 da[2][NTL];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int t = 0; t < NTL; ++t) da[i][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) {
    if (kk + 1 < KS) {
#pragma unroll
      for (int c = 0; c < 5; ++c) load_w(1 + c, kk + 1, w3[(kk + 1) & 1][c]);
    }
#pragma unroll
    for (int t = 0; t < NTL; ++t) {
      const bf16x8 f[3] = {frag_of(0, t, kk), frag_of(1, t, kk), frag_of(2, t, kk)};
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          mma(da[i][t], f[c], w3[kk & 1][c][i]);
          if (c < 2) mma(acc[i][t], w3[kk & 1][3 + c][i], f[c]);
        }
    }
  }
#pragma unroll
  for (int t = 0; t < NTL; t += 2) {
    if (n0 + 16 * t >= n_pad) continue;   // n_pad is a multiple of 32: the pair is in or out
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float v[8] = {da[i][t][0], da[i][t][1], da[i][t][2], da[i][t][3],
                          da[i][t + 1][0], da[i][t + 1][1], da[i][t + 1][2], da[i][t + 1][3]};
      *reinterpret_cast<bf16x8*>(daT + (size_t)(32 * fw + 2 * q + i) * n_pad + n0 + 16 * t + 8 * g) = pack8<bf16s>(v);
    }
#pragma unroll
    for (int u = t; u < t + 2; ++u) {
      float* row = dh + (size_t)node_of(u) * H + fe;
      *reinterpret_cast<f32x4*>(row) = f32x4{acc[0][u][0], acc[1][u][0], acc[0][u][1], acc[1][u][1]};
      *reinterpret_cast<f32x4*>(row + 4) = f32x4{acc[0][u][2], acc[1][u][2], acc[0][u][3], acc[1][u][3]};
    }
  }
}

// ---------------------------------------------------------------------------
// Weight gradients of the GRU over one split of the rows k:
//   P[split][0][i][c] = sum_k a[k][i] G^[k][c]          (dWi)
//   P[split][1][i][c] = sum_k x_c[k][i] G^[k][c]        (dU)
// with x_c = h for the r and z columns and r*h for the n columns, and
//   Pb[split][c] = sum_k G^[k][c]                       (db).
// The rows are the nodes of all T steps at once (K = T * n_pad: a, h, saved
// and G^ stacked over t).  A workgroup owns one split of the rows and a
// slice of IT input features (all of them up to H = 64), every gate column:
// each input row is read once.  Per chunk of KC rows the operands are
// staged node-major in LDS (plain 16-byte copies; a rounded to bf16, r*h
// formed on the way) and read as matrix-core fragments with transposing
// LDS reads; the next chunk's loads are in flight during the products.
// Wave w: matrix w / 4 (dWi or dU) and a quarter of that matrix's tiles.
// ---------------------------------------------------------------------------
#ifndef GGNN_GRU_WGRAD_KC64
#define GGNN_GRU_WGRAD_KC64 64
#endif
#ifndef GGNN_GRU_WGRAD_MAXBUF
#define GGNN_GRU_WGRAD_MAXBUF 2
#endif
template <typename S, int H> struct GruWgradCfg {
  // input features per workgroup: each slice re-reads G^ (3H per row), so
  // slices are as wide as the accumulators allow
  static constexpr int IT = (H >= 256 && sizeof(S) == 2) ? 32 : (H >= 128 ? 4096 / H : H);
  static constexpr int NI = IT / 16, NCT = 3 * H / 16;  // tiles: input, gate columns
  static constexpr int KC = (sizeof(S) == 4 || H >= 256) ? 32 : (H >= 128 ? 64 : (H == 64 ? GGNN_GRU_WGRAD_KC64 : 128));   // rows per chunk
  static constexpr int IW = H == 32 ? 1 : NI;            // input tiles per wave
  static constexpr int CW = H == 32 ? 3 : NCT / 4;       // gate-column tiles per wave
  static constexpr int PA = IT + 16, PG = 3 * H + 16;    // LDS row pitches (elements)
  // LDS buffers: two (the next chunk is written while the current one is
  // read) when they fit in 160 KB.
  static constexpr int NBUF = GGNN_GRU_WGRAD_MAXBUF >= 2 && 2 * KC * (3 * PA + PG) * (int)sizeof(S) <= 160 * 1024 ? 2 : 1;
};

template <typename S, int H>
__global__ __launch_bounds__(512) void gru_wgrad_kernel(const float* __restrict__ a, const S* __restrict__ h,
                                                        const S* __restrict__ saved, const S* __restrict__ ghat,
                                                        float* __restrict__ P, float* __restrict__ Pb, long K,
                                                        int rows_per_split) {
  using C = GruWgradCfg<S, H>;
  constexpr int IT = C::IT, KC = C::KC, IW = C::IW, CW = C::CW, PA = C::PA, PG = C::PG, NBUF = C::NBUF;
  constexpr int NT = 512;
  constexpr int V = 16 / sizeof(S);
  constexpr int NA = KC * IT / V, NG = KC * 3 * H / V;   // 16-byte units per chunk
  constexpr int UA = (NA + NT - 1) / NT, UG = (NG + NT - 1) / NT;
  __shared__ __attribute__((aligned(16))) S sa[NBUF][3][KC * PA];   // a, h, r*h
  __shared__ __attribute__((aligned(16))) S sg[NBUF][KC * PG];      // G^

  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int q = lane % 16, g = lane / 16;
  constexpr int NSL = H / IT;
  const int bid = xcd_swizzle(blockIdx.x, gridDim.x);
  const int sl = bid % NSL, split = bid / NSL;
  const int i0 = sl * IT;
  const long nlo = (long)split * rows_per_split;
  const long nhi = min(K, nlo + rows_per_split);
  const int mat = wave / 4, sub = wave % 4;
  const int it0 = H == 32 ? sub % 2 : 0;
  const int ct0 = H == 32 ? (sub / 2) * 3 : sub * CW;
  const bool do_bias = mat == 0 && sl == 0 && it0 == 0;

  f32x4 acc[IW][CW];
  float bsum[CW];
#pragma unroll
  for (int i = 0; i < IW; ++i)
#pragma unroll
    for (int c = 0; c < CW; ++c) acc[i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < CW; ++c) bsum[c] = 0.f;

  // Register stage of one chunk: per A unit the fp32 a (V values), h and r;
  // per G unit the 16 bytes of G^.
  f32x4 ra[UA][V / 4];
  u32x4 rh[UA], rr[UA], rg[UG];
  auto load_chunk = [&](long c0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      const int lin = u * NT + tid;
      const long row = c0 + lin / (IT / V);
      const int f = i0 + (lin % (IT / V)) * V;
      if ((NA % NT == 0 || lin < NA) && row < nhi) {
#pragma unroll
        for (int x = 0; x < V / 4; ++x) ra[u][x] = *reinterpret_cast<const f32x4*>(a + (size_t)row * H + f + 4 * x);
        rh[u] = *reinterpret_cast<const u32x4*>(h + (size_t)row * H + f);
        rr[u] = *reinterpret_cast<const u32x4*>(saved + (size_t)row * 3 * H + f);
      } else {   // rows past the split (a ragged last chunk) contribute zeros
#pragma unroll
        for (int x = 0; x < V / 4; ++x) ra[u][x] = f32x4{0.f, 0.f, 0.f, 0.f};
        rh[u] = u32x4{0u, 0u, 0u, 0u};
        rr[u] = u32x4{0u, 0u, 0u, 0u};
      }
    }
#pragma unroll
    for (int u = 0; u < UG; ++u) {
      const int lin = u * NT + tid;
      const long row = c0 + lin / (3 * H / V);
      const int c = (lin % (3 * H / V)) * V;
      rg[u] = ((NG % NT == 0 || lin < NG) && row < nhi)
                  ? *reinterpret_cast<const u32x4*>(ghat + (size_t)row * 3 * H + c)
                  : u32x4{0u, 0u, 0u, 0u};
    }
  };
  auto store_chunk = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < UA; ++u) {
      const int lin = u * NT + tid;
      if (NA % NT == 0 || lin < NA) {
        const int r = lin / (IT / V), f = (lin % (IT / V)) * V;
        const S* ph = reinterpret_cast<const S*>(&rh[u]);
        const S* pr = reinterpret_cast<const S*>(&rr[u]);
        float av[V], rhv[V];
#pragma unroll
        for (int x = 0; x < V; ++x) {
          av[x] = ra[u][x / 4][x % 4];
          rhv[x] = to_f<S>(ph[x]) * to_f<S>(pr[x]);
        }
        u32x4 wa, wr;
        if constexpr (sizeof(S) == 2) {
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            wa[x] = pk2(av[2 * x], av[2 * x + 1]);
            wr[x] = pk2(rhv[2 * x], rhv[2 * x + 1]);
          }
        } else {
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            wa[x] = __float_as_uint(av[x]);
            wr[x] = __float_as_uint(rhv[x]);
          }
        }
        *reinterpret_cast<u32x4*>(&sa[buf][0][r * PA + f]) = wa;
        *reinterpret_cast<u32x4*>(&sa[buf][1][r * PA + f]) = rh[u];
        *reinterpret_cast<u32x4*>(&sa[buf][2][r * PA + f]) = wr;
      }
    }
#pragma unroll
    for (int u = 0; u < UG; ++u) {
      const int lin = u * NT + tid;
      if (NG % NT == 0 || lin < NG) {
        const int r = lin / (3 * H / V), c = (lin % (3 * H / V)) * V;
        *reinterpret_cast<u32x4*>(&sg[buf][r * PG + c]) = rg[u];
      }
    }
  };

  // Splits start at multiples of KC rows; a last chunk that runs past the
  // split is zero-filled.
  if (nlo < nhi) load_chunk(nlo);
  int buf = 0;
  for (long c0 = nlo; c0 < nhi; c0 += KC, buf = NBUF == 2 ? buf ^ 1 : 0) {
    if (NBUF == 1 && c0 > nlo) __syncthreads();   // the previous chunk is fully read
    store_chunk(buf);
    __syncthreads();
    if (c0 + KC < nhi) load_chunk(c0 + KC);
#pragma unroll
    for (int k0 = 0; k0 < KC; k0 += 32) {
      frag_t<S> fa[IW][2];   // [.][0]: a (dWi) or h (dU r, z columns); [.][1]: r*h (dU n columns)
#pragma unroll
      for (int i = 0; i < IW; ++i) {
        const int n0 = 16 * (it0 + i);
        fa[i][0] = tr_frag(sa[buf][mat == 0 ? 0 : 1], PA, k0, n0, lane);
        if (mat == 1 && (ct0 + CW) * 16 > 2 * H) fa[i][1] = tr_frag(sa[buf][2], PA, k0, n0, lane);
      }
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const int ct = ct0 + c;
        const frag_t<S> fb = tr_frag(sg[buf], PG, k0, 16 * ct, lane);
        if (do_bias) {
#pragma unroll
          for (int x = 0; x < 8; ++x) bsum[c] += static_cast<float>(fb[x]);
        }
        const int src = (mat == 1 && 16 * ct >= 2 * H) ? 1 : 0;
#pragma unroll
        for (int i = 0; i < IW; ++i) mma(acc[i][c], src ? fa[i][1] : fa[i][0], fb);
      }
    }
  }
  // D[i = i0 + 16 (it0 + i) + 4g + j][c = 16 (ct0 + c) + q]
  float* out = P + ((size_t)split * 2 + mat) * H * 3 * H;
#pragma unroll
  for (int i = 0; i < IW; ++i)
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        out[(size_t)(i0 + 16 * (it0 + i) + 4 * g + j) * 3 * H + 16 * (ct0 + c) + q] = acc[i][c][j];
  if (do_bias) {
#pragma unroll
    for (int c = 0; c < CW; ++c) {
      float v = bsum[c];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (g == 0) Pb[(size_t)split * 3 * H + 16 * (ct0 + c) + q] = v;
    }
  }
}

}  // namespace dev

namespace {
// Row split of the weight-gradient contraction: about 256 workgroups (one
// per compute unit, 8 waves each) over splits x input-feature slices;
// splits are multiples of 128 rows.
struct Split {
  int nsplit, per;
};
#ifndef GGNN_GRU_WGRAD_WGS
#define GGNN_GRU_WGRAD_WGS 256
#endif
// At H = 256 in bf16 the contraction of csrc/wgrad_wide.hip runs instead:
// six output tiles per split, 144 KB of LDS per workgroup (one per compute
// unit), so 42 splits (252 workgroups) of a multiple of 32 rows.
#ifndef GGNN_GRU_WGRAD256_LDS
#define GGNN_GRU_WGRAD256_LDS 1
#endif
#ifndef GGNN_GRU_WGRAD_PACE
#define GGNN_GRU_WGRAD_PACE 1
#endif
bool gru_wgrad256(long K, int H, bool f32) { return GGNN_GRU_WGRAD256_LDS && H == 256 && !f32 && K % 32 == 0; }
Split gru_split(long K, int H, bool f32) {
  if (gru_wgrad256(K, H, f32)) {
    const long want = GGNN_GRU_WGRAD_WGS / 6;
    const long per = std::max(32L, ((K + want - 1) / want + 31) / 32 * 32);
    return {(int)((K + per - 1) / per), (int)per};
  }
  const long slices = (H >= 256 && !f32) ? H / 32 : (H >= 128 ? H / (4096 / H) : 1);
  const long want = GGNN_GRU_WGRAD_WGS / slices > 0 ? GGNN_GRU_WGRAD_WGS / slices : 1;
  long per = ((K + want - 1) / want + 127) / 128 * 128;
  return {(int)((K + per - 1) / per), (int)per};
}

template <typename S, int H>
constexpr bool gru_big() {
  return sizeof(S) == 2 && H >= 128;
}

template <typename S, int H>
hipError_t gru_pack_h(const void* Wi, const void* U, void* packed, hipStream_t st) {
  if constexpr (gru_big<S, H>()) {
    const int units = 2 * dev::gru_pack_units(H);
    hipLaunchKernelGGL((dev::gru_pack_kernel<S, H>), dim3((units + 255) / 256), dim3(256), 0, st,
                       static_cast<const S*>(Wi), static_cast<const S*>(U), static_cast<S*>(packed));
    return hipGetLastError();
  }
  return hipSuccess;   // no kernel reads the packed form
}

template <typename S, int H>
hipError_t gru_fwd_h(int n_pad, const float* a, const void* h, const void* Wi, const void* U, const float* b,
                     void* h_out, void* saved, const void* packed, hipStream_t st) {
  if constexpr (sizeof(S) == 2) {
    const S* pk = gru_big<S, H>() ? static_cast<const S*>(packed) : nullptr;
    constexpr int NW = H >= 128 ? 1 : 128 / H;
#define GGNN_GRU_COLS(NTL, PK)                                                                                 \
  hipLaunchKernelGGL((dev::gru_fwd_cols_kernel<H, NTL, NW, PK>), dim3((n_pad + 16 * NTL * NW - 1) / (16 * NTL * NW)), \
                     dim3(H / 32 * NW * 64), 0, st, a, static_cast<const S*>(h), static_cast<const S*>(Wi),     \
                     static_cast<const S*>(U), pk, b, static_cast<S*>(h_out), static_cast<S*>(saved), n_pad)
    // The fewest node tiles per wave that leave no compute unit two workgroups: 16, 32 or 64 nodes (times NW); above
    // that 64, so that the weights are read less often.  One / two / four tiles, us: H = 64, 8,192 nodes 4.9 / 5.8 /
    // 7.9, 16,384 7.3 / 6.5 / 8.6, 262,144 (nothing saved) 55 / 45 / 41; H = 32, 16,384 4.0 / 5.1 / 6.6, 32,768 5.7 /
    // 5.6 / 7.1; H = 128, 6,400 9.4 / 7.9 / 10.3, 16,384 15.0 / 11.3 / 10.2; H = 256, 2,048 14.9 / 17.5 / 23.1, 8,192
    // 28.5 / 20.0 / 25.5, 16,384 53 / 37 / 29.
    constexpr int one = 256 * 16 * NW;
    const int tiles = n_pad <= one ? 1 : (n_pad <= 2 * one ? 2 : 4);
#define GGNN_GRU_COLS_PICK(PK) \
  if (tiles == 1)              \
    GGNN_GRU_COLS(1, PK);      \
  else if (tiles == 2)         \
    GGNN_GRU_COLS(2, PK);      \
  else                         \
    GGNN_GRU_COLS(4, PK);
    if constexpr (gru_big<S, H>()) {
      if (pk != nullptr) {
        GGNN_GRU_COLS_PICK(true)
      } else {
        GGNN_GRU_COLS_PICK(false)
      }
    } else {
      GGNN_GRU_COLS_PICK(false)
    }
#undef GGNN_GRU_COLS_PICK
#undef GGNN_GRU_COLS
    return hipGetLastError();
  } else {
    constexpr int WAVES = 4;
    hipLaunchKernelGGL((dev::gru_fwd_kernel<H, WAVES>), dim3((n_pad + 16 * WAVES - 1) / (16 * WAVES)),
                       dim3(WAVES * 64), 0, st, a, static_cast<const float*>(h), static_cast<const float*>(Wi),
                       static_cast<const float*>(U), b, static_cast<float*>(h_out), static_cast<float*>(saved), n_pad);
    return hipGetLastError();
  }
}

template <typename S, int H>
hipError_t gru_bwd_nodes_h(int n_pad, const float* dh_out, const void* h, const void* saved, const void* Wi,
                           const void* U, void* da, float* dh, void* ghat, const void* packed, hipStream_t st) {
  if constexpr (gru_big<S, H>()) {
    // the reverse region follows the forward one
    const S* pk = packed ? static_cast<const S*>(packed) + (size_t)dev::gru_pack_units(H) * 8 : nullptr;
#define GGNN_GRU_BWD_COLS(NTL, PK)                                                                                \
  hipLaunchKernelGGL((dev::gru_bwd_cols_kernel<H, NTL, PK>), dim3((n_pad + 16 * NTL - 1) / (16 * NTL)),           \
                     dim3(H / 32 * 64), 0, st, dh_out, static_cast<const S*>(h), static_cast<const S*>(saved),    \
                     static_cast<const S*>(Wi), static_cast<const S*>(U), pk, static_cast<S*>(da), dh,            \
                     static_cast<S*>(ghat), n_pad)
    // 32 nodes per workgroup on small grids, else 64, so that the weights are read less often (whole reverse with
    // the weight gradients, H = 256: 70 us against 77 at 8,192 nodes, 104 against 84 at 12,352; H = 128: 29 / 31 and
    // 39 / 35).
    const bool small = n_pad <= 8192;
    if (small && pk != nullptr)
      GGNN_GRU_BWD_COLS(2, true);
    else if (small)
      GGNN_GRU_BWD_COLS(2, false);
    else if (pk != nullptr)
      GGNN_GRU_BWD_COLS(4, true);
    else
      GGNN_GRU_BWD_COLS(4, false);
#undef GGNN_GRU_BWD_COLS
    return hipGetLastError();
  } else {
    constexpr int WAVES = 4;
    hipLaunchKernelGGL((dev::gru_bwd_kernel<S, H, WAVES>), dim3((n_pad + 16 * WAVES - 1) / (16 * WAVES)),
                     dim3(WAVES * 64), 0, st, dh_out, static_cast<const S*>(h), static_cast<const S*>(saved),
                     static_cast<const S*>(Wi), static_cast<const S*>(U), static_cast<S*>(da), dh,
                     static_cast<S*>(ghat), n_pad);
    return hipGetLastError();
  }
}

template <typename S, int H>
hipError_t gru_wgrad_h(long K, const float* a, const void* h, const void* saved, const void* ghat, float* dWi,
                       float* dU, float* db, void* ws, ReduceList* defer, hipStream_t st) {
  Split sp = gru_split(K, H, sizeof(S) == 4);
  float* P = static_cast<float*>(ws);
  float* Pb = P + (size_t)sp.nsplit * 2 * H * 3 * H;
  hipError_t err;
  if (sizeof(S) == 2 && H == 256 && gru_wgrad256(K, H, false)) {
    int* prog = reinterpret_cast<int*>(Pb + (size_t)sp.nsplit * 3 * H);   // pacing counters
    err = launch_gru_wgrad256(sp.nsplit, sp.per, K, a, h, saved, ghat, P, Pb, GGNN_GRU_WGRAD_PACE ? prog : nullptr,
                              st);
  } else {
    const int blocks = sp.nsplit * (H / dev::GruWgradCfg<S, H>::IT);
    hipLaunchKernelGGL((dev::gru_wgrad_kernel<S, H>), dim3(blocks), dim3(512), 0, st, a,
                       static_cast<const S*>(h), static_cast<const S*>(saved), static_cast<const S*>(ghat), P, Pb,
                       K, sp.per);
    err = hipGetLastError();
  }
  if (err != hipSuccess) return err;
  const long slice = 2L * H * 3 * H;  // partials are [split][which][H][3H]
  err = reduce_or_defer(P, dWi, sp.nsplit, H * 3 * H, slice, defer, st);
  if (err != hipSuccess) return err;
  err = reduce_or_defer(P + (size_t)H * 3 * H, dU, sp.nsplit, H * 3 * H, slice, defer, st);
  if (err != hipSuccess) return err;
  return reduce_or_defer(Pb, db, sp.nsplit, 3 * H, 3L * H, defer, st);
}

#define GGNN_GRU_SWITCH(CALL)                  \
  switch (H) {                                 \
    case 32: { constexpr int HH = 32; CALL; }  \
    case 64: { constexpr int HH = 64; CALL; }  \
    case 128: { constexpr int HH = 128; CALL; } \
    case 256: { constexpr int HH = 256; CALL; } \
  }                                            \
  return hipErrorInvalidValue;

template <typename S>
hipError_t gru_pack_t(int H, const void* Wi, const void* U, void* packed, hipStream_t st) {
  GGNN_GRU_SWITCH(return (gru_pack_h<S, HH>(Wi, U, packed, st)))
}
template <typename S>
hipError_t gru_fwd_t(int n_pad, int H, const float* a, const void* h, const void* Wi, const void* U, const float* b,
                     void* h_out, void* saved, const void* packed, hipStream_t st) {
  GGNN_GRU_SWITCH(return (gru_fwd_h<S, HH>(n_pad, a, h, Wi, U, b, h_out, saved, packed, st)))
}
template <typename S>
hipError_t gru_bwd_nodes_t(int n_pad, int H, const float* dh_out, const void* h, const void* saved, const void* Wi,
                           const void* U, void* da, float* dh, void* ghat, const void* packed, hipStream_t st) {
  GGNN_GRU_SWITCH(return (gru_bwd_nodes_h<S, HH>(n_pad, dh_out, h, saved, Wi, U, da, dh, ghat, packed, st)))
}
template <typename S>
hipError_t gru_wgrad_t(long K, int H, const float* a, const void* h, const void* saved, const void* ghat, float* dWi,
                       float* dU, float* db, void* ws, ReduceList* defer, hipStream_t st) {
  GGNN_GRU_SWITCH(return (gru_wgrad_h<S, HH>(K, a, h, saved, ghat, dWi, dU, db, ws, defer, st)))
}
#undef GGNN_GRU_SWITCH
}  // namespace

#if GGNN_DT_BF16   // dtype-independent helpers: built once
size_t ghat_bytes(int dt, long rows, int H) {
  size_t b = (size_t)rows * 3 * H * (dt == GGNN_BF16 ? 2 : 4);
  return (b + 255) / 256 * 256;
}

size_t gru_wgrad_workspace(long K, int H) {
  // large enough for the split of either dtype
  Split sp = gru_split(K, H, false);
  const Split s32 = gru_split(K, H, true);
  if (s32.nsplit > sp.nsplit) sp = s32;
  // partials, bias partials, then 8 pacing counters per split (H = 256 bf16)
  return ((size_t)sp.nsplit * 2 * H * 3 * H + (size_t)sp.nsplit * 3 * H + (size_t)sp.nsplit * 8) * sizeof(float);
}

size_t gru_pack_bytes(int dt, int H) {
  return dt == GGNN_BF16 && H >= 128 ? (size_t)12 * H * H * 2 : 0;
}

size_t gru_bwd_workspace(int dt, int n_pad, int H) {
  return ghat_bytes(dt, n_pad, H) + gru_wgrad_workspace(n_pad, H);
}

hipError_t launch_gru_bwd(int dt, int n_pad, int H, const float* dh_out, const float* a, const void* h,
                          const void* saved, const void* Wi, const void* U, void* da, float* dh, float* dWi,
                          float* dU, float* db, void* ws, hipStream_t st) {
  void* ghat = ws;
  void* part = static_cast<char*>(ws) + ghat_bytes(dt, n_pad, H);
  hipError_t err = launch_gru_bwd_nodes(dt, n_pad, H, dh_out, h, saved, Wi, U, da, dh, ghat, st);
  if (err != hipSuccess) return err;
  ReduceList red;   // the partial sums of dWi, dU and db in one launch
  err = launch_gru_wgrad(dt, n_pad, H, a, h, saved, ghat, dWi, dU, db, part, st, &red);
  return err == hipSuccess ? launch_reduce_multi(red, st) : err;
}
#endif

namespace GGNN_IMPL_NS {
hipError_t launch_gru_pack(int H, const void* Wi, const void* U, void* packed, hipStream_t st) {
  return gru_pack_t<dev::dt_t>(H, Wi, U, packed, st);
}

hipError_t launch_gru_fwd(int n_pad, int H, const float* a, const void* h, const void* Wi, const void* U,
                          const float* b, void* h_out, void* saved, const void* packed, hipStream_t st) {
  return gru_fwd_t<dev::dt_t>(n_pad, H, a, h, Wi, U, b, h_out, saved, packed, st);
}

hipError_t launch_gru_bwd_nodes(int n_pad, int H, const float* dh_out, const void* h, const void* saved,
                                const void* Wi, const void* U, void* da, float* dh, void* ghat, const void* packed,
                                hipStream_t st) {
  return gru_bwd_nodes_t<dev::dt_t>(n_pad, H, dh_out, h, saved, Wi, U, da, dh, ghat, packed, st);
}

hipError_t launch_gru_wgrad(long K, int H, const float* a, const void* h, const void* saved, const void* ghat,
                            float* dWi, float* dU, float* db, void* ws, ReduceList* defer, hipStream_t st) {
  return gru_wgrad_t<dev::dt_t>(K, H, a, h, saved, ghat, dWi, dU, db, ws, defer, st);
}
}  // namespace GGNN_IMPL_NS

}  // namespace ggnn
