// Step on a 1-bit block band with the weights read straight from global memory: float32 (every size) and the bf16
// sizes that the other step kernels serve badly (small grids at H >= 128, blocks that do not fit in LDS whole at
// H <= 64), the products of the fused step of Eq. 3 in the operand order of Algorithm 1:
//   forward:  a[k]    = sum_e (sum_s bits[e][k][s] X[k-1+s]) W_e   (+ deg_e b_e)
//   reverse:  dM_e[k] = sum_s bits_t[e][k][s] da[k-1+s]            (stored)
//             dX[k]   = dX_in[k] + sum_e dM_e[k] W_e^T
//
// fp32: what bounds the aggregation is the matrix-core rate: an fp32 k step
// of 32 nodes takes eight v_mfma_f32_16x16x4_f32 of 32 cycles.  The band's
// entries are 0 or 1, exact in bf16, so the states are split instead, once,
// when they are staged: x = hi + mid + lo with bf16 parts (8 + 8 + 8
// significant bits, cut off, so the split is exact; below about 2^-110 the low
// part falls under the smallest bf16 subnormal, an error of less than 2^-133
// of a state), and a k step is three
// v_mfma_f32_16x16x32_bf16 of 16 cycles with float accumulation: the same
// sums of the same values at 5.3 times the rate.  The transform by W_e stays
// on the fp32 instructions: there both operands have 24 bits.
//
// bf16: the aggregate enters the transform as hi + lo (forward) or rounded as
// stored (reverse), as in the other step kernels.  On small grids those are
// bound by how few waves they start: the wide kernel shares every weight
// between a block's rows through LDS, at the price of a barrier per 32 weight
// rows and B / 32 waves per block.  Here a workgroup's waves take the
// edge types side by side and add their sums once at the end.
//
// The transform's contraction over features is split into slices of HQ
// features, (A_e X) W_e = sum_q (A_e X[:, q]) W_e[q, :]: per slice the three
// node blocks' parts (3 x 3 B x HQ bf16) are staged once in LDS and reused by
// every edge type, and the type loop has no barrier.
//
// Measured on 20,000 nodes, B = 128, H = 64, 10 types, per pass of two steps
// forward and reverse: 1055 -> 439 us against the fp32 form that staged
// 64-node chunks per type and multiplied them in fp32 (205 us per step launch
// there); the distance from a 64-bit reference 1.6e-6 -> 1.3e-6 of the norm
// (fewer roundings per sum).  Bound now by the transform's fp32 products.
// bf16, 12,352 nodes, B = 64, H = 128, 7 types: 60 -> 28 us per forward and
// 51 -> 25 us per reverse launch against the wide kernel, bound by the chain
// of a wave's types (bit rows, products, weights).
#include "band_frag.h"
#include "device_common.h"
#include "kernels.h"

namespace ggnn {
namespace dev {

template <typename S, int H, int B, int WAVES, int TG, int NTW_>
struct DirectCfg {
  static constexpr bool F32 = sizeof(S) == 4;
  static constexpr int PARTS = F32 ? 3 : 1;
  // Features per slice: as many as the parts of three blocks (in LDS) and the
  // slice's aggregate (in registers, next to the output sums) leave room for.
  static constexpr int HQF = B >= 512 ? 16 : (B >= 128 || H == 32 || H == 256 ? 32 : 64);
  static constexpr int HQB = B >= 512 || H == 32 ? 32 : (B >= 256 || H == 64 || H == 256 ? 64 : 128);
  static constexpr int HQ = F32 ? HQF : HQB;
  static constexpr int NQ = H / HQ, MQ = HQ / 16, MT = H / 16;
  static constexpr int NTW = NTW_, RPW = 16 * NTW;   // 16-row tiles and rows per wave
  static constexpr int R = WAVES * RPW, NT = TG * WAVES * kWave;
  static constexpr int RB = B / 32;              // bit-row bytes per lane and block (= k steps per block)
  // k order of a block's columns (as in the bf16 step kernels): contiguous
  // where a register transpose of the bit bytes exists (and trivially for one
  // byte), so that empty k steps can be skipped; else lane group g holds
  // columns g B/4 .. (g + 1) B/4 - 1.
  static constexpr bool KCONT = RB == 1 || RB == 4 || RB == 8;
  static constexpr int PLANE = 3 * B * HQ;       // elements of one part of the staged window
  // The groups' partial sums meet in LDS, one row tile at a time.
  static constexpr int RED = TG == 1 ? 0 : TG * WAVES * MT * 1024;
  static constexpr int LDS = PARTS * PLANE * 2 > RED ? PARTS * PLANE * 2 : RED;
  // The forward with W^T is a form of its own where the registers that gathering columns of W takes would be spilled.
  static constexpr bool WT_ARG = !F32 && H >= 128;
  // Output tiles whose weights are loaded together.
  static constexpr int GM = F32 ? (MQ >= 4 || H == 256 ? 2 : 4) : (HQ == 128 ? 2 : 4);
};

// x = hi + mid + lo, each with at most eight significant bits (the low words
// of the returned floats are zero); an infinite x is its own hi part.
__device__ __forceinline__ void split3(float x, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  hi = __float_as_uint(x) & 0xFFFF0000u;
  float r = x - __uint_as_float(hi);
  r = __builtin_isinf(x) ? 0.f : r;
  mid = __float_as_uint(r) & 0xFFFF0000u;
  lo = __float_as_uint(r - __uint_as_float(mid));
}
// Eight floats -> three bf16 fragments.
__device__ __forceinline__ void split3x8(const float (&v)[8], u32x4 (&o)[3]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t a[3], b[3];
    split3(v[2 * i], a[0], a[1], a[2]);
    split3(v[2 * i + 1], b[0], b[1], b[2]);
#pragma unroll
    for (int p = 0; p < 3; ++p) o[p][i] = __builtin_amdgcn_perm(b[p], a[p], 0x07060302u);   // the two high halves
  }
}

template <int NB> struct DirectBits {
  static constexpr int NW = NB < 4 ? 1 : NB / 4;
  uint32_t w[NW];
  __device__ __forceinline__ void load(const uint8_t* p) {
    if constexpr (NB == 1) {
      w[0] = *p;
    } else if constexpr (NB == 2) {
      w[0] = *reinterpret_cast<const uint16_t*>(p);
    } else {
#pragma unroll
      for (int i = 0; i < NW; ++i) w[i] = reinterpret_cast<const uint32_t*>(p)[i];
    }
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = 0u;
  }
  __device__ __forceinline__ uint32_t any() const {
    uint32_t a = 0u;
#pragma unroll
    for (int i = 0; i < NW; ++i) a |= w[i];
    return a;
  }
  __device__ __forceinline__ uint32_t byte(int i) const { return (w[i / 4] >> (8 * (i % 4))) & 0xFFu; }
  __device__ __forceinline__ int popc() const {
    int c = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) c += __popc(w[i]);
    return c;
  }
};

// Workgroup: R = 16 NTW WAVES rows of block row k, TG * WAVES waves; wave w takes
// R / WAVES of these rows and the edge types w / WAVES, w / WAVES + TG, ...
// (dealt round robin: with fewer types than groups, or one more than a
// multiple of them, the waves that have the most work are on different SIMDs;
// with contiguous ranges 2 types of 8 groups fell to waves 3 and 7, which
// share one).  V = X (forward, [n_pad][H]) or da (reverse, [H][n_pad]); W
// [E][H][H]; Wt = W_e^T or NULL (forward: rows of W_e^T, else columns of W;
// where the form WT says which, see DirectCfg).
template <typename S, int H, int B, int WAVES, int TG, int NTW_, bool REV, bool WT>
__global__ __launch_bounds__(TG * WAVES * kWave) void step_direct_kernel(
    const uint8_t* __restrict__ bits, const S* __restrict__ V, const S* __restrict__ W, const S* __restrict__ Wt,
    const float* __restrict__ bias, float* out, int n_pad, int E, const float* dX_in, S* __restrict__ dM, long ldm) {
  using C = DirectCfg<S, H, B, WAVES, TG, NTW_>;
  constexpr bool F32 = C::F32;
  constexpr int NT = C::NT, HQ = C::HQ, NQ = C::NQ, MQ = C::MQ, MT = C::MT, NTW = C::NTW, RB = C::RB, GM = C::GM;
  constexpr int ROWB = B / 8, TPR = B / C::R;
  static_assert(C::LDS <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(16))) char lds[C::LDS];
  bf16s* const xs = reinterpret_cast<bf16s*>(lds);   // [part][block s][fragment order]

  const int nb = n_pad / B;
  const int t = xcd_swizzle(blockIdx.x, gridDim.x);
  const int k = t / TPR;
  const int tid = threadIdx.x, lane = tid % kWave, wave = (tid / kWave) % WAVES, tg = tid / (WAVES * kWave);
  const int q = lane % 16, g = lane / 16;
  const int rw = (t % TPR) * C::R + C::RPW * wave;
  const int s_lo = (k == 0) ? 1 : 0, s_hi = (k == nb - 1) ? 1 : 2;

  auto load_bits = [&](int e, DirectBits<RB> (&dst)[3][NTW]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const uint8_t* p = bits + ((((size_t)e * nb + k) * 3 + s) * B + rw + q) * ROWB + g * RB;
#pragma unroll
      for (int n = 0; n < NTW; ++n) {
        if (s < s_lo || s > s_hi) {
          dst[s][n].zero();
        } else {
          dst[s][n].load(p + (size_t)16 * n * ROWB);
        }
      }
    }
  };

  // One slice of the three blocks, in fragment order.  fp32: a unit is eight
  // nodes of four features (forward: eight 16-byte row loads) or of one
  // feature (reverse), split into its parts.  bf16: an 8 x 8 tile transposed in registers (forward) or eight nodes of
  // one feature (reverse).
  auto at = [&](int s, int f, int c) __attribute__((always_inline)) {   // feature slot f, nodes c .. c + 7 of block s
    const int kk = C::KCONT ? c / 32 : (c % (B / 4)) / 8, gg = C::KCONT ? (c / 8) % 4 : c / (B / 4);
    return xs + s * B * HQ + fo<bf16s>(kk * MQ + f / 16, f % 16 + 16 * gg, 0);
  };
  auto stage = [&](int qs) __attribute__((always_inline)) {
    auto put = [&](int s, int f, int c, const float (&v)[8]) __attribute__((always_inline)) {
      u32x4 o[3];
      split3x8(v, o);
#pragma unroll
      for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4*>(at(s, f, c) + p * C::PLANE) = o[p];
    };
    if constexpr (F32 && !REV) {
      constexpr int UB = (B / 8) * (HQ / 4);
      for (int u = tid; u < 3 * UB; u += NT) {
        const int s = u / UB, r = u % UB, f0 = 4 * (r % (HQ / 4)), c = 8 * (r / (HQ / 4));
        if (s < s_lo || s > s_hi) continue;
        f32x4 x[8];
        const S* p = V + (size_t)((k - 1 + s) * B + c) * H + qs * HQ + f0;
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = *reinterpret_cast<const f32x4*>(p + (size_t)i * H);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float v[8] = {x[0][j], x[1][j], x[2][j], x[3][j], x[4][j], x[5][j], x[6][j], x[7][j]};
          put(s, f0 + j, c, v);
        }
      }
    } else if constexpr (F32) {
      constexpr int UB = (B / 8) * HQ;
      for (int u = tid; u < 3 * UB; u += NT) {
        const int s = u / UB, r = u % UB, f = 16 * (r / (16 * (B / 8))) + r % 16, c = 8 * ((r / 16) % (B / 8));
        if (s < s_lo || s > s_hi) continue;
        const S* p = V + (size_t)(qs * HQ + f) * n_pad + (k - 1 + s) * B + c;
        const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
        const float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
        put(s, f, c, v);
      }
    } else if constexpr (!REV) {
      constexpr int UB = (B / 8) * (HQ / 8);
      for (int u = tid; u < 3 * UB; u += NT) {
        // eight neighbouring lanes take eight node octets of one feature octet: their LDS writes fall on
        // different lane groups' pieces
        const int s = u / UB, r = u % UB, c = 8 * (r % (B / 8)), f0 = 8 * (r / (B / 8));
        if (s < s_lo || s > s_hi) continue;
        u32x4 x[8];
        tile_load<bf16s>(x, V + (size_t)((k - 1 + s) * B + c) * H + qs * HQ + f0, H);
#pragma unroll
        for (int j = 0; j < 8; ++j)
          *reinterpret_cast<u32x4*>(at(s, feature_slot(f0 + j), c)) = tile_row_T<bf16s>(x, j);
      }
    } else {
      constexpr int UB = (B / 8) * HQ;
      for (int u = tid; u < 3 * UB; u += NT) {
        const int s = u / UB, r = u % UB, f = 16 * (r / (16 * (B / 8))) + r % 16, c = 8 * ((r / 16) % (B / 8));
        if (s < s_lo || s > s_hi) continue;
        *reinterpret_cast<u32x4*>(at(s, feature_slot(f), c)) =
            *reinterpret_cast<const u32x4*>(V + (size_t)(qs * HQ + f) * n_pad + (k - 1 + s) * B + c);
      }
    }
  };

  f32x4 acc[NTW][MT];
#pragma unroll
  for (int n = 0; n < NTW; ++n)
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[n][m] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int qs = 0; qs < NQ; ++qs) {
    DirectBits<RB> cur[3][NTW], nxt[3][NTW];
    if (tg < E) load_bits(tg, cur);
    if (qs > 0) __syncthreads();   // every wave is done with the previous slice
    stage(qs);
    __syncthreads();
    for (int e = tg; e < E; e += TG) {
      if (e + TG < E) load_bits(e + TG, nxt);
      // Weight fragments of output tile mo (A operand: row = output feature
      // 16 mo + q; fp32: k = the slice's features 16 m + 4 g + {0..3}, bf16:
      // 32 kk + 8 g + {0..7}).
      constexpr int GMT = GM < MT ? GM : MT, WF = F32 ? MQ : HQ / 32;   // tiles per load, 16-byte pieces per tile
      auto load_w = [&](int mo, u32x4 (&wf)[WF]) __attribute__((always_inline)) {
        const int f = qs * HQ + (F32 ? 4 : 8) * g, o = 16 * mo + q;
        constexpr int step = F32 ? 16 : 32;
#pragma unroll
        for (int m = 0; m < WF; ++m) {
          if (REV || (C::WT_ARG ? WT : Wt != nullptr)) {
            wf[m] = *reinterpret_cast<const u32x4*>((REV ? W : Wt) + ((size_t)e * H + o) * H + f + step * m);
          } else {   // a column of W_e
            const S* p = W + ((size_t)e * H + f + step * m) * H + o;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              if constexpr (F32)
                wf[m][i] = __float_as_uint(p[(size_t)i * H]);
              else
                wf[m][i] = static_cast<uint32_t>(p[(size_t)(2 * i) * H]) |
                           (static_cast<uint32_t>(p[(size_t)(2 * i + 1) * H]) << 16);
            }
          }
        }
      };
      u32x4 wf[2][GMT][WF];
#pragma unroll
      for (int i = 0; i < GMT; ++i) load_w(i, wf[0][i]);   // in flight during the aggregation

      float fd[NTW];
      if (!REV && bias != nullptr && qs == 0) {
#pragma unroll
        for (int n = 0; n < NTW; ++n) {
          int d = cur[0][n].popc() + cur[1][n].popc() + cur[2][n].popc();
          d += __shfl_xor(d, 16);
          d += __shfl_xor(d, 32);
          fd[n] = static_cast<float>(d);
        }
      }
      f32x4 P[NTW][MQ];
#pragma unroll
      for (int n = 0; n < NTW; ++n)
#pragma unroll
        for (int m = 0; m < MQ; ++m) P[n][m] = f32x4{0.f, 0.f, 0.f, 0.f};
      const uint32_t godd = static_cast<uint32_t>(g & 1);
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        uint32_t any = 0u;
#pragma unroll
        for (int n = 0; n < NTW; ++n) any |= cur[s][n].any();
        if (!wave_any(any)) continue;   // no edge of this type from the block into the wave's rows
        if constexpr (RB == 4 || RB == 8) {
#pragma unroll
          for (int n = 0; n < NTW; ++n) bytes_to_contiguous<RB>(cur[s][n].w, godd);
        }
        const bf16s* xb = xs + s * B * HQ;
#pragma unroll
        for (int kk = 0; kk < RB; ++kk) {
          if constexpr (C::KCONT && RB > 1) {
            uint32_t step = 0u;
#pragma unroll
            for (int n = 0; n < NTW; ++n) step |= cur[s][n].byte(kk);
            if (!wave_any(step)) continue;
          }
          bf16x8 bf[NTW];
#pragma unroll
          for (int n = 0; n < NTW; ++n) bf[n] = bits_frag(cur[s][n].byte(kk));
#pragma unroll
          for (int p = C::PARTS - 1; p >= 0; --p)   // the small parts first
#pragma unroll
            for (int m = 0; m < MQ; ++m) {
              const bf16x8 af = load_fragi<bf16s>(xb + p * C::PLANE, kk * MQ + m, lane);
#pragma unroll
              for (int n = 0; n < NTW; ++n) mma(P[n][m], af, bf[n]);
            }
        }
      }
      // The aggregate as operand: fp32 the accumulators themselves; bf16
      // fragments of eight features, forward as hi + lo, reverse rounded (the
      // stored dM).
      constexpr int NP = REV ? 1 : 2;
      bf16x8 pf[F32 ? 1 : NP][NTW][F32 ? 1 : WF];
      if constexpr (!F32) {
#pragma unroll
        for (int n = 0; n < NTW; ++n)
#pragma unroll
          for (int kk = 0; kk < WF; ++kk) {
            float v8[8];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              v8[j] = P[n][2 * kk][j];
              v8[4 + j] = P[n][2 * kk + 1][j];
            }
            if constexpr (REV)
              pf[0][n][kk] = pack8<bf16s>(v8);
            else
              split8(v8, pf[0][n][kk], pf[NP - 1][n][kk]);
          }
      }
      if constexpr (REV) {
#pragma unroll
        for (int n = 0; n < NTW; ++n) {
          S* row = dM + ((size_t)e * ldm + (size_t)k * B + rw + 16 * n + q) * H + qs * HQ + (F32 ? 4 : 8) * g;
#pragma unroll
          for (int m = 0; m < WF; ++m) {
            if constexpr (F32)
              *reinterpret_cast<f32x4*>(row + 16 * m) = P[n][m];
            else
              *reinterpret_cast<bf16x8*>(row + 32 * m) = pf[0][n][m];
          }
        }
      }
      // acc[n][mo] += W rows x aggregate
#pragma unroll
      for (int mo = 0; mo < MT; mo += GMT) {
        const int b = (mo / GMT) & 1;
        if (mo + GMT < MT) {
#pragma unroll
          for (int i = 0; i < GMT; ++i) load_w(mo + GMT + i, wf[1 - b][i]);
        }
#pragma unroll
        for (int m = 0; m < WF; ++m) {
          if constexpr (F32) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
              for (int i = 0; i < GMT; ++i)
#pragma unroll
                for (int n = 0; n < NTW; ++n)
                  acc[n][mo + i] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(wf[b][i][m][j]), P[n][m][j],
                                                                        acc[n][mo + i], 0, 0, 0);
          } else {
#pragma unroll
            for (int part = 0; part < NP; ++part)
#pragma unroll
              for (int i = 0; i < GMT; ++i)
#pragma unroll
                for (int n = 0; n < NTW; ++n)
                  mma(acc[n][mo + i], __builtin_bit_cast(bf16x8, wf[b][i][m]), pf[part][n][m]);
          }
        }
      }
      if (!REV && bias != nullptr && qs == 0) {
#pragma unroll
        for (int mo = 0; mo < MT; ++mo) {
          const f32x4 b4 = *reinterpret_cast<const f32x4*>(bias + (size_t)e * H + 16 * mo + 4 * g);
#pragma unroll
          for (int n = 0; n < NTW; ++n)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[n][mo][j] += fd[n] * b4[j];
        }
      }
      if (e + TG < E) {
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
          for (int n = 0; n < NTW; ++n) cur[s][n] = nxt[s][n];
      }
    }
  }

  // Output rows: lane (q, g) holds features 16 m + 4 g .. + 3 of row 16 n + q.
  auto write = [&](int n, int m, f32x4 v) __attribute__((always_inline)) {
    const size_t at = ((size_t)k * B + rw + 16 * n + q) * H + 16 * m + 4 * g;
    if (REV && dX_in != nullptr) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(dX_in + at);
      v = f32x4{b[0] + v[0], b[1] + v[1], b[2] + v[2], b[3] + v[3]};
    }
    *reinterpret_cast<f32x4*>(out + at) = v;
  };
  if constexpr (TG == 1) {
#pragma unroll
    for (int n = 0; n < NTW; ++n)
#pragma unroll
      for (int m = 0; m < MT; ++m) write(n, m, acc[n][m]);
  } else {
    // Per row tile: every group leaves its sums, then the groups share the
    // output tiles (tile m by group m % TG), adding in group order.
    f32x4* red = reinterpret_cast<f32x4*>(lds);
#pragma unroll
    for (int n = 0; n < NTW; ++n) {
      __syncthreads();
#pragma unroll
      for (int m = 0; m < MT; ++m) red[((tg * WAVES + wave) * MT + m) * kWave + lane] = acc[n][m];
      __syncthreads();
      for (int m = tg; m < MT; m += TG) {
        f32x4 v = red[(wave * MT + m) * kWave + lane];
#pragma unroll
        for (int gi = 1; gi < TG; ++gi) {
          const f32x4 r = red[((gi * WAVES + wave) * MT + m) * kWave + lane];
          v = f32x4{v[0] + r[0], v[1] + r[1], v[2] + r[2], v[3] + r[3]};
        }
        write(n, m, v);
      }
    }
  }
}

}  // namespace dev

namespace {
using S = dev::dt_t;
struct DirectArgs {
  bool rev;
  const void *bits, *V, *W, *Wt;
  const float* bias;
  float* out;
  const float* dX_in;
  void* dM;
  long ldm;
  int n_pad, E;
};

enum : int { kRev = 1, kFwdWt = 2, kFwd = 4, kAll = 7 };   // the directions that a form is built for

template <int H, int B, int WAVES, int TG, int FOR, int NTW = 2>
hipError_t direct_launch(const DirectArgs& A, hipStream_t st) {
  using C = dev::DirectCfg<S, H, B, WAVES, TG, NTW>;
  const dim3 grid((unsigned)(A.n_pad / C::R)), block(C::NT);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, static_cast<const uint8_t*>(A.bits), static_cast<const S*>(A.V),
                       static_cast<const S*>(A.W), static_cast<const S*>(A.Wt), A.bias, A.out, A.n_pad, A.E, A.dX_in,
                       static_cast<S*>(A.dM), A.ldm);
    return hipGetLastError();
  };
  if (A.rev) {
    if constexpr (FOR & kRev) return go(dev::step_direct_kernel<S, H, B, WAVES, TG, NTW, true, true>);
  } else if (A.Wt != nullptr || !C::WT_ARG) {
    if constexpr (FOR & kFwdWt) return go(dev::step_direct_kernel<S, H, B, WAVES, TG, NTW, false, true>);
  } else {
    if constexpr (C::WT_ARG && (FOR & kFwd)) return go(dev::step_direct_kernel<S, H, B, WAVES, TG, NTW, false, false>);
  }
  return hipErrorNotSupported;
}

// Rows and type groups of a workgroup, by the number of 32-row tiles: up to one tile per compute unit, one per
// workgroup and eight type groups (a wave walks few types, and all eight stage the window); from there on as many rows
// as leave each compute unit a workgroup, since a second round of workgroups costs as much as the first.
#if GGNN_DT_BF16
// The aggregate, us, 4 types, eight groups / 2 tiles x 4 groups / 4 x 2: H = 64, B = 256: 8.7 / 9.6 / 12.6 at 64 tiles, 17 /
// 10.5 / 13 at 512, 64 / 40 / 28 at 2,048; H = 128, B = 128: 12.6 / 14.7 / 22, 25 / 17 / 23, 91 / 61 / 48.  At H = 256 the
// forward without W^T (column gathers) keeps four waves per workgroup, which leaves it 512 registers a lane (with eight
// waves 36 to 100 of 256 are spilled): B = 256, 4 types 63 -> 38 us at 128 tiles, 96 -> 58 at 512, 320 -> 191 at 2,048.
// At B = 32 a block is one tile: two groups (H = 128, 4 types, 768 tiles: 30 -> 25 us, four groups 32).
template <int H, int B>
hipError_t direct_pick(const DirectArgs& A, hipStream_t st) {
  const int tiles = A.n_pad / 32;
  const bool no_wt = !A.rev && A.Wt == nullptr;
  if constexpr (H == 32 ? B < 256 : H == 64 && B < 64) {
    return hipErrorNotSupported;   // the fused kernel's sizes
  } else if constexpr (H == 32 ? B == 256 : H == 64 && B < 256) {
    return direct_launch<H, B, 1, 8, kAll>(A, st);   // up to 128 tiles
  } else if constexpr (H == 256 && B < 512) {
    if (no_wt) {
      if (tiles <= 256) return direct_launch<H, B, 1, 4, kFwd>(A, st);
      if constexpr (B == 32) {
        return direct_launch<H, B, 1, 2, kFwd>(A, st);
      } else {
        if constexpr (B >= 128) {
          if (tiles > 512) return direct_launch<H, B, 4, 1, kFwd>(A, st);
        }
        return direct_launch<H, B, 2, 2, kFwd>(A, st);
      }
    }
    if (tiles <= 256) return direct_launch<H, B, 1, 8, kRev | kFwdWt>(A, st);   // up to 512 tiles
    return direct_launch<H, B, B == 32 ? 1 : 2, B == 32 ? 2 : 4, kRev | kFwdWt>(A, st);
  } else {
    if (tiles <= (B == 512 && !A.rev ? 128 : 256)) return direct_launch<H, B, 1, 8, kAll>(A, st);
    if constexpr (B == 32) {
      if (no_wt && A.E > 6) return direct_launch<H, B, 1, 8, kFwd>(A, st);
      return direct_launch<H, B, 1, 2, kAll>(A, st);
    } else if constexpr (B == 64) {
      if (no_wt) return direct_launch<H, B, 2, 2, kFwd>(A, st);
      return direct_launch<H, B, 2, 4, kRev | kFwdWt>(A, st);
    } else {
      if (tiles <= 512) return direct_launch<H, B, 2, 4, kAll>(A, st);
      return direct_launch<H, B, 4, 2, kAll>(A, st);
    }
  }
}
#else
// A forward step with its GRU and a reverse step, us, eight groups / 2 tiles x 4 groups / 4 x 2, H = 64, B = 128, 10 types:
// 65 / 81 / 116 at 256 tiles, 109 / 85 / 119 at 512, 202 / 154 / 132 at 1,024; 2 types 44 / 45 / 47, 68 / 47 / 50, 126 / 84 /
// 62.
template <int H, int B>
hipError_t direct_pick(const DirectArgs& A, hipStream_t st) {
  const int tiles = A.n_pad / 32;
  if constexpr (H == 256) {
    // One type: 16 rows per wave, so that two waves share the transform of a tile that one would do alone (B = 32, 63
    // tiles: the aggregate 55 -> 38 us, the reverse step 52 -> 33; 512 tiles 110 -> 57, 120 -> 58).
    if (A.E == 1 && tiles <= 256) return direct_launch<H, B, 2, 4, kAll, 1>(A, st);
    if (A.E == 1 && tiles <= 512) return direct_launch<H, B, B == 32 ? 2 : 4, 2, kAll, 1>(A, st);
  }
  if constexpr (B == 32) {   // four groups up to four types and up to 512 tiles, above that two
    if (tiles > 512) return direct_launch<H, B, 1, 2, kAll>(A, st);
    if (tiles > 256 || A.E <= 4) return direct_launch<H, B, 1, 4, kAll>(A, st);
    return direct_launch<H, B, 1, 8, kAll>(A, st);
  } else {
    if (tiles <= 256) return direct_launch<H, B, 1, 8, kAll>(A, st);
    if (tiles <= 512) return direct_launch<H, B, 2, 4, kAll>(A, st);
    return direct_launch<H, B, B == 64 ? 2 : 4, 2, kAll>(A, st);
  }
}
#endif

template <int H>
hipError_t direct_h(int B, const DirectArgs& A, hipStream_t st) {
  switch (B) {
    case 32: return direct_pick<H, 32>(A, st);
    case 64: return direct_pick<H, 64>(A, st);
    case 128: return direct_pick<H, 128>(A, st);
    case 256: return direct_pick<H, 256>(A, st);
    case 512: return direct_pick<H, 512>(A, st);
  }
  return hipErrorInvalidValue;
}
}  // namespace

namespace GGNN_IMPL_NS {
hipError_t launch_step_direct(bool rev, int n_pad, int B, int H, int E, const void* bits, const void* V,
                              const void* W, const void* Wt, const float* bias, float* out, const float* dX_in,
                              void* dM, long ldm, hipStream_t st) {
  const DirectArgs A{rev, bits, V, W, Wt, bias, out, dX_in, dM, ldm, n_pad, E};
  switch (H) {
    case 32: return direct_h<32>(B, A, st);
    case 64: return direct_h<64>(B, A, st);
    case 128: return direct_h<128>(B, A, st);
    case 256: return direct_h<256>(B, A, st);
  }
  return hipErrorInvalidValue;
}
}  // namespace GGNN_IMPL_NS

}  // namespace ggnn
