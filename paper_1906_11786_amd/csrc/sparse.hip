// Sparse propagation over an explicit edge list, for evaluation on every edge
// of graphs whose bandwidth exceeds the block size a model was trained with:
// the weights learned on the block band are the same parameters the sparse
// model uses, so they can be evaluated with messages passed along all edges
// (Experiments, "Training time to validation accuracy").
//
//   a[i] = sum_e ( sum_{j -> i of type e} X[j] ) W_e  (+ deg_e(i) b_e)
//
// in the operand order of Algorithm 1 (aggregate per type, then transform),
// the aggregate gathered exactly from the receiver-major lists of
// ggnn_sparse_csr.  A wave takes 16 receivers: lane (q, g) gathers, for
// receiver q, features 32kk + 8g .. + 7 of every sender row (the four lanes of
// a receiver read whole rows together), sums them in float32, and the
// per-type transform runs on the matrix cores with the aggregate as the B
// operand (bf16 hi + lo in bf16 mode) and rows of W_e^T as the A operand.
// Two forms: one workgroup per 16 receivers, on small graphs with the types
// dealt to its waves (sparse_step_kernel), and, on larger graphs at H <= 64,
// one workgroup per compute unit with all types' weights in LDS
// (sparse_lds_kernel); launch_sparse_step says where which runs.
#include "device_common.h"
#include "kernels.h"

namespace ggnn {
namespace dev {

// On small graphs (few groups of 16 receivers) the waves of a workgroup share
// 16 receivers and split the edge types among them (wave w takes types w,
// w + NW, ...), which multiplies the waves in flight by NW and shortens each
// wave's chain of dependent loads (list bounds, column index, sender row) by
// the same factor. Their partial results are added through LDS in wave
// order, so the output does not depend on timing. NW = 8 up to H = 64, 4
// above (the partials take NW * H * 64 bytes of LDS). Larger graphs give
// every SIMD several waves already: there NW = 1 (one wave walks all types).
template <int H>
constexpr int sparse_waves() { return H <= 64 ? 8 : 4; }
#ifndef GGNN_SPARSE_SPLIT_MAX_GROUPS
#define GGNN_SPARSE_SPLIT_MAX_GROUPS 2048
#endif

template <typename S, int H, int NW>
__global__ __launch_bounds__(NW * kWave) void sparse_step_kernel(
    const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, const S* __restrict__ X,
    const S* __restrict__ Wt, const float* __restrict__ bias, float* __restrict__ out, int n_pad, int E) {
  constexpr int HK = H / 32, MT = H / 16;
  constexpr int NP = sizeof(S) == 2 ? 2 : 1;
  // partial results: red[wave][mo][lane], one f32x4 per lane and output tile
  __shared__ f32x4 red[NW > 1 ? NW : 1][NW > 1 ? MT : 1][kWave];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int q = lane % 16, g = lane / 16;
  const int n0 = blockIdx.x * 16;
  if (n0 >= n_pad) return;   // uniform over the workgroup, before its one barrier
  const int node = n0 + q;

  f32x4 acc[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Up to two of the wave's edge types per pass: their gathers are
  // independent, so both lists' loads are in flight together. Each list is
  // still walked in order, so every type's sum is formed as with one type at
  // a time. Above H = 64 a second set of partial sums costs occupancy.
  constexpr int NE = H <= 64 ? 2 : 1;
  for (int k0 = 0; wave + NW * k0 < E; k0 += NE) {
    // List bounds of the pass's types; a type index past E is clamped to the
    // node's last bound and so gets an empty list.
    int lo[NE], len[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int e = wave + NW * (k0 + i);
      const int a0 = e < E ? e : E, a1 = e + 1 < E ? e + 1 : E;
      lo[i] = row_ptr[(size_t)node * E + a0];
      len[i] = row_ptr[(size_t)node * E + a1] - lo[i];
    }
    float p[NE][HK][8];
#pragma unroll
    for (int i = 0; i < NE; ++i)
#pragma unroll
      for (int kk = 0; kk < HK; ++kk)
#pragma unroll
        for (int x = 0; x < 8; ++x) p[i][kk][x] = 0.f;
    int steps = len[0];
#pragma unroll
    for (int i = 1; i < NE; ++i) steps = len[i] > steps ? len[i] : steps;
    // Every list's loads are issued before any sum is formed, so the chains
    // of the types overlap, and nothing branches on which lists are
    // exhausted. A lane inside the loop has a non-empty list, so col[0]
    // exists; it stands in for an exhausted list (it names a valid sender)
    // and the values it brings are dropped.
    for (int j = 0; j < steps; ++j) {
      int c[NE];
#pragma unroll
      for (int i = 0; i < NE; ++i) c[i] = col[j < len[i] ? lo[i] + j : 0];
      frag_t<S> v[NE][HK];
#pragma unroll
      for (int i = 0; i < NE; ++i) {
        const S* row = X + (size_t)c[i] * H + 8 * g;
#pragma unroll
        for (int kk = 0; kk < HK; ++kk) v[i][kk] = load8(row + 32 * kk);
      }
#pragma unroll
      for (int i = 0; i < NE; ++i) {
        const bool live = j < len[i];
#pragma unroll
        for (int kk = 0; kk < HK; ++kk)
#pragma unroll
          for (int x = 0; x < 8; ++x) p[i][kk][x] += live ? static_cast<float>(v[i][kk][x]) : 0.f;
      }
    }
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int e = wave + NW * (k0 + i);
      if (e >= E) break;
      frag_t<S> pf[NP][HK];
#pragma unroll
      for (int kk = 0; kk < HK; ++kk) {
        if constexpr (NP == 2) {
          split8(p[i][kk], pf[0][kk], pf[NP - 1][kk]);
        } else {
          pf[0][kk] = pack8<S>(p[i][kk]);
        }
      }
      const S* we = Wt + (size_t)e * H * H;
#pragma unroll
      for (int mo = 0; mo < MT; ++mo) {
#pragma unroll
        for (int kk = 0; kk < HK; ++kk) {
          const frag_t<S> wf = load8(we + (size_t)(16 * mo + q) * H + 32 * kk + 8 * g);
#pragma unroll
          for (int part = 0; part < NP; ++part) mma(acc[mo], wf, pf[part][kk]);
        }
      }
      if (bias != nullptr) {
        const float d = static_cast<float>(len[i]);
#pragma unroll
        for (int mo = 0; mo < MT; ++mo) {
          const f32x4 b4 = *reinterpret_cast<const f32x4*>(bias + (size_t)e * H + 16 * mo + 4 * g);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[mo][j] += d * b4[j];
        }
      }
    }
  }
  if constexpr (NW == 1) {
    // acc[mo] = D[feature 16mo + 4g + j][receiver q]
#pragma unroll
    for (int mo = 0; mo < MT; ++mo)
      *reinterpret_cast<f32x4*>(out + (size_t)node * H + 16 * mo + 4 * g) = acc[mo];
    return;
  }
#pragma unroll
  for (int mo = 0; mo < MT; ++mo) red[wave][mo][lane] = acc[mo];
  __syncthreads();
  // acc[mo] = D[feature 16mo + 4g + j][receiver q]; wave w writes the tiles
  // mo = w, w + NW, ..., each the sum of the waves' parts in order.
  for (int mo = wave; mo < MT; mo += NW) {
    f32x4 sum = red[0][mo][lane];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const f32x4 t = red[w][mo][lane];
#pragma unroll
      for (int j = 0; j < 4; ++j) sum[j] += t[j];
    }
    *reinterpret_cast<f32x4*>(out + (size_t)node * H + 16 * mo + 4 * g) = sum;
  }
}

// ---------------------------------------------------------------------------
// The same step for H <= 64 with every type's weights in LDS (they fit up to
// E = 14 at H = 64 in bf16): one workgroup of 16 waves per compute unit, walking over
// its share of the receivers, 16 of them per wave at a time.  What the kernel
// above is bound by on large graphs is the number of cache lines its loads
// touch: per 16 receivers and type the weight fragments alone take
// (H / 16) (H / 32) loads of 16 lines.  Here they are read from LDS in fragment
// order, and the wave's list bounds and senders (one contiguous piece of
// row_ptr and col each) are copied to LDS with coalesced loads, which leaves
// the sender rows as the only gathers; the next type's first PF rows per
// receiver are in flight while a type is summed and transformed.  A few long
// lists in a group (a receiver that many nodes send to) are shared by the
// wave's lanes; every other sum is formed in list order, as above.  100,000
// nodes, H = 64, 10 types, two senders per receiver and type: 101 -> 45 us per
// launch; with eight receivers of 2,000 more senders each 671 -> 159 us (812 without
// the sharing), at 20,000 nodes 186 -> 91 (527).
// ---------------------------------------------------------------------------
constexpr int kSparseWaves = 16;      // per workgroup
constexpr int kSparseLong = 48;       // a list of one receiver and type with more senders is shared by the wave,
constexpr int kSparseShared = 4;      // if at most so many of the 16 receivers have one
constexpr int kSparseCols = 448;      // senders of 16 receivers kept in LDS (others are read from memory)
__host__ __device__ constexpr int sparse_rp_ints(int E) { return (16 * E + 1 + 63) / 64 * 64; }
template <typename S, int H>
__host__ __device__ constexpr long sparse_lds_bytes(int E) {
  return (long)E * H * H * (int)sizeof(S) + kSparseWaves * 4L * (sparse_rp_ints(E) + kSparseCols);
}

// Orders one wave's LDS accesses before and after (other lanes of the wave read what a lane wrote).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename S, int H>
__global__ __launch_bounds__(kSparseWaves * kWave) void sparse_lds_kernel(
    const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, const S* __restrict__ X,
    const S* __restrict__ Wt, const float* __restrict__ bias, float* __restrict__ out, int n_pad, int E) {
  constexpr int HK = H / 32, MT = H / 16, V = 16 / (int)sizeof(S);
  constexpr int NP = sizeof(S) == 2 ? 2 : 1;
  constexpr int PF = HK * sizeof(S) <= 4 ? 2 : 1;   // rows in flight ahead (fp32 at H = 64: few registers left)
  __shared__ __attribute__((aligned(16))) char lds[160 * 1024];
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int q = lane % 16, g = lane / 16;
  S* const wl = reinterpret_cast<S*>(lds);
  int32_t* const rp = reinterpret_cast<int32_t*>(lds + (size_t)E * H * H * sizeof(S)) +
                      wave * (sparse_rp_ints(E) + kSparseCols);
  int32_t* const cl = rp + sparse_rp_ints(E);

  // Weights in fragment order: fragment (e, mo, kk), unit = one 16-byte piece of a lane's eight elements.
  const int units = E * H * H / V;
  for (int u = tid; u < units; u += kSparseWaves * kWave) {
    const int e = u / (H * H / V), r = u % (H * H / V), o = r / (H / V), f = (r % (H / V)) * V;
    const u32x4 v = *reinterpret_cast<const u32x4*>(Wt + (size_t)e * H * H + (size_t)o * H + f);
    const int idx = (e * MT + o / 16) * HK + f / 32;
    *reinterpret_cast<u32x4*>(wl + fo<S>(idx, o % 16 + 16 * ((f % 32) / 8), f % 8)) = v;
  }
  __syncthreads();

  // Consecutive groups of 16 receivers go to one workgroup, and consecutive
  // workgroups to one XCD, so that shared senders are found in its caches.
  const int groups = n_pad / 16, wg = xcd_swizzle(blockIdx.x, gridDim.x);
  const int g_lo = (int)((long)wg * groups / gridDim.x), g_hi = (int)((long)(wg + 1) * groups / gridDim.x);
  for (int grp = g_lo + wave; grp < g_hi; grp += kSparseWaves) {
    const int n0 = 16 * grp;
    const int32_t* src = row_ptr + (size_t)n0 * E;
    const int count = 16 * E + 1;
    // Wave-private LDS: the wave's own writes and reads are kept in order by
    // wavefront fences, no barrier.
    for (int i = lane; i < count; i += kWave) rp[i] = src[i];
    wave_lds_order();
    const int first = __builtin_amdgcn_readfirstlane(rp[0]);
    const int total = __builtin_amdgcn_readfirstlane(rp[16 * E]) - first;
    const int kept = total < kSparseCols ? total : kSparseCols;
    for (int i = lane; i < kept; i += kWave) cl[i] = col[first + i];
    wave_lds_order();
    auto sender = [&](int k) __attribute__((always_inline)) {   // k-th sender of the group
      return total <= kSparseCols ? cl[k] : (k < kSparseCols ? cl[k] : col[first + k]);
    };
    f32x4 acc[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m] = f32x4{0.f, 0.f, 0.f, 0.f};

    int lo[2], len[2];
    frag_t<S> v[2][PF][HK];   // the first PF sender rows of this type and the next
    auto fetch = [&](int e, int b) __attribute__((always_inline)) {
      lo[b] = rp[q * E + e] - first;
      len[b] = rp[q * E + e + 1] - first - lo[b];
#pragma unroll
      for (int j = 0; j < PF; ++j) {
#pragma unroll
        for (int kk = 0; kk < HK; ++kk) v[b][j][kk] = frag_t<S>{};
        if (j < len[b]) {
          const S* row = X + (size_t)sender(lo[b] + j) * H + 8 * g;
#pragma unroll
          for (int kk = 0; kk < HK; ++kk) v[b][j][kk] = load8(row + 32 * kk);
        }
      }
    };
    auto one = [&](int e, int b) __attribute__((always_inline)) {
      if (e + 1 < E) fetch(e + 1, 1 - b);
      float p[HK][8];
#pragma unroll
      for (int kk = 0; kk < HK; ++kk)
#pragma unroll
        for (int x = 0; x < 8; ++x) {
          p[kk][x] = static_cast<float>(v[b][0][kk][x]);
          if constexpr (PF == 2) p[kk][x] += static_cast<float>(v[b][1][kk][x]);
        }
      // PF rows at a time (a lane past its list's end adds zeros), a few long lists apart.
      uint64_t todo = __builtin_amdgcn_ballot_w64(len[b] > kSparseLong) & 0xFFFFu;
      if (__builtin_popcountll(todo) > kSparseShared) todo = 0;
      const int most = (todo >> q) & 1 ? PF : len[b];
      for (int j = PF; j < most; j += PF) {
        frag_t<S> r[PF][HK];
#pragma unroll
        for (int i = 0; i < PF; ++i) {
#pragma unroll
          for (int kk = 0; kk < HK; ++kk) r[i][kk] = frag_t<S>{};
          if (j + i < most) {
            const S* row = X + (size_t)sender(lo[b] + j + i) * H + 8 * g;
#pragma unroll
            for (int kk = 0; kk < HK; ++kk) r[i][kk] = load8(row + 32 * kk);
          }
        }
#pragma unroll
        for (int i = 0; i < PF; ++i)
#pragma unroll
          for (int kk = 0; kk < HK; ++kk)
#pragma unroll
            for (int x = 0; x < 8; ++x) p[kk][x] += static_cast<float>(r[i][kk][x]);
      }
      // A long list is shared by the 16 lane groups of four: group i takes rows PF + i, PF + 16 + i, ...; their sums meet
      // in a butterfly, so that its rows are not one chain of loads behind which 15 receivers wait.
      for (; todo != 0; todo &= todo - 1) {
        const int r = __builtin_ctzll(todo);
        const int rlo = __builtin_amdgcn_readlane(lo[b], r), rlen = __builtin_amdgcn_readlane(len[b], r);
#pragma unroll
        for (int kk = 0; kk < HK; ++kk) {
          float part[8];
#pragma unroll
          for (int x = 0; x < 8; ++x) part[x] = 0.f;
#pragma unroll 1
          for (int j = PF + q; j < rlen; j += 16) {
            const frag_t<S> w = load8(X + (size_t)sender(rlo + j) * H + 8 * g + 32 * kk);
#pragma unroll
            for (int x = 0; x < 8; ++x) part[x] += static_cast<float>(w[x]);
          }
#pragma unroll
          for (int x = 0; x < 8; ++x) {
#pragma unroll
            for (int off = 1; off < 16; off *= 2) part[x] += __shfl_xor(part[x], off);
            p[kk][x] += q == r ? part[x] : 0.f;
          }
        }
      }
#pragma unroll
      for (int kk = 0; kk < HK; ++kk) {
        frag_t<S> pf[NP];
        if constexpr (NP == 2) {
          split8(p[kk], pf[0], pf[NP - 1]);
        } else {
          pf[0] = pack8<S>(p[kk]);
        }
#pragma unroll
        for (int mo = 0; mo < MT; ++mo) {
          const frag_t<S> wf = load_fragi<S>(wl, (e * MT + mo) * HK + kk, lane);
#pragma unroll
          for (int part = 0; part < NP; ++part) mma(acc[mo], wf, pf[part]);
        }
      }
      if (bias != nullptr) {
        const float d = static_cast<float>(len[b]);
#pragma unroll
        for (int mo = 0; mo < MT; ++mo) {
          const f32x4 b4 = *reinterpret_cast<const f32x4*>(bias + (size_t)e * H + 16 * mo + 4 * g);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[mo][j] += d * b4[j];
        }
      }
    };
    fetch(0, 0);
    for (int e = 0; e < E; e += 2) {
      one(e, 0);
      if (e + 1 < E) one(e + 1, 1);
    }
#pragma unroll
    for (int mo = 0; mo < MT; ++mo)
      *reinterpret_cast<f32x4*>(out + (size_t)(n0 + q) * H + 16 * mo + 4 * g) = acc[mo];
    wave_lds_order();   // this group's lists are read before the next group's are written
  }
}

}  // namespace dev

namespace GGNN_IMPL_NS {
hipError_t launch_sparse_step(int n_pad, int H, int E, const int32_t* row_ptr, const int32_t* col, const void* X,
                              const void* Wt, const float* bias, float* a, hipStream_t st) {
  using S = dev::dt_t;
  const int blocks = n_pad / 16;   // n_pad is a multiple of 32 (checked by the caller)
  const bool split = blocks <= GGNN_SPARSE_SPLIT_MAX_GROUPS;
  // All weights in LDS where they fit and the grid is large enough.  Up to 2,048 groups the other form shares 16
  // receivers among eight waves, which counts the more the more types and edges a receiver has and the less the
  // transform takes (H = 32).  Random senders, 0.5 / 2 / 8 / 30 per receiver and type, other form / this one, us:
  // H = 64, E = 4 at 1,024 groups 12.7 / 9.7, 16.2 / 12.8, 27 / 25, 64 / 58; E = 10 there 19 / 17, 26 / 24, 47 / 52,
  // 117 / 130, at 1,250 groups 24 / 18, 34 / 26, 66 / 57, 167 / 142; E = 14 at 1,250 30 / 23, 42 / 34, 81 / 74, 209 / 208.
  // H = 32: E = 2 at 1,024 groups 6.6 / 6.0 to 24 / 24; E = 4 there 8.0 / 9.3 to 32 / 43, at 1,250 10 / 9 to 47 / 44; E = 10 at
  // 1,250 10 / 11 to 92 / 104, at 2,048 121 / 131 with 30 per type; from 2,500 on (one wave per 16 receivers in both)
  // faster in each.
  auto lds_applies = [&](int HH) {
    const int least = HH == 64 ? (E <= 4 ? 1024 : 1250) : (E <= 2 ? 1024 : (E <= 4 ? 1250 : GGNN_SPARSE_SPLIT_MAX_GROUPS + 1));
    return blocks >= least;
  };
#define GGNN_SPARSE_LDS(HH)                                                                                        \
  if (lds_applies(HH) && dev::sparse_lds_bytes<S, HH>(E) <= 160 * 1024) {                                          \
    hipLaunchKernelGGL((dev::sparse_lds_kernel<S, HH>), dim3(256), dim3(dev::kSparseWaves * 64), 0, st, row_ptr, col, \
                       static_cast<const S*>(X), static_cast<const S*>(Wt), bias, a, n_pad, E);                    \
    return hipGetLastError();                                                                                       \
  }
#define GGNN_SPARSE_NW(HH, NWV)                                                                               \
  hipLaunchKernelGGL((dev::sparse_step_kernel<S, HH, NWV>), dim3(blocks), dim3((NWV) * 64), 0, st, row_ptr, col, \
                     static_cast<const S*>(X), static_cast<const S*>(Wt), bias, a, n_pad, E)
#define GGNN_SPARSE(HH)                                  \
  if (split) {                                           \
    GGNN_SPARSE_NW(HH, dev::sparse_waves<HH>());         \
  } else {                                               \
    GGNN_SPARSE_NW(HH, 1);                               \
  }
  switch (H) {
    case 32: GGNN_SPARSE_LDS(32) GGNN_SPARSE(32); break;
    case 64: GGNN_SPARSE_LDS(64) GGNN_SPARSE(64); break;
    case 128: GGNN_SPARSE(128); break;
    case 256: GGNN_SPARSE(256); break;
    default: return hipErrorInvalidValue;
  }
#undef GGNN_SPARSE
#undef GGNN_SPARSE_LDS
#undef GGNN_SPARSE_NW
  return hipGetLastError();
}
}  // namespace GGNN_IMPL_NS

}  // namespace ggnn
