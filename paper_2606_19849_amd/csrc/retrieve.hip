// Query-side chunk retrieval for gfx950: representative features, cosine
// scores and top-k selection (ViCoStream, Sec. 3, query-time decoding).
//
//   token_mean_kernel   mean over tokens of a [L][dm] bf16 embedding block,
//                       fp32 out (a chunk's feature at ingest, or the query's)
//   chunk_scores_kernel s_i = <q, c_i> / (|q| |c_i|) over the feature table
//   topk_kernel         the k best chunks with s >= tau_q (ties: smaller
//                       index), written in stream order together with their
//                       store segments, for the gathered attention
//
// All three are bound by HBM or by launch latency; none of them needs a
// workspace.  Every reduction runs in a fixed order, so results repeat
// bit for bit.

#include <type_traits>

#include "attn_common.h"

namespace vico {
namespace {

constexpr int kMeanThreads = 1024;   // 16 waves split the tokens; 4 columns per lane
constexpr int kMeanCols = 256;       // columns per work-group
constexpr int kTopkThreads = 1024;
constexpr int kTopkRegKeys = 8;      // scores kept in registers per thread (N <= 8192 read once)

__global__ __launch_bounds__(kMeanThreads) void token_mean_kernel(const uint16_t* __restrict__ x, int L, int dm,
                                                                  float* __restrict__ out) {
  constexpr int NW = kMeanThreads / 64;
  __shared__ f32x4 part[NW][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = blockIdx.x * kMeanCols + lane * 4;
  f32x4 acc{0.f, 0.f, 0.f, 0.f};
  if (col < dm) {
    const uint16_t* p = x + col;
    for (int t = wave; t < L; t += NW) {
      const uint2 v = *(const uint2*)(p + (int64_t)t * dm);
      acc[0] += __uint_as_float(v.x << 16);
      acc[1] += __uint_as_float(v.x & 0xFFFF0000u);
      acc[2] += __uint_as_float(v.y << 16);
      acc[3] += __uint_as_float(v.y & 0xFFFF0000u);
    }
  }
  part[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && col < dm) {
    f32x4 s = part[0][lane];
    for (int w = 1; w < NW; ++w) s += part[w][lane];
    *(f32x4*)(out + col) = f32x4{s[0] / (float)L, s[1] / (float)L, s[2] / (float)L, s[3] / (float)L};
  }
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// One wave per chunk (grid-stride over chunks).  |q|^2, <q, c_i> and |c_i|^2
// are summed in one walk over the features, kScoreBatch float4 of q and of
// the row per lane loaded before any is used, so a 3584-feature row costs two
// memory latencies.  Each lane adds its columns in increasing order and the
// wave reduction is fixed, so every wave gets the same |q|^2 bits.
constexpr int kScoreBatch = 8;
__global__ __launch_bounds__(256) void chunk_scores_kernel(const float* __restrict__ qf, const float* __restrict__ cf,
                                                           int N, int dm, float* __restrict__ scores) {
  const int lane = threadIdx.x & 63;
  const int gw = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int nw = (gridDim.x * blockDim.x) >> 6;
  const int n4 = dm / 4;
  for (int i = gw; i < N; i += nw) {
    const float* row = cf + (int64_t)i * dm;
    float dot = 0.f, cc = 0.f, qq = 0.f;
    for (int c0 = lane; c0 < n4; c0 += 64 * kScoreBatch) {
      f32x4 q[kScoreBatch], v[kScoreBatch];
#pragma unroll
      for (int u = 0; u < kScoreBatch; ++u) {
        const int c = min(c0 + 64 * u, n4 - 1);      // in range; the sums below skip c >= n4
        q[u] = *(const f32x4*)(qf + 4 * c);
        v[u] = *(const f32x4*)(row + 4 * c);
      }
#pragma unroll
      for (int u = 0; u < kScoreBatch; ++u)
        if (c0 + 64 * u < n4) {
          qq += q[u][0] * q[u][0] + q[u][1] * q[u][1] + q[u][2] * q[u][2] + q[u][3] * q[u][3];
          dot += q[u][0] * v[u][0] + q[u][1] * v[u][1] + q[u][2] * v[u][2] + q[u][3] * v[u][3];
          cc += v[u][0] * v[u][0] + v[u][1] * v[u][1] + v[u][2] * v[u][2] + v[u][3] * v[u][3];
        }
    }
    qq = wave_sum(qq);
    dot = wave_sum(dot);
    cc = wave_sum(cc);
    if (lane == 0) {
      const float den = sqrtf(cc) * sqrtf(qq);
      scores[i] = den > 0.f ? dot / den + 0.0f : 0.0f;   // + 0 turns -0 into +0
    }
  }
}

// Order-preserving map of a (non-NaN) float to an unsigned key.
__device__ __forceinline__ uint32_t order_key(float s) {
  const uint32_t u = __float_as_uint(s + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

struct TopkArgs {
  const float* scores;
  int N, k;
  float min_score;
  const int64_t* chunk_start;
  const int32_t* chunk_len;
  int32_t* out_chunks;
  float* out_scores;
  int64_t* seg_start;
  int32_t* seg_len;
  int32_t* out_count;
};

// Radix select of the k-th largest key, 8 bits at a time from the top, then
// one numbering of the selected scores in index order.  One work-group, bound
// by the latency of its barriers and LDS round trips, so it makes few: every
// digit has its own histogram (cleared together), every wave finds the digit
// for itself from the histogram (no second barrier), and the scores kept in
// registers are numbered in one step from their ballots.  6 barriers (3 where
// all candidates are taken); with three barriers per digit and four per
// numbering step it took 6.5 us at 256 scores and 9.4 at 1800, now 4.9 and 6.8
// (traced).
//
// NT threads: 256 for up to 256 scores (fewer waves to wait for), else 1024.
// The first NR * NT keys stay in registers; further ones are read again.  2
// and 8 keys per thread are separate kernels: at 1800 scores the walk over 8
// mostly empty registers took 10.0 us against 6.8.
template <int NT, int NR>
__global__ __launch_bounds__(NT) void topk_kernel(TopkArgs a) {
  constexpr int NW = NT / 64;
  static_assert(NR * NW <= 128, "a wave scans the per-wave counts of all register keys, two per lane");
  __shared__ int hist[4][256];
  __shared__ int cnt_gt[128], cnt_eq[128];           // selected / equal keys per (register, wave)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // key of score i, 0 for "not a candidate" (0 is the key of a NaN pattern,
  // which is never a candidate)
  auto key_of = [&](int i) __attribute__((always_inline)) -> uint32_t {
    const float s = a.scores[i];
    return (!isnan(s) && s >= a.min_score) ? order_key(s) : 0u;
  };
  uint32_t kr[NR];
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const int i = tid + j * NT;
    kr[j] = i < a.N ? key_of(i) : 0u;
  }
  for (int i = tid; i < 4 * 256; i += NT) (&hist[0][0])[i] = 0;
  __syncthreads();

  // digits of the k-th largest key.  Lane l of every wave holds bins 255-4l ..
  // 252-4l and finds where the count from the top first reaches `remaining`.
  uint32_t prefix = 0, mask = 0;
  int remaining = a.k;
  bool take_all = false;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const int shift = 24 - 8 * d;
    auto count = [&](uint32_t k) __attribute__((always_inline)) {
      if (k != 0u && (k & mask) == prefix) atomicAdd(&hist[d][(k >> shift) & 255u], 1);
    };
#pragma unroll
    for (int j = 0; j < NR; ++j) count(kr[j]);
    for (int i = tid + NR * NT; i < a.N; i += NT) count(key_of(i));
    __syncthreads();
    int c[4], tot = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      c[e] = hist[d][255 - 4 * lane - e];
      tot += c[e];
    }
    int incl = tot;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o, 64);
      incl += lane >= o ? y : 0;
    }
    if (d == 0 && __builtin_amdgcn_readlane(incl, 63) <= a.k) {      // no more candidates than asked for
      take_all = true;
      break;
    }
    const int before = incl - tot;
    const int hit = __builtin_ctzll(__builtin_amdgcn_ballot_w64(before < remaining && incl >= remaining));
    int cum = __builtin_amdgcn_readlane(before, hit), bin = 255 - 4 * hit;
#pragma unroll
    for (int e = 0; e < 3; ++e) {                    // which of the lane's four bins (wave-uniform)
      const int n = __builtin_amdgcn_readlane(c[e], hit);
      const bool past = bin == 255 - 4 * hit - e && cum + n < remaining;
      cum += past ? n : 0;
      bin -= past ? 1 : 0;
    }
    remaining -= cum;
    prefix |= (uint32_t)bin << shift;
    mask |= 255u << shift;
  }
  // prefix = key of the k-th best; keys above it are all taken, and
  // `remaining` of those equal to it, earliest first.  A selected score's place
  // is the number of taken ones before it.
  auto is_gt = [&](uint32_t k) __attribute__((always_inline)) { return k != 0u && (take_all || k > prefix); };
  auto is_eq = [&](uint32_t k) __attribute__((always_inline)) { return k != 0u && !take_all && k == prefix; };
  auto put = [&](int pos, int i) __attribute__((always_inline)) {
    a.out_chunks[pos] = i;
    a.out_scores[pos] = a.scores[i];
    if (a.seg_start) {
      a.seg_start[pos] = a.chunk_start[i];
      a.seg_len[pos] = a.chunk_len[i];
    }
  };
  const uint64_t below = (1ull << lane) - 1;
  // numbers NG groups of NT consecutive scores; key(j) is this thread's key in group j, i0 the first score
  int gt_seen = 0, eq_seen = 0;
  auto number = [&](auto groups, auto&& key, int i0) __attribute__((always_inline)) {
    constexpr int NG = decltype(groups)::value;
#pragma unroll
    for (int j = 0; j < NG; ++j) {
      const uint64_t g = __builtin_amdgcn_ballot_w64(is_gt(key(j))), q = __builtin_amdgcn_ballot_w64(is_eq(key(j)));
      if (lane == 0) {
        cnt_gt[j * NW + wave] = __builtin_popcountll(g);
        cnt_eq[j * NW + wave] = __builtin_popcountll(q);
      }
    }
    __syncthreads();
    // exclusive counts before each (group, wave): two entries per lane, every wave for itself
    constexpr int NE = NG * NW;
    const int e0 = 2 * lane < NE ? cnt_gt[2 * lane] : 0, e1 = 2 * lane + 1 < NE ? cnt_gt[2 * lane + 1] : 0;
    const int f0 = 2 * lane < NE ? cnt_eq[2 * lane] : 0, f1 = 2 * lane + 1 < NE ? cnt_eq[2 * lane + 1] : 0;
    int ig = e0 + e1, iq = f0 + f1;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int yg = __shfl_up(ig, o, 64), yq = __shfl_up(iq, o, 64);
      ig += lane >= o ? yg : 0;
      iq += lane >= o ? yq : 0;
    }
#pragma unroll
    for (int j = 0; j < NG; ++j) {
      const int w = __builtin_amdgcn_readfirstlane(j * NW + wave), src = w >> 1;
      const int gt_w = __builtin_amdgcn_readlane(ig, src) - __builtin_amdgcn_readlane(e1, src) -
                       ((w & 1) ? 0 : __builtin_amdgcn_readlane(e0, src));
      const int eq_w = __builtin_amdgcn_readlane(iq, src) - __builtin_amdgcn_readlane(f1, src) -
                       ((w & 1) ? 0 : __builtin_amdgcn_readlane(f0, src));
      const bool gt = is_gt(key(j)), eq = is_eq(key(j));
      const uint64_t g = __builtin_amdgcn_ballot_w64(gt), q = __builtin_amdgcn_ballot_w64(eq);
      const int gt_before = gt_seen + gt_w + __builtin_popcountll(g & below);
      const int eq_before = eq_seen + eq_w + __builtin_popcountll(q & below);
      if (gt || (eq && eq_before < remaining)) put(gt_before + min(eq_before, remaining), i0 + j * NT + tid);
    }
    gt_seen += __builtin_amdgcn_readlane(ig, 63);
    eq_seen += __builtin_amdgcn_readlane(iq, 63);
  };
  number(std::integral_constant<int, NR>{}, [&](int j) __attribute__((always_inline)) { return kr[j]; }, 0);
  for (int i0 = NR * NT; i0 < a.N; i0 += NT) {
    const int i = i0 + tid;
    const uint32_t k = i < a.N ? key_of(i) : 0u;
    __syncthreads();                                 // the counts of the step before have been read
    number(std::integral_constant<int, 1>{}, [&](int) __attribute__((always_inline)) { return k; }, i0);
  }
  const int taken = gt_seen + min(eq_seen, take_all ? 0 : remaining);
  for (int j = taken + tid; j < a.k; j += NT) {
    a.out_chunks[j] = -1;
    a.out_scores[j] = -INFINITY;
    if (a.seg_start) {
      a.seg_start[j] = 0;
      a.seg_len[j] = 0;
    }
  }
  if (tid == 0) a.out_count[0] = taken;
}

}  // namespace

hipError_t launch_token_mean(const uint16_t* x, int L, int dm, float* out, hipStream_t stream) {
  const int blocks = (dm + kMeanCols - 1) / kMeanCols;
  hipLaunchKernelGGL(token_mean_kernel, dim3(blocks), dim3(kMeanThreads), 0, stream, x, L, dm, out);
  return hipGetLastError();
}

hipError_t launch_chunk_scores(const float* qf, const float* cf, int N, int dm, float* scores, hipStream_t stream) {
  const int waves = N < 4096 ? N : 4096;
  const int blocks = (waves + 3) / 4;
  hipLaunchKernelGGL(chunk_scores_kernel, dim3(blocks), dim3(256), 0, stream, qf, cf, N, dm, scores);
  return hipGetLastError();
}

hipError_t launch_topk(const float* scores, int N, int k, float min_score, const int64_t* chunk_start,
                       const int32_t* chunk_len, int32_t* out_chunks, float* out_scores, int64_t* seg_start,
                       int32_t* seg_len, int32_t* out_count, hipStream_t stream) {
  TopkArgs a{scores, N, k, min_score, chunk_start, chunk_len, out_chunks, out_scores, seg_start, seg_len, out_count};
  // the smallest form whose registers hold all scores
  if (N <= 256)
    hipLaunchKernelGGL((topk_kernel<256, 1>), dim3(1), dim3(256), 0, stream, a);
  else if (N <= 2 * kTopkThreads)
    hipLaunchKernelGGL((topk_kernel<kTopkThreads, 2>), dim3(1), dim3(kTopkThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((topk_kernel<kTopkThreads, kTopkRegKeys>), dim3(1), dim3(kTopkThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace vico
