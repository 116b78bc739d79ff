// Attention of few query rows, straight from memory into registers (gfx950).
//
// The decode step, the short query and the small chunk: softmax(Q K^T /
// sqrt(d)) V for row tiles of 16 or 32 packed (token, query head) rows
// over the keys [sink | store segments or ring window | tail, causal]
// (ViCoStream Sec. 3; query rows of Eq. (4), and its vision rows for a chunk).
//
// What bounds it, and the form taken.  Such calls read each key once or a few
// times and compute little, so they are bound by the latency from the launch
// to the last key's arrival and by how many bytes are in flight; staging tiles
// in LDS for one or two computing waves serialises a work-group behind its
// barriers.  Here every wave works alone: it takes 32-key blocks of its
// work-group's key range in turn, loads them into registers and keeps its own
// running softmax state.
// There is no barrier before the end, where the waves' states are merged
// through LDS.  8 waves: 12 measured the same on the 20.5k-key decode step
// (16.1 us a layer with its merge; staged through LDS 22.6), 16 at 128
// registers each spill (24.4).
//   * v_mfma_f32_16x16x32_bf16.  S^T = K Q^T: the A operand wants 8
//     consecutive dims of one key row per lane, which is a 16-byte load.  The
//     32 keys are two 16-key products whose row order is chosen so that lane
//     group j = lane/16 ends with the logits of keys 8j .. 8j+7: P^T is then
//     the B operand of the second product as it stands.
//     A wave's 16 consecutive lanes then ask for 16 different rows, 16 bytes of
//     each, and the CU takes such a load at a fraction of the rate of one that
//     covers whole rows (reading the same bytes row by row took 2.1 us off an
//     8.2 us call of 5 row tiles).  STAGE: K comes by whole rows into the wave's own LDS and
//     is read back as fragments; no barrier, the stage is the wave's part of
//     the merge buffer.  It costs a pass through LDS on the way of each block,
//     so it is for calls whose row tiles read the same keys, out of the
//     caches; where one tile streams them from HBM it is 5 % slower.
//   * O^T = V^T P^T: the A operand wants 8 consecutive keys of one dim per
//     lane.  A lane loads VE = d/16 consecutive dims of its 8 keys (each load
//     covers 4 whole rows) and transposes them in registers (one v_perm_b32
//     per two values); product e takes dims VE*m + e, so O^T leaves each lane
//     with VE consecutive dims of 4 dim groups.
//   * The segment table sits in the lanes (up to 64 entries, lane = segment):
//     clamped, prefix-summed and searched with wave operations, so that no
//     LDS or barrier stands between the table and the first key load.

#include "attn_common.h"

namespace vico {
namespace {

template <int D, int NRB, int NW, bool STAGE>
__global__ __launch_bounds__(NW * 64, 1) void attn_rows_kernel(RowsArgs a) {
  constexpr int NKS = D / 32;              // k-steps of Q K^T
  constexpr int VE = D / 16;               // dims per lane of a V row
  constexpr int RT = 16 * NRB;             // rows of the work-group
  constexpr int BK = kRowsBlock;           // keys per block
  constexpr int OS = D + 8;                // row stride of the merge buffer (floats)
  static_assert(BK == 32, "two 16-key products per block");
  typedef uint32_t vrow_t __attribute__((ext_vector_type(VE / 2)));

  __shared__ __attribute__((aligned(16))) float o_s[NW][RT][OS];
  __shared__ float m_s[NW][RT], l_s[NW][RT];

  // ---- the append's share: slots that no work-group of this launch reads
  const int n_work = gridDim.x - a.app_blocks;
  if ((int)blockIdx.x >= n_work) {
    append_units(a.app, (int64_t)(blockIdx.x - n_work) * blockDim.x + threadIdx.x, (int64_t)a.app_blocks * blockDim.x);
    return;
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, j = lane >> 4;
  const int g = a.Hq / a.Hkv;
  const int NR = g * a.Lq;

  // ---- work item: row tiles of one key range side by side (they share its K/V in an XCD's L2)
  const int L = xcd_remap(blockIdx.x, n_work);
  const int rt = L % a.n_rt;
  const int part = (L / a.n_rt) % a.parts;
  const int kv = L / (a.n_rt * a.parts);

  // ---- segment table: lane s holds segment s.  Loads first.
  int64_t st = 0;
  int sl = 0;
  if (a.seg_start) {
    const int sc = min(lane, a.n_segs - 1);
    st = a.seg_start[sc];
    sl = a.seg_len[sc];
  } else {
    st = lane == 0 ? a.seg0 : 0;
    sl = lane == 0 ? a.len0 : a.len1;
  }

  // ---- Q rows as B fragments; rows past the end repeat the last one and are never stored
  bf16x8 qf[NRB][NKS];
  int tok[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    const int r = min(rt * RT + rb * 16 + n, NR - 1);
    tok[rb] = r / g;
    const uint16_t* qp = a.q + ((int64_t)tok[rb] * a.Hq + kv * g + r % g) * D + j * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[rb][ks] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qp + ks * 32));
  }

  // clamp to the store; incl = keys in segments 0 .. s, shift: slot of gathered key i = i + shift
  const int64_t lo = st > 0 ? st : 0, en = st + (int64_t)sl, hi = en < (int64_t)a.cap ? en : (int64_t)a.cap;
  const bool some = lane < a.n_segs && hi > lo;
  const int len = some ? (int)(hi - lo) : 0, slot = some ? (int)lo : 0;
  int incl = len;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o, 64);
    incl += lane >= o ? y : 0;
  }
  const int shift = slot - (incl - len);
  const int S = a.S;
  const int SG = S + __builtin_amdgcn_readlane(incl, 63);      // sink and gathered keys
  const int tail0 = a.T - a.Lq;

  // ---- last visible key of this lane's rows, of the tile's first and last row
  auto last_key = [&](int t) __attribute__((always_inline)) { return SG + (a.bidir ? a.T - 1 : tail0 + t); };
  int key_lim[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) key_lim[rb] = last_key(tok[rb]);
  const int first_lim = last_key(min(rt * RT, NR - 1) / g);
  const int n_blocks = (last_key((min((rt + 1) * RT, NR) - 1) / g) + BK) / BK;
  const int b_lo = (int)((int64_t)n_blocks * part / a.parts);
  const int b_hi = (int)((int64_t)n_blocks * (part + 1) / a.parts);

  // ---- block loader
  const int rbytes = a.Hkv * D * 2;
  const int ka = 8 * (n >> 2) + (n & 3);                       // this lane's key of the first product; second: + 4
  const uint32_t k_off = (uint32_t)(kv * D * 2 + j * 16);
  const uint32_t v_off = (uint32_t)(kv * D * 2 + n * (VE * 2));
  // K in the wave's LDS: row r at r * RBY, its 16-byte unit u at u ^ swz(r), where swz(r) takes the row's
  // low bits and one above (16 lanes of a fragment read then touch all banks).  Load i brings rows of KR * i.
  constexpr int RBY = D * 2, KR = 512 / D, NKL = BK / KR;
  const int lr = lane / (RBY / 16), lu = lane % (RBY / 16);
  const uint32_t k_lane = STAGE ? (uint32_t)(lr * rbytes) : (uint32_t)(ka * rbytes) + k_off;
  const uint32_t k_unit = (uint32_t)((lu ^ lr) * 16);
  const int swz0 = n & (RBY / 16 - 1);
  char* const k_stage = (char*)&o_s[wave][0][0];
  const char* const k_frag = k_stage + ka * RBY;
  const uint32_t k_fu = (uint32_t)((swz0 ^ j) * 16);
  static_assert(BK * RBY <= RT * OS * 4, "the stage lies in the wave's part of the merge buffer");
  const uint32_t v_lane = (uint32_t)(8 * j * rbytes) + v_off;
  auto vload = [&](rsrc_t r, uint32_t off, uint32_t so) __attribute__((always_inline)) {
    if constexpr (VE == 8) return __builtin_amdgcn_raw_buffer_load_b128(r, off, so, 0);
    else return __builtin_amdgcn_raw_buffer_load_b64(r, off, so, 0);
  };
  auto load_block = [&](int b, u32x4 (&kr)[2][NKS], vrow_t (&vr)[8]) __attribute__((always_inline)) {
    const int k0 = b * BK, k1 = k0 + BK;
    // one tensor and consecutive rows: base + fixed per-lane offsets
    const uint16_t *bk = nullptr, *bv = nullptr;
    int rows = 0, row0 = 0;
    if (k1 <= S) {
      bk = a.sink_k; bv = a.sink_v; rows = S; row0 = k0;
    } else if (k0 >= SG) {
      if (k1 <= SG + a.T) { bk = a.tail_k; bv = a.tail_v; rows = a.T; row0 = k0 - SG; }
    } else if (k0 >= S && k1 <= SG) {
      const int i0 = k0 - S;
      const int s = __builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= i0));      // segment of key i0
      if (i0 + BK <= __builtin_amdgcn_readlane(incl, s)) {
        bk = a.store_k; bv = a.store_v; rows = a.cap;
        row0 = i0 + __builtin_amdgcn_readlane(shift, s);
      }
    }
    if (bk) {
      const rsrc_t rk = make_rsrc(bk, rows * rbytes), rv = make_rsrc(bv, rows * rbytes);
      const uint32_t so = (uint32_t)row0 * (uint32_t)rbytes;
      if constexpr (STAGE) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // the last block's fragments are read
#pragma unroll
        for (int i = 0; i < NKL; ++i) {
          const uint32_t x = D == 128 ? 64 * ((i ^ (i >> 1)) & 1) + 128 * (i >> 2) : 64 * (i & 1);
          load_lds16(rk, (lds_void*)(k_stage + i * 1024), k_lane + (k_unit ^ x), so + (uint32_t)(kv * RBY + i * KR * rbytes));
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < 8; ++i) vr[i] = vload(rv, v_lane, so + i * rbytes);
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");        // K is there; the 8 V loads may be under way
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int ks = 0; ks < NKS; ++ks)
            kr[h][ks] = *(const u32x4*)(k_frag + h * 4 * RBY + (k_fu ^ (uint32_t)(64 * (ks ^ h))));
      } else {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int ks = 0; ks < NKS; ++ks)
            kr[h][ks] = __builtin_amdgcn_raw_buffer_load_b128(rk, k_lane + ks * 64, so + h * 4 * rbytes, 0);
#pragma unroll
        for (int i = 0; i < 8; ++i) vr[i] = vload(rv, v_lane, so + i * rbytes);
      }
      return;
    }
    // a block across regions or segments: lane i resolves key k0 + i%32 (row,
    // and tensor in the top two bits; 3: past the tail), the lanes fetch their
    // rows' entries.  Past the tail the last tail row is read; its logits
    // are masked, its values are replaced by zeros.
    const int kk = k0 + (lane & 31), i = kk - S;
    int sh = 0;
    if (k1 > S && k0 < SG && SG > S) {     // wave-uniform: the segments that the block's keys reach
      int s = __builtin_popcountll(__builtin_amdgcn_ballot_w64(incl <= max(k0 - S, 0)));
      int begin = s > 0 ? __builtin_amdgcn_readlane(incl, s - 1) : 0;
      while (begin < min(k1, SG) - S) {
        const int end = __builtin_amdgcn_readlane(incl, s), d = __builtin_amdgcn_readlane(shift, s);
        sh = i >= begin && i < end ? d : sh;
        begin = end;
        ++s;
      }
    }
    const uint32_t where = kk < S ? (uint32_t)kk : kk < SG ? (uint32_t)(i + sh) | (1u << 30)
                         : kk < SG + a.T ? (uint32_t)(kk - SG) | (2u << 30) : (uint32_t)(a.T - 1) | (3u << 30);
    typedef const __attribute__((address_space(1))) char* gptr;
    auto row_of = [&](int key, const uint16_t* sink, const uint16_t* store, const uint16_t* tail, uint32_t unit,
                      bool& real) __attribute__((always_inline)) {
      const uint32_t w = (uint32_t)__shfl((int)where, key, 64), t = w >> 30;
      real = t != 3;
      const uint16_t* base = t == 0 ? sink : t == 1 ? store : tail;
      return (gptr)base + ((uint64_t)(w & 0x3FFFFFFFu) * (uint32_t)rbytes + unit);
    };
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bool real;
      const gptr p = row_of(ka + 4 * h, a.sink_k, a.store_k, a.tail_k, k_off, real);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) kr[h][ks] = *(const __attribute__((address_space(1))) u32x4*)(p + ks * 64);
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      bool real;
      const gptr p = row_of(8 * j + r, a.sink_v, a.store_v, a.tail_v, v_off, real);
      const vrow_t x = *(const __attribute__((address_space(1))) vrow_t*)p;
      vr[r] = real ? x : vrow_t{};
    }
  };

  // ---- running state: row n of each 16-row block, shared by the lanes n, n+16, n+32, n+48
  f32x4 o[NRB][VE];
  float m_run[NRB], l_run[NRB], neg_m[NRB];        // neg_m: -m_run, +inf while there is no max
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
#pragma unroll
    for (int e = 0; e < VE; ++e) o[rb][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run[rb] = -INFINITY;
    neg_m[rb] = INFINITY;
    l_run[rb] = 0.f;
  }
  const float c = a.scale_log2;

  auto compute_block = [&](int b, const u32x4 (&kr)[2][NKS], const vrow_t (&vr)[8]) __attribute__((always_inline)) {
    bf16x8 pf[NRB];
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
      f32x4 s[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        s[h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
          s[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kr[h][ks]), qf[rb][ks], s[h], 0, 0, 0);
      }
      if (b * BK + BK - 1 > first_lim) {
#pragma unroll
        for (int v = 0; v < 8; ++v)
          s[v / 4][v % 4] = b * BK + 8 * j + v > key_lim[rb] ? -INFINITY : s[v / 4][v % 4];
      }
      // probabilities against the running max; raised when a lane's sum of 8
      // (which bounds each) passes kLaneSumLimit, or there is no max yet
      float e[8], sum;
      auto expo = [&](float nm) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 8; ++v) e[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[v / 4][v % 4], c, nm));
        sum = ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
      };
      expo(neg_m[rb]);
      if (__builtin_amdgcn_ballot_w64(!(sum <= kLaneSumLimit))) {
        float mx = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                         fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float m_new = fmaxf(m_run[rb], mx * c);
        const float alpha = (m_new == m_run[rb]) ? 1.f : __builtin_amdgcn_exp2f(m_run[rb] - m_new);
        l_run[rb] *= alpha;
#pragma unroll
        for (int d = 0; d < VE; ++d) o[rb][d] *= alpha;
        m_run[rb] = m_new;
        neg_m[rb] = -m_new;
        expo(m_new == -INFINITY ? 0.f : -m_new);
      }
      l_run[rb] += sum;
#pragma unroll
      for (int v = 0; v < 8; ++v) pf[rb][v] = (__bf16)e[v];
    }
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      u32x4 w;           // value e of this lane's 8 keys
#pragma unroll
      for (int p = 0; p < 4; ++p)
        w[p] = __builtin_amdgcn_perm(vr[2 * p + 1][e / 2], vr[2 * p][e / 2], (e & 1) ? 0x07060302u : 0x05040100u);
      const bf16x8 vf = __builtin_bit_cast(bf16x8, w);
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) o[rb][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[rb], o[rb][e], 0, 0, 0);
    }
  };

  // ---- the wave's blocks.  (Loading the next block while one is computed was
  // measured 1-7 % slower: the other waves' loads fill the gap, and the
  // second set of registers only lengthens the start.)
  for (int b = b_lo + wave; b < b_hi; b += NW) {
    u32x4 kr[2][NKS];
    vrow_t vr[8];
    load_block(b, kr, vr);
    compute_block(b, kr, vr);
  }

  // ---- merge of the waves: O^T lane (n, j) holds row n, dims VE*(4j+i) + e
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    float l = l_run[rb];
    l += __shfl_xor(l, 16, 64);
    l += __shfl_xor(l, 32, 64);
    if (j == 0) {
      m_s[wave][rb * 16 + n] = m_run[rb];
      l_s[wave][rb * 16 + n] = l;
    }
    float* op = &o_s[wave][rb * 16 + n][VE * 4 * j];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < VE; e += 4)
        *(f32x4*)(op + i * VE + e) = f32x4{o[rb][e][i], o[rb][e + 1][i], o[rb][e + 2][i], o[rb][e + 3][i]};
  }
  __syncthreads();
  constexpr int NQ = D / 4;
  const int rows = min(RT, NR - rt * RT);
  for (int it = tid; it < rows * NQ; it += NW * 64) {
    const int r = it / NQ, dq = it % NQ;
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) m = fmaxf(m, m_s[w][r]);
    const float m_use = m == -INFINITY ? 0.f : m;
    float l = 0.f;
    f32x4 acc{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = __builtin_amdgcn_exp2f(m_s[w][r] - m_use);      // 0 for a wave that saw no key of the row
      l += f * l_s[w][r];
      acc += f * *(const f32x4*)&o_s[w][r][dq * 4];
    }
    acc *= l > 0.f ? 1.f / l : 0.f;
    const float lse2 = l > 0.f ? m_use + __log2f(l) : -INFINITY;
    const int pr = rt * RT + r, t = pr / g, h = kv * g + pr % g;
    if (a.parts > 1) {
      const int64_t prow = ((int64_t)part * a.Hq + h) * a.Lq + t;      // the merge kernel's layout
      *(f32x4*)(a.ws_o + prow * D + dq * 4) = acc;
      if (dq == 0) a.ws_lse[prow] = part_lse(l, lse2);
      continue;
    }
    const int64_t oo = ((int64_t)t * a.Hq + h) * D + dq * 4;
    if (a.out_f32) *(f32x4*)((float*)a.out + oo) = acc;
    else *(bf16x4*)((__bf16*)a.out + oo) = bf16x4{(__bf16)acc[0], (__bf16)acc[1], (__bf16)acc[2], (__bf16)acc[3]};
    if (dq == 0 && a.lse) a.lse[(int64_t)h * a.Lq + t] = lse2 * kLn2;
  }
}

template <int D>
hipError_t launch(const RowsArgs& a, hipStream_t stream) {
  const dim3 grid(a.n_rt * a.parts * a.Hkv + a.app_blocks);
  if (a.row_blocks == 1) {
    if (a.stage) hipLaunchKernelGGL((attn_rows_kernel<D, 1, 8, true>), grid, dim3(512), 0, stream, a);
    else hipLaunchKernelGGL((attn_rows_kernel<D, 1, 8, false>), grid, dim3(512), 0, stream, a);
  } else if (a.row_blocks == 2) {
    if (a.stage) hipLaunchKernelGGL((attn_rows_kernel<D, 2, 8, true>), grid, dim3(512), 0, stream, a);
    else hipLaunchKernelGGL((attn_rows_kernel<D, 2, 8, false>), grid, dim3(512), 0, stream, a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_rows(const RowsArgs& a, hipStream_t stream) {
  if (a.n_segs > kRowsMaxSegments || a.n_rt < 1 || a.parts < 1) return hipErrorInvalidValue;
  return a.D == 128 ? launch<128>(a, stream) : launch<64>(a, stream);
}

}  // namespace vico
