// Bounded chunk-prefill attention for gfx950 (CDNA4).
//
// Computes softmax(Q K^T / sqrt(d)) V for the rows of one visual chunk over
// the keys [sink | W newest history tokens (read through ring slots) |
// chunk keys 0..i] -- the bounded visual attention of ViCoStream (Sec. 3,
// "LLM Prefilling and Decoding"; visibility as in the vision rows of Eq. (4),
// at token granularity, causal inside the chunk).
//
// Mapping onto the hardware
//   * Work-group = 8 waves (two per SIMD, one work-group per CU) = 256 query
//     rows (one key range when split).  Each wave owns 32 rows for the whole
//     key loop; every K/V tile brought into LDS serves all 256 rows.  The
//     rows are 256 tokens of one query head, or packed (token, head) pairs
//     of all query heads of one KV head, token-major (row r: token r / g,
//     head kv*g + r % g) when that takes fewer row tiles: a chunk length
//     that is not a multiple of 256 leaves every query head's last row tile
//     part-empty, and packing leaves one part-filled row tile per KV head
//     instead.  Both forms read the same K/V; the packed one is its own
//     kernel, attn_fwd_packed_kernel.
//   * The tile body (S^T = K Q^T and O^T = V^T P^T on v_mfma_f32_32x32x16_bf16,
//     the exponentiate-first online softmax, software-pipelined over 32-key
//     halves) is PipeTile of attn_pipe.h.
//   * K/V tiles: 64 keys, four buffers each in LDS, loaded three tiles ahead
//     with one barrier per tile.  Loads go straight to LDS through buffer
//     resources: consecutive tiles inside one tensor (a run) share the
//     resource and advance a scalar offset; a tile that straddles two tensors
//     or the ring end resolves each key row (ring slot = ws + k, minus R once
//     past the end) and loads each tensor's rows with the other lanes switched
//     off.  Keys past the chunk end read as zero (out of range).  No copies.
//   * Causal chunk: only tiles that reach past the first row of a wave run the
//     mask on their logits, and a wave computes up to its last row's last tile;
//     from there it only takes part in the loads.  With the bidirectional option (Eq. (4) read
//     literally: a chunk sees all of itself) every row's last key is the
//     chunk's last key, so only the tile holding the chunk end is masked.
//   * Work-groups are renumbered so that consecutive logical ids (the query
//     heads, or the packed row tiles, of one KV head) land on the same XCD
//     and share its L2.
//   * Optional split of the key range (for chunks too small to fill 256 CUs):
//     each split writes fp32 O and log2-sum-exp; a merge kernel combines them.

#include <type_traits>

#include "attn_common.h"
#include "attn_pipe.h"

namespace vico {
namespace {

// The kernel body; PACKED selects the packed (token, head) rows.  Inlined
// into one kernel per row form (attn_fwd_kernel, attn_fwd_packed_kernel).
template <int D, bool PACKED>
__device__ __forceinline__ void attn_fwd_body(const AttnArgs& a, int n_rt, int gq) {
  constexpr int RB = kRowBlocks;
  typedef PipeTile<D, RB> Tile;
  constexpr int BN = kKeyTile;         // keys per tile
  constexpr int BM = kBlockM;          // rows per work-group
  constexpr int NW = kThreads / 64;          // waves per work-group
  // LDS tiles: dense rows of 2*D bytes (the direct loads below write each
  // wave's 64 x 16 bytes contiguously), units swizzled as the tile body reads them
  constexpr int UPR = Tile::UPR;       // 16-byte units per row
  constexpr int RBY = D * 2;           // bytes per LDS row
  constexpr uint32_t TBY = BN * RBY;         // bytes of one K (or V) tile
  constexpr int NLD = TBY / 1024 / NW;       // direct 1 KiB loads per wave per tile (K or V)
  constexpr int RPL = 1024 / RBY;            // rows per direct load
  constexpr int NDB = Tile::NDB, NKS = Tile::NKS;
  static_assert(NLD * NW * 1024 == TBY, "direct loads cover the tile");
  static_assert(BM == NW * RB * 32, "work-group rows");
  static_assert(BN == 64, "two 32-key halves per tile");

  // Tile t (counted from the segment's first) lives in K and V buffer t mod NB.
  // The pipelined body multiplies V one half after K, so with one barrier per
  // tile the loads run NB - 1 = AHEAD tiles ahead.  One array and one address
  // register per fragment kind, advanced once per tile: the direct loads are
  // assembly, so the compiler has no loads in flight to confuse with the reads.
  constexpr int NB = kBuffers, AHEAD = NB - 1;
  constexpr uint32_t kKBase = NB * TBY;
  __shared__ __attribute__((aligned(16))) uint8_t lds[2 * NB * TBY];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void*)lds;

  // ---- the append's share: slots that no work-group of this launch reads
  const int n_work = gridDim.x - a.app_blocks;
  if ((int)blockIdx.x >= n_work) {
    const AppendArgs ap{a.kc, a.vc, a.app_rk, a.app_rv, a.C, a.R, a.app_p0, a.Hkv * a.D};
    append_units(ap, (int64_t)(blockIdx.x - n_work) * kThreads + threadIdx.x, (int64_t)a.app_blocks * kThreads);
    return;
  }

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31;
  const int hh = lane >> 5;
  const int C = a.C, S = a.S, SW = a.S + a.Wv;
  const int P = PACKED ? a.pack : 1;   // query heads packed into the rows of a row tile
  const int NR = C * P;                // packed rows of one head group

  // last key visible to chunk token `tok`: its own position (causal), or the
  // chunk's last key when the chunk attends to itself bidirectionally
  auto last_key_of_tok = [&](int tok) __attribute__((always_inline)) {
    return SW + (a.bidir ? C - 1 : min(tok, C - 1));
  };
  // packed row r of a head group is chunk token r / P of query head (group
  // base) + r % P; rows past the group's end stand for its last row
  auto tok_of = [&](int r) __attribute__((always_inline)) { return min(r, NR - 1) / P; };
  // key tiles seen by row tile rt: keys up to its last row's last key
  auto tiles_of = [&](int rt) __attribute__((always_inline)) {
    return (last_key_of_tok(tok_of((rt + 1) * BM - 1)) + BN) / BN;
  };

  // ---- one segment of work: key tiles [t_lo, t_hi) of row tile rt of head
  // group qh of KV head kv (query heads kv*g + qh*P .. + P-1).  `partial`
  // segments write fp32 O and log2-sum-exp to workspace slot `part` (of
  // n_parts) for the merge kernel; others write the output.  All waves of the
  // work-group run the same segments.
  auto segment = [&](int kv, int rt, int qh, int t_lo, int t_hi, int part, int n_parts, bool partial)
      __attribute__((always_inline)) {
  const int h0 = (kv * gq + qh) * P;
  const int row0 = rt * BM;
  const int n_tiles = tiles_of(rt);

  // this wave: packed rows wrow0 .. wrow0 + 31 in one block (RB); this lane:
  // token tok[rb] of head h[rb] in each block
  const int wrow0 = row0 + wave * (RB * 32);
  const bool wave_active = wrow0 < NR;
  const int wave_first_lim = last_key_of_tok(tok_of(wrow0));      // last key of the wave's first row
  // the wave computes tiles [t_lo, t_end): past its last row's last key it only
  // keeps loading for the others (P = 0 there is not enough: 0 times an
  // infinite or NaN value of a later token is NaN)
  const int t_end =
      wave_active ? min(t_hi, last_key_of_tok(tok_of(wrow0 + RB * 32 - 1)) / BN + 1) : t_lo;
  int tok[RB], h[RB], key_lim[RB];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    const int r = min(wrow0 + rb * 32 + l32, NR - 1);
    tok[rb] = r / P;
    h[rb] = h0 + r % P;
    key_lim[rb] = last_key_of_tok(tok[rb]);
  }

  // ---- the wave's Q rows and running state.  The Q loads are unconditional:
  // rows past the group's end repeat its last row (the clamped address) and
  // are never stored, and a row's softmax only mixes the two lanes of that row.
  bf16x8 qf[RB][NKS];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) WaveTile<D>::load_q(qf[rb], a.q + ((int64_t)tok[rb] * a.Hq + h[rb]) * D + hh * 8);

  // ---- tile loader.  Direct load n of wave w fills chunk w*NLD + n of the tile
  // (RPL rows); the layout says which row and unit each lane fetches.  The
  // byte offset is counted from the tile's first row, less n * 1024: a load's
  // immediate offset counts on both sides, in LDS (where load n belongs
  // n * 1024 further on) and in memory.  Not negative: row n * RPL starts at
  // least n * 1024 bytes into the tile.
  const int rbytes = a.Hkv * D * 2;                            // bytes per token row in HBM
  auto k_row = [&](int n, int& unit) __attribute__((always_inline)) {
    int row;
    Tile::k_source(wave * NLD + n, lane, row, unit);
    return (wave * NLD + n) * RPL + row;
  };
  auto v_row = [&](int n, int& unit) __attribute__((always_inline)) {
    int row;
    Tile::v_source(lane, row, unit);
    return (wave * NLD + n) * RPL + row;
  };
  uint32_t ld_k[NLD], ld_v[NLD];
#pragma unroll
  for (int n = 0; n < NLD; ++n) {
    int unit;
    const int rk = k_row(n, unit);
    ld_k[n] = (uint32_t)(rk * rbytes + kv * D * 2 + unit * 16 - n * 1024);
    const int rv = v_row(n, unit);
    ld_v[n] = (uint32_t)(rv * rbytes + kv * D * 2 + unit * 16 - n * 1024);
  }

  // A run of tiles that lie in one tensor, without a ring end: their loads
  // share the two buffer resources and differ in the scalar offset.  run_left
  // counts the tiles left in it.  A tile across a boundary (mixed) is a run
  // of one with empty resources (its direct loads then read nothing), to be
  // filled by load_tile_rows; past the segment's last tile the run is empty
  // and endless, so every step issues the same number of loads.
  u32x4 run_k, run_v;
  uint32_t run_so;
  int run_left;
  bool mixed;
  auto start_run = [&](int t) __attribute__((always_inline)) {
    const int k0 = t * BN;
    const uint16_t *bk = a.kc, *bv = a.vc;
    int rows = 0, row0 = 0, n = 1;           // tensor rows, the tile's first row, tiles in the run
    mixed = false;
    if (t >= t_hi) {
      n = 1 << 30;
    } else if (k0 + BN <= S) {
      bk = a.sink_k; bv = a.sink_v;
      rows = S; row0 = k0;
      n = (S - k0) / BN;
    } else if (k0 >= SW && k0 + BN <= SW + C) {
      rows = C; row0 = k0 - SW;
      n = (SW + C - k0) / BN;
    } else {
      int slot0 = a.ws + (k0 - S);
      if (slot0 >= a.R) slot0 -= a.R;
      if (k0 >= S && k0 + BN <= SW && slot0 + BN <= a.R) {
        bk = a.ring_k; bv = a.ring_v;
        rows = a.R; row0 = slot0;
        n = min(SW - k0, a.R - slot0) / BN;
      } else {
        mixed = true;
      }
    }
    const uint64_t pk = (uint64_t)bk, pv = (uint64_t)bv;
    run_k = u32x4{(uint32_t)pk, (uint32_t)(pk >> 32) & 0xFFFFu, (uint32_t)(rows * rbytes), 0x00020000u};
    run_v = u32x4{(uint32_t)pv, (uint32_t)(pv >> 32) & 0xFFFFu, (uint32_t)(rows * rbytes), 0x00020000u};
    run_so = (uint32_t)row0 * (uint32_t)rbytes;
    run_left = n;
  };

  // direct load n (0 .. NLD-1: K, NLD .. 2*NLD-1: V) of the run's tile to the
  // buffers at byte offset `boff`.  m0 holds a load's LDS address.  The compiler
  // has m0 for itself (it takes no claim of it), so every load sets it and gives
  // it back.  The loads have no result registers.  Wait states that the compiler
  // does not know assembly to need: one after a write of m0, five after a VALU
  // write of a scalar operand (the reload of a scalar kept in a VGPR lane is one).
  const uint32_t my_part = (uint32_t)(wave * NLD * 1024);
  auto load_direct = [&](auto idx, uint32_t boff) __attribute__((always_inline)) {
    constexpr int i = decltype(idx)::value, n = i % NLD;
    const uint32_t off = i < NLD ? ld_k[n] : ld_v[n], so = run_so;
    const uint32_t to = lds0 + my_part + boff + (i < NLD ? kKBase : 0u);
    const u32x4 rs = i < NLD ? run_k : run_v;
    uint32_t m0;
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %5\n\ts_nop 4\n\t"
        "buffer_load_dwordx4 %1, %2, %3 offen offset:%4 lds\n\ts_mov_b32 m0, %0"
        : "=&s"(m0)
        : "v"(off), "s"(rs), "s"(so), "n"(n * 1024), "s"(to)
        : "memory");
  };

  // mixed tiles: each lane resolves its key row and the row's tensor; one
  // direct load per tensor, for that tensor's lanes only (a lane that does not
  // take part leaves its 16 bytes of LDS alone).  Rows past the chunk's end
  // are read out of range, as zeros.  The lanes are switched off inside the
  // assembly: the surrounding code has no divergent branch.
  auto load_tile_rows = [&](uint32_t boff, int t) __attribute__((always_inline)) {
    const int k0 = t * BN;
    auto from = [&](const uint16_t* p, int n, int row, uint32_t unit_off, bool take, uint32_t to)
        __attribute__((always_inline)) {
      const uint64_t lanes = __builtin_amdgcn_ballot_w64(take);
      if (lanes == 0) return;
      const uint64_t u = (uint64_t)p;
      const u32x4 rs = u32x4{(uint32_t)u, (uint32_t)(u >> 32) & 0xFFFFu, (uint32_t)(n * rbytes), 0x00020000u};
      uint64_t all;
      uint32_t m0;
      asm volatile(
          "s_mov_b64 %0, exec\n\ts_mov_b32 %1, m0\n\ts_mov_b64 exec, %2\n\ts_mov_b32 m0, %3\n\ts_nop 4\n\t"
          "buffer_load_dwordx4 %4, %5, 0 offen lds\n\ts_mov_b32 m0, %1\n\ts_mov_b64 exec, %0"
          : "=&s"(all), "=&s"(m0)
          : "s"(lanes), "s"(to), "v"((uint32_t)row * (uint32_t)rbytes + unit_off), "s"(rs)
          : "memory");
    };
    auto rows = [&](const uint16_t* sink, const uint16_t* ring, const uint16_t* chunk, int kk, uint32_t unit_off, uint32_t to)
        __attribute__((always_inline)) {
      int slot = a.ws + (kk - S);
      slot = slot >= a.R ? slot - a.R : slot;
      from(sink, S, kk, unit_off, kk < S, to);
      from(ring, a.R, slot, unit_off, kk >= S && kk < SW, to);
      from(chunk, C, kk - SW, unit_off, kk >= SW, to);
    };
#pragma unroll 1
    for (int n = 0; n < NLD; ++n) {
      int unit;
      const int rk = k_row(n, unit);
      const uint32_t to = lds0 + my_part + boff + n * 1024;
      rows(a.sink_k, a.ring_k, a.kc, k0 + rk, (uint32_t)(kv * D * 2 + unit * 16), to + kKBase);
      const int rv = v_row(n, unit);
      rows(a.sink_v, a.ring_v, a.vc, k0 + rv, (uint32_t)(kv * D * 2 + unit * 16), to);
    }
  };

  // ---- key loop.  Step t multiplies S of tile t's second half and of tile
  // t+1's first half, P V of tile t-1's second half and of tile t's first.
  // The barrier between the two halves certifies tile t+1 and frees V of tile
  // t-1 (last read in this step's first half), whose buffers take tile
  // t+AHEAD; its loads go out one by one in the slots of the second half.
  constexpr int NL = 2 * NLD;                      // direct loads per wave and tile
  constexpr int LSTEP = (Tile::NSLOT - 2) / (NL + 1);      // slots between two of them
  static_assert(LSTEP >= 1, "a tile's loads fit a body's slots");
  // Tile t+1 has landed (the loads of the AHEAD-2 tiles after it may be in
  // flight), for this wave and every other.  (Not __syncthreads(): that would
  // wait for all of them, and for the fragment reads.)
  auto landed = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"((AHEAD - 2) * NL) : "memory");
  };
  // the rest of a tile's load, after its direct loads
  auto finish_load = [&](uint32_t boff, int t) __attribute__((always_inline)) {
    run_so += (uint32_t)(BN * rbytes);
    if (__builtin_expect(--run_left == 0, 0)) {
      if (mixed) load_tile_rows(boff, t);
      start_run(t + 1);
    }
  };
  auto load_whole = [&](uint32_t boff, int t) __attribute__((always_inline)) {
    unrolled<2 * NLD>([&](auto i) __attribute__((always_inline)) { load_direct(i, boff); });
    finish_load(boff, t);
  };

  f32x16 o[RB][NDB];
  float m_run[RB], l_run[RB], neg_m[RB];
  uint32_t k_rd[2], v_rd, v_nx;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
    for (int db = 0; db < NDB; ++db) o[rb][db] = f32x16{};
    m_run[rb] = -INFINITY;
    neg_m[rb] = INFINITY;
    l_run[rb] = 0.f;
  }
  Tile::start(k_rd, v_nx);
  k_rd[0] += lds0 + kKBase;                        // tile 0 of the segment: buffer 0
  k_rd[1] += lds0 + kKBase;
  v_nx += lds0;
  v_rd = v_nx + (NB - 1) * TBY;                    // the tile before it: the last buffer
  if (t_lo < t_hi) {
    start_run(t_lo);
#pragma unroll 1
    for (int i = 0; i < AHEAD; ++i) load_whole(i * TBY, t_lo + i);
    // the pipeline's first P V multiplies zero probabilities with the last 16
    // rows of the last V buffer: any bits there must be finite
    if (tid < 16 * UPR)
      *(__attribute__((address_space(3))) u32x4*)(uintptr_t)(lds0 + (NB - 1) * TBY + 48 * RBY + tid * 16) =
          u32x4{0, 0, 0, 0};
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((AHEAD - 1) * NL) : "memory");   // tile t_lo
    uint32_t boff = 0;                             // buffer offset of tile t
    constexpr uint32_t kWrap = NB * TBY - 1;
    static_assert((NB & (NB - 1)) == 0, "buffer offsets wrap by a mask");
    int t = t_lo;
    if (t < t_end) {
      bf16x8 vf[NDB] = {};
      Tile wt{qf, k_rd, v_rd, v_nx, o, m_run, l_run, neg_m, vf, a.scale_log2};
      f32x16 s0[RB], s1[RB];
      bf16x8 p0[RB][2] = {}, p1[RB][2] = {};
      wt.first_logits(s0);
      const int t_mask = wave_first_lim < 63 ? 0 : (wave_first_lim - 63) / BN + 1;   // tiles from here on may need the mask
      if (t_lo >= t_mask) Tile::mask(t_lo * BN, key_lim, hh, s0);
      wt.first_max(s0);
      for (; t < t_end; ++t) {
        if (__builtin_expect(t >= t_mask, 0)) Tile::mask(t * BN, key_lim, hh, s0);
        uint32_t next = 0;                         // of tile t+1
        wt.template half<32, 48, 0>(s0, s1, p1, p0, [&](auto slot) __attribute__((always_inline)) {
          constexpr int s = decltype(slot)::value;
          if constexpr (s == Tile::NQK + Tile::NPV) {
            next = (boff + TBY) & kWrap;
            k_rd[0] += next - boff;                // K of tile t+1
            k_rd[1] += next - boff;
            v_rd = v_nx;                           // V of tile t
          }
        });
        landed();
        if (__builtin_expect(t >= t_mask, 0)) Tile::mask(t * BN + 32, key_lim, hh, s1);
        const uint32_t fill = (boff + AHEAD * TBY) & kWrap;
        wt.template half<0, 16, 32>(s1, s0, p0, p1, [&](auto slot) __attribute__((always_inline)) {
          constexpr int s = decltype(slot)::value, i = s / LSTEP - 1;
          if constexpr (s % LSTEP == 0 && i >= 0 && i < NL) load_direct(std::integral_constant<int, i>{}, fill);
        });
        v_nx += next - boff;                       // V of tile t+1
        boff = next;
        finish_load(fill, t + AHEAD);
      }
      // V of the wave's last tile is read here, before the barrier of the step that reuses its buffer
      wt.template last_values<48>(p1);
    }
    for (; t < t_hi; ++t) {
      landed();
      load_whole((boff + AHEAD * TBY) & kWrap, t + AHEAD);
      boff = (boff + TBY) & kWrap;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the empty loads past the last tile
  }

  if (!wave_active) return;
#pragma unroll
  for (int rb = 0; rb < RB; ++rb) {
    // row totals over the two lanes of a row
    const float l_tot = pair_sum(l_run[rb]);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;                              // 0 for an empty row
    const float lse2 = l_tot > 0.f ? m_run[rb] + __log2f(l_tot) : -INFINITY;
    if (wrow0 + rb * 32 + l32 >= NR) continue;
    const int row = tok[rb], hd = h[rb];
    if (partial || a.out_f32) {
      float* op = partial ? a.ws_o + (((int64_t)part * a.Hq + hd) * C + row) * D
                          : (float*)a.out + ((int64_t)row * a.Hq + hd) * D;
      op += hh * 4;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const f32x16& x = o[rb][db];
          *(f32x4*)(op + db * 32 + q4 * 8) =
              f32x4{x[q4 * 4] * inv, x[q4 * 4 + 1] * inv, x[q4 * 4 + 2] * inv, x[q4 * 4 + 3] * inv};
        }
    } else {
      __bf16* op = (__bf16*)a.out + ((int64_t)row * a.Hq + hd) * D + hh * 4;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const f32x16& x = o[rb][db];
          *(bf16x4*)(op + db * 32 + q4 * 8) =
              bf16x4{(__bf16)(x[q4 * 4] * inv), (__bf16)(x[q4 * 4 + 1] * inv), (__bf16)(x[q4 * 4 + 2] * inv),
                     (__bf16)(x[q4 * 4 + 3] * inv)};
        }
    }
    if (hh != 0) continue;
    if (!partial) {
      if (a.lse) a.lse[(int64_t)hd * C + row] = lse2 * kLn2;
    } else {
      a.ws_lse[((int64_t)part * a.Hq + hd) * C + row] = part_lse(l_tot, lse2);
      // a row tile that ends in this segment uses no later parts
      if (t_hi == n_tiles)
        for (int p2 = part + 1; p2 < n_parts; ++p2) a.ws_lse[((int64_t)p2 * a.Hq + hd) * C + row] = -INFINITY;
    }
  }
  };   // segment

  // ---- schedule
  const int L = xcd_remap(blockIdx.x, n_work);
  if (!a.balanced) {
    // one row tile (one key range of it when split) per work-group
    const int qh = L % gq;
    int rest = L / gq;
    const int rt = n_rt - 1 - rest % n_rt;   // longest row tiles first
    rest /= n_rt;
    const int sp = rest % a.splits;
    const int kv = rest / a.splits;
    const int nt = tiles_of(rt);
    const int t_lo = (int)((int64_t)nt * sp / a.splits);
    const int t_hi = (int)((int64_t)nt * (sp + 1) / a.splits);
    segment(kv, rt, qh, t_lo, t_hi, sp, a.splits, a.splits > 1);
  } else {
    // Balanced: the (row tile, key tile) pairs of all row tiles, in the order
    // kv, row tile (longest first), head group, are cut into gridDim.x equal
    // ranges.  A row tile cut between work-groups is finished by the merge
    // kernel; part = index of the work-group among those covering it.
    const int64_t G = n_work, T = a.total_tiles;
    int64_t pos = (int64_t)L * T / G;
    const int64_t end = (int64_t)(L + 1) * T / G;
    bool first = true;
    while (pos < end) {
      int64_t base = 0;
      int kv = 0, rt = 0, qh = 0, nt = 1;
      for (int k = 0; k < a.Hkv; ++k)
        for (int ri = 0; ri < n_rt; ++ri) {
          const int r = n_rt - 1 - ri;
          const int n = tiles_of(r);
          const int64_t blk = (int64_t)gq * n;
          if (pos >= base && pos < base + blk) {
            kv = k; rt = r; nt = n; qh = (int)((pos - base) / n);
          }
          base += blk;
        }
      // start of the containing row tile in the global order
      int64_t task_start = 0;
      for (int k = 0; k < kv; ++k)
        for (int ri = 0; ri < n_rt; ++ri) task_start += (int64_t)gq * tiles_of(ri);
      for (int ri = 0; ri < n_rt - 1 - rt; ++ri) task_start += (int64_t)gq * tiles_of(n_rt - 1 - ri);
      task_start += (int64_t)qh * nt;
      const int lo = (int)(pos - task_start);
      const int hi = (int)(min(end, task_start + nt) - task_start);
      const int owner = (int)(((task_start + 1) * G - 1) / T);   // work-group holding the row tile's first key tile
      if (!first) __syncthreads();      // the previous segment is done with the LDS buffers
      segment(kv, rt, qh, lo, hi, L - owner, a.splits, true);
      first = false;
      pos = task_start + hi;
    }
  }
}

template <int D>
__global__ __launch_bounds__(kThreads, kWgPerCU) void attn_fwd_kernel(AttnArgs a, int n_rt, int gq) {
  attn_fwd_body<D, false>(a, n_rt, gq);
}

template <int D>
__global__ __launch_bounds__(kThreads, kWgPerCU) void attn_fwd_packed_kernel(AttnArgs a, int n_rt, int gq) {
  attn_fwd_body<D, true>(a, n_rt, gq);
}

}  // namespace

hipError_t launch_attention(const AttnArgs& a, int grid, hipStream_t stream) {
  const int g = a.Hq / a.Hkv;
  if (a.pack < 1 || g % a.pack != 0) return hipErrorInvalidValue;
  const int gq = g / a.pack;
  const int n_rt = (int)(((int64_t)a.C * a.pack + kBlockM - 1) / kBlockM);
  const dim3 gr(grid + a.app_blocks), bl(kThreads);
  if (a.pack == 1) {
    if (a.D == 128) hipLaunchKernelGGL(attn_fwd_kernel<128>, gr, bl, 0, stream, a, n_rt, gq);
    else hipLaunchKernelGGL(attn_fwd_kernel<64>, gr, bl, 0, stream, a, n_rt, gq);
  } else {
    if (a.D == 128) hipLaunchKernelGGL(attn_fwd_packed_kernel<128>, gr, bl, 0, stream, a, n_rt, gq);
    else hipLaunchKernelGGL(attn_fwd_packed_kernel<64>, gr, bl, 0, stream, a, n_rt, gq);
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (a.splits > 1) return launch_merge(a, stream);   // appends too, when asked
  if (!a.app_rk || a.app_blocks > 0) return err;
  const AppendArgs ap{a.kc, a.vc, a.app_rk, a.app_rv, a.C, a.R, a.app_p0, a.Hkv * a.D};
  return launch_append(ap, stream);
}

}  // namespace vico
