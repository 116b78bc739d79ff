// The tile body of the chunk-prefill kernels (gfx950): a wave's query rows
// against K/V tiles in LDS, as one software-pipelined instruction stream.
//
// Why this form.  A wave that multiplies, exponentiates and multiplies again
// leaves the matrix cores idle while it exponentiates, and the second wave of
// the SIMD fills only part of that: a 64-key tile took 3600 engine cycles for
// 2112 cycles of MFMA work.  Here one loop body holds three independent
// pieces of work on 32 keys ("half j" of a tile):
//     S(j+1) = K Q^T        the next half's logits        (MFMA)
//     O     += V^T P(j-1)   the previous half's values    (MFMA)
//     P(j)   = exp2(S(j))   this half's probabilities     (VALU)
// The body is cut into slots of one MFMA each (16 at head size 128 and one
// 32-row block); every slot carries its share of the exponentials, sums and
// packing and the LDS reads of a later MFMA, so that the VALU and LDS work
// issues in the shadow of the 32-cycle MFMAs.  A tile then takes 2785 cycles;
// the clock falls from 2.15 to 1.8-1.9 GHz (the chip is at its power limit),
// which leaves 6-9 % on long key ranges: 7B chunk (28/4 heads, 16384 keys +
// 2048) 482 -> 450 us, 3B heads over 65536 keys 975 -> 909 us.
//
// Registers.  The compiler's own choice is all MFMA results in one kind of
// register, which copies either the logits (read by the VALU) or O back and
// forth, or spills.  So the MFMAs are written as assembly with O and the Q
// fragments in accumulation registers and the logits in VGPRs.  The compiler
// knows neither that these are MFMAs nor their wait states, hence the rules
// below:
//   * VALU reads of an MFMA result need up to 18 wait states.  Logits: all of
//     a body's Q K^T slots are followed by the P V slots of the second 16
//     keys (2 to 8 MFMAs of 8 wait states and the VALU work of their slots)
//     before the next body reads them.  O: settle() around VALU accesses.
//   * MFMA reads of a VALU result need 2 wait states: P is packed in the body
//     before the one that multiplies it; K and V fragments come from LDS (the
//     compiler waits for those, also in front of assembly); settle() after
//     every VALU write of O.
//   * No divergent branch between the first and the last of these MFMAs: a
//     register copy that the compiler puts at the join, before the lanes are
//     switched on again, reaches only some of them.  Masks are selects, a tile's
//     rows are loaded with the lanes switched off inside the assembly
//     (load_tile_rows), and every other branch of the key loop is wave-uniform.
//     The kernel's two branches on lanes lie outside: the zeroing of a V buffer
//     before the loop (whole waves) and the stores after settle().
#pragma once

#include <type_traits>
#include <utility>

#include "attn_common.h"

namespace vico {

template <int N, class F, int... I>
__device__ __forceinline__ void unrolled_(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(0), f(1), ... f(N-1) with compile-time indexes
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled_<N>(f, std::make_integer_sequence<int, N>{});
}

// O += A B with O in accumulation registers
__device__ __forceinline__ void mfma_o(f32x16& o, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(o) : "v"(a), "v"(b));
}
// S = A B and S += A B with B (the Q fragment) in accumulation registers
__device__ __forceinline__ void mfma_s_first(f32x16& s, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(s) : "v"(a), "a"(b));
}
__device__ __forceinline__ void mfma_s(f32x16& s, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(s) : "v"(a), "a"(b));
}

// Keeps the computation of x where it is written (in its slot).
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }

template <int D, int RB>                            // RB: 32-row blocks of the wave
struct PipeTile {
  static constexpr int NKS = D / 16;                 // k-steps of Q K^T
  static constexpr int NDB = D / 32;                 // 32-dim blocks of O^T
  static constexpr int RBY = D * 2;                  // bytes per LDS row
  static constexpr int NPV = NDB * RB;               // MFMAs of P V over 16 keys
  static constexpr int NQK = NKS * RB;               // MFMAs of Q K^T over 32 keys
  static constexpr int NSLOT = 2 * NPV + NQK;
  static constexpr int NE = 16 * RB;                 // probabilities per lane of a half
  // slot s exponentiates elements first_e(s) .. first_e(s+1)-1: all done
  // two slots before the body's end, where the check of the sums follows
  // (one element per slot: two in the first two slots, then one)
  static constexpr int first_e(int s) {
    return s <= 0 ? 0 : s >= NSLOT - 2 ? NE : NE == NSLOT ? (s == 1 ? 2 : s + 2) : s * NE / (NSLOT - 2);
  }

  // The wave's state lives in the kernel as locals (as in WaveTile).
  bf16x8 (&qf)[RB][NKS];       // Q rows
  uint32_t (&k_rd)[2];         // LDS addresses of the lane's K fragments (even, odd k-steps), current K buffer
  uint32_t& v_rd;              //   and of its V^T fragments, V buffer of the tile whose P is multiplied
  uint32_t& v_nx;              //   V buffer of the current tile
  f32x16 (&o)[RB][NDB];        // O^T accumulators
  float (&m_run)[RB];          // running max (log2 units) of the lane's row of each block
  float (&l_run)[RB];          // the lane's sum of probabilities
  float (&neg_m)[RB];          // -m_run (so +inf, which makes every probability inf or NaN, while there is no max)
  bf16x8 (&vf)[NDB];           // V^T fragments of the next 16 keys to multiply
  const float c;               // softmax scale * log2(e)

  // LDS layout of a tile: chunks of 1024 bytes (what one direct load of a wave
  // writes) with RPC rows each, arranged so that a fragment read has no bank
  // conflict (64 banks of 4 bytes) and all fragments of a tile are immediate
  // offsets from one or two addresses.
  //   K: 16-byte unit u of row r at slot u ^ (chunk mod CPB), row r mod RPC
  //      inside the slot; a read takes one unit of 16 consecutive rows = CPB
  //      chunks, whose slots the XOR makes distinct.
  //   V: 64-byte segments, segment-major: a transposing read takes one segment
  //      of 4 consecutive rows, 256 contiguous bytes.
  static constexpr int RPC = 1024 / RBY;             // rows per chunk
  static constexpr int CPB = 16 / RPC;               // chunks per 16 rows
  static constexpr int UPR = D / 8;                  // 16-byte units per row
  static __device__ __forceinline__ void start(uint32_t (&krd)[2], uint32_t& vrd) {
    const int lane = threadIdx.x & 63, l32 = lane & 31, hh = lane >> 5;
    const int c = l32 / RPC;
#pragma unroll
    for (int odd = 0; odd < 2; ++odd)
      krd[odd] = (uint32_t)(c * 1024 + ((2 * odd + hh) ^ (c & (CPB - 1))) * (RPC * 16) + (l32 % RPC) * 16);
    // lane 4j+q of 16-lane group G supplies key (G/2)*4 + j, dims (G%2)*16 + 4q .. +3 of the segment's 32
    const int r = hh * 4 + ((lane & 15) >> 2);
    vrd = (uint32_t)(r / RPC * 1024 + (r % RPC) * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8);
  }
  // which row of its chunk and which unit of the row lane `lane` of a direct load fetches
  static __device__ __forceinline__ void k_source(int chunk, int lane, int& row, int& unit) {
    row = lane % RPC;
    unit = (lane / RPC) ^ (chunk & (CPB - 1));
  }
  static __device__ __forceinline__ void v_source(int lane, int& row, int& unit) {
    row = (lane / 4) % RPC;
    unit = lane / (4 * RPC) * 4 + lane % 4;
  }
  // K fragment of k-step ks, rows KR .. KR+31; V^T fragment of 32-dim block db, rows VR .. VR+15
  template <int KR>
  __device__ __forceinline__ bf16x8 read_k(int ks) const {
    const uint32_t a = k_rd[ks & 1] + KR * RBY + (ks >> 1) * (4 * RPC * 16);
    return *(const __attribute__((address_space(3))) bf16x8*)(uintptr_t)a;
  }
  template <int VR>
  static __device__ __forceinline__ bf16x8 read_v(uint32_t v, int db) {
    const uint32_t a = v + VR * RBY + db * (RPC * 64);
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(uintptr_t)a);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(uintptr_t)(a + 8 * RBY));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }

  // Logits of the first half (nothing to overlap with yet).
  __device__ __forceinline__ void first_logits(f32x16 (&s)[RB]) const {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      mfma_s_first(s[rb], read_k<0>(0), qf[rb][0]);
#pragma unroll
      for (int ks = 1; ks < NKS; ++ks) mfma_s(s[rb], read_k<0>(ks), qf[rb][ks]);
    }
    asm volatile("s_nop 15\n\ts_nop 7");
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) asm volatile("" : "+v"(s[rb]));
  }

  // Causal mask of a half: see WaveTile::mask_half.
  static __device__ __forceinline__ void mask(int k0h, const int (&key_lim)[RB], int hh, f32x16 (&s)[RB]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) WaveTile<D>::mask_half(k0h, key_lim[rb], hh, s[rb]);
  }

  // The running max from the first half's logits (nothing to rescale yet), so
  // that the first half needs no raise().
  __device__ __forceinline__ void first_max(const f32x16 (&s)[RB]) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[rb][v]);
      m_run[rb] = pair_max(mx) * c;
      neg_m[rb] = -m_run[rb];
    }
  }

  // Wait states between MFMA writes of O and VALU accesses to it, and back.
  __device__ __forceinline__ void settle() const {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int db = 0; db < NDB; ++db) asm volatile("" : "+a"(o[rb][db]));
    asm volatile("s_nop 15\n\ts_nop 7");
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int db = 0; db < NDB; ++db) asm volatile("" : "+a"(o[rb][db]));
  }

  // One loop body: sn = logits of the next half (keys at LDS row KR of the K
  // buffer k_rd points to), O += the previous half (probabilities pp; its first
  // 16 keys' V fragments are in vf, its second 16 keys at row VR of v_rd), pc =
  // probabilities of the logits sc; vf = V fragments at row NR of v_nx.
  // Probabilities are taken against the running max; when a lane's sum of them
  // (which bounds each) passes kLaneSumLimit, or a row has no max yet, raise()
  // redoes them.
  // side(s) adds the kernel's own work to slot s.  k_rd has been read for the
  // last time in slot NQK - RB, v_rd in slot NQK + NPV - RB, v_nx in slot
  // NSLOT - RB.
  template <int KR, int VR, int NR, class Side>
  __device__ __forceinline__ void half(const f32x16 (&sc)[RB], f32x16 (&sn)[RB], const bf16x8 (&pp)[RB][2],
                                       bf16x8 (&pc)[RB][2], Side&& side) {
    float y[NE], x[NE], sum[RB][2];
    uint32_t pw[RB][2][4];
    bf16x8 kf[NKS], v2[NDB];
    float ls[RB], total;
    unrolled<NSLOT>([&](auto slot) __attribute__((always_inline)) {
      constexpr int s = decltype(slot)::value;
      {
        // fragments are read NPV slots before the MFMAs that use them
        if constexpr (s % RB == 0) {
          if constexpr (s < NQK) kf[s / RB] = read_k<KR>(s / RB);
          else if constexpr (s < NQK + NPV) v2[(s - NQK) / RB] = read_v<VR>(v_rd, (s - NQK) / RB);
        }
        if constexpr (s < NPV) {
          mfma_o(o[s % RB][s / RB], vf[s / RB], pp[s % RB][0]);
        } else if constexpr (s < NPV + NQK) {
          constexpr int q = s - NPV;
          if constexpr (q < RB) mfma_s_first(sn[q], kf[0], qf[q][0]);
          else mfma_s(sn[q % RB], kf[q / RB], qf[q % RB][q / RB]);
        } else {
          constexpr int q = s - NPV - NQK;
          mfma_o(o[q % RB][q / RB], v2[q / RB], pp[q % RB][1]);
          if constexpr (q % RB == 0) vf[q / RB] = read_v<NR>(v_nx, q / RB);
        }
        side(slot);
      }
      // softmax, one stage per slot: scaled logits, then exponentials, then
      // sums, then packing, so that no instruction waits for the one before it
      constexpr int e0 = first_e(s), e1 = first_e(s + 1), e2 = first_e(s + 2), em = first_e(s - 1),
                    ep = first_e(s - 2);
#pragma unroll
      for (int e = s == 0 ? 0 : e1; e < (s == 0 ? e1 : 0); ++e) y[e] = __builtin_fmaf(sc[e / 16][e % 16], c, neg_m[e / 16]);
#pragma unroll
      for (int e = e1; e < e2; ++e) {
        y[e] = __builtin_fmaf(sc[e / 16][e % 16], c, neg_m[e / 16]);
        pin(y[e]);
      }
#pragma unroll
      for (int e = em; e < e0; ++e) {
        float& a = sum[e / 16][e & 1];
        a = e % 16 < 2 ? x[e] : a + x[e];
        if (e % 16 >= 2) pin(a);
      }
#pragma unroll
      for (int e = ep; e < (s == NSLOT - 1 ? e0 : em); ++e)
        if (e & 1) {      // the pair's sums were a slot ago: packed in the slots without an LDS read
          typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
          uint32_t& w = pw[e / 16][(e % 16) / 8][(e % 8) / 2];
          w = __builtin_bit_cast(uint32_t, bf16x2{(__bf16)x[e - 1], (__bf16)x[e]});
          asm volatile("" : "+v"(w));
        }
#pragma unroll
      for (int e = e0; e < e1; ++e) x[e] = __builtin_amdgcn_exp2f(y[e]);
#pragma unroll
      for (int e = e0; e < e1; ++e) pin(x[e]);
      if constexpr (s == NSLOT - 1) {
        total = 0.f;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
          ls[rb] = sum[rb][0] + sum[rb][1];
          total = rb == 0 ? ls[0] : total + ls[rb];
        }
        pin(total);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int kp = 0; kp < 2; ++kp)
        pc[rb][kp] = __builtin_bit_cast(bf16x8, u32x4{pw[rb][kp][0], pw[rb][kp][1], pw[rb][kp][2], pw[rb][kp][3]});
    // (also true of NaN: a row without a max, or NaN logits)
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(total <= kLaneSumLimit)) != 0, 0)) raise(sc, pc, ls);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) l_run[rb] += ls[rb];
  }

  // Raises the running max of every row to this half's, rescales O and l and
  // takes the half's probabilities again (rare, wave-uniform).
  __device__ __forceinline__ void raise(const f32x16 (&sc)[RB], bf16x8 (&pc)[RB][2], float (&ls)[RB]) {
    settle();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sc[rb][v]);
      // branch-free per lane: a divergent branch here would keep two copies of O
      const float m_new = fmaxf(m_run[rb], pair_max(mx) * c);
      const float alpha = (m_new == m_run[rb]) ? 1.f : __builtin_amdgcn_exp2f(m_run[rb] - m_new);
      l_run[rb] *= alpha;
#pragma unroll
      for (int db = 0; db < NDB; ++db) o[rb][db] *= alpha;
      m_run[rb] = m_new;
      neg_m[rb] = -m_new;
      const float nm = (m_new == -INFINITY) ? 0.f : -m_new;      // no visible key yet: probabilities 0
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[rb][v], c, nm));
        if (v & 1) s1 = v == 1 ? e : s1 + e;
        else s0 = v == 0 ? e : s0 + e;
        pc[rb][v / 8][v % 8] = (__bf16)e;
      }
      ls[rb] = s0 + s1;
    }
    settle();
  }

  // O += the last half: vf and row VR of v_rd.
  template <int VR>
  __device__ __forceinline__ void last_values(const bf16x8 (&pp)[RB][2]) {
    bf16x8 v2[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) v2[db] = read_v<VR>(v_rd, db);
    asm volatile("s_nop 1");       // pp may have been written by the VALU just before
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) mfma_o(o[rb][db], vf[db], pp[rb][0]);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int rb = 0; rb < RB; ++rb) mfma_o(o[rb][db], v2[db], pp[rb][1]);
    settle();
  }
};

}  // namespace vico
