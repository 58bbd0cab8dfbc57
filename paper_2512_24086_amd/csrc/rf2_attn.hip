// Block-sparse flash attention (Sec. 3.1, eqs. 1-4 with the block skip rule) for gfx950.
//
// Two kernels with the same arithmetic: block_sparse_attn_kernel (d = 64; K and V^T in LDS rings, described first) and
// stream_attn_kernel (d = 128; operands from memory into registers, described where it begins).
//
// One workgroup owns one Q block (b_q rows, or 128 of 256) of one (batch, head) and walks that row's
// list of kept K/V blocks (b_k rows each; b_q and b_k may differ).  Every wavefront owns 32 query rows
// and sees all keys of the list, so there is nothing to merge at the end; a workgroup needs 40 KiB
// of LDS and 128 registers per lane (d = 64), so four workgroups share a compute unit (four wavefronts per
// SIMD) and each hides the barriers, LDS latencies and vector-ALU phases of the others.
// Launches that would leave compute units idle or wait for a few long lists instead give a list to KS such
// groups of wavefronts, each with a contiguous share of it and with rings of its own, which merge their
// results through LDS (rf2_attn_cut.h has the rule and the measurements).
//
// Both products are computed transposed so that no register shuffling is needed between them
// (v_mfma_f32_32x32x16_bf16, D = A(32xk) * B(kx32) + C):
//   S^T[key][query]  = K (A, from LDS)  * Q^T (B, registers, loaded once)
//   O^T[chan][query] = V^T (A, from LDS) * P^T (B, registers = exp of the S^T accumulators)
// In the accumulator layout lane l holds query column l%32 and, per 32-key tile, keys
// 8*(i/4) + 4*(l/32) + i%4 for i = 0..15.  Eight consecutive accumulator values are exactly one
// B operand of the second product provided the A operand (V^T) lists the keys of each 16-key
// group in the order 0-3, 8-11, 4-7, 12-15 -- the order rf2_permute writes.  Row statistics are
// per lane (one query column) plus one exchange with lane l^32.
//
// Softmax (eqs. 2, 3) without a per-unit row maximum: a probability is exp2(fma(q.k, c, -m_ref c))
// with c = log2(e)/sqrt(d), the subtraction of eq. (2) riding on the multiply-add that applies the
// scale.  m_ref is set exactly from the first unit of the row and afterwards only moved when the row
// sum of a unit leaves the range fp32/bf16 carry without loss (> 2^40, or not finite); the final
// division by the row sum makes the reference point irrelevant.  The common path is one fused
// multiply-add, one exp2, one add and half a bf16 pack per probability.
//
// The loop is software-pipelined over "units" (one 32-key tile; a 64-key part of a K/V block is
// two units): step s issues the matrix products S_{s+1} and O += V P_{s-1} around the softmax
// arithmetic of unit s.  K and V^T parts stream from global memory straight into LDS rings (3 K
// parts, 2 V^T parts); the workgroup meets at one barrier per part (every second step).
#include "rf2_internal.h"

#include <cfloat>
#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// BQ rows per Q block (one workgroup), BK rows per K/V block (Sec. 3.1: b_q and b_k).
// KS groups of NW wavefronts walk a contiguous share of the row's list each and merge at the end.
template <int D, int BQ, int BK, int KS>
struct AttnCfg {
  static constexpr int NW = BQ / 32;            // wavefronts, 32 query rows each
  static constexpr int NT = NW * 64;            // threads of a group
  static constexpr int KH = BK / 2;             // K block rows r and r + KH share a part (see rf2.h)
  static constexpr int PB = BK / 64;            // 64-key parts per K/V block
  static constexpr int UB = BK / 32;            // 32-key units per K/V block
  static constexpr int DS = D / 16;             // k-steps of the first product
  static constexpr int DT = D / 32;             // 32-channel tiles of the output
  static constexpr int TILE_BYTES = BK * D * 2;
  static constexpr int PART_BYTES = 64 * D * 2;
  static constexpr int LPW = PART_BYTES / 1024 / NW;   // 1 KiB direct-to-LDS loads per wavefront per part
  static constexpr int NK = 3, NV = 2;                 // ring depths in parts
  static constexpr int RING_BYTES = (NK + NV) * PART_BYTES;   // per group
  // the merge passes a group's accumulators and row statistics through its rings
  static_assert(KS == 1 || NW * (DT * 4096 + 256) <= RING_BYTES, "merge buffer");
  static_assert(LPW >= 1 && 2 * LPW < 63, "vmcnt range");
};

// rf2_permute stores every K and V^T block as PB contiguous parts in exactly the order the
// operand reads below walk them ([chunk][64 rows][8 bf16], see rf2.h), so a part is copied
// verbatim: each wavefront-wide load deposits 64 x 16 B at consecutive LDS addresses (M0 = LDS
// base of that KiB), wavefront w taking KiB u*NW + w for u = 0..LPW-1.  In LDS the 16 lanes of a
// quarter-wave read 16 consecutive 16-byte slots (no bank conflicts) and all reads of a product
// share one per-lane base address plus compile-time offsets.
// The load is written in assembly on purpose: the compiler then does not track it, and the only
// waits for it are the explicit vmcnt waits of ring_barrier below (its own bookkeeping of
// direct-to-LDS loads falls back to waiting for every outstanding load before unrelated LDS reads).
//
// The S^T product is issued through assembly so that its accumulators are ordinary vector
// registers that the softmax arithmetic reads in place.  The compiler does not know these
// statements are MFMAs, so what it would do for an MFMA is done by hand:
//  * between the last MFMA of a chain and the first vector-ALU read of its result lie the wait states
//    an 8-pass MFMA needs.  In the loop the chain ends in slot NQ-1 of a step and its accumulators are
//    first read in the following step, behind the NP matrix products of the remaining slots (their
//    order is frozen by the scheduling barriers), so nothing is added there; the chain of the
//    prologue is followed by code the compiler orders freely and ends in qk_last_wait, which carries
//    the wait states itself (18 >= the 12 needed);
//  * the first MFMA of a chain takes the constant 0 as its addend, so no register is read by the
//    matrix core after issue except the A and B operands;
//  * A and B operands are read at issue; they come from LDS reads and the resident Q fragments.
__device__ __forceinline__ void qk_first(f32x16& S, const bf16x8& a, const bf16x8& b) {
  asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(S) : "v"(a), "v"(b));
}
__device__ __forceinline__ void qk_next(f32x16& S, const bf16x8& a, const bf16x8& b) {
  asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(S) : "v"(a), "v"(b));
}
__device__ __forceinline__ void qk_last_wait(f32x16& S, const bf16x8& a, const bf16x8& b) {
  asm("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0\n\t"
      "s_nop 7\n\ts_nop 7\n\ts_nop 1"
      : "+v"(S)
      : "v"(a), "v"(b));
}

// Tells the compiler that a pointer is the same in every lane (it then lives in scalar registers).
__device__ __forceinline__ const unsigned char* uniform_ptr(const void* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const unsigned char*)(((uint64_t)hi << 32) | lo);
}

// One wavefront-wide direct-to-LDS load: 64 x 16 B from g + voff (scalar base, per-lane 32-bit
// byte offset) to the KiB of LDS at `lds_kib`.
// M0 is written here and named as clobbered.  The compiler reserves M0 for itself (and says so with a
// warning, silenced below): it sets M0 immediately in front of each of its own uses (LDS-direct builtins,
// relative moves, message and GWS instructions), none of which this translation unit contains.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma_one(uint32_t lds_kib, const unsigned char* g, uint32_t voff) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_kib), "v"(voff), "s"(g) : "memory", "m0");
}
#pragma clang diagnostic pop

// A whole part (LPW KiB per wavefront): wavefront w takes KiB u*NW + w for u = 0..LPW-1.
template <int NW, int LPW>
__device__ __forceinline__ void dma_part(unsigned char* lds, const unsigned char* g, int wave, uint32_t tid16) {
  const uint32_t lds_base = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)lds;
  g = uniform_ptr(g);
#pragma unroll
  for (int u = 0; u < LPW; ++u) dma_one(lds_base + (uint32_t)((u * NW + wave) * 1024), g + u * (NW * 1024), tid16);
}

// Workgroup barrier of the loop: waits until at most N of this wavefront's direct-to-LDS loads
// are still in flight, then s_barrier.  __syncthreads() cannot be used there: its release fence
// would wait for ALL outstanding loads, i.e. also for the parts prefetched for later steps.  LDS
// operand reads have completed before the barrier because the MFMAs consuming them were issued;
// the asm memory clobbers keep the compiler from moving LDS accesses across.
template <int N>
__device__ __forceinline__ void ring_barrier() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Head and Q block of a workgroup, from its XCD and its number there.  False: no work.
// Workgroups with equal blockIdx % 8 share an XCD (which of the eight it is varies from launch to launch).  Slots of an XCD, in
// issue order: the all-column sink rows of every head first, then the ordinary rows head by head.  A sink row is several times
// longer than an ordinary one; issued first (longest jobs first) none of them is left running alone at the end, and the short
// rows fill the tail evenly.
struct RowOrder {
  const int32_t* shares;       // [8][per_xcd]: ordinary Q block of each slot of a head, -1 = none; null: rows in one run
  int per_xcd;                 // slots of a head on an XCD, or of all heads
  int n_bh, rows, sink_begin, n_sink, sink_slots;
};
__device__ __forceinline__ bool row_of(const RowOrder& w, int xcd, int slot, int& bh, int& qi) {
  if (slot < w.sink_slots) {
    // The sink rows of all heads, numbered head by head, are cut into 8 contiguous runs of sink_slots rows, one per XCD: an
    // XCD gets whole heads where it can (with 40 heads of 29 sink rows: five heads each).  Rows of one head have the same
    // list (every column) and the same length: side by side on one XCD they run in step and find each other's tiles in its L2.
    const int g = xcd * w.sink_slots + slot;
    bh = g / w.n_sink;
    qi = w.sink_begin + g % w.n_sink;
    return g < w.n_bh * w.n_sink;
  }
  const int t = slot - w.sink_slots;
  if (w.shares == nullptr) {     // the ordinary rows likewise (see rf2_cut_stream)
    const int plain = w.rows - w.n_sink, g = xcd * w.per_xcd + t;
    bh = g / plain;
    qi = g % plain;
    qi += qi >= w.sink_begin ? w.n_sink : 0;
    return g < w.n_bh * plain;
  }
  // The work table deals a head's ordinary rows to 8 shares of slightly different size (contiguous ranges); the share an XCD
  // takes rotates with the head so that no XCD collects the large shares of every head.
  bh = t / w.per_xcd;
  qi = w.shares[((xcd + bh) & 7) * w.per_xcd + t % w.per_xcd];
  return qi >= 0;
}

// (second launch bound: wavefronts per SIMD the register budget is sized for, which is what LDS admits: four workgroups of
// 40 KiB rings per compute unit, whatever KS; a 64-row Q block has two wavefronts per group)
template <int D, int BQ, int BK, int KS>
__global__ void __launch_bounds__(BQ * 2 * KS, BQ == 128 ? 4 : 2) block_sparse_attn_kernel(
    const __bf16* __restrict__ qp, const __bf16* __restrict__ kp, const __bf16* __restrict__ vp,
    const int32_t* __restrict__ blk_idx, const int32_t* __restrict__ blk_cnt, __bf16* __restrict__ op,
    float* __restrict__ lse, RowOrder order, int Tb, int k_row, int last_valid, float scale_log2, const int32_t* __restrict__ scatter, int n_tokens,
    int heads, rf2_strides st, int split) {
  // split: log2 of the workgroups that share a list (a Q block of the mask has BQ << split rows); they are neighbours
  // on one XCD.  Tb: K/V blocks per head (columns of the block mask); last_valid: tokens in the last one.
  using C = AttnCfg<D, BQ, BK, KS>;
  // Part P lives in slot P % NK of the K ring (first) and slot P % NV of the V^T ring (behind it).
  __shared__ __attribute__((aligned(1024))) unsigned char ring[KS * C::RING_BYTES];
  constexpr uint32_t VRING = C::NK * C::PART_BYTES;

  const int xcd = blockIdx.x & 7, share = (int)(blockIdx.x >> 3) & ((1 << split) - 1), slot = (int)(blockIdx.x >> 3) >> split;
  int bh, qi;
  if (!row_of(order, xcd, slot, bh, qi)) return;
  const int Tq = order.rows;
  const size_t row_id = (size_t)bh * Tq + qi;
  int cnt = blk_cnt[row_id];
  const bool dense = (cnt == Tb);
  cnt = dense ? Tb : min(max(cnt, 0), k_row);
  const int32_t* __restrict__ list = blk_idx + row_id * k_row;
  // Only the last listed block can be the ragged last block of the sequence (lists ascend).
  bool ragged = false;
  if (cnt > 0 && last_valid < BK) {
    const int jl = dense ? cnt - 1 : list[cnt - 1];
    ragged = min(max(jl, 0), Tb - 1) == Tb - 1;
  }
  int NPARTS = cnt * C::PB;
  // (a last part without any valid key is left out, so that every group has a valid key in its first unit)
  if (KS > 1 && C::PB > 1 && ragged && last_valid <= 32) --NPARTS;
  // Group `grp` walks the parts from P0 on, as many as there are; all groups pass the same number of barriers.
  const int grp = KS > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x / C::NT) : 0;
  const int parts = (NPARTS + KS - 1) / KS, P0 = grp * parts;
  const int U = KS > 1 ? 2 * max(min(parts, NPARTS - P0), 0) : 2 * parts;   // 32-key units to process (even)

  const int tid = KS > 1 ? (int)threadIdx.x % C::NT : (int)threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wavefront-uniform, kept in a scalar register
  const uint32_t tid16 = (uint32_t)tid * 16u;
  const int l32 = lane & 31, lh = lane >> 5;
  const size_t q_head_off = (size_t)bh * (Tq << split) * BQ * D;   // elements; qp and op
  const int q_row = ((qi << split) + share) * BQ + 32 * wave + l32;   // this lane's query row in its head
  const size_t k_head_off = (size_t)bh * Tb * BK * D;   // kp and vp
  const unsigned char* const kbase = uniform_ptr(kp + k_head_off);
  const unsigned char* const vbase = uniform_ptr(vp + k_head_off);
  // LDS byte offsets of this lane's first operand chunk inside a K part / a V^T part, for the
  // first 32-key tile of the part; the second tile lies K_TILE / V_TILE bytes further.
  const uint32_t k_lane = (uint32_t)(grp * C::RING_BYTES + (lh * 64 + l32) * 16);
  const uint32_t v_lane = (uint32_t)(grp * C::RING_BYTES + (lh * D + l32) * 16);
  constexpr uint32_t K_TILE = 32 * 16, V_TILE = 4 * D * 16;
  // Part P of the list is part P % PB of listed block P / PB (P clamped: loads past the end
  // re-fetch the last part into a free slot, which keeps the outstanding-load count uniform).
  // A list entry is read one odd step before it is needed (list_entry) and turned into an offset
  // only when it is used (part_off), so that no step waits for a scalar memory load.
  // (part numbers are never negative: unsigned division and remainder are a shift and a mask)
  auto list_entry = [&](int P) {
    const int it = (int)((unsigned)min(P, NPARTS - 1) / (unsigned)C::PB);
    return dense ? it : list[it];
  };
  auto part_off = [&](int entry, int P) {
    const int j = min(max(entry, 0), Tb - 1);            // a corrupt list can give wrong results, never a fault
    return (uint32_t)j * (uint32_t)C::TILE_BYTES + ((unsigned)min(P, NPARTS - 1) % (unsigned)C::PB) * (uint32_t)C::PART_BYTES;
  };
  auto part_at = [&](int P) { return (size_t)part_off(list_entry(P0 + P), P0 + P); };
  unsigned char* const gring = ring + grp * C::RING_BYTES;
  const uint32_t ring_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)gring;
  const int partial_begin = ragged ? max((cnt - 1) * C::UB - 2 * P0, 0) : U;   // first unit of the ragged block

  bf16x8 qf[C::DS];
  f32x16 o[C::DT];
#pragma unroll
  for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
  // Softmax reference m_ref (per query column, in units of the raw products q.k) and nmc = -m_ref * c,
  // the addend of the multiply-add in front of every exp2.  l_run lags one unit behind: rs_last, the
  // row sum of the latest unit, is still to be added.
  // (a group without any part of its own weighs nothing in the merge, however small the others' references are)
  float m_ref = KS > 1 && U == 0 ? -FLT_MAX : 0.f, nmc = 0.f, l_run = 0.f, rs_last = 0.f;

  // ---- building blocks ------------------------------------------------------------------
  // One step has NQ + NP "slots" of one MFMA each: slots 0..NQ-1 are the k-steps of
  // S^T_{s+1} = K Q^T (eq. 1, unscaled), slots NQ.. are the (channel tile, k-step) pairs of
  // O^T += V^T P^T_{s-1} (eq. 4).
  constexpr int NQ = C::DS, NP = C::DT * 2, NSLOT = NQ + NP;
  constexpr int PD = 4;                                  // operand reads run this many slots ahead
  constexpr int SPP = NSLOT / 8;                         // slots per pair of probabilities (8 pairs per unit)
  static_assert(NSLOT % 8 == 0 && NQ >= 2 && 2 * C::LPW <= NSLOT, "slot plan");
  auto k_operand = [&](uint32_t k_addr, int c) -> bf16x8 {        // chunk 2c+lh of the tile
    return *reinterpret_cast<const bf16x8*>(ring + k_addr + c * 2048);
  };
  auto v_operand = [&](uint32_t v_addr, int dt, int ks) -> bf16x8 {   // key chunk 2ks+lh, channel 32dt+l32
    return *reinterpret_cast<const bf16x8*>(ring + v_addr + (2 * ks * D + 32 * dt) * 16);
  };
  auto operand = [&](uint32_t k_addr, uint32_t v_addr, int g) -> bf16x8 {
    return g < NQ ? k_operand(k_addr, g) : v_operand(v_addr, (g - NQ) / 2, (g - NQ) % 2);
  };
  // largest accumulator of one unit per query column (both lane halves end up with the same value)
  auto rowmax = [&](const f32x16& S) -> float {
    float v = S[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) v = fmaxf(v, S[i]);
    // exchange with lane l^32 on the vector ALU (an LDS shuffle would wait for operand reads in flight)
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  };
  // Moves the reference to `to` (per query column, where `move`): everything accumulated so far is rescaled
  // (eqs. 3, 4).  The accumulators hold raw products, so nothing else changes.
  auto move_reference = [&](bool move, float to) {
    const float delta = move ? to - m_ref : 0.f;
    // (the very first move may go down; nothing has been accumulated then, any finite factor will do)
    const float alpha = __builtin_amdgcn_exp2f(-fmaxf(delta, 0.f) * scale_log2);
    if constexpr (KS > 1) m_ref = move ? to : m_ref;     // (from -FLT_MAX a difference does not lead to `to`)
    else m_ref += delta;
    nmc = -m_ref * scale_log2;
    l_run *= alpha;
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[dt][i] *= alpha;
  };
  // The probabilities P of the unit whose accumulators are in S were out of range; O holds all
  // earlier units, so the reference moves up and P (and rs_last) are recomputed.
  auto redo_unit = [&](f32x16& S, bf16x8 (&P)[2]) {
    const float mx = rowmax(S);
    move_reference(mx > m_ref, mx);
    rs_last = 0.f;
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      const float p0 = __builtin_amdgcn_exp2f(fmaf(S[i], scale_log2, nmc));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(S[i + 1], scale_log2, nmc));
      const bf16x2 pk = {(__bf16)p0, (__bf16)p1};
      rs_last += p0 + p1;
      P[i / 8][i % 8] = pk[0];
      P[i / 8][i % 8 + 1] = pk[1];
    }
  };
  // Rare work before the step of unit s: redo of unit s-1 (its accumulators are still in Sprev, the
  // buffer this step overwrites), the first unit (sets the reference exactly), and the units of the
  // ragged last block (keys past the end of the sequence are masked here).
  auto pre_step = [&](f32x16& S, f32x16& Sprev, bf16x8 (&Pprev)[2], uint32_t v_addr, int s, bool redo) {
    if (redo) redo_unit(Sprev, Pprev);
    if (s == 0 || s >= partial_begin) {
      // the pending product V P_{s-1} must reach O before O is rescaled; it is then neutralised
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const int dt = j % C::DT, ks = j / C::DT;
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(v_addr, dt, ks), Pprev[ks], o[dt], 0, 0, 0);
      }
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) Pprev[ks][e] = (__bf16)0.f;
      if (s >= partial_begin) {
        const int t = s & 1, p = (P0 + (s >> 1)) % C::PB;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = t * C::KH + 32 * p + 8 * (i / 4) + 4 * lh + (i % 4);
          if (key >= last_valid) S[i] = -INFINITY;
        }
      }
      // (minus infinity in all products of a later unit of a list is no reference: it weighs nothing, also where a group begins)
      const float mx = KS > 1 && grp > 0 ? fmaxf(rowmax(S), -FLT_MAX) : rowmax(S);
      // first unit: exact reference (it has at least one valid key); later: only upwards
      const bool move = (s == 0) ? true : (mx > m_ref);
      if (__builtin_amdgcn_ballot_w64(move) != 0ull) {
        l_run += rs_last;                                  // unit s-1 is in O now: rescale it with the rest
        rs_last = 0.f;
        move_reference(move, mx);
      }
    }
  };

  int entry_k = 0, entry_v = 0;       // list entries of the parts loaded by the next odd step
  bool slow = true, redo = false;     // pre_step is needed for the coming unit / the latest unit must be redone
  // Step s (unit s = tile s%2 of part s/2): products S_{s+1} and V P_{s-1} around the softmax
  // arithmetic of unit s, in NSLOT slots of {operand read PD slots ahead, one MFMA, part of the
  // softmax arithmetic, one direct-to-LDS load}.  Odd steps s = 2P+1 start with the barrier and
  // issue the loads of V^T part P+NV-1 (into the slot of part P-1) and K part P+NK (into the slot of
  // part P); the V^T part is needed at the next barrier and goes first, the K loads may stay in
  // flight across it.
  auto step = [&](auto odd_tag, int s, int kslot, int vslot, int kfree, int vfree, f32x16& Scur, f32x16& Snext,
                  bf16x8 (&Pprev)[2], bf16x8 (&Pcur)[2]) {
    constexpr bool ODD = decltype(odd_tag)::value;
    if constexpr (ODD) ring_barrier<C::LPW>();
    // Through the step that issues a part's loads a wavefront takes precedence over the other wavefront
    // of its SIMD (which belongs to the other workgroup of the compute unit and is, as a rule, in an even
    // step): its loads leave earlier.  Measured +0.6 ... +1.1 % on 128- and 256-row Q blocks; a 64-row Q
    // block has its SIMD to itself (-0.2 %).
    constexpr bool PRIO = ODD && BQ >= 128;
    if constexpr (PRIO) __builtin_amdgcn_s_setprio(2);
    // unit s+1 and unit s-1 are both tile (s+1)%2 of their parts
    const uint32_t k_addr = (uint32_t)(kslot * C::PART_BYTES) + (ODD ? 0u : K_TILE) + k_lane;
    const uint32_t v_addr = VRING + (uint32_t)(vslot * C::PART_BYTES) + (ODD ? 0u : V_TILE) + v_lane;
    if (slow) pre_step(Scur, Snext, Pprev, v_addr, s, redo);
    l_run += rs_last;
    uint32_t k_dst = 0, v_dst = 0, k_voff = 0, v_voff = 0;
    if constexpr (ODD) {
      const int P = s >> 1;
      k_dst = ring_lds + (uint32_t)(kfree * C::PART_BYTES + wave * 1024);
      v_dst = ring_lds + VRING + (uint32_t)(vfree * C::PART_BYTES + wave * 1024);
      k_voff = tid16 + part_off(entry_k, P0 + P + C::NK);
      v_voff = tid16 + part_off(entry_v, P0 + P + C::NV - 1);
    }
    // the entries fetched by the previous odd step are consumed before the next fetches are issued:
    // scalar loads return out of order, so a wait for the old ones would also wait for new ones
    __builtin_amdgcn_sched_barrier(0);
    float rs = 0.f, e0 = 0.f, e1 = 0.f;
    bf16x8 opnd[NSLOT];
#pragma unroll
    for (int g = 0; g < PD; ++g) opnd[g] = operand(k_addr, v_addr, g);
    if constexpr (ODD) {
      const int P = s >> 1;
      entry_k = list_entry(P0 + P + 1 + C::NK);   // for the next odd step
      entry_v = list_entry(P0 + P + C::NV);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int g = 0; g < NSLOT; ++g) {
      if (g + PD < NSLOT) opnd[g + PD] = operand(k_addr, v_addr, g + PD);
      if (g == 0) qk_first(Snext, opnd[g], qf[g]);
      else if (g < NQ) qk_next(Snext, opnd[g], qf[g]);
      else {
        const int dt = (g - NQ) / 2, ks = (g - NQ) % 2;
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(opnd[g], Pprev[ks], o[dt], 0, 0, 0);
      }
      if (g % SPP == 0) {
        // exponentials of pair g/SPP now, sum and bf16 packing of the previous pair (its exponentials
        // have long left the pipeline: no instruction here waits for the one before it)
        const int i = 2 * (g / SPP);
        if (i > 0) {
          const bf16x2 pk = {(__bf16)e0, (__bf16)e1};
          rs = (i == 2) ? e0 + e1 : rs + (e0 + e1);
          Pcur[(i - 2) / 8][(i - 2) % 8] = pk[0];
          Pcur[(i - 2) / 8][(i - 2) % 8 + 1] = pk[1];
        }
        e0 = __builtin_amdgcn_exp2f(fmaf(Scur[i], scale_log2, nmc));
        e1 = __builtin_amdgcn_exp2f(fmaf(Scur[i + 1], scale_log2, nmc));
        if (i == 14) {
          const bf16x2 pk = {(__bf16)e0, (__bf16)e1};
          rs += e0 + e1;
          Pcur[1][6] = pk[0];
          Pcur[1][7] = pk[1];
        }
      }
      if constexpr (ODD) {
        // from slot 0 on (-1.4 % from the slots of the second product on), V^T first
        if (g < C::LPW) dma_one(v_dst + g * (C::NW * 1024), vbase + g * (C::NW * 1024), v_voff);
        else if (g < 2 * C::LPW) dma_one(k_dst + (g - C::LPW) * (C::NW * 1024), kbase + (g - C::LPW) * (C::NW * 1024), k_voff);
      }
      // Slots stay in this order: the operand reads keep their PD-slot lead over the MFMAs that
      // consume them (left alone, the scheduler packs each read right in front of its consumer).
      __builtin_amdgcn_sched_barrier(0);
    }
    // Keep the softmax arithmetic inside this block (its results are only consumed by the next
    // step, and the compiler would otherwise sink it there, out from under the MFMAs).
    asm volatile("" : "+v"(Pcur[0]), "+v"(Pcur[1]), "+v"(rs));
    if constexpr (PRIO) __builtin_amdgcn_s_setprio(0);
    rs_last = rs;
    redo = __builtin_amdgcn_ballot_w64(!(rs <= 1.0995e12f)) != 0ull;   // rare: above 2^40 or not finite
    slow = redo || (s + 1 >= partial_begin);
  };

  if (U > 0) {
    // ---- prologue: fill the rings, load Q, S of unit 0 -------------------------------------
    // (at raised priority: a row that starts has nothing to compute on until its first parts arrive; +0.3 %)
    __builtin_amdgcn_s_setprio(3);
#pragma unroll
    for (int P = 0; P < C::NK; ++P) dma_part<C::NW, C::LPW>(gring + P * C::PART_BYTES, kbase + part_at(P), wave, tid16);
#pragma unroll
    for (int P = 0; P < C::NV - 1; ++P)
      dma_part<C::NW, C::LPW>(gring + VRING + P * C::PART_BYTES, vbase + part_at(P), wave, tid16);
    // the slot of "part -1" (read by step 0 with zero probabilities) gets the list's first part, as finite as the list is
    dma_part<C::NW, C::LPW>(gring + VRING + (C::NV - 1) * C::PART_BYTES, vbase + part_off(list_entry(0), 0), wave, tid16);
    {
      const __bf16* qrow = qp + q_head_off + (size_t)q_row * D + 8 * lh;
#pragma unroll
      for (int ds = 0; ds < C::DS; ++ds) qf[ds] = *reinterpret_cast<const bf16x8*>(qrow + 16 * ds);
    }
    f32x16 Sa, Sb;
    bf16x8 Pa[2], Pb[2];
    ring_barrier<0>();
#pragma unroll
    for (int ds = 0; ds < C::DS; ++ds) {
      const bf16x8 a = k_operand(k_lane, ds);
      if (ds == 0) qk_first(Sa, a, qf[ds]);
      else if (ds < C::DS - 1) qk_next(Sa, a, qf[ds]);
      else qk_last_wait(Sa, a, qf[ds]);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int e = 0; e < 8; ++e) Pb[ks][e] = (__bf16)0.f;   // "P_{-1}": step 0 adds V * 0
#pragma unroll
    for (int i = 0; i < 16; ++i) Sb[i] = 0.f;
    entry_k = list_entry(P0 + C::NK);
    entry_v = list_entry(P0 + C::NV - 1);

    __builtin_amdgcn_s_setprio(0);
    // ---- steady state: two steps per part ---------------------------------------------------
    int k0 = 0, k1 = 1;                                   // K ring slots of parts P and P+1
    int vm = C::NV - 1, vc = 0;                           // V^T ring slots of parts P-1 and P
    // (the loop starts on a 64-byte line of the instruction cache: against where it otherwise falls, pairs of runs of both
    // builds, 720p and a 256-row clip +0.5 ... +1.0 %, long video +0.1 ... +0.7, 480p and d = 64 0, 64-row blocks -0.4)
    asm volatile(".p2align 6");
    for (int s = 0; s < U; s += 2) {
      // even step: S of unit s+1 (part P, tile 1), V P of unit s-1 (part P-1, tile 1)
      step(std::false_type{}, s, k0, vm, 0, 0, Sa, Sb, Pb, Pa);
      // odd step: S of unit s+2 (part P+1, tile 0), V P of unit s (part P, tile 0)
      step(std::true_type{}, s + 1, k1, vc, k0, vm, Sb, Sa, Pa, Pb);
      k0 = k1;
      k1 = (k1 == C::NK - 1) ? 0 : k1 + 1;
      vm = vc;
      vc = (vc == C::NV - 1) ? 0 : vc + 1;
    }
    // ---- last product: O += V P_{U-1} (tile 1 of the last part; P_{U-1} is in Pb) ---------------
    if constexpr (KS > 1)
      for (int s = U; s < 2 * parts; s += 2) __builtin_amdgcn_s_barrier();   // (the longer groups are still walking)
    ring_barrier<0>();
    if (redo) redo_unit(Sb, Pb);
    l_run += rs_last;
    {
      const uint32_t v_addr = VRING + (uint32_t)(vm * C::PART_BYTES) + V_TILE + v_lane;
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const int dt = j % C::DT, ks = j / C::DT;
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(v_addr, dt, ks), Pb[ks], o[dt], 0, 0, 0);
      }
    }
  } else if (KS > 1 && parts > 0) {
    for (int s = -4; s < 2 * parts; s += 2) __builtin_amdgcn_s_barrier();    // prologue, one per part, last product
  }

  // ---- normalise (the final division of eq. 4) and write the 32 rows of this wavefront ----------
  const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
  float l_tot = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  // ---- merge of the groups: group dt * KS / DT finishes channel tile dt ---------------------------
  // Every group leaves the tiles it does not finish and its row statistics in its own rings (free once all
  // wavefronts have passed the barrier) and rescales what it reads to the largest reference of the row.
  auto finishes = [&](int dt) { return KS == 1 || grp == dt * KS / C::DT; };
  if constexpr (KS > 1) {
    float4* const tiles = reinterpret_cast<float4*>(gring) + wave * C::DT * 256 + lane;
    float2* const stats = reinterpret_cast<float2*>(gring + C::NW * C::DT * 4096) + wave * 32 + l32;
    __syncthreads();
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
      if (!finishes(dt))
#pragma unroll
        for (int g = 0; g < 4; ++g)
          tiles[(dt * 4 + g) * 64] = make_float4(o[dt][4 * g], o[dt][4 * g + 1], o[dt][4 * g + 2], o[dt][4 * g + 3]);
    if (lh == 0) *stats = make_float2(m_ref, l_tot);
    __syncthreads();
    float m_all = m_ref;
    float2 st_of[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      st_of[k] = *reinterpret_cast<const float2*>(reinterpret_cast<const unsigned char*>(stats) + (k - grp) * C::RING_BYTES);
      m_all = fmaxf(m_all, st_of[k].x);
    }
    const float own = __builtin_amdgcn_exp2f((m_ref - m_all) * scale_log2);
    l_tot = 0.f;
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[dt][i] *= own;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const float w = __builtin_amdgcn_exp2f((st_of[k].x - m_all) * scale_log2);
      l_tot = fmaf(st_of[k].y, w, l_tot);
      const float4* const from = reinterpret_cast<const float4*>(reinterpret_cast<const unsigned char*>(tiles) + (k - grp) * C::RING_BYTES);
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt)
        if (k != grp && finishes(dt))
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const float4 x = from[(dt * 4 + g) * 64];
            o[dt][4 * g] = fmaf(x.x, w, o[dt][4 * g]);
            o[dt][4 * g + 1] = fmaf(x.y, w, o[dt][4 * g + 1]);
            o[dt][4 * g + 2] = fmaf(x.z, w, o[dt][4 * g + 2]);
            o[dt][4 * g + 3] = fmaf(x.w, w, o[dt][4 * g + 3]);
          }
    }
    m_ref = m_all;
  }
  const float f = l_tot > 0.f ? 1.0f / l_tot : 0.f;      // a row with no kept key yields zeros
  const size_t row = (size_t)q_row;
  // plain output: row `row` of the permuted layout; fused inverse permutation: the token's raster row
  const int target = scatter ? scatter[row] : (int)row;
  if (target < 0) return;                                 // padding row of the last block
  __bf16* orow = scatter ? op + ((bh / heads) * st.batch + (bh % heads) * st.head + (long long)target * st.token) * D
                         : op + q_head_off + row * D;
#pragma unroll
  for (int dt = 0; dt < C::DT; ++dt)
    if (finishes(dt))
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 pk;
#pragma unroll
        for (int e = 0; e < 4; ++e) pk[e] = (__bf16)(o[dt][4 * g + e] * f);
        *reinterpret_cast<bf16x4*>(orow + 32 * dt + 8 * g + 4 * lh) = pk;
      }
  if (lse != nullptr && lh == 0 && grp == 0)
    lse[scatter ? (size_t)bh * n_tokens + target : (size_t)bh * (Tq << split) * BQ + row] =
        m_ref * scale_log2 * 0.6931471805599453f + __logf(l_tot);
}

// ==== d = 128: operands from memory into registers ===============================================================
//
// A wavefront owns 64 query rows (two tiles of 32) and loads the operands of both products straight from memory into
// registers, two steps ahead of their use: a part of the operand layout is read in 1 KiB pieces, each of which is one
// operand and feeds two MFMAs.  There is no LDS and no barrier between the wavefronts that work on a launch, so one
// wavefront per SIMD (442 of its 512 registers) keeps the matrix cores 76 % busy on 720p; against rings in LDS with
// wavefronts of 32 rows (4 to a workgroup of 128 rows, two per SIMD, 69 %) an operand is moved half as often and nothing
// passes through LDS, which the power limit turns into clock: 1.55 GHz instead of 1.50.  720p, 40 heads, 20.7 -> 19.1 ms
// (1,216 TFLOP/s); 480p 4.00 -> 3.73 ms; with 64-row Q blocks, where the rings leave one wavefront of 32 rows per SIMD,
// 5.13 -> 4.03 ms and 720p, 20 heads, 13.3 -> 10.8 ms.
//
// A workgroup has QH x KS wavefronts: QH times 64 neighbouring query rows of a Q block, whose wavefronts ask for the same
// tiles at about the same time and find each other's in the L1 cache (720p, QH = 2 against two workgroups of 64 rows,
// 20.0 -> 19.2 ms), times KS shares of the list: wavefront k of a share walks parts k, k + KS, ... of it, and the
// shares are merged through LDS at the end.  rf2_cut_stream (rf2_attn_cut.h) chooses QH and KS.
//
// Registers: O^T 128 and Q 64 accumulation registers, S^T of two units 64, P of two units 32, operands of two steps 128.

// The S^T product in assembly, as above, with the Q operand in accumulation registers (volatile: the statements
// keep their places between the loads and the softmax arithmetic).
__device__ __forceinline__ void qk_stream(f32x16& S, const bf16x8& a, const bf16x8& b, bool first) {
  if (first) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(S) : "v"(a), "a"(b));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(S) : "v"(a), "a"(b));
}

template <int D, int BK, int QH, int KS>
__global__ void __launch_bounds__(64 * QH * KS, 1) stream_attn_kernel(
    const __bf16* __restrict__ qp, const __bf16* __restrict__ kp, const __bf16* __restrict__ vp,
    const int32_t* __restrict__ blk_idx, const int32_t* __restrict__ blk_cnt, __bf16* __restrict__ op,
    float* __restrict__ lse, RowOrder order, int Tb, int k_row, int last_valid, float scale_log2,
    const int32_t* __restrict__ scatter, int n_tokens, int heads, rf2_strides st, int split) {
  // split: log2 of the workgroups that share a Q block; they are neighbours on one XCD.  Tb: K/V blocks per head (columns of
  // the block mask); last_valid: tokens in the last one.
  constexpr int BQ = 64 * QH, KH = BK / 2, PB = BK / 64, DS = D / 16, DT = D / 32;
  constexpr int TILE_BYTES = BK * D * 2, PART_BYTES = 64 * D * 2;
  const int xcd = blockIdx.x & 7, share = (int)(blockIdx.x >> 3) & ((1 << split) - 1), slot = (int)(blockIdx.x >> 3) >> split;
  int bh, qi;
  if (!row_of(order, xcd, slot, bh, qi)) return;
  const int Tq = order.rows;
  const size_t row_id = (size_t)bh * Tq + qi;
  int cnt = blk_cnt[row_id];
  const bool dense = (cnt == Tb);
  cnt = dense ? Tb : min(max(cnt, 0), k_row);
  const int32_t* __restrict__ list = blk_idx + row_id * k_row;
  // Only the last listed block can be the ragged last block of the sequence (lists ascend).
  bool ragged = false;
  if (cnt > 0 && last_valid < BK) {
    const int jl = dense ? cnt - 1 : list[cnt - 1];
    ragged = min(max(jl, 0), Tb - 1) == Tb - 1;
  }
  int NPARTS = cnt * PB;
  // (a last part without any valid key is left out, so that every wavefront has a valid key in its first unit)
  if (KS > 1 && PB > 1 && ragged && last_valid <= 32) --NPARTS;
  const int wave = QH * KS > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : 0;
  const int half = wave % QH, grp = wave / QH;
  const int parts = KS > 1 ? max(NPARTS - grp + KS - 1, 0) / KS : NPARTS;    // this wavefront's: grp, grp + KS, ...
  const int U = 2 * parts;                                                   // its 32-key units (even)
  const int lane = (int)threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
  const size_t q_head_off = (size_t)bh * (Tq << split) * BQ * D;             // elements; qp and op
  const int q_row = ((qi << split) + share) * BQ + 64 * half + l32;          // this lane's query row of tile 0 in its head
  const size_t k_head_off = (size_t)bh * Tb * BK * D;                        // kp and vp
  // (buffer loads: scalar offsets of tile and operand beside a constant per-lane one; nothing past a head's K or V is read)
  const unsigned head_bytes = (unsigned)Tb * (unsigned)TILE_BYTES;
  const auto kbuf = __builtin_amdgcn_make_buffer_rsrc((void*)uniform_ptr(kp + k_head_off), 0, head_bytes, 0x00020000);
  const auto vbuf = __builtin_amdgcn_make_buffer_rsrc((void*)uniform_ptr(vp + k_head_off), 0, head_bytes, 0x00020000);
  const uint32_t k_lane = (uint32_t)((lh * 64 + l32) * 16), v_lane = (uint32_t)((lh * D + l32) * 16);
  constexpr uint32_t K_TILE = 32 * 16, V_TILE = 4 * D * 16;     // the second 32-key tile of a part
  // Operand c of the K tile, operand j = 2 dt + ks of the V^T tile, that begins at byte `off` of the head.
  auto k_load = [&](uint32_t off, int c) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(kbuf, k_lane + c % 2 * 2048, off + c / 2 * 4096, 0));
  };
  auto v_load = [&](uint32_t off, int j) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(vbuf, v_lane + j / 2 * 512, off + j % 2 * 2 * D * 16, 0));
  };
  // Part P of the list is part P % PB of listed block P / PB (P clamped: loads past the end fetch the last part again).
  auto list_entry = [&](int P) {
    const int it = (int)((unsigned)min(P, NPARTS - 1) / (unsigned)PB);
    return dense ? it : list[it];
  };
  auto part_off = [&](int entry, int P) {
    const int j = min(max(entry, 0), Tb - 1);            // a corrupt list can give wrong results, never a fault
    return (uint32_t)j * (uint32_t)TILE_BYTES + ((unsigned)min(P, NPARTS - 1) % (unsigned)PB) * (uint32_t)PART_BYTES;
  };
  auto part_of = [&](int P) { return P * KS + grp; };    // list part of this wavefront's part P
  const int partial_begin = ragged ? 2 * (max((cnt - 1) * PB - grp + KS - 1, 0) / KS) : U;   // first unit of the ragged block

  bf16x8 qf[2][DS];
  f32x16 o[2][DT];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[q][dt][i] = 0.f;
  // Softmax state per tile and query column, as in the other kernel; m_ref is exact from the first unit of the wavefront.
  // (a wavefront without any part of its own weighs nothing in the merge, however small the others' references are)
  float m_ref[2], nmc[2] = {}, l_run[2] = {}, rs_last[2] = {};
  m_ref[0] = m_ref[1] = KS > 1 && U == 0 ? -FLT_MAX : 0.f;
  constexpr int NQ = DS, NP = DT * 2;                    // operands of a step: K, V^T
  static_assert(NQ + NP == 16, "one pair of probabilities of each tile for every operand");
  // k-step ks of the second product's B operand from the packed probabilities of a unit
  auto operand_p = [](const uint32_t (&P)[8], int ks) {
    const u32x4 w = {P[4 * ks], P[4 * ks + 1], P[4 * ks + 2], P[4 * ks + 3]};
    return __builtin_bit_cast(bf16x8, w);
  };
  auto rowmax = [&](const f32x16& S) -> float {
    float v = S[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) v = fmaxf(v, S[i]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  };
  // The accumulators are scaled where they are, through one vector register (left to the compiler, the copies cost the
  // registers of the loop).  The wait states in front cover a product in flight, those behind a product that follows.
  auto move_reference = [&](int q, bool move, float to) {
    const float delta = move ? to - m_ref[q] : 0.f;
    const float alpha = __builtin_amdgcn_exp2f(-fmaxf(delta, 0.f) * scale_log2);
    if constexpr (KS > 1) m_ref[q] = move ? to : m_ref[q];     // (from -FLT_MAX a difference does not lead to `to`)
    else m_ref[q] += delta;
    nmc[q] = -m_ref[q] * scale_log2;
    l_run[q] *= alpha;
    asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        float x = o[q][dt][i], t;
        asm volatile("v_accvgpr_read_b32 %1, %0\n\ts_nop 1\n\tv_mul_f32 %1, %1, %2\n\ts_nop 1\n\tv_accvgpr_write_b32 %0, %1"
                     : "+a"(x), "=&v"(t) : "v"(alpha));
        o[q][dt][i] = x;
      }
    asm volatile("s_nop 7" ::: "memory");
  };
  // The probabilities P of the unit whose accumulators are in S were out of range; O holds all earlier units, so the reference
  // moves up and P (and rs_last) are recomputed.
  auto redo_unit = [&](const f32x16 (&S)[2], uint32_t (&P)[2][8]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float mx = rowmax(S[q]);
      move_reference(q, mx > m_ref[q], mx);
      rs_last[q] = 0.f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(S[q][i], scale_log2, nmc[q]));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(S[q][i + 1], scale_log2, nmc[q]));
        const bf16x2 pk = {(__bf16)p0, (__bf16)p1};
        rs_last[q] += p0 + p1;
        P[q][i / 2] = __builtin_bit_cast(uint32_t, pk);
      }
    }
  };
  // Keys past the end of the sequence, in the units of the ragged block.
  auto mask_unit = [&](f32x16 (&S)[2], int s) {
    const int t = s & 1, p = part_of(s >> 1) % PB;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int key = t * KH + 32 * p + 8 * (i / 4) + 4 * lh + (i % 4);
      if (key >= last_valid) S[0][i] = S[1][i] = -INFINITY;
    }
  };

  bool slow = partial_begin == 0, redo = false;   // mask the coming unit / the latest unit must be redone
  bf16x8 kr[2][NQ], vr[2][NP];                    // operands of the coming even and odd step
  // Step s: products S_{s+1} and V P_{s-1} around the softmax arithmetic of unit s, operand by operand.  Its registers are
  // reloaded for step s+2 (K tile at k_off, V^T tile at v_off) as soon as both MFMAs that read them are issued.  An MFMA
  // takes eight issue slots of the SIMD; behind the first of an operand come the exponentials of a pair of
  // probabilities, behind the second its sum and packing and the load.
  auto step = [&](auto odd_tag, int s, f32x16 (&Scur)[2], f32x16 (&Snext)[2], uint32_t (&Pprev)[2][8], uint32_t (&Pcur)[2][8],
                  uint32_t k_off, uint32_t v_off) {
    constexpr int ODD = decltype(odd_tag)::value ? 1 : 0;
    if (slow) {
      if (redo) redo_unit(Snext, Pprev);          // (the accumulators of unit s-1 are still in the buffer this step overwrites)
      if (s > 0 && s >= partial_begin) mask_unit(Scur, s);
    }
    l_run[0] += rs_last[0];
    l_run[1] += rs_last[1];
    __builtin_amdgcn_sched_barrier(0);
    float rs[2] = {}, e0 = 0.f, e1 = 0.f;
#pragma unroll
    for (int g = 0; g < NQ + NP; ++g) {
      const int tile = g / 8, i = 2 * (g % 8), j = g - NQ;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (g < NQ) qk_stream(Snext[q], kr[ODD][g], qf[q][g], g == 0);
        else o[q][j / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[ODD][j], operand_p(Pprev[q], j % 2), o[q][j / 2], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (q == 0) {
          e0 = __builtin_amdgcn_exp2f(fmaf(Scur[tile][i], scale_log2, nmc[tile]));
          e1 = __builtin_amdgcn_exp2f(fmaf(Scur[tile][i + 1], scale_log2, nmc[tile]));
          asm volatile("" : "+v"(e0), "+v"(e1));
        } else {
          if (g < NQ) kr[ODD][g] = k_load(k_off, g);
          else vr[ODD][j] = v_load(v_off, j);
          asm volatile("" ::: "memory");          // (the load stays here: the compiler would move it to its use in the next round)
          const bf16x2 pk = {(__bf16)e0, (__bf16)e1};
          uint32_t w = __builtin_bit_cast(uint32_t, pk);
          rs[tile] = (i == 0) ? e0 + e1 : rs[tile] + (e0 + e1);
          asm volatile("" : "+v"(w), "+v"(rs[tile]));
          Pcur[tile][i / 2] = w;
        }
        __builtin_amdgcn_sched_barrier(0);        // the slots stay in this order
      }
    }
    rs_last[0] = rs[0];
    rs_last[1] = rs[1];
    redo = __builtin_amdgcn_ballot_w64(!(rs[0] + rs[1] <= 1.0995e12f)) != 0ull;    // rare: above 2^40 or not finite
    slow = redo || (s + 1 >= partial_begin);
  };

  if (U > 0) {
    uint32_t off0 = part_off(list_entry(part_of(0)), part_of(0)), off1 = part_off(list_entry(part_of(1)), part_of(1));   // parts P, P + 1
    bf16x8 k0[NQ];
#pragma unroll
    for (int c = 0; c < NQ; ++c) k0[c] = k_load(off0, c);
#pragma unroll
    for (int c = 0; c < NQ; ++c) kr[0][c] = k_load(off0 + K_TILE, c);
    {
      // (between the operands of the two steps: in the loop as many loads lie between an operand's load and its use, and the
      // compiler's wait counts are the smaller of the two)
      const __bf16* qrow = qp + q_head_off + (size_t)q_row * D + 8 * lh;
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int ds = 0; ds < DS; ++ds) qf[q][ds] = *reinterpret_cast<const bf16x8*>(qrow + q * 32 * D + 16 * ds);
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int c = 0; c < NQ; ++c) kr[1][c] = k_load(off1, c);
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      vr[1][j] = v_load(off0, j);
#pragma unroll
      for (int e = 0; e < 8; ++e) vr[0][j][e] = (__bf16)0.f;       // step 0 has no unit before it: it adds 0 x 0
    }
    f32x16 Sa[2], Sb[2];
    uint32_t Pa[2][8], Pb[2][8];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int ds = 0; ds < DS; ++ds) qk_stream(Sa[q], k0[ds], qf[q][ds], ds == 0);
      asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 1" : "+v"(Sa[q]));   // (what an 8-pass MFMA needs before its result is read)
#pragma unroll
      for (int e = 0; e < 8; ++e) Pb[q][e] = 0u;
#pragma unroll
      for (int i = 0; i < 16; ++i) Sb[q][i] = 0.f;
    }
    if (partial_begin == 0) mask_unit(Sa, 0);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      // (minus infinity in all products of a later unit of a list is no reference: it weighs nothing, also where a share begins)
      m_ref[q] = KS > 1 && grp > 0 ? fmaxf(rowmax(Sa[q]), -FLT_MAX) : rowmax(Sa[q]);
      nmc[q] = -m_ref[q] * scale_log2;
    }
    // A list entry is read a round before it is turned into an offset, so that no step waits for a scalar memory load.
    int entry = list_entry(part_of(2));
    for (int s = 0; s < U; s += 2) {
      const int P = s >> 1;
      // (two wavefronts that walk one list meet every 16 parts: left alone they drift apart, out of reach of each other's
      // tiles in L1.  720p, 24 heads, 11.25 -> 10.99 ms; every part or every 4th: as much, and dearer on short lists.  Four
      // wavefronts of a 256-row Q block lose 2 %)
      if (QH == 2 && KS == 1 && P % 16 == 0) __builtin_amdgcn_s_barrier();
      const uint32_t off2 = part_off(entry, part_of(P + 2));
      entry = list_entry(part_of(P + 3));
      // even step: S of unit s+1 (part P, tile 1), V P of unit s-1; loads K of part P+1, tile 1 and V of part P, tile 1
      step(std::false_type{}, s, Sa, Sb, Pb, Pa, off1 + K_TILE, off0 + V_TILE);
      // odd step: S of unit s+2 (part P+1, tile 0), V P of unit s; loads K of part P+2, tile 0 and V of part P+1, tile 0
      step(std::true_type{}, s + 1, Sb, Sa, Pa, Pb, off2, off1);
      off0 = off1;
      off1 = off2;
    }
    // ---- last product: O += V P_{U-1} -----------------------------------------------------------------
    if (redo) redo_unit(Sb, Pb);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      l_run[q] += rs_last[q];
#pragma unroll
      for (int j = 0; j < NP; ++j)
        o[q][j / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[0][j], operand_p(Pb[q], j % 2), o[q][j / 2], 0, 0, 0);
    }
  }

  // ---- normalise (the final division of eq. 4) and write this wavefront's rows ------------------------------------
  float l_tot[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run[q]), __float_as_uint(l_run[q]), false, false);
    l_tot[q] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
  }
  // ---- merge of the shares: wavefront x KS / TILES finishes 32 x 32 tile x = q DT + dt ----------------------------
  // Every wavefront leaves the tiles it does not finish and its row statistics in LDS and rescales what it reads to the
  // largest reference of the row.
  constexpr int TILES = 2 * DT;
  auto finishes = [&](int q, int dt) { return KS == 1 || grp == (q * DT + dt) * KS / TILES; };
  if constexpr (KS > 1) {
    __shared__ float4 tiles[QH][KS][TILES - TILES / KS][4][64];
    __shared__ float2 stats[QH][KS][2][32];
    auto place = [&](int owner, int x) { return x < owner * TILES / KS ? x : x - TILES / KS; };   // (its own tiles take no place)
#pragma unroll
    for (int x = 0; x < TILES; ++x)
      if (!finishes(x / DT, x % DT)) {
        const f32x16& t = o[x / DT][x % DT];
        float4* const to = &tiles[half][grp][place(grp, x)][0][lane];
#pragma unroll
        for (int g = 0; g < 4; ++g) to[g * 64] = make_float4(t[4 * g], t[4 * g + 1], t[4 * g + 2], t[4 * g + 3]);
      }
    if (lh == 0) {
      stats[half][grp][0][l32] = make_float2(m_ref[0], l_tot[0]);
      stats[half][grp][1][l32] = make_float2(m_ref[1], l_tot[1]);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float m_all = m_ref[q];
      float2 st_of[KS];
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        st_of[k] = stats[half][k][q][l32];
        m_all = fmaxf(m_all, st_of[k].x);
      }
      const float own = __builtin_amdgcn_exp2f((m_ref[q] - m_all) * scale_log2);
      l_tot[q] = 0.f;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
        if (finishes(q, dt))
#pragma unroll
          for (int i = 0; i < 16; ++i) o[q][dt][i] *= own;
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const float w = __builtin_amdgcn_exp2f((st_of[k].x - m_all) * scale_log2);
        l_tot[q] = fmaf(st_of[k].y, w, l_tot[q]);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          if (k != grp && finishes(q, dt)) {
            const float4* const from = &tiles[half][k][place(k, q * DT + dt)][0][lane];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const float4 x = from[g * 64];
              o[q][dt][4 * g] = fmaf(x.x, w, o[q][dt][4 * g]);
              o[q][dt][4 * g + 1] = fmaf(x.y, w, o[q][dt][4 * g + 1]);
              o[q][dt][4 * g + 2] = fmaf(x.z, w, o[q][dt][4 * g + 2]);
              o[q][dt][4 * g + 3] = fmaf(x.w, w, o[q][dt][4 * g + 3]);
            }
          }
      }
      m_ref[q] = m_all;
    }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float f = l_tot[q] > 0.f ? 1.0f / l_tot[q] : 0.f;   // a row with no kept key yields zeros
    const size_t row = (size_t)q_row + 32 * q;
    // plain output: row `row` of the permuted layout; fused inverse permutation: the token's raster row
    const int target = scatter ? scatter[row] : (int)row;
    if (target < 0) continue;                                 // padding row of the last block
    __bf16* orow = scatter ? op + ((bh / heads) * st.batch + (bh % heads) * st.head + (long long)target * st.token) * D
                           : op + q_head_off + row * D;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      if (finishes(q, dt))
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          bf16x4 pk;
#pragma unroll
          for (int e = 0; e < 4; ++e) pk[e] = (__bf16)(o[q][dt][4 * g + e] * f);
          *reinterpret_cast<bf16x4*>(orow + 32 * dt + 8 * g + 4 * lh) = pk;
        }
    if (lse != nullptr && lh == 0 && finishes(q, 0))
      lse[scatter ? (size_t)bh * n_tokens + target : (size_t)bh * (Tq << split) * BQ + row] =
          m_ref[q] * scale_log2 * 0.6931471805599453f + __logf(l_tot[q]);
  }
}

struct AttnArgs {
  const void *qp, *kp, *vp;
  const int32_t *blk_idx, *blk_cnt;
  void* out;
  float* lse;
  bool scatter;
};

// Numbering of a plan's rows, and the slots of an XCD: its run of the sink rows of all heads, then its ordinary rows.
RowOrder row_order(const rf2_plan* plan, unsigned* slots) {
  const rf2_info& in = plan->info;
  const int n_bh = plan->cfg.batch * plan->cfg.heads, n_sink = in.sink_block_end - in.sink_block_begin;
  const int sink_slots = (int)(((int64_t)n_bh * n_sink + 7) / 8);
  const int run = (int)(((int64_t)n_bh * (in.n_blocks - n_sink) + 7) / 8);
  const bool whole = plan->cut.whole_heads;
  *slots = (unsigned)sink_slots + (whole ? (unsigned)run : (unsigned)n_bh * (unsigned)plan->plain_per_xcd);
  return {whole ? nullptr : plan->d_row_order, whole ? run : plan->plain_per_xcd, n_bh, in.n_blocks, in.sink_block_begin, n_sink, sink_slots};
}

template <int D, int BQ, int BK, int KS>
int launch_ring(const rf2_plan* plan, const AttnArgs& a, hipStream_t st) {
  using C = AttnCfg<D, BQ, BK, KS>;
  const rf2_info& in = plan->info;
  const int split = plan->cfg.block > BQ ? 1 : 0;
  unsigned slots;
  const RowOrder order = row_order(plan, &slots);
  if (slots == 0) return RF2_OK;
  block_sparse_attn_kernel<D, BQ, BK, KS><<<dim3((8u * slots) << split), dim3(C::NT * KS), 0, st>>>(
      (const __bf16*)a.qp, (const __bf16*)a.kp, (const __bf16*)a.vp, a.blk_idx, a.blk_cnt, (__bf16*)a.out, a.lse, order,
      in.n_blocks_k, in.k_row, in.last_block_valid_k, (float)(1.4426950408889634 / sqrt((double)D)),
      a.scatter ? plan->d_perm : nullptr, (int)in.N, plan->cfg.heads, rf2_qkv_strides(plan), split);
  RF2_LAUNCH_CHECK();
  return RF2_OK;
}

template <int D, int BK, int QH, int KS>
int launch_stream(const rf2_plan* plan, const AttnArgs& a, hipStream_t st) {
  const rf2_info& in = plan->info;
  const int share = plan->cfg.block / (64 * QH), split = share / 2;      // workgroups of a Q block: 1, 2, 4
  if (share < 1) return RF2_ERR_UNSUPPORTED;                             // (no cut has more rows than a Q block)
  unsigned slots;
  const RowOrder order = row_order(plan, &slots);
  if (slots == 0) return RF2_OK;
  stream_attn_kernel<D, BK, QH, KS><<<dim3((8u * slots) << split), dim3(64 * QH * KS), 0, st>>>(
      (const __bf16*)a.qp, (const __bf16*)a.kp, (const __bf16*)a.vp, a.blk_idx, a.blk_cnt, (__bf16*)a.out, a.lse, order,
      in.n_blocks_k, in.k_row, in.last_block_valid_k, (float)(1.4426950408889634 / sqrt((double)D)),
      a.scatter ? plan->d_perm : nullptr, (int)in.N, plan->cfg.heads, rf2_qkv_strides(plan), split);
  RF2_LAUNCH_CHECK();
  return RF2_OK;
}

template <int D, int BK>
int dispatch_cut(const rf2_plan* plan, const AttnArgs& a, hipStream_t st) {
  const rf2_attn_cut& cut = plan->cut;
  if constexpr (D == 128) {
#define RF2_ATTN_CASE(QH, KS) \
  if (cut.rows == 64 * QH && cut.groups == KS) return launch_stream<D, BK, QH, KS>(plan, a, st);
    RF2_ATTN_CASE(1, 1)
    RF2_ATTN_CASE(2, 1)
    RF2_ATTN_CASE(4, 1)
    RF2_ATTN_CASE(1, 2)
    RF2_ATTN_CASE(2, 2)
    RF2_ATTN_CASE(1, 4)
#undef RF2_ATTN_CASE
  } else {
#define RF2_ATTN_CASE(Q, KS) \
  if (cut.rows == Q && cut.groups == KS) return launch_ring<D, Q, BK, KS>(plan, a, st);
    RF2_ATTN_CASE(64, 1)
    RF2_ATTN_CASE(128, 1)
    RF2_ATTN_CASE(256, 1)
    RF2_ATTN_CASE(64, 2)
    RF2_ATTN_CASE(128, 2)
    RF2_ATTN_CASE(64, 4)
    RF2_ATTN_CASE(128, 4)
#undef RF2_ATTN_CASE
  }
  return RF2_ERR_UNSUPPORTED;
}

template <int D>
int dispatch_blocks(const rf2_plan* plan, const AttnArgs& a, hipStream_t st) {
  if (plan->info.block_k == 128) return dispatch_cut<D, 128>(plan, a, st);
  if (plan->info.block_k == 64) return dispatch_cut<D, 64>(plan, a, st);
  return RF2_ERR_UNSUPPORTED;
}

int dispatch_attn(const rf2_plan* plan, const void* qp, const void* kp, const void* vp, const int32_t* blk_idx,
                  const int32_t* blk_cnt, void* out, float* lse, bool scatter, void* stream) {
  if (!plan || !qp || !kp || !vp || !blk_idx || !blk_cnt || !out) return RF2_ERR_INVALID_ARG;
  if (const int rc = rf2_check_device(plan)) return rc;
  hipStream_t st = (hipStream_t)stream;
  const AttnArgs a{qp, kp, vp, blk_idx, blk_cnt, out, lse, scatter};
  if (plan->cfg.head_dim == 128) return dispatch_blocks<128>(plan, a, st);
  if (plan->cfg.head_dim == 64) return dispatch_blocks<64>(plan, a, st);
  return RF2_ERR_UNSUPPORTED;
}

}  // namespace

extern "C" int rf2_block_sparse_attn(const rf2_plan* plan, const void* qp, const void* kp, const void* vp,
                                     const int32_t* blk_idx, const int32_t* blk_cnt, void* op, float* lse,
                                     void* stream) {
  return dispatch_attn(plan, qp, kp, vp, blk_idx, blk_cnt, op, lse, false, stream);
}

extern "C" int rf2_block_sparse_attn_unpermuted(const rf2_plan* plan, const void* qp, const void* kp, const void* vp,
                                                const int32_t* blk_idx, const int32_t* blk_cnt, void* o, float* lse,
                                                void* stream) {
  return dispatch_attn(plan, qp, kp, vp, blk_idx, blk_cnt, o, lse, true, stream);
}
