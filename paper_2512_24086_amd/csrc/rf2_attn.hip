// Block-sparse flash attention (Sec. 3.1, eqs. 1-4 with the block skip rule) for gfx950.
//
// A wavefront owns 64 query rows (two tiles of 32) of one Q block of one (batch, head) and walks that row's list of kept K/V
// blocks (b_k rows each; b_q and b_k may differ), or a share of it.
//
// Both products are computed transposed so that no register shuffling is needed between them
// (v_mfma_f32_32x32x16_bf16, D = A(32xk) * B(kx32) + C):
//   S^T[key][query]  = K (A)   * Q^T (B, registers, loaded once)
//   O^T[chan][query] = V^T (A) * P^T (B, registers = exp of the S^T accumulators)
// In the accumulator layout lane l holds query column l%32 and, per 32-key tile, keys
// 8*(i/4) + 4*(l/32) + i%4 for i = 0..15.  Eight consecutive accumulator values are exactly one
// B operand of the second product provided the A operand (V^T) lists the keys of each 16-key
// group in the order 0-3, 8-11, 4-7, 12-15 -- the order rf2_permute writes.  Row statistics are
// per lane (one query column) plus one exchange with lane l^32.
//
// Operands come straight from memory into registers, 1.5 to 2 steps ahead of their use: a part (64 keys) of the layout that
// rf2_permute writes is read in 1 KiB pieces, each of which is one A operand and feeds two MFMAs.  There is no LDS in the
// loop, and no barrier except where wavefronts that share tiles or a list meet now and then (MEET).  Against rings in LDS with wavefronts of 32 rows, 4 to a workgroup, an operand
// is moved half as often and nothing passes through LDS, which the power limit turns into clock.  d = 128 (one wavefront per
// SIMD, 442 to 446 of its 512 registers, matrix cores 76 % busy on 720p where the rings kept two wavefronts 69 % busy): 720p, 40
// heads, 20.7 -> 19.1 ms on one card (18.0 to 20.1 from card to card, 1,292 to 1,158 TFLOP/s), 480p 4.00 -> 3.54 ms; with 64-row Q blocks, where the rings left one wavefront of 32
// rows per SIMD, 480p 5.13 -> 3.98 ms and 720p, 20 heads, 13.3 -> 10.8 ms.  d = 64 (two wavefronts per SIMD, 242 to 249 registers of 256 each) is
// bound by vector issue and power either way: 480p 2.12 -> 2.07 ms, 720p, 20 heads, 5.48 -> 5.38; with 64-row Q blocks 2.47 ->
// 2.12 ms.
//
// A workgroup has QH x KS wavefronts: QH times 64 neighbouring query rows of a Q block, whose wavefronts ask for the same
// tiles at about the same time and find each other's in the L1 cache (720p, d = 128, QH = 2 against two workgroups of 64 rows,
// 20.0 -> 19.2 ms), times KS shares of the list: wavefront k of a share walks parts k, k + KS, ... of it, and the
// shares are merged through LDS at the end.  rf2_cut_stream (rf2_attn_cut.h) chooses QH and KS.
//
// Softmax (eqs. 2, 3) without a per-unit row maximum: a probability is exp2(fma(q.k, c, -m_ref c))
// with c = log2(e)/sqrt(d), the subtraction of eq. (2) riding on the multiply-add that applies the
// scale.  m_ref is set exactly from the first 32-key unit of the wavefront and afterwards only moved when the row
// sum of a unit leaves the range fp32/bf16 carry without loss (> 2^40, or not finite); the final
// division by the row sum makes the reference point irrelevant.  The common path is one fused
// multiply-add, one exp2, one add and half a bf16 pack per probability.
#include "rf2_internal.h"

#include <algorithm>
#include <cfloat>
#include <type_traits>

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

// The S^T product is issued through assembly so that its accumulators are ordinary vector registers that the softmax
// arithmetic reads in place (the statements are volatile: they keep their places between loads and arithmetic).  The
// compiler does not know that they are MFMAs, so what it would do for an MFMA is done by hand:
//  * between the last MFMA of a chain and the first vector-ALU read of its result lie the 12 wait states that an 8-pass MFMA
//    needs: in the loop the frozen slots of at least one more MFMA with the arithmetic behind it, in front of the loop a wait;
//  * the first MFMA of a chain takes the constant 0 as its addend, so no register is read by the
//    matrix core after issue except the A and B operands;
//  * A and B operands are read at issue; they come from loads (the compiler waits for them) and the resident Q fragments.
// ACC: Q lies in accumulation registers.
template <bool ACC>
__device__ __forceinline__ void qk(f32x16& S, const bf16x8& a, const bf16x8& b, bool first) {
  if constexpr (ACC) {
    if (first) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(S) : "v"(a), "a"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(S) : "v"(a), "a"(b));
  } else {
    if (first) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(S) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(S) : "v"(a), "v"(b));
  }
}

// Tells the compiler that a pointer is the same in every lane (it then lives in scalar registers).
__device__ __forceinline__ const unsigned char* uniform_ptr(const void* p) {
  const uint64_t v = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const unsigned char*)(((uint64_t)hi << 32) | lo);
}

// Place of 16-byte chunk `chunk` of row `row` among rows of CPR chunks in LDS: 16 lanes that move the same chunk of neighbouring
// rows, or the chunks of a row in turn, meet different banks.
template <int CPR>
__device__ __forceinline__ int row_slot(int row, int chunk) {
  return row * CPR + (chunk ^ (row / (16 / CPR) % CPR));
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

// Parameters of both kernels, what a row needs first in front: the first 14 words arrive in registers (a compiler flag in
// build.py), the others are read from memory.  shares to sink_slots: RowOrder.  split: log2 of the workgroups that share a Q block; they are neighbours on one XCD.  Tb: K/V blocks
// per head (columns of the block mask); last_valid: tokens in the last one; perm: token of a permuted row; fused: output in the
// caller's token order; meets: wavefronts of four shares meet (see rf2_cut_stream).
#define RF2_STREAM_PARAMS \
  const int32_t *__restrict__ shares, int per_xcd, int n_bh, int rows, int sink_begin, int n_sink, int sink_slots, int split, int k_row, \
      const int32_t *__restrict__ blk_idx, const int32_t *__restrict__ blk_cnt, const __bf16 *__restrict__ qp, \
      const __bf16 *__restrict__ kp, const __bf16 *__restrict__ vp, const int32_t *__restrict__ perm, __bf16 *__restrict__ op, \
      float *__restrict__ lse, int Tb, int last_valid, float scale_log2, int n_tokens, int heads, bool fused, bool meets, rf2_strides st
#define RF2_STREAM_ARGS(split) \
  shares, per_xcd, n_bh, rows, sink_begin, n_sink, sink_slots, split, k_row, blk_idx, blk_cnt, qp, kp, vp, perm, op, lse, Tb, last_valid, \
      scale_log2, n_tokens, heads, fused, meets, st

// One workgroup: number `share` of those of a Q block, number `slot` of the XCD's rows.
template <int D, int BK, int QH, int KS>
__device__ __forceinline__ void attend(RF2_STREAM_PARAMS, int xcd, int slot, int share) {
  constexpr int BQ = 64 * QH, KH = BK / 2, PB = BK / 64, DS = D / 16, DT = D / 32;
  constexpr int TILE_BYTES = BK * D * 2, PART_BYTES = 64 * D * 2;
  int bh, qi;
  if (!row_of({shares, per_xcd, n_bh, rows, sink_begin, n_sink, sink_slots}, xcd, slot, bh, qi)) return;
  const int Tq = rows;
  const size_t row_id = (size_t)bh * Tq + qi;
  const auto* const list = (const __attribute__((address_space(4))) int32_t*)(blk_idx + row_id * k_row);   // (scalar loads)
  const int wave = QH * KS > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : 0;
  const int half = wave % QH, grp = wave / QH;
  const int lane = (int)threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
  // The start of a row is a chain of latencies that nothing covers, so what can be asked for at once is: the count, the list's
  // entries of the wavefront's first three parts and its last one as if it were full (behind the count lies whatever the caller
  // left, inside the list and clamped like any entry; it is replaced or never multiplied), Q, and the rows of the output.  (One
  // after the other: tiny layer 21.9 us, now 21.2, image of 24 heads 137.9, now 135.0; 480p and larger layers +0.0 to +0.4 %.)
  int cnt = blk_cnt[row_id];
  int ahead[3];
#pragma unroll
  for (int p = 0; p < 3; ++p) ahead[p] = list[min((p * KS + grp) / PB, k_row - 1)];
  int tail = list[k_row - 1];
  __builtin_amdgcn_sched_barrier(0);
  const size_t q_head_off = (size_t)bh * (Tq << split) * BQ * D;             // elements; qp and op
  const int q_row = ((qi << split) + share) * BQ + 64 * half + l32;          // this lane's query row of tile 0 in its head
  bf16x8 q_in[2][DS];
  const __bf16* const q_from = qp + q_head_off + (size_t)(q_row - l32) * D + 8 * lane;
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int i = 0; i < DS; ++i) q_in[q][i] = *reinterpret_cast<const bf16x8*>(q_from + q * 32 * D + i * 512);
  int token = perm[q_row - l32 + lane];                                      // of the wavefront's row `lane`; -1: padding of the last block
  // where the head's rows go, and how far they are apart
  uint64_t out_at = (uint64_t)(fused ? op + ((bh / heads) * st.batch + (bh % heads) * st.head) * D : op + q_head_off);
  uint32_t out_pitch = fused ? (uint32_t)st.token * (D * 2) : D * 2;
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" : "+s"(out_at), "+s"(out_pitch));
  asm("" : "+s"(cnt), "+s"(tail), "+s"(ahead[0]), "+s"(ahead[1]), "+s"(ahead[2]));   // (left alone, the entries wait for the count)
  const bool dense = (cnt == Tb);
  cnt = dense ? Tb : min(max(cnt, 0), k_row);
  // Only the last listed block can be the ragged last block of the sequence (lists ascend).
  bool ragged = false;
  if (cnt > 0 && last_valid < BK) {
    const int jl = dense ? cnt - 1 : cnt == k_row ? tail : list[cnt - 1];
    ragged = min(max(jl, 0), Tb - 1) == Tb - 1;
  }
  int NPARTS = cnt * PB;
  // (a last part without any valid key is left out, so that every wavefront has a valid key in its first unit)
  if (KS > 1 && PB > 1 && ragged && last_valid <= 32) --NPARTS;
  const int parts = KS > 1 ? max(NPARTS - grp + KS - 1, 0) / KS : NPARTS;    // this wavefront's: grp, grp + KS, ...
  const int U = 2 * parts;                                                   // its 32-key units (even)
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
  // (its entry is read without a branch and, where the row keeps all blocks, not used)
  auto list_entry = [&](int P) { return list[min((int)((unsigned)min(P, NPARTS - 1) / (unsigned)PB), k_row - 1)]; };
  auto part_off = [&](int entry, int P) {
    const int it = (int)((unsigned)min(P, NPARTS - 1) / (unsigned)PB);
    const int j = min(max(dense ? it : entry, 0), Tb - 1);     // a corrupt list can give wrong results, never a fault
    return (uint32_t)j * (uint32_t)TILE_BYTES + ((unsigned)min(P, NPARTS - 1) % (unsigned)PB) * (uint32_t)PART_BYTES;
  };
  auto part_of = [&](int P) { return P * KS + grp; };    // list part of this wavefront's part P
  const int partial_begin = ragged ? 2 * (max((cnt - 1) * PB - grp + KS - 1, 0) / KS) : U;   // first unit of the ragged block

  // Q and O pass through LDS on their way between memory, where a wavefront moves whole rows, and registers, where a lane has
  // pieces of one row: 16 or 8 bytes a lane at a stride of a row keep the address unit of a compute unit busy for 64 cycles an
  // instruction, 2,048 of them for the O of a wavefront, where whole rows take 16.  (480p, us from row to row of a place, beside a
  // loop of 125: last product to last store acknowledged 3.2 -> 2.0, end to next start 1.7 -> 0.9, start to first unit 2.8 -> 2.6,
  // with the arguments in registers.  Layers: tiny 21.0 -> 19.5 us, image 130 -> 126.5, 480p 3,867 -> 3,840, with 64-row blocks 4,136 ->
  // 4,089; attention alone, d = 64 480p 2,129 -> 2,103, ten heads of 256-row blocks 463.6 -> 455.4, long video +0.5 %.)
  constexpr int TILES = 2 * DT, OWN = TILES >= KS ? TILES / KS : 1;          // 32 x 32 tiles of O, those that a wavefront finishes
  constexpr int OC = 4 * std::min(OWN, DT);                                  // 16-byte chunks of a row that it finishes
  __shared__ uint4 out_rows[QH * KS][32 * OC];
  __shared__ int targets[QH * KS][64];                                       // where these rows go
  __shared__ float4 tiles[QH][KS][KS > 1 ? TILES - TILES / KS : 1][KS > 1 ? 4 : 1][KS > 1 ? 64 : 1];
  bf16x8 qf[2][DS];
  // plain output: the row of the permuted layout; fused inverse permutation: the token's raster row
  auto note_targets = [&] {
    asm volatile("" : "+v"(token));          // (left alone, it is waited for before the first tiles are asked for)
    targets[wave][lane] = fused ? token : q_row - l32 + lane;
  };
  auto spread_q = [&] {
    note_targets();
    uint4* const staged = KS > 1 ? reinterpret_cast<uint4*>(&tiles[half][grp]) : out_rows[wave];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int i = 0; i < DS; ++i)
        staged[row_slot<D / 8>(lane / (D / 8) + i * (512 / D), lane % (D / 8))] = __builtin_bit_cast(uint4, q_in[q][i]);
      wave_fence();
#pragma unroll
      for (int ds = 0; ds < DS; ++ds) qf[q][ds] = __builtin_bit_cast(bf16x8, staged[row_slot<D / 8>(l32, 2 * ds + lh)]);
      wave_fence();
    }
  };

  f32x16 o[2][DT];
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[q][dt][i] = 0.f;
  // Softmax reference m_ref (per query tile and column, in units of the raw products q.k) and nmc = -m_ref * c, the addend of the
  // multiply-add in front of every exp2.  l_run lags one unit behind: rs_last, the row sum of the latest unit, is still to be
  // added.  (A wavefront without any part of its own weighs nothing in the merge, however small the others' references are.)
  float m_ref[2], nmc[2] = {}, l_run[2] = {}, rs_last[2] = {};
  m_ref[0] = m_ref[1] = KS > 1 && U == 0 ? -FLT_MAX : 0.f;
  constexpr int NQ = DS, NP = DT * 2;                    // operands of a unit: K, V^T
  // k-step ks of the second product's B operand from the packed probabilities of a unit
  auto operand_p = [](const uint32_t (&P)[8], int ks) {
    const u32x4 w = {P[4 * ks], P[4 * ks + 1], P[4 * ks + 2], P[4 * ks + 3]};
    return __builtin_bit_cast(bf16x8, w);
  };
  // largest accumulator of one unit per query column (both lane halves end up with the same value)
  auto rowmax = [&](const f32x16& S) -> float {
    float v = S[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) v = fmaxf(v, S[i]);
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
  };
  // Moves the reference of tile q to `to` (per query column, where `move`): everything accumulated so far is rescaled
  // (eqs. 3, 4).  The accumulators hold raw products, so nothing else changes.
  auto move_reference = [&](int q, bool move, float to) {
    const float delta = move ? to - m_ref[q] : 0.f;
    const float alpha = __builtin_amdgcn_exp2f(-fmaxf(delta, 0.f) * scale_log2);
    if constexpr (KS > 1) m_ref[q] = move ? to : m_ref[q];     // (from -FLT_MAX a difference does not lead to `to`)
    else m_ref[q] += delta;
    nmc[q] = -m_ref[q] * scale_log2;
    l_run[q] *= alpha;
    if constexpr (D == 64) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[q][dt][i] *= alpha;
    } else {
      // In accumulation registers: scaled where they are, through one vector register (left to the compiler, the copies cost
      // the registers of the loop).  The wait states in front cover a product in flight, those behind one that follows.
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
    }
  };
  // Probabilities of the unit of tile q whose accumulators are in S, once more: they were out of range (rare), O holds all earlier
  // units, so the reference moves up and P (and rs_last) are recomputed.
  auto redo_tile = [&](int q, const f32x16& S, uint32_t (&P)[8]) {
    const float mx = rowmax(S);
    move_reference(q, mx > m_ref[q], mx);
    rs_last[q] = 0.f;
#pragma unroll
    for (int i = 0; i < 16; i += 2) {
      const float p0 = __builtin_amdgcn_exp2f(fmaf(S[i], scale_log2, nmc[q]));
      const float p1 = __builtin_amdgcn_exp2f(fmaf(S[i + 1], scale_log2, nmc[q]));
      const bf16x2 pk = {(__bf16)p0, (__bf16)p1};
      rs_last[q] += p0 + p1;
      P[i / 2] = __builtin_bit_cast(uint32_t, pk);
    }
  };
  constexpr float RANGE = 1.0995e12f;     // 2^40
  // Keys past the end of the sequence, in unit s of the ragged block.
  auto mask_tile = [&](f32x16& S, int s) {
    const int left = last_valid - ((s & 1) * KH + 32 * (part_of(s >> 1) % PB)) - 4 * lh;     // (held against constants)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (8 * (i / 4) + i % 4 >= left) S[i] = -INFINITY;
  };
  // S and the references of the wavefront's first unit.
  auto first_unit = [&](f32x16 (&S)[2], const bf16x8 (&k0)[NQ]) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int ds = 0; ds < DS; ++ds) qk<D == 128>(S[q], k0[ds], qf[q][ds], ds == 0);
      asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 1" : "+v"(S[q]));
    }
    if (partial_begin == 0) mask_tile(S[0], 0), mask_tile(S[1], 0);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      // (minus infinity in all products of a later unit of a list is no reference: it weighs nothing, also where a share begins)
      m_ref[q] = KS > 1 && grp > 0 ? fmaxf(rowmax(S[q]), -FLT_MAX) : rowmax(S[q]);
      nmc[q] = -m_ref[q] * scale_log2;
    }
  };
  // Offset of this wavefront's part p < 3, from the entry that was asked for ahead (past the end of the list: any part in bounds).
  auto first_off = [&](int p) {
    const int P = part_of(p), j = min(max(dense ? P / PB : ahead[p], 0), Tb - 1);
    return (uint32_t)j * (uint32_t)TILE_BYTES + (unsigned)(P % PB) * (uint32_t)PART_BYTES;
  };
  // Two wavefronts that ask for the same tiles meet every 16 parts: left alone they drift apart, out of reach of each other's
  // tiles in L1 (d = 128, 720p, 24 heads, 11.25 -> 10.99 ms, 480p 3.59 -> 3.56; every part or every 4th: no more, and dearer on
  // short lists; d = 64, KS = 2, 480p 2.122 -> 2.109 ms.  Four wavefronts of a 256-row Q block lose 2 %).
  // Four shares of a long list: at every part, for its tiles in L2 (rf2_cut_stream says where).
  constexpr int MEET = QH == 2 && (D == 64 || KS == 1) ? 16 : D == 128 && KS == 4 ? 1 : 0;
  const bool meeting = MEET == 16 || (MEET > 0 && meets);
  auto meet = [&](int part = 0) {
    if (meeting && part % std::max(MEET, 1) == 0) __builtin_amdgcn_s_barrier();
  };
  // Every wavefront of a list meets as often as the one with the most parts: also one that has a part less, or none.
  const int most = (NPARTS + KS - 1) / KS;
  // The order of the loads in front of the loops is that of the loops: the compiler's wait counts are the smaller of the two.

  if constexpr (D == 128) {
    // Registers: O^T 128 and Q 64 accumulation registers, S^T of two units 64, P of two units 32, operands of two steps 128.
    bf16x8 kr[2][NQ], vr[2][NP];                    // operands of the coming even and odd step
    // Step s: products S_{s+1} and V P_{s-1} around the softmax arithmetic of unit s, operand by operand.  Its registers are
    // reloaded for step s+2 (K tile at k_off, V^T tile at v_off) as soon as both MFMAs that read them are issued.  An MFMA
    // takes eight issue slots of the SIMD, two of them its own; behind the first of an operand come the exponentials of a pair of
    // probabilities (two slots each) and their arguments, which fills it, behind the second its sum and packing and the load, and what
    // else there is to do: `spare(g)`.
    // The wavefront issues one instruction after the other, so what stood between two steps (offsets, the list, the checks of the
    // last unit, branches around the rare cases) held up the MFMAs; in their open slots it does not (attention at 480p 3,496 -> 3,404
    // us, 720p +1.3 to 2.6 %, ten heads of 256-row blocks 454.5 -> 449.7, 480p with 64-row blocks, whose operands come late, 3,854 ->
    // 3,856).  Wavefronts that share a long list drift further apart at this pace: four shares meet for that, two were left 1 to 3 %
    // slower on long launches of 64-row blocks (12 heads of 75,600 tokens 6,630 -> 6,780, 16 of 69,012 10,236 -> 10,551; meeting every 4 or
    // 16 parts and one wait per operand change that by less than launches of one binary differ).  K and V through rings in LDS, filled for both wavefronts at once, was 9 % slower (480p): writes to LDS take
    // longer to issue than the loads that they save.
    auto step = [&](auto odd_tag, int s, f32x16 (&Scur)[2], f32x16 (&Snext)[2], uint32_t (&Pprev)[2][8], uint32_t (&Pcur)[2][8],
                    uint32_t k_off, uint32_t v_off, auto spare) {
      constexpr int ODD = decltype(odd_tag)::value ? 1 : 0;
      __builtin_amdgcn_sched_barrier(0);
      float rs[2] = {}, e0 = 0.f, e1 = 0.f;
      int limit = 0;
#pragma unroll
      for (int g = 0; g < NQ + NP; ++g) {
        const int tile = g / 8, i = 2 * (g % 8), j = g - NQ;
        if (g % 2 == 0) {                         // (one wait for two operands)
          if (g < NQ) asm volatile("" ::"v"(kr[ODD][g + 1]));
          else asm volatile("" ::"v"(vr[ODD][j + 1]));
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (g < NQ) qk<true>(Snext[q], kr[ODD][g], qf[q][g], g == 0);
          else o[q][j / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[ODD][j], operand_p(Pprev[q], j % 2), o[q][j / 2], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          if (q == 0) {
            e0 = __builtin_amdgcn_exp2f(fmaf(Scur[tile][i], scale_log2, nmc[tile]));
            e1 = __builtin_amdgcn_exp2f(fmaf(Scur[tile][i + 1], scale_log2, nmc[tile]));
            asm volatile("" : "+v"(e0), "+v"(e1));
          } else {
            if (g < NQ) kr[ODD][g] = k_load(k_off, g);
            else vr[ODD][j] = v_load(v_off, j);
            asm volatile("" ::: "memory");        // (the load stays here: the compiler would move it to its use in the next round)
            const bf16x2 pk = {(__bf16)e0, (__bf16)e1};
            uint32_t w = __builtin_bit_cast(uint32_t, pk);
            rs[tile] = (i == 0) ? e0 + e1 : rs[tile] + (e0 + e1);
            asm volatile("" : "+v"(w), "+v"(rs[tile]));
            Pcur[tile][i / 2] = w;
            if (i == 0) {
              l_run[tile] += rs_last[tile];
              asm volatile("" : "+v"(l_run[tile]));
            }
            if (g == 13) {
              limit = s + 1 >= partial_begin ? __builtin_bit_cast(int, -1.f) : __builtin_bit_cast(int, RANGE);
              asm volatile("" : "+s"(limit));
            }
            spare(g);
          }
          __builtin_amdgcn_sched_barrier(0);      // the slots stay in this order
        }
      }
      rs_last[0] = rs[0];
      rs_last[1] = rs[1];
      // One branch, hardly ever taken: unit s is out of range, or unit s+1 has keys past the end of the sequence.
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(rs[0] + rs[1] <= __builtin_bit_cast(float, limit))) != 0ull, 0)) {
        if (__builtin_amdgcn_ballot_w64(!(rs[0] + rs[1] <= RANGE)) != 0ull) redo_tile(0, Scur[0], Pcur[0]), redo_tile(1, Scur[1], Pcur[1]);
        if (s + 1 >= partial_begin) mask_tile(Snext[0], s + 1), mask_tile(Snext[1], s + 1);
      }
    };
    if (KS > 1 && U == 0 && most > 0) meet(0);
    if (U > 0) {
      uint32_t off0 = first_off(0), off1 = first_off(1);   // parts P, P + 1
      bf16x8 k0[NQ];
#pragma unroll
      for (int c = 0; c < NQ; ++c) k0[c] = k_load(off0, c);
#pragma unroll
      for (int c = 0; c < NQ; ++c) kr[0][c] = k_load(off0 + K_TILE, c);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int c = 0; c < NQ; ++c) kr[1][c] = k_load(off1, c);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        vr[1][j] = v_load(off0, j);
#pragma unroll
        for (int e = 0; e < 8; ++e) vr[0][j][e] = (__bf16)0.f;     // step 0 has no unit before it: it adds 0 x 0
      }
      f32x16 Sa[2], Sb[2];
      uint32_t Pa[2][8], Pb[2][8];
      spread_q();
      first_unit(Sa, k0);
      // (arrived before the loop, whose waits would else be those of its first round: vr[0] is not on its way yet)
#pragma unroll
      for (int c = 0; c < NQ; ++c) asm volatile("" : "+v"(kr[0][c]));
#pragma unroll
      for (int q = 0; q < 2; ++q) {
#pragma unroll
        for (int e = 0; e < 8; ++e) Pb[q][e] = 0u;
#pragma unroll
        for (int i = 0; i < 16; ++i) Sb[q][i] = 0.f;
      }
      // A list entry is read a round before it is turned into an offset, so that no step waits for a scalar memory load.
      int entry = ahead[2];
      for (int s = 0; s < U;) {
        meet();
        const int end = meeting ? min(U, s + 2 * MEET) : U;
        do {
          const int P = s >> 1;
          uint32_t off2 = 0;
          // even step: S of unit s+1 (part P, tile 1), V P of unit s-1; loads K of part P+1, tile 1 and V of part P, tile 1
          step(std::false_type{}, s, Sa, Sb, Pb, Pa, off1 + K_TILE, off0 + V_TILE, [&](int g) {
            if (g == 3) {
              off2 = part_off(entry, part_of(P + 2));
              asm volatile("" : "+s"(off2));
            } else if (g == 5) {
              entry = list_entry(part_of(P + 3));
            }
          });
          // odd step: S of unit s+2 (part P+1, tile 0), V P of unit s; loads K of part P+2, tile 0 and V of part P+1, tile 0
          step(std::true_type{}, s + 1, Sb, Sa, Pa, Pb, off2, off1, [](int) {});
          off0 = off1;
          off1 = off2;
          s += 2;
        } while (s < end);
      }
      if (KS > 1 && parts < most) meet(parts);
      // last product: O += V P_{U-1}
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        l_run[q] += rs_last[q];
#pragma unroll
        for (int j = 0; j < NP; ++j)
          o[q][j / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[0][j], operand_p(Pb[q], j % 2), o[q][j / 2], 0, 0, 0);
      }
    }
  } else {
    // The two tiles half a step apart, so that one S and one P of each are enough: O^T 64, Q 32, S^T 32, P 16, operands of two
    // steps 64 registers, two wavefronts per SIMD (with the tiles in step as above 274 registers, one wavefront: 480p 2.34 ms).
    bf16x8 kr[2][NQ], vr[2][NP];                    // operands of even and odd units
    f32x16 S[2];
    uint32_t P[2][8];
    // Half of step s for tile T: S_T of unit s+1 and O_T += V P_T of unit s, in turn, around the softmax arithmetic of the other
    // tile X (unit s of tile 1 in the first half, unit s+1 of tile 0 in the second).  In the second half the operands'
    // registers are reloaded for step s+2.
    // (checks, offsets and the list between MFMAs as above: 480p 2,078 -> 2,027 us, tiny layer 19.4 -> 19.1, with 64-row blocks 480p
    // 2,117 -> 2,108.)
    auto half_step = [&](auto tile_tag, auto odd_tag, int s, uint32_t k_off, uint32_t v_off, auto spare) {
      constexpr int T = decltype(tile_tag)::value ? 1 : 0, X = 1 - T, ODD = decltype(odd_tag)::value ? 1 : 0;
      __builtin_amdgcn_sched_barrier(0);
      float rs = 0.f, e[2][2];
      int limit = 0;
      // sum and packing of pair p, a slot behind its exponentials: no instruction waits for the one before it
      auto finish_pair = [&](int p) {
        const bf16x2 pk = {(__bf16)e[p & 1][0], (__bf16)e[p & 1][1]};
        uint32_t w = __builtin_bit_cast(uint32_t, pk);
        rs = p == 0 ? e[0][0] + e[0][1] : rs + (e[p & 1][0] + e[p & 1][1]);
        asm volatile("" : "+v"(w), "+v"(rs));
        P[X][p] = w;
      };
#pragma unroll
      for (int g = 0; g < NQ + NP; ++g) {
        const int j = g / 2;
        if (g % 2 == 0) qk<false>(S[T], kr[1 - ODD][j], qf[T][j], j == 0);
        else o[T][j / 2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[ODD][j], operand_p(P[T], j % 2), o[T][j / 2], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (T == 1) {
          if (g % 2 == 0) kr[1 - ODD][j] = k_load(k_off, j);
          else vr[ODD][j] = v_load(v_off, j);
          asm volatile("" ::: "memory");
        }
        if (g > 0) finish_pair(g - 1);
        if (g == 0) {
          l_run[T] += rs_last[T];
          asm volatile("" : "+v"(l_run[T]));
        }
        if (g == 5) {
          limit = s + 1 >= partial_begin ? __builtin_bit_cast(int, -1.f) : __builtin_bit_cast(int, RANGE);
          asm volatile("" : "+s"(limit));
        }
        spare(g);
        e[g & 1][0] = __builtin_amdgcn_exp2f(fmaf(S[X][2 * g], scale_log2, nmc[X]));
        e[g & 1][1] = __builtin_amdgcn_exp2f(fmaf(S[X][2 * g + 1], scale_log2, nmc[X]));
        asm volatile("" : "+v"(e[g & 1][0]), "+v"(e[g & 1][1]));
        if (g == 7) finish_pair(7);
        __builtin_amdgcn_sched_barrier(0);
      }
      rs_last[X] = rs;
      // One branch, hardly ever taken: the unit of X is out of range, or unit s+1 of T has keys past the end of the sequence.
      if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(rs <= __builtin_bit_cast(float, limit))) != 0ull, 0)) {
        // (a unit past the end of the list is none of this wavefront's)
        if ((X == 1 || s + 1 < U) && __builtin_amdgcn_ballot_w64(!(rs <= RANGE)) != 0ull) redo_tile(X, S[X], P[X]);
        if (s + 1 >= partial_begin) mask_tile(S[T], s + 1);
      }
    };
    if (KS > 1 && U == 0 && most > 0) meet(0);
    if (U > 0) {
      const uint32_t off0 = first_off(0);
      uint32_t off1 = first_off(1);                                      // part P + 1
      bf16x8 k0[NQ];
#pragma unroll
      for (int c = 0; c < NQ; ++c) k0[c] = k_load(off0, c);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
          kr[1 - u][j] = k_load(u == 0 ? off0 + K_TILE : off1, j);
          asm volatile("" ::: "memory");
          vr[u][j] = v_load(u == 0 ? off0 : off0 + V_TILE, j);
          asm volatile("" ::: "memory");
        }
      }
      spread_q();
      first_unit(S, k0);
      redo_tile(0, S[0], P[0]);                     // probabilities of tile 0 of the first unit (the reference stays where it is)
#pragma unroll
      for (int e = 0; e < 8; ++e) P[1][e] = 0u;
      int entry = ahead[2];
      const auto nothing = [](int) {};
      for (int s = 0; s < U;) {
        meet();
        const int end = meeting ? min(U, s + 2 * MEET) : U;
        do {
          const int p = s >> 1;
          uint32_t off2 = 0;
          // loads in step s (part P, tile 0): K of part P+1, tile 1, V of part P+1, tile 0; in step s+1: K of part P+2, tile 0, V of part P+1, tile 1
          half_step(std::false_type{}, std::false_type{}, s, 0, 0, [&](int g) {
            if (g == 3) {
              off2 = part_off(entry, part_of(p + 2));
              asm volatile("" : "+s"(off2));
            } else if (g == 4) {
              entry = list_entry(part_of(p + 3));
            }
          });
          half_step(std::true_type{}, std::false_type{}, s, off1 + K_TILE, off1, nothing);
          half_step(std::false_type{}, std::true_type{}, s + 1, 0, 0, nothing);
          half_step(std::true_type{}, std::true_type{}, s + 1, off2, off1 + V_TILE, nothing);
          off1 = off2;
          s += 2;
        } while (s < end);
      }
      if (KS > 1 && parts < most) meet(parts);
    }
  }

  if (U == 0) note_targets();

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
  auto finishes = [&](int q, int dt) { return KS == 1 || grp == (q * DT + dt) * KS / TILES; };
  if constexpr (KS > 1) {
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
    if (KS == 1 || grp * TILES / KS / DT == q) {                // (of more wavefronts than tiles some have none)
      if (KS <= TILES || grp * TILES % KS == 0) {
        uint4* const staged = out_rows[wave];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          if (finishes(q, dt))
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              bf16x4 pk;
#pragma unroll
              for (int e = 0; e < 4; ++e) pk[e] = (__bf16)(o[q][dt][4 * g + e] * f);
              reinterpret_cast<bf16x4*>(&staged[row_slot<OC>(l32, (4 * dt + g) % OC)])[lh] = pk;
            }
        wave_fence();
        // (all reads ahead of the stores, which may stand behind branches: rows past the last token are not written)
        __attribute__((address_space(1))) unsigned char* const to = (__attribute__((address_space(1))) unsigned char*)out_at + (OC < D / 8 ? 64 * (grp * TILES / KS % DT) : 0) + 16 * (lane % OC);
        uint4 piece[OC / 2];
        int row_to[OC / 2];
#pragma unroll
        for (int i = 0; i < OC / 2; ++i) {
          const int r = lane / OC + i * (64 / OC);
          piece[i] = staged[row_slot<OC>(r, lane % OC)];
          row_to[i] = targets[wave][32 * q + r];
        }
#pragma unroll
        for (int i = 0; i < OC / 2; ++i) asm volatile("" : "+v"(piece[i].x), "+v"(piece[i].y), "+v"(piece[i].z), "+v"(piece[i].w), "+v"(row_to[i]));
        auto store = [&](int i) {
          const u32x4 x = {piece[i].x, piece[i].y, piece[i].z, piece[i].w};
          *reinterpret_cast<__attribute__((address_space(1))) u32x4*>(to + (uint64_t)(uint32_t)row_to[i] * out_pitch) = x;
        };
        if (!fused || q_row - l32 + 64 <= n_tokens) {
#pragma unroll
          for (int i = 0; i < OC / 2; ++i) store(i);
        } else {
#pragma unroll
          for (int i = 0; i < OC / 2; ++i)
            if (row_to[i] >= 0) store(i);
        }
        wave_fence();
      }
    }
    if (lse != nullptr && lh == 0 && finishes(q, 0)) {
      const int t = targets[wave][32 * q + l32];
      if (t >= 0)
        lse[fused ? (size_t)bh * n_tokens + t : (size_t)bh * (Tq << split) * BQ + t] =
            m_ref[q] * scale_log2 * 0.6931471805599453f + __logf(l_tot[q]);
    }
  }
}

template <int D, int BK, int QH, int KS>
__global__ void __launch_bounds__(64 * QH * KS, D == 128 ? 1 : 2) stream_attn_kernel(RF2_STREAM_PARAMS) {
  const int at = (int)(blockIdx.x >> 3);
  attend<D, BK, QH, KS>(RF2_STREAM_ARGS(split), (int)(blockIdx.x & 7), at >> split, at & ((1 << split) - 1));
}

// QH = 2 for the row slots `lead` to `whole` of an XCD, KS = 2 in front of them (its sink rows, or none) and behind them (see
// rf2_cut_stream): workgroups of two wavefronts either way, `split` is that of the former.  1,536 tiles of an image layer (24 heads) fill 1,024 places one and a half
// times: as one cut two rounds or three half ones, so in one and a half, 102.6 -> 94.4 us (the layer 135.9 -> 128.3).  With 77 text
// tokens, whose rows are three times as long as the others, 98.4 -> 84.3 us (the layer 145.8 -> 132.1).
template <int D, int BK>
__global__ void __launch_bounds__(128, 1) mixed_attn_kernel(RF2_STREAM_PARAMS, int lead, int whole) {
  const int xcd = (int)(blockIdx.x & 7), at = (int)(blockIdx.x >> 3);
  const int inside = at - (lead << (split + 1)), behind = inside - ((whole - lead) << split);
  if (inside >= 0 && behind < 0) {
    attend<D, BK, 2, 1>(RF2_STREAM_ARGS(split), xcd, lead + (inside >> split), inside & ((1 << split) - 1));
  } else {
    const int half = inside < 0 ? at : behind;
    attend<D, BK, 1, 2>(RF2_STREAM_ARGS(split + 1), xcd, (inside < 0 ? 0 : whole) + (half >> (split + 1)), half & ((2 << split) - 1));
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

template <int D, int BK, int QH, int KS>
int launch_stream(const rf2_plan* plan, const AttnArgs& a, hipStream_t st) {
  const rf2_info& in = plan->info;
  const int share = plan->cfg.block / (64 * QH), split = share / 2;      // workgroups of a Q block: 1, 2, 4
  if (share < 1) return RF2_ERR_UNSUPPORTED;                             // (no cut has more rows than a Q block)
  unsigned slots;
  const RowOrder order = row_order(plan, &slots);
  if (slots == 0) return RF2_OK;
  const auto launch = [&](auto kernel, unsigned grid, auto... more) {
    kernel<<<dim3(grid), dim3(64 * QH * KS), 0, st>>>(
        order.shares, order.per_xcd, order.n_bh, order.rows, order.sink_begin, order.n_sink, order.sink_slots, split, in.k_row, a.blk_idx,
        a.blk_cnt, (const __bf16*)a.qp, (const __bf16*)a.kp, (const __bf16*)a.vp, plan->d_perm, (__bf16*)a.out, a.lse, in.n_blocks_k,
        in.last_block_valid_k, (float)(1.4426950408889634 / sqrt((double)D)), (int)in.N, plan->cfg.heads, a.scatter, plan->cut.meets,
        rf2_qkv_strides(plan), more...);
  };
  if constexpr (D == 128 && QH == 2 && KS == 1) {
    const unsigned lead = plan->cut.halved_sinks ? (unsigned)order.sink_slots : 0u;
    const unsigned whole = std::max(lead, std::min(slots, (unsigned)plan->cut.whole_slots));
    if (plan->cut.whole_slots > 0 && (lead > 0 || whole < slots)) {
      launch(mixed_attn_kernel<D, BK>, 8u * (((whole - lead) << split) + ((slots - whole + lead) << (split + 1))), (int)lead, (int)whole);
      RF2_LAUNCH_CHECK();
      return RF2_OK;
    }
  }
  launch(stream_attn_kernel<D, BK, QH, KS>, (8u * slots) << split);
  RF2_LAUNCH_CHECK();
  return RF2_OK;
}

template <int D, int BK>
int dispatch_cut(const rf2_plan* plan, const AttnArgs& a, hipStream_t st) {
  const rf2_attn_cut& cut = plan->cut;
#define RF2_ATTN_CASE(QH, KS) \
  if (cut.rows == 64 * QH && cut.groups == KS) return launch_stream<D, BK, QH, KS>(plan, a, st);
  RF2_ATTN_CASE(1, 1)
  RF2_ATTN_CASE(1, 2)
  RF2_ATTN_CASE(1, 4)
  RF2_ATTN_CASE(2, 2)
  if constexpr (D == 128) {
    RF2_ATTN_CASE(2, 1)
    RF2_ATTN_CASE(4, 1)
  } else {
    RF2_ATTN_CASE(1, 8)
  }
#undef RF2_ATTN_CASE
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
