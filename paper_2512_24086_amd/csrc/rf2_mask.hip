// Block-mask prediction: S_hat = qbar kbar^T (Sec. 3.2, eq. 7) in fp32 on the matrix cores,
// then per-row top-n selection (eq. 8) with the first-frame sink (Sec. 3.4), fused in one
// kernel.  A workgroup owns 16 rows (Q blocks) of one head: its wavefronts first fill a 16 x Tk
// strip of order-preserving integer keys of the scores in LDS (Tk = number of K blocks; the mask
// is Tq x Tk, square unless b_q != b_k), then each wavefront finds the threshold key of its rows
// by a guided search and emits the ascending block lists.
// The cumulative-mass variant (RF2_SELECT_CDF) runs the same search on probability mass
// instead of counts: the threshold is the largest key whose upper set carries >= tau of the
// row's softmax mass.
//
// What bounds it: on the 720p layer (591 x 591 scores, 40 heads) the fp32 MFMAs take 23 us of the
// matrix cores at full rate, the search and the emission about as much of the vector and of the
// scalar issue slots; a workgroup is a chain of load, multiply, search and store, so what counts is how
// many of them a compute unit holds.  The Q operand is read from LDS and the K operand is
// reloaded in place, four chunks of 16 channels ahead, which keeps a wavefront of up to 768 columns within 72 registers: six
// wavefronts per SIMD where LDS holds three workgroups of eight (up to 688 columns, 752 at d = 64; two up to 1,120 and 1,184, one
// beyond).  K is loaded four lanes to 64 bytes of a row and turned into the operand's order, 16 rows to a quarter of the lanes, through
// the place in LDS where the tile's keys go afterwards: loaded in that order, each lane's 16 bytes lie in a line of their own, and the address
// unit of a compute unit was busy with 64 cycles an instruction, 46 us of the 720p layer (without the search and the lists 54 us).  720p
// 69.0 -> 56.1 us, d = 64 46.5 -> 43.7, one head 17.2 -> 14.2, long video by count 103.6 -> 86.9, by mass 131.9 -> 117.2.  (Turned by
// DPP moves within quads, 67 and 134.5 us; with eight chunks ahead, 57.0 and 118.2.)  A probe of the
// search costs a compare and a population count per 64 keys; on bell-shaped rows, as smooth fields give, the
// normal-distribution guess and interpolation need 4 or 5 of them where a bitwise search that stops at the first exact
// count needs 15.5 (other rows: see MAX_GUIDED).  720p: 104 -> 70 us; cumulative mass on the long video (929 x 929, 24
// heads): 291 -> 146 us; with few workgroups 12-50 -> 8-15 us, all before K came so.  No load of K, no read of a key and no store of a list entry
// stands behind a branch: buffers drop what lies outside of kbar or of the list.  (Behind branches the compiler waited for the
// whole next K tile at the end of each, and every entry cost four scalar instructions: 720p 70.1 -> 69.4 us (68.7 to 69.8 in
// three runs), long video, cumulative mass, 145.0 -> 134.8.)  Wavefronts that share a K tile (32, 48 or 64 rows per
// workgroup) halve the L2 reads and are slower (98-122 us on 720p).
#include "rf2_internal.h"

#include <algorithm>
#include <cmath>

namespace {

typedef __attribute__((ext_vector_type(4), may_alias)) float f32x4;

// Order-preserving map float -> uint32 (larger float <=> larger key); -0 is folded into +0.
__device__ __forceinline__ uint32_t order_key(float x) {
  const uint32_t u = __float_as_uint(x + 0.f);
  return u ^ (uint32_t)(((int32_t)u >> 31) | (int32_t)0x80000000);
}

// The float whose order_key is k.
__device__ __forceinline__ float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// The same value in every lane, as a scalar.
__device__ __forceinline__ float uniform(float x) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(x)));
}

__device__ __forceinline__ int popc64(unsigned long long m) { return __builtin_popcountll(m); }
// Set bits of m below this lane.
__device__ __forceinline__ int rank_below(unsigned long long m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Reductions over the wavefront on the vector ALU (DPP row shifts and row broadcasts); the total forms in lane 63 and
// is handed to every lane as a scalar.  An LDS shuffle would cost a trip through LDS for each of the six steps.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xf, false);
}
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v, uint32_t neutral, Op op) {
  v = op(v, dpp<0x111, 0xf>(neutral, v));             // lane i with lane i-1, then i-2, i-4, i-8 of its row of 16
  v = op(v, dpp<0x112, 0xf>(neutral, v));
  v = op(v, dpp<0x114, 0xf>(neutral, v));
  v = op(v, dpp<0x118, 0xf>(neutral, v));
  v = op(v, dpp<0x142, 0xa>(neutral, v));             // lane 15 / 47 to the row behind it
  v = op(v, dpp<0x143, 0xc>(neutral, v));             // lane 31 to the upper half
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
// Sum over the wavefront, every lane with lane ^ 32, then ^ 16, 8, 4, 2, 1: this order of the additions is part of the result
// (a cumulative-mass row is cut where these fp32 sums say).  Halves and rows of 16 trade places through permlane swaps;
// after them all lanes of a row hold values of period 8, 4, 2, 1, so a rotation by as much reaches the same partner's value.
__device__ __forceinline__ float wave_sum(float x) {
  const auto add = [](uint32_t a, uint32_t b) { return __uint_as_float(a) + __uint_as_float(b); };
  uint32_t v = __float_as_uint(x);
  const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  v = __float_as_uint(add(h[0], h[1]));
  const auto q = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = __float_as_uint(add(q[0], q[1]));
  v = __float_as_uint(add(v, dpp<0x128, 0xf>(v, v)));
  v = __float_as_uint(add(v, dpp<0x124, 0xf>(v, v)));
  v = __float_as_uint(add(v, dpp<0x122, 0xf>(v, v)));
  return uniform(add(v, dpp<0x121, 0xf>(v, v)));
}
// Sum over a row of 16 lanes, in the last of them.
__device__ __forceinline__ float row_sum(float x) {
  x += __uint_as_float(dpp<0x111, 0xf>(0u, __float_as_uint(x)));
  x += __uint_as_float(dpp<0x112, 0xf>(0u, __float_as_uint(x)));
  x += __uint_as_float(dpp<0x114, 0xf>(0u, __float_as_uint(x)));
  return x + __uint_as_float(dpp<0x118, 0xf>(0u, __float_as_uint(x)));
}
__device__ __forceinline__ uint32_t wave_max_u(uint32_t x) {
  return wave_reduce(x, 0u, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
}
__device__ __forceinline__ uint32_t wave_min_u(uint32_t x) {
  return wave_reduce(x, ~0u, [](uint32_t a, uint32_t b) { return a < b ? a : b; });
}

// First guesses of a row's threshold search (see rf2_mask_prepare).
struct Guess {
  float z, slope;
};

// Keys of columns that take no part in a row's search: below every candidate's (columns past the row) and above
// (sink columns: counted by every probe and always taken).
constexpr uint32_t PAST_KEY = 0u, SINK_KEY = 0xffffffffu;

// A search keeps a bracket [lo, top] around the threshold.  Its first two probes come from the guesses, then the measure
// (count or mass) is interpolated between the ends, or the bracket halved where that has not halved its keys.  Where
// scores are not bell-shaped (outliers, several levels, many magnitudes) interpolation gains little: after MAX_GUIDED
// probes, for counts also after three in a row that leave more than half of the bracket's keys, the bracket's integer range
// is halved, at a third of the time for a count (a mass costs more than its guess), and every TIGHTEN probes it is drawn in to
// the keys it holds (equal scores end there).  Whatever the probes are, the threshold found is the same.
// (720p, 40 heads, us, bitwise search -> with up to 12 guided probes and none of this -> now: scores all equal 126 -> 192 -> 69,
// over many magnitudes 99 -> 128 -> 83, one column in ten far above 101 -> 130 -> 90, smooth fields 104 -> 72 -> 70; cumulative
// mass, four levels 171 -> 205 -> 109, smooth fields 170 -> 95 -> 95)
constexpr int TIGHTEN = 8;
__device__ __forceinline__ uint32_t halfway(uint32_t lo, uint32_t top) { return lo + ((top - lo) >> 1) + 1u; }
__device__ __forceinline__ uint32_t next_probe(float t, uint32_t lo, uint32_t top) {
  const uint32_t k = order_key(t);
  return k - lo - 1u < top - lo ? k : halfway(lo, top);    // lo < k <= top; any float, NaN too, is safe here
}
// The smallest and the largest key of the bracket (which holds one) become its ends.
template <int EMAX>
__device__ __forceinline__ void draw_in(const uint32_t (&key)[EMAX], uint32_t& lo, uint32_t& top) {
  uint32_t least = ~0u, most = 0u;
#pragma unroll
  for (int e = 0; e < EMAX; ++e) {
    const bool in = key[e] - lo <= top - lo;
    least = min(least, in ? key[e] : ~0u);
    most = max(most, in ? key[e] : 0u);
  }
  lo = wave_min_u(least);
  top = wave_max_u(most);
}

// LDS of a workgroup behind its strip of keys: the Q operand and each wavefront's share of the rows' sums.  Behind, because the
// last row's reads of keys pass the end of the strip: they end in here, and nothing is allocated for them.  (With words of their own
// the widest rows of a step lost a workgroup per compute unit; 12 heads, us, with them -> now: d = 128, 1,120 columns 116.6 -> 88.4, by
// mass 148.7 -> 110.9, 688 columns, by mass, 58.3 -> 55.1; d = 64, 752 columns 36.0 -> 34.6, by mass 50.9 -> 46.7.)
template <int D, int NW>
struct BehindKeys {
  float qs[16][D + 4];                              // (+4: the 16 rows of an operand read start in different banks)
  float stat[NW][16][2];                            // sum and sum of squares over a wavefront's columns
};

// NW wavefronts per workgroup of R = 16 rows.  Second launch bound, wavefronts per SIMD: up to 768 columns LDS holds three workgroups
// of eight (six), beyond two.  At d = 64 it holds four where rows have up to 512 columns; for that many a wavefront may have 64 vector
// registers and, as the trap handler has 16 of its own, 80 scalar ones (eight).  Left alone the kernel takes 67 and up to 93: three
// workgroups.  (By count, us, three -> four: 200 columns x 1,014 strips 19.5 -> 18.1, 304 x 1,007 23.6 -> 21.8, 512 x 1,024 30.9 -> 28.2;
// where three are enough 304 x 760 18.2 -> 18.3, 300 x 266 13.4 -> 13.5.  By mass four cost up to 1 % where three are
// enough, 304 x 760 29.5 -> 29.8: left at three.)
template <int D, int EMAX, bool CDF, int NW>
__global__ void __launch_bounds__(NW * 64, NW == 8 ? (D == 64 && EMAX <= 8 && !CDF ? 8 : EMAX <= 12 ? 6 : 4) : 4) predict_mask_kernel(
    const float* __restrict__ qbar, const float* __restrict__ kbar, int32_t* __restrict__ blk_idx,
    int32_t* __restrict__ blk_cnt, uint8_t* __restrict__ mask_dense, float* __restrict__ scores,
    int Tq, int Tb, int LD, int row_sink_begin, int row_sink_end, int sink_begin, int sink_end, int k_row,
    float tau, float scale_log2, Guess guess, int n_strips, int n_work) {
  // Tb, sink_begin, sink_end describe the COLUMNS (K blocks) from here on; rows use Tq and row_sink_*.
  constexpr int R = 16;
  constexpr int MAX_GUIDED = CDF ? 10 : 8;
  constexpr int FULL = EMAX <= 12 ? EMAX - 2 : EMAX == 32 ? 24 : EMAX - 4;    // a row has more than 64 FULL columns (choose_instance)
  extern __shared__ __attribute__((aligned(16))) uint32_t keys[];   // [R][LD]
  auto& [qs, stat] = *reinterpret_cast<BehindKeys<D, NW>*>(keys + R * LD);
  // Workgroups with equal blockIdx % 8 share an XCD and take a contiguous run of the strips, numbered head by head:
  // the strips that read one head's kbar meet in one L2.
  const int work = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  if (work >= n_work) return;
  const int bh = work / n_strips;
  const int i0 = (work % n_strips) * R;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const float* __restrict__ qb = qbar + (size_t)bh * Tq * D;
  // kbar of the head as a buffer: columns past the row read as zero and cost nothing, so no load stands behind a branch.
  const auto kbuf = __builtin_amdgcn_make_buffer_rsrc((void*)(kbar + (size_t)bh * Tb * D), 0, (unsigned)Tb * D * 4, 0x00020000);
  // Lane l has 16 bytes of row l / 4 of the tile.
  auto k_load = [&](int ct, int kk) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(kbuf, ((ct * 16 + lane / 4) * D + 4 * (lane & 3)) * 4 + 64 * kk, 0, 0));
  };

  // ---- scores: 16 x 16 tiles with v_mfma_f32_16x16x4_f32 -------------------------------
  // Lane (lr, lk) feeds row lr of each operand.  Per 16 channels it has 4 consecutive
  // floats from 16*kk + 4*lk on; MFMA step e uses element e, so "k slot lk" stands for channel
  // 16*kk + 4*lk + e in both operands (a dot product does not care about summation order).
  const int n_ct = (Tb + 15) / 16;
  constexpr int NC = D / 16, NB = 4;              // chunks of 16 channels; those on their way
  f32x4 b[NB];
#pragma unroll
  for (int kk = 0; kk < NB; ++kk) b[kk] = k_load(wave, kk);
  for (int c = threadIdx.x; c < R * (D / 4); c += NW * 64) {
    const int row = c / (D / 4), ch = c % (D / 4) * 4;
    *reinterpret_cast<f32x4*>(&qs[row][ch]) = *reinterpret_cast<const f32x4*>(qb + (size_t)min(i0 + row, Tq - 1) * D + ch);
  }
  __syncthreads();
  float sum[4] = {}, sum2[4] = {};
  for (int ct = wave; ct < n_ct; ct += NW) {
    // the registers of a chunk are reloaded with the one NB chunks on, at last of the wavefront's next column tile, as soon as
    // its products are issued (its copy in LDS is read by other lanes than wrote it, and before the next chunk's is written: the fences)
    uint32_t* const tile = &keys[ct * 16];
    f32x4* const put = reinterpret_cast<f32x4*>(tile + lane / 4 * LD + 4 * (lane & 3));
    const f32x4* const get = reinterpret_cast<const f32x4*>(tile + lr * LD + 4 * lk);
    f32x4 acc = {}, a = *reinterpret_cast<const f32x4*>(&qs[lr][4 * lk]);
    *put = b[0];
    wave_fence();
    f32x4 k = *get;
    wave_fence();
#pragma unroll
    for (int kk = 0; kk < NC; ++kk) {
      const f32x4 a_now = a, k_now = k;
      if (kk + 1 < NC) {
        *put = b[(kk + 1) % NB];
        wave_fence();
        k = *get;
        wave_fence();
        a = *reinterpret_cast<const f32x4*>(&qs[lr][16 * (kk + 1) + 4 * lk]);
      }
      __builtin_amdgcn_sched_barrier(0);      // (left alone, the read comes behind three of the products, into their registers)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a_now[e], k_now[e], acc, 0, 0, 0);
      b[kk % NB] = kk + NB < NC ? k_load(ct, kk + NB) : k_load(ct + NW, kk + NB - NC);
      __builtin_amdgcn_sched_barrier(0);      // (left alone, the loads of all chunks are gathered in twice the registers)
    }
    // acc[i] = S_hat[i0 + 4*lk + i][ct*16 + lr]
    const int j = ct * 16 + lr;
    if (scores != nullptr) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (j < Tb && i0 + 4 * lk + i < Tq) scores[((size_t)bh * Tq + i0 + 4 * lk + i) * Tb + j] = acc[i];
    }
    uint32_t* const kout = &keys[4 * lk * LD + j];
#pragma unroll
    for (int i = 0; i < 4; ++i) kout[i * LD] = min(max(order_key(acc[i]), PAST_KEY + 1u), SINK_KEY - 1u);
    if (ct * 16 + 16 > Tb || (ct * 16 + 16 > sink_begin && ct * 16 < sink_end)) {   // columns that are no candidates
      const bool past = j >= Tb, sink = j >= sink_begin && j < sink_end;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (past || sink) kout[i * LD] = past ? PAST_KEY : SINK_KEY;
        acc[i] = (past || sink) ? 0.f : acc[i];
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sum[i] += acc[i];
      sum2[i] = fmaf(acc[i], acc[i], sum2[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    // the 16 lanes of a row: total in the last of them
    const float s = row_sum(sum[i]), s2 = row_sum(sum2[i]);
    if (lr == 15) { stat[wave][4 * lk + i][0] = s; stat[wave][4 * lk + i][1] = s2; }
  }
  __syncthreads();

  // ---- selection: wavefront `wave` handles rows wave, wave + NW, ... ------------
  const int n_cand = Tb - (sink_end - sink_begin);
  for (int r = wave; r < R; r += NW) {
    const int i = i0 + r;
    if (i >= Tq) break;
    int32_t* __restrict__ out = blk_idx + ((size_t)bh * Tq + i) * k_row;
    uint8_t* __restrict__ mrow = mask_dense ? mask_dense + ((size_t)bh * Tq + i) * Tb : nullptr;
    if (i >= row_sink_begin && i < row_sink_end) {  // sink row: keeps every column
      if (lane == 0) blk_cnt[(size_t)bh * Tq + i] = Tb;
      for (int j = lane; j < k_row; j += 64) out[j] = j;
      if (mrow) for (int j = lane; j < Tb; j += 64) mrow[j] = 1;
      continue;
    }
    uint32_t key[EMAX];
#pragma unroll
    for (int e = 0; e < EMAX; ++e) {
      // (read in any case: without a branch; what lies behind the row is in the strip or in BehindKeys)
      key[e] = keys[r * LD + 64 * e + lane];
      if (e >= FULL) key[e] = 64 * e + lane < Tb ? key[e] : PAST_KEY;
    }
    // (16 lanes over the NW wavefronts' shares; with eight of them every share counts twice)
    const float in_all = (NW == 8 ? 0.5f : 1.0f) / (float)max(n_cand, 1);
    const float sum_r = row_sum(stat[lane % NW][r][0]), sum2_r = row_sum(stat[lane % NW][r][1]);
    const float mean = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(sum_r * in_all), 15));
    const float square = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(sum2_r * in_all), 15));
    const float sigma = uniform(__builtin_amdgcn_sqrtf(fmaxf(square - mean * mean, 0.f)));
    // The threshold T: every key above it is taken, of the keys equal to it the need_eq lowest columns.
    uint32_t T, lo = PAST_KEY + 1u, top = SINK_KEY - 1u;      // bracket: the answer is in [lo, top]
    int need_eq = 0;
    int n_lo = Tb, n_top = Tb - n_cand;             // keys >= lo, keys > top
    if constexpr (!CDF) {
      // Largest T with |{key >= T}| >= k_row (sink columns count); a probe with exactly k_row keys at or above it ends
      // the search early: any T between the k_row-th and the next key gives the same set.  (The scalar
      // unit is as busy as the vector unit, 450 instructions a row, most of them what decides and not what counts: with the first
      // probe on its own, the ends of the loop as one minimum and no flag, and the rows' sums added across lanes, 720p 56.2 ->
      // 55.5 us, d = 64 43.7 -> 42.2, five heads 14.7 -> 14.2, long video 86.8 -> 84.9.)
      if (n_top == k_row) lo = SINK_KEY, n_lo = k_row;        // only the sink columns
      const auto probe = [&](uint32_t cand) {
        int cnt = 0;
#pragma unroll
        for (int e = 0; e < EMAX; ++e) cnt += popc64(__builtin_amdgcn_ballot_w64(key[e] >= cand));
        if (cnt >= k_row) { lo = cand; n_lo = cnt; } else { top = cand - 1u; n_top = cnt; }
        return cnt;
      };
      if (n_lo != k_row && lo < top) {
        float t = mean + guess.z * sigma;
        t += (float)(probe(next_probe(t, lo, top)) - k_row) * sigma * guess.slope;
        int stalled = 0;                            // probes in a row that left more than half of the bracket's keys
        for (int p = 1; min(n_lo - k_row, min(MAX_GUIDED - p, 3 - stalled)) > 0 && lo < top; ++p) {
          const int before = n_lo - n_top;
          probe(next_probe(t, lo, top));
          stalled = 2 * (n_lo - n_top) > before ? stalled + 1 : 0;
          const float fl = key_value(lo), fh = key_value(top);
          if (lo == PAST_KEY + 1u) t = fh - sigma * (0.25f * (float)(1 << p));      // no lower (upper) end yet
          else if (top == SINK_KEY - 1u) t = fl + sigma * (0.25f * (float)(1 << p));
          else t = fl + (fh - fl) * ((stalled & 1) ? 0.5f : (float)(n_lo - k_row) * __builtin_amdgcn_rcpf((float)(n_lo - n_top)));
        }
      }
      for (int p = 0; n_lo != k_row && lo < top; ++p) {
        if (p % TIGHTEN == 0) draw_in(key, lo, top);
        if (lo < top) probe(halfway(lo, top));
      }
      const bool exact = n_lo == k_row;
      T = exact ? lo - 1u : lo;
      need_eq = exact ? 0 : k_row - n_top;          // lo == top: the keys equal to lo share the places left
    } else {
      // Softmax mass of every candidate (relative to the row maximum, unnormalised), then the
      // largest T whose upper set {key >= T} carries at least tau of the total: the columns above
      // T are the shortest prefix of the descending order that reaches tau, up to ties at T.  One key left in the
      // bracket ends the search.
      uint32_t kmax = PAST_KEY + 1u;
#pragma unroll
      for (int e = 0; e < EMAX; ++e) kmax = max(kmax, key[e] == SINK_KEY ? PAST_KEY : key[e]);
      top = wave_max_u(kmax);
      const float mx = key_value(top);
      float ev[EMAX], part = 0.f;
#pragma unroll
      for (int e = 0; e < EMAX; ++e) {
        const float x = __builtin_amdgcn_exp2f((key_value(key[e]) - mx) * scale_log2);
        ev[e] = (key[e] != PAST_KEY && key[e] != SINK_KEY) ? x : 0.f;
        part += ev[e];
      }
      const float total = wave_sum(part), target = tau * total;
      float m_lo = total, m_top = 0.f;
      bool halve = false;
      // (a weight exp(a s) moves the mean of a normal distribution by a sigma^2)
      float t = mean + sigma * (sigma * scale_log2 * 0.6931472f + guess.z);
      const auto probe = [&](uint32_t cand) {
        float mass = 0.f;
        int cnt = 0;
#pragma unroll
        for (int e = 0; e < EMAX; ++e) {
          const bool in = key[e] >= cand;
          mass += in ? ev[e] : 0.f;
          cnt += popc64(__builtin_amdgcn_ballot_w64(in));
        }
        mass = wave_sum(mass);
        const bool up = mass >= target;               // (selects: branches here left the captured variables in scratch memory)
        lo = up ? cand : lo, n_lo = up ? cnt : n_lo, m_lo = up ? mass : m_lo;
        top = up ? top : cand - 1u, n_top = up ? n_top : cnt, m_top = up ? m_top : mass;
        return mass;
      };
      for (int p = 0; n_lo - n_top > 1 && lo < top && p < MAX_GUIDED; ++p) {
        const int before = n_lo - n_top;
        const float mass = probe(next_probe(t, lo, top));
        halve = !halve && p > 1 && 2 * (n_lo - n_top) > before;
        const float fl = key_value(lo), fh = key_value(top);
        if (p == 0) t += (mass / total - tau) * sigma * guess.slope;
        else if (lo == PAST_KEY + 1u) t = fh - sigma * (0.25f * (float)(1 << min(p, 12)));
        else t = fl + (fh - fl) * (halve ? 0.5f : (m_lo - target) * __builtin_amdgcn_rcpf(m_lo - m_top));
      }
      for (int p = 0; n_lo - n_top > 1 && lo < top; ++p) {
        if (p % TIGHTEN == TIGHTEN / 2) draw_in(key, lo, top);    // (first after four: mostly two or three are left to do)
        if (lo < top) probe(halfway(lo, top));
      }
      T = lo - 1u;                                    // (where the sums are no numbers lo is the least key at most: all are kept)
      if (n_lo - n_top > 1) {                         // lo == top: several keys equal to it, of equal mass
        T = lo;
        const float tie = __builtin_amdgcn_exp2f((key_value(lo) - mx) * scale_log2);
        const float left = ceilf((target - m_top) / tie);
        need_eq = left <= (float)n_lo ? max(1, (int)left) : n_lo;      // (not a number: the whole row is kept)
      } else if (n_cand == 0) {
        T = SINK_KEY - 1u;                            // only sink columns
      }
    }
    if (need_eq > 0) {                                // of the keys equal to T, the lowest columns rise above it
      int run = 0;
#pragma unroll
      for (int e = 0; e < EMAX; ++e) {
        const bool eq = key[e] == T;
        const unsigned long long eq_m = __builtin_amdgcn_ballot_w64(eq);
        if (eq && run + rank_below(eq_m) < need_eq) key[e] = T + 1u;
        run += popc64(eq_m);
      }
    }
    // (lanes without an entry store past the end of the row's list, which a buffer drops: no branch around each store)
    const auto list = __builtin_amdgcn_make_buffer_rsrc((void*)out, 0, k_row * 4, 0x00020000);
    int out_run = 0;
#pragma unroll
    for (int e = 0; e < EMAX; ++e) {
      const bool sel = key[e] > T;
      const unsigned long long sel_m = __builtin_amdgcn_ballot_w64(sel);
      __builtin_amdgcn_raw_buffer_store_b32((uint32_t)(64 * e + lane), list, sel ? (out_run + rank_below(sel_m)) * 4 : 1 << 30, 0, 0);
      out_run += popc64(sel_m);
    }
    if (mrow) {
#pragma unroll
      for (int e = 0; e < EMAX; ++e)
        if (64 * e + lane < Tb) mrow[64 * e + lane] = key[e] > T ? 1 : 0;
    }
    if (lane == 0) blk_cnt[(size_t)bh * Tq + i] = out_run;   // top-n: == k_row by construction
  }
}

// Shape of the launch for a plan, and the kernel instance that serves it.
struct MaskLaunch {
  const void* kernel = nullptr;
  int E, LD, NW;
  size_t lds = 0;
};

// The kernel is instantiated for a few row widths (EMAX keys per lane): the search loops run over
// EMAX keys without bounds checks (keys past the row are 0), so a snug width saves compares.
template <int D, int NW>
void choose_instance(MaskLaunch& m, bool cdf) {
  const auto words = [&](int width) {               // strip and what is behind it; where the last row's reads end
    return std::max(16 * m.LD + (int)(sizeof(BehindKeys<D, NW>) / 4), 15 * m.LD + 64 * width);
  };
#define RF2_MASK_CASE(W)                                                                                                        \
  if (m.E <= W) {                                                                                                               \
    m.kernel = cdf ? (const void*)predict_mask_kernel<D, W, true, NW> : (const void*)predict_mask_kernel<D, W, false, NW>;       \
    m.lds = (size_t)words(W) * 4;                                                                                               \
    return;                                                                                                                     \
  }
  RF2_MASK_CASE(2)
  RF2_MASK_CASE(4)
  RF2_MASK_CASE(6)
  RF2_MASK_CASE(8)
  RF2_MASK_CASE(10)
  RF2_MASK_CASE(12)
  RF2_MASK_CASE(16)
  RF2_MASK_CASE(20)
  RF2_MASK_CASE(24)
  RF2_MASK_CASE(32)
#undef RF2_MASK_CASE
}                                                   // (Tk <= 2048: E <= 32)

MaskLaunch mask_launch(const rf2_plan* plan) {
  MaskLaunch m;
  m.E = (plan->info.n_blocks_k + 63) / 64;
  m.LD = (plan->info.n_blocks_k + 15) / 16 * 16 + 4;   // +4: the 4 row groups of a tile store hit distinct banks
  // Up to one workgroup per compute unit a row's search is latency: 16 wavefronts search one row each.  Beyond, a
  // compute unit holds three workgroups of 8 wavefronts but only one of 16 (up to 688 columns: LDS).  (16 against 8 wavefronts: 9.5 / 10.3 us
  // at 28 workgroups, 12.4 / 13.0 at 35, 20.3 / 21.2 at 136; 21.2 / 19.7 us at 320, 92 / 72 us at 1,480.)
  const int64_t strips = (int64_t)((plan->info.n_blocks + 15) / 16) * plan->cfg.batch * plan->cfg.heads;
  m.NW = strips <= 256 ? 16 : 8;
  const bool cdf = (plan->cfg.select_mode == RF2_SELECT_CDF);
  if (plan->cfg.head_dim == 128) m.NW == 8 ? choose_instance<128, 8>(m, cdf) : choose_instance<128, 16>(m, cdf);
  else m.NW == 8 ? choose_instance<64, 8>(m, cdf) : choose_instance<64, 16>(m, cdf);
  return m;
}

// z with P(X > z) = p for a standard normal X, by halving on the complementary error function.
double normal_quantile(double p) {
  double lo = -9.0, hi = 9.0;
  for (int it = 0; it < 60; ++it) {
    const double mid = 0.5 * (lo + hi);
    (0.5 * std::erfc(mid * 0.7071067811865476) > p ? lo : hi) = mid;
  }
  return 0.5 * (lo + hi);
}

}  // namespace

// Called once by rf2_plan_create.  A score strip wider than the default dynamic-LDS limit needs the limit of
// its kernel raised; doing it here keeps rf2_predict_mask free of anything but the launch (so it can be
// recorded into a HIP graph).  The first probe of a row's threshold search is where a normal distribution with the
// mean and variance of the row's scores would have it, the second a Newton step from there: z and 1 / density.
int rf2_mask_prepare(rf2_plan* plan) {
  const MaskLaunch m = mask_launch(plan);
  if (m.lds > 32 * 1024)
    RF2_HIP(hipFuncSetAttribute(m.kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)m.lds));
  const rf2_info& in = plan->info;
  const int n_cand = in.n_blocks_k - (in.sink_block_end_k - in.sink_block_begin_k);
  const bool cdf = (plan->cfg.select_mode == RF2_SELECT_CDF);
  const double n = cdf ? 1.0 : (double)std::max(n_cand, 1);
  const double p = cdf ? (double)plan->cfg.cdf_threshold : in.k_sel / n;
  const double z = (p > 0.0 && p < 1.0) ? normal_quantile(p) : 0.0;
  plan->mask_z = (float)z;
  plan->mask_slope = (float)(2.5066282746310002 * std::exp(0.5 * z * z) / n);
  return RF2_OK;
}

extern "C" int rf2_predict_mask(const rf2_plan* plan, const float* qbar, const float* kbar, int32_t* blk_idx,
                                int32_t* blk_cnt, uint8_t* mask_dense, float* scores, void* workspace,
                                void* stream) {
  (void)workspace;
  if (!plan || !qbar || !kbar || !blk_idx || !blk_cnt) return RF2_ERR_INVALID_ARG;
  if (const int rc = rf2_check_device(plan)) return rc;
  const rf2_config& c = plan->cfg;
  const rf2_info& in = plan->info;
  const MaskLaunch m = mask_launch(plan);
  int Tq = in.n_blocks, Tk = in.n_blocks_k, LD = m.LD;   // rows and columns of the block mask
  int rb = in.sink_block_begin, re = in.sink_block_end, cb = in.sink_block_begin_k, ce = in.sink_block_end_k;
  int k_row = in.k_row;
  float tau = c.cdf_threshold, scale_log2 = (float)(1.4426950408889634 / sqrt((double)c.head_dim));
  Guess guess{plan->mask_z, plan->mask_slope};
  int n_strips = (Tq + 16 - 1) / 16, n_work = n_strips * c.batch * c.heads;    // at most 128 x 65,535
  void* args[] = {&qbar, &kbar, &blk_idx, &blk_cnt, &mask_dense, &scores, &Tq, &Tk, &LD, &rb, &re, &cb, &ce,
                  &k_row, &tau, &scale_log2, &guess, &n_strips, &n_work};
  const dim3 grid((unsigned)((n_work + 7) / 8 * 8), 1, 1);
  RF2_HIP(hipLaunchKernel(m.kernel, grid, dim3(m.NW * 64), args, m.lds, (hipStream_t)stream));
  return RF2_OK;
}
