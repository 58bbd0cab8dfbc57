// How a launch of the attention kernel is cut (host only; also compiled into a test).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <functional>
#include <queue>
#include <vector>

#include "rf2.h"

// rf2_cut_attn: the rule of thresholds for the former kernel, with rings in LDS and wavefronts of 32 rows.  No launch takes it any
// more (rf2_cut_stream, below, does that); a host test still holds it to its measurements.
// How a launch is cut, from the sizes of the plan alone (so that both exits of a layer give the same bits).
// A row of the mask is one workgroup of `groups` (KS) groups of wavefronts that share its list (KS = 1: no merge); a Q block
// of 256 rows is one workgroup of eight wavefronts or two of 128 rows.
// jobs = the launch's work in units of its longest list.  With few jobs and KS = 1 compute units stand idle, or wait for
// the all-column sink rows of a few heads; groups shorten the longest list, and cost a merge, a common barrier and
// half of the workgroups a compute unit holds.  Where the rows are many and short beside the longest (a long tail: video
// with a sink frame) the jobs decide, else how the workgroups themselves fill the compute units: with two groups at d = 128
// and four at d = 64 a compute unit holds one workgroup, with two at d = 64 two, and what a shader engine gets beyond that
// waits for a whole list (rf2_busiest_engine; of 330 launches with equal rows every one with 8, or 16, workgroups at most on
// the busiest engine gained, with more all lost or gained 2 % at most).  KS = 1 -> 2 (us), d = 128, 64-row blocks, rows of 25 parts, 25 rows x
// 9 heads (9 on an engine) 30.8 -> 41.8, of 31 parts, 31 x 7 (7) 34.7 -> 26.7; 128-row blocks, 51 x 5 (9) 108 -> 133; d = 64,
// 64-row blocks, 25 x 20 (17) 29.0 -> 30.6, 31 x 16 (16) 35.7 -> 26.5; KS = 1 -> 4, 128-row blocks, 51 x 5 (9) 77.8 -> 83.7.
// Measured, KS = 1 -> 2 (us), 480p layer (rows of 40, sink rows of 256 blocks), d = 128: 1 head (51 jobs) 469 -> 332,
// 4 heads (204) 580 -> 448, 6 heads (306) 687 -> 616, 8 heads (408) 797 -> 832, 20 heads 1,919 -> 2,060; 64-row blocks,
// 2 heads (206) 461 -> 309, 4 heads (412) 518 -> 555.  Equal rows (3,072-token image, 24 rows of 10 blocks), d = 128:
// 192 workgroups 25.0 -> 24.5, 288 35.2 -> 46.0.  Images with text (2 long rows of 20): 320 workgroups 49.6 -> 40.7,
// 400 51.7 -> 58.0, 64-row blocks 312 43.0 -> 32.9, 468 45.4 -> 46.4.
// d = 64 holds twice the workgroups: 480p, 306 jobs 483 -> 374, 408 jobs 543 -> 480, 510 jobs 613 -> 602, 714 jobs 792 ->
// 817; equal rows, 64-row blocks, 384 workgroups 24.0 -> 18.7, 576 25.4 -> 27.6, 128-row blocks 192 18.2 -> 15.8, 288 23.7 ->
// 24.2; with text, 64-row blocks, 300 jobs 33.2 -> 31.1, 360 34.9 -> 35.6.
// A workgroup that shares a compute unit with fewer others is the dearer the shorter its own list is: the workgroups may be 13
// times as many as the longest list has parts (d = 128; at d = 64 12 to 32 times by the work, 7 for KS = 4).  KS = 1 -> 2 (us),
// d = 128, images with text, 64-row blocks, 750 workgroups, 75 parts (10 times) 1.53 times as fast, 792, 66 parts (12) 1.16, 816,
// 51 parts (16) 55.3 -> 58.8, 760, 38 parts (20) 44.4 -> 50.3; 128-row blocks, 936, 77 (12) 89.2 -> 78.7, 896, 56 (16) 64.4 ->
// 66.7; d = 64, 64-row blocks, 186 jobs (32) 1.16 times, 317 (24) 1.27, 324 (24) 1.20, 408 (20) 1.14, 442 (24) 1.03, 366 (32) 44.4 -> 45.9, 430 (40) 94.6 ->
// 113; without a tail, 295 (16) 1.15, 314 (24) 25.3 -> 29.2; 128-row blocks, 311 (20) 1.07, 369 (20) 1.05, 403 (2.5) 1.13, 436 (20)
// 113 -> 117; KS = 2 -> 4, 744 workgroups, 124 parts (6) 1.17 times, 1,056, 132 (8) 0.82, 1,480, 74 (20) 40.6 -> 65.2 (KS = 1: 54.5).
// KS = 4 against 2 (us): 480p, 51 jobs 250 -> 204, 204 jobs 313 -> 288; 64-row blocks 180 -> 133; with text, 64-row blocks,
// 264 workgroups 28.8 -> 26.0, 312 20.9 -> 24.5; but rows of 20 parts, 128-row blocks 14.5 -> 17.2.
// A list has to be long enough to pay for the merge (equal rows of 64-key parts, KS = 1 -> 2, us): d = 128, 64 workgroups,
// 8 parts 14.0 -> 14.6, 16 parts 21.0 -> 19.7; 192 workgroups, 16 parts 23.6 -> 24.0, 32 parts 38.0 -> 35.2; 256 workgroups,
// 32 parts 41.5 -> 42.0, 64 parts 70.4 -> 65.9; 64-row blocks, 2 parts 8.9 -> 9.2, 4 parts 10.4 -> 10.1; d = 64, 8 parts 10.3 ->
// 10.2, 16 parts 15.7 -> 14.3; 64-row blocks, 4 parts 8.8 -> 8.9, 8 parts 10.0 -> 8.8 (KS = 4: 9.1); 2 -> 4, 128-row
// blocks, 32 parts 21.9 -> 21.8, 64 parts 36.0 -> 33.2; 64-row blocks, 16 parts 10.8 -> 10.9.
// 256-row blocks, one workgroup -> two (us): d = 128, 512 workgroups 683 -> 586 (KS = 2: 452), 760: 576 -> 516, 480 of equal
// length 101 -> 92, 1,024: 813 -> 827, 5,120: 3,830 -> 3,914 (the larger one reads K and V less often); d = 64,
// 1,024: 597 -> 534, 1,280: 641 -> 607, 2,560: 1,115 -> 1,128.  Rows of equal length gain only where the halves fill the compute
// units better (a compute unit holds one whole block at d = 128, two at d = 64, twice as many halves): 65 rows of 130 parts, d =
// 128, 166 -> 125, 130 rows 170 -> 176, 260 381 -> 347, 390 401 -> 412, 455 424 -> 436, 520 607 -> 577, 650 617 -> 645; d = 64, 65
// 118 -> 92, 195 123 -> 129, 260 217 -> 183, 390 233 -> 251, 455 247 -> 263, 520 361 -> 329.  Lists under 20 parts always gain, 3 % or
// more; at d = 64 the halves of long sequences read past an XCD's L2 (16,640 tokens 404 -> 338, 31,160 tokens 237 -> 252).
struct rf2_attn_cut {
  int rows;         // query rows of a workgroup: those of a Q block, or a half or a quarter of them
  int groups;       // groups of wavefronts that share a list
  bool whole_heads; // ordinary rows are numbered head by head and dealt to the XCDs in 8 runs (else every head in 8 shares)
  int whole_slots = 0;  // > 0: row slots of an XCD that are cut so; those behind them get 64-row workgroups of two shares,
  bool halved_sinks = false;      // and so do its sink rows (not then counted as cut so)
};

// Workgroups of a launch that its busiest shader engine gets, `share` workgroups to a row of the mask.  The hardware deals
// workgroup g to XCD g % 8 and there to shader engine (g / 8) % 4, each of 8 compute units, as it comes; the grid's slots
// without work (the kernel's numbering: sink rows of all heads in 8 runs, then every head's ordinary rows in 8 shares that
// rotate with the head) take their turn too, so an engine can get more than its part of the rows.
inline int rf2_busiest_engine(int64_t lists, int rows, int sink_rows, int share) {
  const int plain = rows - sink_rows;
  const int64_t sinks = lists * sink_rows, sink_slots = (sinks + 7) / 8;
  int most = 0, of_share[8] = {}, slots = 0;
  for (int r = 0; r < plain; ++r) ++of_share[(int64_t)r * 8 / plain];
  for (int n : of_share) slots = std::max(slots, n);
  for (int xcd = 0; xcd < 8; ++xcd) {
    int load[4] = {};
    for (int64_t s = 0; s < sink_slots + lists * slots; ++s) {
      const int64_t t = s - sink_slots;
      const bool work = t < 0 ? xcd * sink_slots + s < sinks : t % slots < of_share[(xcd + t / slots) & 7];
      for (int i = 0; work && i < share; ++i) ++load[(s * share + i) & 3];
    }
    for (int n : load) most = std::max(most, n);
  }
  return most;
}

inline rf2_attn_cut rf2_cut_attn(const rf2_config& c, const rf2_info& in) {
  const int64_t lists = (int64_t)c.batch * c.heads, rows = lists * in.n_blocks, share = c.block == 256 ? 2 : 1;
  const int sink_rows = in.sink_block_end - in.sink_block_begin;
  const bool known = in.kept_pairs_per_head >= 0;
  const int64_t wgs = rows * share;
  // (cumulative mass: the lengths of ordinary rows are not known.  Taken as equal; without a sink row, whose length is
  // known, a row is taken to keep what a flat one does, tau (1 + tau) / 2 of the columns: smooth fields kept 0.04 of them
  // at tau = 0.1, 0.25 at 0.3, 0.6 at 0.7, 0.85 at 0.9.  Taken as full, rows of 2 parts got two groups, 9.7 -> 11.8 us
  // at d = 128 with 29 columns, tau = 0.1, and four, 6.4 -> 6.8 us at d = 64 with 25)
  int64_t longest = sink_rows > 0 ? in.n_blocks_k : in.k_row;
  int64_t parts = longest * (in.block_k / 64);
  if (!known && sink_rows == 0) parts = (int64_t)((float)parts * 0.5f * c.cdf_threshold * (1.0f + c.cdf_threshold));
  const int64_t jobs = known ? share * lists * in.kept_pairs_per_head / longest : wgs;
  const bool uneven = wgs >= 2 * jobs, tail = wgs >= 3 * jobs;
  const int busiest = rows <= 2048 ? rf2_busiest_engine(lists, in.n_blocks, sink_rows, (int)share) : 1 << 20;
  int groups = 1;
  if (c.head_dim == 64) {
    const bool fits = c.block == 64 ? busiest <= 16 && parts >= 4
                                    : wgs <= 256 && parts >= (busiest <= 8 || sink_rows > 0 ? 12 : 32);
    const int times = !tail ? 20 : c.block == 64 ? (jobs <= 320 ? 32 : 24) : (jobs <= 400 ? 24 : 12);
    const bool pays = jobs <= (tail ? 512 : 320) && wgs <= times * parts;
    if (uneven ? pays && parts >= (c.block == 64 ? 4 : 12) : fits) groups = 2;
    if ((tail ? jobs <= 256 : wgs <= 280) && parts >= (c.block == 64 ? 24 : 64) &&
        (busiest <= 8 || (sink_rows > 0 && wgs <= 7 * parts)))
      groups = 4;
  } else if ((!uneven ? busiest <= 8 : wgs <= 13 * parts && (tail ? jobs <= (parts >= 256 ? 320 : 256) : wgs <= 320)) &&
             parts >= (c.block == 64 ? 6 : std::max<int64_t>(12, jobs / 6))) {
    groups = 2;
  }
  if (c.block != 256 || groups > 1) return {c.block == 256 ? 128 : c.block, groups};
  const int64_t limit = c.head_dim == 64 ? 2048 : 1024;
  if (rows >= limit) return {256, 1};
  // (cumulative mass with sink rows: spread where a flat ordinary row keeps less than half of the columns)
  const bool spread = known ? uneven : sink_rows > 0 && c.cdf_threshold * (1.0f + c.cdf_threshold) < 1.0f;
  const int whole = rf2_busiest_engine(lists, in.n_blocks, sink_rows, 1);
  const bool full = c.head_dim == 64 ? (whole > 4 && whole < 8) || (whole > 11 && whole <= 16) || (whole > 8 && in.N > 19456)
                                     : (busiest + 7) / 8 >= 2 * ((whole + 7) / 8);
  return {full && parts >= 20 && !spread ? 256 : 128, 1};
}

// ---- the cut of stream_attn_kernel -----------------------------------------------------------------------------------
// A workgroup has QH x KS wavefronts, QH = rows / 64, KS = groups.  Which QH and KS: the pair with the shortest launch in a
// small model of it, made of what a launch is: jobs of two lengths (all-column sink rows first, then the others), dealt in order to
// places that take the next job when they are done.
//   * The busiest shader engine is looked at: 1/8 of the rows go to an XCD, 1/4 of its workgroups to each engine of 8 compute
//     units, which hold 32 wavefronts at d = 128 and 64 at d = 64.
//   * A job lasts 2 (parts / KS) units of a wavefront, plus the start of a row, plus the merge, all counted in units.
//   * A unit takes `idle` us where up to `knee` of the wavefront places are taken and `full` where all are (shared vector issue at d = 64,
//     clock under the power limit, shared L2), along a line with a bow between.  By and large QH = 2 meets tiles in L1, KS = 2 and
//     4 have fewer rows in flight on an XCD: factors of `full`.
// The constants are fitted to launches of 600 to 40,000 tokens, 1 to 40 heads, blocks of 64, 128 and 256 rows, sparsity 0.5 to 0.9,
// with and without sink rows and text (d = 128: 140 launches, d = 64: 125), and to 30 of 480p to long-video layers, each timed with
// several cuts.  d = 128: the model is 4 % off on average, its choice 0.1 % slower than the best cut (6 % at most); d = 64: 7 % off,
// 0.6 % slower (14 % at most, on launches under 100 us).  Against a rule of thresholds for a kernel with rings in LDS, d = 128,
// 1.28 times as fast in the geometric mean.
// E.g. d = 128 (us, QH x KS = 1x1, 1x2, 1x4, 2x1, 2x2): image of 4,096 tokens, 1 head 38, 24, 19, 39, 26; 8 heads 41, 36, 42, 41, 36;
// 16 heads 66, 70, 84, 67, 72; 24 heads 104, 102, 124, 107, 105; 480p 5 heads 672, 492, 532, 665, 493, 40 heads 3,926, 3,974,
// 4,251, 3,506, 3,800; 256-row blocks, 480p, 40 heads, 2x1 3,425, 4x1 3,394, 720p 18,067 and 17,653.  d = 64 (1x1, 1x2, 1x4, 1x8, 2x2): image,
// 2 heads 34, -, -, 15, 21; 24 heads 63, 71, 66, 83, 57; 480p, 2 heads 495, -, -, 140, 263; 40 heads 2,133, 2,206, 2,258, 2,570, 2,107.
struct rf2_stream_model {
  double idle, full, knee, bow;                  // us per unit
  double start, start2, start4;                  // units: start of a row, more of it for QH = 2 and 4
  double merge2, merge4, merge8;                 // units: merge of KS shares
  double rate2, rate4, of2, of4, of8, square;    // factors of `full`: QH = 2, 4; KS = 2, 4, 8; QH = KS = 2 (on top)
  double launch;                                 // us
  int waves;                                     // places of a shader engine
};
inline const rf2_stream_model& rf2_model_of(int head_dim) {
  static const rf2_stream_model d128{0.507, 0.843, 0.372, -0.532, 4.04, 1.95, 6.58, 2.06, 5.02, 0.0, 0.957, 0.918, 0.984, 0.937, 1.0, 1.01, 5.1, 32};
  static const rf2_stream_model d64{0.448, 0.931, 0.21, 0.084, 2.02, 0.85, 0.0, 2.42, 2.85, 6.57, 1.042, 1.0, 1.066, 1.003, 0.97, 0.865, 4.4, 64};
  return head_dim == 128 ? d128 : d64;
}
struct rf2_stream_jobs {
  int64_t sinks, plain;          // jobs of a shader engine
  double sink_parts, plain_parts;
  int64_t halved = 0;            // of 128 rows: as many of the last ones run as two jobs of 64 rows and two shares each,
  bool halved_sinks = false;     // and so do the sink rows
};
inline double rf2_stream_time(const rf2_stream_model& m, rf2_stream_jobs j, int qh, int ks) {
  const int places = m.waves / (qh * ks);
  const double full = m.full * (qh == 4 ? m.rate4 : qh == 2 ? m.rate2 : 1.0) * (ks == 8 ? m.of8 : ks == 4 ? m.of4 : ks == 2 ? m.of2 : 1.0) *
                      (qh == 2 && ks == 2 ? m.square : 1.0);
  const double more = m.start + (qh == 4 ? m.start4 : qh == 2 ? m.start2 : 0.0) + (ks == 8 ? m.merge8 : ks == 4 ? m.merge4 : ks == 2 ? m.merge2 : 0.0);
  const double sink = 2.0 * std::ceil(j.sink_parts / ks) + more, plain = 2.0 * std::ceil(j.plain_parts / ks) + more;
  double us = m.launch;
  // (many rounds of equal jobs: all but the last sixteen at the full rate)
  const auto rounds = [&](int64_t& jobs, double units) {
    const int64_t skip = std::max<int64_t>(jobs / places - 16, 0);
    jobs -= skip * places;
    us += (double)skip * units * full;
  };
  rounds(j.sinks, sink);
  rounds(j.plain, plain);
  std::priority_queue<double, std::vector<double>, std::greater<double>> busy;     // ends of the jobs under way
  std::vector<double> starts, ends;
  const auto deal = [&](double units) {
    double at = 0.0;
    if ((int)busy.size() == places) { at = busy.top(); busy.pop(); }
    starts.push_back(at);
    ends.push_back(at + units);
    busy.push(ends.back());
  };
  const double per = m.of2 / m.rate2, merge = m.start + m.merge2;        // (a unit of KS = 2 in units of QH = 2)
  for (int64_t i = 0; i < j.sinks + j.plain; ++i) {
    const bool first = i < j.sinks;
    if (i < j.sinks + j.plain - j.halved && !(first && j.halved_sinks)) {
      deal(first ? sink : plain);
    } else {
      const double half = (2.0 * std::ceil((first ? j.sink_parts : j.plain_parts) / 2) + merge) * per;
      deal(half);
      deal(half);
    }
  }
  std::sort(ends.begin(), ends.end());
  double last = 0.0;             // (starts ascend)
  for (size_t s = 0, e = 0; e < ends.size();) {
    const bool begins = s < starts.size() && starts[s] < ends[e];
    const double at = begins ? starts[s] : ends[e];
    const double taken = (double)((s - e) * qh * ks) / m.waves, x = std::max(0.0, (taken - m.knee) / (1.0 - m.knee));
    us += (at - last) * (m.idle + (full - m.idle) * (x + m.bow * x * (1.0 - x)));
    last = at;
    begins ? ++s : ++e;
  }
  return us;
}

// Ordinary rows: with whole heads on an XCD its L2 fetches 1/8 of the K and V that it does where every XCD has rows of every
// head, but the Infinity Cache (256 MB) has to hold those of 8 heads at a time.  (every head in 8 shares -> whole heads: 4,096
// tokens x 24 heads, 112 -> 106 us; 480p, 17 MB a head, 3.56 -> 3.52 ms; 48,384 tokens, 25 MB, 4.62 -> 4.61; 60,480 tokens, 31 MB,
// 7.16 -> 7.16; 720p, 39 MB, 18.5 -> 18.8; long video, 61 MB, 13.7 -> 14.1; d = 64: 480p, 8 MB, 2.126 -> 2.107 ms, 720p, 19 MB, 10.98 ->
// 10.87, long video, 30 MB, 8.24 -> 8.31.)  Launches of 64-row blocks have the more different lists in flight and gain at 720p too
// (20 heads 11.6 -> 10.8 ms, d = 64, 40 heads 11.46 -> 11.22; long video, 6 heads, 3.77 -> 3.81).
inline rf2_attn_cut rf2_cut_stream(const rf2_config& c, const rf2_info& in) {
  const rf2_stream_model& m = rf2_model_of(c.head_dim);
  const int64_t lists = (int64_t)c.batch * c.heads, sink_rows = in.sink_block_end - in.sink_block_begin;
  const int64_t sinks = (lists * sink_rows + 7) / 8, plain = (lists * (in.n_blocks - sink_rows) + 7) / 8;      // of an XCD
  const double parts = in.block_k / 64;
  double keeps = in.k_row;
  // (cumulative mass: a row is taken to keep what a flat one does)
  if (in.kept_pairs_per_head < 0) keeps = std::max(1.0, (double)in.k_row * 0.5 * c.cdf_threshold * (1.0 + c.cdf_threshold));
  // (the pairs that were the best of all cuts for some size: at d = 64 2 x 1, 4 x 1 and 2 x 4 never by more than 1 %)
  static const int pairs128[][2] = {{1, 1}, {1, 2}, {1, 4}, {2, 1}, {2, 2}, {4, 1}}, pairs64[][2] = {{1, 1}, {1, 2}, {1, 4}, {1, 8}, {2, 2}};
  const auto* pairs = c.head_dim == 128 ? pairs128 : pairs64;
  rf2_attn_cut best{64, 1, false};
  double least = 0.0;
  for (int i = 0; i < (c.head_dim == 128 ? 6 : 5); ++i) {
    const int qh = pairs[i][0], ks = pairs[i][1];
    if (64 * qh > c.block) continue;
    const int64_t share = c.block / (64 * qh), of_sinks = (sinks * share + 3) / 4, all = ((sinks + plain) * share + 3) / 4;
    const double us = rf2_stream_time(m, {of_sinks, all - of_sinks, in.n_blocks_k * parts, keeps * parts}, qh, ks);
    if (least == 0.0 || us < least) least = us, best = {64 * qh, ks, false, 0};
    // Whole rows only as far as they fill rounds, those of the last, partly filled round as tiles of 64 rows with two shares each: a
    // round of half the length.  Taken where the model sees 3 % in it (its error); launches of many rounds have no such gain.
    // (us, the better of the other cuts -> this: 4,096 tokens, s = 0.5, 17 heads 92.8 -> 81.9, 24 heads 102.6 -> 94.4, 36 heads 155.3 ->
    // 143.2; 6,200 tokens, s = 0.7, 13 heads 87.8 -> 75.1, 25 heads 147.2 -> 133.6; 2,450 tokens, 256-row blocks, 30 heads 68.3 -> 56.9;
    // 3,000 tokens, s = 0.8, 64-row K/V blocks, 22 heads 38.3 -> 35.2.  The model: 81.4, 93.2, 139.3, 74.1, 130.4, 55.8, 32.8.)
    // All-column sink rows among short ones run as halves, too, where their length is what the launch waits for.  (us, before ->
    // halves: image of 4,087 tokens and 77 of text, s = 0.6, 24 heads 98.4 -> 84.3, 28 heads 104.3 -> 101.1; 2,450 and 200, s = 0.7, 33
    // heads 54.5 -> 44.6, 256-row blocks, 39 heads 67.8 -> 57.4; 9 frames of 900 tokens, the first a sink, s = 0.8, 24 heads 192.7 -> 175.8, 16
    // heads 126.5 -> 119.3; where the model sees less than 3 % nothing changes: of 22 launches none got slower.)
    if (c.head_dim == 128 && qh == 2 && ks == 1 && all <= 16 * 16) {
      for (const bool halved_sinks : {false, true}) {
        if (halved_sinks && of_sinks == 0) break;
        for (int64_t whole = std::max<int64_t>(16, all / 16 * 16 - 16);; whole += 4) {
          whole = std::min(whole, all);
          if (whole == all && !halved_sinks) break;
          const double mixed = rf2_stream_time(
              m, {of_sinks, all - of_sinks, in.n_blocks_k * parts, keeps * parts, all - whole, halved_sinks}, 2, 1);
          if (mixed < 0.97 * least)
            least = mixed, best = {128, 1, false, whole == all ? INT32_MAX : (int)(whole * 4 / share), halved_sinks};
          if (whole == all) break;
        }
      }
    }
  }
  best.whole_heads = c.block == 64 || in.N_pad_k * c.head_dim * 4 <= (int64_t)24 << 20;
  return best;
}
