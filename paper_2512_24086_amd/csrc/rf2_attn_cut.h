// How a launch of the attention kernel is cut (host only; also compiled into tests).
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <functional>
#include <queue>
#include <vector>

#include "rf2.h"

// How a launch is cut, from the sizes of the plan alone (so that both exits of a layer give the same bits).
struct rf2_attn_cut {
  int rows;         // query rows of a workgroup: those of a Q block, or a half or a quarter of them
  int groups;       // shares of a row's list, a wavefront each for every 64 of these rows
  bool whole_heads; // ordinary rows are numbered head by head and dealt to the XCDs in 8 runs (else every head in 8 shares)
  int whole_slots = 0;  // > 0: row slots of an XCD that are cut so; those behind them get 64-row workgroups of two shares,
  bool halved_sinks = false;      // and so do its sink rows (not then counted as cut so)
  bool meets = false;             // the wavefronts of four shares meet at every part
};

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
//   * At d = 64 a SIMD holds two wavefronts.  Workgroups of one wavefront spread over the SIMDs; beyond half of the places some share
//     one, run at nearly the full rate's pace, `shared` of it, and the launch waits for them: 1,100 of them take a fifth longer than a
//     line has it.  (Launches whose last round is half to three quarters full, us, the cut without this -> with it: 8 heads of 8,424
//     tokens, 256-row blocks, s = 0.6, 88.7 -> 70.8, 10 x 6,972, s = 0.7, 58.9 -> 49.2, 12 x 6,090, s = 0.6, 69.6 -> 61.7, 3 x 29,412, 92.7 ->
//     83.7, 19 x 10,626, 237.4 -> 216.5; the former kernel, with rings, took 75.1, 52.0, 62.5, 83.7, 223.9.  Of 720 random launches 39 are
//     cut differently, 31 of them faster, by 2 to 20 %, 4 slower, by 3 to 4 %.)
// The constants are fitted to launches of 600 to 40,000 tokens, 1 to 40 heads, blocks of 64, 128 and 256 rows, sparsity 0.5 to 0.9,
// with and without sink rows and text (d = 128: 140 launches, d = 64: 125), and to 30 of 480p to long-video layers, each timed with
// several cuts.  On launches it is not fitted to: d = 128 (130 of them), 5 % off on average, its choice, mixed cuts among them, 0.3 %
// faster than the best single cut, up to 7 % slower, on one (64-row blocks, 46,920 tokens x 46 heads) 22 %; d = 64 (720, of which
// `shared` is taken), 7 % off, the choice 1.3 % slower than the best cut, up to 18 %, under 20 us 24 %.  Against the former kernel,
// with rings in LDS and a rule of thresholds, they are 1.27 and 1.16 times as fast in the geometric mean; none at d = 128 is slower, six
// at d = 64 by more than 5 % (8 % at most).  (All of this was measured when a row's start and end took half as long again and a unit 2 to 3 %
// longer than they do now that Q and O move as whole rows and the checks of a unit stand between its MFMAs; not refitted since.)
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
  double shared;                                 // of `full`: rate where the first SIMDs are shared (0: they never are)
};
inline const rf2_stream_model& rf2_model_of(int head_dim) {
  static const rf2_stream_model d128{0.507, 0.843, 0.372, -0.532, 4.04, 1.95, 6.58, 2.06, 5.02, 0.0, 0.957, 0.918, 0.984, 0.937, 1.0, 1.01, 5.1, 32, 0.0};
  static const rf2_stream_model d64{0.448, 0.931, 0.21, 0.084, 2.02, 0.85, 0.0, 2.42, 2.85, 6.57, 1.042, 1.0, 1.066, 1.003, 0.97, 0.865, 4.4, 64, 0.9};
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
    double unit = m.idle + (full - m.idle) * (x + m.bow * x * (1.0 - x));
    if (m.shared > 0.0 && qh * ks == 1 && taken > 0.5) unit = std::max(unit, full * (m.shared + (1.0 - m.shared) * (2.0 * taken - 1.0)));
    us += (at - last) * unit;
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
  // Four wavefronts that share a list drift apart on long ones, and the workgroups of an XCD then have a wider stretch of K and V in
  // use than its L2 holds.  Meeting at every part keeps them together (requests that miss L2, 118,800 tokens x 3 heads: 660 -> 236 of 1,329
  // million, 73,750 x 5: 226 -> 93 of 599).  Taken where the drift costs more than the meetings: 64-row blocks
  // (no two workgroups with one list), lists of one length, of 256 parts and more, and fewer heads than XCDs, whose K and V are of 28 MB a
  // head, near the 32 MB of all L2s, 44 MB with six and seven heads, and of 40 MB together.
  // (us, without -> with, tokens x heads, sparsity: 118,800 x 3, 0.5, 12,480 -> 9,343; 119,280 x 3, 0.55, 12,699 -> 8,415; 100,800 x 2, 0.5,
  // 128-row K/V blocks, 5,236 -> 4,310; 118,800 x 2, the same, 9,219 -> 8,766; 73,750 x 5, 0.65, 4,898 -> 4,150; 93,492 x 6, 0.5, 15,712 ->
  // 12,170; 62,092 x 3, 0.59, 2,420 -> 2,188; 91,584 x 1, 0.64, 1,915 -> 1,764.  Beyond these lines: 128-row Q blocks,
  // 118,800 x 1, 0.5, 2,894 -> 2,957; by mass, 57,792 x 3, 3,776 -> 3,894; lists of 138 parts, 63,000 x 3, 735 -> 748; 118,800 x 8, 0.8,
  // 11,236 -> 11,465; 44,928 x 1, 0.43, 485 -> 497; 64,428 x 1, 0.62, 709 -> 726; 85,690 x 7, 0.68, 7,362 -> 7,530.)
  best.meets = c.head_dim == 128 && best.rows == 64 && best.groups == 4 && c.block == 64 && lists < 8 && in.k_row < in.n_blocks_k &&
               in.k_row * parts >= 256 && in.N_pad_k * 512 >= (int64_t)(lists <= 5 ? 28 : 44) << 20 && in.N_pad_k * 512 * lists >= (int64_t)40 << 20;
  best.whole_heads = c.block == 64 || in.N_pad_k * c.head_dim * 4 <= (int64_t)24 << 20;
  return best;
}
