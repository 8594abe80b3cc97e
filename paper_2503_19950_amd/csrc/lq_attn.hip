// Decode attention: launch planning and dispatch.
#include <math.h>
#include <stdlib.h>

#include "lq_device.h"
#include "lq_internal.h"

namespace lq {

hipError_t launch_decode_attn_mfma(const Shape& s, const lq_cache& c, const void* q, float scale,
                                   void* out, const Workspace& ws, const lq_plan& plan, hipStream_t st,
                                   const void* k_new, const void* v_new, const SeqArg* seq);

static int env_int(const char* name, int dflt) {
  const char* v = getenv(name);
  return v && *v ? atoi(v) : dflt;
}

int compute_units() {
  static const int cus = env_int("LOGQUANT_ATTN_CUS", 256);
  return cus;
}

// Launch shape: wavefronts per workgroup (12, 8 or 4) and context splits per (b, kv head,
// head group).  Work is counted
// in units of one 64-slot quantized tile; a 32-row fp unit weighs its bytes relative
// to that.  A compute unit holds eight wavefronts of this kernel, i.e. one
// workgroup of 8 or two of 4; the candidate shapes are ranked by
//     rounds * (units per wavefront + fixed) + merge cost per split,
// rounds = how many times the chip has to be refilled, fixed = start-up and merge
// tail of a workgroup expressed in tiles.
static double fp_unit_weight(const Shape& s) {
  const double q_tile_bytes = 64.0 * (s.d * s.bits / 4 + 4 * s.ngc + 4.0 * s.d / s.G);
  const double fp_unit_bytes = 32.0 * 4 * s.d;
  return fp_unit_bytes / q_tile_bytes;
}

// The fp rows' share of the wavefronts, as the plan reports it: the number that, given
// every unit of 32 rows, would be done when the others are done with the tiles (whole
// units counted).  The kernel keeps to it where the context is split and the tiles are
// not drawn, and where there are no tiles; it also enters the rule for drawing them
// (lq_schedule.h).  Else wavefronts take both.
int fp_wave_share(const Shape& s, int NW, int n_fp, int n_q) {
  const int TQ = tiles_of(s, n_q), TF = (n_fp + 31) / 32;
  if (TF == 0) return 0;
  if (TQ == 0) return NW;
  const double r = fp_unit_weight(s);
  int best = 1;
  double best_t = 1e300;
  const int hi = TF < NW - 1 ? TF : NW - 1;
  for (int n = 1; n <= hi; ++n) {
    const double t_fp = (double)((TF + n - 1) / n) * r, t_q = (double)TQ / (NW - n);
    const double t = t_fp > t_q ? t_fp : t_q;
    if (t < best_t - 1e-9) { best_t = t; best = n; }
  }
  return best;
}

void plan_decode(const Shape& s, int n_fp, int n_q, lq_plan* plan, Rows rows) {
  const int TQ = tiles_of(s, n_q), TF = (n_fp + 31) / 32;
  const double r = fp_unit_weight(s);
  const double units = TQ + r * TF;
  const int64_t bytes_read = cache_bytes_read(s, n_fp, n_q);
  const int hb = heads_per_group(s, bytes_read);
  const int groups = s.B * s.Hkv * (s.gh / hb);
  const int cus = compute_units();
  static const int force_wpb = env_int("LOGQUANT_ATTN_WPB", 0);
  static const int force_splits = env_int("LOGQUANT_ATTN_SPLITS", 0);
  const double fixed = 2.5, per_split = 0.02, merge_tail = 1.5;
  int best_wpb = 8, best_splits = 1;
  double best = 1e300;
  bool keep_8 = false;
  for (int wpb = 8; wpb >= 4; wpb -= 4) {   // (12 is derived from 8 below)
    if (force_wpb && force_wpb != 12 && wpb != force_wpb) continue;
    // Rows of different lengths: 4 wavefronts win as they do for lock-step rows (two workgroups to a compute unit cover
    // each other's start and end: 41 rows of up to 1238 tokens, 8 kv heads 44.4 -> 34.9 us a launch, 64 rows of up to
    // 4096 44.5 -> 42; with padding, W = 85, G = 64, 52 of 2963, 4 bits, four layers 182 -> 175, W = 42, 19 of 3807 94 -> 79),
    // but not without tiles (9 rows of up to 540 tokens 9.6 -> 10.0).  Lock-step rows with padding slots, and equal rows
    // through the per-sequence calls, keep to 8 and 12 (with padding 4 are no better on average: of 100 shapes 0.85 to 1.28
    // times as long, 1.02 on average, with one split and with several).
    if (wpb == 4 && !force_wpb && (rows == LOCK_STEP ? s.Wq != s.W : rows == SAME_LENGTH || TQ == 0)) continue;
    const int slots = cus * (8 / wpb);
    int smax = (int)ceil(units / wpb);            // at least one unit per wavefront
    if (smax > max_splits(s)) smax = max_splits(s);
    if (smax < 1) smax = 1;
    const bool unsplit_8 = best < 1e300 && best_splits == 1;   // (wpb == 4: what the candidates of 8 came to)
    for (int sp = 1; sp <= smax; ++sp) {
      if (force_splits && sp != force_splits && force_splits <= smax) continue;
      // Two sets of query heads, rows of one length: not five or more splits among workgroups of 4.  Of 32 shapes that the
      // estimate would split so, 8 wavefronts take 0.81 to 1.04 of the time, 0.93 on average (15 rows x 2 kv heads x 13125
      // tokens, d = 96, 4 bits, 8 heads each, 19.6 -> 16.2 us).  Three splits of 4 are no worse on average (0.94 to 1.23 with
      // 8: 39 x 8 x 5099 tokens 55 -> 68 us), and unsplit 4 are better (8 shapes 1.13 to 1.32).
      if (hb > 4 && wpb == 4 && sp > 3 && rows == LOCK_STEP && !force_wpb) break;
      const int rounds = (sp * groups + slots - 1) / slots;
      // Rows of different lengths, more workgroups than fit at once: the last round is one of short rows and never full,
      // so that 8 wavefronts are done sooner than their count of rounds says.  Where they would not split, 4 do not
      // either (33 to 40 rows of up to 2000 or 3000 tokens, 8 kv heads, 45 tiles a row, 8 launches: 8 wavefronts unsplit
      // 238-264 us, 4 in three splits 255-283, 4 unsplit 223-259); where 8 would split as well, three splits of 4 are
      // the better ones (36 rows of 6000 352 against 370 us unsplit, 34 of 12000 536 against 594).
      const bool instead_of_unsplit_8 = wpb == 4 && rows == DIFFERENT_LENGTHS && sp > 1 && unsplit_8;
      if (instead_of_unsplit_8 && rounds > 1) break;
      // more than one split adds the cross-workgroup merge: a chain of memory round trips
      // (store, ticket, fetch) worth about a tile and a half (measured on the smallest
      // workload: 8.4 us with three splits, 6.8 us with one)
      const double t = rounds * (units / ((double)sp * wpb) + fixed) + per_split * sp + (sp > 1 ? merge_tail : 0.0);
      // At least four tiles to each of their wavefronts: with fewer there is little to split, and every row pays for the
      // merge.  Of 160 shapes of 3 to 86 tiles, four layers, those with fewer than 48 take 8 unsplit 0.75 to 1.08 of the time
      // of 4 in three splits, 0.95 on average (8 kv heads, d = 128: 20 rows of 1106 tokens, 12 tiles, 49 against 66 us, 21 of
      // 878 50 against 60, 18 of 2261, 27 tiles, 4 bits 71 against 73), the others 0.96 to 1.15 (21 of 4196, 60 tiles, 90
      // against 85).  8, and not the 12 below, which take up to 1.2 times as long there (20 of 1106 57, 18 of 2484, 34 tiles,
      // 72 against 62).
      if (instead_of_unsplit_8 && TQ < 4 * sp * wpb) {
        keep_8 = keep_8 || t < best - 1e-9;
        continue;
      }
      if (t < best - 1e-9) { best = t; best_wpb = wpb; best_splits = sp; }
    }
  }
  // Few items (units of fp rows, tiles): one split of 8.  The estimate above divides the work evenly, but an item is not
  // shared, and what a split saves is less than the merge costs: nothing but fp rows, 2 to 128 kv heads, take 0.72 to 0.96
  // of the time up to 20 units (three to a wavefront), 0.80 to 0.90 up to 24 for d = 64 or where the groups alone fill a
  // quarter of the chip; elsewhere 24 units take 1.03.  8, not the 12 below, which would have a second set of empty
  // wavefronts (20 units, d = 128: 1.07 of the time of the splits with 12, 0.95 with 8).  With tiles up to two items to a
  // wavefront: 0.73 to 0.98 of the time, but with more than one unit to a wavefront and few groups the long ones, d = 96 and
  // 128, only up to 14 items (0.96 to 0.99; 15 take 1.00 to 1.05), and d = 128 with one channel group not at all (1.03 to
  // 1.10).  Not caches of three or four channel groups with tiles: their probabilities are rounded, all but a wavefront's
  // heaviest, and with fewer wavefronts outputs are further off (520 tokens, d = 128, G = 32, fp16 2.319e-4 of the 2-norm
  // in three splits, 2.329e-4 in one, though 5.9 instead of 7.5 us; bf16 1.6614e-3 and 1.6688e-3, d = 96 1.6583e-3 and
  // 1.6748e-3).
  const bool easy = s.d == 64 || 4 * groups >= cus;
  const int most_items = TQ == 0 ? (easy ? 24 : 20) : s.ngc > 2 ? 0 : easy || TF <= 8 ? 16 : s.d == 128 && s.ngc == 1 ? 8 : 14;
  if (rows != DIFFERENT_LENGTHS && best_splits > 1 && !force_wpb && !force_splits && TF + TQ <= most_items) {
    best_wpb = 8;
    best_splits = 1;
    keep_8 = true;
  }
  // Twelve wavefronts per workgroup (three per SIMD) for long contexts on few groups: not with fewer than six tiles to a
  // wavefront, and only when the launch fits the chip in one round (64 rows with per-row counts 54 us, with 8 49).  They
  // cover latency with a third wavefront, but where the loads bound the launch that no longer pays: of 70 shapes inside the
  // rule, 8 take 0.82 to 1.06 of their time with several splits (0.98 on average, 37 shapes; 98209 tokens x 8 kv
  // heads, four layers, 19.6 us a launch with 12, 17.8 with 8), with padding 0.92 to 1.09 (1.00, 30 shapes), in one split 0.96 to 0.98 (3 shapes).
  // Only built for 2-bit codes (with 4-bit codes it made no difference: 37.3 against 37.2 us), and not for more than four
  // query heads, whose registers would not fit.
  if (s.bits == 2 && hb <= 4 && (force_wpb == 12 || (!force_wpb && best_wpb == 8 && !keep_8 && units / (best_splits * 8.0) >= 6.0 &&
                                          (int64_t)best_splits * groups <= cus)))
    best_wpb = 12;
  const int splits = best_splits, WPB = best_wpb;
  const int NW = WPB * splits;
  const int nwf = fp_wave_share(s, NW, n_fp, n_q);
  plan->splits = splits;
  plan->waves_per_block = WPB;
  plan->blocks = splits * groups;
  plan->fp_waves = nwf;
  plan->bytes_read = bytes_read;
}

hipError_t launch_decode_attn(const Shape& s, const lq_cache& c, const void* q, float scale,
                              void* out, const Workspace& ws, const lq_plan& plan, hipStream_t st, const SeqArg* seq) {
  return launch_decode_attn_mfma(s, c, q, scale, out, ws, plan, st, nullptr, nullptr, seq);
}

// `c` already counts the new row (n_fp includes it); the row itself is still only in
// k_new / v_new.
hipError_t launch_decode_step(const Shape& s, const lq_cache& c, const void* k_new, const void* v_new,
                              const void* q, float scale, void* out, const Workspace& ws, const lq_plan& plan,
                              hipStream_t st, const SeqArg* seq) {
  return launch_decode_attn_mfma(s, c, q, scale, out, ws, plan, st, k_new, v_new, seq);
}

}  // namespace lq
