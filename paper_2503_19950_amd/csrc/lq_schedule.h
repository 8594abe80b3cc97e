// How the attention kernel's work is dealt to wavefronts: fp rows in units of 32, quantized rows in tiles of 64.
// Integer arithmetic only, used by the kernel, by the choice of its program on the host, and by the host test.
#pragma once
#include <stdint.h>
#ifdef __HIP__
#define LQ_HD __host__ __device__ __forceinline__
#else
#define LQ_HD inline
#endif

namespace lq {

// Division by a number that the host knows, exact for x >= 0 and (x + 1) * n <= 2^32: the reciprocal is rounded down, and
// x + 1 taken instead of x makes up for it.  (B * Hq is at most 65535, and with it every x and n here.)  The attention
// kernel's start is one chain of scalar operations up to its first load: of 180 instructions half were divisions by kernel
// arguments, and the grid's size for them was a second argument load (now 60 to 90 and, without counts per row, one wait:
// 512 tokens 7.92 -> 7.77 us a launch; 8 rows of 8192, four layers, 69.0 -> 67.0; 64 rows of up to 4096, 16 steps,
// 671 -> 664; 8 rows of 2048 37.6 -> 36.7).
struct Divisor {
  int n;
  uint32_t inv;   // floor((2^32 - 1) / n)
  void set(int d) {
    n = d;
    inv = 0xFFFFFFFFu / (uint32_t)d;
  }
  LQ_HD int quotient(int x) const { return (int)(((uint64_t)((uint32_t)x + 1u) * inv) >> 32); }
};

// Pools of tiles that wavefronts draw from, per head group.  Several, because atomics on one address are serialised at
// a rate that a single counter could not sustain.
constexpr int NSUB = 8;

// The tiles that hold tokens.  A filtering event takes Wq slots, its W tokens first; with key groups of 64 or 128 slots
// that is a whole number of tiles, of which those behind the last token are padding: they are not dealt, and nothing of
// them is read (17 rows of 17970 tokens, 8 kv heads, W = 39, groups of 128, d = 96: half of the tiles, 117 -> 68 us a
// launch), nor of the second half of a tile where that is padding (2 rows of 28243 tokens, 32 kv heads, W = 212, groups
// of 64, 4 bits: 46.4 -> 43.7).  Tiles are numbered through the live ones; place() finds a tile in the buffers.
struct LiveTiles {
  int per_event, pad;   // ceil(W / 64) tiles of an event that hold tokens, and the Wq / 64 - per_event that do not
  uint32_t inv;         // ceil(2^31 / per_event)
  void set(int W, int Wq) {
    per_event = (W + 63) / 64;
    pad = Wq / 64 - per_event;
    inv = (uint32_t)(((uint64_t)1 << 31) / per_event + (((uint64_t)1 << 31) % per_event != 0));
  }
  struct Place { int tile, slot0; };   // index of the tile among all, padding included; its first slot within its event
  LQ_HD Place place(int t) const {
    int e = (int)(((uint64_t)(2u * (uint32_t)t) * inv) >> 32);   // t / per_event, or one more (t < 2^30)
    int j = t - e * per_event;
    if (j < 0) { --e; j += per_event; }
    return Place{t + e * pad, 64 * j};
  }
};

// Four programs, chosen per launch.  The wavefronts of all workgroups of a head group are numbered 0..NW-1: place by place
// (the first wavefronts of all splits, then the second ones, ..), so that those that get the most - units, or one tile
// more than others - are the older ones of every compute unit, each with a lighter one on its SIMD.  (Numbered split by
// split the first workgroups had all of it: 8 rows of 8192 tokens, 4 splits, wavefronts done between 11.5 and 17.6 us;
// four layers 69.0 -> 66.5 us, 4 rows of 8192 48.5 -> 44.3, 1 of 20000 41.5 -> 39.4.)
//  APART      a share of the wavefronts, NWF, keeps to the units, the others walk the tiles and have their first loads
//             on the way before anything else.  For several splits with few tiles per wavefront, and for launches
//             without tiles.  (With units and tiles in the same wavefronts and the deal worked out from the counts,
//             every wavefront waited twice for kernel arguments before its first load, and those without tiles ran the
//             whole prologue and epilogue of tiles: 8 rows of 8192 tokens, four layers, 75.9 instead of 73.4 us.)
//  ONE_SPLIT  a single split: every wavefront takes its units and then tiles, with one set of sums for both.  (With a
//             share kept for the units those wavefronts were done long before the others - after 40 of 240 us at 32768
//             tokens x 16 rows x 32 kv heads - and idled.)  When the units do not come out even, the wavefronts with
//             one unit less are a round of tiles ahead of the others (a unit takes about as long as a tile: a lead of
//             0 or 2 rounds measured 1 to 2% slower).
//  DRAWN      several splits, many tiles: the units fall on different compute units, the tiles are drawn from the pools,
//             and the wavefronts with a unit join in when they are done with it.
//  BY_SPLIT   APART with another numbering of the wavefronts.
enum { APART, ONE_SPLIT, DRAWN, BY_SPLIT };

// Several splits: whether the tiles are drawn.  At least five tiles for each wavefront that an even deal would give
// them to, and more wavefronts than pools, also of those that start without a unit.
LQ_HD bool draws_tiles(int dynamic, int NW, int nwf, int TF, int TQ) {
  return dynamic && NW - TF > NSUB && NW - nwf > NSUB && TQ >= 5 * (NW - nwf);
}

// APART or BY_SPLIT, for workgroups of 8: with fewer than two tiles for a wavefront, every compute unit in use and more
// than an eighth of the wavefronts at the units, these are kept together in the first workgroups and leave the others to
// nothing but tiles (8 rows of 2048 tokens, 9 of 32 wavefronts at the units, four layers 37.9 against 39.5 us; 4 of 3000
// 35.2 against 36.1; but 1 row of 2048, 56 workgroups, 32.9 against 31.6).  Of 100 shapes with several splits of 8 and tiles
// that are not drawn, the 9 inside the rule take 0.93 to 1.02 of the time of APART, 0.986 on average, the 91 outside it
// would take 0.96 to 1.13, 1.028 on average.  A program of its own: a choice in the kernel
// delays the first load (8 rows of 4096 tokens 47.7 -> 48.1 us).  Workgroups of 4 and 12 always are BY_SPLIT: of 4, two
// share a compute unit, and place by place both would have their units on the same SIMD (38 rows of up to 10277 tokens
// 162 against 143 us); of 12, none of the shapes measured gains (31898 tokens, 8 heads of 8, 72.5 against 71.5 us).
LQ_HD bool keeps_units_together(int NW, int nwf, int TQ, bool chip_full) {
  return chip_full && TQ < 2 * (NW - nwf) && 8 * nwf > NW;
}

template <int PROG, int NWB>
struct Deal {
  int NWF, NWQ;          // wavefronts that start with a unit, and with a tile (ONE_SPLIT: all of them count here)
  int unit0, unit_step;  // this wavefront's units, if it takes any
  int first;             // its first tile (DRAWN: negative for those that start with a unit)
  int step1;             // from the first tile to the second, where they are not drawn
  int pool_of;           // the pool it draws from

  // split, wave: this wavefront; nwf: the share of wavefronts for the units in APART and BY_SPLIT; TF: number of units
  LQ_HD Deal(int splits, int split, int wave, int nwf, int TF) {
    const int NW = PROG == ONE_SPLIT ? NWB : splits * NWB;
    NWF = PROG == ONE_SPLIT ? 0 : PROG == DRAWN ? (TF < NW ? TF : NW) : nwf;
    NWQ = NW - NWF;
    unit0 = PROG == ONE_SPLIT ? wave : PROG == BY_SPLIT ? split * NWB + wave : wave * splits + split;
    unit_step = PROG == APART || PROG == BY_SPLIT ? NWF : NW;
    if (PROG == ONE_SPLIT) {
      const int nh = TF % NWB, nl = NWB - nh;   // wavefronts with one unit more, and the others
      const bool ahead = nh > 0 && wave >= nh;
      first = nh == 0 ? wave : ahead ? wave - nh : 2 * nl + wave;
      step1 = ahead ? nl : NWB;
      pool_of = 0;
    } else {
      first = unit0 - NWF;
      step1 = NWQ;
      // DRAWN: a pool is drawn from by wavefronts of many workgroups and, within those, of places far apart: the older
      // wavefronts of a workgroup are faster.  (Numbered like the units, a pool belonged to one workgroup at 2, 4 and 8
      // splits, and one that started late kept all its tiles; with one place to a pool, 131072 tokens of 4-bit codes
      // took 144 instead of 137 us for four layers; with neighbouring places, shapes of 3, 5 and 9 splits 2 to 4% more.)
      // In the others only wavefronts without units draw: the first eight cover all pools, and more than eight draw.
      const int gw = split * NWB + wave;
      pool_of = (PROG == DRAWN ? 3 * gw + gw / NSUB : PROG == APART ? first + 3 * (first / NSUB) : first) % NSUB;
    }
  }
  LQ_HD bool takes_units(int TF) const { return unit0 < (PROG == APART || PROG == BY_SPLIT ? NWF : TF); }
  LQ_HD bool takes_tiles() const { return PROG == ONE_SPLIT || PROG == DRAWN || unit0 >= NWF; }
  // Tiles that are not drawn: the second, then every NWQ-th.
  LQ_HD int second() const { return first + step1; }
  LQ_HD int after(int t) const { return t + NWQ; }
  // Tiles that are drawn: the first two of a wavefront without units are fixed, the v-th draw from its pool gives
  LQ_HD int drawn(int v) const { return 2 * NWQ + v * NSUB + pool(); }
  LQ_HD int pool() const { return pool_of; }
};

}  // namespace lq
