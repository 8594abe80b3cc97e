// Runs the attention kernel's own deal (csrc/lq_schedule.h) for random launches, the drawing wavefronts in random
// order, and checks that every unit of fp rows and every tile is taken exactly once.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "lq_schedule.h"

using namespace lq;
static std::mt19937 rng(2503);
static int any(int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); }
static int one_of(std::initializer_list<int> v) { return v.begin()[rng() % v.size()]; }

struct Wave { int ta, tb, kd, pool; bool on; };

static void fail(const char* what, int prog, int NWB, int NS, int nwf, int TF, int TQ) {
  printf("%s: program %d, %d wavefronts, %d splits, nwf %d, units %d, tiles %d\n", what, prog, NWB, NS, nwf, TF, TQ);
  exit(1);
}

template <int PROG, int NWB>
static void check(int NS, int nwf, int TF, int TQ, bool dyn) {
  std::vector<int> units(TF, 0), tiles(TQ, 0), counter(NSUB, 0), drawers(NSUB, 0), groups(NSUB, 0), last(NSUB, -1);
  std::vector<Wave> w;
  for (int split = 0; split < NS; ++split)
    for (int wave = 0; wave < NWB; ++wave) {
      const Deal<PROG, NWB> d(NS, split, wave, nwf, TF);
      if (d.takes_units(TF))
        for (int u = d.unit0; u < TF; u += d.unit_step) {
          if (u < 0) fail("unit below 0", PROG, NWB, NS, nwf, TF, TQ);
          ++units[u];
        }
      if (!d.takes_tiles()) continue;
      if (dyn) {   // the kernel's loop, one step of a random wavefront at a time (below)
        if (d.pool() < 0 || d.pool() >= NSUB) fail("no such pool", PROG, NWB, NS, nwf, TF, TQ);
        ++drawers[d.pool()];
        if (last[d.pool()] != split) { last[d.pool()] = split; ++groups[d.pool()]; }
        w.push_back({d.first, d.second(), 0, d.pool(), true});
        continue;
      }
      if (d.first < 0) fail("tile below 0", PROG, NWB, NS, nwf, TF, TQ);
      for (int ta = d.first, tb = d.second(); ta < TQ; ta = tb, tb = d.after(tb)) ++tiles[ta];
    }
  if (dyn) {
    for (int p = 0; p < NSUB; ++p) {
      if (!drawers[p]) fail("a pool that nobody draws from", PROG, NWB, NS, nwf, TF, TQ);
      // a workgroup that starts late can only be relieved by others that draw from its pools
      if (PROG == DRAWN && NS * NWB >= 2 * NSUB && groups[p] < 2) fail("a pool of one workgroup", PROG, NWB, NS, nwf, TF, TQ);
    }
    std::vector<Deal<PROG, NWB>> deal;
    for (int split = 0; split < NS; ++split)
      for (int wave = 0; wave < NWB; ++wave) {
        const Deal<PROG, NWB> d(NS, split, wave, nwf, TF);
        if (d.takes_tiles()) deal.push_back(d);
      }
    for (size_t i = 0; i < w.size(); ++i)
      if (PROG == DRAWN && deal[i].takes_units(TF)) {
        const int ka = counter[w[i].pool]++, kb = counter[w[i].pool]++;
        w[i].ta = deal[i].drawn(ka);
        w[i].tb = deal[i].drawn(kb);
      }
    for (size_t left = w.size(); left;) {
      const size_t i = rng() % w.size();
      if (!w[i].on) continue;
      if (w[i].ta < TQ) {
        const bool more = w[i].tb < TQ;
        const int kd = counter[w[i].pool]++;
        ++tiles[w[i].ta];
        if (more) { w[i].ta = w[i].tb; w[i].tb = deal[i].drawn(kd); continue; }
      }
      w[i].on = false;
      --left;
    }
  }
  for (int u = 0; u < TF; ++u)
    if (units[u] != 1) fail("unit not taken once", PROG, NWB, NS, nwf, TF, TQ);
  for (int t = 0; t < TQ; ++t)
    if (tiles[t] != 1) fail("tile not taken once", PROG, NWB, NS, nwf, TF, TQ);
}

template <int NWB>
static void all() {
  int drawn = 0;
  for (int i = 0; i < 4000; ++i) {
    const int TQ = one_of({0, 1, 2, 3, 63, 64, 65, any(0, 400), any(0, 4000)});
    const int TF = one_of({1, 2, NWB - 1, NWB, NWB + 1, any(1, 24), any(1, 100)});
    check<ONE_SPLIT, NWB>(1, 0, TF, TQ, false);
    const int NS = one_of({1, 2, 3, 4, 5, 8, 16, 32, any(1, 64)}), NW = NS * NWB;
    const int nwf = TQ == 0 ? NW : any(1, TF < NW - 1 ? TF : NW - 1);   // as fp_wave_share gives it
    check<APART, NWB>(NS, nwf, TF, TQ, false);
    check<BY_SPLIT, NWB>(NS, nwf, TF, TQ, false);
    if (NS > 1 && draws_tiles(1, NW, nwf, TF, TQ)) {
      check<APART, NWB>(NS, nwf, TF, TQ, true);
      check<BY_SPLIT, NWB>(NS, nwf, TF, TQ, true);
      check<DRAWN, NWB>(NS, nwf, TF, TQ, true);
      ++drawn;
    }
  }
  printf("%d wavefronts: %d launches with drawn tiles\n", NWB, drawn);
  if (drawn < 300) exit(2);
}

// Every slot with a token lies in exactly one of the tiles that LiveTiles numbers, at the slot it says.
static void live_tiles() {
  for (int i = 0; i < 20000; ++i) {
    const int G = one_of({64, 128}), W = one_of({1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, any(1, 700), any(1, 60000)});
    const int Wq = (W + G - 1) / G * G, per_event = (W + 63) / 64;
    LiveTiles l;
    l.set(W, Wq);
    for (int k = 0; k < 8; ++k) {
      const int e = one_of({0, 1, 2, any(0, 50), (1 << 25) / (Wq / 64)}), j = one_of({0, per_event - 1, any(0, per_event - 1)});
      const LiveTiles::Place p = l.place(e * per_event + j);
      if (p.tile != e * (Wq / 64) + j || p.slot0 != 64 * j) { printf("W %d, Wq %d, event %d, tile %d\n", W, Wq, e, j); exit(3); }
    }
  }
}

// What the kernel divides: numbers below B * Hq <= 65535, by a factor of that product.
static void divisors() {
  for (int n = 1; n <= 65535; ++n) {
    Divisor d;
    d.set(n);
    const int last = 65535 / n * n - 1;   // the largest number there is with this divisor
    for (int x : {0, 1, n - 1, n, n + 1, last / n * n, last, any(0, last), any(0, last)})
      if (x <= last && d.quotient(x) != x / n) { printf("%d / %d\n", x, n); exit(4); }
  }
}

int main() {
  divisors();
  live_tiles();
  all<4>();
  all<8>();
  all<12>();
  return 0;
}
