// Rules that decide how a call runs, as plain functions of the sizes they
// depend on: no result depends on them.  Constant expressions, so the kernels,
// the host code and a compiler without HIP read the same ones.
#pragma once

#include <stdint.h>

namespace tc {

// ---- late passes of the time sort ----------------------------------------------
// Blocks of the passes that only time ranges past 33 bits use (milliseconds over
// a year have 35).  Others leave them idle, and an idle block costs its launch:
// an eighth of the tiles, but as many as the CUs hold at once, which an active
// pass needs.  A multiple of 8 where it is not every tile (tiles go to the XCDs
// by their index mod 8).  The build with an eighth of the tiles and with these:
// 36-bit times, 5e5 edges 307 and 270 us, 2e6 468 and 410, 5e6 1,051 and 1,012;
// 60-bit times, 5e5 462 and 307, 2e6 838 and 609; 22-bit times (the passes idle)
// 249 and 246, 369 and 372, 946 and 949.
constexpr int64_t late_pass_blocks(int64_t ntiles) {
  const int64_t eighth = (ntiles + 63) / 64 * 8, resident = 2 * 256;
  const int64_t b = eighth > resident ? eighth : resident;
  return b < ntiles ? b : ntiles;
}

// ---- run table of the build ----------------------------------------------------
// Whether the graph's runs are few for its edges: n vertices have at most n^2
// pairs.  Grouping the runs by table segment costs per edge, inserting them one
// by one per run, and few runs are long ones, whose ends both ways search for.
// The whole build, grouped and inserted, us: 3e6 edges of 40, 1,000 and 1,700
// vertices 429, 510, 588 and 388, 499, 624; 2e7 of 40, 1,000 and 3,000 1,750,
// 2,355, 2,509 and 1,632, 2,312, 2,772; 6e7 of 40, 1,700 and 5,500 5,180, 8,310,
// 7,578 and 4,710, 8,107, 8,682.
constexpr bool few_pairs(int64_t n, int64_t m) { return n * n < m / 8; }

// ---- windows of small graphs ---------------------------------------------------
// Whether every edge's windows are searched by its own thread in the lists of
// its end vertices (two launches) instead of by merge passes (seven).  Searches
// in the source's lists share lines with their neighbours in scan order; those
// in the destination's lists do not, and leave the XCD's L2 as the graph grows,
// the sooner the longer the lists.  Every delta adds a search to the first way
// and little to the second.  The lines, in 65,536 edges, lie below the first
// size at which the searches were the slower way on any of twenty graphs: degree
// exponents of 1.8 to 2.4 with 2 to 20 edges a vertex, and (long lists, 128
// edges a vertex and more) uniform and skewed ones of 20 to 2,000 vertices.
// Merge passes and searches, us, exponent 1.8, 20 edges a vertex:
//   both sides, one delta    786,432 edges 113 and 113
//   both sides, two          589,824 131 and 123, 655,360 131 and 140
//   both sides, four         589,824 205 and 195, 655,360 204 and 223
//   destination only, one    524,288 75 and 63, 589,824 84 and 87
//   destination only, four   458,752 130 and 114, 524,288 131 and 140
//   source only, one, eight  786,432 76 and 44, 263 and 138
// 300 vertices:
//   both sides, one, four    524,288 92 and 71, 150 and 157; 458,752 143 and 136
//   destination, one, eight  524,288 73 and 64; 393,216 147 and 168
constexpr int64_t kDirectEdges = (int64_t)12 << 16;  // the most any call searches
constexpr bool direct_windows(int64_t n, int64_t m, int deltas, bool source, bool destination) {
  // one, two, three or four, five to eight deltas
  constexpr uint8_t both[2][4] = {{12, 9, 9, 9}, {8, 8, 7, 6}};
  constexpr uint8_t dest[2][4] = {{8, 8, 7, 7}, {8, 7, 6, 5}};
  const int lists = m >= 128 * n ? 1 : 0;
  const int d = deltas <= 2 ? deltas - 1 : (deltas <= 4 ? 2 : 3);
  const int64_t line = !destination ? 12 : (source ? both[lists][d] : dest[lists][d]);
  return m > 0 && m <= line << 16;
}

// ---- order of a chunk's samples ------------------------------------------------
// Whether a chunk's samples are put in rank order before the path kernel.  That
// costs two launches and 4 bytes a sample, and makes neighbouring slots share
// lines of the graph.  One delta, not ordered and ordered, graphs of 1e5, 1e6
// and 2e7 edges: 2.6e5 samples 66, 67, 81 and 72, 72, 86 us; 5.2e5 87, 94, 118
// and 89, 92, 118; 7.9e5 105, 110, 147 and 103, 108, 143; 1e7 681 to 1,170 and
// 558 to 924.  One ordering serves every delta of the call: 2.6e5 samples of
// two 70, 82, 121 and 75, 76, 112, of four 130, 145, 213 and 119, 124, 190;
// 7.9e5 of two 100, 128, 233 and 104, 110, 192, of four 211, 257, 439 and 179,
// 199, 354.
// A per-sample output array is then written far apart by neighbouring slots, a
// partial line each.  One array (4 or 8 bytes a sample) costs less than the
// order gains; from two arrays on the order is the slower way.  Not ordered and
// ordered, 8e6 samples over 3e5, 3e6 and 2e7 edges: P alone 528, 773, 937 and
// 419, 723, 920 us; P and one motif's X 534, 792, 954 and 466, 933, 1,088; e1..e3
// and X 610, 913, 1,095 and 872, 1,372, 1,463; every output of six motifs 1,144,
// 2,276, 3,165 and 2,465, 3,552, 4,419.
constexpr uint32_t kOrderFrom = 3u << 18;
constexpr bool orders_samples(uint32_t samples, uint32_t arrays) {
  return samples >= kOrderFrom && arrays <= 1u;
}

// ---- merged ListCount pass: items per claim ------------------------------------
// Its blocks claim tickets from one counter, which serves a claim in about
// 12 ns.  An item claimed alone holds a pass of short items to that; sixteen
// long items in a row on one block are the pass's critical path when the
// queue is short.  So tickets are of sixteen items while more than sixteen a
// block are left, of four while more than four a block are, then of one: no
// block is left with more of them than the queue's share of a block and one
// ticket.  Six motifs, 6e7 edges, the whole call with tickets of sixteen for
// three quarters of any queue, with these, and with one item a claim: 1e3
// samples 655, 253 and 244 us; 3e4 1,102, 516 and 519 us; 1e6 4.28, 4.24 and
// 4.25 ms; 4e6 (5.3e5 items) 13.3, 13.3 and 13.4 ms.
constexpr uint32_t kWideResident = 2560;  // blocks at five wavefronts per SIMD on 256 CUs

// Blocks the tickets are shared among.  Windows of 2^32 and more put lists of
// every length in the queue, most of them short: the claims weigh more there,
// and half the blocks is the middle way.  Over 1e6 and 5e6 edges in
// milliseconds, for all the blocks, half and a quarter of them: 1e5 samples of
// one motif 458, 415 and 390 us (one item a claim 486), 3e4 samples of six
// 1,066, 1,093 and 1,374 us (1,174).
constexpr uint32_t wide_shares(uint32_t launched, bool any_length) {
  const uint32_t b = launched < kWideResident ? launched : kWideResident;
  return any_length ? (b + 1u) / 2u : b;
}

struct WideDeal {
  uint32_t n, t16, t4;  // items, tickets of 16, tickets of 4
  constexpr WideDeal(uint32_t items, uint32_t shares)
      : n(items),
        t16(items > 16u * shares ? (items - 16u * shares) / 16u : 0u),
        t4(items - 16u * t16 > 4u * shares ? (items - 16u * t16 - 4u * shares) / 4u : 0u) {}
  // items of ticket t: *lo .. *hi - 1, none past the last ticket
  constexpr void range(uint32_t t, uint32_t* lo, uint32_t* hi) const {
    if (t < t16) {
      *lo = t * 16u;
      *hi = *lo + 16u;
    } else if (t - t16 < t4) {
      *lo = t16 * 16u + (t - t16) * 4u;
      *hi = *lo + 4u;
    } else {
      const uint64_t i = (uint64_t)t16 * 16u + (uint64_t)t4 * 4u + (t - t16 - t4);
      *lo = (uint32_t)(i < n ? i : n);
      *hi = i < n ? *lo + 1u : n;
    }
  }
};

}  // namespace tc
