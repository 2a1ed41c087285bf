// Rules that decide how a call runs, as plain functions of the sizes they
// depend on: no result depends on them.  Constant expressions, so the kernels,
// the host code and a compiler without HIP read the same ones.
#pragma once

#include <stdint.h>

namespace tc {

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
