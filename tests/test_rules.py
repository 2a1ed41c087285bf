"""CPU tests of the rules that decide how a call runs (csrc/tc_rules.h, plain
constant expressions), compiled into a small program with g++."""
import heapq
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2409_08975_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstring>
#include "tc_rules.h"
int main() {
  char what[32];
  long long a, b, c;
  while (std::scanf("%31s %lld %lld %lld", what, &a, &b, &c) == 4) {
    if (!std::strcmp(what, "shares")) {
      std::printf("%u\n", tc::wide_shares((uint32_t)a, b != 0));
    } else if (!std::strcmp(what, "order")) {
      std::printf("%d\n", tc::orders_samples((uint32_t)a, (uint32_t)b));
    } else if (!std::strcmp(what, "direct")) {  // c: source, destination, vertices
      std::printf("%d\n", tc::direct_windows(c >> 2, a, (int)b, (c & 1) != 0, (c & 2) != 0));
    } else if (!std::strcmp(what, "few")) {
      std::printf("%d\n", tc::few_pairs(a, b));
    } else if (!std::strcmp(what, "late")) {
      std::printf("%lld\n", (long long)tc::late_pass_blocks(a));
    } else if (!std::strcmp(what, "tickets")) {
      const tc::WideDeal d((uint32_t)a, (uint32_t)b);
      for (uint32_t t = 0;; ++t) {
        uint32_t lo, hi;
        d.range(t, &lo, &hi);
        if (lo == hi) break;
        std::printf("%u:%u ", lo, hi);
      }
      uint32_t lo, hi;
      d.range(0xFFFFFFFFu, &lo, &hi);
      std::printf("%u:%u\n", lo, hi);
    }
  }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = d / "rules.cpp", d / "rules"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)

    def ask(*queries):
        text = "".join("%s %d %d %d\n" % (q + (0,) * (4 - len(q))) for q in queries)
        return subprocess.run([str(exe)], input=text, capture_output=True, text=True,
                              check=True).stdout.splitlines()
    return ask


def _tickets(line):
    return [tuple(map(int, x.split(":"))) for x in line.split()]


@pytest.mark.parametrize("blocks", [1, 16, 32, 2560, 4096])
@pytest.mark.parametrize("any_length", [False, True])
def test_merged_pass_tickets(rules, blocks, any_length):
    """Tickets hand out every item once, and no block is left with a row of
    them while others idle: with items of one cost, claimed in order by
    `blocks` blocks, the last block ends within two items of the queue's
    share of a block (with tickets for half the blocks, once the queue is past
    two items a block, within eight more)."""
    shares = int(rules(("shares", blocks, any_length))[0])
    live = min(blocks, 2560)
    assert shares == (live + 1) // 2 if any_length else shares == live
    sizes = [1, 2, 15, 16, 17, 63, 64, 65, 1000, 1001, 4 * shares, 4 * shares + 1, 8000, 16 * shares + 1, 40000,
             40001, 16 * shares + 17, 200003]
    for n, line in zip(sizes, rules(*(("tickets", n, shares) for n in sizes))):
        *tickets, past = _tickets(line)
        assert past == (n, n)
        assert [lo for lo, _ in tickets] == [0] + [hi for _, hi in tickets[:-1]] and tickets[-1][1] == n
        assert {hi - lo for lo, hi in tickets} <= {1, 4, 16}
        ends = [0] * live
        for lo, hi in tickets:
            heapq.heapreplace(ends, ends[0] + hi - lo)
        slack = 8 if any_length and n > 2 * live else 0
        assert max(ends) <= n / live + 2 + slack, n


def test_sample_order_and_outputs(rules):
    """Long chunks are put in rank order, which scatters the per-sample
    outputs, only for at most one output array a sample."""
    sizes = [1, 1 << 16, (3 << 18) - 1, 3 << 18, 10**6, 1 << 25]
    for arrays in (0, 1, 2, 3, 5, 20):
        got = [int(x) for x in rules(*(("order", n, arrays) for n in sizes))]
        assert got == [int(n >= 3 << 18 and arrays <= 1) for n in sizes]


# Sizes (in 65,536 edges) up to which searching every edge's windows was
# measured faster than the merge passes, and the first at which it was slower
# on some graph: with fewer than 128 edges a vertex, and with more.
@pytest.mark.parametrize("sides,deltas,faster,slower,long_faster,long_slower", [
    (3, 1, 12, None, 8, 9), (3, 2, 9, 10, 8, 9), (3, 4, 9, 10, 7, 8), (3, 8, 9, 11, 6, 7), (2, 1, 8, 9, 8, 9),
    (2, 2, 8, 9, 7, 8), (2, 4, 7, 8, 6, 7), (2, 8, 7, 8, 5, 6), (1, 1, 12, None, 12, None), (1, 8, 12, None, 12, None)])
def test_windows_of_small_graphs(rules, sides, deltas, faster, slower, long_faster, long_slower):
    """Windows are searched edge by edge only at sizes where that was not
    measured slower on any of the graphs, and at all of them up to 5 * 2^16."""
    line = [m for m in range(1, 14 << 16, 4096)] + [k << 16 for k in range(1, 15)]
    for n, top, bad in ((1 << 16, faster, slower), (300, long_faster, long_slower)):
        ask = [("direct", m, deltas, sides | n << 2) for m in line]
        got = dict(zip(line, map(int, rules(*ask))))
        assert all(got[m] for m in line if m <= 5 << 16)
        assert not any(got[m] for m in line if m > top << 16)
        assert bad is None or not got[bad << 16]
    assert rules(("direct", 0, deltas, sides | 4)) == ["0"]


@pytest.mark.parametrize("m,inserted,grouped", [
    (1700000, 400, 1000), (3 * 10**6, 400, 1700), (5 * 10**6, 700, 1700), (10**7, 700, 1700), (2 * 10**7, 1000, 3000),
    (6 * 10**7, 1700, 5500)])
def test_run_table_of_few_vertices(rules, m, inserted, grouped):
    """Vertex counts at which inserting the runs one by one was measured the
    faster build, and at which grouping them was; the largest counts do not
    overflow."""
    ask = [1, 2, 40, inserted, grouped, 30000, 2**31 - 1]
    assert rules(*(("few", n, m) for n in ask)) == ["1"] * 4 + ["0"] * 3


def test_late_time_passes_fill_the_chip(rules):
    """Passes of wide time ranges get a block per tile up to the 512 blocks
    the CUs hold, then at least those and an eighth of the tiles."""
    tiles = [1, 7, 8, 160, 489, 511, 512, 513, 1221, 4095, 4096, 4883, 73243]
    for n, b in zip(tiles, map(int, rules(*(("late", n) for n in tiles)))):
        assert b == n if n <= 512 else 512 <= b <= max(512, n // 8 + 8) and b % 8 == 0
