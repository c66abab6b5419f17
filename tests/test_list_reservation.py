"""CPU replay of how the raster's groups reserve their runs of the list (vs_lists.h): whatever finds no room, no two runs
may overlap.  The reservation is the kernel's own code, compiled for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_02482_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# usage: driver PART_WORDS GROUPS LO HI SEED THREADS: needs drawn from LO..HI; prints runs, words in them, overlaps of the
# rule below and of one that leaves in the counters what found no room
DRIVER = r'''
#include <algorithm>
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>
#include "vs_lists.h"

static std::atomic<uint64_t> counters[vs::kParts];
static std::atomic<uint32_t> narrow[vs::kParts];

static uint32_t leaves_it(uint32_t need, uint32_t part_words, uint32_t own) {
  for (uint32_t q = 0; q < (uint32_t)vs::kParts; ++q) {
    const uint32_t p = (own + q) % vs::kParts;
    const uint32_t from = narrow[p].fetch_add(need);
    if (from <= part_words - need) return p * part_words + from;
  }
  return vs::kGroupNoRun;
}

int main(int, char** a) {
  const uint32_t part = strtoul(a[1], 0, 0), groups = strtoul(a[2], 0, 0), lo = strtoul(a[3], 0, 0), hi = strtoul(a[4], 0, 0);
  const int threads = atoi(a[6]);
  std::mt19937 rng(atoi(a[5]));
  std::vector<uint32_t> need(groups), base(groups);
  for (auto& n : need) n = std::uniform_int_distribution<uint32_t>(lo, hi)(rng);
  const vs::ListRoom room = {part, ~0u, vs::kParts};
  for (int rule = 0; rule < 2; ++rule) {
    for (auto& c : counters) c = 0;
    std::atomic<uint32_t> next(0);
    auto work = [&] {
      for (uint32_t g; (g = next++) < groups;)
        base[g] = rule ? leaves_it(need[g], part, g & 7)
                       : vs::reserve_run(need[g], need[g] / 2, room, g, [](uint32_t p) { return counters[p].load(); },
                                         [](uint32_t p, uint64_t n) { return counters[p].fetch_add(n); });
    };
    std::vector<std::thread> pool;
    for (int t = 0; t < threads; ++t) pool.emplace_back(work);
    for (auto& t : pool) t.join();
    std::vector<std::pair<uint64_t, uint64_t>> runs;
    uint64_t words = 0, overlaps = 0, outside = 0, past = 0;
    for (uint32_t g = 0; g < groups; ++g)
      if (base[g] != vs::kGroupNoRun) {
        runs.push_back({base[g], base[g] + (uint64_t)need[g]});
        words += need[g];
        outside += base[g] / part != (base[g] + need[g] - 1) / part || base[g] / part >= vs::kParts;
      }
    std::sort(runs.begin(), runs.end());
    for (size_t i = 1; i < runs.size(); ++i) overlaps += runs[i].first < runs[i - 1].second;
    for (auto& c : counters) past += (uint32_t)c.load() > part;
    printf("%zu %llu %llu %llu %llu\n", runs.size(), (unsigned long long)words, (unsigned long long)overlaps,
           (unsigned long long)outside, (unsigned long long)past);
  }
}
'''


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("lists")
    src, exe = d / "driver.hip", d / "driver"
    src.write_text(DRIVER)
    subprocess.check_call([HIPCC, "--offload-host-only", "-O2", "-std=c++17", "-pthread", "-I", CSRC, str(src), "-o", str(exe)])

    def run(*args):
        rows = subprocess.check_output([str(exe), *[str(a) for a in args]], text=True).split("\n")[:2]
        return [tuple(int(x) for x in r.split()) for r in rows]
    return run


# a layer of 16 M triangles with 160-pixel boxes in bins of 8 pixels: 15,625 groups of about 0.3 M words, of which a view of
# 1024^2 with the automatic workspace has room for a few hundred; small runs in a small list; mixed ones
@pytest.mark.parametrize("threads", [1, 6])
@pytest.mark.parametrize("part,groups,lo,hi", [
    (16_000_000, 15_625, 290_000, 330_000), (1_000, 200_000, 1, 1_001), (16_384, 1_000_000, 300, 9_000), (64, 500, 1, 64)])
def test_no_two_runs_overlap(driver, part, groups, lo, hi, threads):
    (runs, words, overlaps, outside, past), _ = driver(part, groups, lo, hi, 5, threads)
    assert overlaps == 0 and outside == 0 and past == 0
    assert 0 < runs and words <= 8 * part
    # the list is used: what is left in a part is less than the largest run
    assert words > 8 * (part - hi)


def test_the_replay_finds_overlaps(driver):
    """A rule that leaves failed additions in the counters wraps them within the 16 M triangles' groups."""
    _, (_, _, overlaps, _, _) = driver(16_000_000, 15_625, 290_000, 330_000, 5, 1)
    assert overlaps > 0
