"""CPU replay of how the raster's groups reserve their runs of the list (vs_lists.h): whatever finds no room, no two runs
may overlap.  The reservation is the kernel's own code, compiled for the host."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_02482_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# usage: driver PART_WORDS GROUPS LO HI SEED THREADS: needs drawn from LO..HI; prints runs, words in them, overlaps of the
# rule and of one that leaves in counters of 32 bits what found no room
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
                                         [](uint32_t p, uint64_t n) { return counters[p].fetch_add(n); }, [](uint64_t) { return (uint64_t)0; });
    };
    std::vector<std::thread> pool;
    for (int t = 0; t < threads; ++t) pool.emplace_back(work);
    for (auto& t : pool) t.join();
    std::vector<std::pair<uint64_t, uint64_t>> runs;
    uint64_t words = 0, overlaps = 0, outside = 0;
    for (uint32_t g = 0; g < groups; ++g)
      if (base[g] != vs::kGroupNoRun) {
        runs.push_back({base[g], base[g] + (uint64_t)need[g]});
        words += need[g];
        outside += base[g] / part != (base[g] + need[g] - 1) / part || base[g] / part >= vs::kParts;
      }
    std::sort(runs.begin(), runs.end());
    for (size_t i = 1; i < runs.size(); ++i) overlaps += runs[i].first < runs[i - 1].second;
    printf("%zu %llu %llu %llu\n", runs.size(), (unsigned long long)words, (unsigned long long)overlaps,
           (unsigned long long)outside);
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
    (runs, words, overlaps, outside), _ = driver(part, groups, lo, hi, 5, threads)
    assert overlaps == 0 and outside == 0
    assert 0 < runs and words <= 8 * part
    # the list is used: what is left in a part is less than the largest run
    assert words > 8 * (part - hi)


def test_the_replay_finds_overlaps(driver):
    """A rule that leaves failed additions in counters of 32 bits wraps them within the 16 M triangles' groups."""
    _, (_, _, overlaps, _) = driver(16_000_000, 15_625, 290_000, 330_000, 5, 1)
    assert overlaps > 0


# every order in which the groups' loads and additions can follow each other: prints orders, and those with overlapping runs
ORDERS = r'''
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <thread>
#include <vector>
#include <algorithm>
#include "vs_lists.h"

struct Group { uint32_t need, base; bool waiting, done; };
static std::mutex mu;
static std::condition_variable cv;
static std::vector<Group> groups;
static uint64_t counter[2];
static int turn;   // the group whose step is next, -1: the scheduler's

static void step(int g) {   // wait to be let on
  std::unique_lock<std::mutex> l(mu);
  groups[g].waiting = true;
  cv.notify_all();
  cv.wait(l, [&] { return turn == g; });
  turn = -1;
  groups[g].waiting = false;
}

static void work(int g, vs::ListRoom room) {
  const auto load = [&](uint32_t p) { step(g); return counter[p]; };
  const auto add = [&](uint32_t p, uint64_t n) { step(g); const uint64_t c = counter[p]; counter[p] += n; return c; };
  groups[g].base = RESERVE;
  std::unique_lock<std::mutex> l(mu);
  groups[g].done = true;
  cv.notify_all();
}

int main(int, char** a) {
  const uint32_t limit = atoi(a[1]), taken = atoi(a[2]), parts = atoi(a[3]);
  std::vector<uint32_t> needs;
  for (char** q = a + 4; *q; ++q) needs.push_back(atoi(*q));
  const vs::ListRoom room = {limit, ~0u, (int32_t)parts};
  std::vector<std::pair<int, int>> choice;   // taken, of how many
  long orders = 0, overlaps = 0;
  do {
    counter[0] = counter[1] = taken; groups.assign(needs.size(), {0, 0, false, false}); turn = -1;
    for (size_t g = 0; g < needs.size(); ++g) groups[g].need = needs[g];
    std::vector<std::thread> pool;
    for (size_t g = 0; g < needs.size(); ++g) pool.emplace_back(work, (int)g, room);
    for (size_t at = 0;; ++at) {
      std::unique_lock<std::mutex> l(mu);
      cv.wait(l, [] { return turn == -1 && std::all_of(groups.begin(), groups.end(), [](const Group& g) { return g.waiting || g.done; }); });
      std::vector<int> can;
      for (size_t g = 0; g < groups.size(); ++g) if (!groups[g].done) can.push_back((int)g);
      if (can.empty()) break;
      if (at == choice.size()) choice.push_back({0, (int)can.size()});
      turn = can[choice[at].first];
      cv.notify_all();
    }
    for (auto& t : pool) t.join();
    ++orders;
    bool bad = false;
    for (size_t i = 0; i < groups.size(); ++i) if (groups[i].base != vs::kGroupNoRun) {
      bad |= groups[i].base % limit < taken || groups[i].base % limit + groups[i].need > limit || groups[i].base / limit >= parts;
      for (size_t j = 0; j < i; ++j) if (groups[j].base != vs::kGroupNoRun)
        bad |= groups[i].base < groups[j].base + groups[j].need && groups[j].base < groups[i].base + groups[i].need;
    }
    overlaps += bad;
    while (!choice.empty() && choice.back().first + 1 == choice.back().second) choice.pop_back();
    if (!choice.empty()) ++choice.back().first;
  } while (!choice.empty());
  printf("%ld %ld\n", orders, overlaps);
}
'''
# as it is, and a rule that takes a failed addition off again
KERNEL = "vs::reserve_run(groups[g].need, 0, room, g, load, add, [](uint64_t) { return (uint64_t)0; })"
GIVES_BACK = ("[&]() -> uint32_t { const uint64_t t = add(0, groups[g].need); if (t <= room.words - groups[g].need) return (uint32_t)t; "
              "add(0, 0ull - groups[g].need); return vs::kGroupNoRun; }()")


def _orders(tmp_path, reserve, *args):
    src, exe = tmp_path / "orders.hip", tmp_path / "orders"
    src.write_text(ORDERS.replace("RESERVE", reserve))
    subprocess.check_call([HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-pthread", "-I", CSRC, str(src), "-o", str(exe)])
    return [int(x) for x in subprocess.check_output([str(exe), *map(str, args)], text=True).split()]


@pytest.mark.parametrize("limit,taken,parts,needs", [(10, 4, 1, (7, 5, 1, 5)), (10, 4, 2, (7, 5, 6)), (10, 7, 2, (2, 2, 2, 2)), (6, 5, 2, (1, 3, 1))])
def test_no_order_of_groups_overlaps(tmp_path, limit, taken, parts, needs):
    orders, overlaps = _orders(tmp_path, KERNEL, limit, taken, parts, *needs)
    assert orders > 20 and overlaps == 0


def test_the_orders_find_a_rule_that_gives_back(tmp_path):
    """Words given back after another group's were taken above them are handed out twice."""
    orders, overlaps = _orders(tmp_path, GIVES_BACK, 10, 4, 1, 7, 5, 1, 5)
    assert orders > 20 and overlaps > 0
