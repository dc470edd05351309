"""The work split of decode, walked on the CPU as its kernels walk it: the
header that the launcher and the kernels share is compiled with the host
compiler and every worker's piece is followed cache by cache.  Each filled slot
is read exactly once and nothing past a fill, a cache split over several
workers finds its partials in slots of its own within the workspace, pieces
differ by at most one unit, and every resident slot has work in calls that
memory bounds."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

from paper_2406_14909_amd import build as B

pytestmark = pytest.mark.skipif(shutil.which(B.CXX) is None, reason="no host compiler")

_WALK = r"""
#include <string.h>
#include <vector>
#include "decode_split.h"
using namespace moa;

// 0 when the split is sound; otherwise the number of the broken rule.
// out: workers, unit shift, longest and shortest piece (units), most partials of a cache
extern "C" int walk(int hkv, const int64_t* fill, int batch, int64_t slots, int round_shift, int paired,
                    int64_t* out) {
  DecodeArgs a;
  memset(&a, 0, sizeof(a));
  a.hkv = hkv;
  a.batch = batch;
  for (int g = 0; g < hkv; ++g) a.seg_start[g + 1] = a.seg_start[g] + fill[g];
  a.seq_keys = a.seg_start[hkv];
  split_decode(a, slots, round_shift, paired != 0);
  const int64_t workers = a.workers;
  if (workers < 1 || workers > slots) return 1;
  if (a.seq_keys != a.seg_start[hkv] || worker_start(a, workers) != a.seq_keys * batch) return 2;
  std::vector<int64_t> next(size_t(batch) * hkv, 0);        // virtual keys of each cache covered so far
  std::vector<char> used(workers + size_t(batch) * hkv, 0); // partial slots
  int64_t longest = 0, shortest = INT64_MAX, parts = 0;
  for (int w = 0; w < workers; ++w) {
    int64_t x = worker_start(a, w);
    const int64_t end = worker_start(a, w + 1);
    if (end <= x) return 3;                                 // a worker without work
    longest = std::max(longest, (end - x) >> a.unit_shift);
    shortest = std::min(shortest, (end - x) >> a.unit_shift);
    int b = int(mul_floor(x, a.inv_seq_keys)), g = 0;
    int64_t r = x - b * a.seq_keys;
    while (a.seg_start[g + 1] <= r) ++g;
    while (x < end) {
      if (b >= batch) return 4;
      const int64_t len = a.seg_start[g + 1] - a.seg_start[g], lo = r - a.seg_start[g];
      const int64_t hi = std::min(len, lo + (end - x));
      const int64_t c = int64_t(b) * hkv + g;
      if (lo != next[c] || hi <= lo) return 5;              // a gap or an overlap
      next[c] = hi;
      if (lo >= fill[g]) return 6;                          // a piece past the cache's fill
      const int64_t base = int64_t(b) * a.seq_keys + a.seg_start[g];
      const int w0 = worker_of(a, base), w1 = worker_of(a, base + len - 1);
      if (w < w0 || w > w1) return 7;                       // the merge would miss this worker
      const bool whole = lo == 0 && hi == len;
      if (whole != (w0 == w1)) return 8;
      if (!whole) {
        const int64_t slot = w + c;
        if (slot >= int64_t(used.size()) || used[slot]++) return 9;
        parts = std::max<int64_t>(parts, w1 - w0 + 1);
      }
      x += hi - lo;
      r += hi - lo;
      if (hi == len && ++g == hkv) {
        g = 0;
        ++b;
        r = 0;
      }
    }
  }
  for (int64_t c = 0; c < int64_t(next.size()); ++c)
    if (next[c] < fill[c % hkv]) return 10;                 // keys left out
  out[0] = workers;
  out[1] = a.unit_shift;
  out[2] = longest;
  out[3] = shortest;
  out[4] = parts;
  return 0;
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("split")
    src, out = tmp / "walk.cpp", tmp / "walk.so"
    src.write_text(_WALK)
    r = subprocess.run([B.CXX, "-std=c++17", "-O1", "-g", "-shared", "-fPIC", "-Wall", "-Wextra", f"-I{B.INCLUDE}",
                        f"-I{B.CSRC}", str(src), "-o", str(out)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    assert r.returncode == 0, r.stdout.decode(errors="replace")
    lib = ctypes.CDLL(str(out))

    def call(fills, batch, slots, round_shift, paired=False):
        n = len(fills)
        res = (ctypes.c_int64 * 5)()
        st = lib.walk(n, (ctypes.c_int64 * n)(*fills), batch, ctypes.c_int64(slots), round_shift, int(paired), res)
        assert st == 0, (st, fills, batch, slots, round_shift, paired)
        out = dict(zip(("workers", "shift", "longest", "shortest", "parts"), res))
        assert out["longest"] - out["shortest"] <= 1, out
        return out

    return call


@pytest.mark.parametrize("paired", [False, True])
@pytest.mark.parametrize("round_shift", [6, 7, 8])
@pytest.mark.parametrize("slots", [768, 1024])
def test_every_slot_works_where_memory_bounds_the_call(walk, slots, round_shift, paired):
    """Just above a whole number of rounds per slot, handing every worker
    ceil(rounds / slots) rounds left up to half of the slots without work."""
    for ratio in (2.05, 2.5, 3.05, 4.05, 5.05, 8.05, 12.05, 15.5, 17.0, 40.0):
        for hkv, batch in ((8, 4), (8, 16), (32, 4), (32, 16)):
            per_cache = max(1, round(ratio * slots / (hkv * batch)))
            s = walk([(per_cache << round_shift) - 37] * hkv, batch, slots, round_shift, paired)
            assert s["workers"] == slots, (ratio, hkv, batch, s)


@pytest.mark.parametrize("slots,batch", [(768, 7), (1024, 14), (768, 20), (768, 16), (1024, 23)])
def test_uneven_caches_are_cut_at_whole_rounds(walk, slots, batch):
    """Pieces of equal keys cross from one cache to the next with a partial round
    on both sides, which costs up to a tenth of a call of a few rounds per slot."""
    for ratio in (2.1, 3.05, 4.6, 7.5, 12.3):
        per_cache = ratio * slots / (8 * batch)
        fills = [max(1, int(128 * per_cache * x)) for x in (.25, .5, 1.75, 1.0, .5, 2.0, 1.5, .5)]
        s = walk(fills, batch, slots, 7)
        assert s["shift"] == 7 and s["workers"] == slots, (ratio, s)
    s = walk([int(40 * 128 * slots / (8 * batch))] * 7 + [1], batch, slots, 7)
    assert s["shift"] == 0                                   # a partial round weighs nothing
    if slots % (8 * batch) == 0:
        assert walk([int(3.05 * 128 * slots / (8 * batch))] * 8, batch, slots, 7)["shift"] == 0   # aligned


@pytest.mark.parametrize("fills,batch,workers,longest", [
    ([12064] * 8, 1, 380, 2), ([24064] * 8, 1, 502, 3),     # few partials for the merge
    ([100064], 1, 196, 4), ([131136], 1, 205, 5),           # long caches: many, but not a work-group each
    ([33064], 1, 130, 2), ([32768], 1, 64, 4), ([32769], 1, 129, 2),
    ([10936, 16064, 32064, 40064, 50064, 60064, 66064, 66064], 1, 768, 4),   # no slot idles
])
def test_partials_of_few_long_caches(walk, fills, batch, workers, longest):
    s = walk(fills, batch, 768, 7)
    assert (s["workers"], s["longest"]) == (workers, longest), s



@pytest.mark.parametrize("rounds,workers,longest", [
    (700, 700, 1), (768, 768, 1),              # a round each
    (769, 385, 2), (792, 396, 2), (1024, 512, 2),   # some worker has two: all of them
    (1025, 768, 2), (1200, 768, 2),            # too many slots would idle
    (1344, 672, 2), (1536, 768, 2),
])
def test_paired_rounds(walk, rounds, workers, longest):
    s = walk([100] * (rounds % 8 or 8) + [1], 1, 768, 7, True)       # (a small one: no limit applies)
    assert s["workers"] == (rounds % 8 or 8) + 1
    s = walk([128 * 1] * 1, rounds, 768, 7, True)
    assert (s["workers"], s["longest"]) == (workers, longest)
    if rounds > 768:
        assert walk([128], rounds, 768, 7, False)["workers"] == 768


def test_every_key_once_and_partials_apart(walk):
    rng = random.Random(7)
    for _ in range(400):
        hkv, batch = rng.choice([1, 2, 3, 7, 8, 32, 64]), rng.choice([1, 1, 2, 5, 23])
        shift, slots = rng.choice([6, 7, 8]), rng.choice([1, 2, 256, 768, 1024, 8192])
        top = rng.choice([1, 65, 300, 3000, 20000])
        fills = [rng.choice([1, rng.randint(1, top), (rng.randint(1, top) >> shift << shift) + rng.choice([0, 1])]) or 1
                 for _ in range(hkv)]
        s = walk(fills, batch, slots, shift, rng.random() < 0.5)
        if s["shift"]:
            assert s["parts"] <= 256 + 2, s        # kMaxParts pieces, begun and ended inside other ones


@pytest.mark.parametrize("fills,batch", [([1], 1), ([1] * 64, 1), ([64], 1), ([65], 1), ([128 * 64], 1), ([128 * 64 + 1], 1),
                                         ([1 << 20], 1), ([(1 << 30) - 1, 1], 1), ([64 + 4096] * 8, 300),
                                         ([(1 << 30) - 1] * 64, 30000)])
@pytest.mark.parametrize("slots", [1, 1024])
@pytest.mark.parametrize("paired", [False, True])
def test_split_at_extremes(walk, fills, batch, slots, paired):
    walk(fills, batch, slots, 7, paired)
