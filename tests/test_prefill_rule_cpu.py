"""The grid of a bf16 prefill launch and the choice of its kernel, on the CPU: the
launcher's header is compiled with the host compiler and its work-groups are
dealt to the dies as the kernel reads them from its block index."""
import ctypes
import random
import shutil
import subprocess

import pytest

from paper_2406_14909_amd import build as B

pytestmark = pytest.mark.skipif(shutil.which(B.CXX) is None, reason="no host compiler")

_DEAL = r"""
#include <string.h>
#include <vector>
#include "prefill_rule.h"
using namespace moa;

// shape: waves, key groups; out: work-groups of the fullest die, the grid's own count of them,
// tiles of the longest chain.  Returns 0, or the number of the broken rule.
extern "C" int deal(int batch, int hq, int hkv, int head_dim, int64_t n, int window, int sink, int* shape, int64_t* out) {
  PrefillArgs a;
  memset(&a, 0, sizeof(a));
  a.n = n; a.batch = batch; a.hq = hq; a.hkv = hkv; a.group = hq / hkv; a.num_sink = sink;
  for (int g = 0; g < hkv; ++g) a.window[g] = window;
  const PrefillShape s = prefill_shape(a, head_dim);
  shape[0] = s.waves;
  shape[1] = s.key_groups;
  const PrefillGrid g = prefill_grid(a, 32 * s.waves);
  std::vector<int64_t> die(kNumXcd, 0);
  std::vector<char> seen(size_t(batch) * hq * g.tiles, 0);
  const int64_t per_unit = a.group * g.qchunk, hb = int64_t(hkv) * batch;
  for (int64_t i = 0; i < g.blocks; ++i) {
    const int64_t xcd = i % kNumXcd, local = i / kNumXcd, round = local / per_unit, within = local % per_unit;
    const int64_t unit = round * kNumXcd + ((round & 1) ? kNumXcd - 1 - xcd : xcd);
    if (unit >= g.n_units) continue;
    const int64_t qt = (g.n_chunks - 1 - unit / hb) * g.qchunk + (g.qchunk - 1 - within / a.group);
    if (qt >= g.tiles) continue;
    const int64_t head = (unit % hb) / batch * a.group + within % a.group, b = unit % batch;
    if (qt < 0 || seen[(b * hq + head) * g.tiles + qt]++) return 1;
    ++die[xcd];
  }
  for (char c : seen)
    if (!c) return 2;
  out[0] = *std::max_element(die.begin(), die.end());
  out[1] = g.per_die;
  return out[0] <= out[1] ? 0 : 3;
}

extern "C" void shape_f32(int batch, int hq, int hkv, int head_dim, int64_t n, int window, int* out) {
  PrefillArgs a;
  memset(&a, 0, sizeof(a));
  a.n = n; a.batch = batch; a.hq = hq; a.hkv = hkv; a.group = hq / hkv;
  for (int g = 0; g < hkv; ++g) a.window[g] = window;
  const PrefillF32Shape s = prefill_f32_shape(a, head_dim);
  out[0] = s.shared;
  out[1] = s.key_groups;
  out[2] = s.row_blocks;
}
"""


@pytest.fixture(scope="module")
def deal(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("rule")
    src, out = tmp / "deal.cpp", tmp / "deal.so"
    src.write_text(_DEAL)
    r = subprocess.run([B.CXX, "-std=c++17", "-O1", "-shared", "-fPIC", "-Wall", "-Wextra", f"-I{B.INCLUDE}",
                        f"-I{B.CSRC}", str(src), "-o", str(out)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    assert r.returncode == 0, r.stdout.decode(errors="replace")
    lib = ctypes.CDLL(str(out))

    def call(b, hq, hkv, d, n, window, sink=4):
        shape, res = (ctypes.c_int * 2)(), (ctypes.c_int64 * 2)()
        st = lib.deal(b, hq, hkv, d, ctypes.c_int64(n), window, sink, shape, res)
        assert st == 0, (st, b, hq, hkv, d, n, window)
        return tuple(shape), res[0]

    call.lib = lib
    return call


def test_every_row_tile_once_and_split_work_groups_fit_their_die(deal):
    """A work-group of two key groups has (head_dim 64: half) a compute unit's LDS.
    The earlier rule counted the whole chip's and gave one die four times what
    it holds: 8 query heads of one KV head x 1,024 tokens 32.1 -> 50.0 us."""
    rng = random.Random(5)
    for _ in range(600):
        hkv = rng.choice([1, 1, 2, 3, 4, 5, 8, 9, 10, 17, 32])
        hq, d = hkv * rng.choice([g for g in (1, 2, 4, 8) if hkv * g <= 64]), rng.choice([64, 128])
        n = int(round(2 ** rng.uniform(0, 13)))
        w = max(1, int(n * rng.choice([0.05, 0.3, 0.5, 1.0])))
        b = rng.choice([1, 1, 2, 3])
        (waves, groups), fullest = deal(b, hq, hkv, d, n, w)
        assert (waves, groups) in ((4, 1), (4, 2), (2, 2))
        if groups == 2:
            slots = 32 if d == 128 else 64
            even = w < 0.8 * n or n < 20 * 64             # no row's chain is much longer than another's
            if even and (waves == 4 or d == 128):
                assert fullest <= slots, (b, hq, hkv, d, n, w, waves, fullest)
            assert fullest <= 2 * slots


@pytest.mark.parametrize("args,shape", [
    ((1, 32, 32, 128, 512, 512), (2, 2)), ((1, 32, 32, 128, 513, 513), (4, 2)), ((1, 32, 32, 128, 192, 192), (4, 1)),
    ((1, 8, 1, 128, 1024, 1024), (4, 1)), ((1, 8, 1, 128, 256, 256), (2, 2)), ((1, 16, 2, 128, 777, 388), (4, 1)),
    ((1, 16, 16, 128, 3000, 3000), (4, 2)), ((1, 9, 9, 128, 4096, 2048), (4, 1)), ((1, 32, 32, 128, 4096, 4096), (4, 1)),
    ((1, 8, 1, 64, 4096, 204), (2, 2)), ((1, 8, 1, 64, 1024, 307), (4, 1)), ((1, 16, 16, 64, 512, 512), (2, 2)),
    ((8, 32, 32, 128, 8192, 8192), (4, 1)), ((1, 1, 1, 128, 1, 1), (4, 1)),
])
def test_shape_at_the_measured_sizes(deal, args, shape):
    assert deal(*args)[0] == shape


SHARED, FOUR_32, FOUR_64, TWO_64 = (1, 1, 1), (0, 4, 1), (0, 4, 2), (0, 2, 2)


@pytest.mark.parametrize("args,shape", [
    # long prompts, which the kernels without shared tiles made up to 16 % slower
    ((1, 64, 8, 64, 8192, 8192), SHARED), ((1, 32, 8, 64, 8192, 4096), SHARED), ((1, 32, 8, 64, 4096, 4096), SHARED),
    ((1, 32, 32, 64, 8192, 8192), SHARED), ((1, 8, 8, 64, 16384, 16384), SHARED), ((8, 32, 32, 64, 4096, 2048), SHARED),
    ((1, 8, 8, 64, 8192, 1638), SHARED), ((1, 64, 8, 64, 2048, 2048), SHARED), ((1, 16, 2, 64, 16384, 16384), SHARED),
    ((1, 8, 8, 64, 8192, 8192), FOUR_32), ((1, 64, 8, 64, 2048, 1024), FOUR_64), ((1, 16, 2, 64, 8192, 8192), FOUR_64),
    ((1, 32, 32, 64, 4096, 4096), FOUR_64), ((8, 16, 16, 64, 1024, 1024), FOUR_64), ((1, 8, 8, 64, 1501, 1501), FOUR_32),
    ((1, 32, 32, 64, 2048, 2048), FOUR_32), ((1, 32, 32, 64, 1024, 204), TWO_64), ((1, 1, 1, 64, 1, 1), FOUR_32),
    ((1, 32, 8, 64, 4096, 81), TWO_64), ((8, 16, 16, 64, 2048, 40), TWO_64),
    ((1, 32, 32, 128, 4096, 4096), (0, 1, 1)), ((2, 16, 8, 128, 800, 800), (0, 2, 1)), ((1, 4, 4, 128, 99, 1), (0, 4, 1)),
])
def test_f32_shape_at_the_measured_sizes(deal, args, shape):
    out = (ctypes.c_int * 3)()
    b, hq, hkv, d, n, w = args
    deal.lib.shape_f32(b, hq, hkv, d, ctypes.c_int64(n), w, out)
    assert tuple(out) == shape
