"""How the shared prefixes of a decode batch are cut into tiles (csrc/prefix_plan.h), compiled for the host: every shared unit of every
member is in one tile per KV head, and no tile is the time of the whole launch."""
import ctypes
import random
import subprocess
import sys

import numpy as np
import pytest

from paper_2604_11554_amd import build

SOURCE = """
#include "prefix_plan.h"
extern "C" int64_t words(int n, int Hkv) { return (int64_t)rlx::shared_prefix_words(n, Hkv); }
extern "C" int64_t plain_units(int hd, int n_layers) { return rlx::shared_prefix_plain_units(hd, n_layers); }
extern "C" void range(int lo, int hi, int max_blocks, int* out) {
  const rlx::PrefixRange r = rlx::prefix_range(lo, hi, max_blocks);
  out[0] = r.lo; out[1] = r.hi;
}
extern "C" void fill(int n, int Hq, int Hkv, const int32_t* leader, const int32_t* pages, int most_tiles, int64_t plain_units,
                     int32_t* out) {
  rlx::shared_prefix_build(n, Hq, Hkv, leader, pages, most_tiles, plain_units, out);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("prefix")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-ftrapv", "-I", build.CSRC, str(d / "plan.cpp"), "-o",
                    str(d / "plan.so")], check=True, capture_output=True)
    l = ctypes.CDLL(str(d / "plan.so"))
    l.words.restype = l.plain_units.restype = ctypes.c_int64
    return l


def _tiles(lib, groups, Hq, Hkv, most_tiles, plain_units=284):
    """groups: (members, pages of every member) -> header, per-sequence arrays, tiles (row, kvh, lo, hi, members)"""
    leader, pages = [], []
    for p in groups:
        leader += [len(pages)] * len(p)
        pages += p
    n, m = len(pages), len(pages) * Hkv
    out = np.full(lib.words(n, Hkv) + 4, -99, np.int32)
    a, b = np.array(leader, np.int32), np.array(pages, np.int32)
    lib.fill(n, Hq, Hkv, a.ctypes.data_as(ctypes.c_void_p), b.ctypes.data_as(ctypes.c_void_p), most_tiles, ctypes.c_int64(plain_units),
             out.ctypes.data_as(ctypes.c_void_p))
    assert (out[-4:] == -99).all()
    out = out[:-4]
    assert out[0] == n and out[1] <= m
    start, tile0, chunks, col0 = out[8:8 + 4 * n].reshape(4, n)
    t = out[8 + 4 * n:8 + 4 * n + 4 * m].reshape(4, m)
    mem = out[8 + 4 * n + 4 * m:].reshape(m, 16)
    return out[:8], start, tile0, chunks, col0, [(*t[:, i].tolist(), mem[i].tolist()) for i in range(out[1])]


@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (4, 2), (16, 1), (32, 4), (2, 2)])
@pytest.mark.parametrize("most_tiles", [0, 16, 512])
def test_every_shared_unit_of_every_member_is_in_one_tile(lib, Hq, Hkv, most_tiles):
    rng = random.Random(Hq * 1000 + Hkv * 10 + most_tiles)
    group = Hq // Hkv
    MS = min(16, 32 // group)
    for _ in range(60):
        groups = [[rng.choice([0, 1, 2, 3, 17, rng.randint(0, 400)]) for _ in range(rng.choice([1, 1, 2, 5, 9, 33]))]
                  for _ in range(rng.randint(1, 60))]
        head, start, tile0, chunks, col0, tiles = _tiles(lib, groups, Hq, Hkv, most_tiles)
        n, seen = 0, set()
        for p in groups:
            units = min(p) // 2 if len(p) > 1 else 0
            for j in range(len(p)):
                i = n + j
                assert start[i] == units
                if not units:
                    assert chunks[i] == 0
                    continue
                first = n + j // MS * MS
                assert col0[i] == (i - first) * group and 1 <= chunks[i] <= 4
                for h in range(Hkv):
                    at = 0
                    for c in range(chunks[i]):
                        row, kvh, lo, hi, mem = tiles[tile0[i] + c * Hkv + h]
                        assert (row, kvh, lo) == (n, h, at) and hi > lo and mem[i - first] == i
                        assert [x for x in mem if x >= 0] == list(range(first, min(first + MS, n + len(p))))
                        seen.add(tile0[i] + c * Hkv + h)
                        at = hi
                    assert at == units
            n += len(p)
        assert seen == set(range(len(tiles)))
        shared = [p for p in groups if len(p) > 1 and min(p) >= 2]
        few = sum(min(p) // 2 for p in shared) * Hkv <= 284
        assert head[3] == int(len(shared) > 0 and (few or any(len(p) > MS for p in shared)))
        longest = [0] * (len(tiles) + 1)                      # of the tiles of a run of chunks: the list comes longest first
        firsts = sorted({tile0[i] for i in range(n) if chunks[i]})
        longest = [max(t[3] - t[2] for t in tiles[a:b]) for a, b in zip(firsts, firsts[1:] + [len(tiles)])]
        assert longest == sorted(longest, reverse=True)


def _lengths(lib, units, members=8, most_tiles=512):
    _, _, _, _, _, tiles = _tiles(lib, [[2 * u] * members for u in units], 32, 8, most_tiles)
    return len(tiles), max(t[3] - t[2] for t in tiles)


def test_a_long_prefix_among_short_ones_is_split(lib):
    # 32 query and 8 KV heads on 512 workgroups: as many groups as one chunk each fills the device with, and more than that
    assert _lengths(lib, [40] * 63 + [937]) == (63 * 8 + 4 * 8, 235)
    assert _lengths(lib, [40] * 64 + [937]) == (64 * 8 + 4 * 8, 235)
    assert _lengths(lib, [8] * 96 + [937], members=2) == (96 * 8 + 2 * 8, 469)     # pairs: the descriptor has room for two chunks each
    n, longest = _lengths(lib, [16 + 48 * i // 69 for i in range(70)] + [500, 500])
    assert longest <= 125 and n <= 80 * 8
    # no longer than twice an even deal, or a quarter of the prefix
    rng = random.Random(3)
    for _ in range(200):
        units = [rng.choice([1, 9, rng.randint(1, 100), rng.randint(1, 3000)]) for _ in range(rng.randint(1, 150))]
        even = -(-sum(units) * 8 // 512)
        n, longest = _lengths(lib, units)
        assert longest <= max(8, 2 * even, max(-(-u // 4) for u in units))


def test_chunks_are_as_many_as_one_round_takes(lib):
    # even prefixes: the shortest chunks that fit 512 workgroups, one each where nothing shorter does
    assert _lengths(lib, [64] * 16) == (512, 16) and _lengths(lib, [64] * 32) == (512, 32) and _lengths(lib, [64] * 33) == (264, 64)
    assert _lengths(lib, [40] * 65) == (520, 40) and _lengths(lib, [40] * 128) == (1024, 40)
    # MoE policies: the same chunks whatever the number of tiles is
    assert _lengths(lib, [40] * 128, most_tiles=0) == (4096, 10) and _lengths(lib, [17] * 8, most_tiles=0) == (192, 6)


@pytest.mark.timeout(20)
def test_page_counts_of_any_size(lib):
    # the search halves its range: 256 groups of the largest counts there are take no longer than others, and nothing overflows
    top = 2 ** 31 - 1
    assert _lengths(lib, [top // 2] * 256, members=4) == (2048, top // 2)
    assert _lengths(lib, [3] * 255 + [top // 2], members=4) == (255 * 8 + 32, -(-(top // 2) // 4))
    _, start, _, _, _, tiles = _tiles(lib, [[top] * 2] * 8, 32, 8, 512)
    assert start[0] == top // 2 and max(t[3] for t in tiles) == top // 2


def test_a_tiles_units_are_in_the_block_table_whatever_the_words_hold(lib):
    # what the kernel does with them: entries 2 lo + 0 .. 63, capped at the last one, then units lo + wave .. hi - 1
    out, top = (ctypes.c_int * 2)(), 2 ** 31 - 1
    words = [-top - 1, -1, 0, 1, 3, 7, 8, 9, 2 ** 30 - 1, 2 ** 30, top - 3, top]
    for lo in words:
        for hi in words:
            for max_blocks in (1, 2, 15, 16, 1 << 20):
                lib.range(lo, hi, max_blocks, out)
                assert 0 <= out[0] <= out[1] <= max_blocks // 2, (lo, hi, max_blocks)
                assert 2 * out[0] + 63 <= top and (out[0] == out[1] or 2 * (out[1] - 1) + 1 < max_blocks)
                if 0 <= lo < hi <= max_blocks // 2:
                    assert (out[0], out[1]) == (lo, hi)


# the entry with the descriptor of 65 536 rows and 64 KV heads to stage (320 MB) in a process that may have 64 MB more than it has; of the
# model it looks at the configuration that a handle begins with, and it returns before it touches a device
OUT_OF_MEMORY = """
import ctypes as C, resource
from paper_2604_11554_amd import binding as B
l = B.lib()
n, model = 65536, (C.c_char * 65536)()
cfg = B.ModelConfig.from_buffer(model)
cfg.n_q_heads, cfg.n_kv_heads = 64, 64
leader, pages = (C.c_int32 * n)(), (C.c_int32 * n)(*[4] * n)
have = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (have + (64 << 20),) * 2)
rc = l.rlx_shared_prefix_build(C.addressof(model), n, leader, pages, 4096, 1 << 40, None)
print(rc, l.rlx_last_error().decode())
"""


def test_no_exception_leaves_the_entry():
    r = subprocess.run([sys.executable, "-c", OUT_OF_MEMORY], cwd=build.HERE + "/..", capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stderr)
    assert r.stdout.split(" ", 1)[0] == "-2" and "host allocation failed" in r.stdout, r.stdout


def test_which_pages_are_copied_without_the_streaming_mark(lib):
    # 160 MB of a unit's 16 KB (heads of 128, 8 KB of 64) per KV head and layer
    assert [lib.plain_units(hd, n) for hd, n in ((128, 36), (128, 48), (128, 2), (64, 2), (128, 100000))] == [284, 213, 5120, 10240, 0]
    flag = lambda groups, units: _tiles(lib, groups, 32, 8, 512, units)[0][3]  # noqa: E731
    assert [flag([[2 * 17] * 8] * 2, u) for u in (271, 272)] == [0, 1]          # 34 units of eight KV heads
    assert flag([[2 * 17] * 9], 0) == 1                                          # nine members: two tiles read the pages
    assert flag([[0] * 8], 1000) == 0
