"""The buckets by which prefill attention orders its query tiles (csrc/tile_order.h), compiled for the host."""
import ctypes
import random
import subprocess

from paper_2604_11554_amd import build

SOURCE = """
#include "tile_order.h"
extern "C" int bucket(int keys, int longest) { return rlx::tile_bucket(keys, longest, rlx::tile_shift(longest)); }
"""


def test_every_tile_has_a_bucket_and_longer_ones_come_first(tmp_path):
    (tmp_path / "order.hip").write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", build.CSRC,
                    str(tmp_path / "order.hip"), "-o", str(tmp_path / "order.so")], check=True, capture_output=True)
    f = ctypes.CDLL(str(tmp_path / "order.so")).bucket
    rng = random.Random(1)
    for longest in [0, 1, 2, 1022, 1023, 1024, 1025, 32768, 2 ** 31 - 1] + [rng.randint(1, 2 ** 31 - 1) for _ in range(200)]:
        # a cached length below zero is outside the contract, but no reason to count past the buckets
        keys = sorted({-2 ** 31, -1024, -64, -1, 0, 1, longest // 2, max(longest - 1, 0), longest} | {rng.randint(0, longest) for _ in range(50)})
        got = [f(k, longest) for k in keys]
        assert all(0 <= b < 1024 for b in got), longest
        assert all(a >= b for a, b in zip(got, got[1:])), longest
        if longest >= 512:
            assert got[-1] <= 511                                     # the longest is in the front half: the buckets are used
        if 0 < longest < 1024:
            assert [f(k, longest) for k in range(longest + 1)] == [1023 - k for k in range(longest + 1)]
