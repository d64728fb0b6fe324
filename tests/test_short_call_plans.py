"""How short calls cut their products (csrc/flow_plan.h), compiled for the host: every plan covers K once and is one of the kernels
that are built, the form is chosen where it says, and the products of test_gpu_short_calls.py reach every tiling."""
import ctypes
import random
import subprocess

import pytest

from paper_2604_11554_amd import build

import rollout_inputs as RI
import test_gpu_norm_inside as GN
import test_gpu_short_calls as G

SOURCE = """
#include "flow_plan.h"
extern "C" int store_plan(int N, int K, int T, int units, int planes) {
  const rlx::FlowPlan p = rlx::flow_store_plan(N, K, T, 16, units, planes);
  return p.rt * 100 + p.splits;
}
extern "C" int store_form(int N, int K, int T, int units, int planes) { return rlx::flow_store_form(N, K, T, units, planes); }
extern "C" int norm_fits(int T, int K) { return rlx::flow_norm_fits(T, K); }
extern "C" int norm_form(int T, int K, int planes_o, int planes_down) { return rlx::flow_norm_form(T, K, planes_o, planes_down); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    (d / "plans.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", build.CSRC, str(d / "plans.cpp"), "-o", str(d / "plans.so")],
                   check=True, capture_output=True)
    return ctypes.CDLL(str(d / "plans.so"))


def test_every_plan_covers_k_once_with_a_kernel_that_is_built(lib):
    rng = random.Random(5)
    for _ in range(20000):
        N, K = 8 * rng.randint(1, 2500), 16 * rng.randint(1, 1200)
        planes, units = rng.choice([1, 2]), rng.choice([256, 256, 1, 64, 304])
        T = rng.randint(1, 128 if planes == 1 else 96)
        rt, splits = divmod(lib.store_plan(N, K, T, units, planes), 100)
        steps = (K // 16 + 1) // 2
        per = -(-steps // splits)
        assert rt in ((2, 4, 5, 8) if T <= 64 else (2, 4, 5)), (N, K, T, rt)
        assert 1 <= splits <= 16 and (splits - 1) * per < steps <= splits * per, (N, K, T, splits)
        assert splits == 1 or per >= 4                                 # a step for each of the four waves


def test_the_form_of_a_store(lib):
    # fp16 in one term: up to 128 tokens, whatever the widths
    assert [lib.store_form(6144, 2560, t, 256, 1) for t in (1, 49, 64, 65, 128, 129)] == [1, 1, 1, 1, 1, 0]
    # bf16 in two: up to 96 but for 49 to 64 where the other form cuts K in five or fewer: 256 // 43 = 5, 256 // 42 = 6
    for rows, narrow in ((1, 1), (2560, 1), (128 * 42, 1), (128 * 42 + 1, 0), (6144, 0), (40000, 0)):
        assert [lib.store_form(rows, 2560, t, 256, 2) for t in (1, 48, 49, 64, 65, 96, 97, 128)] == [1, 1, narrow, narrow, 1, 1, 0, 0]
    # activations of more than 5 MiB: 96 tokens of 13 653 columns in two terms, of 27 306 in one
    assert [lib.store_form(5120, k, 96, 256, 2) for k in (13648, 13664)] == [1, 0]
    assert [lib.store_form(5120, k, 96, 256, 1) for k in (27296, 27312)] == [1, 0]


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
def test_the_compared_products_reach_every_tiling(lib, fmt):
    planes = 2 if fmt == "bf16" else 1
    stores = set()
    for s in G.WIDE.values():
        for t in G.WIDE_TOKENS:
            token_tiles = next(n for n in (1, 2, 3, 4, 6, 8) if t <= 16 * n)
            for N, K in ((s.q_dim + 2 * s.kv_dim, s.d_model), (s.d_model, s.q_dim), (s.d_model, s.d_ff)):
                if lib.store_form(N, K, t, 256, planes):
                    stores.add((lib.store_plan(N, K, t, 256, planes) // 100, token_tiles))
    # all (row tiles, token tiles) that any product of up to 16 384 x 12 288 takes
    want = {(rt, n) for rt in (2, 4, 5) for n in (1, 2, 3, 4, 6)} | {(8, n) for n in (2, 3, 4)}
    want |= {(8, 1)} if planes == 2 else {(rt, 8) for rt in (2, 4, 5)}
    assert stores == want, stores ^ want


def test_where_the_norm_goes_into_the_products(lib):
    s = RI.TINY_DENSE

    def inside(T, d, q_dim, d_ff, planes):
        o, down = (lib.store_plan(d, k, T, 256, planes) % 100 for k in (q_dim, d_ff))
        return lib.norm_form(T, d, o, down)

    # the compared calls: all but the last ones, on either side of three slices per thread
    last = {80: 13, 512: 8, 1024: 5, 2544: 2, 5120: 1}
    for planes in (1, 2):
        for d, d_ff, rows in GN.SHAPES:
            assert [inside(T, d, s.q_dim, d_ff, planes) for T in rows] == [int(T <= last[d]) for T in rows], (planes, d)
            assert last[d] in rows and last[d] + 1 in rows
        # measured: d_model, width of the attention output, d_ff: rows that gain, rows that lose (or are even)
        for d, q_dim, d_ff, yes, no in ((256, 256, 688, 10, 12), (512, 512, 1536, 6, 8), (1024, 2048, 3072, 4, 5), (1536, 1536, 8960, 3, 4),
                                        (2048, 2048, 6144, 2, 3), (2560, 4096, 9728, 2, 3), (4096, 4096, 12288, 1, 2)):
            assert [inside(T, d, q_dim, d_ff, planes) for T in (yes, no)] == [1, 0], (planes, d)
    # more planes, fewer rows; never past what the kernels are built for
    assert [lib.norm_form(4, 512, p, p) for p in (2, 6, 13, 14, 16)] == [1, 1, 1, 0, 0]
    for T in range(1, 40):
        for d in (16, 48, 256, 1024, 5120, 5136, 20480):
            assert lib.norm_fits(T, d) == int(T <= 16 and T * d <= 5120)
            assert lib.norm_form(T, d, 1, 1) <= lib.norm_fits(T, d)
