"""The rule by which a token's experts are chosen (csrc/topk_rule.h), compiled for the host: 64 lanes, each the best of its
experts, the largest key of all.  Whatever the logits are, the ids are different ones of [0, E)."""
import ctypes
import subprocess

import numpy as np
import pytest

from paper_2604_11554_amd import build

SOURCE = """
#include "topk_rule.h"
template <int NJ> static void choose(const float* logits, int n_experts, int top_k, int* ids, float* ranks) {
  float rank[64][NJ];
  for (int lane = 0; lane < 64; ++lane)
    for (int j = 0; j < NJ; ++j) rank[lane][j] = lane + 64 * j < n_experts ? rlx::topk_rank(logits[lane + 64 * j]) : rlx::TOPK_GONE;
  for (int k = 0; k < top_k; ++k) {
    uint64_t best = 0;
    for (int lane = 0; lane < 64; ++lane) {
      const uint64_t key = rlx::topk_lane_key<NJ>(rank[lane], lane);
      if (key > best) best = key;
    }
    ids[k] = rlx::topk_key_id(best);
    ranks[k] = rlx::topk_key_rank(best);
    if (ids[k] < 0 || ids[k] >= n_experts) return;
    rank[ids[k] % 64][ids[k] / 64] = rlx::TOPK_GONE;
  }
}
extern "C" void choose_experts(const float* logits, int n_experts, int top_k, int* ids, float* ranks) {
  if (n_experts <= 128) choose<2>(logits, n_experts, top_k, ids, ranks);
  else choose<4>(logits, n_experts, top_k, ids, ranks);
}
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("topk")
    (d / "choose.hip").write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-I", build.CSRC,
                    str(d / "choose.hip"), "-o", str(d / "choose.so")], check=True, capture_output=True)
    lib = ctypes.CDLL(str(d / "choose.so"))

    def f(logits, top_k):
        z = np.ascontiguousarray(logits, np.float32)
        ids, ranks = np.full(top_k, -7, np.int32), np.zeros(top_k, np.float32)
        lib.choose_experts(z.ctypes.data_as(ctypes.c_void_p), len(z), top_k, ids.ctypes.data_as(ctypes.c_void_p),
                           ranks.ctypes.data_as(ctypes.c_void_p))
        return ids, ranks

    return f


@pytest.mark.parametrize("n_experts", [1, 2, 31, 64, 65, 128, 129, 256])
def test_the_ids_are_different_experts_whatever_the_logits_are(choose, n_experts):
    rng = np.random.default_rng(n_experts)
    nan, inf = np.float32(np.nan), np.float32(np.inf)
    rows = {"numbers": rng.standard_normal(n_experts), "ties": rng.integers(-1, 2, n_experts), "nan": np.full(n_experts, nan),
            "minus": np.full(n_experts, -inf), "plus": np.full(n_experts, inf), "lowest": np.full(n_experts, np.finfo(np.float32).min)}
    for p in (0.1, 0.5, 0.97):
        z = rng.standard_normal(n_experts)
        for bad in (nan, inf, -inf):
            z = np.where(rng.random(n_experts) < p, bad, z)
        rows["mixed %.2f" % p] = z
    for name, z in rows.items():
        z = np.asarray(z, np.float32)
        rank = np.where(np.isnan(z) | (z == -inf), np.finfo(np.float32).min, z)
        for k in sorted({1, min(8, n_experts), min(64, n_experts)}):
            ids, ranks = choose(z, k)
            np.testing.assert_array_equal(ids, np.argsort(-rank, kind="stable")[:k], err_msg=name)
            np.testing.assert_array_equal(ranks, rank[ids], err_msg=name)
