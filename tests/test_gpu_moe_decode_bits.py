"""MoE decode keeps the order of its sums: the router's near-ties turn on the last bits of its input, so another order of
the same sums sends tokens to other experts.  The logits and the routing of a few decode steps are compared bit for bit
with those of the library at commit 9132d03 on an MI355X (CRC-32 of every row), recorded in golden/moe_decode_crc.json by
`digests` below; nothing else has a claim to these bits."""
import json
import os
import zlib

import numpy as np
import pytest
import torch

import rollout_inputs as RI

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "moe_decode_crc.json")
TWO_KV = RI.TINY_MOE.replace(n_q_heads=8, n_kv_heads=2, head_dim=128)
# shape, format, prompt lengths, members of a sampling group per prompt, attention grid (0: the default)
CASES = {
    "ragged": (RI.TINY_MOE, "bf16", [1, 31, 32, 33, 97, 130, 250, 511, 600, 1100], 1, 0),
    "ragged_hd128": (TWO_KV, "bf16", [5, 64, 129, 300, 700], 1, 0),
    "ragged_one_term": (TWO_KV, "bf16 one term", [5, 64, 129, 300, 700], 1, 0),
    "ragged_f16": (RI.TINY_MOE, "f16", [1, 31, 130, 250, 700], 1, 0),
    "pairs_are_shares": (TWO_KV, "bf16", [150] * 6, 1, 12),     # as many workgroups as pairs of equal length
    "few_shares": (RI.TINY_MOE, "bf16", [40, 350, 3, 900], 1, 3),
    "many_rows": (RI.TINY_MOE, "bf16", [1 + 7 * (i % 13) for i in range(70)], 1, 0),
    "rows_200": (RI.TINY_MOE, "bf16", [1 + i % 40 for i in range(200)], 1, 0),   # GEMMs of 129 to 256 tokens
    "rows_300": (TWO_KV, "bf16", [1 + i % 40 for i in range(300)], 1, 0),        # ... and of more: activations in rows
    "groups": (RI.TINY_MOE, "bf16", [75, 300, 20], 3, 0),
}
STEPS = 4


def digests(name):
    """[step][row] CRC-32 of the row's logits, and of the step's routing as the last entry."""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s, fmt, lens, members, grid = CASES[name]
    model = synthetic.model_from_shape(s, 3, fmt=fmt.split()[0], activation_split=0 if "one" in fmt else 1)
    if grid:
        model.set_attention_grid(grid)
    rng = np.random.default_rng(21)
    toks = [rng.integers(0, s.vocab - 2, n).astype(np.int32) for n in lens]
    rows = len(lens) * members
    blocks = [(n + STEPS + 31) // 16 for n in lens]
    eng = pkg.RolloutEngine(model, n_blocks=sum(blocks) * members, max_seqs=rows, max_chunk_tokens=sum(lens),
                            max_blocks_per_seq=max(blocks))
    out = []
    for i, t in enumerate(toks):
        lead = eng.add_sequence(50 + i, reserve_tokens=16 * blocks[i])
        eng.prefill([lead], [t[:-1] if len(t) > 1 else t], sample_last=[False])
        for k in range(1, members):
            eng.fork(lead, 90 + 10 * i + k, reserve_tokens=16 * blocks[i])
    for step in range(STEPS):
        eng.tokens[:rows] = torch.tensor(rng.integers(0, s.vocab - 2, rows), dtype=torch.int32, device="cuda:0")
        forced = torch.tensor(rng.integers(0, s.vocab - 2, rows), dtype=torch.int32, device="cuda:0")
        o = eng.decode_step(forced=forced, want_logits=True, want_routing=True)
        z = np.ascontiguousarray(o.logits.cpu().numpy())
        assert np.isfinite(z).all()
        out.append([zlib.crc32(r.tobytes()) for r in z] + [zlib.crc32(o.routing.cpu().numpy().tobytes())])
    model.close()
    return out


@pytest.mark.parametrize("name", sorted(CASES))
def test_moe_decode_steps_have_the_recorded_bits(name):
    with open(GOLDEN) as f:
        want = json.load(f)[name]
    got = digests(name)
    bad = [(s, r) for s in range(STEPS) for r in range(len(want[s])) if got[s][r] != want[s][r]]
    assert not bad, "(step, row) that differ, the last row being the routing: %s" % bad
