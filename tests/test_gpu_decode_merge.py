"""Decode attention merges the parts of a (sequence, KV head) pair with four threads per output where a call has few
pairs and with two where it has many (512 pairs and up).  One long sequence, cut into dozens of parts, is decoded alone, among
hundreds of short ones and among hundreds of finished ones; pairs of equal length are cut by several grids."""
import numpy as np
import pytest
import torch

import rollout_inputs as RI

pytestmark = pytest.mark.gpu

HEADS = {64: RI.TINY_DENSE, 128: RI.TINY_DENSE.replace(head_dim=128, n_q_heads=4, n_kv_heads=1)}


@pytest.mark.parametrize("head_dim", sorted(HEADS))
@pytest.mark.parametrize("others", ["short", "finished"])
@pytest.mark.parametrize("keys", [40, 1023, 3000])
def test_a_long_sequence_among_many_others(keys, others, head_dim):
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = HEADS[head_dim]
    n = (512 + s.n_kv_heads - 1) // s.n_kv_heads
    model = synthetic.model_from_shape(s, 3)
    long = np.random.default_rng(5).integers(0, s.vocab - 2, keys).astype(np.int32)
    logits = []
    for short in (0, n - 1):
        toks = [long] + [long[:1 + i % 3] for i in range(short)]
        rows = list(range(len(toks)))
        blocks = [(t.size + 2 + 15) // 16 for t in toks]
        eng = pkg.RolloutEngine(model, n_blocks=sum(blocks), max_seqs=len(toks), max_chunk_tokens=keys + 3 * len(toks),
                                max_blocks_per_seq=max(blocks))
        for i in rows:
            eng.add_sequence(i, reserve_tokens=16 * blocks[i])
        eng.prefill([0], [long], forced=[int(long[0])])
        if short:
            eng.prefill(rows[1:], toks[1:], forced=[int(long[0])] * short)
        if others == "finished":
            eng.finished[1:len(toks)] = 1
        out = eng.decode_step(forced=torch.full((len(toks),), int(long[0]), dtype=torch.int32, device="cuda"), want_logits=True)
        logits.append(out.logits.cpu().numpy())
    # the same products; sums in another grouping (other GEMM forms and parts) flip the last bit of a few bf16 keys and
    # values (2^-9 of an element) of unit-variance logits: the bar of the calls compared form against form
    assert np.isfinite(logits[1][:1 if others == "finished" else None]).all()
    d = np.abs(logits[0][0] - logits[1][0]).max()
    assert d < 5e-3, d
    model.close()


@pytest.mark.parametrize("head_dim", sorted(HEADS))
@pytest.mark.parametrize("keys", [97, 130, 2200])
def test_pairs_that_are_exactly_a_workgroup(keys, head_dim):
    """With as many workgroups as pairs and equal contexts every pair is cut into as many shares as a workgroup has waves;
    other grids cut the same pairs elsewhere, or not at all."""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s, n = HEADS[head_dim], 3
    model = synthetic.model_from_shape(s, 3)
    rng = np.random.default_rng(6)
    toks = [rng.integers(0, s.vocab - 2, keys - 1).astype(np.int32) for _ in range(n)]
    logits = []
    for grid in (n * s.n_kv_heads, n * s.n_kv_heads + 1, 1, 512):
        model.set_attention_grid(grid)
        blocks = (keys + 17) // 16
        eng = pkg.RolloutEngine(model, n_blocks=n * blocks, max_seqs=n, max_chunk_tokens=n * keys, max_blocks_per_seq=blocks)
        for i in range(n):
            eng.add_sequence(i, reserve_tokens=16 * blocks)
        eng.prefill(list(range(n)), toks, forced=[1] * n)
        out = eng.decode_step(forced=torch.ones(n, dtype=torch.int32, device="cuda"), want_logits=True)
        logits.append(out.logits.cpu().numpy())
    # one layer's sums in another grouping: as above
    assert np.isfinite(logits[0]).all()
    assert max(np.abs(z - logits[0]).max() for z in logits[1:]) < 5e-3
    model.close()


@pytest.mark.parametrize("shape", ["tiny_dense", "tiny_moe"])
def test_groups_of_equal_own_length_on_any_grid(shape):
    """Members of a sampling group whose own keys are equally many: the grid decides whether a pair lies in one share (its
    own part then goes beside the prefix chunks) or in several.  Every grid equals plain attention without the descriptor."""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = {"tiny_dense": RI.TINY_DENSE, "tiny_moe": RI.TINY_MOE}[shape]
    model = synthetic.model_from_shape(s, 3)
    rng = np.random.default_rng(8)
    prompt = rng.integers(0, s.vocab - 2, 200).astype(np.int32)
    own = [rng.integers(0, s.vocab - 2, 130).astype(np.int32) for _ in range(3)]
    logits = []
    for grid, share in ((512, False), (1, True), (3, True), (3 * s.n_kv_heads, True), (12 * s.n_kv_heads, True), (512, True)):
        model.set_attention_grid(grid)
        eng = pkg.RolloutEngine(model, n_blocks=120, max_seqs=3, max_chunk_tokens=512, max_blocks_per_seq=24)
        eng.share_prefix_attention = share
        lead = eng.add_sequence(1, reserve_tokens=340)
        eng.prefill([lead], [prompt], sample_last=[False])
        rows = [lead] + [eng.fork(lead, 2 + i, reserve_tokens=340) for i in range(2)]
        eng.prefill(rows, own, forced=[5] * 3)
        out = eng.decode_step(forced=torch.full((3,), 7, dtype=torch.int32, device="cuda"), want_logits=True)
        logits.append(out.logits.cpu().numpy())
    # one step's sums in another grouping, as above
    assert np.isfinite(logits[0]).all()
    assert max(np.abs(z - logits[0]).max() for z in logits[1:]) < 5e-3
    assert any(not np.array_equal(z, logits[0]) for z in logits[1:])     # the descriptor was used
    model.close()
