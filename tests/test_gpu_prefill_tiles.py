"""Prefill attention takes its query tiles from a list sorted by the keys they walk, and pairs long ones with short ones where all
workgroups are resident at once (257 to 512 of them on 256 units).  Many ragged sequences in one call, with and without cached
keys, against the same sequences one by one."""
import numpy as np
import pytest

import rollout_inputs as RI

pytestmark = pytest.mark.gpu


# tiles x 2 KV heads: a few, 257..512, more; 1100 sequences fill the list's first pass over them more than once
@pytest.mark.parametrize("n_seqs,longest", [(3, 200), (90, 150), (200, 150), (1100, 9)])
def test_ragged_sequences_equal_single_ones(n_seqs, longest):
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_DENSE
    model = synthetic.model_from_shape(s, 5)
    rng = np.random.default_rng(n_seqs)
    lens = rng.integers(1, longest + 1, n_seqs)
    cached = rng.integers(0, longest + 1, n_seqs) * (rng.random(n_seqs) < 0.5)
    toks = [rng.integers(0, s.vocab - 2, c + n).astype(np.int32) for c, n in zip(cached, lens)]
    blocks = [(len(t) + 15) // 16 for t in toks]
    eng = pkg.RolloutEngine(model, n_blocks=sum(blocks), max_seqs=n_seqs, max_chunk_tokens=int(max(lens.sum(), cached.sum())),
                            max_blocks_per_seq=max(blocks))
    for i in range(n_seqs):
        eng.add_sequence(i, reserve_tokens=16 * blocks[i])
    rows = [i for i in range(n_seqs) if cached[i]]
    if rows:
        eng.prefill(rows, [toks[i][:cached[i]] for i in rows], sample_last=[False] * len(rows))
    got = eng.prefill(list(range(n_seqs)), [t[c:] for t, c in zip(toks, cached)], want_logits=True).logits.cpu().numpy()
    worst = 0.0
    for i in rng.permutation(n_seqs)[:25]:
        one = pkg.RolloutEngine(model, n_blocks=blocks[i], max_seqs=1, max_chunk_tokens=len(toks[i]), max_blocks_per_seq=blocks[i])
        one.add_sequence(1, reserve_tokens=16 * blocks[i])
        worst = max(worst, float(np.abs(one.prefill([0], [toks[i]], want_logits=True).logits.cpu().numpy()[0] - got[i]).max()))
    print("%d sequences, %d tokens: %.1e" % (n_seqs, lens.sum(), worst), flush=True)
    model.close()
    # other GEMM forms, so sums in another order, and now and then a cached code's last bit: the bar of long against short calls
    assert worst <= 5e-3
