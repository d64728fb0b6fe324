"""Calls of few tokens: the products make their normalised rows themselves, and the residual stream changes its place with every
addition.  Rows at the edges of the form (float4 slices per thread: up to 3, up to 5; rows that cost more than they save, where the norm
is a kernel of its own; widths that end inside a 32-wide step) go through a chunk of one token each and two decode steps of three
layers, against the oracle under teacher forcing; the log-probabilities, which the last stage takes from the rows that the LM head
left, against the logits; and a scoring call of the same rows, whose final norm reads the residual stream where it ended up."""
import numpy as np
import pytest
import torch

import oracle as O
import rollout_inputs as RI

pytestmark = pytest.mark.gpu

# Per layer the bars of the other short-call tests (largest difference over the logits' root mean square: two bf16 terms keep 16
# bits; a cached value with the neighbouring code moves its row; one fp16 term): the layers' parts add up, and a row's context of
# up to three cached tokens carries theirs.
LAYERS = 3
BAR = {"bf16": 7e-3 * LAYERS, "f16": 1e-2 * LAYERS}
TYPICAL = {"bf16": 1e-4 * LAYERS, "f16": 5e-3 * LAYERS}      # half of the rows, as long as they see no token but their own


# d_model, d_ff, rows (test_short_call_plans.py holds the first ones of each to the form and the last ones to the other): 512 has 128
# slices a row, so 6 rows fill three per thread and 8 four; 5 rows of 1024 and one of 5120 fill five
SHAPES = [(80, 688, (1, 13, 14, 16, 17)), (512, 1024, (1, 6, 7, 8, 9, 10, 11)), (1024, 1024, (4, 5, 6)), (2544, 688, (1, 2, 3)),
          (5120, 688, (1, 2))]


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("d_model,d_ff,rows", SHAPES)
def test_few_tokens_match_the_oracle(d_model, d_ff, rows, fmt):
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_DENSE.replace(n_layers=LAYERS, d_model=d_model, d_ff=d_ff, vocab=264, qk_norm=True)
    model = synthetic.model_from_shape(s, 0, **(dict(fmt="f16", activation_split=0) if fmt == "f16" else {}))
    toks = np.random.default_rng(d_model).integers(0, s.vocab - 2, (3, max(rows))).astype(np.int32)
    ora = O.OracleRollout(O.OracleModel(s, 0, fmt=fmt), n_blocks=max(rows))
    ids = [ora.add_sequence(i) for i in range(max(rows))]
    want = [ora.prefill_chunk(ids, [toks[0, i:i + 1] for i in ids], forced_tokens=[int(t) for t in toks[1]], want_logits=True)]
    for step in (2, 2):
        want.append(ora.decode_step(ids, forced_tokens=[int(t) for t in toks[step]], want_logits=True))
    want = [np.stack(w["logits"]) for w in want]
    for n in rows:
        eng = pkg.RolloutEngine(model, n_blocks=n, max_seqs=n, max_chunk_tokens=n, max_blocks_per_seq=1)
        for i in range(n):
            eng.add_sequence(i, reserve_tokens=16)
        got = [eng.prefill(list(range(n)), [toks[0, i:i + 1] for i in range(n)], forced=[int(t) for t in toks[1, :n]], want_logits=True)]
        for step in (2, 2):
            got.append(eng.decode_step(forced=torch.tensor(toks[step, :n], device="cuda:0"), want_logits=True))
        for k, (g, w) in enumerate(zip(got, want)):
            off = np.sort(np.abs(g.logits[:n].cpu().numpy() - w[:n]).max(axis=1)) / np.sqrt((w * w).mean())
            print("d_model %d %s, %d rows, call %d: %.2e %.2e" % (d_model, fmt, n, k, off[n // 2], off[-1]), flush=True)
            assert off[-1] <= BAR[fmt], (n, k, off)
            if n > 2 and k == 0:
                assert off[n // 2 - 1] <= TYPICAL[fmt], (n, k, off)
            # 1e-5 is what 32-bit sums over the vocabulary and over d_model leave
            z, at = g.logits[:n].cpu().numpy().astype(np.float64), (1, 2, 2)[k]
            lp = z[np.arange(n), toks[at, :n]] - np.log(np.exp(z).sum(axis=1))
            assert np.abs(lp - g.logprobs[:n].cpu().numpy()).max() < 3e-5, (n, k)
        eng = pkg.RolloutEngine(model, n_blocks=n, max_seqs=n, max_chunk_tokens=n, max_blocks_per_seq=1)
        for i in range(n):
            eng.add_sequence(i, reserve_tokens=16)
        lp, _ = eng.score(list(range(n)), [toks[0, i:i + 1] for i in range(n)], [toks[1, i:i + 1] for i in range(n)])
        z = want[0][:n].astype(np.float64)
        lp = lp.cpu().numpy() - (z[np.arange(n), toks[1, :n]] - np.log(np.exp(z).sum(axis=1)))
        # two logits' distances
        assert np.abs(lp).max() <= 2 * BAR[fmt] * np.sqrt((z * z).mean()), (n, lp)
    model.close()
