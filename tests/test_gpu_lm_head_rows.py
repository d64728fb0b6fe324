"""LM heads of 65 to 256 rows: draws and log-probabilities against the logits that come with them, and those against calls of at most 64
rows, whose LM head has the short form.  Small vocabularies take tiles of 128 x 128; tiles of 320 vocabulary rows by 128 or 256
tokens take over where their rounds fit the vocabulary better (test_lm_head_plan.py holds these calls to it)."""
import numpy as np
import pytest

import rollout_inputs as RI

pytestmark = pytest.mark.gpu


def _engine(pkg, model, n, lens):
    blocks = [(x + 31) // 16 for x in lens]
    eng = pkg.RolloutEngine(model, n_blocks=sum(blocks), max_seqs=n, max_chunk_tokens=sum(lens), max_blocks_per_seq=max(blocks))
    for i in range(n):
        eng.add_sequence(7000 + i, temperature=0.7 if i % 3 else 0.0, reserve_tokens=16 * blocks[i])
    return eng


# the last tile of 128 ids, two waves of 64: 353 = 2 x 128 + 64 + 33, one id past a weight tile in the second wave; 705 = 5 x 128 + 65: the
# second wave has one id; 161 = 128 + 33: it has none, and the first one's second weight tile one
@pytest.mark.parametrize("vocab,d_model", [(353, 80), (705, 48), (161, 272)])
@pytest.mark.parametrize("n_rows", [96, 200, 256])
def test_draws_of_65_to_256_rows(n_rows, vocab, d_model):
    _draws(n_rows, vocab, d_model, 1)


# rows, vocabulary, d_model; 81 793 = 255 x 320 + 160 + 33: the last tile's second wave has one id past a weight tile; 81 665 = 255 x 320 +
# 65: the second wave has none, the first one's third weight tile one; d_model 272 ends inside a stage
WIDE_TILES = [(96, 81793, 272), (128, 81665, 272), (129, 81665, 272), (256, 81793, 272)]


@pytest.mark.parametrize("n_rows,vocab,d_model", WIDE_TILES)
def test_draws_in_tiles_of_320(n_rows, vocab, d_model):
    _draws(n_rows, vocab, d_model, 7)


def _draws(n_rows, vocab, d_model, every):
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    model = synthetic.model_from_shape(RI.TINY_DENSE.replace(vocab=vocab, d_model=d_model), 5)
    toks = [np.array([i % (vocab - 2)], np.int32) for i in range(n_rows)]
    out = _engine(pkg, model, n_rows, [1] * n_rows).prefill(list(range(n_rows)), toks, want_sampled=True, want_logits=True)
    z, drawn, lp = (x.cpu().numpy() for x in (out.logits, out.sampled, out.logprobs))
    from oracle import gumbel_noise
    for i in sorted({*range(0, n_rows, every), n_rows - 1}):
        t = 0.7 if i % 3 else 1.0
        row = z[i].astype(np.float64) / t
        score = row + (gumbel_noise(7000 + i, 1, vocab) if i % 3 else 0.0)
        # 1e-5 is the error of the kernel's noise, 1e-5 that of 32-bit sums over the vocabulary
        assert score.max() - score[drawn[i]] < 3e-5, i
        assert abs(row[drawn[i]] - np.log(np.exp(row - row.max()).sum()) - row.max() - lp[i]) < 3e-5, i
    eng = _engine(pkg, model, n_rows, [1] * n_rows)
    for a in range(0, n_rows, 64):
        rows = list(range(a, min(a + 64, n_rows)))
        short = eng.prefill(rows, [toks[i] for i in rows], want_logits=True).logits.cpu().numpy()
        # sums in another order (1e-7 relative each) flip the last bit of a cached key or value here and there, logits of unit variance
        assert np.abs(short - z[rows]).max() < 5e-3
    model.close()
