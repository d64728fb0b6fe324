"""Products of short calls of dense policies: calls of up to 128 tokens deal K to the waves of a workgroup in 32-wide steps, on
16-row weight tiles and 16-token tiles.  One-token sequences at the edges of the token tiles go through one layer whose widths
reach every weight tiling of gate/up (F / 8 row tiles on 256 units: 2, 4, 5, 6 and 8 per workgroup, and the 32-row form past
that) and K with an odd number of 16-wide steps, against the oracle on the same weights."""
import numpy as np
import pytest

import oracle as O
import rollout_inputs as RI

pytestmark = pytest.mark.gpu

TOKENS = (1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 128)
# Largest difference over the logits' root mean square, of nine rows in ten and of every row.  bf16 in two terms keeps 16 bits:
# 2^-17 / sqrt(3) per product, four products in a row, 4.5 sigma: 4e-5.  A row whose cached value got the neighbouring code of an
# element of 3 sigma moves by 2^-8 * 3 / sqrt(256) of its attention's part, times 4.5 sigma: 3.3e-3.  One fp16 term is
# 2^-12 / sqrt(3) off: 1.3e-3, and its codes 2^-11.  Twice to four times that.
BAR = {"bf16": (1e-4, 7e-3), "f16": (5e-3, 1e-2)}


# ... and where the long-call form begins: gate/up in tiles of 160 (9728) and of 192 (11008) weight rows.  (Up to 256 tokens: there
# the norm leaves its factor to the products, as in short calls.  Above, rows are rounded to two terms after it and keys and values
# are sums of fewer planes, so a tenth of the rows and more have a value with the neighbouring code, 2.9e-3 at most: the second
# bar's case, which the first one does not allow for.)
LONG = (129, 200, 256)


@pytest.mark.parametrize("d_model,d_ff", [(528, 9728), (528, 11008), (80, 9744)])
def test_calls_just_above_match_the_oracle(d_model, d_ff):
    _compare(d_model, d_ff, "bf16", LONG)


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("d_model,d_ff", [(256, 688), (80, 4112), (528, 8208), (80, 9728), (80, 10256), (80, 12304), (80, 16400)])
def test_short_calls_match_the_oracle(d_model, d_ff, fmt):
    _compare(d_model, d_ff, fmt, TOKENS)


def _compare(d_model, d_ff, fmt, tokens):
    worst = {n: (float(rows[int(0.9 * (n - 1))]), float(rows[-1])) for n, rows in
             _row_errors(RI.TINY_DENSE.replace(n_layers=1, d_model=d_model, d_ff=d_ff, vocab=264, qk_norm=True), fmt, tokens)}
    assert all(w[0] <= BAR[fmt][0] and w[1] <= BAR[fmt][1] for w in worst.values()), worst


def _row_errors(s, fmt, tokens):
    """(tokens of the call, its rows' largest differences over the root mean square, in ascending order) of every call"""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    kw = dict(fmt="f16", activation_split=0) if fmt == "f16" else {}
    model = synthetic.model_from_shape(s, 0, **kw)
    toks = np.random.default_rng(s.d_ff).integers(0, s.vocab - 2, tokens[-1]).astype(np.int32)
    want = O.forward_full(O.OracleModel(s, 0, fmt=fmt), [toks[i:i + 1] for i in range(len(toks))])
    want = np.stack([w["logits"][-1] for w in want])
    rms = np.sqrt((want * want).mean())
    eng = pkg.RolloutEngine(model, n_blocks=len(toks), max_seqs=len(toks), max_chunk_tokens=len(toks), max_blocks_per_seq=1)
    for i in range(len(toks)):
        eng.add_sequence(i, reserve_tokens=16)
    out = []
    for n in tokens:
        eng.ctx_lens.zero_()
        o = eng.prefill(list(range(n)), [toks[i:i + 1] for i in range(n)], want_logits=True)
        rows = np.sort(np.abs(o.logits[:n].cpu().numpy() - want[:n]).max(axis=1) / rms)
        print("d_model %d d_ff %d %s, %d tokens: %.2e %.2e" % (s.d_model, s.d_ff, fmt, n, rows[int(0.9 * (n - 1))], rows[-1]), flush=True)
        out.append((n, rows))
    model.close()
    return out


# Wide products, whose cuts of the rows and of K the narrow ones above do not reach (test_short_call_plans.py says which they are):
# q|k|v of 6144 rows (384 row tiles, no multiple of five, in three segments) from 159 k-steps of 16 with an output projection to
# 2544 rows (ends inside a tile), of 10 368 rows, of 8320 rows from few columns, and a down projection of 3456 x 4608.
WIDE = {"q_o": RI.TINY_DENSE.replace(n_layers=1, d_model=2544, n_q_heads=32, n_kv_heads=8, head_dim=128, d_ff=688, vocab=264),
        "heads": RI.TINY_DENSE.replace(n_layers=1, d_model=1664, n_q_heads=63, n_kv_heads=9, head_dim=128, d_ff=688, vocab=264),
        "flat": RI.TINY_DENSE.replace(n_layers=1, d_model=272, n_q_heads=104, n_kv_heads=13, head_dim=64, d_ff=688, vocab=264),
        "down": RI.TINY_DENSE.replace(n_layers=1, d_model=3456, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ff=4608, vocab=264)}
WIDE_TOKENS = (1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 128)


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("name", sorted(WIDE))
def test_wide_products_of_short_calls_match_the_oracle(name, fmt):
    s = WIDE[name]
    for n, rows in _row_errors(s, fmt, WIDE_TOKENS):
        # of a row's kv_dim values each gets the neighbouring code with a chance of 1600 in six million; four sigma of the count
        p = 1 - (1 - 1600 / 6e6) ** s.kv_dim
        flipped = n * p + 4 * (n * p * (1 - p)) ** 0.5 + 1
        assert (rows > BAR[fmt][0]).sum() <= flipped and rows[-1] <= BAR[fmt][1], (n, rows)


# rows of LM heads: one token tile (the last of whose rows hold their temperature, seed and position at its very end), and two
# rows more, which take the form that stages the activations
@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("d_model,vocab", [(256, 2056), (272, 35)])
def test_draws_of_few_rows_match_the_oracle(d_model, vocab, fmt):
    """Draws and log-probabilities of 1 to 18 dense rows, each with its own temperature (greedy ones among them) and seed; the
    rows of a call are the first ones of the next, so both forms of the LM head are held to the same oracle on the same rows."""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_DENSE.replace(n_layers=1, d_model=d_model, vocab=vocab)
    model = synthetic.model_from_shape(s, 0, **(dict(fmt="f16", activation_split=0) if fmt == "f16" else {}))
    rng = np.random.default_rng(vocab)
    toks = rng.integers(0, s.vocab - 2, 18).astype(np.int32)
    temps = np.array([0.0, 1.0, 0.5, 1.7, 0.8, 0.0, 1.2, 0.6, 2.0, 1.0, 0.7, 0.5, 1.5, 0.0, 0.9, 1.3, 0.5, 0.0])
    seeds = [int(x) for x in rng.integers(1, 1 << 62, 18)]
    z = np.stack([w["logits"][-1] for w in O.forward_full(O.OracleModel(s, 0, fmt=fmt), [toks[i:i + 1] for i in range(18)])])
    z = z.astype(np.float64)
    # a logit is off by the second bar at most (above), a difference of two logits or of one and the log-sum-exp by twice that
    bar = 2 * BAR[fmt][1] * np.sqrt((z * z).mean())
    eng = pkg.RolloutEngine(model, n_blocks=18, max_seqs=18, max_chunk_tokens=18, max_blocks_per_seq=1)
    for i in range(18):
        eng.add_sequence(seeds[i], temperature=float(temps[i]), reserve_tokens=16)
    drawn = 0
    for n in (1, 10, 11, 12, 15, 16, 17, 18):
        eng.ctx_lens.zero_()
        out = eng.prefill(list(range(n)), [toks[i:i + 1] for i in range(n)], want_sampled=True)
        got, lp = out.sampled.cpu().numpy(), out.logprobs.cpu().numpy()
        for i in range(n):
            t = temps[i] if temps[i] > 0 else 1.0
            score = z[i] / t + (O.gumbel_noise(seeds[i], 1, vocab) if temps[i] > 0 else 0.0)
            want = z[i][got[i]] / t - np.log(np.exp(z[i] / t).sum())
            tag = "%d rows, row %d, temperature %.1f" % (n, i, temps[i])
            assert score[got[i]] >= score.max() - bar / t, tag
            assert abs(float(lp[i]) - want) <= bar / t, tag
            drawn += int(got[i] != int(np.argmax(score)))
    assert drawn <= 4, drawn                     # of 100 draws and 16 greedy picks: scores closer than the bar are rare
    model.close()
