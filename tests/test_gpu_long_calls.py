"""Long calls take GEMM forms of their own (activations in rows, tiles of 128 or 64 tokens, K cut into planes where the tiles
leave the device idle): the layers' products from 129 tokens on in dense policies and from 257 in MoE ones, LM heads and
scoring from 65 rows on.  They are compared with the same tokens handed over in calls of at most 64, all of whose products
take the short forms: the same products, sums in another grouping."""
import numpy as np
import pytest

import rollout_inputs as RI

pytestmark = pytest.mark.gpu

# widths at the edges of the tiles: K = 688 and 2064 have an odd number of 16-wide k-steps, N = 2056 / 24 experts and the
# vocabulary are no multiple of a weight tile, 2064 is long enough to be cut into planes
SHAPES = {
    "tiny_dense": RI.TINY_DENSE,
    "wide_dense": RI.TINY_DENSE.replace(d_model=528, d_ff=2064, vocab=2056, n_q_heads=8, n_kv_heads=1, qk_norm=True),
    "tiny_moe": RI.TINY_MOE.replace(n_experts=24, vocab=2056),
}
# tokens of every sequence: just past the limits, around the 64- and 128-token tiles, a few hundred ragged ones
LENGTHS = {"129": [129], "130": [2, 128], "257": [257], "320": [64, 1, 255], "385": [129, 256], "ragged": [256, 31, 200, 97, 1, 250, 255, 118]}


@pytest.mark.parametrize("lengths", sorted(LENGTHS))
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_long_calls_equal_the_same_tokens_in_short_calls(name, lengths):
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = SHAPES[name]
    lens = LENGTHS[lengths]
    model = synthetic.model_from_shape(s, 3)
    rng = np.random.default_rng(11)
    toks = [rng.integers(0, s.vocab - 2, n).astype(np.int32) for n in lens]
    rows = list(range(len(lens)))
    blocks = [(n + 31) // 16 for n in lens]

    def engine():
        eng = pkg.RolloutEngine(model, n_blocks=sum(blocks), max_seqs=len(lens), max_chunk_tokens=sum(lens),
                                max_blocks_per_seq=max(blocks))
        for i in rows:
            eng.add_sequence(i, reserve_tokens=16 * blocks[i])
        return eng

    long_eng, short_eng = engine(), engine()
    out = long_eng.prefill(rows, toks, want_logits=True, want_routing=True)
    lp, _ = (lambda e: e.score(rows, toks, [np.roll(t, -1) for t in toks]))(engine())
    replay = out.routing.cpu().numpy() if s.is_moe else None
    offs = np.concatenate([[0], np.cumsum(lens)])
    logits, lp_short = [], []
    scorer = engine()
    for i in rows:                               # one sequence per call, at most 64 tokens at a time
        for a in range(0, len(toks[i]), 64):
            b = min(a + 64, len(toks[i]))
            o = short_eng.prefill([i], [toks[i][a:b]], want_logits=True)
            scored, _ = scorer.score([i], [toks[i][a:b]], [np.roll(toks[i], -1)[a:b]],
                                     replay_routing=None if replay is None else [replay[offs[i] + a:offs[i] + b]])
            lp_short.append(scored.cpu().numpy())
        logits.append(o.logits.cpu().numpy()[0])
    dz = np.abs(out.logits.cpu().numpy() - np.stack(logits)).max()
    dlp = np.abs(lp.cpu().numpy() - np.concatenate(lp_short)).max()
    # Both sides hold activations to 16 significand bits and round the same keys and values to bf16; sums in another
    # order (1e-7 relative each) flip the last bit of a few of those (2^-9 of an element).  Logits have unit variance:
    # the short forms are within 5e-4 of the oracle here, the bar of the project is 0.05.
    assert dz < 5e-3, dz
    assert dlp < 5e-3, dlp
    model.close()


@pytest.mark.parametrize("vocab,d_model", [(2048, 256), (2056, 256), (35, 256), (2056, 272)])
@pytest.mark.parametrize("n_rows", [65, 128, 130, 257])
def test_lm_heads_of_many_rows_draw_what_short_ones_draw(n_rows, vocab, d_model):
    """More than 64 sampled rows take the long-call LM head (records of 64 ids, rows of activations): same draws and
    log-probabilities as calls of at most 64 rows; 2056 and 35 ids end inside a tile, 272 has an odd number of k-steps: the
    last one is read from LDS right before the epilogue takes the stage buffers."""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_DENSE.replace(vocab=vocab, d_model=d_model)
    model = synthetic.model_from_shape(s, 5)
    toks = [np.array([i % (vocab - 2)], np.int32) for i in range(n_rows)]
    sampled, logprobs = [], []
    for step in (n_rows, 64):
        got = []
        for a in range(0, n_rows, step):
            part = toks[a:a + step]
            eng = pkg.RolloutEngine(model, n_blocks=len(part), max_seqs=len(part), max_chunk_tokens=len(part),
                                    max_blocks_per_seq=1)
            for j in range(len(part)):
                eng.add_sequence(7000 + a + j, temperature=0.7 if (a + j) % 3 else 0.0, reserve_tokens=16)
            out = eng.prefill(list(range(len(part))), part, want_sampled=True)
            got.append((out.sampled.cpu().numpy(), out.logprobs.cpu().numpy()))
        sampled.append(np.concatenate([g[0] for g in got]))
        logprobs.append(np.concatenate([g[1] for g in got]))
    # the logits differ by the order of their sums only (~1e-6): a draw may differ where two scores are that close
    same = sampled[0] == sampled[1]
    assert same.mean() >= 0.99, np.nonzero(~same)
    # log-probabilities of unit-variance logits: 1e-6 of the sums, and up to one flipped last bit of a cached key
    assert np.abs(logprobs[0] - logprobs[1])[same].max() < 1e-3
    model.close()


@pytest.mark.parametrize("head_dim", [64, 128])
def test_values_of_tokens_at_any_slot_are_appended_alike(head_dim):
    """Calls above 1024 tokens store the values of four tokens in neighbouring slots of a page together, of two, or one
    by one: sequences that begin at every slot remainder, in one call of 1222 tokens and in two of fewer."""
    import torch

    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_DENSE.replace(name="tiny_rope", n_q_heads=2 * 64 // head_dim, n_kv_heads=1, head_dim=head_dim, qk_norm=True)
    before, lens = [0, 1, 2, 3, 5, 16, 17, 30], [301, 1, 2, 3, 258, 7, 350, 300]
    rng = np.random.default_rng(4)
    toks = [rng.integers(0, s.vocab - 2, b + n).astype(np.int32) for b, n in zip(before, lens)]
    model = synthetic.model_from_shape(s, 3)
    pools = []
    for calls in ([range(8)], [range(5), range(5, 8)]):
        eng = pkg.RolloutEngine(model, n_blocks=192, max_seqs=8, max_chunk_tokens=2048, max_blocks_per_seq=32)
        for i in range(8):
            eng.add_sequence(i, reserve_tokens=16 * 20 + 64)
        for i in range(1, 8):
            eng.prefill([i], [toks[i][:before[i]]], sample_last=[False])
        for rows in calls:
            eng.prefill(list(rows), [toks[i][before[i]:] for i in rows], sample_last=[False] * len(rows))
        torch.cuda.synchronize()
        pools.append(eng.kv_pool.view(torch.int16).cpu().numpy().copy())
    layer0 = 192 * 2 * 16 * head_dim             # the first layer's inputs are the same bits in both
    assert (pools[0][:layer0] != 0).sum() >= sum(map(len, toks)) * head_dim
    assert np.array_equal(pools[0][:layer0], pools[1][:layer0])
    model.close()


def test_values_of_calls_of_129_to_256_tokens_are_as_exact_as_those_of_short_calls():
    """Values are rounded to 16 bits as q|k|v leaves them, so its sums decide how many of them get the neighbouring code.
    Against a product in 64 bits: a call of 256 tokens may have no more such codes than the same tokens in calls of 64,
    which cut K finer than time alone would ask of the longer call (half a million values per call, twelve calls)."""
    import torch

    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_DENSE.replace(n_layers=1, d_model=2560, n_q_heads=16, n_kv_heads=16, head_dim=128, d_ff=16, vocab=2048)
    tensor = synthetic.device_random_tensor(s, 3)
    model = synthetic.device_random_model(s, 3)
    f64 = torch.float64
    h = tensor(-1, "embed").to(f64)
    x = h / torch.sqrt((h * h).mean(-1, keepdim=True) + s.rms_eps) * tensor(0, "attn_norm").to(f64)
    want = (x @ tensor(0, "wv").to(f64).t()).to(torch.bfloat16)
    n, off = 256, {256: 0, 64: 0}
    for call in range(12):
        toks = np.random.default_rng(call).choice(s.vocab - 2, n, replace=False).astype(np.int32)
        for per in off:
            eng = pkg.RolloutEngine(model, n_blocks=n, max_seqs=n, max_chunk_tokens=n, max_blocks_per_seq=1)
            for i in range(n):
                eng.add_sequence(i, reserve_tokens=1)
            for a in range(0, n, per):
                eng.prefill(list(range(a, a + per)), [toks[i:i + 1] for i in range(a, a + per)], sample_last=[False] * per)
            pages = eng.kv_pool.view(torch.bfloat16).view(n, s.n_kv_heads, 2, 16 * s.head_dim)
            got = pages[eng.block_table[:n, 0].long(), :, 1].view(n, s.kv_dim, 16)[:, :, 0]
            ref = want[torch.from_numpy(toks).long().to(got.device)]
            assert bool(((got.float() - ref.float()).abs() <= 2.0 ** -7 * ref.float().abs() + 1e-5).all())
            off[per] += int((got != ref).sum())
    # of six million values about 1500 each; the square root is the scatter of the count.  (In two ranges of K instead of four:
    # a quarter more.)
    print("codes off", off)
    assert off[64] > 500, off
    assert off[256] <= 1.05 * off[64] + 3 * off[64] ** 0.5, off
    model.close()
