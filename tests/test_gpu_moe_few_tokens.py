"""MoE calls of a few tokens, whose expert products give workgroups only to the experts that have rows: the first and the last
expert, neighbours, gaps longer than a 64-expert word, one expert for all tokens, and as many experts as a call may have, scored
with that routing replayed against the oracle that replays the same."""
import numpy as np
import pytest

import oracle as O
import rollout_inputs as RI

pytestmark = pytest.mark.gpu

# two-term bf16 keeps 16 bits per product and a cached key or value may get the neighbouring code (2^-8 of one element): the
# same bar as scoring in chunks against scoring whole
BAR = 2e-3   # largest seen 2.3e-4


@pytest.mark.parametrize("n_experts,top_k,d_ff_expert", [(256, 3, 208), (128, 8, 96), (70, 2, 64), (3, 2, 96), (1, 1, 32)])
def test_few_tokens_reach_few_experts(n_experts, top_k, d_ff_expert):
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_MOE.replace(n_layers=2, n_experts=n_experts, top_k=top_k, d_ff_expert=d_ff_expert, vocab=264)
    model, omodel = synthetic.model_from_shape(s, 0), O.OracleModel(s, 0)
    rng = np.random.default_rng(n_experts)
    for n in (1, 2, 5, 17):
        toks = rng.integers(0, s.vocab - 2, n).astype(np.int32)
        targets = np.roll(toks, -1)
        ends = np.concatenate([np.arange(top_k // 2), np.arange(n_experts - (top_k - top_k // 2), n_experts)])
        sets = {"first": np.arange(top_k), "last": np.arange(n_experts - top_k, n_experts), "ends": ends}
        routes = {k: np.broadcast_to(v, (n, s.n_layers, top_k)) for k, v in sets.items()}
        routes["any"] = np.argsort(rng.random((n, s.n_layers, n_experts)), axis=-1)[..., :top_k]
        for name, r in routes.items():
            r = np.ascontiguousarray(r, dtype=np.int32)
            eng = pkg.RolloutEngine(model, n_blocks=4, max_seqs=1, max_chunk_tokens=32, max_blocks_per_seq=4)
            eng.add_sequence(1, reserve_tokens=32)
            lp, got = eng.score([0], [toks], [targets], replay_routing=[r], want_routing=True)
            z = O.forward_full(omodel, [toks], forced_routing=[r])[0]["logits"].astype(np.float64)
            z -= z.max(axis=1, keepdims=True)
            want = z[np.arange(n), targets] - np.log(np.exp(z).sum(axis=1))
            d = float(np.abs(lp.cpu().numpy() - want).max())
            print("%d experts, %d tokens, %s: %.1e" % (n_experts, n, name, d), flush=True)
            assert d <= BAR
            np.testing.assert_array_equal(got.cpu().numpy().reshape(r.shape), r)
    model.close()


@pytest.mark.parametrize("n", [1, 2, 5, 33, 300])
def test_rows_that_are_not_numbers_stay_with_themselves(n):
    """Injected embeddings that are NaN, in every row or in one: their router logits are NaN, their experts the first ones, their
    logits NaN; the other rows are what they are beside an ordinary row, and so is the next call."""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_MOE.replace(n_layers=2, vocab=264)
    model = synthetic.model_from_shape(s, 0)
    eng = pkg.RolloutEngine(model, n_blocks=n, max_seqs=n, max_chunk_tokens=n, max_blocks_per_seq=1)
    for i in range(n):
        eng.add_sequence(i, reserve_tokens=16)
    toks = np.random.default_rng(n).integers(0, s.vocab - 2, (n, 1)).astype(np.int32)

    def call(nan_rows):
        eng.ctx_lens.zero_()
        eng.kv_pool.zero_()
        t, e = toks.copy(), [None] * n
        for i in nan_rows:
            t[i] = -1
            e[i] = np.full((1, s.d_model), 0x7FC0, np.uint16)
        out = eng.prefill(list(range(n)), list(t), e, forced=[5] * n, want_logits=True, want_routing=True)
        return out.logits.cpu().numpy(), out.routing.cpu().numpy()

    want, routing = call([])
    for nan_rows in (range(n), [n // 2]):
        got, routed = call(nan_rows)
        for i in range(n):
            if i in nan_rows:
                assert np.isnan(got[i]).all()
                np.testing.assert_array_equal(routed[i], np.broadcast_to(np.arange(s.top_k), routed[i].shape))
            else:
                np.testing.assert_array_equal(got[i], want[i])
                np.testing.assert_array_equal(routed[i], routing[i])
    again, routed = call([])
    np.testing.assert_array_equal(again, want)
    np.testing.assert_array_equal(routed, routing)
    model.close()


@pytest.mark.parametrize("n_experts", [32, 200])
def test_experts_whose_logits_are_not_numbers_come_last(n_experts):
    """Three router rows are numbers, fewer than a token has experts: those come first, by their logits, then the smallest ids of
    the others, whose weight is zero."""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_MOE.replace(n_layers=1, n_experts=n_experts, vocab=264)
    numbers = [5, 9, n_experts - 1]

    def tensor(layer, name):
        t = RI.tensor_bits(s, 0, layer, name)
        if name == "w_router":
            keep = t[numbers].copy()
            t = np.full_like(t, 0x7FC0)
            t[numbers] = keep
        return t

    model = pkg.RolloutModel(synthetic.config_from_shape(s), tensor)
    rest = [e for e in range(n_experts) if e not in numbers][:s.top_k - 3]
    for n in (1, 7, 40, 300):
        eng = pkg.RolloutEngine(model, n_blocks=n, max_seqs=n, max_chunk_tokens=n, max_blocks_per_seq=1)
        for i in range(n):
            eng.add_sequence(i, reserve_tokens=16)
        toks = np.random.default_rng(n).integers(0, s.vocab - 2, (n, 1)).astype(np.int32)
        out = eng.prefill(list(range(n)), list(toks), forced=[5] * n, want_logits=True, want_routing=True)
        routed = out.routing.cpu().numpy()[:, 0]
        np.testing.assert_array_equal(np.sort(routed[:, :3]), np.broadcast_to(numbers, (n, 3)))
        np.testing.assert_array_equal(routed[:, 3:], np.broadcast_to(rest, (n, s.top_k - 3)))
        assert np.isfinite(out.logits.cpu().numpy()).all()
    model.close()
