"""What rlx_workspace_bytes promises (every smaller call fits, and writes nothing past it) and what the fixed array of
rollout_decode_step_static holds."""
import numpy as np
import pytest
import torch

import rollout_inputs as RI

pytestmark = pytest.mark.gpu

GUARD = 0xA5


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("shape", ["tiny_dense", "tiny_moe"])
@pytest.mark.parametrize("max_tokens,total", [(300, 256), (300, 129), (300, 40), (2000, 256), (2000, 257), (2000, 1999)])
def test_a_chunk_with_empty_sequences_fits_the_workspace(max_tokens, total, shape, fmt):
    """300 rows of which some bring no token: the number of rows is above the 256 tokens up to which a call cuts its sums
    sixteen ways, the number of tokens is not.  The same tokens without the empty rows give the same outputs."""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import binding as B
    from paper_2604_11554_amd import synthetic

    s = {"tiny_dense": RI.TINY_DENSE, "tiny_moe": RI.TINY_MOE}[shape]
    model = synthetic.model_from_shape(s, 3, fmt=fmt)
    rng = np.random.default_rng(total)
    lens = [0] * 300
    full = rng.permutation(300)[:min(total, 210)]
    for i in full:
        lens[i] = 1
    lens[full[0]] += total - sum(lens)
    toks = [rng.integers(0, s.vocab - 2, n).astype(np.int32) for n in lens]
    got = []
    for rows in (list(range(300)), sorted(int(i) for i in full)):
        eng = pkg.RolloutEngine(model, n_blocks=300 + max(lens) // 16 + 2, max_seqs=len(rows), max_chunk_tokens=max_tokens,
                                max_blocks_per_seq=max(lens) // 16 + 2)
        size = B.rlx_workspace_bytes(model.handle, len(rows), max_tokens, eng.max_blocks)
        buf = torch.full((size + 65536,), GUARD, dtype=torch.uint8, device="cuda:0")
        eng.workspace = buf[:size]
        for i in rows:
            eng.add_sequence(i, reserve_tokens=max(lens[i], 1))
        n = len(rows)
        out = eng.prefill(list(range(n)), [toks[i] for i in rows], forced=[5] * n, want_logits=True)
        assert bool((buf[size:] == GUARD).all()), "written past the workspace"
        keep = [j for j, i in enumerate(rows) if lens[i]]
        got.append((out.logits.cpu().numpy()[keep], out.logprobs.cpu().numpy()[keep]))
    # the same GEMM forms on the same tokens; the LM head may take other tiles for 300 rows than for 210, whose sums have
    # the same order
    assert np.isfinite(got[0][0]).all()
    assert np.abs(got[0][0] - got[1][0]).max() <= 1e-5 and np.abs(got[0][1] - got[1][1]).max() <= 1e-5
    model.close()


def test_the_workspace_grows_with_the_call():
    from paper_2604_11554_amd import binding as B
    from paper_2604_11554_amd import synthetic

    for s, kw in ((RI.TINY_DENSE, {}), (RI.TINY_MOE, {}), (RI.TINY_DENSE, {"fmt": "f16"}), (RI.TINY_MOE, {"activation_split": 0})):
        model = synthetic.device_random_model(s, **kw)
        tokens = [1, 64, 65, 128, 129, 255, 256, 257, 300, 511, 1023, 1024, 1025, 2047, 2049, 8191, 8193, 20000]
        seqs = [1, 7, 64, 65, 128, 129, 256, 257, 300, 1024, 2000]
        need = {(a, t): B.rlx_workspace_bytes(model.handle, a, t, 64) for a in seqs for t in tokens if a <= t}
        for (a, t), n in need.items():
            assert all(m <= n for (b, u), m in need.items() if b <= a and u <= t), (s.name, kw, a, t)
        model.close()


# shapes and the most sequences that a step on the fixed array took at commit 9132d03
FIXED = {"tiny_wide_head": (RI.TINY_DENSE.replace(vocab=151936), 1246),
         "mid_dense": (RI.TINY_DENSE.replace(d_model=1040, d_ff=2736, n_q_heads=16, n_kv_heads=4, vocab=32000), 1295),
         "mid_moe": (RI.TINY_MOE.replace(vocab=32000, d_model=1024, d_ff_expert=400), 1292),
         "hd128": (RI.TINY_DENSE.replace(head_dim=128, n_q_heads=16, n_kv_heads=1, vocab=8000, d_model=528), 1696)}


def _fits(B, model, n):
    """Without arrays a step that fits is refused for them, one that does not for its size: nothing runs either way."""
    with pytest.raises(B.RlxError) as e:
        B.rollout_decode_step_static(model.handle, None, 1, n, None, None, None, 8, None, None, None, None, None, None)
    assert e.value.code in (B.RLX_EINVAL, B.RLX_ENOMEM)
    return e.value.code == B.RLX_EINVAL


# ... and at commit 98e1273, whose plans of a step's attention were smaller than a share's record is now
@pytest.mark.parametrize("shape,kw,took", [
    (RI.TINY_DENSE, {}, 4212), (RI.TINY_DENSE, {"fmt": "f16"}, 4905), (RI.TINY_MOE, {}, 3904),
    (RI.TINY_MOE, {"activation_split": 0}, 4488), (RI.TINY_DENSE.replace(vocab=35, d_model=128), {}, 4659),
    (FIXED["mid_dense"][0], {}, 1427), (FIXED["mid_moe"][0], {"fmt": "f16"}, 1604), (FIXED["hd128"][0], {}, 1850)])
def test_the_fixed_array_takes_what_it_took(shape, kw, took):
    from paper_2604_11554_amd import binding as B
    from paper_2604_11554_amd import synthetic

    model = synthetic.device_random_model(shape, **kw)
    assert all(_fits(B, model, n) for n in (1, 171, 172, 256, 257, took // 2, took - 1, took))
    assert not _fits(B, model, took + 200)
    model.close()


@pytest.mark.parametrize("name", sorted(FIXED))
def test_the_largest_step_on_the_fixed_array(name):
    """What the fixed array took it still takes, and the largest step that it takes today equals the step on a workspace."""
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import binding as B
    from paper_2604_11554_amd import synthetic

    s, took = FIXED[name]
    model = synthetic.device_random_model(s)
    assert all(_fits(B, model, n) for n in (1, 128, 129, 256, 257, 258, 300, took // 2, took - 1, took))
    n = next(n for n in range(2 * took, took - 1, -1) if _fits(B, model, n))
    eng = pkg.RolloutEngine(model, n_blocks=n, max_seqs=n, max_chunk_tokens=n, max_blocks_per_seq=1)
    for i in range(n):
        eng.add_sequence(i, reserve_tokens=16)
    toks = np.random.default_rng(9).integers(0, s.vocab - 2, n).astype(np.int32)
    eng.prefill(list(range(n)), [toks[i:i + 1] for i in range(n)], sample_last=[False] * n)
    state = [eng.tokens, eng.ctx_lens, eng.finished, eng.kv_pool]
    eng.tokens[:n] = torch.from_numpy(toks).to("cuda:0")
    before = [t.clone() for t in state]
    forced = torch.from_numpy(np.roll(toks, 1).copy()).to("cuda:0")
    got = []
    for static in (False, True):
        for t, b in zip(state, before):
            t.copy_(b)
        lp = torch.empty(n, dtype=torch.float32, device="cuda:0")
        args = (n, eng.tokens, eng.ctx_lens, eng.block_table, eng.max_blocks, eng.seeds, eng.temperature, eng.max_ctx,
                eng.finished, forced, lp)
        if static:
            B.rollout_decode_step_static(model.handle, eng.kv_pool, eng.n_blocks, *args)
        else:
            B.rollout_decode_step(model.handle, eng.kv_pool, eng.n_blocks, eng.workspace, *args)
        torch.cuda.synchronize()
        got.append(lp.cpu().numpy())
    # dense: fewer K planes, so sums in another order (1e-7 relative each) and here and there a cached code's last bit;
    # log-probabilities of unit-variance logits as in the calls compared form against form
    assert np.isfinite(got[1]).all()
    assert np.abs(got[0] - got[1]).max() < (0 if s.is_moe else 5e-3) + 1e-12
    model.close()
