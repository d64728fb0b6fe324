"""Shared-prefix tiles where their list is walked more than once, where a tile has more units than a window of its block-table
entries, and where several tiles read the same pages: logits against decode steps that attend every row's pages by itself."""
import numpy as np
import pytest
import torch

import rollout_inputs as RI

pytestmark = pytest.mark.gpu


# groups, members, pages of the shared prefix (16 positions each) per group in turn: 260 groups x 2 KV heads are 520 tiles of one
# chunk, more than the 512 workgroups, of 35 and of 3 units; 70 groups: chunks of up to a quarter of 40 units; 9 members of a
# head group of four, 20 of one of two: more than a tile's columns; 290 pages: chunks of 37 units; 257 groups: more tiles than workgroups
# at one chunk each, and prefixes of 65 units in four chunks among others of three; the last two: more pages than are copied without the
# streaming mark (both layers' 344 and 281 MB)
@pytest.mark.parametrize("heads,groups,members,pages,fmt", [((4, 2, 64), 260, 2, (70, 7), "bf16"), ((4, 2, 64), 70, 3, (80, 33, 5), "f16"),
                                                            ((4, 1, 128), 3, 9, (21, 40), "bf16"), ((4, 2, 128), 2, 20, (9, 66), "f16"),
                                                            ((16, 1, 64), 2, 3, (290, 18), "bf16"),
                                                            ((4, 2, 64), 257, 4, (6,) * 64 + (130,), "bf16"),
                                                            ((4, 2, 64), 300, 2, (70,), "bf16"), ((4, 2, 128), 130, 2, (66,), "f16")])
def test_prefix_tiles_match_attention_by_row(heads, groups, members, pages, fmt):
    import paper_2604_11554_amd as pkg
    from paper_2604_11554_amd import synthetic

    s = RI.TINY_DENSE.replace(n_layers=2, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=heads[2], vocab=264, qk_norm=True)
    model = synthetic.model_from_shape(s, 0, **(dict(fmt="f16", activation_split=0) if fmt == "f16" else {}))
    n, widest = groups * members, max(pages) + 2
    eng = pkg.RolloutEngine(model, n_blocks=groups * (max(pages) + 1) + 2 * n, max_seqs=n, max_chunk_tokens=n, max_blocks_per_seq=widest)
    ctx = []
    for i in range(n):
        p = pages[i // members % len(pages)]
        if i % members == 0:
            eng.add_sequence(i, reserve_tokens=16 * (p + 1))
            eng.ctx_lens[i] = 16 * p + 1
        else:
            eng.fork(i - i % members, i, reserve_tokens=16 * (p + 1))
        ctx.append(16 * p + 1 + i % 9)
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    eng.kv_pool.view(torch.float16 if fmt == "f16" else torch.bfloat16).normal_(generator=gen)
    toks = torch.tensor(np.random.default_rng(2).integers(0, s.vocab - 2, n), dtype=torch.int32, device="cuda:0")
    lens, pool, got = torch.tensor(ctx, dtype=torch.int32, device="cuda:0"), eng.kv_pool.clone(), []
    desc = eng._shared_prefix()
    assert desc is not None and int(desc[:8].view(torch.int32)[1].item()) > 0
    for shared in (True, False):
        eng.share_prefix_attention = shared
        eng.kv_pool.copy_(pool)
        eng.ctx_lens.copy_(lens)
        eng.tokens[:n] = toks
        eng.finished.zero_()
        got.append(eng.decode_step(forced=toks, want_logits=True).logits[:n].cpu().numpy())
    model.close()
    # the merges of the softmax add in another order: 1e-7 of a sum each, and in the second layer, here and there, the other
    # 16-bit code of a cached element or (fp16) of an activation; logits of about unit variance
    assert np.isfinite(got[0]).all()
    assert np.abs(got[0] - got[1]).max() <= (2e-3 if fmt == "bf16" else 1e-2), float(np.abs(got[0] - got[1]).max())
