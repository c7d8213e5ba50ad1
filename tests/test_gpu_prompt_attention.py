"""Prompt attention where one row's maximum moves late and its tile's other rows stand still (run with -m gpu)."""
import pytest
import torch

import synth
from oracle import transformer
from tests.test_gpu_prefill import LOGIT_TOL, _custom, _rel_err
from tests.util import bf16_pair, gpu_available, oracle_model

pytestmark = pytest.mark.gpu

LOOK, SEEN, ASK, VOCAB = 7, 11, 13, 1008


def late_maximum(heads, kv, dh):
    """Weights of two layers in which every score is 0 but that of id LOOK against id SEEN, 30, in the first, and of ASK against
    LOOK in the second, so that ASK's logits show what the first layer made of LOOK's row."""
    cfg = _custom(synth.ModelShape(2, 256, heads, kv, 512, VOCAB, head_dim=dh), 1, 460)
    w = bf16_pair(cfg)
    ids = [LOOK, SEEN, ASK]
    emb, layers = w[0]["tok_embed"], w[0]["layers"]
    emb[:, :3] = 0.0
    emb[ids] = 0.0
    emb[ids, [0, 1, 2]] = 16.0       # 16 behind the norm too
    layers[0]["wo"][:3] = layers[0]["w_down"][:3] = 0.0
    layers[0]["wo"].mul_(4.0)
    layers[0]["wv"].mul_(4.0)
    slow = dh // 2 - 1               # the slowest of the rotated pairs
    for lay, query, key, score in ((layers[0], 0, 1, 30.0), (layers[1], 2, 0, 200.0)):
        lay["attn_norm"].fill_(1.0)
        for name, n, column, x in (("wq", heads, query, 1.25), ("wk", kv, key, score * dh ** 0.5 / 256 / 1.25)):
            lay[name].zero_()
            lay[name].view(n, dh, 256)[:, slow, column] = x
    return cfg, w


# SEEN in a chunk of 64 positions that all of LOOK's tile sees (256 .. 319) or in the diagonal one, at a chunk's ends, in the very
# first; a tile of 16 rows is 16 tokens, 4, and 1 or 2 and parts (groups of 1, 4 and 9).  A row that keeps what it had summed before
# its maximum moved, put into the oracle, makes an error of 0.22 and more
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("heads,kv,dh", [(2, 2, 128), (8, 2, 64), (9, 1, 128)])
@pytest.mark.parametrize("seen,look", [(256, 330), (319, 321), (290, 383), (385, 391), (0, 450), (449, 450)])
def test_one_row_of_a_tile_moves_its_maximum(heads, kv, dh, seen, look):
    from paper_2408_11850_amd import harness
    cfg, w = late_maximum(heads, kv, dh)
    target, draft = harness.build_pair(cfg, weights=w)
    ctx = harness.make_context(cfg, target, draft, 8, temperature=1.0)
    import paper_2408_11850_amd as amd
    ctx.set_option(amd.SPEC_OPT_PREFILL, 1)
    prompt = [i if i not in (LOOK, SEEN, ASK) else 500 for i in synth.prompt_tokens(460, VOCAB, 7).tolist()]
    prompt[seen], prompt[look] = SEEN, LOOK
    ctx.prefill(prompt, which_mask=1)
    ocm = transformer.CachedModel(oracle_model(w[0], cfg.target), 512)
    ocm.feed(prompt[:-1])
    toks = [prompt[-1], ASK]
    assert _rel_err(ctx.verify(toks, want_logits=True), ocm.feed(toks)) <= LOGIT_TOL
    ctx.close()
