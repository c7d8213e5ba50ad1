"""Decode attention in one launch over more than 1216 positions, where there are KV heads enough (run with -m gpu)."""
import ctypes as C

import pytest

import synth
from oracle import transformer
from tests.test_gpu_forward import LOGIT_TOL, _custom, _rel_err, _setup
from tests.test_gpu_row_bits import assert_rows_share_their_bits
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def room(max_seq):
    """Positions there is room for in the pages of a context."""
    return (-(-max_seq // 64) + 1) * 64


def one_launch_room(kv_heads):
    import paper_2408_11850_amd as amd
    amd.load_library()
    return C.CDLL(amd.LIB_PATH)._Z25attention_one_launch_roomi(kv_heads)


# 56 KV heads: one launch up to room for 3072 positions.  Contexts around the rounds of chunks that a workgroup has in flight (7
# waves, two each: 448 positions), and the last ones there is room for; one part of 16-row tiles more at M = 17
def test_long_rounds_against_the_oracle():
    cfg = _custom(synth.ModelShape(2, 256, 56, 56, 512, 1008, head_dim=64), 1)
    cfg.n_prompt = 2100
    amd, ctx, tm, _ = _setup(cfg, gamma_max=31)
    assert 1216 < room(2100 + 64 + 64) <= one_launch_room(56)
    ids = synth.prompt_tokens(2200, 1008, 7).tolist()
    ocm = transformer.CachedModel(tm, 2304)
    fed = 0
    for context in (895, 897, 1024, 1343, 1345, 1792, 2099):
        ctx.prefill(ids[:context + 1])
        ocm.feed(ids[fed:context])
        ref = ocm.feed(ids[context:context + 17])
        for m in (1, 5, 17):
            assert _rel_err(ctx.verify(ids[context:context + m], want_logits=True), ref[:m]) <= LOGIT_TOL, (context, m)
            ctx.rollback_kv(amd.SPEC_TARGET, context)
        ocm.rollback(context)
        fed = context
        print(f"  context {context}: ok", flush=True)
    ctx.close()


# rows share their bits on both sides of the lines: 56 heads in one launch (room for 2304 and 3072 positions) and split (3136),
# 48 and 32 in one (1216) and split (1280)
@pytest.mark.parametrize("heads,max_seq,one", [(56, 2240, True), (56, 3008, True), (56, 3009, False), (48, 1152, True),
                                               (48, 1153, False), (32, 1152, True), (32, 1153, False)])
def test_rows_keep_their_bits(heads, max_seq, one):
    assert (room(max_seq) <= one_launch_room(heads)) == one
    assert_rows_share_their_bits(synth.ModelShape(2, 256, heads, heads, 512, 1008, head_dim=64), max_seq, (300, max_seq - 20))
