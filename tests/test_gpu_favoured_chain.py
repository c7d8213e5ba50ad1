"""Which chain's waves issue first changes no bit of what either model computes (run with -m gpu)."""
import ctypes as C

import numpy as np
import pytest

import synth
from tests.test_gpu_stale_cache import model
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def favoured_now(ctx):
    """The chain in front in the next forwards of a context: 0 the target's, 1 the draft's, -1 neither."""
    import paper_2408_11850_amd as amd
    f = C.CDLL(amd.LIB_PATH)._Z12favoured_nowPK8spec_ctx
    f.argtypes = [C.c_void_p]
    return f(ctx._ctx)


# 8 target layers and a draft of the first: one draft pass is 0.2 target passes, so windows of 1 put the target in front, of 5
# neither and of 16 the draft.  Rows of every projection layout: up to 8 tokens, one row tile and two, K slices.
@pytest.mark.parametrize("shape", [(256, 4, 512), (2048, 16, 704)])
def test_the_favoured_chain_changes_no_bits(shape):
    import paper_2408_11850_amd as amd
    d, heads, ffn = shape
    target = model(synth.ModelShape(8, d, heads, heads, ffn, 1008), 3)
    draft = target.prefix(1, synth.ModelShape(1, d, heads, heads, ffn, 1008))
    ids = synth.prompt_tokens(90, 1008, 7).tolist()
    seen = []
    for gamma, front in ((1, amd.SPEC_TARGET), (5, -1), (16, amd.SPEC_DRAFT)):
        ctx = amd.SpecContext(target, draft, gamma_max=gamma, max_seq=256, temperature=0.7)
        assert favoured_now(ctx) == front
        ctx.prefill(ids[:40])
        out = []
        for m in (1, 5, 12, 20, 32):
            out.append(ctx.verify(ids[40:40 + m], want_logits=True).copy())
            ctx.rollback_kv(amd.SPEC_TARGET, 39)
        out.append([ctx.draft_step(0.37, want_token=True) for _ in range(2)])
        seen.append(out)
        ctx.close()
    for other in seen[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(seen[0], other))


def test_a_loop_leaves_the_favoured_chain_as_it_was():
    """Loops of short and long windows on one context, each with the graphs of its own favoured chain: the same tokens and logits
    again, and between them the choice that the context was made with."""
    import paper_2408_11850_amd as amd
    target = model(synth.ModelShape(8, 256, 4, 4, 512, 1008), 3)
    draft = target.prefix(1, synth.ModelShape(1, 256, 4, 4, 512, 1008))
    ids = synth.prompt_tokens(90, 1008, 7).tolist()
    ctx = amd.SpecContext(target, draft, gamma_max=16, max_seq=256, temperature=0.7)
    ctx.prefill(ids[:40])
    seen = {}
    for algo, gamma in ((amd.ALGO_PEARL, 1), (amd.ALGO_PEARL, 16), (amd.ALGO_PEARL, 5), (amd.ALGO_AR, 0)) * 2:
        tokens, _ = ctx.generate(algo, gamma, 24, synth.make_uniforms(24, max(gamma, 1), 5))
        assert favoured_now(ctx) == amd.SPEC_DRAFT, (algo, gamma)
        ctx.rewind(40 + 24)
        logits = ctx.verify(tokens[-1:], want_logits=True).copy()
        ctx.rewind(40)
        was = seen.setdefault((algo, gamma), (tokens, logits))
        assert was[0] == tokens and np.array_equal(was[1], logits), (algo, gamma)
    ctx.calibrate_gamma(4, 2, concurrent=True)
    assert favoured_now(ctx) == amd.SPEC_DRAFT
    ctx.close()
