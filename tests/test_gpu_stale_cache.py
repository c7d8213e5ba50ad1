"""What an earlier prompt left in the pages of a cache does not reach a later one's logits (run with -m gpu)."""
import numpy as np
import pytest
import torch

import synth
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def model(s, seed, poison=None):
    """A packed model of random weights; `poison`: a token whose embedding is not finite."""
    import paper_2408_11850_amd as amd
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def tensor(layer, name):
        if name in ("attn_norm", "ffn_norm", "final_norm"):
            return torch.randn(s.d_model, generator=gen, device="cuda").mul_(0.3).add_(1.0).to(torch.bfloat16)
        n, k = (s.vocab, s.d_model) if layer is None else synth.layer_matrix_shapes(s)[name]
        t = torch.randn(n, k, generator=gen, device="cuda").mul_(0.9 / k ** 0.5).to(torch.bfloat16)
        if name == "tok_embed" and poison is not None:
            t[poison] = float("nan")
        return t

    return amd.pack_model(s, tensor)


# room for 320, 512, 1024, 1088 and 1280 positions: each kernel that a context's room chooses, splits in the last.  Behind the poisoned token every
# position holds NaN; the second prompt fills whole chunks of 32 (64 positions), so that nothing stale lies among its own, or
# none at all
@pytest.mark.parametrize("max_seq", [256, 448, 960, 1024, 1153])
@pytest.mark.parametrize("heads,kv,dh", [(2, 2, 128), (8, 1, 64)])
def test_a_poisoned_prompt_does_not_reach_the_next_one(max_seq, heads, kv, dh):
    import paper_2408_11850_amd as amd
    from tests.test_gpu_attention_room import one_launch_room, room
    assert (room(max_seq) > one_launch_room(kv)) == (max_seq == 1153)
    s = synth.ModelShape(2, 256, heads, kv, 512, 1008, head_dim=dh)
    m = model(s, 3, poison=5)
    ids = [i if i != 5 else 6 for i in synth.prompt_tokens(max_seq, s.vocab, 7).tolist()]
    ctx = amd.SpecContext(m, m, gamma_max=8, max_seq=max_seq)
    clean = {}
    for n in (1, 65):
        ctx.prefill(ids[:n], which_mask=1)
        clean[n] = ctx.verify(ids[n - 1:n + 4], want_logits=True).copy()
        assert np.isfinite(clean[n]).all()
    for n in (1, 65):
        ctx.prefill(ids[:100] + [5] + ids[101:max_seq - 16], which_mask=1)
        assert not np.isfinite(ctx.verify(ids[:1], want_logits=True)).any()
        ctx.prefill(ids[:n], which_mask=1)
        got = ctx.verify(ids[n - 1:n + 4], want_logits=True)
        assert np.array_equal(got, clean[n]), (n, np.isfinite(got).all())
    ctx.close()
