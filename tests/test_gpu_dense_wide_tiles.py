"""The large and the 256 x 192 tile of the prompt-time projection at their edges (run with -m gpu)."""
import pytest
import torch

import synth
from tests.test_gpu_dense_tiles import LARGE, WIDE, tile
from tests.test_gpu_prefill import _custom, _rel_err, _setup
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# 2045 x 8160: 8 x 32 tiles of 256 x 256, one round (small tiles: 4); 509 x 24544: 2 x 128 of 256 x 192, one round (small: 3).
# K: 1, 2, 3, 5 and 12 steps of 32 (shorter than the rings, odd counts, longer)
@pytest.mark.parametrize("M,N,which", [(2045, 8160, LARGE), (509, 24544, WIDE)])
@pytest.mark.parametrize("K", [32, 64, 96, 160, 384])
@pytest.mark.parametrize("epilogue", [0, 1, 2])
def test_projection_of_a_filled_chip(M, N, which, K, epilogue):
    import paper_2408_11850_amd as amd
    assert tile(M, N, K) == which
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda")  # noqa: E731
    w, x = rnd(N, K).mul_(0.05).to(torch.bfloat16), rnd(M, K).to(torch.bfloat16)
    ref = x.double() @ w.double().T
    packed = amd.binding.pack_matrices([w])
    # as for the other tiles: a chain of K / 32 additions with independent errors, 12 deviations for the largest of 2^24
    f32 = 2.0 ** -24 * (K / 32 + 8) ** 0.5 * 2
    if epilogue == 2:
        got = amd.dense_gemm(x, packed, N, 2).double()
        ref = ref.view(M, -1, 2, 16)
        scale = (ref[:, :, 0].square().mean().sqrt() * (1 + ref[:, :, 1].abs().max())).item() * 2
        ref = (torch.nn.functional.silu(ref[:, :, 0]) * ref[:, :, 1]).reshape(M, -1)
        rel = 2.0 ** -8
    else:
        y0 = rnd(M, N)
        got = amd.dense_gemm(x, packed, N, epilogue, y0.clone() if epilogue else None).double()
        ref = ref + y0.double() if epilogue else ref
        scale, rel = ref.square().mean().sqrt().item(), 0.0
    assert got.shape == ref.shape and torch.isfinite(got).all()
    assert ((got - ref).abs() - rel * ref.abs()).max().item() <= 12 * f32 * scale
    assert ((got - ref).norm() / ref.norm()).item() <= rel + f32


# QKV with its rotation and page append: 997 rows x 12288 take 256 x 192 tiles (a tile holds one and a half heads of 128, three
# of 64), 2045 x 8192 256 x 256, and so do 511 x 25344, 13 tile columns per XCD.  Two layers: the first one's q reaches the
# caches of the second
@pytest.mark.parametrize("shape,n_prompt,which", [(synth.ModelShape(2, 256, 64, 16, 256, 1024, 128), 998, WIDE),
                                                  (synth.ModelShape(2, 256, 128, 32, 256, 1024, 64), 998, WIDE),
                                                  (synth.ModelShape(2, 256, 48, 8, 256, 1024, 128), 2046, LARGE),
                                                  (synth.ModelShape(2, 256, 162, 18, 256, 1024, 128), 512, LARGE)])
def test_dense_and_chunked_prompt_passes_agree(shape, n_prompt, which):
    assert tile(n_prompt - 1, (shape.n_heads + 2 * shape.n_kv_heads) * shape.head_dim, shape.d_model) == which
    amd, ctx, _, _ = _setup(_custom(shape, 1, n_prompt))
    prompt = synth.prompt_tokens(n_prompt, shape.vocab, 7).tolist()
    toks = [prompt[-1]] + synth.prompt_tokens(8, shape.vocab, 8).tolist()
    out = []
    for mode in (0, 1):
        ctx.set_option(amd.SPEC_OPT_PREFILL, mode)
        ctx.prefill(prompt)
        out.append(ctx.verify(toks, want_logits=True))
    err = _rel_err(out[1], out[0])
    print(f"  dense vs chunked: {err:.2e}", flush=True)
    assert err <= 1e-2          # as for the narrower pairs
    ctx.close()
