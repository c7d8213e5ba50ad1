"""The whole-K projections (proj.hip): every way of filling the MFMA operands, every epilogue, at the edges of its range
(run with -m gpu)."""
import numpy as np
import pytest
import torch

import synth
from oracle import transformer
from tests.test_gpu_forward import LOGIT_TOL, _custom, _rel_err, _setup
from tests.util import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


# 8 / 9 and 16 / 17 tokens change the operand layout; N = 16: two half panels; 2048 / 2064: last of the half panels;
# 4112, 8208, 24592: one panel more than a workgroup range (1, 2, 6 per CU); K = 40, 1032: ragged K and odd step counts;
# 4104 with 17 and 25 tokens of a narrow matrix: K slices
@pytest.mark.parametrize("N,K", [(16, 40), (48, 8), (2048, 1032), (2064, 520), (4112, 1032), (8192, 2088), (8208, 264),
                                 (24592, 136), (2048, 4104)])
@pytest.mark.parametrize("M", [1, 8, 9, 16, 17, 25, 32])
def test_projection_at_the_edges_of_the_operand_layouts(M, N, K):
    import paper_2408_11850_amd as amd
    gen = torch.Generator().manual_seed(N * 64 + M)
    w = torch.randn(N, K, generator=gen).mul_(0.05).to(torch.bfloat16)
    x = torch.randn(M, K, generator=gen).to(torch.bfloat16)
    ref = (x.double() @ w.double().T).numpy()
    y = amd.gemm(x.cuda(), amd.binding.pack_matrices([w.cuda()]), N).cpu().double().numpy()
    assert np.isfinite(y).all()
    # one rounding of 2^-24 per addition of a chain whose partial sums grow with the square root of its length; no chain
    # here is longer than 60 additions, rows of y and columns of W are independent
    err = np.linalg.norm(y - ref) / np.linalg.norm(ref)
    assert err <= 2.0 ** -24 * 60 ** 0.5, err
    assert np.abs(y - ref).max() <= 12 * 2.0 ** -24 * 60 ** 0.5 * np.sqrt(np.mean(ref ** 2))


# residual add: 2048 half panels, 4608 single panels, 8448 four at a time, 256 x 24640 K slices; gate/up: 256 and 5632
# half panels, 8400 two or four panels, 24640 half panels again
@pytest.mark.parametrize("d,heads,kv,ffn", [(2048, 4, 2, 5632), (4608, 4, 2, 1376), (8448, 4, 2, 640), (512, 4, 4, 8400),
                                            (256, 2, 1, 24640)])
def test_forwards_at_the_edges_of_the_operand_layouts(d, heads, kv, ffn):
    cfg = _custom(synth.ModelShape(2, d, heads, kv, ffn, 1008, head_dim=128), 1)
    amd, ctx, tm, _ = _setup(cfg)
    prompt = synth.prompt_tokens(40, 1008, 7).tolist()
    toks = synth.prompt_tokens(32, 1008, 8).tolist()
    ctx.prefill(prompt)
    ocm = transformer.CachedModel(tm, 256)
    ocm.feed(prompt[:-1])
    base = ocm.len
    ref = ocm.feed(toks)
    for m in (1, 8, 9, 16, 17, 32):
        got = ctx.verify(toks[:m], want_logits=True)
        ctx.rollback_kv(amd.SPEC_TARGET, base)
        err = _rel_err(got, ref[:m])
        print(f"  d={d} ffn={ffn} m={m}: {err:.2e}", flush=True)
        assert err <= LOGIT_TOL, (m, err)
    ctx.close()
