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
# 4104 with 17 and 25 tokens of a narrow matrix: K slices; 14352 and 16384: from 9 tokens on one and two workgroups per CU, below
# and at four panels per CU; 24592: four panels at a time, up to 8 tokens from K = 1568 on PAIR; 4624: uneven shares, K slices
# from 4096 on
@pytest.mark.parametrize("N,K", [(16, 40), (48, 8), (2048, 1032), (2064, 520), (4112, 1032), (8192, 2088), (8208, 264),
                                 (24592, 136), (2048, 4104), (14352, 264), (16384, 264), (24592, 2056), (4624, 4088), (4624, 4104)])
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


# Residual adds and SiLU * mul in every layout that up to 8 tokens take (asserted in test_abi.py); 256 x 24640: K slices
FORWARDS = [(2048, 4, 2, 5632), (4608, 4, 2, 1376), (8448, 4, 2, 640), (512, 4, 4, 8400), (256, 2, 1, 24640), (2304, 11, 1, 1376),
            (4096, 4, 2, 2304), (4096, 16, 2, 2048), (4608, 4, 2, 2560), (8448, 4, 2, 2560), (512, 4, 4, 1376)]


@pytest.mark.parametrize("d,heads,kv,ffn", FORWARDS)
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


def _shifted(t):
    """The same values one element off the allocation's grid."""
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
    v = buf[1:1 + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 4 == 2
    return v


# K slices, panels, half panels; the operand's rows start 2 bytes off every vector
@pytest.mark.parametrize("M,N,K", [(1, 2048, 2048), (7, 4112, 1032), (17, 2064, 4104), (32, 48, 40)])
def test_projection_of_activations_at_an_odd_address(M, N, K):
    import paper_2408_11850_amd as amd
    gen = torch.Generator().manual_seed(N + M)
    w = torch.randn(N, K, generator=gen).mul_(0.05).to(torch.bfloat16)
    x = torch.randn(M, K, generator=gen).to(torch.bfloat16)
    ref = (x.double() @ w.double().T).numpy()
    y = amd.gemm(_shifted(x.cuda()), amd.binding.pack_matrices([w.cuda()]), N).cpu().double().numpy()
    assert np.linalg.norm(y - ref) <= 2.0 ** -24 * 60 ** 0.5 * np.linalg.norm(ref)   # as above


def test_embedding_and_gains_at_odd_addresses_give_the_same_bits():
    """A model whose embedding and norm gains are views one element into their allocations: prompt passes of both kinds,
    draft steps and forwards of every layout of the residual add equal those of the aligned model."""
    import paper_2408_11850_amd as amd
    for d, ffn in ((256, 1376), (4608, 1376), (8448, 640)):
        s = synth.ModelShape(2, d, 4, 2, ffn, 1008, head_dim=64)
        outs = []
        for shift in (False, True):
            gen = torch.Generator(device="cuda").manual_seed(d)

            def tensor(layer, name):
                if name in ("attn_norm", "ffn_norm", "final_norm"):
                    return torch.randn(d, generator=gen, device="cuda").mul_(0.3).add_(1.0).to(torch.bfloat16)
                n, k = (s.vocab, d) if layer is None else synth.layer_matrix_shapes(s)[name]
                return torch.randn(n, k, generator=gen, device="cuda").mul_(0.9 / k ** 0.5).to(torch.bfloat16)

            model = amd.pack_model(s, tensor)
            if shift:
                model.tok_embed, model.final_norm = _shifted(model.tok_embed), _shifted(model.final_norm)
                for lay in model.layers:
                    lay["attn_norm"], lay["ffn_norm"] = _shifted(lay["attn_norm"]), _shifted(lay["ffn_norm"])
            ctx = amd.SpecContext(model, model, gamma_max=31, max_seq=256)
            got = []
            for mode in (0, 1):
                ctx.set_option(amd.SPEC_OPT_PREFILL, mode)
                ctx.prefill(synth.prompt_tokens(90, s.vocab, 7).tolist())
                got.append(np.asarray([ctx.draft_step(0.3, True), ctx.draft_step(0.6, True)]))
                ctx.drop_drafts()
                ctx.rollback_kv(amd.SPEC_DRAFT, 89)
                for m in (1, 9, 17):
                    got.append(ctx.verify(synth.prompt_tokens(m, s.vocab, 8).tolist(), want_logits=True))
                    ctx.rollback_kv(amd.SPEC_TARGET, 89)
            outs.append(got)
            ctx.close()
        assert all(np.isfinite(g).all() for g in outs[0])
        assert all(np.array_equal(a, b) for a, b in zip(*outs)), d


# Units of work beyond 256 and 512, so that one and two workgroups per CU share them out differently (uneven shares, several
# panel groups per workgroup).  Up to 8 tokens, third: QKV, O and LM head 512 panels, gate/up 512 half units, all two per CU;
# fourth: gate/up 704 half units in 512 workgroups with shares as they fall, LM head 875 panels.  From 9 tokens on, second and
# fifth: gate/up 525 and 544 units, fifth: LM head 1250 panels.  (K slices, and the matrices that take one workgroup per CU in
# both modes, are in all of them; that the modes differ is asserted in test_abi.py)
MODES = [(4608, 40, 4, 5632, 8496), (8448, 64, 4, 8400, 25616), (8192, 32, 16, 4096, 8192), (2048, 16, 16, 5632, 14000),
         (1024, 8, 8, 8704, 20000)]


@pytest.mark.parametrize("d,heads,kv,ffn,vocab", MODES)
def test_launch_modes_give_the_same_bits(d, heads, kv, ffn, vocab):
    import paper_2408_11850_amd as amd
    s = synth.ModelShape(1, d, heads, kv, ffn, vocab, head_dim=128)
    gen = torch.Generator(device="cuda").manual_seed(d)

    def tensor(layer, name):
        if name in ("attn_norm", "ffn_norm", "final_norm"):
            return torch.randn(d, generator=gen, device="cuda").mul_(0.3).add_(1.0).to(torch.bfloat16)
        n, k = (vocab, d) if layer is None else synth.layer_matrix_shapes(s)[name]
        return torch.randn(n, k, generator=gen, device="cuda").mul_(0.9 / k ** 0.5).to(torch.bfloat16)

    model = amd.pack_model(s, tensor)
    ctx = amd.SpecContext(model, model, gamma_max=31, max_seq=256)
    ctx.prefill(synth.prompt_tokens(40, vocab, 7).tolist(), which_mask=1)
    toks = synth.prompt_tokens(32, vocab, 8).tolist()
    for m in (1, 8, 9, 16, 17, 32):
        got = []
        for wgs in (1, 2):
            ctx.set_option(amd.SPEC_OPT_GEMM_WGS_PER_CU, wgs)
            got.append(ctx.verify(toks[:m], want_logits=True))
            ctx.rollback_kv(amd.SPEC_TARGET, 39)
        assert np.isfinite(got[0]).all() and got[0].std() > 0.1 and np.array_equal(got[0], got[1]), m
    ctx.close()
