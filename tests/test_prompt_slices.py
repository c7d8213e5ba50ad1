"""K slices of the prompt pass's residual projections: the rule on the host, the pass on the GPU."""
import ctypes as C

import pytest

import synth
from tests.util import gpu_available


def test_slices_are_whole_stages_and_fit_their_buffer():
    import paper_2408_11850_amd as amd
    amd.load_library()
    lib = C.CDLL(amd.LIB_PATH)
    slices, floats = lib._Z12dense_slicesiii, lib._Z19dense_slices_floatsv
    slices.argtypes, floats.restype = [C.c_int] * 3, C.c_size_t
    seen = set()
    for M in (1, 33, 65, 127, 128, 129, 256, 511, 1000, 1023, 2048, 4096):
        for N in (32, 256, 1000 * 16, 2048, 4096, 7168, 8192):
            for K in (32, 96, 256, 704, 2048, 2784, 5504, 11008, 28672):
                S = slices(M, N, K)
                seen.add(S)
                steps, tiles = K // 32, -(-M // 128) * -(-N // 128)
                assert S == 1 or (2 <= S <= 16 and S * tiles <= 256 and S * M * N <= floats()), (M, N, K, S)
                if S > 1:
                    length = -(-steps // S) + 1 & ~1          # whole stages of two K steps
                    assert length >= 4 and -(-steps // length) == S, (M, N, K, S)
                    assert (S - 1) * length < steps           # no slice is empty
    assert {1, 2, 4, 8} <= seen


# d_model x d_ffn: 1024 x 2784 (87 K steps, the last slice ends with half a stage), 256 x 2752, 2048 x 704; prompts of one row
# tile, one row more, and two and a bit
@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a GPU")
@pytest.mark.parametrize("d,heads,ffn", [(1024, 8, 2784), (256, 2, 2752), (2048, 16, 704)])
@pytest.mark.parametrize("n_prompt", [66, 129, 130, 300])
def test_sliced_prompt_pass_matches_oracle(d, heads, ffn, n_prompt):
    from oracle import transformer
    from tests.test_gpu_prefill import LOGIT_TOL, _custom, _rel_err, _setup
    shape = synth.ModelShape(3, d, heads, heads, ffn, 1024)
    amd, ctx, tm, _ = _setup(_custom(shape, 1, n_prompt))
    lib = C.CDLL(amd.LIB_PATH)
    assert lib._Z12dense_slicesiii(n_prompt - 1, d, max(d, ffn // 32 * 32)) > 1
    ctx.set_option(amd.SPEC_OPT_PREFILL, 1)
    for seed in (7, 9):                       # the second prompt finds the first one's sums in the buffers
        prompt = synth.prompt_tokens(n_prompt, 1024, seed).tolist()
        toks = [prompt[-1]] + synth.prompt_tokens(6, 1024, 8).tolist()
        ctx.prefill(prompt, which_mask=1)
        ocm = transformer.CachedModel(tm, n_prompt + 16)
        ocm.feed(prompt[:-1])
        err = _rel_err(ctx.verify(toks, want_logits=True), ocm.feed(toks))
        print(f"  d={d} ffn={ffn} n={n_prompt}: max logit error / range = {err:.2e}", flush=True)
        assert err <= LOGIT_TOL
    ctx.close()
