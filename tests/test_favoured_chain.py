"""Which of two overlapped chains issues first (host only)."""
import ctypes as C

import pytest

import paper_2408_11850_amd as amd
import synth


def front(target, draft, gamma):
    amd.load_library()
    f = C.CDLL(amd.LIB_PATH)._Z14favoured_chainRK15spec_model_descS1_i
    d = [amd.ModelDesc(s.n_layers, s.d_model, s.n_heads, s.n_kv_heads, s.head_dim, s.d_ffn, s.vocab, s.rope_theta, s.rms_eps)
         for s in (target, draft)]
    return f(C.byref(d[0]), C.byref(d[1]), gamma)


@pytest.mark.parametrize("pair", ["7b_1b", "33b_1b", "70b_7b"])
@pytest.mark.parametrize("gamma", [1, 4, 8, 16])
def test_the_draft_of_a_target_with_long_kernels(pair, gamma):
    cfg = synth.config(pair)
    assert front(cfg.target, cfg.draft, gamma) == amd.SPEC_DRAFT


# the small pair's shapes at depths target / draft: what each measured step ran fastest with, or level with
@pytest.mark.parametrize("depths,gamma,which", [((24, 4), 4, 0), ((12, 4), 2, 0), ((16, 1), 3, 0), ((24, 2), 8, -1), ((24, 3), 6, -1),
                                                ((24, 4), 5, -1), ((20, 4), 6, 1), ((12, 4), 8, 1)])
def test_brief_kernels_go_by_the_longer_chain(depths, gamma, which):
    s = synth.config("small").target
    assert front(synth._truncate(s, depths[0]), synth._truncate(s, depths[1]), gamma) == which
