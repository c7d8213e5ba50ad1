"""Up to which room a decode attention is one launch (host only)."""
import ctypes as C

import paper_2408_11850_amd as amd


def test_the_line_lies_where_one_launch_is_ahead():
    """56 KV heads give 224 of 256 CUs a part of a head; with fewer, a context near the end of a longer room fell behind."""
    amd.load_library()
    f = C.CDLL(amd.LIB_PATH)._Z25attention_one_launch_roomi
    assert [f(h) for h in (1, 8, 32, 47, 48, 52, 55)] == [1216] * 7
    assert [f(h) for h in (56, 57, 64, 128)] == [3072] * 4
