"""Which launches touch weights ahead: the rules against what was measured. No GPU needed."""
import ctypes as C

import pytest

import workload as W
from host_rules import library


def touched(config, role, rows, position, beside=False):
    """For a layer of this model: the O, gate/up and down weights; the model: all layers and the vocabulary head."""
    d = W.get_config(config).models()[role]
    qd, kvd = d.n_q_heads * d.head_dim, d.n_kv_heads * d.head_dim
    layer = 2 * qd * d.d_model + 6 * d.d_model * d.ffn
    model = d.n_layers * (layer + 2 * d.d_model * (qd + 2 * kvd)) + (2 * d.d_model * d.vocab if d.head == "lm" else 0)
    f = library()._Z15weights_touchedimmbb
    f.restype, f.argtypes = C.c_bool, [C.c_int, C.c_size_t, C.c_size_t, C.c_bool, C.c_bool]
    return f(rows, layer, model, position, beside)


def test_models_and_rows():
    for rows in (1, 16, 256):
        for config, role in (("c2_small", "target"), ("c2_small", "prm"), ("c3_1p5b", "target"), ("c3_1p5b", "draft")):
            assert touched(config, role, rows, False)
        assert touched("c4_7b", "draft", rows, True)
        assert not touched("c2_small", "draft", rows, False)        # fits the Infinity Cache, unless others are beside it
        assert touched("c2_small", "draft", rows, False, True)
        assert not touched("c2_small", "draft", rows, True) and not touched("c2_small", "target", rows, True)
        assert not touched("c3_1p5b", "draft", rows, True)          # 27 MB a layer
        assert not touched("c4_7b", "target", rows, False) and not touched("c4_7b", "target", rows, True)
    assert not touched("c3_1p5b", "target", 257, False) and not touched("c3_1p5b", "target", 257, True)


@pytest.mark.parametrize("own,position,groups", [
    (8, True, 16), (64, True, 2), (80, True, 2), (128, True, 1),
    (88, True, 0), (96, True, 0), (112, True, 0), (129, True, 0), (160, True, 0), (256, True, 0),
    (8, False, 16), (112, False, 2), (160, False, 1), (256, False, 1), (264, False, 0)])
def test_workgroups_that_touch(own, position, groups):
    f = library()._Z12ahead_groupsiib
    f.restype, f.argtypes = C.c_int, [C.c_int, C.c_int, C.c_bool]
    assert f(own, 128, position) == groups
    assert f(own, 0, position) == 0
