"""The binding's checks of device buffers (no GPU): tables that were marshalled once go through one
native call, lists of tensors through Python; both refuse the same calls with the same words."""
import numpy as np
import pytest
import torch

import paper_2602_05754_amd as tf

SHAPES, T = [(8, 16), (24, 8), (16, 16)], 12


def _backward(wrap, change=None, mask=(0, 1, 0), io=tf.TF_BF16):
    """tf_stage_backward without a context: what passes the binding's checks is refused by the library."""
    dt = torch.bfloat16
    t = {"W": [torch.zeros(k, n, dtype=dt) for k, n in SHAPES], "X": [torch.zeros(T, k, dtype=dt) for k, n in SHAPES],
         "dY": [torch.zeros(T, n, dtype=dt) for k, n in SHAPES], "dX": [torch.zeros(T, k, dtype=dt) for k, n in SHAPES],
         "dW": [torch.zeros(k, n) for k, n in SHAPES]}
    if change:
        change(t)
    t = {k: wrap(v) for k, v in t.items()}
    with pytest.raises((ValueError, tf.TfError)) as e:
        tf.tf_stage_backward(None, SHAPES, T, io, t["W"], t["X"], t["dY"], np.array(mask, np.uint8), t["dX"], t["dW"], tf.TF_F32)
    return e.type, str(e.value)


def _adamw(wrap, change=None):
    n = [5, 64, 33]
    t = {k: [torch.zeros(q) for q in n] for k in ("p", "m", "v", "grad", "ema", "ema_abs")}
    t["p_lowp"] = [torch.zeros(5, dtype=torch.bfloat16), None, torch.zeros(33, dtype=torch.bfloat16)]
    if change:
        change(t)
    t = {k: wrap(v) for k, v in t.items()}
    with pytest.raises((ValueError, tf.TfError)) as e:
        tf.tf_masked_adamw(None, n, t["p"], t["m"], t["v"], t["grad"], tf.TF_F32, [1] * 3, 1e-3, 0.9, 0.99, 1e-8, 0.0, p_lowp=t["p_lowp"],
                           tensor_freeze_mask=np.array([0, 0, 1], np.uint8), ema=t["ema"], ema_abs=t["ema_abs"], ema_decay=0.9)
    return e.type, str(e.value)


def test_calls_that_pass_the_checks_reach_the_library():
    for run in (_backward, _adamw):
        assert run(list) == run(tf.PtrTable)
        assert run(tf.PtrTable)[0] is tf.TfError                       # no context


@pytest.mark.parametrize("name", ["W", "X", "dY", "dX", "dW"])
@pytest.mark.parametrize("i", [0, 2])
@pytest.mark.parametrize("fault", ["short", "type"])
def test_backward_buffers(name, i, fault):
    def change(t):
        x = t[name][i]
        t[name][i] = x.reshape(-1)[:-1].clone() if fault == "short" else x.to(torch.float16 if x.element_size() == 2 else torch.int32)
    got = _backward(list, change), _backward(tf.PtrTable, change)
    assert got[0][0] is ValueError and got[1][0] is ValueError and f"{name}[{i}]" in got[0][1] and f"{name}[{i}]" in got[1][1]


@pytest.mark.parametrize("name", ["X", "dW"])
def test_buffers_of_frozen_layers_are_not_looked_at(name):
    def change(t):
        t[name][1] = torch.zeros(1)
    assert _backward(tf.PtrTable, change) == _backward(tf.PtrTable) == _backward(list, change)
    assert _backward(tf.PtrTable, change, mask=(0, 0, 0))[0] is ValueError


@pytest.mark.parametrize("name", ["p", "m", "v", "grad", "p_lowp", "ema", "ema_abs"])
def test_optimizer_buffers(name):
    def change(t):
        t[name][0] = t[name][0][:4].clone()
    for wrap in (list, tf.PtrTable):
        kind, text = _adamw(wrap, change)
        assert kind is ValueError and f"{name}[0]" in text

    def frozen(t):
        t[name][2] = t[name][2][:4].clone()
    assert _adamw(tf.PtrTable, frozen)[0] is tf.TfError


def test_tables_of_another_length_and_raw_pointers():
    def fewer(t):
        t["dX"] = t["dX"][:2]
    assert _backward(tf.PtrTable, fewer)[0] is ValueError

    def raw(t):
        t["W"][0] = 4096                                                # a pointer of unknown size passes
    assert _backward(tf.PtrTable, raw)[0] is tf.TfError


@pytest.mark.parametrize("number", [int, np.int64, np.int32, float])
def test_type_codes_and_sizes_of_other_number_types(number):
    """What int() takes, as from an array of codes, works for tables as for lists."""
    for wrap in (list, tf.PtrTable):
        t = {k: wrap(v) for k, v in {
            "W": [torch.zeros(k, n, dtype=torch.bfloat16) for k, n in SHAPES], "X": [torch.zeros(T, k, dtype=torch.bfloat16) for k, n in SHAPES],
            "dY": [torch.zeros(T, n, dtype=torch.bfloat16) for k, n in SHAPES], "dX": [torch.zeros(T, k, dtype=torch.bfloat16) for k, n in SHAPES],
            "dW": [torch.zeros(k, n) for k, n in SHAPES]}.items()}
        with pytest.raises(tf.TfError):                                 # no context: it has passed the checks
            tf.tf_stage_backward(None, SHAPES, number(T), number(tf.TF_BF16), t["W"], t["X"], t["dY"], None, t["dX"], t["dW"], number(tf.TF_F32))


def test_a_device_number_of_another_number_type():
    class Ctx:
        device_id, handle = np.int64(0), None

        def last_hip_error(self):
            return 0
    with pytest.raises(ValueError) as e:                                # host tensors: refused for that, by name
        tf.tf_stage_backward(Ctx(), SHAPES[:1], T, tf.TF_F32, *[tf.PtrTable([torch.zeros(T, 16)])] * 3, None,
                             *[tf.PtrTable([torch.zeros(T, 16)])] * 2, tf.TF_F32)
    assert "GPU 0" in str(e.value)
