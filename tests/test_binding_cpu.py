"""What the Python binding derives from a call before it reaches the device: no GPU needed."""
import numpy as np
import pytest
import torch

import paper_2603_04127_amd as dk


def _tensors(B=2, H=3, L=40, d=64, m=128):
    X = torch.zeros(B, H, L, d)
    return X, torch.zeros(H, d, d), torch.zeros(H, m, d)


def test_plan_follows_a_scale_that_changes_in_place():
    # a temperature kept in a tensor: the object stays the same while its value moves
    X, M, W = _tensors()
    t = torch.tensor(0.125)
    assert dk._plan(dk.OP_ATTN_FWD, False, X, X, M, W, scale=t)[0].scale == 0.125
    assert dk._decode_params(X[:, :, 0], X[:, :, 0], M, W, t).scale == 0.125
    t.fill_(0.5)
    assert dk._plan(dk.OP_ATTN_FWD, False, X, X, M, W, scale=t)[0].scale == 0.5
    assert dk._decode_params(X[:, :, 0], X[:, :, 0], M, W, t).scale == 0.5


@pytest.mark.parametrize("scale", [np.float64(0.25), np.array(0.25), torch.tensor(0.25)])
def test_plan_takes_every_number_for_a_scale(scale):
    X, M, W = _tensors()
    assert dk._plan(dk.OP_FEATURIZE, False, X, None, M, W, scale=scale)[0].scale == 0.25


def test_plan_refuses_what_equals_an_option_without_being_one():
    # 128.0 == 128 and hashes alike; the parameter block takes whole numbers only, also after 128 has been used
    X, M, W = _tensors()
    for make in (lambda **kw: dk._plan(dk.OP_ATTN_CAUSAL_FWD, False, X, X, M, W, **kw), ):
        assert make(chunk=128)[0].chunk == 128 and make(path=dk.PATH_F32)[0].path == 1
        for bad in (dict(chunk=128.0), dict(path=1.0)):
            with pytest.raises(TypeError):
                make(**bad)


def test_plan_follows_schedule_overrides_that_change_in_place():
    X, M, W = _tensors()
    wgs = torch.tensor(64)
    assert dk._plan(dk.OP_ATTN_FWD, False, X, X, M, W, sched={"kv_wgs": wgs})[0].sched_kv_wgs == 64
    wgs.fill_(128)
    assert dk._plan(dk.OP_ATTN_FWD, False, X, X, M, W, sched={"kv_wgs": wgs})[0].sched_kv_wgs == 128
    with pytest.raises(ValueError):
        dk._plan(dk.OP_ATTN_FWD, False, X, X, M, W, sched={"kv_wgs": 1, 3: 4})


@pytest.mark.parametrize("shape", [(3, 64), (2, 3, 1, 64)])
def test_decode_refuses_rows_of_another_rank(shape):
    _, M, W = _tensors()
    x = torch.zeros(shape)
    with pytest.raises(ValueError):
        dk._decode_params(x, x, M, W, 0.0)


class _Tagged(torch.Tensor):
    """A tensor subclass, as libraries around torch make them."""


@pytest.mark.parametrize("make", [lambda: torch.zeros(2, 3, 1, 64).as_strided((2, 3, 1, 64), (192, 64, 7, 1)),
                                  lambda: torch.zeros(2, 3, 1, 64).as_subclass(_Tagged),
                                  lambda: torch.nn.Parameter(torch.zeros(2, 3, 1, 64))])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_results_are_plain_contiguous_tensors(make, dtype):
    # whatever kind of tensor the values are, and whatever strides their dimensions of size one have
    V = make()
    out = dk._result(V, dtype, V)
    assert type(out) is torch.Tensor and out.dtype == dtype and out.shape == V.shape and not out.requires_grad
    assert out.stride() == torch.empty(V.shape).stride()
