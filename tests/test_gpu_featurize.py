"""MFMA feature map: one to fourteen waves a workgroup, runs of several tiles, remainders of a tile."""
import numpy as np
import pytest
import torch

import paper_2603_04127_amd as dk
from oracle import dark_oracle as O
from tests import parity_util as U

pytestmark = pytest.mark.gpu

# B, H, L, d, m
SHAPES = [(1, 1, 1, 64, 64), (1, 2, 33, 64, 64), (1, 1, 95, 64, 128), (1, 3, 64, 64, 192), (2, 1, 31, 64, 896),
          (1, 1, 129, 128, 384), (1, 1, 45, 128, 64), (48, 48, 97, 64, 256), (2, 3, 1, 128, 64), (5, 3, 1025, 128, 64),
          (60, 12, 256, 128, 64), (7, 50, 1000, 128, 128), (9, 40, 1001, 128, 128)]


@pytest.mark.parametrize("is_query", [True, False])
@pytest.mark.parametrize("shape", SHAPES)
def test_featurize(shape, is_query):
    B, H, L, d, m = shape
    inp = U.random_problem(61, B, H, L, d, d, m, 8, bf16=True, w_shared=H == 3, amp=1.5)
    dev = U.to_device(inp, True)
    phi, stab = dk.dark_featurize(dev["Q"], dev["M"], dev["W"], is_query, path=dk.PATH_FUSED)
    torch.cuda.synchronize()
    phi, stab = phi.float().cpu().numpy(), stab.cpu().numpy()
    for b, h in {(0, 0), (B - 1, H - 1), (B // 2, H // 3)}:
        want, c = O.featurize(inp["Q"][b, h], inp["M"][h], inp["W"] if inp["W"].ndim == 2 else inp["W"][h], is_query)
        got = stab[b, h]
        assert np.abs(got - c).max() <= 2e-2   # the shift is itself a logit computed from fp16-rounded operands
        adj = phi[b, h] * np.exp((got - c)[:, None] if is_query else (got - c))
        U.assert_close(adj, want, U.TOL["bf16"], f"phi[{b},{h}] {shape}")


@pytest.mark.parametrize("is_query", [True, False])
def test_more_heads_than_one_launch_takes(is_query):
    # 2^26 + 3 batch entries of one row, a workgroup of 64 threads each: more threads than a launch has.
    B = (1 << 26) + 3
    g = torch.Generator(device="cuda").manual_seed(7)
    X = torch.empty(B, 1, 1, 64, dtype=torch.bfloat16, device="cuda")
    X.view(-1, 64)[:] = torch.randn(8191, 64, generator=g, device="cuda").to(torch.bfloat16).repeat(B // 8191 + 1, 1)[:B]
    W = torch.randn(1, 64, 64, generator=g, device="cuda")
    phi, stab = dk.dark_featurize(X, None, W, is_query, path=dk.PATH_FUSED)
    few = slice(B - 8191, B)
    want, c = dk.dark_featurize(X[few].contiguous(), None, W, is_query, path=dk.PATH_FUSED)
    torch.cuda.synchronize()
    assert torch.equal(phi[few], want) and torch.equal(stab[few], c)
    assert torch.equal(phi[:3], phi[8191:8194])
    del X, phi
    torch.cuda.empty_cache()
