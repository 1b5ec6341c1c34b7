"""MFMA backward of causal attention: slices of several tiles with every kind of remainder, and single gradients."""
import numpy as np
import pytest
import torch

import paper_2603_04127_amd as dk
from oracle import dark_oracle as O
from tests import parity_util as U

pytestmark = pytest.mark.gpu

# B, H, L: as many (b,h) as it takes for a slice of several tiles; the last tile of a slice has 1, 8, 32 or 31 tokens
SHAPES = [(1, 3, 65), (2, 64, 200), (4, 64, 97), (2, 128, 127)]


@pytest.mark.parametrize("shape", SHAPES)
def test_slices_of_several_tiles(shape):
    B, H, L = shape
    inp = U.random_problem(91, B, H, L, 64, 64, 256, 64, bf16=True, w_shared=H == 128, amp=1.5, backward=True)
    dev = U.to_device(inp, True)
    g = dk.dark_attn_bwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], dev["dOut"], True, path=dk.PATH_FUSED)
    torch.cuda.synchronize()
    want = dict(zip(("dQ", "dK", "dV", "dM"), U.oracle_bwd(inp, True)))
    for k in want:
        U.assert_close_grad(g[k].cpu().numpy(), want[k], U.TOL["bf16"], f"{k} {shape}")


@pytest.mark.parametrize("need", [("dQ",), ("dK",), ("dV",), ("dM",)])
def test_single_gradients(need):
    # Each gradient alone is bit for bit what it is among the others.
    inp = U.random_problem(92, 2, 4, 333, 64, 64, 256, 64, bf16=True, backward=True)
    dev = U.to_device(inp, True)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], dev["dOut"], True)
    full = dk.dark_attn_bwd(*args, path=dk.PATH_FUSED)
    one = dk.dark_attn_bwd(*args, need=need, path=dk.PATH_FUSED)
    torch.cuda.synchronize()
    assert np.isfinite(full[need[0]].cpu().numpy()).all()
    assert torch.equal(full[need[0]], one[need[0]])


# Slices that end in the middle of a 64-token tile of the key pass: 96 + 34, 160 + 130 and 160 + 160 + 130 positions.
@pytest.mark.parametrize("shape", [(4, 32, 130), (2, 64, 290), (1, 85, 450)])
def test_slices_of_an_odd_number_of_tiles(shape):
    B, H, L = shape
    inp = U.random_problem(93, B, H, L, 64, 64, 256, 64, bf16=True, amp=1.5, backward=True)
    dev = U.to_device(inp, True)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"])
    out, saved = dk.dark_attn_causal_fwd_save(*args, path=dk.PATH_FUSED, out_dtype=torch.float32)
    g = dk.dark_attn_bwd(*args, dev["dOut"], True, saved=saved, path=dk.PATH_FUSED)
    torch.cuda.synchronize()
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, True), U.TOL["bf16"], f"out {shape}")
    want = dict(zip(("dQ", "dK", "dV", "dM"), U.oracle_bwd(inp, True)))
    for k in want:
        U.assert_close_grad(g[k].cpu().numpy(), want[k], U.TOL["bf16"], f"{k} {shape}")


def test_infinity_at_the_end_of_an_odd_slice():
    # The key pass fills the rest of the slice's last tile with rows of its own: an infinite value of V in the slice's last row (its
    # 96 positions end inside a tile of 64) stays infinite in the rows after the slice.
    inp = U.random_problem(94, 4, 32, 130, 64, 64, 256, 64, bf16=True, amp=1.0)
    dev = U.to_device(inp, True)
    dev["V"][:, :, 95, 7] = float("inf")
    out = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_FUSED)[:, :, 96:].float().cpu().numpy()
    torch.cuda.synchronize()
    assert np.isposinf(out[..., 7]).all()
    assert np.isfinite(np.delete(out, 7, axis=-1)).all()


# Forward, slices of 1, 2, 3, 5 and 17 tiles of 32 with a ragged last one, by the state kernel that walks tiles in pairs (at d = 64 only
# on request): 30; 96 + 34; 64 + 56; 160 + 130; 96 + 96 + 68; 160 + 160 + 130; 64 heads of 3 x 544 + 468 positions.
@pytest.mark.parametrize("d,shape,wgs", [(d, (1, 2, L), w) for d in (64, 128) for L, w in
                                         ((30, 2), (130, 4), (120, 4), (290, 4), (260, 6), (450, 6))] + [(128, (1, 64, 2100), 256)])
@pytest.mark.parametrize("out_f32", [False, True])
def test_state_kernel_on_odd_tiles(d, shape, wgs, out_f32):
    B, H, L = shape
    inp = U.random_problem(95, B, H, L, d, d, 256, d, bf16=True, amp=1.5)
    dev = U.to_device(inp, True)
    out = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_FUSED,
                                  out_dtype=torch.float32 if out_f32 else None, sched={"cs_wgs": wgs, "cs_state": 1})
    torch.cuda.synchronize()
    for h in sorted({0, H // 2, H - 1}):
        Q, K, V, M, W = U.head(inp, 0, h)
        U.assert_close(out[0, h].float().cpu().numpy(), O.attn_causal(Q, K, V, M, W), U.TOL["bf16"], f"d={d} {shape} head {h}")
