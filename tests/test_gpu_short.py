"""GPU parity of the two-launch forward pass of short sequences (bf16 inputs) at the edges of its tiles and of its rule."""
import numpy as np
import pytest

import paper_2603_04127_amd as dk
from tests import parity_util as U
from tests.test_gpu_parity import _drifting_keys, _reround

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# B, H, L, d, m: one key, a tile of 32 at, below and above its edge; eight waves with a tile each, with one more and with an
# odd number of tiles; workgroups of one, a ragged and several steps of 32 queries; more blocks of features than CUs; the
# longest sequence of the rule and the first one past it.
SHAPES = [(1, 1, 1, 64, 256), (1, 2, 31, 64, 256), (2, 1, 32, 64, 512), (1, 3, 33, 128, 256), (1, 2, 255, 64, 256),
          (1, 1, 256, 128, 256), (2, 2, 257, 64, 512), (3, 12, 509, 64, 256), (5, 13, 90, 64, 256), (3, 11, 97, 128, 256),
          (1, 1, 1024, 128, 256), (1, 1, 1025, 128, 256), (1, 2, 2048, 64, 256), (1, 2, 2049, 64, 256)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("out_f32", [False, True])
def test_short_forward(shape, out_f32):
    B, H, L, d, m = shape
    inp = U.random_problem(91, B, H, L, d, d, m, d, bf16=True, amp=1.5, w_shared=m == 512)
    dev = U.to_device(inp, True)
    out = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], out_dtype=torch.float32 if out_f32 else None)
    torch.cuda.synchronize()
    U.assert_close(out.float().cpu().numpy(), U.oracle_attn(inp, False), U.TOL["bf16"], f"{shape} f32 out={out_f32}")


@pytest.mark.parametrize("L", [200, 700])   # a tile a wave, and three, whose shifts are raised
@pytest.mark.parametrize("general", [False, True])
def test_key_logits_that_rise_along_the_sequence(L, general):
    inp = U.random_problem(92, 1, 2, L, 64, 64, 256, 64, bf16=True, amp=1.0)
    inp["K"] = _drifting_keys(inp["K"], 8.0, 39, 6.0)
    _reround(inp, "K")
    dev = U.to_device(inp, True)
    # a schedule of the general kernels (their own number of workgroups) takes the call to them
    out = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], sched={"kv_wgs": 512} if general else None)
    torch.cuda.synchronize()
    U.assert_close(out.float().cpu().numpy(), U.oracle_attn(inp, False), U.TOL["bf16"], f"rising logits, L={L}")


def test_shifts_of_the_feature_blocks_differ():
    # draws whose length grows along the features: every block of 64 features has its own shift, far from its neighbours'
    inp = U.random_problem(93, 1, 2, 300, 64, 64, 256, 64, bf16=True, amp=2.0)
    inp["W"] *= np.linspace(0.2, 5.0, 256, dtype=np.float32)[None, :, None]
    dev = U.to_device(inp, True)
    out = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"])
    ref = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32)
    torch.cuda.synchronize()
    # logits of a hundred in fp16 operands: 2^-11 of them is a relative error of several per cent, on either MFMA path; the
    # general kernels are held to the same figure
    gen = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], sched={"kv_wgs": 512})
    torch.cuda.synchronize()
    e, g = ((x.float() - ref.float()).norm() / ref.float().norm() for x in (out, gen))
    assert torch.isfinite(out.float()).all() and e <= 1.1 * g + 2e-3, (e, g)
