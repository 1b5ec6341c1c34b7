"""GPU parity of the causal forward pass by kernel values (bf16 inputs, d = 128, short sequences) at the edges of its tiles."""
import ctypes

import numpy as np
import pytest

import paper_2603_04127_amd as dk
from tests import parity_util as U
from tests.test_gpu_parity import _drifting_keys, _reround

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# B, H, L: one position, a tile of 32 and a workgroup of 64 at, below and above their edge; one tile for each of the four waves
# that share the keys, with one more; a number of (b,h) that is and one that is not a multiple of 8; the longest
# sequences of the rule with more workgroups than CUs (36 tiles; 28,000 tiles of kernel values) and the first ones past it;
# pairs of tiles of queries: fewest tiles (8), an odd number with a middle tile, as many workgroups as CUs and one
# (b,h) more, the longest sequence and the first one past it; odd numbers of (b,h), which the XCDs take in runs, with grids that
# are and are not multiples of 8.
SHAPES = [(1, 1, 1), (1, 2, 31), (2, 1, 32), (1, 3, 33), (1, 2, 64), (1, 1, 65), (1, 8, 128), (2, 2, 129), (1, 16, 300),
          (1, 1, 1152), (1, 1, 1153), (9, 10, 544), (9, 10, 545),
          (1, 2, 224), (1, 2, 225), (1, 1, 257), (1, 1, 545), (16, 4, 256), (13, 5, 256), (1, 1, 2048), (1, 1, 2049),
          (1, 3, 257), (3, 3, 700), (1, 7, 1000)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("out_f32", [False, True])
def test_causal_forward(shape, out_f32):
    B, H, L = shape
    inp = U.random_problem(95, B, H, L, 128, 128, 256, 128, bf16=True, amp=1.5, w_shared=L == 129)
    dev = U.to_device(inp, True)
    out = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], out_dtype=torch.float32 if out_f32 else None)
    if B * H > 64:   # the oracle takes minutes there: the scan, which the other shapes' oracle holds to the same figure
        ref = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], out_dtype=torch.float32, sched={"cs_wgs": 256})
        want = ref.cpu().numpy()
    else:
        want = U.oracle_attn(inp, True)
    torch.cuda.synchronize()
    U.assert_close(out.float().cpu().numpy(), want, U.TOL["bf16"], f"{shape} f32 out={out_f32}")


@pytest.mark.parametrize("scan", [False, True])
def test_key_logits_that_rise_along_the_sequence(scan):
    inp = U.random_problem(96, 1, 2, 700, 128, 128, 256, 128, bf16=True, amp=1.0)
    inp["K"] = _drifting_keys(inp["K"], 8.0, 36, 6.0)
    _reround(inp, "K")
    dev = U.to_device(inp, True)
    # a schedule of the scan (its own number of workgroups) takes the call to it
    out = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], sched={"cs_wgs": 256} if scan else None)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy()
    assert np.isfinite(got).all()
    U.assert_close(got, U.oracle_attn(inp, True), U.TOL["bf16"], "rising key logits")


def test_identity_geometry_keeps_the_exact_key_norms():
    # M = None at d = 128: both forward passes stay on the kernels that take |k|^2 in fp32 (the same bits as with a schedule of theirs)
    inp = U.random_problem(97, 1, 2, 300, 128, 128, 256, 128, bf16=True, amp=1.5)
    dev = U.to_device(inp, True)
    for fn, sched in ((dk.dark_attn_fwd, {"kv_wgs": 256}), (dk.dark_attn_causal_fwd, {"cs_wgs": 256})):
        a = fn(dev["Q"], dev["K"], dev["V"], None, dev["W"])
        b = fn(dev["Q"], dev["K"], dev["V"], None, dev["W"], sched=sched)
        torch.cuda.synchronize()
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), fn.__name__


# two tiles of queries from both ends, also with the middle tile alone and with a ragged last tile; neighbours
@pytest.mark.parametrize("shape", [(1, 2, 300), (1, 1, 257), (1, 2, 129), (5, 13, 500)])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_infinite_values_stay_infinite(shape, value):
    # An infinite element of V is its column's result in every row that attends to it, whatever the sign of a kernel value's
    # second bf16; other columns, and rows of the tiles of 32 before it, are as without it.
    B, H, L = shape
    inp = U.random_problem(98, B, H, L, 128, 128, 256, 128, bf16=True, amp=1.0)
    dev = U.to_device(inp, True)
    want = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], out_dtype=torch.float32)
    V = dev["V"].clone()
    V[B - 1, H - 1, 70, 5] = value
    got = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], V, dev["M"], dev["W"], out_dtype=torch.float32)
    torch.cuda.synchronize()
    col = got[B - 1, H - 1, :, 5].clone()
    assert torch.equal(col[:64], want[B - 1, H - 1, :64, 5])
    seen = col[70:]   # (rows 64 to 69: a weight of zero times an infinity, NaN as in the scan)
    assert torch.isnan(seen).all() if value != value else (seen == value).all()
    got[B - 1, H - 1, :, 5] = want[B - 1, H - 1, :, 5]
    assert torch.equal(got, want)


# more (b,h) than a round of workgroups, where the tiles' features take more memory than the scan's states; one head, where they do not
@pytest.mark.parametrize("shape", [(8, 16, 448), (4, 16, 560), (1, 1, 300)])
def test_a_workspace_that_holds_the_scan_is_enough(shape):
    B, H, L = shape
    inp = U.random_problem(99, B, H, L, 128, 128, 256, 128, bf16=True, amp=1.5)
    dev = U.to_device(inp, True)
    args = [dev[n] for n in ("Q", "K", "V", "M", "W")]
    p, s = (dk.make_params(B, H, L, 128, 128, 256, 128, io_dtype=dk.DARK_BF16, sched=x) for x in (None, {"cs_wgs": 256}))
    full, scan = dk.workspace_bytes(p, dk.OP_ATTN_CAUSAL_FWD), dk.workspace_bytes(s, dk.OP_ATTN_CAUSAL_FWD)
    assert (full > scan) == (B * H > 1)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")

    def call(nbytes):
        out = torch.empty_like(dev["V"])
        st = dk.lib().dark_attn_causal_fwd(ctypes.byref(p), *(t.data_ptr() for t in args), out.data_ptr(), ws.data_ptr(), nbytes, dk._stream())
        torch.cuda.synchronize()
        return st, out.view(torch.int16)

    values = dk.dark_attn_causal_fwd(*args).view(torch.int16)
    by_scan = dk.dark_attn_causal_fwd(*args, sched={"cs_wgs": 256}).view(torch.int16)
    st, out = call(full)
    assert st == dk.DARK_OK and torch.equal(out, values)
    st, out = call(scan)
    assert st == dk.DARK_OK and torch.equal(out, by_scan if full > scan else values)
    assert call(scan - 256)[0] == dk.DARK_EWORKSPACE
