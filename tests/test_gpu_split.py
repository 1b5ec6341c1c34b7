"""GPU parity of the three-plane fp32 path (d = r = dv = 64, m a multiple of 64) at the edges of its tiles."""
import ctypes

import numpy as np
import pytest

import paper_2603_04127_amd as dk
from oracle import dark_oracle as O
from tests import parity_util as U
from tests.test_gpu_parity import _drifting_keys, _reround

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# B, H, L, m: a tile of 32 tokens and a workgroup of 128 queries at, one below and one above their edge; one, two, an
# odd number and many groups of 64 features; a last 256-feature block that is short; several slices of keys; enough
# rows that a wave has its 32 queries to itself (more than 1536 tiles).
SHAPES = [(1, 1, 1, 64), (1, 2, 31, 64), (2, 1, 32, 128), (1, 3, 33, 192), (1, 2, 127, 256), (2, 2, 128, 256),
          (1, 1, 129, 320), (1, 2, 1000, 512), (1, 1, 2085, 64), (8, 8, 801, 128)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("bf16", [False, True])
def test_bidirectional(shape, bf16):
    B, H, L, m = shape
    inp = U.random_problem(71, B, H, L, 64, 64, m, 64, bf16=bf16, amp=1.5, w_shared=m == 128)
    dev = U.to_device(inp, bf16)
    out = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32, out_dtype=torch.float32)
    torch.cuda.synchronize()
    # Three planes are fp32's 24 bits and the sums are fp32: the benchmark's fp32 tolerance, whatever the inputs are.
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, False), U.TOL["f32"], f"{shape} bf16={bf16}")


# One workgroup for all keys of 32 features: its longest sequences (at m = 64, 128, 256 and beyond) and the first ones past them, a
# wave with two tiles beside waves with one, one block of features too many, several batch entries of a head.
@pytest.mark.parametrize("shape", [(1, 1, 288, 64), (1, 1, 289, 64), (2, 2, 320, 128), (1, 2, 384, 256), (1, 2, 385, 256),
                                   (3, 2, 290, 320), (4, 8, 40, 256), (3, 11, 40, 256)])
@pytest.mark.parametrize("bf16", [False, True])
def test_keys_in_one_workgroup(shape, bf16):
    B, H, L, m = shape
    inp = U.random_problem(78, B, H, L, 64, 64, m, 64, bf16=bf16, amp=1.5, w_shared=m == 128)
    dev = U.to_device(inp, bf16)
    out = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32, out_dtype=torch.float32)
    torch.cuda.synchronize()
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, False), U.TOL["f32"], f"{shape} bf16={bf16}")


@pytest.mark.parametrize("bf16", [False, True])
def test_keys_in_one_workgroup_raise_their_shift(bf16):
    # key logits that rise along the sequence: a wave's second tile lies far above its first
    inp = U.random_problem(79, 1, 2, 380, 64, 64, 256, 64, bf16=bf16, amp=1.0)
    inp["K"] = _drifting_keys(inp["K"], 6.0, 41, 4.0)
    if bf16:
        _reround(inp, "K")
    dev = U.to_device(inp, bf16)
    out = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32, out_dtype=torch.float32)
    torch.cuda.synchronize()
    # logits of several hundred, whose fp32 rounding is a relative error of about 1e-4 (as in test_shifts_are_raised)
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, False), 5e-4, f"rising key logits bf16={bf16}")


@pytest.mark.parametrize("shape", [(9, 17, 70, 64), (3, 45, 33, 128), (2, 130, 20, 64)])
@pytest.mark.parametrize("bf16", [False, True])
def test_key_norms_of_short_sequences(shape, bf16):
    # the preparation's workgroups take the keys of a head in all batch entries: tiles of several entries in one workgroup, ragged
    # ones among them (more heads than k_sp_keys takes)
    B, H, L, m = shape
    inp = U.random_problem(84, B, H, L, 64, 64, m, 64, bf16=bf16, amp=1.5)
    dev = U.to_device(inp, bf16)
    out = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32, out_dtype=torch.float32)
    torch.cuda.synchronize()
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, False), U.TOL["f32"], f"{shape} bf16={bf16}")


def test_shifts_are_raised():
    # Logits that grow along the features: the queries' running shifts are raised from group to group (the keys' slices are of
    # one tile here, see test_shift_raised_from_far_below).  The logits reach several hundred, whose fp32 rounding (2^-24 of
    # them, times a few terms) is a relative error of about 1e-4.
    inp = U.random_problem(72, 1, 2, 400, 64, 64, 256, 64, amp=2.0)
    inp["K"] *= np.linspace(0.1, 3.0, 400, dtype=np.float32)[None, None, :, None]
    inp["W"] *= np.linspace(0.2, 4.0, 256, dtype=np.float32)[None, :, None]
    dev = U.to_device(inp, False)
    out = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32)
    torch.cuda.synchronize()
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, False), 5e-4, "growing logits")


@pytest.mark.parametrize("shape", SHAPES[:8])
@pytest.mark.parametrize("bf16", [False, True])
def test_bidirectional_backward(shape, bf16):
    B, H, L, m = shape
    inp = U.random_problem(73, B, H, L, 64, 64, m, 64, bf16=bf16, amp=1.5, w_shared=m == 128, backward=True)
    dev = U.to_device(inp, bf16)
    g = dk.dark_attn_bwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], dev["dOut"], False, path=dk.PATH_F32)
    torch.cuda.synchronize()
    want = dict(zip(("dQ", "dK", "dV", "dM"), U.oracle_bwd(inp, False)))
    for k in want:   # the fp32 backward's tolerance, on either input type (gradients are fp32)
        if L == 1 and k != "dV":
            # out = v whatever Q, K and M are: these gradients vanish identically, as differences of equal terms of
            # order |dOut| |v| |A| < 100 in fp32 (2^-24 of that, over the sums, stays below 1e-4).
            assert np.abs(g[k].cpu().numpy()).max() < 1e-4
            continue
        U.assert_close(g[k].cpu().numpy(), want[k], 2e-4, f"{k} {shape} bf16={bf16}")


# bf16 inputs and m = 256, where eight waves share the features of a tile: slices of one to five tiles, last tiles of 1, 8 and 32 rows;
# `spread`: the row maxima of the waves lie far apart (the logits' fp32 rounding grows with them, see test_shifts_are_raised).
@pytest.mark.parametrize("shape,spread", [((4, 32, 97), False), ((2, 64, 200), False), ((3, 85, 160), False), ((1, 2, 300), True)])
def test_bidirectional_backward_of_shared_tiles(shape, spread):
    B, H, L = shape
    inp = U.random_problem(94, B, H, L, 64, 64, 256, 64, bf16=True, amp=1.5, backward=True)
    if spread:
        inp["W"] *= np.linspace(0.2, 2.0, 256, dtype=np.float32)[None, :, None]
    dev = U.to_device(inp, True)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], dev["dOut"], False)
    g = dk.dark_attn_bwd(*args)
    alone = {k: dk.dark_attn_bwd(*args, need=(k,))[k] for k in g}
    torch.cuda.synchronize()
    want = dict(zip(("dQ", "dK", "dV", "dM"), U.oracle_bwd(inp, False)))
    for k in want:
        U.assert_close(g[k].cpu().numpy(), want[k], 5e-4 if spread else 2e-4, f"{k} {shape}")
        assert torch.equal(g[k], alone[k])


@pytest.mark.parametrize("shape", [(1, 1, 2500), (2, 3, 777)])
def test_dq_alone_forms_no_states(shape):
    # bf16 inputs and m = 256: the query pass of dQ alone leaves out the states of the key side (and cuts a long sequence into more
    # slices), with the same bits.  What it does not write of its workspace is at least the room of one state a slice.
    B, H, L = shape
    inp = U.random_problem(96, B, H, L, 64, 64, 256, 64, bf16=True, amp=1.5, backward=True)
    dev = U.to_device(inp, True)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], dev["dOut"])
    full = dk.dark_attn_bwd(*args, False)
    p = dk.make_params(B, H, L, 64, 64, 256, 64, io_dtype=dk.DARK_BF16)
    ws = torch.full((dk.workspace_bytes(p, dk.OP_ATTN_BWD) // 4 + 64,), 0x7f123456, dtype=torch.int32, device="cuda")
    at = (-ws.data_ptr()) % 256 // 4
    dQ = torch.empty(B, H, L, 64, device="cuda")
    null = ctypes.c_void_p(None)
    status = dk.lib().dark_attn_bwd(ctypes.byref(p), 0, *(x.data_ptr() for x in args), dQ.data_ptr(), null, null, null,
                                    ws[at:].data_ptr(), 4 * (ws.numel() - at), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert status == 0
    assert torch.equal(dQ, full["dQ"])
    slices = -(-L // (32 * -(-L // (32 * min(64, 256 // (B * H))))))
    assert (ws == 0x7f123456).sum().item() >= B * H * slices * 256 * 64


@pytest.mark.parametrize("m,bf16", [(64, False), (256, False), (128, True), (256, True)])
def test_gradients_of_a_large_loss(m, bf16):
    # The gradients are linear in dOut, by a power of two exactly, while they and the sums they are made of stay in the fp32 range:
    # here the largest come to 2^121.  (1e-6: what the unscaled problem loses to planes below the normal range.)
    inp = U.random_problem(95, 1, 2, 1100, 64, 64, m, 64, bf16=bf16, amp=1.5, backward=True)
    dev = U.to_device(inp, bf16)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"])
    g = dk.dark_attn_bwd(*args, dev["dOut"], False, path=dk.PATH_F32)
    big = dk.dark_attn_bwd(*args, dev["dOut"] * 2.0 ** 112, False, path=dk.PATH_F32)
    torch.cuda.synchronize()
    for k in g:
        assert torch.isfinite(big[k]).all(), k
        diff = big[k].double() * 2.0 ** -112 - g[k].double()
        assert diff.norm() <= 1e-6 * g[k].double().norm(), k


@pytest.mark.parametrize("need", [("dQ",), ("dV",), ("dK",), ("dM",), ("dW",)])
def test_backward_single_gradients(need):
    # Each gradient alone is bit for bit what it is among the others.
    inp = U.random_problem(74, 2, 2, 200, 64, 64, 128, 64, amp=1.0, backward=True)
    dev = U.to_device(inp, False)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], dev["dOut"], False)
    full = dk.dark_attn_bwd(*args, need=("dQ", "dK", "dV", "dM", "dW"))
    one = dk.dark_attn_bwd(*args, need=need)
    torch.cuda.synchronize()
    assert torch.equal(full[need[0]], one[need[0]])


# chunks of 32 positions: one below, at and above an edge, up to the 32 chunks of one pass of the scan, every wave count
CAUSAL_SHAPES = [(1, 1, 1, 64), (1, 2, 31, 128), (2, 1, 32, 64), (1, 3, 33, 192), (1, 2, 255, 256), (2, 2, 257, 128),
                 (1, 1, 1000, 256), (2, 3, 290, 64)]


@pytest.mark.parametrize("shape", CAUSAL_SHAPES)
@pytest.mark.parametrize("bf16", [False, True])
def test_causal(shape, bf16):
    B, H, L, m = shape
    inp = U.random_problem(75, B, H, L, 64, 64, m, 64, bf16=bf16, amp=1.5, w_shared=m == 128, backward=True)
    dev = U.to_device(inp, bf16)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"])
    out = dk.dark_attn_causal_fwd(*args, path=dk.PATH_F32, out_dtype=torch.float32)
    g = dk.dark_attn_bwd(*args, dev["dOut"], True, path=dk.PATH_F32)
    torch.cuda.synchronize()
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, True), U.TOL["f32"], f"{shape} bf16={bf16}")
    want = dict(zip(("dQ", "dK", "dV", "dM"), U.oracle_bwd(inp, True)))
    for k in want:
        if L == 1 and k != "dV":   # vanish identically, see above
            assert np.abs(g[k].cpu().numpy()).max() < 1e-4
            continue
        U.assert_close(g[k].cpu().numpy(), want[k], 2e-4, f"{k} {shape} bf16={bf16}")


def test_causal_single_gradients():
    inp = U.random_problem(76, 2, 2, 200, 64, 64, 128, 64, amp=1.0, backward=True)
    dev = U.to_device(inp, False)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], dev["dOut"], True)
    full = dk.dark_attn_bwd(*args, need=("dQ", "dK", "dV", "dM", "dW"))
    for k in full:
        one = dk.dark_attn_bwd(*args, need=(k,))
        torch.cuda.synchronize()
        assert torch.equal(full[k], one[k]), k


def test_causal_key_logits_rise_and_fall():
    # Keys that grow along the sequence and shrink again, logits of several hundred (fp32 rounding of about 1e-4): the rows of
    # the growing half.  (The norm term holds the rise of a feature's largest logit at some 27 nats; see
    # test_causal_drift_beyond_the_exponent_range.)
    inp = U.random_problem(77, 1, 2, 500, 64, 64, 128, 64, amp=1.0)
    ramp = np.concatenate([np.linspace(0.05, 4.0, 250), np.linspace(4.0, 0.05, 250)]).astype(np.float32)
    inp["K"] *= ramp[None, None, :, None]
    inp["W"] *= 2.0
    dev = U.to_device(inp, False)
    out = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32)
    torch.cuda.synchronize()
    got, want = out.cpu().numpy(), U.oracle_attn(inp, True)
    U.assert_close(got[:, :, :250], want[:, :, :250], 5e-4, "rising")


@pytest.mark.parametrize("bf16", [False, True])
def test_static_scratch_falls_back_to_the_general_kernels(bf16):
    # 960 features of three positions: the three-plane kernels need more than the static scratch, the general ones do not,
    # and serve such a problem on either entry point: the same bits.
    inp = U.random_problem(78, 4, 12, 3, 64, 64, 960, 64, bf16=bf16, amp=1.0)
    dev = U.to_device(inp, bf16)
    p = dk.make_params(4, 12, 3, 64, 64, 960, 64, io_dtype=dk.DARK_BF16 if bf16 else dk.DARK_F32, path=dk.PATH_F32)
    assert dk.workspace_bytes(p, dk.OP_ATTN_FWD) <= dk.static_scratch_bytes()
    out = torch.empty_like(dev["V"])
    dk.dark_attn_fwd_static(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], out, path=dk.PATH_F32)
    ref = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    U.assert_close(out.float().cpu().numpy(), U.oracle_attn(inp, False), U.TOL["bf16" if bf16 else "f32"], f"static bf16={bf16}")


@pytest.mark.parametrize("L", [45, 801])
def test_rows_past_the_end_stay_out_whatever_the_norms(L):
    # Every key's norm term lies far above any fixed stand-in for the norm of the rows past the end of a tile: the output is
    # the value of the shortest key, the others' features vanish.
    inp = U.random_problem(79, 1, 2, L, 64, 64, 128, 64, amp=1.0)
    inp["Q"] *= np.float32(1e-16)
    inp["K"] *= np.float32(1e16)
    for h in range(2):
        x = inp["K"][0, h].astype(np.float64) @ inp["M"][h].T.astype(np.float64)
        n = np.square(x).sum(-1) / 16.0
        assert n.min() > 1e31 and n.max() < 1e36
    dev = U.to_device(inp, False)
    out = dk.dark_attn_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32)
    torch.cuda.synchronize()
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, False), U.TOL["f32"], f"huge norms L={L}")


def _first_tile_far_below(amp, bf16):
    # 64 (b,h) of 801 keys at m = 128: slices of 128 keys, four tiles each.  The first tile of every slice holds keys `amp`
    # times as long, whose logits lie far below those of the tiles after it.
    inp = U.random_problem(80, 8, 8, 801, 64, 64, 128, 64, bf16=bf16, amp=1.0, backward=True)
    first = (np.arange(801) % 128) < 32
    inp["K"][:, :, first] *= np.float32(amp)
    if bf16:
        _reround(inp, "K")
    return inp, first


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("amp", [30.0, 1000.0, 1e25])
def test_shift_raised_from_far_below(amp, bf16):
    # The running shift starts at the first tile's logits (-1e3, -1e6; -inf at 1e25, where the norm term overflows fp32) and
    # is raised by the second tile, whose logits are of order ten and must keep their precision: the fp32 tolerance.
    inp, first = _first_tile_far_below(amp, bf16)
    dev = U.to_device(inp, bf16)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"])
    out = dk.dark_attn_fwd(*args, path=dk.PATH_F32, out_dtype=torch.float32)
    g = dk.dark_attn_bwd(*args, dev["dOut"], False, path=dk.PATH_F32)
    torch.cuda.synchronize()
    for b, h in ((0, 0), (7, 7)):
        Q, K, V, M, W = U.head(inp, b, h)
        lg = O.logits(K, M, W) / np.log(2.0)
        assert (lg[~first][:96].max(0) - lg[first][:32].max(0)).min() > 20.0   # every feature's shift is raised
        U.assert_close(out[b, h].cpu().numpy(), O.attn_bidir(Q, K, V, M, W), U.TOL["f32"], f"out {b},{h} x{amp:g}")
        if amp < 1e20:
            dQ, dK, dV, _ = O.attn_bwd_brute(Q, K, V, M, W, inp["dOut"][b, h], False)
            for name, want in (("dQ", dQ), ("dV", dV), ("dK", dK)):
                U.assert_close(g[name][b, h].cpu().numpy(), want, 2e-4, f"{name} {b},{h} x{amp:g}")


def test_causal_keys_whose_norm_overflows():
    # A chunk whose keys' norm terms overflow fp32: their features vanish, and the rows after it are those of the other keys.
    inp = U.random_problem(81, 1, 2, 300, 64, 64, 128, 64, amp=1.0)
    inp["K"][:, :, :32] *= np.float32(1e25)
    dev = U.to_device(inp, False)
    out = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], path=dk.PATH_F32)
    torch.cuda.synchronize()
    want = np.stack([[O.attn_brute(*U.head(inp, 0, h), True) for h in range(2)]])
    U.assert_close(out[:, :, 32:].cpu().numpy(), want[:, :, 32:], U.TOL["f32"], "after the chunk")


@pytest.mark.parametrize("shape,causal,bound", [
    # bound: error of dV on the general fp32 kernels for this problem (2-norm, mean of the seeds), which the three-plane kernels
    # must not exceed; they show 0.6 to 0.75e-6 (1.04 to 1.32e-6 when their logits were summed in one accumulator)
    ((1, 2, 600, 64), False, 1.11e-6), ((1, 2, 127, 256), False, 1.19e-6),
    ((1, 2, 600, 64), True, 1.03e-6), ((1, 2, 127, 256), True, 0.94e-6)])
def test_value_gradients_are_as_precise_as_on_the_general_kernels(shape, causal, bound):
    B, H, L, m = shape
    errs = []
    for seed in range(173, 177):
        inp = U.random_problem(seed, B, H, L, 64, 64, m, 64, amp=1.5, backward=True)
        dev = U.to_device(inp, False)
        g = dk.dark_attn_bwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], dev["dOut"], causal, need=("dV",))
        torch.cuda.synchronize()
        want = U.oracle_bwd(inp, causal)[2]
        errs.append(np.linalg.norm(g["dV"].cpu().numpy() - want) / np.linalg.norm(want))
    assert np.mean(errs) <= bound, errs


@pytest.mark.parametrize("B,H,L,m,bf16", [(3, 5, 32768, 256, False), (1, 14, 32768, 256, True), (7, 2, 65536, 128, False)])
def test_causal_forward_in_groups(B, H, L, m, bf16):
    # More chunk states than one group holds: whole batch entries with a smaller last group, heads of one entry, both weights.
    g = torch.Generator(device="cuda").manual_seed(5)
    t = torch.bfloat16 if bf16 else torch.float32
    Q, K, V = (torch.randn(B, H, L, 64, generator=g, device="cuda").to(t) for _ in range(3))
    M = torch.eye(64, device="cuda") + 0.1 * torch.randn(H, 64, 64, generator=g, device="cuda")
    W = torch.randn(*((m, 64) if bf16 else (H, m, 64)), generator=g, device="cuda")
    out = dk.dark_attn_causal_fwd(Q, K, V, M, W, path=dk.PATH_F32)
    for b, h in ((0, 0), (B - 1, H - 1), (B // 2, H // 2)):
        one = [x[b:b + 1, h:h + 1].contiguous() for x in (Q, K, V)]
        ref = dk.dark_attn_causal_fwd(*one, M[h:h + 1].contiguous(), W if bf16 else W[h:h + 1].contiguous(), path=dk.PATH_F32)
        torch.cuda.synchronize()
        assert torch.equal(out[b, h], ref[0, 0]), (b, h)


def test_chunks_shorter_than_the_kernels_own_keep_their_range():
    # chunk = 16: the first sixteen keys lie 100 nats and more below the next sixteen, in every feature.  Under one shift for
    # all 32 their features would vanish and the first rows come out 0/0; under a shift per 16 they are ordinary.
    inp = U.random_problem(82, 1, 2, 200, 64, 64, 128, 64, amp=1.0, backward=True)
    inp["W"] *= np.float32(0.3)
    for h in range(2):
        x = inp["K"][0, h, :16].astype(np.float64)
        n = np.square(x @ inp["M"][h].T.astype(np.float64)).sum(-1) / 16.0
        inp["K"][0, h, :16] = x * np.sqrt(140.0 / n)[:, None]
        lg = O.logits(inp["K"][0, h], inp["M"][h], inp["W"][h])
        assert (lg[16:32].max(0) - lg[:16].max(0)).min() > 90.0 and np.ptp(lg[:16], axis=0).max() < 60.0
    dev = U.to_device(inp, False)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"])
    out = dk.dark_attn_causal_fwd(*args, chunk=16)
    g = dk.dark_attn_bwd(*args, dev["dOut"], True, chunk=16)
    torch.cuda.synchronize()
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, True), U.TOL["f32"], "chunk=16")
    for name, want in zip(("dQ", "dK", "dV", "dM"), U.oracle_bwd(inp, True)):
        U.assert_close(g[name].cpu().numpy(), want, 2e-4, f"{name} chunk=16")


@pytest.mark.parametrize("chunk", [16, 32, 100, 512])
def test_causal_chunk_is_only_a_schedule(chunk):
    # below 32 positions the general kernels, from 32 on the chunked ones
    inp = U.random_problem(83, 1, 2, 333, 64, 64, 128, 64, amp=1.5)
    dev = U.to_device(inp, False)
    out = dk.dark_attn_causal_fwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], chunk=chunk)
    torch.cuda.synchronize()
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, True), U.TOL["f32"], f"chunk={chunk}")


# more than the 32 chunks of one pass of the scan: what is carried from pass to pass, and a last pass of one or two chunks
@pytest.mark.parametrize("shape", [(1, 2, 1025, 64), (1, 1, 2085, 128)])
@pytest.mark.parametrize("bf16", [False, True])
def test_causal_scan_of_several_passes(shape, bf16):
    test_causal(shape, bf16)


def test_causal_drift_beyond_the_exponent_range():
    # Every feature's key logits rise by more than 90 nats over 600 positions and fall again, by less than 40 inside a chunk:
    # running shifts, the factors between chunks (both directions) and two passes of the scan.  All rows, all gradients, on the
    # scale of the tensor (logits of two hundred: fp32 rounding of up to 1e-4).
    inp = U.random_problem(84, 1, 2, 1200, 64, 64, 64, 64, amp=1.0, backward=True)
    K = _drifting_keys(inp["K"], 8.0, 84, 6.0)
    inp["K"] = np.concatenate([K[:, :, ::2], K[:, :, ::-2]], axis=2)
    for h in range(2):
        lg = O.logits(inp["K"][0, h], inp["M"][h], inp["W"][h])
        tiles = [lg[i:i + 32] for i in range(0, 1200, 32)]
        assert (lg.max(0) - tiles[0].max(0)).min() > 90.0 and (lg.max(0) - tiles[-1].max(0)).min() > 90.0
        assert max(np.ptp(t, axis=0).max() for t in tiles) < 40.0
    dev = U.to_device(inp, False)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"])
    out = dk.dark_attn_causal_fwd(*args)
    g = dk.dark_attn_bwd(*args, dev["dOut"], True)
    torch.cuda.synchronize()
    U.assert_close(out.cpu().numpy(), U.oracle_attn(inp, True), 5e-4, "drift")
    for name, want in zip(("dQ", "dK", "dV", "dM"), U.oracle_bwd(inp, True)):
        U.assert_close_grad(g[name].cpu().numpy(), want, 5e-4, f"{name} drift")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("shared", [False, True])
def test_gradient_of_the_draws(causal, shared):
    inp = U.random_problem(85, 2, 3, 150, 64, 64, 128, 64, w_shared=shared, amp=1.5, backward=True)
    dev = U.to_device(inp, False)
    g = dk.dark_attn_bwd(dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"], dev["dOut"], causal, need=("dW",))
    torch.cuda.synchronize()
    want = np.zeros(inp["W"].shape)
    for b in range(2):
        for h in range(3):
            dW = O.attn_bwd_brute(*U.head(inp, b, h), inp["dOut"][b, h], causal, with_dW=True)[4]
            want[... if shared else h] += dW
    U.assert_close(g["dW"].cpu().numpy().reshape(-1, 64), want.reshape(-1, 64), 2e-4, f"dW shared={shared} causal={causal}")


# The lines of the dispatch of many short sequences, one position below and one above: B, H, L, m, causal, bf16
SHORT = [(48, 16, 128, 256, True, False), (48, 16, 129, 256, True, False), (48, 16, 128, 256, True, True),
         (48, 16, 129, 256, True, True), (128, 16, 72, 128, True, False), (128, 16, 73, 128, True, False),
         (128, 16, 48, 128, True, True), (128, 16, 49, 128, True, True), (45, 16, 20, 256, False, False),
         (45, 16, 21, 256, False, False), (257, 8, 8, 128, False, False), (257, 8, 9, 128, False, False),
         (129, 8, 8, 896, False, True), (129, 8, 9, 896, False, True)]


@pytest.mark.parametrize("shape", SHORT)
def test_many_heads_of_short_sequences(shape):
    # What a head gets among many (either kernel, by the number of heads) is what it gets in a problem of its own.
    B, H, L, m, causal, bf16 = shape
    inp = U.random_problem(83, B, H, L, 64, 64, m, 64, bf16=bf16, amp=1.0, w_shared=True, backward=True)
    few = {k: v[-1:] if k in ("Q", "K", "V", "dOut") else v for k, v in inp.items()}
    dev = U.to_device(inp, bf16)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"])
    fwd = dk.dark_attn_causal_fwd if causal else dk.dark_attn_fwd
    out = fwd(*args, path=dk.PATH_F32, out_dtype=torch.float32)
    g = dk.dark_attn_bwd(*args, dev["dOut"], causal, path=dk.PATH_F32)
    torch.cuda.synchronize()
    U.assert_close(out[-1:].cpu().numpy(), U.oracle_attn(few, causal), U.TOL["f32"], f"{shape}")
    want = dict(zip(("dQ", "dK", "dV"), U.oracle_bwd(few, causal)))
    for k in want:
        U.assert_close(g[k][-1:].cpu().numpy(), want[k], 2e-4, f"{k} {shape}")


def test_vanished_rows_leave_later_keys_alone():
    # The first chunk's keys are so long that its first rows see none that counts (0/0): a key after such a row does not depend on it.
    inp = U.random_problem(97, 1, 4, 100, 64, 64, 64, 64, amp=1.5, backward=True)
    inp["K"][:, :, :32] *= np.float32(1e3)
    dev = U.to_device(inp, False)
    args = (dev["Q"], dev["K"], dev["V"], dev["M"], dev["W"])
    out = dk.dark_attn_causal_fwd(*args, path=dk.PATH_F32)
    dK = dk.dark_attn_bwd(*args, dev["dOut"], True, path=dk.PATH_F32)["dK"]
    torch.cuda.synchronize()
    seen = 0
    for h in range(4):
        gone = torch.nonzero(~torch.isfinite(out[0, h]).all(-1)).flatten().tolist()
        after = gone[-1] + 1 if gone else 0
        assert after <= 32
        seen += bool(gone) and after < 32
        assert torch.isfinite(dK[0, h, after:]).all(), f"head {h}: rows up to {after - 1} have vanished"
    assert seen   # some head has such rows and keys after them in the chunk
