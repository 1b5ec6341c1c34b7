"""dark_decode_step: the causal recurrence one token at a time against the oracle's causal attention."""
import numpy as np
import pytest

import paper_2603_04127_amd as dk
from oracle import dark_oracle as O
from tests import parity_util as U

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _np(t):
    return t.detach().float().cpu().numpy()


@pytest.mark.parametrize("shape", [
    # B, H, L,  d,  r,  m,   dv, bf16, shared W, identity
    (2, 3, 70, 24, 16, 80,  40, False, False, False),   # a thread per column
    (1, 2, 50, 7,  5,  33,  3,  False, False, False),
    (2, 2, 90, 64, 64, 256, 64, True,  False, False),   # 16-byte state accesses
    (1, 2, 40, 64, 64, 256, 64, True,  True,  False),
    (1, 2, 40, 32, 32, 64,  16, False, False, True),
])
def test_decode_matches_causal_attention(shape):
    B, H, L, d, r, m, dv, bf16, shared, ident = shape
    inp = U.random_problem(81, B, H, L, d, r, m, dv, bf16=bf16, w_shared=shared, amp=2.0)
    if ident:
        inp["M"] = np.broadcast_to(np.eye(d, dtype=np.float32), (H, d, d)).copy()
    dev = U.to_device(inp, bf16)
    state = dk.decode_state(B, H, m, dv)
    outs = []
    for t in range(L):
        outs.append(dk.dark_decode_step(dev["Q"][:, :, t].contiguous(), dev["K"][:, :, t].contiguous(),
                                        dev["V"][:, :, t].contiguous(), None if ident else dev["M"], dev["W"], state))
    torch.cuda.synchronize()
    got = _np(torch.stack(outs, dim=2))
    want = U.oracle_attn(inp, True)
    e = U.assert_close(got, want, U.TOL["bf16" if bf16 else "f32"], f"decode {shape}")
    print(f"decode {shape}: {U.fmt(e)}")
    # the state is the causal state: z = sum_l phi(k_l) under the stored shift
    S, z, c = state
    for b in range(B):
        for h in range(H):
            Q, K, V, M, W = U.head(inp, b, h)
            lg = O.logits(K, M, W)
            zw = np.exp(lg - float(c[b, h])).sum(0)
            assert abs(float(c[b, h]) - lg.max()) <= 1e-3 * max(1.0, abs(lg.max()))
            assert np.abs(_np(z[b, h]) - zw).max() <= 2e-3 * zw.max()


def test_decode_rescales_when_the_key_logits_rise():
    """Keys whose logits grow by tens of nats from token to token: every step raises the shift."""
    inp = U.random_problem(82, 1, 2, 60, 24, 16, 80, 40, bf16=False, amp=1.0)
    ramp = np.linspace(4.0, 0.5, 60, dtype=np.float32)[None, None, :, None]
    inp["K"] = inp["K"] * ramp
    dev = U.to_device(inp, False)
    state = dk.decode_state(1, 2, 80, 40)
    outs = [dk.dark_decode_step(dev["Q"][:, :, t].contiguous(), dev["K"][:, :, t].contiguous(),
                                dev["V"][:, :, t].contiguous(), dev["M"], dev["W"], state) for t in range(60)]
    torch.cuda.synchronize()
    U.assert_close(_np(torch.stack(outs, dim=2)), U.oracle_attn(inp, True), U.TOL["f32"], "decode, rising logits")


@pytest.mark.parametrize("shape", [
    # B, H, L,  d,   m,   bf16, identity: every instantiation of the kernel for d = r = dv in {64, 128}
    (2, 2, 30, 64,  128, False, False),
    (1, 2, 30, 64,  256, False, True),
    (1, 2, 30, 64,  512, True,  False),
    (2, 1, 30, 128, 128, True,  False),
    (1, 3, 30, 128, 256, False, False),
    (1, 2, 30, 128, 256, True,  True),
])
def test_decode_row_kernel(shape):
    B, H, L, d, m, bf16, ident = shape
    inp = U.random_problem(83, B, H, L, d, d, m, d, bf16=bf16, amp=1.5, w_shared=m == 128)
    if ident:
        inp["M"] = np.broadcast_to(np.eye(d, dtype=np.float32), (H, d, d)).copy()
    dev = U.to_device(inp, bf16)
    S, z, c = state = dk.decode_state(B, H, m, d)
    outs = [dk.dark_decode_step(dev["Q"][:, :, t].contiguous(), dev["K"][:, :, t].contiguous(),
                                dev["V"][:, :, t].contiguous(), None if ident else dev["M"], dev["W"], state)
            for t in range(L)]
    torch.cuda.synchronize()
    U.assert_close(_np(torch.stack(outs, dim=2)), U.oracle_attn(inp, True), U.TOL["bf16" if bf16 else "f32"], f"{shape}")
    for b in range(B):
        for h in range(H):
            _, K, V, M, W = U.head(inp, b, h)
            phi = np.exp(O.logits(K, M, W) - float(c[b, h]))
            assert np.abs(_np(z[b, h]) - phi.sum(0)).max() <= 1e-4 * phi.sum(0).max()     # the fp32 tolerance
            Sw = phi.T @ V.astype(np.float64)
            assert np.abs(_np(S[b, h]) - Sw).max() <= 1e-4 * np.abs(Sw).max()


def test_decode_step_of_more_heads_than_one_launch_of_the_row_kernel_takes():
    # 2^22 (b,h) of 1024 threads are more than a launch has; the general kernel's 256 fit.  137 GB of state.
    B, d, m = 1 << 22, 64, 128
    if torch.cuda.mem_get_info()[0] < 160e9:
        pytest.skip("needs 150 GB of device memory")
    g = torch.Generator(device="cuda").manual_seed(6)
    q, k, v = (torch.randn(B, 1, d, generator=g, device="cuda") for _ in range(3))
    state = dk.decode_state(B, 1, m, d)
    out = dk.dark_decode_step(q, k, v, None, torch.randn(1, m, d, generator=g, device="cuda"), state)
    torch.cuda.synchronize()
    assert torch.allclose(out, v, rtol=1e-5, atol=1e-6)   # one token: its own value
    del state, out
    torch.cuda.empty_cache()
