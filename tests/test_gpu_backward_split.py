"""GPU parity of the split backward (the calls with a workspace).

Tiles that do not fill the GPU share their sums out over several workgroups and
another kernel adds the parts up (the sums of fp32 parts are ordered otherwise
than those of the call without: not the same bits). Each geometry runs with the
workspace (the binding's ordinary call) and without (the C entry point that takes none), and
both are held to the oracle within the bound of the backward's other tests,
|err| <= 2e-2 x RMS + 2^-8 |g| + 2^-8 m with m the sum of absolute products.
"""
import ctypes

import numpy as np
import pytest
import torch

from gpu_helpers import say
from oracle import ChunkGeometry, full_sequence_attention_backward
from synth import bf16_bits_to_f32, f32_to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tm():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2506_03099_amd import tm as binding
    binding.lib()
    return binding


def _bf16(rng, shape, norm):
    x = rng.standard_normal(shape).astype(np.float32)
    if norm:
        x /= np.sqrt(np.mean(x * x, axis=-1, keepdims=True))
    bits = f32_to_bf16_bits(x)
    return bf16_bits_to_f32(bits), torch.from_numpy(bits.view(np.int16)).view(torch.bfloat16).cuda()


# B, H, D, T, C, R, W, frames, splits?
CASES = [
    (1, 1, 128, 100, 3, 1, 1, 11, True),   # dK/dV of c_0 and of the chunks
    (1, 2, 64, 70, 7, 2, 0, 16, True),     # D = 64, ragged tiles, two chunks
    (1, 3, 128, 131, 1, 1, 3, 9, True),    # the window reaches past the last chunk: short query ranges
    (2, 2, 128, 300, 2, 3, 1, 3, True),    # c_0 alone: every tile is one of its own
    (1, 24, 64, 130, 3, 1, 1, 13, True),   # only c_0's dK/dV
    (1, 2, 128, 50, 2, 1, 1, 5, False),    # too short
    (1, 1, 128, 64, 7, 1, 1, 15, True),    # all three; c_0's query tile has one key tile: an empty part
]


@pytest.mark.parametrize("B,H,D,T,C,R,W,frames,splits", CASES)
def test_split_backward_matches_oracle(tm, B, H, D, T, C, R, W, frames, splits):
    say(f"split backward: B={B} H={H} D={D} T={T} C={C} R={R} W={W} frames={frames}")
    rng = np.random.default_rng(T)
    L = frames * T
    (q, qd), (k, kd), (v, vd) = (_bf16(rng, (B, L, H, D), i < 2) for i in range(3))
    do, dod = _bf16(rng, (B, L, H, D), False)
    desc = tm.make_desc(B, H, D, T, C, R, W, "bf16")
    d = ctypes.byref(desc)
    assert (tm.lib().tm_sparse_causal_attn_bwd_workspace(d, frames) > 0) == splits
    lse = torch.empty(B, H, L, dtype=torch.float32, device="cuda")
    o = tm.tm_sparse_causal_attn_fwd(desc, qd, -1, k=kd, v=vd, n_frames=frames, lse=lse)
    got = {"workspace": tm.tm_sparse_causal_attn_bwd(desc, frames, qd, kd, vd, o, lse, dod)}
    again = tm.tm_sparse_causal_attn_bwd(desc, frames, qd, kd, vd, o, lse, dod)
    plain = [torch.full_like(qd, float("nan")) for _ in range(3)]
    delta = torch.empty_like(lse)
    p = tm._ptr
    st = tm.lib().tm_sparse_causal_attn_bwd(d, frames, p(qd), p(kd), p(vd), p(o), p(lse), p(dod), p(delta),
                                            *map(p, plain), tm._stream(None))
    assert st == tm.TM_OK, tm.tm_last_error()
    got["plain"] = plain
    torch.cuda.synchronize()
    heads = sorted({0, H - 1})
    want, mags = full_sequence_attention_backward(q, k, v, do, ChunkGeometry(T, C, R, W), heads=heads,
                                                  magnitudes=True)
    for route, grads in got.items():
        for name, g, w, m in zip(("dq", "dk", "dv"), grads, want, mags):
            g = g.float().cpu().numpy()[:, :, heads].astype(np.float64)
            assert np.all(np.isfinite(g)), f"{route} {name}"
            bound = 2e-2 * np.sqrt(np.mean(w ** 2)) + 2.0 ** -8 * np.abs(w) + 2.0 ** -8 * m
            worst = float(np.max(np.abs(g - w) / bound))
            say(f"  {route} {name}: worst err / bound = {worst:.3f}")
            assert worst <= 1.0, f"{route} {name}: error {worst:.3f} x the bound"
    for a, b in zip(got["workspace"], again):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


def test_split_backward_workspace_is_checked(tm):
    desc = tm.make_desc(1, 1, 128, 100, 3, 1, 1, "bf16")
    d, p = ctypes.byref(desc), tm._ptr
    n = tm.lib().tm_sparse_causal_attn_bwd_workspace(d, 11)
    assert n > 0
    q, k, v, o, do, dq, dk, dv = (torch.zeros((1, 1100, 1, 128), dtype=torch.bfloat16, device="cuda") for _ in range(8))
    lse, delta = (torch.zeros((1, 1, 1100), dtype=torch.float32, device="cuda") for _ in range(2))
    call = lambda ws, size: tm.lib().tm_sparse_causal_attn_bwd_ws(  # noqa: E731
        d, 11, p(q), p(k), p(v), p(o), p(lse), p(do), p(delta), p(dq), p(dk), p(dv), ws, size, tm._stream(None))
    ws = torch.empty(n + 16, dtype=torch.uint8, device="cuda")
    assert call(p(ws), n) == tm.TM_OK
    assert call(p(ws), n - 1) == tm.TM_OK  # too small: not used
    assert call(None, 0) == tm.TM_OK
    assert call(p(ws) + 8, n) == tm.TM_E_ARG  # misaligned
    assert call(p(ws) + (1 << 40), n) == tm.TM_E_ARG  # not device memory
    big = torch.zeros(n + (1 << 20), dtype=torch.uint8, device="cuda")
    q = big[:1100 * 256].view(torch.bfloat16)  # the workspace covers an input
    assert call(p(big), n) == tm.TM_E_ARG
    torch.cuda.synchronize()


def test_split_backward_with_plain_addresses(tm):
    # q given as an address, the outputs as tensors: the call without a workspace
    desc = tm.make_desc(1, 1, 128, 100, 3, 1, 1, "bf16")
    rng = np.random.default_rng(5)
    q, k, v, do = (_bf16(rng, (1, 1100, 1, 128), i < 2)[1] for i in range(4))
    d = ctypes.byref(desc)
    assert tm.lib().tm_sparse_causal_attn_bwd_workspace(d, 11) > 0
    lse = torch.empty(1, 1, 1100, dtype=torch.float32, device="cuda")
    o = tm.tm_sparse_causal_attn_fwd(desc, q, -1, k=k, v=v, n_frames=11, lse=lse)
    p = tm._ptr
    delta = torch.empty_like(lse)
    want, got = ([torch.full_like(q, float("nan")) for _ in range(3)] for _ in range(2))
    st = tm.lib().tm_sparse_causal_attn_bwd(d, 11, p(q), p(k), p(v), p(o), p(lse), p(do), p(delta),
                                            *map(p, want), tm._stream(None))
    assert st == tm.TM_OK, tm.tm_last_error()
    tm.tm_sparse_causal_attn_bwd(desc, 11, p(q), k, v, o, lse, do, None, *got)
    torch.cuda.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
