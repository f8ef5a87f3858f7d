"""GPU parity of the audio cross-attention on both sides of the line up to which
each stream has a workgroup of its own (batch * heads * frames * parts * streams
up to three quarters of the 256 CUs) and past which the streams are taken in
turn. Bars as in the other audio tests: face rows of the fp32 output within
2e-2 x RMS of the oracle, rows without a face exactly zero, the bf16 output the
rounded fp32 output, in place as well.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import assert_close, assert_rounds_to, say
from oracle import audio_cross_attention
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


# H, D, T, frames, M
CASES = [
    (64, 64, 90, 1, 3),     # 192 workgroups: a stream each
    (65, 64, 90, 1, 3),     # 195: in turn
    (48, 128, 70, 2, 2),    # 192
    (49, 128, 70, 2, 2),    # 196
    (3, 64, 2100, 1, 4),    # two parts per frame, a stream each
    (2, 128, 300, 3, 32),   # the most streams, 192 workgroups, most of them without rows
]


@pytest.mark.parametrize("H,D,T,frames,M", CASES)
def test_audio_streams(tm, H, D, T, frames, M):
    say(f"audio streams: H={H} D={D} T={T} frames={frames} M={M}")
    A, Fa, w, first = 8, 5, 1, 1
    n = T * frames
    rng = np.random.default_rng(H + M)
    q, qd = _bf16(rng, (1, n, H, D), True)
    ak, akd = _bf16(rng, (1, M, Fa * A, H, D), True)
    av, avd = _bf16(rng, (1, M, Fa * A, H, D), False)
    face = rng.integers(-1, M + 1, size=(1, n)).astype(np.int32)  # M: no face
    face[face == 1] = -1  # a stream without rows
    fd = torch.from_numpy(face).cuda()
    desc = tm.make_audio_desc(1, H, D, T, A, Fa, M, w)
    o = tm.tm_audio_cross_attn_fwd(desc, qd, first, akd, avd, fd)
    of = tm.tm_audio_cross_attn_fwd_f32out(desc, qd, first, akd, avd, fd)
    inplace = qd.clone()
    tm.tm_audio_cross_attn_fwd(desc, inplace, first, akd, avd, fd, o=inplace)
    torch.cuda.synchronize()
    assert_rounds_to(o, of, "streams")
    assert torch.equal(inplace.view(torch.int16), o.view(torch.int16))
    heads = sorted({0, H - 1})
    valid = np.where((face >= 0) & (face < M), face, -1)
    want = audio_cross_attention(q, ak, av, valid, tokens_per_frame=T, audio_per_frame=A,
                                 first_frame=first, half_window=w, heads=heads)
    got = of.cpu().numpy()[:, :, heads]
    sel = valid >= 0
    assert np.all(got[~sel] == 0)
    assert_close(got[sel], want[sel], "bf16", f"H={H} M={M}")
