"""GPU parity of the fp32 attention kernel where its key split changes.

The kernel shares a query tile's keys out over 1, 2, 4 or 8 groups of waves,
chosen on the host from the number of 32-row query blocks and of keys. Each of
CASES lands on one of them as a whole sequence (row-major V), each of STREAMS
streamed (dimension-major V from the cache; test_plan.py holds the counts), with
ragged rows, ranges that end inside a 32-key block and, in the stream, cache
regions that start off 32-key blocks.
Bar: max |gpu - oracle| <= 1e-4 x RMS, log-sum-exp within 1e-4.
"""
import numpy as np
import pytest
import torch

from gpu_helpers import LSE_ATOL, assert_close, from_dev, say, to_dev
from oracle import ChunkGeometry, StreamHistory, full_sequence_attention
from synth import draw_chunk, draw_qkv_sequence
from synth.inputs import Workload

pytestmark = pytest.mark.gpu

# B, H, D, T, C, R, W, frames: key groups of the whole sequence
CASES = [
    (1, 2, 64, 5, 1, 1, 1, 3, 1),      # 15 keys: one group whatever the fill
    (1, 2, 128, 33, 1, 1, 1, 2, 2),    # 66 keys: two groups
    (1, 3, 128, 41, 2, 1, 1, 6, 4),    # few rows, D = 128: four groups
    (1, 2, 64, 41, 2, 3, 2, 9, 8),     # few rows, D = 64: eight groups
    (8, 64, 64, 35, 1, 1, 1, 3, 2),    # 512 (batch, head) pairs of 6 blocks
    (16, 64, 64, 33, 1, 1, 1, 3, 1),   # 1024 pairs of 6 blocks: one group
    (8, 64, 128, 35, 1, 1, 1, 3, 2),
    (16, 64, 128, 33, 1, 1, 1, 3, 1),
]


# H, D, T, C, R, W, chunk: key groups of the streamed chunk (all rows). At D = 64, 8
# groups where they share the 32-key blocks of the ranges about as evenly as 4 do.
STREAMS = [
    (2, 64, 50, 2, 1, 2, 3, 8),    # 14 blocks in 4 ranges
    (2, 64, 64, 2, 1, 1, 2, 4),    # 10 blocks
    (3, 64, 44, 2, 1, 2, 3, 4),    # 11 blocks, ragged ends
    (1, 64, 64, 3, 1, 0, 1, 8),    # 8 blocks
    (2, 128, 50, 2, 1, 2, 3, 4),   # D = 128: never 8
]


@pytest.fixture(scope="module")
def tm():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2506_03099_amd import tm as binding
    binding.lib()
    return binding


@pytest.mark.parametrize("H,D,T,C,R,W,chunk,groups", STREAMS)
def test_f32_streamed_key_groups(tm, H, D, T, C, R, W, chunk, groups):
    say(f"f32 stream: H={H} D={D} T={T} C={C} R={R} W={W} chunk={chunk} ({groups} key groups)")
    g = ChunkGeometry(T, C, R, W)
    desc = tm.make_desc(1, H, D, T, C, R, W, "f32")
    w = Workload(760 + T, "f32_groups", "f32", 1, H, D, T, C, R, W)
    cache, hist = tm.KVCache(desc), StreamHistory(g)
    for t in range(chunk + 1):
        c = draw_chunk(w, t)
        qd, kd, vd = (to_dev(c[x]) for x in "qkv")
        tm.tm_kv_append(cache, t, kd, vd)
        hist.append(t, c["k"], c["v"])
    lse = torch.empty(1, H, C * T, dtype=torch.float32, device="cuda")
    o = from_dev(tm.tm_sparse_causal_attn_fwd(desc, qd, chunk, cache=cache, lse=lse))
    want, want_lse = hist.attend(c["q"], chunk)
    assert_close(o, want, "f32", "stream")
    assert np.max(np.abs(lse.cpu().numpy() - want_lse)) <= LSE_ATOL["f32"]


def _overflow(x, blocked, sign):
    """Rows of q (sign 0) or k whose scores overflow to -inf in fp32 where ``blocked``."""
    if sign == 0:
        return np.abs(x) * np.float32(1e20)
    y = x * np.float32(1e-20)
    y[:, blocked] = np.float32(-1e20)
    return y


# D, T, C, R, W, frames (sequence), chunk (streamed): 4 key groups at D = 128, 8 at 64
@pytest.mark.parametrize("D,T,C,R,W,frames,chunk", [(128, 50, 2, 1, 2, 9, 3), (64, 50, 2, 1, 2, 9, 3)])
@pytest.mark.parametrize("where", ["late", "alternate", "early"])
def test_f32_scores_of_minus_infinity(tm, D, T, C, R, W, frames, chunk, where):
    # Finite inputs whose scores overflow to -inf: over whole key groups ("late": from
    # the 100th key on), over the first block of some groups only ("alternate": every
    # other 32 keys), and over the row's first keys. They weigh nothing.
    say(f"f32 -inf: D={D} {where}")
    B, H = 1, 2
    g = ChunkGeometry(T, C, R, W)
    desc = tm.make_desc(B, H, D, T, C, R, W, "f32")
    blocked = {"late": lambda p: p >= 100, "alternate": lambda p: p // 32 % 2 == 1, "early": lambda p: p < 40}[where]
    w = Workload(750, "f32_inf", "f32", B, H, D, T, C, R, W, n_frames=frames)
    d = draw_qkv_sequence(w)
    d["q"] = _overflow(d["q"], None, 0)
    d["k"] = _overflow(d["k"], blocked(np.arange(frames * T)), 1)
    q, k, v = (to_dev(d[n]) for n in "qkv")
    lse = torch.empty(B, H, frames * T, dtype=torch.float32, device="cuda")
    o = tm.tm_sparse_causal_attn_fwd(desc, q, -1, k=k, v=v, n_frames=frames, lse=lse)
    torch.cuda.synchronize()
    with np.errstate(over="ignore"):
        want, want_lse = full_sequence_attention(d["q"], d["k"], d["v"], g)
    assert_close(from_dev(o), want, "f32", "sequence")
    assert np.max(np.abs(lse.cpu().numpy() - want_lse)) <= LSE_ATOL["f32"]

    cache, hist, seen = tm.KVCache(desc), StreamHistory(g), 0
    for t in range(chunk + 1):
        c = draw_chunk(w, t)
        n = c["k"].shape[1]
        c["q"] = _overflow(c["q"], None, 0)
        c["k"] = _overflow(c["k"], blocked(seen + np.arange(n)), 1)
        seen += n
        qd, kd, vd = (to_dev(c[x]) for x in "qkv")
        tm.tm_kv_append(cache, t, kd, vd)
        hist.append(t, c["k"], c["v"])
        o = from_dev(tm.tm_sparse_causal_attn_fwd(desc, qd, t, cache=cache))
    with np.errstate(over="ignore"):
        want = hist.attend(c["q"], chunk)[0]
    assert_close(o, want, "f32", "stream")


def _heads(B, H):
    """(batch, head) pairs to compare: all of a small case, the corners of a large one."""
    if B * H <= 16:
        return [(b, h) for b in range(B) for h in range(H)]
    return [(0, 0), (0, H - 1), (B // 2, 3), (B - 1, H - 1)]


@pytest.mark.parametrize("B,H,D,T,C,R,W,frames,groups", CASES)
def test_f32_key_groups(tm, B, H, D, T, C, R, W, frames, groups):
    say(f"f32: B={B} H={H} D={D} T={T} C={C} R={R} W={W} frames={frames} ({groups} key groups)")
    g = ChunkGeometry(T, C, R, W)
    desc = tm.make_desc(B, H, D, T, C, R, W, "f32")
    w = Workload(700 + groups, "f32_groups", "f32", B, H, D, T, C, R, W, n_frames=frames)
    d = draw_qkv_sequence(w)
    q, k, v = (to_dev(d[n]) for n in "qkv")
    lse = torch.empty(B, H, frames * T, dtype=torch.float32, device="cuda")
    o = tm.tm_sparse_causal_attn_fwd(desc, q, -1, k=k, v=v, n_frames=frames, lse=lse)
    torch.cuda.synchronize()
    o, lse = from_dev(o), lse.cpu().numpy()
    for b, h in _heads(B, H):
        one = [d[n][b:b + 1, :, h:h + 1] for n in "qkv"]
        want, want_lse = full_sequence_attention(*one, g)
        assert_close(o[b:b + 1, :, h:h + 1], want, "f32", f"sequence b={b} h={h}")
        assert np.max(np.abs(lse[b, h] - want_lse[0, 0])) <= LSE_ATOL["f32"]

    # streamed: chunk 2 of 2 (its last rows missing) over c_0 and the window
    cache = tm.KVCache(desc)
    hist = {p: StreamHistory(g) for p in _heads(B, H)}
    for t in range(3):
        n = None if t < 2 else max(1, C * T - 3)
        c = draw_chunk(w, t, n)
        qd, kd, vd = (to_dev(c[x]) for x in "qkv")
        tm.tm_kv_append(cache, t, kd, vd)
        for (b, h), s in hist.items():
            s.append(t, c["k"][b:b + 1, :, h:h + 1], c["v"][b:b + 1, :, h:h + 1])
        o = from_dev(tm.tm_sparse_causal_attn_fwd(desc, qd, t, cache=cache))
    for (b, h), s in hist.items():
        want = s.attend(c["q"][b:b + 1, :, h:h + 1], 2)[0]
        assert_close(o[b:b + 1, :, h:h + 1], want, "f32", f"stream b={b} h={h}")
