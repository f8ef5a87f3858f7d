"""GPU parity of the forward's key split (the calls with a workspace).

Query tiles that do not fill the GPU share their keys out over several
workgroups and a second kernel merges the parts; without a workspace the parts
run one after the other, to the same bits. Each geometry runs with the
workspace (the binding's ordinary calls) and without (the C entry points that
take none). The fp32 output of both is held to the oracle within
2^-9 * (P |V|) + 1e-4 * RMS per element: every weight is rounded to bf16 for the
P V product (relative error at most 2^-9), and the rest is fp32. The
log-sum-exps are held to 1e-4, and the bf16 output is the rounded fp32 output on
each route. Whether a geometry splits at all is part of the case.
"""
import ctypes

import numpy as np
import pytest
import torch

from gpu_helpers import LSE_ATOL, assert_rounds_to, from_dev, say, to_dev
from oracle import ChunkGeometry, StreamHistory, full_sequence_attention
from synth import bf16_bits_to_f32, draw_chunk, draw_qkv_sequence, f32_to_bf16_bits
from synth.inputs import Workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tm():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2506_03099_amd import tm as binding
    binding.lib()
    return binding


def _plain(tm, desc, q, q_chunk, cache=None, k=None, v=None, n_frames=0, lse=None, f32=False):
    """The call without a workspace."""
    L = tm.lib()
    o = torch.empty(q.shape, dtype=torch.float32 if f32 else q.dtype, device="cuda")
    fn = L.tm_sparse_causal_attn_fwd_f32out if f32 else L.tm_sparse_causal_attn_fwd
    st = fn(ctypes.byref(desc), tm._ptr(q), q_chunk, cache.handle if cache else None, tm._ptr(k),
            tm._ptr(v), n_frames, tm._ptr(o), tm._ptr(lse), tm._stream(None))
    assert st == tm.TM_OK, tm.tm_last_error()
    return o


def _plain_into(tm, desc, q, q_chunk, o, lse, k=None, v=None, n_frames=0):
    st = tm.lib().tm_sparse_causal_attn_fwd(ctypes.byref(desc), tm._ptr(q), q_chunk, None, tm._ptr(k), tm._ptr(v),
                                            n_frames, tm._ptr(o), tm._ptr(lse), tm._stream(None))
    assert st == tm.TM_OK, tm.tm_last_error()


def _bytes(tm, desc, q_chunk, cache=None, n_frames=0):
    return tm.lib().tm_sparse_causal_attn_fwd_workspace(
        ctypes.byref(desc), q_chunk, cache.handle if cache else None, n_frames)


def _assert_bound(got, want, mag, what):
    """|got - want| <= 2^-9 mag + 1e-4 RMS(want), mag the weights times |V|."""
    bound = 2.0 ** -9 * mag + 1e-4 * float(np.sqrt(np.mean(np.square(want, dtype=np.float64))))
    assert np.all(np.isfinite(got)), f"{what}: non-finite output"
    worst = float(np.max(np.abs(got - want) / bound))
    say(f"  {what}: worst err / bound = {worst:.3f}")
    assert worst <= 1.0, f"{what}: error {worst:.3f} x the bound"


def _both(tm, desc, q, q_chunk, heads, want, mag, want_lse, what, **kw):
    B, n, H = q.shape[:3]
    for route in ("workspace", "plain"):
        lse = torch.full((B, H, n), float("nan"), dtype=torch.float32, device="cuda")
        if route == "workspace":
            o = tm.tm_sparse_causal_attn_fwd(desc, q, q_chunk, lse=lse, **kw)
            of = tm.tm_sparse_causal_attn_fwd_f32out(desc, q, q_chunk, **kw)
        else:
            o = _plain(tm, desc, q, q_chunk, lse=lse, **kw)
            of = _plain(tm, desc, q, q_chunk, f32=True, **kw)
        torch.cuda.synchronize()
        assert_rounds_to(o, of, f"{what} {route}")
        _assert_bound(from_dev(of)[:, :, heads], want, mag, f"{what} {route}")
        assert np.max(np.abs(lse.cpu().numpy()[:, heads] - want_lse)) <= LSE_ATOL["bf16"]


# B, H, D, T, C, R, W, rows of the streamed chunk 3 (0: all), splits?
STREAM = [
    (1, 2, 128, 300, 3, 1, 1, 0, True),     # 8 tiles, at most 16 parts, fewer by the keys
    (1, 3, 64, 301, 2, 2, 2, 250, True),    # D = 64, ragged rows and regions, four ranges
    (2, 5, 128, 500, 3, 3, 0, 33, True),    # one 33-row tile per head
    (1, 258, 64, 150, 2, 1, 3, 0, True),    # two rounds of 256 whole tiles, then 4 split ones
    (1, 40, 128, 64, 1, 1, 1, 0, False),    # too few keys to share out
    (1, 129, 64, 200, 1, 1, 3, 0, False),   # more than half a round
]


@pytest.mark.parametrize("B,H,D,T,C,R,W,rows,splits", STREAM)
def test_split_stream(tm, B, H, D, T, C, R, W, rows, splits):
    say(f"split stream: B={B} H={H} D={D} T={T} C={C} R={R} W={W} rows={rows}")
    g = ChunkGeometry(T, C, R, W)
    desc = tm.make_desc(B, H, D, T, C, R, W, "bf16")
    heads = sorted({0, H // 2, H - 1})
    w = Workload(800 + T, "split", "bf16", B, H, D, T, C, R, W)
    cache, hist, hist_abs = tm.KVCache(desc), StreamHistory(g), StreamHistory(g)
    for t in range(4):
        d = draw_chunk(w, t, rows if t == 3 and rows else None)
        q, k, v = (to_dev(d[n], d[n + "_bits"], "bf16") for n in "qkv")
        tm.tm_kv_append(cache, t, k, v)
        kh, vh = (np.ascontiguousarray(d[n][:, :, heads]) for n in "kv")
        hist.append(t, kh, vh)
        hist_abs.append(t, kh, np.abs(vh))
    assert (_bytes(tm, desc, 3, cache) > 0) == splits
    qh = np.ascontiguousarray(d["q"][:, :, heads])
    want, want_lse = hist.attend(qh, 3)
    _both(tm, desc, q, 3, heads, want, hist_abs.attend(qh, 3)[0], want_lse, "stream", cache=cache)


# B, H, D, T, C, R, W, frames, splits?
SEQUENCE = [
    (1, 2, 128, 256, 3, 1, 1, 8, True),     # parts outnumber c_0's key tiles
    (1, 1, 64, 200, 2, 3, 2, 11, True),
    (2, 16, 128, 100, 2, 1, 1, 13, False),  # 256 tiles: a full round
]


@pytest.mark.parametrize("B,H,D,T,C,R,W,frames,splits", SEQUENCE)
def test_split_sequence(tm, B, H, D, T, C, R, W, frames, splits):
    say(f"split sequence: B={B} H={H} D={D} T={T} C={C} R={R} W={W} frames={frames}")
    desc = tm.make_desc(B, H, D, T, C, R, W, "bf16")
    d = draw_qkv_sequence(Workload(820 + T, "split", "bf16", B, H, D, T, C, R, W, n_frames=frames))
    q, k, v = (to_dev(d[n], d[n + "_bits"], "bf16") for n in "qkv")
    assert (_bytes(tm, desc, -1, None, frames) > 0) == splits
    heads = sorted({0, H - 1})
    qh, kh, vh = (d[n][:, :, heads] for n in "qkv")
    g = ChunkGeometry(T, C, R, W)
    want, want_lse = full_sequence_attention(qh, kh, vh, g)
    mag = full_sequence_attention(qh, kh, np.abs(vh), g)[0]
    _both(tm, desc, q, -1, heads, want, mag, want_lse, "sequence", k=k, v=v, n_frames=frames)


def test_split_parts_of_minus_infinity(tm):
    # scores of the last 700 keys overflow to -inf: whole parts see nothing else
    H, D, T = 1, 128, 400
    rng = np.random.default_rng(3)
    x = [rng.standard_normal((1, 4 * T, H, D)).astype(np.float32) for _ in range(3)]
    x[0][...] = np.abs(x[0]) * 1e20
    x[1][:, :900] *= 1e-20
    x[1][:, 900:] = -1e20
    bits = [f32_to_bf16_bits(a) for a in x]
    q, k, v = (to_dev(None, b, "bf16") for b in bits)
    desc = tm.make_desc(1, H, D, T, 3, 1, 1, "bf16")
    assert _bytes(tm, desc, -1, None, 4) > 0
    with np.errstate(over="ignore"):
        g = ChunkGeometry(T, 3, 1, 1)
        qh, kh, vh = (bf16_bits_to_f32(b) for b in bits)
        want, want_lse = full_sequence_attention(qh, kh, vh, g)
        mag = full_sequence_attention(qh, kh, np.abs(vh), g)[0]
    _both(tm, desc, q, -1, [0], want, mag, want_lse, "-inf parts", k=k, v=v, n_frames=4)


def _low_scores(d, blocked):
    """q and k whose scores lie near -300 in the log2 domain, or at -inf where
    ``blocked`` (keys): dimension 0 carries the offset, the others are as drawn."""
    D = d["q"].shape[-1]
    d["q"][..., 0] = 64.0
    d["k"][..., 0] = np.float32(-300 * np.log(2) * np.sqrt(D) / 64)
    d["k"][:, blocked, :, 0] = -3e38  # times 64: past the largest fp32
    for n in "qk":
        d[n + "_bits"] = f32_to_bf16_bits(d[n])
        d[n] = bf16_bits_to_f32(d[n + "_bits"])
    return d


@pytest.mark.parametrize("D", [128, 64])
def test_split_parts_that_start_at_minus_infinity(tm, D):
    # Two of three 64-key tiles score -inf: most parts start with one and go on with
    # scores far below 0, which weigh as much as those of the other parts.
    say(f"split parts that start at -inf: D={D}")
    blocked = lambda p: p // 64 % 3 != 2  # noqa: E731
    B, H, T, C, R, W, frames = 1, 2, 256, 3, 1, 1, 8
    g = ChunkGeometry(T, C, R, W)
    desc = tm.make_desc(B, H, D, T, C, R, W, "bf16")
    d = draw_qkv_sequence(Workload(890, "split", "bf16", B, H, D, T, C, R, W, n_frames=frames))
    d = _low_scores(d, blocked(np.arange(frames * T)))
    q, k, v = (to_dev(d[n], d[n + "_bits"], "bf16") for n in "qkv")
    assert _bytes(tm, desc, -1, None, frames) > 0
    with np.errstate(over="ignore"):
        want, want_lse = full_sequence_attention(d["q"], d["k"], d["v"], g)
        mag = full_sequence_attention(d["q"], d["k"], np.abs(d["v"]), g)[0]
    _both(tm, desc, q, -1, [0, 1], want, mag, want_lse, "sequence", k=k, v=v, n_frames=frames)

    w = Workload(891, "split", "bf16", B, H, D, T, C, R, W)
    cache, hist, hist_abs, seen = tm.KVCache(desc), StreamHistory(g), StreamHistory(g), 0
    for t in range(4):
        d = draw_chunk(w, t)
        n = d["k"].shape[1]
        d = _low_scores(d, blocked(seen + np.arange(n)))
        seen += n
        q, k, v = (to_dev(d[x], d[x + "_bits"], "bf16") for x in "qkv")
        tm.tm_kv_append(cache, t, k, v)
        hist.append(t, d["k"], d["v"])
        hist_abs.append(t, d["k"], np.abs(d["v"]))
    assert _bytes(tm, desc, 3, cache) > 0
    with np.errstate(over="ignore"):
        want, want_lse = hist.attend(d["q"], 3)
        mag = hist_abs.attend(d["q"], 3)[0]
    _both(tm, desc, q, 3, [0, 1], want, mag, want_lse, "stream", cache=cache)


def test_split_off_the_current_stream_and_under_capture(tm):
    # neither takes a workspace: the bits of the call without one, replay after replay
    desc = tm.make_desc(1, 2, 128, 256, 3, 1, 1, "bf16")
    d = draw_qkv_sequence(Workload(840, "split", "bf16", 1, 2, 128, 256, 3, 1, 1, n_frames=8))
    q, k, v = (to_dev(d[n], d[n + "_bits"], "bf16") for n in "qkv")
    want = _plain(tm, desc, q, -1, k=k, v=v, n_frames=8)
    o = torch.empty_like(q)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    tm.tm_sparse_causal_attn_fwd(desc, q, -1, k=k, v=v, n_frames=8, o=o, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), want.view(torch.int16))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tm.tm_sparse_causal_attn_fwd(desc, q, -1, k=k, v=v, n_frames=8, o=o)
    for _ in range(3):
        o.zero_()
        tm.tm_sparse_causal_attn_fwd(desc, q, -1, k=k, v=v, n_frames=8)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o.view(torch.int16), want.view(torch.int16))


# B, H, D, T, C, R, W, rows of the streamed chunk 3 (0: all)
ROUTES = [
    (1, 2, 128, 300, 3, 1, 1, 0),     # 8 split tiles: four workgroups walk each tile's parts
    (2, 5, 128, 500, 3, 3, 0, 33),    # 33 rows: most of these workgroups have none
    (1, 3, 64, 301, 2, 2, 2, 250),
    (1, 20, 128, 300, 3, 1, 1, 777),  # 80 split tiles: two workgroups each, O in private memory
    (1, 33, 64, 200, 2, 3, 3, 0),     # 66 at D = 64
    (1, 258, 64, 150, 2, 1, 3, 0),    # 512 whole tiles beside 4 split ones
]


def _same_bits(got, want):
    for a, b in zip(got, want):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("B,H,D,T,C,R,W,rows", ROUTES)
def test_split_bits_do_not_depend_on_the_workspace_streamed(tm, B, H, D, T, C, R, W, rows):
    say(f"split routes, stream: B={B} H={H} D={D} T={T} C={C} R={R} W={W} rows={rows}")
    desc = tm.make_desc(B, H, D, T, C, R, W, "bf16")
    w = Workload(860 + T, "split", "bf16", B, H, D, T, C, R, W)
    cache = tm.KVCache(desc)
    for t in range(4):
        d = draw_chunk(w, t, rows if t == 3 and rows else None)
        q, k, v = (to_dev(d[n], d[n + "_bits"], "bf16") for n in "qkv")
        tm.tm_kv_append(cache, t, k, v)
    assert _bytes(tm, desc, 3, cache) > 0
    lse = [torch.empty((B, H, q.shape[1]), dtype=torch.float32, device="cuda") for _ in range(2)]
    want = (tm.tm_sparse_causal_attn_fwd(desc, q, 3, cache=cache, lse=lse[0]), lse[0],
            tm.tm_sparse_causal_attn_fwd_f32out(desc, q, 3, cache=cache))
    got = (_plain(tm, desc, q, 3, cache=cache, lse=lse[1]), lse[1], _plain(tm, desc, q, 3, cache=cache, f32=True))
    torch.cuda.synchronize()
    _same_bits(got, want)


# B, H, D, T, C, R, W, frames
SEQUENCE_ROUTES = [
    (1, 2, 128, 256, 3, 1, 1, 8),     # c_0's tiles have fewer key tiles than there are parts
    (1, 1, 64, 200, 2, 3, 2, 11),
    (1, 10, 128, 250, 3, 1, 1, 7),    # 70 split tiles
    (1, 12, 64, 250, 3, 1, 1, 7),     # 84 at D = 64
]


@pytest.mark.parametrize("B,H,D,T,C,R,W,frames", SEQUENCE_ROUTES)
def test_split_bits_do_not_depend_on_the_workspace_sequence(tm, B, H, D, T, C, R, W, frames):
    say(f"split routes, sequence: B={B} H={H} D={D} T={T} C={C} R={R} W={W} frames={frames}")
    desc = tm.make_desc(B, H, D, T, C, R, W, "bf16")
    d = draw_qkv_sequence(Workload(880 + T, "split", "bf16", B, H, D, T, C, R, W, n_frames=frames))
    q, k, v = (to_dev(d[n], d[n + "_bits"], "bf16") for n in "qkv")
    for chunk in (-1, 2):  # the whole sequence, and one chunk's queries
        if chunk >= 0:
            start = R * T + (chunk - 1) * C * T
            q = q[:, start:start + C * T].contiguous()
        kw = dict(k=k, v=v, n_frames=frames)
        assert _bytes(tm, desc, chunk, None, frames) > 0
        lse = [torch.empty((B, H, q.shape[1]), dtype=torch.float32, device="cuda") for _ in range(3)]
        want = (tm.tm_sparse_causal_attn_fwd(desc, q, chunk, lse=lse[0], **kw), lse[0],
                tm.tm_sparse_causal_attn_fwd_f32out(desc, q, chunk, **kw))
        got = (_plain(tm, desc, q, chunk, lse=lse[1], **kw), lse[1], _plain(tm, desc, q, chunk, f32=True, **kw))
        inplace = q.clone()
        _plain_into(tm, desc, inplace, chunk, inplace, lse[2], **kw)
        torch.cuda.synchronize()
        _same_bits(got, want)
        _same_bits((inplace, lse[2]), want)


def test_split_captured_chunk_has_the_eager_bits(tm):
    # a streamed chunk's attention captured once, replayed on new queries each time, with
    # eager calls in between; and the same call on a side stream
    desc = tm.make_desc(1, 5, 128, 300, 3, 1, 1, "bf16")
    w = Workload(895, "split", "bf16", 1, 5, 128, 300, 3, 1, 1)
    cache = tm.KVCache(desc)
    for t in range(4):
        d = draw_chunk(w, t)
        q, k, v = (to_dev(d[n], d[n + "_bits"], "bf16") for n in "qkv")
        tm.tm_kv_append(cache, t, k, v)
    assert _bytes(tm, desc, 3, cache) > 0
    o, lse = torch.empty_like(q), torch.empty((1, 5, q.shape[1]), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        tm.tm_sparse_causal_attn_fwd(desc, q, 3, cache=cache, o=o, lse=lse)
    for i in range(4):
        q.copy_(torch.roll(q, i + 1, 1))
        want_lse = torch.empty_like(lse)
        want = tm.tm_sparse_causal_attn_fwd(desc, q, 3, cache=cache, lse=want_lse)
        o.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        _same_bits((o, lse), (want, want_lse))
        side = torch.cuda.Stream()
        o.zero_()
        torch.cuda.synchronize()
        tm.tm_sparse_causal_attn_fwd(desc, q, 3, cache=cache, o=o, lse=lse, stream=side)
        torch.cuda.synchronize()
        _same_bits((o, lse), (want, want_lse))


def test_split_with_plain_addresses(tm):
    # tensors given as addresses: the call without a workspace
    desc = tm.make_desc(1, 2, 128, 256, 3, 1, 1, "bf16")
    d = draw_qkv_sequence(Workload(840, "split", "bf16", 1, 2, 128, 256, 3, 1, 1, n_frames=8))
    q, k, v = (to_dev(d[n], d[n + "_bits"], "bf16") for n in "qkv")
    assert _bytes(tm, desc, -1, None, 8) > 0
    want = _plain(tm, desc, q, -1, k=k, v=v, n_frames=8)
    o = torch.empty_like(q)
    tm.tm_sparse_causal_attn_fwd(desc, q.data_ptr(), -1, k=k.data_ptr(), v=v.data_ptr(), n_frames=8,
                                 o=o.data_ptr())
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), want.view(torch.int16))


def test_split_workspace_is_checked(tm):
    desc = tm.make_desc(1, 2, 128, 256, 3, 1, 1, "bf16")
    q, k, v = (torch.zeros((1, 2048, 2, 128), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    o = torch.empty_like(q)
    n = _bytes(tm, desc, -1, None, 8)
    call = lambda ws, size: tm.lib().tm_sparse_causal_attn_fwd_ws(  # noqa: E731
        ctypes.byref(desc), tm._ptr(q), -1, None, tm._ptr(k), tm._ptr(v), 8, tm._ptr(o), 0, None, ws,
        size, tm._stream(None))
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    assert call(tm._ptr(ws), n) == tm.TM_OK
    assert call(tm._ptr(ws), n - 1) == tm.TM_OK  # too small: not used
    assert call(tm._ptr(ws) + 8, n) == tm.TM_E_ARG
    assert call(tm._ptr(q), n) == tm.TM_E_ARG
    torch.cuda.synchronize()
