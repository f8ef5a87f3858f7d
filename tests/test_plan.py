"""How the host lays calls out: key groups of the fp32 forward, parts of the split
bf16 forward and of the backward, as the planners (through the sanitizer build's
``--plan``) print them, for the geometries that the GPU tests run because they
land on one side or the other of a rule.
"""
import os
import subprocess

import pytest

import test_gpu_backward_split as bwd
import test_gpu_f32 as f32
import test_gpu_split as split

DRIVER = os.path.join(os.path.dirname(os.path.abspath(__file__)), "sanitize", "host_abi_driver")


def _plan(dtype, B, H, D, T, C, R, W, form, *args):
    if not os.path.exists(DRIVER):
        pytest.skip("tests/sanitize/host_abi_driver is not built (run build())")
    cmd = [DRIVER, "--plan", dtype, *map(str, (B, H, D, T, C, R, W)), form, *map(str, args)]
    words = subprocess.run(cmd, capture_output=True, text=True, check=True, timeout=60).stdout.split()
    return {k: int(v) for k, v in zip(words[::2], words[1::2])}


@pytest.mark.parametrize("B,H,D,T,C,R,W,frames,groups", f32.CASES)
def test_f32_sequence_key_groups(B, H, D, T, C, R, W, frames, groups):
    assert _plan("f32", B, H, D, T, C, R, W, "seq", frames, -1)["key_groups"] == groups


@pytest.mark.parametrize("H,D,T,C,R,W,chunk,groups", f32.STREAMS)
def test_f32_streamed_key_groups(H, D, T, C, R, W, chunk, groups):
    assert _plan("f32", 1, H, D, T, C, R, W, "stream", chunk, C * T)["key_groups"] == groups


@pytest.mark.parametrize("D,groups", [(128, 4), (64, 8)])
def test_f32_key_groups_of_the_minus_infinity_test(D, groups):
    assert _plan("f32", 1, 2, D, 50, 2, 1, 2, "seq", 9, -1)["key_groups"] == groups
    assert _plan("f32", 1, 2, D, 50, 2, 1, 2, "stream", 3, 100)["key_groups"] == groups


@pytest.mark.parametrize("B,H,D,T,C,R,W,rows,split_tiles", [
    (1, 2, 128, 300, 3, 1, 1, 0, 8), (2, 5, 128, 500, 3, 3, 0, 33, 10), (1, 3, 64, 301, 2, 2, 2, 250, 3),
    (1, 20, 128, 300, 3, 1, 1, 777, 80), (1, 33, 64, 200, 2, 3, 3, 0, 66), (1, 258, 64, 150, 2, 1, 3, 0, 4)])
def test_split_tiles_of_the_route_tests(B, H, D, T, C, R, W, rows, split_tiles):
    # without a workspace, four workgroups per split tile up to 64 tiles, two beyond
    assert (B, H, D, T, C, R, W, rows) in split.ROUTES
    p = _plan("bf16", B, H, D, T, C, R, W, "stream", 3, rows or C * T)
    assert p["tiles"] - p["whole"] == split_tiles and p["parts"] > 1


@pytest.mark.parametrize("B,H,D,T,C,R,W,frames,split_tiles", [
    (1, 2, 128, 256, 3, 1, 1, 8, 16), (1, 1, 64, 200, 2, 3, 2, 11, 11), (1, 10, 128, 250, 3, 1, 1, 7, 70),
    (1, 12, 64, 250, 3, 1, 1, 7, 84)])
def test_split_tiles_of_the_sequence_route_tests(B, H, D, T, C, R, W, frames, split_tiles):
    assert (B, H, D, T, C, R, W, frames) in split.SEQUENCE_ROUTES
    p = _plan("bf16", B, H, D, T, C, R, W, "seq", frames, -1)
    assert p["tiles"] - p["whole"] == split_tiles and p["parts"] > 1


# c_0's dK/dV, the chunks' dK/dV, dQ: which of them the backward's cases split
@pytest.mark.parametrize("case,ref,chunks,q", [
    (bwd.CASES[0], True, True, False), (bwd.CASES[1], True, True, False), (bwd.CASES[2], True, True, False),
    (bwd.CASES[3], True, False, True), (bwd.CASES[4], True, False, False), (bwd.CASES[5], False, False, False),
    (bwd.CASES[6], True, True, True)])
def test_backward_parts(case, ref, chunks, q):
    B, H, D, T, C, R, W, frames = case[:8]
    p = _plan("bf16", B, H, D, T, C, R, W, "bwd", frames)
    assert (p["k_ref_parts"] > 1, p["k_chunk_parts"] > 1, p["q_parts"] > 1) == (ref, chunks, q)
