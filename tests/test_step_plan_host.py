"""Block shapes of the whole Sinkhorn steps (compiled for the host), and where a one-call step keeps their column sums (host-only
query); no GPU.  The two halves of a split call
run forward and backward without waiting for each other, so a half's backward must not write where the other half's
sums lie, nor the reverse, unless the streams are joined between the directions."""
import itertools
import os
import subprocess

import pytest

from paper_2605_08123_amd import binding as b

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2605_08123_amd", "csrc")
SIZES = [(1, 1), (31, 7), (65, 0), (100, 99), (300, 128), (333, 5000), (700, 160), (701, 64), (3001, 100), (4096, 128), (9000, 300),
         (16384, 256), (16500, 480), (33001, 256), (40000, 97), (65536, 256), (70001, 200), (262144, 256)]


def written_by_backward(N, L, R, dtype):
    """[(start, end, problem)] in bytes: the vectors g_u, vbar_R, ubar_R, ... [1 + 2 R][N][ldw], the fp32 packs
    [2][N][ldw][4 (2 R + 3) / 4] (each with room for R groups of four) and the packs of bf16 columns [4][N][ldw][16]."""
    ldw = (L + 3) // 4 * 4
    out, at = [], 0
    for _ in range(1 + 2 * R):
        out += [(at + 4 * ldw * n, at + 4 * ldw * (n + 1), n) for n in range(N)]
        at += 4 * ldw * N
    row = 16 * ((2 * R + 3) // 4)
    for _ in range(2):
        out += [(at + row * ldw * n, at + row * ldw * (n + 1), n) for n in range(N)]
        at += 16 * R * ldw * N
    for _ in range(4):
        out += [(at + 32 * ldw * n, at + 32 * ldw * (n + 1), n) for n in range(N)]
        at += 32 * ldw * N
    return out, at


@pytest.mark.parametrize("dtype,d", itertools.product((b.SKA_F32, b.SKA_BF16), (32, 64, 128)))
def test_sums_of_a_split_step_lie_apart_from_the_other_half(dtype, d):
    apart = 0
    for (L, W), N, R, lengths in itertools.product(SIZES, (2, 3, 5, 8), (1, 2, 3, 7), (False, True)):
        p = b.query_step_plan(N, 1, L, d, W, 16, R, False, dtype, one_call=True, lengths=lengths)
        if not p.whole_steps:
            continue
        written, end = written_by_backward(N, L, R, dtype)
        half = lambda n: n >= N // 2
        sums = [(off + n * p.sums_stride, off + n * p.sums_stride + p.sums_bytes, n) for off in p.sums_offset for n in range(N)]
        assert all(s >= 4 * ((L + 3) // 4 * 4) * N and e <= end for s, e, _ in sums)   # behind g_u, which the output map writes
        assert all(e0 <= s1 or e1 <= s0 for (s0, e0, _), (s1, e1, _) in itertools.combinations(sums, 2))
        if not p.sums_apart:   # the streams are joined; a default split (5e7 edges per half) never needs it
            assert (N // 2) * L * (2 * min(W, L) + 1) < 5e7, (L, W, N)
            continue
        apart += 1
        for s0, e0, n0 in sums:
            for s1, e1, n1 in written:
                assert half(n0) == half(n1) or e0 <= s1 or e1 <= s0, (L, W, N, R, n0, n1)
    assert apart > 20


def test_forward_alone_keeps_its_sums_inside_the_workspace():
    for (L, W), N, R, (dustbin, lengths) in itertools.product(SIZES, (1, 3), (1, 2, 5), ((False, False), (True, False), (False, True))):
        total = b.sinkhorn_attn_workspace_bytes(N, 1, L, 64, W, 16, R, dustbin)
        p = b.query_step_plan(N, 1, L, 64, W, 16, R, dustbin, lengths=lengths)
        if p.whole_steps:
            ends = [off + (N - 1) * p.sums_stride + p.sums_bytes for off in p.sums_offset]
            assert min(p.sums_offset) >= 2 * N * L * 64 and max(ends) <= total   # behind the prescaled operand
            assert ends[0] <= p.sums_offset[1]
        small = b.query_step_plan(N, 1, L, 64, W, 16, R, dustbin, workspace_bytes=2 * N * L * 64)
        assert not small.whole_steps   # room for the prescaled operand alone


def test_launches_that_wait_start_one_after_the_other(tmp_path):
    """gate.cpp: chains of steps and of half-steps go through one gate per device."""
    exe = str(tmp_path / "gate")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", CSRC, "-o", exe, os.path.join(HERE, "gate.cpp")], check=True)
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


def test_block_shapes(tmp_path):
    """step_shapes.cpp over the shapes that the rule takes: each has an instance that fits LDS, and no wavefront reads a tile
    outside it."""
    exe = str(tmp_path / "step_shapes")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__host__=", "-D__device__=", "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "step_shapes.cpp")], check=True)
    run = subprocess.run([exe], capture_output=True, text=True)
    print(run.stdout)
    assert run.returncode == 0, run.stdout
