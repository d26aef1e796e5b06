"""The choice of the GEMM kernel (csrc/gemm_choice.h, compiled for the host):
the sizes that the GPU tests use for each kernel do reach it, and the rule's
invariants over a range of sizes."""
import os
import random
import subprocess

import pytest

from tests import gemm_kinds

HERE = os.path.dirname(os.path.abspath(__file__))
CUS = 256


@pytest.fixture(scope="module")
def kinds(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("choice") / "gemm_choice")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "host_gemm_choice.cpp"),
                    "-o", exe], check=True)

    def of(calls, mode="amax"):
        flags = {"amax": "1 1", "delayed": "0 1", "none": "0 0"}[mode]
        text = "".join(f"{M} {N} {K} {CUS} {int(fused)} {int(mx)} {flags}\n" for M, N, K, fused, mx in calls)
        return subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()
    return of


@pytest.mark.parametrize("table,fused,mx", [("PLAIN", 0, 0), ("PLAIN_INSIDE", 0, 0), ("FUSED", 1, 0),
                                            ("MX", 0, 1), ("MX_INSIDE", 0, 1)])
def test_the_gpu_tests_reach_the_kernels_they_name(kinds, table, fused, mx):
    entries = getattr(gemm_kinds, table)
    for mode in ("amax", "delayed", "none"):
        assert kinds([(*s, fused, mx) for s in entries.values()], mode) == list(entries)


def test_choices_that_depend_on_the_mode(kinds):
    """Many small workgroups with a statistic and little K; the fused pair
    kernel with an intermediate that outgrows the last-level cache."""
    for K, M, want in ((64, 2048, "big"), (512, 2048, "big"), (1024, 2048, "big"), (1025, 2048, "pair"),
                       (512, 1536, "big"), (513, 1536, "pair"), (512, 1408, "pair")):
        assert kinds([(M, 4096, K, 0, 0)], "amax") == kinds([(M, 4096, K, 0, 0)], "delayed") == [want], (M, K)
        assert kinds([(M, 4096, K, 0, 0)], "none") == kinds([(M, 4096, K, 1, 0)], "amax") == ["pair"], (M, K)
    assert kinds([(3001, 12288, 5504, 1, 0)], "amax") == ["pair-rounds"]
    assert kinds([(3001, 12288, 8192, 1, 0)], "amax") == ["fused8-rounds"]
    assert kinds([(3001, 12288, 8192, 1, 0)], "none") == ["pair-rounds"]
    # (block scales, whose kernels sum K differently, in no mode)
    for K, M, want in ((64, 2048, "big"), (256, 1856, "big"), (257, 2048, "wave-rounds"), (256, 1792, "wave-rounds")):
        for mode in ("amax", "delayed", "none"):
            assert kinds([(M, 1024, K, 0, 1)], mode) == [want], (M, K, mode)
    assert kinds(list((*s, 0, 0) for s in gemm_kinds.SHORT_K), "amax") == ["big"] * len(gemm_kinds.SHORT_K)
    assert kinds(list((*s, 0, 0) for s in gemm_kinds.SHORT_K), "none") == ["pair"] * len(gemm_kinds.SHORT_K)


def test_tiles_fit_the_kernels(kinds):
    """The single pass of the wave kernel holds its tiles (at most two), and
    the mid kernels' deep rings have one tile per workgroup."""
    rng = random.Random(5)
    size = lambda: int(2 ** rng.uniform(0, 15))
    calls = [(size(), size(), size(), f, m) for _ in range(4000) for f, m in ((0, 0), (1, 0), (0, 1))]
    for (M, N, K, fused, mx), kind in zip(calls, kinds(calls)):
        tm = 16 if M <= 16 else (32 if M <= 32 else 64)
        tiles = -(-M // tm) * -(-N // 64)
        if kind.startswith("wave"):
            assert tiles <= (2 * CUS if mx else CUS), (M, N, K)
        if kind.startswith("mid"):
            assert "rounds" not in kind and K >= 4096 and not mx, (M, N, K)
        if kind.startswith("fused8"):
            assert fused, (M, N, K)
