"""Plans of the projections (host only).

The K split does not change within a block of rows, so a buffer sized for a
block's last row holds every shorter call, as the workspace assumes; and the
plans are near the fastest of the measured ones."""
import ctypes
import os

import pytest

import paper_2410_20290_amd as sr
from test_gpu_gemm import KERNEL_SHAPES

KINDS = ["reg", "stream", "tile128", "tile256", "wring", "dma3"]


class Plan(ctypes.Structure):
    """GemmPlan (csrc/kernels.h)."""
    _fields_ = [(n, ctypes.c_int) for n in ("kind", "splits", "stream", "stream_bn")]


def plan(M, N, K, paired=False, fused=False):
    f = sr.lib()._ZN2sr9gemm_planEiiiibb
    f.restype, f.argtypes = Plan, [ctypes.c_int] * 4 + [ctypes.c_bool] * 2
    p = f(sr.SR_BF16, M, N, K, paired, fused)
    return KINDS[p.kind], p.splits


@pytest.mark.parametrize("N,K,mode", [(6144, 4096, 0), (4096, 14336, 1), (14336, 4096, 2), (2048, 8192, 1),
                                      (1536, 512, 2), (512, 1536, 0), (8192, 512, 0), (384, 320, 0)])
def test_split_is_constant_within_a_block_of_rows(N, K, mode):
    scratch = lambda M: int(sr.lib().sr_projection_scratch(sr.SR_BF16, M, N, K, mode))
    ends = [0, 32, 64, 112, 128] + list(range(256, 6401, 128))
    for lo, hi in zip(ends, ends[1:]):
        per_row = {scratch(M) / M for M in range(lo + 1, hi + 1)}
        assert len(per_row) == 1, (lo, hi, per_row)


def measured():
    """[(shape, M, N, K, paired, fused, {(kind, splits): us})]"""
    path = os.path.join(os.path.dirname(__file__), "..", "profiles", "gemm_plan_sweep.csv")
    for line in open(path):
        if line.startswith(("#", "shape,")):
            continue
        shape, N, K, paired, M, fused, times = line.strip().split(",")
        us = {}
        for t in times.split():
            k, v = t.split("=")
            us[(k.split(":")[0], int(k.split(":")[1]))] = float(v)
        yield shape, int(M), int(N), int(K), paired == "1", fused != "none", us


def test_plans_are_near_the_fastest_measured():
    """Over all measured projections above the streaming range, each plan's
    measured time against the fastest one's: 1.5 % on average.  At whole row
    tiles (multiples of 256, no element-wise edge) at most 20 %; and the 8B QKV
    projection of 512 rows, whose reduction had been priced at twice its time
    (unsplit tiles, 28 % slower), at most 5 %."""
    loss = {}
    for shape, M, N, K, paired, fused, us in measured():
        if M > 128:
            loss[(shape, M, fused)] = us[plan(M, N, K, paired, fused)] / min(us.values())
    assert len(loss) > 500
    assert sum(loss.values()) / len(loss) <= 1.015
    assert max(v for (_, M, _), v in loss.items() if M % 256 == 0) <= 1.2
    for M in (420, 512):
        assert loss[("8b.qkv", M, False)] <= 1.05 and loss[("1b.qkv", M, False)] <= 1.08


def test_streaming_plans_are_near_the_fastest_measured():
    loss = []
    for shape, M, N, K, paired, fused, us in measured():
        if M <= 128 and plan(M, N, K, paired, fused) in us:
            loss.append(us[plan(M, N, K, paired, fused)] / min(us.values()))
    assert len(loss) > 150
    assert sum(loss) / len(loss) <= 1.01 and max(loss) <= 1.2


@pytest.mark.parametrize("kernel,splits,mode,M,N,K", KERNEL_SHAPES)
def test_kernel_shapes_reach_their_kernel(kernel, splits, mode, M, N, K):
    assert plan(M, N, K, mode == 2) == (kernel, splits)


def test_kernel_shapes_cover_every_tile_kernel():
    have = {(k, mode == 2, s > 1) for k, s, mode, _, _, _ in KERNEL_SHAPES}
    for k in ("tile128", "tile256", "dma3"):
        assert {(k, p, s) for p in (False, True) for s in (False, True)} <= have
    assert {("wring", False, False), ("wring", True, False)} <= have   # (never split)


@pytest.mark.parametrize("N,K,paired", [(6144, 4096, False), (4096, 4096, False), (4096, 14336, False),
                                        (14336, 4096, True), (128256, 4096, False), (3072, 2048, False),
                                        (2048, 8192, False), (768, 512, False), (512, 1536, False), (384, 320, False),
                                        (8192, 2048, True)])
@pytest.mark.parametrize("fused", [False, True])
def test_partials_of_every_row_count_fit_the_workspace(N, K, paired, fused):
    """The workspace is sized by gemm_partial_elems_upto from the ends of the
    blocks of rows: no call of up to M_max rows writes more, for limits at a
    block's end and inside one, and it grows with M_max."""
    if paired and fused:
        pytest.skip("partials are left by unpaired projections only")
    upto = sr.lib()._ZN2sr23gemm_partial_elems_uptoEiiiibb
    upto.restype, upto.argtypes = ctypes.c_size_t, [ctypes.c_int] * 4 + [ctypes.c_bool] * 2

    def partials(M):
        s = plan(M, N, K, paired, fused)[1]
        return s * M * N * (2 if paired else 1) if s > 1 or fused else 0
    most, at = 0, {}
    for M in range(1, 2601):
        most = max(most, partials(M))
        at[M] = most
    last = 0
    for M in (1, 31, 32, 33, 64, 65, 100, 112, 113, 128, 129, 200, 256, 257, 500, 512, 513, 1000, 1024, 1025, 2000, 2600):
        n = int(upto(sr.SR_BF16, M, N, K, paired, fused))
        assert n >= at[M] and n >= last, (M, n, at[M])
        last = n
