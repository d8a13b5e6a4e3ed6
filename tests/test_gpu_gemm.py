"""Projection GEMM parity (sr_projection) against a float64 product of the
same bf16/fp32 inputs, over ragged shapes, every epilogue and the split-K
path.  The max-abs error is bounded relative to the oracle product's
max-abs: 1e-2 where the output is rounded to bf16, else 1e-4."""
import numpy as np
import pytest

from gpu_util import need_gpu, say

pytestmark = pytest.mark.gpu


def bf16_round(a):
    u = a.astype(np.float32).view(np.uint32)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.view(np.float32)


SHAPES = [(1, 64, 64), (17, 100, 128), (33, 1000, 512), (100, 384, 4096), (129, 130, 64), (300, 257, 1024),
          (512, 512, 14336), (1000, 96, 192), (1100, 300, 256), (2048, 520, 1024), (4000, 129, 64),
          (128, 200, 1024), (64, 64, 14336), (21, 4100, 1792), (112, 130, 384),
          # a few hundred rows, many columns, short K (128 x 128 tiles)
          (300, 49152, 256), (257, 24576, 128),
          # the 103-row QKV projection of the 8B shape
          (103, 6144, 4096),
          # 65-112 rows, long K, ragged N
          (70, 2000, 8192), (103, 4096, 14336),
          # 65-112 rows with 2 to 6 K steps of 256 per work-group
          (97, 4150, 512), (65, 4200, 768), (100, 4096, 4096), (112, 4100, 1280), (77, 4200, 1536),
          # 65-112 rows, more than 65536 columns (the LM head's tiles), ragged N
          (103, 66000, 384), (70, 65601, 128),
          # paired few-row tiles with 512-byte rows per copy (K steps of 256), ragged N
          (21, 4100, 2048),
          # thousands of rows, ragged in M and N, ten K steps
          (2600, 1100, 640),
          # 128 x 128 tiles: one to four K steps, ragged edges, one and two
          # work-groups a CU, K split; the rows where the choice changes
          (113, 130, 64), (129, 127, 128), (300, 200, 192), (771, 2048, 512), (513, 4100, 256), (200, 2048, 2048),
          (640, 300, 3072), (1500, 1000, 448),
          # thousands of rows, one to five K steps
          (5000, 2600, 64), (5100, 2570, 128), (4900, 2600, 320),
          # few rows, short K: no split where a reduction would cost more
          (64, 1536, 512), (21, 8192, 512)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("mode", [0, 1, 2, 3])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_projection(dtype, mode, M, N, K):
    torch, sr = need_gpu()
    if dtype == "f32" and K > 4096:
        pytest.skip("fp32 model shapes stay small")
    say(f"projection {dtype} mode={mode} M={M} N={N} K={K}")
    rng = np.random.default_rng(M * 7 + N + K + mode)
    x = rng.normal(0, 1, size=(M, K)).astype(np.float32)
    w = rng.normal(0, 0.05, size=((2, N, K) if mode == 2 else (N, K))).astype(np.float32)
    if dtype == "bf16":
        x, w = bf16_round(x), bf16_round(w)
        xt = torch.from_numpy(x.view(np.uint32) >> 16).to(torch.int32).to(torch.int16).cuda()
        wt = torch.from_numpy((w.view(np.uint32) >> 16).astype(np.uint16).view(np.int16)).cuda()
        xt = torch.from_numpy((x.view(np.uint32) >> 16).astype(np.uint16).view(np.int16)).cuda()
    else:
        xt, wt = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    x64, w64 = x.astype(np.float64), w.astype(np.float64)
    if mode == 2:
        g, u = x64 @ w64[0].T, x64 @ w64[1].T
        ref = g / (1 + np.exp(-g)) * u
    else:
        ref = x64 @ w64.T
    init = rng.normal(size=(M, N)).astype(np.float32)
    if mode in (0, 1):
        out = torch.from_numpy(init.copy()).cuda()
    else:
        out = torch.zeros((M, N), dtype=torch.int16 if dtype == "bf16" else torch.float32, device="cuda")
    sr.projection(xt, wt, mode, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    if mode in (2, 3) and dtype == "bf16":
        got = (got.view(np.uint16).astype(np.uint32) << 16).view(np.float32)
    if mode == 1:
        ref = ref + init
    scale = np.abs(ref).max()
    rtol = 1e-2 if (mode in (2, 3) and dtype == "bf16") else 1e-4
    assert np.abs(got - ref).max() <= rtol * scale, np.abs(got - ref).max()


# (kernel, splits, mode, M, N, K): every tile kernel paired and not, with and
# without a K split, at each remainder of its three-step loop, ragged in M and N;
# that the plans are these is asserted without a GPU (test_gemm_plan.py)
KERNEL_SHAPES = [("dma3", 1, 1, 129, 16390, 1024), ("dma3", 1, 3, 256, 16390, 1088), ("dma3", 1, 0, 129, 16390, 1152),
                 ("dma3", 1, 2, 129, 8200, 1024), ("dma3", 1, 2, 129, 8200, 1088), ("dma3", 1, 2, 129, 8200, 1152),
                 ("dma3", 8, 1, 129, 2050, 8192), ("dma3", 8, 0, 200, 4096, 14336), ("dma3", 4, 2, 129, 2050, 4096),
                 ("tile256", 1, 1, 1500, 8200, 640), ("tile256", 1, 3, 1500, 8200, 704),
                 ("tile256", 1, 0, 3100, 2570, 1152), ("tile256", 1, 2, 1500, 4100, 640),
                 ("tile256", 1, 2, 1500, 4100, 704), ("tile256", 1, 2, 1500, 4100, 768),
                 ("tile256", 4, 1, 771, 4096, 14336), ("tile256", 4, 3, 129, 8200, 8192),
                 ("tile256", 8, 2, 129, 2050, 14336),
                 ("wring", 1, 0, 129, 40000, 1024), ("wring", 1, 3, 129, 40000, 1088), ("wring", 1, 1, 129, 40000, 1152),
                 ("wring", 1, 2, 129, 24600, 640), ("wring", 1, 2, 129, 24600, 704), ("wring", 1, 2, 200, 16390, 1152),
                 ("tile128", 2, 1, 129, 257, 1536), ("tile128", 4, 3, 129, 257, 2048), ("tile128", 8, 0, 129, 257, 8192),
                 ("tile128", 2, 2, 129, 257, 1536), ("tile128", 1, 0, 300, 514, 256), ("tile128", 1, 2, 300, 514, 192)]


@pytest.mark.parametrize("kernel,splits,mode,M,N,K", KERNEL_SHAPES)
def test_projection_tile_kernels(kernel, splits, mode, M, N, K):
    torch, sr = need_gpu()
    say(f"projection {kernel} splits={splits} mode={mode} M={M} N={N} K={K}")
    bf = torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(M + N + K + mode)
    x = torch.empty((M, K), dtype=bf, device="cuda").normal_(0, 1, generator=g)
    w = torch.empty((2, N, K) if mode == 2 else (N, K), dtype=bf, device="cuda").normal_(0, 0.05, generator=g)
    out = torch.randn((M, N), generator=g, device="cuda").to(bf if mode >= 2 else torch.float32)
    x64, w64 = x.double(), w.double()
    if mode == 2:
        ga, up = x64 @ w64[0].T, x64 @ w64[1].T
        ref = ga / (1 + torch.exp(-ga)) * up
    else:
        ref = x64 @ w64.T + (out.double() if mode == 1 else 0)
    sr.projection(x, w, mode, out)
    torch.cuda.synchronize()
    assert float((out.double() - ref).abs().max()) <= (1e-2 if mode >= 2 else 1e-4) * float(ref.abs().max())


@pytest.mark.parametrize("M", [8, 41, 103, 120])
def test_projection_paired_8b(M):
    """The 8B gate/up projection (N 14336, K 4096) at the row counts of the
    decode rounds: every few-row tile kind with its rotated K order."""
    torch, sr = need_gpu()
    N, K = 14336, 4096
    say(f"paired projection bf16 M={M} N={N} K={K}")
    rng = np.random.default_rng(M)
    x = bf16_round(rng.normal(0, 1, size=(M, K)).astype(np.float32))
    w = bf16_round(rng.normal(0, 0.02, size=(2, N, K)).astype(np.float32))
    xt = torch.from_numpy((x.view(np.uint32) >> 16).astype(np.uint16).view(np.int16)).cuda()
    wt = torch.from_numpy((w.view(np.uint32) >> 16).astype(np.uint16).view(np.int16)).cuda()
    out = torch.zeros((M, N), dtype=torch.int16, device="cuda")
    sr.projection(xt, wt, 2, out)
    torch.cuda.synchronize()
    got = (out.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32)
    x64, w64 = x.astype(np.float64), w.astype(np.float64)
    g, u = x64 @ w64[0].T, x64 @ w64[1].T
    ref = g / (1 + np.exp(-g)) * u
    assert np.abs(got - ref).max() <= 1e-2 * np.abs(ref).max(), np.abs(got - ref).max()


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(5, 33, 64), (17, 100, 192), (1090, 1000, 64)])
def test_projection_f32_unaligned(M, N, K, mode):
    """fp32 operands that are only 4-byte aligned (scalar loads), on the
    split-K and the whole-K tiles.  Bound: K + 2 roundings of sums of |x w|,
    2^-24 each, on max-abs products well below 1."""
    torch, sr = need_gpu()
    say(f"projection f32 unaligned mode={mode} M={M} N={N} K={K}")
    rng = np.random.default_rng(M + N + K + mode)
    x = rng.normal(0, 1, size=(M, K)).astype(np.float32)
    w = rng.normal(0, 0.05, size=((2, N, K) if mode == 2 else (N, K))).astype(np.float32)
    xt = torch.from_numpy(np.concatenate([np.zeros(1, np.float32), x.ravel()])).cuda()[1:].view(M, K)
    wt = torch.from_numpy(np.concatenate([np.zeros(1, np.float32), w.ravel()])).cuda()[1:].view(w.shape)
    init = rng.normal(size=(M, N)).astype(np.float32)
    out = torch.from_numpy(init.copy()).cuda()
    sr.projection(xt, wt, mode, out)
    torch.cuda.synchronize()
    x64, w64 = x.astype(np.float64), w.astype(np.float64)
    if mode == 2:
        g, u = x64 @ w64[0].T, x64 @ w64[1].T
        ref = g / (1 + np.exp(-g)) * u
    else:
        ref = x64 @ w64.T + (init if mode == 1 else 0)
    bound = (K + 2) * 2.0 ** -24 * max(1.0, float((np.abs(x64) @ np.abs(w64.reshape(-1, K)).T).max())) ** 2
    assert np.abs(out.cpu().numpy() - ref).max() <= bound


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("which", ["x", "w"])
@pytest.mark.parametrize("M,N,K", [(20, 100, 256), (50, 100, 256), (70, 200, 192), (100, 200, 256), (600, 300, 1024),
                                   (1100, 300, 256)])
def test_projection_bf16_unaligned(M, N, K, which, mode):
    """bf16 operands that start on a 2-byte boundary: no 16-byte copy into LDS
    takes them, the register-staged tiles do, at every row count that has a
    streaming or an LDS-DMA tile plan."""
    torch, sr = need_gpu()
    say(f"projection bf16 unaligned {which} mode={mode} M={M} N={N} K={K}")
    g = torch.Generator(device="cuda").manual_seed(M + N + K + mode)

    def operand(shape, std, odd):
        t = torch.empty(int(np.prod(shape)) + 8, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
        return t[odd:odd + int(np.prod(shape))].view(shape)
    x = operand((M, K), 1.0, int(which == "x"))
    w = operand((2, N, K) if mode == 2 else (N, K), 0.05, int(which == "w"))
    x64, w64 = x.double(), w.double()
    if mode == 2:
        ga, up = x64 @ w64[0].T, x64 @ w64[1].T
        ref, out = ga / (1 + torch.exp(-ga)) * up, torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
    else:
        out = torch.randn((M, N), generator=g, device="cuda")
        ref = x64 @ w64.T + out.double()
    sr.projection(x, w, mode, out)
    torch.cuda.synchronize()
    assert float((out.double() - ref).abs().max()) <= (1e-2 if mode == 2 else 1e-4) * float(ref.abs().max())
