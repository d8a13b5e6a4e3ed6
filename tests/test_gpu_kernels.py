"""Kernel-level parity: Philox, the sampler, the cut and the KV compaction
against the oracle, bit-exact (they are integer decisions)."""
import numpy as np
import pytest

from gpu_util import need_gpu, say
from oracle import sampler as osamp
from oracle import specrej
from oracle.philox import philox4x32_10_np

pytestmark = pytest.mark.gpu


def test_philox_bit_exact():
    torch, sr = need_gpu()
    rng = np.random.default_rng(0)
    n = 100_003
    ctr = rng.integers(0, 2**32, size=(n, 4), dtype=np.uint64).astype(np.uint32)
    for seed in (0, 42, (7 << 32) | 99, 2**64 - 1):
        out = torch.empty((n, 4), dtype=torch.int32, device="cuda")
        sr.philox_fill(seed, torch.from_numpy(ctr.view(np.int32)).cuda(), out)
        got = out.cpu().numpy().view(np.uint32)
        ref = philox4x32_10_np(ctr[:, 0], ctr[:, 1], ctr[:, 2], ctr[:, 3], seed & 0xFFFFFFFF, seed >> 32)
        assert np.array_equal(got, np.stack(ref, axis=1))


def oracle_tokens(logits, cand, step, temperature, seed):
    return np.array([osamp.sample(logits[r], temperature, seed, int(cand[r]), step) for r in range(len(cand))])


@pytest.mark.parametrize("vocab", [1, 2, 63, 64, 65, 511, 512, 8192, 32000, 128256])
@pytest.mark.parametrize("temperature", [1.0, 0.7, 0.0])
def test_sampler_bit_exact(vocab, temperature):
    torch, sr = need_gpu()
    say(f"sampler vocab={vocab} T={temperature}")
    rng = np.random.default_rng(vocab)
    rows = 37
    logits = (rng.standard_normal((rows, vocab)) * rng.uniform(0.5, 6.0, size=(rows, 1))).astype(np.float32)
    logits[0, : min(vocab, 5)] = -np.inf           # excluded tokens
    logits[1] = 3.0                                # all equal
    logits[2, vocab // 2] = 80.0                   # near-deterministic
    cand = rng.permutation(4096)[:rows].astype(np.int32)
    for step in (0, 1, 1023):
        tok = torch.empty(rows, dtype=torch.int32, device="cuda")
        sr.sample(torch.from_numpy(logits).cuda(), torch.from_numpy(cand).cuda(), step, temperature, 42, tok)
        got = tok.cpu().numpy()
        ref = oracle_tokens(logits, cand, step, temperature, 42)
        assert np.array_equal(got, ref), (step, np.flatnonzero(got != ref)[:5])


def test_sampler_weights_near_boundaries():
    """Logits spread over the whole exp range, many rows: every weight must
    round exactly as the oracle's float32 steps."""
    torch, sr = need_gpu()
    rng = np.random.default_rng(11)
    rows, vocab = 512, 4096
    logits = rng.uniform(-30, 0, size=(rows, vocab)).astype(np.float32)
    cand = np.arange(rows, dtype=np.int32)
    tok = torch.empty(rows, dtype=torch.int32, device="cuda")
    sr.sample(torch.from_numpy(logits).cuda(), torch.from_numpy(cand).cuda(), 5, 1.0, 7, tok)
    assert np.array_equal(tok.cpu().numpy(), oracle_tokens(logits, cand, 5, 1.0, 7))


@pytest.mark.parametrize("b,keep", [(1, 1), (2, 1), (7, 3), (64, 16), (103, 21), (512, 103), (1000, 999),
                                    (4096, 410)])
def test_select_bit_exact(b, keep):
    torch, sr = need_gpu()
    rng = np.random.default_rng(b)
    scores = rng.normal(size=b).astype(np.float32)
    scores[rng.integers(0, b, size=b // 5)] = np.float32(0.25)   # ties
    if b > 4:
        scores[1] = np.nan
        scores[2] = -np.inf
        scores[3] = -0.0
    cand = rng.permutation(8192)[:b].astype(np.int32)
    acc = torch.empty(b, dtype=torch.int32, device="cuda")
    sr.select(torch.from_numpy(scores).cuda(), torch.from_numpy(cand).cuda(), keep, acc)
    got = acc.cpu().numpy()
    sd = {int(c): float(s) for c, s in zip(cand, scores)}
    kept = set(specrej.top_k([int(c) for c in cand], sd, keep))
    ref = np.array([1 if int(c) in kept else 0 for c in cand])
    assert got.sum() == keep and np.array_equal(got, ref)


@pytest.mark.parametrize("elem_bytes,hd", [(2, 128), (2, 64), (4, 32)])
def test_compact_bit_exact(elem_bytes, hd):
    torch, sr = need_gpu()
    rng = np.random.default_rng(hd)
    nl, hkv, b, cap_src, cap_dst, length = 3, 2, 37, 20, 33, 19
    dt = np.uint16 if elem_bytes == 2 else np.uint32
    sb = b * hkv * cap_src * hd + 17
    db = b * hkv * cap_dst * hd + 5
    src = rng.integers(0, 2**15, size=2 * nl * sb).astype(dt)
    flags = (rng.random(b) < 0.4).astype(np.int32)
    flags[0] = 1
    tdt = torch.int16 if elem_bytes == 2 else torch.int32
    s_t = torch.from_numpy(src.view(np.int16 if elem_bytes == 2 else np.int32)).cuda()
    d_t = torch.zeros(2 * nl * db, dtype=tdt, device="cuda")
    src_row = torch.full((b,), -1, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    sr.compact(s_t, sb, d_t, db, torch.from_numpy(flags).cuda(), nl, hkv, hd, elem_bytes, cap_src, cap_dst, length,
               src_row, cnt)
    torch.cuda.synchronize()
    kept = np.flatnonzero(flags)
    assert int(cnt.item()) == len(kept)
    assert np.array_equal(src_row.cpu().numpy()[: len(kept)], kept)
    dst = d_t.cpu().numpy().view(dt)
    for blk in range(2 * nl):
        S = src[blk * sb: blk * sb + b * hkv * cap_src * hd].reshape(b, hkv, cap_src, hd)
        Dd = dst[blk * db: blk * db + b * hkv * cap_dst * hd].reshape(b, hkv, cap_dst, hd)
        assert np.array_equal(Dd[: len(kept), :, :length], S[kept, :, :length])
        assert not Dd[len(kept):].any() and not Dd[:, :, length:].any()


@pytest.mark.parametrize("b,keep_frac,length,hkv,hd", [(1, 1.0, 1, 1, 64), (300, 0.0, 5, 2, 64), (257, 1.0, 65, 3, 128),
                                                       (4096, 0.02, 3, 1, 64), (9, 0.5, 0, 2, 64),
                                                       (40, 0.6, 130, 8, 128)])
def test_compact_edges(b, keep_frac, length, hkv, hd):
    """Compaction at the edges of its packing and chunks: one row, no row and
    every row kept, the most rows, no tokens, runs of just over one and two
    16 KB chunks."""
    torch, sr = need_gpu()
    say(f"compact b={b} keep={keep_frac} len={length} hkv={hkv} hd={hd}")
    rng = np.random.default_rng(b + length)
    nl, cap = 2, max(length, 1)
    blk = b * hkv * cap * hd
    src = torch.from_numpy(rng.integers(0, 2**15, size=(2 * nl, b, hkv, cap, hd)).astype(np.int16)).cuda()
    dst = torch.zeros_like(src)
    flags = (rng.random(b) < keep_frac).astype(np.int32)
    src_row = torch.full((b,), -1, dtype=torch.int32, device="cuda")
    cnt = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    sr.compact(src, blk, dst, blk, torch.from_numpy(flags).cuda(), nl, hkv, hd, 2, cap, cap, length, src_row, cnt)
    torch.cuda.synchronize()
    kept = np.flatnonzero(flags)
    assert int(cnt.item()) == len(kept)
    assert np.array_equal(src_row.cpu().numpy()[: len(kept)], kept) and bool((src_row[len(kept):] == -1).all())
    ref = torch.zeros_like(src)
    ref[:, : len(kept), :, :length] = src[:, torch.from_numpy(kept).cuda(), :, :length]
    assert torch.equal(dst, ref)


@pytest.mark.parametrize("b,keep_frac,length,cap,hkv,hd,nl", [(600, 0.2, 127, 130, 4, 128, 4),   # runs of two chunks
                                                             (600, 0.9, 16, 16, 4, 128, 32),    # more chunks than work-groups
                                                             (600, 0.0, 127, 127, 4, 128, 4),
                                                             (4096, 1.0, 33, 34, 2, 128, 4)])
def test_compact_large(b, keep_frac, length, cap, hkv, hd, nl):
    """From 512 MB of rows that may move, the flags are packed by a launch of
    their own and the copy walks the row list."""
    torch, sr = need_gpu()
    say(f"compact large b={b} keep={keep_frac} len={length} hkv={hkv} hd={hd} nl={nl}")
    assert b * hkv * length * hd * 2 * 2 * nl >= 512 << 20
    g = torch.Generator(device="cuda").manual_seed(b + length)
    blk = b * hkv * cap * hd
    src = torch.randint(-2**15, 2**15, (2 * nl, b, hkv, cap, hd), generator=g, dtype=torch.int16, device="cuda")
    flags = (torch.rand(b, generator=g, device="cuda") < keep_frac).int()
    dst = torch.full_like(src, 3)
    src_row = torch.full((b,), -1, dtype=torch.int32, device="cuda")
    cnt = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    sr.compact(src, blk, dst, blk, flags, nl, hkv, hd, 2, cap, cap, length, src_row, cnt)
    torch.cuda.synchronize()
    kept = torch.nonzero(flags).flatten()
    n = len(kept)
    assert int(cnt.item()) == n and torch.equal(src_row[:n].long(), kept) and bool((src_row[n:] == -1).all())
    assert torch.equal(dst[:, :n, :, :length], src[:, kept, :, :length])
    assert bool((dst[:, n:] == 3).all()) and bool((dst[:, :, :, length:] == 3).all())


@pytest.mark.parametrize("vocab", [24576, 24577, 24579, 32768, 50257, 131071, 262144])
@pytest.mark.parametrize("temperature", [1.0, 0.3, 0.0])
def test_sampler_segment_edges(vocab, temperature):
    """Vocabularies around the change of segment length, odd ones (rows that
    are not 16-byte aligned) and the largest; NaN, infinities, several
    maxima, rows without a distribution and late steps."""
    torch, sr = need_gpu()
    say(f"sampler edges vocab={vocab} T={temperature}")
    rng = np.random.default_rng(vocab + 1)
    rows = 13
    logits = (rng.standard_normal((rows, vocab)) * rng.uniform(0.5, 8.0, size=(rows, 1))).astype(np.float32)
    logits[0, ::3] = np.nan
    logits[1] = -np.inf
    logits[2, 5:] = -np.inf
    logits[3, vocab - 40:] = 9.0                    # many weights of exactly 2^32, at the row's end
    logits[4] = np.nextafter(np.float32(1), np.float32(0))
    logits[4, 7::11] = 1.0
    logits[5] = -0.0
    logits[5, vocab // 3] = 0.0
    logits[6] = np.nan
    logits[7, vocab - 1] = 60.0
    logits[8] -= 3.0e38
    cand = rng.permutation(4096)[:rows].astype(np.int32)
    for step in (0, 517):
        tok = torch.empty(rows, dtype=torch.int32, device="cuda")
        sr.sample(torch.from_numpy(logits).cuda(), torch.from_numpy(cand).cuda(), step, temperature, 1 << 40 | 9, tok)
        with np.errstate(all="ignore"):
            ref = oracle_tokens(logits, cand, step, temperature, 1 << 40 | 9)
        assert np.array_equal(tok.cpu().numpy(), ref), (step, np.flatnonzero(tok.cpu().numpy() != ref))
