"""Decode attention (sr_decode_attention) and prefill attention
(sr_prefill_attention) against the oracle's float64 attention on the same
bf16 / fp32 inputs: shared prefix plus each row's own keys, ragged tails, no
prefix, prefix only, cached history before the new tokens, every query-group
size and head size the kernels take.  Each row's max-abs error is bounded
relative to the max-abs of that row of the oracle's output: 1e-2 for bf16,
1e-5 for fp32."""
import numpy as np
import pytest

from gpu_util import need_gpu, say
from oracle.transformer import causal_attention, decode_attention

pytestmark = pytest.mark.gpu


def bf16_round(a):
    u = a.astype(np.float32).view(np.uint32)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.view(np.float32)


def to_dev(torch, a, bf16):
    if bf16:
        return torch.from_numpy((a.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16).view(np.int16)).cuda()
    return torch.from_numpy(a.astype(np.float32)).cuda()


CASES = [
    # dtype, hd, hq, hkv, rows, P, lt, cap
    ("bf16", 128, 32, 8, 103, 256, 300, 320),
    ("bf16", 128, 32, 8, 21, 256, 700, 704),
    ("bf16", 128, 32, 8, 40, 256, 1, 128),
    ("bf16", 128, 32, 8, 128, 256, 50, 64),
    ("bf16", 128, 32, 8, 160, 256, 20, 32),
    ("bf16", 128, 32, 8, 512, 256, 127, 128),     # first round of the 8B schedule
    ("bf16", 128, 32, 8, 512, 256, 1, 128),
    ("bf16", 128, 32, 8, 1024, 256, 33, 40),      # largest row count of the MFMA streaming form
    ("bf16", 128, 64, 8, 300, 256, 0, 16),
    ("bf16", 128, 16, 8, 129, 40, 300, 320),
    ("bf16", 128, 8, 8, 130, 70, 33, 40),         # one query head per KV head; prefix not a multiple of 64
    ("bf16", 128, 32, 8, 160, 600, 10, 16),       # prefix longer than the stage ring
    ("bf16", 128, 64, 8, 12, 100, 90, 96),
    ("bf16", 128, 32, 8, 17, 0, 77, 80),
    ("bf16", 128, 32, 8, 5, 256, 0, 16),
    ("bf16", 128, 8, 8, 3, 31, 5, 8),
    ("bf16", 128, 16, 2, 9, 64, 130, 130),
    ("bf16", 64, 32, 8, 33, 256, 129, 130),
    ("bf16", 64, 8, 2, 7, 128, 33, 40),
    # row groups sharing the prefix: head_dim 64 at the 1B run's rows, four
    # and eight query heads per KV head, a partial last group
    ("bf16", 64, 32, 8, 256, 256, 129, 130),
    ("bf16", 64, 32, 8, 66, 256, 500, 512),
    ("bf16", 64, 8, 2, 64, 128, 33, 40),
    ("bf16", 128, 64, 8, 101, 256, 77, 80),
    ("bf16", 128, 32, 8, 64, 33, 1, 8),
    # one, two and three blocks a wave; a partial prefix block before the tail;
    # one block in all; tails of whole blocks
    ("bf16", 128, 32, 8, 3, 33, 64, 64),
    ("bf16", 64, 32, 8, 2, 1, 31, 32),
    ("bf16", 64, 8, 8, 5, 95, 97, 100),
    ("bf16", 128, 8, 8, 7, 0, 31, 31),
    ("bf16", 128, 32, 8, 64, 65, 32, 33),
    ("bf16", 128, 64, 8, 70, 31, 161, 161),
    ("bf16", 64, 16, 8, 90, 200, 64, 64),
    ("f32", 32, 4, 4, 16, 32, 17, 64),
    ("f32", 32, 8, 1, 6, 5, 3, 3),
]


@pytest.mark.parametrize("dtype,hd,hq,hkv,rows,P,lt,cap", CASES)
def test_decode_attention(dtype, hd, hq, hkv, rows, P, lt, cap):
    torch, sr = need_gpu()
    say(f"decode attention {dtype} hd={hd} hq={hq} hkv={hkv} rows={rows} P={P} lt={lt} cap={cap}")
    bf16 = dtype == "bf16"
    rng = np.random.default_rng(hd + hq + rows + P + lt)
    q = rng.normal(size=(rows, hq, hd)).astype(np.float32)
    kp, vp = rng.normal(size=(2, hkv, P, hd)).astype(np.float32)
    kt, vt = rng.normal(size=(2, rows, hkv, cap, hd)).astype(np.float32)
    if bf16:
        kp, vp, kt, vt = (bf16_round(a) for a in (kp, vp, kt, vt))
    out = torch.zeros((rows, hq * hd), dtype=torch.int16 if bf16 else torch.float32, device="cuda")
    qd = torch.from_numpy(q).cuda()
    kpd = to_dev(torch, kp, bf16) if P else None
    vpd = to_dev(torch, vp, bf16) if P else None
    sr.decode_attention(qd, kpd, vpd, to_dev(torch, kt, bf16), to_dev(torch, vt, bf16), lt, out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    if bf16:
        got = (got.view(np.uint16).astype(np.uint32) << 16).view(np.float32)
    got = got.reshape(rows, hq, hd)
    worst = 0.0
    for r in range(rows):
        k = np.concatenate([kp.transpose(1, 0, 2), kt[r, :, :lt].transpose(1, 0, 2)], axis=0).astype(np.float64)
        v = np.concatenate([vp.transpose(1, 0, 2), vt[r, :, :lt].transpose(1, 0, 2)], axis=0).astype(np.float64)
        ref = decode_attention(q[r].astype(np.float64), k, v, hkv)
        worst = max(worst, float(np.abs(got[r] - ref).max() / np.abs(ref).max()))
    tol = 1e-2 if bf16 else 1e-5
    assert worst <= tol, worst


PREFILL_CASES = [
    # dtype, hd, hq, hkv, rows, P, t0, lr, cap
    ("bf16", 128, 32, 8, 3, 40, 37, 29, 70),      # matrix-core kernel, ragged tiles
    ("bf16", 128, 32, 8, 2, 256, 128, 100, 636),  # 8B shapes: second scoring round
    ("bf16", 128, 32, 8, 2, 256, 0, 128, 128),    # 8B shapes: first scoring round (one 32-query block a work-group)
    ("bf16", 128, 32, 8, 2, 7, 45, 130, 200),     # ragged last block
    ("bf16", 64, 32, 8, 2, 30, 3, 150, 160),      # head_dim 64
    ("bf16", 128, 16, 8, 2, 20, 5, 70, 80),       # 2 query heads per KV head: 2 blocks a work-group, 3 blocks
    ("bf16", 128, 8, 8, 2, 0, 16, 33, 49),
    ("bf16", 128, 16, 2, 2, 17, 0, 50, 64),
    ("bf16", 128, 32, 8, 1, 5, 0, 1, 1),
    ("bf16", 64, 8, 2, 3, 33, 20, 17, 40),
    # edges of the 32-query blocks and of the 32- and 64-key tiles, grids of one
    # work-group and of hundreds, for every group size
    ("bf16", 128, 32, 8, 1, 31, 0, 32, 32),
    ("bf16", 128, 32, 8, 1, 0, 63, 33, 96),
    ("bf16", 64, 16, 8, 1, 64, 0, 65, 65),
    ("bf16", 128, 32, 8, 32, 33, 31, 64, 96),
    ("bf16", 128, 16, 8, 33, 64, 0, 65, 70),
    ("bf16", 64, 8, 8, 34, 3, 62, 63, 130),
    ("bf16", 64, 32, 4, 40, 127, 1, 70, 71),
    ("f32", 32, 4, 4, 2, 5, 9, 11, 20),
    ("f32", 64, 8, 2, 1, 0, 0, 1, 1),
    ("f32", 32, 8, 1, 2, 3, 64, 40, 110),
]


@pytest.mark.parametrize("dtype,hd,hq,hkv,rows,P,t0,lr,cap", PREFILL_CASES)
def test_prefill_attention(dtype, hd, hq, hkv, rows, P, t0, lr, cap):
    """The new tokens' outputs equal the last lr rows of the causal attention
    of the whole sequence (prefix, cached tokens, new tokens)."""
    torch, sr = need_gpu()
    say(f"prefill attention {dtype} hd={hd} hq={hq} hkv={hkv} rows={rows} P={P} t0={t0} lr={lr} cap={cap}")
    bf16 = dtype == "bf16"
    rng = np.random.default_rng(hd + hq + rows + P + t0 + lr)
    q = rng.normal(size=(rows, lr, hq, hd)).astype(np.float32)
    kp, vp = rng.normal(size=(2, hkv, P, hd)).astype(np.float32)
    ko, vo = rng.normal(size=(2, rows, hkv, cap, hd)).astype(np.float32)   # beyond t0 + lr: never read
    if bf16:
        kp, vp, ko, vo = (bf16_round(a) for a in (kp, vp, ko, vo))
    out = torch.zeros((rows, lr, hq * hd), dtype=torch.int16 if bf16 else torch.float32, device="cuda")
    kpd = to_dev(torch, kp, bf16) if P else None
    vpd = to_dev(torch, vp, bf16) if P else None
    sr.prefill_attention(torch.from_numpy(q).cuda(), kpd, vpd, to_dev(torch, ko, bf16), to_dev(torch, vo, bf16), t0,
                         out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    if bf16:
        got = (got.view(np.uint16).astype(np.uint32) << 16).view(np.float32)
    got = got.reshape(rows, lr, hq, hd)
    T = P + t0 + lr
    worst = 0.0
    for r in range(rows):
        k = np.concatenate([kp.transpose(1, 0, 2), ko[r, :, :t0 + lr].transpose(1, 0, 2)], axis=0).astype(np.float64)
        v = np.concatenate([vp.transpose(1, 0, 2), vo[r, :, :t0 + lr].transpose(1, 0, 2)], axis=0).astype(np.float64)
        qf = np.zeros((T, hq, hd))
        qf[T - lr:] = q[r]
        ref = causal_attention(qf, k, v, hkv)[T - lr:]
        worst = max(worst, float(np.abs(got[r] - ref).max() / np.abs(ref).max()))
    tol = 1e-2 if bf16 else 1e-5
    assert worst <= tol, worst


@pytest.mark.parametrize("hd,hq,hkv,rows,P,t0,lr", [(64, 8, 2, 9, 128, 0, 37), (128, 32, 8, 1, 0, 0, 20),
                                                    (128, 16, 8, 3, 1, 2, 30), (64, 32, 8, 40, 70, 0, 33),
                                                    (128, 64, 8, 5, 90, 0, 70)])
def test_prefill_attention_after_nans(hd, hq, hkv, rows, P, t0, lr):
    """A call whose keys and values are all NaN leaves them in LDS; the next
    call reads none of them (keys past the last one, stages never filled)."""
    torch, sr = need_gpu()
    say(f"prefill after NaN hd={hd} hq={hq} hkv={hkv} rows={rows} P={P} t0={t0} lr={lr}")
    bf = torch.bfloat16
    nan = torch.full((64, 8, 192, 128), float("nan"), dtype=bf, device="cuda")
    qn = torch.zeros((64, 192, 32, 128), dtype=torch.float32, device="cuda")
    sr.prefill_attention(qn, None, None, nan, nan, 0, torch.empty((64, 192, 32 * 128), dtype=bf, device="cuda"))
    g = torch.Generator(device="cuda").manual_seed(hd + lr)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    q = rnd(rows, lr, hq, hd)
    kp, vp = (rnd(hkv, P, hd).to(bf), rnd(hkv, P, hd).to(bf)) if P else (None, None)
    ko, vo = rnd(rows, hkv, t0 + lr, hd).to(bf), rnd(rows, hkv, t0 + lr, hd).to(bf)
    out = torch.empty((rows, lr, hq * hd), dtype=bf, device="cuda")
    sr.prefill_attention(q, kp, vp, ko, vo, t0, out)
    got = out.double().cpu().numpy().reshape(rows, lr, hq, hd)
    for r in range(rows):
        k, v = (np.concatenate([([] if p is None else [p.double().cpu().numpy()]) + [o[r].double().cpu().numpy()]][0],
                               axis=1).transpose(1, 0, 2) for p, o in ((kp, ko), (vp, vo)))
        qf = np.zeros((P + t0 + lr, hq, hd))
        qf[P + t0:] = q[r].double().cpu().numpy()
        ref = causal_attention(qf, k, v, hkv)[P + t0:]
        assert np.abs(got[r] - ref).max() <= 1e-2 * np.abs(ref).max()


def dev_attention64(torch, q, k, v):
    """float64 attention on the device: q [..., G, hd] against k, v [..., T, hd]."""
    s = torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous()) / q.shape[-1] ** 0.5
    return torch.matmul(torch.softmax(s, -1), v.double())


@pytest.mark.parametrize("hd,hq,hkv", [(128, 32, 8), (64, 8, 8), (64, 16, 8), (128, 64, 8)])
@pytest.mark.parametrize("blind", [33, 64, 100])
@pytest.mark.parametrize("how", ["inf", "overflow"])
def test_attention_first_scores_minus_infinity(hd, hq, hkv, blind, how):
    """The first `blind` keys score -inf for every query (infinite key
    components, or products that overflow), all later ones are finite: those
    keys weigh 0 and the others form the softmax, in prefill and in both
    decode forms, also where a wave's first blocks hold no finite score."""
    torch, sr = need_gpu()
    say(f"-inf scores hd={hd} hq={hq} hkv={hkv} blind={blind} {how}")
    bf, rows, P, lr, lt, G = torch.bfloat16, 2, 130, 40, 70, hq // hkv
    g = torch.Generator(device="cuda").manual_seed(hd + hq + blind)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")

    def queries(*s):
        q = rnd(*s)
        q[..., :16] = 2.0   # (16 products of -3e38 x 2 / sqrt(hd) overflow)
        return q
    kp, vp = rnd(hkv, P, hd).to(bf), rnd(hkv, P, hd).to(bf)
    kp[:, :blind, :16] = -float("inf") if how == "inf" else -3.0e38
    ko, vo = rnd(rows, hkv, lr, hd).to(bf), rnd(rows, hkv, lr, hd).to(bf)
    q = queries(rows, lr, hq, hd)
    out = torch.empty((rows, lr, hq * hd), dtype=bf, device="cuda")
    sr.prefill_attention(q, kp, vp, ko, vo, 0, out)
    got = out.double().view(rows, lr, hkv, G, hd)
    assert bool(torch.isfinite(got).all())
    for r in range(rows):
        for t in range(lr):
            k, v = (torch.cat([a[:, blind:], b[r][:, : t + 1]], 1) for a, b in ((kp, ko), (vp, vo)))
            ref = dev_attention64(torch, q[r, t].view(hkv, G, hd), k, v)
            assert float((got[r, t] - ref).abs().max()) <= 1e-2 * float(ref.abs().max())
    for nrow in (5, 70):   # one row a work-group, row groups
        kt, vt = rnd(nrow, hkv, lt, hd).to(bf), rnd(nrow, hkv, lt, hd).to(bf)
        qd = queries(nrow, hq, hd)
        o = torch.empty((nrow, hq * hd), dtype=bf, device="cuda")
        sr.decode_attention(qd, kp, vp, kt, vt, lt, o)
        k, v = (torch.cat([a[:, blind:].expand(nrow, -1, -1, -1), b], 2) for a, b in ((kp, kt), (vp, vt)))
        ref = dev_attention64(torch, qd.view(nrow, hkv, G, hd), k, v)
        dec = o.double().view(nrow, hkv, G, hd)
        assert bool(torch.isfinite(dec).all())
        assert float((dec - ref).abs().max()) <= 1e-2 * float(ref.abs().max())


def rounded_attention64(torch, q, k, v, mask=None):
    """(float64 attention, the same with the roundings the matrix-core kernels
    make: scaled queries, the probabilities relative to the column's maximum
    and the output to bf16)."""
    def attend(s, rnd):
        if mask is not None:
            s = s.masked_fill(mask, -float("inf"))
        p = torch.exp2(s - s.amax(-1, keepdim=True))
        return torch.matmul(rnd(p), v.double()) / p.sum(-1, keepdim=True)
    bf = lambda x: x.to(torch.bfloat16).double()
    kt = k.double().transpose(-1, -2).contiguous()
    scale = np.log2(np.e) / np.sqrt(q.shape[-1])
    return (attend(torch.matmul(q.double() * scale, kt), lambda p: p),
            bf(attend(torch.matmul(bf(q * np.float32(scale)), kt), bf)))


def no_further_off(torch, got, q, k, v, share, mask=None):
    """The error's 2-norm is at most `share` of the rounded form's.  The kernels
    round a little less than it: every maximum of a wave's run so far is exactly
    1 when it is met (measured 0.95-0.973 of it in decoding, 0.984 in prefill).
    With probabilities relative to a stale maximum the largest is rounded too:
    0.99-1.02 and 1.025-1.03.  Over the >= 80 000 outputs here the ratio moves
    by 0.002."""
    ref, emu = rounded_attention64(torch, q, k, v, mask)
    err, bound = float((got.double() - ref).norm()), float((emu - ref).norm())
    say(f"error {err / float(ref.norm()):.6f}, of the rounded form {bound / float(ref.norm()):.6f}")
    assert err <= share * bound


@pytest.mark.parametrize("hd,hq,hkv,rows,P,lt", [(128, 32, 8, 96, 256, 300), (64, 32, 8, 128, 256, 300),
                                                 (128, 32, 8, 21, 256, 700), (64, 32, 8, 37, 256, 699),
                                                 (128, 8, 8, 140, 300, 200)])
def test_decode_attention_error(hd, hq, hkv, rows, P, lt):
    torch, sr = need_gpu()
    say(f"decode attention error hd={hd} hq={hq} rows={rows} P={P} lt={lt}")
    bf, G = torch.bfloat16, hq // hkv
    g = torch.Generator(device="cuda").manual_seed(hd + rows)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    q, kp, vp = rnd(rows, hq, hd), rnd(hkv, P, hd).to(bf), rnd(hkv, P, hd).to(bf)
    kt, vt = rnd(rows, hkv, lt, hd).to(bf), rnd(rows, hkv, lt, hd).to(bf)
    out = torch.empty((rows, hq * hd), dtype=bf, device="cuda")
    sr.decode_attention(q, kp, vp, kt, vt, lt, out)
    k, v = (torch.cat([a.expand(rows, -1, -1, -1), b], 2) for a, b in ((kp, kt), (vp, vt)))
    no_further_off(torch, out.view(rows, hkv, G, hd), q.view(rows, hkv, G, hd), k, v, 0.982)


@pytest.mark.parametrize("hd,hq,hkv,rows,P,t0,lr", [(128, 32, 8, 3, 256, 128, 200), (64, 32, 8, 4, 256, 0, 300),
                                                    (128, 8, 8, 5, 100, 60, 200), (64, 64, 8, 2, 64, 100, 200)])
def test_prefill_attention_error(hd, hq, hkv, rows, P, t0, lr):
    torch, sr = need_gpu()
    say(f"prefill attention error hd={hd} hq={hq} rows={rows} P={P} t0={t0} lr={lr}")
    bf, G, T = torch.bfloat16, hq // hkv, P + t0 + lr
    g = torch.Generator(device="cuda").manual_seed(hd + lr)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    q, kp, vp = rnd(rows, lr, hq, hd), rnd(hkv, P, hd).to(bf), rnd(hkv, P, hd).to(bf)
    ko, vo = rnd(rows, hkv, t0 + lr, hd).to(bf), rnd(rows, hkv, t0 + lr, hd).to(bf)
    out = torch.empty((rows, lr, hq * hd), dtype=bf, device="cuda")
    sr.prefill_attention(q, kp, vp, ko, vo, t0, out)
    k, v = (torch.cat([a.expand(rows, -1, -1, -1), b], 2) for a, b in ((kp, ko), (vp, vo)))
    by_head = lambda x: x.view(rows, lr, hkv, G, hd).permute(0, 2, 3, 1, 4)   # [rows][hkv][G][lr][hd]
    mask = torch.arange(T, device="cuda")[None, :] > (P + t0 + torch.arange(lr, device="cuda"))[:, None]
    no_further_off(torch, by_head(out), by_head(q), k.unsqueeze(2), v.unsqueeze(2), 1.0, mask)


@pytest.mark.parametrize("odd", ["kpre", "vpre", "kown", "vown"])
@pytest.mark.parametrize("hd,hq,hkv,P,t0,lr", [(128, 32, 8, 50, 20, 40), (64, 8, 8, 50, 0, 70), (64, 64, 8, 0, 9, 33)])
def test_prefill_attention_unaligned(hd, hq, hkv, P, t0, lr, odd):
    """Keys or values that start on a 2-byte boundary: no 16-byte copy into LDS
    takes them, the vector kernel does."""
    if P == 0 and odd in ("kpre", "vpre"):
        pytest.skip("no prefix")
    torch, sr = need_gpu()
    say(f"prefill attention unaligned {odd} hd={hd} hq={hq} P={P} t0={t0} lr={lr}")
    rows, G, T = 2, hq // hkv, P + t0 + lr
    g = torch.Generator(device="cuda").manual_seed(hd + lr)

    def operand(name, *shape):
        n = int(np.prod(shape))
        t = torch.randn(n + 8, generator=g, device="cuda").to(torch.bfloat16)
        return t[int(name == odd):][:n].view(shape)
    q = torch.randn((rows, lr, hq, hd), generator=g, device="cuda")
    kp, vp = (operand(n, hkv, P, hd) if P else None for n in ("kpre", "vpre"))
    ko, vo = (operand(n, rows, hkv, t0 + lr, hd) for n in ("kown", "vown"))
    out = torch.empty((rows, lr, hq * hd), dtype=torch.bfloat16, device="cuda")
    sr.prefill_attention(q, kp, vp, ko, vo, t0, out)
    got = out.double().view(rows, lr, hkv, G, hd)
    for r in range(rows):
        for t in (0, 1, 31, 32, lr - 1):
            k, v = (torch.cat(([a] if P else []) + [b[r]], 1)[:, : P + t0 + t + 1] for a, b in ((kp, ko), (vp, vo)))
            ref = dev_attention64(torch, q[r, t].view(hkv, G, hd), k, v)
            assert float((got[r, t] - ref).abs().max()) <= 1e-2 * float(ref.abs().max())
