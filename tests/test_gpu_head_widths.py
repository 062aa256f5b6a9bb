"""The matrix-core kernels for head widths other than bf16 x 128 (score_any.hip, nearest_any.hip) against the oracle:
widths that fill their operand steps and widths that do not, prompts around the 32-row block and the strip of 16, 32 or
64 rows, grids on both sides of the size from which a wave holds several groups of stationary rows."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_2406_18139_amd import build, lookm
from tests import parity

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32
SHAPES = [(1, 33, 8, BF), (2, 95, 24, BF), (2, 129, 40, BF), (3, 161, 72, BF), (1, 257, 104, BF), (2, 97, 160, BF),
          (1, 63, 200, BF), (2, 200, 256, BF), (1, 31, 16, F32), (2, 65, 24, F32), (1, 96, 48, F32), (2, 127, 72, F32),
          (1, 160, 96, F32), (2, 70, 128, F32), (1, 130, 168, F32), (1, 90, 248, F32),
          (16, 1100, 64, BF), (9, 1999, 80, BF), (16, 1100, 32, F32), (10, 900, 136, BF), (12, 800, 128, F32)]


@pytest.mark.parametrize("H,L,d,dtype", SHAPES)
def test_scores_and_matching_at_every_head_width(H, L, d, dtype):
    g = torch.Generator().manual_seed(1000 * d + L)
    q = torch.randn(H, L, d, generator=g).to(dtype)
    k = torch.randn(H, L, d, generator=g).to(dtype)
    heads = sorted({0, H // 2, H - 1})              # the oracle on three heads of a wide layer
    # the fp32 sum of d products is off by about sqrt(d) 2^-24 |q||k| / sqrt(d) <= 16 * 16 * 2^-24 in a logit and twice
    # that (logit and log-sum-exp) in an exponential: 3e-5 for the widest heads, 1e-5 measured
    ref = oracle.scores(q[heads].contiguous(), k[heads].contiguous())
    s = lookm.lookm_scores(q.cuda(), k.cuda())
    assert torch.equal(s, lookm.lookm_scores(q.cuda(), k.cuda()))
    got = s.cpu().numpy().astype(np.float64)
    assert (np.abs(got[heads] - ref) / ref).max() < 3e-5
    np.testing.assert_allclose(got.sum(1), L, rtol=1e-5)
    rng = np.random.default_rng(d)
    B = max(1, int(L * rng.choice([0.1, 0.45, 0.9])))
    kept = np.stack([np.sort(rng.choice(L, B, replace=False)) for _ in range(H)]).astype(np.int32)
    ev = np.stack([np.setdiff1d(np.arange(L), kept[h]) for h in range(H)]).astype(np.int32)
    a, sim = lookm.lookm_nearest(k.cuda(), torch.from_numpy(kept).cuda(), torch.from_numpy(ev).cuda())
    a, sim, kf = a.cpu().numpy(), sim.cpu().numpy(), k.float().numpy()
    assert sum(parity.check_nearest(kf[h], kept[h], ev[h], a[h], sim[h]) for h in heads) == 0   # rows in the tie band


@pytest.mark.parametrize("H", [1, 16])                  # strips of 16 rows; of 64 and 32 rows
@pytest.mark.parametrize("d,dtype", [(16, BF), (64, BF), (96, BF), (256, BF), (8, F32), (64, F32), (128, F32), (200, F32)])
def test_scores_of_prompts_that_end_inside_a_strip(H, d, dtype):
    """Prompts around the pieces that a strip's rows and a block's rows are loaded in (4 to 16 rows a wave): rows past the end
    repeat the last one.  fp32 logits are off by at most sqrt(d) 2^-24 |q||k| / sqrt(d), twice that in an exponential (3e-5)."""
    extra = 270 if H > 1 else 0
    for L in [extra + n for n in (1, 2, 7, 8, 9, 15, 17, 31, 32, 33, 63, 64, 65, 97)]:
        g = torch.Generator().manual_seed(1000 * d + L)
        q, k = torch.randn(H, L, d, generator=g).to(dtype), torch.randn(H, L, d, generator=g).to(dtype)
        got = lookm.lookm_scores(q.cuda(), k.cuda()).cpu().numpy().astype(np.float64)
        heads = [0, H - 1]
        np.testing.assert_allclose(got[heads], oracle.scores(q[heads].contiguous(), k[heads].contiguous()), rtol=3e-5, err_msg=str(L))
        lse = torch.from_numpy(oracle.row_lse(q, k)).float().cuda()
        own = lookm.lookm_scores_lse(q.cuda(), k.cuda(), lse).cpu().numpy()
        np.testing.assert_allclose(own, got, rtol=3e-5, err_msg=str(L))


@pytest.mark.parametrize("H,kvh,L,d,dtype,window", [(6, 2, 150, 80, BF, 45), (16, 8, 700, 64, BF, 333), (8, 2, 210, 40, F32, 1)])
def test_grouped_heads_windows_and_supplied_lse(H, kvh, L, d, dtype, window):
    g = torch.Generator().manual_seed(d)
    q, k = torch.randn(H, L, d, generator=g).to(dtype), torch.randn(kvh, L, d, generator=g).to(dtype)
    s = lookm.lookm_scores_grouped(q.cuda(), k.cuda()).cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(s, oracle.scores_grouped(q, k), rtol=3e-5)
    kr = k.repeat_interleave(H // kvh, 0)
    w = lookm.lookm_scores_window(q.cuda(), kr.cuda(), window).cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(w, oracle.scores_window(q, kr, window), rtol=3e-5, atol=1e-12)
    lse = torch.from_numpy(oracle.row_lse(q, kr)).float().cuda()
    own = lookm.lookm_scores_lse(q.cuda(), kr.cuda(), lse).cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(own, oracle.scores(q, kr), rtol=3e-5)


@pytest.mark.parametrize("d,dtype", [(80, BF), (64, BF), (24, F32), (64, F32)])      # widths that leave a step unfilled, and full ones
def test_infinite_keys_and_nan_queries_stay_where_they_are(d, dtype):
    L, at = 203, 40
    g = torch.Generator().manual_seed(d)
    q, k = torch.randn(1, L, d, generator=g).to(dtype), torch.randn(1, L, d, generator=g).to(dtype)
    q[:, :, 0] = -1.0
    k[:, at, 0] = float("inf")                      # every logit of this key is -inf: it weighs nothing
    logits = (q.double()[0] @ k.double()[0].t()) / d ** 0.5
    p = torch.softmax(logits.masked_fill(torch.ones(L, L).triu(1).bool(), -float("inf")), 1)
    got = lookm.lookm_scores(q.cuda(), k.cuda()).cpu().double()[0]
    np.testing.assert_allclose(got.numpy(), p.sum(0).numpy(), rtol=3e-5)
    bad = 77
    q[:, bad] = float("nan")                        # reaches the keys up to it, and no later one
    got = lookm.lookm_scores(q.cuda(), k.cuda()).cpu().double()[0]
    assert got[:bad + 1].isnan().all()
    np.testing.assert_allclose(got[bad + 1:].numpy(), p[bad + 1:].sum(0)[bad + 1:].numpy(), rtol=3e-5)
    window = L - bad - 1                            # rows bad + 1 .. L - 1: the window begins inside the row's block
    got = lookm.lookm_scores_window(q.cuda(), k.cuda(), window).cpu().double()[0]
    np.testing.assert_allclose(got.numpy(), p[bad + 1:].sum(0).numpy(), rtol=3e-5)


@pytest.mark.parametrize("d", [8, 24, 64, 72, 96, 128])
@pytest.mark.parametrize("what", ["plain", "infinite key", "key that rounds to infinity in bf16", "nan query", "tiny and huge", "tiny keys, huge queries", "tiny conserved keys"])
def test_fp32_products_from_bf16_parts(d, what):
    """fp32 with strips of 32 rows multiplies bf16 parts, with strips of 16 rows (few heads) floats: both are off by the fp32
    rounding of a sum of d products, 3e-5 in an exponential, and agree where a block holds what the parts cannot hold."""
    L, H = 203, 40
    g = torch.Generator().manual_seed(d)
    q, k = torch.randn(1, L, d, generator=g), torch.randn(1, L, d, generator=g)
    if what == "infinite key":
        q[:, :, 0] = -1.0
        k[:, 40, 0] = float("inf")
    if what == "key that rounds to infinity in bf16":
        q[:, :, 1] = 1e-38
        k[:, 50, 1] = 3.4e38
    if what == "nan query":
        q[:, 77] = float("nan")
    if what == "tiny keys, huge queries":      # a key's third part is less than a bf16 holds
        q *= 2.0 ** 122
        k *= 2.0 ** -122
    if what == "tiny conserved keys":
        k[:, ::3] *= 2.0 ** -122
    if what == "tiny and huge":
        q *= 1e-30
        k *= 1e30
    one = lookm.lookm_scores(q.cuda(), k.cuda())
    many = lookm.lookm_scores(q.repeat(H, 1, 1).cuda(), k.repeat(H, 1, 1).cuda())
    assert torch.equal(many.nan_to_num(-1), many[:1].nan_to_num(-1).expand_as(many))
    np.testing.assert_allclose(many[0].cpu().numpy(), one[0].cpu().numpy(), rtol=3e-5)
    if what != "nan query":
        p = torch.softmax(((q.double()[0] @ k.double()[0].t()) / d ** 0.5).masked_fill(torch.ones(L, L).triu(1).bool(), -float("inf")), 1)
        np.testing.assert_allclose(many[0].cpu().double().numpy(), p.sum(0).numpy(), rtol=3e-5)
    kept, ev = torch.arange(0, L, 3, dtype=torch.int32)[None], torch.tensor([i for i in range(L) if i % 3], dtype=torch.int32)[None]
    a1, s1 = lookm.lookm_nearest(k.cuda(), kept.cuda(), ev.cuda())
    big = 80                                                  # 135 evicted keys: five strips of 32 a head
    am, sm = lookm.lookm_nearest(k.repeat(big, 1, 1).cuda(), kept.repeat(big, 1).cuda(), ev.repeat(big, 1).cuda())
    assert torch.equal(am, a1.expand_as(am)) and torch.equal(sm.nan_to_num(-9), sm[:1].nan_to_num(-9).expand_as(sm))
    np.testing.assert_allclose(sm[0].cpu().numpy(), s1[0].cpu().numpy(), rtol=1e-5, atol=1e-6)


@pytest.mark.parametrize("d", [8, 24, 64, 128])
@pytest.mark.parametrize("sharp", [1.0, 4.0])
def test_fp32_products_from_parts_are_no_further_off(d, sharp):
    """Scores against binary64, sixteen heads at once (strips of 32 rows, bf16 parts) and the same heads one by one (strips of 16,
    the fp32 instruction), over 45000 scores: the rms of the first is not above the second's (a sample's scatter is 0.5 %), nor,
    on average over the heads, is the largest error of a head (2 to 4 %)."""
    H, L = 16, 700
    rms, largest = torch.zeros(2, dtype=torch.double), torch.zeros(2, dtype=torch.double)
    for seed in range(4):
        g = torch.Generator().manual_seed(10 * d + seed)
        q, k = (torch.randn(H, L, d, generator=g).cuda() for _ in range(2))
        q *= sharp
        logits = torch.stack([q[h].double() @ k[h].double().t().contiguous() for h in range(H)]) / d ** 0.5
        ref = torch.softmax(logits.masked_fill_(torch.ones(L, L, device="cuda").triu(1).bool(), -float("inf")), 2).sum(1)
        for i, got in enumerate((lookm.lookm_scores(q, k), torch.cat([lookm.lookm_scores(q[h:h + 1], k[h:h + 1]) for h in range(H)]))):
            error = ((got.double() - ref) / ref).cpu()
            rms[i] += error.pow(2).mean()
            largest[i] += error.abs().amax(1).mean()
    assert rms[0].sqrt() <= 1.01 * rms[1].sqrt() and largest[0] <= 1.05 * largest[1], (rms.sqrt(), largest)


def small_value_in_every_strip(x, rows=None):
    """One value that bf16 parts hold only in part in every 32 rows, in the second sixteen of some and the first of others."""
    rows = torch.arange(x.shape[1]) if rows is None else rows
    x[:, rows[5::64], 0] = 2.0 ** -105
    x[:, rows[51::64], 1] = -2.0 ** -105
    return x


@pytest.mark.parametrize("d", [8, 24, 56, 64, 104, 128])
def test_fp32_strips_that_bf16_parts_do_not_hold(d):
    """Strips of 32 rows with such a value multiply floats, like strips of 16 rows: the same instruction in the same order, so
    the same bits.  A strip with a NaN row does too, and nothing else changes for it."""
    L, H = 203, 40
    g = torch.Generator().manual_seed(d)
    q, k = (small_value_in_every_strip(torch.randn(1, L, d, generator=g)) for _ in range(2))
    for nan_rows in ([], [77, 150]):
        q[:, nan_rows] = float("nan")
        one = lookm.lookm_scores(q.cuda(), k.cuda())
        many = lookm.lookm_scores(q.repeat(H, 1, 1).cuda(), k.repeat(H, 1, 1).cuda())
        assert torch.equal(many.nan_to_num(-1), one.nan_to_num(-1).expand_as(many))
        assert torch.isnan(many).sum() == H * ((nan_rows[-1] + 1) if nan_rows else 0)
    kept, ev = torch.arange(0, L, 3, dtype=torch.int32)[None], torch.tensor([i for i in range(L) if i % 3], dtype=torch.int32)[None]
    big = 80                                                  # 135 evicted keys: five strips of 32 a head
    plain = torch.randn(1, L, d, generator=g)
    short = plain.clone()
    short[:, ::3] *= 2.0 ** -120
    for k in (small_value_in_every_strip(plain, ev[0].long()), short):      # short conserved keys beside longer evicted ones
        a1, s1 = lookm.lookm_nearest(k.cuda(), kept.cuda(), ev.cuda())
        am, sm = lookm.lookm_nearest(k.repeat(big, 1, 1).cuda(), kept.repeat(big, 1).cuda(), ev.repeat(big, 1).cuda())
        assert torch.equal(am, a1.expand_as(am)) and torch.equal(sm, s1.expand_as(sm))


def test_fp32_strips_known_to_need_floats_skip_the_parts():
    """Such strips cost what the fp32 instruction costs, 1.5 times the parts' time at 128 dims (with the parts first and the rows
    from memory again: 3.6 times)."""
    H, L, d = 16, 1483, 128
    g = torch.Generator().manual_seed(0)
    plain = [torch.randn(H, L, d, generator=g).cuda() for _ in range(2)]
    small = [small_value_in_every_strip(x.clone()) for x in plain]
    ws = lookm.alloc_workspace(H, L, d, 0, lookm.F32, "cuda")
    times = {}
    for _ in range(5):
        for name, (q, k) in (("plain", plain), ("small", small)):
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            lookm.lookm_scores(q, k, workspace=ws)
            begin.record()
            for _ in range(20):
                lookm.lookm_scores(q, k, workspace=ws)
            end.record()
            end.synchronize()
            times[name] = min(times.get(name, float("inf")), begin.elapsed_time(end))
    assert times["small"] < 2.2 * times["plain"], times


@pytest.mark.parametrize("d,dtype", [(64, BF), (80, BF), (256, BF), (24, F32), (128, F32)])
def test_scores_logits_that_jump_late_in_the_row(d, dtype):
    # the twin of the test of that name for bf16 x 128: a block more than 64 binades above the row's reference makes pass 1
    # take a new one, in the middle of rows, in interior and in diagonal blocks
    H, L = 2, 900
    g = torch.Generator().manual_seed(d)
    q, k = torch.randn(H, L, d, generator=g), torch.randn(H, L, d, generator=g) * 0.02
    for j in (130, 131, 400, 777, 899):
        k[:, j] *= 1500.0
    q, k = q.to(dtype), k.to(dtype)
    logits = (q.double() @ k.double().transpose(1, 2)) / d ** 0.5 * np.log2(np.e)
    assert (logits[:, 400:, 400] - logits[:, 400:, :400].amax(2)).max() > 64
    s = lookm.lookm_scores(q.cuda(), k.cuda()).cpu().numpy().astype(np.float64)
    ref = oracle.scores(q, k)
    assert np.all(np.isfinite(s))
    # logits of up to 150 in magnitude, rounded to 2^-17 in their sums and in the log-sum-exp
    big = ref > 1e-6
    assert (np.abs(s - ref)[big] / ref[big]).max() < 1e-4
    assert np.abs(s - ref)[~big].max() < 1e-9
    np.testing.assert_allclose(s.sum(1), L, rtol=1e-5)


@pytest.mark.parametrize("d,dtype,group,window,own_lse", [(64, F32, 1, 0, False), (64, BF, 1, 0, False), (24, BF, 2, 0, False), (128, F32, 1, 40, False),
                                                          (8, F32, 1, 0, True), (256, BF, 1, 0, False)])
def test_weights_below_the_normal_range_are_kept(d, dtype, group, window, own_lse):
    # The first key takes all the attention; the others' logits lie 60 to 103 below (natural units), their weights around and
    # far below 2^-126 = e^-87.3, down to the smallest number fp32 has.
    L = 300
    q, k = torch.zeros(group, L, d), torch.zeros(1, L, d)
    q[..., 0] = 8.0 * d ** 0.5
    k[0, 1:, 0] = -torch.linspace(60, 103, L - 1) / 8
    q, k = q.to(dtype), k.to(dtype)
    logits = (q.double() @ k[0].double().t()) / d ** 0.5
    p = torch.softmax(logits.masked_fill(torch.ones(L, L).triu(1).bool(), -float("inf")), 2)
    want = p[:, L - window if window else 0:].sum((0, 1))
    qg, kg = q.cuda(), k.cuda()
    if own_lse:
        lse = torch.logsumexp(logits.masked_fill(torch.ones(L, L).triu(1).bool(), -float("inf")), 2).float()
        got = lookm.lookm_scores_lse(qg, kg, lse.cuda())
    elif window:
        got = lookm.lookm_scores_window(qg, kg, window)
    else:
        got = lookm.lookm_scores_grouped(qg, kg)
    got = got.cpu().double()[0]
    # exponents of up to 150 binades are rounded to 2^-17: 5e-6 of the weight and once more for the log-sum-exp; a subnormal
    # weight is rounded to 2^-149, and its sum over the rows with it
    assert ((got - want).abs() <= 2e-5 * want + group * L * 2.0 ** -149).all()
    assert (want < 2.0 ** -126).sum() > 50 and got[1:].unique().numel() > 250


@pytest.mark.parametrize("d,dtype", [(64, BF), (80, BF), (256, BF), (24, F32), (128, F32)])
def test_nearly_equal_cosines_are_decided_by_the_sum_in_the_order_of_the_dims(d, dtype):
    # Evicted keys that read the same backwards, and for each a conserved key and its mirror image: equal dots and norms in
    # exact arithmetic, so that only the rounding of a particular order of the sum tells them apart.
    n = 150
    g = torch.Generator().manual_seed(d)
    half = torch.randn(n, d // 2, generator=g)
    e = torch.cat([half, half.flip(1)], 1).to(dtype)
    c = (e.float() + 0.3 * torch.randn(n, d, generator=g)).to(dtype)
    k = torch.cat([e, c, c.flip(1)])[None].contiguous()
    perm = torch.randperm(2 * n, generator=g)       # slot -> conserved key; both orders of the pairs, near and far apart
    k[0, n:] = k[0, n:][perm]
    at = torch.argsort(perm)
    pair = torch.stack([at[:n], at[n:]], 1).sort(1).values.numpy()
    kf = k[0].double().numpy()
    dot = np.zeros((n, 2), np.float32)
    for i in range(d):                              # fused multiply-adds: one rounding to fp32 per dim
        dot = (kf[:n, None, i] * kf[n + pair, i] + dot.astype(np.float64)).astype(np.float32)
    rn = (1 / np.sqrt((kf[n + pair] ** 2).sum(-1))).astype(np.float32)
    val = dot * rn
    want = np.where(val[:, 1] > val[:, 0], pair[:, 1], pair[:, 0])
    assert 0.1 < (val[:, 0] != val[:, 1]).mean() and 0.03 < (want == pair[:, 1]).mean()
    kept, ev = (torch.arange(n, 3 * n)[None].int().cuda(), torch.arange(n)[None].int().cuda())
    a, _ = lookm.lookm_nearest(k.cuda(), kept, ev)
    assert (a.cpu().numpy()[0] == want).all()


def test_more_heads_than_one_grid_dimension_holds():
    # 2^24 workgroups of 256 threads are 2^32: a batch of prompts folded into the heads passes that with a workgroup per head
    H, d = (1 << 24) + 200_001, 8
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn((H, 2, d), generator=g, device="cuda").to(BF)
    logits = (x[:, 1, None].float() * x.float()).sum(2) / d ** 0.5          # of row 1; row 0 sees key 0 alone
    want = torch.softmax(logits, 1)
    want[:, 0] += 1
    assert (lookm.lookm_scores(x, x) - want).abs().max() < 1e-5
    k = torch.cat([x, torch.randn((H, 1, d), generator=g, device="cuda").to(BF)], 1)
    kept = torch.tensor([0, 2], dtype=torch.int32, device="cuda").repeat(H, 1)
    ev = torch.ones((H, 1), dtype=torch.int32, device="cuda")
    a, sim = lookm.lookm_nearest(k, kept, ev)
    cos = torch.nn.functional.cosine_similarity(k[:, 1, None].float(), k[:, ::2].float(), dim=2)
    assert (sim[:, 0] - cos.max(1).values).abs().max() < 1e-5
    clear = (cos[:, 0] - cos[:, 1]).abs() > 1e-5
    assert torch.equal(a[clear, 0].long(), cos.argmax(1)[clear])


@pytest.mark.parametrize("d,dtype,n,padding", [(64, BF, 150, 40), (80, BF, 60, 700), (256, BF, 40, 3), (24, F32, 150, 0), (128, F32, 90, 300),
                                               (32, BF, 1200, 0)])
def test_more_than_two_nearly_equal_cosines(d, dtype, n, padding):
    # Evicted keys that are the same read backwards and with their halves swapped.  For each, a conserved key in its four
    # arrangements - equal dots and norms in exact arithmetic - and one of them twice: five candidates apart by roundings.
    g = torch.Generator().manual_seed(d + n)
    quarter = torch.randn(n, d // 4, generator=g)
    a = torch.cat([quarter, quarter.flip(1)], 1)
    e = torch.cat([a, a], 1).to(dtype)
    c = (e.float() + 0.3 * torch.randn(n, d, generator=g)).to(dtype)
    swap = lambda x: torch.cat([x[:, d // 2:], x[:, :d // 2]], 1)
    arranged = [c, c.flip(1), swap(c), swap(c.flip(1))]
    twice = torch.stack(arranged)[torch.randint(0, 4, (n,), generator=g), torch.arange(n)]
    other = torch.randn(padding, d, generator=g).to(dtype)         # conserved keys of no interest, one of them NaN
    if padding:
        other[padding // 2, 1] = float("nan")
    k = torch.cat([e, *arranged, twice, other])[None].contiguous()
    perm = torch.randperm(5 * n + padding, generator=g)
    k[0, n:] = k[0, n:][perm]
    kf = k[0].double().numpy()
    dot = np.zeros((n, 5 * n + padding), np.float32)
    for i in range(d):                              # fused multiply-adds: one rounding to fp32 per dim
        dot = (kf[:n, None, i] * kf[None, n:, i] + dot.astype(np.float64)).astype(np.float32)
    val = dot * (1 / np.sqrt((kf[n:] ** 2).sum(-1))).astype(np.float32)
    want = np.where(np.isnan(val), -np.inf, val).argmax(1)       # the lowest slot of the largest value
    kept, ev = (torch.arange(n, 6 * n + padding)[None].int().cuda(), torch.arange(n)[None].int().cuda())
    got, _ = lookm.lookm_nearest(k.cuda(), kept, ev)
    assert (got.cpu().numpy()[0] == want).all()
    # every conserved key a copy of the same one, and an evicted key of zeros among the others: the lowest slot
    k[0, n:] = c[0]
    k[0, 1] = 0
    got, _ = lookm.lookm_nearest(k.cuda(), kept, ev)
    assert (got == 0).all()


@pytest.mark.parametrize("d", [40, 48, 56, 64])
@pytest.mark.parametrize("group", [1, 4])
def test_remainders_by_dots_and_by_subtraction(d, group):
    """Between 577 and 1152 strips of 32 rows (pass 1: 2816) that go along 3500 rows and more the remainders of fp32 parts are
    differences, otherwise they are dots: the same bits.  Eight heads of 110 strips against each half of them; of grouped heads the
    strips of pass 2 go along four queries a row, and are too few for it."""
    L = 3517
    g = torch.Generator(device="cuda").manual_seed(d)
    q, k = torch.randn(8, L, d, generator=g, device="cuda"), torch.randn(8 // group, L, d, generator=g, device="cuda")
    halves = [lookm.lookm_scores_grouped(q[a:a + 4].contiguous(), k[a // group:(a + 4) // group].contiguous()) for a in (0, 4)]
    assert torch.equal(lookm.lookm_scores_grouped(q, k), torch.cat(halves))


def test_bf16_parts_bit_for_bit():
    """The three parts of a float are the nearest bf16 of what the parts before leave, whichever instruction works the remainders out
    and in either place of a pair: four million floats of every exponent that bf16 holds, both signs, subnormal ones and subnormal
    remainders among them, next to others of any magnitude.  An odd last step leaves zeros."""
    lib = ctypes.CDLL(str(build.SPLIT_CHECK if build.SPLIT_CHECK.exists() else build.build_split_check()))
    n = 1 << 22
    g = torch.Generator().manual_seed(3)
    bits = torch.randint(0, 1 << 23, (n,), generator=g, dtype=torch.int32)                # mantissas; a quarter of them short
    bits &= torch.where(torch.rand(n, generator=g) < 0.25, torch.full((), 0x7f8000), torch.full((), 0x7fffff)).int()
    bits |= torch.randint(0, 255, (n,), generator=g, dtype=torch.int32) << 23
    bits = torch.minimum(bits, torch.full((), 0x7f7f7fff, dtype=torch.int32))             # above: rounds to infinity
    x = torch.where(torch.rand(n, generator=g) < 0.5, -1.0, 1.0) * bits.view(torch.float32)
    x[:8] = torch.tensor([0.0, -0.0, 2.0 ** -149, -2.0 ** -149, 2.0 ** -126, 3.3895e38, -3.3895e38, 1.0])
    rest, want = x.clone(), []
    for _ in range(3):
        want.append(rest.bfloat16())
        rest = rest - want[-1].float()
    want = torch.stack([w.view(torch.int16).view(n // 8, 8) for w in want], 1)            # [groups, part, value]
    out = torch.empty(3, n // 8, 3, 8, dtype=torch.int16, device="cuda")
    xg = x.cuda()
    assert lib.split_check(ctypes.c_void_p(xg.data_ptr()), n // 8, *(ctypes.c_void_p(o.data_ptr()) for o in out),
                           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    dots, differences, half = out.cpu()
    assert torch.equal(differences, want)
    assert torch.equal(dots, want)
    assert torch.equal(half[:, :, :4], want[:, :, :4]) and not half[:, :, 4:].any()
