"""GPU parity, stage by stage, through the C ABI: each kernel against the oracle function for the
same step, on sizes that span several tiles and a ragged tail, plus the degenerate cases."""
import numpy as np
import pytest
import torch

import oracle
from paper_2406_18139_amd import lookm
from tests import parity

pytestmark = pytest.mark.gpu


def rand_qk(H, L, d, dtype, seed, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    q = (torch.randn(H, L, d, generator=g) * scale).to(dtype)
    k = (torch.randn(H, L, d, generator=g) * scale).to(dtype)
    return q, k


@pytest.mark.parametrize("H,L,d,dtype", [
    (3, 700, 128, torch.bfloat16),      # matrix-core path: 3 strips of 256, ragged tail
    (2, 256, 128, torch.bfloat16),      # exactly one strip
    (1, 1, 128, torch.bfloat16),        # single token
    (2, 65, 128, torch.bfloat16),
    (2, 333, 64, torch.bfloat16),       # other widths, bf16
    (2, 256, 64, torch.float32),        # the tiny configuration's shape
    (1, 130, 8, torch.float32),
    (1, 97, 256, torch.float32),
])
def test_scores_match_oracle(H, L, d, dtype):
    q, k = rand_qk(H, L, d, dtype, seed=L * 7 + d)
    s = lookm.lookm_scores(q.cuda(), k.cuda()).cpu().numpy().astype(np.float64)
    ref = oracle.scores(q, k)
    rel = np.abs(s - ref) / ref
    print(f"scores H={H} L={L} d={d} {dtype}: max rel err {rel.max():.3e}")
    assert rel.max() < 2e-5        # far inside the 1e-3 bar
    np.testing.assert_allclose(s.sum(1), L, rtol=1e-5)


@pytest.mark.parametrize("L", [2, 31, 63, 64, 127, 128, 129, 191, 255, 257, 320, 511, 513, 767, 1023, 1025, 1300])
def test_scores_around_tile_and_strip_boundaries(L):
    """Lengths on both sides of the 32-row block, 64-row tile and 256-row strip boundaries of the matrix-core
    kernels: ragged last tiles, waves with nothing to do, tiles skipped above the diagonal."""
    q, k = rand_qk(2, L, 128, torch.bfloat16, seed=1000 + L)
    s = lookm.lookm_scores(q.cuda(), k.cuda()).cpu().numpy().astype(np.float64)
    ref = oracle.scores(q, k)
    assert np.all(np.isfinite(s))
    assert (np.abs(s - ref) / ref).max() < 2e-5
    np.testing.assert_allclose(s.sum(1), L, rtol=1e-5)


def test_scores_large_logits_and_determinism():
    q, k = rand_qk(2, 600, 128, torch.bfloat16, seed=5, scale=4.0)   # logits up to ~ +-60
    a = lookm.lookm_scores(q.cuda(), k.cuda())
    b = lookm.lookm_scores(q.cuda(), k.cuda())
    assert torch.equal(a, b)
    ref = oracle.scores(q, k)
    s = a.cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(s))
    big = ref > 1e-6
    assert (np.abs(s - ref)[big] / ref[big]).max() < 1e-4
    np.testing.assert_allclose(s.sum(1), 600, rtol=1e-5)


def test_scores_logits_that_jump_late_in_the_row():
    # pass 1 sums a block against the row's current reference and only takes a new maximum when that overflows:
    # tiny keys first, then a few keys whose logits lie hundreds of binades higher (and lower), forces the refresh
    # in the middle of rows, in interior and in diagonal tiles
    H, L, d = 2, 900, 128
    g = torch.Generator().manual_seed(12)
    q = torch.randn(H, L, d, generator=g)
    k = torch.randn(H, L, d, generator=g) * 0.02
    for j in (130, 131, 400, 777, 899):
        k[:, j] *= 1500.0                                   # logits of about +-300
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    a = lookm.lookm_scores(q.cuda(), k.cuda())
    assert torch.equal(a, lookm.lookm_scores(q.cuda(), k.cuda()))
    s = a.cpu().numpy().astype(np.float64)
    ref = oracle.scores(q, k)
    assert np.all(np.isfinite(s))
    big = ref > 1e-6
    assert (np.abs(s - ref)[big] / ref[big]).max() < 1e-4
    assert np.abs(s - ref)[~big].max() < 1e-9
    np.testing.assert_allclose(s.sum(1), L, rtol=1e-5)


def test_scores_zero_queries_closed_form():
    L = 1000
    q = torch.zeros(1, L, 128, dtype=torch.bfloat16)
    k = torch.randn(1, L, 128, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16)
    s = lookm.lookm_scores(q.cuda(), k.cuda()).cpu().numpy()[0].astype(np.float64)
    inv = 1.0 / np.arange(1, L + 1)
    np.testing.assert_allclose(s, np.cumsum(inv[::-1])[::-1], rtol=2e-6)


@pytest.mark.parametrize("H,L,d,dtype", [(3, 700, 128, torch.bfloat16), (2, 333, 64, torch.bfloat16),
                                         (2, 256, 64, torch.float32)])
def test_scores_from_a_supplied_row_lse(H, L, d, dtype):
    # the row log-sum-exp a prefill kernel would hold (here: the oracle's, rounded to fp32) replaces pass 1
    q, k = rand_qk(H, L, d, dtype, seed=L + d)
    lse = torch.from_numpy(oracle.row_lse(q, k)).float()
    s = lookm.lookm_scores_lse(q.cuda(), k.cuda(), lse.cuda()).cpu().numpy().astype(np.float64)
    ref = oracle.scores(q, k)
    rel = np.abs(s - ref) / ref
    print(f"scores from row_lse H={H} L={L} d={d} {dtype}: max rel err {rel.max():.3e}")
    assert rel.max() < 2e-5
    own = lookm.lookm_scores(q.cuda(), k.cuda()).cpu().numpy().astype(np.float64)
    assert (np.abs(own - s) / ref).max() < 1e-5       # both routes agree


@pytest.mark.parametrize("H,L,nbytes", [(8, 700, 278016), (32, 700, 1095424), (8, 1482, 675328), (32, 2896, 7579648)])
@pytest.mark.parametrize("window", [0, 300])
def test_compression_in_the_smallest_workspace(H, L, nbytes, window):
    # a smaller workspace than lookm_workspace_bytes gives: longer chunks, nothing written past its end
    d, B = 128, {(8, 700): 200, (32, 700): 160, (8, 1482): 400, (32, 2896): 1000}[H, L]
    q, k = rand_qk(H, L, d, torch.bfloat16, seed=L + H)
    qg, kg, mask = q.cuda(), k.cuda(), torch.ones(L, dtype=torch.uint8, device="cuda")
    run = lambda ws: lookm.lookm_compress(qg, kg, kg, mask, B, 16, "averaged", want_scores=True, workspace=ws, score_window=window)
    full = run(None)
    ws = torch.full((nbytes + 256 + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    start = -ws.data_ptr() % 256
    small = run(ws[start:start + nbytes])
    assert (ws[start + nbytes:] == 0xA5).all()
    # the same fp32 sums in another order: a few last bits in the log-sum-exp and in the column sum, 1.7e-6 measured
    np.testing.assert_allclose(small.scores.cpu().numpy(), full.scores.cpu().numpy(), rtol=1e-5)
    assert (small.kept_idx == full.kept_idx).float().mean() > 0.999      # two scores within that may trade places
    again = run(ws[start:start + nbytes])
    assert torch.equal(again.scores, small.scores) and torch.equal(again.k_out, small.k_out)


@pytest.mark.parametrize("H,L,d,dtype,windows", [
    (2, 700, 128, torch.bfloat16, (1, 63, 64, 65, 300, 699, 700)),      # matrix cores: inside one tile, across chunks
    (2, 3000, 128, torch.bfloat16, (17, 256, 1000, 2999)),
    (1, 333, 64, torch.bfloat16, (5, 200)),                             # other widths
    (2, 256, 64, torch.float32, (16, 255)),
])
def test_window_scores_match_oracle(H, L, d, dtype, windows):
    q, k = rand_qk(H, L, d, dtype, seed=L + d)
    qg, kg = q.cuda(), k.cuda()
    for w in windows:
        s = lookm.lookm_scores_window(qg, kg, w).cpu().numpy().astype(np.float64)
        ref = oracle.scores_window(q, k, w)
        assert np.all(np.isfinite(s))
        # columns that only far-away rows look at can be tiny: relative where it matters, absolute below
        np.testing.assert_allclose(s, ref, rtol=2e-5, atol=1e-12)
        np.testing.assert_allclose(s.sum(1), w, rtol=2e-5)
    full = lookm.lookm_scores(qg, kg)
    assert torch.equal(lookm.lookm_scores_window(qg, kg, L), full)       # the whole prompt: the same launches


@pytest.mark.parametrize("H,kvh,L,d,dtype", [
    (8, 2, 700, 128, torch.bfloat16),       # matrix cores, groups of four
    (6, 3, 1500, 128, torch.bfloat16),
    (4, 1, 300, 64, torch.bfloat16),        # other widths, one key head for all query heads
    (4, 2, 256, 64, torch.float32),
])
def test_grouped_scores_match_oracle(H, kvh, L, d, dtype):
    g = torch.Generator().manual_seed(H * 100 + L)
    q = torch.randn(H, L, d, generator=g).to(dtype)
    k = torch.randn(kvh, L, d, generator=g).to(dtype)
    s = lookm.lookm_scores_grouped(q.cuda(), k.cuda()).cpu().numpy().astype(np.float64)
    ref = oracle.scores_grouped(q, k)
    np.testing.assert_allclose(s, ref, rtol=2e-5)
    # the same sum taken from single-head launches: one query head per key head, repeated keys
    grp = H // kvh
    single = lookm.lookm_scores(q.cuda(), k.repeat_interleave(grp, 0).cuda()).view(kvh, grp, L)
    np.testing.assert_allclose(s, single.double().sum(1).cpu().numpy(), rtol=1e-6)


def select_case(scores, mask, B, M):
    sg = torch.from_numpy(np.asarray(scores, np.float32)).cuda()
    mg = torch.from_numpy(np.asarray(mask, np.uint8)).cuda()
    kept, ev = lookm.lookm_select(sg, mg, B, M)
    return kept.cpu().numpy(), ev.cpu().numpy()


@pytest.mark.parametrize("seed", range(8))
def test_select_matches_oracle_with_ties(seed):
    rng = np.random.default_rng(seed)
    H = 3
    L = int(rng.integers(1, 5000))
    M = int(rng.integers(0, min(L, 70) + 1))
    mask = (rng.random(L) < 0.8).astype(np.uint8)
    coarse = seed % 2 == 0
    scores = (rng.integers(1, 40, (H, L)) / 8.0 if coarse else rng.random((H, L)) + 1e-3).astype(np.float32)
    P = oracle.protected_count(mask, M)
    for B in sorted({P, min(L, P + 1), (P + L) // 2, max(P, L - 1), L}):
        kept, ev = select_case(scores, mask, B, M)
        for h in range(H):
            rk, re_ = oracle.select(scores[h].astype(np.float64), mask, B, M)
            assert kept[h].tolist() == rk.tolist(), (L, M, B, h)
            assert ev[h].tolist() == re_.tolist(), (L, M, B, h)


def test_select_scores_in_a_narrow_range_or_all_equal():
    # keys are re-based to the head's own range before the radix digits are taken
    rng = np.random.default_rng(5)
    L, M = 3000, 10
    mask = (rng.random(L) < 0.9).astype(np.uint8)
    P = oracle.protected_count(mask, M)
    narrow = (1.0 + rng.integers(0, 50, (1, L)) * 2.0 ** -23).astype(np.float32)     # 50 adjacent floats
    # positive, as Eq. 4 scores are, and within what the oracle's literal binary64 add of Eq. 5 resolves
    wide = (10.0 ** rng.uniform(-7, 7, (1, L))).astype(np.float32)
    same = np.full((1, L), 0.37, np.float32)
    two = np.where(rng.random((1, L)) < 0.5, np.float32(1.0e-7), np.float32(3.0e7)).astype(np.float32)
    for scores in (narrow, wide, same, two):
        for B in (P + 1, P + 700, L - 1):
            kept, ev = select_case(scores, mask, B, M)
            rk, re_ = oracle.select(scores[0].astype(np.float64), mask, B, M)
            assert kept[0].tolist() == rk.tolist() and ev[0].tolist() == re_.tolist(), B


@pytest.mark.parametrize("seed", range(4))
def test_select_literal_rule_matches_oracle_for_every_budget(seed):
    # Eq. 8 as printed: below |T u R| the text tokens compete by score and no image token is conserved
    rng = np.random.default_rng(40 + seed)
    H = 2
    L = int(rng.integers(50, 3000))
    M = int(rng.integers(0, 40))
    mask = (rng.random(L) < 0.5).astype(np.uint8)
    scores = (rng.integers(1, 60, (H, L)) / 8.0 if seed % 2 else rng.random((H, L)) + 1e-3).astype(np.float32)
    sg = torch.from_numpy(scores).cuda()
    mg = torch.from_numpy(mask).cuda()
    P = oracle.protected_count(mask, M)
    budgets = sorted({M, M + 1, (M + P) // 2, P - 1, P, P + 1, (P + L) // 2, L} & set(range(M, L + 1)))
    for B in budgets:
        kept, ev = lookm.lookm_select(sg, mg, B, M, rule="literal")
        kept, ev = kept.cpu().numpy(), ev.cpu().numpy()
        for h in range(H):
            rk, re_ = oracle.select(scores[h].astype(np.float64), mask, B, M, "literal")
            assert kept[h].tolist() == rk.tolist() and ev[h].tolist() == re_.tolist(), (L, M, B, h)
        if B < P:
            with pytest.raises(lookm.LookmError) as e:
                lookm.lookm_select(sg, mg, B, M)                     # the default rule still refuses
            assert e.value.code == lookm.ERR_BUDGET_BELOW_PROTECTED


def test_select_degenerate_cases():
    L = 300
    scores = np.random.default_rng(0).random((2, L)).astype(np.float32)
    ones = np.ones(L, np.uint8)
    kept, ev = select_case(scores, ones, 0, 0)                      # nothing conserved
    assert kept.shape == (2, 0) and ev[0].tolist() == list(range(L))
    kept, ev = select_case(scores, ones, L, L)                      # the window is the whole prompt
    assert kept[1].tolist() == list(range(L)) and ev.shape == (2, 0)
    kept, _ = select_case(scores, np.zeros(L, np.uint8), L, 0)      # all text
    assert kept[0].tolist() == list(range(L))
    kept, _ = select_case(scores, ones, 40, 0)                      # text prior off: plain top-B
    for h in range(2):
        assert kept[h].tolist() == np.sort(np.argsort(-scores[h], kind="stable")[:40]).tolist()
    neg = -scores                                                   # negative and zero scores order correctly
    neg[:, 5] = 0.0
    neg[:, 6] = -0.0
    kept, _ = select_case(neg, ones, 3, 0)
    for h in range(2):
        assert kept[h].tolist() == oracle.select(neg[h].astype(np.float64), ones, 3, 0)[0].tolist()


def test_select_reports_budget_below_protected():
    L = 64
    mask = np.zeros(L, np.uint8)
    mask[10:50] = 1
    sg = torch.rand(2, L, device="cuda")
    with pytest.raises(lookm.LookmError) as e:
        lookm.lookm_select(sg, torch.from_numpy(mask).cuda(), 20, 4)   # 24 text + 4 recent (text) -> 24 > 20
    assert e.value.code == lookm.ERR_BUDGET_BELOW_PROTECTED


def split(L, B, seed):
    rng = np.random.default_rng(seed)
    kept = np.sort(rng.choice(L, B, replace=False)).astype(np.int32)
    return kept, np.setdiff1d(np.arange(L, dtype=np.int32), kept)


@pytest.mark.parametrize("H,L,B,d,dtype", [
    (2, 900, 200, 128, torch.bfloat16),    # matrix-core path: ragged conserved and evicted tiles
    (2, 600, 64, 128, torch.bfloat16),
    (1, 300, 1, 128, torch.bfloat16),      # one conserved key
    (1, 300, 299, 128, torch.bfloat16),    # one evicted key
    (1, 32768, 32000, 128, torch.bfloat16),  # the longest prompt the library takes, nearly all of it conserved: nine chunks of 112 blocks
    (2, 500, 130, 64, torch.bfloat16),     # other widths
    (2, 256, 154, 64, torch.float32),
    (1, 100, 30, 8, torch.float32),
])
def test_nearest_matches_oracle(H, L, B, d, dtype):
    g = torch.Generator().manual_seed(L + B)
    cent = torch.randn(H, 16, d, generator=g)
    k = (cent[:, torch.randint(0, 16, (L,), generator=g)] + 0.3 * torch.randn(H, L, d, generator=g)).to(dtype)
    kept = np.stack([split(L, B, 10 + h)[0] for h in range(H)])
    ev = np.stack([split(L, B, 10 + h)[1] for h in range(H)])
    a, s = lookm.lookm_nearest(k.cuda(), torch.from_numpy(kept).cuda(), torch.from_numpy(ev).cuda())
    a, s = a.cpu().numpy(), s.cpu().numpy()
    kf = k.float().numpy()
    ties = sum(parity.check_nearest(kf[h], kept[h], ev[h], a[h], s[h]) for h in range(H))
    print(f"nearest H={H} L={L} B={B} d={d}: {ties} tie-band rows")
    assert ties == 0


def test_nearest_exact_ties_and_zero_keys():
    L, d = 200, 128
    g = torch.Generator().manual_seed(3)
    k = torch.randn(1, L, d, generator=g).to(torch.bfloat16)
    kept, ev = split(L, 50, 4)
    k[0, kept[7]] = k[0, kept[3]]                   # duplicate conserved keys: lower slot must win
    k[0, kept[30]] = k[0, kept[3]] * 2
    k[0, ev[5]] = k[0, kept[3]] * 0.5
    k[0, ev[9]] = 0                                 # zero evicted key: cosine 0 with everything -> slot 0
    k[0, kept[0]] = 0                               # zero conserved key
    a, s = lookm.lookm_nearest(k.cuda(), torch.from_numpy(kept)[None].cuda(), torch.from_numpy(ev)[None].cuda())
    a, s = a.cpu().numpy()[0], s.cpu().numpy()[0]
    ra, rs = oracle.nearest(k[0], kept, ev)
    assert a[5] == 3 and ra[5] == 3 and abs(s[5] - 1.0) < 1e-6
    assert a[9] == 0 and ra[9] == 0 and s[9] == 0.0
    assert np.array_equal(a, ra)


def test_nearest_when_every_cosine_is_negative():
    """Evicted keys that point away from every conserved key: the best cosine is negative, where the integer order
    of float bits is the reverse of their value order - those rows are decided by the exact pass over all slots."""
    L, d, B = 700, 128, 300
    g = torch.Generator().manual_seed(5)
    v = torch.randn(d, generator=g)
    k = torch.empty(1, L, d)
    kept, ev = split(L, B, 6)
    k[0, kept] = v + 0.3 * torch.randn(B, d, generator=g)
    k[0, ev] = -v + 0.3 * torch.randn(L - B, d, generator=g)
    k = k.to(torch.bfloat16)
    a, s = lookm.lookm_nearest(k.cuda(), torch.from_numpy(kept)[None].cuda(), torch.from_numpy(ev)[None].cuda())
    ra, rs = oracle.nearest(k[0].float().numpy(), kept, ev)
    assert rs.max() < 0
    assert np.array_equal(a.cpu().numpy()[0], ra)
    np.testing.assert_allclose(s.cpu().numpy()[0], rs, rtol=0, atol=parity.SIM_ATOL)


@pytest.mark.parametrize("H,Le", [(1, 512), (16, 12288), (3, 30000)])
def test_nearest_near_ties_between_far_apart_blocks(H, Le):
    """Pairs (and triples) of conserved keys whose cosines to an evicted key differ by a few 1e-7 - less than the
    matrix cores' fp32 values can tell apart - sitting 8, 16 or 32 blocks of 32 slots apart.  The matching must
    still be the binary64 one on every row: every block that holds a contender has to reach the exact pass.  With
    16 heads x 48 strips the conserved axis is ONE chunk of 64 blocks, so the members of a pair fall into the same
    block class of the same lane (two contenders that a set of class bits would show as one); with one head the
    axis is cut into 8 chunks and the members sit in different chunks; the third shape has chunks of 12 blocks.
    The twin of a key differs from it in one component (0 against 2^-7), where the evicted keys hold +-2^-7: the
    dot product moves by 2^-14 in about a hundred."""
    d, B = 128, 2048
    g = torch.Generator().manual_seed(11)
    kept_k = torch.randn(B, d, generator=g)
    kept_k[:, 5] = 0
    n_src = 256
    for s in range(n_src):
        for off in ((256,), (512,), (1024,), (256, 512))[s % 4]:
            kept_k[s + off] = kept_k[s]
            kept_k[s + off, 5] = 2.0 ** -7
    src = torch.arange(Le) % n_src
    ev_k = kept_k[src] + 0.05 * torch.randn(Le, d, generator=g)
    ev_k[:, 5] = (2.0 ** -7) * (1 - 2 * (torch.arange(Le) // n_src % 2)).float()
    k1 = torch.cat([kept_k, ev_k]).to(torch.bfloat16)
    k = k1[None].expand(H, -1, -1).contiguous()                       # every head holds the same keys
    kept = np.tile(np.arange(B, dtype=np.int32), (H, 1))
    ev = np.tile(np.arange(B, B + Le, dtype=np.int32), (H, 1))
    a, s = lookm.lookm_nearest(k.cuda(), torch.from_numpy(kept).cuda(), torch.from_numpy(ev).cuda())
    a, s = a.cpu().numpy(), s.cpu().numpy()
    assert all(np.array_equal(a[h], a[0]) and np.array_equal(s[h], s[0]) for h in range(H))
    rows = np.arange(0, Le, max(1, Le // 800))                        # the oracle on a sample of a long list
    ra, rs = oracle.nearest(k1.float().numpy(), kept[0], ev[0][rows])
    twins = int(np.sum(ra >= n_src))
    print(f"near ties: {len(rows)} rows checked, {twins} matched to a twin, {int(np.sum(a[0][rows] != ra))} differ")
    assert len(rows) // 8 < twins < len(rows)                         # both members of a pair win somewhere
    assert np.array_equal(a[0][rows], ra)
    np.testing.assert_allclose(s[0][rows], rs, rtol=0, atol=parity.SIM_ATOL)


@pytest.mark.parametrize("B,Le", [(1024, 4000), (64, 3000), (8, 2000), (2, 600)])
def test_nearest_keys_without_a_similar_conserved_key(B, Le):
    """Evicted keys unrelated to every conserved key: best cosines of 0.35 (1024 conserved keys) down to 0.1 (two).
    The rounding errors of the fp32 dot products grow like 1 / cos relative to the value, so the band inside which
    the matching is decided exactly widens with them, and below a cosine of 0.08 every slot is decided exactly.
    Every conserved key has a twin 2^-14 away in the dot product, so near ties are the rule here; every row must
    still get the binary64 answer."""
    d = 128
    g = torch.Generator().manual_seed(B)
    half = torch.randn(B // 2, d, generator=g)
    half[:, 5] = 0
    twin = half.clone()
    twin[:, 5] = 2.0 ** -7
    kept_k = torch.cat([half, twin])
    ev_k = torch.randn(Le, d, generator=g)
    ev_k[:, 5] = (2.0 ** -7) * (1 - 2 * (torch.arange(Le) % 2)).float()
    k = torch.cat([kept_k, ev_k])[None].to(torch.bfloat16)
    kept = np.arange(B, dtype=np.int32)[None]
    ev = np.arange(B, B + Le, dtype=np.int32)[None]
    a, s = lookm.lookm_nearest(k.cuda(), torch.from_numpy(kept).cuda(), torch.from_numpy(ev).cuda())
    a, s = a.cpu().numpy()[0], s.cpu().numpy()[0]
    ra, rs = oracle.nearest(k[0].float().numpy(), kept[0], ev[0])
    print(f"dissimilar keys, B={B}: best cosines {rs.min():.3f} .. {rs.max():.3f}, {int(np.sum(a != ra))} rows differ")
    assert np.array_equal(a, ra)
    np.testing.assert_allclose(s, rs, rtol=0, atol=parity.SIM_ATOL)


@pytest.mark.parametrize("H,B,Le", [(16, 2048, 12288), (32, 3072, 9216), (2, 1000, 3000)])
def test_nearest_near_ties_scattered_over_the_conserved_axis(H, B, Le):
    """Near-tied conserved keys at random slots (any lane, any entry of a block, any chunk; some in threes), with
    cosine gaps from 3e-8 to 4e-6 - from far below to just above what the matrix-core values resolve - and an
    evicted key for each that prefers one or the other by the sign of one small component.  Chunks of 64, 48 and 8
    blocks: every counter width of the block marks.  The matching must be the binary64 one on every checked row."""
    d = 128
    rng = np.random.default_rng(B + Le)
    g = torch.Generator().manual_seed(B)
    kept_k = torch.randn(B, d, generator=g)
    kept_k[:, 5] = 0
    n_src = B // 5
    slots = rng.permutation(B)
    src_slot, twin_slot, third_slot = slots[:n_src], slots[n_src:2 * n_src], slots[2 * n_src:3 * n_src]
    p_exp = rng.integers(6, 10, n_src)
    for i in range(n_src):
        kept_k[twin_slot[i]] = kept_k[src_slot[i]]
        kept_k[twin_slot[i], 5] = 2.0 ** -int(p_exp[i])
        if i % 3 == 0:
            kept_k[third_slot[i]] = kept_k[src_slot[i]]
            kept_k[third_slot[i], 5] = -(2.0 ** -int(p_exp[i]))
    which = torch.from_numpy(rng.integers(0, n_src, Le))
    ev_k = kept_k[torch.from_numpy(src_slot)[which]] + 0.05 * torch.randn(Le, d, generator=g)
    q_exp = torch.from_numpy(rng.integers(5, 10, Le)).float()
    sign = torch.from_numpy(rng.choice([-1.0, 1.0], Le)).float()
    ev_k[:, 5] = sign * 2.0 ** -q_exp
    k1 = torch.cat([kept_k, ev_k]).to(torch.bfloat16)
    k = k1[None].expand(H, -1, -1).contiguous()
    kept = np.tile(np.arange(B, dtype=np.int32), (H, 1))
    ev = np.tile(np.arange(B, B + Le, dtype=np.int32), (H, 1))
    a, s = lookm.lookm_nearest(k.cuda(), torch.from_numpy(kept).cuda(), torch.from_numpy(ev).cuda())
    a, s = a.cpu().numpy(), s.cpu().numpy()
    assert all(np.array_equal(a[h], a[0]) and np.array_equal(s[h], s[0]) for h in range(H))
    rows = np.arange(0, Le, max(1, Le // 1500))
    ra, rs = oracle.nearest(k1.float().numpy(), kept[0], ev[0][rows])
    print(f"scattered near ties: {len(rows)} rows checked, {int(np.sum(a[0][rows] != ra))} differ")
    assert np.array_equal(a[0][rows], ra)
    np.testing.assert_allclose(s[0][rows], rs, rtol=0, atol=parity.SIM_ATOL)


@pytest.mark.parametrize("mode", ["averaged", "pivotal", "weighted", "none"])
@pytest.mark.parametrize("H,L,B,d,dtype", [
    (2, 700, 150, 128, torch.bfloat16),
    (2, 256, 154, 64, torch.float32),
    (1, 120, 40, 8, torch.float32),
    (1, 300, 77, 256, torch.bfloat16),
    (2, 9000, 2100, 16, torch.bfloat16),     # register-resident sort, 8 entries per thread
    (1, 7000, 5200, 8, torch.float32),       # budget too large for 16 counter rows in LDS: general sort
    (1, 20000, 1500, 8, torch.bfloat16),     # more than 16 K evicted tokens: general sort
])
def test_merge_matches_oracle(mode, H, L, B, d, dtype):
    g = torch.Generator().manual_seed(L * 3 + B)
    k = torch.randn(H, L, d, generator=g).to(dtype)
    v = (torch.randn(H, L, d, generator=g) * 2).to(dtype)
    rng = np.random.default_rng(B)
    kept = np.stack([split(L, B, 20 + h)[0] for h in range(H)])
    ev = np.stack([split(L, B, 20 + h)[1] for h in range(H)])
    # skewed assignment: a few slots collect many members, many collect none
    assign = np.minimum((rng.random((H, L - B)) ** 3 * B).astype(np.int32), B - 1)
    sim = rng.uniform(0.1, 1.0, (H, L - B)).astype(np.float32)
    ko, vo = lookm.lookm_merge(k.cuda(), v.cuda(), torch.from_numpy(kept).cuda(), torch.from_numpy(ev).cuda(),
                               torch.from_numpy(assign).cuda(), torch.from_numpy(sim).cuda(), mode)
    ko, vo = ko.float().cpu().numpy(), vo.float().cpu().numpy()
    for h in range(H):
        parity.check_merge(k[h].float().numpy(), kept[h], ev[h], assign[h], sim[h], mode, ko[h], dtype)
        parity.check_merge(v[h].float().numpy(), kept[h], ev[h], assign[h], sim[h], mode, vo[h], dtype)


def test_merge_everything_into_one_slot():
    # the worst skew: all evicted rows matched to one conserved row
    H, L, B, d = 1, 2000, 10, 128
    g = torch.Generator().manual_seed(9)
    k = torch.randn(H, L, d, generator=g).to(torch.bfloat16)
    kept, ev = split(L, B, 1)
    assign = np.full((1, L - B), 4, np.int32)
    sim = np.full((1, L - B), 0.5, np.float32)
    ko, vo = lookm.lookm_merge(k.cuda(), k.cuda(), torch.from_numpy(kept)[None].cuda(), torch.from_numpy(ev)[None].cuda(),
                               torch.from_numpy(assign).cuda(), torch.from_numpy(sim).cuda(), "averaged")
    parity.check_merge(k[0].float().numpy(), kept, ev, assign[0], sim[0], "averaged", ko[0].float().cpu().numpy(),
                       torch.bfloat16)
    assert torch.equal(ko, vo)


def test_mfma_probe_reports_a_plausible_rate():
    """The measurement aid runs, and the rate it reports lies between a tenth of the datasheet peak and the peak."""
    for mode in (0, 1, 2):        # constant / random operands with 32x32x16, random operands with 16x16x32
        t = lookm.lookm_probe_mfma(mode, 3, iters=256, reps=6)
        assert 250.0 < t < 2600.0, (mode, t)


def merge_kernel(H, B, Le, d):
    """Which kernels merge these lists (the rule of the library; test_which_lists_are_sorted holds it against the library's own
    profile): waves that collect their slots' members, workgroups that do, or a sort before the merge."""
    lanes = 1 << max(0, (-(-d // 8) - 1).bit_length())
    workgroups = H * -(-B // (256 // lanes))
    if lanes >= 8 and Le <= 256 and Le <= 4 * B and H * B * lanes // 64 <= 2048:
        return "waves"
    if lanes >= 8 and Le <= 4096 and workgroups <= (3584 if 8 * lanes != d or Le < 256 else 5120) and workgroups * Le <= 4 << 20:
        return "workgroups"
    return "sort"


@pytest.mark.parametrize("d,dtype", [(64, torch.float32), (40, torch.bfloat16), (128, torch.bfloat16), (200, torch.float32)])
@pytest.mark.parametrize("B,Le", [(1, 1), (16, 63), (16, 64), (16, 65), (17, 65), (70, 257), (154, 102), (256, 1023), (256, 1024), (257, 1025), (500, 1000),
                                  (2, 300), (12, 1023), (31, 4000)])
def test_merge_with_and_without_a_sort(d, dtype, B, Le):
    """Three heads take one way, many more the others: the same heads on all of them.  Waves and workgroups that collect their slots'
    members and the merge of a sorted list all add a slot's members in ascending position, the latter two
    in up to 256 pieces: fp32 sums of n terms in two orders differ by at most n 2^-23 times the largest term, and a bf16
    row rounded from either by one unit in the last place, 2^-7 of its value, more."""
    L = B + Le
    ways = {merge_kernel(H, B, Le, d): H for H in range(16500, 0, -3)}     # the fewest heads that go each way
    assert "sort" in ways and len(ways) == (3 if 1 < Le <= min(256, 4 * B) else 2), ways
    g = torch.Generator().manual_seed(B + Le + d)
    k, v = torch.randn(3, L, d, generator=g).to(dtype).cuda(), torch.randn(3, L, d, generator=g).to(dtype).cuda()
    perm = torch.stack([torch.randperm(L, generator=g) for _ in range(3)])
    kept, ev = perm[:, :B].sort(1)[0].int().cuda(), perm[:, B:].sort(1)[0].int().cuda()
    u = torch.rand(3, Le, generator=g)
    assign = torch.stack([(u[0] * B).long(), torch.full((Le,), B - 1), (u[2] ** 4 * B).long()]).int().cuda()   # even, one set, uneven
    sim = torch.rand(3, Le, generator=g).cuda()
    args = (k, v, kept, ev, assign, sim)
    for mode in ("averaged", "pivotal", "weighted"):
        ko, vo = lookm.lookm_merge(*args, mode)
        for H in ways.values():
            if H == 3:
                continue
            ks, vs = lookm.lookm_merge(*(x.repeat((H // 3,) + (1,) * (x.dim() - 1)) for x in args), mode)
            bound = Le * 2.0 ** -23 * 6.0                                # |terms| < 6 here
            for a, b in ((ks[-3:], ko), (vs[-3:], vo)):
                diff = (a.float() - b.float()).abs()
                assert (diff <= bound + (2.0 ** -7 * b.float().abs() if dtype == torch.bfloat16 else 0.0)).all()
                assert torch.equal(a[1, :B - 1], b[1, :B - 1])           # rows without members: copies
        for h in range(3):
            ref = oracle.merge(k[h].float().cpu().numpy(), *(x[h].cpu().numpy() for x in (kept, ev, assign, sim)), mode)
            assert np.abs(ko[h].float().cpu().numpy() - ref).max() < (2e-2 if dtype == torch.bfloat16 else 1e-4)


@pytest.mark.parametrize("d,dtype", [(64, torch.float32), (64, torch.bfloat16), (104, torch.bfloat16), (256, torch.float32)])
@pytest.mark.parametrize("sizes", [[33, 32, 0, 65, 31, 200, 1, 40], [0, 0, 0, 0, 0, 0, 0, 700], [64, 64, 64, 64, 64, 64, 64, 64]])
def test_large_sets_without_a_sort(d, dtype, sizes):
    """1017 members, shared out evenly to a workgroup's lane groups whatever slots they belong to."""
    check_large_sets(d, dtype, sizes, 301, 1017, "workgroups")


@pytest.mark.parametrize("d,dtype", [(64, torch.float32), (64, torch.bfloat16), (104, torch.bfloat16), (256, torch.float32)])
@pytest.mark.parametrize("sizes", [[33, 32, 0, 65, 31, 40, 1, 50], [64, 64, 64, 64, 0, 0, 0, 0], [32, 33, 34, 31, 33, 32, 32, 29], [0, 0, 0, 0, 0, 0, 0, 200],
                                   [33, 0, 0, 0, 0, 0, 0, 223]])
def test_large_sets_of_the_shortest_lists(d, dtype, sizes):
    """Sets of more than 32 members are shared out to a wave's two to eight lane groups, one after the other."""
    check_large_sets(d, dtype, sizes, 301, 256, "waves")


def check_large_sets(d, dtype, sizes, B, Le, kernel):
    """Slots 0 to 7 and the last eight have the given sizes (those of one wave at 64 dims), the others share the rest.  fp32 sums
    of n terms below 6 in any order are within n 2^-23 6 of each other; a bf16 row is rounded once more, 2^-8 of its value."""
    assert merge_kernel(2, B, Le, d) == kernel
    L = B + Le
    g = torch.Generator().manual_seed(d)
    k, v = torch.randn(2, L, d, generator=g).to(dtype), torch.randn(2, L, d, generator=g).to(dtype)
    perm = torch.stack([torch.randperm(L, generator=g) for _ in range(2)])
    kept, ev = perm[:, :B].sort(1)[0].int(), perm[:, B:].sort(1)[0].int()
    assign = torch.randint(8, B - 8, (2, Le), generator=g).int()
    for h, base in ((0, 0), (1, B - 8)):
        at = torch.randperm(Le, generator=g)
        for slot, n in enumerate(sizes):
            assign[h, at[:n]], at = base + slot, at[n:]
    sim = torch.rand(2, Le, generator=g)
    args = (k, v, kept, ev, assign, sim)
    for mode in ("averaged", "pivotal", "weighted"):
        got = lookm.lookm_merge(*(x.cuda() for x in args), mode)
        for x, out in zip((k, v), got):
            for h in range(2):
                ref = torch.from_numpy(oracle.merge(x[h].float().numpy(), *(y[h].numpy() for y in (kept, ev, assign, sim)), mode))
                bound = max(sizes) * 2.0 ** -23 * 6 + (2.0 ** -8 * ref.abs() if dtype == torch.bfloat16 else 0.0)
                assert ((out[h].double().cpu() - ref).abs() <= bound + 1e-6).all()


@pytest.mark.parametrize("d,dtype", [(64, torch.float32), (128, torch.bfloat16), (256, torch.bfloat16)])
@pytest.mark.parametrize("B,Le", [(70, 255), (64, 256), (257, 257), (300, 1000), (33, 2049), (200, 3071), (70, 4095), (129, 4096), (129, 4097)])
def test_merge_that_scans_the_list_and_merge_of_a_sorted_one(d, dtype, B, Le):
    """Up to 4096 entries the merge's workgroups collect their slots' members from the list, for few enough workgroups; enough
    heads take the sort.  Both add the same members in the same order: equal bit for bit.  Even sets, all in one, uneven.  (Up to 256
    entries three heads have a kernel of their own, which adds in another order: the oracle's tolerance only.)"""
    L = B + Le
    many = min(H for H in range(3, 6000, 3) if merge_kernel(H, B, Le, d) == "sort")
    assert (merge_kernel(3, B, Le, d) == "waves") == (Le <= 256)
    g = torch.Generator().manual_seed(B + Le + d)
    k, v = torch.randn(3, L, d, generator=g).to(dtype).cuda(), torch.randn(3, L, d, generator=g).to(dtype).cuda()
    perm = torch.stack([torch.randperm(L, generator=g) for _ in range(3)])
    kept, ev = perm[:, :B].sort(1)[0].int().cuda(), perm[:, B:].sort(1)[0].int().cuda()
    u = torch.rand(3, Le, generator=g)
    assign = torch.stack([(u[0] * B).long(), torch.full((Le,), B - 1), (u[2] ** 4 * B).long()]).int().cuda()
    args = (k, v, kept, ev, assign, torch.rand(3, Le, generator=g).cuda())
    for mode in ("averaged", "pivotal", "weighted"):
        scanned = lookm.lookm_merge(*args, mode)
        for a, b in zip(scanned, lookm.lookm_merge(*(x.repeat((many // 3,) + (1,) * (x.dim() - 1)) for x in args), mode)):
            assert Le <= 256 or torch.equal(a, b[:3]) and torch.equal(a, b[-3:])
        for h in range(3):
            ref = oracle.merge(k[h].float().cpu().numpy(), *(x[h].cpu().numpy() for x in args[2:]), mode)
            assert np.abs(scanned[0][h].float().cpu().numpy() - ref).max() < (2e-2 if dtype == torch.bfloat16 else 1e-4)


@pytest.mark.parametrize("Le,kernel", [(256, "waves"), (1020, "workgroups")])
def test_one_large_set_does_not_set_the_time_of_a_merge(Le, kernel):
    """All members in one set against as many on 256 slots: 13.5 us against 5.2 and 20.4 against 6.8.  (256 members that the set's
    own lane group adds up by itself take 41.9 us.)"""
    H, B, d = 8, 256, 128
    assert merge_kernel(H, B, Le, d) == kernel
    L = B + Le
    g = torch.Generator().manual_seed(5)
    k, v = (torch.randn(H, L, d, generator=g).bfloat16().cuda() for _ in range(2))
    perm = torch.stack([torch.randperm(L, generator=g) for _ in range(H)])
    kept, ev = perm[:, :B].sort(1)[0].int().cuda(), perm[:, B:].sort(1)[0].int().cuda()
    sim = torch.rand(H, Le, generator=g).cuda()
    assigns = {"even": torch.randint(0, B, (H, Le), generator=g).int().cuda(), "one": torch.full((H, Le), 100, dtype=torch.int32).cuda()}
    graphs, times = {}, {}
    for name, assign in assigns.items():
        lookm.lookm_merge(k, v, kept, ev, assign, sim, "weighted")
        graphs[name] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graphs[name]):
            for _ in range(20):
                lookm.lookm_merge(k, v, kept, ev, assign, sim, "weighted")
    for _ in range(5):
        for name, graph in graphs.items():
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            graph.replay()
            begin.record()
            graph.replay()
            end.record()
            end.synchronize()
            times[name] = min(times.get(name, float("inf")), begin.elapsed_time(end))
    assert times["one"] < 5 * times["even"], times


@pytest.mark.parametrize("L", [1, 64, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049])
@pytest.mark.parametrize("what", ["spread", "equal", "crowded"])
def test_selection_at_the_edges_of_its_workgroup_sizes(L, what):
    """256, 512 and 1024 threads, digits of 10, 11 and 12 bits: distinct scores, all equal, and most of them within a few ulp of
    each other next to a far larger one (more digits).  Exact, ties to the lower position."""
    g = torch.Generator().manual_seed(L)
    s = torch.rand(2, L, generator=g) + 0.5
    if what == "equal":
        s.fill_(0.75)
    if what == "crowded":
        s = 1.0 + torch.randint(0, 40, (2, L), generator=g).float() * 2.0 ** -23
        s[:, 0] = 1e30
    mask = (torch.rand(L, generator=g) < 0.8).to(torch.uint8)
    M = min(5, L)
    protected = lookm.protected_count(mask, M)
    for B in {protected, L, protected + (L - protected) // 3, max(protected, L - 1)}:
        if B < 1:
            continue
        kept, ev = lookm.lookm_select(s.cuda(), mask.cuda(), B, M)
        for h in range(2):
            rank = torch.where((mask == 0) | (torch.arange(L) >= L - M), float("inf"), s[h].double())
            want = torch.sort(torch.sort(-rank, stable=True)[1][:B])[0]
            assert torch.equal(kept[h].cpu().long(), want)
            rest = torch.ones(L, dtype=torch.bool)
            rest[want] = False
            assert torch.equal(ev[h].cpu().long(), torch.nonzero(rest)[:, 0])


@pytest.mark.parametrize("H,L", [(1, 64), (3, 256), (2, 257), (8, 512), (8, 513), (32, 1024), (1, 1024), (8, 1025), (32, 2048), (8, 2048), (2, 2048), (1, 2048), (40, 2049), (32, 4096), (2, 4096), (32, 4097)])
@pytest.mark.parametrize("what", ["mixed", "images", "text first"])
def test_selection_that_sums_the_chunks(H, L, what):
    """Up to 4096 positions the selection adds up the score chunks of the competing tokens itself, one to sixteen of them (see the test
    below for which); with the scores asked for, and beyond, a kernel of its own does.  The same sums: kept tokens and cache are equal bit for bit, under an
    observation window and with a row log-sum-exp too."""
    g = torch.Generator().manual_seed(L + H)
    q, k, v = (torch.randn(H, L, 128, generator=g).bfloat16().cuda() for _ in range(3))
    mask = torch.ones(L, dtype=torch.uint8)
    if what == "mixed":
        mask = (torch.rand(L, generator=g) < 0.7).to(torch.uint8)
    if what == "text first":
        mask[:L // 2] = 0
    M = 16
    protected = lookm.protected_count(mask, M)
    B = protected + (L - protected) // 5
    lse = torch.randn(H, L, generator=g).cuda() + 5.0
    for extra in ({}, {"score_window": min(L, 64)}, {"row_lse": lse}):
        without = lookm.lookm_compress(q, k, v, mask.cuda(), B, M, "weighted", **extra)
        asked = lookm.lookm_compress(q, k, v, mask.cuda(), B, M, "weighted", want_scores=True, **extra)
        assert torch.equal(without.kept_idx, asked.kept_idx)
        assert torch.equal(without.k_out, asked.k_out) and torch.equal(without.v_out, asked.v_out)


def kernel_times(H, L, B, d, dtype, mode="weighted", row_lse=False, scores=False):
    """lookm_job_profile of a prompt whose image tokens are all but the first eight and the last sixteen."""
    g = torch.Generator(device="cuda").manual_seed(L)
    q, k, v = (torch.randn(H, L, d, generator=g, device="cuda").to(dtype) for _ in range(3))
    mask = torch.ones(L, dtype=torch.uint8, device="cuda")
    mask[:8] = 0
    out = lookm.alloc_outputs(H, L, d, B, dtype, "cuda", scores)
    ws = lookm.alloc_workspace(H, L, d, B, lookm.BF16 if dtype == torch.bfloat16 else lookm.F32, "cuda")
    lse = torch.randn(H, L, generator=g, device="cuda") + 5.0 if row_lse else None
    return lookm.lookm_job_profile(lookm.make_job(q, k, v, mask, B, 16, mode, out, ws, row_lse=lse), 3)


@pytest.mark.parametrize("skipped,args", [
    ({"score_colsum_fold", "bucket"}, dict(H=8, L=700, B=300, d=128, dtype=torch.bfloat16)),
    ({"score_colsum_fold", "bucket", "score_lse", "score_lse_fold"}, dict(H=8, L=700, B=300, d=128, dtype=torch.bfloat16, row_lse=True)),
    ({"score_colsum_fold", "bucket", "nearest", "nearest_fold"}, dict(H=8, L=700, B=300, d=128, dtype=torch.bfloat16, mode="none")),
    ({"bucket"}, dict(H=8, L=700, B=300, d=128, dtype=torch.bfloat16, scores=True)),
    (set(), dict(H=8, L=5000, B=800, d=128, dtype=torch.bfloat16)),
    ({"score_lse_fold", "score_colsum_fold", "nearest_fold", "bucket"}, dict(H=2, L=256, B=154, d=64, dtype=torch.float32)),
    ({"score_lse_fold", "score_colsum_fold", "nearest_fold"}, dict(H=2, L=5000, B=800, d=64, dtype=torch.bfloat16)),
])
def test_profile_reads_zero_for_what_is_not_launched(skipped, args):
    ms = kernel_times(**args)
    del ms["rnorm"]                     # the price of the events: an empty interval
    assert {name for name, t in ms.items() if t == 0.0} == skipped, ms


@pytest.mark.parametrize("H,L,summed", [(1, 1024, True), (1, 1025, False), (1, 2048, False), (2, 1088, False), (2, 2048, True), (8, 2048, True),
                                        (40, 2049, True), (8, 2896, False), (32, 4096, True), (32, 4097, False),
                                        (192, 2100, True), (193, 2100, False), (256, 2048, True)])
def test_which_prompts_have_their_chunks_summed_in_the_selection(H, L, summed):
    """Sixteen chunks at most (1 x 1024, 2 x 2048), past 2048 positions eight (32 x 4096; 8 x 2896 has twelve) of 192 heads at most; 1 x 1025
    has seventeen, 1 x 2048 thirty-two."""
    assert (kernel_times(H, L, L // 2, 128, torch.bfloat16)["score_colsum_fold"] == 0.0) == summed


@pytest.mark.parametrize("H,B,Le,d,dtype,sort", [
    (256, 512, 58, 128, torch.bfloat16, True), (32, 2448, 230, 256, torch.bfloat16, True),      # short lists, many workgroups
    (128, 448, 255, 128, torch.bfloat16, False), (128, 449, 255, 128, torch.bfloat16, True),    # 3584 and 3712 of them
    (128, 448, 300, 80, torch.bfloat16, False), (128, 449, 300, 80, torch.bfloat16, True),      # .. of rows that leave lanes idle
    (128, 640, 256, 128, torch.bfloat16, False), (128, 641, 256, 128, torch.bfloat16, True),    # 5120 and 5248
    (80, 1024, 300, 128, torch.float32, False), (80, 1025, 300, 128, torch.float32, True),
    (64, 1024, 2048, 64, torch.bfloat16, False), (64, 1024, 2049, 64, torch.bfloat16, True),    # 2^22 entries gone through, and more
    (2, 100, 4096, 64, torch.bfloat16, False), (2, 100, 4097, 64, torch.bfloat16, True)])
def test_which_lists_are_sorted(H, B, Le, d, dtype, sort):
    """Where the merge's workgroups go through the list themselves no sort is launched."""
    assert (kernel_times(H, B + Le, B, d, dtype)["bucket"] > 0.0) == sort == (merge_kernel(H, B, Le, d) == "sort")
