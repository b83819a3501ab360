"""Diversity set by pools (Sec. 4.1) on the GPU where the pool's rounds end
early: every pick against float64 distances to the GPU's own selected set."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_37581_amd import trevs
from parity import assert_scores_close, check_fps_picks

pytestmark = pytest.mark.gpu


def clustered(rng, N, d, clusters, dup, zeros):
    """Rows of N tokens: `clusters` tight clusters (size, spread), `dup` copies of
    one row, `zeros` zero rows, the rest independent; and which are independent."""
    Z = rng.standard_normal((N, d))
    order = rng.permutation(N)
    at = 0
    for size, spread in clusters:
        Z[order[at:at + size]] = rng.standard_normal(d) + spread * rng.standard_normal((size, d))
        at += size
    Z[order[at:at + dup]] = rng.standard_normal(d)
    at += dup
    Z[order[at:at + zeros]] = 0.0
    at += zeros
    return Z, np.sort(order[at:])


# (N, d, K, K_d, dtype, per sample: clusters, copies, zero rows).  Pools hold at
# most 4096 tokens, so a cluster of 5000 far tokens fills one and ends its round
# after the first pick; three of them leave picks for the full Gram matrix.
CASES = {
    "second-round-bf16": (8192, 256, 768, 192, "bf16", [([(5000, 0.05)], 0, 0), ([], 0, 0)]),
    "unfinished-bf16": (20000, 64, 1024, 256, "bf16", [([(5000, 0.02)] * 3, 0, 0), ([(300, 0.02)] * 9, 0, 0)]),
    "unfinished-odd-f32": (16387, 20, 600, 150, "f32", [([(4500, 0.02)] * 3, 0, 0)]),
    "copies-and-zeros-bf16": (6000, 128, 640, 160, "bf16", [([], 2500, 0), ([], 300, 900)]),
    "pool-of-all-bf16": (2304, 1024, 1152, 288, "bf16", [([(500, 0.1)], 100, 3)] * 2),
    # one tight cluster: most pairs are marked, and rows of G are no multiple of four
    "pool-of-one-cluster-bf16": (2305, 1024, 800, 200, "bf16", [([(1700, 0.05)], 0, 0), ([(850, 0.05)] * 2, 0, 0)]),
    "pool-tail-f32": (3000, 1028, 700, 175, "f32", [([(200, 0.1)] * 4, 50, 1)]),
}


@pytest.mark.parametrize("name", CASES)
def test_picks_of_clustered_tokens(name):
    N, d, K, k_div, dtype, samples = CASES[name]
    rng = np.random.default_rng(sum(map(ord, name)))
    B, H, M = len(samples), 4, 8
    print(f"[picks] {name}: B={B} N={N} d={d} K={K} K_d={k_div}", flush=True)
    Z = np.empty((B, N, d), dtype=np.float32)
    cls = rng.standard_normal((B, H, N)).astype(np.float32)
    for b, (clusters, dup, zeros) in enumerate(samples):
        Z[b], free = clustered(rng, N, d, clusters, dup, zeros)
        cls[b][:, rng.choice(free, K - k_div, replace=False)] += 8.0  # the pivots: no cluster holds one
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Zt = torch.from_numpy(Z).to(dt)
    T = torch.from_numpy(rng.standard_normal((B, M, d)).astype(np.float32)).to(dt).cuda()
    call = trevs.Prellm(torch.from_numpy(cls).to(dt).cuda(), Zt.cuda(), T, k_keep=K, k_div=k_div,
                        textual_ratio=0.0, want_scores=True)
    call()
    torch.cuda.synchronize()
    kept, picks = call.kept_idx.cpu().numpy(), call.div_idx.cpu().numpy()
    score = call.score.cpu().numpy()
    assert torch.equal(call.kept_feats.cpu(), torch.stack([Zt[b][torch.from_numpy(kept[b]).long()] for b in range(B)]))
    for b in range(B):
        pivots = np.setdiff1d(kept[b], picks[b])
        assert pivots.size == K - k_div and np.unique(picks[b]).size == k_div, b
        assert np.array_equal(pivots, oracle.topk_ascending(score[b].astype(np.float64), K - k_div)), b
        assert np.array_equal(kept[b], np.sort(np.concatenate([pivots, picks[b]]))), b
        check_fps_picks(Zt[b].double().numpy(), pivots, picks[b])
    again = call.div_idx.clone()
    call()
    assert torch.equal(again, call.div_idx)


@pytest.mark.parametrize("N,d,K,k_div,dtype,huge", [
    (2304, 1024, 2304, 288, "bf16", 3),     # a pool of all tokens, every token kept
    (2304, 1024, 1152, 288, "bf16", 1200),  # a pool of all tokens, fewer distances than picks
    (3000, 1028, 3000, 175, "f32", 1),
    (300, 64, 300, 40, "bf16", 33),         # the full Gram matrix at once
    (9000, 64, 400, 256, "bf16", 8700),     # rounds that find too little, then the full Gram matrix
])
def test_tokens_without_a_distance(N, d, K, k_div, dtype, huge):
    """Finite rows whose products overflow have no distance (infinity times 1/infinity).
    The tokens that have one are picked first; then the others fill the set in
    index order, and the kept list is complete."""
    print(f"[picks-overflow] N={N} d={d} K={K} K_d={k_div} {dtype} huge={huge}", flush=True)
    rng = np.random.default_rng(N + huge)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Z = rng.standard_normal((2, N, d)).astype(np.float32)
    cls = rng.standard_normal((2, 4, N)).astype(np.float32)
    rows = np.sort(rng.permutation(N)[:huge])
    usable = np.setdiff1d(np.arange(N), rows)
    Z[0, rows] = 3e38 * np.where(rng.random((huge, d)) < 0.5, -1.0, 1.0)  # sample 1 has none
    for b in range(2):
        cls[b][:, rng.choice(usable, min(K - k_div, usable.size), replace=False)] += 8.0
    Zt = torch.from_numpy(Z).to(dt)
    T = torch.from_numpy(rng.standard_normal((2, 8, d)).astype(np.float32)).to(dt).cuda()
    call = trevs.Prellm(torch.from_numpy(cls).to(dt).cuda(), Zt.cuda(), T, k_keep=K, k_div=k_div,
                        textual_ratio=0.0, ratio_mode="budget", want_scores=True)
    call()
    torch.cuda.synchronize()
    kept, picks, sal = call.kept_idx.cpu().numpy(), call.div_idx.cpu().numpy(), call.sal.cpu().numpy()
    for b in range(2):
        pivots = oracle.topk_ascending(sal[b].astype(np.float64), K - k_div)
        assert np.array_equal(kept[b], np.unique(np.concatenate([pivots, picks[b]]))), b
        assert kept[b].size == K and kept[b][0] >= 0 and kept[b][-1] < N, b
        have = usable if b == 0 else np.arange(N)
        with_distance = np.setdiff1d(have, pivots)
        n = min(k_div, with_distance.size)
        assert np.isin(picks[b][:n], with_distance).all(), b
        check_fps_picks(Zt[b][torch.from_numpy(have)].double().numpy(), np.searchsorted(have, np.intersect1d(pivots, have)),
                        np.searchsorted(have, picks[b][:n]))
        left = np.setdiff1d(np.arange(N), np.concatenate([pivots, picks[b][:n]]))
        assert np.array_equal(picks[b][n:], left[:k_div - n]), b


@pytest.mark.parametrize("d", [4096, 16384])
def test_picks_do_not_depend_on_nearer_tokens(d):
    """fp32 rows of equal magnitudes, whose sums of squares collect rounding errors
    of one sign: the relevance pass's norms and those of the Gram matrix differ
    most here (about 1.5e-5 and 6e-5 of the norm).  Thousands of tokens nearer to the
    pivot than the picks must not change the picks, whatever their norms decide
    about the pool.  Distances are 0.1 and a few 1e-5 steps, set by one extra
    coordinate; magnitudes of a power of two have exact norms (the pivot, the
    nearer tokens and some others)."""
    rng = np.random.default_rng(d)
    m = d - 4
    sign = rng.choice([-1.0, 1.0], m)
    flips = m // 20

    def row(c, y):  # at distance 0.1 + y
        s = sign.copy()
        s[rng.permutation(m)[:flips]] *= -1.0
        x = 1.0 - 2.0 * flips / m
        z = np.zeros(d, dtype=np.float32)
        z[:m] = np.float32(c) * s
        z[m] = np.float32(c) * np.sqrt(m * ((x / (x - y)) ** 2 - 1.0))
        return z

    near, unit = 1e-4, 2.0 ** -7
    few = [row(unit, near) for _ in range(3)]
    picked = [row(unit, near + 3e-5 + 1e-7 * i) for i in range(8)]
    for c in unit * rng.uniform(1.0, 2.0, 16):
        picked += [row(c, near + y) for y in np.arange(-8e-5, 8e-5, 8e-6)]
    pivot = np.zeros(d, dtype=np.float32)
    pivot[:m] = unit * sign
    small = np.stack([pivot] + picked + few)
    rest = np.stack([row(unit, near) for _ in range(512)])[np.arange(5000) % 512]
    order = []
    for Z, k_div in ((small, len(picked) + 2), (np.concatenate([small, rest]), 256)):
        N = Z.shape[0]
        print(f"[picks-norms] d={d} N={N} K_d={k_div}", flush=True)
        cls = torch.zeros((1, 1, N))
        cls[0, 0, 0] = 8.0
        call = trevs.Prellm(cls.cuda(), torch.from_numpy(Z)[None].cuda(), torch.ones((1, 1, d)).cuda(),
                            k_keep=k_div + 1, k_div=k_div, textual_ratio=0.0, ratio_mode="budget")
        call()
        order.append(call.div_idx.cpu().numpy()[0])
    n = int(np.argmax(order[0] > len(picked)))  # up to the first of the nearer tokens
    assert 8 < n < 250, n
    assert np.array_equal(order[0][:n], order[1][:n]), (order[0][:n], order[1][:n])


@pytest.mark.parametrize("N,d,clusters,spread,zeros", [
    (8192, 256, 40, 0.3, 0), (9001, 1032, 8, 0.0, 0), (8192, 1024, 20, 0.0, 0),
    (8192, 256, 30, 0.1, 5000), (20001, 64, 9, 0.0, 9000),  # zero rows: distance 1, more than a pool holds
])
def test_picks_of_rounds_and_of_the_full_matrix(N, d, clusters, spread, zeros):
    """Few picks are made in rounds, more than 2048 over the Gram matrix of all
    tokens; the former are the beginning of the latter, bit for bit in bf16, near
    ties included (clusters leave much of them to the second round; those of
    copies of one row leave distances of a rounding error)."""
    k_piv, size = 576, (N - 606 - zeros) // clusters
    rng = np.random.default_rng(N + clusters)
    Z = np.empty((2, N, d), dtype=np.float32)
    cls = torch.zeros((2, 1, N))
    for b in range(2):
        Z[b], free = clustered(rng, N, d, [(size, spread)] * clusters, 0, zeros)
        cls[b, 0, torch.from_numpy(free[:k_piv])] = 8.0
    Zt = torch.from_numpy(Z).bfloat16().cuda()
    picks = []
    for k_div in (192, 2100):
        print(f"[picks-prefix] N={N} d={d} clusters={clusters} spread={spread} zeros={zeros} K_d={k_div}", flush=True)
        call = trevs.Prellm(cls.bfloat16().cuda(), Zt, torch.ones((2, 1, d), dtype=torch.bfloat16, device="cuda"),
                            k_keep=k_piv + k_div, k_div=k_div, textual_ratio=0.0, ratio_mode="budget")
        call()
        picks.append(call.div_idx.cpu().numpy())
    assert np.array_equal(picks[0], picks[1][:, :192])


@pytest.mark.parametrize("cosine", [1e-5, 1e-4])
def test_picks_among_distances_an_ulp_apart(cosine):
    """Mutually orthogonal rows with one small cosine to the pivots: thousands of
    distances within an ulp or two of each other, which the norms' rounding can
    order either way.  The picks of a pool are those over all tokens, bit for bit."""
    m, N, k_piv = 2048, 8192, 400
    H = np.ones((1, 1))
    while H.shape[0] < m:
        H = np.block([[H, H], [H, -H]])
    rng = np.random.default_rng(m)
    Z = np.zeros((1, N, m + 8), dtype=np.float32)
    c = rng.uniform(1.0, 2.0, N)
    Z[0, :, :m] = H[rng.integers(0, 2000, N)] * c[:, None]
    Z[0, :, m] = cosine * np.sqrt(m) * c
    piv = rng.permutation(N)[:k_piv]
    Z[0, piv] = 0.0
    Z[0, piv, m] = rng.uniform(1.0, 2.0, k_piv)
    cls = torch.zeros((1, 1, N))
    cls[0, 0, torch.from_numpy(piv)] = 8.0
    picks = []
    for k_div in (192, 2100):
        print(f"[picks-ulp] N={N} d={m + 8} cosine={cosine} K_d={k_div}", flush=True)
        call = trevs.Prellm(cls.bfloat16().cuda(), torch.from_numpy(Z).bfloat16().cuda(),
                            torch.ones((1, 1, m + 8), dtype=torch.bfloat16, device="cuda"), k_keep=k_piv + k_div,
                            k_div=k_div, textual_ratio=0.0, ratio_mode="budget")
        call()
        picks.append(call.div_idx.cpu().numpy())
    assert np.array_equal(picks[0], picks[1][:, :192])


@pytest.mark.parametrize("B,N,d,K,k_div,dtype,spread", [
    (2, 5003, 264, 901, 225, "bf16", 0.02),  # 256-row tiles, rows of G not a multiple of four
    (8, 1999, 264, 400, 100, "bf16", 0.02),  # 128-row tiles
    (4, 3001, 260, 600, 150, "f32", 0.05),
    (2, 5003, 264, 901, 225, "bf16", 1.0),   # the rounds suffice
])
def test_picks_of_slowly_changing_features(B, N, d, K, k_div, dtype, spread):
    """Features that change slowly over the image, the pivots at its beginning: a pool
    holds runs of near tokens and gives few picks, and most are made over the Gram
    matrix of the tokens that are no pivots.  In bf16 they are, bit for bit, the
    beginning of those over the matrix of all tokens (more than 2048 picks)."""
    rng = np.random.default_rng(N + d)
    x = np.arange(N) / 64.0
    i, f = x.astype(int), (x % 1.0)[None, :, None]
    knots = rng.standard_normal((B, N // 64 + 2, d))
    Z = knots[:, i] * (1 - f) + knots[:, i + 1] * f + spread * rng.standard_normal((B, N, d))
    Z = np.ascontiguousarray(Z, dtype=np.float32)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    Zt = torch.from_numpy(Z).to(dt)
    cls = torch.zeros((B, 1, N))
    cls[:, :, :K - k_div] = 8.0
    picks = []
    for n in (k_div, 2100)[:2 if N > 4500 else 1]:
        print(f"[picks-smooth] B={B} N={N} d={d} K_r={K - k_div} K_d={n} {dtype} spread={spread}", flush=True)
        call = trevs.Prellm(cls.to(dt).cuda(), Zt.cuda(), torch.ones((B, 1, d), dtype=dt, device="cuda"),
                            k_keep=K - k_div + n, k_div=n, textual_ratio=0.0, ratio_mode="budget")
        call()
        picks.append(call.div_idx.cpu().numpy())
    if dtype == "bf16" and len(picks) == 2:
        assert np.array_equal(picks[0], picks[1][:, :k_div])
    for b in range(B):
        assert np.unique(picks[0][b]).size == k_div, b
        check_fps_picks(Zt[b].double().numpy(), np.arange(K - k_div), picks[0][b])


@pytest.mark.parametrize("d,dtype", [(1032, "bf16"), (1024, "bf16"), (1028, "f32")])
def test_relevance_text_lengths_at_block_edges(d, dtype):
    """Question lengths around the 32-row text blocks (the blocks past the last
    row are skipped), one and two text chunks, whole and partial last slabs."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    for M in (32, 64, 128, 160):
        rng = np.random.default_rng(M + d)
        Zt = torch.from_numpy(rng.standard_normal((6, 200, d)).astype(np.float32)).to(dt)
        T = torch.from_numpy(rng.standard_normal((6, M, d)).astype(np.float32)).to(dt)
        cls = torch.from_numpy(rng.standard_normal((6, 4, 200)).astype(np.float32)).to(dt)
        lens = np.array([1, M // 2 - 1, M // 2, M // 2 + 1, M - 1, M], dtype=np.int32)
        call = trevs.Prellm(cls.cuda(), Zt.cuda(), T.cuda(), torch.from_numpy(lens).cuda(), k_keep=20,
                            want_scores=True)
        call()
        z = torch.nn.functional.normalize(Zt.double(), dim=2)
        t = torch.nn.functional.normalize(T.double(), dim=2)
        c = (z @ t.transpose(1, 2)).clamp_min(0.0).square()
        want = torch.stack([c[b, :, :int(lens[b])].mean(1).sqrt() for b in range(6)])
        assert_scores_close(call.rel.cpu().numpy(), want.numpy(), f"s^t M={M}")
