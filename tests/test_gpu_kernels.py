"""Kernels against plain float64 references at the sizes where their tilings can go wrong: edges of tiles and stages,
remainders, the smallest and largest of each branch's range."""
import threading

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _pkg():
    import paper_2403_12983_amd as pkg
    return pkg


def _gram_err(H, X, lam):
    """largest entrywise error of H over sqrt(H_ii H_jj)"""
    Hr = X.T @ X + lam * np.eye(X.shape[1])
    d = np.sqrt(np.diag(Hr))
    return np.max(np.abs(H - Hr) / np.outer(d, d))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,d1,m,pad", [(1, 1, 1, 0), (31, 63, 5, 1), (32, 64, 64, 0), (33, 65, 63, 3), (65, 129, 1, 2),
                                        (4097, 64, 65, 0), (5000, 191, 130, 1), (96, 1024, 1024, 0), (2050, 1000, 33, 7)])
def test_small_tile_float64_products(dtype, n, d1, m, pad):
    """The 64 x 64 float64 products with contraction-major operands (X^T X from rows at any alignment, H W), with and without
    the contraction cut into ranges.  Sums are float64, so H and G are float32 roundings of the exact values: 2^-24 = 6e-8,
    relative to sqrt(H_ii H_jj) (to the entries' own sizes for G, through H's rounding: 2e-7 of |H| |W|)."""
    g = torch.Generator().manual_seed(n * 7 + d1)
    X = torch.randn(n, d1 + pad, generator=g).to(dtype)[:, :d1]
    W = torch.randn(d1, m, generator=g).to(dtype)
    Xg = torch.empty(n, d1 + pad, dtype=dtype, device=DEV)[:, :d1]
    Xg.copy_(X)
    H = torch.empty(d1, d1, device=DEV)
    G = torch.empty(d1, m, device=DEV)
    sc = torch.empty(2, dtype=torch.float64, device=DEV)
    _pkg().osscar_gram_static(Xg, W.to(DEV), H, G, sc, 1e-3, 1e-2)
    torch.cuda.synchronize()
    Xd, Wd = X.double().numpy(), W.double().numpy()
    lam = 1e-3 + 1e-2 * np.sum(Xd * Xd) / d1
    assert abs(sc[0].item() - lam) <= 1e-12 * lam
    Hn = H.cpu().double().numpy()
    assert _gram_err(Hn, Xd, lam) <= 6.1e-8 and np.array_equal(Hn, Hn.T)
    Gr = Hn @ Wd                                     # the product of the H that was written
    assert np.max(np.abs(G.cpu().double().numpy() - Gr) / np.maximum(np.abs(Gr), 1e-12 * np.max(np.abs(Gr)))) <= 6.1e-8
    assert abs(sc[1].item() - np.sum(Wd * Gr)) <= 1e-7 * np.sum(np.abs(Wd * Gr))


@pytest.mark.parametrize("d1,m", [(64, 64), (288, 64), (191, 130), (1024, 1024)])
def test_static_gram_with_the_weights_where_g_goes(d1, m):
    """G may take the place of W: the same result as with a buffer of its own, up to the float64 sums' order (other ranges of the contraction:
    G the same to float32's rounding, 6e-8 of an entry, c0 through it)."""
    g = torch.Generator(device=DEV).manual_seed(d1)
    X = torch.randn(512, d1, generator=g, device=DEV)
    for dtype in (torch.float32, torch.bfloat16):
        out = []
        for in_place in (False, True):
            g.manual_seed(m)
            G = torch.empty(d1, m, device=DEV)
            W = G.view(-1).view(dtype)[:d1 * m].view(d1, m) if in_place else torch.empty(d1, m, dtype=dtype, device=DEV)
            W.copy_(torch.randn(d1, m, generator=g, device=DEV))
            H, sc = torch.empty(d1, d1, device=DEV), torch.empty(2, dtype=torch.float64, device=DEV)
            _pkg().osscar_gram_static(X, W, H, G, sc, 1e-3, 1e-2)
            torch.cuda.synchronize()
            out.append((H, G, sc))
        (H0, G0, s0), (H1, G1, s1) = out
        assert torch.equal(H0, H1) and torch.allclose(G1, G0, rtol=1.2e-7, atol=1e-9 * G0.abs().max().item())
        assert s1[0] == s0[0] and abs(s1[1] - s0[1]) <= 1e-7 * abs(s0[1])


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_patch_rows_in_several_pieces(dtype):
    """float32 maps (and bf16 maps whose patch width is no multiple of eight) write their patches out as rows, as many as the
    staging buffer holds: 9408 patches of 126 columns take two pieces."""
    g = torch.Generator().manual_seed(3)
    B, C, S, m = 3, 14, 56, 8
    F = torch.randn(B, C, S, S, generator=g).to(dtype)
    W = torch.randn(C * 9, m, generator=g).to(dtype)
    s = _pkg().Solver(C * 9, m, C, 9, C // 2, 1, dtype, dtype, DEV)
    s.osscar_gram_conv(F.to(DEV), 3, 3, 1, 1, True, W.to(DEV), 0.5, 0.0)
    H = s.osscar_get_tensor(0).cpu().double().numpy()
    s.close()
    X = torch.nn.functional.unfold(F.double(), 3, padding=1).permute(0, 2, 1).reshape(-1, C * 9).numpy()
    assert X.shape[0] == 9408 and _gram_err(H, X, 0.5) <= 6.1e-8


@pytest.mark.parametrize("side", [True, False])
@pytest.mark.parametrize("kr", [1, 15, 16, 17, 113, 127, 128, 129, 255, 257, 385, 600])
def test_sweep_inverse_at_the_edges_of_its_blocks(kr, side):
    """P = H_KK^-1 where the last pivot block and its last 16 x 16 tile are full, ragged or one row, on one stream and on two.
    The sweep is float64 (condition number below 20: 1e-14), so P is the float32 rounding of the inverse: 2^-24."""
    from paper_2403_12983_amd import binding
    pkg = _pkg()
    d1 = kr + 5
    g = torch.Generator().manual_seed(kr)
    A = torch.randn(2 * d1, d1, generator=g, dtype=torch.float64)
    H = (A.T @ A / (2 * d1) + 0.2 * torch.eye(d1, dtype=torch.float64)).float()
    H = torch.tril(H) + torch.tril(H, -1).T
    s = pkg.Solver(d1, 3, d1, 1, kr, 1, torch.float32, torch.float32, DEV)
    binding.side_stream(side)
    try:
        s.osscar_set_quadratic(H.to(DEV), torch.randn(d1, 3, generator=g).to(DEV), 1.0, np.ones(d1))
        groups = sorted(np.random.default_rng(kr).choice(d1, kr, replace=False).tolist())
        s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, groups)
        P = s.osscar_get_tensor(2).cpu().double().numpy()
    finally:
        binding.side_stream(True)
        s.close()
    R = np.linalg.inv(H.double().numpy()[np.ix_(groups, groups)])
    d = np.sqrt(np.diag(R))
    assert np.array_equal(P, P.T) and np.max(np.abs(P - R) / np.outer(d, d)) <= 6.1e-8


@pytest.mark.parametrize("d1,m,chunks", [
    (8, 8, [1, 600]), (136, 72, [5000, 63, 2048]),      # ranges of the contraction into copies, fewer of them later, ragged stages
    (2048, 8, [2048, 500]), (1000, 1000, [1537]),
    (3528, 2056, [8200]),                                # wide tiles, ragged in both directions and in the last stage
    (3592, 2056, [700, 8129, 16384 + 64]),               # both kernels on one layer, a second repacked piece
])
def test_packed_gram_in_ranges_and_in_wide_tiles(d1, m, chunks):
    """H = X^T X and G = X^T Y from bf16 rows, chunk by chunk.  Products are exact; the matrix core adds 16 rows at a time in
    float32 and may cut off up to one unit in the last place, 2^-23 of the partial sum, each time; sums restart every 1024 rows
    at most and go on in rounded float32 and, from range to range, in float64.  64 such steps on a sum that grows evenly: at most
    64 / 2 * 2^-23 = 3.8e-6 of sqrt(H_ii H_jj); measured 3e-7, on the diagonal, and held to three times that."""
    n = sum(chunks)
    g = torch.Generator(device=DEV).manual_seed(d1 + n)
    X = torch.randn(n, d1, generator=g, device=DEV).to(torch.bfloat16)
    Y = torch.randn(n, m, generator=g, device=DEV).to(torch.bfloat16)
    W = torch.zeros(d1, m, dtype=torch.bfloat16, device=DEV)
    s = _pkg().Solver(d1, m, d1, 1, max(1, d1 // 2), 1, torch.bfloat16, torch.bfloat16, DEV, target_output=True)
    r0 = 0
    for c in chunks:
        last = r0 + c == n
        s.osscar_gram_target(X[r0:r0 + c], Y[r0:r0 + c], *((True, W, 0.0, 1e-2) if last else (False,)))
        r0 += c
    H, G = s.osscar_get_tensor(0).cpu().double().numpy(), s.osscar_get_tensor(1).cpu().double().numpy()
    lam = s.osscar_get_scalars()[0]
    s.close()
    Hr, Gr = np.zeros((d1, d1)), np.zeros((d1, m))
    for r0 in range(0, n, 4096):
        Xd, Yd = X[r0:r0 + 4096].double(), Y[r0:r0 + 4096].double()
        Hr += (Xd.T @ Xd).cpu().numpy()
        Gr += (Xd.T @ Yd).cpu().numpy()
    Hr += lam * np.eye(d1)
    dx, dy = np.sqrt(np.diag(Hr)), np.sqrt((Y.double() ** 2).sum(0).cpu().numpy())
    assert np.array_equal(H, H.T) and np.max(np.abs(H - Hr) / np.outer(dx, dx)) <= 1e-6
    assert np.max(np.abs(G - Gr) / np.outer(dx, dy)) <= 1e-6


@pytest.mark.parametrize("q,p,m", [(2, 40, 3), (9, 15, 64), (15, 6, 130), (16, 7, 128), (17, 5, 33), (33, 5, 257), (48, 4, 1), (63, 4, 40),
                                   (64, 6, 300)])
def test_swaps_of_groups_of_every_tile_count(q, p, m):
    """Groups of 1 - 4 tiles of 16 rows, full and ragged, after three swaps (the middle one towards a higher index, the others
    towards a lower one) and, from the dense layer, after single removals: the state and every score against float64 inverses
    of the kept set.  The state is float32 and every swap rounds it again: a few times 2^-24 = 6e-8 times the condition number
    (below 20) per swap, 1e-5 in all; scores are squares of it."""
    pkg = _pkg()
    d1, k = p * q, p // 2 + 1
    g = torch.Generator().manual_seed(q * 100 + p)
    A = torch.randn(2 * d1, d1, generator=g, dtype=torch.float64)
    H = (A.T @ A / (2 * d1) + 0.2 * torch.eye(d1, dtype=torch.float64)).float()
    H = torch.tril(H) + torch.tril(H, -1).T
    W = torch.randn(d1, m, generator=g, dtype=torch.float64)
    G = (H.double() @ W).float()
    Hd, Gd = H.double().numpy(), G.double().numpy()

    def check(s, kept):
        rows = lambda gs: np.concatenate([np.arange(x * q, x * q + q) for x in sorted(gs)])
        out = [x for x in range(p) if x not in kept]
        K, C = rows(kept), rows(out)
        P = np.linalg.inv(Hd[np.ix_(K, K)])
        B = P @ Gd[K]
        V = P @ Hd[np.ix_(K, C)]
        R = Gd[C] - V.T @ Gd[K]
        S = Hd[np.ix_(C, C)] - Hd[np.ix_(C, K)] @ V
        T = lambda i: s.osscar_get_tensor(i).cpu().double().numpy()
        assert T(8).astype(int).tolist() == sorted(kept)
        for got, ref in ((T(2), P), (T(3), B), (T(4), V), (T(5), R)):
            assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)
        rem, add = T(6), T(7)
        for n, x in enumerate(sorted(kept)):
            b, pb = B[n * q:n * q + q], P[n * q:n * q + q, n * q:n * q + q]
            assert abs(rem[x] - np.sum(b * np.linalg.solve(pb, b))) <= 2e-5 * rem[x]
        for n, x in enumerate(out):
            r, sb = R[n * q:n * q + q], S[n * q:n * q + q, n * q:n * q + q]
            assert abs(add[x] - np.sum(r * np.linalg.solve(sb, r))) <= 2e-5 * add[x]

    kept = set(range(0, 2 * k, 2)) if 2 * k <= p else set(range(k))
    s = pkg.Solver(d1, m, p, q, k, 4, torch.float32, torch.float32, DEV)
    s.osscar_set_quadratic(H.to(DEV), G.to(DEV), float(np.sum(W.numpy() * Gd)), np.ones(p))
    s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, sorted(kept))
    check(s, kept)
    for go, gi in ((max(kept), min(set(range(p)) - kept)), (None, None), (None, None)):
        if go is None:
            go, gi = min(kept), max(set(range(p)) - kept)
        s.osscar_apply_swap(go, gi)
        kept = kept - {go} | {gi}
        check(s, kept)
    s.close()
    s = pkg.Solver(d1, m, p, q, k, 4, torch.float32, torch.float32, DEV, from_dense=True)
    s.osscar_set_quadratic(H.to(DEV), G.to(DEV), float(np.sum(W.numpy() * Gd)), np.ones(p))
    s.osscar_init_greedy(2)
    check(s, set(s.osscar_get_tensor(8).cpu().tolist()))
    s.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,d1,m,pad", [(1024, 2817, 129, 1), (9001, 2945, 5, 0), (1500, 2943, 2050, 3)])
def test_gram_in_digits(dtype, n, d1, m, pad):
    """X^T X and X^T Y of rows that the packed kernels do not take, on the int8 matrix cores (in two pieces for 9001 rows), with
    columns of very different sizes, rare large values (their panels of 128 columns: float64 sums) and an empty column.  What the
    digits drop is 1e-9 of sqrt(H_ii H_jj), so H and G are float32 roundings of the exact sums: 2^-24 + 1e-9."""
    g = torch.Generator(device=DEV).manual_seed(n)
    scale = torch.exp2(torch.randint(-20, 20, (d1,), generator=g, device=DEV).float())
    X = torch.randn(n, d1 + pad, generator=g, device=DEV)
    X[torch.randint(0, n, (50,), generator=g, device=DEV), torch.randint(0, d1, (50,), generator=g, device=DEV)] *= 100
    X[:, :d1] *= scale
    X[:, 7] = 0
    X = X.to(dtype)[:, :d1]
    Y = torch.randn(n, m, generator=g, device=DEV).to(dtype)
    W = torch.zeros(d1, m, dtype=dtype, device=DEV)
    s = _pkg().Solver(d1, m, d1, 1, d1 // 2, 1, dtype, dtype, DEV, target_output=True)
    s.osscar_gram_target(X, Y, True, W, 0.0, 0.0)
    H, G = s.osscar_get_tensor(0), s.osscar_get_tensor(1)
    Xd, Yd = X.double(), Y.double()
    Hr, Gr = Xd.T @ Xd, Xd.T @ Yd
    dx, dy = Hr.diagonal().sqrt().clamp_min(1e-300), Yd.square().sum(0).sqrt()
    assert torch.equal(H, H.T) and ((H.double() - Hr).abs() / dx[:, None] / dx).max().item() <= 6.1e-8
    assert ((G.double() - Gr).abs() / dx[:, None] / dy).max().item() <= 6.1e-8
    # an infinity or a NaN spoils its own row and column and, through the trace in the ridge, the diagonal
    Xb = X.clone()
    Xb[3, 11], Xb[n - 1, d1 - 1] = float("nan"), float("inf")
    s.osscar_gram_target(Xb, Y, True, W, 1.0, 0.0)
    H2 = s.osscar_get_tensor(0)
    s.close()
    bad = torch.zeros(d1, dtype=torch.bool, device=DEV)
    bad[11] = bad[d1 - 1] = True
    expect = bad[:, None] | bad[None, :] | torch.eye(d1, dtype=torch.bool, device=DEV)
    assert torch.equal(~torch.isfinite(H2), expect)


@pytest.mark.parametrize("p,k,t_hat,equal", [(5, 2, 3, 0), (40, 3, 37, 0), (1000, 900, 7, 0), (1030, 1000, 10, 300), (3000, 2936, 64, 0),
                                             (8193, 8140, 10, 0), (8193, 8100, 20, 8193)])
def test_simultaneous_picks(p, k, t_hat, equal):
    """The cheapest groups of the dense layer, by rank and (many equal costs: more than the list holds) one by one, on both
    sides of the two register sizes.  H = 1 and G = diag: the cost of removing row i is G_i^2, whatever has been removed before, so the
    picks are a stable sort (lowest index on ties)."""
    pkg = _pkg()
    rng = np.random.default_rng(p + k)
    cost = rng.permutation(p).astype(np.float64) + 1
    cost[rng.permutation(p)[:equal]] = 0.5 if equal < p else 7.0
    s = pkg.Solver(p, 1, p, 1, k, 1, torch.float32, torch.float32, DEV, from_dense=True)
    H = torch.eye(p, device=DEV)
    G = torch.from_numpy(np.sqrt(cost)).float().to(DEV).reshape(p, 1)
    s.osscar_set_quadratic(H, G, float(cost.sum()), np.ones(p))
    s.osscar_init_greedy(t_hat)
    kept = set(s.osscar_get_tensor(8).cpu().tolist())
    s.close()
    g2 = G.double().cpu().numpy().ravel() ** 2
    order = np.lexsort((np.arange(p), np.round(g2, 3)))
    assert kept == set(order[p - k:].tolist())


@pytest.mark.parametrize("dtype,B,C,S", [(torch.float32, 3, 320, 36), (torch.bfloat16, 2, 321, 24)])
def test_patch_rows_in_digits(dtype, B, C, S):
    """Wide patch matrices (2880 and 2889 columns) of maps that the packed kernels do not take: the patches are written out as rows
    and cut into digits behind them, 3888 patches in two pieces.  H is the float32 rounding of the exact sums: 2^-24 + 1e-9."""
    g = torch.Generator(device=DEV).manual_seed(C)
    F = torch.randn(B, C, S, S, generator=g, device=DEV).clamp_min(0).to(dtype)
    W = torch.randn(C * 9, 4, generator=g, device=DEV).to(dtype)
    s = _pkg().Solver(C * 9, 4, C, 9, C // 2, 1, dtype, dtype, DEV)
    s.osscar_gram_conv(F, 3, 3, 1, 1, True, W, 0.5, 0.0)
    H = s.osscar_get_tensor(0).double()
    s.close()
    X = torch.nn.functional.unfold(F.double(), 3, padding=1).permute(0, 2, 1).reshape(-1, C * 9).contiguous()
    Hr = X.T @ X + 0.5 * torch.eye(C * 9, dtype=torch.float64, device=DEV)
    d = Hr.diagonal().sqrt()
    assert torch.equal(H, H.T) and ((H - Hr).abs() / d[:, None] / d).max().item() <= 6.1e-8


def _range_rows(n, ntiles):
    """rows of one range of a packed product's contraction: as many ranges as bring 2048 tiles together, of at least 8 stages of 64"""
    stages = (n + 63) // 64
    ranges = min(stages, -(-2048 // ntiles)) if ntiles < 1024 else 1
    return 64 * max(-(-stages // ranges), min(stages, 8))


@pytest.mark.parametrize("d1,m,n", [(1024, 512, 4096), (2048, 2048, 16384), (2056, 72, 9000), (4096, 8, 16384)])
def test_packed_gram_joins_its_ranges_in_float64(d1, m, n):
    """Three ranges of the contraction contribute 2^25, 1 and -2^25 to an entry: 1 if they meet in float64, 0 in float32.  With
    one copy of the result per range, with several ranges to a copy, and in wide tiles."""
    t, tm = (d1 + 127) // 128, (m + 127) // 128
    for target, tiles in ((False, t * (t + 1) // 2), (True, t * tm)):
        rows = _range_rows(n, tiles)
        assert 2 * rows < n
        X = torch.zeros(n, d1, dtype=torch.bfloat16, device=DEV)
        Y = torch.zeros(n, m, dtype=torch.bfloat16, device=DEV)
        X[0, 0::2], X[0, 1::2], Y[0] = 2.0 ** 12, 2.0 ** 13, 2.0 ** 13
        X[rows], Y[rows] = 1.0, 1.0
        X[2 * rows, 0::2], X[2 * rows, 1::2], Y[2 * rows] = 2.0 ** 12, -2.0 ** 13, -2.0 ** 13
        s = _pkg().Solver(d1, m, d1, 1, d1 // 2, 1, torch.bfloat16, torch.bfloat16, DEV, target_output=True)
        s.osscar_gram_target(X, Y, True, torch.zeros(d1, m, dtype=torch.bfloat16, device=DEV), 0.0, 0.0)
        H, G = s.osscar_get_tensor(0), s.osscar_get_tensor(1)
        s.close()
        got = G[0::2] if target else H[0::2, 1::2]
        assert got.min().item() == 1.0 and got.max().item() == 1.0


@pytest.mark.parametrize("d1,m", [(2048, 512), (4096, 2048)])
def test_product_with_bf16_weights_joins_its_ranges_in_float64(d1, m):
    """G = H W from three bf16 pieces of H: the rows k0, k1, k2 of three ranges contribute 2^25, 1 and -2^25."""
    rows = _range_rows(d1, (d1 // 128) * (m // 128))
    k = [0, rows, 2 * rows]
    assert k[2] < d1
    X = torch.zeros(64, d1, dtype=torch.bfloat16, device=DEV)
    X[0], X[1] = 2.0 ** 12, 1.0
    X[0, k], X[1, k] = torch.tensor([2.0 ** 13, 0, 2.0 ** 13], device=DEV).bfloat16(), torch.tensor([0, 1.0, 0], device=DEV).bfloat16()
    W = torch.zeros(d1, m, dtype=torch.bfloat16, device=DEV)
    W[k[0]], W[k[1]], W[k[2]] = 1.0, 1.0, -1.0
    s = _pkg().Solver(d1, m, d1, 1, d1 // 2, 1, torch.bfloat16, torch.bfloat16, DEV)
    s.osscar_gram(X, True, W, 0.0, 0.0)
    G = s.osscar_get_tensor(1)
    s.close()
    G = G[[i for i in range(d1) if i not in k]]
    assert G.min().item() == 1.0 and G.max().item() == 1.0


@pytest.mark.parametrize("d1,m,dtype", [(1024, 1024, torch.float32), (1100, 1028, torch.float32), (1031, 1025, torch.float32),
                                        (1031, 1025, torch.bfloat16), (1536, 1536, torch.bfloat16), (3584, 3520, torch.float32)])
def test_product_with_weights_small_where_activations_are_large(d1, m, dtype):
    """G = H W without the bf16 pieces, W inversely proportional to the channels' scales (eight of them 100 times the rest), where
    every term counts alike, and with one weight per column 10^4 times the others.  Sums are float64, so an entry of G is the
    float32 rounding of the exact one: 2^-24, and 2^-52 per term of |H| |W|."""
    g = torch.Generator(device=DEV).manual_seed(d1)
    rnd = lambda *a: torch.randn(*a, generator=g, device=DEV)
    scale = torch.exp(rnd(d1))
    scale[torch.randint(0, d1, (8,), generator=g, device=DEV)] *= 100
    X = (rnd(2 * d1, d1) * scale).to(dtype)
    W = (rnd(d1, m) / scale[:, None]).to(dtype)
    W[torch.randint(0, d1, (m,), generator=g, device=DEV), torch.arange(m, device=DEV)] *= 1e4
    s = _pkg().Solver(d1, m, d1, 1, d1 // 2, 1, dtype, dtype, DEV)
    s.osscar_gram(X, True, W, 0.0, 0.0)
    H, G = s.osscar_get_tensor(0).double(), s.osscar_get_tensor(1).double()
    Gr, size = H @ W.double(), H.abs() @ W.double().abs()
    assert ((G - Gr).abs() <= 2.0 ** -24 * 1.01 * Gr.abs() + d1 * 2.0 ** -52 * size).all()
    # an infinite weight and a NaN spoil their columns, and only those
    W[5, 3], W[d1 - 1, m - 1] = float("inf"), float("nan")
    s.osscar_gram(X, True, W, 0.0, 0.0)
    G2 = s.osscar_get_tensor(1)
    s.close()
    bad = torch.zeros(m, dtype=torch.bool, device=DEV)
    bad[3] = bad[m - 1] = True
    assert torch.equal(~torch.isfinite(G2), bad.expand(d1, m)) and torch.equal(G2[:, ~bad].double(), G[:, ~bad])


@pytest.mark.parametrize("p,k,t_hat", [(1000, 872, 64), (1000, 800, 40), (2050, 1900, 50)])
def test_block_removal_stops_at_a_row_that_was_not_looked_ahead(p, k, t_hat):
    """Of every 1024 rows 32 have their products computed ahead, so an iteration of more than that meets rows without: the block
    pivot asks for a stop, the host applies what is pending and removes the rest one by one.  Same removals as with the state updated in
    place after each, and the weights of the float64 inverse (a float32 state after 150 removals, condition number below 20: 1e-5)."""
    pkg = _pkg()
    m = 24
    g = torch.Generator().manual_seed(p + t_hat)
    A = torch.randn(2 * p, p, generator=g, dtype=torch.float64)
    H = (A.T @ A / (2 * p) + 0.2 * torch.eye(p, dtype=torch.float64)).float()
    H = torch.tril(H) + torch.tril(H, -1).T
    # half of the costs among the first 1024 rows, far below the others'
    W = torch.randn(p, m, generator=g, dtype=torch.float64) * torch.linspace(0.5, 3.0, p, dtype=torch.float64)[:, None]
    G = (H.double() @ W).float()
    s = pkg.Solver(p, m, p, 1, k, 1, torch.float32, torch.float32, DEV, from_dense=True)
    s.osscar_set_quadratic(H.to(DEV), G.to(DEV), float((W * G.double()).sum()), np.ones(p))
    _, ahead, _ = s.osscar_init_greedy(t_hat)
    kept, B = s.osscar_get_tensor(8).cpu().tolist(), s.osscar_get_tensor(3).cpu().double().numpy()
    _, in_place, _ = s.osscar_init_greedy(t_hat, 0, pkg.OSSCAR_SEARCH_EAGER)
    s.close()
    assert ahead == in_place and len(kept) == k and not set(kept) & set(sum(ahead, []))
    assert max(sum(x < 1024 for x in step) for step in ahead) > 32
    Br = np.linalg.solve(H.double().numpy()[np.ix_(kept, kept)], G.double().numpy()[kept])
    assert np.linalg.norm(B - Br) <= 1e-5 * np.linalg.norm(Br)


def test_map_of_more_than_2_to_the_31_patches():
    """A tall narrow float32 map with wide padding: 33 * (2^26 + 32) patches of two columns, all but 2^26 of them zero.  H is the
    float32 rounding of the float64 sums, whose 2^26 additions are in order within ranges: 2^-24 + 2^-53 * 2^20."""
    g = torch.Generator(device=DEV).manual_seed(31)
    F = torch.randn(1, 2, 1 << 26, 1, generator=g, device=DEV)
    W = torch.ones(2, 3, device=DEV)
    s = _pkg().Solver(2, 3, 2, 1, 1, 1, torch.float32, torch.float32, DEV)
    s.osscar_gram_conv(F, 1, 1, 1, 16, True, W, 0.0, 0.0)
    H = s.osscar_get_tensor(0).double().cpu()
    s.close()
    X = F.reshape(2, -1).double()
    Hr = torch.tensor([[(X[i] * X[j]).sum().item() for j in range(2)] for i in range(2)], dtype=torch.float64)
    d = Hr.diagonal().sqrt()
    assert ((H - Hr).abs() / d[:, None] / d).max().item() <= 6.1e-8


@pytest.mark.parametrize("q", [2, 17])
def test_reciprocals_of_pivots_are_rounded_correctly(q):
    """Groups whose diagonal block is diagonal: the gain of adding one is the sum of its squares over the diagonal, with two nonzero
    terms a bit-exact chain of one division, product and sum.  An infinite diagonal entry adds nothing."""
    pkg = _pkg()
    p, k = 200, 1
    rng = np.random.default_rng(q)
    h = np.exp(rng.uniform(-3, 3, (p, q))).astype(np.float32)
    b = rng.standard_normal((p, q)).astype(np.float32)
    b[:, 2:] = 0
    h[7, 0] = np.inf
    s = pkg.Solver(p * q, 1, p, q, k, 1, torch.float32, torch.float32, DEV)
    s.osscar_set_quadratic(torch.diag(torch.from_numpy(h.ravel())).to(DEV), torch.from_numpy(b.reshape(-1, 1)).to(DEV), 1e6, np.ones(p))
    s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, [0])
    add = s.osscar_get_tensor(7).cpu().numpy()
    s.close()
    hd, b2 = h.astype(np.float64), b.astype(np.float64) ** 2
    ref = (1.0 / hd[:, 0]) * b2[:, 0] + (1.0 / hd[:, 1]) * b2[:, 1]
    assert np.array_equal(add[1:], ref[1:])


@pytest.mark.parametrize("d1,m,p,q,k,swaps,dtype,dense,target,nbytes", [
    (288, 64, 32, 9, 16, 50, torch.float32, False, False, 14547200), (576, 64, 64, 9, 32, 50, torch.bfloat16, True, False, 27382016),
    (1024, 512, 16, 64, 8, 20, torch.bfloat16, False, False, 63750400), (1536, 640, 1536, 1, 768, 60, torch.bfloat16, False, True, 144641536),
    (3001, 40, 3001, 1, 1499, 60, torch.float32, False, False, 263547392)])
def test_a_workspace_without_the_extras_serves_the_layer(monkeypatch, d1, m, p, q, k, swaps, dtype, dense, target, nbytes):
    """A context takes less than osscar_workspace_bytes, down to what the arrays themselves need (the sizes here), and gives the same
    layer: sums in another order only (float64), so the kept sets are equal and the weights agree to float32 (1e-6 in the
    2-norm, cond below 100).  Below that it refuses."""
    pkg = _pkg()
    g = torch.Generator(device=DEV).manual_seed(d1)
    n = 3 * d1 + 77
    X = torch.randn(n, d1, generator=g, device=DEV).clamp_min(0).to(dtype)
    W = torch.randn(d1, m, generator=g, device=DEV).to(dtype)
    Y = torch.randn(n, m, generator=g, device=DEV).to(dtype)
    lib = pkg.load_library()

    def layer():
        s = pkg.Solver(d1, m, p, q, k, swaps, dtype, dtype, DEV, from_dense=dense, target_output=target)
        for r0 in range(0, n, 2048):
            more = (True, W, 0.0, 1e-2) if r0 + 2048 >= n else (False,)
            if target:
                s.osscar_gram_target(X[r0:r0 + 2048], Y[r0:r0 + 2048], *more)
            else:
                s.osscar_gram(X[r0:r0 + 2048], *more)
        s.osscar_init_greedy(2) if dense else s.osscar_init_support()
        s.osscar_local_search(swaps)
        What, support, obj = s.osscar_backsolve()
        size = s.workspace_bytes
        s.close()
        return What.double(), support.tolist(), obj, size

    full = layer()
    assert full[3] > nbytes
    monkeypatch.setattr(lib, "osscar_workspace_bytes", lambda desc: nbytes)
    less = layer()
    assert less[1] == full[1] and abs(less[2] - full[2]) <= 1e-6 * abs(full[2])
    assert (less[0] - full[0]).norm().item() <= 1e-6 * full[0].norm().item()
    monkeypatch.setattr(lib, "osscar_workspace_bytes", lambda desc: nbytes // 2)
    with pytest.raises(pkg.OsscarError) as e:
        layer()
    assert e.value.status == 2


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,d1,m,where", [(1500, 2901, 130, None), (9001, 2817, 70, None), (2500, 2945, 257, (128, 256)), (1100, 2883, 5, (2816, 2883))])
def test_gram_of_columns_with_rare_large_values(dtype, n, d1, m, where):
    """One value of 300 sigma in every column, or in those of one panel of 128 (a full one and the last): digits relative to it would leave
    the column's other products with too few bits, so the tiles of such panels are float64 sums: the float32 rounding of the
    exact entry, 2^-24, and 2^-53 per term.  The other tiles are digits: 2^-24 + 1e-9 of sqrt(H_ii H_jj)."""
    g = torch.Generator(device=DEV).manual_seed(n + d1)
    X = torch.randn(n, d1 + 1, generator=g, device=DEV)
    lo, hi = where or (0, d1)
    X[torch.randint(0, n, (hi - lo,), generator=g, device=DEV), torch.arange(lo, hi, device=DEV)] = 300.0
    X, Y = X.to(dtype)[:, :d1], torch.randn(n, m, generator=g, device=DEV).to(dtype)
    W = torch.zeros(d1, m, dtype=dtype, device=DEV)
    s = _pkg().Solver(d1, m, d1, 1, d1 // 2, 1, dtype, dtype, DEV, target_output=True)
    s.osscar_gram_target(X, Y, True, W, 0.0, 0.0)
    H, G = s.osscar_get_tensor(0).double(), s.osscar_get_tensor(1).double()
    s.close()
    Xd, Yd = X.double(), Y.double()
    exact = torch.zeros(d1, dtype=torch.bool, device=DEV)
    exact[lo:hi] = True
    for got, A, B, ex in ((H, Xd, Xd, exact[:, None] | exact), (G, Xd, Yd, exact[:, None].expand(d1, m))):
        ref, size = A.T @ B, A.abs().T @ B.abs()
        norm = A.square().sum(0).sqrt()[:, None] * B.square().sum(0).sqrt()
        assert ((got - ref).abs() <= 2.0 ** -24 * 1.01 * ref.abs() + n * 2.0 ** -53 * size)[ex].all()
        assert ((got - ref).abs() <= 6.1e-8 * norm).all()


@pytest.mark.parametrize("n,d1,m,kind", [(3000, 130, 20, 14), (3000, 2881, 20, 30)])
def test_the_log_holds_the_products_of_the_gram_phase(n, d1, m, kind):
    """X^T X (float64 sums, and in digits for wide layers: 16 more), X^T Y and G = H W of float32 rows, and the allocation-free call's."""
    from paper_2403_12983_amd import binding as B
    g = torch.Generator(device=DEV).manual_seed(d1)
    X, W = torch.randn(n, d1, generator=g, device=DEV), torch.randn(d1, m, generator=g, device=DEV)
    s = _pkg().Solver(d1, m, d1, 1, d1 // 2, 1, torch.float32, torch.float32, DEV, target_output=True)
    B.gemm_log(True)
    try:
        s.osscar_gram(X, True, W, 0.0, 1e-2)
        one = B.gemm_log_read()
        B.gemm_log(True)
        s.osscar_gram_target(X, X[:, :m].contiguous(), True, W, 0.0, 1e-2)
        two = B.gemm_log_read()
        B.gemm_log(True)
        if d1 <= 1024:
            _pkg().osscar_gram_static(X, W, torch.empty(d1, d1, device=DEV), torch.empty(d1, m, device=DEV),
                                      torch.empty(2, dtype=torch.float64, device=DEV))
        static = B.gemm_log_read()
    finally:
        B.gemm_log(False)
        s.close()
    def rows_of(log, M, N, k):
        """contraction lengths of the products of this shape and kind, durations positive"""
        assert (log[:, 4] > 0).all()
        return log[(log[:, 0] == M) & (log[:, 1] == N) & (log[:, 3] == k)][:, 2].sum()
    assert rows_of(one, d1, d1, kind) == n and rows_of(one, d1, m, 0) == d1
    assert rows_of(two, d1, d1, kind) == n and rows_of(two, d1, m, 2 + (kind & 16)) == n
    if d1 <= 1024:
        assert rows_of(static, d1, d1, 14) == n and rows_of(static, d1, m, 0) == d1


@pytest.mark.parametrize("d1,n", [(64, 64), (8, 1), (1000, 1000), (1000, 2100), (2048, 130)])
def test_packed_gram_adds_the_same_in_small_and_large_launches(d1, n):
    """Launches of few workgroups add to the float64 result with atomics, larger ones with loads and stores: two equal chunks give
    exactly twice the sums of one, and again the same bits."""
    g = torch.Generator(device=DEV).manual_seed(d1 + n)
    X = torch.randn(n, d1, generator=g, device=DEV).bfloat16()
    W = torch.zeros(d1, 8, dtype=torch.bfloat16, device=DEV)
    s = _pkg().Solver(d1, 8, d1, 1, d1 // 2, 1, torch.bfloat16, torch.bfloat16, DEV)
    H = []
    for chunks in (1, 2, 2):
        for _ in range(chunks - 1):
            s.osscar_gram(X)
        s.osscar_gram(X, True, W, 0.0, 0.0)
        H.append(s.osscar_get_tensor(0))
    s.close()
    assert torch.equal(H[1], H[2]) and torch.equal(H[1], 2 * H[0])
    Hr = (X.double().T @ X.double()).cpu().numpy()
    d = np.sqrt(np.diag(Hr))
    assert np.max(np.abs(H[0].cpu().double().numpy() - Hr) / np.outer(d, d)) <= 1e-6


@pytest.mark.parametrize("p,m,k,swaps", [(31, 3, 15, 40), (33, 20, 17, 40), (257, 36, 100, 90), (8192, 33, 4000, 70), (8193, 8, 4100, 70),
                                         (16384, 40, 8000, 66), (16385, 17, 8001, 66)])
def test_swaps_in_one_launch(p, m, k, swaps):
    """One launch per swap, at the edges of its workgroups' rows (32, 64 and 128), past a flush: the same swaps as with the state updated in
    place, with the products computed ahead and without (then every pivot's are fetched).  The runs may part only where two groups
    score alike (1e-5, the bar on choices); up to there the exact changes agree to 1e-6 of the objective (float32 storage)."""
    pkg = _pkg()
    g = torch.Generator().manual_seed(p)
    X = (torch.randn(2 * p + 64 if p < 1000 else 1024, p, generator=g) * torch.exp(0.5 * torch.randn(p, generator=g))).to(DEV)
    W = (torch.randn(p, m, generator=g) / p ** 0.5).to(DEV)
    s = pkg.Solver(p, m, p, 1, k, swaps, torch.float32, torch.float32, DEV)
    s.osscar_gram(X, True, W, 0.0, 5e-2)
    runs = []
    for flags in (pkg.OSSCAR_SEARCH_EAGER, 0, pkg.OSSCAR_SEARCH_NO_LOOKAHEAD):
        s.osscar_init_support()
        r = s.osscar_local_search(swaps, 0.0, flags | pkg.OSSCAR_SEARCH_ALWAYS_ACCEPT)
        assert r["iters"] == r["accepted"] == swaps
        runs.append((r, s.osscar_get_counters(), s.osscar_backsolve()))
    s.close()
    (e, _, (We, Se, _)), (a, ca, _), (b, cb, _) = runs
    assert cb["lookahead_misses"] >= 2 * min(swaps, k) and ca["lookahead_misses"] < cb["lookahead_misses"]
    for r, _, (Wr, Sr, _) in runs[1:]:
        same = (r["trace_out"] == e["trace_out"]) & (r["trace_in"] == e["trace_in"])
        n = swaps if same.all() else int(np.argmin(same))
        assert n == swaps or e["trace_gap"][n].min() <= 1e-5
        assert np.allclose(r["trace_obj"][:n], e["trace_obj"][:n], rtol=1e-6, atol=0)
        if n == swaps:
            assert Sr.tolist() == Se.tolist() and torch.linalg.norm(Wr - We) <= 1e-5 * torch.linalg.norm(We)


@pytest.mark.parametrize("p,m,k,swaps", [(63, 8, 30, 40), (64, 504, 32, 40), (65, 520, 32, 40), (129, 1032, 60, 70), (4097, 1000, 2000, 70),
                                         (16320, 512, 8000, 66), (16321, 520, 8000, 66), (25472, 24, 12000, 66), (25473, 24, 12000, 66)])
def test_products_computed_ahead_in_64_rows(p, m, k, swaps):
    """The same at the edges of the products' 64-row workgroups, of their last stage of 32 columns, of the cut of the columns in two (from 512 on,
    below 256 workgroups) and of the 199 workgroups of 128 rows beyond which these do them.  Bounds as there: three bf16 terms a factor
    leave 2^-24 of a product, as the float32 storage does."""
    test_swaps_in_one_launch(p, m, k, swaps)


def _same_swaps(r, e, Wr, We, Sr, Se):
    """The search r took the swaps of e, except behind a choice between two groups that score alike."""
    n = min(r["iters"], e["iters"])
    same = (r["trace_out"][:n] == e["trace_out"][:n]) & (r["trace_in"][:n] == e["trace_in"][:n])
    n = n if same.all() else int(np.argmin(same))
    assert n == e["iters"] == r["iters"] or e["trace_gap"][n].min() <= 1e-9
    assert np.allclose(r["trace_obj"][:n], e["trace_obj"][:n], rtol=1e-9, atol=0)
    assert np.allclose(r["trace_gap"][:n], e["trace_gap"][:n], rtol=1e-5, atol=1e-9)
    if n == e["iters"]:
        assert r["accepted"] == e["accepted"] and Sr.tolist() == Se.tolist() and torch.linalg.norm(Wr - We) <= 1e-6 * torch.linalg.norm(We)


@pytest.mark.parametrize("p,m,k,swaps", [(31, 3, 15, 40), (32, 8, 16, 40), (600, 72, 300, 90), (8192, 40, 4000, 150), (8193, 8, 4100, 70),
                                         (16384, 40, 8000, 66), (16385, 16, 8001, 66), (32768, 8, 16384, 66), (32769, 8, 16384, 10)])
def test_runs_of_swaps(p, m, k, swaps):
    """Many swaps in one launch, at the edges of the workgroups' rows and on either side of the 256 workgroups that can be resident together, and
    moves of given pairs: the same swaps as with a launch each, also where every wait is given up at once.  Both ways are float64 algebra on
    the same stored numbers, in another order: the objective agrees to 1e-9 (1e-16 times the square of |z0| / |z|, below 1e3 here), and the
    choices part only where two groups score alike."""
    pkg = _pkg()
    g = torch.Generator(device=DEV).manual_seed(p)
    X = torch.randn(2 * p + 64 if p < 1000 else 1024, p, generator=g, device=DEV) * torch.exp(0.5 * torch.randn(p, generator=g, device=DEV))
    W = torch.randn(p, m, generator=g, device=DEV) / p ** 0.5
    s = pkg.Solver(p, m, p, 1, k, swaps, torch.float32, torch.float32, DEV)
    s.osscar_gram(X, True, W, 0.0, 5e-2)
    out = []
    for flags in (pkg.OSSCAR_SEARCH_LAUNCH_PER_SWAP, 0, pkg.OSSCAR_SEARCH_IMPATIENT):
        s.osscar_init_support()
        r = s.osscar_local_search(swaps, 0.0, flags)
        out.append((r, s.osscar_get_counters(), s.osscar_backsolve()))
    moves = []
    for flags in (pkg.OSSCAR_SEARCH_LAUNCH_PER_SWAP, 0):
        s.osscar_init_support()
        moves.append((s.osscar_block_search(5, min(7, k), 0.0, flags), s.osscar_backsolve()))
    s.close()
    (e, ce, (We, Se, _)) = out[0]
    assert ce["runs"] == 0 and (out[1][1]["runs"] > 0) == (p <= 32768)
    assert out[2][1]["runs"] == out[2][1]["runs_given_up"] == (p <= 32768)
    for r, c, (Wr, Sr, _) in out[1:]:
        _same_swaps(r, e, Wr, We, Sr, Se)
    (a, (Wa, Sa, _)), (b, (Wb, Sb, _)) = moves
    assert a["moves"] == b["moves"] and a["accepted"] == b["accepted"] and Sa.tolist() == Sb.tolist()
    assert abs(a["obj_final"] - b["obj_final"]) <= 1e-9 * abs(a["obj_final"]) and torch.linalg.norm(Wa - Wb) <= 1e-6 * torch.linalg.norm(Wa)


@pytest.mark.parametrize("p,m,k,swaps", [(600, 72, 300, 180), (2000, 400, 900, 250), (8193, 8, 4100, 250), (16385, 16, 8001, 200)])
def test_run_given_up_with_swaps_pending(p, m, k, swaps):
    """A run that goes on behind fetched products, with the swaps of the run before still pending, is given up, with another run already
    enqueued behind it: the same swaps as with a launch each.  Neighbouring columns are correlated, so that some pivots' products have to be
    fetched.  Bounds as above."""
    pkg = _pkg()
    g = torch.Generator(device=DEV).manual_seed(p)
    X = torch.randn(2 * p + 64 if p < 1000 else 1024, p, generator=g, device=DEV) * torch.exp(0.5 * torch.randn(p, generator=g, device=DEV))
    X = X + 0.3 * torch.roll(X, -1, dims=1)
    W = torch.randn(p, m, generator=g, device=DEV) / p ** 0.5
    s = pkg.Solver(p, m, p, 1, k, swaps, torch.float32, torch.float32, DEV)
    s.osscar_gram(X, True, W, 0.0, 5e-2)
    out = []
    for flags in (pkg.OSSCAR_SEARCH_LAUNCH_PER_SWAP, pkg.OSSCAR_SEARCH_IMPATIENT_LATER):
        s.osscar_init_support()
        r = s.osscar_local_search(swaps, 0.0, flags | pkg.OSSCAR_SEARCH_ALWAYS_ACCEPT)
        out.append((r, s.osscar_get_counters(), s.osscar_backsolve()))
    s.close()
    (e, ce, (We, Se, _)), (r, c, (Wr, Sr, _)) = out
    assert ce["runs_given_up"] == 0 and ce["lookahead_misses"] > 0
    assert c["runs_given_up"] == 1 and c["runs"] >= 3
    _same_swaps(r, e, Wr, We, Sr, Se)


def test_two_searches_at_once():
    """Two contexts on two streams and two threads, each with runs that want every compute unit: whether or not a run is given up for it, the
    swaps are those of a launch each with the GPU to itself.  Bounds as above."""
    pkg = _pkg()
    p, m, k, swaps = 8192, 64, 4096, 300
    solvers, alone, both = [], [], [[], []]
    for seed in (1, 2):
        with torch.cuda.stream(torch.cuda.Stream()):
            g = torch.Generator(device=DEV).manual_seed(seed)
            X = torch.randn(1024, p, generator=g, device=DEV) * torch.exp(0.5 * torch.randn(p, generator=g, device=DEV))
            W = torch.randn(p, m, generator=g, device=DEV) / p ** 0.5
            s = pkg.Solver(p, m, p, 1, k, swaps, torch.float32, torch.float32, DEV)
            s.osscar_gram(X, True, W, 0.0, 5e-2)
        s.osscar_init_support()
        alone.append((s.osscar_local_search(swaps, 0.0, pkg.OSSCAR_SEARCH_LAUNCH_PER_SWAP), s.osscar_backsolve()))
        solvers.append(s)
    together = threading.Barrier(2, timeout=60)

    def work(i):
        for _ in range(4):
            solvers[i].osscar_init_support()
            together.wait()
            r = solvers[i].osscar_local_search(swaps)
            both[i].append((r, solvers[i].osscar_get_counters(), solvers[i].osscar_backsolve()))

    threads = [threading.Thread(target=work, args=(i,)) for i in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s in solvers:
        s.close()
    for (e, (We, Se, _)), calls in zip(alone, both):
        assert len(calls) == 4
        for r, c, (Wr, Sr, _) in calls:
            assert c["runs"] > 0
            _same_swaps(r, e, Wr, We, Sr, Se)


@pytest.mark.parametrize("target", [False, True])
@pytest.mark.parametrize("d1,m,chunks", [(1096, 72, [1, 2048, 63, 700, 0]), (2048, 8, [2048] * 9), (2056, 520, [16384 - 128, 64, 64, 1, -130, 200]),
                                         (1504, 40, [5000, 20000, 5000, 0]), (8, 8, [70, 1, 300])])
def test_rows_of_several_calls_in_one_product(d1, m, chunks, target):
    """Calls whose rows wait for a full buffer: one row, rows up to the buffer's last stage, more than a buffer, a chunk at another alignment
    in between (negative), a last call without rows.  The activations are small whole numbers, so every sum is exact in float32 (below
    2^24) and H and G must be exact; in the first two columns only three rows, of different calls, are not zero: they contribute 2^25, 1 and
    -2^25 to an entry, and meet in float64."""
    n = sum(abs(c) for c in chunks)
    g = torch.Generator(device=DEV).manual_seed(d1 + n)
    X = torch.randint(-3, 4, (n, d1), generator=g, device=DEV).bfloat16()
    Y = torch.randint(-3, 4, (n, m), generator=g, device=DEV).bfloat16()
    X[:, :2] = 0.0
    X[0, :2] = torch.tensor([2.0 ** 12, 2.0 ** 13], device=DEV).bfloat16()
    X[abs(chunks[0]) + abs(chunks[1]) // 2, :2] = 1.0
    X[n - 1, :2] = torch.tensor([2.0 ** 12, -2.0 ** 13], device=DEV).bfloat16()
    W = torch.zeros(d1, m, dtype=torch.bfloat16, device=DEV)
    s = _pkg().Solver(d1, m, d1, 1, d1 // 2, 1, torch.bfloat16, torch.bfloat16, DEV, target_output=target)
    r0 = 0
    for i, c in enumerate(chunks):
        x, y = X[r0:r0 + abs(c)], Y[r0:r0 + abs(c)]
        if c < 0:
            x = torch.cat([x[:, :1], x], 1)[:, 1:]
        args = (True, W, 0.0, 0.0) if i + 1 == len(chunks) else (False,)
        s.osscar_gram_target(x, y, *args) if target else s.osscar_gram(x, *args)
        r0 += abs(c)
    H, G = s.osscar_get_tensor(0).double(), s.osscar_get_tensor(1).double()
    s.close()
    Xd = X.double()
    Hr = Xd.T @ Xd
    off = torch.ones(d1, d1, dtype=torch.bool, device=DEV)
    off[0], off[:, 0], off[1], off[:, 1] = False, False, False, False      # beyond 2^24 but for the entry where the large terms cancel
    assert torch.equal(H[off], Hr[off]) and H[0, 1] == Hr[0, 1] == H[1, 0] == 1.0
    if target:
        assert torch.equal(G[2:], (Xd.T @ Y.double())[2:])


@pytest.mark.parametrize("target", [False, True])
@pytest.mark.parametrize("d1,m,chunks", [(4096, 1096, [2048] * 8 + [0]), (4104, 2000, [2048] * 8 + [1, -130, 66]), (5632, 1536, [4000, 4000, 5000]),
                                         (2056, 3720, [1000, 3000, 4500, 66])])
def test_tiles_that_do_not_fill_a_round(d1, m, chunks, target):
    """The same where the result's 256 x 128 tiles (272, 289 with remainders on either side, 506, which stay whole, and 45 beside 270 of the target's)
    leave a last round of the compute units nearly empty and are cut along the rows."""
    test_rows_of_several_calls_in_one_product(d1, m, chunks, target)


@pytest.mark.parametrize("costs", ["shuffled", "equal", "ascending"])
@pytest.mark.parametrize("p,t_hat", [(40, 3), (70, 16), (1030, 10), (8192, 16), (8193, 7), (30100, 16), (30144, 16), (30145, 16)])
def test_picks_of_block_removals(p, t_hat, costs):
    """The rows of an iteration come from sorted lists of every 64 rows: fewer rows than a list, more lists than groups of them, the last size
    whose entries are all staged (30144 rows, 471 lists of 17) and the first with 16 of each (30145), where the 17th of a list, read
    where it lies, is the one that ends the gap when one list holds the cheapest rows (ascending costs).  With H = I the cost of a row
    is its weights' squared norm, whatever has left, so the removals go by that norm; of equal ones the lowest rows leave first, past
    those whose products are computed ahead."""
    pkg = _pkg()
    m, iters = 8, 3
    k = p - iters * t_hat
    g = torch.Generator().manual_seed(p)
    scale = torch.ones(p) if costs == "equal" else 1.0 + (torch.arange(p) if costs == "ascending" else torch.randperm(p, generator=g)).float() / p
    W = (torch.ones(p, m) * scale[:, None]).to(DEV)
    H = torch.eye(p, device=DEV)
    s = pkg.Solver(p, m, p, 1, k, 1, torch.float32, torch.float32, DEV, from_dense=True)
    s.osscar_set_quadratic(H, W, float((W.double() ** 2).sum()), np.ones(p))
    obj, steps, gaps = s.osscar_init_greedy(t_hat)
    s.close()
    order = np.argsort(scale.double().numpy(), kind="stable")
    assert [len(x) for x in steps] == [t_hat] * iters and sum(steps, []) == order[:iters * t_hat].tolist()
    cost = np.append(scale.double().numpy()[order] ** 2, np.inf)
    for i, gap in enumerate(gaps):
        lo, hi = cost[(i + 1) * t_hat - 1], cost[(i + 1) * t_hat]
        assert abs(gap - (hi - lo) / lo) <= 1e-6      # (neighbours differ by 2 / p, 6.6e-5 at the largest p)


@pytest.mark.parametrize("p", [2, 255, 257, 2048, 2049])
def test_selection_of_groups(p):
    """Groups of two rows around the selection's sizes: one score, a wave and a workgroup more or less, and on either side of the
    size from which a launch of its own selects.  H = the identity times the group's own factor, so that a group's cost and gain are
    its own rows' squares over that factor, and every value that can be asked for is known: three moves take the smallest kept
    and the largest excluded score, the lowest index of equal ones (there are many), and the objective follows exactly up to
    its float64 sums (scores are sums of two small whole numbers)."""
    pkg = _pkg()
    q, m, d1, k = 2, 3, 2 * p, p // 2
    gen = torch.Generator().manual_seed(p)
    val = torch.randint(1, 6, (p,), generator=gen)                              # a group's rows: (val, 0, 0), (0, 1, 0)
    G = torch.zeros(d1, m)
    G[0::2, 0] = val.float()
    G[1::2, 1] = 1.0
    kept = set(torch.randperm(p, generator=gen)[:k].tolist())
    score = [float(v) ** 2 + 1.0 for v in val.tolist()]
    s = pkg.Solver(d1, m, p, q, k, 4, torch.float32, torch.float32, DEV)
    s.osscar_set_quadratic(torch.eye(d1).to(DEV), G.to(DEV), 0.0, np.ones(p))
    s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, sorted(kept))
    moves = []
    for _ in range(3):
        r = s.osscar_local_search(max_swaps=1, rel_tol=0.0)
        g, j = min((score[x], x) for x in kept)[1], min((-score[x], x) for x in range(p) if x not in kept)[1]
        if score[j] <= score[g]:
            assert r["accepted"] == 0
            break
        assert r["accepted"] == 1 and (r["trace_out"][0], r["trace_in"][0]) == (g, j)
        assert abs((r["obj_initial"] - r["obj_final"]) - (score[j] - score[g])) <= 1e-9 * sum(score)
        kept = kept - {g} | {j}
        moves.append((g, j))
    assert s.osscar_get_tensor(8).cpu().numpy().astype(int).tolist() == sorted(kept)


@pytest.mark.parametrize("p,q,block", [(3, 1, 1), (40, 1, 20), (130, 1, 64), (70, 2, 5), (8193, 1, 10)])
def test_pairs_of_block_moves(p, q, block):
    """Block moves of rows and of groups, the smallest and the largest block: H = the identity, so that a score is the sum of the group's own squares and
    stays what it is; a move takes the cheapest kept and the dearest excluded groups, the lowest index of equal ones first, until
    a move does not pay, which is taken back (the whole block, from its last pair)."""
    pkg = _pkg()
    gen = torch.Generator().manual_seed(p)
    val = torch.randint(1, 6, (p,), generator=gen)
    G = torch.zeros(p * q, 3)
    G[0::q, 0] = val.float()
    kept = set(torch.randperm(p, generator=gen)[:p // 2].tolist())
    score = [float(v) ** 2 for v in val.tolist()]
    s = pkg.Solver(p * q, 3, p, q, p // 2, 4, torch.float32, torch.float32, DEV)
    s.osscar_set_quadratic(torch.eye(p * q).to(DEV), G.to(DEV), 0.0, np.ones(p))
    s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, sorted(kept))
    r = s.osscar_block_search(max_iters=4, block=block, rel_tol=0.0)
    moves = 0
    for i in range(r["iters"]):
        out = sorted(kept, key=lambda x: (score[x], x))[:block]
        inn = sorted(set(range(p)) - kept, key=lambda x: (-score[x], x))[:block]
        take = min(len(out), len(inn))
        assert (r["moves"][i][0], r["moves"][i][1]) == (out[:take], inn[:take])
        if sum(score[x] for x in inn[:take]) > sum(score[x] for x in out[:take]):
            kept = kept - set(out[:take]) | set(inn[:take])
            moves += 1
    assert r["accepted"] == moves and s.osscar_get_tensor(8).cpu().numpy().astype(int).tolist() == sorted(kept)
    assert abs(r["obj_final"] + sum(score[x] for x in kept)) <= 1e-9 * sum(score)


@pytest.mark.parametrize("before", [1, 2, 3])
def test_rebuilt_state_that_is_not_definite_is_an_error(before):
    """H with two equal rows a, b: once a is kept, the Schur complement of b is rounding, of either sign.  a enters by the `before`-th
    swap, after which the state is rebuilt.  Whether the rebuilt one is positive shows in a state built from that kept set at once: the score of b is
    its squared norm over it, or over one where it is not.  Where it is not the search is an error, whatever the number of launches before."""
    pkg = _pkg()
    p, k, m, a, b = 40, 20, 3, 30, 35
    wrong = 0
    for seed in range(16):
        g = torch.Generator().manual_seed(seed)
        X = torch.randn(400, p, generator=g, dtype=torch.float64)
        X[:, b] = X[:, a]
        H = (X.T @ X).float()
        H[b], H[:, b] = H[a], H[:, a]
        H[b, b] = H[a, a]
        G = torch.randn(p, m, generator=g)
        for i in range(before):
            G[20 + i] = 1000.0 / 2.0 ** i                   # enter first, in this order
        G[20 + before - 1] = 1.0
        G[a] = G[b] = 1000.0 / 2.0 ** (before - 1)
        s = pkg.Solver(p, m, p, 1, k, 8, torch.float32, torch.float32, DEV)
        s.osscar_set_quadratic(H.to(DEV), G.to(DEV), 1e6, np.ones(p))
        s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, list(range(k)))
        r = s.osscar_local_search(before, 0.0, pkg.OSSCAR_SEARCH_ALWAYS_ACCEPT)
        assert r["trace_in"].tolist() == [20 + i for i in range(before - 1)] + [a]
        kept = sorted(set(range(k)) - set(r["trace_out"].tolist()) | set(r["trace_in"].tolist()))
        s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, kept)
        gain = float(s.osscar_get_tensor(7)[b])
        row = s.osscar_get_tensor(5)[sorted(set(range(p)) - set(kept)).index(b)].double()
        positive = gain > 2.0 * float((row * row).sum())    # (the complement is far below one)
        s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, list(range(k)))
        if not positive:
            wrong += 1
            with pytest.raises(pkg.OsscarError) as e:
                s.osscar_local_search(before + 1, 0.0, pkg.OSSCAR_SEARCH_ALWAYS_ACCEPT, refresh_every=before)
            assert e.value.status == 3
        s.close()
    assert wrong > 0


@pytest.mark.parametrize("p,m,block", [(300, 20, 64), (300, 20, 17), (700, 192, 32), (1030, 8, 10)])
def test_block_moves_whose_products_are_not_computed_ahead(p, m, block):
    """Moves in which every pair (no look-ahead) or most pairs (few rows are looked ahead in a small layer) have to fetch their products:
    the same moves as in place, to 1e-6 of the objective (float32 storage), and no more than about two launches a pair.  Launches enqueued
    again after every fetch took up to 6.5 times as long as four launches a pair here and are now as long or shorter; the search in place takes
    about as long, and the bar is twice its time."""
    pkg = _pkg()
    g = torch.Generator().manual_seed(p)
    X = (torch.randn(2 * p + 64, p, generator=g) * torch.exp(0.5 * torch.randn(p, generator=g))).to(DEV)
    W = (torch.randn(p, m, generator=g) / p ** 0.5).to(DEV)
    s = pkg.Solver(p, m, p, 1, p // 2, 1, torch.float32, torch.float32, DEV)
    s.osscar_gram(X, True, W, 0.0, 5e-2)
    runs = []
    for flags in (pkg.OSSCAR_SEARCH_EAGER, 0, pkg.OSSCAR_SEARCH_NO_LOOKAHEAD):
        ms = []
        for _ in range(3):
            s.osscar_init_support()
            r = s.osscar_block_search(3, block, 0.0, flags | pkg.OSSCAR_SEARCH_ALWAYS_ACCEPT)
            ms.append(s.osscar_get_timers()[3])
        s.osscar_init_support()
        back = s.osscar_block_search(3, block, 0.9, flags)      # turned down: taken back, the last pair first
        assert r["iters"] == r["accepted"] == 3 and back["iters"] == 1 and back["accepted"] == 0
        assert back["obj_final"] == back["obj_initial"]
        runs.append((r, min(ms), s.osscar_backsolve()))
    s.close()
    (e, te, (We, Se, _)), others = runs[0], runs[1:]
    for r, t, (Wr, Sr, _) in others:
        assert r["moves"] == e["moves"]
        assert np.allclose(r["trace_obj"], e["trace_obj"], rtol=1e-6, atol=0)
        assert Sr.tolist() == Se.tolist() and torch.linalg.norm(Wr - We) <= 1e-5 * torch.linalg.norm(We)
        print(f"p {p} block {block}: in place {te:.2f} ms, delayed {t:.2f} ms")
        assert t <= 2.0 * te


def _exact_gram(d1, m, chunks, target):
    """H and G of calls of `chunks` rows of small whole numbers (every sum exact in float32), the timers, the same in float64"""
    n = sum(chunks)
    g = torch.Generator(device=DEV).manual_seed(d1 + n)
    X = torch.randint(-3, 4, (n, d1), generator=g, device=DEV).bfloat16()
    Y = torch.randint(-3, 4, (n, m), generator=g, device=DEV).bfloat16()
    W = torch.zeros(d1, m, dtype=torch.bfloat16, device=DEV)
    s = _pkg().Solver(d1, m, d1, 1, 1, 1, torch.bfloat16, torch.bfloat16, DEV, target_output=target)
    r0 = 0
    for i, c in enumerate(chunks):
        args = (True, W, 0.0, 0.0) if i + 1 == len(chunks) else (False,)
        s.osscar_gram_target(X[r0:r0 + c], Y[r0:r0 + c], *args) if target else s.osscar_gram(X[r0:r0 + c], *args)
        r0 += c
    H, G, t = s.osscar_get_tensor(0).double(), s.osscar_get_tensor(1).double(), s.osscar_get_timers()
    s.close()
    Xd = X.double()
    assert torch.equal(H, Xd.T @ Xd) and (not target or torch.equal(G, Xd.T @ Y.double()))
    return t


@pytest.mark.parametrize("d1,m,chunks,launches", [(512, 64, [6000, 6000], 2), (1000, 72, [2100, 3000, 1], 3), (520, 8, [2048, 2048, 65, 700], 4),
                                                  (1000, 72, [1024, 1000, 900], 1), (2048, 512, [2048, 3000], 1)])
def test_rows_that_wait_when_the_layer_ends(d1, m, chunks, launches):
    """Rows of several calls that do not fill the buffer: together where they keep half of the compute units busy or the calls are short, else a
    launch per call.  Sums of small whole numbers are exact either way.  (512 columns, two calls of 6000 rows: eight workgroups took the
    whole contraction, three times as long as the two launches.)"""
    t = _exact_gram(d1, m, chunks, False)
    assert t[14] == launches and sum(chunks) <= t[15] < sum(chunks) + 128 * len(chunks)
    if launches == 2:
        ms = [min(u[13] * u[14] for u in [_exact_gram(d1, m, c, False) for _ in range(3)]) for c in (chunks, [sum(chunks)])]
        assert ms[0] <= 2.0 * ms[1]
    _exact_gram(d1, m, chunks, True)


@pytest.mark.parametrize("d1,chunks,launches,rows", [(8192, [9000, 9000], 1, 9000), (8192, [300, 5000], 2, 5300), (8192, [4608, 4608], 1, 9216),
                                                     (5120, [9000, 9000], 2, 18000)])
def test_long_calls_are_multiplied_by_themselves(d1, chunks, launches, rows):
    """Where the 256 x 192 tiles fill the chip, a call of more than 4608 rows does not wait (launches and rows are those of the last call): collected
    in the buffer, calls of 12000 rows of 8192 columns took 1.15 times as long.  At 5120 columns, 287 tiles, they wait."""
    t = _exact_gram(d1, 8, chunks, False)
    assert (t[14], t[15]) == (launches, rows)


def test_the_timers_hold_the_products_of_rows_that_waited():
    """A finalizing call without rows multiplies the rows of the calls before it: their time is the Gram accumulation's."""
    g = torch.Generator(device=DEV).manual_seed(1)
    X = torch.randn(4096, 2048, generator=g, device=DEV).bfloat16()
    W = torch.zeros(2048, 8, dtype=torch.bfloat16, device=DEV)
    s = _pkg().Solver(2048, 8, 2048, 1, 1, 1, torch.bfloat16, torch.bfloat16, DEV)
    s.osscar_gram(X[:2048])
    s.osscar_gram(X[2048:])
    s.osscar_gram(None, True, W, 0.0, 1e-2)
    t = s.osscar_get_timers()
    s.close()
    assert t[14] == 1 and 0.5 * t[13] <= t[0] <= t[13] + 1.0      # ms; the product is 0.05


@pytest.mark.parametrize("p,k", [(32768, 300), (32769, 70)])
def test_swaps_in_more_workgroups_than_compute_units(p, k):
    """One launch per swap with 128 rows a workgroup: 256 of them, and one more, which starts when others have ended and have entered the swap
    in what only grows.  H = the identity with neighbouring rows coupled by 0.3: the same swaps as with the state updated in place (rows that
    score alike to 1e-5 apart), past a flush, with and without products computed ahead."""
    pkg = _pkg()
    m, swaps = 8, 66
    g = torch.Generator(device=DEV).manual_seed(p)
    H = torch.eye(p, device=DEV)
    H.diagonal(1).fill_(0.3)
    H.diagonal(-1).fill_(0.3)
    G = torch.randn(p, m, generator=g, device=DEV)
    s = pkg.Solver(p, m, p, 1, k, swaps, torch.float32, torch.float32, DEV)
    s.osscar_set_quadratic(H, G, 10.0 * float((G.double() ** 2).sum()), np.ones(p))
    del H
    kept = torch.randperm(p, generator=torch.Generator().manual_seed(p))[:k].tolist()
    runs = []
    for flags in (pkg.OSSCAR_SEARCH_EAGER, 0, pkg.OSSCAR_SEARCH_NO_LOOKAHEAD):
        s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, kept)
        r = s.osscar_local_search(swaps, 0.0, flags | pkg.OSSCAR_SEARCH_ALWAYS_ACCEPT)
        assert r["iters"] == r["accepted"] == swaps
        runs.append((r, s.osscar_backsolve()))
    s.close()
    e, (We, Se, _) = runs[0]
    for r, (Wr, Sr, _) in runs[1:]:
        same = (r["trace_out"] == e["trace_out"]) & (r["trace_in"] == e["trace_in"])
        n = swaps if same.all() else int(np.argmin(same))
        assert n == swaps or e["trace_gap"][n].min() <= 1e-5
        assert np.allclose(r["trace_obj"][:n], e["trace_obj"][:n], rtol=1e-6, atol=0)
        if n == swaps:
            assert Sr.tolist() == Se.tolist() and torch.linalg.norm(Wr - We) <= 1e-5 * torch.linalg.norm(We)


@pytest.mark.parametrize("p,m,swaps", [(1024, 16383, 30), (40, 4100, 8), (513, 4097, 30)])
def test_products_fetched_for_long_rows(p, m, swaps):
    """Pivots whose products are fetched, rows of 16383 columns (read four at a time, the last three apart) and of just more than 4096 (from where
    workgroups without rows help): the same swaps as in place, and no more than three times its time.  Column by column, with one
    request of a row of K in flight at a time, by the layer's own workgroups, it took six times as long with 16383 columns."""
    pkg = _pkg()
    g = torch.Generator(device=DEV).manual_seed(5)
    X = torch.randn(2 * p + 152, p, generator=g, device=DEV) * torch.exp(0.5 * torch.randn(p, generator=g, device=DEV))
    W = torch.randn(p, m, generator=g, device=DEV) / p ** 0.5 * (1.0 + torch.arange(p, device=DEV)[:, None] / p)
    s = pkg.Solver(p, m, p, 1, p // 2, swaps, torch.float32, torch.float32, DEV)
    s.osscar_gram(X, True, W, 0.0, 5e-2)
    runs = []
    for flags in (pkg.OSSCAR_SEARCH_EAGER, pkg.OSSCAR_SEARCH_NO_LOOKAHEAD):
        ms = []
        for _ in range(3):
            s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, list(range(0, p, 2))[:p // 2])
            r = s.osscar_local_search(swaps, 0.0, flags)
            ms.append(s.osscar_get_timers()[3])
        runs.append((r, min(ms)))
    s.close()
    (e, te), (r, t) = runs
    print(f"in place {te:.2f} ms, fetched {t:.2f} ms")
    assert e["iters"] == swaps and r["trace_out"].tolist() == e["trace_out"].tolist() and r["trace_in"].tolist() == e["trace_in"].tolist()
    assert np.allclose(r["trace_obj"], e["trace_obj"], rtol=1e-6, atol=0)
    assert t <= 3.0 * te


def test_flushes_without_products_computed_ahead():
    """Every pending pivot has a slot for its products when none are computed ahead: 128 swaps of rows that are not swapped twice are two flushes
    and no pause, and so are 256 removals."""
    pkg = _pkg()
    p, m = 600, 4
    G = (1.0 + torch.randperm(p, generator=torch.Generator().manual_seed(1)).float() / p)[:, None] * torch.ones(p, m)
    s = pkg.Solver(p, m, p, 1, 300, 128, torch.float32, torch.float32, DEV, from_dense=True)
    s.osscar_set_quadratic(torch.eye(p).to(DEV), G.to(DEV), 1e4, np.ones(p))
    worst = torch.argsort(G[:, 0])[:300].tolist()
    s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, sorted(worst))
    r = s.osscar_local_search(128, 0.0, pkg.OSSCAR_SEARCH_NO_LOOKAHEAD)
    c = s.osscar_get_counters()
    assert r["accepted"] == 128 and r["trace_out"].tolist() == worst[:128]
    assert (c["lookahead_misses"], c["flushes"], c["pauses"]) == (256, 2, 0)
    obj, steps, _ = s.osscar_init_greedy(7, 0, pkg.OSSCAR_SEARCH_NO_LOOKAHEAD)
    assert sum(steps, []) == worst
    s.close()


@pytest.mark.parametrize("flags", ["", "OSSCAR_SEARCH_LAUNCH_PER_SWAP"])
@pytest.mark.parametrize("p,at", [(128, 0), (128, 5), (128, 6), (128, 7), (2000, 0), (2000, 7), (8256, 7), (16448, 3)])
def test_rows_without_a_score_do_not_disturb_the_picks(p, at, flags):
    """Outside groups whose score is NaN (a NaN in their row of G) are picked by nothing, and every other row is where it would be without
    them: with H = I the swaps exchange the smallest kept |G_i| for the largest outside ones, in order, and no pivot's products are missing."""
    pkg = _pkg()
    m, swaps, k = 8, 30, p // 2
    G = torch.randn(p, m, generator=torch.Generator().manual_seed(p))
    G[k:] *= 2.0
    G[k + at::8] = float("nan")
    s = pkg.Solver(p, m, p, 1, k, swaps, torch.float32, torch.float32, DEV)
    s.osscar_set_quadratic(torch.eye(p).to(DEV), G.to(DEV), 1e6, np.ones(p))
    s.osscar_init_support(pkg.OSSCAR_INIT_GIVEN, range(k))
    r = s.osscar_local_search(swaps, 0.0, getattr(pkg, flags, 0))
    c = s.osscar_get_counters()
    s.close()
    score = (G.double() ** 2).sum(1)
    assert r["trace_out"].tolist() == torch.argsort(score[:k])[:swaps].tolist()
    assert r["trace_in"].tolist() == (k + torch.argsort(-score[k:].nan_to_num(0.0))[:swaps]).tolist()
    assert r["accepted"] == swaps and c["lookahead_misses"] == 0
