"""Kernels against plain float64 references at the sizes where their tilings can go wrong: edges of tiles and stages,
remainders, the smallest and largest of each branch's range."""
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
