"""Left-looking LU (stmg_batched_lu in FP64 and FP32, patch systems) on special
matrices and batches: NaN entries, against the persistent right-looking kernel
(explicit launch parameters); tiny complex pivots; matrices beyond the
left-looking kernel's limit beside others (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def factor(A, dt, config=None):
    from paper_2602_13841_amd import stmg
    m = len(A)
    F = torch.tensor(A, dtype=dt, device="cuda")
    piv = torch.full((m,), -1, dtype=torch.int32, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    stmg.batched_lu(F, [0], [m], piv, [0], info, config=config)
    return F.cpu().numpy(), piv.cpu().numpy(), int(info.item())


@pytest.mark.parametrize("m", [3, 40, 130, 300, 600])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_nan_pivots(prec, m):
    """NaN is below every number in the pivot search: a zero is taken before
    it, and a column without a number keeps its row and is no zero pivot."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt = torch.float64 if prec == "f64" else torch.float32
    rng = np.random.Generator(np.random.PCG64(83))
    right_looking = (1, [16, 16, 16, 8, 4], 256)
    # [NaN, 0, 0, ...] and zeros elsewhere: the first zero, in every column
    A = np.zeros((m, m))
    A[0, 0] = np.nan
    F, piv, info = factor(A, dt)
    _, ref, ref_info = factor(A, dt, right_looking)
    assert piv[0] == 1 and info == m - 1
    assert np.array_equal(piv, ref) and info == ref_info
    # no number in column 0, hence in none
    A = rng.uniform(-1, 1, (m, m))
    A[:, 0] = np.nan
    F, piv, info = factor(A, dt)
    _, ref, ref_info = factor(A, dt, right_looking)
    assert np.array_equal(piv, np.arange(m)) and np.array_equal(piv, ref) and info == ref_info == 0
    # one NaN: its row is the last pivot, the others are factored without it
    A = rng.uniform(-1, 1, (m, m))
    A[0, 0], A[2, 0] = np.nan, 8.0
    F, piv, info = factor(A, dt)
    assert piv[0] == 2 and info == 0
    assert np.all(np.isfinite(F[:-1])) and np.all(np.isnan(F[-1]))


@pytest.mark.parametrize("d,n,r,nu,tau", [(3, (2, 1, 1), 2, 3e-19, 1e19), (2, (2, 2), 3, 3e-20, 1e20)],
                         ids=["3d_r2", "2d_r3"])
def test_small_complex_pivots(d, n, r, nu, tau):
    """Almost no viscosity and a long slab without Dirichlet faces: FP32 patch
    systems whose velocity pivots (1e-20 and below 5.4e-20) have a squared
    modulus with a reciprocal beyond the FP32 range.  The pivots' own
    reciprocals are finite, and so is a sweep."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13841_amd import stmg
    ctx = stmg.Context(d, n, r, 1, nu, tau, dirichlet_faces=0, prec_mg=stmg.STMG_F32, fgmres_maxit=1)
    ctx.smoother_rebuild(torch.zeros(ctx.N, dtype=torch.float64, device="cuda"))
    b = 1e-10 * torch.rand(ctx.N, generator=torch.Generator().manual_seed(1), dtype=torch.float64)
    x = torch.zeros(ctx.N, dtype=torch.float32, device="cuda")
    ctx.vanka_smooth(0, b.to("cuda", torch.float32), x)
    assert bool(torch.isfinite(x).all()) and bool(x.any())


@pytest.mark.parametrize("prec,big", [("f64", 1281), ("f32", 1857)])
def test_oversized_beside_others(prec, big):
    """Matrices above the left-looking limit run beside the rest of the batch:
    each is factored as it is alone (bit for bit), with the fixed staging too,
    and on a stream that still holds earlier work."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13841_amd import stmg
    dt = torch.float64 if prec == "f64" else torch.float32
    rng = np.random.Generator(np.random.PCG64(84))
    sizes = [40, big, 395, 600, 17]
    mats = [rng.uniform(-1, 1, (m, m)) for m in sizes]
    want = [factor(A, dt) for A in mats]
    a_off = np.concatenate([[0], np.cumsum(np.square(sizes))[:-1]])
    p_off = np.concatenate([[0], np.cumsum(sizes)[:-1]])
    flat = torch.tensor(np.concatenate([A.ravel() for A in mats]), dtype=dt, device="cuda")
    stream = torch.cuda.Stream()
    for noalloc in (False, True):
        piv = torch.full((sum(sizes),), -1, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            F = torch.zeros_like(flat)
            for _ in range(50):   # the matrices arrive with the last of these copies
                F.copy_(flat)
            stmg.batched_lu(F, a_off, sizes, piv, p_off, noalloc=noalloc)
        F, piv = F.cpu().numpy(), piv.cpu().numpy()
        for m, a, p, (G, q, _) in zip(sizes, a_off, p_off, want):
            assert np.array_equal(F[a:a + m * m].reshape(m, m), G) and np.array_equal(piv[p:p + m], q)


@pytest.mark.parametrize("m", [20, 33, 47, 64, 130, 300, 600, 700])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_nonfinite_entries_stay_where_elimination_puts_them(prec, m):
    """NaN and infinities above the diagonal: the factors are not finite
    exactly where the elimination l_ik u_kj reaches, and agree elsewhere with
    the factors of the matrix without them.  (Dominant diagonal: no
    interchanges.)"""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt, u = (torch.float64, 2.0 ** -53) if prec == "f64" else (torch.float32, 2.0 ** -24)
    rng = np.random.Generator(np.random.PCG64(85))
    A = rng.uniform(0.5, 1, (m, m)) + 4 * m * np.eye(m)
    clean, _, _ = factor(A, dt)
    for bad in ([(m - 3, m - 1)], [(m // 2, m - 2), (m - 2, m - 1)], [(1, m - 5), (2, m - 1)], [(m - 20, m - 4)]):
        B, hit = A.copy(), np.zeros((m, m), dtype=bool)
        for (i, j), v in zip(bad, (np.nan, -np.inf)):
            B[i, j], hit[i, j] = v, True
        for k in range(m):
            hit[k + 1:, k] |= hit[k, k]
            hit[k + 1:, k + 1:] |= hit[k + 1:, k, None] | hit[None, k, k + 1:]
        for config in (None, (1, [16, 16, 16, 8, 4], 256)):
            F, piv, info = factor(B, dt, config)
            assert info == 0 and np.array_equal(piv, np.arange(m))
            assert np.array_equal(~np.isfinite(F), hit), (bad, config)
            ok = ~hit
            assert np.all(np.abs(F[ok] - clean[ok]) <= 8 * m * u * np.abs(clean[ok]) + 8 * m * u)
