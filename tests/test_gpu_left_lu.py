"""Left-looking batched LU (stmg_batched_lu in FP64 and FP32) at the edges of
its tiles, panels and size classes, against LAPACK's definition (GPU).

Checked on each matrix: the interchanges are those of partial pivoting (every
multiplier at most 1), and P A = L U to the backward error bound of Gaussian
elimination, |P A - L U| <= gamma_m |L| |U| entrywise, with gamma_m = m u / (1 -
m u) (blocked products and inverses of 16-column unit triangles included: a
factor of 4 covers them).  Ties go to the first row, as LAPACK's idamax."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# remainders of 4, 8, 16 and 32 columns, both sides of 128, 256, 512 and 1280
# rows, the largest sizes of each precision and (FP64 1281, FP32 1857) the first
# that the persistent kernel takes
SIZES = {"f64": [1, 2, 7, 16, 17, 31, 33, 85, 128, 129, 255, 257, 395, 512, 513, 790, 1279, 1280, 1281],
         "f32": [1, 3, 16, 32, 41, 64, 127, 129, 202, 256, 511, 513, 606, 1185, 1281, 1856, 1857]}


def factor(mats, dt, noalloc=False):
    from paper_2602_13841_amd import stmg
    sizes = np.array([len(M) for M in mats], dtype=np.int32)
    a_off = np.concatenate([[0], np.cumsum(sizes.astype(np.int64) ** 2)[:-1]])
    p_off = np.concatenate([[0], np.cumsum(sizes.astype(np.int64))[:-1]])
    A = torch.tensor(np.concatenate([M.ravel() for M in mats]), dtype=dt, device="cuda")
    piv = torch.full((int(sizes.sum()),), -1, dtype=torch.int32, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    stmg.batched_lu(A, a_off, sizes, piv, p_off, info, noalloc=noalloc)
    A, piv = A.double().cpu().numpy(), piv.cpu().numpy()
    return [(A[o:o + m * m].reshape(m, m), piv[p:p + m]) for m, o, p in zip(sizes, a_off, p_off)], int(info.item())


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_backward_error(prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt, u = (torch.float64, 2.0 ** -53) if prec == "f64" else (torch.float32, 2.0 ** -24)
    rng = np.random.Generator(np.random.PCG64(81))
    mats = []
    for m in SIZES[prec]:
        M = rng.uniform(-1, 1, (m, m)) * 10.0 ** rng.uniform(-1, 1, (m, 1))   # rows of different size: real pivoting
        mats.append(M.astype(np.float32).astype(np.float64) if prec == "f32" else M)
    for noalloc in (False, True):
        out, info = factor(mats, dt, noalloc)
        assert info == 0
        for M, (F, piv) in zip(mats, out):
            m = len(M)
            assert np.all(piv >= np.arange(m)) and np.all(piv < m)
            PA = M.copy()
            for j, p in enumerate(piv):
                PA[[j, p]] = PA[[p, j]]
            L, U = np.tril(F, -1) + np.eye(m), np.triu(F)
            assert np.max(np.abs(L)) <= 1.0 + 4 * u
            g = m * u / (1 - m * u)
            # one more rounding of the FP32 factors read back is within the bound
            assert np.all(np.abs(PA - L @ U) <= 4 * g * (np.abs(L) @ np.abs(U)) + 1e-300), m


def test_ties_and_zero_pivots():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # +-1 entries: many equal candidates; the first of them is taken
    rng = np.random.Generator(np.random.PCG64(82))
    mats = [rng.choice([-1.0, 1.0], (m, m)) for m in (5, 40, 130, 300, 600)]
    for dt in (torch.float64, torch.float32):
        out, _ = factor(mats, dt)
        for M, (F, piv) in zip(mats, out):
            assert piv[0] == 0   # every entry of the first column has modulus 1
        # a zero matrix: every pivot is zero, counted, no interchange
        out, info = factor([np.zeros((35, 35)), np.eye(20)], dt)
        assert info == 35 and np.array_equal(out[0][1], np.arange(35)) and np.array_equal(out[1][1], np.arange(20))
        assert np.array_equal(out[1][0], np.eye(20))


@pytest.mark.parametrize("m", [1, 20, 35, 64, 100, 130, 257, 513])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_negative_zero_pivots(prec, m):
    """A column of -0 is a zero pivot like one of +0: counted, no interchange,
    and the other columns factored as usual."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dt = torch.float64 if prec == "f64" else torch.float32
    out, info = factor([-np.zeros((m, m))], dt)
    assert info == m and np.array_equal(out[0][1], np.arange(m)) and not out[0][0].any()
    # a diagonal matrix (exact in both precisions), its last and a middle
    # column -0, negated zeros everywhere off the diagonal
    M = -np.zeros((m, m))
    d = 1.0 + np.arange(m) % 5
    d[[m // 2, m - 1]] = -0.0
    np.fill_diagonal(M, -d)
    for mats in ([M], [M, -M, np.eye(40)]):   # alone and beside others
        out, info = factor(mats, dt)
        assert info == len({m // 2, m - 1}) * min(len(mats), 2)
        for A, (F, piv) in zip(mats, out):
            assert np.array_equal(piv, np.arange(len(A))) and np.array_equal(F, A)
