"""3D volume pass of the Jacobian and the residual at every degree, number of
time nodes and quadrature (GPU).

Each degree has its own split of the row stage (r = 3: one thread per row and
half of its points while two halves fit the workgroup; below: one thread per
row and component), the number of time nodes sets the workgroup and the LDS
layout.  Bar as for the other operator tests: FP64 to 1e-12 of the oracle's
largest value, FP32 to 1e-5.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2602_13841_amd import inputs as I  # noqa: E402

pytestmark = pytest.mark.gpu


def dev(a, dtype=torch.float64):
    return torch.tensor(np.asarray(a), dtype=dtype, device="cuda")


def rel(a, b):
    return float(np.max(np.abs(a.double().cpu().numpy() - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("mapped", [False, True], ids=["affine", "mapped"])
@pytest.mark.parametrize("k", [0, 1, 2, 3])
@pytest.mark.parametrize("r,nq", [(1, 3), (1, 4), (2, 4), (2, 5), (3, 5), (3, 7)])
def test_volume_pass(r, nq, k, mapped):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13841_amd import stmg
    n = (2, 1, 1) if mapped else (1, 2, 1)
    vert = I.perturbed_vertices(3, n, 0.2, 7 + r) if mapped else None
    prob = oracle.Problem(dim=3, n=n, r=r, k=k, nu=0.02, tau=0.1, vertices=vert, dirichlet_mask=None, nq=nq)
    slab = oracle.Slab(prob)
    ctx = stmg.Context(3, n, r, k, 0.02, 0.1, vertices=vert, dirichlet_faces=prob.dirichlet_mask, n_q=nq)
    U, X = I.uniform(slab.N, 11), I.uniform(slab.N, 12)
    want = slab.jacobian(U) @ X
    assert rel(ctx.jacobian_vmult(dev(U), dev(X)), want) < 1e-12
    assert rel(ctx.jacobian_vmult(dev(U, torch.float32), dev(X, torch.float32)), want) < 1e-5
    rhs, vprev = I.uniform(slab.N, 13), I.uniform(slab.Nv, 14)
    ctx.set_slab_data(dev(rhs), dev(vprev))
    assert rel(ctx.residual(dev(U)), slab.residual(U, rhs, vprev)) < 1e-12
    ctx.set_slab_data(None, None)
    assert rel(ctx.residual(dev(U)), slab.residual(U)) < 1e-12


# the FP32 Jacobian's rule on the number of cells (256 CUs): r = 2 from 1025 on,
# r = 3 outside 641 ... 896; interior cells on both sides of each line
@pytest.mark.parametrize("r,k,n,mapped", [(2, 2, (8, 8, 16), False), (2, 2, (8, 10, 14), False),
                                          (3, 1, (8, 8, 10), False), (3, 1, (6, 10, 12), True),
                                          (3, 1, (8, 8, 14), False), (3, 1, (8, 10, 12), True)],
                         ids=["r2_1024", "r2_1120", "r3_640", "r3_720_mapped", "r3_896", "r3_960_mapped"])
def test_volume_pass_many_cells(r, k, n, mapped):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13841_amd import stmg
    vert = I.perturbed_vertices(3, n, 0.2, 7 + r) if mapped else None
    slab = oracle.Slab(oracle.Problem(dim=3, n=n, r=r, k=k, nu=0.02, tau=0.1, vertices=vert))
    ctx = stmg.Context(3, n, r, k, 0.02, 0.1, vertices=vert, fgmres_maxit=1)
    U, X = I.uniform(slab.N, 11), I.uniform(slab.N, 12)
    # sampled rows of the oracle's element action; FP32 against FP64 everywhere
    rng = np.random.Generator(np.random.PCG64(15))
    rows = np.sort(np.concatenate([rng.choice(slab.nt * slab.Nv, 30, replace=False),
                                   slab.nt * slab.Nv + rng.choice(slab.nt * slab.Np, 10, replace=False)]))
    want = slab.vmult_rows(U, X, rows)
    got = ctx.jacobian_vmult(dev(U), dev(X)).cpu().numpy()
    scale = np.max(np.abs(got))
    assert np.max(np.abs(got[rows] - want)) < 1e-12 * scale
    assert rel(ctx.jacobian_vmult(dev(U, torch.float32), dev(X, torch.float32)), got) < 1e-5
