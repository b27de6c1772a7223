"""Left-looking patch LU and sweeps of the time-decoupled systems on every
system size (21 to 395 unknowns, real and complex), against the full
space-time patch factorization (GPU).

Bars: those of the time-decoupled splitting on the other cases
(test_time_decoupled_equals_full_patch): 1e-10 in FP64, 1e-4 in FP32."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2602_13841_amd import inputs as I  # noqa: E402

pytestmark = pytest.mark.gpu

# dimension, degree, k: k = 0 has one real system, 1 one complex, 2 both
CASES = [(d, r, k) for d in (2, 3) for r in (1, 2, 3) for k in (0, 1, 2)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("d,r,k", CASES, ids=[f"{d}d_r{r}_k{k}" for d, r, k in CASES])
def test_sweep_equals_full_patch(d, r, k, prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13841_amd import stmg
    p, dt, tol = (stmg.STMG_F64, torch.float64, 1e-10) if prec == "f64" else (stmg.STMG_F32, torch.float32, 1e-4)
    n = (4,) * d if r == 1 else (2, 4, 2)[:d]
    vert = I.perturbed_vertices(d, n, 0.2, 71)
    out = []
    for td in (1, 0):
        ctx = stmg.Context(d, n, r, k, 0.02, 0.05, vertices=vert, prec_mg=p, vanka_time_decoupled=td, max_levels=2)
        for seed in (72, 73):   # two states in the same buffers
            ctx.smoother_rebuild(torch.tensor(I.uniform(ctx.N, seed), device="cuda"))
        x = torch.tensor(0.1 * I.uniform(ctx.N, 74), dtype=dt, device="cuda")
        ctx.vanka_smooth(0, torch.tensor(I.uniform(ctx.N, 75), dtype=dt, device="cuda"), x)
        out.append(x.double().cpu().numpy())
        ctx.close()
    assert np.max(np.abs(out[0] - out[1])) <= tol * np.max(np.abs(out[1]))
