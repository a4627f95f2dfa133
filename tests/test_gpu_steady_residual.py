"""The steady solver's linear tolerance: the true residual of a Newton system
ends at or below lin_tol ||R||, also where the recursive residual of the
flexible GMRES gets there before it.

The first step of the study's example starts from zero, so its matrix is the
oracle's Stokes matrix J. ||R - J dx|| is formed from the library's R and dx
in extended precision. Two roundings stand between it and the residual that
the library checks: those of its products in double precision (taken as the
difference of the two precisions here) and those of the entries of J (taken as
the effect of a random relative change of 2^-53); the bar is lin_tol plus both."""
import numpy as np
import pytest

from oracle import fem, mesh, problems, steady
from tests.gpu_common import rel, require_gpu

pytestmark = pytest.mark.gpu


def _product(J, x):
    p = J.data.astype(np.longdouble) * x.astype(np.longdouble)[J.indices]
    y = np.zeros(J.shape[0], dtype=np.longdouble)
    np.add.at(y, np.repeat(np.arange(J.shape[0]), np.diff(J.indptr)), p)
    return y


@pytest.mark.parametrize("n,restart,lin_tol", [(12, 60, 1e-12), (24, 150, 1e-14),
                                               (48, 150, 5e-14), (64, 150, 1e-13)])
def test_true_residual_meets_the_tolerance(n, restart, lin_tol):
    torch, I = require_gpu()
    print(f"steady residual n={n} restart={restart} lin_tol={lin_tol}", flush=True)
    s = I.Steady(I.Mesh.unit_square(n), nu=1.0, restart=restart, lin_tol=lin_tol)
    s.set_builtin(I.IPCS_SOL_STEADY_PAPER_2D)
    st = s.step()
    R, dx = (np.concatenate([u.ravel(), p]) for u, p in map(s.vector, (0, 1)))
    S = fem.Space(*mesh.unit_square(n, n))
    J = steady.SteadyNewton(S, problems.SteadyPaper2D(1.0), 1.0).jacobian()
    exact = R.astype(np.longdouble) - _product(J, dx)
    other = J.copy()
    other.data = J.data * (1 + 2.0 ** -53 * np.random.default_rng(n).uniform(-1, 1, J.nnz))
    scale = np.linalg.norm(R)
    res = float(np.linalg.norm(exact.astype(float))) / scale
    rounding = [float(np.linalg.norm(v)) / scale
                for v in ((R - J @ dx - exact).astype(float), (other - J) @ dx)]
    print(f"  residual {res:.3e} roundings {rounding}", st, flush=True)
    assert res <= lin_tol + sum(rounding)


def test_one_cycle_decides_for_the_inner_solves():
    """Convection dominates on 24^2 squares at nu = 0.002 from the second Newton
    step on: the inner solves give the oracle's fields (1e-10, as the steady
    solver's other tests), after a single multigrid cycle that gains too little.
    A linear iteration cap between one cycle and two shows the cycles: it ends the
    inner solves too, and the count that is left is the multigrid one."""
    torch, I = require_gpu()
    print("steady: fallback to the inner solves", flush=True)
    n, nu, restart, cap = 24, 0.002, 60, 100
    m = I.Mesh.unit_square(n)
    o = steady.SteadyNewton(fem.Space(*mesh.unit_square(n, n)), problems.SteadyPaper2D(nu), nu)
    o.run()
    s = I.Steady(m, nu=nu, restart=restart)
    s.set_builtin(I.IPCS_SOL_STEADY_PAPER_2D)
    st = s.solve()
    errs = [rel(s.velocity()[c], o.U[c]) for c in range(2)] + [rel(s.pressure(), o.P)]
    print(" ", errs, st, flush=True)
    assert st["inner_it"] > 0 and max(errs) <= 1e-10
    s = I.Steady(m, nu=nu, restart=restart, lin_maxit=cap)
    s.set_builtin(I.IPCS_SOL_STEADY_PAPER_2D)
    s.step()
    with pytest.raises(I.IpcsError) as e:
        s.solve()
    print(" ", e.value.stats, flush=True)
    assert e.value.code == I.IPCS_E_NOT_CONVERGED
    assert e.value.stats["lin_it"] == restart
