"""The steady solver's two preconditioners against the oracle's Newton iteration:
the multigrid one where viscosity dominates (no inner iterations), the inner
Jacobi solves after a multigrid cycle that gains too little, and the meshes
between (no vertex off the boundary, a coarsest level, both product forms).

Bars: those of the steady solver's other tests, 1e-10 for both fields (both
sides iterate to relative changes below 1e-10 on systems solved to 1e-12)."""
import numpy as np
import pytest

from oracle import fem, mesh, problems, steady
from tests.gpu_common import rel, require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nu,inner", [(2, 1.0, False), (5, 0.5, False),
                                        (13, 1.0, False), (14, 0.05, False), (21, 2.0, False),
                                        (10, 0.001, None)])
def test_steady_example_matches_the_oracle(n, nu, inner):
    torch, I = require_gpu()
    print(f"steady multigrid n={n} nu={nu}", flush=True)
    S = fem.Space(*mesh.unit_square(n, n))
    o = steady.SteadyNewton(S, problems.SteadyPaper2D(nu), nu)
    o.run()
    s = I.Steady(I.Mesh.unit_square(n), nu=nu)
    for again in range(2):      # the second solve starts anew
        s.set_builtin(I.IPCS_SOL_STEADY_PAPER_2D)
        st = s.solve()
        U, P = s.velocity(), s.pressure()
        eu, ep = max(rel(U[c], o.U[c]) for c in range(2)), rel(P, o.P)
        print(f"  u {eu:.2e} p {ep:.2e}", st, flush=True)
        assert eu <= 1e-10 and ep <= 1e-10
        if inner is not None:
            assert (st["inner_it"] > 0) == inner, st


@pytest.mark.parametrize("dim,n,nu", [(2, 12, 0.005), (3, 3, 0.3), (3, 4, 1.0)])
def test_polynomial_state(dim, n, nu):
    torch, I = require_gpu()
    print(f"steady multigrid polynomial dim={dim} n={n} nu={nu}", flush=True)
    m = I.Mesh.unit_square(n) if dim == 2 else I.Mesh.unit_cube(n)
    s = I.Steady(m, nu=nu)
    s.set_builtin(I.IPCS_SOL_POLY_STEADY_2D if dim == 2 else I.IPCS_SOL_POLY_STEADY_3D)
    st = s.solve()
    S = fem.Space(*(mesh.unit_square(n, n) if dim == 2 else mesh.unit_cube(n, n, n)))
    pb = problems.PolySteady2D(nu) if dim == 2 else problems.PolySteady3D(nu)
    print(st, flush=True)
    assert np.abs(s.velocity() - pb.u(S.xu, 0.0).T).max() <= 1e-11
    assert np.abs(s.pressure() - pb.p(S.xp, 0.0)).max() <= 1e-10


def test_long_vectors_are_orthonormalized_by_the_general_kernels():
    """More rows than the five-launch Gram-Schmidt takes (131072), and the
    largest mesh below: the polynomial state to ten times the relative change
    at which the iteration stops (1e-10)."""
    torch, I = require_gpu()
    for n in (120, 122):
        print(f"steady multigrid n={n}", flush=True)
        s = I.Steady(I.Mesh.unit_square(n), nu=1.0)
        s.set_builtin(I.IPCS_SOL_POLY_STEADY_2D)
        st = s.solve()
        S = fem.Space(*mesh.unit_square(n, n))
        assert (2 * len(S.xu) + len(S.xp) > 131072) == (n == 122)
        pb = problems.PolySteady2D(1.0)
        u, p = pb.u(S.xu, 0.0).T, pb.p(S.xp, 0.0)
        print(rel(s.velocity(), u), rel(s.pressure(), p), st, flush=True)
        assert rel(s.velocity(), u) <= 1e-9 and rel(s.pressure(), p) <= 1e-9
