"""The pressure solve's true residual on both of its forms: after short momentum
solves (multigrid) and after long ones (Jacobi). ||r - Kp dP|| <= tol ||r|| in the
library's own Kp and right-hand side, a tenth more for the rounding of the product
here (some 1e-14 to 2e-13 of ||r|| at these sizes, against a tolerance of 1e-11).
The fields of a step agree with those of the Jacobi form named by the parameters
to what the tolerance leaves of the increment, 1e-9."""
import numpy as np
import pytest

from tests.gpu_common import rel, require_gpu, residual

pytestmark = pytest.mark.gpu

TOL = 1e-11


@pytest.mark.parametrize("dim,n,pair,nu,long", [
    (2, 60, 0, 0.003, False), (2, 60, 0, 1.0, True), (2, 160, 0, 0.003, False),
    (2, 160, 0, 0.3, True), (2, 31, 1, 0.003, False), (2, 31, 1, 1.0, True),
    (3, 14, 0, 0.01, False), (3, 14, 0, 20.0, True)])
def test_either_form_meets_the_tolerance(dim, n, pair, nu, long):
    torch, I = require_gpu()
    print(f"pressure residual dim={dim} n={n} pair={pair} nu={nu}", flush=True)
    m = I.Mesh.unit_square(n, pair=pair) if dim == 2 else I.Mesh.unit_cube(n, pair=pair)
    out = []
    for rows in (0, 384):
        r = I.Run(m, I.ipcs_params_default(nu=nu, dt=1e-3, tol_p=TOL, poisson_part_rows=rows))
        if dim == 2:
            r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (4 * np.pi,))
        else:
            r.set_builtin(I.IPCS_SOL_BELTRAMI_3D, ())
        r.phase(I.IPCS_PHASE_ASM)
        mom = max(r.phase(I.IPCS_PHASE_MOMENTUM)["it_mom"][:dim])
        st = r.phase(I.IPCS_PHASE_PRESSURE)
        res = residual(r.matrix(I.IPCS_MAT_KP), r.field(I.IPCS_FIELD_DP),
                       r.field(I.IPCS_FIELD_RHS_P))
        r.phase(I.IPCS_PHASE_CORRECTION)
        print(f"  rows {rows}: momentum {mom}, pressure {st['it_p']}, residual {res:.2e}", flush=True)
        assert res <= 1.1 * TOL
        out.append((mom, r.velocity(), r.pressure()))
    (mom, U, P), (_, V, Q) = out
    assert (mom > 40) == long
    assert rel(U, V) <= 1e-9 and rel(P, Q) <= 1e-9
