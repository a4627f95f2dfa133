"""Multigrid CG on a mesh whose last product is past 8192 blocks of the usual
size (1024^2 squares): the blocks grow, the solve keeps its form and meets its
tolerance in the library's own matrix."""
import numpy as np
import pytest

from tests.gpu_common import require_gpu, residual

pytestmark = pytest.mark.gpu


def test_past_the_usual_block_count():
    torch, I = require_gpu()
    print("multigrid CG n=1024", flush=True)
    tol = 1e-10     # the rounding of r - Kp dP alone is some 1e-11 of r here
    r = I.Run(I.Mesh.unit_square(1024), I.ipcs_params_default(nu=1e-4, dt=1e-3, tol_p=tol))
    r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (4 * np.pi,))
    r.phase(I.IPCS_PHASE_ASM)
    mom = max(r.phase(I.IPCS_PHASE_MOMENTUM)["it_mom"][:2])
    st = r.phase(I.IPCS_PHASE_PRESSURE)
    res = residual(r.matrix(I.IPCS_MAT_KP), r.field(I.IPCS_FIELD_DP),
                   r.field(I.IPCS_FIELD_RHS_P))
    print(mom, st, res, flush=True)
    assert st["it_p"] < 60 and res <= 1.2 * tol
