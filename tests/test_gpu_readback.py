"""Fields read back through the pinned halves: what was set comes back, value by
value, for fields below one half (524288 values), just below and above it, over
several chunks (a chunk then holds the end of one component and the start of
the next), and pressures of more than one chunk."""
import numpy as np
import pytest

from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n", [(2, 1), (2, 16), (2, 255), (2, 256), (2, 384), (2, 725), (3, 30)])
def test_state_comes_back(dim, n):
    torch, I = require_gpu()
    print(f"read back dim={dim} n={n}", flush=True)
    m = I.Mesh.unit_square(n) if dim == 2 else I.Mesh.unit_cube(n)
    r = I.Run(m, I.ipcs_params_default(nu=0.01, dt=1e-3))
    rng = np.random.default_rng(n)
    for _ in range(2):
        u, p = rng.standard_normal((dim, r.n2)), rng.standard_normal(r.n1)
        r.set_state(u, p, 0.0)
        assert np.array_equal(r.velocity(), u)
        assert np.array_equal(r.pressure(), p)
