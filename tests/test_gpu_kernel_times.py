"""The timing hook sees the pressure multigrid and the one-block solves: every
launch of a masked kernel is counted, and the step's result keeps its bits."""
import numpy as np
import pytest

from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu

STEPS = 2


def _run(I, n, dim=2, pair=0, prec=0, timed=True):
    m = I.Mesh.unit_square(n, pair=pair) if dim == 2 else I.Mesh.unit_cube(n, pair=pair)
    r = I.Run(m, I.ipcs_params_default(nu=0.003, dt=1e-3, precision=prec))
    r.set_builtin(*((I.IPCS_SOL_TAYLOR_GREEN_2D, (4 * np.pi,)) if dim == 2 else
                    (I.IPCS_SOL_BELTRAMI_3D, ())))
    if timed:
        r.kernel_timing((1 << I.IPCS_NKERNEL) - 1)
    st = r.advance(STEPS)
    ms, cnt = r.kernel_times()
    print(f"  {dim}D n={n} pair={pair} prec={prec}", st[-1]["it_p"], cnt, flush=True)
    assert all((t > 0.0) == (k > 0) for t, k in zip(ms, cnt))
    return st, ms, cnt, r.velocity(), r.pressure()


@pytest.mark.parametrize("dim,n,pair,prec,with_w,products", [
    (2, 64, 0, 0, True, 3), (2, 64, 0, 1, True, 3), (2, 300, 0, 0, False, 5),
    (2, 300, 0, 1, False, 5), (3, 14, 0, 0, True, 3)])
def test_multigrid_kernels(dim, n, pair, prec, with_w, products):
    torch, I = require_gpu()
    print("kernel times: multigrid", flush=True)
    st, _, cnt, U, P = _run(I, n, dim, pair, prec)
    its = sum(s["it_p"] for s in st)
    assert 0 < its < 60 * STEPS * max(1, st[0]["ir_outer"])
    assert cnt[I.IPCS_KERNEL_MG_UPDATE_P] >= its
    assert cnt[I.IPCS_KERNEL_MG_PRODUCT_P] == products * cnt[I.IPCS_KERNEL_MG_UPDATE_P]
    assert cnt[I.IPCS_KERNEL_PCG_SPMV_P] == (0 if with_w else cnt[I.IPCS_KERNEL_MG_UPDATE_P])
    assert cnt[I.IPCS_KERNEL_PCG_FUSED_P] == 0
    _, _, none, V, Q = _run(I, n, dim, pair, prec, timed=False)
    assert not any(none)
    np.testing.assert_array_equal(U, V)
    np.testing.assert_array_equal(P, Q)


def test_one_block_solves():
    torch, I = require_gpu()
    print("kernel times: one block", flush=True)
    _, _, cnt, U, P = _run(I, 16)
    for k in (I.IPCS_KERNEL_ONE_BLOCK_MOM, I.IPCS_KERNEL_ONE_BLOCK_P, I.IPCS_KERNEL_ONE_BLOCK_CORR):
        assert cnt[k] == STEPS
    assert cnt[I.IPCS_KERNEL_BICG_SPMV] == cnt[I.IPCS_KERNEL_PCG_FUSED_P] == 0
    _, _, _, V, Q = _run(I, 16, timed=False)
    np.testing.assert_array_equal(U, V)
    np.testing.assert_array_equal(P, Q)


def test_kernels_without_a_launcher_of_their_own_and_shorter_outputs():
    torch, I = require_gpu()
    import ctypes as C
    print("kernel times: bounds", flush=True)
    r = I.Run(I.Mesh.unit_square(12), I.ipcs_params_default(poisson_part_rows=-1))
    r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (np.pi,))
    r.advance(1)
    U = r.velocity()
    for k in (-1, I.IPCS_KERNEL_MG_PRODUCT_P, I.IPCS_KERNEL_ONE_BLOCK_CORR, I.IPCS_NKERNEL):
        with pytest.raises(I.IpcsError) as e:
            I.ipcs_profile_kernel(r.h, k, 2)
        assert e.value.code == I.IPCS_E_INVALID
    r.advance(1)      # the solver's states are as they were
    np.testing.assert_equal(np.isfinite(r.velocity()).all() and (r.velocity() != U).any(), True)
    ms, cnt = (C.c_double * 12)(*[-1.0] * 12), (C.c_int64 * 12)(*[-1] * 12)
    assert I.lib.ipcs_kernel_times(r.h, ms, cnt, 11) == I.IPCS_OK      # as many as there were
    assert ms[10] == 0.0 and ms[11] == -1.0 and cnt[11] == -1
    assert I.lib.ipcs_kernel_times(r.h, ms, cnt, 10) == I.IPCS_E_INVALID


@pytest.mark.parametrize("maxit,one_block", [(100000, True), (100001, False)])
def test_no_single_launch_without_a_bound(maxit, one_block):
    """A one-block solve cannot be ended by the host: past an iteration cap of
    100000 small systems take the polled forms, to the same fields (1e-9: both
    meet the default tolerance of 1e-12)."""
    torch, I = require_gpu()
    print(f"kernel times: maxit {maxit}", flush=True)
    m, out = I.Mesh.unit_square(16), []
    for cap in (20000, maxit):
        r = I.Run(m, I.ipcs_params_default(nu=0.01, dt=1e-3, maxit=cap))
        r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (np.pi,))
        r.kernel_timing((1 << I.IPCS_NKERNEL) - 1)
        r.advance(STEPS)
        cnt = r.kernel_times()[1]
        out.append((r.velocity(), r.pressure()))
    print(" ", cnt, flush=True)
    for k in (I.IPCS_KERNEL_ONE_BLOCK_MOM, I.IPCS_KERNEL_ONE_BLOCK_P, I.IPCS_KERNEL_ONE_BLOCK_CORR):
        assert cnt[k] == (STEPS if one_block else 0)
    for a, b in zip(*out):
        assert np.linalg.norm(a - b) <= 1e-9 * np.linalg.norm(a)
