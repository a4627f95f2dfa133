"""A pressure solve that multigrid does not bring to the tolerance: the Jacobi
form repeats it. A tolerance out of reach (1e-16) ends both, with the Jacobi
form's status and the state of the last completed step."""
import numpy as np
import pytest

from tests.gpu_common import require_gpu

pytestmark = pytest.mark.gpu


def _run(I, torch, rows=0, prec=None, stream=None, n=60):
    p = I.ipcs_params_default(nu=0.01, dt=1e-3, tol_p=1e-16, poisson_part_rows=rows,
                              precision=I.IPCS_FP64 if prec is None else prec)
    if prec == I.IPCS_MIXED:
        p.tol_ir = 1e-16
    r = I.Run(I.Mesh.unit_square(n), p, stream=stream)
    r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (np.pi,))
    return r


def _failed(I, r):
    with pytest.raises(I.IpcsError) as e:
        r.advance(1)
    assert e.value.stats[0].failed_solve == 2
    return e.value.code, e.value.stats[0].it_p, e.value.stats[0].checks_p


def test_the_iterations_of_both_forms_are_counted():
    torch, I = require_gpu()
    print("failed multigrid solve: iterations", flush=True)
    named = _failed(I, _run(I, torch, rows=384))
    both = _failed(I, _run(I, torch))
    print(" ", named, both, flush=True)
    assert both[0] == named[0] and both[1] > named[1] and both[2] >= named[2]
    # a batch counts as a run alone does, in both precisions
    for prec in (I.IPCS_FP64, I.IPCS_MIXED):
        alone = _failed(I, _run(I, torch, prec=prec))
        for step in (I.ipcs_batch_step, I.ipcs_batch_step_noalloc):
            s = torch.cuda.Stream()
            r = _run(I, torch, prec=prec, stream=s)
            rc, st = step([r.h], s.cuda_stream)
            print(" ", prec, alone, rc, st[0]["it_p"], st[0]["checks_p"], flush=True)
            assert (rc, st[0]["it_p"], st[0]["checks_p"]) == alone


def test_the_next_solves_go_to_the_jacobi_form_at_once():
    torch, I = require_gpu()
    print("failed multigrid solve: remembered", flush=True)
    named = _failed(I, _run(I, torch, rows=384))
    r = _run(I, torch)
    U0 = r.velocity()
    first, second = _failed(I, r), _failed(I, r)
    r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (np.pi,))   # a new state tries again
    third = _failed(I, r)
    I.ipcs_set_time_step(r.h, 1e-3)                       # and so do new parameters
    fourth = _failed(I, r)
    print(" ", named, first, second, third, fourth, flush=True)
    assert second == named and first == third == fourth and first[1] > second[1]
    np.testing.assert_array_equal(r.velocity(), U0)
    s = torch.cuda.Stream()
    b = _run(I, torch, stream=s)
    its = [I.ipcs_batch_step([b.h], s.cuda_stream)[1][0]["it_p"] for _ in range(2)]
    assert its == [first[1], second[1]]


def test_a_failed_solve_is_no_guide_for_the_next_ones_length():
    """A solve of known length launches that many iterations before it looks at
    the status. After a failed solve (more than the 18 iterations of a first one)
    and a new state, a solve that is done at its start (everything is zero)
    launches 19."""
    torch, I = require_gpu()
    print("failed multigrid solve: length", flush=True)
    r = I.Run(I.Mesh.unit_square(60), I.ipcs_params_default(nu=0.01, dt=1e-3, tol_p=1e-16))
    x = np.random.default_rng(1).standard_normal((2, r.n2))
    r.set_state(x, np.zeros(r.n1), 0.0)
    r.kernel_timing(1 << I.IPCS_KERNEL_MG_UPDATE_P)
    _failed(I, r)
    first = r.kernel_times()[1][I.IPCS_KERNEL_MG_UPDATE_P]
    r.set_state(0 * x, np.zeros(r.n1), 0.0)
    r.kernel_timing(1 << I.IPCS_KERNEL_MG_UPDATE_P)
    st = r.advance(1)[0]
    print(" ", first, r.kernel_times()[1][I.IPCS_KERNEL_MG_UPDATE_P], st, flush=True)
    assert st["it_p"] == 0 and first > 19
    assert r.kernel_times()[1][I.IPCS_KERNEL_MG_UPDATE_P] == 19
