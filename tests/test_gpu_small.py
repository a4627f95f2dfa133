"""Whole solves in one block per system (small systems) against the oracle: the
sizes where a thread takes one row more or the matrix leaves the registers, rows
of every width, both value types, and the ends of a solve.

Bars: the repository's field bar, 1e-10 at tolerance 1e-13 (mixed form 1e-5, as
its other tests). Iteration counts: sums are formed in another order than in the
per-iteration kernels, which moves a count by a few at most."""
import numpy as np
import pytest

from tests.gpu_common import field_errors, make_pair, require_gpu

pytestmark = pytest.mark.gpu

FIELD_TOL = 1e-10


# velocity rows of 512 and 1024 threads: 1 to 5 each; pressure rows up to 2048
@pytest.mark.parametrize("dim,n,p3,opt", [
    (2, 3, False, {}), (2, 10, False, {}), (2, 11, False, {}), (2, 15, False, {"semi": True}),
    (2, 19, False, {}), (2, 20, False, {"chorin": True}), (2, 22, False, {}), (2, 31, False, {}),
    (2, 44, False, {}), (3, 1, False, {}), (3, 4, False, {"semi": True}), (3, 5, False, {}),
    (3, 9, False, {}), (2, 2, True, {}), (2, 7, True, {"semi": True}), (2, 18, True, {}),
    (3, 2, True, {}), (3, 3, True, {})])
def test_steps_match_the_oracle(dim, n, p3, opt):
    torch, I = require_gpu()
    print(f"one-block solves dim={dim} n={n} p3={p3} {opt}", flush=True)
    S, o, r = make_pair(I, dim, n, "tg" if dim == 2 else "beltrami", 0.01, 0.005, p3=p3, **opt)
    for step in range(2):
        st = r.advance(1)[0]
        o.step()
        errs = field_errors(o, r)
        print(f"  step {step}:", st["it_mom"], st["it_p"], st["it_corr"], errs, flush=True)
        assert max(errs) <= FIELD_TOL


@pytest.mark.parametrize("n", [6, 16, 24, 27])
def test_mixed_steps_match_the_oracle(n):
    torch, I = require_gpu()
    print(f"one-block solves, mixed form n={n}", flush=True)
    # the step the 1e-5 bar was set at (FP32 rounding enters the pressure as 1/dt)
    S, o, r = make_pair(I, 2, n, "tg", 0.01, 0.01, precision=I.IPCS_MIXED, tol_ir=1e-10)
    for _ in range(2):
        st = r.advance(1)[0]
        o.step()
        assert st["ir_outer"] >= 1 and st["res_p"] <= 1e-10, st
        assert max(field_errors(o, r)) <= 1e-5


def test_unstructured_rows():
    """Moved and relabelled vertices: rows of uneven width."""
    torch, I = require_gpu()
    from paper_2605_25403_amd.workloads import jittered_mesh
    for n in (9, 17):
        print(f"one-block solves, jittered mesh n={n}", flush=True)
        S, o, r = make_pair(I, 2, n, "tg", 0.01, 0.005, arrays=jittered_mesh(2, n, 3))
        for _ in range(2):
            r.advance(1)
            o.step()
            assert max(field_errors(o, r)) <= FIELD_TOL


@pytest.mark.parametrize("n", [8, 16, 24])
def test_ends_of_a_solve(n):
    """An iteration cap, a tolerance out of reach, a zero right-hand side and a
    value that is not finite end as they do in the per-iteration kernels."""
    torch, I = require_gpu()
    print(f"one-block solves: ends, n={n}", flush=True)

    def run(**kw):
        r = I.Run(I.Mesh.unit_square(n), I.ipcs_params_default(nu=0.01, dt=0.01, **kw))
        r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (np.pi,))
        return r

    for kw, solve, codes in ((dict(maxit=2), 1, (I.IPCS_E_NOT_CONVERGED,)),
                             (dict(tol_p=1e-17), 2, (I.IPCS_E_NOT_CONVERGED, I.IPCS_E_BREAKDOWN))):
        r = run(**kw)
        U0 = r.velocity()
        with pytest.raises(I.IpcsError) as e:
            r.advance(1)
        assert e.value.code in codes and e.value.stats[0].failed_solve == solve
        np.testing.assert_array_equal(r.velocity(), U0)
    r = run(maxit=2)
    try:
        r.advance(1)
    except I.IpcsError as e:
        assert max(e.stats[0].it_mom) == 2
    # rest: every solve of the step has a zero right-hand side
    r = I.Run(I.Mesh.unit_square(n), I.ipcs_params_default(nu=0.01, dt=0.01))
    st = r.advance(1)[0]
    assert st["status"] == 0 and st["it_p"] == 0 and not np.any(r.velocity())
    r = run()
    U = r.velocity()
    U[0, U.shape[1] // 2] = np.nan
    r.set_state(U, r.pressure(), 0.0)
    with pytest.raises(I.IpcsError) as e:
        r.advance(1)
    assert e.value.code == I.IPCS_E_NONFINITE
