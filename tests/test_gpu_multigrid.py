"""The multigrid-preconditioned CG of the pressure Poisson system, the default
above 2560 pressure rows after a momentum solve of at most 40 iterations (after
a longer one the Jacobi form), against the oracle and against the Jacobi form
of the same call (poisson_part_rows = 384).

Bars. Either form ends with ||r - Kp dP|| <= tol ||r|| confirmed on the true
residual: dP in the oracle's Kp is held to that, with a tenth more for the
rounding of the oracle's own product. Fields against the oracle take the
repository's field bar (1e-10 at tolerance 1e-13)."""
import numpy as np
import pytest

from tests.gpu_common import field_errors, make_pair, rel, require_gpu, residual

pytestmark = pytest.mark.gpu

FIELD_TOL = 1e-10


# (dim, n, P3-P2, kind, options): from just above the line; three levels and
# more; both directions of a ragged last block
CASES = [(2, 50, False, "tg", {}), (2, 67, False, "john", {}), (2, 53, False, "tg", {"semi": True}),
         (2, 50, False, "tg", {"chorin": True}), (3, 13, False, "beltrami", {}),
         (3, 17, False, "beltrami", {"semi": True}), (2, 26, True, "tg", {}),
         (2, 31, True, "john", {}), (3, 7, True, "beltrami", {})]


@pytest.mark.parametrize("dim,n,p3,kind,opt", CASES)
def test_steps_match_the_oracle(dim, n, p3, kind, opt):
    torch, I = require_gpu()
    print(f"multigrid CG dim={dim} n={n} p3={p3} {kind} {opt}", flush=True)
    nu, dt = (1.0, 0.002) if kind == "john" else (0.01, 0.005)
    S, o, r = make_pair(I, dim, n, kind, nu, dt, p3=p3, **opt)
    assert r.n1 > 2560
    for step in range(2):
        r.phase(I.IPCS_PHASE_ASM)
        mom = max(r.phase(I.IPCS_PHASE_MOMENTUM)["it_mom"][:dim])
        st = r.phase(I.IPCS_PHASE_PRESSURE)
        # the Jacobi form takes 60 and more here
        assert (st["it_p"] < 60) == (mom <= 40), (mom, st)
        res = residual(o.Kp, r.field(I.IPCS_FIELD_DP), r.field(I.IPCS_FIELD_RHS_P))
        r.phase(I.IPCS_PHASE_CORRECTION)
        o.step()
        errs = field_errors(o, r)
        print(f"  step {step}: it_p {st['it_p']} residual {res:.2e}", errs, flush=True)
        assert res <= 1.1e-13 or mom > 40
        assert max(errs) <= FIELD_TOL


def test_unstructured_mesh_and_previous_start():
    """Moved and relabelled vertices; the start from the previous increment."""
    torch, I = require_gpu()
    from paper_2605_25403_amd.workloads import jittered_mesh
    print("multigrid CG on a jittered mesh", flush=True)
    for p3, n in ((False, 55), (True, 29)):
        arrays = jittered_mesh(2, n, 11)
        S, o, r = make_pair(I, 2, n, "tg", 0.01, 0.005, arrays=arrays, p3=p3,
                            poisson_start=I.IPCS_START_PREVIOUS)
        for step in range(3):
            st = r.advance(1)[0]
            o.step()
            errs = field_errors(o, r)
            print(f"  p3={p3} step {step}: it_p {st['it_p']}", st["it_mom"], errs, flush=True)
            assert (st["it_p"] < 80) == (max(st["it_mom"][:2]) <= 40), st
            assert max(errs) <= FIELD_TOL


@pytest.mark.parametrize("dim,n,pair,prec_name", [
    (2, 300, 0, "fp64"), (2, 300, 0, "mixed"), (3, 36, 0, "fp64"), (3, 36, 0, "mixed"),
    (2, 150, 1, "fp64"), (3, 14, 1, "mixed")])
def test_large_systems_meet_the_tolerance(dim, n, pair, prec_name):
    """Sizes on both sides of the switch from three products to five: the
    solve in the library's own Kp and right-hand side, and the fields of two
    steps against the Jacobi form's (both within the tolerance of the exact
    increment, which the pressure's condition leaves within 1e-9 here)."""
    torch, I = require_gpu()
    print(f"multigrid CG dim={dim} n={n} pair={pair} {prec_name}", flush=True)
    prec = I.IPCS_FP64 if prec_name == "fp64" else I.IPCS_MIXED
    mesh = I.Mesh.unit_square(n, pair=pair) if dim == 2 else I.Mesh.unit_cube(n, pair=pair)
    out = []
    for rows in (0, 384):
        r = I.Run(mesh, I.ipcs_params_default(nu=0.003, dt=1e-3, precision=prec,
                                              poisson_part_rows=rows))
        if dim == 2:
            r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (4 * np.pi,))
        else:
            r.set_builtin(I.IPCS_SOL_BELTRAMI_3D, ())
        r.advance(1)
        r.phase(I.IPCS_PHASE_ASM)
        mom = max(r.phase(I.IPCS_PHASE_MOMENTUM)["it_mom"][:dim])
        st = r.phase(I.IPCS_PHASE_PRESSURE)
        if rows == 0:
            # the FP64 values of the mixed form's matrix round to its FP32 export
            if prec_name == "fp64":
                res = residual(r.matrix(I.IPCS_MAT_KP), r.field(I.IPCS_FIELD_DP),
                               r.field(I.IPCS_FIELD_RHS_P))
                assert res <= 1.1e-12, res
            else:
                assert st["res_p"] <= 1e-10 and st["ir_outer"] >= 1, st
            assert (st["it_p"] < 60) == (mom <= 40), (mom, st)
        r.phase(I.IPCS_PHASE_CORRECTION)
        out.append((r.velocity(), r.pressure(), st["it_p"]))
    (U, P, a), (V, Q, b) = out
    print("  iterations", a, b, rel(U, V), rel(P, Q), flush=True)
    assert rel(U, V) <= 1e-9 and rel(P, Q) <= 1e-9


def test_batch_equals_runs_alone():
    """Multigrid systems of both depths and both value types share launches
    with Jacobi ones; every run is bitwise the run alone."""
    torch, I = require_gpu()
    print("multigrid CG in a batch", flush=True)
    cases = [(64, 0, I.IPCS_FP64), (300, 0, I.IPCS_FP64), (52, 0, I.IPCS_MIXED),
             (30, 0, I.IPCS_FP64), (64, 384, I.IPCS_FP64), (110, 0, I.IPCS_MIXED)]
    meshes = {n: I.Mesh.unit_square(n) for n, _, _ in cases}

    def mk(n, rows, prec, stream=None):
        r = I.Run(meshes[n], I.ipcs_params_default(nu=0.003, dt=1e-3, precision=prec,
                                                   poisson_part_rows=rows), stream=stream)
        r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (4 * np.pi,))
        return r

    alone = []
    for c in cases:
        r = mk(*c)
        r.advance(3)
        alone.append((r.velocity(), r.pressure()))
    for step in (I.ipcs_batch_step, I.ipcs_batch_step_noalloc):
        s = torch.cuda.Stream()
        runs = [mk(*c, stream=s) for c in cases]
        for _ in range(3):
            rc, st = step([r.h for r in runs], s.cuda_stream)
            assert rc == I.IPCS_OK, st
        for (U, P), r in zip(alone, runs):
            np.testing.assert_array_equal(r.velocity(), U)
            np.testing.assert_array_equal(r.pressure(), P)


def test_unreachable_tolerance_falls_back_and_fails():
    """A tolerance out of reach: the multigrid solve stalls, the Jacobi form is
    tried and its failure is reported; the state stays at the last step and the
    next step at a reachable tolerance runs."""
    torch, I = require_gpu()
    print("multigrid CG: unreachable tolerance", flush=True)
    r = I.Run(I.Mesh.unit_square(60), I.ipcs_params_default(nu=0.01, dt=1e-3, tol_p=1e-16))
    r.set_builtin(I.IPCS_SOL_TAYLOR_GREEN_2D, (np.pi,))
    U0 = r.velocity()
    with pytest.raises(I.IpcsError) as e:
        r.advance(1)
    assert e.value.code in (I.IPCS_E_NOT_CONVERGED, I.IPCS_E_BREAKDOWN)
    assert e.value.stats[0].failed_solve == 2
    np.testing.assert_array_equal(r.velocity(), U0)
