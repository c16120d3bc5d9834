"""GPU kernels at the sizes where their work split can go wrong.

The step's kernels from degree 3 on are persistent: one workgroup per compute
unit, its wavefronts walking over the elements of one of eight ranges.  Edges:
fewer elements than ranges (6), than a workgroup has wavefronts, ranges of
unequal length (750 = 8 x 94 - 2), and more elements than wavefronts on the
card (4374), in every degree and precision.  Small meshes are
compared with the FP64 oracle; the large one, FP32 and split-BF16 against the
FP64 library (whose kernels are others).

Tolerances are the ones of the parity tests, derived from the arithmetic: two
Cauchy-Kovalevskaya steps accumulate a few hundred roundings, 1e-10 in FP64; in FP32 and the split
form (FP32 state and accumulation) 1e-5; a sum over 4374 elements does not
change a relative L2 norm.
"""
import numpy as np
import pytest

from oracle.refmat import RefElement
from oracle.sources import PointSources, Receivers
from oracle.step import from_workload as oracle_from
from workloads import make_workload

from _metrics import assert_within, errors

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16": 1e-5}


def _api():
    from paper_2502_09714_amd import api
    return api


def _to_lib(U):
    return U.permute(0, 2, 1).contiguous().numpy()


_ORACLE = {}


def _oracle(N, n):
    if (N, n) not in _ORACLE:
        w = make_workload("c2", n=n, N=N)
        S = oracle_from(w)
        U = S.project(w.ic)
        _ORACLE[N, n] = (w, _to_lib(U), _to_lib(S.run(U, 2)))
    return _ORACLE[N, n]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("N,n", [(1, 1), (2, 1), (3, 1), (4, 1), (1, 5), (2, 3), (3, 2), (4, 2)])
def test_step_on_few_elements(N, n, prec):
    w, U0, U2 = _oracle(N, n)
    sim = _api().from_workload(w, prec, state=False)
    sim.set_state(U0)
    sim.step(2)
    e = errors(sim.get_state(), U2, RefElement(N).V.numpy())
    print(N, n, prec, e, flush=True)
    assert_within(e, TOL[prec], f"degree {N}, {6 * n ** 3} elements, {prec}")
    sim.close()


@pytest.mark.parametrize("predictor", ["ck", "picard"])
@pytest.mark.parametrize("N,n", [(3, 5), (3, 9), (4, 9)])
def test_step_more_elements_than_wavefronts(N, n, predictor):
    """The state after two steps; with the Picard predictor its own output, the
    time-point states (its corrector is another set of kernels, whose BF16 form
    has the 3e-3 bar of the Picard parity tests)."""
    w = make_workload("c2", n=n, N=N)
    want = None
    for prec in ("fp64", "fp32", "bf16"):
        sim = _api().from_workload(w, prec)
        if predictor == "ck":
            sim.step(2)
            got = sim.get_state()
        else:
            sim.set_predictor("picard", 0)
            sim.step(1)
            got = sim.get_time_point_states()
            got = got.transpose(0, 2, 1, 3).reshape(got.shape[0], 10, -1)
        sim.close()
        if want is None:
            want = got
            continue
        what = f"degree {N}, {6 * n ** 3} elements, {predictor}, {prec}"
        if predictor == "ck":
            e = errors(got, want, RefElement(N).V.numpy())
            print(what, e, flush=True)
            assert_within(e, TOL[prec], what)
        else:
            for g in (slice(0, 6), slice(6, 9), slice(9, 10)):
                e = np.linalg.norm(got[:, g] - want[:, g]) / np.linalg.norm(want[:, g])
                print(what, g, e, flush=True)
                assert e < TOL[prec], what


@pytest.mark.parametrize("N,n", [(4, 3), (4, 9)])
def test_adjoint_points_split_form(N, n):
    """The adjoint of the volume terms, FP32 (split products) against FP64, on
    lognormal moduli (no ties of the two sides' speeds)."""
    w = make_workload("c3", n=n, N=N)
    out = []
    rng = np.random.default_rng(5)
    lam = None
    for prec in ("fp64", "fp32"):
        sim = _api().from_workload(w, prec)
        if lam is None:
            lam = rng.standard_normal(sim.get_state().shape)
        lam_n, gmu, gcd = sim.adjoint_step_host(lam)
        out.append((lam_n - lam, gmu, gcd))
        sim.close()
    for a, b, k in zip(out[1], out[0], ("lambda", "dJ/dmu0", "dJ/dCd")):
        e = np.linalg.norm(a - b) / np.linalg.norm(b)
        print(N, n, k, e, flush=True)
        assert e < 1e-5, k


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 1e-5)])
def test_sources_and_receivers_sharing_an_element(prec, tol):
    """Three sources in one element with a receiver in it, one source elsewhere,
    receivers in elements without sources, two of them in one."""
    w = make_workload("c4", n=4, N=2)
    s = {k: (np.repeat(np.asarray(v), 4, axis=0) if np.ndim(v) else v) for k, v in w.sources.items()}
    x = np.array(s["xyz"], dtype=np.float64)
    x[1] += [3.0, 2.0, -1.0]
    x[2] += [-2.0, 1.0, 1.0]
    x[3] += [2500.0, 900.0, 700.0]
    s["xyz"] = x
    S = oracle_from(w)
    sim = _api().from_workload(w, prec, state=False)
    sim.set_point_sources(**s)
    rec = np.stack([x[0] + 1.0, x[0] + [1800.0, 700.0, 500.0], x[0] + [1801.0, 701.0, 501.0],
                    x[3] + 2.0])
    sim.set_receivers(rec)
    U = S.project(w.ic)
    sim.set_state(_to_lib(U))
    t = 0.45
    sim.set_time(t)
    src, R = PointSources(S, **s), Receivers(S, rec)
    want = []
    for _ in range(4):
        U = S.step(U) + src.increment(t, t + S.dt)
        t += S.dt
        want.append(R.sample(U).numpy())
    sim.step(4)
    want, got = np.stack(want), sim.get_seismograms()
    assert np.linalg.norm(got - want) / np.linalg.norm(want) < tol
    d = _to_lib(U)[:, :9]
    assert np.linalg.norm(sim.get_state()[:, :9] - d) / np.linalg.norm(d) < tol
    sim.close()
