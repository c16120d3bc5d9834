"""Clustered steps and the internal-variable law on the step's kernels from degree 3 on, at the sizes of their
element lists; handles in BF16 form.

The small cases are compared with the FP64 oracle under the bars of the parity tests (1e-10 in FP64, 1e-5 in
FP32: a few hundred roundings per step).  On the large mesh, 5 of 6000 elements take the finer step: one list
is longer than the launch has wavefronts (256 compute units x 16), the other shorter than the eight ranges it is
cut into.  Elements that no finer element reaches within the step must come out as from the global step
without lists, to rounding (1e-6), and all of them in FP32 as in FP64.
"""
import numpy as np
import pytest

from oracle.lts import LtsSolver
from oracle.refmat import RefElement
from oracle.step import from_workload as oracle_from
from workloads import make_workload

from _metrics import assert_within, errors
from _patch import face_partners

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-5, "bf16": 1e-5}


def _sim(w, prec, state=True):
    from paper_2502_09714_amd import api
    return api.from_workload(w, prec, state=state)


def _to_lib(U):
    return U.permute(0, 2, 1).contiguous().numpy()


def _thirds(w):
    """Clusters 0, 1, 2 by thirds of the cube along x (neighbours at most one apart)."""
    cent = w.mesh["xyz"][w.mesh["tets"]].mean(axis=1)
    return np.minimum(2, (3.0 * cent[:, 0] / w.mesh["length"]).astype(np.int32)).astype(np.int32)


_ORACLE = {}


def _lts_case(N, law):
    if (N, law) not in _ORACLE:
        w = make_workload("c2", n=3, N=N, rheology=law)
        S = oracle_from(w)
        U0 = S.project(w.ic)
        cl, dt0 = _thirds(w), w.dt / 4
        _ORACLE[N, law] = (w, cl, dt0, _to_lib(U0), _to_lib(LtsSolver(S, cl, dt0).run(U0, 1)))
    return _ORACLE[N, law]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("N,law", [(4, "cdm"), (4, "ivm"), (3, "ivm")])
def test_three_clusters(N, law, prec):
    w, cl, dt0, U0, want = _lts_case(N, law)
    sim = _sim(w, prec, state=False)
    sim.set_state(U0)
    sim.set_clusters(cl, dt0)
    sim.step_lts(1)
    e = errors(sim.get_state(), want, RefElement(N).V.numpy())
    print(N, law, prec, e, flush=True)
    assert_within(e, TOL[prec], f"three clusters, degree {N}, {law}, {prec}")
    sim.close()


@pytest.mark.parametrize("N", [3, 4])
def test_long_and_short_lists(N):
    w = make_workload("c2", n=10, N=N)
    nbr = face_partners(w.mesh)
    cl = np.ones(w.ne, dtype=np.int32)
    cl[:5] = 0
    near = cl == 0
    for _ in range(2):                      # flux integrals reach the neighbours; their neighbours for good measure
        near[nbr[near][nbr[near] >= 0]] = True
    out = {}
    for prec in ("fp64", "fp32"):
        sim = _sim(w, prec)
        U0 = sim.get_state()
        sim.set_params(w.dt, w.alpha_max)
        sim.step(1)
        whole = sim.get_state()
        sim.set_state(U0)
        sim.set_clusters(cl, w.dt / 2)
        sim.step_lts(1)
        out[prec] = sim.get_state()
        sim.close()
        tol = 1e-13 if prec == "fp64" else 1e-6
        e = np.linalg.norm((out[prec] - whole)[~near]) / np.linalg.norm(whole[~near])
        print(N, prec, int(near.sum()), e, flush=True)
        assert e < tol
        assert np.abs((out[prec] - whole)[cl == 0]).max() > 0
    assert_within(errors(out["fp32"], out["fp64"], RefElement(N).V.numpy()), TOL["fp32"], f"lists, degree {N}")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("N,n", [(1, 1), (2, 1), (3, 1), (4, 1), (3, 2), (4, 2)])
def test_ivm_on_few_elements(N, n, prec):
    key = ("few", N, n)
    if key not in _ORACLE:
        w = make_workload("c2", n=n, N=N, rheology="ivm")
        S = oracle_from(w)
        U = S.project(w.ic)
        _ORACLE[key] = (w, _to_lib(U), _to_lib(S.run(U, 2)))
    w, U0, want = _ORACLE[key]
    sim = _sim(w, prec, state=False)
    sim.set_state(U0)
    sim.step(2)
    e = errors(sim.get_state(), want, RefElement(N).V.numpy())
    print(N, n, prec, e, flush=True)
    assert_within(e, TOL[prec], f"internal-variable law, degree {N}, {6 * n ** 3} elements, {prec}")
    sim.close()


@pytest.mark.parametrize("law", ["cdm", "ivm"])
@pytest.mark.parametrize("N", [1, 2, 3, 4])
def test_bf16_handles_step_as_fp32_ones(N, law):
    """Their Cauchy-Kovalevskaya step, global and clustered, is the FP32 one to the bit."""
    w = make_workload("c2", n=3, N=N, rheology=law)
    out = []
    for prec in ("fp32", "bf16"):
        sim = _sim(w, prec)
        sim.step(2)
        sim.set_clusters(_thirds(w), w.dt / 4)
        sim.step_lts(1)
        out.append(sim.get_state())
        sim.close()
    assert np.array_equal(out[0], out[1])
