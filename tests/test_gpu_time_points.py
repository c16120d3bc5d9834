"""dgd_get_time_point_states: what it returns after each kind of call."""
import numpy as np
import pytest

from oracle.quadrature import time_rule
from workloads import make_workload

pytestmark = pytest.mark.gpu

# one prediction from states that agree to rounding; FP32 states are extrapolated to the step's start from the
# N + 1 time points (Lebesgue constant below 10), so a factor 10 above the rounding of the states
TOL = {"fp64": 1e-13, "fp32": 2e-5}


def _sim(w, prec):
    from paper_2502_09714_amd import api
    return api.from_workload(w, prec)


def _rel(a, b):
    """Largest relative difference over the quantity groups, of (E, Nt, 10, L) arrays."""
    return max(np.linalg.norm((a - b)[:, :, g]) / np.linalg.norm(b[:, :, g])
               for g in (slice(0, 6), slice(6, 9), slice(9, 10)))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [1, 2, 3, 4])
def test_after_clustered_steps(N, prec):
    """The prediction is local to the element: each element's states are those that a global step of the
    length of its own predicts from the state at its start (the value at tau = 0 of the polynomial through
    them).  Clusters that are replaced afterwards do not change them."""
    w = make_workload("c2", n=3, N=N)
    sim = _sim(w, prec)
    cent = w.mesh["xyz"][w.mesh["tets"]].mean(axis=1)
    cl = (cent[:, 0] < 0.5 * w.mesh["length"]).astype(np.int32)
    dt0 = 0.5 * w.dt
    sim.set_clusters(cl, dt0)
    sim.step_lts(2)
    got = sim.get_time_point_states()
    sim.set_clusters(1 - cl, 0.25 * dt0)
    assert np.array_equal(sim.get_time_point_states(), got)
    sim.set_clusters(None)
    sim.set_params(3.0 * w.dt, w.alpha_max)
    assert np.array_equal(sim.get_time_point_states(), got)
    sim.close()
    tau = time_rule(N)[0].numpy()
    at0 = np.array([np.prod([-tau[k] / (tau[j] - tau[k]) for k in range(N + 1) if k != j]) for j in range(N + 1)])
    start = np.einsum("z,ezpl->epl", at0, got)
    ref = _sim(w, prec)
    ref.set_state(np.ascontiguousarray(start))
    for c in (0, 1):
        ref.set_params(dt0 * 2 ** c, w.alpha_max)
        ref.set_state(np.ascontiguousarray(start))
        ref.step(1)
        e = _rel(got[cl == c], ref.get_time_point_states()[cl == c])
        print(N, prec, "cluster", c, e, flush=True)
        assert e < TOL[prec]
    ref.close()


@pytest.mark.parametrize("N,n", [(4, 10), (3, 13)])
def test_query_in_slices(N, n):
    """More elements than one slice of the query's 64 MiB of scratch (4793 at degree 4, 10485 at degree 3):
    every element's states extrapolate to the state it was set to."""
    w = make_workload("c2", n=n, N=N)
    sim = _sim(w, "fp64")
    U = sim.get_state()
    sim.step(1)
    got = sim.get_time_point_states()
    sim.close()
    tau = time_rule(N)[0].numpy()
    at0 = np.array([np.prod([-tau[k] / (tau[j] - tau[k]) for k in range(N + 1) if k != j]) for j in range(N + 1)])
    start = np.einsum("z,ezpl->epl", at0, got)
    scale = np.abs(got).max(axis=(0, 1, 3))[None, :, None]
    assert (np.abs(start - U) / scale).max() < 1e-12


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [1, 2, 4])
def test_backward_leaves_the_last_steps(N, prec):
    """Replayed steps of dgd_backward are not the solver's last one."""
    w = make_workload("c4", n=3, N=N)
    sim = _sim(w, prec)
    sim.forward_checkpointed(5, 2)
    run = sim.get_time_point_states()
    cot = np.ones((5, sim.nrec, 3))
    grad = sim.backward(cot)
    assert np.array_equal(sim.get_time_point_states(), run)
    sim.step(2)
    later = sim.get_time_point_states()
    again = sim.backward(cot)
    assert np.array_equal(sim.get_time_point_states(), later)
    assert np.array_equal(again[0], grad[0]) and np.array_equal(again[1], grad[1])
    sim.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("N", [1, 2, 3, 4])
def test_first_picard_and_adjoint_call_keep_them(N, prec):
    """The first call that needs time-point states on the device takes the derivatives' place, with their
    content; the states of an adjoint step and of Picard steps replace them."""
    w = make_workload("c4", n=3, N=N)
    sim, ref = _sim(w, prec), _sim(w, prec)
    U0 = sim.get_state()
    sim.step(2)
    pts = sim.get_time_point_states()
    sim.set_predictor("picard")
    assert np.array_equal(sim.get_time_point_states(), pts)
    sim.set_predictor("ck")
    sim.set_state(U0)
    sim.set_time(0.0)
    sim.step(2)                                     # derivatives now beside or in the states' memory
    assert np.array_equal(sim.get_time_point_states(), pts)
    U2 = sim.get_state()
    sim.adjoint_step_host(np.ones_like(U2))
    ref.set_state(U2)
    ref.step(1)
    tol = {"fp64": 1e-13, "fp32": 1e-5, "bf16": 1e-5}[prec]
    assert _rel(sim.get_time_point_states(), ref.get_time_point_states()) < tol
    assert np.array_equal(sim.get_state(), U2)
    sim.set_predictor("picard")
    sim.step(1)
    pic = sim.get_time_point_states()
    sim.set_predictor("ck")
    assert np.array_equal(sim.get_time_point_states(), pic)
    sim.set_mesh(w.mesh["xyz"], w.mesh["tets"], w.mesh["face_tag"], w.mesh["periodic_map"])
    sim.set_material(**{k: w.material[k] for k in ("rho", "lambda0", "mu0", "gamma_r", "xi0", "Cd")})
    sim.set_state(U0)
    assert not sim.get_time_point_states().any()
    sim.close()
    ref.close()


def test_memory_of_the_time_point_states():
    """Derivatives and time-point states share one buffer, allocated with the mesh: neither the Picard
    predictor nor the adjoint asks for either again (degree 4 FP32: 7000 and 4352 bytes an element)."""
    import torch
    w = make_workload("c2", n=14, N=4)

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    sim = _sim(w, "fp32")
    sim.step(1)
    f0 = free()
    sim.set_predictor("picard")
    assert f0 - free() == 0
    sim.set_predictor("ck")
    lam = np.zeros((w.ne, 10, sim.L))
    sim.adjoint_step_host(lam)
    faces = 2 * w.ne + 6 * 14 * 14                  # interior ones and half of the boundary's twelve triangles a square
    adjoint = 4 * (2 * 36 * 16 + 5 * 36 * 16 + 9 * 35) * w.ne + 8 * (2 + 35) * w.ne + \
        4 * (2 * 5 * 25 * 10) * faces + 16 * faces
    assert f0 - free() <= adjoint + (24 << 20)      # ten buffers, rounded to 2 MiB
    sim.close()
