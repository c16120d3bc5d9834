"""Non-finite damage and inadmissible moduli show in the waves and raise the flag."""
import numpy as np
import pytest

from workloads import make_workload

pytestmark = pytest.mark.gpu


def _run(w, prec, predictor, change=None):
    from paper_2502_09714_amd import api
    from paper_2502_09714_amd._lib import DGDError
    sim = api.from_workload(w, prec)
    sim.set_predictor(predictor)
    if change is not None:
        U = sim.get_state()
        change(U)
        sim.set_state(U)
    with pytest.raises(DGDError, match="ENUMERIC"):
        sim.step(1)
        sim.synchronize()
    U = sim.get_state()
    sim.close()
    return U


@pytest.mark.parametrize("predictor", ["ck", "picard"])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("N", [1, 2, 3, 4])
def test_nan_damage_reaches_the_waves(N, prec, predictor):
    """A stress with a NaN in it enters the velocities, and through the prediction (any further order or
    sweep) the strains of the element, too.  (Periodic: a boundary flux carries the NaN by its moduli.)"""
    w = make_workload("c2", n=3, N=N, periodic=True)

    def change(U):
        U[17, 9, 0] = np.nan

    U = _run(w, prec, predictor, change)
    assert not np.isfinite(U[17, :9]).any()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_ivm_negative_p_modulus_is_flagged(prec):
    """lambda0 + 2 mu0 < 0 has no wave speed."""
    from paper_2502_09714_amd import api
    from paper_2502_09714_amd._lib import DGDError
    w = make_workload("c2", n=3, N=2, periodic=True)
    sim = api.from_workload(w, prec)
    m = w.material
    mu = np.asarray(m["mu0"])
    sim.set_material_ivm(m["rho"], -3.0 * mu, mu, np.full_like(mu, 1e4), np.full_like(mu, 1.0))
    with pytest.raises(DGDError, match="ENUMERIC"):
        sim.step(1)
        sim.synchronize()
    sim.close()
