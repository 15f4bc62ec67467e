"""How far the explicit step's FP32 stress is from C e: no further than the product with the 21 entries of C, rounded
to FP32 and summed by fused multiply-adds, would be on the same strains (that product is emulated here, an FP32 product
and sum in FP64 rounded once).  The stress is read off a lattice of one grain under a uniaxial load, its displacements
held (glob_alpha = 0), whose first step moves the macroscopic strain by Sigma - <sigma(E_0)> (glob_alphaE = 1; the
stress sums resolve 3e-9 of it)."""
import numpy as np
import pytest

import oracle as O
from paper_1009_0457_amd import hmc as H
from paper_1009_0457_amd.synth import haar_euler

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)


def by_entries(c, e):
    """The FP32 product of (n, 6, 6) stiffnesses and (n, 6) strains."""
    c, e = c.astype(np.float32).astype(np.float64), e.astype(np.float64)
    s = np.zeros(e.shape)
    for j in range(6):
        s = (c[:, :, j] * e[:, None, j] + s).astype(np.float32).astype(np.float64)
    return s


def test_rounding_of_the_step_stress():
    K, n = 4, 200
    load = np.array([0.0, 0.0, 150.0, 0.0, 0.0, 0.0])
    p = H.hmc_default_params(K, 26, 1)
    p.glob_alpha, p.glob_alphaE = 0.0, 1.0
    euler = haar_euler(np.random.default_rng(4), n)
    C = np.asarray(O.tables(euler, p.C11, p.C12, p.C44)[0]).reshape(n, 6, 6)
    lat = H.Lattice(p, 1)
    strain, stress = [], []
    for e in euler:
        lat.set_orientations(e[None])
        lat.set_spins(np.zeros(K ** 3, np.int32))
        lat.set_load(load)
        lat.stress_refresh(0, True)
        E0 = lat.macro_strain()
        lat.stress_refresh(1, True)
        strain.append(E0.astype(np.float32))
        stress.append(load * 1e-3 - (lat.macro_strain() - E0))
    lat.close()
    strain = np.array(strain)
    want = np.einsum("nij,nj->ni", C, strain.astype(np.float64))

    def rms(s):
        return np.sqrt(np.mean(np.sum((s - want) ** 2, 1) / np.sum(want ** 2, 1)))

    here, entries = rms(np.array(stress)), rms(by_entries(C, strain))
    print(f"[stress rounding] {here:.2e}, by the entries {entries:.2e} over {n} orientations", flush=True)
    assert here <= entries
