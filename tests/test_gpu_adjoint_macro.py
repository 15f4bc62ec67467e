"""The gradient's macroscopic terms, with the relaxation switched off (step lengths 0): the state is the uniform strain
E_0 = mean(S_q) Sigma, of 512 random grains mixed over 16^3 sites, and the load derivative mean(S) sum_v C_v E_0 in
closed form.  What FP32 leaves are the grains' table entries, rounded by at most 2^-24 of themselves and in no relation
to each other, so that over 512 grains 6e-8 averages to 3e-9; 1e-8 allows for C, S and the products.  A macroscopic
strain or stress in FP32 would show: its rounding, up to 6e-8 of a component, is the same in every voxel."""
import numpy as np
import pytest

import oracle as O
from paper_1009_0457_amd import hmc as H
from paper_1009_0457_amd.synth import haar_euler, random_spins

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)


def test_load_derivative_of_a_uniform_strain():
    K, Q = 16, 512
    rng = np.random.default_rng(7)
    euler, spins = haar_euler(rng, Q), random_spins(K, Q, 3)
    p = H.hmc_default_params(K, 26, 1)
    p.glob_alpha = p.glob_alphaE = 0.0
    Ct, St, _ = O.tables(euler, p.C11, p.C12, p.C44)
    share = np.bincount(spins, minlength=Q) / K ** 3
    C, S = (np.einsum("q,qij->ij", share, np.asarray(t).reshape(Q, 6, 6)) for t in (Ct, St))
    lat = H.Lattice(p, Q)
    lat.set_orientations(euler)
    lat.set_spins(spins)
    for load in rng.uniform(-200, 200, (6, 6)):
        lat.set_load(load)
        U = lat.elastic_forward(1, 1)
        E = lat.macro_strain()
        _, got = lat.elastic_backward(1.0)
        want = K ** 3 * 1e-3 * S @ (C @ E)
        err = np.linalg.norm(got - want) / np.linalg.norm(want)
        print(f"[macro] load derivative off by {err:.2e}, energy by {U / (0.5 * K ** 3 * E @ C @ E) - 1:.2e}", flush=True)
        assert err <= 1e-8
        assert abs(U / (0.5 * K ** 3 * E @ C @ E) - 1) <= 1e-8
    lat.close()
