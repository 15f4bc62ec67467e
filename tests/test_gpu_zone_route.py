"""Which relaxations the zone solve takes by conjugate gradients, and that the others keep the heavy-ball steps.

Steps that the gradients cannot stand for are held to the FP64 oracle within the zone solve's tolerance, 1e-5 of
max(|dPi|, W_p / 10) (see test_gpu_zone_krylov, whose check this is).  The route itself is read off the bits: variant 4
always takes the steps, with the arithmetic of the automatic choice's, so its energies are equal to the last bit where
the automatic choice takes them too, and differ in some trials' last bits where it takes gradients."""
import numpy as np
import pytest

import test_gpu_zone_krylov as Z
from paper_1009_0457_amd import autotune as A
from paper_1009_0457_amd import hmc as H
from paper_1009_0457_amd.synth import voronoi_polycrystal

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)


# lightly damped steps, whose last residuals are polynomials of a degree that a Krylov basis of a converged solve
# does not resolve: beta^n_r is 4e-5, 0.13, 2e-3 and 0.02
@pytest.mark.parametrize("K,h,nr,beta", [(10, 2, 200, 0.95), (10, 2, 200, 0.99), (10, 2, 600, 0.99), (8, 3, 400, 0.99)])
def test_lightly_damped_steps(K, h, nr, beta):
    Z.test_zone_energies_match_the_heavy_ball_oracle(K, h, nr, Z.NICKEL, 1.0, 1.0, beta)


# steps near the longest that the rule takes on T
@pytest.mark.parametrize("K,h,nr", [(10, 2, 200), (8, 3, 400)])
def test_long_steps(K, h, nr):
    Z.test_zone_energies_match_the_heavy_ball_oracle(K, h, nr, Z.NICKEL, 1.0, 1.55, None)


# constants at the edge of the rule, whose trials fill the kernel's table or nearly do
@pytest.mark.parametrize("K,h,nr,c", [(12, 2, 1000, (100.0, 61.0, 120.0)), (12, 2, 1000, (250.0, 60.0, 29.5)),
                                      (12, 3, 600, (100.0, 57.0, 120.0))])
def test_full_tables(K, h, nr, c):
    Z.test_zone_energies_match_the_heavy_ball_oracle(K, h, nr, c, 1.0, 1.0, None)


def energies(K, h, nr, c, variant):
    m = voronoi_polycrystal(K, 10, 70 + K)
    p = H.hmc_default_params(K, 26, h)
    p.kT, p.proposal, p.zone_steps, p.zone_variant = 0.8, 1, nr, variant
    p.C11, p.C12, p.C44 = c
    lam, mu = max(c[0] + 2 * c[1], c[0] - c[1], 2 * c[2]), 0.5 * (c[0] - c[1]) / (2 * h + 1) ** 2
    a, b = (4 * lam) ** 0.5, mu ** 0.5
    p.zone_alpha, p.zone_beta = 4.0 / (a + b) ** 2, ((a - b) / (a + b)) ** 2
    lat = H.Lattice(p, m.Q)
    lat.set_orientations(m.euler)
    lat.set_spins(m.spins)
    lat.set_load([60.0, -90.0, 140.0, 25.0, 0.0, -35.0])
    lat.stress_refresh(200, True)
    rec = lat.colour_pass(5, records=True)
    lat.close()
    return rec["dPi"]


# nickel at the two lengths around the shortest that gradients take; crystals whose slowest shear is C44's, on which
# gradients take longer than 1/2 (C11 - C12) says: some 105 steps for the first, more than their table holds for the rest
ROUTES = [(10, 2, 148, Z.NICKEL, False), (10, 2, 149, Z.NICKEL, True), (8, 3, 231, Z.NICKEL, False),
          (8, 3, 232, Z.NICKEL, True), (10, 2, 120, (34.6, 5.8, 5.05), False), (10, 2, 200, (34.6, 5.8, 5.05), True),
          (10, 2, 600, (250.0, 60.0, 10.0), False), (10, 2, 600, (250.0, 0.0, 2.0), False),
          (10, 2, 1000, (250.0, 60.0, 2.0), False), (8, 3, 1000, (250.0, 60.0, 2.0), False)]


@pytest.mark.parametrize("K,h,nr,c,gradients", ROUTES)
def test_route(K, h, nr, c, gradients):
    print(f"[zone route] K={K} h={h} steps={nr} C={c}", flush=True)
    automatic, steps = energies(K, h, nr, c, 0), energies(K, h, nr, c, 4)
    assert np.count_nonzero(steps) > 20
    assert np.array_equal(automatic, steps) != gradients


@pytest.mark.parametrize("K,h,nr", [(10, 2, 200), (8, 3, 400)])
def test_variant_3_keeps_the_steps(K, h, nr):
    """One wavefront of whole trials per work-group, at lengths that the automatic choice takes by gradients."""
    print(f"[zone route] variant 3 K={K} h={h} steps={nr}", flush=True)
    automatic, one, two = (energies(K, h, nr, Z.NICKEL, v) for v in (0, 3, 4))
    assert np.array_equal(one, two) and not np.array_equal(one, automatic)


def test_autotuner_times_the_gradients():
    """A long relaxation has variant 0 among the candidates, a short one does not."""
    for nr, want in ((200, True), (60, False)):
        m = voronoi_polycrystal(12, 10, 21)
        p = H.hmc_default_params(12, 26, 2)
        p.kT, p.proposal, p.zone_steps = 0.8, 1, nr
        lat = H.Lattice(p, m.Q)
        lat.set_orientations(m.euler)
        lat.set_spins(m.spins)
        lat.set_load([80.0, -60.0, 120.0, 20.0, 0.0, -30.0])
        lat.stress_refresh(100, True)
        res = A.tune_zone_variant(lat, 2)
        print(f"[zone route] autotune steps={nr}: {res}", flush=True)
        assert ("0" in res["ms_per_solve"]) == want and {"1", "2", "3", "4", "5"} <= set(res["ms_per_solve"])
        lat.close()
