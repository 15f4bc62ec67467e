"""Which zone relaxations go by conjugate gradients, from the host-only query: by length, zone size and variant, by
the slowest shear of the crystal, and by how the heavy-ball steps are damped.  No call here touches a GPU."""
import os

import pytest

H = pytest.importorskip("paper_1009_0457_amd.hmc")
if not os.path.exists(H.LIB_PATH):
    pytest.skip("libhmc.so not built", allow_module_level=True)


def by_gradients(h, nr, variant=0, c=None, beta=None, alpha_scale=1.0):
    p = H.hmc_default_params(16, 26, h)
    if c is not None:
        p.C11, p.C12, p.C44 = c
        lam = max(c[0] + 2 * c[1], c[0] - c[1], 2 * c[2])
        a, b = (4 * lam) ** 0.5, (0.5 * (c[0] - c[1])) ** 0.5 / (2 * h + 1)
        p.zone_alpha, p.zone_beta = 4 / (a + b) ** 2, ((a - b) / (a + b)) ** 2
    p.zone_steps, p.zone_variant = nr, variant
    p.zone_alpha *= alpha_scale
    if beta is not None:
        p.zone_beta = beta
    return H.hmc_zone_by_gradients(p)


@pytest.mark.parametrize("h,nr,want", [(0, 4000, False), (1, 4000, False), (2, 148, False), (2, 149, True), (2, 4000, True),
                                       (3, 231, False), (3, 232, True), (2, 0, False)])
def test_length_and_zone_size(h, nr, want):
    assert by_gradients(h, nr) == want
    for variant in (1, 2, 3, 4, 5):          # these name a kernel of heavy-ball steps (or none: 0 there too)
        assert not by_gradients(h, nr, variant)


@pytest.mark.parametrize("c,nr,want", [((34.6, 5.8, 5.05), 135, False), ((34.6, 5.8, 5.05), 137, True),
                                       ((250.0, 60.0, 30.0), 200, True), ((250.0, 60.0, 10.0), 4000, False),
                                       ((250.0, 0.0, 2.0), 4000, False)])
def test_slowest_shear(c, nr, want):
    assert by_gradients(2, nr, c=c) == want


@pytest.mark.parametrize("beta,nr,want", [(0.95, 200, False), (0.95, 314, False), (0.95, 315, True), (0.99, 1000, False),
                                          (0.0, 200, False), (1.0, 4000, False), (-0.5, 200, False), (-1.5, 200, False)])
def test_damping(beta, nr, want):
    """0.95^314 is above 1e-7, 0.95^315 below; the default alpha needs a beta of 0.2 at least to be stable."""
    assert by_gradients(2, nr, beta=beta) == want


def test_step_length():
    assert by_gradients(2, 200, alpha_scale=0.01) and by_gradients(2, 200, beta=0.0, alpha_scale=0.5)
    # stable up to 2 (1 + beta) over 4 times the <111> modulus, 346.6 GPa: 1.56 times the default
    assert by_gradients(2, 200, alpha_scale=1.56) and not by_gradients(2, 200, alpha_scale=1.57)
    assert not by_gradients(2, 200, alpha_scale=-1.0)


def test_constants_changed_alone():
    """The texture experiment's nickel on another set's step lengths."""
    for h, nr in ((2, 200), (3, 400)):
        p = H.hmc_default_params(100, 26, h)
        p.zone_steps = nr
        p.C11, p.C12, p.C44 = 250.8, 150.0, 123.5
        assert H.hmc_zone_by_gradients(p)
