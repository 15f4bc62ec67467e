"""The zone solve where conjugate gradients cannot stand for the heavy-ball steps: the relaxation keeps the
steps themselves.  Energies against the FP64 oracle within the zone solve's tolerance, 1e-5 of max(|dPi|, W_p / 10)
(see test_gpu_zone_krylov, whose check this is)."""
import pytest

import test_gpu_zone_krylov as Z

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)


# lightly damped steps, whose last residuals are polynomials of a degree that a Krylov basis of a converged solve
# does not resolve: beta^n_r is 4e-5, 0.13, 2e-3 and 0.02
@pytest.mark.parametrize("K,h,nr,beta", [(10, 2, 200, 0.95), (10, 2, 200, 0.99), (10, 2, 600, 0.99), (8, 3, 400, 0.99)])
def test_lightly_damped_steps(K, h, nr, beta):
    Z.test_zone_energies_match_the_heavy_ball_oracle(K, h, nr, Z.NICKEL, 1.0, 1.0, beta)
