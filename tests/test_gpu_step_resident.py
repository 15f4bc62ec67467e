"""The explicit step at the line between its kernels: tiles of 1, 2 or 4 layers go to the shallow kernel while a launch has
at most 512 blocks, to the marched one beyond.  A replica of a batch past the line has, to the last
bit, the stress of itself alone, before it."""
import numpy as np
import pytest

from paper_1009_0457_amd import hmc as H
from paper_1009_0457_amd.synth import haar_euler, random_spins

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

SIG = [120.0, -40.0, 80.0, 30.0, -20.0, 10.0]


# 512 and 640 blocks of 32^3, 680 of 34^3, 680 at depth 2, 500 and 600 of 40^3 at depth 4
@pytest.mark.parametrize("K,depth,n", [(32, 1, 4), (32, 1, 5), (34, 1, 2), (34, 2, 4), (40, 4, 5), (40, 4, 6)])
def test_batch_across_the_line_equals_alone(K, depth, n):
    tiles = -(-K // 32) * -(-K // 8) * -(-K // depth)
    print(f"[resident] K={K} depth={depth}: {n} x {tiles} blocks", flush=True)
    Q = 12
    euler = haar_euler(np.random.default_rng(K), Q)
    spins = [random_spins(K // 2, Q, 9 * r + K).reshape((K // 2,) * 3).repeat(2, 0).repeat(2, 1).repeat(2, 2).ravel()
             for r in range(n)]
    common = H.hmc_default_params(K, 26, 1)
    common.refresh_tile_z = depth
    reps = []
    for r in range(n):
        rep = H.hmc_default_replica(common, K, Q)
        for i in range(6):
            rep.sigma_MPa[i] = SIG[(i + r) % 6]
        reps.append(rep)
    b = H.Batch(common, reps)
    for r in range(n):
        b.set_replica(r, euler, spins[r])
    b.stress_refresh(21, True)
    lat = H.Lattice(common, Q)
    lat.set_orientations(euler)
    for r in range(n):
        lat.set_spins(spins[r])
        lat.set_load(np.roll(SIG, -r))
        lat.stress_refresh(21, True)
        assert torch.equal(lat.get_stress(), b.get_stress(r)), r
    lat.close()
    b.close()
