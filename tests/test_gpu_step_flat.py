"""The shallow explicit step (tiles of depth 1, 2 and 4) at the edges of its tiles: lattices narrower
than a tile, edges that leave a remainder in x, y and z (a cut last tile at depth 4), an edge at which
the equal tiles are shallower than asked for (which the other kernel takes), and a batch of both.  FP32
steps on FP32 tables stay within 1e-6 of the FP64 oracle's field over so few steps (each step adds
about a unit in the last place of the strain, 6e-8)."""
import numpy as np
import pytest

import oracle as O
from paper_1009_0457_amd import hmc as H
from paper_1009_0457_amd.synth import voronoi_polycrystal

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

SIG = np.array([120.0, -40.0, 80.0, 30.0, -20.0, 10.0])
STEPS = 40


def oracle_field(m, p, sig_MPa):
    Ct, St, _ = O.tables(m.euler, p.C11, p.C12, p.C44)
    _, E, s, _ = O.global_solve(m.K, m.spins, Ct, St, sig_MPa * 1e-3, STEPS, True, p.glob_alpha, p.glob_beta,
                                p.glob_alphaE)
    return E, s


@pytest.mark.parametrize("K", [4, 6, 10, 26, 34])
@pytest.mark.parametrize("depth", [1, 2, 4])
def test_shallow_step_matches_oracle(K, depth):
    print(f"[flat step] K={K} depth={depth}", flush=True)
    m = voronoi_polycrystal(K, max(2, K ** 3 // 300), 80 + K)
    p = H.hmc_default_params(K, 26, 1)
    p.refresh_tile_z = depth
    lat = H.Lattice(p, m.Q)
    lat.set_orientations(m.euler)
    lat.set_spins(m.spins)
    lat.set_load(SIG)
    lat.stress_refresh(STEPS, True)
    E, s = oracle_field(m, p, SIG)
    got = lat.get_stress().cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - s) <= 1e-6 * np.linalg.norm(s)
    assert np.linalg.norm(lat.macro_strain() - E) <= 1e-6 * np.linalg.norm(E)
    lat.close()


def test_shallow_step_in_a_batch_equals_alone():
    """Replicas of different edges at one depth, each bit-identical to itself alone."""
    Ks = (34, 6, 16)
    micros = [voronoi_polycrystal(K, max(2, K ** 3 // 300), 90 + K) for K in Ks]
    for depth in (1, 2):
        print(f"[flat step] batch {Ks} depth={depth}", flush=True)
        common = H.hmc_default_params(Ks[0], 26, 1)
        common.refresh_tile_z = depth
        reps = []
        for K, m in zip(Ks, micros):
            r = H.hmc_default_replica(common, K, m.Q)
            for i in range(6):
                r.sigma_MPa[i] = float(SIG[i])
            reps.append(r)
        b = H.Batch(common, reps)
        for i, m in enumerate(micros):
            b.set_replica(i, m.euler, m.spins)
        b.stress_refresh(STEPS, True)
        for i, (K, m) in enumerate(zip(Ks, micros)):
            p = H.hmc_default_params(K, 26, 1)
            p.refresh_tile_z = depth
            lat = H.Lattice(p, m.Q)
            lat.set_orientations(m.euler)
            lat.set_spins(m.spins)
            lat.set_load(SIG)
            lat.stress_refresh(STEPS, True)
            assert torch.equal(lat.get_stress(), b.get_stress(i)), (depth, K)
            lat.close()
        b.close()


@pytest.mark.parametrize("K", [4, 6, 26, 34])
def test_shallow_adjoint_step_matches_the_deep_one(K):
    """The gradient by the depth-1 adjoint kernel against the tiled kernel at depth 8 (two to five blocks in
    z above K = 8, the last one cut): the same sums in another order.  Each of the FP32 steps, forward and
    backward, adds up to a unit in the last place (6e-8) to its field, so the two stay within 2e-6 of the
    largest derivative over so few of them."""
    m = voronoi_polycrystal(K, max(2, K ** 3 // 300), 95 + K)
    grads = []
    for depth in (1, 8):
        print(f"[flat adjoint] K={K} depth={depth}", flush=True)
        p = H.hmc_default_params(K, 26, 1)
        p.refresh_tile_z = depth
        lat = H.Lattice(p, m.Q)
        lat.set_orientations(m.euler)
        lat.set_spins(m.spins)
        lat.set_load(SIG)
        lat.elastic_forward(STEPS, 15)
        grads.append([np.asarray(g, dtype=np.float64) for g in lat.elastic_backward(1.0)])
        lat.close()
    for flat, deep in zip(*grads):
        assert np.abs(flat - deep).max() <= 2e-6 * np.abs(deep).max()
