"""The explicit step with 8 material points per cell at the edges of its tiles: the smallest meshes, mesh
edges that leave a cut tile in x, y or z, and an odd number of steps (which ends in the other displacement
buffer).  FP32 steps on FP32 tables stay within 1e-6 of the FP64 oracle's field over so few steps (each step
adds about a unit in the last place of the strain, 6e-8)."""
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


@pytest.mark.parametrize("K,steps", [(4, 40), (6, 41), (14, 40), (34, 41), (46, 30)])
def test_step_matches_oracle(K, steps):
    print(f"[mp8 step] K={K} steps={steps}", flush=True)
    m = voronoi_polycrystal(K, max(2, K ** 3 // 300), 110 + K)
    p = H.hmc_default_params(K, 26, 1)
    H.hmc_set_material_points(p, 8)
    lat = H.Lattice(p, m.Q)
    lat.set_orientations(m.euler)
    lat.set_spins(m.spins)
    lat.set_load(SIG)
    lat.stress_refresh(steps, True)
    got = lat.get_stress().cpu().numpy().astype(np.float64)
    Ct, St, _ = O.tables(m.euler, p.C11, p.C12, p.C44)
    _, E, s, info = O.global_solve_mp8(K, m.spins, Ct, St, SIG * 1e-3, steps, True, p.glob_alpha, p.glob_beta,
                                       p.glob_alphaE)
    assert np.linalg.norm(got - s) <= 1e-6 * np.linalg.norm(s)
    assert np.linalg.norm(lat.macro_strain() - E) <= 1e-6 * np.linalg.norm(E)
    assert abs(lat.energy()[1] - info["U"]) <= 2e-6 * abs(info["U"])
    lat.close()


def test_many_blocks_equal_few():
    """Four lattices of 64^3 in one batch have enough blocks that lanes keep their rows from point to point; each
    ends bit-identical to itself alone, where they are read for every point."""
    K, steps = 64, 12
    print("[mp8 step] batch of four", K, flush=True)
    m = voronoi_polycrystal(K, 400, 7)
    common = H.hmc_default_params(K, 26, 1)
    H.hmc_set_material_points(common, 8)
    reps = []
    for r in range(4):
        rep = H.hmc_default_replica(common, K, m.Q)
        for i in range(6):
            rep.sigma_MPa[i] = float(SIG[(i + r) % 6])
        reps.append(rep)
    b = H.Batch(common, reps)
    for r in range(4):
        b.set_replica(r, m.euler, m.spins)
    b.stress_refresh(steps, True)
    lat = H.Lattice(common, m.Q)
    lat.set_orientations(m.euler)
    lat.set_spins(m.spins)
    for r in range(4):
        lat.set_load(np.roll(SIG, -r))
        lat.stress_refresh(steps, True)
        assert torch.equal(lat.get_stress(), b.get_stress(r)), r
    lat.close()
    b.close()
