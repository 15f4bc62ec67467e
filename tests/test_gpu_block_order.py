"""Race detection for the kernels that the sizes of test_gpu_race do not reach: the marched explicit step with tiles of
8, 16 and 32 rows, the marched adjoint step, the zero-load launches of two colours (alone and in a batch) and the
explicit step with 8 points per cell.  Results must be bit-identical under the default, the reversed and the shuffled
order of the work-groups."""
import numpy as np
import pytest

from paper_1009_0457_amd import hmc as H
from paper_1009_0457_amd.synth import haar_euler, random_spins

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

LOAD = [60.0, -90.0, 120.0, 10.0, 30.0, -20.0]


def grains(K, Q, seed, edge=8):
    """Random grains of edge^3 sites."""
    n = -(-K // edge)
    s = random_spins(n, Q, seed).reshape(n, n, n)
    return np.ascontiguousarray(s.repeat(edge, 0).repeat(edge, 1).repeat(edge, 2)[:K, :K, :K]).ravel()


def lattice(K, order, Q=20, **fields):
    p = H.hmc_default_params(K, 26, 1)
    if fields.pop("points", 1) == 8:
        H.hmc_set_material_points(p, 8)
    for k, v in fields.items():
        setattr(p, k, v)
    lat = H.Lattice(p, Q)
    lat.set_block_order(order)
    lat.set_orientations(haar_euler(np.random.default_rng(K), Q))
    lat.set_spins(grains(K, Q, K))
    return lat


def same(outs):
    for o in outs[1:]:
        for a, b in zip(o, outs[0]):
            assert torch.equal(a, b) if torch.is_tensor(a) else np.array_equal(a, b)


# (edge, depth): tiles of 8 rows, of 8 with a remainder in every direction, of 16 (512 blocks of them) and of 32
@pytest.mark.parametrize("K,depth", [(64, 8), (50, 16), (128, 8), (256, 32)])
def test_marched_step(K, depth):
    print(f"[block order] marched step K={K} depth={depth}", flush=True)
    outs = []
    for order in (0, 1, 2):
        lat = lattice(K, order, refresh_tile_z=depth)
        lat.set_load(LOAD)
        lat.stress_refresh(12, True)
        outs.append((lat.get_stress(), lat.macro_strain()))
        lat.close()
    same(outs)


@pytest.mark.parametrize("K,depth", [(40, 2), (40, 8)])
def test_marched_adjoint_step(K, depth):
    print(f"[block order] marched adjoint K={K} depth={depth}", flush=True)
    outs = []
    for order in (0, 1, 2):
        lat = lattice(K, order, refresh_tile_z=depth)
        lat.set_load(LOAD)
        U = lat.elastic_forward(20, 6)
        outs.append((U, *lat.elastic_backward(1.0)))
        lat.close()
    same(outs)


@pytest.mark.parametrize("K", [34, 100])
def test_two_colours_a_launch(K):
    print(f"[block order] two colours K={K}", flush=True)
    outs = []
    for order in (0, 1, 2):
        lat = lattice(K, order, Q=5, lambda_el=0.0, kT=0.8)
        lat.sweep(3)
        outs.append((lat.get_spins(),))
        stats = lat.stats()
        outs[-1] += (stats["accepted"], stats["real_flips"])
        lat.close()
    same(outs)


def test_two_colours_a_launch_in_a_batch():
    K, Q, n = 30, 5, 6
    print("[block order] two colours, batch", flush=True)
    common = H.hmc_default_params(K, 26, 0)
    outs = []
    for order in (0, 1, 2):
        reps = []
        for r in range(n):
            rep = H.hmc_default_replica(common, K, Q)
            rep.kT, rep.seed, rep.lambda_el = 0.8, 20 + r, 0.0
            reps.append(rep)
        b = H.Batch(common, reps)
        b.set_block_order(order)
        for r in range(n):
            b.set_replica(r, haar_euler(np.random.default_rng(1), Q), grains(K, Q, 50 + r, 2))
        b.sweep(3)
        outs.append([b.get_spins(r) for r in range(n)])
        b.close()
    same(outs)


@pytest.mark.parametrize("K", [34, 64])
def test_eight_points_per_cell(K):
    print(f"[block order] 8 points K={K}", flush=True)
    outs = []
    for order in (0, 1, 2):
        lat = lattice(K, order, points=8)
        lat.set_load(LOAD)
        lat.stress_refresh(15, True)
        outs.append((lat.get_stress(), lat.macro_strain()))
        lat.close()
    same(outs)
