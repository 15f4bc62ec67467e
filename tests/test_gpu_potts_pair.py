"""Sweeps at zero load with 26 neighbours, whose launches take two colours each, against the eight single-colour
passes: the same spins and statistics, on edges that fill a block's rows, leave a remainder or need two sites a
thread, for both proposals, alone, in a batch and from a graph."""
import numpy as np
import pytest

from paper_1009_0457_amd import hmc as H
from paper_1009_0457_amd.synth import haar_euler, random_spins

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

SWEEPS = 3


def lattice(K, Q, euler, spins, proposal, seed, stream=None):
    p = H.hmc_default_params(K, 26, 0)
    p.lambda_el, p.kT, p.proposal, p.seed = 0.0, 0.8, proposal, seed
    lat = H.Lattice(p, Q, stream=stream) if stream is not None else H.Lattice(p, Q)
    lat.set_orientations(euler)
    lat.set_spins(spins)
    return lat


def by_colours(lat):
    for s in range(SWEEPS):
        lat.set_sweep_index(s)
        for colour in range(8):
            lat.colour_pass(colour)
    return lat.get_spins().cpu().numpy(), lat.stats()


@pytest.mark.parametrize("proposal", [0, 1])
@pytest.mark.parametrize("K", [2, 4, 6, 34, 64, 100, 206])
def test_pairs_equal_single_colours(K, proposal):
    print(f"[potts pair] K={K} proposal={proposal}", flush=True)
    Q = 5
    spins = random_spins(K // 2, Q, K).reshape((K // 2,) * 3)   # grains of eight sites
    spins = spins.repeat(2, 0).repeat(2, 1).repeat(2, 2).ravel()
    euler = haar_euler(np.random.default_rng(K), Q)
    want, stats = by_colours(lattice(K, Q, euler, spins, proposal, 11))
    for graphs in (False, True):
        lat = lattice(K, Q, euler, spins, proposal, 11, torch.cuda.Stream() if graphs else None)
        if graphs:
            lat.set_graphs(True)
        lat.sweep(SWEEPS)
        got = lat.get_spins()
        lat.synchronize()   # the lattice's own stream
        assert np.array_equal(got.cpu().numpy(), want), graphs
        assert lat.stats() == stats, graphs
        lat.close()


def test_batch_pairs_equal_single_colours():
    K, Q = 30, 4
    print(f"[potts pair] batch of five {K}", flush=True)
    common = H.hmc_default_params(K, 26, 0)
    common.lambda_el = 0.0
    euler = haar_euler(np.random.default_rng(1), Q)
    reps, fields = [], []
    for r in range(5):
        rep = H.hmc_default_replica(common, K, Q)
        rep.kT, rep.seed, rep.lambda_el = 0.8, 20 + r, 0.0
        reps.append(rep)
        fields.append(random_spins(K, Q, 50 + r))
    b = H.Batch(common, reps)
    for r in range(5):
        b.set_replica(r, euler, fields[r])
    b.sweep(SWEEPS)
    for r in range(5):
        want, _ = by_colours(lattice(K, Q, euler, fields[r], 0, 20 + r))
        assert np.array_equal(b.get_spins(r).cpu().numpy(), want), r
    b.close()
