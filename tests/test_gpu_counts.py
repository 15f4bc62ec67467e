"""Counts over the sites against numpy: unlike bonds and texture histograms on lattices from the smallest to
several blocks, and grain labels of a percolating two-spin field, whose one large cluster is united across
many blocks."""
import numpy as np
import pytest

from grains import grain_labels
from paper_1009_0457_amd import hmc as H
from paper_1009_0457_amd.synth import haar_euler, random_spins

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)


def lattice(K, neighbors, Q, spins):
    p = H.hmc_default_params(K, neighbors, 0)
    p.lambda_el = 0.0
    lat = H.Lattice(p, Q)
    euler = haar_euler(np.random.default_rng(K), Q)
    lat.set_orientations(euler)
    lat.set_spins(spins)
    return lat, euler


@pytest.mark.parametrize("neighbors", [6, 26])
@pytest.mark.parametrize("K", [2, 4, 6, 34, 66])
def test_unlike_bonds(K, neighbors):
    print(f"[counts] bonds K={K} neighbors={neighbors}", flush=True)
    spins = random_spins(K, 5, K)
    lat, _ = lattice(K, neighbors, 5, spins)
    f = spins.reshape(K, K, K)
    n = 0
    for dz in (-1, 0, 1):
        for dy in (-1, 0, 1):
            for dx in (-1, 0, 1):
                if (dx, dy, dz) != (0, 0, 0) and (neighbors == 26 or abs(dx) + abs(dy) + abs(dz) == 1):
                    n += np.count_nonzero(f != np.roll(f, (dz, dy, dx), (0, 1, 2)))
    assert lat.energy()[0] == n // 2
    lat.close()


@pytest.mark.parametrize("K", [2, 6, 34, 66])
def test_texture_histogram(K):
    print(f"[counts] texture K={K}", flush=True)
    Q, nbins = 40, 6
    spins = random_spins(K, Q, K + 1)
    lat, euler = lattice(K, 6, Q, spins)
    h = np.asarray(lat.texture_histogram((1.0, 0.0, 0.0)))
    one = np.zeros((Q, nbins), np.int64)   # the bin of each grain, from a field of that grain alone
    for q in range(Q):
        lat.set_spins(np.full(K ** 3, q, np.int32))
        one[q] = np.asarray(lat.texture_histogram((1.0, 0.0, 0.0)))
    assert np.all(one.sum(1) == K ** 3) and np.all((one == 0) | (one == K ** 3))
    assert np.array_equal(h, (np.bincount(spins, minlength=Q)[:, None] * (one > 0)).sum(0))
    lat.close()


@pytest.mark.parametrize("K", [34, 66])
def test_labels_of_a_percolating_field(K):
    print(f"[counts] labels K={K}", flush=True)
    spins = random_spins(K, 2, K + 2)
    lat, _ = lattice(K, 6, 2, spins)
    lab, n = lat.grain_labels()
    lab, ref = lab.cpu().numpy(), grain_labels(spins, K)
    first = np.full(ref.max() + 1, K ** 3)
    np.minimum.at(first, ref, np.arange(K ** 3))
    assert n == ref.max() + 1 and np.array_equal(lab, first[ref])
    lat.close()


@pytest.mark.parametrize("K", [2, 6, 34])
def test_spins_in_and_out_at_any_alignment(K):
    """The wide conversions (16-byte aligned arrays) and the plain ones give back the same spins."""
    print(f"[counts] spins in and out K={K}", flush=True)
    spins = torch.as_tensor(random_spins(K, 9, K + 3)).cuda()
    lat, _ = lattice(K, 6, 9, np.zeros(K ** 3, np.int32))
    for shift in (0, 1):
        store = torch.zeros(K ** 3 + 4, dtype=torch.int32, device="cuda:0")
        view = store[shift:shift + K ** 3]
        view.copy_(spins)
        H.hmc_set_spins(lat.ctx, view)
        out = torch.full((K ** 3 + 4,), -1, dtype=torch.int32, device="cuda:0")
        H.hmc_get_spins(lat.ctx, out[shift:shift + K ** 3])
        lat.synchronize()
        assert torch.equal(out[shift:shift + K ** 3], spins)
        assert bool((out[shift + K ** 3:] == -1).all()) and bool((out[:shift] == -1).all())
    bad = spins.clone()
    bad[K ** 3 - 1] = 9
    with pytest.raises(H.HmcError):
        H.hmc_set_spins(lat.ctx, bad)
    lat.close()
