"""The gradient with its workspace in device-visible memory of another kind than the usual: fine-grained device
memory and managed memory give the gradient of ordinary device memory to the last bit, with both adjoint kernels
(tiles of depth 1, and the tiled step at depth 4)."""
import ctypes as C

import numpy as np
import pytest

from paper_1009_0457_amd import hmc as H
from paper_1009_0457_amd.synth import voronoi_polycrystal

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no HIP device", allow_module_level=True)

K, STEPS, EVERY = 12, 30, 8


class Memory:
    """Device-visible memory of `kind`, with what the bindings ask of a workspace tensor."""

    def __init__(self, kind, nbytes):
        self.hip, self.p, self.n = C.CDLL("libamdhip64.so"), C.c_void_p(), nbytes
        if kind == "managed":
            st = self.hip.hipMallocManaged(C.byref(self.p), C.c_size_t(nbytes), C.c_uint(1))
        else:
            st = self.hip.hipExtMallocWithFlags(C.byref(self.p), C.c_size_t(nbytes), C.c_uint(1))   # fine-grained
        assert st == 0 and self.p.value % 256 == 0

    def data_ptr(self):
        return self.p.value

    def numel(self):
        return self.n

    def free(self):
        assert self.hip.hipFree(self.p) == 0


@pytest.mark.parametrize("kind", ["fine-grained", "managed"])
@pytest.mark.parametrize("depth", [1, 4])
def test_gradient_in_other_memory(kind, depth):
    print(f"[adjoint memory] {kind} depth={depth}", flush=True)
    m = voronoi_polycrystal(K, 8, 5)
    p = H.hmc_default_params(K, 26, 1)
    p.refresh_tile_z = depth
    lat = H.Lattice(p, m.Q)
    lat.set_orientations(m.euler)
    lat.set_spins(m.spins)
    lat.set_load([60.0, -90.0, 120.0, 10.0, 30.0, -20.0])
    U = lat.elastic_forward(STEPS, EVERY)
    euler, load = lat.elastic_backward(1.0)
    ws = Memory(kind, H.hmc_adjoint_workspace_bytes(lat.ctx, STEPS, EVERY))
    assert H.hmc_elastic_forward(lat.ctx, STEPS, EVERY, ws) == U
    e, s = H.hmc_elastic_backward(lat.ctx, ws, 1.0, lat.Q)
    torch.cuda.synchronize()
    assert np.array_equal(e, euler) and np.array_equal(s, load)
    lat.close()
    ws.free()
