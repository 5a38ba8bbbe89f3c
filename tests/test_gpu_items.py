"""Work items of the sweep: results do not depend on their size, bit for bit, and
a lattice whose item list cannot grow stays as it was."""
import numpy as np
import pytest

from paper_1007_1388_amd import inputs, lbm
from tests.helpers import gpu_lattice, prepare

pytestmark = pytest.mark.gpu


def _cavity(n=128):
    rho, u = inputs.perturbed_fields((n, n, n), seed=3, drho=1e-3, du=1e-2)
    return dict(dims=(n, n, n), walls=(True, True, True), wall_u={"+z": (0.05, 0.0, 0.0)}, tau=0.6, init=(rho, u))


class _Deny:
    """Stands in for torch in a lattice's allocator: refuses requests under `limit` bytes."""

    def __init__(self, torch, limit):
        self.cuda, self.torch, self.limit, self.refused = self, torch, limit, 0

    def caching_allocator_alloc(self, n, device, stream):
        if n < self.limit:
            self.refused += 1
            raise MemoryError
        return self.torch.cuda.caching_allocator_alloc(n, device, stream)

    def caching_allocator_delete(self, ptr):
        self.torch.cuda.caching_allocator_delete(ptr)


def test_geometry_that_cannot_grow_the_item_list_leaves_the_lattice():
    """16-bit storage takes twice the items with obstacles: the list is refused, the mask's and the staging memory not."""
    import torch
    case = _cavity()
    solid = inputs.porous_spheres(case["dims"], 0.1, (3, 6), 2, (False,) * 3)
    lat, ref = (gpu_lattice(case, precision="f16s") for _ in range(2))
    for a in (lat, ref):
        prepare(a, case)
        a.step(2)
    items = lat.info()["n_items"]
    lat._alloc.torch = deny = _Deny(torch, 1 << 20)
    with pytest.raises(lbm.LBMError) as e:
        lat.set_geometry(solid)
    assert e.value.status == lbm.LBM_ENOMEM and deny.refused == 1
    lat._alloc.torch = torch
    info = lat.info()
    assert info["n_items"] == items and not info["has_obstacles"]
    for a in (lat, ref):
        a.step(3)
    assert np.array_equal(lat.get_state(as_fp64=False), ref.get_state(as_fp64=False))
    # and with the memory at hand
    for a in (lat, ref):
        a.set_geometry(solid)
        a.step(2)
    assert lat.info()["n_items"] == 2 * items and lat.info()["has_obstacles"]
    assert np.array_equal(lat.get_state(as_fp64=False), ref.get_state(as_fp64=False))
    lat.close()
    ref.close()
