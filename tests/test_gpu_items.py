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


def _items(dims, rows):
    return dims[2] * -(-dims[1] // rows)


def test_explicit_item_cells_are_taken_as_they_are():
    """Any value but the default, whatever the sweep would choose: rows of item_cells / nx, 16-bit rows rounded up to
    whole rounds of the four waves (a 64-cell row is one task)."""
    dims = (64, 96, 80)
    for prec, wants in (("f64", {64: 1, 256: 4, 511: 7, 1024: 16}), ("f32", {64: 1, 256: 4, 511: 7, 1024: 16}),
                        ("f16s", {64: 4, 256: 4, 448: 8, 1024: 16})):
        lat = lbm.Lattice(dims, walls=(True,) * 3, tau=0.6, precision=prec)
        for cells, rows in wants.items():
            lat.set_schedule(item_cells=cells)
            assert lat.info()["n_items"] == _items(dims, rows), (prec, cells)
            assert lat.schedule["item_cells"] == cells
        lat.close()


@pytest.mark.parametrize("prec,dims,chosen,whole", [
    ("f64", (128, 64, 96), 2, 4), ("f32", (256, 60, 96), 1, 2),      # half
    ("f64", (64, 32, 32), 4, 8),                                     # half: few items
    ("f64", (192, 40, 64), 2, 2),                                    # three tasks a row: whole
    ("f16s", (128, 128, 128), 8, 4), ("bf16s", (256, 96, 96), 4, 2),  # double
    ("f16s", (160, 128, 110), 4, 4), ("f16s", (128, 64, 64), 4, 4),  # 640-cell items already; few items
])
def test_the_sweeps_choice_of_items(prec, dims, chosen, whole):
    """item_cells = 512 against the same lattice with whole items (520 cells): fewer or more items, the same bits."""
    rho, u = inputs.perturbed_fields(dims, seed=3, drho=1e-3, du=1e-2)
    case = dict(dims=dims, walls=(True, True, True), wall_u={"+z": (0.05, 0.0, 0.0)}, tau=0.6, init=(rho, u))
    a, b = (gpu_lattice(case, precision=prec) for _ in range(2))
    b.set_schedule(item_cells=520)
    for lat in (a, b):
        prepare(lat, case)
        lat.step(3)
    assert (a.info()["n_items"], b.info()["n_items"]) == (_items(dims, chosen), _items(dims, whole))
    assert np.array_equal(a.get_state(as_fp64=False), b.get_state(as_fp64=False))
    a.close()
    b.close()


def test_obstacles_come_and_go_on_a_lattice_whose_items_change():
    case = _cavity()
    solid = inputs.porous_spheres(case["dims"], 0.1, (3, 6), 2, (False,) * 3)
    a, b = (gpu_lattice(case, precision="f16s") for _ in range(2))
    b.set_schedule(item_cells=520)
    for mask, items in ((None, 2048), (solid, 4096), (1 - solid, 4096), (None, 2048), (solid, 4096)):
        for lat in (a, b):
            lat.set_geometry(mask)
            if mask is None:
                prepare(lat, case)
            lat.step(3)
        assert (a.info()["n_items"], b.info()["n_items"]) == (items, 4096)
        assert np.array_equal(a.get_state(as_fp64=False), b.get_state(as_fp64=False))
    a.close()
    b.close()


def test_autotune_skips_lines_of_another_meaning_of_item_cells(tmp_path):
    """A cached choice whose key lacks the mark of the present meaning does not count."""
    cache = str(tmp_path / "tune.txt")
    case = _cavity(32)
    lat = gpu_lattice(case, precision="f32")
    lat.autotune(cache, trial_steps=1)
    line = open(cache).read()
    assert "|i2|" in line
    with open(cache, "w") as fh:
        fh.write(line.replace("|i2|", "|"))
    lat.autotune(cache, trial_steps=1)
    assert len([l for l in open(cache).read().splitlines() if l.strip()]) == 2
    lat.close()
