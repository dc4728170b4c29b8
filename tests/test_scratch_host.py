"""Scratch sizes: a box has room for a third node-force field only where particles
can take two-step sweeps in it.  No kernel is launched here."""
import ctypes

import pytest


def _sizes(box, storage, n, q=19):
    from paper_1909_13412_amd import _abi

    lib = _abi.load()
    g = _abi.GridDesc(*box, 0.8, _abi.STORAGE[storage], 16, q, 0)
    grid, part = ctypes.c_size_t(), ctypes.c_size_t()
    assert lib.lbm_grid_scratch_bytes(ctypes.byref(g), ctypes.byref(grid)) == 0
    assert lib.lbm_particle_scratch_bytes(ctypes.byref(g), n, ctypes.byref(part)) == 0
    return grid.value, part.value


@pytest.mark.parametrize("box,storage,n,third", [
    ((256, 256, 256), "f32", 0, False), ((256, 256, 256), "f32", 4096, True), ((256, 256, 256), "bf16", 4096, True),
    ((64, 64, 64), "f64", 16, False), ((128, 128, 64), "f16", 16, False),  # too small
    ((8192, 8192, 4), "f32", 16, False),  # planes of 4 GiB and more
], ids=str)
def test_two_node_force_fields_and_a_third_where_it_is_used(box, storage, n, third):
    cells = box[0] * box[1] * box[2]
    grid, part = _sizes(box, storage, n)
    field = 24 * cells + cells // 8
    # two fields, and sums of every wavefront (32 bytes)
    assert 2 * field <= grid < 2 * field + cells + 1000000
    assert (part >= field) == third
    assert part < 400 * n + (field + 1000000 if third else 0) + 1


@pytest.mark.parametrize("q", [15, 19])
@pytest.mark.parametrize("storage", ["f32", "bf16", "f16", "f64"])
@pytest.mark.parametrize("box", [(256, 256, 256), (64, 64, 64), (8192, 8192, 4)])
def test_scratch_for_many_particles_serves_fewer(box, storage, q):
    sizes = [_sizes(box, storage, n, q)[1] for n in (1, 100, 512, 4000, 5000, 55925, 65536, 65537, 1 << 20, 1 << 24)]
    # (the pair lists of the sets that can have them, too)
    assert sizes == sorted(sizes), sizes


@pytest.mark.parametrize("n,third", [(8, True), (100000, False)])
def test_ensemble_scratch(n, third):
    from paper_1909_13412_amd import _abi

    lib = _abi.load()
    desc = _abi.EnsembleDesc(2, _abi.STORAGE["f32"], 16, _abi.FRICTION["stokeslet"], 10.0, 1.0, 0.0, 0.0, 0, 0)
    reps = (_abi.ReplicaDesc * 2)(*[_abi.ReplicaDesc(128, 128, 96, n, 0.8, k, k, 0) for k in range(2)])
    lat, scr = ctypes.c_size_t(), ctypes.c_size_t()
    assert lib.lbm_ens_bytes(ctypes.byref(desc), reps, ctypes.byref(lat), ctypes.byref(scr)) == 0
    cells = 2 * 128 * 128 * 96
    field = 24 * cells + cells // 8
    rest = 1000000 + 400 * 2 * n
    fields = 3 if third else 2
    assert fields * field <= scr.value < fields * field + rest
