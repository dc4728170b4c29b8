"""Pair repulsion of crowded cells: long cutoffs and clusters cost what their
lists are long, and give the sum over all pairs."""
import time
import warnings

import numpy as np
import pytest

from helpers import announce, nmax_err


def _lattice(r, L, storage="f32"):
    from paper_1909_13412_amd import Lattice

    lat = Lattice(L, L, L, 0.8, storage=storage)
    # no fluid forces: a cluster coupled to the same few nodes would not be stable
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")  # the volume fraction is beyond the method's range
        lat.particles_couple(r, np.zeros_like(r), kT=0.0, radius=0.5, friction="bd")
    return lat


@pytest.mark.gpu
def test_pair_time_grows_no_faster_than_the_lists():
    # 8 and 512 particles per cell: the lists are 64 times as long.  A walk that
    # starts over for every few particles takes a multiple of that.
    import torch

    n, L = 4096, 32
    lat = _lattice(np.random.default_rng(1).random((n, 3)) * L, L)

    def us(a_f, rc):
        lat.set_pair_force(a_f, rc)
        lat.step(2)
        best = np.inf
        for _ in range(3):
            torch.cuda.synchronize()
            t = time.perf_counter()
            lat.step(5)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t) / 5 * 1e6)
        return best

    none, few, many = us(0.0, 1.0), us(1e-9, 4.0), us(1e-9, 16.0)
    announce(f"us per step: no pairs {none:.1f}, 8 per cell {few:.1f}, 512 per cell {many:.1f}")
    assert many - none <= 64 * (few - none)


@pytest.mark.gpu
@pytest.mark.parametrize("n,L,rc,cluster", [(700, 8, 4.0, 0), (900, 24, 1.5, 300), (257, 9, 2.2, 257)])
def test_pair_forces_of_long_lists(n, L, rc, cluster):
    rng, a = np.random.default_rng(n), 0.05
    r = rng.random((n, 3)) * L
    r[:cluster] = np.array([L - 0.1, 0.05, 4.2]) + 0.2 * rng.standard_normal((cluster, 3))
    announce(f"pair forces: {n} particles in {L}^3, cutoff {rc}, cluster of {cluster}")
    lat = _lattice(r, L, "f64")
    lat.set_pair_force(a, rc)
    for _ in range(2):  # the lists are emptied and built again
        pos = lat.particles()[0].cpu().numpy()
        lat.step(1)
        d = pos[:, None] - pos[None]
        d -= L * np.rint(d / L)
        dist = np.sqrt((d * d).sum(2))
        near = (dist > 0) & (dist < rc)
        mag = np.where(near, a * (1 - dist / rc) / np.where(near, dist, 1.0), 0.0)
        ref = (mag[..., None] * d).sum(1)
        # n terms of size <= a, a few roundings each
        err = np.max(np.abs(lat.pair_forces().cpu().numpy() - ref))
        assert err <= 16 * n * a * 2.0 ** -53


@pytest.mark.gpu
@pytest.mark.parametrize("where", [5.0, np.nan, np.inf])
def test_particles_all_in_one_cell(where):
    # the positions of a run that has diverged, or of a careless start; in a
    # sparse box (r_c = 1), whose lists are not put in order
    import torch

    n = 16384
    announce(f"{n} particles at {where}")
    lat = _lattice(np.full((n, 3), where), 32)
    lat.set_pair_force(0.05, 1.0)
    lat.step(1)
    torch.cuda.synchronize()
    t = time.perf_counter()
    lat.step(2)
    torch.cuda.synchronize()
    t = time.perf_counter() - t
    announce(f"{t * 1e3:.1f} ms for two steps")
    # n loads of 1 us, one after another, would be 33 ms; n^2 / 4 of 0.1 us 13 s
    assert t < 1.0
    assert torch.count_nonzero(lat.pair_forces()).item() == 0  # no direction at distance zero


@pytest.mark.gpu
@pytest.mark.parametrize("n,rc,spread", [(34, 4.5, None), (12, 1.2, 1.0)])
def test_adjoint_of_crowded_cells_matches_oracle(oracle_mod, n, rc, spread):
    # lists put in order (34 particles in 8 cells) and a cluster in a sparse box
    from oracle import adjoint as A
    from paper_1909_13412_amd import Lattice
    from test_gpu_adjoint import BOX, _case

    f0, r0, v0, cf, cr, cv = _case(oracle_mod, 21, n=n)
    rng = np.random.default_rng(21)
    r0 = rng.random((n, 3)) * np.array(BOX) if spread is None else 3.0 + spread * rng.random((n, 3))
    cells = np.prod(np.floor(np.array(BOX) / rc))
    assert (n > 4 * cells) == (spread is None)
    theta, N, every, seed = (0.05, 0.8, 10.0, 1e-4), 4, 3, 14  # weak friction: many particles share nodes
    announce(f"adjoint of crowded cells: {n} particles, cutoff {rc}")
    nx, ny, nz = BOX
    lat = Lattice(nx, ny, nz, theta[1], storage="f64")
    lat.set_populations(f0)
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")
        lat.particles_couple(r0, v0, mass=theta[2], gamma=theta[0], kT=theta[3], seed=seed)
    lat.set_pair_force(0.02, rc)
    g = {k: t.cpu().numpy() for k, t in lat.adjoint(lat.record(N, every), cf, cr, cv).items()}
    ref = A.vjp(f0, r0, v0, np.array(theta), A.noise(n, N, seed), cf, cr, cv, pair=(0.02, rc))
    errs = [nmax_err(g[k], x) for k, x in zip(("pop", "r", "v", "params"), ref)]
    announce(f"  errors {errs}")
    assert max(errs) < 1e-10  # the bound of the sparse case, over fewer steps
