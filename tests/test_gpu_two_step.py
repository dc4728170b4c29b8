"""The two-step sweep (and the particle update one step ahead of it) against the
same steps taken one at a time: every bit of the populations, particles, VACF
sums and recorded sums.  The oracle bounds of the single steps therefore hold
for it too."""
import warnings

import numpy as np
import pytest

from helpers import announce

# (box, storage, velocities, friction, particles, options): tiles with
# remainders in x, y and z, rows that are no whole wavefront, one tile across a
# periodic edge, a box of few planes, every friction model
CASES = [
    ((96, 80, 70), "f32", 19, "stokeslet", 40, {}),
    ((100, 77, 71), "f32", 19, "stokeslet_cube", 60, dict(vacf=True)),
    ((201, 201, 53), "f16", 15, "stokeslet", 9, dict(body=True)),
    ((130, 129, 130), "bf16", 19, "stokeslet2dx", 64, dict(series=5)),
    ((33, 257, 64), "f64", 19, "pointwise", 50, dict(fext=True)),
    ((257, 33, 65), "f64", 15, "stokeslet_cube", 50, {}),
    ((1030, 260, 2), "f32", 19, "stokeslet", 31, dict(pair=True, vacf=True)),
    ((20, 164, 165), "bf16", 19, "bd", 100, dict(body=True)),
    ((64, 128, 65), "f32", 19, "stokeslet", 0, dict(body=True, series=3)),
    ((160, 112, 120), "f16", 19, "stokeslet", 400, dict(pair=True)),
]


def _make(case, seed=7):
    from paper_1909_13412_amd import Lattice
    from paper_1909_13412_amd.inputs import particle_positions, particle_velocities, perturbed_fields

    box, storage, q, friction, n, opt = case
    lat = Lattice(*box, 0.7, storage=storage, velocities=q)
    rho, u = perturbed_fields(box[::-1], seed)
    lat.set_equilibrium(rho, u)
    if opt.get("body"):
        lat.set_body_force((1e-5, -2e-5, 3e-6))
    if n:
        r, v = particle_positions(n, box, seed), particle_velocities(n, 1e-3, seed)
        r[0] = (0.0, box[1] - 1e-9, box[2] - 0.25)  # on and across the periodic faces
        r[-1] = np.floor(r[-1]) + 0.5
        if n > 8:
            r[1:5] = r[5] + 0.3 * np.arange(4)[:, None]  # particles sharing nodes
        lat.particles_couple(r, v, mass=10.0, gamma=1.0, kT=1e-4, radius=0.5, seed=seed, friction=friction)
        if opt.get("fext"):
            lat.set_particle_force(1e-3 * np.cos(np.arange(3 * n)).reshape(n, 3))
        if opt.get("pair"):
            lat.set_pair_force(0.05, 1.0)
        if opt.get("vacf"):
            lat.vacf_config(9, 2)
    if opt.get("series"):
        lat.series_config(opt["series"], 4)
    return lat


def _state(lat, case):
    out = {"f": lat.populations().cpu().numpy()}
    if case[4]:
        out["r"], out["v"] = (t.cpu().numpy() for t in lat.particles())
        out["fh"], out["fr"] = (t.cpu().numpy() for t in lat.particle_forces())
        if case[5].get("vacf"):
            acc, cnt = lat.vacf()
            out["acc"], out["cnt"] = acc.cpu().numpy(), cnt
        if case[5].get("pair"):
            out["pair"] = lat.pair_forces().cpu().numpy()
    if case[5].get("series"):
        out["series"] = lat.series()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{'x'.join(map(str, c[0]))}-{c[1]}-q{c[2]}-{c[3]}")
def test_two_step_sweep_equals_single_steps(case):
    announce(f"two-step sweep: {case}")
    ones, twos = _make(case), _make(case)
    taken = 0
    # odd and even starts; five steps hold one two-step sweep too many to keep
    # an even number of them
    for n in (4, 1, 9, 3, 5, 8):
        for _ in range(n):
            ones.step(1)
        twos.profile_enable(True)
        twos.step(n)
        prof = twos.profile_read()
        taken += n - prof["collide_launches"]
        assert prof["particle_launches"] == (n if case[4] else 0)
        a, b = _state(ones, case), _state(twos, case)
        for k in a:
            assert np.array_equal(a[k], b[k]), (k, n)
        assert np.all(np.isfinite(b["f"]))
        # n steps leave the state in the lattice n swaps away
        raw = [(x.pop_a if ones.step_count % 2 == 0 else x.pop_b)[:4096].cpu() for x in (ones, twos)]
        assert bool((raw[0] == raw[1]).all())
        assert ones.step_count == twos.step_count
    # the two-step sweep took part
    assert taken >= 4, taken


@pytest.mark.gpu
def test_particle_set_replaced_after_a_two_step_sweep():
    # The fields of both steps of a sweep are released when another particle
    # set follows, and when a plain step follows.
    case = CASES[0]
    lats = [_make(case), _make(case)]
    from paper_1909_13412_amd.inputs import particle_positions, particle_velocities

    r, v = particle_positions(11, case[0], 3), particle_velocities(11, 1e-3, 3)
    for k, lat in enumerate(lats):
        for n in (4, 1, 4):
            for _ in range(n if k else 1):
                lat.step(1 if k else n)
        lat.particles_couple(r, v, mass=10.0, gamma=1.0, kT=1e-4, radius=0.5, seed=4)
        for n in (1, 4, 2):
            for _ in range(n if k else 1):
                lat.step(1 if k else n)
    a, b = (_state(lat, case) for lat in lats)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


# Boxes of unlike shape (one too small for more than a tile, one with several
# tiles and slabs and remainders), graph replays and plain launches
@pytest.mark.gpu
@pytest.mark.parametrize("storage,friction,graph", [("f32", "stokeslet", True), ("bf16", "stokeslet_cube", False),
                                                    ("f64", "bd", True), ("f16", "pointwise", True),
                                                    ("f64", "stokeslet", False)])
def test_ensemble_two_step_sweep_equals_single_steps(storage, friction, graph):
    from paper_1909_13412_amd import Ensemble, _abi
    from paper_1909_13412_amd.inputs import particle_positions, particle_velocities

    boxes = [((96, 48, 60), 0.7, 40), ((9, 7, 5), 0.9, 3), ((130, 33, 51), 0.8, 25), ((50, 51, 25), 0.65, 70),
             ((320, 128, 89), 0.75, 30)]
    reps = [dict(nx=b[0], ny=b[1], nz=b[2], tau=tau, seed=40 + k, replica=k, r=particle_positions(n, b, k),
                 v=particle_velocities(n, 1e-3, k)) for k, (b, tau, n) in enumerate(boxes)]
    kw = dict(storage=storage, kT=1e-4, radius=0.5, friction=friction)
    announce(f"ensemble two-step sweep: {storage} {friction} graph {graph}")
    ones, twos = Ensemble(reps, **kw), Ensemble(reps, **kw)
    ones.use_graph(False)
    twos.use_graph(graph)
    for e in (ones, twos):
        e.vacf_config(7, 3)
    G = _abi.LBM_ENS_GRAPH_STEPS
    done = replays = 0
    # odd starts, and graphs from every even step number mod 6
    for n in (4, 1, 6, G + 3, 2 * G, 2, G + 5):
        for _ in range(n):
            ones.step(1)
        twos.step(n)
        replays += (n - (done & 1 if n else 0)) // G if graph else 0
        done += n
        assert twos.graph_replays == replays
        for k in range(len(boxes)):
            assert np.array_equal(ones.populations(k).cpu().numpy(), twos.populations(k).cpu().numpy()), (n, k)
        for a, b in ((ones.r, twos.r), (ones.v, twos.v), (ones.vacf()[0], twos.vacf()[0])):
            assert np.array_equal(a.cpu().numpy(), b.cpu().numpy()), n
        assert np.array_equal(ones.vacf()[1], twos.vacf()[1])
        raw = [(x.pop_a if done % 2 == 0 else x.pop_b)[:4096].cpu() for x in (ones, twos)]
        assert bool((raw[0] == raw[1]).all())


@pytest.mark.gpu
@pytest.mark.parametrize("n", [2, 5, 9, 70])
def test_pair_forces_of_crowded_cells(n):
    # More particles of one cell than a walk of its list takes at a time (4),
    # against the sum over all pairs in FP64, in the kernels' rounding.
    from paper_1909_13412_amd import Lattice

    box, rc, a = np.array([12.0, 10.0, 9.0]), 1.5, 0.05
    rng = np.random.default_rng(n)
    r = np.concatenate([np.array([11.9, 0.05, 4.2]) + 0.3 * rng.standard_normal((n, 3)), rng.random((20, 3)) * box])
    lat = Lattice(12, 10, 9, 0.8, storage="f64")
    with warnings.catch_warnings():
        warnings.simplefilter("ignore")  # the volume fraction is beyond the method's range
        lat.particles_couple(r, np.zeros_like(r), kT=0.0, radius=0.5)
    lat.set_pair_force(a, rc)
    for _ in range(2):  # the list is emptied and built again
        pos = lat.particles()[0].cpu().numpy()
        lat.step(1)
        d = pos[:, None] - pos[None]
        d -= box * np.rint(d / box)
        dist = np.sqrt((d * d).sum(2))
        near = (dist > 0) & (dist < rc)
        mag = np.where(near, a * (1 - dist / rc) / np.where(near, dist, 1.0), 0.0)
        ref = (mag[..., None] * d).sum(1)
        # n terms of size <= a, a few roundings each
        assert np.max(np.abs(lat.pair_forces().cpu().numpy() - ref)) <= 16 * (n + 20) * a * 2.0 ** -53
