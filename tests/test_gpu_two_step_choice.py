"""Which ensembles take two-step sweeps."""
import numpy as np
import pytest

from helpers import announce


def _ensemble(box, n, storage="f32", boxes=2):
    from paper_1909_13412_amd import Ensemble
    from paper_1909_13412_amd.inputs import particle_positions

    reps = [dict(nx=box[0], ny=box[1], nz=box[2], tau=0.8, seed=k, replica=k, r=particle_positions(n, box, k),
                 v=np.zeros((n, 3))) for k in range(boxes)]
    return Ensemble(reps, storage=storage, kT=1e-4, radius=0.5)


@pytest.mark.gpu
def test_remembered_choice_follows_the_particles_at_hand():
    # 262 and 160000 nodes per particle: the first are too dense for two-step sweeps
    dense, sparse, box = 5000, 8, (128, 128, 80)
    announce("ensemble choice: tuned dense, then sparse; tuned sparse, then dense")
    first = _ensemble(box, dense)
    assert not first.two_step
    first.autotune(3)
    assert not first.two_step
    later = _ensemble(box, sparse)
    assert later.two_step  # nothing was tried against it
    later.autotune(3)
    assert _ensemble(box, sparse).two_step == later.two_step
    assert not _ensemble(box, dense).two_step
