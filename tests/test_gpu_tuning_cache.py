"""The batch tuner's cache file: an entry answers for the batch it was measured on
and no other, and not for a choice among other passes."""
import hashlib
import json

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1411_7051_amd import Batch, Lattice, inputs  # noqa: E402

SIZES = [(130, 64), (300, 41), (59, 130)]


def batch(**extra):
    out = []
    for i, (nx, ny) in enumerate(SIZES):
        c = inputs.random_medium(nx, ny, seed=i, bc_x=inputs.PRESSURE, rho_in=1.01, rho_out=1.0,
                                 init=1)
        out.append(Lattice(c.eps, c.k, c.kn0, storage="f16", **dict(c.params, **extra)))
    return Batch(out)


def test_entry_of_an_older_file(tmp_path):
    """A file from before tile passes keys a batch by device, storage, boundary
    kinds and sizes alone and names single steps."""
    b = batch()
    d = b.lattices[0].desc
    key = json.dumps([torch.cuda.get_device_name(b.device), int(d.storage), int(d.bc_x),
                      int(d.bc_y), sorted(SIZES)])
    old = hashlib.sha1(key.encode()).hexdigest()[:16]
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({old: [64, 1, 0, 1, 5.0]}))
    assert b.signature() != old
    assert b.autotune(reps=2, cache=str(cache)) > 0  # measured, not answered
    assert set(json.loads(cache.read_text())) == {old, b.signature()}


@pytest.mark.parametrize("extra", [dict(f_eps=0.5), dict(gx=1e-6), dict(correlation=1),
                                   dict(kn_local=0), dict(rho_ref=1.5)])
def test_entries_of_other_models(extra):
    assert batch(**extra).signature() != batch().signature()


def test_round_trip(tmp_path):
    cache = str(tmp_path / "tune.json")
    b = batch()
    assert b.tile_steps > 0
    b.autotune(reps=3, cache=cache)
    c = batch()
    assert np.isnan(c.autotune(cache=cache))
    assert c.tile_steps == b.tile_steps
    assert c.launch == b.launch
    for x in (b, c):
        x.step(23)
    for p, q in zip(b.lattices, c.lattices):
        assert torch.equal(p.save_state(), q.save_state())


@pytest.mark.parametrize("per_launch,want", [(0, "tile"), (1, "single"), (2, "two_step")])
def test_choices_in_the_file(tmp_path, per_launch, want):
    b = batch()
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({b.signature(): [64, 2, 0, per_launch, 5.0]}))
    assert np.isnan(b.autotune(reps=2, cache=str(cache)))
    assert (b.tile_steps > 0) == (want == "tile")
    if want != "tile":
        assert b.steps_per_launch == per_launch
    assert b.launch[:3] == (64, 2, 0)
