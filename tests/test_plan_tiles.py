"""The tile a plan reports is the tile its step kernel runs on, and can be asked
for; the autotuner's stored choices belong to the kernels they were timed on."""
import dataclasses

import numpy as np
import pytest

from paper_2304_05639_amd import inputs, lenia


def _global_world(H, W, R=13):
    rng = np.random.default_rng(H * W)
    return dataclasses.replace(inputs.orbium_like_world(seed=3, R=R), H=H, W=W,
                               A=rng.random((1, H, W)).astype(np.float32))


def _tile(plan):
    i = plan.info()
    return i.tile_y, i.tile_x


@pytest.mark.parametrize("H,W,ok", [(13, 64, True), (12, 64, False), (64, 63, False)])
def test_quad_tile_of_global_worlds_validates_where_it_fits(H, W, ok):
    w = _global_world(H, W)
    assert (lenia.validate(w, tile=(4, 64)) == lenia.OK) == ok
    for tile in ((8, 32), (16, 32)):
        assert lenia.validate(w, tile=tile) == lenia.OK
    # localized genes on one channel have no such form
    loc = dataclasses.replace(w, localized=1, genotype_update=0, m=None, s=None, h=None)
    assert lenia.validate(loc, tile=(4, 64)) == lenia.ERR_UNSUPPORTED


def test_quad_tile_of_ring_worlds_validates_where_it_fits():
    for H, W, ok in ((12, 64, True), (11, 64, False), (64, 63, False)):
        w = inputs.ring_test_world(H, W, seed=1, n_blobs=1)
        assert (lenia.validate(w, tile=(4, 64)) == lenia.OK) == ok
        assert lenia.validate(w, tile=(8, 32)) == lenia.OK


@pytest.mark.gpu
@pytest.mark.parametrize("H,W,default", [(13, 64, (4, 64)), (40, 100, (4, 64)), (40, 63, (8, 32))])
def test_global_plan_reports_the_tile_that_runs(H, W, default):
    """The 4 x 64 form sums in another order than the one-cell kernels, so the
    bits tell which kernel ran: the default's are those of its own tile asked
    for, and those of 8 x 32 are those of 16 x 32 (each cell's sums do not
    depend on the one-cell kernel's tile)."""
    import torch
    w = _global_world(H, W)
    A = torch.tensor(w.A, device="cuda")
    plan = lenia.Plan(w)
    assert _tile(plan) == default
    A1 = plan.step(A)[0]
    again = lenia.Plan(w, tile=default)
    assert _tile(again) == default and torch.equal(again.step(A)[0], A1)
    u = []
    for tile in ((8, 32), (16, 32)):
        p = lenia.Plan(w, tile=tile)
        assert _tile(p) == tile
        u.append(p.potentials(A))
    assert torch.equal(u[0], u[1])
    assert torch.equal(plan.potentials(A), u[0]) == (default != (4, 64))
    b = lenia.BatchedPlan([w, w])
    assert _tile(b) == default


@pytest.mark.gpu
def test_global_plan_is_not_autotuned(tmp_path, monkeypatch):
    """One form fits, so there is nothing to time and nothing to store."""
    monkeypatch.setenv("LENIA_TUNE_CACHE", str(tmp_path / "tune.txt"))
    assert _tile(lenia.Plan(_global_world(40, 100), autotune=True)) == (4, 64)
    assert not (tmp_path / "tune.txt").exists()


# (290 tiles of 4 x 64 and 219 of 8 x 32, 525 and 494, 2500 and 1875; 256 and 256,
# 896 and 832, 750 and 564)
@pytest.mark.gpu
@pytest.mark.parametrize("H,W,default", [(577, 86, (8, 32)), (300, 400, (8, 32)), (5000, 80, (8, 32)),
                                           (256, 256, (4, 64)), (512, 400, (4, 64)), (1500, 70, (4, 64))])
def test_ring_default_fills_compute_units_evenly(H, W, default):
    w = inputs.ring_test_world(64, 64, seed=1, n_blobs=1)
    w.H, w.W = H, W
    assert _tile(lenia.Plan(w)) == default
    assert _tile(lenia.Plan(w, tile=(4, 64))) == (4, 64)


@pytest.mark.gpu
@pytest.mark.parametrize("H,W,default", [(12, 64, (4, 64)), (30, 63, (8, 32))])
def test_ring_plan_reports_the_tile_that_runs(H, W, default):
    import torch
    w = inputs.ring_test_world(H, W, seed=1, n_blobs=1)
    A, P = torch.tensor(w.A, device="cuda"), torch.tensor(w.P, device="cuda")
    plan, again = lenia.Plan(w), lenia.Plan(w, tile=default)
    assert _tile(plan) == _tile(again) == default
    assert all(torch.equal(x, y) for x, y in zip(plan.step(A, P), again.step(A, P)))
    assert _tile(lenia.Plan(w, tile=(8, 32))) == (8, 32)


@pytest.mark.gpu
def test_stored_choices_of_other_kernels_are_not_taken(tmp_path, monkeypatch):
    """A choice stored under a key that does not name the kernels it was timed on
    (as earlier versions wrote it) is timed again, and two batches that differ
    in a later world only do not share one."""
    import torch
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("LENIA_TUNE_CACHE", str(cache))
    worlds = [inputs.test_world(64, 64, seed=40 + i, n_blobs=1) for i in range(5)]
    narrow = inputs.test_world(64, 48, seed=45, n_blobs=1)
    arch = torch.cuda.get_device_properties(0).gcnArchName
    # 3-channel table (1), updated genes (mode 2)
    old = [f"{arch}:t1:R12:m2:single:64x64:n1 16 32 0.001",
           f"{arch}:t1:R12:m2:batch:64x64:64x64:64x64:64x64:n5 16 32 0.001"]
    cache.write_text("\n".join(old) + "\n")
    lenia.Plan(worlds[0], autotune=True)
    assert len(cache.read_text().splitlines()) == 3
    for n, batch in enumerate((worlds, worlds[:4] + [narrow])):
        first = _tile(lenia.BatchedPlan(batch, autotune=True))
        lines = cache.read_text().splitlines()
        assert len(lines) == 4 + n                    # timed and stored
        assert tuple(map(int, lines[-1].split()[1:3])) == first
        assert _tile(lenia.BatchedPlan(batch, autotune=True)) == first
        assert len(cache.read_text().splitlines()) == 4 + n   # found
