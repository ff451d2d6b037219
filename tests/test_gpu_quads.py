"""The quad kernels (four cells per lane) at the edges of their range: the
smallest worlds they serve, tiles that end at the right and bottom edge, sides
that no vector width divides."""
import dataclasses

import numpy as np
import pytest

from paper_2304_05639_amd import inputs

from gpu_helpers import TOL_STATE, dev, gpu_step, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_05639_amd import lenia
    lenia.lib()
    return lenia


@pytest.mark.parametrize("H,W,R", [(12, 64, 12), (13, 65, 12), (30, 127, 12), (12, 32, 12), (15, 33, 12),
                                   (41, 63, 12), (13, 64, 13), (22, 70, 13), (13, 35, 13)])
def test_step_equals_one_cell_per_lane(L, H, W, R):
    """The 4 x 64 (and, below 64 columns, 8 x 32) quad step against the step of
    one cell per lane: the same sums in the same order, so the same bits, for
    one step with and without saved potentials and for four steps (zero-gene
    tile flags), on a world with empty, living and masked cells."""
    w = inputs.test_world(H, W, seed=500 + H + W, n_blobs=max(1, H * W // 1200), R=R)
    quads, cells = L.Plan(w), L.Plan(w, tile=(16, 32))
    assert (quads.info().tile_y, quads.info().tile_x) == ((4, 64) if W >= 64 else (8, 32))
    for n in (1, 4):
        a, b = gpu_step(quads, w.A, w.P, n_steps=n), gpu_step(cells, w.A, w.P, n_steps=n)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    sa, sb = quads.new_saved().zero_(), cells.new_saved().zero_()
    a, b = gpu_step(quads, w.A, w.P, saved=sa), gpu_step(cells, w.A, w.P, saved=sb)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    for x, y in zip(quads.saved_views(sa), cells.saved_views(sb)):
        assert np.array_equal(host(x), host(y))


@pytest.mark.parametrize("H,W,R", [(13, 64, 13), (14, 65, 13), (51, 131, 13), (12, 66, 12)])
def test_global_step(L, oracle, H, W, R):
    """Global genes on one channel: the state and the saved potentials against
    the oracle (tolerance of the FP32 form), and a batch of the same world
    against the single plan, bit for bit."""
    import torch
    rng = np.random.default_rng(H * W)
    w = dataclasses.replace(inputs.orbium_like_world(seed=3, R=R), H=H, W=W,
                            A=rng.random((1, H, W)).astype(np.float32))
    plan = L.Plan(w)
    saved = plan.new_saved()
    A1, _ = gpu_step(plan, w.A, None, saved=saved)
    r = oracle.step(oracle.Desc.from_world(w), w.A)
    assert np.abs(A1 - r["A"]).max() <= TOL_STATE
    u, alpha = plan.saved_views(saved)
    assert np.abs(host(u) - r["U"]).max() <= 2e-6 and (host(alpha) == 1).all()
    assert torch.equal(plan.potentials(dev(w.A)), u)
    As = [dev(w.A), dev(w.A)]
    L.BatchedPlan([w, w]).step(As, None, n_steps=1)
    assert all(np.array_equal(host(A), A1) for A in As)


@pytest.mark.parametrize("H,W,R", [(12, 64, 12), (17, 65, 12), (26, 130, 12), (13, 67, 13)])
def test_backward(L, oracle, H, W, R):
    """The adjoint against the oracle's, every cell living and away from the
    clips (so that every entry is compared).  gA and gP: FP32 sums of some 400
    terms, 2e-5 of the largest entry; the shell heights, a difference of such
    sums over all cells, 1e-4."""
    rng = np.random.default_rng(H + W)
    w = inputs.test_world(H, W, seed=7, n_blobs=0, dt=0.02, R=R)
    w.A = rng.uniform(0.3, 0.6, (3, H, W)).astype(np.float32)
    w.P = np.stack([rng.uniform(lo, hi, (15, H, W)) for lo, hi in ((0.1, 0.4), (0.03, 0.1), (0.1, 1.0))]).astype(np.float32)
    gA1 = rng.standard_normal(w.A.shape).astype(np.float32)
    gP1 = rng.standard_normal(w.P.shape).astype(np.float32)
    plan = L.Plan(w)
    A, P = dev(w.A), dev(w.P)
    saved = plan.new_saved()
    plan.step(A, P, saved=saved)
    g = oracle.step_vjp(oracle.Desc.from_world(w), w.A, w.P, gA1, gP1)
    for got, want, tol in zip(plan.backward(A, P, saved, dev(gA1), dev(gP1)), (g["gA"], g["gP"], g["gbeta"]), (2e-5, 2e-5, 1e-4)):
        assert np.abs(host(got) - want).max() <= tol * np.abs(want).max()


@pytest.mark.parametrize("H,W,R", [(4, 64, 12), (5, 65, 12), (25, 63, 12), (51, 131, 13), (40, 96, 12)])
def test_step_from_given_potentials(L, H, W, R):
    """The two-kernel step of the transform form (its second kernel in quads
    where the world holds a 4 x 64 tile) against the one-kernel step, which
    treats one cell at a time: identical bits, and the saved alpha set exactly
    where genes remain."""
    w = inputs.test_world(H, W, seed=900 + H + W, n_blobs=max(1, H * W // 600), R=R)
    two, one = L.Plan(w, conv=3), L.Plan(w, conv=3, dft_fused=True)
    for n in (1, 3):
        a, b = gpu_step(two, w.A, w.P, n_steps=n), gpu_step(one, w.A, w.P, n_steps=n)
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    saved = two.new_saved().zero_()
    a = gpu_step(two, w.A, w.P, saved=saved)
    alpha = host(two.saved_views(saved)[1])
    assert np.array_equal(alpha != 0, (a[1] > 0).any(axis=(0, 1)))
