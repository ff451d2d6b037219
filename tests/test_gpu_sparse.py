"""Worlds that are partly empty.  In long calls tiles whose genes the call has
already written as 0 are passed over, come alive when a gene front reaches them,
and share cells with the tiles moved up at the right and bottom edges.  Cells
whose alpha fails on a gene that is read late lose the genes stored before."""
import numpy as np
import pytest

from paper_2304_05639_amd import inputs

from gpu_helpers import dev

pytestmark = pytest.mark.gpu
STEPS = 12


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2304_05639_amd import lenia
    lenia.lib()
    return lenia


def _front_world(H, W, R):
    """Matter everywhere but in a corner patch, genes in a block that ends nine
    cells before the bottom and right edges: the genes spread by a cell a step."""
    rng = np.random.default_rng(H * W + R)
    w = inputs.test_world(H, W, seed=7, n_blobs=0, dt=0.02, R=R)
    w.A = rng.uniform(0.3, 0.6, (3, H, W)).astype(np.float32)
    w.A[:, 24:40, 12:28] = 0.0
    w.P = np.stack([rng.uniform(lo, hi, (15, H, W)) for lo, hi in ((0.1, 0.4), (0.03, 0.1), (0.1, 1.0))]).astype(np.float32)
    keep = np.zeros((H, W), bool)
    keep[20:H - 9, 10:W - 9] = True
    w.P *= keep
    return w


def _tiles(H, W, ty, tx):
    return [(min(y, H - ty), min(x, W - tx)) for y in range(0, H, ty) for x in range(0, W, tx)]


def _chain(L, w, tile=(16, 32)):
    """The states of STEPS single-step calls (of the one-cell kernel)."""
    plan = L.Plan(w, tile=tile)
    out = [(dev(w.A), dev(w.P))]
    for _ in range(STEPS):
        out.append(plan.step(*out[-1]))
    return out


def _assert_reaches(states, H, W, ty, tx):
    """From the third step of a call on (the first whose buffer the call has
    written before), tiles stay empty and come alive, at the moved edges too."""
    tiles = _tiles(H, W, ty, tx)
    zero = [[not P[:, :, y:y + ty, x:x + tx].any().item() for y, x in tiles] for _, P in states]
    moved = [y % ty != 0 or x % tx != 0 for y, x in tiles]
    stays = [[zero[t - 2][i] and zero[t][i] for i in range(len(tiles))] for t in range(3, STEPS + 1)]
    wakes = [[zero[t - 2][i] and not zero[t][i] for i in range(len(tiles))] for t in range(3, STEPS + 1)]
    for rows in (stays, wakes):
        assert any(any(r) for r in rows)
        assert any(x and m for r in rows for x, m in zip(r, moved))


# at most 256 tiles, and more; 4 x 64 tiles, and 8 x 32 below 64 columns
SIZES = [(97, 161, 12), (97, 63, 12), (261, 321, 12), (1033, 63, 12), (261, 321, 13)]


@pytest.mark.parametrize("H,W,R", SIZES)
@pytest.mark.parametrize("n_steps", [3, STEPS])
def test_long_call_equals_single_steps(L, H, W, R, n_steps):
    import torch
    w = _front_world(H, W, R)
    states = _chain(L, w)
    plan = L.Plan(w)
    i = plan.info()
    _assert_reaches(states, H, W, i.tile_y, i.tile_x)
    A, P = dev(w.A), dev(w.P)
    # other values in the plan's buffers and in the outputs
    plan.step(A, torch.where(P > 0, P, 0.3), n_steps=2)
    A2, P2 = torch.full_like(A, float("nan")), torch.full_like(P, float("nan"))
    plan.step(A, P, A2, P2, n_steps=n_steps)
    assert torch.equal(A2, states[n_steps][0]) and torch.equal(P2, states[n_steps][1])


def test_batch_equals_single_steps(L):
    import torch
    worlds = [_front_world(H, W, 12) for H, W in ((97, 161), (261, 321), (40, 64))]
    As, Ps = [dev(w.A) for w in worlds], [dev(w.P) for w in worlds]
    L.BatchedPlan(worlds).step(As, Ps, n_steps=STEPS)
    for w, A, P in zip(worlds, As, Ps):
        a, p = _chain(L, w)[-1]
        assert torch.equal(A, a) and torch.equal(P, p)


@pytest.mark.parametrize("H,W", [(97, 161), (40, 64)])
def test_ring_long_call_equals_single_steps(L, H, W):
    """(The one-cell ring kernel sums in another order: single steps of the same
    kernel, which a call of one step runs without the tile list.)"""
    import torch
    w = inputs.ring_test_world(H, W, seed=5, n_blobs=0)
    w.A = np.random.default_rng(H).uniform(0.3, 0.6, (3, H, W)).astype(np.float32)
    if H > 80:
        w.P[..., :20, :] = w.P[..., H - 9:, :] = w.P[..., :10] = w.P[..., W - 9:] = 0.0
    else:
        w.P[..., 4:20, :] = 0.0
    states = _chain(L, w, (4, 64))
    if H > 80:
        _assert_reaches(states, H, W, 4, 64)
    plan = L.Plan(w)
    A, P = dev(w.A), dev(w.P)
    plan.step(A, torch.where(P > 0, P, 0.3), n_steps=2)
    A2, P2 = torch.full_like(A, float("nan")), torch.full_like(P, float("nan"))
    plan.step(A, P, A2, P2, n_steps=STEPS)
    assert torch.equal(A2, states[-1][0]) and torch.equal(P2, states[-1][1])


@pytest.mark.parametrize("H,W,R", [(45, 131, 12), (45, 35, 12), (261, 321, 12), (45, 131, 13)])
@pytest.mark.parametrize("dft", [False, True])
def test_genes_that_fail_late(L, oracle, H, W, R, dft):
    """One gene of one kernel is 0 in single cells (which then diffuse from
    their neighbours), in crosses, rows and blocks; another kernel's elsewhere.
    Against the kernel of one cell per lane, and alpha against the oracle's."""
    import torch
    w = _front_world(H, W, R)
    rng = np.random.default_rng(3)
    w.P = np.maximum(w.P, 0.1).astype(np.float32)
    for p, k in ((2, 14), (2, 2), (1, 11), (0, 9)):
        gone = rng.random((H, W)) < 0.002
        gone[rng.integers(H)] = gone[:, rng.integers(W)] = True
        y, x = rng.integers(H - 9), rng.integers(W - 11)
        gone[y:y + 9, x:x + 11] = True
        near = gone.copy()   # disks without any value above the cutoff
        for dy, dx in ((0, 1), (0, -1), (1, 0), (-1, 0)):
            near |= np.roll(gone, (dy, dx), (0, 1))
        w.P[p, k][near] = 0.0
    a, b = (L.Plan(w, conv=3), L.Plan(w, conv=3, dft_fused=True)) if dft else (L.Plan(w), L.Plan(w, tile=(16, 32)))
    A, P = dev(w.A), dev(w.P)
    for n in (1, 3):
        x, y = a.step(A, P, n_steps=n), b.step(A, P, n_steps=n)
        assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1])
    saved = a.new_saved()
    _, P1 = a.step(A, P, saved=saved)
    alpha = a.saved_views(saved)[1].cpu().numpy() != 0
    r = oracle.step(oracle.Desc.from_world(w), w.A, w.P)
    sure = (r["amb"] & 1) == 0
    assert np.array_equal(alpha[sure], (r["alpha"] != 0)[sure])
    assert 0.02 < (~alpha).mean() < 0.9
    assert not P1[:, :, torch.tensor(~alpha, device="cuda")].any()
