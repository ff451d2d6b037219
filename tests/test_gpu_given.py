"""The two-kernel step of the transform form: which kernel follows the transforms
depends on the world's size and rows, and every choice gives the same bits."""
import numpy as np
import pytest

from paper_2304_05639_amd import inputs

from gpu_helpers import dev

pytestmark = pytest.mark.gpu


# below and from 2^16 cells; from the size whose 111 planes exceed 256 MiB, rows of
# whole lines, odd rows, and rows that are not whole lines in planes that are, and in
# planes of whole half lines
@pytest.mark.parametrize("H,W", [(1023, 64), (1024, 64), (257, 259), (6000, 100), (787, 768), (788, 768), (779, 779),
                                 (800, 760), (804, 756), (9700, 64)])
def test_two_kernel_step_equals_one_kernel_step(H, W):
    import torch
    from paper_2304_05639_amd import lenia
    g = torch.Generator(device="cuda")
    g.manual_seed(H * W)
    w = inputs.test_world(64, 64, seed=3, n_blobs=0)
    w.H, w.W = H, W
    A = torch.zeros(3, H, W, device="cuda")
    P = torch.rand((3, 15, H, W), generator=g, device="cuda") * 0.3 + 0.05
    # matter in half of the rows, genes that fail in a strip and at single cells
    A[:, :H // 2] = torch.rand((3, H // 2, W), generator=g, device="cuda")
    P[2, 14, :, 10:19] = 0.0
    P[1, 6][torch.rand((H, W), generator=g, device="cuda") < 0.3] = 0.0
    two, one = lenia.Plan(w, conv=3), lenia.Plan(w, conv=3, dft_fused=True)
    for n in (1, 3):
        a, b = two.step(A, P, n_steps=n), one.step(A, P, n_steps=n)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
        assert 0.05 < a[1][0, 0].count_nonzero().item() / (H * W) < 0.6
    saved = two.new_saved()
    a, b = two.step(A, P, saved=saved), one.step(A, P)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert torch.equal(two.saved_views(saved)[1] != 0, a[1].flatten(0, 1).any(0))
