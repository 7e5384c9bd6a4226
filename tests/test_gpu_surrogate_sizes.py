"""The surrogate's two launch forms at the sizes where they change or leave remainders, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2509_08721_amd import sapo
from tests.test_gpu_surrogate import case, run_and_check

pytestmark = pytest.mark.gpu


# 24576 and 14336 tokens (rows of whole groups of four, other rows): the last sizes of the single launch; 1023 .. 1025:
# edges of a gradient block; odd sizes: mask remainders
@pytest.mark.parametrize("S,T", [(1, 15), (1, 17), (11, 93), (1, 1024), (5, 205), (64, 384), (3, 8196), (64, 512), (23, 623), (2, 7169), (57, 575), (8, 4097), (300, 129)])
def test_surrogate_sizes(S, T):
    run_and_check(*case(S, T, 100 + S))


@pytest.mark.parametrize("n_rows", [8, 320])
def test_surrogate_mask_bytes_and_alignment(n_rows):
    """Any non-zero mask byte counts, a mask that is not 16-byte aligned gives the same result, and so does a call
    without a gradient."""
    ln, lo, mask, adv = case(n_rows, 130, 7)
    dev = [torch.from_numpy(x).cuda() for x in (ln, lo, mask, adv)]
    loss, grad = sapo.sapo_clipped_surrogate(*dev)
    rng = np.random.default_rng(1)
    odd = torch.from_numpy((mask * rng.integers(1, 256, mask.shape)).astype(np.uint8)).cuda()
    shifted = torch.empty(odd.numel() + 3, dtype=torch.uint8, device="cuda")[3:].view(odd.shape)
    shifted.copy_(odd)
    loss2, grad2 = sapo.sapo_clipped_surrogate(dev[0], dev[1], odd, dev[3])
    loss3, grad3 = sapo.sapo_clipped_surrogate(dev[0], dev[1], shifted, dev[3])
    loss4, none = sapo.sapo_clipped_surrogate(*dev, want_grad=False)
    assert none is None
    assert torch.equal(grad, grad2) and torch.equal(grad, grad3)
    assert float(loss) == float(loss2) == float(loss4) and float(loss3) == pytest.approx(float(loss), rel=1e-6)
