"""The surrogate's two launch forms at the sizes where they change or leave remainders, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2509_08721_amd import sapo
from tests.test_gpu_surrogate import case, run_and_check

pytestmark = pytest.mark.gpu


# 24576 and 16384 tokens (rows of whole groups of four, other rows): the last sizes of the single launch; 1023 .. 1025:
# edges of a gradient block; odd sizes: mask remainders
@pytest.mark.parametrize("S,T", [(1, 15), (1, 17), (11, 93), (1, 1024), (5, 205), (64, 384), (3, 8196), (64, 512), (23, 623), (2, 7169), (57, 575), (8, 4097), (300, 129), (8192, 2), (5462, 3)])
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


@pytest.mark.parametrize("over", ["logp_new", "logp_old"])
@pytest.mark.parametrize("S,T", [(8, 33), (64, 384), (300, 129)])
def test_surrogate_gradient_over_its_inputs(S, T, over):
    """The gradient written over the log-probs it is taken from: what a call with an output of its own gives, at sizes
    that take one launch and two otherwise."""
    ln, lo, mask, adv = case(S, T, 300 + S)
    ref_loss, ref_grad = run_and_check(ln, lo, mask, adv)
    dev = [torch.from_numpy(x).cuda() for x in (ln, lo, mask, adv)]
    out = dev[0] if over == "logp_new" else dev[1]
    loss = torch.empty(1, device="cuda")
    sapo.sapo_clipped_surrogate_noalloc(*dev, loss, out)
    # the sum's order is that of the two launches: fp64, so the loss agrees to the last bits of its fp32
    assert float(loss) == pytest.approx(ref_loss, rel=2e-7) and np.array_equal(out.cpu().numpy().astype(np.float64), ref_grad)
