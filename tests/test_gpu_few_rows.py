"""Decode steps with few rows: the row-count-dependent kernels give each row the same bits.

Up to 16 rows the projections run on k_skinny_few, up to 64 on k_skinny16 with as many 16-token groups as hold rows; a
row's sums are taken in the same order everywhere, so a call with the first P prompts repeats the first P rows of a
call with 64 bit for bit.  (The 64-row call itself is checked against the oracle in test_gpu_mfma.py.)
"""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2509_08721_amd import sapo
from paper_2509_08721_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = {
    "mini": W.MINI_BF16,
    # down projection long enough for half tiles; tile counts that are no multiple of 8
    "long_ffn": replace(W.MINI_BF16, d_model=384, d_ff=2368, n_layers=3),
    # the widest output in half tiles, next to the prefetching workgroups
    "wide_ffn": replace(W.MINI_BF16, d_model=1280, n_q_heads=20, d_ff=2368),
    # d > 1024: gate/up in units of two tiles, the token-parallel LM head
    "wide": replace(W.MINI_BF16_HD128, d_model=1152, d_ff=640),
}


@pytest.fixture(scope="module", params=sorted(SHAPES))
def full(request):
    shape = SHAPES[request.param]
    gw = sapo.sapo_weights_create(shape, W.make_weights(shape, 31, std=0.05))
    assert gw.uses_mfma
    prompts = torch.from_numpy(np.random.default_rng(5).integers(0, shape.vocab, size=(64, 21)).astype(np.int32)).cuda()
    tok, lp = sapo.sapo_rollout_generate(gw, prompts, 1, 12, 1.0, 17)
    return gw, prompts, tok.cpu().numpy(), lp.cpu().numpy()


@pytest.mark.parametrize("rows", [1, 7, 15, 16, 17, 32, 33, 48, 49, 63])
def test_first_rows_are_bit_identical(full, rows):
    gw, prompts, tok64, lp64 = full
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):   # plain launches, then the captured step
        with torch.cuda.stream(stream):
            tok, lp = sapo.sapo_rollout_generate(gw, prompts[:rows].contiguous(), 1, 12, 1.0, 17)
        torch.cuda.synchronize()
        assert np.array_equal(tok.cpu().numpy(), tok64[:rows])
        assert np.array_equal(lp.cpu().numpy(), lp64[:rows])
