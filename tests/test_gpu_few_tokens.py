"""Scoring calls and prompts of few tokens: the GEMM tiles and attention splits chosen by size give every token the same bits.

SAPO_BIG_TILE=256 forces the 256-token tiles (checked against the oracle in test_gpu_mfma.py and test_gpu_full.py); by
default calls of few tokens run on k_gemm_mid / k_gemm_qkv_mid, which keep every output's chain of MFMAs.
"""
import os
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2509_08721_amd import sapo
from paper_2509_08721_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = {
    "hd64": replace(W.MINI_BF16, d_model=384, d_ff=576, n_layers=3, max_seq=1024),
    "hd128": replace(W.MINI_BF16_HD128, max_seq=1024),
}


@pytest.fixture(scope="module", params=sorted(SHAPES))
def model(request):
    shape = SHAPES[request.param]
    gw = sapo.sapo_weights_create(shape, W.perturb_norm_gains(W.make_weights(shape, 41, std=0.05), 41))
    assert gw.uses_mfma
    return shape, gw


# (sequences, tokens each): one token, edges of the 32- and 64-token tiles, sizes that take each of the tiles
@pytest.mark.parametrize("S,T", [(1, 2), (1, 31), (1, 33), (3, 43), (5, 129), (1, 1000), (7, 357), (20, 250)])
def test_scores_are_bit_identical_to_the_large_tiles(model, S, T):
    shape, gw = model
    rng = np.random.default_rng(S * 1000 + T)
    tokens = torch.from_numpy(rng.integers(0, shape.vocab, size=(S, T)).astype(np.int32)).cuda()
    mask = torch.from_numpy((rng.random((S, T)) < 0.6).astype(np.uint8)).cuda()
    rewards = torch.from_numpy(rng.random(S).astype(np.float32)).cuda()
    lp, _ = sapo.sapo_score_logprobs(gw, tokens, mask, rewards, 1)
    os.environ["SAPO_BIG_TILE"] = "256"
    try:
        ref, _ = sapo.sapo_score_logprobs(gw, tokens, mask, rewards, 1)
        torch.cuda.synchronize()
    finally:
        os.environ.pop("SAPO_BIG_TILE", None)
    assert np.array_equal(lp.cpu().numpy(), ref.cpu().numpy())
