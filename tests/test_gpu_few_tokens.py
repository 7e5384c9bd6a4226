"""Scoring calls and prompts of few tokens: the GEMM tiles and attention splits chosen by size give every token the same bits.

SAPO_BIG_TILE=256 forces the 256-token tiles (checked against the oracle in test_gpu_mfma.py and test_gpu_full.py); by
default calls of few tokens run on k_gemm_mid / k_gemm_qkv_mid, which keep every output's chain of MFMAs.  The query heads
per wave of the attention follow the number of sequences, and the vocabulary groups of the scorer the number of scored rows, not
that switch: a call of few sequences is compared with the same sequences in a larger one for those.
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


# two layers each: attention waves of 1, 2 and 4 heads at head dim 64 (1, 8 and 16 sequences of 300), 1 and 2 heads at 128;
# scorer groups of several sizes
@pytest.mark.parametrize("shape", [replace(W.HALF_B, n_layers=2), replace(W.ONE_HALF_B, n_layers=2)], ids=["hd64", "hd128"])
def test_a_sequence_scores_the_same_alone_and_among_others(shape):
    gw = sapo.sapo_weights_create(shape, W.make_weights(shape, 43))
    assert gw.uses_mfma
    rng = np.random.default_rng(44)
    S, T = 16, 300
    tokens = torch.from_numpy(rng.integers(0, shape.vocab, size=(S, T)).astype(np.int32)).cuda()
    mask = torch.ones((S, T), dtype=torch.uint8, device="cuda")
    rewards = torch.zeros(S, device="cuda")
    positions = [(0, 0), (0, 15), (0, 16), (0, 100), (0, 255), (0, 256), (0, 299)]
    logits = sapo.sapo_debug_logits(gw, tokens, positions)
    lp, _ = sapo.sapo_score_logprobs(gw, tokens, mask, rewards, 1)
    for n in (1, 2, 8):
        few = tokens[:n].contiguous()
        assert torch.equal(sapo.sapo_debug_logits(gw, few, positions), logits)      # layers and attention: every bit
        a, _ = sapo.sapo_score_logprobs(gw, few, mask[:n].contiguous(), rewards[:n].contiguous(), 1)
        assert torch.equal(a, lp[:n])
        again, _ = sapo.sapo_score_logprobs(gw, few, mask[:n].contiguous(), rewards[:n].contiguous(), 1)
        assert torch.equal(a, again)
    gw.close()


# the last one's (max, sum of exponentials) pairs take more than the layers' buffers, where they lie
@pytest.mark.parametrize("shape", [replace(W.HALF_B, n_layers=1), replace(W.MINI_BF16, max_seq=1024),
                                   replace(W.MINI_BF16, n_layers=1, vocab=131072, max_seq=1024)],
                         ids=["vocabulary of 151936", "mini", "mini with a vocabulary of 131072"])
def test_log_probs_keep_their_bits_whatever_else_is_scored(shape):
    """The scorer's workgroups follow the number of rows that the masks name; a sequence's log-probs are the same bits with other
    sequences' masks empty, sparse or full, with fewer sequences, and at positions its own mask adds none to."""
    gw = sapo.sapo_weights_create(shape, W.make_weights(shape, 45))
    rng = np.random.default_rng(46)
    S, T = 14, 301
    tokens = torch.from_numpy(rng.integers(0, shape.vocab, size=(S, T)).astype(np.int32)).cuda()
    rewards = torch.zeros(S, device="cuda")
    full = torch.ones((S, T), dtype=torch.uint8, device="cuda")
    want, _ = sapo.sapo_score_logprobs(gw, tokens, full, rewards, 1)
    for share in (0.0, 0.05, 0.3, 0.8):
        mask = torch.from_numpy((rng.random((S, T)) < share).astype(np.uint8)).cuda()
        mask[0] = 1
        lp, _ = sapo.sapo_score_logprobs(gw, tokens, mask, rewards, 1)
        assert torch.equal(lp, torch.where(mask != 0, want, torch.zeros_like(want))), share
    for n in (1, 3, 9):
        lp, _ = sapo.sapo_score_logprobs(gw, tokens[:n].contiguous(), full[:n].contiguous(), rewards[:n].contiguous(), 1)
        assert torch.equal(lp, want[:n]), n
    gw.close()


def test_workspace_of_scoring_has_no_room_of_its_own_for_the_scorer():
    """A call's workspace is what its layers need, the rows to score and their final norms: a (max, sum of exponentials) per row
    and 128 entries of the vocabulary, 467 MB here, lies where the layers' buffers were."""
    shape = replace(W.HALF_B, n_layers=1)
    gw = sapo.sapo_weights_create(shape, W.make_weights(shape, 47))
    S, T = 64, 768
    d, q, kv, F = shape.d_model, shape.q_dim, shape.kv_dim, shape.d_ff
    layers = 4 * d + 2 * d + 4 * (q + 2 * kv) + 2 * q + 2 * q + 2 * F + 4 * (d // 64 + 3)   # bytes per token
    assert sapo.sapo_score_workspace_bytes(gw, S, T) <= S * T * (layers + 2 * 2 * kv * shape.n_layers + 2 * d + 12) + (1 << 20)
    gw.close()
