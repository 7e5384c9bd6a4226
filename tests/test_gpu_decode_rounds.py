"""Decode projections over several rounds of k steps, and the ways a decode row finds its sequence."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import sapo_oracle as O
from paper_2509_08721_amd import sapo, workloads as W
from tests.parity import oracle_logprobs_for

pytestmark = pytest.mark.gpu

# As in test_gpu_mfma_edges.py.  A k step left out is 1 / 44 of a sum's variance, 0.1 and more in a log-prob here.
LOGPROB_TOL = 2e-2


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.fixture(scope="module")
def model():
    # 44 k steps (QKV, O, gate/up: two rounds of three from 65 rows on) and 164 (down: one step beyond the 20 that a wave of
    # the launch keeps in flight), the last of them for half the waves only
    shape = replace(W.MINI_BF16, d_model=1408, n_q_heads=22, d_ff=5248, vocab=512)
    w = W.make_weights(shape, 41, std=0.02)
    return shape, sapo.sapo_weights_create(shape, w), O.Model(shape, w)


@pytest.mark.parametrize("rows", [1, 16, 17, 40, 64, 70, 130])
def test_rounds_of_k_steps(model, rows):
    shape, gw, oracle = model
    prompts = np.random.default_rng(rows).integers(0, shape.vocab, size=(rows, 9)).astype(np.int32)
    toks, lps = sapo.sapo_rollout_generate(gw, dev(prompts), 1, 4, 1.0, 3)
    toks, lps = toks.cpu().numpy(), lps.cpu().numpy()
    seqs = sorted({0, rows // 2, rows - 1})
    for s, ref in oracle_logprobs_for(oracle, prompts, 1, toks, seqs).items():
        assert np.max(np.abs(lps[s] - ref)) <= LOGPROB_TOL, s


@pytest.mark.parametrize("rows", [3, 24, 100])
def test_rows_by_table_and_in_order_are_the_same(model, rows):
    """Prompts of one length: their lengths given one by one, or a stop token that no row draws, make the attention look
    up each row's sequence and length; neither may change a bit."""
    shape, gw, _ = model
    prompts = np.random.default_rng(rows).integers(0, shape.vocab, size=(rows, 33)).astype(np.int32)
    n_new = min(20, (shape.vocab - 1) // rows)   # fewer draws than ids: one of them is not drawn
    assert n_new >= 4
    toks, lps = sapo.sapo_rollout_generate(gw, dev(prompts), 1, n_new, 1.0, 5)
    by_length = sapo.sapo_rollout_generate_ragged(gw, dev(prompts), [33] * rows, 1, n_new, 1.0, 5)
    assert torch.equal(by_length[0], toks) and torch.equal(by_length[1], lps)
    unused = int(np.setdiff1d(np.arange(shape.vocab), toks.cpu().numpy())[0])
    stopped = sapo.sapo_rollout_generate_stop(gw, dev(prompts), 1, n_new, 1.0, 5, unused)
    assert torch.equal(stopped[0], toks) and torch.equal(stopped[1], lps)
