"""The small-decoder kernels (one workgroup per sequence) against the shape-generic ones, which the other tests hold to
the oracle: tile edges, both prefill forms, every attention form, ragged prompts, stop tokens, biases."""
import os
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2509_08721_amd import sapo, workloads as W

pytestmark = pytest.mark.gpu

SHAPES = {
    "tiny": W.TINY,
    "hd12": replace(W.TINY, n_q_heads=9, n_kv_heads=3, head_dim=12, d_model=36, d_ff=100, vocab=301),   # no matrix-core attention
    "hd32": replace(W.TINY, n_q_heads=2, n_kv_heads=1, head_dim=32, d_model=132, d_ff=260, n_layers=3, vocab=1003),
    "hd64": replace(W.TINY, n_q_heads=10, n_kv_heads=5, head_dim=64, d_model=60, d_ff=64, n_layers=1, vocab=600),
}


def handles(shape, seed, bias=False):
    w = W.perturb_norm_gains(W.make_weights(shape, seed, std=0.05), seed)
    if bias:
        w = W.add_qkv_bias(w, shape, seed)
    small = sapo.sapo_weights_create(shape, w)
    os.environ["SAPO_FORCE_GENERIC"] = "1"
    try:
        generic = sapo.sapo_weights_create(shape, w)
    finally:
        del os.environ["SAPO_FORCE_GENERIC"]
    return small, generic


def kernels_of(call):
    """The kernels a call launches."""
    sapo.sapo_profile_start()
    call()
    return set(sapo.sapo_profile_stop())


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("S,T,G", [(1, 1, 1), (4, 15, 2), (3, 16, 3), (6, 17, 2), (5, 33, 1), (2, 130, 1)])
def test_small_scoring(name, S, T, G):
    shape = SHAPES[name]
    small, generic = handles(shape, 11, bias=name == "hd32")
    rng = np.random.default_rng(S * T)
    tok = torch.from_numpy(rng.integers(0, shape.vocab, (S, T)).astype(np.int32)).cuda()
    mask = torch.from_numpy((rng.random((S, T)) < 0.5).astype(np.uint8)).cuda()
    rew = torch.from_numpy((rng.random(S) < 0.5).astype(np.float32)).cuda()
    assert kernels_of(lambda: sapo.sapo_score_logprobs(small, tok, mask, rew, G)) == {"k_small"}
    for temp in (1.0, 0.7):
        a = sapo.sapo_score_logprobs_at(small, tok, mask, rew, G, temp)
        b = sapo.sapo_score_logprobs_at(generic, tok, mask, rew, G, temp)
        assert float((a[0] - b[0]).abs().max()) <= 2e-5 and torch.equal(a[1], b[1])


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("P,G,Lp,N", [(1, 1, 1, 1), (2, 3, 16, 5), (3, 2, 17, 40), (2, 2, 100, 3)])
def test_small_rollouts(name, P, G, Lp, N):
    shape = SHAPES[name]
    small, generic = handles(shape, 12, bias=name == "hd64")
    rng = np.random.default_rng(P * Lp + N)
    prompts = torch.from_numpy(rng.integers(0, shape.vocab, (P, Lp)).astype(np.int32)).cuda()
    for temp in (1.0, 0.0):
        a = sapo.sapo_rollout_generate(small, prompts, G, N, temp, 5)
        b = sapo.sapo_rollout_generate(generic, prompts, G, N, temp, 5)
        assert torch.equal(a[0], b[0]) and float((a[1] - b[1]).abs().max()) <= 2e-5
    # prompts of different lengths, with a stop token that some row emits
    lens = [int(x) for x in rng.integers(1, Lp + 1, P)]
    stop = int(a[0][0, N // 2])
    for st in (-1, stop):
        a = sapo.sapo_rollout_generate_ragged(small, prompts, lens, G, N, 1.0, 6, stop_token=st)
        b = sapo.sapo_rollout_generate_ragged(generic, prompts, lens, G, N, 1.0, 6, stop_token=st)
        assert torch.equal(a[0], b[0]) and float((a[1] - b[1]).abs().max()) <= 2e-5
        assert st < 0 or torch.equal(a[2], b[2])


@pytest.mark.parametrize("P,G,Lp,N", [(2, 2, 18, 9), (1, 3, 30, 45), (2, 1, 380, 21)])
def test_small_rollouts_by_what_fits_in_lds(P, G, Lp, N):
    """A sequence's keys and values and the LM head in LDS (contexts of 27), the keys and values alone (75), neither (401)."""
    shape = replace(W.TINY, max_seq=512)
    small, generic = handles(shape, 21)
    prompts = torch.from_numpy(np.random.default_rng(Lp).integers(0, shape.vocab, (P, Lp)).astype(np.int32)).cuda()
    assert kernels_of(lambda: sapo.sapo_rollout_generate(small, prompts, G, N, 1.0, 8)) == {"k_small"}
    a = sapo.sapo_rollout_generate(small, prompts, G, N, 1.0, 8)
    b = sapo.sapo_rollout_generate(generic, prompts, G, N, 1.0, 8)
    assert torch.equal(a[0], b[0]) and float((a[1] - b[1]).abs().max()) <= 2e-5


@pytest.mark.parametrize("hd", [12, 16, 32, 64])
def test_small_bf16_rollouts_are_scored_alike(hd):
    """bf16: a rollout's log-probs are those that scoring gives its tokens (roundings to bf16 may fall either way)."""
    shape = replace(W.TINY, dtype="bf16", head_dim=hd, d_model=64 if hd != 12 else 48)
    small, _ = handles(shape, 22)
    prompts = torch.from_numpy(np.random.default_rng(hd).integers(0, shape.vocab, (2, 13)).astype(np.int32)).cuda()
    tok, lp = sapo.sapo_rollout_generate(small, prompts, 3, 30, 1.0, 9)
    seqs = torch.cat([prompts.repeat_interleave(3, 0), tok], 1).contiguous()
    mask = torch.zeros_like(seqs, dtype=torch.uint8)
    mask[:, 13:] = 1
    ref = sapo.sapo_score_logprobs(small, seqs, mask, torch.zeros(6, device="cuda"), 3)[0][:, 13:]
    assert float((ref - lp).abs().max()) <= 2e-2


def test_small_norm_of_rows_whose_squares_overflow():
    """Residuals of 1e20: their sum of squares is infinite, its inverse root 0 and the normalised row 0, as in the generic kernels, so
    the logits behind such a token are all 0 (untied head)."""
    shape = replace(W.TINY, tied_embeddings=False)
    w = W.make_weights(shape, 23, std=0.05)
    w["embed"][3:6] *= 1e21
    small = sapo.sapo_weights_create(shape, w)
    os.environ["SAPO_FORCE_GENERIC"] = "1"
    try:
        generic = sapo.sapo_weights_create(shape, w)
    finally:
        del os.environ["SAPO_FORCE_GENERIC"]
    tok = torch.tensor([[9, 3, 17, 4, 4, 30, 5, 11]], dtype=torch.int32, device="cuda")
    a, b = (sapo.sapo_score_logprobs(h, tok, torch.ones_like(tok, dtype=torch.uint8), torch.zeros(1, device="cuda"), 1)[0][0] for h in (small, generic))
    assert float((a - b).abs().max()) <= 2e-5 and float((a[[2, 4, 5, 7]] + np.log(shape.vocab)).abs().max()) <= 2e-5
    for prompt in (tok, tok[:, :5].contiguous()):
        a, b = (sapo.sapo_rollout_generate(h, prompt, 2, 6, 1.0, 4) for h in (small, generic))
        assert torch.equal(a[0], b[0]) and float((a[1] - b[1]).abs().max()) <= 2e-5


def test_small_bf16_follows_the_generic_kernels():
    shape = replace(W.TINY, dtype="bf16")
    small, generic = handles(shape, 13)
    assert not small.uses_mfma
    rng = np.random.default_rng(3)
    tok = torch.from_numpy(rng.integers(0, shape.vocab, (4, 50)).astype(np.int32)).cuda()
    mask = torch.ones((4, 50), dtype=torch.uint8, device="cuda")
    rew = torch.zeros(4, device="cuda")
    a, b = (sapo.sapo_score_logprobs(h, tok, mask, rew, 2)[0] for h in (small, generic))
    assert float((a - b).abs().max()) <= 2e-2     # roundings to bf16 may fall either way


def test_large_models_do_not_take_the_small_path():
    shape = replace(W.TINY, d_model=512, n_q_heads=8, n_kv_heads=8, head_dim=64, d_ff=2048)
    w = sapo.sapo_weights_create(shape, W.make_weights(shape, 1))
    tok = torch.zeros((1, 8), dtype=torch.int32, device="cuda")
    names = kernels_of(lambda: sapo.sapo_score_logprobs(w, tok, torch.ones_like(tok, dtype=torch.uint8), torch.zeros(1, device="cuda"), 1))
    assert "k_small" not in names


def test_large_batches_leave_the_small_path():
    """Thousands of sequences cost the small path a round of workgroups per 256 of them; from some size on the generic
    kernels take the call.  The rows are the same: the first prompts of a large call repeat a small call's tokens."""
    shape = W.TINY
    small, _ = handles(shape, 14)
    rng = np.random.default_rng(9)
    prompts = torch.from_numpy(rng.integers(0, shape.vocab, (1536, 5)).astype(np.int32)).cuda()
    G, N = 8, 6
    a = sapo.sapo_rollout_generate(small, prompts[:64].contiguous(), G, N, 1.0, 5)
    assert kernels_of(lambda: sapo.sapo_rollout_generate(small, prompts[:64].contiguous(), G, N, 1.0, 5)) == {"k_small"}
    b = sapo.sapo_rollout_generate(small, prompts, G, N, 1.0, 5)
    assert "k_small" not in kernels_of(lambda: sapo.sapo_rollout_generate(small, prompts, G, N, 1.0, 5))
    assert torch.equal(a[0], b[0][:512]) and float((a[1] - b[1][:512]).abs().max()) <= 2e-5
    # long prompts and few steps: the prompts' tiles decide, and they are cheaper on the small path
    long = torch.from_numpy(rng.integers(0, shape.vocab, (1024, 200)).astype(np.int32)).cuda()
    assert kernels_of(lambda: sapo.sapo_rollout_generate(small, long, 1, 2, 1.0, 5)) == {"k_small"}


def test_large_batches_can_be_captured():
    """Under the caller's stream capture a large batch stays on the small path, whose launches can be recorded; replays
    repeat the eager call's tokens."""
    shape = W.TINY
    small, _ = handles(shape, 15)
    rng = np.random.default_rng(10)
    P, G, N = 1536, 8, 6
    prompts = torch.from_numpy(rng.integers(0, shape.vocab, (P, 5)).astype(np.int32)).cuda()
    ws = torch.empty(sapo.sapo_rollout_workspace_bytes(small, P, 5, G, N) + 256, dtype=torch.uint8, device="cuda")
    tok = torch.empty((P * G, N), dtype=torch.int32, device="cuda")
    lp = torch.empty((P * G, N), device="cuda")
    call = lambda: sapo.sapo_rollout_generate(small, prompts, G, N, 1.0, 5, workspace=ws, out_tokens=tok, out_logprobs=lp)
    sapo.sapo_rollout_generate(small, prompts[:2].contiguous(), G, N, 1.0, 5)
    call()
    want = tok.clone(), lp.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        tok.zero_(); lp.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(tok, want[0]) and float((lp - want[1]).abs().max()) <= 2e-5
        call()                                      # the program's own eager call between two replays
        torch.cuda.synchronize()
        assert torch.equal(tok, want[0])
