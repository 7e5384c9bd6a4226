"""Scoring passes and prompts whose padding is left out: every row keeps the bits it has without.

A scoring pass of at least 2560 positions runs only the positions that a scored token depends on, side by side, and behind the
last layer's attention only the rows that predict a scored token; smaller passes (checked against the oracle in test_gpu_mfma.py
and test_gpu_full.py) run all of them.  A row's log-prob has the same bits whatever else is scored, so the two are compared
sequence by sequence, bit for bit.  Prompts of different lengths are left out of the same way from 1024 positions on.
"""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2509_08721_amd import sapo
from paper_2509_08721_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = {
    "hd64": replace(W.MINI_BF16, d_model=384, d_ff=576, n_layers=3, max_seq=1024),
    "hd128": replace(W.MINI_BF16_HD128, d_ff=832, max_seq=1024),
    # more query features than an FFN is wide: the last layer runs for all rows, and a scoring pass as its rows lie
    "wide_queries": replace(W.MINI_BF16_HD128, max_seq=1024),
}
NARROWS = {"hd64": True, "hd128": True, "wide_queries": False}


def make(name):
    shape = SHAPES[name]
    assert (shape.d_model <= shape.q_dim + 2 * shape.kv_dim and shape.q_dim <= shape.d_ff) == NARROWS[name]
    gw = sapo.sapo_weights_create(shape, W.perturb_norm_gains(W.make_weights(shape, 41, std=0.05), 41))
    assert gw.uses_mfma
    return shape, gw


@pytest.fixture(scope="module", params=[n for n in sorted(SHAPES) if NARROWS[n]])
def model(request):
    return make(request.param)


@pytest.fixture(scope="module", params=sorted(SHAPES))
def any_model(request):
    return make(request.param)


def masks(S, T, kind, rng):
    m = np.zeros((S, T), np.uint8)
    if kind == "ends":          # answers that end anywhere, the row's first and last token included
        for s in range(S):
            last = int(rng.integers(0, T)) if s > 1 else (0, T - 1)[s]
            m[s, int(rng.integers(0, last + 1)):last + 1] = 1
    elif kind == "holes":       # scattered tokens, whole rows without any
        m = (rng.random((S, T)) < rng.random((S, 1)) ** 4).astype(np.uint8)
        m[::3] = 0
    elif kind == "one":         # a single scored token in the whole call
        m[S // 2, T // 2] = 1
    elif kind == "full":
        m[:] = 255              # any value but zero counts
    return m


# (sequences, tokens each): page and tile edges; the smallest pass that packs; (900, 150): two passes of the call
@pytest.mark.parametrize("S,T,kind", [(10, 256, "ends"), (20, 129, "holes"), (9, 301, "ends"), (40, 65, "ends"), (16, 161, "full"),
                                      (16, 161, "one"), (16, 161, "none"), (5, 1000, "ends"), (900, 150, "ends")])
def test_scores_keep_their_bits_without_the_padding(model, S, T, kind):
    shape, gw = model
    rng = np.random.default_rng(S * 1000 + T)
    tokens = torch.from_numpy(rng.integers(0, shape.vocab, size=(S, T)).astype(np.int32)).cuda()
    mask = torch.from_numpy(masks(S, T, kind, rng)).cuda()
    rewards = torch.from_numpy(rng.random(S).astype(np.float32)).cuda()
    assert S * T >= 2560
    for temperature in (1.0, 0.7):
        lp, adv = sapo.sapo_score_logprobs_at(gw, tokens, mask, rewards, 1, temperature)
        n = 2559 // T
        ref = [sapo.sapo_score_logprobs_at(gw, tokens[s:s + n].contiguous(), mask[s:s + n].contiguous(), rewards[s:s + n].contiguous(), 1,
                                           temperature)[0] for s in range(0, S, n)]
        lp = lp.cpu().numpy()
        assert np.array_equal(lp, torch.cat(ref).cpu().numpy())
        on = mask.cpu().numpy() != 0
        on[:, 0] = False
        assert np.all(lp[~on] == 0.0) and np.all(lp[on] < 0.0)


# more sequences in a pass than the second dimension of a grid holds
def test_scores_of_many_short_sequences(model):
    shape, gw = model
    S, T = 65600, 2
    rng = np.random.default_rng(3)
    tokens = torch.from_numpy(rng.integers(0, shape.vocab, size=(S, T)).astype(np.int32)).cuda()
    mask = torch.from_numpy((rng.random((S, T)) < 0.7).astype(np.uint8)).cuda()
    rewards = torch.zeros(S, device="cuda")
    lp = sapo.sapo_score_logprobs(gw, tokens, mask, rewards, 1)[0]
    for s in (0, 30000, 65500):
        part = slice(s, s + 100)
        ref = sapo.sapo_score_logprobs(gw, tokens[part].contiguous(), mask[part].contiguous(), rewards[part].contiguous(), 1)[0]
        assert torch.equal(lp[part], ref) and (ref[:, 1] < 0).any()


# the workspace of a call before does not show: the same bits from memory full of NaN patterns
def test_scores_do_not_depend_on_what_the_workspace_holds(model):
    shape, gw = model
    S, T = 12, 257
    rng = np.random.default_rng(7)
    tokens = torch.from_numpy(rng.integers(0, shape.vocab, size=(S, T)).astype(np.int32)).cuda()
    mask = torch.from_numpy(masks(S, T, "ends", rng)).cuda()
    rewards = torch.zeros(S, device="cuda")
    ws = torch.zeros(sapo.sapo_score_workspace_bytes(gw, S, T) + 256, dtype=torch.uint8, device="cuda")
    a = sapo.sapo_score_logprobs(gw, tokens, mask, rewards, 1, workspace=ws)[0].cpu().numpy()
    ws.fill_(255)
    b = sapo.sapo_score_logprobs(gw, tokens, mask, rewards, 1, workspace=ws)[0].cpu().numpy()
    assert np.array_equal(a, b) and np.isfinite(a).all()


# P prompts of up to Lp tokens, packed where they are shorter (P Lp >= 1024 and a row tile of 128 or a sixteenth less) and with the
# last layer for their last rows only (P Lp >= 512, also where rows of padding lie between), against the same prompts one at a time,
# which run neither
@pytest.mark.parametrize("P,Lp,G,kind", [(9, 120, 4, "packed"), (5, 257, 3, "packed"), (40, 33, 1, "packed"), (5, 120, 2, "full"),
                                         (3, 257, 3, "full"), (17, 31, 1, "full"), (33, 32, 1, "full"), (7, 100, 3, "padded"),
                                         (20, 31, 1, "padded"), (9, 120, 2, "padded"), (5, 300, 1, "padded")])
def test_rollouts_keep_their_bits_without_the_prompts_padding(any_model, P, Lp, G, kind):
    shape, gw = any_model
    rng = np.random.default_rng(P * 100 + Lp)
    lens = [Lp] * P if kind == "full" else [1, Lp] + [int(x) for x in rng.integers(1, Lp + 1, size=P - 2)]
    if kind == "padded" and P * Lp >= 1024:   # fewer rows of padding than a tile
        lens = [Lp - int(x) for x in rng.integers(0, 127 // P + 1, size=P)]
    left_out = P * Lp - sum(lens)
    packed = P * Lp >= 1024 and left_out >= max(128, P * Lp // 16)
    prompts = torch.from_numpy(rng.integers(0, shape.vocab, size=(P, Lp)).astype(np.int32)).cuda()
    assert P * Lp >= 512 and Lp < 512 and packed == (kind == "packed") and (left_out > 0) == (kind != "full")
    tok, lp, _ = sapo.sapo_rollout_generate_ragged(gw, prompts, lens, G, 3, 0.0, 5)
    for p in range(P):
        t, ref, _ = sapo.sapo_rollout_generate_ragged(gw, prompts[p:p + 1].contiguous(), lens[p:p + 1], G, 3, 0.0, 5)
        # greedy tokens; log-probs up to the order in which the parts of a log-sum-exp of at most 1024 entries are merged
        assert torch.equal(tok[p * G:(p + 1) * G], t)
        assert np.abs(lp[p * G:(p + 1) * G].cpu().numpy() - ref.cpu().numpy()).max() <= 1e-5
