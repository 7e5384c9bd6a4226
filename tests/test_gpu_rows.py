"""Decode steps of 65 .. 256 rows against the oracle: row counts at the edges of the 32- and 128-row blocks, widths of the FFN
and of the model that take each number of feature blocks per workgroup (2 .. 5, with a last tile that is not full), fewer
stages of K than parts, rows with more sums of squares than are requested ahead."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import sapo_oracle as O
from paper_2509_08721_amd import sapo
from paper_2509_08721_amd import workloads as W
from tests.parity import measured_logit_eps, oracle_logprobs_for, teacher_forced_token_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,F,S,std", [
    (128, 64, 65, 0.05),        # one stage of K for eight parts
    (128, 256, 96, 0.05), (128, 576, 97, 0.05), (256, 320, 128, 0.05), (256, 704, 129, 0.05), (384, 512, 160, 0.05),
    (256, 4160, 192, 0.02),     # gate/up: 260 blocks, 3 per workgroup
    (128, 6272, 255, 0.02),     # 392 blocks, 4
    (128, 8256, 256, 0.02),     # 516 blocks, 5, the last tile one block
    (1152, 128, 200, 0.02),     # down: 36 blocks, 3
    (1664, 128, 131, 0.02),     # 52 blocks, 4; 52 parts of the sums of squares
    (2176, 192, 254, 0.02),     # 68 blocks, 5, the last tile three
    (3200, 64, 70, 0.01),       # two blocks per part of the sums of squares
])
def test_rows_follow_the_oracle(d, F, S, std):
    shape = replace(W.MINI_BF16, n_layers=2, d_model=d, d_ff=F)
    w = W.perturb_norm_gains(W.make_weights(shape, 11, std=std), 11)
    gw = sapo.sapo_weights_create(shape, w)
    assert gw.uses_mfma
    ma, Lp, N, seed = O.Model(shape, w), 9, 5, 77
    prompts = np.random.default_rng(S).integers(0, shape.vocab, size=(S, Lp)).astype(np.int32)
    st = torch.cuda.Stream()

    def run(stream):
        t, l = sapo.sapo_rollout_generate(gw, torch.from_numpy(prompts).cuda(), 1, N, 1.0, seed, stream=stream)
        torch.cuda.synchronize()
        return t.cpu().numpy(), l.cpu().numpy()

    toks, lps = run(None)
    with torch.cuda.stream(st):
        for _ in range(2):      # the captured step, replayed
            t2, l2 = run(st)
            assert np.array_equal(t2, toks) and np.array_equal(l2.view(np.uint32), lps.view(np.uint32))
    seqs = sorted({0, 31, 32, 63, 64, S // 2, S - 2, S - 1})
    eps = max(measured_logit_eps(sapo, gw, ma, np.concatenate([prompts[s], toks[s]]), Lp - 1) for s in seqs)
    assert eps <= 5e-2, eps
    n, exact, near, bad = teacher_forced_token_check(ma, prompts, 1, toks, 1.0, seed, seqs, delta=1e-3 + 2 * eps)
    assert not bad, bad[:5]
    ref = oracle_logprobs_for(ma, prompts, 1, toks, seqs)
    assert max(np.max(np.abs(ref[s] - lps[s])) for s in seqs) <= 2e-2
    gw.close()


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("P,G", [(1, 2), (3, 3), (5, 3), (3, 5), (2, 12), (1, 16), (7, 11)])   # the last one not a multiple of its group, and 77 rows
def test_rows_dealt_in_groups_of_siblings(hd, P, G):
    """Decode attention deals rows to the XCDs in groups of 1, 2, 4 or 8: every row is there once, whatever the number of
    siblings, also where a group holds rows of two prompts."""
    shape = replace(W.MINI_BF16 if hd == 64 else W.MINI_BF16_HD128, n_layers=1)
    w = W.make_weights(shape, 12, std=0.05)
    gw = sapo.sapo_weights_create(shape, w)
    ma, Lp, N, seed = O.Model(shape, w), 21, 4, 78
    prompts = np.random.default_rng(P * G).integers(0, shape.vocab, size=(P, Lp)).astype(np.int32)
    toks, lps = sapo.sapo_rollout_generate(gw, torch.from_numpy(prompts).cuda(), G, N, 1.0, seed)
    toks, lps = toks.cpu().numpy(), lps.cpu().numpy()
    seqs = list(range(P * G))
    eps = max(measured_logit_eps(sapo, gw, ma, np.concatenate([prompts[s // G], toks[s]]), Lp - 1) for s in seqs[::5])
    n, exact, near, bad = teacher_forced_token_check(ma, prompts, G, toks, 1.0, seed, seqs, delta=1e-3 + 2 * max(eps, 5e-3))
    assert not bad, bad[:5]
    ref = oracle_logprobs_for(ma, prompts, G, toks, seqs)
    assert max(np.max(np.abs(ref[s] - lps[s])) for s in seqs) <= 2e-2
    gw.close()
