"""Decode steps of 65 .. 256 rows against the oracle: row counts at the edges of the 32- and 128-row blocks, widths of the FFN
and of the model that take each number of feature blocks per workgroup (2 .. 5, with a last tile that is not full), fewer
stages of K than parts, rows with more sums of squares than are requested ahead, each tile of the O projection in front."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import sapo_oracle as O
from paper_2509_08721_amd import sapo
from paper_2509_08721_amd import workloads as W
from tests.parity import measured_logit_eps, oracle_logprobs_for, teacher_forced_token_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,F,S,std,heads", [(*c, (4, 2)) for c in [
    (128, 64, 65, 0.05),        # one stage of K for eight parts
    (128, 256, 96, 0.05), (128, 576, 97, 0.05), (256, 320, 128, 0.05), (256, 704, 129, 0.05), (384, 512, 160, 0.05),
    (256, 4160, 192, 0.02),     # gate/up: 260 blocks, 3 per workgroup
    (128, 6272, 255, 0.02),     # 392 blocks, 4
    (128, 8256, 256, 0.02),     # 516 blocks, 5, the last tile one block
    (1152, 128, 200, 0.02),     # down: 36 blocks, 3
    (1664, 128, 131, 0.02),     # 52 blocks, 4; 52 parts of the sums of squares
    (2176, 192, 254, 0.02),     # 68 blocks, 5, the last tile three
    (3200, 64, 70, 0.01),       # two blocks per part of the sums of squares
    (1280, 128, 100, 0.02),     # O projection: two tiles x two token groups; QKV: two x one, K in two rounds
    (3200, 64, 193, 0.01),      # O projection: four tiles x four token groups per workgroup
]] + [                          # O projection: K of 2304, two workgroups of two token groups per block, each with its sums
    (256, 320, 65, 0.05, (36, 4)), (640, 192, 150, 0.02, (36, 4)), (128, 64, 256, 0.05, (36, 4))])
def test_rows_follow_the_oracle(d, F, S, std, heads):
    shape = replace(W.MINI_BF16, n_layers=2, d_model=d, d_ff=F, n_q_heads=heads[0], n_kv_heads=heads[1])
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


@pytest.mark.parametrize("d,F,S", [(256, 320, 66), (128, 4160, 129), (128, 8256, 200), (1664, 192, 100)])   # 2, 3, 5 feature blocks; 52 parts
def test_rows_that_half_cannot_hold_before_their_norm(d, F, S):
    """The FFN of 65 .. 256 rows reads half(residual x gain) and scales behind the product.  Rows whose product is beyond half's
    range, and rows far below its normal range, get what their normalised values give, next to ordinary rows in the same
    wave: embeddings of three sizes (peaks of 32000, 4 and 1e-6; ffn gains of 8), no attention output, an FFN whose output
    outweighs the residual.  Step 0 comes from the prompt's pass, which clamps as documented: steps 1 on are compared.
    Halves are good to 2^-11 of the largest of the values that meet in a logit: the general tolerance."""
    shape = replace(W.MINI_BF16, n_layers=1, d_model=d, d_ff=F, tied_embeddings=False, rms_eps=1e-15)
    rng = np.random.default_rng(S)
    w = W.perturb_norm_gains(W.make_weights(shape, 13, std=0.05 * (128 / d) ** 0.5), 13)
    lw = w["layers"][0]
    lw["wo"] = np.zeros_like(lw["wo"])
    lw["ffn_norm"] = (8.0 * lw["ffn_norm"]).astype(np.float32)
    lw["w_down"] = W.f32_to_bf16_bits(W.bf16_bits_to_f32(lw["w_down"]) * np.float32(250.0 / (F / 256) ** 0.5))
    size = np.array([32000.0, 4.0, 1e-6], np.float32)[rng.integers(0, 3, shape.vocab)]
    e = W.bf16_bits_to_f32(w["embed"])
    w["embed"] = W.f32_to_bf16_bits((e / np.abs(e).max() * size[:, None]).astype(np.float32))
    gw = sapo.sapo_weights_create(shape, w)
    assert gw.uses_mfma
    ma, Lp, N, seed = O.Model(shape, w), 5, 6, 79
    prompts = rng.integers(0, shape.vocab, size=(S, Lp)).astype(np.int32)
    toks, lps = sapo.sapo_rollout_generate(gw, torch.from_numpy(prompts).cuda(), 1, N, 1.0, seed)
    toks, lps = toks.cpu().numpy(), lps.cpu().numpy()
    seqs = list(range(0, S, 3))
    assert len({float(size[toks[s, t]]) for s in seqs for t in range(N - 1)}) == 3
    n, exact, near, bad = teacher_forced_token_check(ma, prompts, 1, toks, 1.0, seed, seqs, steps=range(1, N), delta=2e-2)
    assert not bad, bad[:5]
    ref = oracle_logprobs_for(ma, prompts, 1, toks, seqs)
    assert max(np.max(np.abs(ref[s] - lps[s])[1:]) for s in seqs) <= 2e-2
    gw.close()
