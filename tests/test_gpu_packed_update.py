"""Updates on answers that end before their row does: what lies behind a sequence's last masked token goes through neither pass.

Loss, log-probs and every gradient against the float64 reference (the bounds of test_gpu_update.py), with the whole set at once and in
micro-batches (some of them without a masked token, which run all rows as they lie), and the same bits whatever the padding holds.
"""
from dataclasses import replace

import numpy as np
import pytest
import torch

from paper_2509_08721_amd import workloads as W
from tests.test_gpu_update import SHAPES, dev, read_all, reference_on_gpu, sapo, tiles_shape  # noqa: F401  (sapo: the fixture)

pytestmark = pytest.mark.gpu


def case(shape, seed, S, T, kind):
    from oracle import sapo_update_oracle as U
    w = W.perturb_norm_gains(W.make_weights(shape, seed, std=0.25), seed)
    rng = np.random.default_rng([seed, S, T])
    tokens = rng.integers(0, shape.vocab, size=(S, T)).astype(np.int32)
    mask = np.zeros((S, T), np.uint8)
    for s in range(S):
        last = (int(rng.integers(1, T)), 1, T // 2, T - 1)[min(s, 3)] if s < 4 else int(rng.integers(0, T))
        mask[s, max(0, last - int(rng.integers(0, T))):last + 1] = 1
    if kind == "holes":
        mask &= rng.random((S, T)) < 0.3
        mask[0, 1] = 1
    if kind == "gaps":          # sequences (with one or two to a micro-batch: micro-batches) without a masked token; one masked at 0 only
        mask[2:4] = 0
        mask[S - 1] = 0
        mask[S - 1, 0] = 1
    adv = rng.standard_normal(S).astype(np.float32)
    params = U.parameter_list(shape, w)
    _, lp, _ = U.loss_and_gradients(shape, params, tokens, mask, np.zeros((S, T), np.float32), adv)
    u = rng.uniform(-0.4, 0.4, size=lp.shape)
    u[(np.abs(np.exp(-u) - 1.28) < 0.02) | (np.abs(np.exp(-u) - 0.8) < 0.02)] = 0.0   # clear of the clip bounds
    return w, params, tokens, mask, (lp + u * (mask != 0)).astype(np.float32), adv


def leaves_rows_out(mask, s_micro):
    """Is every micro-batch without a sixteenth of its rows and 128 of them at least, those behind the last masked tokens?"""
    S, T = mask.shape
    for s in range(0, S, s_micro or S):
        m = mask[s:s + (s_micro or S)]
        needed = sum(int(np.flatnonzero(r)[-1]) if r.any() else 0 for r in m)
        if needed == 0 or m.size - needed < max(128, m.size // 16):
            return False
    return True


# the sets of 576 rows and more are large enough to leave rows out
@pytest.mark.parametrize("name,S,T", [("tiny", 7, 32), ("ragged_untied", 5, 13), ("hd128", 5, 70), ("tiny", 9, 64), ("ragged_untied", 12, 50),
                                      ("hd128", 7, 100), ("tiny_long", 4, 300), ("hd24", 4, 40)])
@pytest.mark.parametrize("kind", ["ends", "holes", "gaps"])
@pytest.mark.parametrize("s_micro", [None, 2])
def test_update_without_the_padding(sapo, name, S, T, kind, s_micro):  # noqa: F811
    from oracle import sapo_update_oracle as U
    shape = SHAPES[name]
    w, params, tokens, mask, logp_old, adv = case(shape, 900 + len(name), S, T, kind)
    packed = name != "hd24" and leaves_rows_out(mask, s_micro)
    assert packed or S * T < 576 or s_micro
    ref_loss, ref_lp, ref_g = U.loss_and_gradients(shape, params, tokens, mask, logp_old, adv)
    gmax = max(float(np.max(np.abs(x))) for x in ref_g)
    bits = None
    for padding in (0, 1):
        t = tokens.copy()
        for s in range(S):
            on = np.flatnonzero(mask[s])
            end = int(on[-1]) + 1 if len(on) else 0
            if padding:
                t[s, end:] = (t[s, end:] + 1 + np.arange(T - end)) % shape.vocab
        tr = sapo.sapo_trainer_create(shape, w)
        ws = None
        if s_micro:
            ws = torch.empty(sapo.sapo_trainer_workspace_bytes_for(tr, S, T, s_micro) + 256, dtype=torch.uint8, device="cuda").fill_(255)
        loss, lp = sapo.sapo_policy_update(tr, dev(t), dev(mask), dev(logp_old), dev(adv), workspace=ws)
        torch.cuda.synchronize()
        loss, lp, g = float(loss.cpu()[0]), lp.cpu().numpy(), read_all(sapo, tr, 1)
        tr.close()
        if bits is None:
            assert np.max(np.abs(lp - ref_lp)) < 2e-4 and abs(loss - ref_loss) < 1e-4 * max(1.0, abs(ref_loss))
            for a, b in zip(g, ref_g):
                assert float(np.max(np.abs(a - b))) <= 2e-4 * max(float(np.max(np.abs(b))), 1e-3 * gmax) + 1e-7
            bits = (loss, lp, g)
        elif packed:   # rows that nothing depends on do not show in a bit
            assert loss == bits[0] and np.array_equal(lp, bits[1]) and all(np.array_equal(a, b) for a, b in zip(g, bits[2]))


# What the decoders of the workloads run: head dims 64 and 128, an FFN width in multiples of 64 (its passes write packed operands),
# every number of pieces, with projection biases.  Row totals in and out of step with the blocks of 16, 64 and 128; in micro-batches
# of `s_micro` sequences.  Tolerances as in test_gpu_update.py for the same models and pieces.
@pytest.mark.parametrize("pieces", [1, 2, 3])
@pytest.mark.parametrize("head_dim,d_ff,S,T,kind,s_micro", [
    (64, 128, 11, 129, "ends", None), (64, 64, 9, 200, "holes", None), (64, 192, 6, 301, "gaps", None), (64, 128, 8, 160, "ends", 4),
    (128, 64, 11, 129, "ends", None), (128, 192, 6, 301, "holes", None), (128, 128, 9, 160, "gaps", 5)])
def test_packed_gradients(sapo, head_dim, d_ff, S, T, kind, s_micro, pieces):  # noqa: F811
    from oracle import sapo_update_oracle as U
    grad_tol, logp_tol = {3: (2e-4, 2e-4), 2: (1e-3, 5e-4), 1: (5e-2, 2e-2)}[pieces]
    shape = replace(tiles_shape(head_dim, d_ff), max_seq=512)
    w = W.perturb_norm_gains(W.make_weights(shape, 50 + T, std=0.25 if pieces > 1 else 0.02), T)
    w = W.add_qkv_bias(w, shape, 3, std=0.1)
    rng = np.random.default_rng([head_dim, S, T])
    tokens = rng.integers(0, shape.vocab, size=(S, T)).astype(np.int32)
    mask = np.zeros((S, T), np.uint8)
    for s in range(S):
        last = int(rng.integers(T // 8, T * 3 // 4)) if s else T - 1
        mask[s, max(1, last - 30):last + 1] = 1
    if kind == "holes":
        mask &= rng.random((S, T)) < 0.3
    if kind == "gaps":
        mask[1] = 0
        mask[S - 1] = 0
        mask[S - 1, 0] = 1
    least = 192 if pieces == 1 else 128
    for s in range(0, S, s_micro or S):
        m = mask[s:s + (s_micro or S)]
        assert m.size - sum(int(np.flatnonzero(r)[-1]) if r.any() else 0 for r in m) >= max(least, m.size // 16)
    adv = np.where(np.arange(S) % 2 == 0, 1.25, -0.75).astype(np.float32)
    params = U.parameter_list(shape, w)
    _, lp0, _ = reference_on_gpu(shape, params, tokens, mask, np.zeros((S, T), np.float32), adv)
    # ratios clear of 1, where the loss of either sign has one branch, and of the clip bounds
    logp_old = (lp0 + np.where(rng.random((S, T)) < 0.5, -0.1, 0.1) * (mask != 0)).astype(np.float32)
    ref_loss, ref_lp, ref_g = reference_on_gpu(shape, params, tokens, mask, logp_old, adv)
    tr = sapo.sapo_trainer_create(shape, w)
    sapo.sapo_trainer_set_matmul_pieces(tr, pieces)
    ws = None
    if s_micro:
        ws = torch.empty(sapo.sapo_trainer_workspace_bytes_for(tr, S, T, s_micro) + 256, dtype=torch.uint8, device="cuda").fill_(255)
    loss, lp = sapo.sapo_policy_update(tr, dev(tokens), dev(mask), dev(logp_old), dev(adv), workspace=ws)
    torch.cuda.synchronize()
    assert np.max(np.abs(lp.cpu().numpy() - ref_lp)) < logp_tol and abs(float(loss.cpu()[0]) - ref_loss) < logp_tol
    gmax = max(float(np.max(np.abs(b))) for b in ref_g)
    for i, (a, b) in enumerate(zip(read_all(sapo, tr, 1), ref_g)):
        if pieces == 1:   # bf16 operands: the tensor's norm
            assert np.linalg.norm(a - b) <= grad_tol * max(np.linalg.norm(b), 1e-3 * gmax), (i, np.linalg.norm(a - b), np.linalg.norm(b))
        else:
            assert float(np.max(np.abs(a - b))) <= grad_tol * max(float(np.max(np.abs(b))), 1e-3 * gmax) + 1e-7, i
    tr.close()


# operands of one and two pieces: a sequence's log-probs have the same bits with and without other sequences' padding
@pytest.mark.parametrize("pieces", [1, 2])
def test_log_probs_keep_their_bits(sapo, pieces):  # noqa: F811
    shape = W.MINI_BF16
    S, T = 6, 150
    w = W.make_weights(shape, 5, std=0.05)
    rng = np.random.default_rng(6)
    tokens = rng.integers(0, shape.vocab, size=(S, T)).astype(np.int32)
    ends = np.zeros((S, T), np.uint8)
    for s in range(S):
        ends[s, 3:int(rng.integers(10, T // 2))] = 1
    full = np.ones((S, T), np.uint8)
    old, adv = np.zeros((S, T), np.float32), np.zeros(S, np.float32)
    out = []
    for mask in (ends, full):
        tr = sapo.sapo_trainer_create(shape, w)
        sapo.sapo_trainer_set_matmul_pieces(tr, pieces)
        _, lp = sapo.sapo_policy_update(tr, dev(tokens), dev(mask), dev(old), dev(adv))
        out.append(lp.cpu().numpy())
        tr.close()
    assert np.array_equal(out[0], np.where(ends != 0, out[1], np.float32(0)))
