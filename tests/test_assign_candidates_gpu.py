"""The greedy pass where values that the ordinary inputs do not hold meet the
candidate set (GPU): predictions and queues that are no numbers or infinite on
instances that are no candidates, and qualities below zero on some that are.

The reference is the loop itself in float64, step by step from the GPU's own
picks: a pick must be a candidate whose score is within 1e-5 of the best one
(fp32 scores of unit scale are good to about 1e-6), and the state of every
instance must be what its picks make it.
"""
import dataclasses

import numpy as np
import pytest
import torch

import test_parity_options_gpu as opt

pytestmark = pytest.mark.gpu

NEG_NAN = np.array([0xffc00000], np.uint32).view(np.float32)[0]
COUNTS = [13, 64, 200, 300, 700]   # one row of lanes; one, four slots; eight waves of one, two


def replay(res, qh, lh, pl, inst, w, mask=None, label=""):
    """Checks the picks, chosen scores and final state of `res`."""
    m = inst.model
    p, a = inst.prefill_q.astype(np.float64), inst.decode_q.astype(np.float64)
    up = np.ones(len(m), bool) if mask is None else mask != 0
    with np.errstate(all="ignore"):
        for r in range(len(qh)):
            q, lv = qh[r].astype(np.float64)[m], lh[r].astype(np.float64)[m]
            C = pl[r] * inst.price_in.astype(np.float64) + lv * inst.price_out
            cand = up & (C <= np.inf) & ~np.isnan(q)
            g = int(res["assign"][r])
            if not cand.any():
                assert g == -1 and np.isnan(res["chosen"][r]), f"{label} request {r}: picked {g}"
                continue
            T = (p + pl[r]) / inst.prefill_rate + (a + lv) / inst.decode_rate
            cm, tm = C[cand].max(), T[cand].max()
            S = w[0] * q + w[2] * (1 - (C / cm if cm > 0 else 0)) + \
                w[1] * (1 - (T / tm if tm > 0 else 0))
            best = S[cand].max()
            assert g >= 0 and cand[g], f"{label} request {r}: {g} is no candidate"
            assert S[g] >= best - 1e-5 * max(1.0, abs(best)), \
                f"{label} request {r}: picked {g} at {S[g]}, best {best}"
            assert abs(res["chosen"][r] - S[g]) <= 1e-4 * max(1.0, abs(S[g]))
            p[g] += pl[r]
            a[g] += lv[g]
    picked = np.isin(np.arange(len(m)), res["assign"])
    for f, ref, start in (("p", p, inst.prefill_q), ("a", a, inst.decode_q)):
        same = res[f].view(np.uint32) == start.astype(np.float32).view(np.uint32)
        assert same[~picked].all(), f"{label}: the state of an instance never picked changed"
        assert np.allclose(res[f][picked], ref[picked], rtol=1e-4), label


def run(qh, lh, pl, inst, w, mask=None, label=""):
    opt.say(f"candidates {label}")
    res = opt.run_assign_ex(qh, lh, pl, inst, w, mask=mask)
    replay(res, qh, lh, pl, inst, w, mask, label)


@pytest.mark.parametrize("nan", [np.float32(np.nan), NEG_NAN], ids=["nan", "negative nan"])
@pytest.mark.parametrize("I", COUNTS)
def test_predictions_that_are_no_numbers(I, nan):
    """A NaN predicted length (no labels, or fewer neighbours than k) makes the
    instances of that model no candidates of that request."""
    B, M = 70, 5
    for w in ((0.3, 0.4, 0.3), (0.6, 0.0, 0.4)):
        qh, lh, pl, inst = opt.random_case(B, M, I, seed=I)
        lh[::3, 1] = nan                  # one model
        lh[5], qh[5] = nan, nan           # every model
        lh[6] = nan
        lh[0] = nan                       # the first request
        run(qh, lh, pl, inst, w, label=f"nan lengths I={I} w={w}")


@pytest.mark.parametrize("value", [np.nan, NEG_NAN, np.inf, -np.inf],
                         ids=["nan", "negative nan", "inf", "negative inf"])
@pytest.mark.parametrize("I", COUNTS)
def test_queues_of_masked_instances(I, value):
    """What a lost instance's queue figures hold decides nothing and stays."""
    B, M = 70, 5
    mask = (np.arange(I) % 3 != 0).astype(np.uint8)   # (the lowest index among the lost)
    for w in ((0.3, 0.4, 0.3), (0.6, 0.0, 0.4), (0.0, 1.0, 0.0)):
        qh, lh, pl, inst = opt.random_case(B, M, I, seed=I + 1)
        for f in ("prefill_q", "decode_q"):
            q = getattr(inst, f).astype(np.float32).copy()
            q[mask == 0] = value
            run(qh, lh, pl, dataclasses.replace(inst, **{f: q}), w, mask,
                f"{f} {value} I={I} w={w}")
        r = inst.decode_rate.astype(np.float32).copy()
        r[mask == 0] = 0.0                # (a lost instance that decodes nothing)
        run(qh, lh, pl, dataclasses.replace(inst, decode_rate=r), w, mask,
            f"decode rate 0 I={I} w={w}")


@pytest.mark.parametrize("I", COUNTS)
def test_negative_qualities(I):
    """A candidate whose quality is below zero is one all the same, in the
    maxima and for the pick (the best score is not below zero here)."""
    B, M = 70, 5
    for w in ((0.3, 0.4, 0.3), (0.6, 0.4, 0.0), (0.8, 0.1, 0.1)):
        qh, lh, pl, inst = opt.random_case(B, M, I, seed=I + 2)
        qh -= np.float32(0.6)
        qh[:, 0] = np.float32(0.05)       # one model's is not
        qh[::4, 0] = -np.float32(0.01)    # (or hardly below)
        run(qh, lh, pl, inst, w, label=f"negative qualities I={I} w={w}")
