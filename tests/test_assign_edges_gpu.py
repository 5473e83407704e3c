"""The greedy pass where its kernels change hands and at the ends of their
groups (GPU): instance counts around 16, 64, 128, 256 and 512, step counts
around the producers' groups and the 64-step blocks, against the oracle under
the repository's acceptance rule, and the decided rows against the picks.
"""
import numpy as np
import pytest
import torch

import test_parity_options_gpu as opt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("I", [1, 16, 17, 64, 65, 128, 129, 256, 257, 511, 512, 513, 1000, 1024])
@pytest.mark.parametrize("B", [1, 2, 7, 8, 9, 65])
def test_assign_at_the_edges(B, I):
    opt.say(f"assign edges B={B} I={I}")
    M = min(I, 5)
    qh, lh, pl, inst = opt.random_case(B, M, I, seed=1000 * B + I)
    C = opt.costs(lh, pl, inst)
    budget = np.quantile(C, 0.6, axis=1).astype(np.float32)
    budget[0] = 0.0                     # a request without a candidate
    mask = (np.arange(I) % 3 != 1).astype(np.uint8)
    for w, kw in (((0.3, 0.4, 0.3), {}), ((0.3, 0.4, 0.3), dict(budget=budget, mask=mask)),
                  ((0, 1, 0), dict(mask=mask))):
        for order in (0, 1):
            res = opt.run_assign_ex(qh, lh, pl, inst, w, order=order, **kw)
            opt.check(res, qh, lh, pl, inst, w, order, label=f"w={w} order={order}", **kw)


@pytest.mark.parametrize("I", [13, 64, 200, 300, 700])
def test_decided_rows_hold_the_chosen_scores(I):
    m = opt.rb()
    B, w = 70, (0.3, 0.4, 0.3)
    qh, lh, pl, inst = opt.random_case(B, 5, I, seed=I)
    qh[3, :] = np.nan                   # a request without a score has no candidate
    outs = []
    for want in (False, True):
        gi = m.DeviceInstances.from_host(inst, opt.DEV)
        dec = torch.empty(B, I, device=opt.DEV) if want else None
        asg, ch = m.rb_assign(opt.dev(qh), opt.dev(lh), opt.dev(pl), gi, w, decided=dec)
        torch.cuda.synchronize()
        outs.append((asg.cpu().numpy(), ch.cpu().numpy(), gi.prefill_q.cpu().numpy(),
                     gi.decode_q.cpu().numpy()))
    for x, y in zip(*outs):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32))
    asg, ch = outs[0][:2]
    dec = dec.cpu().numpy()
    assert asg[3] == -1 and np.isnan(ch[3]) and np.isnan(dec[3]).all()
    for r in range(B):
        if asg[r] >= 0:
            assert dec[r, asg[r]].view(np.uint32) == ch[r].view(np.uint32)
            assert np.nanargmax(dec[r]) == asg[r] or np.nanmax(dec[r]) - ch[r] < 1e-5
