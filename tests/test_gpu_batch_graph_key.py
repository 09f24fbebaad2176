"""A captured batch is replayed only for the batch it was captured from: the drift
correction of a station decides which launches a job has and whether it joins the
fused rounds at all, so the same buffers with that flag changed are another batch.
"""
import dataclasses

import pytest
import torch

from synth import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lanes_only", [True, False])
def test_drift_flag_is_part_of_the_batch(lanes_only):
    from paper_1502_06894_amd import xcorr as xc
    corr = xc.Correlator(0)
    jobs = [configs.small_job(n_stations=2 + k, n_subbands=1, n_pols=1, n_chan=256, C=2,
                              n_frames=40 + 30 * k, seed=k) for k in range(4)]
    for j in jobs:
        xc.job_to_device(j)
    other = list(jobs)
    other[1] = dataclasses.replace(jobs[1], stations=[
        dataclasses.replace(st, rate_correct=i == 0) for i, st in enumerate(jobs[1].stations)])
    refs = {False: [corr.correlate(j) for j in jobs], True: [corr.correlate(j) for j in other]}
    assert not torch.equal(refs[False][1][0], refs[True][1][0])
    ws = max((corr.batch_workspace(b, lanes_only=lanes_only) for b in (jobs, other)),
             key=lambda t: t.numel())
    outs = [corr.alloc_output(j) for j in jobs]
    for flag in (False, True, False, True, True):
        for v, w in outs:
            v.zero_()
            w.zero_()
        corr.correlate_batch(other if flag else jobs, outs=outs, workspace=ws, graph=True,
                             lanes_only=lanes_only)
        torch.cuda.synchronize()
        for k, ((v, w), (rv, rw)) in enumerate(zip(outs, refs[flag])):
            assert torch.equal(v, rv) and torch.equal(w, rw), (flag, k)
