"""Accumulator slots and weights need no cleared workspace.

A job's first block stores its slots and the delay kernel counts the weights;
blocks with fewer slices leave the others alone.  So a workspace full of NaN
bit patterns gives what one full of zeros does, and the weights are the oracle's.
"""
import numpy as np
import pytest
import torch

from oracle import fx
from synth import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def xc():
    from paper_1502_06894_amd import xcorr
    return xcorr


@pytest.fixture(scope="module")
def corr(xc):
    return xc.Correlator(0)


# 64-frame chunks of the delay kernel and their remainders, more stations than a
# workgroup has waves, blocks of one and several slices and a short last one
@pytest.mark.parametrize("S,nf,fpb,prec", [
    (2, 63, 0, 0), (3, 65, 0, 0), (17, 130, 50, 0), (2, 2100, 900, 0), (2, 1, 0, 0),
    (5, 700, 300, 1), (5, 700, 300, 2),
])
def test_dirty_workspace(xc, corr, S, nf, fpb, prec):
    job = configs.small_job(n_stations=S, n_subbands=1, n_pols=1, n_chan=128, C=2, n_frames=nf,
                            realistic=False, seed=S)
    st = job.stations[1]
    st.frames = st.frames.clone()
    st.frames[0, 0] = 0
    W = fx.correlate(job, threads=8)[1]
    xc.job_to_device(job)
    ws = corr.alloc_workspace(job, precision=prec, frames_per_block=fpb)
    out = []
    for byte in (0, 255):
        ws.fill_(byte)
        out.append(corr.correlate(job, precision=prec, frames_per_block=fpb, workspace=ws))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert np.array_equal(out[1][1].cpu().numpy(), W.astype(np.float32))


@pytest.mark.parametrize("lanes_only", [False, True])
def test_dirty_batch_and_graph(xc, corr, lanes_only):
    jobs = [configs.small_job(n_stations=2 + k, n_subbands=1, n_pols=1, n_chan=128 << (k % 2), C=2,
                              n_frames=90 + 70 * k, seed=k) for k in range(4)]
    for j in jobs:
        xc.job_to_device(j)
    ws = corr.batch_workspace(jobs, lanes_only=lanes_only)
    refs = [corr.correlate(j) for j in jobs]
    for graph in (False, True, True, True):
        ws.fill_(255)
        outs = [corr.alloc_output(j) for j in jobs] if not graph else outs
        got = corr.correlate_batch(jobs, outs=outs, workspace=ws, graph=graph,
                                   lanes_only=lanes_only)
        torch.cuda.synchronize()
        for (v, w), (rv, rw) in zip(got, refs):
            assert torch.equal(v, rv) and torch.equal(w, rw), graph
        for v, w in outs:
            v.fill_(0)
            w.fill_(0)
