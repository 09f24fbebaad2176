"""A captured single call holds its descriptor: it replays with its own job's
results however many other calls the correlator has made since.  Nor does a call
wait for the calls before it: the host can be any number of them ahead."""
import dataclasses
import time

import numpy as np
import pytest
import torch

from synth import configs

pytestmark = pytest.mark.gpu


def _with_phase(job):
    """The job's own fringe phase as explicit polynomials per subband."""
    return dataclasses.replace(job, stations=[
        dataclasses.replace(st, phase_poly=np.outer(job.lo_hz, st.delay_poly))
        for st in job.stations])


# descriptors of one launch, and of four (19 stations, 8 subbands of phase polynomials)
@pytest.mark.parametrize("S,nsb,phase", [(3, 2, False), (19, 8, True)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_replays_after_other_calls(S, nsb, phase, noalloc):
    from paper_1502_06894_amd import xcorr as xc
    corr = xc.Correlator(0)
    job = configs.small_job(n_stations=S, n_subbands=nsb, n_pols=1, n_chan=256, C=8, n_frames=24,
                            seed=S)
    job = _with_phase(job) if phase else job
    others = [configs.small_job(n_stations=2 + 5 * k, n_subbands=1 + k, n_pols=1,
                                n_chan=128 << k, C=4, n_frames=30 + k, seed=k) for k in range(4)]
    others[3] = _with_phase(others[3])
    for j in [job] + others:
        xc.job_to_device(j)
    call = corr.correlate_noalloc if noalloc else corr.correlate
    ref = [call(j) for j in [job] + others]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        vis, w = call(job)
    for rep in range(4):
        for i in range(11):
            got = call(others[i % 4])
        torch.cuda.synchronize()
        assert torch.equal(got[0], ref[1 + 10 % 4][0]) and torch.equal(got[1], ref[1 + 10 % 4][1])
        vis.zero_()
        w.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(vis, ref[0][0]) and torch.equal(w, ref[0][1]), rep


def test_host_runs_ahead():
    from paper_1502_06894_amd import xcorr as xc
    corr = xc.Correlator(0)
    job = configs.small_job(n_stations=2, n_subbands=1, n_pols=1, n_chan=128, C=2, n_frames=60)
    xc.job_to_device(job)
    ws = corr.alloc_workspace(job)
    ref = corr.correlate(job, workspace=ws)
    a = torch.randn(4096, 4096, device="cuda")
    b = a @ a
    torch.cuda.synchronize()
    t0 = time.monotonic()
    for _ in range(400):
        torch.mm(a, a, out=b)
    got = [corr.correlate(job, workspace=ws) for _ in range(30)]
    t1 = time.monotonic()
    torch.cuda.synchronize()
    t2 = time.monotonic()
    assert t1 - t0 < 0.5 * (t2 - t0), (t1 - t0, t2 - t0)
    for v, w in got:
        assert torch.equal(v, ref[0]) and torch.equal(w, ref[1])
