"""Single calls captured into a graph by the caller: a graph that never runs
holds up neither the calls after it nor the end of the correlator; one that runs
gives the eager call's results."""
import time

import pytest
import torch

from synth import configs

pytestmark = pytest.mark.gpu


def test_captured_call_that_never_runs():
    from paper_1502_06894_amd import xcorr as xc
    job = configs.small_job(n_stations=3, n_subbands=2, n_pols=2, n_chan=256, C=4, n_frames=24)
    xc.job_to_device(job)
    corr = xc.Correlator(0)
    ref = corr.correlate(job)
    torch.cuda.synchronize()
    graphs = []
    for _ in range(2):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            vis, w = corr.correlate(job)
        graphs.append(g)
    for _ in range(3):                                 # the last one runs, its slot not reused yet
        graphs[-1].replay()
        torch.cuda.synchronize()
        assert torch.equal(vis, ref[0]) and torch.equal(w, ref[1])
    t0 = time.monotonic()
    for _ in range(20):                                # more than twice around the ring of slots
        got = corr.correlate(job)
        torch.cuda.synchronize()
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    corr.close()
    assert time.monotonic() - t0 < 5.0                 # (a wait for a graph's slot: 10 s)
