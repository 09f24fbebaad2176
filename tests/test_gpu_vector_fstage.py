"""The vector F stage: what jobs run whose fringe phase curves too much inside a
frame for the matrix cores, and what those jobs' tuned variants select.

The jobs here leave 1e-3 turns of curvature in a frame: the matrix form would be
off by some 2e-4 of the spectra's RMS, far outside the bounds below, so results
within them are the vector kernels'.
"""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import fx
from synth import configs
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

SPEC_TOL = 3e-6     # the vector F stage's bound, as for every job before the matrix form
VIS_TOL = 1e-5


@pytest.fixture(scope="module")
def xc():
    from paper_1502_06894_amd import xcorr
    return xcorr


@pytest.fixture(scope="module")
def corr(xc):
    return xc.Correlator(0)


def _curved(**kw):
    """A small job with 1e-3 turns (N^2 phi2) of fringe curvature in station 1's frames."""
    job = configs.small_job(**kw)
    t0 = job.sub_start / job.fs_hz
    c2 = 1e-3 * job.fs_hz ** 2 / (max(job.lo_hz) * job.N ** 2)
    st = job.stations[1]
    p = np.array(st.delay_poly, np.float64)
    p[:3] += [c2 * t0 * t0, -2 * c2 * t0, c2]        # + c2 (t - t0)^2
    return dataclasses.replace(job, stations=[job.stations[0],
                                              dataclasses.replace(st, delay_poly=p),
                                              *job.stations[2:]])


def _check(job, nf, spec, vis, w, V, W):
    for s in range(job.n_stations):
        for sb in range(job.n_subbands):
            for p in range(job.n_pols):
                Y = fx.station_spectra(job, s, sb, p, np.arange(nf))[0]
                assert rel_l2(spec[sb, :, s * job.n_pols + p, :], Y) < SPEC_TOL, (s, sb, p)
    assert np.array_equal(w.cpu().numpy(), W.astype(np.float32))
    for sb in range(job.n_subbands):
        for bl in range(job.n_baselines):
            assert rel_l2(vis[sb, bl].cpu().numpy(), V[sb, bl]) < VIS_TOL, (sb, bl)


# every length, one and two polarisations; input counts around a lean task's four
@pytest.mark.parametrize("n_chan,C,nsb,P,nf", [
    (128, 4, 2, 2, 37), (128, 8, 5, 1, 19), (256, 4, 1, 2, 21), (256, 1, 1, 1, 9),
    (512, 8, 3, 2, 11), (512, 16, 5, 1, 7), (1024, 4, 2, 2, 9), (1024, 8, 5, 1, 5),
    (2048, 16, 3, 2, 5), (2048, 2, 1, 1, 3), (4096, 2, 1, 2, 4), (4096, 8, 5, 1, 3),
    (8192, 4, 1, 2, 2), (8192, 16, 5, 1, 3), (16384, 8, 3, 2, 3), (16384, 2, 1, 1, 2),
])
def test_default_and_variants(xc, corr, n_chan, C, nsb, P, nf):
    """The default against the oracle; variants 1-4 and 8 alike bit for bit (up to
    4096 channels); the default is the variant it is said to be."""
    job = _curved(n_stations=3, n_subbands=nsb, n_pols=P, n_chan=n_chan, C=C, n_frames=nf,
                  seed=n_chan + 7 * nsb + P)
    V, W = fx.correlate(job, threads=8)
    cpu = job.stations
    job = dataclasses.replace(job, stations=[dataclasses.replace(s) for s in cpu])
    xc.job_to_device(job)
    host = dataclasses.replace(job, stations=cpu)
    vis, w = corr.correlate(job)
    spec = corr.debug_spectra(job, 0, nf)
    _check(host, nf, spec.cpu().numpy(), vis, w, V, W)
    if n_chan > 4096:
        return
    got = {}
    try:
        for v in (1, 2, 3, 4, 8, 5, 7):
            corr.set_tuning(fstage_waves_per_simd=v)
            got[v] = corr.debug_spectra(job, 0, nf)
            vis, w = corr.correlate(job)
            if v in (5, 7):
                _check(host, nf, got[v].cpu().numpy(), vis, w, V, W)
    finally:
        corr.set_tuning(fstage_waves_per_simd=0)
    for v in (2, 3, 4, 8):
        assert torch.equal(got[v], got[1]), v
    lean = n_chan >= 4096 or (P == 1 and 512 <= n_chan <= 2048)
    assert torch.equal(spec, got[7 if lean else 1])
    if 256 <= n_chan <= 1024:                        # (split tables: other roundings)
        assert not torch.equal(got[7], got[1])


def test_fused_batch(xc, corr):
    """Curved jobs of every length of the fused batch, one and two polarisations,
    beside smooth ones of the same lengths: the same bits as each job alone."""
    jobs = []
    for i, n_chan in enumerate([128, 256, 512, 1024, 2048, 4096, 8192]):
        for P in (1, 2):
            kw = dict(n_subbands=1 + i % 3, n_pols=P, n_chan=n_chan, C=8,
                      n_frames=max(3, 4000 // n_chan + 5 * P), seed=40 * i + P)
            jobs.append(_curved(n_stations=2 + (i + P) % 3, **kw))
            jobs.append(configs.small_job(n_stations=2 + i % 2, **kw))
    host = [dataclasses.replace(j, stations=[dataclasses.replace(s) for s in j.stations])
            for j in jobs]
    for j in jobs:
        xc.job_to_device(j)
    refs = [corr.correlate(j) for j in jobs]
    ws = corr.batch_workspace(jobs, n_lanes=3)
    outs = [corr.alloc_output(j) for j in jobs]
    for graph in (False, True, True):
        for v, w in outs:
            v.zero_()
            w.zero_()
        corr.correlate_batch(jobs, n_lanes=3, graph=graph, outs=outs, workspace=ws)
        torch.cuda.synchronize()
        for k, ((v, w), (rv, rw)) in enumerate(zip(outs, refs)):
            assert torch.equal(v, rv) and torch.equal(w, rw), (graph, k)
    for k in range(0, len(jobs), 4):
        V, W = fx.correlate(host[k], threads=8)
        assert np.array_equal(refs[k][1].cpu().numpy(), W.astype(np.float32)), k
        assert rel_l2(refs[k][0].cpu().numpy(), V) < VIS_TOL, k
