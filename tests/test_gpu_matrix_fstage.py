"""The F stage on the matrix cores against the FP64 oracle.

Bound: the phases are products of about five FP32 phasors (each within half a
turn's rounding, 2^-25 turns, and its sine's), the transform log2 N rounded
stages: an error below (5 x 1.9e-7 / sqrt(3) + 16 x 6e-8 x 0.5) ~ 1e-6 of the
spectrum's RMS.
"""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import fx
from synth import configs
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

SPEC_TOL = 1e-6
VIS_TOL = 1e-5


@pytest.fixture(scope="module")
def xc():
    from paper_1502_06894_amd import xcorr
    return xcorr


@pytest.fixture(scope="module")
def corr(xc):
    return xc.Correlator(0)


# frames around the group a workgroup takes (32, 16, 8, 4, 2 and 1 frames), inputs
# around a task's four, every number of streams per word
@pytest.mark.parametrize("n_chan,C,nsb,P,nf", [
    (128, 16, 5, 1, 33), (128, 1, 1, 1, 1), (256, 8, 3, 2, 17), (256, 2, 1, 1, 15),
    (512, 4, 1, 2, 9), (512, 16, 6, 1, 7), (1024, 16, 5, 2, 5), (1024, 1, 1, 1, 3),
    (2048, 2, 2, 1, 3), (2048, 16, 7, 1, 1), (4096, 8, 3, 1, 2), (8192, 4, 1, 2, 2),
    (8192, 16, 5, 1, 1), (16384, 8, 3, 2, 3), (16384, 2, 1, 1, 2),
])
def test_spectra(xc, corr, n_chan, C, nsb, P, nf):
    """Spectra of every input, with a bad recording frame in one station and
    the end of another cut off (their frames' spectra are zero)."""
    job = configs.small_job(n_stations=3, n_subbands=nsb, n_pols=P, n_chan=n_chan, C=C,
                            n_frames=nf, seed=n_chan + 10 * nsb + P)
    job.stations[0].frames = job.stations[0].frames.clone()
    job.stations[0].frames[0, 0] = 0
    if job.stations[2].frames.shape[0] > 1:
        job.stations[2].frames = job.stations[2].frames[:-1].contiguous()
    ref = {(s, sb, p): fx.station_spectra(job, s, sb, p, np.arange(nf))
           for s in range(3) for sb in range(nsb) for p in range(P)}
    V, W = fx.correlate(job, threads=8)
    xc.job_to_device(job)
    spec = corr.debug_spectra(job, 0, nf).cpu().numpy()
    for (s, sb, p), r in ref.items():
        got, Y = spec[sb, :, s * P + p, :], r[0]
        for f in range(nf):
            if not np.any(Y[f]):
                assert not np.any(got[f]), (s, sb, p, f)
            else:
                assert rel_l2(got[f], Y[f]) < SPEC_TOL, (s, sb, p, f)
    vis, w = corr.correlate(job)
    assert np.array_equal(w.cpu().numpy(), W.astype(np.float32))
    vis = vis.cpu().numpy()
    for sb in range(nsb):
        for bl in range(job.n_baselines):
            if W[sb, bl] > 0:
                assert rel_l2(vis[sb, bl], V[sb, bl]) < VIS_TOL, (sb, bl)


@pytest.mark.parametrize("n_chan,nf", [(128, 8192), (512, 3000), (1024, 3000), (4096, 700)])
def test_every_frame(xc, corr, n_chan, nf):
    """Every matrix (one per group of frames and subband) is good: no frame of a
    long run is further from the vector kernel's than both kernels' bounds, and
    their chains of phasors (16 steps, 1.2e-7 each, there), allow."""
    job = configs.small_job(n_stations=2, n_subbands=3, n_pols=1, n_chan=n_chan, C=4, n_frames=nf,
                            seed=5)
    xc.job_to_device(job)
    spec = corr.debug_spectra(job, 0, nf)
    try:
        corr.set_tuning(fstage_waves_per_simd=7)
        ref = corr.debug_spectra(job, 0, nf)
    finally:
        corr.set_tuning(fstage_waves_per_simd=0)
    err = torch.linalg.vector_norm(spec - ref, dim=-1) / torch.linalg.vector_norm(ref, dim=-1)
    assert err.max().item() < 5e-6


@pytest.mark.parametrize("scale,matrix", [(0.9, True), (1.1, False)])
def test_curvature_rule(xc, corr, scale, matrix):
    """A fringe phase whose curvature inside a frame leaves less than 3e-8 turns
    out of the matrix product takes the matrix cores; a stronger one the vector
    kernel, at N = 8192 the lean tasks, bit for bit."""
    job = configs.small_job(n_stations=2, n_subbands=1, n_pols=1, n_chan=4096, C=4, n_frames=4,
                            realistic=False, phase_zero=False, seed=11)
    N, t0 = job.N, job.sub_start / job.fs_hz
    c2 = scale * 3e-8 / (0.0325 * N * N) * job.fs_hz ** 2 / job.lo_hz[0]
    st = job.stations[1]
    p = np.array(st.delay_poly, np.float64)
    p[:3] += [c2 * t0 * t0, -2 * c2 * t0, c2]        # tau = the constant + c2 (t - t0)^2
    job = dataclasses.replace(job, stations=[job.stations[0],
                                             dataclasses.replace(st, delay_poly=p)])
    Y = fx.station_spectra(job, 1, 0, 0, np.arange(4))[0]
    xc.job_to_device(job)
    spec = corr.debug_spectra(job, 0, 4)
    try:
        corr.set_tuning(fstage_waves_per_simd=7)
        lean = corr.debug_spectra(job, 0, 4)
    finally:
        corr.set_tuning(fstage_waves_per_simd=0)
    assert torch.equal(spec, lean) != matrix
    if matrix:
        assert rel_l2(spec[0, :, 1].cpu().numpy(), Y) < SPEC_TOL
