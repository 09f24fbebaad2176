"""The matrix-core F stage's tasks over several rounds of its workgroups: every
spectrum is written, whatever the number and the sizes of a station's input groups.

Tolerance: the matrix and the vector kernel are within 1e-6 and 3e-6 of the oracle's
spectra, frame by frame (the bounds of their own tests), so within 5e-6 of each other.
"""
import pytest
import torch

from synth import configs

pytestmark = pytest.mark.gpu


# input groups of a station: 4 + 1, 4 + 2, 4 + 4 + 2 (at a multiple of three resident
# workgroups, and not), 4 + 3, 1, 4 x 4; some three to five rounds, the last one partial
@pytest.mark.parametrize("n_chan,C,S,nsb,P,nf", [
    (128, 8, 3, 5, 1, 12001), (256, 8, 5, 3, 2, 3999), (512, 16, 3, 5, 2, 2503),
    (1024, 16, 3, 5, 2, 1801), (2048, 8, 3, 5, 1, 1501), (2048, 8, 5, 3, 2, 701),
    (4096, 8, 5, 7, 1, 301), (8192, 8, 2, 3, 2, 403), (16384, 4, 5, 3, 1, 203),
    (16384, 16, 2, 8, 2, 151),
])
def test_every_spectrum(n_chan, C, S, nsb, P, nf):
    from paper_1502_06894_amd import xcorr as xc
    corr = xc.Correlator(0)
    job = configs.small_job("cuda", n_stations=S, n_subbands=nsb, n_pols=P, n_chan=n_chan, C=C,
                            n_frames=nf, seed=n_chan + nsb)
    stale = torch.full((nsb, nf, S * P, n_chan), float("nan"), dtype=torch.complex64, device="cuda")
    del stale                                        # (what the spectra's memory holds before)
    spec = corr.debug_spectra(job, 0, nf, frames_per_block=nf)
    try:
        corr.set_tuning(fstage_waves_per_simd=7)
        ref = corr.debug_spectra(job, 0, nf, frames_per_block=nf)
    finally:
        corr.set_tuning(fstage_waves_per_simd=0)
    torch.cuda.synchronize()
    worst = 0.0
    for sb in range(nsb):
        d = torch.linalg.vector_norm(spec[sb] - ref[sb], dim=-1)
        n = torch.linalg.vector_norm(ref[sb], dim=-1)
        assert torch.isfinite(d).all() and n.min().item() > 0.0
        worst = max(worst, (d / n).max().item())
    assert 0.0 < worst < 5e-6, worst


def test_fused_batch_rounds():
    """The same over the fused batch's tasks, which go over all jobs of a length: the
    bits of each job alone."""
    from paper_1502_06894_amd import xcorr as xc
    corr = xc.Correlator(0)
    jobs = []
    for k, (n_chan, S, nsb, P, nf) in enumerate([
            (256, 5, 3, 2, 2501), (256, 3, 5, 1, 3000), (2048, 4, 3, 2, 401), (2048, 5, 7, 1, 203),
            (2048, 3, 1, 1, 300), (8192, 3, 5, 1, 99), (8192, 2, 5, 2, 101)]):
        jobs.append(configs.small_job("cuda", n_stations=S, n_subbands=nsb, n_pols=P,
                                      n_chan=n_chan, C=16, n_frames=nf, seed=k))
    ws = corr.batch_workspace(jobs, n_lanes=2)
    ws.fill_(255)
    got = corr.correlate_batch(jobs, n_lanes=2, workspace=ws)
    torch.cuda.synchronize()
    for k, (j, (v, w)) in enumerate(zip(jobs, got)):
        rv, rw = corr.correlate(j)
        assert torch.equal(v, rv) and torch.equal(w, rw), k
