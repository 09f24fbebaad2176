"""The delay-drift correction on the matrix cores against the FP64 oracle.

Bound: the regular spectra's 1e-6 of their RMS (five FP32 phasors a sample, log2 N
rounded stages) and the same for the correction, which is below a fifth of the
spectrum at the rates here, plus the rounding of its sum: 1.3e-6.
"""
import dataclasses

import numpy as np
import pytest

from oracle import fx
from synth import configs, shape
from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu

SPEC_TOL = 1.3e-6


# every frame length of the kernel; frames around the group a workgroup takes; inputs
# around a task's four; one, two and all stations corrected, not in sequence
@pytest.mark.parametrize("n_chan,C,nsb,P,nf,flagged", [
    (128, 16, 5, 1, 33, (1,)), (256, 8, 2, 2, 15, (0, 3)), (512, 4, 1, 2, 17, (1, 2)),
    (1024, 16, 5, 1, 7, (3,)), (2048, 2, 2, 1, 3, (0, 1, 2, 3)), (4096, 8, 1, 2, 2, (0, 2)),
    (8192, 4, 3, 1, 1, (2,)), (16384, 2, 1, 1, 1, ()),
])
def test_corrected_spectra(n_chan, C, nsb, P, nf, flagged):
    """Corrected and other stations' spectra, with a bad recording frame and the
    end of a recording cut off; the correction shows in the spectra."""
    from paper_1502_06894_amd import xcorr as xc
    fs, t0 = configs.FS_16MHZ, configs.SUB_START_S
    rate = min(3e-4, 0.1 / (2 * n_chan))
    rates = [rate, -rate, 0.5 * rate, -0.7 * rate]
    job = shape.build_job(n_stations=4, n_subbands=nsb, n_pols=P, n_chan=n_chan, C=C, fs=fs,
                          lo_hz=[configs.LO0_HZ + 16e6 * b for b in range(nsb)],
                          sub_start=int(t0 * fs), n_frames=nf,
                          delay_polys=[[0.03 - r * t0, r, 0.0] for r in rates],
                          shifts=[0] * 4, phase_zero=False, seed=n_chan + nsb, margin=4096)
    plain = job
    job = dataclasses.replace(job, stations=[
        dataclasses.replace(st, rate_correct=i in flagged) for i, st in enumerate(job.stations)])
    job.stations[0].frames = job.stations[0].frames.clone()
    job.stations[0].frames[0, 0] = 0
    if job.stations[2].frames.shape[0] > 1:
        job.stations[2].frames = job.stations[2].frames[:-1].contiguous()
    idx = np.arange(nf)
    ref = {(s, sb, p): fx.station_spectra(job, s, sb, p, idx)[0]
           for s in range(4) for sb in range(nsb) for p in range(P)}
    for s in flagged:
        Y, Y0 = ref[s, 0, 0], fx.station_spectra(plain, s, 0, 0, idx)[0]
        if s not in (0, 2):
            assert rel_l2(Y0, Y) > 1e-3
    xc.job_to_device(job)
    spec = xc.Correlator(0).debug_spectra(job, 0, nf).cpu().numpy()
    for (s, sb, p), Y in ref.items():
        got = spec[sb, :, s * P + p, :]
        for f in range(nf):
            if not np.any(Y[f]):
                assert not np.any(got[f]), (s, sb, p, f)
            else:
                assert rel_l2(got[f], Y[f]) < SPEC_TOL, (s, sb, p, f)
