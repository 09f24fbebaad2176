"""FP16 spectra from the matrix-core F stage, which jobs of 1024 frames and more run
from 512 to 16384 points.

Against the vector kernel's FP16 spectra (variant 7): the two differ by some 1.2e-6
of the spectra's RMS, so about that over an FP16 step (2^-10 of it) of the values, 1.2e-3, land on
the neighbouring one, 9.8e-4 off: 3.4e-5 a value, 4.8e-5 a product, 1.5e-6 of the
products' scale after 1024 frames; the bound is 5e-6 (of sqrt(A_i A_j), RMS over
channels).  Against FP32: each component is rounded once, 2^-11, so products are
within (2 u + u^2) sqrt(A_i A_j), plus a tenth for the FP32 stages.
"""
import pytest
import torch

from synth import configs

pytestmark = pytest.mark.gpu


def _scale(vis, M):
    """sqrt(A_i A_j) of every baseline, [n_sb][nbl][n_chan]."""
    diag = [i * M - i * (i - 1) // 2 for i in range(M)]
    A = vis[:, diag].real
    i = [a for a in range(M) for _ in range(a, M)]
    j = [b for a in range(M) for b in range(a, M)]
    return (A[:, i] * A[:, j]).sqrt()


# partial frame groups (16, 8, 4, 2 frames), odd input counts, every exponent word layout;
# the last frame count below the rule
@pytest.mark.parametrize("n_chan,C,nsb,P,S,nf", [
    (256, 8, 5, 1, 3, 1037), (256, 2, 1, 2, 2, 1024), (512, 4, 3, 1, 5, 1031),
    (1024, 8, 3, 2, 3, 1026), (1024, 1, 1, 1, 2, 1024), (2048, 4, 3, 1, 3, 1025),
    (4096, 8, 5, 1, 2, 1024), (8192, 4, 3, 1, 3, 1024), (8192, 2, 1, 2, 2, 1027),
    (2048, 4, 3, 1, 3, 1023),
])
def test_fp16_matrix_spectra(n_chan, C, nsb, P, S, nf):
    from paper_1502_06894_amd import xcorr as xc
    corr = xc.Correlator(0)
    job = configs.small_job("cuda", n_stations=S, n_subbands=nsb, n_pols=P, n_chan=n_chan, C=C,
                            n_frames=nf, seed=n_chan + nsb)
    st = job.stations[1]
    st.frames = st.frames.clone()
    st.frames[st.frames.shape[0] // 2, 0] = 0        # a bad recording frame
    ref, w_ref = corr.correlate(job)
    got, w = corr.correlate(job, precision=xc.XC_FP16_MFMA)
    try:
        corr.set_tuning(fstage_waves_per_simd=7)
        vec, w_vec = corr.correlate(job, precision=xc.XC_FP16_MFMA)
    finally:
        corr.set_tuning(fstage_waves_per_simd=0)
    assert torch.equal(w, w_ref) and torch.equal(w_vec, w_ref)
    ref, got, vec = (x.to(torch.complex128) for x in (ref, got, vec))
    sc = _scale(ref, S * P)
    u = 2.0 ** -11
    assert ((got - ref).abs() / sc).max().item() < 1.1 * (2 * u + u * u)
    d = ((got - vec).abs() / sc).square().mean(-1).sqrt().max().item()
    print(f"\n{n_chan} channels, {nf} frames: matrix against vector {d:.2e}")
    if nf >= 1024:
        assert 0.0 < d < 5e-6
    else:
        assert d == 0.0                              # (4096 points: variant 7 rounds as the default)
