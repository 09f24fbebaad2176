"""Fringe search by chunks of delay columns: every rate transform's layout, with
and without the zero upper half, against the oracle; maps without a clear peak."""
import numpy as np
import pytest
import torch

from tests.test_gpu_fringe import _check, _vis_set, corr, xc  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n_sb,nbl,n_chan,D,R,dw,rw", [
    (16, 1, 3, 128, 256, 32, 0, 0), (17, 1, 2, 129, 256, 32, 0, 0),
    (33, 1, 2, 256, 512, 64, 40, 9), (32, 2, 2, 512, 1024, 64, 0, 0),
    (100, 1, 2, 300, 512, 256, 0, 0), (200, 1, 1, 256, 256, 256, 0, 30),
    (200, 1, 1, 200, 512, 512, 60, 0), (256, 1, 1, 256, 256, 512, 0, 0),
    (7, 5, 9, 256, 512, 8, 0, 0), (16, 1, 1, 256, 256, 16, 0, 0), (1, 1, 1, 200, 256, 2, 0, 0),
])
def test_chunks_parity(corr, T, n_sb, nbl, n_chan, D, R, dw, rw):  # noqa: F811
    rng = np.random.default_rng(T + D + R)
    V = _vis_set(rng, T, n_sb, nbl, n_chan, D, R)
    _check(corr, V, D, R, 15625.0, 0.5, dw, rw)


def test_ties_and_not_a_number(corr):  # noqa: F811
    """Equal values everywhere give the first bin of the window; a map with no
    number in it gives bin 0 and leaves the other maps alone."""
    T, n_chan, D, R = 64, 256, 512, 128
    V = torch.zeros((T, 1, 4, n_chan), dtype=torch.complex64, device="cuda")
    V[0, 0, 1, 0] = 3.0                              # |G| = 3 in every bin
    V[:, 0, 2] = 1.0
    V[5, 0, 2, 7] = float("nan")
    t = torch.arange(T, device="cuda")[:, None]
    k = torch.arange(n_chan, device="cuda")[None, :]
    V[:, 0, 3] = torch.polar(torch.ones((T, n_chan), device="cuda"),
                             2 * np.pi * (k * 100 / D + t * (-20) / R))
    peaks, _ = corr.fringe_search(V, D, R, 1.0, 1.0)
    for m in (0, 1):
        assert (peaks[0, m]["delay_bin"], peaks[0, m]["rate_bin"]) == (0, 0)
    assert peaks[0, 0]["amp"] == 0.0
    assert abs(peaks[0, 1]["amp"] - 3.0 / (T * n_chan)) < 1e-6
    assert (peaks[0, 2]["delay_bin"], peaks[0, 2]["rate_bin"]) == (0, 0)
    assert np.isnan(peaks[0, 2]["amp"])
    assert (peaks[0, 3]["delay_bin"], peaks[0, 3]["rate_bin"]) == (100, -20)
