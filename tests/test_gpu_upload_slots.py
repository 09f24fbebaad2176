"""Many calls ahead of the device: descriptors go through a ring of pinned slots,
each reused only after its upload has read it, on one stream and on two."""
import pytest
import torch

from synth import configs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("streams", [1, 2])
def test_calls_ahead_of_the_device(streams):
    from paper_1502_06894_amd import xcorr as xc
    corr = xc.Correlator(0)
    jobs = [configs.small_job(n_stations=2 + k % 3, n_subbands=1, n_pols=1, n_chan=128, C=2,
                              n_frames=60 + k, seed=k) for k in range(5)]
    for j in jobs:
        xc.job_to_device(j)
    refs = []
    for j in jobs:
        refs.append(corr.correlate(j))
        torch.cuda.synchronize()
    ss = [torch.cuda.Stream() for _ in range(streams)]
    big = torch.randn(4096, 4096, device="cuda")
    got = []
    for s in ss:
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            for _ in range(60):
                big @ big                              # keep the device behind the host
    for i in range(40):                                # five times around the ring
        s = ss[i % streams]
        with torch.cuda.stream(s):
            got.append(corr.correlate(jobs[i % 5], stream=s))
    torch.cuda.synchronize()
    for i, (v, w) in enumerate(got):
        assert torch.equal(v, refs[i % 5][0]) and torch.equal(w, refs[i % 5][1]), i
