"""The plain FP32 engine's work items: diagonal tiles in pairs (odd and even
counts, pairs that span two channels), off-diagonal tiles, K splits of any
count, accumulation, and corr_correlate_static on the same split."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import CORR_DUMP_INTEG, Correlator, _lib, make_config

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# input counts around the 64-row tiles and their 16 x 16 thread blocks (4 rows each); 1 to 3 channels give odd and
# even numbers of diagonal tiles; sample counts around the 16-sample stages and the 4-stage minimum of a split
@pytest.mark.parametrize("n_in,n_ch", [(1, 1), (4, 3), (33, 2), (61, 5), (64, 1), (64, 4), (65, 3), (128, 1), (130, 3),
                                       (193, 2)])
@pytest.mark.parametrize("T", [1, 15, 17, 64, 129, 1100])
def test_integer_samples_are_exact(n_in, n_ch, T):
    x = synth.ci8(seed=n_in + T, n_channels=n_ch, n_inputs=n_in, n_samples=T)
    want = oracle.xengine_ci8(x)
    for sample, d in (("ci8", torch.from_numpy(x).to(DEV)), ("cf32", torch.from_numpy(x).to(DEV).float())):
        c = Correlator(n_in, n_ch, engine="fp32", sample_type=sample, max_abs=7, device=DEV)
        c.correlate(d)
        got, n, exact = c.dump(CORR_DUMP_INTEG | 8, device_out=False)     # keep: the next pass adds to it
        assert n == T and exact and np.array_equal(got.numpy().astype(np.int64), want), sample
        c.correlate(d)
        got, n, _ = c.dump(CORR_DUMP_INTEG, device_out=False)
        assert n == 2 * T and np.array_equal(got.numpy().astype(np.int64), 2 * want), sample
        c.close()


@pytest.mark.parametrize("n_in,n_ch,T", [(64, 40, 900), (100, 7, 555), (200, 3, 1000)])
def test_float_samples_and_the_static_call(n_in, n_ch, T):
    rng = np.random.default_rng(n_in)
    x = rng.standard_normal((n_ch, n_in, T, 2)).astype(np.float32)
    d = torch.from_numpy(x).to(DEV)
    c = Correlator(n_in, n_ch, engine="fp32", sample_type="cf32", max_abs=0, device=DEV)
    c.correlate(d)
    got = c.dump(CORR_DUMP_INTEG, device_out=True)[0]
    c.close()
    out = torch.zeros_like(got)
    cfg = make_config(n_in, n_ch, engine="fp32", sample_type="cf32", max_abs=0)
    _lib.corr_correlate_static(cfg, d.data_ptr(), T, T, out.data_ptr(), False, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), out.view(torch.int32))
    want = oracle.xengine_cf64(x)
    # sums of 2T products of unit variance: rounding of at most one ulp an addition, relative to the sum's scale
    err = np.linalg.norm(got.cpu().numpy().astype(np.float64) - want) / np.linalg.norm(want)
    assert err < 2 * T * 2.0 ** -24, err
