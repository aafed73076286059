"""The plain FP32 engine on up to 32 inputs, whose channels share a workgroup (4 of
up to 32 inputs, 8 of up to 16): every input count around the 4-row blocks and
the panel's rows, channel counts that do and do not fill the last workgroup."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import CORR_DUMP_INTEG, Correlator, _lib, make_config

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_in", [1, 3, 4, 5, 8, 13, 16, 17, 20, 31, 32, 33])
@pytest.mark.parametrize("n_ch,T", [(1, 1), (2, 17), (3, 130), (4, 64), (5, 1100), (7, 15), (8, 33), (9, 257), (17, 500)])
def test_integer_samples_are_exact(n_in, n_ch, T):
    x = synth.ci8(seed=n_in + T, n_channels=n_ch, n_inputs=n_in, n_samples=T)
    want = oracle.xengine_ci8(x)
    for sample, d in (("ci8", torch.from_numpy(x).to(DEV)), ("cf32", torch.from_numpy(x).to(DEV).float())):
        c = Correlator(n_in, n_ch, engine="fp32", sample_type=sample, max_abs=7, device=DEV)
        c.correlate(d)
        c.correlate(d)   # adds to the first pass
        got, n, _ = c.dump(CORR_DUMP_INTEG, device_out=False)
        c.close()
        assert n == 2 * T and np.array_equal(got.numpy().astype(np.int64), 2 * want), sample


@pytest.mark.parametrize("n_in,n_ch,T", [(16, 40, 900), (32, 7, 555), (21, 30, 3000)])
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
