"""FP16 / FP8 staging of rows of every length (a workgroup's lanes share one row
or several) against the oracle's encoder, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import Correlator

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# around the powers of two of a row's lanes (2 or 4 samples each), the 256 lanes
# of a workgroup, its rows, and the 4-fold steps of the maximum's loop
@pytest.mark.parametrize("T", [1, 2, 3, 4, 5, 8, 9, 15, 17, 64, 65, 129, 255, 257, 513, 1023, 1025, 2049, 4097])
@pytest.mark.parametrize("engine", ["f16", "f8"])
def test_rows_of_every_length(engine, T):
    for n_in, n_ch in ((1, 2), (5, 2), (67, 1)):
        x = np.stack([synth.complex_float(7 + T, ch, n_in, T) for ch in range(n_ch)])
        x[0, n_in - 1, T - 1, 1] = -40.0   # the channel's largest value is its last one
        c = Correlator(n_in, n_ch, engine=engine, sample_type="cf32", max_abs=0, ring_samples=T, device=DEV)
        c.correlate(torch.from_numpy(x).to(DEV))
        st, sc = c.stage_read()
        c.close()
        for ch in range(n_ch):
            if engine == "f16":
                want = oracle.f16_encode(x[ch].astype(np.float64))
            else:
                s = oracle.e4m3_scale(x[ch].astype(np.float64))
                assert sc[ch] == s, (n_in, ch)
                want = oracle.e4m3_encode(x[ch].astype(np.float64) * s)
            assert np.array_equal(st[ch].reshape(-1), np.asarray(want).reshape(-1)), (n_in, ch)
