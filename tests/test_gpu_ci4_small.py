"""CI4 passes of up to 64 inputs (64-row tiles) against the oracle, bit for bit:
around the 16-, 32- and 64-row blocks, the 16-byte pieces, the 64-byte stages,
the pipeline's depth and the K splits, aligned rows longer than the pass."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import CORR_DUMP_INTEG, Correlator

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_in,n_ch", [(1, 2), (16, 3), (31, 2), (33, 1), (63, 2), (64, 40), (65, 1)])
def test_up_to_64_inputs(n_in, n_ch):
    for T in (1, 15, 16, 17, 63, 64, 65, 191, 193, 257, 1000, 2049):
        x = synth.ci8(seed=n_in + T, n_channels=n_ch, n_inputs=n_in, n_samples=T)
        want = oracle.xengine_ci8(x)
        row = (T + 15) // 16 * 16 + 16
        b = np.full((n_ch, n_in, row), 0x77, np.uint8)   # what lies past the pass would show in the sums
        b[:, :, :T] = (x[..., 0].astype(np.int32) & 15) << 4 | x[..., 1].astype(np.int32) & 15
        c = Correlator(n_in, n_ch, engine="i8", sample_type="ci4", max_abs=7, device=DEV)
        c.correlate(torch.from_numpy(b).to(DEV), n_samples=T)
        out, n, exact = c.dump(CORR_DUMP_INTEG, device_out=False)
        c.close()
        assert n == T and exact
        assert np.array_equal(out.numpy().astype(np.int64), want), T
