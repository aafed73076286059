"""Products at the edges of a tile's row groups (16 rows, 32, 64, 128 and their
neighbours) on the matrix-core engines, in a first pass and in one that adds to
it.  Samples are integers in [-7, 7]: exact in FP16 and in scaled FP8, with sums
below 2^24, so every engine must equal the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import Correlator

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("engine", ["i8", "fp32m", "f16", "f8"])
@pytest.mark.parametrize("n_in", [1, 3, 16, 17, 31, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 113, 128, 145, 193])
def test_rows(engine, n_in):
    n_ch, T = 3, 104
    x = synth.ci8(seed=900 + n_in, n_channels=n_ch, n_inputs=n_in, n_samples=T)
    want = oracle.xengine_ci8(x)
    float_in = engine != "i8"
    d = torch.from_numpy(x).to(DEV)
    d = d.float().contiguous() if float_in else d
    c = Correlator(n_in, n_ch, engine=engine, sample_type="cf32" if float_in else "ci8",
                   max_abs=7 if engine in ("i8", "fp32m") else 0, ring_samples=T if engine in ("f16", "f8") else 0, device=DEV)
    for passes in (1, 2):
        for _ in range(passes):
            c.correlate(d)
        out, n, _ = c.dump()
        assert n == passes * T and np.array_equal(out.cpu().numpy().astype(np.float64), passes * want.astype(np.float64))
    c.close()
