"""Later calls of an integration add to the products of the earlier ones, every
engine and tile shape: one call, then further ones of other lengths, against the
oracle's sum over all samples.  The samples are integers whose sums every engine
holds exactly, so nothing may differ."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import CORR_DUMP_INTEG, Correlator

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CUTS = (0, 40, 56, 96, 97, 160)   # short passes: one K split, so products are added by the X-engine itself


# on both sides of the 16-, 32-, 64- and 128-row tiles
@pytest.mark.parametrize("n_in,n_ch", [(1, 3), (17, 2), (63, 2), (64, 3), (65, 2), (100, 1), (129, 2), (257, 1)])
@pytest.mark.parametrize("engine,sample,ring", [("i8", "ci8", 0), ("i8", "ci4", 0), ("fp32", "ci8", 0), ("fp32m", "cf32", 0),
                                                ("f16", "cf32", 0), ("f16", "cf32", 64), ("f8", "cf32", 0),
                                                ("f8", "cf32", 64)])
def test_calls_add_up(engine, sample, ring, n_in, n_ch):
    x = synth.ci8(seed=n_in, n_channels=n_ch, n_inputs=n_in, n_samples=CUTS[-1])
    want = oracle.xengine_ci8(x)
    c = Correlator(n_in, n_ch, engine=engine, sample_type=sample, max_abs=0 if sample == "cf32" else 7,
                   ring_samples=ring, device=DEV)
    for rep in range(2):   # the second integration stores over what the first one left
        for t0, t1 in zip(CUTS, CUTS[1:]):
            part = x[:, :, t0:t1]
            if engine == "fp32m" and (t1 - t0) % 2:   # whole pairs of samples: a zero one added
                part = np.concatenate([part, np.zeros_like(part[:, :, :1])], axis=2)
            if sample == "ci4":   # rows of a multiple of 16 bytes
                b = np.zeros((n_ch, n_in, (t1 - t0 + 15) // 16 * 16), np.uint8)
                b[:, :, :t1 - t0] = ((part[..., 0].astype(np.int32) & 15) << 4 | part[..., 1].astype(np.int32) & 15)
                c.correlate(torch.from_numpy(b).to(DEV), n_samples=t1 - t0)
            else:
                v = part.astype(np.float32) if sample == "cf32" else part
                c.correlate(torch.from_numpy(np.ascontiguousarray(v)).to(DEV))
        out, n, _ = c.dump(CORR_DUMP_INTEG, device_out=False)
        assert n == CUTS[-1] + 2 * (engine == "fp32m")   # two odd parts
        assert np.array_equal(out.numpy().astype(np.int64), want), rep
    c.close()
