"""The converting FP16 engine on 129 to 256 inputs, where one workgroup takes a
channel, against the oracle on integer samples (whose sums it holds exactly) and
on passes around the steady loop's first and last stage; passes and channel
counts on the other side of the rule run the tiles and must agree too."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import CORR_DUMP_INTEG, Correlator

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# 129 to 256 inputs around the 32-row blocks; 128 channels and few samples: one split, half a round of workgroups
# (127: less); a few channels and many samples: K splits that fill half a round (22 channels: less)
@pytest.mark.parametrize("n_in,n_ch,T", [(129, 128, 400), (160, 128, 401), (161, 128, 415), (255, 128, 416), (256, 128, 417),
                                         (256, 127, 417), (200, 128, 399), (192, 130, 431), (224, 128, 432), (250, 128, 433),
                                         (129, 24, 8000), (256, 23, 6500), (130, 22, 8000)])
def test_integer_samples_are_exact(n_in, n_ch, T):
    x = synth.ci8(seed=n_in + T, n_channels=min(n_ch, 6), n_inputs=n_in, n_samples=T)
    x = np.tile(x, ((n_ch + 5) // 6, 1, 1, 1))[:n_ch]
    want = oracle.xengine_ci8(x[:6])
    c = Correlator(n_in, n_ch, engine="f16", sample_type="cf32", max_abs=0, device=DEV)
    stride = T + 1 + T % 2                       # odd: rows at any multiple of 8 bytes
    d = torch.full((n_ch, n_in, stride, 2), 9.0, device=DEV)   # what lies past the pass would show in the sums
    d[:, :, :T] = torch.from_numpy(x).to(DEV).float()
    for rep in (1, 2):                           # the second pass adds to the first
        c.correlate(d, n_samples=T)
    out, n, _ = c.dump(CORR_DUMP_INTEG, device_out=False)
    c.close()
    got = out.numpy().astype(np.int64)
    assert n == 2 * T
    for ch in range(n_ch):
        assert np.array_equal(got[ch], 2 * want[ch % 6]), ch
