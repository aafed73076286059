"""Read-outs by every route: the one-launch kernel into device memory (any
4-byte alignment, sizes that are not whole 16-byte pieces), the pinned staging
of small results for host memory, the runtime's copy for larger ones, and
plans beyond the pinned slots, each with and without the long-run fold.
Integer samples: the integration must equal the oracle and the long-run sum
the sum of the folded integrations, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import (CORR_DUMP_FOLD, CORR_DUMP_INTEG, CORR_DUMP_LONGRUN, CORR_DUMP_NO_RESET, Correlator,
                                 _lib)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dump_to(c, what, where, count, dtype):
    """Dump `count` scalars to host memory, or to device memory `where` bytes past an allocation's start;
    what lies around the result must stay as it was."""
    size = count * np.dtype(dtype).itemsize
    if where == "host":
        out = np.zeros(count, dtype)
        n, exact = _lib.corr_dump(c.plan, what, out.ctypes.data, False)
        return out, n, exact
    buf = torch.full((where + size + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    n, exact = _lib.corr_dump(c.plan, what, buf.data_ptr() + where, True)
    h = buf.cpu().numpy()
    assert (h[:where] == 0x5A).all() and (h[where + size:] == 0x5A).all()
    return h[where:where + size].copy().view(dtype), n, exact


# (1, 1): one product; (5, 3): 45 products, a partial 16-byte piece at the end; (40, 3) staged for the host;
# (64, 8): 133 KB, past the staging room (its long-run sum is past it from (40, 11) on)
@pytest.mark.parametrize("n_in,n_ch", [(1, 1), (5, 3), (40, 3), (40, 11), (64, 8)])
@pytest.mark.parametrize("where", [0, 4, 8, "host"])
@pytest.mark.parametrize("engine", ["i8", "fp32"])
def test_every_dump_mode(engine, where, n_in, n_ch):
    xs = [synth.ci8(seed=60 + k, n_channels=n_ch, n_inputs=n_in, n_samples=96) for k in range(3)]
    want = [oracle.xengine_ci8(x).reshape(-1) for x in xs]
    count, dt = want[0].size, np.int32 if engine == "i8" else np.float32
    c = Correlator(n_in, n_ch, engine=engine, max_abs=7, fp64_longrun=True, device=DEV)
    for k, x in enumerate(xs):
        c.correlate(torch.from_numpy(x).to(DEV))
        if k == 0:      # read, keep, then fold without a copy
            got, n, exact = dump_to(c, CORR_DUMP_INTEG | CORR_DUMP_NO_RESET, where, count, dt)
            assert n == 96 and exact and np.array_equal(got.astype(np.int64), want[0])
            _lib.corr_dump(c.plan, CORR_DUMP_FOLD, 0, False)
        elif k == 1:    # fold and read the integration
            got, n, exact = dump_to(c, CORR_DUMP_FOLD | CORR_DUMP_INTEG, where, count, dt)
            assert n == 96 and exact and np.array_equal(got.astype(np.int64), want[1])
        else:           # fold and read the long-run sum
            got, n, exact = dump_to(c, CORR_DUMP_FOLD | CORR_DUMP_LONGRUN, where, count, np.float64)
            assert n == 96 and exact and np.array_equal(got, sum(want).astype(np.float64))
    # nothing accumulated: the long-run sum is unchanged, the integration reads as zeros
    got, n, _ = dump_to(c, CORR_DUMP_FOLD | CORR_DUMP_LONGRUN, where, count, np.float64)
    assert n == 0 and np.array_equal(got, sum(want).astype(np.float64))
    got, n, _ = dump_to(c, CORR_DUMP_INTEG, where, count, dt)
    assert n == 0 and not got.any()
    c.close()


def test_more_plans_than_pinned_slots():
    x = synth.ci8(seed=70, n_channels=2, n_inputs=9, n_samples=64)
    want, d = oracle.xengine_ci8(x), torch.from_numpy(x).to(DEV)
    plans = [Correlator(9, 2, engine="i8", max_abs=7, device=DEV) for _ in range(40)]
    for turn in range(2):
        for k, c in enumerate(plans):
            c.correlate(d)
            out, n, exact = c.dump(CORR_DUMP_INTEG, device_out=bool((k + turn) & 1))
            assert n == 64 and exact and np.array_equal(out.cpu().numpy().astype(np.int64), want), k
        for c in plans[::3]:      # slots come back and are taken again
            c.close()
        plans = [Correlator(9, 2, engine="i8", max_abs=7, device=DEV) if k % 3 == 0 else c for k, c in enumerate(plans)]
    for c in plans:
        c.close()
