"""A read-out into device memory that ends past its allocation is refused by the
runtime, as any copy there is; one that ends with it is not.  (9, 5) has 1800
bytes of products, so the pages of an allocation of its own hold the result in
either case."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import CORR_DUMP_INTEG, Correlator, _lib

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("missing", [0, 4, 64])
def test_destination_within_its_allocation(missing):
    hip = _lib.lib()          # the runtime that the library is linked to
    x = synth.ci8(seed=81, n_channels=5, n_inputs=9, n_samples=64)
    want = oracle.xengine_ci8(x)
    size = want.size * 4
    c = Correlator(9, 5, engine="i8", max_abs=7, device=DEV)
    c.correlate(torch.from_numpy(x).to(DEV))
    ptr = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(ptr), ctypes.c_size_t(size + 64 - missing)) == 0
    try:
        if missing:
            with pytest.raises(_lib.CorrError):
                _lib.corr_dump(c.plan, CORR_DUMP_INTEG, ptr.value + 64, True)
            hip.hipGetLastError()
        else:
            n, exact = _lib.corr_dump(c.plan, CORR_DUMP_INTEG, ptr.value + 64, True)
            got = np.zeros(want.size, np.int32)
            assert hip.hipMemcpy(ctypes.c_void_p(got.ctypes.data), ctypes.c_void_p(ptr.value + 64),
                                 ctypes.c_size_t(size), 2) == 0
            assert n == 64 and exact and np.array_equal(got, want.reshape(-1).astype(np.int32))
    finally:
        torch.cuda.synchronize()
        hip.hipFree(ptr)
        c.close()
