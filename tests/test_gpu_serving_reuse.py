"""The serving queue under reuse: a caller's ring that is rewritten between jobs
while one grid keeps running (its caches may hold the former samples), slots
that serve many jobs in turn, and more jobs at once than there are slots.
Every result must equal the oracle bit for bit."""
import time

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_0906_1887_amd import Scheduler

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def wait_all(s, ids, timeout=60.0):
    t0 = time.time()
    while ids:
        left = []
        for j in ids:
            r = s.poll(j)
            if r is None:
                left.append(j)
            else:
                assert r[0] == 0
        ids = left
        assert time.time() - t0 < timeout, f"{len(ids)} jobs not done"


def result(n_in, n_ch):
    return torch.empty((n_ch, n_in * (n_in + 1) // 2, 2), dtype=torch.int32, device=DEV)


def test_ring_rewritten_while_the_grid_runs():
    n_in, n_ch, T = 16, 64, 96
    xs = [synth.ci8(seed=300 + k, n_channels=n_ch, n_inputs=n_in, n_samples=T) for k in range(4)]
    want = [torch.from_numpy(oracle.xengine_ci8(x).astype(np.int32)) for x in xs]
    src = [torch.from_numpy(x).to(DEV) for x in xs]
    ring, out = torch.empty_like(src[0]), result(n_in, n_ch)
    busy = torch.zeros((256, 64, 4000, 2), dtype=torch.int8, device=DEV)     # keeps the grid from idling
    spare = [result(64, 256) for _ in range(3)]
    torch.cuda.synchronize()
    s = Scheduler(64 << 20, 2)
    st = torch.cuda.current_stream()
    try:
        for k in range(60):
            background = [s.submit(64, 256, 4000, o, d_samples=busy.data_ptr()) for o in spare]
            ring.copy_(src[k % 4])
            st.synchronize()               # the ring holds the new samples (the grid runs on)
            wait_all(s, [s.submit(n_in, n_ch, T, out, d_samples=ring.data_ptr())])
            got = torch.empty(out.shape, dtype=out.dtype, pin_memory=True)
            got.copy_(out, non_blocking=True)
            st.synchronize()
            assert torch.equal(got, want[k % 4]), k
            wait_all(s, background)
    finally:
        s.close()


def test_many_jobs_through_few_slots():
    shapes = [(5, 3, 40), (130, 2, 72), (16, 64, 200), (64, 8, 1000)]
    xs = [synth.ci8(seed=320 + k, n_channels=c, n_inputs=n, n_samples=t) for k, (n, c, t) in enumerate(shapes)]
    want = [oracle.xengine_ci8(x) for x in xs]
    dev = [torch.from_numpy(x).to(DEV) for x in xs]
    torch.cuda.synchronize()
    s = Scheduler(64 << 20, 2)
    try:
        outs = [result(*shapes[k % 4][:2]) for k in range(200)]
        wait_all(s, [s.submit(*shapes[k % 4], o, d_samples=dev[k % 4].data_ptr()) for k, o in enumerate(outs)])
        torch.cuda.synchronize()
        for k, o in enumerate(outs):
            assert np.array_equal(o.cpu().numpy().astype(np.int64), want[k % 4]), k
        assert s.stats()["completed"] == 200
    finally:
        s.close()
