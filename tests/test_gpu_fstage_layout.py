"""F-stage calls of every split (4, 8 or 16 inputs per workgroup, chosen by the
size of the call) and input alignment give the same codes.

Each call is compared, bit for bit, with the same blocks given 15 at a time:
those launches have 4 inputs per workgroup and a ragged block group.
The arithmetic of a block (of a pair of real inputs) does not depend on the
split, so nothing may differ; the small calls' spectra and codes are held to
the FP64 transform."""
import numpy as np
import pytest
import torch

import fcheck
import oracle
import synth
from paper_0906_1887_amd import Correlator

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SCALE = {"r8": float(np.float32(1.0 / 90.0)), "cw16": 1.0 / 16.0, "cb8": 1.0 / 16.0}  # parts of about 2 levels rms


def make(fmt, taps, n_in, ring):
    return Correlator(n_in, 128, engine="i8", fft_size=256 if fmt == "r8" else 128, max_abs=7, requant_scale=SCALE[fmt],
                      ring_samples=ring, device=DEV, volt_format=fmt, pfb_taps=taps)


def raw_rows(fmt, blocks, n_in):
    if fmt == "r8":
        return synth.real_voltages(seed=3, index=n_in, n_blocks=blocks, n_inputs=n_in).reshape(-1, n_in)
    if fmt == "cw16":
        rec, _ = synth.capture_records(seed=3, index=n_in, n_records=blocks * 128, n_streams=1, w_per=n_in)
        return np.ascontiguousarray(rec[0, :, 1:]).view(np.int16)
    return synth.complex_bytes(seed=3, index=n_in, n_samples=blocks * 128, n_inputs=n_in)[0]


# n_in x block counts on both sides of each rule (1024 workgroups of 16 or of 8
# real inputs, 768 of 8 complex ones), with a ragged last block group; n_in that
# are multiples of 16, 8, 4 and of none
CASES = [("r8", 0, 64, 4083), ("r8", 0, 64, 4103), ("r8", 0, 72, 1819), ("r8", 0, 72, 1803), ("r8", 0, 20, 77),
         ("r8", 0, 13, 40), ("r8", 0, 1, 33), ("r8", 4, 64, 2059), ("r8", 4, 64, 2027), ("r8", 4, 12, 50),
         ("r8", 4, 5, 21), ("cw16", 0, 64, 1545), ("cw16", 0, 64, 1519), ("cw16", 0, 12, 45), ("cw16", 0, 3, 18),
         ("cb8", 0, 64, 1545), ("cb8", 0, 64, 1519), ("cb8", 0, 12, 45), ("cb8", 0, 7, 18),
         # the last input group reads back into the row; the fewest inputs
         ("r8", 0, 62, 300), ("r8", 0, 3, 35), ("r8", 4, 1, 18), ("r8", 4, 30, 65), ("cw16", 0, 61, 129),
         ("cw16", 0, 2, 17), ("cw16", 0, 1, 34), ("cb8", 0, 58, 100), ("cb8", 0, 1, 31), ("cb8", 0, 2, 16)]


@pytest.mark.parametrize("fmt,taps,n_in,n_blocks", CASES)
def test_split_and_alignment_do_not_change_a_code(fmt, taps, n_in, n_blocks):
    fft = 256 if fmt == "r8" else 128
    hist = max(0, taps - 1)
    raw = raw_rows(fmt, n_blocks + hist, n_in)
    c = make(fmt, taps, n_in, n_blocks + 8)
    flat = torch.zeros(raw.size + 32, dtype=torch.from_numpy(raw[:0]).dtype, device=DEV)

    def at(offset, b0, b1):
        """Blocks b0 .. b1 - 1, with their history, as a view `offset` elements into the buffer."""
        flat[offset:offset + raw.size] = torch.from_numpy(raw.reshape(-1)).to(DEV)
        row = fft * n_in
        return flat[offset + b0 * row:offset + (b1 + hist) * row].view(-1, n_in)

    # reference: 15 blocks a call; the last call's spectra against the transform
    for b0 in range(0, n_blocks, 15):
        b1 = min(n_blocks, b0 + 15)
        dbg = torch.empty((128, n_in, b1 - b0, 2), dtype=torch.float32, device=DEV)
        if b0 == 0:
            x = at(0, 0, n_blocks)
        c.channelise(x[b0 * fft:(b1 + hist) * fft], first_seq=b0, spectra_dbg=dbg)
    want = c.ring_read().numpy()
    if taps == 0:
        last = raw[b0 * fft:b1 * fft]
        if fmt == "r8":
            X, bound = oracle.dft_real(last, 256), fcheck.real_bound(last, 256)
        else:
            lv = oracle.unpack_w16(last.view(np.uint16)) if fmt == "cw16" else oracle.unpack_b8(last.view(np.uint8))
            X, bound = oracle.dft_complex(lv, 128), fcheck.complex_bound(lv, 128)
        fcheck.check_spectra_requant(X, dbg.cpu().numpy(), want[:, :, b0:b1], SCALE[fmt], 7, bound, fmt)
    c.close()
    for offset in (0, 1, 2, 4, 8):
        c = make(fmt, taps, n_in, n_blocks + 8)
        c.channelise(at(offset, 0, n_blocks), first_seq=0)
        got = c.ring_read().numpy()
        c.close()
        assert np.array_equal(got, want), f"buffer offset {offset}"
