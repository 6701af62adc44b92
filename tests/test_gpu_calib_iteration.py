"""GPU parity of one k-means iteration where its launch changes form: element counts at either side of the look-up's lower
limit (3 Mi elements of 16 signposts) and at whole and ragged rounds of the grid, starts whose thresholds lie near zero, in one
cell of the look-up or beside each other's rounding.  Tolerance: see test_gpu_calib.py."""
import numpy as np
import pytest

import kvq_synth as S
from oracle import kvq_calib_oracle as C

pytestmark = pytest.mark.gpu

ATOL = 2e-6


def _start(kind, bits):
    k = 1 << bits
    c = np.linspace(-1, 1, k).astype(np.float32)
    if kind == "zero":                       # the middle threshold at a few 1e-8
        c[k // 2 - 1], c[k // 2] = np.float32(-0.06), np.float32(0.06 + 3e-8)
    if kind == "close":                      # two thresholds in one cell, signposts at the smallest distance that is counted on
        c[3] = c[2] + np.float32(2.0 ** -15)
        c[4] = c[3] + np.float32(2.0 ** -15)
    if kind == "closer":                     # below it
        c[3] = c[2] + np.float32(2.0 ** -17)
    return np.sort(c)


@pytest.mark.parametrize("bits,n,kind", [
    (4, (3 << 20) - 1, "even"), (4, 3 << 20, "even"), (4, (3 << 20) + 5, "zero"), (4, 3 << 20, "close"), (4, 3 << 20, "closer"),
    (4, 512 * 1024, "zero"), (4, 512 * 1024 + 2049, "even"), (3, 1024 * 1024 + 1, "close"), (2, 3 * 512 * 1024 - 3, "even"),
    (2, 2047, "even"), (3, 2048, "even"), (4, 2049, "zero"),
])
def test_iterations_match_oracle(bits, n, kind):
    import torch
    import paper_2401_18079_amd as K
    x, w = S.gen_calibration(4711 + n, n)
    c0 = _start(kind, bits)
    got = K.kvq_calibrate_nuq(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), bits, 2, c0)
    ref = C.nuq_signposts(x, w, c0, 2)
    assert np.allclose(got, ref, rtol=0, atol=ATOL), (got, ref)


def test_on_a_stream_of_the_caller():
    import torch
    import paper_2401_18079_amd as K
    x, w = S.gen_calibration(4712, 70001)
    c0 = _start("even", 4)
    dx, dw = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got = K.kvq_calibrate_nuq(dx, dw, 4, 2, c0, stream=side)
    assert np.allclose(got, C.nuq_signposts(x, w, c0, 2), rtol=0, atol=ATOL)
