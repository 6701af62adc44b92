"""Per-channel Key calibration at the edges of its launch rule: every channel grouping, row counts around the
tail sample's threshold, outlier counts from none to almost half, unaligned input.  Bit-exact against the oracle."""
import numpy as np
import pytest

from oracle import kvq_calib_oracle as C

pytestmark = pytest.mark.gpu


def _keys(T, D, seed, kind):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((T, D)) * np.exp(rng.standard_normal(D)) + rng.standard_normal(D)
    if kind == "drift":                       # later rows ever larger: the sampled rows are no random sample
        x = x * (1.0 + np.arange(T)[:, None] / 7.0)
    elif kind == "coarse":                    # a handful of distinct values, zeros of both signs among them
        x = np.round(x) * 0.5
    return x.astype(np.float16)


@pytest.mark.parametrize("T,D,p,shift,kind", [
    (1200, 4096, 0.01, 0, "plain"),           # 16 channels per workgroup
    (513, 5120, 0.02, 0, "coarse"),           # 16, row steps with a remainder
    (1009, 2048, 0.01, 0, "plain"), (1008, 2048, 0.01, 0, "drift"),         # 8
    (8177, 2048, 0.01, 0, "plain"),           # 8; the smallest row count whose rows are sampled
    (8176, 2048, 0.01, 0, "drift"),           # 8; one row fewer: no sample
    (1100, 1024, 0.0563, 0, "plain"), (1100, 1024, 0.07, 0, "drift"),       # 4
    (8200, 1024, 0.0622, 0, "plain"),         # 4; 2 (k + 1) just fits the sample of 513 rows
    (8200, 1024, 0.0625, 0, "drift"),         # 4; and just does not
    # 16 and 1, sampled.  (Not "drift" over so many rows and channels: its factor of up to 1287 takes values past the
    # largest fp16 number, and infinite inputs are outside the call's contract.)
    (9000, 4096, 0.01, 0, "plain"), (9001, 515, 0.01, 0, "coarse"),
    (3000, 514, 0.01, 0, "drift"),            # 2
    (3000, 300, 0.99, 0, "coarse"),           # 1; both sides meet in the middle
    (1500, 515, 0.01, 0, "plain"),            # 1; odd row length
    (1100, 4096, 0.0, 1, "coarse"),           # 1; input not 16-byte aligned; no outliers
    (32768, 24, 0.01, 0, "drift"),            # the most rows
    (3, 4096, 0.5, 0, "plain"),               # fewer rows than a workgroup step
])
def test_channel_constants_at_the_edges(T, D, p, shift, kind):
    import torch
    import paper_2401_18079_amd as K
    x = _keys(T, D, T + D, kind)
    buf = torch.zeros(T * D + shift, dtype=torch.float16, device="cuda")
    dev = buf[shift:].view(T, D)
    dev.copy_(torch.from_numpy(x))
    got = K.kvq_calibrate_key_channels(dev, p)
    for name, a, b in zip(("s", "z", "lo", "hi"), got, C.key_channel_constants(x, p)):
        assert np.array_equal(a, b), (name, np.nonzero(a != b)[0][:5])


@pytest.mark.parametrize("bits,n,kind", [
    (4, 100003, "plain"), (3, 5, "plain"), (2, 1 << 20, "plain"),
    (4, 50001, "close"),                      # two decision points in one cell of the look-up
    (3, 50002, "unsorted"),                   # signposts that do not ascend
    (4, 50003, "wide"),                       # signposts beyond [-1, 1]
    (3, 40000, "equal"),                      # signposts that coincide
    (4, 40001, "far"),                        # values far outside the signposts
    # from 6 Mi elements of 16 signposts on the look-up is taken; the last size below it, and every way out of it
    (4, (6 << 20) - 1, "plain"), (4, 6 << 20, "plain"), (4, (6 << 20) + 3, "close"), (4, (6 << 20) + 2, "unsorted"),
    (4, (6 << 20) + 1, "wide"), (4, (6 << 20) + 5, "equal"), (4, (6 << 20) + 6, "far"),
])
def test_signposts_where_the_look_up_could_part_from_the_search(bits, n, kind):
    import torch
    import paper_2401_18079_amd as K
    rng = np.random.default_rng(n + bits)
    k = 1 << bits
    c = np.linspace(-1, 1, k)
    if kind == "close":
        c[1:4] = [-0.5, -0.4999, -0.4998]
    elif kind == "unsorted":
        c = rng.permutation(c)
    elif kind == "wide":
        c = c * 3.0
    elif kind == "equal":
        c[2] = c[1]
    c = c.astype(np.float32)
    x = rng.standard_normal(n) * 0.4
    mid = (np.sort(c)[1:] + np.sort(c)[:-1]) / 2
    x[::7] = rng.choice(mid, x[::7].size)     # on the decision points, and next to them
    x = x.astype(np.float32)
    x[::14] = np.nextafter(x[::14], np.float32(9.0))
    if kind == "far":
        x[::101] = rng.choice(np.float32([127.5, -300.0, 1e6, -3e8]), x[::101].size)
    w = np.exp(rng.standard_normal(n)).astype(np.float32)
    got = K.kvq_calibrate_nuq(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), bits, 1, c)
    # one iteration: the assignment is exact, the sums are fp64 in another order (a few ulps of fp64), one rounding to fp32
    idx = C.nearest(x, c)
    ref = c.astype(np.float64)
    for j in range(k):
        m = idx == j
        if w[m].sum() > 0:
            ref[j] = (w[m].astype(np.float64) * x[m]).sum() / w[m].astype(np.float64).sum()
    ref = np.sort(ref)
    assert np.all(np.abs(got - ref) <= 2.0 ** -23 * np.maximum(np.abs(ref), 1e-12 * n)), (got, ref)
