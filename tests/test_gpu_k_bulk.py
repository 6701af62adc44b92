"""The bulk Key append with packed keys: every width of its rule and the call lengths at either side of it, runs that end short,
constants at which a short cut does not hold (open thresholds with elements beyond the code range, thresholds at zero of either
sign, scales of a few bits, zero or huge, signposts whose codes cannot be counted), full outlier arrays, infinities and NaN.
Bit-exact against the oracle, or, where constants or elements are outside its contract, against one-token calls, which another
kernel takes."""
import numpy as np
import pytest

import kvq_synth as S
from oracle import kvq_oracle as O
from kvq_testlib import Setup, compare_caches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,bits,T,n0,blocked", [
    (8, 2, 64, 0, False), (8, 3, 65, 1, True), (8, 4, 63, 0, False), (16, 3, 129, 3, False), (24, 4, 131, 0, True), (32, 2, 255, 1, False),
    (32, 3, 1027, 0, False), (32, 4, 700, 5, True), (40, 3, 64, 1, False), (40, 4, 771, 0, False), (48, 2, 130, 0, False), (56, 4, 129, 1, False),
    (64, 3, 515, 0, False), (64, 4, 128, 0, True), (36, 3, 130, 0, False),
])
def test_keys_match_the_oracle(heads, bits, T, n0, blocked):
    import torch
    import paper_2401_18079_amd as K
    wl = S.workload("c2", n_kv_heads=heads, n_q_heads=heads, bits=bits)
    st = Setup(wl)
    cap = (n0 + T + 127) // 128 * 128
    k, v = st.k(0, n0 + T), st.v(0, n0 + T)
    oc = O.OracleCache(bits, heads, heads, cap, st.k_side, wl.rope_base, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi,
                       cap_nnz_k=max(1024, st.cap_nnz_k(cap)))
    nnz = max(1024, st.cap_nnz_k(cap))
    gc = K.KvqCache(bits, heads, heads, cap, st.k_side, wl.rope_base, nnz, nnz_block_entries=1024 if blocked else None)
    K.kvq_lut_load(gc, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi)
    for a, b in ((0, n0), (n0, n0 + T)):
        if a < b:
            oc.append_k(k[a:b]); oc.append_v(v[a:b])
            K.kvq_quantize_append_kv(gc, torch.from_numpy(k[a:b]).cuda(), torch.from_numpy(v[a:b]).cuda())
    bad = compare_caches(oc, gc)
    assert not bad, bad


def _constants(D, rng, kind):
    s = np.exp(rng.standard_normal(D)).astype(np.float16)
    z = rng.standard_normal(D).astype(np.float16)
    lo, hi = (z - s).astype(np.float16), (z + s).astype(np.float16)
    if kind == "open":
        lo[:], hi[:] = np.float16(-65504), np.float16(65504)
        s[::3] = np.float16(1e-3)                        # elements far beyond the code range that are no outliers
    elif kind == "odd":
        e = np.arange(D) % 16
        lo[e == 0], hi[e == 1] = np.float16(0.0), np.float16(0.0)
        lo[e == 2], hi[e == 3] = np.float16(-0.0), np.float16(-0.0)
        s[e == 4] = np.float16(2.0 ** -24)
        s[e == 5] = np.float16(0.0)
        s[e == 6], z[e == 6] = np.float16(60000), np.float16(-60000)
        lo[e == 7], hi[e == 7] = np.float16(2.0), np.float16(-2.0)               # everything is an outlier
        lo[e == 8], hi[e == 8] = np.float16(np.nan), np.float16(np.nan)          # nothing is
        lo[e == 9], hi[e == 10] = np.float16(-np.inf), np.float16(np.inf)
        s[e == 11] = np.float16(-1.0)
        z[e == 12] = np.float16(np.inf)
    return s, z, lo, hi


@pytest.mark.parametrize("heads,bits,kind,posts,nnz", [
    (8, 2, "open", "plain", 1 << 16), (8, 3, "open", "plain", 1 << 16), (16, 4, "open", "plain", 1 << 17),
    (8, 3, "odd", "plain", 1 << 17), (16, 4, "odd", "plain", 1 << 18), (24, 2, "odd", "plain", 1 << 18),
    (8, 3, "plain", "wide", 1 << 17), (8, 4, "odd", "close", 1 << 17),           # codes that thresholds do not give
    (8, 3, "plain", "plain", 3000), (8, 4, "odd", "plain", 20001),               # full arrays
])
def test_constants_at_the_edges_as_in_one_token_calls(heads, bits, kind, posts, nnz):
    import torch
    import paper_2401_18079_amd as K
    rng = np.random.default_rng(heads + bits + nnz)
    D, T, n0 = heads * 128, 67, 1
    s, z, lo, hi = _constants(D, rng, kind)
    lut = np.linspace(-1, 1, 1 << bits).astype(np.float32)
    if posts == "wide":
        lut = lut * 3
    elif posts == "close":
        lut[2] = lut[1] + np.float32(2.0 ** -10) / 64
    x = (rng.standard_normal((n0 + T, D)) * 2 * np.exp(0.5 * rng.standard_normal(D))).astype(np.float16)
    x[5, :200] = np.float16(0.0); x[5, 200:400] = np.float16(-0.0)
    x[9, rng.permutation(D)[:60]] = np.float16(6e4)
    x[20, rng.permutation(D)[:9]] = np.float16(np.nan)
    x[33, rng.permutation(D)[:9]] = np.float16(np.inf)
    x[34, rng.permutation(D)[:3]] = np.float16(-np.inf)
    dev = torch.from_numpy(x).cuda()
    got = []
    for whole in (True, False):
        gc = K.KvqCache(bits, heads, heads, 128, 1, 10000.0, nnz)
        K.kvq_lut_load(gc, lut, lut, s, z, lo, hi)
        K.kvq_quantize_append_k(gc, dev[:n0])
        if whole:
            K.kvq_quantize_append_k(gc, dev[n0:])
        else:
            for t in range(n0, n0 + T):
                K.kvq_quantize_append_k(gc, dev[t:t + 1])
        torch.cuda.synchronize()
        n = int(gc.k_ptr.cpu().numpy().view(np.uint32)[n0 + T])
        got.append((gc.status(), n, {f: getattr(gc, f).cpu().numpy().copy() for f in ("k_codes", "k_ptr")},
                    gc.k_idx.cpu().numpy()[:n].copy(), gc.k_val.cpu().numpy()[:n].copy()))
    a, b = got
    assert a[0] == b[0] and (a[0] != 0) == (a[1] == nnz) and a[1] == b[1], (a[:2], b[:2])
    for f in a[2]:
        assert np.array_equal(a[2][f].view(np.uint8), b[2][f].view(np.uint8)), f
    assert np.array_equal(a[3].view(np.uint16), b[3].view(np.uint16))
    va, vb = a[4].view(np.float16), b[4].view(np.float16)
    assert np.array_equal(va.view(np.uint16)[~np.isnan(va)], vb.view(np.uint16)[~np.isnan(vb)]) and np.array_equal(np.isnan(va), np.isnan(vb))


@pytest.mark.parametrize("heads,bits,posts", [(8, 2, "plain"), (16, 3, "plain"), (8, 4, "plain"), (40, 4, "plain"), (8, 2, "near"), (8, 3, "near"),
                                              (32, 4, "near")])
def test_codes_of_outliers_beyond_the_code_range(heads, bits, posts):
    """Channels whose outlier thresholds lie well within the code range, as calibrated ones do, and elements far beyond both: there fp32
    distances to different signposts round to the same number, and the smaller index wins."""
    import torch
    import paper_2401_18079_amd as K
    rng = np.random.default_rng(heads * 8 + bits)
    D, T, n0 = heads * 128, 131, 1
    s, z = np.full(D, 0.01, np.float16), np.zeros(D, np.float16)
    s[D // 2:], z[D // 2:] = np.float16(0.25), np.float16(-0.5)
    lo, hi = (z - s).astype(np.float16), (z + s).astype(np.float16)
    lut = np.linspace(-1, 1, 1 << bits).astype(np.float32)
    if posts == "near":                                  # two signposts 2^-10 apart at either end: codes can still be counted
        lut[1], lut[-2] = lut[0] + np.float32(2.0 ** -10), lut[-1] - np.float32(2.0 ** -10)
    x = (z + s * rng.standard_normal((n0 + T, D)) * 0.3).astype(np.float16)
    for t in range(n0 + T):
        at = rng.permutation(D)[:64]
        far = np.concatenate([[6e4, -6e4, 1200, -1200, 120, -120], rng.uniform(1.2, 1.35, 10), rng.uniform(30, 33, 10), rng.uniform(-2000, 2000, 38)])
        x[t, at] = far.astype(np.float16)
    v = rng.standard_normal((n0 + T, D)).astype(np.float16)
    nnz = 1 << 16
    oc = O.OracleCache(bits, heads, heads, 256, 4, 10000.0, lut, lut, s, z, lo, hi, cap_nnz_k=nnz)
    gc = K.KvqCache(bits, heads, heads, 256, 4, 10000.0, nnz)
    K.kvq_lut_load(gc, lut, lut, s, z, lo, hi)
    for a, b in ((0, n0), (n0, n0 + T)):
        oc.append_k(x[a:b]); oc.append_v(v[a:b])
        K.kvq_quantize_append_kv(gc, torch.from_numpy(x[a:b]).cuda(), torch.from_numpy(v[a:b]).cuda())
    bad = compare_caches(oc, gc)
    assert not bad, bad


# Thresholds by head, each on every fifth channel among ordinary ones: no channel's range ends at the code range, so that the packed keys alone decide.
_EDGES = {
    "none": lambda z, s: (z - s, z + s), "lo +0": lambda z, s: (0.0 * z, abs(z) + s), "lo -0": lambda z, s: (-0.0 * abs(z), abs(z) + s),
    "hi +0": lambda z, s: (-abs(z) - s, 0.0 * abs(z)), "hi -0": lambda z, s: (-abs(z) - s, -0.0 * abs(z)),
    "zeros": lambda z, s: (0.0 * abs(z), -0.0 * abs(z)), "crossed": lambda z, s: (z + s, z - s), "infinite": lambda z, s: (z + np.inf, z - np.inf),
    "one value": lambda z, s: (z, z), "smallest": lambda z, s: (0 * z - 2.0 ** -24, 0 * z + 2.0 ** -24), "largest": lambda z, s: (0 * z - 65504.0, 0 * z + 65504.0),
}


@pytest.mark.parametrize("heads,bits,scales", [(16, 2, "normal"), (16, 3, "normal"), (24, 4, "normal"), (40, 3, "normal"), (24, 2, "mixed"), (16, 4, "mixed")])
def test_thresholds_at_the_edges_among_ordinary_channels(heads, bits, scales):
    """Against the oracle; with scales outside its contract on channels of their own heads ("mixed"), against one-token calls."""
    import torch
    import paper_2401_18079_amd as K
    rng = np.random.default_rng(100 * heads + bits)
    D, T, n0, nnz = heads * 128, 67, 1, heads * 128 * 68
    c = np.arange(D)
    s, z = np.exp(rng.standard_normal(D)).clip(0.1, 8).astype(np.float16), rng.standard_normal(D).astype(np.float16)
    names, head, special = list(_EDGES), c // 128, (c % 5 == 3)
    kind = np.where(special, head % len(names), 0)
    s[kind == names.index("largest")] = np.float16(600)
    z32, s32 = z.astype(np.float32), s.astype(np.float32)
    lo, hi = np.empty(D, np.float16), np.empty(D, np.float16)
    for i, name in enumerate(names):
        a, b = _EDGES[name](z32, s32)
        lo[kind == i], hi[kind == i] = a.astype(np.float16)[kind == i], b.astype(np.float16)[kind == i]
    crossed = ~(lo <= hi)
    assert np.all(crossed | ((lo >= z32 - 126 * s32) & (hi <= z32 + 126 * s32)))
    if scales == "mixed":
        odd = special & (head >= len(names))
        s[odd & (c % 3 == 0)], s[odd & (c % 3 == 1)], s[odd & (c % 3 == 2)] = np.float16(0), np.float16(-1), np.float16(2.0 ** -24)
    lut = np.linspace(-1, 1, 1 << bits).astype(np.float32)
    x = (z32 + 0.6 * s32 * rng.standard_normal((n0 + T, D))).astype(np.float16)
    at = rng.integers(0, 12, x.shape)                    # the thresholds themselves, their neighbours, zeros and the smallest numbers
    finite = ~np.isinf(lo)
    with np.errstate(over="ignore"):
        beside = np.nextafter(lo, np.float16(-np.inf)), np.nextafter(hi, np.float16(np.inf))
    for i, y in enumerate((lo, hi, *beside)):
        x = np.where((at == i) & finite & np.isfinite(y), y, x)
    for i, y in enumerate((0.0, -0.0, 2.0 ** -24, -2.0 ** -24)):
        x = np.where(at == 4 + i, np.float16(y), x)
    for t in range(0, n0 + T, 3):                        # tokens of which a few elements are out of the code range
        x[t, rng.permutation(D)[:24]] = np.float16(6e4) * rng.choice([-1, 1], 24).astype(np.float16)
    v = rng.standard_normal((n0 + T, D)).astype(np.float16)
    dev, dev_v = torch.from_numpy(x).cuda(), torch.from_numpy(v).cuda()

    def filled(step):
        gc = K.KvqCache(bits, heads, heads, 128, 4, 10000.0, nnz)
        K.kvq_lut_load(gc, lut, lut, s, z, lo, hi)
        for t in [0] + list(range(n0, n0 + T, step)):
            e = n0 if t < n0 else min(t + step, n0 + T)
            K.kvq_quantize_append_k(gc, dev[t:e])
            K.kvq_quantize_append_v(gc, dev_v[t:e])
        torch.cuda.synchronize()
        assert gc.status() == 0
        return gc

    gc = filled(T)
    if scales == "normal":
        oc = O.OracleCache(bits, heads, heads, 128, 4, 10000.0, lut, lut, s, z, lo, hi, cap_nnz_k=nnz)
        oc.append_k(x); oc.append_v(v)
        bad = compare_caches(oc, gc)
        assert not bad, bad
    else:
        ref = filled(1)
        for f in ("k_codes", "k_ptr", "k_idx"):
            assert torch.equal(getattr(gc, f), getattr(ref, f)), f
        a, b = (r.k_val.cpu().numpy().view(np.float16) for r in (gc, ref))
        assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a.view(np.uint16)[~np.isnan(a)], b.view(np.uint16)[~np.isnan(b)])


def _append_ms(gc, k, timer):
    import torch
    import paper_2401_18079_amd as K
    best = []
    for _ in range(6):
        timer.start()
        for _ in range(8):
            gc.c.n_tokens_k = 0
            K.kvq_quantize_append_k(gc, k)
        timer.stop()
        torch.cuda.synchronize()
        best.append(timer.elapsed_ms())
    return min(best)


@pytest.mark.parametrize("what", ["infinite", "NaN"])
def test_infinities_and_nan_cost_no_more_than_other_elements(what):
    """A factor of 2.9 when every lane that met one coded its elements one by one."""
    import torch
    import paper_2401_18079_amd as K
    heads, T = 32, 4096
    wl = S.workload("c2", n_kv_heads=heads, n_q_heads=heads, bits=4)
    st = Setup(wl)
    x = torch.from_numpy(np.asarray(st.k(0, 256)).view(np.float16)).cuda().repeat(T // 256, 1)
    y = x.clone()
    y[:, 7] = float("inf") if what == "infinite" else float("nan")
    gc = K.KvqCache(4, heads, heads, T, 20, wl.rope_base, 1 << 20)
    K.kvq_lut_load(gc, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi)
    timer = K.binding.HipEventTimer()
    a, b = _append_ms(gc, y, timer), _append_ms(gc, x, timer)
    assert a < 1.5 * b, (a, b)


def test_codes_that_are_searched_for_cost_little():
    """Signposts past 1, whose codes thresholds do not give: four instructions a signpost and element more.  A factor of 4.8 when the bulk
    kernel's lanes searched for their codes one after the other."""
    import torch
    import paper_2401_18079_amd as K
    heads, T = 32, 4096
    wl = S.workload("c2", n_kv_heads=heads, n_q_heads=heads, bits=3)
    st = Setup(wl)
    x = torch.from_numpy(np.asarray(st.k(0, 256)).view(np.float16)).cuda().repeat(T // 256, 1)
    timer, ms = K.binding.HipEventTimer(), []
    for scale in (1.5, 1.0):
        gc = K.KvqCache(3, heads, heads, T, 20, wl.rope_base, 1 << 20)
        K.kvq_lut_load(gc, st.lut_k * np.float32(scale), st.lut_v * np.float32(scale), st.s, st.z, st.lo, st.hi)
        ms.append(_append_ms(gc, x, timer))
    assert ms[0] < 2.5 * ms[1], ms


@pytest.mark.parametrize("heads,bits,T", [(32, 3, 64), (32, 4, 200), (32, 2, 64), (16, 4, 1000), (40, 4, 64), (8, 3, 4096)])
def test_searched_codes_match_the_oracle(heads, bits, T):
    """The kernels that such tables take, Keys and Values, at either side of their rule."""
    import torch
    import paper_2401_18079_amd as K
    wl = S.workload("c2", n_kv_heads=heads, n_q_heads=heads, bits=bits)
    st = Setup(wl)
    cap = (T + 127) // 128 * 128
    k, v = st.k(0, T), st.v(0, T)
    lut_k, lut_v = st.lut_k * np.float32(1.5), st.lut_v * np.float32(1.5)
    nnz = max(1024, st.cap_nnz_k(cap))
    oc = O.OracleCache(bits, heads, heads, cap, st.k_side, wl.rope_base, lut_k, lut_v, st.s, st.z, st.lo, st.hi, cap_nnz_k=nnz)
    gc = K.KvqCache(bits, heads, heads, cap, st.k_side, wl.rope_base, nnz)
    K.kvq_lut_load(gc, lut_k, lut_v, st.s, st.z, st.lo, st.hi)
    oc.append_k(k); oc.append_v(v)
    K.kvq_quantize_append_kv(gc, torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda())
    bad = compare_caches(oc, gc)
    assert not bad, bad
