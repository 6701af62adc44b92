"""The dense Value kernel at the edges of its tiles (64 tokens), of its head groups and of its weight scale,
against the oracle.  Outlier-free caches: what is compared is the dense kernel and the reduction alone."""
import numpy as np
import pytest

import kvq_synth as S
from kvq_testlib import Setup, fill_both

pytestmark = pytest.mark.gpu


def _weights(kind, Hq, L, rng):
    p = rng.random((Hq, L)) / L
    if kind == "growing":                 # twenty-odd orders of magnitude, ascending: every wavefront its own scale
        p = 2.0 ** (np.arange(L) * (90.0 / L) - 70.0)[None, :] * rng.uniform(0.5, 1.0, (Hq, L))
    elif kind == "signed":
        p = rng.standard_normal((Hq, L)) * np.exp(3.0 * rng.standard_normal((Hq, L)))
    elif kind == "one":                   # a single weight in the last tile, everything before it zero
        p = np.zeros((Hq, L))
        p[:, L - 1] = rng.random(Hq) + 0.5
    return p.astype(np.float32)


@pytest.mark.parametrize("bits,kv,hq,L,sink,kind", [
    (2, 1, 1, 1, 0, "plain"),             # one token: half a pair
    (3, 2, 2, 63, 0, "plain"),            # a ragged tile
    (4, 2, 4, 64, 0, "growing"),          # exactly one tile
    (2, 2, 8, 65, 1, "plain"),            # a second tile with one token, four heads per KV head
    (3, 1, 8, 1025, 0, "growing"),        # eight, several workgroups per head
    (4, 1, 16, 513, 4, "signed"),         # sixteen heads per KV head
    (2, 1, 8, 2049, 0, "signed"),
    (3, 2, 6, 700, 2, "growing"),         # three heads per KV head
    (4, 1, 6, 300, 0, "one"),             # six
    (3, 4, 4, 8191, 0, "one"),
    (2, 3, 12, 1664, 0, "growing"),       # four, a context of whole tiles
    (4, 5, 5, 4097, 0, "growing"),        # a head count that does not divide the compute units
])
def test_weighted_sums_match_the_oracle(bits, kv, hq, L, sink, kind):
    import torch
    import paper_2401_18079_amd as K
    from oracle import kvq_oracle as O
    wl = S.workload("c2", n_kv_heads=kv, n_q_heads=hq, bits=bits, outlier_fraction=0.0)
    st = Setup(wl)
    cap = (L + 127) // 128 * 128
    oc = O.OracleCache(bits, kv, hq, cap, 0, wl.rope_base, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi,
                       cap_nnz_k=1024, n_sink=sink)
    gc = K.KvqCache(bits, kv, hq, cap, 0, wl.rope_base, 1024, n_sink=sink)
    K.kvq_lut_load(gc, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi)
    fill_both(st, oc, gc, L, [1024])
    rng = np.random.default_rng(L + bits)
    p = _weights(kind, hq, L, rng)
    out = torch.full((hq, 128), 7.0, device="cuda")
    K.kvq_pv_matvec(gc, torch.from_numpy(p).cuda(), out)
    ref = oc.pv(p)
    # every product and every partial sum is rounded to fp32 at most: 2^-24 of the terms' sizes each, the
    # roundings of a chain of a few dozen sums (64 allowed) adding up at worst
    vmax = np.abs(st.v(0, L).astype(np.float64)).max(axis=1)
    bound = 64 * 2.0 ** -24 * 1.25 * (np.abs(p.astype(np.float64)) @ vmax)[:, None] + 1e-300
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= bound), float((err / bound).max())


def _plan(kv, hq, L):
    """Heads per group, workgroups per head group and wavefronts per workgroup, as the launch rule has them."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tiles = (L + 63) // 64
    rg = 1 if hq * tiles <= 16 * cus else 2 if hq * tiles <= 48 * cus else 4 if hq * tiles <= 192 * cus else 8
    while (hq // kv) % rg:
        rg //= 2
    slabs = max(1, min(cus // (hq // rg), (tiles + 7) // 8, 512))
    return rg, slabs, 8 if rg == 8 else 16


@pytest.mark.parametrize("bits,kv,hq,L,sink,group", [
    (2, 1, 63, 20011, 0, 1), (3, 1, 63, 20011, 2, 1), (4, 3, 63, 20032, 0, 1),
    (2, 1, 62, 9001, 0, 2), (3, 1, 62, 9001, 1, 2), (4, 1, 62, 8960, 0, 2),
    (2, 1, 60, 20011, 1, 4), (3, 1, 60, 20011, 0, 4), (4, 5, 60, 20001, 4, 4),
    (2, 1, 64, 49999, 0, 8), (3, 2, 64, 49999, 4, 8), (4, 1, 64, 49984, 0, 8),
])
def test_scales_lowered_between_the_tiles_of_a_wavefront(bits, kv, hq, L, sink, group):
    """A wavefront takes every WAVES-th tile of its workgroup.  Weights that grow by 2^7 and more from one of them to
    the next, by another factor for each head, lower the scale of sums that are not zero and still count for 2^-7 of
    the result: a factor on the wrong head or row is far outside the bound."""
    import torch
    import paper_2401_18079_amd as K
    from oracle import kvq_oracle as O
    rg, slabs, waves = _plan(kv, hq, L)
    tiles = (L + 63) // 64
    assert rg == group and tiles // slabs > waves, "several tiles per wavefront"
    wl = S.workload("c2", n_kv_heads=kv, n_q_heads=hq, bits=bits, outlier_fraction=0.0)
    st = Setup(wl)
    cap = (L + 127) // 128 * 128
    oc = O.OracleCache(bits, kv, hq, cap, 0, wl.rope_base, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi,
                       cap_nnz_k=1024, n_sink=sink)
    gc = K.KvqCache(bits, kv, hq, cap, 0, wl.rope_base, 1024, n_sink=sink)
    K.kvq_lut_load(gc, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi)
    fill_both(st, oc, gc, L, [4096])
    rng = np.random.default_rng(L + bits)
    tile = np.arange(L) // 64
    first = np.array([s * tiles // slabs for s in range(slabs)])
    step = (tile - first[np.searchsorted(first, tile, side="right") - 1]) // waves     # which of its tiles a wavefront has
    growth = 7.0 + (5 * np.arange(hq) % 9) / 2.0
    growth[::7] = 0.0                         # and heads whose scale stays
    p = (2.0 ** (growth[:, None] * (step - step.max())[None, :]) * rng.uniform(0.5, 1.0, (hq, L))).astype(np.float32)
    out = torch.full((hq, 128), 7.0, device="cuda")
    K.kvq_pv_matvec(gc, torch.from_numpy(p).cuda(), out)
    ref = oc.pv(p)
    # roundings as above: the sums of a wavefront, of the wavefronts and of the workgroups, 64 allowed
    vmax = np.concatenate([np.abs(st.v(t, min(4096, L - t)).astype(np.float64)).max(axis=1) for t in range(0, L, 4096)])
    bound = 64 * 2.0 ** -24 * 1.25 * (np.abs(p.astype(np.float64)) @ vmax)[:, None] + 1e-300
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref)
    worst = float((err / bound).max())
    assert worst <= 1.0
