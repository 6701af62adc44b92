"""Codes of the appends where counting thresholds could part from the exhaustive search over the signposts: values
on and next to the decision points, far outliers, signpost tables that are not monotone to count on.  Bit-exact
against the oracle, Keys and Values, every routine that the call size selects."""
import numpy as np
import pytest

import kvq_synth as S
from kvq_testlib import Setup, compare_caches
from oracle import kvq_oracle as O

pytestmark = pytest.mark.gpu


def _table(kind, bits, rng):
    n = 1 << bits
    t = np.sort(rng.uniform(-1, 1, n))
    t[0], t[-1] = -1.0, 1.0
    if kind == "equal":                    # codes that are never chosen
        t[n // 2] = t[n // 2 - 1]
        t[-2] = 1.0
    elif kind == "close":                  # nearer to each other than the counting allows
        t = np.concatenate([np.arange(n - 2) * 2.0 ** -20, [0.5, 1.0]])
    elif kind == "wide":                   # signposts beyond [-1, 1]
        t = t * 300.0
    elif kind == "gap":                    # the smallest difference that is counted
        t[1] = -1.0 + 2.0 ** -10
    return np.sort(t).astype(np.float32)


def _rows(T, D, s, z, lut, rng):
    """fp16 rows around s * x + z for x on the midpoints of neighbouring signposts, on signposts, and far outside."""
    lut = O.store_lut(lut)
    mid = (lut[1:] + lut[:-1]) / 2
    x = rng.choice(np.concatenate([mid, mid, lut, [130.0, -127.0, 4000.0, -3e4]]), size=(T, D))
    x = s.astype(np.float64) * x + z
    x = np.clip(x, -6e4, 6e4).astype(np.float16)
    step = rng.integers(-1, 2, size=(T, D)).astype(np.int16)            # the fp16 neighbours on either side too
    return (x.view(np.int16) + np.where(np.abs(x) > 1e-3, step, 0)).astype(np.int16).view(np.float16)


@pytest.mark.parametrize("heads,T", [(2, 1), (3, 70), (16, 1), (32, 65), (8, 1030), (40, 3), (40, 520), (65, 2), (5, 2048)])
@pytest.mark.parametrize("bits,kind", [(2, "equal"), (3, "plain"), (3, "close"), (4, "gap"), (4, "wide"), (4, "equal")])
def test_codes_at_the_decision_points(heads, T, bits, kind):
    import torch
    import paper_2401_18079_amd as K
    rng = np.random.default_rng(bits * 1000 + heads * 7 + T)
    wl = S.workload("c2", n_kv_heads=heads, n_q_heads=heads, bits=bits)
    st = Setup(wl)
    D, cap = wl.D, (T + 127) // 128 * 128
    lut_k, lut_v = _table(kind, bits, rng), _table(kind, bits, rng)
    s = np.exp2(rng.integers(-3, 2, D)).astype(np.float16)
    z = rng.integers(-2, 3, D).astype(np.float16)
    lo, hi = (z - 4 * s).astype(np.float16), (z + 4 * s).astype(np.float16)
    oc = O.OracleCache(bits, heads, heads, cap, st.k_side, wl.rope_base, lut_k, lut_v, s, z, lo, hi, cap_nnz_k=T * D)
    gc = K.KvqCache(bits, heads, heads, cap, st.k_side, wl.rope_base, T * D)
    K.kvq_lut_load(gc, lut_k, lut_v, s, z, lo, hi)
    k, v = _rows(T, D, s, z, lut_k, rng), _rows(T, D, np.ones(1), np.zeros(1), lut_v, rng)
    oc.append_k(k); oc.append_v(v)
    K.kvq_quantize_append_kv(gc, torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda())
    assert not compare_caches(oc, gc)
