"""Value appends of one to four heads, a wavefront per token: every width, the call lengths at either side of the rule, outlier counts
from none to almost half of the channels, rows full of ties.  Bit-exact against the oracle."""
import numpy as np
import pytest

import kvq_synth as S
from oracle import kvq_oracle as O
from kvq_testlib import Setup, compare_caches, tie_vectors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,bits,T,n0,k", [
    (1, 2, 1, 1, 0), (1, 3, 70, 0, 1), (1, 4, 260, 3, 63), (2, 3, 1, 0, 2), (2, 4, 65, 1, 30), (2, 2, 257, 0, 127), (3, 4, 1, 1, 3),
    (3, 2, 66, 0, 64), (3, 3, 300, 1, 65), (4, 3, 2048, 1, 3), (4, 2, 2047, 0, 3), (4, 4, 2049, 0, 255), (4, 3, 1, 0, 100),
])
@pytest.mark.parametrize("together", [False, True])
def test_narrow_values_match_the_oracle(heads, bits, T, n0, k, together):
    import torch
    import paper_2401_18079_amd as K
    wl = S.workload("c2", n_kv_heads=heads, n_q_heads=heads, bits=bits)
    st = Setup(wl)
    D, cap = wl.D, (n0 + T + 127) // 128 * 128
    rng = np.random.default_rng(heads * 100 + T + k)
    v = (rng.standard_normal((n0 + T, D)) * np.exp(0.5 * rng.standard_normal((n0 + T, 1)))).astype(np.float16)
    v[::3] = rng.choice(np.float16([-2.0, -0.5, 0.25, 0.5, 3.0]), v[::3].shape)
    if 1 <= k <= D // 8:
        ties = tie_vectors(D, k, rng)
        v[1::3] = ties[rng.integers(0, len(ties), len(v[1::3]))]
    keys = st.k(0, n0 + T)
    nnz = max(1024, st.cap_nnz_k(cap), 2 * k * cap)
    oc = O.OracleCache(bits, heads, heads, cap, k, wl.rope_base, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi, cap_nnz_k=nnz)
    gc = K.KvqCache(bits, heads, heads, cap, k, wl.rope_base, nnz)
    K.kvq_lut_load(gc, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi)
    for a, b in ((0, n0), (n0, n0 + T)):
        if a == b:
            continue
        oc.append_k(keys[a:b]); oc.append_v(v[a:b])
        kd, vd = torch.from_numpy(keys[a:b]).cuda(), torch.from_numpy(v[a:b]).cuda()
        if together:
            K.kvq_quantize_append_kv(gc, kd, vd)
        else:
            K.kvq_quantize_append_k(gc, kd); K.kvq_quantize_append_v(gc, vd)
    bad = compare_caches(oc, gc)
    assert not bad, bad
