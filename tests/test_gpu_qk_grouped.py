"""The grouped Key kernel at the edges of its tiles, head groupings and table forms: every score against the oracle."""
import numpy as np
import pytest

import kvq_synth as S
from kvq_testlib import Setup, fill_both

pytestmark = pytest.mark.gpu


def _grouping(kv, r, L):
    """KV heads per workgroup and tokens per tile, as the launch rule has them: the largest grouping with workgroups
    for five eighths of the compute units."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count

    def workgroups(kvh, nt):
        groups = kv // kvh
        return min(max(cus // groups, 1), 256, (L + nt - 1) // nt) * groups
    most = 2 if r == 8 else 4
    if kv % most == 0 and workgroups(most, 1024) >= cus * 5 // 8:
        return most, 1024
    if most == 4 and kv % 2 == 0 and workgroups(2, 512) >= cus * 5 // 8:
        return 2, 512
    return 1, 512


@pytest.mark.parametrize("bits,kv,r,L,kvh,nt", [
    (3, 4, 2, 63, 1, 512), (4, 2, 2, 513, 1, 512),      # a ragged wavefront / one token of a second tile
    (2, 1, 4, 1, 1, 512), (3, 3, 4, 511, 1, 512), (4, 5, 4, 1024, 1, 512), (2, 4, 4, 40000, 1, 512),
    (2, 8, 8, 129, 1, 512), (3, 1, 8, 640, 1, 512), (4, 2, 8, 1537, 1, 512),
    (4, 8, 4, 20500, 2, 512), (2, 4, 4, 40500, 2, 512), (3, 4, 4, 41000, 2, 512), (3, 4, 2, 41001, 2, 512),
    (4, 8, 2, 20481, 2, 512),
    (2, 8, 4, 82000, 4, 1024), (3, 4, 4, 164000, 4, 1024), (3, 4, 2, 165000, 4, 1024), (4, 4, 2, 164001, 4, 1024),
    (4, 2, 8, 165000, 2, 1024),
])
def test_every_score_matches_the_oracle(bits, kv, r, L, kvh, nt):
    import torch
    import paper_2401_18079_amd as K
    assert _grouping(kv, r, L) == (kvh, nt)
    wl = S.workload("c4", n_kv_heads=kv, n_q_heads=kv * r, bits=bits, context=L)
    st = Setup(wl)
    cap = (L + 127) // 128 * 128
    if L <= 2000:
        st_lo = 0
    else:
        st_lo = L - 1500                     # the oracle takes a window at the start and one at the end
    gc = st.gpu_cache(cap)
    from kvq_synth.device import DeviceGen
    dg = DeviceGen(wl, 0, st.kprof, st.vprof)
    for t in range(0, L, 4096):
        K.kvq_quantize_append_k(gc, dg.k(t, min(4096, L - t)))
    q = S.gen_q(wl, 0, 0)
    scores = torch.full((kv * r, cap), 7.0, device="cuda")
    K.kvq_qk_matvec(gc, torch.from_numpy(q).cuda(), 0.0883, scores)
    got = scores.cpu().numpy()
    assert np.all(got[:, L:] == 7.0)
    assert not np.any(got[:, :L] == 7.0)
    # the oracle's cache holds the window alone, at positions from 0: the query is rotated back by the window's start
    # instead (<q, R_{t0+n} k> = <R_{t0}^T q, R_n k>)
    from oracle import kvq_oracle as O
    for t0 in {0, st_lo}:
        T = min(1500, L - t0)
        oc = O.OracleCache(bits, kv, kv, 1536, st.k_side, wl.rope_base, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi,
                           cap_nnz_k=st.cap_nnz_k(1536))
        oc.append_k(st.k(t0, T))
        theta = wl.rope_base ** (-np.arange(64) / 64.0)
        a, b = q[:, :64].astype(np.float64), q[:, 64:].astype(np.float64)
        c, s = np.cos(t0 * theta), np.sin(t0 * theta)
        back = np.concatenate([a * c + b * s, b * c - a * s], axis=1)        # R_{t0}^T q
        ref = np.zeros((kv * r, T))
        for j in range(r):
            ref[j::r] = oc.qk(back[j::r].astype(np.float32), 0.0883)
        err = np.abs(got[:, t0:t0 + T] - ref)
        # 128 products and sums in fp32, sines and cosines good to 1e-6, and the oracle's query rounded to fp32
        bound = 2e-5 * np.sqrt(np.mean(ref ** 2, axis=1, keepdims=True)) + 2e-5 * np.abs(ref)
        assert np.all(err <= bound), (t0, float((err / bound).max()))
    # the scores between: the same cache with one query head per KV head, by the kernel for that (both within the
    # bound of the oracle)
    gc.c.n_q_heads = kv
    for j in range(r):
        one = torch.zeros((kv, cap), device="cuda")
        K.kvq_qk_matvec(gc, torch.from_numpy(np.ascontiguousarray(q[j::r])).cuda(), 0.0883, one)
        ref = one.cpu().numpy()[:, :L].astype(np.float64)
        err = np.abs(got[j::r, :L] - ref)
        bound = 4e-5 * np.sqrt(np.mean(ref ** 2, axis=1, keepdims=True)) + 4e-5 * np.abs(ref)
        assert np.all(err <= bound), (j, float((err / bound).max()))
