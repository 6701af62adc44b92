"""The sparse and dense Value kernels as one launch, at the edges of its rule and of its plan, against the oracle and
with either storage of the outliers."""
import numpy as np
import pytest

import kvq_synth as S
from kvq_testlib import Setup, fill_both, matvec_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,kv,hq,L,sink,p,full", [
    (3, 1, 1, 2048, 0, 0.01, False),        # the shortest context that takes it
    (2, 8, 8, 2049, 0, 0.01, False),        # a last tile and a last run with one token
    (4, 2, 4, 4095, 3, 0.01, False),        # sink tokens, two heads per group at most
    (3, 1, 8, 9001, 0, 0.01, False),        # eight heads on one
    (4, 1, 6, 2500, 1, 0.01, False),        # a ratio that is not a power of two
    (2, 8, 64, 2100, 0, 0.01, False),       # 64 query heads
    (3, 5, 40, 2777, 0, 0.02, False),       # a head count that leaves compute units over
    (4, 2, 2, 3000, 0, 0.0, False),         # no outliers
    (3, 2, 4, 3000, 0, 0.02, True),         # outlier arrays that run full: tokens with fewer outliers, then none
])
def test_one_launch_against_the_oracle(bits, kv, hq, L, sink, p, full):
    import torch
    import paper_2401_18079_amd as K
    from oracle import kvq_oracle as O
    wl = S.workload("c2", n_kv_heads=kv, n_q_heads=hq, bits=bits, outlier_fraction=p)
    st = Setup(wl)
    cap = (L + 1 + 127) // 128 * 128
    k_side = st.k_side if p else 0
    nnz = st.cap_nnz_k(cap)
    nnz_v = max(1024, 2 * k_side * L)
    if full:
        nnz_v = nnz_v // 2 // 1024 * 1024                                # half the tokens, the last of them in part
    oc = O.OracleCache(bits, kv, hq, cap, k_side, wl.rope_base, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi,
                       cap_nnz_k=nnz, n_sink=sink)
    gc, bc = (K.KvqCache(bits, kv, hq, cap, k_side, wl.rope_base, nnz, nnz_v, n_sink=sink, nnz_block_entries=be)
              for be in (None, 1024))
    for c in (gc, bc):
        K.kvq_lut_load(c, st.lut_k, st.lut_v, st.s, st.z, st.lo, st.hi)
        fill_both(st, oc if c is gc else None, c, L, [1024])
    assert (gc.status() != 0) == full and (bc.status() != 0) == full
    if full:                                                             # (the oracle's have room for all: hand it these)
        oc.v_ptr[:L + 1] = gc.v_ptr.cpu().numpy().view(np.uint32)[:L + 1]
    w = np.random.default_rng(L + bits).random((hq, L)).astype(np.float32) / L
    q = torch.from_numpy(S.gen_q(wl, 0, 0)).cuda()
    scale = 1.0 / np.sqrt(128.0)
    scores = torch.zeros((hq, cap), device="cuda")
    outs = []
    for c in (gc, bc):
        out, attended = (torch.full((hq, 128), 7.0, device="cuda") for _ in range(2))
        K.kvq_pv_matvec(c, torch.from_numpy(w).cuda(), out)
        ok, worst = matvec_close(out.cpu().numpy(), oc.pv(w), rel=1e-4)
        assert ok, f"worst error / bound = {worst:.3f}"
        if hq // kv in (1, 2, 4, 8):                                     # (the ratios that the Key half takes)
            K.kvq_attention_decode(c, q, scale, scores, attended)
            # (twice the mat-vec tolerance: a score error delta multiplies a weight by e^delta)
            ok, worst = matvec_close(attended.cpu().numpy(), oc.pv(O.softmax(scores[:, :L].cpu().numpy())), rel=2e-3)
            assert ok, f"attention: worst error / bound = {worst:.3f}"
        outs.append(out)
    assert torch.equal(*outs)                                            # the same terms in the same order


@pytest.mark.parametrize("bits,kv,hq,L,sink,p", [
    (2, 1, 2, 55001, 0, 0.02),          # several sub-ranges a wavefront, in units of eight tokens
    (4, 8, 64, 4401, 2, 0.01),          # two heads per group
    (3, 8, 32, 26003, 0, 0.01),         # likewise, units of eight
    (3, 8, 64, 12345, 1, 0.01),         # four heads per group
    (2, 4, 32, 99003, 0, 0.01),         # eight: workgroups of eight wavefronts, units of sixteen
    (4, 8, 64, 50007, 0, 0.005),
])
def test_longer_runs_and_groups_of_heads(bits, kv, hq, L, sink, p):
    """Plans in which a wavefront walks through several sub-ranges, and those of every head group."""
    test_one_launch_against_the_oracle(bits, kv, hq, L, sink, p, False)


@pytest.mark.parametrize("bits,kv,hq,k_side,longest", [
    (3, 32, 32, 20, 160000), (4, 40, 40, 26, 120000), (2, 16, 32, 10, 400000), (3, 8, 64, 5, 300000), (2, 4, 32, 3, 400000),
    (4, 1, 8, 1, 600000),
])
def test_one_context_ends_the_one_launch(bits, kv, hq, k_side, longest):
    """A decoder does not fall back and forth between the two forms as its context grows."""
    import paper_2401_18079_amd as K
    c = K.KvqCache(bits, kv, hq, 256, k_side, 10000.0, 1024, 1024)
    D, lut = kv * 128, np.linspace(-1, 1, 1 << bits, dtype=np.float32)
    K.kvq_lut_load(c, lut, lut, *[np.full(D, v, np.float16) for v in (1, 0, -1, 1)])
    c.c.cap_tokens = (longest // 128 + 2) * 128        # (host arithmetic only: the arrays are not touched)
    at = sorted({n for m in np.geomspace(2047, longest, 300).astype(int) for n in (m - m % 8 - 1, m - m % 8, m)
                 if 2047 <= n <= longest} | {131071, 131072} & set(range(longest)))
    seen = []
    for n in at:
        c.c.n_tokens_k = c.c.n_tokens_v = int(n)
        seen.append(K.kvq_decode_step_launches(c))
    c.c.n_tokens_k = c.c.n_tokens_v = 2000
    assert seen[0] == K.kvq_decode_step_launches(c) - 1
    assert sum(a != b for a, b in zip(seen, seen[1:])) <= 1, [n for n, a, b in zip(at[1:], seen, seen[1:]) if a != b]


def test_contexts_on_either_side_of_the_rule():
    import paper_2401_18079_amd as K
    cache = lambda kv, hq, cap, **kw: K.KvqCache(2, kv, hq, cap, 1, 10000.0, 4096, **kw)

    def launches(c, n):
        c.c.n_tokens_k = c.c.n_tokens_v = n
        return K.kvq_decode_step_launches(c)

    c = cache(1, 1, 600064)
    K.kvq_lut_load(c, *[np.linspace(-1, 1, 4, dtype=np.float32)] * 2, *[np.full(128, v, np.float16) for v in (1, 0, -1, 1)])
    assert [launches(c, n) for n in (0, 2046, 2047, 600000)] == [6, 6, 5, 5]
    c = cache(32, 32, 1 << 16)               # more sparse work than the launch saves
    K.kvq_lut_load(c, *[np.linspace(-1, 1, 4, dtype=np.float32)] * 2, *[np.full(4096, v, np.float16) for v in (1, 0, -1, 1)])
    c.c.k_side_v = 20
    assert [launches(c, n) for n in (2046, 2047, 60000)] == [6, 5, 5]
    c.c.k_side_v = 2000
    assert launches(c, 60000) == 6
    c = cache(1, 1, 4096, nnz_block_entries=1024)
    K.kvq_lut_load(c, *[np.linspace(-1, 1, 4, dtype=np.float32)] * 2, *[np.full(128, v, np.float16) for v in (1, 0, -1, 1)])
    assert launches(c, 3000) == 5
