"""Precision of the dense Value kernel against 64 bits where its number formats could cost some: small weights beside
large ones, and the long sums of a million-token context."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
U = 2.0 ** -24                            # half a unit in the last place of fp32, relative


def _cache(bits, kv, hq, cap, lut):
    import paper_2401_18079_amd as K
    gc = K.KvqCache(bits, kv, hq, cap, 0, 10000.0, 1024)
    D = kv * 128
    one, zero = np.ones(D, np.float16), np.zeros(D, np.float16)
    K.kvq_lut_load(gc, lut, lut, one, zero, np.full(D, -65504, np.float16), np.full(D, 65504, np.float16))
    return gc


@pytest.mark.parametrize("bits,kv,hq,L", [
    (2, 1, 1, 640), (3, 2, 4, 640), (4, 1, 8, 640),
    (3, 1, 62, 9024), (4, 1, 60, 20032), (2, 1, 64, 49984),         # two, four and eight heads per wavefront
])
def test_weights_far_below_the_largest_keep_all_their_bits(bits, kv, hq, L):
    """The first token of every tile of 64 has weight 1 and the Value 0 in the channels compared; all others weigh
    2^-20 (1 + 0.99 * 2^-13): if the part below 2^-13 of such a weight is dropped, every sum is 1.2e-4 too small."""
    import torch
    import paper_2401_18079_amd as K
    lut = np.sort(np.concatenate([[-1.0, 0.0, 1.0], np.linspace(0.1, 0.9, (1 << bits) - 3)])).astype(np.float32)
    stored = np.array([K.kvq_stored_signpost(float(x)) for x in lut], np.float32)
    gc = _cache(bits, kv, hq, (L + 127) // 128 * 128, lut)
    rng = np.random.default_rng(bits + hq)
    v = rng.choice(stored[stored > 0], size=(L, kv * 128)).astype(np.float16)
    v[::64] = 0.0
    v[:, 0::128], v[:, 1::128] = 1.0, -1.0                        # every token: scale 1, zero-point 0
    for t in range(0, L, 4096):
        K.kvq_quantize_append_v(gc, torch.from_numpy(v[t:t + 4096]).cuda())
    p = np.full((hq, L), 2.0 ** -20 * (1.0 + 0.99 * 2.0 ** -13))
    p[:, ::64] = 1.0
    p = (p * 2.0 ** (-5.0 * (np.arange(hq) % 8))[:, None]).astype(np.float32)
    out = torch.zeros((hq, 128), device="cuda")
    K.kvq_pv_matvec(gc, torch.from_numpy(p).cuda(), out)
    got = out.cpu().numpy().astype(np.float64)
    for q in range(hq):
        h = q // (hq // kv)
        ref = p[q].astype(np.float64) @ v[:, h * 128:(h + 1) * 128].astype(np.float64)
        # positive terms: the products of a few tiles, their wavefronts' and workgroups' sums, each rounded to fp32 once
        worst = float(np.max(np.abs(got[q, 2:] / ref[2:] - 1.0)))
        assert worst <= 96 * U, q


def test_sums_over_a_million_tokens_are_those_of_short_chains():
    """Random codes and weights.  A sum of m zero-mean terms whose partial sums are all rounded is off by u sqrt(m / 2)
    of its size (u: half a unit in the last place, evenly spread, mantissas evenly spread too: 2^-24 / sqrt(6)).
    Allowed: 32 roundings in a chain of 1024 tokens (one per matrix instruction), 8 chains, 16 wavefronts, 8 workgroups
    and the 32 partial results of the reduction.  One chain over a wavefront's 8192 tokens would have 256."""
    import torch
    import paper_2401_18079_amd as K
    kv, L = 32, 1 << 20
    lut = np.float32([-1.0, -0.375, 0.375, 1.0])
    gc = _cache(2, kv, kv, L, lut)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    gc.v_codes.random_(0, 256, generator=g)
    gc.v_sz.view(-1, 2)[:, 0] = 0x3C00                            # scale 1, zero-point 0
    gc.c.n_tokens_v = L
    p = torch.rand(kv, L, generator=g, device="cuda")
    out = torch.zeros((kv, 128), device="cuda")
    K.kvq_pv_matvec(gc, p, out)
    # field j of the chunk of (head, half, token pair): two tokens' codes, low bits first; 16-byte pieces of 64 pairs
    chunks = gc.v_codes.view(kv, 2, L // 128, 2, 64, 16)
    table = torch.from_numpy(lut).double().cuda()
    err = size = 0.0
    for h in (0, 13, 31):
        for half in (0, 1):
            b = chunks[h, half].permute(0, 2, 1, 3).reshape(L // 2, 32).int()            # [pair][byte]
            f = torch.stack([b & 15, b >> 4], 2).reshape(L // 2, 64)                      # [pair][field]
            ref = torch.zeros(64, dtype=torch.float64, device="cuda")
            for t in (0, 1):
                ref += p[h, t::2].double() @ table[((f >> (2 * t)) & 3).long()]
            err += float(((out[h, 64 * half:64 * half + 64].double() - ref) ** 2).sum())
            size += float((ref ** 2).sum())
    bound = U / np.sqrt(6.0) * np.sqrt((32 + 8 + 16 + 8 + 32) / 2)
    assert np.sqrt(err / size) <= bound, (np.sqrt(err / size), bound)
