"""Range of the sparse Value sums: channels that hold a large residual in every token, with equal scores over a long
context (every token then weighs as much as the largest), whatever number of tokens a workgroup sums.

The append stores such a Value as signpost + fp16 residual, good to half a unit in the residual's last place: 2^-11 of
it.  The sums of equal terms add less than that again (fp32, a few dozen roundings)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _cache(bits, kv, hq, L, value, blocked=False):
    """L tokens with `value` in channel 3 of every second head, -value / 2 in channel 100, and small values elsewhere."""
    import torch
    import paper_2401_18079_amd as K
    D, lut = kv * 128, np.linspace(-1.0, 1.0, 1 << bits).astype(np.float32)
    c = K.KvqCache(bits, kv, hq, (L + 127) // 128 * 128, (kv + 1) // 2, 10000.0, 1024, (kv + 1) * L + 4096,
                   nnz_block_entries=1 << 16 if blocked else None)
    one = np.ones(D, np.float16)
    K.kvq_lut_load(c, lut, lut, one, 0 * one, np.full(D, -65504, np.float16), np.full(D, 65504, np.float16))
    x = torch.randn((4096, D), generator=torch.Generator("cuda").manual_seed(5), device="cuda").half()
    x[:, 3::256], x[:, 100::256] = value, -value / 2
    for t in range(0, L, 4096):
        K.kvq_quantize_append_kv(c, torch.zeros_like(x[:L - t]), x[:L - t])
    assert c.status() == 0
    return c


def _close(out, kv, value):
    out = out.reshape(kv, -1, 128)[::2]
    assert np.max(np.abs(out[..., 3] / value - 1.0)) <= 2.0 ** -10
    assert np.max(np.abs(out[..., 100] / (-value / 2) - 1.0)) <= 2.0 ** -10


CASES = [
    (3, 8, 8, 65536, 20000.0, False),       # (within 2^23 over a workgroup of a launch of its own for the sparse sums)
    (2, 4, 16, 65536, 20000.0, False),
    (4, 1, 8, 100001, 20000.0, False),
    (4, 2, 2, 300000, 6500.0, True),
    (3, 32, 32, 131072, 25000.0, False),
]


@pytest.mark.parametrize("bits,kv,hq,L,value,blocked", CASES + [
    (4, 1, 1, 2048, 65000.0, False),        # almost the largest fp16 number, from the shortest shared launch ...
    (3, 1, 1, 400000, 65000.0, False),
    (3, 40, 40, 150001, 65000.0, False),    # ... to contexts with a launch of their own for the sparse sums
    (2, 8, 64, 262144, 65000.0, True),
])
def test_attention_holds_any_fp16_residual(bits, kv, hq, L, value, blocked):
    import torch
    import paper_2401_18079_amd as K
    c = _cache(bits, kv, hq, L, value, blocked)
    scores, out = torch.zeros((hq, c.c.cap_tokens), device="cuda"), torch.zeros((hq, 128), device="cuda")
    K.kvq_attention_decode(c, torch.zeros((hq, 128), device="cuda"), 1.0, scores, out)
    _close(out.cpu().numpy().astype(np.float64), kv, value)


@pytest.mark.parametrize("bits,kv,hq,L,value,blocked", CASES)
def test_weights_of_one(bits, kv, hq, L, value, blocked):
    """A caller's weights: a shared launch holds what the sparse sums hold in a launch of their own."""
    import torch
    import paper_2401_18079_amd as K
    c = _cache(bits, kv, hq, L, value, blocked)
    out = torch.zeros((hq, 128), device="cuda")
    K.kvq_pv_matvec(c, torch.ones((hq, L), device="cuda"), out)
    _close(out.cpu().numpy().astype(np.float64) / L, kv, value)
