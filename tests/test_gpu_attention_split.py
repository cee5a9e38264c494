"""Attention workgroups that split keys (forward, dQ) and queries (dK/dV) over more wavefronts."""
import re

import pytest

from tests import test_gpu_kernels as K
from tests.gpu_util import launches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel_set", [5, 6, 7])
@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("b,s,h,hkv,hd", K.ATT_SHAPES + [(1, 33, 2, 2, 128), (2, 64, 1, 1, 64), (1, 65, 2, 1, 128), (1, 129, 3, 3, 64), (1, 257, 2, 2, 128)])
def test_four_key_parts_and_two_query_parts(kernel_set, causal, b, s, h, hkv, hd):
    """kernel_set 5 forces the shape, 7 both passes of its backward in one launch, 6 those of the shape with half as many parts: one row, one past a 32-key part, past a 64-row tile, past a 128-key step and past two steps,
    so that parts without a key and query blocks without a row occur; oracle and tolerances of the other shapes."""
    K.test_attention("bf16", kernel_set, causal, b, s, h, hkv, hd)


ONE4, ONE2 = "bwd 4 2", "bwd 2 1"                     # one launch, two wavefronts per SIMD and workgroup or one
ONE_PAIR, TWO_PAIRS = "dq 256 2, dkv 64 1", "dq 256 2, dkv 64 2"
# (causal, b, s, h, hkv, hd, scratch): what the backward launches.  64-row tiles x (h + hkv x splits) is the count that the lines are drawn by.
BACKWARD = [
    ((0, 1, 320, 25, 25, 128, 0), ONE4), ((0, 1, 320, 26, 26, 128, 0), ONE_PAIR), ((0, 1, 321, 21, 21, 128, 0), ONE4), ((0, 1, 321, 22, 22, 128, 0), TWO_PAIRS),
    ((1, 1, 320, 25, 25, 128, 0), ONE4), ((1, 1, 320, 26, 26, 128, 0), ONE2), ((1, 1, 320, 51, 51, 128, 0), ONE2), ((1, 1, 320, 52, 52, 128, 0), ONE_PAIR),
    ((1, 2, 65, 33, 33, 128, 0), ONE2), ((1, 1, 321, 22, 22, 128, 0), ONE4), ((1, 1, 321, 42, 42, 128, 0), ONE4), ((1, 1, 321, 43, 43, 128, 0), ONE_PAIR),
    ((0, 1, 2048, 8, 8, 128, 0), TWO_PAIRS), ((1, 1, 2048, 8, 8, 128, 0), ONE4),
    ((1, 2, 300, 32, 8, 128, 0), ONE4), ((1, 3, 81, 40, 20, 128, 0), ONE4), ((1, 3, 81, 40, 20, 128, 1), ONE2 + ", reduce"),      # long chains of query heads, and split
    ((0, 1, 321, 21, 21, 64, 0), ONE4), ((0, 1, 321, 22, 22, 64, 0), ONE2), ((1, 1, 321, 42, 42, 64, 0), ONE4), ((1, 1, 321, 43, 43, 64, 0), ONE2),
    ((1, 1, 320, 25, 25, 64, 0), ONE4), ((1, 1, 320, 26, 26, 64, 0), ONE2),
    ((0, 1, 128, 192, 192, 64, 0), ONE2), ((0, 1, 128, 193, 193, 64, 0), ONE_PAIR), ((0, 1, 129, 160, 160, 64, 0), ONE2), ((0, 1, 129, 161, 161, 64, 0), ONE_PAIR),
    ((0, 1, 385, 68, 68, 64, 0), ONE2), ((0, 1, 385, 69, 69, 64, 0), TWO_PAIRS),
    ((0, 1, 512, 32, 8, 64, 0), TWO_PAIRS), ((0, 1, 512, 32, 8, 64, 1), ONE2 + ", reduce"), ((1, 1, 300, 64, 16, 64, 0), ONE_PAIR),
]
FORWARD = [((1, 1, 999, 2, 2, 128), "256 2"), ((1, 1, 1000, 2, 2, 128), "512 4"), ((1, 2, 1000, 8, 1, 128), "512 4"), ((1, 2, 1000, 9, 1, 128), "256 2"),
           ((1, 2, 1000, 16, 1, 64), "512 4"), ((1, 2, 1000, 17, 1, 64), "256 2")]


def _names(kernels):
    out = []
    for name, _, _ in kernels:
        m = re.search(r"attn_(fwd|dq|dkv|bwd|dkv_reduce)_kernel(?:ILi\d+E(?:Li(\d+)E)(?:Li(\d+)E))?", name)
        out.append("reduce" if m[1] == "dkv_reduce" else f"{m[1]} {m[2]} {m[3]}")
    return ", ".join(out)


@pytest.mark.parametrize("shape,expect", BACKWARD)
def test_backward_launches_at_the_lines(shape, expect):
    """The kernels themselves, on both sides of every line of the rule (a capture: nothing runs, so the buffers are only names)."""
    import torch
    causal, b, s, h, hkv, hd, scratch = shape
    t = torch.zeros(256, dtype=torch.uint8, device="cuda:0")
    need = K.L().stage_kernel_attention_bwd_scratch_bytes(b, s, h, hkv, hd)
    assert not scratch or need > 0
    got = launches(lambda stream: K.L().stage_kernel_attention_bwd_ws(1, b, s, h, hkv, hd, causal, *([K.P(t)] * 7 if scratch else [K.P(t)] * 6 + [None]),
                                                                      need if scratch else 0, 0, stream))
    assert _names(got) == expect


@pytest.mark.parametrize("shape,expect", FORWARD)
def test_forward_launches_at_the_lines(shape, expect):
    import torch
    causal, b, s, h, hkv, hd = shape
    t = torch.zeros(256, dtype=torch.uint8, device="cuda:0")
    got = launches(lambda stream: K.L().stage_kernel_attention_fwd(1, b, s, h, hkv, hd, causal, K.P(t), K.P(t), K.P(t), 0, stream))
    assert _names(got) == "fwd " + expect


@pytest.mark.parametrize("causal,b,s,h,hkv,hd", [x[:6] for x, _ in BACKWARD if not x[6]] + [(1, 1, 1000, 2, 2, 128), (1, 2, 1000, 2, 1, 64), (0, 1, 2048, 5, 5, 64)])
def test_the_rule_at_its_lines(causal, b, s, h, hkv, hd):
    """Both directions against the oracle on either side of every line of the rule, and where the forward takes four key parts."""
    K.test_attention("bf16", 0, causal, b, s, h, hkv, hd)


@pytest.mark.parametrize("kernel_set", [5, 6, 7])
@pytest.mark.parametrize("b,s,h,hkv,hd", [(1, 392, 8, 1, 128), (2, 300, 12, 2, 64)])
def test_two_query_parts_with_split_query_heads(kernel_set, b, s, h, hkv, hd):
    K.test_attention_bwd_with_split_query_heads(kernel_set, 1, b, s, h, hkv, hd)


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("part", ["q", "k", "v", "do"])
@pytest.mark.parametrize("s,hd,causal,at", [(37, 128, 1, 20), (37, 64, 0, 36), (150, 128, 1, 0), (150, 64, 1, 141), (300, 64, 1, 130), (300, 128, 0, 299)])
def test_infinities_and_nan_spread_as_with_two_parts(part, value, s, hd, causal, at):
    """An infinity or NaN of one position makes the same elements non-finite, in the same way, whatever the number of key and query parts and
    whether the backward is one launch, and leaves the others as they were."""
    import torch
    h, hkv = 2, 1
    g = torch.Generator().manual_seed(36)
    qkv, do = torch.randn((s, (h + 2 * hkv) * hd), generator=g), torch.randn((s, h * hd), generator=g)
    if part == "do":
        do[at, hd + 3] = value
    else:
        qkv[at, {"q": hd, "k": h * hd, "v": (h + hkv) * hd}[part] + 5] = value
    qkv, do = qkv.to("cuda:0").bfloat16(), do.to("cuda:0").bfloat16()
    o, dqkv = {}, {}
    for ks in (4, 5, 6, 7):
        o[ks], dqkv[ks] = torch.zeros_like(do), torch.zeros_like(qkv)
        lse, delta = (torch.zeros((h, s), device="cuda:0") for _ in range(2))
        assert K.L().stage_kernel_attention_fwd(1, 1, s, h, hkv, hd, causal, K.P(qkv), K.P(o[ks]), K.P(lse), ks, None) == 0
        assert K.L().stage_kernel_attention_fwd(1, 1, s, h, hkv, hd, causal, K.P(qkv), K.P(o[4]), K.P(lse), 4, None) == 0
        assert K.L().stage_kernel_attention_bwd(1, 1, s, h, hkv, hd, causal, K.P(qkv), K.P(o[4]), K.P(lse), K.P(do), K.P(dqkv[ks]), K.P(delta), ks, None) == 0
    for got in (o, dqkv):
        ref = got[4].float()
        fin = torch.isfinite(ref)
        for ks in (5, 6, 7):
            x = got[ks].float()
            assert torch.equal(torch.isnan(x), torch.isnan(ref)) and torch.equal(x[torch.isinf(ref)], ref[torch.isinf(ref)]) and torch.equal(torch.isfinite(x), fin), ks
            if fin.any():
                assert (x[fin] - ref[fin]).abs().max() <= K.KTOL["bf16"] * ref[fin].abs().max(), ks
