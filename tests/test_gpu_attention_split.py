"""Attention workgroups that split keys (forward, dQ) and queries (dK/dV) over more wavefronts."""
import pytest

from tests import test_gpu_kernels as K

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel_set", [5, 6, 7])
@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("b,s,h,hkv,hd", K.ATT_SHAPES + [(1, 33, 2, 2, 128), (2, 64, 1, 1, 64), (1, 65, 2, 1, 128), (1, 129, 3, 3, 64), (1, 257, 2, 2, 128)])
def test_four_key_parts_and_two_query_parts(kernel_set, causal, b, s, h, hkv, hd):
    """kernel_set 5 forces the shape, 7 both passes of its backward in one launch, 6 those of the shape with half as many parts: one row, one past a 32-key part, past a 64-row tile, past a 128-key step and past two steps,
    so that parts without a key and query blocks without a row occur; oracle and tolerances of the other shapes."""
    K.test_attention("bf16", kernel_set, causal, b, s, h, hkv, hd)


@pytest.mark.parametrize("causal,b,s,h,hkv,hd", [(0, 1, 320, 26, 26, 128), (0, 1, 321, 22, 22, 128), (1, 1, 1000, 2, 2, 128), (1, 2, 1000, 2, 1, 64),
                                                 (1, 2, 321, 26, 26, 64), (1, 2, 320, 52, 26, 64), (1, 1, 2049, 1, 1, 64), (0, 1, 2048, 5, 5, 64)])
def test_the_rule_at_its_lines(causal, b, s, h, hkv, hd):
    """Where the rule changes shape: the backward in one launch up to 256, 512 and 960 workgroups, dK/dV above 320 positions, the forward
    from 1000, dQ from 2048."""
    K.test_attention("bf16", 0, causal, b, s, h, hkv, hd)


@pytest.mark.parametrize("kernel_set", [5, 6, 7])
@pytest.mark.parametrize("b,s,h,hkv,hd", [(1, 392, 8, 1, 128), (2, 300, 12, 2, 64)])
def test_two_query_parts_with_split_query_heads(kernel_set, b, s, h, hkv, hd):
    K.test_attention_bwd_with_split_query_heads(kernel_set, 1, b, s, h, hkv, hd)
