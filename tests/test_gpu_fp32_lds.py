"""fp32 products whose 32 x 32 tiles take their operands through LDS."""
import pytest

from tests import test_gpu_fp32 as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("M,N,K", F.SHAPES[:-2] + [(32, 32, 32), (31, 28, 36), (64, 96, 288), (33, 64, 544), (100, 1536, 772)])
def test_products_through_lds(mode, M, N, K):
    """kernel_set 3: one tile and less, one past a tile, reductions of less than a 32-deep slice, of one, of eight and one more (the wavefronts'
    first round), of two rounds and a ragged rest; tolerance of the other shapes."""
    F.test_products(mode, 3, M, N, K)


@pytest.mark.parametrize("act", [0, 1])
@pytest.mark.parametrize("M,f,K", [(1, 4, 4), (17, 20, 36), (65, 36, 132), (130, 100, 524), (33, 48, 1060)])
def test_fused_activations_through_lds(act, M, f, K):
    F.test_fused_activations(act, 3, M, f, K)


@pytest.mark.parametrize("mode,M,N,K", [(0, 448, 512, 1408), (1, 448, 512, 1536), (1, 512, 512, 260), (1, 512, 516, 260), (1, 200, 640, 640)])
def test_one_round_by_the_rule(mode, M, N, K):
    """Products that the rule gives to 32 x 32 tiles, of less than a round and of more than one."""
    F.test_products(mode, 0, M, N, K)


@pytest.mark.parametrize("act,M,f,K", [(0, 1020, 1024, 36), (0, 1028, 1024, 36), (1, 1020, 512, 36), (1, 1028, 512, 36)])
def test_activations_on_either_side_of_four_rounds(act, M, f, K):
    """Activations over more than four tiles per compute unit take their operands straight into registers."""
    F.test_fused_activations(act, 3, M, f, K)
