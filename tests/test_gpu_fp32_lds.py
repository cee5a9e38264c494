"""fp32 products whose 32 x 32 tiles take their operands through LDS."""
import re

import pytest

from tests import test_gpu_fp32 as F
from tests.gpu_util import launches
from tests.test_gpu_kernels import L, P

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


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("M,N,K", [(278, 384, 384), (214, 576, 2720), (819, 128, 2848), (127, 1344, 160)])
def test_no_further_from_64_bits_than_small_tiles(mode, M, N, K):
    """A wavefront of a 32 x 32 tile sums no more terms in one register than one of a 16 x 16 tile, which splits the reduction over twice as
    many: the two are as far from 64 bits (2-norms over at least 1e5 outputs, which repeat themselves to about one in the square root
    of that; 10 % allowed.  With one sum per wavefront 5 to 36 % further)."""
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(M + K + mode)
    a, b = (torch.randn(s, generator=g, device="cuda:0") for s in ((M, K), (N, K) if mode else (K, N)))
    exact = a.double() @ (b.double().t().contiguous() if mode else b.double())

    def off(kernel_set):
        c = torch.empty((M, N), device="cuda:0")
        assert L().stage_kernel_gemm(0, mode, M, N, K, P(a), K, P(b), b.shape[1], P(c), N, None, 0, 0, kernel_set, None) == 0
        torch.cuda.synchronize()
        return float((c.double() - exact).norm() / exact.norm())

    small, through_lds = off(4), off(3)
    assert through_lds <= 1.1 * small


FORWARD, RESID, DGRAD, GELU, SWIGLU, DGELU, DSWIGLU = range(7)
# (kind, M, N, K): tile and whether its operands go through LDS, on both sides of every line (256 compute units); SwiGLU's N counts gate and up
RULE = [
    ((FORWARD, 448, 512, 256), (32, True)), ((FORWARD, 448, 512, 260), (32, False)), ((FORWARD, 448, 512, 1276), (32, False)), ((FORWARD, 448, 512, 1284), (32, True)),
    ((FORWARD, 512, 1024, 256), (32, True)), ((FORWARD, 516, 1024, 256), (32, False)), ((FORWARD, 516, 1024, 288), (32, True)),
    ((FORWARD, 448, 2336, 512), (32, True)), ((FORWARD, 448, 2816, 512), (32, False)), ((FORWARD, 700, 3072, 768), (32, True)),
    ((FORWARD, 1024, 2432, 512), (64, False)), ((FORWARD, 1084, 4032, 448), (64, False)), ((RESID, 448, 512, 1408), (32, True)),
    ((DGRAD, 516, 1024, 64), (64, False)), ((DGRAD, 1084, 1024, 64), (32, False)), ((SWIGLU, 114, 2040, 1024), (32, False)), ((DGRAD, 516, 1024, 96), (32, True)), ((DGRAD, 512, 1024, 64), (32, True)), ((DGRAD, 448, 512, 504), (32, False)),
    ((DGRAD, 700, 1024, 1288), (32, True)), ((DGRAD, 171, 4000, 1536), (64, False)), ((DGRAD, 1024, 2432, 1024), (32, True)), ((DGRAD, 1084, 4032, 448), (64, False)),
    ((GELU, 512, 1024, 512), (32, True)), ((GELU, 516, 1024, 512), (32, False)), ((GELU, 448, 512, 264), (32, False)),
    ((SWIGLU, 448, 1024, 256), (32, False)), ((SWIGLU, 448, 1024, 288), (32, True)), ((SWIGLU, 448, 1664, 512), (32, True)), ((SWIGLU, 448, 2048, 512), (64, False)), ((SWIGLU, 448, 2816, 512), (32, False)),
    ((SWIGLU, 900, 2600, 640), (64, False)), ((SWIGLU, 1084, 4032, 448), (64, False)),
    ((DGELU, 512, 1024, 256), (32, True)), ((DGELU, 516, 1024, 256), (64, False)), ((DGELU, 900, 2600, 640), (32, True)), ((DSWIGLU, 516, 1024, 288), (32, True)),
    ((DSWIGLU, 451, 1536, 1280), (32, True)), ((DSWIGLU, 171, 4000, 1280), (64, False)), ((DSWIGLU, 195, 1000, 200), (32, False)),
]


@pytest.mark.parametrize("shape,expect", RULE)
def test_tile_and_form_by_the_rule(shape, expect):
    """Read off the launched kernel (a capture: nothing runs, so the buffers are only names)."""
    import torch
    kind, M, N, K = shape
    t = P(torch.zeros(256, dtype=torch.uint8, device="cuda:0"))
    if kind <= DGRAD:
        (name, _, _), = launches(lambda s: L().stage_kernel_gemm(0, int(kind == DGRAD), M, N, K, t, K, t, K if kind == DGRAD else N, t, N, t if kind == RESID else None, N, 0, 0, s))
    elif kind <= SWIGLU:
        f = N // 2 if kind == SWIGLU else N
        (name, _, _), = launches(lambda s: L().stage_kernel_gemm_act(0, int(kind == SWIGLU), M, f, K, t, K, t, N, t, N, t, f, 0, s))
    else:
        (name, _, _), = launches(lambda s: L().stage_kernel_gemm_act_bwd(0, int(kind == DSWIGLU), M, N, K, t, K, t, K, t, (1 + (kind == DSWIGLU)) * N, t, 0, s))
    m = re.search(r"gemm32_kernelILi\d+ELi(\d+)ELi\d+ELi\d+ELi\d+ELb([01])E", name)
    assert (16 * int(m[1]), m[2] == "1") == expect


@pytest.mark.parametrize("mode,M,N,K", [(0, 516, 1024, 256), (0, 448, 512, 260), (1, 448, 512, 504), (0, 65, 140, 1276)])
def test_straight_to_registers_by_the_rule(mode, M, N, K):
    F.test_products(mode, 0, M, N, K)


@pytest.mark.parametrize("act,M,f,K", [(0, 516, 1024, 96), (1, 448, 512, 256), (1, 65, 100, 264)])
def test_activations_straight_to_registers_by_the_rule(act, M, f, K):
    F.test_fused_activations(act, 0, M, f, K)
