"""GPU parity of the block tiles of middle size against the oracle, each shape by name: rows and tokens past a tile, stages that end
one to three chunks early, fewer stages than the ring holds, output rows of no whole 16 bytes, both weight forms, bias, accumulators, unequal
problems, more of them than a launch holds."""
import pytest

from gpu_util import sbn
from test_gpu_kernels_by_name import _run

pytestmark = pytest.mark.gpu

SHAPES = [(1, 16, 128), (33, 130, 256), (97, 64, 2560), (64, 129, 384), (129, 300, 512), (200, 514, 640), (300, 520, 1280), (65, 1100, 2688), (128, 128, 1024),
          (40, 95, 3456)]


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("problem", SHAPES)
@pytest.mark.parametrize("bias,acc", [(False, False), (True, True)])
@pytest.mark.parametrize("form", range(3))
def test_block_edges(form, problem, N, M, bias, acc):
    _run(sbn().SBN_KERNEL_BLOCKS + form, [problem], N, M, bias, acc)


@pytest.mark.parametrize("N,M", [(2, 4), (8, 8)])
@pytest.mark.parametrize("form", range(3))
def test_block_groups_and_adversarial_inputs(form, N, M):
    base = [(1100, 256), (518, 384), (64, 128), (95, 1152)]
    toks = [17, 64, 100, 128, 200, 257, 600, 33, 31, 65, 1]
    _run(sbn().SBN_KERNEL_BLOCKS + form, [(t, *base[i % 4]) for i, t in enumerate(toks)], N, M, bias=True)
    _run(sbn().SBN_KERNEL_BLOCKS + form, [(64, 256, 512)], N, M, adversarial=True)
