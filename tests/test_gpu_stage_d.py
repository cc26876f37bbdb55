"""GPU parity of the compaction and arc kernels where their rounds and block
sums can go wrong: masks denser than the emission's LDS stage (1D noise, two
thirds of the vertices critical), row lengths around the 64-vertex mask word,
chunks of one and of several rounds, and the last block's header."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2303_02724_amd import workloads as W
from tests.gpu_util import KEYS, assert_same, gpu_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(16383,), (70001,), (3, 5461), (257, 63), (255, 65), (1030, 1027), (129, 64, 65),
                                   (20, 21, 22, 23)], ids=lambda s: "x".join(map(str, s)))
def test_dense_masks_and_block_sums(shape):
    f = W.random_field(shape, 40 + len(shape), "uniform")
    for minima in (False, True):
        ctx = f"shape={shape} minima={minima}"
        print(ctx, flush=True)
        n = f.size
        g = gpu_graph(f, minima, cap_max=n, cap_sad=n, cap_arc=8 * n)
        assert_same(g, O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)
