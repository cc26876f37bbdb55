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


def _few_saddles(kind):
    """Fields with few saddles, so that the paths' vertices are recorded in the
    first walk and copied in the second: a valley between two long slopes
    (paths around and far beyond the recorded 128 steps), a smooth 3D field,
    and a saddle with twenty paths (more than are recorded)."""
    if kind == "twenty":
        from tests.test_oracle_pins import twenty_arc_saddle
        return twenty_arc_saddle()[0]
    if kind == "smooth":
        return W.gaussian_random_field((48, 50, 70), 9, corr_len=5.0, workers=4)
    steps = int(kind)
    x = np.abs(np.arange(2 * steps + 1, dtype=np.float32) - steps)
    return np.stack([x, x - 0.5, x - 0.75])


@pytest.mark.parametrize("kind", ["smooth", "twenty", "126", "127", "128", "129", "1500"])
def test_recorded_paths(kind):
    from paper_2303_02724_amd import eg
    import torch
    f = np.ascontiguousarray(_few_saddles(kind), dtype=np.float32)
    for minima in (False, True):
        want = O.extremum_graph(f, minima)
        wp = O.paths(f, want["ptr"], want["saddles"], minima)
        _, p = eg.build_paths(torch.from_numpy(f).cuda(), minima=minima)
        for a, b, name in zip((p.pair_offsets, p.path_offsets, p.vertices), wp,
                              ("pair_offsets", "path_offsets", "vertices")):
            assert np.array_equal(a.cpu().numpy(), b), f"{kind} minima={minima} {name}"


@pytest.mark.parametrize("shape", [(4, 4, 4, 4, 5), (9, 9, 9, 9, 9)], ids=["one-round", "several-blocks"])
def test_paths_of_5d_noise(shape):
    """Blocks of the 5D path kernels hold other numbers of threads than those
    of the 5D arc kernels."""
    from paper_2303_02724_amd import eg
    import torch
    f = W.random_field(shape, 19, "uniform")
    for minima in (False, True):
        want = O.extremum_graph(f, minima)
        wp = O.paths(f, want["ptr"], want["saddles"], minima)
        _, p = eg.build_paths(torch.from_numpy(f).cuda(), minima=minima)
        for a, b, name in zip((p.pair_offsets, p.path_offsets, p.vertices), wp,
                              ("pair_offsets", "path_offsets", "vertices")):
            assert np.array_equal(a.cpu().numpy(), b), f"{shape} minima={minima} {name}"


@pytest.mark.parametrize("corr_len", [0.8, 1.2, 1.5, 1.65])
def test_paths_recorded_for_few_steps(corr_len):
    """Scratch for 4 to 26 steps of every path, of which the longest take 10 to
    20: around the fewest steps for which paths are recorded."""
    from paper_2303_02724_amd import eg
    import torch
    f = W.gaussian_random_field((48, 50, 70), 9, corr_len=corr_len, workers=4)
    for minima in (False, True):
        want = O.extremum_graph(f, minima)
        wp = O.paths(f, want["ptr"], want["saddles"], minima)
        _, p = eg.build_paths(torch.from_numpy(f).cuda(), minima=minima)
        for a, b, name in zip((p.pair_offsets, p.path_offsets, p.vertices), wp,
                              ("pair_offsets", "path_offsets", "vertices")):
            assert np.array_equal(a.cpu().numpy(), b), f"{corr_len} minima={minima} {name}"
