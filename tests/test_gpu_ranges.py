"""GPU parity at the edges of the slab tiles, the exit list's regions and the
untiled label passes: last axes around the slab tiles' rows of 8 and the
64-vertex mask word, grids of enough tiles for eight regions with room for all,
some or none of their exits, and paths longer than the first label pass
follows, around the entries a workgroup holds."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2303_02724_amd import workloads as W
from tests.gpu_util import KEYS, assert_same, gpu_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lead", [(3, 5, 9), (5, 2, 3, 5), (2, 3, 2, 3, 5)], ids=["4d", "5d", "6d"])
@pytest.mark.parametrize("x", [1, 7, 8, 9, 15, 63, 64, 65])
def test_slab_rows_of_eight(lead, x):
    f = W.random_field((*lead, x), 60 + x, "uniform")
    f[..., ::3] = np.round(f[..., ::3] * 4) / 4  # ties too
    for minima in (False, True):
        ctx = f"shape={f.shape} minima={minima}"
        print(ctx, flush=True)
        g = gpu_graph(f, minima, cap_max=f.size, cap_sad=f.size, cap_arc=8 * f.size)
        assert_same(g, O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)


@pytest.mark.parametrize("shape", [(1030, 1027), (65, 66, 515)], ids=["2d", "3d"])
@pytest.mark.parametrize("exits_log2", [None, 1, 6, 12, 16])
def test_eight_exit_regions(shape, exits_log2):
    from paper_2303_02724_amd import eg
    f = W.gaussian_random_field(shape, 7, corr_len=6.0, workers=4)
    tuning = 0 if exits_log2 is None else eg.tuning(exits_log2=exits_log2)
    for minima in (False, True):
        ctx = f"shape={shape} exits<=2^{exits_log2} minima={minima}"
        print(ctx, flush=True)
        assert_same(gpu_graph(f, minima, tuning=tuning), O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)


@pytest.mark.parametrize("shape", [(4,), (5,), (6,), (1023,), (70001,), (2, 2, 2, 1500), (1500, 2, 2, 3),
                                   (700, 1, 1, 1, 3), (1, 1, 1, 1, 2, 900)], ids=lambda s: "x".join(map(str, s)))
def test_long_untiled_paths(shape):
    i = np.arange(int(np.prod(shape)), dtype=np.float32)
    peaks = np.abs(i - 0.4 * i.size)  # one slope down and one up: a maximum at either end
    for f in (i.reshape(shape), peaks.astype(np.float32).reshape(shape)):
        for minima in (False, True):
            ctx = f"shape={shape} minima={minima}"
            print(ctx, flush=True)
            assert_same(gpu_graph(f, minima), O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)


def test_slab_of_more_threads_than_a_launch_holds():
    """A 4D grid of one long row takes eight threads per vertex: more blocks than
    one launch, the last of them ragged.  The same row as a 1D grid, whose
    kernels hold one thread per vertex, has the same graph."""
    import torch
    from paper_2303_02724_amd import eg
    n = 2 ** 28 + 37
    f = torch.arange(n, device="cuda:0", dtype=torch.int32).remainder_(1000).sub_(500).abs_().to(torch.float32)
    f[-20:] += 3
    want = None
    for shape in ((n,), (1, 1, 1, n)):
        print(shape, flush=True)
        r = eg.build(f.view(shape), want_ptr=True, cap_max=1 << 18, cap_sad=1 << 18, cap_arc=1 << 20)
        got = [r.labels.view(-1), r.ptr.view(-1), r.maxima, r.saddles, r.saddle_beta, r.arc_offsets, r.arc_maxima]
        if want is None:
            want = got
            assert r.maxima.numel() > n // 1000
        else:
            assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("shape", [(2 ** 22 + 5,), (2, 2, 2, 2 ** 19 + 1)], ids=["1d", "4d"])
def test_long_slopes_take_few_sweeps(shape):
    """Every vertex on one slope, more of them than the label kernels hold at
    once: the sweeps multiply the reach, they do not walk (150 sweeps where the
    youngest waves held one end of every run)."""
    import torch
    from paper_2303_02724_amd import eg
    n = int(np.prod(shape))
    f = torch.arange(n, device="cuda:0", dtype=torch.float32).view(shape)
    r = eg.build(f)
    assert torch.all(r.labels == n - 1)
    assert r.passes <= 30, r.passes


@pytest.mark.parametrize("shape", [(3, 65537), (3, 70001), (32769, 5), (2, 3, 66001), (8200, 3, 9)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("exits_log2", [None, 9])
def test_exit_lists_of_long_axes(shape, exits_log2):
    """1024 tiles along an axis and more: the exits' sweeps are dealt out another
    way than on other grids."""
    from paper_2303_02724_amd import eg
    tuning = 0 if exits_log2 is None else eg.tuning(exits_log2=exits_log2)
    slope = np.arange(int(np.prod(shape)), dtype=np.float32).reshape(shape)
    slope = slope if max(shape) == shape[-1] else np.ascontiguousarray(slope[::-1])
    for f in (slope, W.gaussian_mixture(shape, 8, n_gauss=6, noise=1e-2)):
        for minima in (False, True):
            ctx = f"shape={shape} exits<=2^{exits_log2} minima={minima}"
            print(ctx, flush=True)
            g = gpu_graph(f, minima, tuning=tuning, cap_max=f.size, cap_sad=f.size, cap_arc=4 * f.size)
            assert_same(g, O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)


@pytest.mark.parametrize("lead", [(3, 2, 2), (4, 1, 4), (5, 2, 2, 2), (2, 2, 1, 2), (2, 2, 1, 2, 2), (3, 1, 2, 2, 2)],
                         ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("x", [9, 16, 17, 32, 33, 63, 64, 65, 97])
def test_wide_slab_rows_of_thin_grids(lead, x):
    """Axes shorter than the slab tiles before the last one: rows of 32 (16 in
    6D) instead of 8, at the edges of the rows and of the 64-vertex mask word."""
    f = W.random_field((*lead, x), 80 + x, "uniform")
    f[..., ::3] = np.round(f[..., ::3] * 4) / 4  # ties too
    for minima in (False, True):
        ctx = f"shape={f.shape} minima={minima}"
        print(ctx, flush=True)
        g = gpu_graph(f, minima, cap_max=f.size, cap_sad=f.size, cap_arc=8 * f.size)
        assert_same(g, O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)


@pytest.mark.parametrize("shape", [(2, 3, 3, 511), (2, 3, 3, 512), (2, 2, 530, 3), (3, 2, 2, 2, 515), (2, 2, 2, 2, 2, 513),
                                   (600, 3, 3, 5), (600, 5, 6, 9)], ids=lambda s: "x".join(map(str, s)))
def test_untiled_labels_around_long_axes(shape):
    """Axes of 512 vertices and more close to the last one: the label kernels
    deal their entries out another way than on other grids."""
    slope = np.arange(int(np.prod(shape)), dtype=np.float32).reshape(shape)
    for f in (slope, W.random_field(shape, 90, "uniform"), W.gaussian_mixture(shape, 9, n_gauss=5, noise=1e-3)):
        for minima in (False, True):
            ctx = f"shape={shape} minima={minima}"
            print(ctx, flush=True)
            g = gpu_graph(f, minima, cap_max=f.size, cap_sad=f.size, cap_arc=8 * f.size)
            assert_same(g, O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)
