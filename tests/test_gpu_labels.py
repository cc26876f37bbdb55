"""GPU parity of the label pass on its fallback paths: tiles whose exit-list
entries do not fit the list keep vertex codes, which the label passes resolve
by walking the label array.  The exit list is capped through the tuning word
(EG_TUNE_EXITS, a launch choice that never changes results), so the fallback
runs on every tile of these fields; outputs are compared with the oracle
element by element, and the header must report success (no label left
unresolved by the last pass)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2303_02724_amd import eg, workloads as W
from tests.gpu_util import KEYS, assert_same, gpu_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("exits_log2", [1, 6, 12])
@pytest.mark.parametrize("tile3", [0, 1, 2])
def test_3d_exit_list_overflow(exits_log2, tile3):
    f = W.gaussian_random_field((37, 45, 150), 21, corr_len=3.0, workers=4)  # ragged tiles in every axis
    for minima in (False, True):
        ctx = f"3d exits<=2^{exits_log2} tile3={tile3} minima={minima}"
        print(ctx, flush=True)
        g = gpu_graph(f, minima, tuning=eg.tuning(tile3=tile3, exits_log2=exits_log2))
        assert_same(g, O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)


@pytest.mark.parametrize("exits_log2", [1, 8])
def test_2d_exit_list_overflow(exits_log2):
    f = W.gaussian_mixture((333, 260), 22, n_gauss=8, noise=1e-3)
    for minima in (False, True):
        ctx = f"2d exits<=2^{exits_log2} minima={minima}"
        print(ctx, flush=True)
        g = gpu_graph(f, minima, tuning=eg.tuning(exits_log2=exits_log2))
        assert_same(g, O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)


def test_long_paths_with_vertex_codes_only():
    """A ramp: one steepest-ascent path through every tile of the grid, each
    tile holding vertex codes only, with 16 links per pass: the chain of codes
    crosses far more tiles than one pass follows links."""
    f = np.arange(30 * 70 * 200, dtype=np.float32).reshape(30, 70, 200)[:, :, ::-1].copy()
    g = gpu_graph(f, tuning=eg.tuning(hops=16, exits_log2=1))
    want = O.extremum_graph(f)
    assert_same(g, want, KEYS + ["ptr"], "ramp, vertex codes")


def test_batch_exit_list_overflow():
    import torch
    shapes = [(300, 257), (33, 40, 70), (1, 1), (150, 3, 2)]
    fields = [W.gaussian_mixture(sh, 30 + i, n_gauss=6, noise=1e-3) for i, sh in enumerate(shapes)]
    ts = [torch.from_numpy(f).cuda() for f in fields]
    for minima in (False, True):
        bb = eg.BatchBuilder([f.shape for f in fields], minima=minima, tuning=eg.tuning(hops=16, exits_log2=3))
        res = bb.run(ts)
        for f, r in zip(fields, res):
            got = {"labels": r.labels.reshape(-1).cpu().numpy(), "maxima": r.maxima.cpu().numpy(),
                   "saddles": r.saddles.cpu().numpy(), "saddle_beta": r.saddle_beta.cpu().numpy(),
                   "arc_offsets": r.arc_offsets.cpu().numpy(), "arc_maxima": r.arc_maxima.cpu().numpy()}
            assert_same(got, O.extremum_graph(f, minima), KEYS, f"batch exits<=8 {f.shape} minima={minima}")


@pytest.mark.parametrize("exits_log2", [1, 12])
def test_long_slopes_with_capped_lists_take_few_sweeps(exits_log2):
    """A slope through 16385 tiles whose list holds next to nothing, alone and in
    a batch: the labels are swept, not walked one link per tile."""
    import torch
    fs = [torch.arange(n, dtype=torch.float32, device="cuda:0").expand(2, -1).contiguous()
          for n in (2 ** 20 + 3, 2 ** 17)]
    tuning = eg.tuning(exits_log2=exits_log2)
    alone = eg.build(fs[0], tuning=tuning)
    batch = eg.BatchBuilder([f.shape for f in fs], tuning=tuning).run(fs)
    for f, r in ((fs[0], alone), *zip(fs, batch)):
        assert torch.all(r.labels == f.numel() - 1)
        assert 0 < r.passes <= 30, r.passes
