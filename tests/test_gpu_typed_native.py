"""GPU parity of 3D fields read in their own sample type: against the oracle
and against the general path (the order surrogate, which stage-wise launches
still take), for every type, both graphs, shapes at the edges of the 64x8x8
tile, and values that the tiles' 32-bit keys cannot tell apart: both ends of
the integer ranges (the clamped keys), float64 samples equal after rounding,
beyond float32's range and below it, -0 and infinities, and plateaus."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2303_02724_amd import eg
from paper_2303_02724_amd import workloads as W
from tests.gpu_util import KEYS, assert_same

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1, 1), (2, 1, 3), (3, 70, 2), (8, 8, 64), (9, 10, 67), (17, 16, 129)]


def _ends(shape, seed, dtype):
    """Samples crowded at the ends of the type's range and around its middle."""
    rng = np.random.Generator(np.random.PCG64(seed))
    dt = np.dtype(dtype)
    if dt == np.float64:
        vals = np.array([1e300, 2e300, -1e300, np.inf, -np.inf, 1e-320, 2e-320, -1e-320, 0.0, -0.0, 1.0,
                         1.0 + 2.0 ** -40, 1.0 + 2.0 ** -39, -1.0 - 2.0 ** -50, np.finfo(np.float64).max])
    else:
        lo, hi = int(np.iinfo(dt).min), int(np.iinfo(dt).max)
        mid = (lo + hi) // 2
        vals = np.array([lo, lo + 1, lo + 2, mid, mid + 1, hi - 2, hi - 1, hi], dtype=dt)
    return vals[rng.integers(0, vals.size, size=shape)].astype(dt)


def _np(b, r):
    return {"labels": r.labels.reshape(-1).cpu().numpy(), "ptr": r.ptr.reshape(-1).cpu().numpy(),
            "maxima": r.maxima.cpu().numpy(), "saddles": r.saddles.cpu().numpy(),
            "saddle_beta": r.saddle_beta.cpu().numpy(), "arc_offsets": r.arc_offsets.cpu().numpy(),
            "arc_maxima": r.arc_maxima.cpu().numpy()}


@pytest.mark.parametrize("dt", W.TYPED)
def test_native_types_equal_oracle_and_surrogate(dt):
    for shape in SHAPES:
        n = int(np.prod(shape))
        for kind, f in (("clusters", W.typed_field(shape, 70 + n % 7, dt)), ("ends", _ends(shape, 71 + n % 7, dt))):
            t = torch.from_numpy(np.ascontiguousarray(f)).to("cuda:0")
            for minima in (False, True):
                ctx = f"dtype={dt} shape={shape} kind={kind} minima={minima}"
                print(ctx, flush=True)
                caps = {"cap_max": n, "cap_sad": n, "cap_arc": 6 * n}
                b = eg.Builder(shape, minima=minima, want_ptr=True, **caps)
                native = _np(b, b.run(t))
                assert_same(native, O.extremum_graph(f, minima), KEYS + ["ptr"], ctx)
                p = b.paths(t)
                s = eg.Builder(shape, minima=minima, want_ptr=True, **caps)
                for stage in ("classify", "label", "arcs"):
                    s.launch(t, stage=stage)
                assert_same(_np(s, s.finish()), native, KEYS + ["ptr"], ctx + " surrogate")
                q = s.paths(eg.order_field(t))
                for k in ("pair_offsets", "path_offsets", "vertices"):
                    assert torch.equal(getattr(p, k), getattr(q, k)), f"{ctx} paths {k}"


def test_native_nan_and_misaligned_view():
    f = W.typed_field((9, 10, 67), 5, "float64")
    f[8, 9, 66] = np.nan
    for minima in (False, True):
        with pytest.raises(eg.EGError) as ei:
            eg.build(torch.from_numpy(f).to("cuda:0"), minima=minima)
        assert ei.value.status == eg.EG_ERR_NAN
    g = W.typed_field((9, 10, 67), 6, "uint8")  # a view at an odd address
    raw = torch.zeros(g.size + 1, dtype=torch.uint8, device="cuda:0")
    raw[1:].copy_(torch.from_numpy(g.reshape(-1)))
    r = eg.build(raw[1:].view(g.shape), want_ptr=True)
    assert_same(_np(None, r), O.extremum_graph(g, False), KEYS + ["ptr"], "odd address")


def test_typed_entry_refuses_what_it_does_not_read():
    b = eg.Builder((40, 50))
    t = torch.zeros((40, 50), dtype=torch.float64, device="cuda:0")
    import ctypes
    for dtype in (eg.DTYPES[torch.float64], -1, 10):
        st = eg.lib().eg_build_typed(dtype, ctypes.c_void_p(t.data_ptr()), 2, b._dims, None, ctypes.byref(b.out))
        assert st == eg.EG_ERR_ARG


# default tiles on one side of 512 (eight exit regions), the named tile's on
# the other: 256 and 512 (64x8x4), 392 and 784, 600 and 300 (64x4x16)
@pytest.mark.parametrize("dt", ["float64", "uint8", "float32"])
@pytest.mark.parametrize("shape,tile3", [((64, 128, 128), 2), ((112, 112, 128), 2), ((1200, 4, 256), 1),
                                         ((128, 128, 128), 2)], ids=["256-512", "392-784", "600-300", "512-1024"])
def test_tiles_of_the_tuning_word_and_exit_regions(shape, tile3, dt):
    rng = np.random.Generator(np.random.PCG64(17))  # noise: half of a tile's faces are exits
    f = rng.integers(0, 256, size=shape).astype(dt) if dt == "uint8" else rng.standard_normal(shape).astype(dt)
    t = torch.from_numpy(f).to("cuda:0")
    n = f.size
    caps = {"cap_max": n, "cap_sad": n, "cap_arc": 4 * n}
    for minima in (False, True):
        want = O.extremum_graph(f, minima)
        for tile in (tile3, 0):
            ctx = f"dtype={dt} shape={shape} tile3={tile} minima={minima}"
            print(ctx, flush=True)
            b = eg.Builder(shape, minima=minima, want_ptr=True, tuning=eg.tuning(tile3=tile), **caps)
            assert_same(_np(b, b.run(t)), want, KEYS + ["ptr"], ctx)
        # stage by stage, the tile changed in between
        print(f"{ctx} tile changed between stages", flush=True)
        b.launch(t, stage="classify")
        b.out.tuning = eg.tuning(tile3=tile3)
        b.launch(t, stage="label")
        b.launch(t, stage="arcs")
        assert_same(_np(b, b.finish()), want, KEYS + ["ptr"], f"{ctx} tile changed between stages")


@pytest.mark.parametrize("dt", ["int64", "uint64", "int32", "uint32"])
def test_tiles_of_the_two_limits_alone(dt):
    """Nothing between the ends of the type in any tile, either end first."""
    lo, hi = int(np.iinfo(dt).min), int(np.iinfo(dt).max)
    rng = np.random.Generator(np.random.PCG64(23))
    for vals in ((lo, hi), (lo, lo + 1, hi - 1, hi), (lo, lo + 2 ** 20, hi)):
        vals = np.array(vals, dtype=dt)
        for shape in ((5, 6, 7), (9, 17, 130)):
            for first in (0, -1):
                f = vals[rng.integers(0, vals.size, size=shape)]
                f[::8, ::8, ::64] = vals[first]  # the first sample of every tile
                n = f.size
                for minima in (False, True):
                    ctx = f"dtype={dt} {len(vals)} values, {vals[first]} first, shape={shape} minima={minima}"
                    print(ctx, flush=True)
                    b = eg.Builder(shape, minima=minima, want_ptr=True, cap_max=n, cap_sad=n, cap_arc=6 * n)
                    assert_same(_np(b, b.run(torch.from_numpy(f).to("cuda:0"))), O.extremum_graph(f, minima),
                                KEYS + ["ptr"], ctx)
