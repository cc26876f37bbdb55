"""The header read of finish(), run() and paths(): the pinned buffer that a
thread keeps for it serves calls under any torch mode, whichever mode the first
of them ran under."""
import threading

import pytest
import torch

from oracle import oracle as O
from paper_2303_02724_amd import eg
from paper_2303_02724_amd import workloads as W

pytestmark = pytest.mark.gpu


def _in_new_thread(f):
    """f() in a thread of its own, which has read no header yet."""
    out = []

    def body():
        try:
            f()
        except BaseException as e:  # noqa: BLE001 - handed to the test
            out.append(e)

    t = threading.Thread(target=body)
    t.start()
    t.join()
    if out:
        raise out[0]


@pytest.mark.parametrize("first", ["inference", "default_device"])
def test_first_read_under_a_torch_mode(first):
    f = W.gaussian_mixture((40, 50), 3, n_gauss=4, noise=1e-3)
    want = O.extremum_graph(f)
    t = torch.from_numpy(f).cuda()

    def calls():
        with torch.inference_mode() if first == "inference" else torch.device("cuda"):
            b = eg.Builder(f.shape)
            assert b.run(t).counts["saddles"] == len(want["saddles"])
        b = eg.Builder(f.shape, want_ptr=True)
        assert b.run(t).counts["saddles"] == len(want["saddles"])
        assert b.paths(t).pair_offsets.numel() == len(want["saddles"]) + 1

    _in_new_thread(calls)


def test_paths_of_a_larger_graph_without_retries():
    """Path buffers sized for an earlier field grow to the pairs that the build
    has counted, which is no retry."""
    small = W.gaussian_mixture((60, 70), 5, n_gauss=2)
    large = W.random_field((60, 70), 6, "uniform")
    b = eg.Builder(small.shape, want_ptr=True, cap_max=small.size, cap_sad=small.size, cap_arc=4 * small.size)
    for f in (small, large):
        t = torch.from_numpy(f).cuda()
        b.run(t)
        p = b.paths(t, max_retries=0)
        want = O.extremum_graph(f)
        for a, w in zip((p.pair_offsets, p.path_offsets, p.vertices), O.paths(f, want["ptr"], want["saddles"])):
            assert (a.cpu().numpy() == w).all()
    assert p.path_offsets.numel() > 64
