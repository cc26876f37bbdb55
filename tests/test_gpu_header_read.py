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
