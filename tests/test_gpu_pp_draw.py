"""k-means++ draws formed in the launch of the weights (calls that count
nothing): the same seeds, bit for bit, as the separate draw kernel (calls with
statistics, pinned to the oracle elsewhere), at the edges of the chunks of 2048
rows, and at and past the largest number of chunks that takes one launch
(256, a thread each)."""
import numpy as np
import pytest
import torch

import synth

import paper_1902_09527_amd as km

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,d,k", [(1, 3, 1), (5, 2, 5), (2047, 4, 7), (2048, 4, 9), (2049, 5, 33), (256 * 2048, 2, 6),
                                   (256 * 2048 - 1, 1, 4),
                                   (256 * 2048 + 1, 3, 6), (60000, 17, 300)])
@pytest.mark.parametrize("prune", [True, False], ids=["prune", "noprune"])
def test_one_launch_draw_is_bit_exact(n, d, k, prune):
    print("case", n, d, k, prune, flush=True)
    g = torch.Generator(device=DEV).manual_seed(n + d)
    X = torch.randn(n, d, device=DEV, generator=g)
    X[: n // 3] += 7.0
    u = np.random.default_rng(n).random(k)
    one = km.kmeanspp(X, k, u, prune=prune)
    two = km.kmeanspp(X, k, u, prune=prune, count=True)
    for key in ("idx", "C", "D2"):
        assert torch.equal(one[key], two[key]), key


def test_one_launch_draw_when_every_row_is_a_seed():
    X = torch.ones(5000, 3, device=DEV)          # all weights zero after the first seed: the uniform rule
    u = np.random.default_rng(4).random(6)
    one, two = km.kmeanspp(X, 6, u), km.kmeanspp(X, 6, u, count=True)
    assert torch.equal(one["idx"], two["idx"]) and float(one["D2"].max()) == 0.0


def test_one_launch_draw_repeats_on_one_workspace():
    X = torch.from_numpy(synth.blobs(30000, 6, 20, seed=9)[0]).to(DEV)
    ws = torch.empty(km.kmeanspp_workspace_bytes(30000, 6, 20) + 256, dtype=torch.uint8, device=DEV)
    ref = None
    for q in range(5):                           # the counter is left ready, whatever the workspace held
        if q == 2:
            ws.fill_(255)
        u = np.random.default_rng(11).random(20)
        r = km.kmeanspp(X, 20, u, workspace=ws)["idx"]
        assert ref is None or torch.equal(r, ref)
        ref = r
