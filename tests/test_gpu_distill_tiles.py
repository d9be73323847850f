"""The fused distillation kernel on both sides of its lines: 256 tiles (one launch, or a second one that adds
the tiles' sums), narrow and wide tiles, every number of channels per lane, rows on the 4-element grid and
off it (quads that straddle lines, partial quads at the end of an image, images of fewer than four
positions).  Bars as in test_gpu_distill; the workspace starts as NaN there, and here it also carries
what calls of other shapes left in it."""
import numpy as np
import pytest
import torch

from paper_2511_12653_amd import binding as fq

import _gpu_harness as H
from test_gpu_distill import _pair, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype, shape", [
    # narrow tiles are 64 (FP16) / 32 (FP32) positions: 256 of them, one more, 256 wide ones, one more
    (np.float16, (1, 3, 16384)), (np.float16, (1, 3, 16388)), (np.float16, (1, 3, 32768)), (np.float16, (1, 3, 32772)),
    (np.float32, (1, 3, 8192)), (np.float32, (1, 3, 8196)), (np.float32, (1, 3, 16384)), (np.float32, (1, 3, 16388)),
    (np.float16, (5, 7, 4096 + 1)), (np.float32, (5, 7, 2048 + 3)),          # the same off the grid
    (np.float16, (2, 33, 32768 - 3)), (np.float32, (3, 65, 8192 - 1)),
    # channels per lane, off the grid; on it in test_gpu_distill
    *[(np.float16, (1, c, 131)) for c in (64, 65, 128, 129, 192, 193, 256, 257, 384, 385, 512)],
    *[(np.float32, (1, c, 131)) for c in (128, 129, 256, 257, 384, 385, 512)],
    *[(np.float16, (1, c, 16700)) for c in (64, 128, 192)],                   # wide
    *[(np.float32, (1, c, 8300)) for c in (128, 256, 384, 512)],
    # ends of images
    *[(d, (9, 5, m)) for d in (np.float16, np.float32) for m in (1, 2, 3, 5, 63, 65, 127, 129)],
    # more than 256 images of one or a few tiles
    *[(d, (n, 5, m)) for d in (np.float16, np.float32) for n, m in ((300, 9), (1100, 4), (300, 32), (129, 96), (130, 65))],
    (np.float32, (300, 130, 16)), (np.float32, (65, 130, 160)), (np.float32, (600, 70, 64)),
])
def test_tiles(oracle, dtype, shape):
    a, b = _pair(shape[1] * 7 + shape[2], shape, dtype)
    _run(a, b, 0.6, oracle, upstream=64.0, label="tiles")


def test_workspace_shared_by_calls_of_different_shapes(oracle):
    """Calls in turn on one workspace that nothing initialises: one launch, one launch with other tiles,
    a second launch, two reads.  What is left in it is never taken for a tile of the next call."""
    shapes = [(1, 9, 3000), (2, 40, 5001), (1, 3, 40000), (1, 530, 257), (1, 9, 3000)]
    pairs = [_pair(40 + i, s, np.float16) for i, s in enumerate(shapes)]
    H.say("distill: one workspace, shapes %s" % (shapes,))
    ds, outs, keep = [], [], []
    for (a, b), (n, c, m) in zip(pairs, shapes):
        da, db = H.dev(a), H.dev(b)
        out, ga = torch.full((3,), -1.0, dtype=torch.float64, device="cuda"), torch.zeros_like(da)
        ds.append(fq.FqDistill.from_torch(n, c, m, da, db, out, ga, lam=0.5))
        outs.append(out)
        keep.append((da, db, ga))
    ws = torch.full((max(fq.fq_distill_workspace_bytes(d) for d in ds) // 8,), float("nan"), dtype=torch.float64,
                    device="cuda")
    refs = [oracle.distill(a, b, 0.5, float(np.float32(1e-8)), 1.0) for a, b in pairs]
    for rep in range(20):
        for out in outs:
            out.fill_(-1.0)
        for d in ds:
            fq.fq_distill_loss(d, ws)
        torch.cuda.synchronize()
        for out, ref, (_, _, ga) in zip(outs, refs, keep):
            got = out.cpu().numpy()
            assert np.all(np.abs(got - np.array(ref[:3])) <= 1e-12 * np.maximum(1.0, np.abs(ref[:3]))), rep
            assert H.ulp_distance(ga.cpu().numpy(), ref[3]).max() <= 1


@pytest.mark.parametrize("tiles", [1, 2, 63, 65, 256])
@pytest.mark.parametrize("start", [0.0, float("nan")])
def test_tiles_that_come_late(tiles, start):
    """The gathering wavefront gives up at once, so the tiles behind it finish the loss: the flag, the claim and
    the records' way back to zero, eager and replayed, against the call that polls."""
    H.say("distill without polling: %d tiles, workspace starts as %r" % (tiles, start))
    shape = (1, 5, 64 * tiles)
    gen = torch.Generator(device="cuda").manual_seed(tiles)
    a, b = ((torch.randn(shape, generator=gen, device="cuda") * 1.5).half() for _ in range(2))
    out, want = (torch.zeros(3, dtype=torch.float64, device="cuda") for _ in range(2))
    ga, want_ga = torch.zeros_like(a), torch.zeros_like(a)
    d = fq.FqDistill.from_torch(*shape, a, b, out, ga, lam=0.5)
    polls = fq.FqDistill.from_torch(*shape, a, b, want, want_ga, lam=0.5)
    words = fq.fq_distill_workspace_bytes(d) // 8
    ws, ws_polls = (torch.full((words,), start, dtype=torch.float64, device="cuda") for _ in range(2))
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            fq.fq_distill_loss_no_poll(d, ws)
    torch.cuda.synchronize()
    for rep in range(8):
        a.mul_(1.0 - 0.03 * rep)
        out.fill_(float("nan"))
        ga.zero_()
        fq.fq_distill_loss(polls, ws_polls)
        torch.cuda.synchronize()
        if rep % 2:
            graph.replay()
        else:
            fq.fq_distill_loss_no_poll(d, ws)
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(ga.view(torch.int16), want_ga.view(torch.int16)), rep
        left = ws.view(torch.int64)
        assert not bool(left[:tiles * 4 + 1].any()), "a record or the flag is left after pass %d" % rep
