"""hb_run_iteration_noalloc under HIP graph capture: a replay computes the
captured batch, whatever the layer ran in between (its pinned metadata staging
is refilled by every eager call), and eager calls after a capture work."""
import numpy as np
import pytest

from gemmcover import COVER
from hb_workloads import make_weights

pytestmark = pytest.mark.gpu

NB = 1024


def _layer(torch):
    from paper_2503_22562_amd.harness import DeviceLayer
    dl = DeviceLayer(COVER, make_weights(COVER), NB, 256, 64)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(91)
    for p in (dl.k_pool, dl.v_pool):
        p.normal_(0.0, 1.0, generator=gen)
    return dl, gen


def _batch(rng, blocks, lens):
    """Requests of these (chunk_len, context_len) over disjoint blocks of `blocks`."""
    out, at = [], 0
    blocks = rng.permutation(blocks).astype(np.int32)
    for c, x in lens:
        n = -(-(c + x) // 16)
        out.append((c, x, blocks[at:at + n].copy()))
        at += n
    assert at <= len(blocks)
    return out


def test_replay_runs_the_captured_batch(hb):
    import torch
    from paper_2503_22562_amd import hb as H
    rng = np.random.default_rng(92)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        dl, gen = _layer(torch)
        # more than one launch's worth of metadata, K splits and merged decodes; and batches of other sizes
        a = _batch(rng, np.arange(0, 700), [(90, 300)] + [(1, 190 + i) for i in range(40)] + [(1, 1500)])
        others = [_batch(rng, np.arange(*ids), lens) for ids, lens in
                  (((700, 705), [(1, 3)]), ((705, 915), [(30, 700), (1, 2500)]), ((915, NB), [(200, 0)] + [(1, 40)] * 20))]
        x, *xs = [torch.randn(sum(r[0] for r in b), COVER.hidden, device="cuda", generator=gen).to(torch.bfloat16)
                  for b in [a, *others]]
        new = lambda t: torch.full((t.shape[0], COVER.hidden), float("nan"), dtype=torch.float32, device="cuda")

        def run(b, xin):
            y = new(xin)
            H.hb_run_iteration_noalloc(dl.layer, b, xin, y)
            return y

        want = run(a, x)
        want_others = [run(b, xb) for b, xb in zip(others, xs)]
        side.synchronize()
        pools = [p.clone() for p in (dl.k_pool, dl.v_pool)]
        y = new(x)
        side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        H.hb_run_iteration_noalloc(dl.layer, a, x, y)
    with torch.cuda.stream(side):
        for i in range(6):
            got = run(others[i % 3], xs[i % 3])
            y.fill_(float("nan"))
            graph.replay()
            if i % 2:
                side.synchronize()
            after = run(others[(i + 1) % 3], xs[(i + 1) % 3])
            side.synchronize()
            assert torch.equal(y, want), i
            assert torch.equal(got, want_others[i % 3]) and torch.equal(after, want_others[(i + 1) % 3]), i
            assert all(torch.equal(p, q) for p, q in zip((dl.k_pool, dl.v_pool), pools)), i
