"""HIP graph capture. hb_run_iteration_noalloc: a replay computes the captured
batch, whatever the layer ran in between (its pinned metadata staging is
refilled by every eager call), and eager calls after a capture work. The other
enqueuing calls are refused without harm to the capture, the pool or later
calls."""
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


def test_other_calls_are_refused_under_capture(hb):
    import torch
    from hb_workloads import TINY, make_batch, make_model_weights
    from paper_2503_22562_amd import hb as H
    from paper_2503_22562_amd.harness import DeviceModel
    rng = np.random.default_rng(93)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        dl, gen = _layer(torch)
        a = _batch(rng, np.arange(NB), [(30, 100), (1, 400)])
        x = torch.randn(31, COVER.hidden, device="cuda", generator=gen).to(torch.bfloat16)
        k = torch.randn(9000, COVER.n_kv_heads, COVER.head_dim, device="cuda", generator=gen).to(torch.bfloat16)
        short, long = np.arange(8, dtype=np.int32), np.arange(600, dtype=np.int32)
        b = make_batch(TINY, [(5, 0), (1, 0)], seed=94, num_blocks=16)
        reqs = [(r.chunk_len, r.context_len, r.block_table) for r in b.requests]
        dm = DeviceModel(TINY, make_model_weights(TINY, 2, 200), b.num_blocks, b.n_tokens, len(reqs))
        ids = torch.from_numpy(b.token_ids(200).astype(np.int32)).cuda()
        nxt = torch.empty(2, dtype=torch.int32, device="cuda")
        logits = torch.empty((2, 200), dtype=torch.float32, device="cuda")
        H.hb_run_model(dm.model, reqs, ids, nxt, logits)
        want_logits = logits.clone()
        y = dl.run(a, x)
        want = y.clone()
        count = torch.zeros(1, device="cuda")
        side.synchronize()
        pools = [p.clone() for p in (dl.k_pool, dl.v_pool)]
        side.synchronize()
    graph = torch.cuda.CUDAGraph()
    calls = [lambda: H.hb_run_iteration(dl.layer, a, x, y), lambda: H.hb_append_kv(dl.layer, short, 0, k[:100], k[:100]),
             lambda: H.hb_append_kv(dl.layer, long, 5, k, k), lambda: H.hb_run_model(dm.model, reqs, ids, nxt, logits)]
    status = []
    with torch.cuda.graph(graph, stream=side):
        count.add_(1)
        for c in calls:
            try:
                c()
                status.append(0)
            except H.HBError as e:
                status.append(e.status)
    assert status == [H.HB_ERR_HIP] * 4
    with torch.cuda.stream(side):
        graph.replay()
        graph.replay()
        side.synchronize()
        assert count.item() == 2  # the capture went on
        assert all(torch.equal(p, q) for p, q in zip((dl.k_pool, dl.v_pool), pools))
        for _ in range(6):  # more calls than the ring has slots
            y.fill_(float("nan"))
            H.hb_run_iteration(dl.layer, a, x, y)
            logits.fill_(float("nan"))
            H.hb_run_model(dm.model, reqs, ids, nxt, logits)
            side.synchronize()
            assert torch.equal(y, want) and torch.equal(logits, want_logits)
        H.hb_append_kv(dl.layer, long, 5, k, k)
        side.synchronize()
