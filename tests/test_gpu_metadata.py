"""Metadata uploads back to back: batches with metadata small enough for the
copy on the layer's stream and larger ones through the copy stream, enqueued in
turn without a synchronisation in between (more of them than the staging ring
has slots), give the bits of the same batches run one at a time."""
import numpy as np
import pytest

from gemmcover import COVER

pytestmark = pytest.mark.gpu


def _decodes(rng, nb, n, keys):
    """n decodes over shared prefix blocks, each with a last block of its own
    (one of the last 256, which no prefix holds)."""
    full = (keys - 1) // 16
    prefix = rng.permutation(nb - 256)[:full].astype(np.int32)
    return [(1, full * 16 + 3, np.append(prefix, np.int32(nb - 1 - i))) for i in range(n)]


def test_uploads_in_turn_match_single_runs(hb):
    import torch
    from hb_workloads import make_weights
    from paper_2503_22562_amd.harness import DeviceLayer
    nb, rng = 1024, np.random.default_rng(71)
    dl = DeviceLayer(COVER, make_weights(COVER), nb, 256, 256)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(72)
    for p in (dl.k_pool, dl.v_pool):
        p.normal_(0.0, 1.0, generator=gen)
    # 230 x 313 block ids lie above 65536 int32 of metadata, the others below
    batches = [_decodes(rng, nb, *c) for c in ((1, 40), (230, 5000), (7, 900), (33, 2000), (230, 4990), (2, 17))]
    xs = [torch.randn(len(b), COVER.hidden, device="cuda", generator=gen).to(torch.bfloat16) for b in batches]
    assert sum(len(r[2]) for r in batches[1]) > 1 << 16
    want = []
    for b, x in zip(batches, xs):
        want.append(dl.run(b, x).clone())
        torch.cuda.synchronize()
    order = [int(i) for i in rng.integers(0, len(batches), 24)]
    got = [dl.run(batches[i], xs[i]) for i in order]
    torch.cuda.synchronize()
    for n, i in enumerate(order):
        assert torch.all(torch.isfinite(got[n])) and torch.equal(got[n], want[i]), (n, i)


@pytest.mark.parametrize("n,keys", [(2, 17), (230, 5000)], ids=["in-stream", "copy-stream"])
def test_eight_iterations_are_enqueued_without_waiting(hb, n, keys):
    """The call returns with its iteration enqueued: eight of them behind work that
    the stream has not got through, none waiting for the one before."""
    import time

    import torch
    from hb_workloads import make_weights
    from paper_2503_22562_amd.harness import DeviceLayer
    nb, rng = 1024, np.random.default_rng(73)
    dl = DeviceLayer(COVER, make_weights(COVER), nb, 256, 256, pool_fill_bits=0)
    b = _decodes(rng, nb, n, keys)
    x = torch.zeros((n, COVER.hidden), dtype=torch.bfloat16, device="cuda")
    y = dl.run(b, x)
    for _ in range(20):  # every slot's buffers exist
        dl.run(b, x, x_out=y)
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    torch.cuda._sleep(1_000_000)
    torch.cuda.synchronize()
    per_ms = 1_000_000 / (1e3 * (time.perf_counter() - t0))
    busy = torch.cuda.Event()
    torch.cuda._sleep(int(per_ms * 500))
    busy.record()
    for i in range(8):
        dl.run(b, x, x_out=y)
        assert not busy.query(), i
    torch.cuda.synchronize()
