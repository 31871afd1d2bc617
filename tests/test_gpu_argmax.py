"""next_tokens of hb_run_model on planted logits: ties (the lowest index wins),
NaN columns (never chosen), infinities, and a head of NaNs alone (index 0), at
vocabulary sizes around one thread's and one workgroup's share of a row."""
import numpy as np
import pytest

from hb_workloads import TINY, make_batch, make_model_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [8, 4088, 4096, 4104, 32768, 32776, 40000])
def test_next_token_is_the_first_largest_logit(hb, vocab):
    import torch
    from paper_2503_22562_amd.harness import DeviceModel
    b = make_batch(TINY, [(1, 0), (3, 0), (1, 0)], seed=81, num_blocks=16)
    reqs = [(r.chunk_len, r.context_len, r.block_table) for r in b.requests]
    mw = make_model_weights(TINY, 1, vocab)
    dm = DeviceModel(TINY, mw, b.num_blocks, b.n_tokens, len(reqs))
    ids = b.token_ids(vocab)
    rng = np.random.default_rng(vocab)

    def run():
        nxt, logits = dm.run(reqs, ids)
        torch.cuda.synchronize()
        return nxt.cpu().numpy(), logits.cpu().numpy()

    def check(what):
        nxt, lg = run()
        want = np.argmax(np.where(np.isnan(lg), -np.inf, lg), axis=1)
        assert np.array_equal(nxt, want), (what, vocab, nxt, want)
        return nxt, lg

    nxt, lg = check("plain")
    top = int(nxt[0])
    for i in rng.integers(0, vocab, 6):  # copies of the first request's best row: equal logits
        dm.lm_head[int(i)] = dm.lm_head[top]
    nxt, lg = check("ties")
    assert np.count_nonzero(lg[0] == lg[0, nxt[0]]) > 1
    dm.lm_head[int(nxt[0])] = float("nan")
    dm.lm_head[int(nxt[1])] = float("nan")
    check("nan columns")
    dm.lm_head[vocab - 1] = 0
    dm.lm_head[vocab - 1, 0] = float("inf")
    dm.lm_head[vocab // 2] = dm.lm_head[vocab - 1]
    check("infinities")
    dm.lm_head[:] = float("nan")
    nxt, lg = run()
    assert np.isnan(lg).all() and not nxt.any()
