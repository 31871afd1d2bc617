"""Split decodes and their merge against the oracle's attention on the kernel's
own inputs: every group size, both head sizes, and up to 33 parts per group, so
that the merge deals its parts to 1, 2, 4, 8 or 16 column slots."""
import numpy as np
import pytest

from hb_workloads import LayerShape, make_batch, make_weights
from hbref import check_attention_kernel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("group", [1, 2, 4, 8, 16])
def test_split_decodes_and_merge(hb, monkeypatch, group, hd):
    import torch
    from paper_2503_22562_amd import hb as H
    from paper_2503_22562_amd.harness import DeviceLayer, bf16_bits, to_device_bf16
    monkeypatch.setenv("HB_ATTN_SPLIT_ITEM", "64")
    shape = LayerShape(f"merge-g{group}", 128, 2 * group, 2, hd, 64, weight_seed=60 + group)
    # 1 .. 33 parts of four 64-key ranges, and chunks whose columns fill one or several units
    lens = [(1, 8447), (1, 511), (1, 256), (1, 255), (1, 64), (1, 0), (3, 1300), (2, 2047)]
    b = make_batch(shape, lens, seed=70 + group, num_blocks=1024)
    dl = DeviceLayer(shape, make_weights(shape), b.num_blocks, b.n_tokens, len(lens))
    for r, q in enumerate(b.requests):
        if q.context_len:
            k, v = b.prior_kv(r)
            dl.append_kv(q.block_table, 0, k, v)
    dl.run([(q.chunk_len, q.context_len, q.block_table) for q in b.requests], to_device_bf16(b.x_in()))
    torch.cuda.synchronize()
    T = b.n_tokens
    q = bf16_bits(dl.stage(H.HB_STAGE_Q, T))
    o = bf16_bits(dl.stage(H.HB_STAGE_ATTN, T))
    print("worst error / bound", check_attention_kernel(dl, b, np.arange(T), q, o))
