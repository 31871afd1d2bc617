"""Epilogues of the GEMM tiles that the planner reaches with head size 64 and with
bf16 layer output, every tile shape forced in turn (and the small-batch kernel by
its row count): RoPE inside the tile where a wave's columns hold one head or two,
which may be a q and a k head or a k and a v head, checked down to the pool; and
the bf16 store of the down projection, which rounds what the fp32 store keeps."""
import numpy as np
import pytest

import oracle
from hb_workloads import LayerShape, make_batch, make_weights
from hbref import assert_parity, assert_stage, oracle_for_batch

pytestmark = pytest.mark.gpu

LENS = [(200, 40), (1, 7), (1, 300), (90, 0), (1, 64)]  # 293 tokens
HD64 = [
    LayerShape("hd64-k-beside-v", 512, 8, 1, 64, 704, weight_seed=51),  # columns 512-639: the k head, then the v head
    LayerShape("hd64-q-beside-k", 512, 3, 3, 64, 704, weight_seed=52),  # columns 128-255: the last q head, the first k
]
TILES = [t for t in range(15) if t != 1]  # 1: the small-batch kernel
_REF = {}


def _case(shape):
    if shape.name not in _REF:
        b = make_batch(shape, LENS, seed=53, num_blocks=64)
        w = make_weights(shape)
        _REF[shape.name] = (b, w, *oracle_for_batch(b, oracle.weights_to_f64(w), stages=True))
    return _REF[shape.name]


def _layer(b, w):
    from paper_2503_22562_amd.harness import DeviceLayer
    dl = DeviceLayer(b.shape, w, b.num_blocks, b.n_tokens, len(b.requests))
    for r, q in enumerate(b.requests):
        if q.context_len:
            dl.append_kv(q.block_table, 0, *b.prior_kv(r))
    return dl, [(q.chunk_len, q.context_len, q.block_table) for q in b.requests]


def test_the_tile_list_is_the_librarys(hb):
    from paper_2503_22562_amd import hb as H
    assert H.hb_gemm_tile_count() == len(TILES) + 1


@pytest.mark.parametrize("shape", HD64, ids=lambda s: s.name)
@pytest.mark.parametrize("tile", TILES)
def test_rope_of_64_wide_heads_inside_the_tile(hb, monkeypatch, shape, tile):
    import torch
    from paper_2503_22562_amd import hb as H
    from paper_2503_22562_amd.harness import bf16_bits, k_by_slot, to_device_bf16, v_by_slot
    b, w, ref, st = _case(shape)
    monkeypatch.setenv("HB_GEMM_TILE", str(tile))
    monkeypatch.setenv("HB_GEMM_KSPLIT", "1")
    dl, reqs = _layer(b, w)
    T = b.n_tokens
    y = dl.run(reqs, to_device_bf16(b.x_in()))
    torch.cuda.synchronize()
    # tiles 13 and 14 cannot rotate 64-wide heads (96 columns a wave; more than 128
    # accumulator registers) and take QKV with a K split
    qkv = H.hb_layer_gemm_plans(dl.layer)[H.HB_GEMM_QKV]
    assert qkv[0] == tile and (qkv[1] > 1) == (tile in (13, 14)), qkv
    assert_parity(y.cpu().numpy().astype(np.float64), ref)
    q = oracle.bf16_bits_to_f64(bf16_bits(dl.stage(H.HB_STAGE_Q, T)))
    assert_stage(q, st["q"].reshape(T, -1), "q after RoPE")
    k, v = k_by_slot(bf16_bits(dl.k_pool)), v_by_slot(bf16_bits(dl.v_pool))
    t = 0
    for req in b.requests:
        at = [oracle.kv_slot(req.block_table, p) for p in range(req.context_len, req.kv_len)]
        blk, slot = (np.array(i) for i in zip(*at))
        assert_stage(oracle.bf16_bits_to_f64(k[blk, :, slot]), st["k"][t:t + len(at)], "stored K")
        assert_stage(oracle.bf16_bits_to_f64(v[blk, :, slot]), st["v"][t:t + len(at)], "stored V")
        t += len(at)


@pytest.mark.parametrize("tile,ksplit", [(t, k) for t in TILES for k in (1, 2)] + [(-1, 0)])
def test_bf16_output_is_the_rounded_fp32_output(hb, monkeypatch, tile, ksplit):
    import torch
    from paper_2503_22562_amd import hb as H
    from paper_2503_22562_amd.harness import to_device_bf16
    b, w, _, _ = _case(HD64[0])
    if tile < 0:  # the small-batch kernel
        b = make_batch(b.shape, [(50, 40), (1, 7), (1, 300), (1, 0)], seed=54, num_blocks=64)
    monkeypatch.setenv("HB_GEMM_TILE", str(tile))
    monkeypatch.setenv("HB_GEMM_KSPLIT", str(ksplit))
    dl, reqs = _layer(b, w)
    x = to_device_bf16(b.x_in())
    y32, y16 = dl.run(reqs, x, H.HB_OUT_F32), dl.run(reqs, x, H.HB_OUT_BF16)
    torch.cuda.synchronize()
    ran = H.hb_layer_gemm_plans(dl.layer)[H.HB_GEMM_DOWN]
    assert ran == ((tile, ksplit) if tile >= 0 else (1, 1)), ran
    assert torch.isfinite(y32).all() and torch.equal(y16, y32.to(torch.bfloat16))
