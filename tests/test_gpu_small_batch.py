"""The small-batch GEMM kernel (at most 64 rows) against the fp64 oracle: every
activation row group it is built for and one row to either side, on shapes
whose weight row counts take one, two and four row tiles per workgroup, with
fewer K steps than waves, K steps that do not divide among the waves, both head
sizes, and every epilogue (RoPE + pool scatter, residual, SwiGLU)."""
import numpy as np
import pytest

import oracle
from hb_workloads import LayerShape, make_batch, make_weights
from hbref import assert_parity, assert_stage, assert_swiglu_stage, oracle_for_batch

pytestmark = pytest.mark.gpu

SHAPES = [
    LayerShape("few-rows", 320, 4, 2, 64, 192, weight_seed=41),          # K of 3, 4 and 5 steps, one row tile
    LayerShape("wide-qkv", 256, 64, 32, 128, 8192, weight_seed=42),      # 16384 QKV and gate/up rows
    LayerShape("wide-hidden", 8192, 4, 2, 64, 128, weight_seed=43),      # 8192 O and down rows, K of 2 steps
    LayerShape("widest-hidden", 16384, 2, 1, 64, 64, weight_seed=44),    # 16384 O and down rows, K of 1 and 2 steps
]
_CACHE = {}


def _weights(shape):
    if shape.name not in _CACHE:
        w = make_weights(shape)
        _CACHE[shape.name] = (w, oracle.weights_to_f64(w))
    return _CACHE[shape.name]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
@pytest.mark.parametrize("T", [1, 8, 9, 16, 17, 24, 25, 32, 33, 48, 49, 64, 65])
def test_small_batch_parity(hb, shape, T):
    import torch
    from paper_2503_22562_amd import hb as H
    from paper_2503_22562_amd.harness import DeviceLayer, bf16_bits, to_device_bf16
    w, w64 = _weights(shape)
    lens = [(1, 5)] if T == 1 else [(T - 3, 9), (1, 0), (1, 33), (1, 16)]
    b = make_batch(shape, lens, seed=50 + T, num_blocks=32)
    dl = DeviceLayer(shape, w, b.num_blocks, T, len(lens))
    for r, q in enumerate(b.requests):
        if q.context_len:
            k, v = b.prior_kv(r)
            dl.append_kv(q.block_table, 0, k, v)
    y = dl.run([(q.chunk_len, q.context_len, q.block_table) for q in b.requests], to_device_bf16(b.x_in()))
    torch.cuda.synchronize()
    plans = H.hb_layer_gemm_plans(dl.layer)
    assert (len({t for t, _ in plans}) == 1 and all(ks == 1 for _, ks in plans)) or T > 64, plans
    ref, st = oracle_for_batch(b, w64, stages=True)
    assert_parity(y.cpu().numpy().astype(np.float64), ref)
    q = oracle.bf16_bits_to_f64(bf16_bits(dl.stage(H.HB_STAGE_Q, T)))
    assert_stage(q, st["q"].reshape(T, -1), "q after RoPE")
    o = oracle.bf16_bits_to_f64(bf16_bits(dl.stage(H.HB_STAGE_ATTN, T)))
    assert_stage(o, st["o"], "attention output")
    assert_parity(dl.stage(H.HB_STAGE_H2, T).cpu().numpy(), st["h2"], "h2")
    m = oracle.bf16_bits_to_f64(bf16_bits(dl.stage(H.HB_STAGE_MLP, T)))
    assert_swiglu_stage(m, st, w64, shape.rms_eps)
