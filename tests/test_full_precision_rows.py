"""Full-precision rows in the decode launch: weights far below the largest one, and Values that are infinite."""
import math

import numpy as np
import pytest

from paper_2505_10938_amd import binding as B, cache as KC

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g,bits", [(1, 2), (2, 2), (4, 2), (8, 2), (8, 4)])
@pytest.mark.parametrize("drop", [12.3, 16.5, 20.7, 24.5, 26.0, 34.0])
def test_many_tokens_of_small_weight(g, bits, drop):
    """One token that takes nearly all the weight and has Values of zero, 3999 tokens of 2^-drop of it whose Values
    make up the whole output.  The output is 4000 equal terms in fp32 and one rounding to fp16: a relative error of
    2^-11, and of the weights what their scores are off by, |score| 2^-22 < 1e-5."""
    import torch
    n, kv_heads = 4000, 2
    cache = KC.KVCache(KC.make_config(1, 1, g * kv_heads, kv_heads, 32, bits, 32, 32, 4096, 8, 32))
    K = np.zeros((kv_heads, n, 128), np.float16)
    K[:, 1234, 0] = drop * math.sqrt(128) / math.log2(math.e)
    V = np.full((kv_heads, n, 128), 30000.0, np.float16) * np.linspace(0.5, 1.0, 128).astype(np.float16)
    V[:, 1234] = 0
    q = np.zeros((1, g * kv_heads, 128), np.float16)
    q[:, :, 0] = 1
    cache.load_residual(0, torch.from_numpy(K)[None].cuda(), torch.from_numpy(V)[None].cuda())
    out = cache.decode(0, torch.from_numpy(q).cuda()).cpu().numpy().astype(np.float64)
    w = np.exp(K[0, :, 0].astype(np.float64) / math.sqrt(128) - float(K[0, 1234, 0]) / math.sqrt(128))
    want = (w / w.sum()) @ V[0].astype(np.float64)
    # (an output below fp16's normal range, drop = 34 aside, would be off by half of 2^-24 more)
    assert np.all(np.abs(out - want) <= 2.0 ** -11 * 1.02 * np.abs(want) + 2.0 ** -25)


def plant_and_compare(batch, kv_heads, g, context, residual, splits, waves, bits=2):
    """An infinite Value in one channel of one full-precision row is an infinity in that channel of the outputs that
    attend to the row, and changes nothing else."""
    import torch
    G = 32
    nq = G * ((context - residual) // G) if context >= residual + G else 0
    cfg = KC.make_config(1, batch, g * kv_heads, kv_heads, max(nq, G), bits, G, 32, residual, 8, 32)
    assert B.kvq_decode_launch_shape(cfg, 1, nq, context - nq + 40)[:2] == (splits, waves)
    cache = KC.KVCache(cfg)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(context)
    K, V = (torch.randn(batch, kv_heads, context, 128, generator=gen, device="cuda").half() for _ in range(2))
    q = (0.1 * torch.randn(batch, g * kv_heads, 128, generator=gen, device="cuda")).half()
    cache.prefill(0, K, V)
    plain = cache.decode(0, q).cpu()
    assert bool(torch.isfinite(plain).all())
    unit, rows = batch * kv_heads - 1, cache.res_view("v")
    for row in sorted({0, 17, (context - nq) // 2, context - nq - 1} & set(range(context - nq))):
        for value in (float("inf"), float("-inf")):
            kept = rows[unit, row, 77].clone()
            rows[unit, row, 77] = value
            out = cache.decode(0, q).cpu()
            rows[unit, row, 77] = kept
            want = plain.clone()
            want.view(batch * kv_heads, g, 128)[unit, :, 77] = value
            assert torch.equal(out, want), (row, value, out.view(batch * kv_heads, g, 128)[unit, :, 77])


@pytest.mark.parametrize("batch,kv_heads,g,context,residual,splits,waves", [
    (128, 8, 1, 150, 128, 1, 2), (64, 8, 2, 150, 128, 1, 4), (64, 8, 4, 1100, 128, 1, 4), (64, 8, 8, 300, 128, 1, 4),
    (1, 1, 1, 400, 128, 1, 8), (1, 4, 8, 400, 128, 1, 8), (1, 1, 4, 4200, 128, 8, 8),
])
@pytest.mark.parametrize("bits", [2, 4])
def test_infinite_value_in_a_full_precision_row(batch, kv_heads, g, context, residual, splits, waves, bits):
    plant_and_compare(batch, kv_heads, g, context, residual, splits, waves, bits)


@pytest.mark.parametrize("batch,kv_heads,g,context,residual,splits,waves", [
    (1, 1, 1, 40, 32, 1, 3), (1, 1, 1, 150, 32, 1, 4), (1, 1, 2, 300, 32, 1, 5), (1, 1, 8, 400, 32, 1, 6),
    (1, 1, 4, 200, 128, 1, 7), (1, 1, 2, 600, 32, 2, 4), (1, 4, 1, 1100, 128, 2, 7), (1, 1, 8, 1100, 32, 3, 8),
    (1, 4, 1, 2100, 128, 4, 6), (1, 1, 4, 2100, 32, 4, 8), (1, 1, 2, 4200, 128, 8, 5),
])
def test_infinite_value_where_fewer_results_are_merged_than_a_merge_has_room_for(batch, kv_heads, g, context, residual,
                                                                                 splits, waves):
    """The merge of a workgroup's wavefronts takes 4, 8 or 16 results, that of a unit's workgroups eight at a time: the
    places beyond the last result count for nothing, also when the last result is infinite."""
    plant_and_compare(batch, kv_heads, g, context, residual, splits, waves)
