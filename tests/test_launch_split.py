"""How a decode launch is split over workgroups: every state of a cache fits the workspace, covers its tokens and
is resident as a whole, also where the number of units is no power of two."""
import random

import pytest

import kvq_synth as S
from paper_2505_10938_amd import binding as B, cache as KC
from tests import test_gpu_parity as P

COMPUTE_UNITS, WAVES = 256, 8


@pytest.mark.parametrize("units", [1, 8, 37, 92, 128, 148, 184, 255, 256, 257, 304, 341, 400, 512, 513, 600, 1024, 1500, 3000])
@pytest.mark.parametrize("g", [1, 4, 8])
def test_every_state_fits_and_is_resident(units, g):
    rng = random.Random(units * 16 + g)
    for G, R, N, A in ((32, 128, 8, 32), (128, 32, 3, 64), (64, 0, 0, 0), (32, 4096, 8, 32)):
        top = 32768
        cfg = KC.make_config(1, units, g, 1, top, 2, G, 32, R, N, A)
        counters = (units * 4 + 255) // 256 * 256
        room = B.kvq_decode_workspace_bytes(cfg, 1) - counters
        if units <= 960:
            assert room <= 2048 * g * 130 * 4
        states = [0, G, 128, 1024, 4096, 4224, top] + [G * rng.randrange(top // G + 1) for _ in range(40)]
        for n_quant in states:
            for fp_rows in (1, R + G - 1 + N + A):
                splits, waves, per = B.kvq_decode_launch_shape(cfg, 1, n_quant, fp_rows)
                assert 1 <= waves <= WAVES and splits >= 1 and splits * per * 128 >= n_quant
                assert units * splits * g * 130 * 4 <= room
                if splits > 1:                     # the library's own scratch array, 4 MiB, would hold what is exchanged
                    assert counters + units * splits * g * 130 * 4 <= 4 << 20
                if units <= COMPUTE_UNITS * WAVES:
                    assert units * splits <= COMPUTE_UNITS * (WAVES // waves)


@pytest.mark.gpu
@pytest.mark.parametrize("batch,kv_heads,g,bits,context", [
    (19, 8, 4, 2, 128 * 33 + 150),    # 152 units, 3 workgroups of 4 wavefronts
    (23, 4, 2, 4, 128 * 60 + 140),    # 92 units, 5 of 4
    (38, 8, 1, 2, 128 * 20 + 129),    # 304 units, 3 of 2
    (10, 4, 8, 2, 128 * 7 + 160),     # 40 units, 2 of 8
    (1, 1, 4, 2, 128 * 200 + 130),    # 1 unit, 25 of 8
])
def test_outputs_with_unit_counts_that_are_no_power_of_two(batch, kv_heads, g, bits, context):
    w = S.Workload("split", 1, batch=batch, q_heads=kv_heads * g, kv_heads=kv_heads, context=context, bits=bits)
    cfg = KC.make_config(1, w.batch, w.q_heads, w.kv_heads, w.n_quant, bits, 32, 32, w.residual, w.outlier_budget,
                         w.aux_capacity)
    assert B.kvq_decode_launch_shape(cfg, 1, w.n_quant, w.n_res + 40)[0] > 1
    n = batch * kv_heads
    units = sorted({0, n // 2, n - 1})
    P.run_sampled(w, units, regimes=("peaky",))


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [1, 2, 63, 64, 65, 130])
def test_launch_plan_of_any_number_of_sequences(batch):
    """One wavefront plans up to 64 sequences, a workgroup more: the same deal, computed here again."""
    import torch
    rng = random.Random(batch)
    cfg = KC.make_config(1, batch, 4, 1, 8192, 2, 32, 32, 128, 8, 32)
    cache = KC.RaggedKVCache(cfg)
    lengths = [rng.randrange(1, 8192) for _ in range(batch)]
    state = []
    for n in lengths:
        nq = 32 * ((n - 128) // 32) if n >= 160 else 0
        state.append([nq, 0, n - nq, 1])
    cache.seq_state.copy_(torch.tensor(state, dtype=torch.int32))
    cache.longest = max(lengths)
    cache.make_plan()
    plan = cache.plan.cpu().tolist()
    entries = (len(plan) - 8) // 8
    mc = [-(-s[0] // 128) for s in state]
    work = [2 * m + -(-s[2] // 16) + -(-40 // 16) for m, s in zip(mc, state)]
    deal = lambda share: [min(max(-(-w // share), 1), max(m, 1)) for w, m in zip(work, mc)]
    share = next(s for s in range(1, max(work) + 1) if sum(deal(s)) <= entries)
    want = []
    for b, (parts, m, s) in enumerate(zip(deal(share), mc, state)):
        per = -(-m // parts)
        want += [[b, k, parts, min(k * per, m), s[0], 0, s[2], min((k + 1) * per, m)] for k in range(parts)]
    assert plan[0] == len(want)
    assert plan[8:8 + 8 * len(want)] == [x for e in want for x in e]
