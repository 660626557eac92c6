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
@pytest.mark.parametrize("batch,kv_heads,g,bits,context,shape", [
    (19, 8, 4, 2, 128 * 33 + 150, (3, 4)),    # 152 units
    (23, 4, 2, 4, 128 * 60 + 140, (5, 4)),    # 92 units
    (38, 8, 1, 2, 128 * 20 + 129, (3, 2)),    # 304 units
    (10, 4, 8, 2, 128 * 7 + 160, (6, 8)),     # 40 units: 8 mini-chunks, the last two workgroups have none
    (1, 1, 4, 2, 128 * 200 + 130, (25, 8)),   # 1 unit
    (1, 1, 4, 2, 4200, (8, 8)),               # some wavefronts have quantized tokens, some rows, some neither
    (1, 8, 4, 2, 1100, (8, 8)),               # one mini-chunk per workgroup
    (1, 8, 2, 2, 800, (4, 4)),                # the last workgroup has rows alone
    (2, 8, 1, 2, 5300, (12, 4)),              # more partial results than are merged at a time
    (2, 8, 1, 4, 5300, (12, 4)),
])
def test_outputs_with_unit_counts_that_are_no_power_of_two(batch, kv_heads, g, bits, context, shape):
    w = S.Workload("split", 1, batch=batch, q_heads=kv_heads * g, kv_heads=kv_heads, context=context, bits=bits)
    cfg = KC.make_config(1, w.batch, w.q_heads, w.kv_heads, w.n_quant, bits, 32, 32, w.residual, w.outlier_budget,
                         w.aux_capacity)
    assert B.kvq_decode_launch_shape(cfg, 1, w.n_quant, w.n_res + 40)[:2] == shape
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


@pytest.mark.gpu
@pytest.mark.parametrize("batch,kv_heads,g,context,residual,budget,shape", [
    (1, 1, 4, 4200, 128, 8, (8, 8)),      # some wavefronts have quantized tokens, some rows, some neither
    (1, 2, 8, 1100, 100, 3, (2, 8)),
    (2, 2, 1, 2100, 128, 8, (4, 6)),      # all have quantized tokens or rows, few have both
    (1, 8, 4, 1100, 128, 8, (8, 8)),      # one mini-chunk per workgroup
    (1, 8, 2, 800, 128, 8, (4, 4)),       # the last workgroup has rows alone
    (2, 8, 1, 5300, 128, 8, (12, 4)),     # more partial results than are merged at a time, the last ones of rows alone
    (16, 8, 4, 320, 128, 8, (1, 8)),      # two of eight have quantized tokens
    (1, 2, 2, 100, 128, 8, (1, 5)),       # none has
    (1, 1, 1, 9, 32, 0, (1, 1)),          # one wavefront with one group of rows
    (40, 8, 4, 4150, 128, 8, (3, 2)),     # every wavefront has both
])
@pytest.mark.parametrize("paged", [False, True])
def test_step_equals_its_parts_however_the_work_is_dealt(batch, kv_heads, g, context, residual, budget, shape, paged):
    """Rotation, append and attention in one launch against a launch of its own for each: the same bits, in the
    outputs and in the ring."""
    import torch
    nq = 32 * ((context - residual) // 32) if context >= residual + 32 else 0
    cfg = KC.make_config(1, batch, g * kv_heads, kv_heads, max(nq, 32), 2, 32, 32, residual, budget, 32 if budget else 0)
    slots = budget + 32 if budget else 0
    assert B.kvq_decode_launch_shape(cfg, 1, nq, context - nq + 1 + slots)[:2] == shape
    groups = cfg.max_seq // 32
    cache = KC.KVCache(cfg, n_pages=batch * groups if paged else None)
    if paged:
        cache.page_table.copy_(torch.randperm(batch * groups, generator=torch.Generator().manual_seed(3)).view(batch, groups))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(context)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda").half()
    cache.prefill(0, new(batch, kv_heads, context, 128), new(batch, kv_heads, context, 128))
    k, v, q = new(batch, kv_heads, 128), new(batch, kv_heads, 128), new(batch, g * kv_heads, 128)
    angle = torch.arange(64, device="cuda") / 7.0
    rope = torch.cat([angle.cos(), angle.sin()]).float()
    parts = KC.KVCache(cfg, n_pages=batch * groups) if paged else cache.clone()
    if paged:
        for name in ("k_codes", "k_meta", "v_codes", "v_meta", "mask", "page_table", "k_res", "v_res", "pool_k", "pool_v",
                     "pool_idx", "pool_score", "pool_count", "aux_count", "frozen"):
            getattr(parts, name).copy_(getattr(cache, name))
        parts.n_quant, parts.n_res = list(cache.n_quant), list(cache.n_res)
    got = cache.step(0, k, v, q, rope=rope)
    kr, qr = torch.empty_like(k), torch.empty_like(q)
    B.kvq_rope_rotate(cfg, k, kv_heads, rope, 0, kr)
    B.kvq_rope_rotate(cfg, q, g * kv_heads, rope, 0, qr)
    assert not parts.append(0, kr, v)
    want = parts.decode(0, qr)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(got).all()) and float(got.abs().max()) > 0
    assert torch.equal(got, want)
    assert torch.equal(cache.k_res, parts.k_res) and torch.equal(cache.v_res, parts.v_res)
