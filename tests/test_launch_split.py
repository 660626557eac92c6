"""How a decode launch is split over workgroups: every state of a cache fits the workspace, covers its tokens and
is resident as a whole, also where the number of units is no power of two."""
import random

import pytest

import kvq_synth as S
from paper_2505_10938_amd import binding as B, cache as KC
from tests import test_gpu_parity as P

COMPUTE_UNITS, WAVES = 256, 8


@pytest.mark.parametrize("units", [1, 8, 37, 92, 128, 148, 184, 255, 256, 257, 304, 341, 400, 513, 600, 1024, 1500, 3000])
@pytest.mark.parametrize("g", [1, 4, 8])
def test_every_state_fits_and_is_resident(units, g):
    rng = random.Random(units * 16 + g)
    for G, R, N, A in ((32, 128, 8, 32), (128, 32, 3, 64), (64, 0, 0, 0), (32, 4096, 8, 32)):
        top = 32768
        cfg = KC.make_config(1, units, g, 1, top, 2, G, 32, R, N, A)
        room = B.kvq_decode_workspace_bytes(cfg, 1) - (units * 4 + 255) // 256 * 256
        if units <= 960:
            assert room <= 2048 * g * 130 * 4
        states = [0, G, 128, 1024, 4096, 4224, top] + [G * rng.randrange(top // G + 1) for _ in range(40)]
        for n_quant in states:
            for fp_rows in (1, R + G - 1 + N + A):
                splits, waves, per = B.kvq_decode_launch_shape(cfg, 1, n_quant, fp_rows)
                assert 1 <= waves <= WAVES and splits >= 1 and splits * per * 128 >= n_quant
                assert units * splits * g * 130 * 4 <= room
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
