"""Codes, steps and zeros of a prompt of many groups where rounding decides: the kernel that takes many groups turns the
thresholds of a group into fp16 values (2-bit) or multiplies by a reciprocal (4-bit); the step that closes a group while
decoding compares in fp32, as the definition does.  Both are given the same rows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def hard_rows(seed, batch, heads, n, group, value_group, bits, non_finite):
    """fp16 [batch, heads, n, 128] twice: each (group of tokens, channel) of the Keys and each (token, group of channels) of
    the Values one of the kinds below, of very different magnitudes."""
    rng = np.random.default_rng(seed)
    levels = 2 ** bits - 1
    f16 = np.float16

    def groups(count, size):
        step = f16(rng.random((count, 1)) * 2.0 ** rng.integers(-24, 12, (count, 1)) + 2.0 ** -24).astype(np.float64)
        kind = rng.integers(0, 9, (count, 1))
        half = rng.integers(0, 2 * levels + 1, (count, size)) * step / 2          # ties: odd multiples of step / 2
        nudge = rng.integers(-1, 2, (count, size))
        near = np.nextafter(f16(half), f16(1e4) * nudge.astype(f16)).astype(np.float64)
        tiny = rng.integers(-3, 4, (count, size)) * 2.0 ** -24
        lo = -(2 * rng.integers(1, levels + 1, (count, 1)) - 1) * step / 2        # a threshold at (about) zero
        across = np.where(rng.random((count, size)) < 0.6, tiny, lo + rng.integers(0, levels + 1, (count, size)) * step)
        normal = rng.standard_normal((count, size)) * step
        offset = 16.0 * step * rng.integers(1, 2000, (count, 1)) + normal
        zeros = np.where(rng.random((count, size)) < 0.5, -0.0, 0.0)
        constant = np.broadcast_to(step, (count, size))
        wide = rng.choice([-65504.0, 65504.0, 1.0, 2.0 ** -24, -0.0], (count, size))
        x = np.select([kind == k for k in range(9)],
                      [half, near, -half, across, np.where(rng.random((count, size)) < 0.1, lo, across), normal, offset,
                       np.where(kind % 2, zeros, np.where(rng.random((count, 1)) < 0.5, zeros, constant)), wide])
        if non_finite:
            hit = (rng.random((count, 1)) < 0.02) & (rng.random((count, size)) < 0.1)
            x = np.where(hit, rng.choice([np.inf, -np.inf, np.nan], (count, size)), x)
            x = np.where(rng.random((count, 1)) < 0.01, np.nan, x)                # not one number in the group
        with np.errstate(over="ignore"):
            return np.clip(f16(x), f16(-65504), f16(65504)) if not non_finite else f16(x)

    units = batch * heads
    k = groups(units * (n // group) * 128, group).reshape(units, n // group, 128, group).transpose(0, 1, 3, 2)
    v = groups(units * n * (128 // value_group), value_group)
    return (np.ascontiguousarray(k).reshape(batch, heads, n, 128), v.reshape(batch, heads, n, 128))


@pytest.mark.parametrize("non_finite", [False, True])
@pytest.mark.parametrize("budget", [0, 5])
@pytest.mark.parametrize("bits,group,value_group", [(2, 32, 32), (2, 64, 64), (2, 128, 128), (4, 32, 64), (4, 64, 128), (4, 128, 32)])
def test_a_prompt_gives_the_bytes_of_its_tokens_one_by_one(bits, group, value_group, budget, non_finite):
    import torch
    if non_finite and budget:
        pytest.skip("scores that are no numbers are not supported")
    batch, heads, n = 32, 4, 8 * group
    k, v = (torch.from_numpy(x).cuda() for x in hard_rows(bits * group + value_group, batch, heads, n, group, value_group, bits, non_finite))
    if budget:                                                # (scores are exact up to a sum of 2^23; tracing is not the point)
        k = k.clamp(-3e4, 3e4)

    compare_with_steps(k, v, bits, group, value_group, budget)


def compare_with_steps(k, v, bits, group, value_group, budget):
    import torch
    from paper_2505_10938_amd import cache as KC
    batch, heads, n = k.shape[:3]
    prompt, steps = (KC.KVCache(KC.make_config(1, batch, heads, heads, n, bits, group, value_group, 0, budget,
                                               32 if budget else 0, 128)) for _ in range(2))
    prompt.prefill(0, k, v)
    for i in range(n):
        steps.append(0, k[:, :, i].contiguous(), v[:, :, i].contiguous())
    assert prompt.n_quant == steps.n_quant == [n]
    for name in ("k_codes", "k_meta", "v_codes", "v_meta", "mask"):
        assert torch.equal(getattr(prompt, name).view(torch.uint8), getattr(steps, name).view(torch.uint8)), name


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("group,groups", [(32, 63), (32, 64), (32, 65), (64, 7), (64, 8), (64, 9), (128, 1), (128, 2)])
def test_either_side_of_the_change_of_kernels(bits, group, groups):
    """Four units: 256 groups of 32 tokens, 32 of 64 and one of 128 are the first that go to the kernel for many."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(group + groups)
    k, v = (torch.randn(1, 4, group * groups, 128, generator=gen, device="cuda").half() for _ in range(2))
    compare_with_steps(k, v, bits, group, 32, 3)
