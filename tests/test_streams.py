"""Calls on a stream that is not torch's current one: what they prepare on the device (buffers allocated on first use,
temporaries, the state of a sequence) is ordered with their launches, whatever else either stream has to do."""
import pytest

from paper_2505_10938_amd import cache as KC

pytestmark = pytest.mark.gpu

BUSY = 20_000_000      # clock cycles that a stream is kept busy for, about 10 ms: far longer than any call below


def rows(n, heads=2, batch=None, seed=1):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    shape = (heads, n, 128) if batch is None else (batch, heads, n, 128)
    return tuple(torch.randn(shape, generator=gen, device="cuda").half() for _ in range(2))


def handles(stream):
    """The stream as the calls take it: an object, or its handle."""
    return [stream, stream.cuda_stream]


@pytest.mark.parametrize("form", [0, 1])
def test_state_of_a_joining_sequence_is_written_behind_the_calls_before_it(form):
    import torch
    cache = KC.RaggedKVCache(KC.make_config(1, 2, 2, 2, 256, residual=32))
    k, v = rows(300)
    cache.prefill_sequence(1, [k], [v])
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(BUSY)
        before = cache.seq_state.clone()
    cache.prefill_sequence(1, [k[:, :100].contiguous()], [v[:, :100].contiguous()], stream=handles(side)[form])
    torch.cuda.synchronize()
    assert before[1].tolist() == [256, 0, 44, 1]
    assert cache.seq_state[1].tolist() == [64, 0, 36, 1]


@pytest.mark.parametrize("form", [0, 1])
def test_first_prompt_on_a_side_stream(form):
    import torch
    cfg = KC.make_config(1, 1, 2, 2, 256, residual=32)
    k, v = rows(300, batch=1)
    want = KC.KVCache(cfg)
    want.prefill(0, k, v)
    cache = KC.KVCache(cfg)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda._sleep(BUSY)
    cache.prefill(0, k, v, stream=handles(side)[form])
    torch.cuda.synchronize()
    assert int(want.prefill_selected.sum()) > 0
    assert torch.equal(cache.prefill_selected, want.prefill_selected)
    assert torch.equal(cache.k_codes, want.k_codes)


def test_workspace_that_grows_on_a_side_stream():
    import torch
    cfg = KC.make_config(1, 1, 2, 2, 4096, residual=32)
    k, v = rows(4100, batch=1)
    cache = KC.KVCache(cfg)
    cache.prefill(0, k, v)
    q = torch.randn(1, 8, 2, 128, device="cuda").half()
    want = cache.clone().decode_multi(0, q)
    need = KC.B.kvq_decode_workspace_bytes(cfg, 8)
    assert cache.workspace.numel() < need
    side = torch.cuda.Stream()
    stale = torch.full((need,), 0x55, dtype=torch.uint8, device="cuda")     # what freed memory may hold
    torch.cuda.synchronize()
    del stale
    torch.cuda._sleep(BUSY)
    out = torch.empty_like(q)
    cache.decode_multi(0, q, out, stream=side)
    torch.cuda.synchronize()
    assert torch.equal(out, want)


def test_rotated_rows_of_a_step_are_not_reused_on_another_stream(monkeypatch):
    """The two rows that a step rotates ahead of its launches are given back when it returns, while the side stream may
    not have come to them yet: only that stream's next allocations may get their memory."""
    import torch
    cfg = KC.make_config(1, 1, 2, 2, 256, residual=32)
    k, v = rows(63, batch=1)                                  # the next token fills the ring
    cache = KC.KVCache(cfg)
    cache.prefill(0, k, v)
    k_new, v_new, q = (torch.randn(1, 2, 128, device="cuda").half() for _ in range(3))
    a = torch.arange(64, device="cuda") / 64.0
    rope = torch.cat([a.cos(), a.sin()]).float()
    want = cache.clone().step(0, k_new, v_new, q, rope=rope)
    used, rotate = [], KC.B.kvq_rope_rotate

    def noted(cfg, x, heads, rope, stride, out, stream=None):
        used.append(out.data_ptr())
        rotate(cfg, x, heads, rope, stride, out, stream)

    monkeypatch.setattr(KC.B, "kvq_rope_rotate", noted)
    side = torch.cuda.Stream()
    out = torch.empty_like(q)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(BUSY)
    cache.step(0, k_new, v_new, q, out, stream=side, rope=rope)
    later = [torch.full_like(q, 7.0) for _ in range(8)]
    assert len(used) == 2 and not set(used) & {t.data_ptr() for t in later}
    torch.cuda.synchronize()
    assert torch.equal(out, want)
