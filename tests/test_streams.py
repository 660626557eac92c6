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


def ragged(layers=1, batch=2, heads=2, capacity=256, residual=32):
    return KC.RaggedKVCache(KC.make_config(layers, batch, 2 * heads, heads, capacity, residual=residual))


def contents(cache):
    return {x: getattr(cache, x).clone() for x in ("k_codes", "k_meta", "v_codes", "v_meta", "mask", "k_res", "v_res", "pool_k",
                                                   "pool_v", "pool_idx", "pool_score", "pool_count", "aux_count", "seq_state")}


def on_streams(form, stream):
    """Where the calls go: `stream` handed over as an object or as a handle, or made the current one."""
    import contextlib
    import torch
    if form < 2:
        return contextlib.nullcontext(), dict(stream=handles(stream)[form])
    return torch.cuda.stream(stream), {}


@pytest.mark.parametrize("first,second", [(0, 0), (1, 1), (2, 2), (2, 0), (1, 2)])
def test_prompts_that_join_on_two_streams_share_the_flags(first, second):
    """Two long prompts of 24 layers into two slots, and a third into the first one's slot behind a stream that is
    busy: the same bytes as on one stream."""
    import torch
    layers, n = 24, 2083
    prompts = [([], []), ([], []), ([], [])]
    for i, (k, v) in enumerate(prompts):
        for l in range(layers):
            a, b = rows(n - 500 * i, heads=4, seed=100 * i + l)
            k.append(a)
            v.append(b)
    want = ragged(layers, heads=4, capacity=2048)
    for slot, (k, v) in zip((0, 1, 0), prompts):
        want.prefill_sequence(slot, k, v)
        torch.cuda.synchronize()
    cache = ragged(layers, heads=4, capacity=2048)
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    for (slot, busy, form), (k, v), s in zip(((0, False, first), (1, True, second), (0, False, first)), prompts, streams):
        if busy:
            with torch.cuda.stream(s):
                torch.cuda._sleep(BUSY)
        context, where = on_streams(form, s)
        with context:
            cache.prefill_sequence(slot, k, v, **where)
    torch.cuda.synchronize()
    a, b = contents(cache), contents(want)
    for x in a:
        assert torch.equal(a[x], b[x]), x


@pytest.mark.parametrize("form", [0, 1, 2])
@pytest.mark.parametrize("then", [0, 1, 2])
def test_steps_on_another_stream_come_behind_a_prompt(form, then):
    import torch
    k, v = rows(300)
    q, kn, vn = (torch.randn(2, h, 128, device="cuda").half() for h in (4, 2, 2))
    outs = []
    for busy in (False, True):
        cache = ragged()
        cache.prefill_sequence(0, [k[:, :200].contiguous()], [v[:, :200].contiguous()])
        side, other = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        if busy:
            with torch.cuda.stream(side):
                torch.cuda._sleep(BUSY)
        context, where = on_streams(form if busy else 0, side)
        with context:
            cache.prefill_sequence(1, [k], [v], **where)
        if not busy:
            torch.cuda.synchronize()
        context, where = on_streams(then, other)
        with context:
            cache.append(0, kn, vn, **where)
            cache.advance(**where)
            cache.make_plan(**where)
            out = [torch.full_like(q, float("nan")) for _ in range(2)]
            cache.decode(0, q, out[0], planned=True, **where)
            cache.decode(0, q, out[1], **where)
        torch.cuda.synchronize()
        outs.append({"planned": out[0], "ragged": out[1], **contents(cache)})
    for x in outs[0]:
        assert torch.equal(outs[0][x], outs[1][x]), x


@pytest.mark.parametrize("form", [0, 1])
def test_calls_on_the_current_stream_come_behind_a_prompt_on_a_side_stream(form):
    import torch
    k, v = rows(300)
    cache = ragged()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(BUSY)
    cache.prefill_sequence(1, [k], [v], stream=handles(side)[form])
    cache.set_active([True, False])
    twin = cache.clone()
    torch.cuda.synchronize()
    assert cache.seq_state.tolist() == [[0, 0, 0, 1], [256, 0, 44, 0]]
    assert torch.equal(twin.k_codes, cache.k_codes) and int(twin.k_codes.sum()) > 0


def test_a_stream_handed_over_may_go_before_the_rows():
    """Nothing of a stream given by its handle is touched once its work is done."""
    import ctypes
    import torch
    torch.cuda.synchronize()
    hip = KC.B.load_library()                                # (the runtime that it is linked with)
    handle = ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(handle), 1) == 0     # (1: not ordered with the default stream)
    k, v = rows(300)
    want, cache = ragged(), ragged()
    want.prefill_sequence(1, [k], [v])
    torch.cuda.synchronize()
    kk, vv = k.clone(), v.clone()
    torch.cuda.synchronize()
    cache.prefill_sequence(1, [kk], [vv], stream=handle.value)
    assert hip.hipStreamSynchronize(handle) == 0 and hip.hipStreamDestroy(handle) == 0
    del kk, vv
    later = [torch.full_like(k, 7.0) for _ in range(4)]
    out = cache.decode(0, torch.randn(2, 4, 128, device="cuda").half())
    torch.cuda.synchronize()
    assert torch.isfinite(out[1]).all() and not cache._held
    a, b = contents(cache), contents(want)
    for x in a:
        assert torch.equal(a[x], b[x]), x
    del later


def test_rows_of_another_stream_are_kept_for_the_current_one():
    import torch
    k, v = rows(300)
    want, cache = ragged(), ragged()
    want.prefill_sequence(1, [k], [v])
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        kk, vv = k.clone(), v.clone()
    torch.cuda.synchronize()
    torch.cuda._sleep(BUSY)
    cache.prefill_sequence(1, [kk], [vv])
    del kk, vv
    with torch.cuda.stream(side):
        later = [torch.full_like(k, 7.0) for _ in range(8)]
    torch.cuda.synchronize()
    a, b = contents(cache), contents(want)
    for x in a:
        assert torch.equal(a[x], b[x]), x
    del later


def test_a_prompt_under_capture_after_prompts_on_other_streams():
    """A captured prompt waits for and leaves nothing outside of its graph; replays equal the eager call."""
    import torch
    k, v = rows(300)
    k2, v2 = rows(300, seed=2)
    cache, want = ragged(), ragged()
    side = torch.cuda.Stream()
    cache.prefill_sequence(0, [k2], [v2])
    cache.prefill_sequence(0, [k], [v], stream=side)
    want.prefill_sequence(0, [k2], [v2])                     # (pool slots beyond the counts keep what was there before)
    want.prefill_sequence(0, [k], [v])
    torch.cuda.synchronize()
    kk, vv = k2.clone(), v2.clone()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cache.prefill_sequence(1, [kk], [vv])
    for source in ((k2, v2), (k, v), (k2, v2)):
        kk.copy_(source[0])
        vv.copy_(source[1])
        want.prefill_sequence(1, [source[0]], [source[1]])
        cache.prefill_sequence(0, [k], [v], stream=side)
        torch.cuda.current_stream().wait_stream(side)
        graph.replay()
        torch.cuda.synchronize()
        a, b = contents(cache), contents(want)
        for x in a:
            assert torch.equal(a[x], b[x]), x
