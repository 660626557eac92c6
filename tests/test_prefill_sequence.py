"""A sequence's prompt in all layers at once against the same layer by layer: every byte that it leaves."""
import ctypes as C

import pytest

import kvq_synth as S
import paper_2505_10938_amd as P
from paper_2505_10938_amd import binding as B, cache as KC
from tests import helpers as H

NAMES = ("k_codes", "k_meta", "v_codes", "v_meta", "mask", "k_res", "v_res", "pool_k", "pool_v", "pool_idx",
         "pool_score", "pool_count", "aux_count", "frozen")


def test_bad_arguments_rejected_before_launch():
    lib = P.load_library()
    c = KC.make_config(3, 2, 4, 4, 1024, residual=32)
    qc = B.kvq_qcache(256, 256, 256, 256, 256)
    pool = B.kvq_pool(256, 256, 256, 256, 256, 256, 256)
    res = B.kvq_residual(256, 256)
    three = lambda *p: (C.c_void_p * 3)(*p)

    def call(cfg=c, seq=0, k=three(256, 512, 768), v=three(256, 512, 768), n=300, stride=300 * 128, flags=256,
             room=4 * 256, state=256):
        return lib.kvq_prefill_sequence(C.byref(cfg), seq, k, v, stride, n, pool, flags, room, qc, res, state, 1, None)

    bad = B.KVQ_ERR_INVALID_ARG
    assert call(seq=-1) == bad and call(seq=2) == bad
    assert call(k=None) == bad and call(v=None) == bad
    assert call(k=three(256, None, 768)) == bad and call(v=three(256, 512, 776)) == bad
    assert call(n=0) == bad and call(n=1024 + 32 + 32) == bad and call(stride=299 * 128) == bad
    assert call(flags=None) == bad and call(state=264) == bad
    assert call(room=4 * 256 - 1) == B.KVQ_ERR_WORKSPACE     # 256 of the 300 tokens are quantized
    per_step = KC.make_config(3, 2, 4, 4, 1024, residual=32, outlier_budget=0, aux_capacity=0, value_per_step=1)
    assert call(cfg=per_step) == B.KVQ_ERR_UNSUPPORTED
    with pytest.raises(B.KvqError):
        B.kvq_prefill_sequence(c, 0, [256, 512], [256, 512], 300 * 128, 300, pool, 256, 4 * 256, qc, res, 256, 1)


# layers, tokens, layers that the flags have room for, untraced layers, paged, further settings
@pytest.mark.gpu
@pytest.mark.parametrize("layers,n,room,untraced,paged,kw", [
    (3, 700, 3, 0, False, {}),
    (5, 700, 2, 0, False, {}),                                       # two launches of two, one of one
    (34, 300, 34, 0, False, {}),                                     # more than a launch takes
    (4, 700, 4, 1, False, {}),                                       # one layer without a pool ahead of three with one
    (3, 127, 3, 0, False, {}),                                       # nothing is quantized yet
    (3, 128, 3, 0, True, {}),                                        # the shortest prompt with a group
    (2, 9001, 2, 0, True, {}),                                       # segments of workgroups of their own
    (3, 1300, 3, 0, True, dict(bits=4, group_k=64, group_v=64)),
    (3, 1300, 3, 0, False, dict(group_k=128, group_v=128, residual=0)),
    (3, 700, 3, 0, False, dict(outlier_budget=0)),
    (40, 1200, 40, 0, False, dict(outlier_budget=3, aux_capacity=0)),
])
def test_all_layers_at_once_equal_one_by_one(layers, n, room, untraced, paged, kw):
    import torch
    cfg = KC.make_config(layers, 2, 3, 3, 9216 if n > 9000 else 1408, **{**dict(residual=96), **kw},
                         untraced_layers=untraced)
    groups = cfg.max_seq // cfg.group_k
    gen = torch.Generator(device="cuda")
    gen.manual_seed(layers * n)
    new = lambda *s: torch.randn(s, generator=gen, device="cuda").half()
    k, v = ([new(3, n, 128) for _ in range(layers)] for _ in range(2))
    junk = {x: torch.randint(0, 256, (getattr(KC.KVCache(cfg), x).numel(),), generator=gen, device="cuda").byte()
            for x in ("k_res", "v_res", "pool_k", "pool_v", "pool_idx", "pool_score", "pool_count", "aux_count")}

    def cache():                                                     # whatever the slots held before
        c = KC.RaggedKVCache(cfg, n_pages=2 * groups if paged else None)
        if paged:
            c.page_table.copy_(torch.randperm(2 * groups, generator=torch.Generator().manual_seed(1)).view(2, groups))
        for x, t in junk.items():
            getattr(c, x).copy_(t)
        return c

    want, got = cache(), cache()
    nq = cfg.group_k * ((n - cfg.residual) // cfg.group_k) if n >= cfg.residual + cfg.group_k else 0
    flags = torch.zeros(2 * 3 * cfg.max_seq, dtype=torch.uint8, device="cuda")
    for layer in range(layers):
        B.kvq_prefill_quantize_seq(cfg, layer, 1, k[layer], v[layer], n * 128, n, want.pool, flags, want.qcache, want.res)
    if room == layers:
        got.prefill_sequence(1, k, v)
    else:
        B.kvq_prefill_sequence(cfg, 1, k, v, n * 128, n, got.pool, flags, room * 3 * nq, got.qcache, got.res,
                               got.seq_state, 1)
    torch.cuda.synchronize()
    for x in NAMES:
        assert torch.equal(getattr(got, x), getattr(want, x)), x
    assert got.seq_state.tolist() == [[0, 0, 0, 0], [nq, 0, n - nq, 1]]


@pytest.mark.gpu
def test_rows_given_back_before_a_side_stream_reads_them():
    import torch
    cfg = KC.make_config(2, 2, 2, 2, 256, residual=32)
    k, v = ([torch.randn(2, 300, 128, device="cuda").half() for _ in range(2)] for _ in range(2))
    want, got = KC.RaggedKVCache(cfg), KC.RaggedKVCache(cfg)
    want.prefill_sequence(1, k, v, active=False)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)                                # about 10 ms
    got.prefill_sequence(1, [t.clone() for t in k], [t.clone() for t in v], active=False, stream=side)
    later = [torch.full_like(k[0], 7.0) for _ in range(8)]
    torch.cuda.synchronize()
    del later
    for x in NAMES + ("seq_state",):
        assert torch.equal(getattr(got, x), getattr(want, x)), x


@pytest.mark.gpu
@pytest.mark.parametrize("bits,G,groups", [
    (2, 32, 127), (2, 32, 128), (4, 64, 64), (2, 128, 32),
    (2, 32, 47), (2, 32, 48), (4, 32, 48), (2, 64, 15), (2, 64, 16), (4, 64, 16), (2, 128, 23), (2, 128, 24), (4, 128, 16),
    (2, 32, 31), (2, 32, 32), (4, 32, 31), (4, 32, 32), (4, 64, 15), (2, 128, 7), (2, 128, 8), (4, 128, 7), (4, 128, 8),
])
def test_a_large_batch_equals_each_sequence_on_its_own(bits, G, groups):
    """128 units: from 4096 quantized tokens each (2^27 bytes of Keys) the quantization takes the last groups first, from
    1024 (2^25) its loads and stores leave the caches alone.  Each sequence on its own, 8 units, does neither, but goes
    through the same kernel: two units are compared with the oracle as well."""
    import torch
    n = groups * G + 43
    w = S.Workload("batch", 1, 16, 8, 8, n, bits, G, residual=43)
    cfg = KC.make_config(1, 16, 8, 8, groups * G, bits, G, residual=43)
    assert w.n_quant == groups * G
    gen = torch.Generator(device="cuda")
    gen.manual_seed(groups)
    k, v = (torch.randn(16, 8, n, 128, generator=gen, device="cuda").half() for _ in range(2))
    a, b = KC.KVCache(cfg), KC.RaggedKVCache(cfg)
    a.prefill(0, k, v)
    for i in range(16):
        b.prefill_sequence(i, [k[i]], [v[i]])
    torch.cuda.synchronize()
    for x in NAMES:
        assert torch.equal(getattr(a, x), getattr(b, x)), x
    units = [5, 126]
    H.compare_state(a, H.oracle_states(w, k.cpu().numpy(), v.cpu().numpy(), w.n_quant, units), w, w.n_quant, units=units)


@pytest.mark.gpu
def test_an_active_entry_means_that_the_rows_are_there():
    """Another stream looks at the entry and then at the codes, over and over while 32 layers of a prompt join: once
    it finds the sequence active, it finds all codes, mask words and ring rows."""
    import torch
    layers, n = 32, 4240
    cfg = KC.make_config(layers, 2, 8, 8, 4096)
    k, v = ([torch.randn(8, n, 128, device="cuda").half() for _ in range(layers)] for _ in range(2))
    cache = KC.RaggedKVCache(cfg)
    flags = torch.empty(layers * 8 * 4096, dtype=torch.uint8, device="cuda")
    watched = [getattr(cache, x).view(-1, 4)[::1024] for x in ("k_codes", "v_codes", "mask", "k_res", "v_res")]
    side = torch.cuda.Stream()

    def join():
        B.kvq_prefill_sequence(cfg, 1, k, v, n * 128, n, cache.pool, flags, flags.numel(), cache.qcache, cache.res,
                               cache.seq_state, 1, side)

    torch.cuda.synchronize()
    join()
    torch.cuda.synchronize()
    want = [t.clone() for t in watched]
    for x in ("k_codes", "v_codes", "mask", "k_res", "v_res", "seq_state"):
        getattr(cache, x).zero_()
    torch.cuda.synchronize()
    join()
    seen = []
    while not (seen and side.query()) and len(seen) < 1000:
        entry = cache.seq_state[1].clone()
        seen.append((entry, [t.clone() for t in watched]))
    torch.cuda.synchronize()
    assert cache.seq_state[1].tolist() == [4096, 0, 144, 1]
    for entry, got in seen:
        entry = entry.tolist()
        assert entry in ([0, 0, 0, 0], [4096, 0, 144, 1])
        if entry[3]:
            assert all(torch.equal(a, b) for a, b in zip(got, want))
