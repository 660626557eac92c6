"""Which tokens of a prompt are selected when all groups compete at once: flags, pools, counts and the stop
rule against the oracle's group-by-group competition, at the places where the split of the work can go wrong."""
import numpy as np
import pytest

from oracle import kvq_oracle as O

pytestmark = pytest.mark.gpu


def keys(pattern, n, rng):
    """fp16 [n, 128] Key rows."""
    x = rng.standard_normal((n, 128))
    t = np.arange(n)[:, None]
    if pattern == "falling":                     # every token beats all before it: the first groups fill the pools
        x *= np.linspace(40.0, 1.0, n)[:, None]
    elif pattern == "rising":
        x *= np.linspace(1.0, 40.0, n)[:, None]
    elif pattern == "equal":                     # the token index decides everywhere
        x = np.repeat(rng.standard_normal((1, 128)), n, 0)
    elif pattern == "late":                      # the second half lies far below the first: every one of its tokens
        x *= np.where(t < n // 2, 1.0, 0.01)     # is let through the first look
    elif pattern == "saw":                       # falls inside every stretch of 200 tokens
        x *= 1.0 + (199 - t % 200) / 50.0
    elif pattern == "teeth":                     # falls inside every segment of 1024 tokens, all above the first one:
        x *= np.where(t < 1024, 1.0, 40.0 - (t % 1024) / 50.0)   # thousands are let through, few are selected
    return x.astype(np.float16)


def check_selection(K, V, G, N, A, units=None):
    """Flags, pools (slot by slot), counts and the stop flag of prompts K, V (fp16 [heads, n, 128], all quantized).
    `units`: that many units in the call, the prompts given taken in turn."""
    import torch
    from paper_2505_10938_amd import cache as KC
    heads, n, _ = K.shape
    units = units or heads
    of = torch.arange(units) % heads
    cache = KC.KVCache(KC.make_config(1, 1, units, units, n, 2, G, 128, 0, N, A))
    cache.prefill(0, torch.from_numpy(K).cuda()[of][None], torch.from_numpy(V).cuda()[of][None])
    torch.cuda.synchronize()
    flags = cache.prefill_selected.cpu().numpy().reshape(-1)[:units * n].reshape(units, n)
    slots = N + A
    idx = cache.pool_idx.view(torch.int32).cpu().numpy()[:units * slots].reshape(units, slots)
    score = cache.pool_score.view(torch.float64).cpu().numpy()[:units * slots].reshape(units, slots)
    pk = cache.pool_k.view(torch.float16).cpu().numpy()[:units * slots * 128].reshape(units, slots, 128)
    pv = cache.pool_v.view(torch.float16).cpu().numpy()[:units * slots * 128].reshape(units, slots, 128)
    counts = [t.view(torch.int32).cpu().numpy()[:units] for t in (cache.pool_count, cache.aux_count, cache.frozen)]
    for h in range(heads):
        st = O.UnitState(128, 2, G, 128, N, A)
        want, fallen = [], []
        for i in range(0, n, G):
            had = {x["idx"] for x in st.aux}
            want.append(st.trace(K[h, i:i + G], V[h, i:i + G], i // G))
            fallen += sorted((x for x in st.aux if x["idx"] not in had), key=lambda x: (-x["score"], -x["idx"]))
        want = np.concatenate(want).astype(np.uint8)
        scores = O.l1_scores(K[h])
        # the pool ascending by (score, index); what has fallen out by group, inside a group the largest key first
        ranked = sorted(st.pool, key=lambda x: (x["score"], x["idx"]))
        for u in range(h, units, heads):
            assert np.array_equal(flags[u], want)
            assert [c[u] for c in counts] == [len(st.pool), len(st.aux), int(st.frozen)]
            for at, members in ((0, ranked), (N, fallen)):
                m = len(members)
                assert list(idx[u, at:at + m]) == [x["idx"] for x in members]
                rows = idx[u, at:at + m]
                assert np.array_equal(score[u, at:at + m], scores[rows])
                assert np.array_equal(pk[u, at:at + m].view(np.uint16), K[h][rows].view(np.uint16))
                assert np.array_equal(pv[u, at:at + m].view(np.uint16), V[h][rows].view(np.uint16))


PATTERNS = ["noise", "falling", "rising", "equal", "late", "saw", "teeth"]


@pytest.mark.parametrize("pattern", PATTERNS)
@pytest.mark.parametrize("G,N,A,n", [
    (32, 8, 32, 1024), (32, 8, 32, 1056), (128, 64, 64, 1024 + 128), (64, 1, 0, 2048), (32, 64, 64, 8192 + 32),
    (128, 3, 64, 8192 + 1024 + 128), (32, 8, 64, 32), (32, 33, 7, 96), (32, 8, 32, 20480),
])
def test_selection_of_a_prompt_equals_the_group_by_group_competition(G, N, A, n, pattern):
    rng = np.random.default_rng(n + N)
    K = np.stack([keys(pattern, n, rng) for _ in range(2)])
    check_selection(K, rng.standard_normal((2, n, 128)).astype(np.float16), G, N, A)


@pytest.mark.parametrize("units,G,N,A,n", [
    # a workgroup per unit and segment, then one per unit
    (100, 64, 8, 32, 5120 + 64), (60, 32, 3, 64, 9216 + 32), (30, 128, 8, 64, 2048 + 128),
    # one workgroup of 1024 threads per unit: few units that stop early, as many as there are compute units
    (7, 32, 32, 16, 4096 + 32), (14, 128, 64, 0, 1024 + 128), (256, 32, 8, 16, 1024 + 32), (250, 128, 32, 32, 2048 + 128),
    # 512 threads
    (257, 32, 8, 16, 512 + 32), (257, 64, 8, 64, 2048 + 64), (300, 32, 1, 0, 2080), (513, 32, 8, 64, 4096 + 32),
    (515, 128, 64, 64, 1024 + 128),
    # 256 threads
    (513, 32, 8, 32, 32), (513, 32, 8, 32, 160), (600, 64, 3, 32, 256), (1030, 32, 64, 64, 224), (520, 128, 32, 32, 128),
    (520, 32, 0, 8, 64),
])
def test_selection_in_calls_of_many_units(units, G, N, A, n):
    rng = np.random.default_rng(n + N)
    K = np.stack([keys(p, n, rng) for p in PATTERNS])
    check_selection(K, rng.standard_normal((len(PATTERNS), n, 128)).astype(np.float16), G, N, A, units)


@pytest.mark.parametrize("units,n", [
    (2, 992), (2, 1024), (256, 2048), (256, 2016), (300, 512), (300, 1056), (600, 256),   # 1024, 512, 256 threads
    (2, 2048), (2, 1024 + 480),                                                           # candidates first
    (2, 32), (2, 512), (2, 544), (256, 1024 + 512), (256, 1024 + 544),                    # eight rows per team, and more
    (300, 256), (300, 288), (300, 512 + 256), (600, 128), (600, 160),
])
def test_scores_are_told_apart_by_their_last_bit(units, n):
    """Rows of 64 times the largest fp16 value that differ by one subnormal, 2^-24 to 2^-13, in one channel or another:
    sums of 47 bits, of which the last ones decide."""
    rng = np.random.default_rng(n)
    K = np.zeros((2, n, 128), np.float16)
    K[:, :, ::2] = 65504.0
    K[:, :, ::4] *= -1
    t = np.arange(n)
    for h in range(2):
        K[h, t, (37 * t + h) % 64 * 2 + 1] = (rng.permutation(n) * 2.0 ** -24).astype(np.float16)
    check_selection(K, rng.standard_normal(K.shape).astype(np.float16), 32, 8, 32, units)


def plateau_keys(G, n, low, lower):
    """Keys whose L1 norms are set one by one (128 equal channels): everything at 8 but for the tokens given.  The
    first 1024 tokens hold 640 of norm 1 and the next 384 are of norm 1, so that the 1025th token that may be selected
    is in the middle of the group that starts at token 1408: `low` and `lower` are the offsets, inside the group 8192
    tokens after that one, of eight tokens of norm 1/2 each and of eight of norm 1/4."""
    norm = np.full(n, 8.0)
    norm[:640] = 1.0
    norm[1024:1408] = 1.0
    norm[1408 + G // 2 + 4:1408 + G] = 1.0
    for s in range(2048, n, 1024):               # the other segments: few that may be selected
        norm[s:s + 8] = 1.0
    at = 1408 + 8192
    norm[at + low:at + low + 8] = 0.5
    norm[at + lower:at + lower + 8] = 0.25
    return np.repeat((norm / 128.0)[:, None], 128, 1).astype(np.float16)


@pytest.mark.parametrize("N", [15, 16, 17])
@pytest.mark.parametrize("n", [32, 96, 1056, 4096])
def test_first_look_of_few_and_of_many_members(N, n):
    """Up to 16 members the first look bisects over the lanes' smallest entries, with more over all."""
    rng = np.random.default_rng(n + N)
    K = np.stack([keys(pattern, n, rng) for pattern in PATTERNS])
    check_selection(K, rng.standard_normal(K.shape).astype(np.float16), 32, N, 64)


def rows_around(c):
    """Rows A and B (fp16 [128]) with L1 norms a little below c, A's the smaller one.  Summed up in fp32, channel by channel,
    A's is c and B's the number below it.  (u: the distance of fp32 numbers below c.)"""
    u = float(c - np.nextafter(np.float32(c), np.float32(0)))
    a, b = np.zeros((2, 128), np.float16)
    a[[0, 2, 4, 6]] = c - 2 ** 13 * u, 2 ** 12 * u, 2 ** 12 * u - 2 ** 9 * u, 2 ** 9 * u - u / 4
    b[[0, 2, 4, 6]] = c - 2 ** 13 * u, 2 ** 12 * u, 2 ** 11 * u, 2 ** 11 * u - u
    b[[1, 8]] = 0.49 * u
    return a, b


# Groups, members, tokens: with few units and this many auxiliary places the candidates are looked for first.
AROUND = [(32, 3, 2048), (32, 8, 2048), (32, 8, 4096 + 96), (64, 16, 3072), (32, 17, 2048 + 64), (128, 40, 2048 + 256)]


def rows_around_bounds(G, N, n):
    """Keys fp16 [units, n, 128], one unit per c, a number whose last 15 bits are zero: there the first look's scores change.
    Each stretch of 1024 tokens begins with N rows B, which make its bounds, and has a row A a group or two later; the
    norm of all others is 4 c."""
    c = np.array([256.0, 384.0, 448.0, 1028.0, 2560.0, 32768.0])
    K = np.repeat(np.repeat(c[:, None, None] / 32, n, 1), 128, 2).astype(np.float16)
    at = G * -(-N // G) + 8
    for h, x in enumerate(c):
        a, b = rows_around(x)
        for t in range(0, n, 1024):
            K[h, t:t + N] = b
            K[h, t + at] = a
    return c, K, at


@pytest.mark.parametrize("G,N,n", AROUND)
def test_first_look_allows_for_the_rounding_of_its_sums(G, N, n):
    """The candidates' scores are fp32 sums.  A row that has to be selected is above the bound by those, below it exactly."""
    _, K, at = rows_around_bounds(G, N, n)
    check_selection(K, np.random.default_rng(n + N).standard_normal(K.shape).astype(np.float16), G, N, 64)


@pytest.mark.parametrize("G", [32, 64, 128])
@pytest.mark.parametrize("A", [8, 32])
@pytest.mark.parametrize("n", [10240, 12288])
def test_a_group_competes_as_a_whole_wherever_the_prompt_is_cut(G, A, n):
    """Tokens of one group of which the later ones displace the earlier ones, around the place where 8192 tokens
    counted from the middle of a group would end.  Taken in two parts the earlier ones would be selected as well,
    and with A = 8 tracing would stop."""
    K = np.stack([plateau_keys(G, n, G // 2 - 8, G // 2 + 4), plateau_keys(G, n, G // 2 + 4, G // 2 - 8)])
    check_selection(K, np.random.default_rng(G + A).standard_normal(K.shape).astype(np.float16), G, 8, A)


@pytest.mark.parametrize("bits,G,Gv,batch", [
    (bits, G, Gv, batch) for bits, G, Gv, batches in [(2, 32, 32, (15, 16, 17)), (4, 32, 64, (15, 16, 17)), (2, 64, 128, (1, 2, 3)),
                                                      (4, 64, 32, (1, 2, 3)), (2, 32, 32, (48, 49)), (4, 32, 64, (49,)), (2, 64, 128, (49,))]
    for batch in batches])
def test_many_prompts_in_one_call_equal_each_on_its_own(bits, G, Gv, batch):
    """16 groups per sequence.  240, 256 and 272 groups of 32 tokens, 16, 32 and 48 of 64 in one call, on both sides of where
    the quantization changes kernels, against the same prompts one sequence at a time (16 groups per call)."""
    import torch
    from paper_2505_10938_amd import cache as KC
    heads, groups, R = 4, 4, 32
    n = groups * G + R + 5
    gen = torch.Generator(device="cuda")
    gen.manual_seed(batch)
    K, V = (torch.randn(batch, heads, n, 128, generator=gen, device="cuda").half() for _ in range(2))
    K[:, :, ::7] *= 0.05
    cfg = KC.make_config(1, batch, heads, heads, groups * G, bits, G, Gv, R, 3, 32)
    a, b = KC.KVCache(cfg), KC.RaggedKVCache(cfg)
    a.prefill(0, K, V)
    for i in range(batch):
        b.prefill_sequence(i, [K[i]], [V[i]])
    for name in ("k_codes", "k_meta", "v_codes", "v_meta", "mask", "k_res", "v_res", "pool_idx", "pool_count", "aux_count"):
        assert torch.equal(getattr(a, name), getattr(b, name)), name
