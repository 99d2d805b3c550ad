"""The attention planner's rules and item accounting on the host (no GPU).

The chunk: the shortest (a multiple of 128 keys, at least 256, at most one
CU's share of all keys) whose work items fit in two rounds of 256, or, when
even the longest allowed chunk gives more, that chunk.  Then what a call
launches: the keys of a work item, narrow or full work groups, and two
branched plans joined in one launch."""
import ctypes

import numpy as np
import pytest

from paper_2609_34388_amd import binding
from paper_2609_34388_amd import workloads as W
from tests.test_abi import _L, _plan

CUS, ROUND2 = 256, 512


def _items(lay, chunk, g, hkv):
    n = 0
    for r in range(lay.num_requests):
        q, T = int(lay.q_len[r]), int(lay.kv_len[r])
        if q == 0:
            continue
        n += -(-(q * g) // 256) * -(-T // chunk)
    return n * hkv


@pytest.mark.parametrize("spec,seed,nreq", [
    ("tiny", 0, None), ("low", 0, None), ("low", 1, 3),
    ("mid", 0, None), ("mid", 5, None), ("mid", 12, None), ("mid", 1, 4), ("mid", 2, 8), ("mid", 3, 32),
    ("high", 0, None), ("high", 1, 16), ("high", 2, 80),
    ("long", 0, None), ("long", 1, 8), ("long", 2, 24),
])
def test_chunk_is_shortest_fitting_two_rounds(spec, seed, nreq):
    lay = W.make_layout(spec, seed=seed, num_requests=nreq) if nreq else W.make_layout(spec, seed=seed)
    s = lay.spec
    g, hkv = s.num_q_heads // s.num_kv_heads, s.num_kv_heads
    l = _L(R=lay.num_requests, hq=s.num_q_heads, hkv=hkv, D=s.head_dim, num_pages=lay.num_pages,
           ctx=lay.ctx_len, nv=lay.n_verify, n=lay.q_len, pages=np.diff(lay.page_indptr))
    info = _plan(l)
    chunk = info.chunk_keys
    assert info.work_items == _items(lay, chunk, g, hkv)
    up = lambda x: -(-x // 128) * 128
    groups = [(int(lay.kv_len[r]), -(-int(lay.q_len[r]) * g // 256)) for r in range(lay.num_requests)
              if lay.q_len[r] > 0]
    total = sum(T * c for T, c in groups) * hkv
    whole = max(256, up(max(T for T, _ in groups)))
    hi = min(whole, max(256, up(total // CUS)))
    if _items(lay, hi, g, hkv) > ROUND2:
        assert chunk == hi
    elif _items(lay, 256, g, hkv) <= ROUND2:
        assert chunk == 256
    else:
        assert 256 < chunk <= hi and chunk % 128 == 0
        assert _items(lay, chunk, g, hkv) <= ROUND2 < _items(lay, chunk - 128, g, hkv)


@pytest.mark.parametrize("floor", [256, 65536, 65664, 131072, 2**31 - 1])
def test_chunk_never_exceeds_the_longest_item(monkeypatch, floor):
    """RG_ATTN_MIN_CHUNK raises the shortest chunk up to 65536 keys, the most a
    work item takes: the workspace then holds the partials of items that long."""
    monkeypatch.setenv("RG_ATTN_MIN_CHUNK", str(floor))
    R, ctx, n, hq, hkv = 16, 200000, 32, 32, 8
    pages = -(-(ctx + n) // 16)
    l = _L(R=R, hq=hq, hkv=hkv, D=128, num_pages=pages * R, ctx=[ctx] * R, nv=[16] * R, n=[n] * R,
           pages=[pages] * R)
    info = _plan(l)
    chunk = info.chunk_keys
    assert chunk % 128 == 0 and 256 <= chunk <= 65536
    need = R * hkv * -(-(ctx + n) // 65536) * n * (hq // hkv)  # partial columns at the longest item
    assert info.partial_columns >= need
    assert info.workspace_bytes >= need * (128 * 2 + 8)


def _batch(ctx, n, nv=None, hq=32, hkv=8, D=128):
    return _L(R=len(ctx), hq=hq, hkv=hkv, D=D, num_pages=1 << 20, ctx=ctx, nv=nv if nv is not None else [0] * len(ctx),
              n=n)


def _launches(l, branches=None):
    info = binding.AttnLaunchInfo()
    st = binding.library().rg_attention_launches(ctypes.byref(l.c), ctypes.byref(branches.c) if branches else None,
                                                 ctypes.byref(info))
    assert st == 0
    return info


def test_launch_query_validation():
    lib, info = binding.library(), binding.AttnLaunchInfo()
    l = _batch([40, 17], [7, 5], [3, 0])
    assert lib.rg_attention_launches(ctypes.byref(l.c), None, None) == 1
    assert lib.rg_attention_launches(None, None, ctypes.byref(info)) == 1
    bad = binding.make_branches([0, 1, 2], [3, 0], [0, 0], [9, 5])  # rows past the request's
    assert lib.rg_attention_launches(ctypes.byref(l.c), ctypes.byref(bad.c), ctypes.byref(info)) == 2


def _random_batch(seed, max_req):
    rng = np.random.default_rng(seed)
    R = int(rng.integers(1, max_req))
    ctx_max = int(2 ** rng.uniform(5, 16 if R < 40 else 13))
    g = int(rng.choice([1, 2, 4, 8]))
    hkv = int(rng.choice([1, 2, 3, 8]))
    ctx = rng.integers(0, ctx_max, R)
    n = rng.choice([[1, 2, 4], [4, 8, 16, 32], [0, 1, 7, 70]][int(rng.integers(3))], R)
    n[0] = max(1, n[0])
    return ctx, n, g, hkv, int(rng.choice([64, 128]))


@pytest.mark.parametrize("env", [{}, {"RG_ATTN_MIN_CHUNK": "128"}, {"RG_ATTN_MIN_CHUNK": "1024"},
                                 {"RG_ATTN_CHUNK": "384"}, {"RG_ATTN_PERSIST": "1"}])
def test_launches_stay_within_the_workspace(monkeypatch, env):
    """Random batches: a work item is no shorter than the chunk, and the items,
    split requests and partials of the launches follow from its length and fit
    the workspace that the chunk sizes."""
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    for seed in range(150):
        ctx, n, g, hkv, D = _random_batch(seed, 300)
        l = _batch(ctx, n, hq=g * hkv, hkv=hkv, D=D)
        plan, run = _plan(l), _launches(l)
        assert run.run_keys >= plan.chunk_keys and run.run_keys % 128 == 0 and run.run_keys <= 65536
        if "RG_ATTN_CHUNK" in env or "RG_ATTN_PERSIST" in env:
            assert run.run_keys == plan.chunk_keys
        items = split = part = 0
        for c, k in zip(ctx, n):
            if k == 0:
                continue
            nch, M = -(-int(c + k) // run.run_keys), int(k) * g
            items += hkv * -(-M // 256) * nch
            if nch > 1:
                split += 1
                part += hkv * nch * -(-M // 32) * 32
        assert (run.work_items, run.split_requests, run.partial_columns) == (items, split, part)
        assert run.partial_columns <= plan.partial_columns
        words = 4 * plan.sync_words
        assert run.max_launch_partial_columns * (2 * D + 8) <= max(0, plan.workspace_bytes - words)
        if run.narrow:
            assert max(int(k) * g for k in n) <= 128
        if "RG_ATTN_PERSIST" in env:
            assert run.merge_launches == 0
        else:
            assert (run.merge_launches > 0) == (split > 0)


def _run_rule(pairs, hkv, cus, chunk):
    """Keys per work item: the shortest whose items fit one round of `cus`,
    where whole requests do, unless its longest item exceeds 1.35 mean loads
    plus 512 keys; whole where that adds at most 192 keys."""
    longest = max(T for T, _, _ in pairs)
    if len(pairs) * hkv > cus or longest <= chunk:
        return chunk
    run = chunk
    while sum(-(-T // run) for T, _, _ in pairs) * hkv > cus:
        run += 128
    load = sum(T * w for T, _, w in pairs)
    if max(min(run, T) * w for T, _, w in pairs) > 1.35 * load * hkv / cus + 512:
        return chunk
    if max((T - run) * w for T, _, w in pairs) <= 192:
        run = -(-longest // 128) * 128
    return max(chunk, min(65536, run))


def _narrow_rule(pairs, hkv, cus, D, run):
    one_round = sum(-(-T // run) for T, _, _ in pairs) * hkv <= cus
    tiles = max(t for _, t, _ in pairs)
    if tiles > 4:
        return False
    if D == 64:
        return not one_round or run <= 512
    return run <= (2432 if tiles <= 2 else 256 if one_round else 512)


def test_runs_and_work_groups_follow_the_rules():
    narrow = longer = 0
    for seed in range(1000, 1300):
        ctx, n, g, hkv, D = _random_batch(seed, 120)
        pairs = []
        for c, k in zip(ctx, n):
            groups, tiles = -(-int(k) * g // 256), -(-int(k) * g // 32)
            tiles = -(-tiles // max(1, groups))
            pairs += [(int(c + k), 8 if groups > 1 else tiles, max(1.0, tiles / 4))] * groups
        l = _batch(ctx, n, hq=g * hkv, hkv=hkv, D=D)
        chunk, got = _plan(l).chunk_keys, _launches(l)
        run = _run_rule(pairs, hkv, CUS, chunk)
        want_narrow = _narrow_rule(pairs, hkv, CUS, D, run)
        if want_narrow and run == chunk:
            run = _run_rule(pairs, hkv, ROUND2, chunk)
        assert (got.run_keys, bool(got.narrow)) == (run, want_narrow), seed
        narrow += want_narrow
        longer += run > chunk
    assert 30 < narrow < 270 and longer > 30  # both sides of both rules are among the batches


def _branched(R, D=128, hq=32, hkv=8, ctx=100, special=None):
    """R requests of one 2-row branch each; request 7 lists `special` instead:
    (verify rows, branches)."""
    ctx, nv = [ctx] * R, [2] * R
    br = [[(1, 0, 2)] for _ in range(R)]
    if special is not None:
        nv[7], br[7] = special
    n = [v + sum(b[2] for b in bs) for v, bs in zip(nv, br)]
    flat = [b for bs in br for b in bs]
    B = binding.make_branches(np.concatenate([[0], np.cumsum([len(bs) for bs in br])]),
                              *([b[i] for b in flat] for i in range(3)))
    return _batch(ctx, n, nv, hq=hq, hkv=hkv, D=D), B


@pytest.mark.parametrize("D", [64, 128])
def test_two_branched_plans_join_in_one_launch(D):
    for R, launches, joined in ((64, 1, 0), (65, 1, 1), (128, 1, 1), (129, 2, 1), (192, 2, 1), (256, 2, 2)):
        got = _launches(*_branched(R, D))
        assert (got.launches, got.joined_launches, got.split_requests) == (launches, joined, 0), R
    split = _launches(*_branched(65, D, ctx=70000))  # split requests: no join
    assert (split.joined_launches, split.launches, split.merge_launches) == (0, 2, 2)
    l, _ = _branched(65, D)
    plain = _launches(l)  # without branches a plan holds 128 requests
    assert (plain.launches, plain.joined_launches) == (1, 0)


@pytest.mark.parametrize("fits,special", [
    (True, (1023, [(1023, 0, 2)])), (False, (1024, [(1024, 0, 2)])),                   # prefix
    (True, (2, [(1, 0, 1023)])), (False, (2, [(1, 0, 1024)])),                         # rows
    (True, (300, [(a, 0, 1) for a in range(255)])), (False, (300, [(a, 0, 1) for a in range(256)])),  # count
    (True, (512, [(0, 0, 1), (255, 0, 1)])), (False, (512, [(0, 0, 1), (256, 0, 1)])),  # prefix step
    (True, (4093, [(5, 0, 2)])), (False, (4094, [(5, 0, 2)])),                         # rows of the request
    (True, (2, [(1, 15, 16)])),                                                        # lead: any that is accepted
])
def test_packed_fields_at_their_limits(monkeypatch, fits, special):
    monkeypatch.setenv("RG_ATTN_CHUNK", "65536")  # whole requests
    got = _launches(*_branched(65, hq=1, hkv=1, special=special))
    assert (got.joined_launches, got.launches) == ((1, 1) if fits else (0, 2))


@pytest.mark.parametrize("rows,joined", [(16300, 1), (16500, 0)])
def test_query_rows_past_the_packed_field(monkeypatch, rows, joined):
    """The first 64 requests' rows put the others' first row below and past 2^20."""
    monkeypatch.setenv("RG_ATTN_CHUNK", "65536")  # whole requests
    R = 192
    n = [rows] * 64 + [2] * 128
    B = binding.make_branches(np.arange(R + 1), [0] * R, [0] * R, n)
    got = _launches(_batch([10] * R, n, hq=1, hkv=1), B)
    assert got.joined_launches == joined


@pytest.mark.parametrize("n,hkv,joined", [(1, 87376, 1), (1, 87400, 0), (130, 43688, 1), (130, 43700, 0)])
def test_joined_launch_holds_fewer_than_2_32_threads(n, hkv, joined):
    """128 requests of one item per KV head in narrow work groups of 384 threads
    and in full ones of 768: two launches where one would wrap its grid."""
    R = 128
    B = binding.make_branches(np.arange(R + 1), [0] * R, [0] * R, [n] * R)
    got = _launches(_batch([60] * R, [n] * R, hq=hkv, hkv=hkv, D=64), B)
    assert (got.joined_launches, got.launches, got.narrow) == (joined, 2 - joined, n == 1)


@pytest.mark.parametrize("n,hkv,status", [(1, 87376, 0), (1, 87400, 3), (130, 43688, 0), (130, 43700, 3)])
def test_launches_of_2_32_threads_are_refused(n, hkv, status):
    l = _batch([60] * 128, [n] * 128, hq=hkv, hkv=hkv, D=64)
    size = ctypes.c_size_t()
    assert binding.library().rg_draft_verify_attention_workspace(ctypes.byref(l.c), ctypes.byref(size)) == status


def test_workspace_size_does_not_depend_on_the_launch_mode(monkeypatch):
    """More than 128 requests fill several launches that share the workspace;
    one sized in either mode serves the other."""
    longer = 0
    for seed in [53, 126, 132, 150, *range(200, 300)]:
        rng = np.random.default_rng(seed)
        R = int(rng.integers(129, 257))
        base = int(rng.integers(300, 3000))
        ctx = rng.integers(base, base + int(2 ** rng.uniform(5, 10)), R)
        n = rng.choice([1, 16, 22], R, p=[0.4, 0.3, 0.3])  # one, four and six tiles of columns
        l = _batch(ctx, n, hq=8, hkv=1)
        B = binding.make_branches(np.arange(R + 1), [0] * R, [0] * R, n)
        size = {}
        for mode in ("1", "0"):
            monkeypatch.setenv("RG_ATTN_PERSIST", mode)
            branched = ctypes.c_size_t()
            assert binding.library().rg_multibranch_attention_workspace(ctypes.byref(l.c), ctypes.byref(B.c),
                                                                        ctypes.byref(branched)) == 0
            size[mode] = (_plan(l).workspace_bytes, branched.value)
        longer += _launches(l).run_keys > _plan(l).chunk_keys
        assert size["0"] == size["1"], seed
    assert longer > 20
