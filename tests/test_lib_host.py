"""Host-side parity of the native library (CPU only, no kernel launches).

The allocator and the planner of ``libflowkv.so`` run on the host; here they
are checked against the oracle on the same seeded inputs: identical block
lists from every allocator policy, identical runs from the planner, and every
error path of the C ABI forced from the host.
"""

import ctypes
import re
import os

import numpy as np
import pytest
from hypothesis import given, settings, strategies as st

import oracle
from paper_2504_03775_amd import flowkv as fk
from workloads import recipes

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "flowkv.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(flowkv_\w+)\s*\(", text)))


def test_inline_capacity_by_layouts_and_depth():
    """flowkv_inline_capacity: the compact forms' limits, host only."""
    def cap(s, d):
        n = ctypes.c_int64(-9)
        rc = fk.lib().flowkv_inline_capacity(ctypes.byref(s), ctypes.byref(d), ctypes.byref(n))
        return rc, n.value

    for L in (1, 2, fk.INLINE_LAYERS, fk.INLINE_LAYERS + 1, fk.MAX_LAYERS):
        lm = pool(layout=0, L=L, bases=tuple(range(1 << 20, (1 << 20) + L)))
        bm = pool(layout=1, L=L)
        few = L <= fk.INLINE_LAYERS
        want_lm = fk.INLINE_RUNS_LAYER_MAJOR if few else fk.INLINE_RUNS
        assert cap(bm, bm) == (fk.OK, fk.INLINE_RUNS_BLOCK_MAJOR), L
        assert cap(lm, bm) == (fk.OK, want_lm), L
        assert cap(bm, lm) == (fk.OK, want_lm), L
        assert cap(lm, lm) == (fk.OK, want_lm), L
    # the deeper pool decides
    assert cap(pool(layout=0, L=2, bases=(1, 2)), pool(layout=1, L=fk.INLINE_LAYERS + 1)) == \
        (fk.OK, fk.INLINE_RUNS)
    # errors leave the output alone
    for s in (pool(layout=7), pool(L=0), pool(L=fk.MAX_LAYERS + 1)):
        assert cap(s, pool()) == (fk.EINVAL, -9)
        assert cap(pool(), s) == (fk.EINVAL, -9)
    n = ctypes.c_int64()
    assert fk.lib().flowkv_inline_capacity(None, ctypes.byref(pool()), ctypes.byref(n)) == fk.EINVAL
    assert fk.lib().flowkv_inline_capacity(ctypes.byref(pool()), ctypes.byref(pool()), None) == \
        fk.EINVAL


def test_library_exports_every_declared_function():
    names = declared_functions()
    assert len(names) >= 12
    lib = ctypes.CDLL(fk.LIB_PATH)
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(fk.SIGNATURES)


def test_binding_constants_match_the_header():
    text = open(os.path.join(ROOT, "include", "flowkv.h")).read()
    defines = dict(re.findall(r"#define\s+(FLOWKV_\w+)\s+(-?\d+)", text))
    assert int(defines["FLOWKV_INLINE_RUNS"]) == fk.INLINE_RUNS
    assert int(defines["FLOWKV_INLINE_RUNS_BLOCK_MAJOR"]) == fk.INLINE_RUNS_BLOCK_MAJOR
    assert int(defines["FLOWKV_INLINE_LAYERS"]) == fk.INLINE_LAYERS
    assert int(defines["FLOWKV_INLINE_RUNS_LAYER_MAJOR"]) == fk.INLINE_RUNS_LAYER_MAJOR
    assert int(defines["FLOWKV_ATTN_SCRATCH_BYTES"]) == fk.ATTN_SCRATCH_BYTES
    assert int(defines["FLOWKV_ATTN_INLINE_LENS"]) == fk.ATTN_INLINE_LENS
    enums = dict(re.findall(r"\b(FLOWKV_E?\w+)\s*=\s*(-?\d+)", text))
    for name in ("OK", "EINVAL", "ENOSPC", "ERANGE", "EDUP", "ECAP", "EHIP", "ENOMEM"):
        assert int(enums["FLOWKV_" + name]) == getattr(fk, name), name


def test_attention_split_rule_and_workspace():
    """The default split: the smallest power of two from 256 to 1024 giving at
    most 512 (request, split) pairs; the workspace follows it."""
    cases = {(1, 13000): 256, (1, 200000): 512, (32, 20000): 1024, (16, 32000): 1024,
             (16, 8192): 256, (17, 8192): 512, (0, 5): 256, (3, 0): 256, (2000, 100): 1024}
    for (n, T), want in cases.items():
        got = fk.flowkv_decode_attention_split(n, T)
        assert got == want, (n, T, got)
        brute = next((s for s in (256, 512) if n * -(-T // s) <= 512), 1024)
        assert got == brute
        ws = fk.flowkv_decode_attention_workspace(n, 32, 128, T)
        assert ws == n * 32 * -(-T // got) * 130 * 4
    assert fk.flowkv_decode_attention_workspace(2, 8, 64, 1000, 100) == 2 * 8 * 10 * 66 * 4
    for bad in ((-1, 5), (1, -5)):
        with pytest.raises(fk.FlowKVError):
            fk.flowkv_decode_attention_split(*bad)
    with pytest.raises(fk.FlowKVError):
        fk.flowkv_decode_attention_workspace(1, 8, 128, 100, 1025)


def test_strerror_names_every_code():
    for c in (fk.OK, fk.EINVAL, fk.ENOSPC, fk.ERANGE, fk.EDUP, fk.ECAP, fk.EHIP, fk.ENOMEM):
        assert fk.strerror(c) and fk.strerror(c) != "unknown status code"
    assert fk.strerror(12345) == "unknown status code"


# ---- allocator ---------------------------------------------------------------

def both(P, policy, seed=0):
    return fk.Allocator(P, policy, seed), oracle.RefAllocator(P, policy, seed)


@pytest.mark.parametrize("policy", [0, 1, 2])
@settings(max_examples=80, deadline=None)
@given(seed=st.integers(0, 2**63 - 1))
def test_allocator_matches_oracle_on_random_streams(policy, seed):
    g = np.random.default_rng(seed)
    P = int(g.integers(1, 300))
    a, r = both(P, policy, seed)
    pre = g.permutation(P)[: int(g.integers(0, P // 2 + 1))]
    a.mark_used(pre)
    r.mark_used(pre)
    live = []
    for _ in range(80):
        if live and g.random() < 0.45:
            ids = live.pop(int(g.integers(len(live))))
            a.free(ids)
            r.free(ids)
        else:
            n = int(g.integers(0, P // 3 + 2))
            if n > r.free_count():
                with pytest.raises(fk.FlowKVError) as e:
                    a.alloc(n)
                assert e.value.code == fk.ENOSPC
                with pytest.raises(oracle.NoSpace):
                    r.alloc(n)
                continue
            x, y = a.alloc(n), r.alloc(n)
            assert x.tolist() == list(y)
            live.append(x)
        assert a.stats() == r.stats()


@pytest.mark.parametrize("policy", [fk.POLICY_SEGMENT, fk.POLICY_FIFO_SORTED,
                                    fk.POLICY_FIFO_SHUFFLED])
def test_allocator_any_order_and_rejected_lists(policy):
    """Frees of any subset of held blocks in any order, marks of free blocks
    in any order, and rejected lists (a repeat after valid IDs, a free block
    among held ones, a held block among free ones) interleaved: the tables
    and stats stay identical to the oracle's, and a rejected list changes
    nothing."""
    g = np.random.default_rng(31 + policy)
    P = 257
    a, r = both(P, policy, 9)
    held = []
    for _ in range(400):
        op = g.random()
        if op < 0.35:
            n = int(g.integers(0, min(40, r.free_count()) + 1))
            x, y = a.alloc(n), r.alloc(n)
            assert x.tolist() == list(y)
            held.extend(x.tolist())
        elif op < 0.65 and held:
            g.shuffle(held)
            k = int(g.integers(1, len(held) + 1))
            ids, held = held[:k], held[k:]
            a.free(ids)
            r.free(ids)
        elif op < 0.8:
            free_ids = np.setdiff1d(np.arange(P), np.asarray(held, dtype=np.int64))
            ids = g.permutation(free_ids)[: int(g.integers(0, min(12, free_ids.size) + 1))]
            a.mark_used(ids)
            r.mark_used(ids)
            held.extend(ids.tolist())
        else:
            before = a.stats()
            free_ids = np.setdiff1d(np.arange(P), np.asarray(held, dtype=np.int64)).tolist()
            bad = []
            if held:
                bad.append((a.free, held[:3] + [held[0]]))
                if free_ids:
                    bad.append((a.free, held[:2] + free_ids[:1]))
                    bad.append((a.mark_used, free_ids[:2] + held[:1]))
            if len(free_ids) > 1:
                bad.append((a.mark_used, free_ids[:2] + [free_ids[1]]))
            for fn, ids in bad:
                with pytest.raises(fk.FlowKVError) as e:
                    fn(ids)
                assert e.value.code == fk.EDUP
            assert a.stats() == before
        assert a.stats() == r.stats()


@pytest.mark.parametrize("variant", ["segment", "shuffled"])
def test_churn_stream_full_size_identical_tables(variant):
    """The 10,000-op churn workload at its real pool size (65,536 blocks)."""
    wl_c = recipes.churn(lambda P, pol, s: fk.Allocator(P, pol, s), variant)
    wl_o = recipes.churn(lambda P, pol, s: oracle.RefAllocator(P, pol, s), variant)
    assert len(wl_c.tables) == len(wl_o.tables) == 128
    for (s1, d1), (s2, d2) in zip(wl_c.tables, wl_o.tables):
        assert np.array_equal(s1, s2) and np.array_equal(d1, d2)


def test_llama8b_tables_identical_and_fragmented():
    for pol in ("fifo_sorted", "segment"):
        wc = recipes.llama8b_13k(lambda P, p, s: fk.Allocator(P, p, s), pol)
        wo = recipes.llama8b_13k(lambda P, p, s: oracle.RefAllocator(P, p, s), pol)
        (S1, D1), (S2, D2) = wc.tables[0], wo.tables[0]
        assert np.array_equal(S1, S2) and np.array_equal(D1, D2)
        assert S1.tolist() == list(range(813))
        k = len(oracle.plan_ref(S1.tolist(), D1.tolist()))
        assert (150 < k < 400) if pol == "fifo_sorted" else (10 < k < 100)


def test_allocator_errors():
    a = fk.Allocator(10)
    ids = a.alloc(6)
    before = a.stats()
    cases = [(lambda: a.alloc(5), fk.ENOSPC), (lambda: a.alloc(-1), fk.EINVAL),
             (lambda: a.free([10]), fk.ERANGE), (lambda: a.free([-1]), fk.ERANGE),
             (lambda: a.free([ids[0], ids[0]]), fk.EDUP), (lambda: a.free([8]), fk.EDUP),
             (lambda: a.mark_used([ids[1]]), fk.EDUP), (lambda: a.mark_used([7, 7]), fk.EDUP)]
    for fn, code in cases:
        with pytest.raises(fk.FlowKVError) as e:
            fn()
        assert e.value.code == code
    assert a.stats() == before
    assert a.alloc(0).size == 0
    for bad in ((-1, 0), (5, 7)):
        with pytest.raises(fk.FlowKVError) as e:
            fk.Allocator(*bad)
        assert e.value.code == fk.EINVAL


# ---- planner -----------------------------------------------------------------

def as_tuples(segs):
    return [(int(s["src_block"]), int(s["dst_block"]), int(s["n_blocks"])) for s in segs]


@settings(max_examples=300, deadline=None)
@given(st.data())
def test_plan_matches_oracle(data):
    seed = data.draw(st.integers(0, 2**32 - 1))
    g = np.random.default_rng(seed)
    P = int(g.integers(1, 200))
    n = int(g.integers(0, P + 1))
    S = g.permutation(P)[:n]
    D = g.permutation(P)[:n]
    for i in range(1, n):  # contiguous stretches are the interesting case
        if g.random() < 0.7 and S[i - 1] + 1 < P and D[i - 1] + 1 < P \
                and S[i - 1] + 1 not in S[:i] and D[i - 1] + 1 not in D[:i]:
            j = np.flatnonzero(S == S[i - 1] + 1)
            k = np.flatnonzero(D == D[i - 1] + 1)
            if j.size: S[j[0]] = S[i]
            if k.size: D[k[0]] = D[i]
            S[i], D[i] = S[i - 1] + 1, D[i - 1] + 1
    if len(set(S.tolist())) < n or len(set(D.tolist())) < n:
        return
    segs = fk.flowkv_plan(S, D, P, P)
    assert as_tuples(segs) == oracle.plan_ref(S.tolist(), D.tolist())
    assert segs["first"].tolist() == np.concatenate(([0], np.cumsum(segs["n_blocks"])[:-1])).tolist()[:len(segs)]


def test_plan_batch_matches_oracle_and_first_runs_across_batch():
    g = np.random.default_rng(5)
    tables = []
    for n in (5, 0, 9, 1, 7):
        tables.append((g.permutation(40)[:n], g.permutation(100)[:n]))
    # receiver IDs must be disjoint across requests: shift each request
    tables = [(s, d + 100 * i) for i, (s, d) in enumerate(tables)]
    off = np.concatenate(([0], np.cumsum([len(s) for s, _ in tables])))
    S = np.concatenate([s for s, _ in tables])
    D = np.concatenate([d for _, d in tables])
    segs = fk.flowkv_plan_batch(off, S, D, 40, 500)
    ref = oracle.plan_batch_ref([(s.tolist(), d.tolist()) for s, d in tables])
    assert as_tuples(segs) == [r[:3] for r in ref]
    assert segs["first"][0] == 0
    assert (segs["first"][1:] == np.cumsum(segs["n_blocks"])[:-1]).all()
    assert fk.plan_total_blocks(segs) == len(S)


def test_plan_batch_records_map_back_to_their_requests():
    """A batch record carries `first` in place of its request's index; the
    header's rule recovers the index -- the last r with offsets[r] <= first
    -- and it is the oracle's request index for every record, with empty
    requests (equal offsets) in the batch, including at its ends.  Each
    record's blocks then sit inside its request's lists."""
    g = np.random.default_rng(17)
    for trial in range(20):
        sizes = [int(x) for x in g.integers(0, 12, size=int(g.integers(1, 9)))]
        if trial % 4 == 0:
            sizes = [0] + sizes + [0, 0]
        tables = []
        for i, n in enumerate(sizes):
            # a few sender runs of random length, a shuffled receiver side
            S = np.sort(g.choice(60, size=n, replace=False)).astype(np.int32)
            D = (1000 * i + np.sort(g.choice(200, size=n, replace=False))).astype(np.int32)
            tables.append((S, D))
        off = np.concatenate(([0], np.cumsum(sizes))).astype(np.int64)
        S_all = np.concatenate([t[0] for t in tables]) if sum(sizes) else np.zeros(0, np.int32)
        D_all = np.concatenate([t[1] for t in tables]) if sum(sizes) else np.zeros(0, np.int32)
        segs = fk.flowkv_plan_batch(off, S_all, D_all, 60, 1000 * len(sizes) + 200)
        ref = oracle.plan_batch_ref([(a.tolist(), b.tolist()) for a, b in tables])
        req = np.searchsorted(off, segs["first"], side="right") - 1
        assert req.tolist() == [r[3] for r in ref]
        for sg, r in zip(segs, req):
            lo = int(sg["first"]) - int(off[r])
            m = int(sg["n_blocks"])
            assert 0 <= lo and lo + m <= sizes[r]
            assert (tables[r][0][lo:lo + m] == sg["src_block"] + np.arange(m)).all()
            assert (tables[r][1][lo:lo + m] == sg["dst_block"] + np.arange(m)).all()


def test_plan_contiguous_is_one_and_stride2_is_n():
    n = 813
    segs = fk.flowkv_plan(np.arange(n), np.arange(100, 100 + n), 1000, 1000)
    assert as_tuples(segs) == [(0, 100, n)]
    segs = fk.flowkv_plan(2 * np.arange(n), 2 * np.arange(n) + 1, 2000, 2000)
    assert len(segs) == n


def test_planners_are_reentrant_across_threads():
    """flowkv_plan keeps its duplicate-check bitmaps per thread: many threads
    planning at once (ctypes releases the interpreter lock during the call)
    each get the oracle's plan, including right after a rejected plan left
    bits to clear."""
    from concurrent.futures import ThreadPoolExecutor

    g = np.random.default_rng(11)
    cases = []
    for i in range(16):   # long lists, so calls on different threads overlap in time
        P = int(g.integers(100_000, 1_000_000))
        n = int(g.integers(50_000, 200_000))
        S = np.sort(g.permutation(P)[:n]) if i % 3 else g.permutation(P)[:n]
        D = np.sort(g.permutation(P)[:n]) if i % 2 else g.permutation(P)[:n]
        want = np.array(oracle.plan_ref(S.tolist(), D.tolist()), dtype=np.int64).reshape(-1, 3)
        cases.append((S.astype(np.int32), D.astype(np.int32), P, want))

    def same(segs, want):
        got = np.stack([segs["src_block"], segs["dst_block"], segs["n_blocks"]], axis=1)
        return np.array_equal(got, want)

    def worker(t):
        for k in range(len(cases)):
            S, D, P, want = cases[(k * 7 + t) % len(cases)]
            if (k + t) % 5 == 0 and len(D) > 1:   # a repeat: EDUP, bits cleared again
                bad = D.copy()
                bad[-1] = bad[0]
                try:
                    fk.flowkv_plan(S, bad, P, P)
                    return f"thread {t}: repeated receiver block accepted"
                except fk.FlowKVError as e:
                    if e.code != fk.EDUP:
                        return f"thread {t}: code {e.code}"
            if not same(fk.flowkv_plan(S, D, P, P), want):
                return f"thread {t}: case {(k * 7 + t) % len(cases)} differs"
        return None

    with ThreadPoolExecutor(8) as ex:
        errors = [e for e in ex.map(worker, range(8)) if e]
    assert not errors, errors


def first_repeat(ids):
    """Position of the first ID that appeared at an earlier position, or None."""
    seen = set()
    for i, x in enumerate(ids):
        if x in seen:
            return i
        seen.add(x)
    return None


def raw_plan(S, D, P, cap, fill=-9):
    """flowkv_plan with an explicit capacity; returns (code, n_out, records)."""
    S, D = np.ascontiguousarray(S, np.int32), np.ascontiguousarray(D, np.int32)
    out = np.full(4 * max(cap, 1), fill, dtype=np.int32).view(fk.SEGMENT_DTYPE)
    n = ctypes.c_int64(-1)
    rc = fk.lib().flowkv_plan(S.ctypes.data, D.ctypes.data, len(S), P, P, out.ctypes.data, cap,
                              ctypes.byref(n))
    return rc, n.value, out


def test_plan_repeats_capacities_and_reuse_after_errors():
    """Repeats are found a run of IDs at a time: the reported position is the
    first whose ID appeared earlier (receiver list first, then sender);
    an output with room for one record per block is written in the counting
    pass, a smaller one after counting, and ECAP leaves it untouched; after
    every rejected plan the same IDs plan cleanly on the same thread."""
    g = np.random.default_rng(23)
    P = 300
    for case in range(400):
        n = int(g.integers(2, 60))
        # runs of consecutive IDs, as allocators hand them out
        def table():
            ids, x = [], int(g.integers(0, P))
            while len(ids) < n:
                if g.random() < 0.3:
                    x = int(g.integers(0, P))
                ids.append(x % P)
                x += 1
            return ids
        S, D = table(), table()
        rs, rd = first_repeat(S), first_repeat(D)
        rc, _, _ = raw_plan(S, D, P, n)
        if rd is not None or rs is not None:
            assert rc == fk.EDUP, (case, S, D)
            pos, bad = (rd, D) if rd is not None else (rs, S)
            msg = fk.lib().flowkv_last_error().decode()
            assert f"block {bad[pos]} repeated (position {pos})" in msg, (msg, pos, S, D)
            assert msg.startswith("receiver" if rd is not None else "sender"), msg
            # the bits set before the repeat were cleared: the distinct IDs
            # of both lists, in order, plan cleanly now
            S, D = list(dict.fromkeys(S)), list(dict.fromkeys(D))
            k = min(len(S), len(D))
            S, D = S[:k], D[:k]
        want = oracle.plan_ref(S, D)
        need, total = len(want), len(S)
        for cap in sorted({need, total, total + 3}):
            rc, k, out = raw_plan(S, D, P, cap)
            assert rc == fk.OK and k == need, (case, cap, rc)
            assert as_tuples(out[:k]) == want
            assert (out["first"][:k] == np.concatenate(([0], np.cumsum(out["n_blocks"][:k])[:-1]))).all()
        if need > 1:
            rc, k, out = raw_plan(S, D, P, need - 1)
            assert rc == fk.ECAP and k == need
            assert (out.view(np.int32) == -9).all(), "ECAP wrote into the output"
    # a range error after a valid plan of the same IDs leaves nothing behind
    with pytest.raises(fk.FlowKVError):
        fk.flowkv_plan([0, 1, 2], [5, 6, P], P, P)
    assert as_tuples(fk.flowkv_plan([0, 1, 2], [5, 6, 7], P, P)) == [(0, 5, 3)]


def test_plan_batch_repeats_across_and_within_requests():
    """A batch may repeat a sender block across requests (a shared prefix)
    but not within one, and may not repeat a receiver block anywhere.  On
    seeded batches built from runs of IDs the planner either matches the
    oracle's per-request plans or names the first offending position: the
    receiver list over the whole batch is checked first, then each
    request's sender list."""
    g = np.random.default_rng(41)
    P = 400
    outcomes = {"ok": 0, "receiver": 0, "sender": 0}
    for case in range(300):
        tables = []
        for _ in range(int(g.integers(1, 6))):
            n = int(g.integers(0, 25))
            def ids():
                out, x = [], int(g.integers(0, P))
                while len(out) < n:
                    if g.random() < 0.3:
                        x = int(g.integers(0, P))
                    out.append(x % P)
                    x += 1
                return out
            tables.append((ids(), ids()))
        off = np.concatenate(([0], np.cumsum([len(s) for s, _ in tables]))).astype(np.int64)
        S = [x for s, _ in tables for x in s]
        D = [x for _, d in tables for x in d]
        rd = first_repeat(D)
        rs = None
        for r, (sr, _) in enumerate(tables):
            k = first_repeat(sr)
            if k is not None:
                rs = int(off[r]) + k
                break
        if rd is None and rs is None:
            segs = fk.flowkv_plan_batch(off, S, D, P, P)
            want = oracle.plan_batch_ref(tables)
            assert as_tuples(segs) == [w[:3] for w in want], case
            assert fk.plan_total_blocks(segs) == len(S)
            outcomes["ok"] += 1
            continue
        with pytest.raises(fk.FlowKVError) as e:
            fk.flowkv_plan_batch(off, S, D, P, P)
        assert e.value.code == fk.EDUP, case
        pos, ids, side = (rd, D, "receiver") if rd is not None else (rs, S, "sender")
        msg = fk.lib().flowkv_last_error().decode()
        assert msg.startswith(side) and f"block {ids[pos]} repeated (position {pos})" in msg, \
            (case, msg, side, pos)
        outcomes[side] += 1
    assert min(outcomes.values()) >= 20, outcomes


def test_plan_errors():
    P = 16
    cases = [((P,), (0,), fk.ERANGE), ((0,), (-1,), fk.ERANGE), ((1, 1), (2, 3), fk.EDUP),
             ((1, 2), (3, 3), fk.EDUP)]
    for S, D, code in cases:
        with pytest.raises(fk.FlowKVError) as e:
            fk.flowkv_plan(S, D, P, P)
        assert e.value.code == code
    # ECAP reports the need
    S = np.array([0, 2, 4], dtype=np.int32)
    D = np.array([0, 1, 2], dtype=np.int32)
    out = (fk.flowkv_segment * 1)()
    need = ctypes.c_int64(-7)
    rc = fk.lib().flowkv_plan(S.ctypes.data_as(fk._I32P), D.ctypes.data_as(fk._I32P), 3, P, P,
                              out, 1, ctypes.byref(need))
    assert rc == fk.ECAP and need.value == 3
    # batch: a receiver block shared by two requests is rejected, a sender
    # block shared by two requests is allowed
    with pytest.raises(fk.FlowKVError) as e:
        fk.flowkv_plan_batch([0, 1, 2], [1, 2], [5, 5], P, P)
    assert e.value.code == fk.EDUP
    assert len(fk.flowkv_plan_batch([0, 1, 2], [1, 1], [5, 6], P, P)) == 2
    for off in ([1, 2], [0, 3, 2]):             # not from 0, not non-decreasing
        with pytest.raises(fk.FlowKVError) as e:
            fk.flowkv_plan_batch(off, [1, 2], [3, 4], P, P)
        assert e.value.code == fk.EINVAL
    # offsets that end past or short of the lists, or are not one row, never
    # reach the planner (it would read past the lists or drop their tail)
    for off in ([0, 5], [0, 1], [0, 2, 3], [], [[0, 2]]):
        with pytest.raises(ValueError):
            fk.flowkv_plan_batch(off, [1, 2], [3, 4], P, P)
    assert len(fk.flowkv_plan([], [], P, P)) == 0


def test_binding_marshals_plans_or_rejects_them():
    """A host plan is taken as SEGMENT_DTYPE records or as integer (k, 4)
    rows of the same four fields (any integer width), anything else is
    rejected; a device plan must be a contiguous int32 tensor of at least
    n_segs rows on the pools' device (no device is touched here)."""
    import torch
    from types import SimpleNamespace

    plan = fk.flowkv_plan([3, 4, 9], [7, 8, 1], 16, 16)
    rows = plan.view(np.int32).reshape(-1, 4)
    for form in (plan, rows, rows.astype(np.int64), rows.astype(np.uint16), rows.tolist()):
        got = fk._host_segments(form)
        assert got.dtype == fk.SEGMENT_DTYPE and got.flags.c_contiguous
        assert np.array_equal(got.view(np.int32).reshape(-1, 4), rows)
    assert len(fk._host_segments(np.zeros((0, 4), np.int32))) == 0
    for bad in (rows.astype(np.float32), rows[:, :3], rows.reshape(-1), rows.reshape(1, -1, 4)):
        with pytest.raises(ValueError):
            fk._host_segments(bad)

    on = SimpleNamespace(device=torch.device("cuda", 0))
    t = torch.from_numpy(rows.copy())                 # a CPU tensor: wrong device
    assert fk._device_segments(t, 0, on) == 0         # nothing to read, nothing checked
    with pytest.raises(ValueError, match="device plan"):
        fk._device_segments(t, 2, on)
    cpu = SimpleNamespace(device=torch.device("cpu"))
    assert fk._device_segments(t, 2, cpu) == t.data_ptr()
    for bad in (t.to(torch.int64), t.t(), t[:1]):     # dtype, layout, too few rows
        with pytest.raises(ValueError, match="device plan"):
            fk._device_segments(bad, 2, cpu)


# ---- transfer argument checks (rejected before any device call) --------------

def pool(layout=1, L=2, B=8, chunk=4096, bases=(1 << 20,)):
    arr = (ctypes.c_void_p * len(bases))(*bases)
    p = fk.flowkv_pool(layout, L, B, 0, chunk, ctypes.cast(arr, ctypes.POINTER(ctypes.c_void_p)))
    p._keep = arr
    return p


def xfer(src, dst, n_segs=1, total=1, cfg=None, segs=1 << 12):
    c = ctypes.byref(cfg) if cfg is not None else None
    return fk.lib().flowkv_transfer_ex(ctypes.byref(src), ctypes.byref(dst),
                                       ctypes.c_void_p(segs), n_segs, total, c, None)


def test_transfer_rejects_bad_pools_without_touching_the_device():
    bb = 2 * 2 * 4096
    good_src = pool(bases=(1 << 30,))
    good_dst = pool(bases=(1 << 31,))
    # no-op plans succeed without a launch
    assert xfer(good_src, good_dst, n_segs=0, total=0) == fk.OK
    assert xfer(good_src, good_dst, n_segs=5, total=0) == fk.OK
    bad = [
        (pool(bases=(1 << 30,)), pool(bases=((1 << 30) + bb,))),          # overlap
        (pool(bases=((1 << 30) + 8,)), good_dst),                           # misaligned
        (pool(chunk=100, bases=(1 << 30,)), pool(chunk=100, bases=(1 << 31,))),  # not x16
        (pool(L=129, bases=(1 << 30,)), pool(L=129, bases=(1 << 31,))),     # too many layers
        (pool(L=3, bases=(1 << 30,)), good_dst),                            # layer mismatch
        (pool(layout=7, bases=(1 << 30,)), good_dst),                       # bad layout
        (pool(B=0, bases=(1 << 30,)), good_dst),                            # empty pool
        (pool(bases=(0,)), good_dst),                                       # NULL base
        (pool(L=128, chunk=1 << 23, bases=(1 << 30,)), pool(L=128, chunk=1 << 23, bases=(1 << 40,))),
        (pool(layout=0, L=2, bases=(1 << 30, 1 << 30)), good_dst),         # fine for src ...
    ]
    for i, (s, d) in enumerate(bad[:-1]):
        assert xfer(s, d) == fk.EINVAL, i
    # receiver layer tensors that overlap each other
    d = pool(layout=0, L=2, bases=(1 << 33, (1 << 33) + 4096))
    assert xfer(good_src, d, n_segs=0, total=0) == fk.EINVAL
    # launch shapes outside the documented limits
    for cfg in (fk.flowkv_launch_config(96, 8, 0, 0), fk.flowkv_launch_config(2048, 8, 0, 0),
                fk.flowkv_launch_config(256, 3, 0, 0), fk.flowkv_launch_config(256, 8, -1, 0),
                fk.flowkv_launch_config(256, 8, 0, 9), fk.flowkv_launch_config(256, 8, 0, 0, 5),
                fk.flowkv_launch_config(256, 8, 0, 0, -1)):
        assert xfer(good_src, good_dst, n_segs=0, total=0, cfg=cfg) == fk.EINVAL
    # layer ranges of the layer-wise entry point
    def xfer_layers(l0, lc):
        return fk.lib().flowkv_transfer_layers(ctypes.byref(good_src), ctypes.byref(good_dst),
                                               ctypes.c_void_p(1 << 12), 1, 1, l0, lc, None, None)
    for l0, lc in ((-1, 1), (0, 3), (2, 1), (1, 2), (0, -1)):
        assert xfer_layers(l0, lc) == fk.EINVAL, (l0, lc)
    assert xfer_layers(1, 0) == fk.OK  # nothing to move: no launch
    # plans carried in the kernel arguments: at most INLINE_RUNS records
    big = np.zeros(fk.INLINE_RUNS + 1, dtype=fk.SEGMENT_DTYPE)
    rc = fk.lib().flowkv_transfer_inline(ctypes.byref(good_src), ctypes.byref(good_dst),
                                         big.ctypes.data_as(fk._SEGP), len(big), 1, None, None)
    assert rc == fk.ECAP
    # beyond INLINE_RUNS only between block-major pools, only in the
    # planner's form, and at most INLINE_RUNS_BLOCK_MAJOR records
    def inline(src, dst, recs, total):
        return fk.lib().flowkv_transfer_inline(ctypes.byref(src), ctypes.byref(dst),
                                               recs.ctypes.data_as(fk._SEGP), len(recs), total,
                                               None, None)

    def planner_form(k):
        r = np.zeros(k, dtype=fk.SEGMENT_DTYPE)
        r["n_blocks"], r["first"] = 1, np.arange(k)
        return r
    assert inline(good_src, good_dst, planner_form(fk.INLINE_RUNS_BLOCK_MAJOR + 1),
                  fk.INLINE_RUNS_BLOCK_MAJOR + 1) == fk.ECAP
    runs = planner_form(100)
    # a layer-major pool: the compact form up to INLINE_RUNS_LAYER_MAJOR
    # records while neither pool has more than INLINE_LAYERS layers
    lm_src = pool(layout=0, L=2, bases=(1 << 34, (1 << 34) + (1 << 24)))
    k = fk.INLINE_RUNS_LAYER_MAJOR + 1
    assert inline(lm_src, good_dst, planner_form(k), k) == fk.ECAP
    L = fk.INLINE_LAYERS + 1
    deep = [pool(layout=lay, L=L, bases=tuple((1 << 36) * (j + 1) + (i << 24) for i in
                                              range(L if lay == 0 else 1)))
            for j, lay in enumerate((0, 1, 0))]
    k = fk.INLINE_RUNS + 1
    assert inline(deep[0], deep[1], planner_form(k), k) == fk.ECAP
    assert inline(deep[1], deep[2], planner_form(k), k) == fk.ECAP
    gap = runs.copy()
    gap["first"][50] += 1
    assert inline(good_src, good_dst, gap, 100) == fk.ECAP       # runs do not abut
    assert inline(good_src, good_dst, runs, 101) == fk.ECAP      # nor cover total_blocks
    empty = runs.copy()
    empty["n_blocks"][7] = 0
    empty["first"][8:] -= 1
    assert inline(good_src, good_dst, empty, 99) == fk.ECAP      # a run of no blocks
    rc = fk.lib().flowkv_transfer_inline(ctypes.byref(good_src), ctypes.byref(good_dst),
                                         None, 1, 1, None, None)
    assert rc == fk.EINVAL
    rc = fk.lib().flowkv_transfer_inline(ctypes.byref(good_src), ctypes.byref(good_dst),
                                         None, 0, 0, None, None)
    assert rc == fk.OK
    assert xfer(good_src, good_dst, segs=8) == fk.EINVAL  # misaligned plan
    assert xfer(good_src, good_dst, segs=0) == fk.EINVAL  # NULL plan
    assert xfer(good_src, good_dst, n_segs=-1) == fk.EINVAL


def test_transfer_request_rejects_before_any_device_call():
    """flowkv_transfer_request: NULL pools, a negative count, the planner's
    ERANGE and EDUP, and ECAP past the inline capacity (run count reported)
    all return before anything is launched; zero blocks is a no-op."""
    lib = fk.lib()
    bm = pool(layout=1, L=2, B=1000)                             # 16 MB at 1 MiB
    bm2 = pool(layout=1, L=2, B=1000, bases=(1 << 30,))
    lm = pool(layout=0, L=2, B=1000, bases=(1 << 28, 1 << 29))

    def req(src, dst, S, D, n=None):
        S, D = np.ascontiguousarray(S, np.int32), np.ascontiguousarray(D, np.int32)
        k = ctypes.c_int64(-1)
        rc = lib.flowkv_transfer_request(src and ctypes.byref(src), dst and ctypes.byref(dst),
                                         S.ctypes.data, D.ctypes.data,
                                         len(S) if n is None else n, None, ctypes.byref(k), None)
        return rc, k.value

    assert req(None, bm2, [0], [0])[0] == fk.EINVAL
    assert req(bm, bm2, [0], [0], n=-1)[0] == fk.EINVAL
    assert req(bm, bm2, [1000], [0])[0] == fk.ERANGE
    assert req(bm, bm2, [1, 1], [2, 3])[0] == fk.EDUP
    assert req(bm, bm2, [], []) == (fk.OK, 0)
    assert req(bm, bm, [], []) == (fk.EINVAL, -1)                   # overlapping pools
    assert req(bm, bm, [0, 1], [5, 6]) == (fk.EINVAL, -1)           # n_runs left untouched
    stride2 = 2 * np.arange(301)
    assert req(bm, bm2, stride2, stride2 + 1) == (fk.ECAP, 301)      # block-major: 300 fit
    k = fk.INLINE_RUNS_LAYER_MAJOR + 1                                # a layer-major pool
    assert req(bm, lm, np.arange(k) * 2, np.arange(k) * 2) == (fk.ECAP, k)
    L = fk.INLINE_LAYERS + 1                                         # ... of many layers
    bm_deep = pool(layout=1, L=L, B=1000, bases=(1 << 31,))
    lm_deep = pool(layout=0, L=L, B=1000, bases=tuple((1 << 32) + (i << 24) for i in range(L)))
    k = fk.INLINE_RUNS + 1
    assert req(bm_deep, lm_deep, np.arange(k) * 2, np.arange(k) * 2) == (fk.ECAP, k)
    assert req(lm, pool(layout=7), [0], [0]) == (fk.EINVAL, -1)      # bad pool: no planning


def test_abi_check_program_is_built_and_runs_without_python():
    """The build step also builds tests/native/abi_transfer, which uses the
    library through the C ABI alone; its dynamic links resolve, and without
    arguments it prints its usage (before any HIP call)."""
    import subprocess
    exe = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "abi_transfer")
    assert os.path.exists(exe), "run the build step first"
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 2 and "usage: abi_transfer" in r.stderr


def test_binding_shares_torchs_hip_runtime():
    """Device pointers and streams come from torch, so the library must bind
    to torch's HIP runtime: exactly one libamdhip64 may be mapped."""
    assert len(fk._hip_runtimes_loaded()) == 1


# ---- decode attention argument checks (rejected before any device call) ------

def attn(p, layer=0, q=1 << 12, n_req=1, hq=8, hkv=2, dh=128, tables=1 << 16, max_blocks=4,
         lens=1 << 18, max_seq=64, scale=0.1, split=0, out=1 << 20, ws=1 << 24, ws_bytes=1 << 30,
         host_lens=None):
    return fk.lib().flowkv_decode_attention(
        ctypes.byref(p), layer, ctypes.c_void_p(q), n_req, hq, hkv, dh, ctypes.c_void_p(tables),
        max_blocks, ctypes.c_void_p(lens), host_lens, max_seq, scale, split,
        ctypes.c_void_p(out), ctypes.c_void_p(ws), ws_bytes, None)


def test_attention_rejects_bad_arguments_without_touching_the_device():
    chunk = 16 * 2 * 128 * 2                       # bs 16, 2 KV heads, head_dim 128, bf16
    p = pool(L=2, B=8, chunk=chunk)
    assert attn(p, n_req=0) == fk.OK              # nothing to do: no launch
    cases = [
        dict(layer=2), dict(layer=-1), dict(dh=96), dict(hq=6, hkv=4), dict(hq=32, hkv=2),
        dict(split=1025), dict(split=-3), dict(scale=0.0), dict(scale=float("inf")),
        dict(q=(1 << 12) + 8),                     # query not 16-byte aligned
        dict(n_req=70000),                         # past the grid's 65,535 requests
        dict(max_seq=70000, split=1),              # past the grid's 65,535 splits
        dict(max_blocks=-1), dict(q=0), dict(ws=0),
        dict(max_blocks=1 << 27),                  # 2^27 blocks x 16 tokens: past 2^31 - 1
    ]
    for c in cases:
        assert attn(p, **c) == fk.EINVAL, c
    assert attn(p, ws_bytes=16) == fk.ECAP
    assert attn(pool(L=2, B=8, chunk=chunk + 16)) == fk.EINVAL    # chunk not bs x Hkv x Dh x 2
    assert attn(pool(layout=7, L=2, B=8, chunk=chunk)) == fk.EINVAL
    assert attn(pool(L=2, B=8, chunk=chunk, bases=(0,))) == fk.EINVAL   # NULL base
    # the device lengths may be NULL only when the host copy travels in the
    # kernel arguments (at most ATTN_INLINE_LENS requests)
    assert attn(p, lens=0) == fk.EINVAL
    big = np.zeros(fk.ATTN_INLINE_LENS + 1, np.int32)
    assert attn(p, lens=0, n_req=len(big), host_lens=big.ctypes.data, ws_bytes=16) == fk.EINVAL
    assert attn(p, n_req=len(big), host_lens=big.ctypes.data, ws_bytes=16) == fk.ECAP
    ok = np.zeros(fk.ATTN_INLINE_LENS, np.int32)
    assert attn(p, lens=0, n_req=len(ok), host_lens=ok.ctypes.data, ws_bytes=16) == fk.ECAP


def test_binding_host_lengths_are_one_int32_per_request():
    """The binding hands the library a contiguous int32 copy of the host
    lengths, one per request, or nothing."""
    assert fk._host_lens(None, 3) is None
    h = fk._host_lens([5, 0, 7], 3)
    assert h.dtype == np.int32 and h.flags["C_CONTIGUOUS"] and h.tolist() == [5, 0, 7]
    h64 = np.arange(8, dtype=np.int64)[::2]            # strided, int64
    assert fk._host_lens(h64, 4).tolist() == [0, 2, 4, 6]
    for bad in ([1, 2], [[1, 2, 3]], np.zeros((3, 1), np.int32)):
        with pytest.raises(ValueError):
            fk._host_lens(bad, 3)


def attn_noalloc(p, layer=0, q=1 << 12, n_req=1, hq=8, hkv=2, dh=128, tables=1 << 16,
                 max_blocks=4, lens=1 << 18, max_seq=64, scale=0.1, split=0, out=1 << 20,
                 host_lens=None):
    return fk.lib().flowkv_decode_attention_noalloc(
        ctypes.byref(p), layer, ctypes.c_void_p(q), n_req, hq, hkv, dh, ctypes.c_void_p(tables),
        max_blocks, ctypes.c_void_p(lens), host_lens, max_seq, scale, split,
        ctypes.c_void_p(out), None)


def test_noalloc_attention_rejects_before_any_runtime_call():
    """The allocation-free variant checks its arguments as the workspace form
    does, and rejects a call whose partial results exceed the library's
    scratch (ECAP) before it looks the scratch up: on this host, with no GPU,
    every one of these returns without a runtime call."""
    chunk = 16 * 2 * 128 * 2
    p = pool(L=2, B=8, chunk=chunk)
    assert fk.ATTN_SCRATCH_BYTES == 16 << 20
    assert attn_noalloc(p, n_req=0) == fk.OK
    for c in (dict(layer=2), dict(dh=96), dict(hq=6, hkv=4), dict(split=1025), dict(scale=0.0),
              dict(q=(1 << 12) + 8), dict(q=0), dict(out=0), dict(max_blocks=-1),
              dict(lens=0)):
        assert attn_noalloc(p, **c) == fk.EINVAL, c
    # the need is n_req x q_heads x splits x (head_dim + 2) floats: find the
    # largest request count that fits the scratch at 32 query heads over 8
    # KV heads and 20,000 tokens, then one more
    p8 = pool(L=2, B=8, chunk=16 * 8 * 128 * 2)
    per_req = fk.flowkv_decode_attention_workspace(1, 32, 128, 20000, 1024)
    fits = fk.ATTN_SCRATCH_BYTES // per_req
    assert fk.flowkv_decode_attention_workspace(fits + 1, 32, 128, 20000, 1024) \
        > fk.ATTN_SCRATCH_BYTES
    rc = attn_noalloc(p8, n_req=fits + 1, hq=32, hkv=8, max_seq=20000, split=1024)
    assert rc == fk.ECAP
    assert "scratch holds 16777216" in fk.lib().flowkv_last_error().decode()


@pytest.mark.parametrize("private", [True, False])
def test_current_stream_handle_with_and_without_the_private_call(monkeypatch, private):
    """The binding reads the current stream's handle through a private call of
    torch's, and through the public Stream object where torch lacks it; a
    stream that the caller passes is taken as it is."""
    import types

    import torch

    if private:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: 100 + dev,
                            raising=False)
        monkeypatch.setattr(torch.cuda, "current_stream", None)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
        monkeypatch.setattr(torch.cuda, "current_stream",
                            lambda: types.SimpleNamespace(cuda_stream=103))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert fk._stream_handle(None) == 103
    assert fk._stream_handle(types.SimpleNamespace(cuda_stream=7)) == 7
