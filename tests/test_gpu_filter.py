"""GPU parity of FIXED tables that pack first candidates and keep a spill filter:
what packing costs in the stash, small stashes, and the filter's end.

Outputs and contents are exact (the dictionary oracle's); the bounds on counts
of stash entries are stated where they are used.
"""
import sys

import numpy as np
import pytest

import oracle
from paper_2510_15095_amd import workload as wl

pytestmark = pytest.mark.gpu


def case(msg):
    print(f"[case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2510_15095_amd import hive
    return hive


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    return t.cpu().numpy()


def make(H, S, nb, set32=False, **cfg):
    if set32:
        return H.Table(nb, slots_per_bucket=32, entry_bits=32, **cfg)
    return H.Table(nb, slots_per_bucket=S, **cfg)


def values(keys, set32):
    return np.zeros(keys.size, np.uint32) if set32 else wl.values_for(keys)


@pytest.mark.parametrize("S,set32", [(16, False), (32, False), (64, False), (32, True)])
def test_packing_leaves_the_stash_almost_empty(H, S, set32):
    """A build of 2^21 keys to 95% load in one batch: two-choice placement
    leaves 0 to 4 entries in the stash.  Packed first candidates may leave a
    few times that, at most 0.002% of the slots."""
    n = 1 << 21
    nb = int(np.ceil(n / (0.95 * S)))
    case(f"stash of a build to 95% S={S} set32={set32}")
    keys = wl.KeyStream(1500).range(0, n)
    t = make(H, S, nb, set32, max_batch=n)
    t.insert(dev(keys), dev(values(keys, set32)), flags=H.HIVE_UNIQUE)
    st = t.stats()
    assert st["status"] == H.HIVE_OK and st["live"] == n
    assert st["stash_count"] <= 0.00002 * nb * S, st
    _, f = t.lookup(dev(keys))
    assert host(f).all()
    t.close()


def test_a_small_stash_holds_what_two_choice_leaves(H):
    """A stash and pending list of 256 entries each, sized for two-choice
    placement under a bound of 4 displacements (about 50 entries of 2^20 keys at
    95% load): nothing is lost."""
    n = 1 << 20
    case("small stash at 95%")
    keys = wl.KeyStream(1501).range(0, n)
    t = H.Table(int(np.ceil(n / (0.95 * 16))), max_evictions=4, stash_capacity=256, pending_capacity=256, max_batch=n)
    t.insert(dev(keys), dev(wl.values_for(keys)), flags=H.HIVE_UNIQUE)
    st = t.stats()
    assert st["status"] == H.HIVE_OK and st["live"] == n, st
    v, f = t.lookup(dev(keys))
    assert host(f).all() and np.array_equal(host(v), wl.values_for(keys))
    t.close()


def second_share(H, t):
    first, second, _ = H.hive_placement(t.h)
    return second / max(1, first + second)


@pytest.mark.parametrize("executor", [False, True])
@pytest.mark.parametrize("S,set32", [(16, False), (32, False), (64, False), (32, True)])
def test_filter_ends_with_the_first_fill(H, S, set32, executor):
    """A half-full table whose contents are turned over: the first fill packs
    first candidates (hardly a key in its second), and once inserts amount to
    the filter's limit new keys are placed by two-choice again (about 0.4 of
    them in their second candidate in turned-over tables of any width), so that
    no worn filter is left to read."""
    if executor and set32:
        pytest.skip("the executor takes 64-bit entries")
    import torch
    nb = 4096 * 16 // S
    n = nb * S // 2
    case(f"end of the filter S={S} set32={set32} executor={executor}")
    ks = wl.KeyStream(1600 + S)
    t, o = make(H, S, nb, set32, max_batch=n), oracle.O1()
    d = H.hive_drain_create(S, 0, 64, 1, 10_000_000) if executor else None
    keep = []

    def submit(mode, k, v=None, vo=None, fo=None):
        keep.append((k, v, vo, fo))
        assert H.hive_drain_submit(d, t.h, mode, k, v, None, vo, fo, flags=H.HIVE_UNIQUE) is not None
        H.hive_drain_launch(d, 0)
        torch.cuda.synchronize()

    def insert(k):
        if executor:
            submit(H.HIVE_OP_INSERT, dev(k), dev(values(k, set32)))
        else:
            t.insert(dev(k), dev(values(k, set32)), flags=H.HIVE_UNIQUE)
        o.insert(k, values(k, set32))

    def delete(k):
        if executor:
            fo = torch.zeros(k.size, dtype=torch.uint8, device="cuda")
            submit(H.HIVE_OP_DELETE, dev(k), None, None, fo)
        else:
            fo = t.delete(dev(k), flags=H.HIVE_UNIQUE)
        assert np.array_equal(host(fo), o.delete(k))

    def check():
        q = ks.range(max(0, lo - n), hi + n)
        if executor:
            vo = torch.zeros(q.size, dtype=torch.int32, device="cuda").view(torch.uint32)
            f = torch.zeros(q.size, dtype=torch.uint8, device="cuda")
            submit(H.HIVE_OP_LOOKUP, dev(q), None, vo, f)
            v = vo
        else:
            v, f = t.lookup(dev(q))
        ov, of = o.lookup(q)
        assert np.array_equal(host(f), of)
        if not set32:
            assert np.array_equal(host(v), ov)

    lo, hi = 0, n
    insert(ks.range(0, n))
    check()
    assert second_share(H, t) < 0.1
    for _ in range(12):  # three turnovers
        delete(ks.range(lo, lo + n // 4))
        lo += n // 4
        check()
        insert(ks.range(hi, hi + n // 4))
        hi += n // 4
        check()
    assert second_share(H, t) > 0.3
    assert np.array_equal(t.dump(), o.dump())
    t.clear()  # and a cleared table packs again
    o = oracle.O1()
    insert(ks.range(lo, lo + n))
    assert second_share(H, t) < 0.1
    assert np.array_equal(t.dump(), o.dump())
    if executor:
        H.hive_drain_destroy(d)
    t.close()


def test_replays_and_eager_calls_agree_on_the_filter(H):
    """Launches captured while the table had its filter, replayed after eager
    calls dropped it, and eager calls after replays that cleared the table and
    filled it with a filter again: every lookup equals the dictionary's."""
    import torch
    case("filter across replays")
    S, nb = 16, 4096
    n = int(nb * S * 0.9)
    ks = wl.KeyStream(1700)
    a, b = ks.range(0, n), ks.range(n, n + nb * S // 20)
    t = H.Table(nb, max_batch=n)
    q = np.concatenate([a, b, ks.range(2 * n, 3 * n)])
    da, va, db, vb, dq = dev(a), dev(wl.values_for(a)), dev(b), dev(wl.values_for(b)), dev(q)
    gone = a[np.random.default_rng(17).permutation(n)[: 6 * n // 10]]
    dg = dev(gone)
    vo = torch.empty(q.size, dtype=torch.int32, device="cuda").view(torch.uint32)
    fo = torch.empty(q.size, dtype=torch.uint8, device="cuda")

    def fill():
        H.hive_clear(t.h, side)
        H.hive_insert_batch(t.h, da, va, H.HIVE_UNIQUE, side)

    def look():
        H.hive_lookup_batch(t.h, dq, vo, fo, side)

    def more():
        H.hive_insert_batch(t.h, db, vb, H.HIVE_UNIQUE, side)

    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        fill()
        look()
    torch.cuda.synchronize()
    graphs = []
    for step in (look, more, fill):  # `fill` last: the host then counts a full table
        H.hive_clear(t.h, side)  # the host's count starts over, too
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            step()
        graphs.append(g)
    g_look, g_more, g_fill = graphs

    def expect(present, what):
        torch.cuda.synchronize()
        there = np.isin(q, present)
        assert np.array_equal(host(fo).astype(bool), there), what
        assert np.array_equal(host(vo), np.where(there, wl.values_for(q), np.uint32(0xFFFFFFFF))), what

    def run(step):
        """One step, done before the next: replays run on the current stream,
        eager calls on `side`, and a handle takes ordered streams only."""
        if isinstance(step, torch.cuda.CUDAGraph):
            step.replay()
        else:
            step()
        torch.cuda.synchronize()

    for r in range(3):
        run(g_fill)
        run(g_look)
        expect(a, f"filled {r}")
        # eager: inserts without the filter (the host counted the fills' n)
        run(more)
        run(g_look)
        expect(np.concatenate([a, b]), f"dropped {r}")
        # filled again by a replay, then an eager delete of the host that dropped it
        run(g_fill)
        run(lambda: H.hive_delete_batch(t.h, dg, None, H.HIVE_UNIQUE, side))
        run(g_look)
        left = np.setdiff1d(a, gone)
        expect(left, f"deleted {r}")
        for _ in range(2):
            run(g_more)
            run(g_look)
            expect(np.concatenate([left, b]), f"more {r}")
        run(look)
        expect(np.concatenate([left, b]), f"eager lookup {r}")
    t.close()


@pytest.mark.parametrize("kinds", [(15, 15, 15, 15), (15, 0, 4, 0), (0, 15, 0, 15)])
def test_4x16_asked_for_by_name(H, kinds):
    """4 waves and 16 loads by name (15), beside the library's choice (0)."""
    from test_gpu_probe_variants import run_all_kinds
    case(f"probe variants by name {kinds}")
    run_all_kinds(H, H.probe_tuning(*kinds), 0)


@pytest.mark.parametrize("bits", [8, 4, 2, 1])
def test_filters_of_fewer_bits_per_bucket(H, bits):  # noqa: F811
    """Large tables have fewer filter bits a bucket.  Keys that crowd into 3,000
    first candidates, about 12 each, so that many sit elsewhere: lookups of them
    and of absent keys of the same buckets, before and after deletes."""
    import torch
    nb = {8: 4_000_000, 4: 5_400_000, 2: 10_600_000, 1: 21_100_000}[bits]
    got = []
    out = torch.empty(1 << 24, dtype=torch.uint32, device="cuda")
    lo = 1
    while lo < 12 * nb:  # 12 candidates for every bucket
        keys = torch.arange(lo, lo + (1 << 24), dtype=torch.int64, device="cuda").to(torch.uint32)
        H.hive_hash_buckets("bithash1", keys, nb, out)
        got.append(keys.cpu().numpy()[out.cpu().numpy() < 3000])
        lo += 1 << 24
    keys = np.random.default_rng(bits).permutation(np.concatenate(got))
    absent, present = keys[:keys.size // 8], keys[keys.size // 8:]
    gone = present[: present.size // 3]
    case(f"{nb} buckets, {present.size} keys in 3,000 of them")
    t = H.Table(nb, max_batch=1 << 17)
    o = oracle.O1()
    for part in np.array_split(present, 3):
        t.insert(dev(part), dev(wl.values_for(part)))
        o.insert(part, wl.values_for(part))
    elsewhere = t.placement()[1]
    assert elsewhere > present.size // 20, f"only {elsewhere} of {present.size} in second candidates"
    for step in range(2):
        v, f = t.lookup(dev(keys))
        ov, of = o.lookup(keys)
        assert np.array_equal(host(f), of) and np.array_equal(host(v)[of == 1], ov[of == 1])
        assert of.sum() == (present.size if step == 0 else present.size - gone.size)
        if step == 0:
            assert host(t.delete(dev(gone))).sum() == gone.size
            o.delete(gone)
    assert absent.size > 1000
    t.close()
