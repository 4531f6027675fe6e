"""GPU parity of the batch paths at the sizes where they change: claims that
crowd into few buckets, export by trips, dedupe and resize forms.

Everything is exact: outputs, key counts and contents equal the dictionary
oracle's.
"""
import sys

import numpy as np
import pytest

import oracle
from paper_2510_15095_amd import workload as wl

pytestmark = pytest.mark.gpu

M32 = 0xFFFFFFFF


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
@pytest.mark.parametrize("nb,over", [(1, 0), (1, 7), (3, 0), (64, 0), (64, 100)])
def test_claims_crowd_into_full_buckets(H, S, set32, nb, over):
    """One batch fills every slot of the table (and `over` entries go to the
    stash): its claims of one bucket all run side by side, each from a slot of
    its own, and together take every slot."""
    case(f"crowded claims S={S} set32={set32} nb={nb} over={over}")
    n = nb * S + over
    ks = wl.KeyStream(501 + nb)
    keys = ks.range(0, n)
    t, o = make(H, S, nb, set32, stash_capacity=4096, pending_capacity=4096), oracle.O1()
    for part in (keys[: n // 2], keys[n // 2:]):
        t.insert(dev(part), dev(values(part, set32)), flags=H.HIVE_UNIQUE)
        o.insert(part, values(part, set32))
    st = t.stats()
    assert st["status"] == H.HIVE_OK and st["live"] == n
    words, where = t.dump(with_where=True)
    assert np.array_equal(words, o.dump())
    assert np.bincount(where[where >= 0], minlength=nb).max() <= S
    q = ks.range(0, 2 * n)
    v, f = t.lookup(dev(q))
    ov, of = o.lookup(q)
    assert np.array_equal(host(f), of)
    if not set32:
        assert np.array_equal(host(v), ov)
    t.close()


@pytest.mark.parametrize("S,set32", [(16, False), (64, False), (32, True)])
@pytest.mark.parametrize("slots,extra", [(64, 0), (64, 9), (16384, 0), (16384 + 64, 3), (70_400, 300)])
def test_dump_by_trips(H, S, set32, slots, extra):
    """Export of tables of less than a trip of 16,384 words, exactly one, a
    little more and several, with entries in the stash and the pending list,
    with and without places, and into a buffer that is too small (the count
    is whole, the words that fit are entries of the table)."""
    import torch
    nb = slots // S
    n = nb * S * 3 // 4 + extra
    case(f"dump S={S} set32={set32} buckets={nb} entries={n}")
    ks = wl.KeyStream(777 + slots)
    keys = ks.range(0, n)
    t, o = make(H, S, nb, set32, max_evictions=0, stash_capacity=16, pending_capacity=8192), oracle.O1()
    t.insert(dev(keys), dev(values(keys, set32)), flags=H.HIVE_UNIQUE)
    o.insert(keys, values(keys, set32))
    gone = keys[::5]
    t.delete(dev(gone), flags=H.HIVE_UNIQUE)
    o.delete(gone)
    words, where = t.dump(with_where=True)
    assert np.array_equal(words, o.dump())
    assert where.min() >= -2 and where.max() < nb
    small = torch.zeros(len(o) // 2, dtype=torch.uint64, device="cuda")
    assert H.hive_dump(t.h, small) == len(o)
    got = host(small)
    assert np.unique(got).size == got.size and np.isin(got, words).all()
    t.close()


def _range_keys(n, lo):
    """n distinct valid keys whose dedupe hash (key times an odd constant) is
    lo, lo + 1, ...: all in one hash range of any batch size."""
    inv = pow(0x9E3779B1, -1, 1 << 32)
    h = (np.arange(n + 2, dtype=np.uint64) + np.uint64(lo)) & np.uint64(M32)
    k = (h * np.uint64(inv)) & np.uint64(M32)
    return k[(k != 0) & (k != M32)][:n].astype(np.uint32)


def _dedupe_rounds(H, keys, seed, n, set32=False):
    """An insert batch, a mixed batch and a delete batch of n operations each
    over `keys`, with repeats, against the dictionary."""
    rng = np.random.default_rng(seed)
    nb = max(1, int(np.ceil(keys.size / (0.6 * (32 if set32 else 16)))))
    t, o = make(H, 16, nb, set32, stash_capacity=max(1024, keys.size // 4)), oracle.O1()
    ins = keys[rng.integers(0, keys.size, n)]
    vals = np.zeros(n, np.uint32) if set32 else rng.integers(1, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
    t.insert(dev(ins), None if set32 else dev(vals))
    o.insert(ins, vals)
    assert t.stats()["live"] == len(o)
    pick = rng.integers(0, keys.size, n)
    ops = np.array([wl.OP_INSERT, wl.OP_DELETE, wl.OP_LOOKUP, wl.OP_DELETE], np.uint8)[pick % 4]
    v, f = t.mixed(dev(ops), dev(keys[pick]), dev(vals))
    ov, of = o.apply(ops, keys[pick], vals)
    assert np.array_equal(host(f), of)
    if not set32:
        assert np.array_equal(host(v), ov)
    gone = keys[rng.integers(0, keys.size, n)]
    assert np.array_equal(host(t.delete(dev(gone))), o.delete(gone))
    assert t.stats()["live"] == len(o)
    assert np.array_equal(t.dump(), o.dump())
    t.close()


@pytest.mark.parametrize("n", [1, 255, 1023, 1024, 1025, 1 << 14, (1 << 14) + 1, (1 << 17) + 1, (1 << 18) + 1, (1 << 20) + 1])
def test_dedupe_forms(H, n):
    """Batches at the edges of the dedupe's forms: with the probe in one block,
    one launch of several blocks, two launches and each of their chunk sizes."""
    case(f"dedupe n={n}")
    _dedupe_rounds(H, wl.KeyStream(600).range(0, max(4, n // 2)), 600 + n, n)


@pytest.mark.parametrize("set32", [False, True])
@pytest.mark.parametrize("n,distinct", [(12_000, 9_000), (200_000, 30_000), (1_500_000, 40_000)])
def test_dedupe_one_range(H, n, distinct, set32):
    """All keys in one hash range, more than its LDS table takes: the range is
    worked through in sub-ranges."""
    case(f"dedupe in one range n={n} distinct={distinct} set32={set32}")
    _dedupe_rounds(H, _range_keys(distinct, 0x40000000 - 1000), 700 + n, n, set32)


@pytest.mark.parametrize("n", [9_000, 300_000])
def test_dedupe_one_hot_key(H, n):
    """One key takes most of the batch: beyond the records a block holds."""
    case(f"dedupe with a hot key n={n}")
    keys = np.concatenate([np.full(30, 12345, np.uint32), wl.KeyStream(601).range(0, 10)])
    _dedupe_rounds(H, np.unique(keys), 800 + n, n)


def test_dedupe_beyond_four_million(H):
    """More than 2^22 operations: every range takes several sub-ranges."""
    n = 3 * (1 << 22) + 77
    case(f"dedupe n={n}")
    rng = np.random.default_rng(9)
    keys = wl.KeyStream(602).range(0, 1 << 23)
    ins = keys[rng.integers(0, keys.size, n)]
    vals = np.arange(1, n + 1, dtype=np.uint32)
    t, o = H.Table(int(np.ceil(keys.size / (0.7 * 16)))), oracle.O1(keys.size)
    t.insert(dev(ins), dev(vals))
    o.insert(ins, vals)
    assert np.array_equal(t.dump(), o.dump())
    gone = keys[rng.integers(0, keys.size, n)]
    assert np.array_equal(host(t.delete(dev(gone))), o.delete(gone))
    assert t.stats()["live"] == len(o)
    t.close()


def _linear(H, S, nb, mb, **cfg):
    return H.Table(nb, slots_per_bucket=S, addressing=H.HIVE_LINEAR, max_buckets=mb, **cfg)


def _check_linear(t, o, S, nb0, mb, geo):
    """Contents, key count, geometry (up to the equivalent form sp == im + 1)
    and every entry in a candidate bucket of the oracle's addressing."""
    st = t.stats()
    assert st["n_buckets"] == geo and st["live"] == len(o), st
    words, where = t.dump(with_where=True)
    assert np.array_equal(words, o.dump())
    o2 = oracle.O2(S, 8, 16, oracle.ADDR_LINEAR, nb0, max_buckets=mb)
    o2.split(geo - nb0)
    keys = (words & np.uint64(M32)).astype(np.uint32)[where >= 0]
    c1, c2 = o2.candidates(keys)
    w = where[where >= 0]
    assert ((w == c1) | (w == c2)).all()
    return st


@pytest.mark.parametrize("S", [16, 64])
@pytest.mark.parametrize("nb0,deltas", [(1, (1, 1, 2, 60, 4000)), (5, (3, 100, -70, 3000, -2500, 7)),
                                        (1000, (24, 2000, -2900, 5000))])
def test_resize_calls_over_several_rounds(H, S, nb0, deltas):
    """hive_resize over one hashing round and over many, up and down: with
    entries in the stash and the pending list, every key stays reachable and
    in place.  A merge may stop at a pair that does not fit, never beyond
    its target."""
    mb = 1 << 13
    n = nb0 * S + 40
    case(f"resize rounds S={S} nb0={nb0} deltas={deltas}")
    ks = wl.KeyStream(900 + nb0)
    keys = ks.range(0, n)
    t, o = _linear(H, S, nb0, mb, stash_capacity=16, pending_capacity=4096), oracle.O1()
    t.insert(dev(keys), dev(wl.values_for(keys)), flags=H.HIVE_UNIQUE)
    o.insert(keys, wl.values_for(keys))
    nb = nb0
    for d in deltas:
        t.resize(d)
        got = t.stats()["n_buckets"]
        if d > 0:
            assert got == min(mb, nb + d)
        else:
            assert max(nb0, nb + d) <= got <= nb
        nb = got
        _check_linear(t, o, S, nb0, mb, nb)
        q = ks.range(0, 2 * n)
        v, f = t.lookup(dev(q))
        ov, of = o.lookup(q)
        assert np.array_equal(host(f), of) and np.array_equal(host(v), ov)
    t.close()


@pytest.mark.parametrize("nb0,K,post", [(1, 1, 0), (8, 64, 0), (8, 5, 1), (100, 1000, 1)])
def test_growth_before_a_batch_keeps_the_stash_searchable(H, nb0, K, post):
    """Batches that replace, delete and look up stashed keys and, by their new
    keys, grow the table first (over one round or several): the stash is
    drained after the batch, so its entries must be found through the split."""
    S, mb = 16, 1 << 12
    case(f"growth with a stash nb0={nb0} K={K} post={post}")
    ks = wl.KeyStream(950 + nb0 + post)
    t = _linear(H, S, nb0, mb, pre_expand=1, post_policy=post, resize_k=K, lf_expand_pct=100 if not post else 97,
                lf_contract_pct=10, max_evictions=0, stash_capacity=4096, pending_capacity=4096)
    o = oracle.O1()
    at = nb0 * S  # exactly full by the rule: many entries cannot be in their buckets
    keys = ks.range(0, at)
    t.insert(dev(keys), dev(wl.values_for(keys)), flags=H.HIVE_UNIQUE)
    o.insert(keys, wl.values_for(keys))
    rng = np.random.default_rng(nb0)
    for b in range(5):
        live = np.unique((o.dump() & np.uint64(M32)).astype(np.uint32))
        perm = rng.permutation(live)
        a, c = perm.size // 3, 2 * perm.size // 3
        new = ks.range(at, at + nb0 * S * (1 + b % 2))
        at += new.size
        k = np.concatenate([perm[:a], new, perm[a:c], perm[c:]])
        ops = np.concatenate([np.full(a + new.size, wl.OP_INSERT), np.full(c - a, wl.OP_DELETE),
                              np.full(perm.size - c, wl.OP_LOOKUP)]).astype(np.uint8)
        p = rng.permutation(k.size)
        k, ops = k[p], ops[p]
        vals = rng.integers(1, 1 << 32, k.size, dtype=np.uint64).astype(np.uint32)
        v, f = t.mixed(dev(ops), dev(k), dev(vals))
        ov, of = o.apply(ops, k, vals)
        assert np.array_equal(host(f), of) and np.array_equal(host(v), ov), b
        st = t.stats()
        _check_linear(t, o, S, nb0, mb, st["n_buckets"])
    t.close()


def test_large_mixed_batch_counts_its_inserts(H):
    """Beyond 4,096 operations a mixed batch's inserts are counted by a launch
    of their own: growth by the rule on exactly that count, at odd sizes."""
    S, nb0, mb = 16, 64, 1 << 14
    ks = wl.KeyStream(970)
    o2 = oracle.O2(S, 8, 4096, oracle.ADDR_LINEAR, nb0, max_buckets=mb, resize_k=16)
    t = _linear(H, S, nb0, mb, pre_expand=1, resize_k=16)
    at = 0
    for n in (4096, 4097, 9001, 70_001):
        case(f"mixed growth n={n}")
        k = ks.range(at, at + n)
        at += n
        ops = np.where(np.arange(n) % 3 == 0, wl.OP_LOOKUP, wl.OP_INSERT).astype(np.uint8)
        live = t.stats()["live"]
        t.mixed(dev(ops), dev(k), dev(wl.values_for(k)))
        need, nb = live + int((ops == wl.OP_INSERT).sum()), o2.stats()["n_buckets"]
        while need * 100 > 90 * nb * S:
            nb += 16
        o2.split(nb - o2.stats()["n_buckets"])
        st = t.stats()
        assert st["n_buckets"] == nb and st["live"] == need, (n, st, nb)
    t.close()


@pytest.mark.parametrize("S,set32,cfg", [(16, False, {}), (64, False, {}), (32, True, {}), (16, False, {"hash_pair": 1}),
                                         (16, False, {"hash_pair": 2}), (16, False, {"max_evictions": 3}),
                                         (16, False, {"probe_both": 1}), (16, False, {"probe_tuning": 0x4444})])
def test_spilled_keys_stay_reachable(H, S, set32, cfg):
    """Tables with a spill filter (and the kinds without one) at 96% load,
    through rounds of deletes and inserts: keys in their second candidate and
    in the stash are found, replaced and deleted, before and after the first
    deletion, and the same batches through the executor."""
    nb = 257 if S == 16 else 65
    case(f"spilled keys S={S} set32={set32} {cfg}")
    n = int(nb * S * 0.96)
    ks = wl.KeyStream(1200 + S)
    t, o = make(H, S, nb, set32, stash_capacity=2048, pending_capacity=4096, **cfg), oracle.O1()
    rng = np.random.default_rng(1200)
    keys = ks.range(0, n)
    for part in np.array_split(keys, 5):  # the later parts meet full buckets
        t.insert(dev(part), dev(values(part, set32)), flags=H.HIVE_UNIQUE)
        o.insert(part, values(part, set32))
    q = ks.range(0, 3 * n)

    def check():
        v, f = t.lookup(dev(q))
        ov, of = o.lookup(q)
        assert np.array_equal(host(f), of)
        if not set32:
            assert np.array_equal(host(v), ov)
        assert np.array_equal(t.dump(), o.dump())

    check()
    at = n
    for r in range(4):
        again = rng.permutation(keys)[: n // 3]  # replaced where they are
        t.insert(dev(again), dev(values(again, set32) ^ np.uint32(0 if set32 else r + 1)))
        o.insert(again, values(again, set32) ^ np.uint32(0 if set32 else r + 1))
        gone = rng.permutation(keys)[: n // 4]
        assert np.array_equal(host(t.delete(dev(gone))), o.delete(gone))
        new = ks.range(at, at + n // 4)
        at += new.size
        keys = np.concatenate([np.setdiff1d(keys, gone), new])
        t.insert(dev(new), dev(values(new, set32)))
        o.insert(new, values(new, set32))
        check()
    if not set32 and "hash_pair" not in cfg:
        d = H.hive_drain_create(S, 0, 64, 1, 10_000_000)
        keep = []
        for r in range(6):
            pick = rng.permutation(q)[:900]
            ops = np.array([wl.OP_INSERT, wl.OP_DELETE, wl.OP_LOOKUP], np.uint8)[pick % 3]
            vals = rng.integers(1, 1 << 32, pick.size, dtype=np.uint64).astype(np.uint32)
            room = len(o) < n  # no growth past the table
            ops[(ops == wl.OP_INSERT) & (not room)] = wl.OP_LOOKUP
            import torch
            vo = torch.zeros(pick.size, dtype=torch.int32, device="cuda").view(torch.uint32)
            fo = torch.zeros(pick.size, dtype=torch.uint8, device="cuda")
            b = (dev(ops), dev(pick), dev(vals), vo, fo)
            keep.append((b, o.apply(ops, pick, vals)))
            assert H.hive_drain_submit(d, t.h, H.HIVE_OP_MIXED, b[1], b[2], b[0], vo, fo) is not None
        H.hive_drain_launch(d, 0)
        import torch
        torch.cuda.synchronize()
        for (_, _, _, vo, fo), (ov, of) in keep:
            assert np.array_equal(host(fo), of) and np.array_equal(host(vo), ov)
        H.hive_drain_destroy(d)
        check()
    t.close()


@pytest.mark.parametrize("nb", [1 << 21, (1 << 21) + 1])
@pytest.mark.parametrize("n", [1 << 24, (1 << 24) + 1])
def test_large_lookups_on_both_sides_of_the_variant_rule(H, nb, n):
    """Buckets of 256 MiB and just beyond, looked up by 2^24 keys and one
    more, with keys that were never there and keys in either bucket."""
    case(f"large lookups nb={nb} n={n}")
    import torch
    keys = wl.KeyStream(31).range(0, 1 << 16)
    t = make(H, 16, nb)
    t.insert(dev(keys), dev(wl.values_for(keys)))
    gone = keys[::5]
    assert host(t.delete(dev(gone))).all()
    q = np.resize(np.concatenate([keys, wl.KeyStream(31).range(1 << 16, (1 << 16) + 7919)]), n)
    v, f = t.lookup(dev(q))
    there = np.ones(keys.size + 7919, bool)
    there[keys.size:] = False
    there[: keys.size : 5] = False
    there = np.resize(there, n)
    assert np.array_equal(host(f).astype(bool), there)
    assert np.array_equal(host(v), np.where(there, wl.values_for(q), np.uint32(M32)))
    t.close()
