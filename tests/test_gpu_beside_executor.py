"""Plain calls on other tables while a resident executor waits for work: small
batches, deduped batches, a resize down and an export find room beside its
blocks.  (The executor gives up after some seconds without progress, so that
calls which found none would end all the same, late and with its error.)"""
import gc
import time

import numpy as np
import pytest

import oracle
from paper_2510_15095_amd import workload as wl
from test_gpu_batch_paths import H, case, dev, host  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [16, 32])
@pytest.mark.parametrize("blocks", [0, 1])  # per compute unit; 0: one less than fit
def test_plain_calls_run_beside_a_resident_executor(H, S, blocks):  # noqa: F811
    import torch
    ns = [100, 1024, 1 << 14, 1 << 18]
    ks = wl.KeyStream(81)
    sets = [ks.range(0, n)[np.random.default_rng(n).integers(0, n, n)] for n in ns]
    o = oracle.O1()
    for kh in sets:
        o.insert(kh, wl.values_for(kh)[::-1])
    want = o.dump()
    sets = [(dev(k), dev(wl.values_for(k)[::-1])) for k in sets]
    # more pairs than merge_kernel's blocks take in one run, so that all are at work
    t = H.Table(1 << 15, slots_per_bucket=S, addressing=H.HIVE_LINEAR, max_batch=1 << 18, max_buckets=1 << 16)
    words = torch.empty(want.size + 1, dtype=torch.uint64, device="cuda")

    def calls():
        at = [("start", time.time())]
        for k, v in sets:
            t.insert(k, v)
            torch.cuda.current_stream().synchronize()
            at.append((f"insert {k.numel()}", time.time()))
        t.resize(1 << 15)
        t.resize(-(1 << 15))
        torch.cuda.current_stream().synchronize()
        at.append(("resize", time.time()))
        n = H.hive_dump(t.h, words)
        at.append(("export", time.time()))
        return n, [(b[0], b[1] - a[1]) for a, b in zip(at, at[1:])]

    calls()  # code loaded, scratch allocated
    t.clear()
    d = H.hive_drain_create(S, blocks, 4, 4, 4_000_000)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    case(f"calls beside the executor, S {S}, blocks {blocks}")
    gc.collect()  # a table of an earlier test that is freed meanwhile waits for the whole device
    gc.disable()
    try:
        H.hive_drain_launch(d, 1, side)
        n, took = calls()
    finally:
        gc.enable()
    print(took, flush=True)
    assert max(s for _, s in took) < 1.0, f"a call waited for the executor: {took}"
    H.hive_drain_stop(d, side)
    H.hive_drain_destroy(d)
    got = host(words[:n])
    assert np.array_equal(got[np.argsort(got & np.uint64(0xFFFFFFFF), kind="stable")], want)
