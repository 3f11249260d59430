"""outcomes_read takes small reads through the pool's page-locked memory,
large ones straight into page-locked caller memory, and copies into pageable
memory otherwise; lookup takes few results through page-locked memory.  All
must give the same records at and around the 64 KiB edge, at odd addresses,
and with capacities that just hold the records or do not."""

import ctypes

import numpy as np
import pytest

from paper_2606_01387_amd.synth import FULL, from_claims, make_batch, make_faults, make_requests, scaled
from tests.test_gpu_parity import free_gpu, gpu_pool_tensor, note

pytestmark = pytest.mark.gpu


def pinned(torch, dtype, n, shift=0):
    """n records in page-locked memory, `shift` bytes past its start."""
    mem = torch.empty(n * dtype.itemsize + shift, dtype=torch.uint8, pin_memory=True)
    mem.fill_(0xA5)
    return mem, mem.numpy()[shift:].view(dtype)


# 16-byte header and 64 + 40..80 bytes per claim (past 16 MiB the copies serve
# page-locked memory too): 64 KiB hold the bound of
# 455 claims (64 + 2 x 40 bytes each), not of 456
@pytest.mark.parametrize("claims", [1, 454, 455, 456, 600, 1500, 20000, 150000])
def test_read_paths(torch, ck, claims):
    w = scaled(FULL["small-claim-stress"], 128, claims, corrupt_rate=0.05)
    batch = make_batch(w)
    C = batch.num_claims
    note(f"read paths: {C} claims")
    kv = gpu_pool_tensor(torch, w)
    with ck.Pool(w.geometry, w.seed, kv, max_claims=2 * C, max_footprint=2 * batch.num_refs,
                 event_capacity=8 * C) as p:
        db = ck.DeviceBatch(batch)
        p.offload(db)
        p.restore(db, faults=make_faults(w, batch))
        p.read()
        p.check(db)
        want, want_ev = p.read()  # pageable, freshly made
        n_ev = want_ev.size
        seq = int(want_ev["seq"][0])
        calls = 0

        def same(out, ev):
            nonlocal calls
            calls += 1
            assert np.array_equal(out, want)
            assert ev.size == n_ev
            for f in ("claim_id", "aux", "kind", "block_index", "phys_block"):
                assert np.array_equal(ev[f], want_ev[f]), f
            assert np.array_equal(ev["seq"], seq + calls * n_ev + np.arange(n_ev, dtype=np.uint64))

        for shift, extra in ((0, 0), (0, 5), (8, 3), (4, 2), (1, 0)):
            om, out = pinned(torch, ck.OUTCOME_DTYPE, C + extra, shift)
            em, ev = pinned(torch, ck.EVENT_DTYPE, n_ev + extra, shift)
            p.check(db)
            same(*p.read(out=out, events=ev))
            tail = np.concatenate([out[C:].view(np.uint8), ev[n_ev:].view(np.uint8)])
            assert (tail == 0xA5).all()  # nothing past the records is written
        p.check(db)
        same(*p.read(max_outcomes=C, max_events=n_ev))
        # one of the two page-locked
        om, out = pinned(torch, ck.OUTCOME_DTYPE, C)
        p.check(db)
        same(*p.read(out=out, events=np.zeros(n_ev, ck.EVENT_DTYPE)))
        # a capacity one short: refused, nothing dropped, then read whole
        em, ev = pinned(torch, ck.EVENT_DTYPE, n_ev)
        p.check(db)
        for o, e in ((out, ev[:-1]), (out[:-1], ev), (out, np.zeros(n_ev - 1, ck.EVENT_DTYPE))):
            with pytest.raises(ck.ClaimError) as err:
                p.read(out=o, events=e)
            assert err.value.status == ck.ENOSPC
        same(*p.read(out=out, events=ev))
        # outcomes alone keep the events; events alone leave the outcomes
        p.check(db)
        n = ctypes.c_uint32()
        lib = ck.lib()
        om, out = pinned(torch, ck.OUTCOME_DTYPE, C)
        assert lib.outcomes_read(p._h, out.ctypes.data, C, ctypes.byref(n), None, 0, None) == ck.OK
        assert n.value == C and np.array_equal(out, want)
        k = ctypes.c_uint64()
        assert lib.outcomes_read(p._h, None, 0, None, ev.ctypes.data, n_ev, ctypes.byref(k)) == ck.OK
        assert k.value == n_ev
        same(out, ev)
        assert lib.outcomes_read(p._h, None, 0, None, None, 0, None) == ck.OK
        assert lib.outcomes_read(p._h, None, 0, None, ev.ctypes.data, 0, ctypes.byref(k)) == ck.OK
        assert k.value == 0
    del kv
    free_gpu(torch)


@pytest.mark.parametrize("requests", [1, 65, 4096, 4097])
def test_lookup_paths(torch, ck, requests):
    w = scaled(FULL["small-claim-stress"], 128, 300)
    batch = make_batch(w)
    reqs, _ = make_requests(w, batch, num_requests=requests)
    kv = gpu_pool_tensor(torch, w)
    with ck.Pool(w.geometry, w.seed, kv) as p:
        p.offload(ck.DeviceBatch(batch))
        d = ck.DeviceBatch(reqs)
        dev = p.lookup_async(d)
        torch.cuda.synchronize()
        want = dev.cpu().numpy().view(ck.LOOKUP_DTYPE)[:requests]
        first = p.lookup(d)
        none = p.lookup(ck.DeviceBatch(from_claims([])))
        assert none.size == 0
        assert np.array_equal(first, want) and np.array_equal(p.lookup(d), want)
        assert np.array_equal(first, want)  # the first call's records are the caller's own
    del kv
    free_gpu(torch)


def test_lookup_during_a_lookup(torch, ck):
    """A lookup that another thread makes while one waits for its results
    (here from within the call, after its launch) takes memory of its own."""
    w = scaled(FULL["small-claim-stress"], 128, 300)
    batch = make_batch(w)
    reqs, _ = make_requests(w, batch, num_requests=100)
    kv = gpu_pool_tensor(torch, w)
    with ck.Pool(w.geometry, w.seed, kv) as p:
        p.offload(ck.DeviceBatch(batch))
        d, other = ck.DeviceBatch(reqs), ck.DeviceBatch(batch)
        want, want_other = p.lookup(d), p.lookup(other)
        assert not np.array_equal(want, want_other[: want.size])
        queue, inner = p.lookup_async, []

        def lookup_async(b, out=None):
            queue(b, out)
            if b is d:
                inner.append(p.lookup(other))

        p.lookup_async = lookup_async
        assert np.array_equal(p.lookup(d), want)
        assert np.array_equal(inner[0], want_other)
    del kv
    free_gpu(torch)
