"""A refused offload reads no block: the digest that an offload queues before
it waits for the verdict finds none where ids repeat or rows may share
entries, and is not queued where the footprint cannot fit.  So a refusal takes
far less time than an accepted offload of the same blocks (half is the line: a
refusal that waits for the digest takes nine tenths of it, one that does not
less than a fifth), for the one-workgroup front and the larger one, and it
leaves nothing behind that the next offload meets."""

import time

import numpy as np
import pytest

from paper_2606_01387_amd.synth import Geometry, from_claims
from tests.test_gpu_parity import free_gpu, note

pytestmark = pytest.mark.gpu

# 2 GiB in 2 MiB blocks; 2 GiB in 9-row chunks (pieces across chunk ends)
POOLS = {"whole-pieces": Geometry(32, 2, 16, 8, 128, 2, 1024),
         "runs": Geometry(61, 1, 8, 1, 576, 1, 7600)}


def timed(torch, call):
    torch.cuda.synchronize()
    t = time.perf_counter()
    call()
    return time.perf_counter() - t


@pytest.mark.parametrize("claims", [64, 600, 1100])  # one workgroup's front up to 1024 claims
@pytest.mark.parametrize("pool", POOLS)
def test_refused_offload(torch, ck, pool, claims):
    g = POOLS[pool]
    rng = np.random.default_rng(claims)
    order = rng.permutation(g.num_blocks)
    bs = g.block_size
    parts = [order[c::claims] if c < order.size else order[:1] for c in range(claims)]

    def batch(base):
        return from_claims([(base + i, p, rng.integers(0, 32000, len(p) * bs).astype(np.uint32))
                            for i, p in enumerate(parts)])

    note(f"refusals {pool}: {claims} claims")
    kv = torch.randint(0, 255, (g.pool_bytes,), dtype=torch.uint8, device="cuda")
    first = batch(1)
    refs = first.num_refs
    with ck.Pool(g, 11, kv, max_claims=8 * claims, max_footprint=6 * refs + 64,
                 event_capacity=32 * claims) as p:
        accepted, refused = [], []
        for k in range(3):
            db = ck.DeviceBatch(batch(1 + k * 100000))
            accepted.append(timed(torch, lambda: p.offload(db)))
            for _ in range(4):
                def again():
                    with pytest.raises(ck.ClaimError) as e:
                        p.offload(db)
                    assert e.value.status == ck.EDUP
                refused.append(timed(torch, again))
            p.read()
        want = p.block_state()["d_off"]
        # rows that share entries, refused for an id and then accepted whole
        shared = batch(900000)
        shared.block_offsets[4] = shared.block_offsets[2]
        known = batch(900000)
        known.claim_ids[-1] = first.claim_ids[0]
        known.block_offsets[:] = shared.block_offsets
        with pytest.raises(ck.ClaimError) as e:
            p.offload(ck.DeviceBatch(known))
        assert e.value.status == ck.EDUP
        p.offload(ck.DeviceBatch(shared))
        db = ck.DeviceBatch(shared)
        p.restore(db)
        p.check(db)
        out, _ = p.read()
        assert set(out["code"]) <= {ck.MATERIALIZED, ck.UNKNOWN}
        st = p.block_state()
        assert np.array_equal(st["d_off"], want)
        assert np.array_equal(st["d_res"][st["d_res"] != 0], want[st["d_res"] != 0])
    with ck.Pool(g, 11, kv, max_claims=8 * claims, max_footprint=2 * refs - 1,
                 event_capacity=32 * claims) as p:
        p.offload(ck.DeviceBatch(first))
        db = ck.DeviceBatch(batch(100000))
        full = []
        for _ in range(4):
            def over():
                with pytest.raises(ck.ClaimError) as e:
                    p.offload(db)
                assert e.value.status == ck.ENOSPC
            full.append(timed(torch, over))
        assert np.array_equal(p.block_state()["d_off"], want)
    note(f"accepted {min(accepted) * 1e6:.0f} us, known ids {min(refused) * 1e6:.0f} us, "
         f"full {min(full) * 1e6:.0f} us")
    assert min(refused) < min(accepted) / 2 and min(full) < min(accepted) / 2
    del kv
    free_gpu(torch)
