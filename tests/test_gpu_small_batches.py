"""Small batches take one-workgroup kernels: the selection (up to 1024 lanes,
and 65536 blocks to list, one more for 8 of the pool, for more than 4 claims),
the restore (up to 1024 claims) and the check's tail (up to 1024 lanes and
positions, 32768 partials, and as many tokens as one CU hashes); larger ones
the kernels split over workgroups.
At and around those edges both must give the oracle's digests, outcomes and
events: each group width, a claim of several windows, faults, missing
entries, malformed and empty rows, an event log that just holds the call's
events, and pools past the LDS bitmap.  An offload's front (up to 1024 claims and 8192 lanes)
and tail follow the same pattern: acceptance, duplicate ids, identities shared
within and across batches, backward rows, staging."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_01387_amd.synth import MISSING, TINY, FaultSpec, Geometry, Workload, content, from_claims
from tests.helpers import apply_flips, digests
from tests.test_gpu_parity import free_gpu, gpu_pool_tensor, note, same_events, same_outcomes

pytestmark = pytest.mark.gpu

# (claims, blocks per claim): widths 2..64; lanes 1024 and past; positions
# 1024 and past; claims 1024 and past; events 4096 and past
BATCHES = [(1, 1), (1, 200), (16, 64), (17, 60), (32, 32), (33, 32), (512, 2), (513, 2), (128, 8),
           (128, 9), (1, 1024), (1, 1025), (1024, 1), (1025, 1), (4096, 1), (4097, 1)]
# 1 and 40 piece groups; 262144 and 262145 blocks fill the bitmap and pass it
POOLS = {"1-group": Geometry(2, 2, 4, 1, 8, 2, 300), "40-groups": Geometry(80, 2, 4, 1, 8, 2, 1024),
         "bitmap-full": Geometry(1, 1, 2, 1, 8, 1, 262144),
         "past-bitmap": Geometry(1, 1, 2, 1, 8, 1, 262145)}


def small_batch(g, claims, blocks, rng):
    parts = []
    for i in range(claims):
        n = max(1, blocks - int(rng.integers(0, 2)))
        blk = rng.integers(0, g.num_blocks, n).astype(np.uint32)
        tok = rng.integers(0, 32000, n * g.block_size - int(rng.integers(0, g.block_size)))
        kind = rng.integers(0, 12) if claims > 4 else 9
        if kind == 0:
            blk[rng.integers(0, n)] = MISSING
        elif kind == 1:
            tok = tok[: max(0, tok.size - g.block_size)]
        elif kind == 2:
            blk, tok = blk[:0], tok[:0]
        parts.append((1000 + 7 * i, blk, tok.astype(np.uint32)))
    b = from_claims(parts)
    if claims > 8:
        b.claim_ids[3] = 0xFFFFFFFFFFFFFFFF  # a reserved id: a malformed row
    return b


# the large pools repeat three batches, and one lists many blocks on both sides
# of the line
CASES = [(p, c, n) for p in POOLS for c, n in BATCHES
         if POOLS[p].num_blocks < 2000 or (c, n) in ((1, 200), (32, 32), (33, 32))]
CASES += [("bitmap-full", 16, 6140), ("bitmap-full", 16, 6160), ("bitmap-full", 4, 25000)]


@pytest.mark.parametrize("pool,claims,blocks", CASES, ids=[f"{p}-{c}x{n}" for p, c, n in CASES])
def test_small_batch(torch, ck, pool, claims, blocks):
    check_batch(torch, ck, POOLS[pool], pool, claims, blocks)


def check_batch(torch, ck, g, pool, claims, blocks):
    rng = np.random.default_rng(claims * 1000 + blocks)
    w = Workload(name=f"small-{pool}", geometry=g, seed=77, num_claims=0, length=TINY.length,
                 sharing=TINY.sharing, corrupt_rate=0.0, gen_seed=1, content_seed=9)
    batch = small_batch(g, claims, blocks, rng)
    seen = batch.unique_blocks(g.num_blocks)
    nf = min(3, seen.size)
    faults = FaultSpec(rng.choice(seen, nf, replace=False).astype(np.uint32),
                       rng.integers(0, 8 * g.block_bytes, nf).astype(np.uint64),
                       rng.choice(seen, min(2, seen.size), replace=False).astype(np.uint32))
    note(f"small batch {pool} {claims} x {blocks}: {batch.num_refs} refs")
    host = content.pool_host(g, w.content_seed)
    d0, d1 = digests(host, w, seen), digests(apply_flips(host, w, faults), w, seen)
    op = O.OraclePool(g.num_blocks, g.block_size, w.seed)
    assert op.offload(batch, d0) == O.OK
    assert op.restore(batch, faults.load_failed) == O.OK
    want = op.check(batch, d1)
    kv = gpu_pool_tensor(torch, w)
    C = batch.num_claims
    with ck.Pool(g, w.seed, kv, max_claims=C, max_footprint=batch.num_refs,
                 event_capacity=5 * C) as p:
        db = ck.DeviceBatch(batch)
        p.offload(db)
        p.restore(db, faults=faults)
        p.check(db)
        out, ev = p.read()
        st = p.block_state()
        # (the log held exactly the worst case of the three calls)
        p.check(db)
        p.check(db)
        again, ev2 = p.read()
    same_outcomes(out, want)
    same_outcomes(again, want)
    want_ev = op.events()
    same_events(ev, want_ev)
    per = (len(ev2) // 2)
    assert len(ev2) == 2 * per
    assert np.array_equal(ev2["seq"], ev["seq"][-1] + 1 + np.arange(len(ev2), dtype=np.uint64))
    for f in ("claim_id", "aux", "kind", "block_index", "phys_block"):
        assert np.array_equal(ev2[f][:per], ev[f][-per:]) and np.array_equal(ev2[f][per:], ev[f][-per:])
    recorded = np.flatnonzero(st["valid_off"])
    assert np.array_equal(st["d_off"][recorded], d0[recorded])
    assert np.array_equal(st["d_res"][recorded], d1[recorded])
    del kv
    free_gpu(torch)


# the check's tail by its tokens: positions x tokens 20 Mi and past for narrow
# groups and for 256 lanes and more; 256 tokens per lane, and blocks of 128
# tokens and more, where wide groups fill up to 256 lanes
TOKENS = [(32, 512, 1), (64, 512, 1), (128, 512, 1), (32, 24, 30), (64, 24, 30), (64, 1, 250),
          (64, 1, 270), (129, 1, 30), (128, 4, 128), (128, 4, 130), (1024, 40, 2), (1024, 4, 16)]


@pytest.mark.parametrize("bs,claims,blocks", TOKENS, ids=[f"{b}-{c}x{n}" for b, c, n in TOKENS])
def test_small_tail_tokens(torch, ck, bs, claims, blocks):
    check_batch(torch, ck, Geometry(2, 1, bs, 1, 16, 1, 700), f"{bs}-tokens", claims, blocks)


# the front's edges: claims 1024 and past, lanes (claims x width) 8192 and past,
# 8229 positions and past (8192 and one for 8 of the 300 blocks) where claims
# have more than 1024 lanes; the tail's: 256 positions and past for more than
# 256 claims, 512 and past for more than 4, 1024 and past for up to 4
FRONT = [(1, 3), (16, 64), (17, 64), (32, 20), (33, 20), (128, 64), (129, 64), (512, 2), (513, 2),
         (1024, 4), (1024, 9), (1025, 1), (128, 66), (24, 340), (24, 512), (16, 1000),
         (256, 1), (257, 1), (128, 4), (64, 9), (5, 104), (4, 200), (4, 256), (4, 258)]


def family_batch(g, claims, blocks, rng, base, first=None):
    """Claims whose leading blocks are often another's, tokens and blocks or
    tokens alone (the same identity on another block is ambiguous)."""
    parts = [] if first is None else list(first)
    made = []
    for i in range(claims):
        n = max(1, blocks - int(rng.integers(0, 2)))
        blk = rng.integers(0, g.num_blocks, n).astype(np.uint32)
        tok = rng.integers(0, 32000, n * g.block_size).astype(np.uint32)
        if parts and rng.random() < 0.6:
            _, b0, t0 = parts[int(rng.integers(len(parts)))]
            k = int(rng.integers(0, min(n, len(b0), len(t0) // g.block_size) + 1))
            tok[: k * g.block_size] = t0[: k * g.block_size]
            if rng.random() < 0.7:
                blk[:k] = b0[:k]
        parts.append((base + i, blk, tok))
        made.append(parts[-1])
    return made


@pytest.mark.parametrize("claims,blocks", FRONT, ids=[f"{c}x{n}" for c, n in FRONT])
@pytest.mark.parametrize("staged", [False, True], ids=["plain", "staged"])
def test_small_offload(torch, ck, claims, blocks, staged):
    g = Geometry(2, 2, 4, 1, 8, 2, 300)
    rng = np.random.default_rng(claims * 77 + blocks)
    w = Workload(name="small-offload", geometry=g, seed=78, num_claims=0, length=TINY.length,
                 sharing=TINY.sharing, corrupt_rate=0.0, gen_seed=1, content_seed=10)
    one = family_batch(g, claims, blocks, rng, 10)
    two = family_batch(g, claims, blocks, rng, 100000, first=one)
    batches = [from_claims(one), from_claims(two)]
    if claims > 8:  # rows that share entries: one row runs backwards
        third = from_claims(family_batch(g, claims, blocks, rng, 200000, first=two))
        third.block_offsets[4] = third.block_offsets[2]
        batches.append(third)
    note(f"small offload {claims} x {blocks} {'staged' if staged else ''}")
    host = content.pool_host(g, w.content_seed)
    d0 = digests(host, w)
    op = O.OraclePool(g.num_blocks, g.block_size, w.seed)
    kv = gpu_pool_tensor(torch, w)
    refs = sum(b.num_refs for b in batches) + 4 * blocks
    staging = torch.zeros(3 * 300 * g.block_bytes, dtype=torch.uint8, device="cuda") if staged else None
    with ck.Pool(g, w.seed, kv, max_claims=4 * claims, max_footprint=2 * refs,
                 event_capacity=64 * claims + 64) as p:
        slot = 0
        for b in batches:
            db = ck.DeviceBatch(b)
            assert op.offload(b, d0) == O.OK
            p.offload(db, staging=staging)
            if staged:
                ok = np.arange(b.num_claims)[np.diff(b.block_offsets.astype(np.int64)) >= 0]
                seen = np.unique(np.concatenate([b.block_ids[b.block_offsets[c]:b.block_offsets[c + 1]]
                                                 for c in ok]))
                got = staging.cpu().numpy().reshape(-1, g.block_bytes)[slot:slot + seen.size]
                want = host.reshape(g.planes, g.num_blocks, -1).transpose(1, 0, 2)[seen]
                assert np.array_equal(got, want.reshape(seen.size, -1))
                slot += seen.size
            # the same ids again, one id twice in a batch: refused, nothing changes
            with pytest.raises(ck.ClaimError) as e:
                p.offload(db)
            assert e.value.status == ck.EDUP
        if claims > 1:
            twice = family_batch(g, claims, blocks, rng, 300000)
            twice[-1] = (twice[0][0],) + twice[-1][1:]
            with pytest.raises(ck.ClaimError) as e:
                p.offload(ck.DeviceBatch(from_claims(twice)))
            assert e.value.status == ck.EDUP
        assert p.identity_stats() == op.identity_stats()
        for b in batches:
            db = ck.DeviceBatch(b)
            p.restore(db, staging=staging)
            assert op.restore(b) == O.OK
            p.check(db)
            out = op.check(b, d0)
        got, ev = p.read()
        same_outcomes(got, out)
        same_events(ev, op.events())
        for b in batches:
            lk, want = p.lookup(ck.DeviceBatch(b)), op.lookup(b)
            for f in want.dtype.names:
                if f != "pad":
                    assert np.array_equal(lk[f], want[f]), f
    del kv, staging
    free_gpu(torch)
