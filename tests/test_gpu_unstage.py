"""Staged blocks return to the pool in pieces of 2048 16-byte words of a block
where they, their bytes and their chunks are large enough and staging is device
memory, word by word otherwise; large staged offloads to device memory write
past the caches.  Sizes on both sides
of each line, pieces that end inside a chunk and cross chunk ends, and every
kind of digest piece: staging must hold the blocks' bytes, every restored
block its bytes again, in whatever order its claims stage and restore it, and
every other block must stay untouched."""

import numpy as np
import pytest

from paper_2606_01387_amd.synth import TINY, Geometry, Workload, from_claims
from tests.test_gpu_parity import free_gpu, gpu_pool_tensor, note

pytestmark = pytest.mark.gpu

# layers, planes per layer, block size, heads, dim, element bytes, blocks
CASES = [
    Geometry(1, 1, 2, 1, 8, 1, 300),  # blocks of one word
    Geometry(1025, 1, 2, 1, 8, 1, 40),  # 16-byte chunks
    Geometry(7, 1, 64, 1, 576, 1, 60),  # few bytes
    Geometry(8, 2, 16, 1, 256, 2, 890),  # just under and past 112 MiB
    Geometry(8, 2, 16, 1, 256, 2, 905),
    Geometry(8, 2, 1, 1, 8176, 1, 1900),  # chunks just under 8 KiB
    Geometry(15, 1, 16, 1, 256, 2, 2000),  # blocks of just under 4 pieces
    Geometry(8, 2, 16, 1, 256, 2, 1900),  # 4 whole chunks a piece, 4 pieces a block
    Geometry(17, 1, 1, 1, 8208, 1, 1800),  # chunks of 513 words
    Geometry(1, 1, 1, 1, 524304, 1, 470),  # one chunk of 16 pieces and a word
    Geometry(7, 1, 64, 1, 576, 1, 980),  # 36 KiB chunks
    # past 448 MiB: each kind of digest piece stores its stream
    Geometry(32, 2, 16, 8, 128, 2, 240),
    Geometry(61, 1, 64, 1, 576, 1, 230),
    Geometry(80, 2, 16, 1, 128, 2, 760),
    Geometry(61, 1, 8, 1, 576, 1, 1750),
    Geometry(17, 2, 24, 3, 80, 2, 1260),
]


@pytest.mark.parametrize("g", CASES, ids=[f"{g.chunk_bytes}Bx{g.planes}x{g.num_blocks}" for g in CASES])
def test_unstage(torch, ck, g):
    round_trips(torch, ck, g, "device")


# page-locked host memory past the lines that device staging has (112 MiB back,
# 448 MiB out): whole pieces and pieces across chunk ends
HOST = [Geometry(7, 1, 64, 1, 576, 1, 600), Geometry(32, 2, 16, 8, 128, 2, 240),
        Geometry(61, 1, 8, 1, 576, 1, 1750)]


@pytest.mark.parametrize("g", HOST, ids=[f"{g.chunk_bytes}Bx{g.planes}x{g.num_blocks}" for g in HOST])
def test_unstage_host(torch, ck, g):
    round_trips(torch, ck, g, "host")


def round_trips(torch, ck, g, where):
    rng = np.random.default_rng(g.chunk_bytes + g.planes)
    w = Workload(name="unstage", geometry=g, seed=5, num_claims=0, length=TINY.length,
                 sharing=TINY.sharing, corrupt_rate=0.0, gen_seed=1, content_seed=7)
    note(f"unstage from {where} memory {g.chunk_bytes} B x {g.planes} planes, {g.num_blocks} blocks")
    kv = gpu_pool_tensor(torch, w)
    pool = kv.view(g.planes, g.num_blocks, g.chunk_bytes)
    want = pool.clone()
    order = rng.permutation(g.num_blocks)[: g.num_blocks - 3]
    claims = [(i + 1, [int(b)], rng.integers(0, 32000, g.block_size)) for i, b in enumerate(order)]
    batch, part = from_claims(claims), from_claims([claims[4], claims[0]])
    staging = torch.zeros(order.size * g.block_bytes, dtype=torch.uint8,
                          **(dict(device="cuda") if where == "device" else dict(pin_memory=True)))
    with ck.Pool(g, w.seed, kv, max_claims=4096, max_footprint=4096, event_capacity=32768) as p:
        p.offload(ck.DeviceBatch(batch), staging=staging)
        used = torch.from_numpy(np.sort(order)).cuda()
        rows = staging.view(order.size, g.planes, g.chunk_bytes)
        torch.cuda.synchronize()
        assert all(torch.equal(rows[:, l].cuda(), want[l, used]) for l in range(g.planes))
        for b, blocks in ((part, order[[4, 0]]), (from_claims([]), order[:0]), (batch, order)):
            pool.fill_(0x5A)
            p.restore(ck.DeviceBatch(b), staging=staging)
            torch.cuda.synchronize()
            back = torch.zeros(g.num_blocks, dtype=torch.bool, device="cuda")
            back[torch.from_numpy(blocks).cuda()] = True
            for l in range(g.planes):
                assert torch.equal(pool[l, back], want[l, back])
                assert bool((pool[l, ~back] == 0x5A).all())
    del kv, pool, want, staging, rows
    free_gpu(torch)


@pytest.mark.parametrize("blocks", [60, 119, 230])
def test_many_references(torch, ck, blocks):
    """Few blocks under many references (2 to 4 GB of them): the blocks that
    are staged decide how they are copied."""
    g = Geometry(32, 2, 16, 8, 128, 2, 700)
    rng = np.random.default_rng(blocks)
    w = Workload(name="references", geometry=g, seed=5, num_claims=0, length=TINY.length,
                 sharing=TINY.sharing, corrupt_rate=0.0, gen_seed=1, content_seed=7)
    note(f"many references to {blocks} blocks")
    kv = gpu_pool_tensor(torch, w)
    pool = kv.view(g.planes, g.num_blocks, g.chunk_bytes)
    want = pool.clone()
    used = np.sort(rng.choice(g.num_blocks, blocks, replace=False))
    batch = from_claims([(i + 1, rng.permutation(used)[:50], rng.integers(0, 32000, 50 * 16))
                         for i in range(40)])
    used = batch.unique_blocks(g.num_blocks)
    staging = torch.zeros(used.size * g.block_bytes, dtype=torch.uint8, device="cuda")
    with ck.Pool(g, w.seed, kv, max_claims=64, max_footprint=4096, event_capacity=4096) as p:
        db = ck.DeviceBatch(batch)
        p.offload(db, staging=staging)
        pool.fill_(0x5A)
        p.restore(db, staging=staging)
        p.check(db)
        out, _ = p.read()
    assert (out["code"] == ck.MATERIALIZED).all()
    back = torch.zeros(g.num_blocks, dtype=torch.bool, device="cuda")
    back[torch.from_numpy(used.astype(np.int64)).cuda()] = True
    for l in range(g.planes):
        assert torch.equal(pool[l, back], want[l, back])
        assert bool((pool[l, ~back] == 0x5A).all())
    del kv, pool, want, staging
    free_gpu(torch)
