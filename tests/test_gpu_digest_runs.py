"""Chunks that no piece of 24, 16 or 8 rows divides are digested in pieces that
run across chunk ends.  Each width the kernel has (1, 2, 4, 8 and 20 words per
lane), chunks of whole rows and chunks that end inside a row, chunks shorter
than a row, a last piece that ends inside the block's last chunk, a last piece
group with idle waves, head shards, few and many blocks per workgroup: every
block's digest before and after flips must be the oracle's, and a staged copy
the block's bytes."""

import numpy as np
import pytest

from oracle import oracle as O  # noqa: F401
from paper_2606_01387_amd.synth import TINY, FaultSpec, Geometry, Workload, content, from_claims
from tests.helpers import apply_flips, digests
from tests.test_gpu_parity import free_gpu, gpu_pool_tensor, note

pytestmark = pytest.mark.gpu

# (geometry, words per lane): layers, planes per layer, block size, heads,
# dim, element bytes, blocks
CASES = [
    (Geometry(1, 1, 2, 1, 8, 1, 500), 1),  # 16-byte chunks: one row holds a block
    (Geometry(3, 1, 8, 1, 64, 1, 900), 1),  # 3 rows
    (Geometry(3, 2, 8, 1, 64, 1, 700), 2),  # 6 rows: one idle wave
    (Geometry(5, 1, 8, 1, 72, 1, 300), 2),  # chunks of 1.125 rows
    (Geometry(7, 2, 8, 1, 64, 1, 300), 4),  # 14 rows
    (Geometry(2, 2, 4, 1, 24, 2, 300), 1),  # chunks shorter than a row (192 bytes)
    (Geometry(9, 1, 8, 1, 576, 1, 600), 8),  # 9-row chunks
    (Geometry(5, 2, 16, 3, 72, 2, 200), 4),  # 13.5 rows
    (Geometry(40, 1, 16, 1, 40, 1, 300), 8),  # 40 planes of 1.25 rows
    (Geometry(40, 2, 8, 1, 64, 1, 300), 20),  # 80 rows in 4 pieces
    (Geometry(71, 1, 8, 1, 72, 1, 200), 20),  # 71 planes of 1.125 rows: 79.9 rows
    (Geometry(3, 2, 16, 1, 72, 2, 150, total_kv_heads=4, first_kv_head=2), 8),  # a head shard
    (Geometry(2, 1, 24, 5, 96, 1, 100, total_kv_heads=15, first_kv_head=5), 4),
]


@pytest.mark.parametrize("g,lpw", CASES, ids=[f"{g.chunk_bytes}Bx{g.planes}" for g, _ in CASES])
def test_runs(torch, ck, g, lpw):
    rng = np.random.default_rng(g.chunk_bytes + g.planes)
    w = Workload(name="runs", geometry=g, seed=int(rng.integers(1 << 62)), num_claims=0,
                 length=TINY.length, sharing=TINY.sharing, corrupt_rate=0.0, gen_seed=1,
                 content_seed=int(rng.integers(1 << 30)))
    host = content.pool_host(g, w.content_seed)
    kv = gpu_pool_tensor(torch, w)
    want = digests(host, w)
    note(f"runs {g.chunk_bytes} B x {g.planes} planes, {g.num_blocks} blocks")
    for blocks in (np.arange(g.num_blocks), np.sort(rng.choice(g.num_blocks, 9, replace=False))):
        batch = from_claims([(i + 1, [int(b)], rng.integers(0, 32000, g.block_size))
                             for i, b in enumerate(blocks)])
        flips = rng.choice(blocks, 5, replace=False).astype(np.uint32)
        faults = FaultSpec(flips, rng.integers(0, 8 * g.block_bytes, 5).astype(np.uint64),
                           np.zeros(0, np.uint32))
        staging = torch.zeros(blocks.size * g.block_bytes, dtype=torch.uint8, device="cuda")
        with ck.Pool(g, w.seed, kv, max_claims=1024, max_footprint=1024, event_capacity=8192) as p:
            grid = p.digest_grid()
            assert (grid["words_per_lane"], grid["segments"]) == (lpw, 0)
            db = ck.DeviceBatch(batch)
            p.offload(db, staging=staging)
            assert np.array_equal(p.block_state()["d_off"][blocks], want[blocks])
            got = staging.cpu().numpy().reshape(blocks.size, -1)
            bytes_ = host.reshape(g.planes, g.num_blocks, -1).transpose(1, 0, 2)[blocks]
            assert np.array_equal(got, bytes_.reshape(blocks.size, -1))
            p.restore(db, staging=staging, faults=faults)
            p.check(db)
            st = p.block_state()
            assert np.array_equal(st["d_res"][blocks],
                                  digests(apply_flips(host, w, faults), w, blocks)[blocks])
            p.restore(db, staging=staging)  # the bytes again
    del kv, staging
    free_gpu(torch)
