"""The digest kernels over seeded random pool geometries, against the
oracle: block sizes, head counts, head widths and element sizes that give
chunks from 16 bytes to 72 KiB (pieces of 4, 8, 16 and 24 words per lane that
divide the chunk, one or several to a chunk; pieces of 1, 2, 4 and 8 words that
run across chunk ends, where none divides it), planes from 1 to 12, and head
shards at random offsets; and pools of 115 to 1365 planes over 8 to 16 blocks,
with both kinds of pieces, most of which read their piece groups in phases (one
phase would leave much of the grid idle).  Every block's offload digest, and
its restore digest after seeded flips, must equal the oracle's."""

import os

import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_01387_amd.synth import TINY, FaultSpec, Geometry, Workload, content, from_claims
from tests.helpers import apply_flips, digests
from tests.test_gpu_parity import free_gpu, gpu_pool_tensor

pytestmark = pytest.mark.gpu


def random_geometry(rng) -> Geometry:
    while True:
        layers, ppl = int(rng.integers(1, 7)), int(rng.choice([1, 2]))
        bs = int(rng.choice([1, 2, 3, 4, 5, 8, 16, 32, 64]))
        heads = int(rng.choice([1, 1, 2, 3, 4, 8]))
        dim = int(rng.choice([8, 16, 24, 40, 64, 96, 128, 576]))
        eb = int(rng.choice([1, 2]))
        chunk = bs * heads * dim * eb
        if chunk % 16 or chunk > 72 * 1024:
            continue
        nb = int(rng.integers(8, 40))
        if rng.random() < 0.3 and dim * eb % 8 == 0:
            total = heads * int(rng.integers(2, 5))
            first = int(rng.integers(0, total - heads + 1))
            return Geometry(layers, ppl, bs, heads, dim, eb, nb, total_kv_heads=total,
                            first_kv_head=first)
        return Geometry(layers, ppl, bs, heads, dim, eb, nb)


# Chunks of 6 to 36 KiB and the pieces that divide them (4, 16, 16, 24 or 24
# words per lane), and 9-row chunks in pieces of 8 rows across chunk ends, with
# the digest workgroups that 256 CUs hold at once.
_PLANE_CHUNKS = [(6144, 3, 1024), (8192, 1, 256), (12288, 1, 256), (16384, 2, 256), (24576, 2, 256),
                 (32768, 4, 256), (36864, 3, 256), (4608, 9 / 8, 512), (4608, 9 / 8, 512)]


def many_plane_geometry(rng) -> tuple[Geometry, bool]:
    """Planes enough for 34-42 % or 51-84 % as many piece groups of 4 pieces
    (the last group often short) as workgroups fit: one phase would fill at
    most 85 % of the grid.  Most have a multiple of 12 of them, which splits into
    phases that fill it; whether it has is returned too."""
    while True:
        chunk, segs, slots = _PLANE_CHUNKS[int(rng.integers(len(_PLANE_CHUNKS)))]
        lo, hi = (0.34, 0.42) if rng.random() < 0.3 else (0.51, 0.84)
        pgs = int(rng.integers(int(lo * slots), int(hi * slots)))
        phased = rng.random() < 0.7
        if phased:
            pgs += -pgs % 12
        planes = int((4 * pgs - int(rng.integers(0, 4))) / segs)
        if pgs > hi * slots or -(-int(np.ceil(planes * segs)) // 4) != pgs:
            continue
        ppl = 2 if planes % 2 == 0 and rng.random() < 0.5 else 1
        bs = int(rng.choice([1, 2, 4, 8, 16]))
        nb = int(rng.integers(8, 17))  # enough blocks for several workgroups per phase
        if planes * chunk * nb > 160 << 20:
            continue
        return Geometry(planes // ppl, ppl, bs, 1, chunk // bs, 1, nb), phased


# CLAIMKV_SHAPE_SEEDS widens a one-off run; the suite runs the first 60
@pytest.mark.parametrize("seed", range(int(os.environ.get("CLAIMKV_SHAPE_SEEDS", "60"))))
def test_digest_shapes(torch, ck, seed):
    rng = np.random.default_rng(70_000 + seed)
    run_shape(torch, ck, random_geometry(rng), rng, seed)


def digest_grid(torch, ck, g):
    kv = torch.empty(g.pool_bytes, dtype=torch.uint8, device="cuda")
    with ck.Pool(g, 1, kv, max_claims=64, max_footprint=64, event_capacity=64) as pool:
        return pool.digest_grid()


def test_shapes_cover_the_widths(torch, ck):
    """The first 60 seeds reach every width of pieces that divide a chunk, and
    those across chunk ends but the widest (20 words: many rows)."""
    grids = [digest_grid(torch, ck, random_geometry(np.random.default_rng(70_000 + s)))
             for s in range(60)]
    assert {d["words_per_lane"] for d in grids if d["segments"]} == {4, 8, 16, 24}
    assert {d["words_per_lane"] for d in grids if not d["segments"]} >= {1, 2, 4, 8}
    assert {d["segments"] > 1 for d in grids if d["segments"]} == {True, False}


@pytest.mark.parametrize("seed", range(int(os.environ.get("CLAIMKV_PLANE_SEEDS", "24"))))
def test_digest_shapes_many_planes(torch, ck, seed):
    rng = np.random.default_rng(80_000 + seed)
    g, _ = many_plane_geometry(rng)
    run_shape(torch, ck, g, rng, seed)


def test_many_planes_are_read_in_phases(torch, ck):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("grid expectations are for 256 compute units")
    phased = {True: 0, False: 0}  # by whether pieces run across chunk ends
    for seed in range(24):
        g, several = many_plane_geometry(np.random.default_rng(80_000 + seed))
        d = digest_grid(torch, ck, g)
        phases = d["piece_groups"] // d["pga"]
        assert d["pga"] * d["groups"] <= d["slots"]
        assert phases > 1 or not several, (seed, g, d)
        phased[d["segments"] == 0] += phases > 1
    assert phased[False] >= 8 and phased[True] >= 3


def run_shape(torch, ck, g, rng, seed):
    w = Workload(name=f"shape-{seed}", geometry=g, seed=int(rng.integers(0, 2**63)), num_claims=0,
                 length=TINY.length, sharing=TINY.sharing, corrupt_rate=0.0, gen_seed=seed,
                 content_seed=int(rng.integers(0, 2**31)))
    print(f"digest shape seed {seed}: planes {g.planes}, chunk {g.chunk_bytes} B "
          f"(bs {g.block_size}, heads {g.num_kv_heads}/{g.total_kv_heads or g.num_kv_heads}, "
          f"dim {g.head_dim}, elem {g.elem_bytes}), {g.num_blocks} blocks", flush=True)
    # every block, one claim each (a few blocks twice)
    blocks = list(range(g.num_blocks)) + [int(b) for b in rng.integers(0, g.num_blocks, 3)]
    batch = from_claims([(i + 1, [b], rng.integers(0, 32000, g.block_size, dtype=np.uint32))
                         for i, b in enumerate(blocks)])
    nflip = int(rng.integers(1, 6))
    faults = FaultSpec(rng.integers(0, g.num_blocks, nflip).astype(np.uint32),
                       rng.integers(0, 8 * g.block_bytes, nflip).astype(np.uint64),
                       np.zeros(0, np.uint32))
    kv = gpu_pool_tensor(torch, w)
    host = content.pool_host(g, w.content_seed)
    with ck.Pool(g, w.seed, kv, max_claims=128, max_footprint=256, event_capacity=512) as pool:
        db = ck.DeviceBatch(batch)
        pool.offload(db)
        pool.restore(db, faults=faults)
        pool.check(db)
        out, _ = pool.read()
        st = pool.block_state()
    assert np.array_equal(st["d_off"], digests(host, w))
    assert np.array_equal(st["d_res"], digests(apply_flips(host, w, faults), w))
    failed = set(int(b) for b in faults.changed_blocks())
    assert [int(c) for c in out["code"]] == [2 if b in failed else 1 for b in blocks]
    del kv
    free_gpu(torch)
