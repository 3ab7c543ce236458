"""Sets with far fewer particles than cells: their many small blocks take the union ranks' room from
pools, so that the structure's memory follows the particles, and are counted by a wavefront each in
3D, larger unions among them by a workgroup; rows are the oracle's on every path."""
import ctypes

import native_harness as native
import numpy as np
import pytest

import oracle
from paper_2401_08586_amd import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_08586_amd import nnps  # noqa: E402

MODES = {"fp16": nnps.MODE_FP16_RCLL, "fp64": nnps.MODE_FP64_BASELINE, "fp32": nnps.MODE_FP32_RCLL}


def scattered(dim, n, nc, seed, clump=0, wide=2.0):
    """n points over nc^dim cells, the last `clump` of them in the middle, `wide` cells to either side."""
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0, 1, size=(n, dim))
    pos[n - clump:] = 0.5 + rng.uniform(-wide, wide, size=(clump, dim)) / nc
    return W.ParticleSet(np.ascontiguousarray(pos[rng.permutation(n)]), (0.0,) * dim, (1.0,) * dim, 1.0 / nc, 1.0 / nc,
                         f"scattered{dim}d_{n}_in_{nc}_{clump}_{wide}")


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def structure_bytes(ps, mode):
    pos = torch.from_numpy(ps.pos).cuda()
    rp = torch.empty(ps.n + 1, dtype=torch.int64, device="cuda")
    ctx = nnps.Context(0)
    cells = ctx.cells()
    before = free_bytes()
    cells.build(pos, ps.lo, ps.hi, ps.cell_size, ps.radius, mode=mode)
    cells.count(rp)
    used = before - free_bytes()
    cells.close()
    ctx.close()
    return used


@pytest.mark.parametrize("mode", ["fp16", "fp64"])
def test_memory_follows_the_particles(mode):
    """Per particle, beside what an almost empty grid takes: 16 bytes of keys and slots, 48 of
    positions and coordinates, 12 of counts and the inverse order, 8 of row starts, 128 of bits, 108
    of dense lists, 36 of the update's and the blocks' tables, up to 136 of block descriptors and
    statistics, 96 of ranks: under 600. (A full union's place per block took 2048 more.)"""
    n = 400000
    few, many = scattered(3, 1000, 160, 1), scattered(3, n, 160, 2)
    a, b = structure_bytes(few, MODES[mode]), structure_bytes(many, MODES[mode])
    print(f"[gpu] memory {mode}: {a} and {b} bytes, {(b - a) / n:.0f} per particle", flush=True)
    assert (b - a) / n < 600


@pytest.mark.parametrize("half", [False, True], ids=["full", "half"])
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("dim", [2, 3])
def test_sparse_sets_against_the_oracle(dim, mode, half):
    for ps in (scattered(dim, 40000, 128 if dim == 3 else 2000, 3), scattered(dim, 60000, 128 if dim == 3 else 2000, 4, 9000),
               scattered(dim, 60000, 128 if dim == 3 else 2000, 6, 25000, 9.0),  # unions of 500 to 900 in 3D
               scattered(dim, 100, 128 if dim == 3 else 2000, 5)):
        print(f"[gpu] sparse {ps.name} {mode} half={half}", flush=True)
        wrp, wcol, wdist = oracle.search_ps(ps)
        if half:
            rows = np.repeat(np.arange(ps.n), np.diff(wrp))
            keep = wcol > rows
            wrp = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=ps.n))])
            wcol, wdist = wcol[keep], wdist[keep]
        pos = torch.from_numpy(ps.pos).cuda()
        ctx = nnps.Context(0)
        try:
            for dense in (0, -1):  # dense cells in the middle, or all blocks and long rows
                ctx.set_tuning(dense_min_union=dense)
                cells = ctx.cells()
                cells.set_half(half)
                stream = torch.cuda.Stream()
                cells.set_graphs(True)
                nnz = len(wcol)
                rp = torch.empty(ps.n + 1, dtype=torch.int64, device="cuda")
                col = torch.empty(max(nnz, 1), dtype=torch.int32, device="cuda")
                dist = torch.empty(max(nnz, 1), dtype=torch.float32, device="cuda")
                sets = [(pos, ps.lo, ps.hi, ps.cell_size, ps.radius)]
                for rep in range(5):  # two searches, the last after counts without a fill; then replays of a graph
                    col.fill_(-1)
                    dist.fill_(-1)
                    if rep < 2:
                        cells.build(*sets[0], mode=MODES[mode])
                        for _ in range(1 + 2 * rep):
                            assert cells.count(rp) == nnz
                        cells.fill(rp, col, dist)
                    else:
                        torch.cuda.synchronize()
                        cells.batch_step(sets, [rp], [col], [dist], MODES[mode], stream=stream)
                        torch.cuda.synchronize()
                    np.testing.assert_array_equal(rp.cpu().numpy(), wrp, err_msg=ps.name)
                    np.testing.assert_array_equal(col.cpu().numpy()[:nnz], wcol, err_msg=ps.name)
                    d, w = dist.cpu().numpy()[:nnz].astype(np.float64), wdist.astype(np.float64)
                    assert np.all(np.abs(d - w) <= 1e-6 * w), ps.name
                cells.close()
        finally:
            ctx.set_tuning()
            ctx.close()


@pytest.mark.parametrize("mode", [nnps.MODE_FP16_RCLL, nnps.MODE_FP64_BASELINE])
@pytest.mark.parametrize("dim", [2, 3])
def test_block_whose_pool_is_empty(dim, mode):
    """It is counted right and its rows are sent to the long-row path: the other blocks keep
    their ranks, and nothing is written past a pool."""
    n, radius = 200, 0.5
    rng = np.random.default_rng(dim)
    pos = rng.uniform(0.02, 0.98, size=(n, dim))
    want = (((pos[:, None] - pos[None]) ** 2).sum(-1) <= radius * radius).sum(1) - 1
    spos = np.zeros((n, 4))
    spos[:, :dim] = pos
    spos[:, 3] = np.arange(n, dtype=np.int64).view(np.float64)
    rq = np.zeros((n, 4), np.float32)
    rq[:, :dim] = 2 * pos - 1
    nb, cap = 4, 208  # room for one union of 200 in each of 256 pools
    taken = np.zeros((256, 16), np.int32)
    taken[1, 0] = 16  # block 1 finds its pool short of room
    arrays = dict(pos=pos, set_room=np.zeros(native.load().harness_set_bytes(), np.uint8), offs=np.array([0, n], np.int32),
                  cell_offs=np.array([0, 1], np.int32), skey=np.zeros(n, np.uint32), perm=np.arange(n, dtype=np.int32),
                  cell_start=np.array([0, n], np.int32), spos=spos, rq=rq, flags=np.zeros(8, np.int32),
                  bstart=np.minimum(64 * np.arange(nb + 1), n).astype(np.int32), bset=np.zeros(nb, np.int32),
                  nblk=np.array([nb], np.int32), counts=np.zeros(n, np.int32), counts_s=np.zeros(n, np.int32),
                  cbits=np.zeros((32, n), np.uint32), bdesc=np.zeros((nb + 8, 24), np.int32), rpool=taken,
                  branks=np.full(256 * cap + 4096, 0xABCD, np.uint16))
    dev = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in arrays.items()}
    args = native.Args(dim=dim, mode=mode, n=n, radius=radius, nblk_max=nb, rpool_cap=cap)
    for k, v in dev.items():
        setattr(args, k, v.data_ptr())
    torch.cuda.synchronize()
    print(f"[gpu] empty pool {dim}d mode={mode}", flush=True)
    assert native.load().harness_count(ctypes.byref(args)) == 0
    np.testing.assert_array_equal(dev["counts"].cpu().numpy(), want)
    desc, ranks = dev["bdesc"].cpu().numpy(), dev["branks"].cpu().numpy()
    limit = 1024 if dim == 3 else 512
    left = ranks.copy()
    for b in range(nb):
        if b == 1:
            assert desc[b, 3] > limit
            continue
        assert desc[b, 3] == n
        at = 16 * int(desc[b, 23])
        assert at == b * cap
        np.testing.assert_array_equal(ranks[at:at + n], np.arange(n))  # one cell, numbered in order
        left[at:at + n] = 0xABCD
    assert np.all(left == 0xABCD)


@pytest.mark.parametrize("half", [0, 1], ids=["full", "half"])
@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("sparse", [0, 1], ids=["workgroup", "wavefront"])
@pytest.mark.parametrize("span", [1 << 10, 1 << 17, 18_000_000])
def test_ranks_and_bits_of_a_count(span, sparse, mode, half):
    """One cell in 3D, numbered at random in `span` values (sorting keys hold a position beside the
    index up to 2^24): every block's union ranks, kept bits and counts, at the edges of what a
    wavefront ranks (64, 128, 256 candidates) and past it."""
    radius = 0.5
    for n in (1, 2, 63, 64, 65, 127, 129, 192, 255, 256, 257, 600, 1024):
        if n > span:
            continue
        rng = np.random.default_rng(n)
        pos = rng.uniform(0.02, 0.98, size=(n, 3))
        near = ((pos[:, None] - pos[None]) ** 2).sum(-1) <= radius * radius
        perm = rng.permutation(np.concatenate([[0, span - 1], 1 + rng.choice(span - 2, n - 2, replace=False)]) if n > 1
                               else [span - 1]).astype(np.int32)  # distinct, the ends among them
        rank = np.empty(n, np.int64)
        rank[np.argsort(perm)] = np.arange(n)
        spos = np.zeros((n, 4))
        spos[:, :3] = pos
        spos[:, 3] = perm.astype(np.int64).view(np.float64)
        rq = np.zeros((n, 4), np.float32)
        rq[:, :3] = 2 * pos - 1
        nb, cap = (n + 63) // 64, 1024
        arrays = dict(pos=pos, set_room=np.zeros(native.load().harness_set_bytes(), np.uint8),
                      offs=np.array([0, n], np.int32), cell_offs=np.array([0, 1], np.int32), skey=np.zeros(n, np.uint32),
                      perm=perm, cell_start=np.array([0, n], np.int32), spos=spos, rq=rq, flags=np.zeros(8, np.int32),
                      bstart=np.minimum(64 * np.arange(nb + 1), n).astype(np.int32), bset=np.zeros(nb, np.int32),
                      nblk=np.array([nb], np.int32), counts=np.full(span, -1, np.int32), counts_s=np.full(n, -1, np.int32),
                      cbits=np.zeros((32, n), np.uint32), bdesc=np.zeros((nb + 8, 24), np.int32),
                      rpool=np.zeros((256, 16), np.int32), branks=np.full(256 * cap, 0xABCD, np.uint16))
        dev = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in arrays.items()}
        args = native.Args(dim=3, mode=MODES[mode], n=n, half=half, radius=radius, nblk_max=nb, rpool_cap=cap, sparse=sparse)
        for k, v in dev.items():
            setattr(args, k, v.data_ptr())
        torch.cuda.synchronize()
        print(f"[gpu] ranks n={n} span={span} sparse={sparse} {mode} half={half}", flush=True)
        assert native.load().harness_count(ctypes.byref(args)) == 0
        keep = near & ~np.eye(n, dtype=bool)
        if half:
            keep &= perm[None] > perm[:, None]
        counts = np.full(span, -1, np.int32)
        counts[perm] = keep.sum(1)
        np.testing.assert_array_equal(dev["counts"].cpu().numpy(), counts)
        np.testing.assert_array_equal(dev["counts_s"].cpu().numpy(), keep.sum(1))
        desc, ranks = dev["bdesc"].cpu().numpy(), dev["branks"].cpu().numpy()
        bits = dev["cbits"].cpu().numpy()
        want = np.zeros((1024, n), bool)
        want[rank] = keep.T
        got = (bits[:, None, :] >> np.arange(32, dtype=np.uint32)[None, :, None] & 1).reshape(1024, n).astype(bool)
        np.testing.assert_array_equal(got, want)
        for b in range(nb):
            assert desc[b, 3] == n and desc[b, 4] == 0
            at = 16 * int(desc[b, 23])
            np.testing.assert_array_equal(ranks[at:at + n], rank)


@pytest.mark.parametrize("graphs", [False, True], ids=["eager", "graph"])
@pytest.mark.parametrize("n", [1, 100, 3000])
@pytest.mark.parametrize("dim", [2, 3])
def test_updates_in_a_grid_of_few_particles(dim, n, graphs):
    """Builds and updates leave their per-cell counters clear for the next one also where the cells
    are thousands of times the particles: rows after every one of them."""
    nc = 128 if dim == 3 else 1448
    ps = scattered(dim, n, nc, 7)
    ps = W.ParticleSet(np.ascontiguousarray(ps.pos), ps.lo, ps.hi, 3.0 / nc, 3.0 / nc)  # some pairs
    rng = np.random.default_rng(n)
    pos = torch.from_numpy(ps.pos.copy()).cuda()
    print(f"[gpu] sparse updates {dim}d n={n} graphs={graphs}", flush=True)
    ctx = nnps.Context(0)
    try:
        cells = ctx.cells()
        cells.set_graphs(graphs)
        stream = torch.cuda.Stream()
        cells.build(pos, ps.lo, ps.hi, ps.cell_size, ps.radius)
        rp = torch.empty(n + 1, dtype=torch.int64, device="cuda")
        cells.count(rp)
        for step in range(6):
            d = torch.from_numpy(rng.uniform(-0.3, 0.3, size=(n, dim))).cuda()  # far jumps, reflected at the faces
            col = torch.full((64 * n + 64,), -1, dtype=torch.int32, device="cuda")
            dist = torch.empty(col.shape, dtype=torch.float32, device="cuda")
            torch.cuda.synchronize()
            if step == 3:  # a fresh build in between
                cells.batch_step([(pos, ps.lo, ps.hi, ps.cell_size, ps.radius)], [rp], [col], [dist],
                                 nnps.MODE_FP16_RCLL, stream=stream)
            else:
                cells.batch_update_step([rp], [col], [dist], disp=[d], stream=stream)
            torch.cuda.synchronize()
            now = W.ParticleSet(pos.cpu().numpy(), ps.lo, ps.hi, ps.cell_size, ps.radius)
            wrp, wcol, _ = oracle.search_ps(now)
            np.testing.assert_array_equal(rp.cpu().numpy(), wrp)
            np.testing.assert_array_equal(col.cpu().numpy()[:len(wcol)], wcol)
        cells.close()
    finally:
        ctx.close()
