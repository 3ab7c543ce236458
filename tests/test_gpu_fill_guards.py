"""The fills on arrays that do not match each other: a row whose accepted bits and count differ
is left out and reported, every other row comes out right, and nothing is written outside the
rows (the outputs are surrounded by guard words). The library's own passes never leave such
arrays, so a harness makes them. n particles of one cell, all pairs within the radius."""
import ctypes

import native_harness as native
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ERR, LONG_ROW = 0, 4  # index of the error word, its bit for a row that does not match
GUARD = 4096


class Rows:
    """Wanted rows of n particles, and the device arrays a fill of one block or dense cell takes."""

    def __init__(self, dim, n, seed, f64):
        self.dim, self.n, self.f64 = dim, n, f64
        self.rng = np.random.default_rng(seed)
        self.pos = self.rng.uniform(0.05, 0.95, size=(n, dim))
        self.keep = self.rng.random((n, n)) < 0.5  # which candidates a row accepts
        np.fill_diagonal(self.keep, False)
        self.len = self.keep.sum(1).astype(np.int64)
        self.dev = {}

    def put(self, **arrays):
        for k, v in arrays.items():
            self.dev[k] = torch.from_numpy(np.ascontiguousarray(v)).cuda()

    def common(self, mode):
        n = self.n
        rec = np.zeros((n, 4))
        rec[:, :self.dim] = self.pos
        rec[:, 3] = np.arange(n, dtype=np.int64).view(np.float64)
        self.start = np.concatenate([[0], np.cumsum(self.len)])
        self.total = int(self.start[-1])
        self.put(pos=self.pos, row_ptr=self.start, col=np.full(self.total + 2 * GUARD, -7, np.int32),
                 dist=np.full(self.total + 2 * GUARD, -7, np.float32),
                 set_room=np.zeros(native.load().harness_set_bytes(), np.uint8), offs=np.array([0, n], np.int32),
                 cell_offs=np.array([0, 1], np.int32), skey=np.zeros(n, np.uint32), perm=np.arange(n, dtype=np.int32),
                 cell_start=np.array([0, n], np.int32), spos=rec, rq=np.zeros((n, 4), np.float32),
                 flags=np.zeros(8, np.int32))
        self.args = native.Args(dim=self.dim, mode=mode, n=n, half=0, capacity=self.total, radius=2.0, nblk_max=1,
                                t_lo=0x7BFF, t_hi=0x7BFF, t_mid=0x7BFF)

    def fill(self, dense):
        for k, t in self.dev.items():
            at = t.data_ptr() + (GUARD * 4 if k in ("col", "dist") else 0)
            setattr(self.args, k, at)
        torch.cuda.synchronize()
        assert native.load().harness_fill(ctypes.byref(self.args), dense) == 0
        return self.dev["flags"].cpu().numpy()

    def check(self, out):
        """Rows in `out` untouched, the others as wanted, the guards untouched."""
        col, dist = self.dev["col"].cpu().numpy(), self.dev["dist"].cpu().numpy()
        wcol, wdist = np.full(col.shape, -7, np.int32), np.full(dist.shape, -7, np.float64)
        for i in range(self.n):
            if i in out:
                continue
            at = GUARD + self.start[i]
            j = np.nonzero(self.keep[i])[0]
            wcol[at:at + len(j)] = j
            wdist[at:at + len(j)] = np.sqrt(((self.pos[j] - self.pos[i]) ** 2).sum(1))
        np.testing.assert_array_equal(col, wcol)
        assert np.all(np.abs(dist - wdist) <= 1e-6 * np.abs(wdist))


@pytest.mark.parametrize("mode", [0, 1], ids=["fp16", "fp64"])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", [1, 17, 64])
def test_block_row_that_does_not_match_its_count(dim, n, mode):
    for wrong in ([], [0], [n - 1], list(range(0, n, 3)), list(range(n))):
        for delta in (-1, 1, 40):
            r = Rows(dim, n, 7, mode == 1)
            bits = r.keep.copy()
            off = [i for i in wrong if r.len[i] + delta >= 0]
            for i in off:  # the count says otherwise than the bits
                r.len[i] += delta
            r.common(mode)
            words = np.zeros((1024 // 32 if dim == 3 else 512 // 32, n), np.uint32)
            for i in range(n):
                for j in np.nonzero(bits[i])[0]:
                    words[j >> 5, i] |= np.uint32(1 << (j & 31))
            nseg = 9 if dim == 3 else 3
            self_seg = nseg // 2
            desc = np.zeros(24, np.int32)
            desc[:4] = [0, n, 0, n]
            desc[5 + nseg + self_seg + 1:5 + 2 * nseg] = n  # the segments after the targets' own start at the end
            r.put(cbits=words, bdesc=desc, branks=np.arange(1024, dtype=np.uint16), nblk=np.array([1], np.int32),
                  counts_s=r.len.astype(np.int32), rsort=r.start[:n], heavy=np.zeros(n, np.int32))
            flags = r.fill(0)
            assert flags[ERR] == (LONG_ROW if off else 0)
            r.check(off)


def kept_bits(keep):
    """The dense count's bits: per (target, 1024-candidate chunk) 64 words of 16 bits."""
    n = keep.shape[0]
    nchunk = (n + 1023) // 1024
    b = np.zeros((n, nchunk * 1024), bool)
    b[:, :n] = keep
    return (b.reshape(n, nchunk, 64, 16) << np.arange(16)).sum(-1).astype(np.uint16)


@pytest.mark.parametrize("mode", [0, 1], ids=["fp16", "fp64"])
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("n", [1, 17, 63, 1000, 1030])
def test_dense_bits_past_the_list_and_rows_of_another_length(dim, n, mode):
    """Bits past the union's last candidate are no candidates. A row with more accepted bits than
    its length in the row pointers writes that many (the list's first), one with fewer what it has;
    both are reported."""
    for case in ("clean", "past", "short", "long"):
        r = Rows(dim, n, 11, mode == 1)
        bits = kept_bits(r.keep)
        if case == "past":
            nchunk = bits.shape[1]
            lane, bit = (n % 1024) >> 4, n & 15
            if n % 1024:
                bits[:, nchunk - 1, lane] |= np.uint16((0xFFFF << bit) & 0xFFFF)
                bits[:, nchunk - 1, lane + 1:] = 0xFFFF
        off = list(range(0, n, 5)) if case in ("short", "long") else []
        off = [i for i in off if case == "long" or r.len[i] > 0]
        for i in off:
            r.len[i] += 1 if case == "long" else -1
        r.common(mode)
        nchunk = bits.shape[1]
        nu = (n + 63) // 64
        r.put(dbits=bits, wdense=np.ones(1, np.int32), usz=np.array([n], np.int32), uoff=np.array([0, n], np.int64),
              ulist=np.arange(n, dtype=np.int32), unit_off=np.array([0, nu], np.int32), ucell=np.zeros(nu, np.int32),
              dn=np.array([n], np.int32), dboff=np.array([0, n * nchunk], np.int64))
        r.args.dbits_cap = bits.size
        flags = r.fill(1)
        assert flags[ERR] == (LONG_ROW if off else 0), case
        for i in off:  # the reported rows: as far as they go
            j = np.nonzero(r.keep[i])[0]
            at = GUARD + r.start[i]
            m = min(len(j), int(r.len[i]))
            np.testing.assert_array_equal(r.dev["col"][at:at + m].cpu().numpy(), j[:m])
            r.dev["col"][at:at + m] = -7
            r.dev["dist"][at:at + m] = -7
        r.check(off)
