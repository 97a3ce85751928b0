"""Host models of how the split forms write a layer back: the fused epilogue of the
product launches (park, direct pass, mirror pass; tiles of 256, 128 and 64 rows and
pairs of 128-row tiles) and the LDS stores of the one-workgroup kernel.  Every index is
formed as the kernels form it; what lies at a staged slot is followed from the
fragments to the stores."""
import numpy as np
import pytest

PANEL_ROWS, PANEL_K = 256, 32
EMPTY = -1


def panel_index(r, c, pdim):
    return ((r // PANEL_ROWS) * (pdim // PANEL_K) + c // PANEL_K) * PANEL_ROWS * PANEL_K \
        + (r % PANEL_ROWS) * PANEL_K + c % PANEL_K


def park_swz(quad):
    return (quad >> 1) | ((quad & 1) << 3)


class Geometry:
    """Epilogue<T16, NT, SR, BN, WTM, TILE> of a launch with WGM x WGN waves."""

    def __init__(self, tile, wgm, wgn, pair=False):
        self.TILE, self.WGM, self.WGN = tile, wgm, wgn
        self.NT, self.SR = 64 * wgm * wgn, 32 * wgm
        self.H = 2 if pair else 1
        self.BN = self.H * tile
        self.WTM, self.WTN = tile // wgm, self.BN // wgn
        self.FM, self.FN = self.WTM // 32, self.WTN // 32
        self.RS = 4 * self.NT // self.BN
        self.ITER = self.SR // self.RS
        self.LS = self.NT // (self.SR // 4)
        self.MITER = self.BN // self.LS
        self.G = 4
        self.NG, self.MG = self.ITER // self.G, self.MITER // self.G
        assert self.RS * self.ITER == self.SR and self.LS * self.MITER == self.BN
        assert self.NG * self.G == self.ITER and self.MG * self.G == self.MITER


GEOMETRIES = {"256": Geometry(256, 2, 2), "128": Geometry(128, 2, 2), "64": Geometry(64, 2, 2),
              "pair": Geometry(128, 2, 4, pair=True)}


def park(g, m, tiles):
    """The staged strip of round m: slot -> element code (h TILE + row) TILE + col of the
    tile that its value belongs to.  tiles: (r0, c0) per tile of the item."""
    T = np.full(g.SR * g.BN, EMPTY)
    lane = np.arange(64)
    half, q4, k = lane >> 5, (lane & 31) >> 2, lane & 3
    for wm in range(g.WGM):
        for wn in range(g.WGN):
            h = wn * g.WTN // g.TILE
            if h >= len(tiles):
                continue
            for n in range(g.FN):
                c = wn * g.WTN + n * 32 + (lane & 31)
                row0, col0 = wm * g.WTM + m * 32, wn * g.WTN + n * 32 - h * g.TILE
                on_diag = tiles[h][0] == tiles[h][1] and row0 == col0
                for r in range(16):
                    quad = wm * 8 + 2 * (r >> 2) + half
                    strip = 4 * quad * g.BN + 4 * ((c >> 2) ^ park_swz(quad))
                    own = (h * g.TILE + row0 + 8 * (r >> 2) + 4 * half + (r & 3)) * g.TILE \
                        + c - h * g.TILE
                    block = (q4 == 2 * (r >> 2) + half) & on_diag
                    keep = ~block | ((r & 3) <= k)
                    for slot, code in (((strip + (r & 3) * g.BN + (c & 3))[keep], own[keep]),
                                       ((strip + k * g.BN + (r & 3))[block & ((r & 3) < k)],
                                        own[block & ((r & 3) < k)])):
                        assert slot.min(initial=0) >= 0 and slot.max(initial=0) < len(T)
                        assert np.all(T[slot] == EMPTY)          # every slot once
                        T[slot] = code
    return T


def epilogue(g, tiles, kd, pdim, ld):
    """Stores of an item: master and split counts per element of the pdim x pdim problem.
    Addresses are checked against the element they stand for."""
    master = np.zeros((pdim, pdim), dtype=int)
    split = np.zeros((pdim, pdim), dtype=int)
    tid = np.arange(g.NT)
    tr0, c4 = tid // (g.BN // 4), tid % (g.BN // 4)
    h = np.zeros(g.NT, dtype=int) if g.H == 1 else c4 // (g.TILE // 4)
    lcl = c4 * 4 - h * g.TILE
    pad = list(tiles) + [(0, 0)] * (g.H - len(tiles))
    rh, ch = np.array([t[0] for t in pad])[h], np.array([t[1] for t in pad])[h]
    on = (h < len(tiles)) & (ch + lcl < kd)
    diag = rh == ch
    rows_ok = np.minimum(kd - rh, g.TILE)
    mq = tid % (g.SR // 4)
    mlr = (mq // 8) * g.WTM + (mq % 8) * 4
    for m in range(g.FM):
        T = park(g, m, tiles)
        packed = np.zeros(len(T), dtype=bool)                     # the slot holds splits
        for b in range(g.NG):                                     # direct pass
            r0 = b * g.G * g.RS
            r = (r0 // 32) * g.WTM + m * 32 + r0 % 32
            for i in range(g.G):
                quad = (g.RS // 4) * (b * g.G + i) + (0 if g.RS == 4 else tr0 >> 2)
                slot = (tr0 + b * g.G * g.RS + i * g.RS) * g.BN + 4 * (c4 ^ park_swz(quad))
                lr = r + i * g.RS + tr0
                takes = on & (lr < rows_ok) & (~diag | (lr <= lcl + 3))
                for q in range(4):
                    s, row, col, hh = (slot + q)[takes], lr[takes], (lcl + q)[takes], h[takes]
                    up = diag[takes] & (row >> 2 == col >> 2)      # whole 4 x 4 blocks there
                    lo, hi = np.minimum(row, col), np.maximum(row, col)
                    want = (hh * g.TILE + np.where(up, lo, row)) * g.TILE + np.where(up, hi, col)
                    assert np.array_equal(T[s], want)
                    assert not packed[s].any()
                    packed[s] = True
                    gr, gc = rh[takes] + row, ch[takes] + col
                    np.add.at(master, (gr, gc), 1)
                    np.add.at(split, (gr, gc), 1)
                gr, gc = rh + lr, ch + lcl
                mw = (rh + tr0) * ld + ch + lcl + r * ld + i * g.RS * ld
                hd = panel_index(rh + tr0, ch + lcl, pdim) + r * PANEL_K + i * g.RS * PANEL_K
                assert np.array_equal(mw[takes], (gr * ld + gc)[takes])
                assert np.array_equal(hd[takes], panel_index(gr, gc, pdim)[takes])
                assert np.all((hd % 4 == 0)[takes]) and np.all((mw % 4 == 0)[takes])
        for b in range(g.MG):                                     # mirror pass
            t = b * g.G * g.LS // g.TILE
            if t >= len(tiles):
                continue
            row0 = b * g.G * g.LS - t * g.TILE
            tr, tc = tiles[t]
            rows, cols = min(kd - tc, g.TILE), min(kd - tr, g.TILE)
            for i in range(g.G):
                c = tid // (g.SR // 4) + row0 + i * g.LS
                lr = mlr + m * 32
                go = (c < rows) & (lr < cols)
                if tr == tc:
                    go &= lr + 3 < c
                lc = c + t * g.TILE
                slot = 4 * mq * g.BN + 4 * ((lc >> 2) ^ park_swz(mq)) + (lc & 3)
                hm = panel_index(tc + tid // (g.SR // 4), tr + mlr, pdim) \
                    + m * PANEL_ROWS * PANEL_K + row0 * PANEL_K + i * g.LS * PANEL_K
                assert np.array_equal(hm[go], panel_index(tc + c, tr + lr, pdim)[go])
                for q in range(4):
                    s = (slot + q * g.BN)[go]
                    assert packed[s].all()                        # read only what was split
                    assert np.array_equal(T[s], ((t * g.TILE + lr + q) * g.TILE + c)[go])
                    np.add.at(split, (tc + c[go], tr + lr[go] + q), 1)
    return master, split


@pytest.mark.parametrize("name", list(GEOMETRIES))
def test_a_wave_touches_every_bank(name):
    """The staged strip as 64 banks of four bytes: a park of 32 columns of two row groups
    and a row of four-column groups meet no bank more often than they must."""
    g = GEOMETRIES[name]
    lane = np.arange(64)
    quad = lane >> 5
    slot = 4 * quad * g.BN + 4 * (((lane & 31) >> 2) ^ park_swz(quad)) + (lane & 3)
    assert np.bincount(slot % 64, minlength=64).max() == 1
    tr0, c4 = lane // (g.BN // 4), lane % (g.BN // 4)
    slot = tr0 * g.BN + 4 * (c4 ^ park_swz(tr0 >> 2))
    assert np.bincount(slot // 4 % 16, minlength=16).max() == 4    # 1 KB over 64 banks


# N, and the tiles of an item as block positions: on and off the diagonal, past the edge
@pytest.mark.parametrize("name,N,blocks", [
    ("256", 300, [(0, 0)]), ("256", 300, [(0, 1)]), ("256", 300, [(1, 1)]), ("256", 512, [(0, 1)]),
    ("128", 130, [(0, 0)]), ("128", 300, [(1, 2)]), ("128", 300, [(2, 2)]), ("128", 512, [(0, 3)]),
    ("64", 97, [(0, 0)]), ("64", 97, [(0, 1)]), ("64", 97, [(1, 1)]), ("64", 300, [(2, 4)]),
    ("64", 512, [(3, 7)]), ("64", 512, [(7, 7)])])
def test_single_problem_tiles_are_written_once(name, N, blocks):
    """A single problem's launch writes whole tiles (its buffers hold a multiple of 256
    rows): every element of the tile and its mirror gets its splits once, the masters
    the upper side and the 4 x 4 blocks on the diagonal."""
    g = GEOMETRIES[name]
    pdim = -(-N // 256) * 256
    ti, tj = blocks[0]
    tiles = [(ti * g.TILE, tj * g.TILE)]
    master, split = epilogue(g, tiles, pdim, pdim, pdim + 128)
    _check(g, tiles, pdim, pdim, master, split)


@pytest.mark.parametrize("N,blocks", [
    (37, [(0, 0)]), (129, [(0, 0), (0, 1)]), (300, [(0, 0), (0, 1)]), (300, [(0, 2), (1, 2)]),
    (300, [(2, 2)]), (300, [(1, 1), (1, 2)]), (513, [(0, 1), (0, 2)]), (513, [(3, 4), (4, 4)])])
def test_pairs_are_written_once_up_to_the_k_extent(N, blocks):
    """The batch's pairs leave out rows and columns from N rounded up to 32 on."""
    g = GEOMETRIES["pair"]
    pdim, kd = -(-N // 256) * 256, -(-N // 32) * 32
    tiles = [(i * g.TILE, j * g.TILE) for i, j in blocks]
    master, split = epilogue(g, tiles, kd, pdim, pdim)
    _check(g, tiles, kd, pdim, master, split)


def _check(g, tiles, kd, pdim, master, split):
    upper, whole = np.zeros((pdim, pdim), dtype=int), np.zeros((pdim, pdim), dtype=int)
    i, j = np.indices((pdim, pdim))
    for r, c in tiles:
        box = np.zeros((pdim, pdim), dtype=bool)
        box[r:min(r + g.TILE, kd), c:min(c + g.TILE, kd)] = True
        upper += box & ((i <= j) | (i // 4 == j // 4))
        whole += box if r == c else box | box.T
    assert np.array_equal(master, upper) and np.array_equal(split, whole)


# ------------------------------------------------------------------ one workgroup
@pytest.mark.parametrize("nf", [1, 2, 3, 4])
def test_one_workgroup_writes_every_split_once(nf):
    """k_tiny: the splits of the upper fragments, stored from the fragments' registers
    (mirror) and from their quad-transposed copies (direct), 8 bytes at a time: every
    element of the matrix once, with its value or its mirror's, inside the row pitch."""
    pitch = 32 * nf + 8
    lds = np.full(32 * nf * pitch, EMPTY)
    lane = np.arange(64)
    c, rb = lane & 31, 4 * (lane >> 5)

    def store(at, codes, go):
        for q in range(4):
            slot = (at + q)[go]
            assert np.all(lds[slot] == EMPTY)
            lds[slot] = codes[q][go]
        assert np.all(at[go] % 4 == 0)                            # 8-byte stores

    for fi in range(nf):
        for fj in range(fi, nf):
            mbase = (32 * fj + c) * pitch + 32 * fi + rb
            dbase = (32 * fi + rb + (c & 3)) * pitch + 32 * fj + (c & ~3)
            for q4 in range(4):
                r0 = 8 * q4 + rb
                own = [(32 * fi + r0 + q) * 1000 + 32 * fj + c for q in range(4)]
                # lane i of a quad receives entry i of lane j as entry j
                tp = [np.array([own[l & 3][(l & ~3) + q] for l in lane]) for q in range(4)]
                if fi != fj:
                    store(mbase + 8 * q4, own, lane >= 0)
                    store(dbase + 8 * q4 * pitch, tp, lane >= 0)
                else:
                    merged = [np.where(r0 + q <= c, own[q], tp[q]) for q in range(4)]
                    store(mbase + 8 * q4, merged, c >= r0)
                    store(dbase + 8 * q4 * pitch, tp, (c & ~3) > r0)
    m = lds.reshape(32 * nf, pitch)
    i, j = np.indices((32 * nf, 32 * nf))
    assert np.array_equal(m[:, :32 * nf], np.minimum(i, j) * 1000 + np.maximum(i, j))
    assert np.all(m[:, 32 * nf:] == EMPTY)
