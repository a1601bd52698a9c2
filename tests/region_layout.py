"""The exact global selection's regions, restated for the tests that aim at a
region's capacity: lines, regions and capacities from the sizes and k, and how
many candidates and band members an input puts into each region. The workspace
size that follows from it is checked against the library's
(test_region_layout.py), so a change of the library's rule fails there instead of
emptying those tests."""
from __future__ import annotations

import numpy as np

TILE, LINE, LINES_PER_TILE = 8192, 32, 256
BAND_CAP = 4096   # band members of a region that a workgroup keeps in LDS


def layout(sizes, k):
    tiles = sum(-(-n // TILE) for n in sizes)
    nlines, d = tiles * LINES_PER_TILE, sum(sizes)
    threads = 512 if nlines <= 256 * 512 * 8 else 1024
    lpt = 4
    while lpt < -(-nlines // (threads * 256)) and lpt < 16:
        lpt *= 2
    even = -(-nlines // 256)
    lines = max(even, min(max(int(256.0 / 48.0 * float(d) / float(k)), threads), 4 * threads))
    lines = -(-lines // lpt) * lpt
    count = max(1, -(-nlines // lines))
    elems = lines * LINE
    share = -(-(8 * k + 65536) // count)
    rcap = min(elems, max(4096, -(-share // 64) * 64, elems // 64))
    return dict(threads=threads, lpt=lpt, lines=lines, count=count, elems=elems, rcap=rcap,
                tiles=tiles, nlines=nlines)


def workspace_bytes(sizes, k):
    a = layout(sizes, k)
    slots = a["count"] * a["rcap"]
    zeroed = [4 * 2048 * 4, 1024 * 4, 4]  # histograms of levels 1 and 2, the ticket
    parts = [a["tiles"] * 32, 16, 16, sum(-(-n // 256) * 256 for n in zeroed),
             a["nlines"] * 2, slots * 16, slots * 4, slots * 4, a["count"] * 1024 * 4,
             a["count"] * 8, 1024 * a["count"] * 4 * 4, a["count"] * 8]
    return sum(-(-n // 256) * 256 for n in parts)


def region_of(sizes, k):
    """Region of every position of the concatenated list."""
    lines, first = layout(sizes, k)["lines"], 0
    out = []
    for n in sizes:
        out.append((first + np.arange(n, dtype=np.int64) // LINE) // lines)
        first += -(-n // TILE) * LINES_PER_TILE
    return np.concatenate(out)


def counts(x, sizes, k):
    """Per region: candidates (level-1 bin of the key at or above the k-th
    largest's) and band members (in that bin)."""
    key = np.ascontiguousarray(x, np.float32).view(np.uint32) & 0x7FFFFFFF
    top = key >> 20
    b1 = np.partition(top, x.size - k)[x.size - k]
    where, n = region_of(sizes, k), layout(sizes, k)["count"]
    return (np.bincount(where[top >= b1], minlength=n), np.bincount(where[top == b1], minlength=n))


def sample_sizes(top):
    """Sizes up to top: around the powers of two of tiles, spread ones between them,
    each a whole number of tiles, one element more and a tile less one."""
    rng = np.random.default_rng(3)
    tiles = {top // TILE}
    for e in range(int(np.log2(top // TILE)) + 1):
        tiles |= {max(1, (1 << e) + s) for s in (-1, 0, 1)}
        tiles |= {int(t) for t in rng.integers(1 << e, 2 << e, 6)}
    return sorted({n for t in tiles for n in (t * TILE, t * TILE + 1, t * TILE + TILE - 1)
                   if n <= top})


def sample_ks(d, top):
    """Values of k up to min(d, top): the ends, around the powers of two, and where
    the lines per region meet one and four lines per thread or the even split."""
    top = min(d, top)
    a = layout([d], 1)
    ks = {1, top}
    for e in range(18):
        ks |= {(1 << e) + s for s in (-1, 0, 1)}
    for lines in (a["threads"], 2 * a["threads"], 4 * a["threads"], -(-a["nlines"] // 256)):
        k = int(256.0 / 48.0 * d / lines)
        ks |= {k + s for s in (-1, 0, 1)}
    return sorted(k for k in ks if 1 <= k <= top)
