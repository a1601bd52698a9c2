"""Kernel variants at the sizes where a tile, a chunk or a dispatch rule ends,
through the public calls, against the CPU oracle."""
import numpy as np
import pytest

import gen
import oracle
import paper_2010_10458_amd as tk
from gpu_common import announce, assert_bitwise, need_gpu, to_dev, to_host
from test_gpu_update_det import det_update_vs_oracle

pytestmark = pytest.mark.gpu

ORC = None


def orc():
    global ORC
    if ORC is None:
        ORC = oracle.Oracle()
    return ORC


# Ordered sums: (workers, entries per worker, distinct positions of the first
# tile they fall on). 768 entries are one chunk of a tile's accumulation: all
# at one position, just over a chunk, pairs only (as many runs as there can
# be), positions in both counter halves, all entries alone, several chunks.
@pytest.mark.parametrize("P,k,pool", [(1, 768, 1), (769, 1, 1), (205, 5, 1), (2, 384, 384),
                                      (3, 256, 256), (16, 64, 65), (1, 768, 768), (300, 7, 8),
                                      (2, 1, 2), (128, 32, 700)])
@pytest.mark.parametrize("mode", ["plain", "momentum"])
def test_ordered_chunks(P, k, pool, mode):
    rng = np.random.default_rng([P, k, pool])
    d = 4096 + 1111
    # positions on both halves of the first tile and some in the second
    where = np.sort(rng.choice(4096 if pool > 8 else [0, 1, 2047, 2048, 2049, 4094, 4095, 4096],
                               size=pool, replace=False))
    repeat = k > pool  # (repeats within a list are allowed)
    idx = np.stack([np.sort(rng.choice(where, size=k, replace=repeat)) for _ in range(P)])
    val = (rng.standard_normal((P, k)) * 10.0 ** rng.integers(-3, 4, (P, k))).astype(np.float32)
    w0 = gen.params_like([d], config=40)
    b0 = gen.params_like([d], config=41) if mode == "momentum" else None
    lr, mu, wd = (0.1, 0.9, 5e-5) if mode == "momentum" else (0.1, 0.0, 0.0)
    det_update_vs_oracle([d], w0, b0, idx.astype(np.int32), val, lr, mu, wd,
                         label=f"chunk edges pool={pool} {mode}")
