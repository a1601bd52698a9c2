"""Host check: the restated region layout gives the library's workspace size."""
import ctypes

import numpy as np

import paper_2010_10458_amd as tk
import region_layout


def test_region_layout_matches_the_library():
    rng = np.random.default_rng(17)
    nb = ctypes.c_size_t()
    for _ in range(3000):
        T = int(rng.choice([1, 1, 1, 2, 5, 161]))
        top = float(rng.uniform(1, 26 if T == 1 else 22))
        sizes = [max(1, int(2 ** rng.uniform(0, top))) for _ in range(T)]
        d = sum(sizes)
        k = min(d, max(1, int(d * 10 ** rng.uniform(-5, 0))))
        assert tk.lib().tkef_sparsify_workspace((ctypes.c_int64 * T)(*sizes), T, tk.GLOBAL, 0.0, k,
                                                ctypes.byref(nb), None) == tk.OK
        assert nb.value == region_layout.workspace_bytes(sizes, k), (sizes, k)
    for d, k in ((340_000_000, 340_000), (340_000_000, 3_400_000), (2**31 - 1, 1), (2**31 - 1, 2**30)):
        assert tk.lib().tkef_sparsify_workspace((ctypes.c_int64 * 1)(d), 1, tk.GLOBAL, 0.0, k,
                                                ctypes.byref(nb), None) == tk.OK
        assert nb.value == region_layout.workspace_bytes([d], k), (d, k)
