"""The general kernel where its forms change over: one position a lane or four, positions numbered through the outputs or through
the padded rows, images dealt to the XCDs or not; rows of every length about its steps of 4, 8 and 16 nonzeros, in any order."""
import numpy as np
import pytest

import paper_1802_10280_amd as esc
from helpers import DeviceLayer, oracle_full, to_dev
from paper_1802_10280_amd import workloads as wl

gpu = pytest.mark.gpu

# N, C, H, W, M, R, S, stride, pad, sparsity
SHAPES = [
    (3, 24, 9, 13, 37, 3, 3, 1, 1, 0.6),      # one position; through the padded rows; images share a wave
    (3, 24, 9, 12, 37, 3, 3, 1, 1, 0.6),      # ... through the outputs
    (2, 20, 7, 7, 35, 5, 5, 1, 2, 0.6),       # padding over half of the map: through the outputs
    (3, 24, 11, 13, 37, 3, 3, 2, 1, 0.6),     # stride 2
    (1, 5, 1, 1, 33, 1, 1, 1, 0, 0.2),        # a single position
    (16, 24, 33, 37, 95, 3, 3, 1, 1, 0.8),    # four positions; rows not in fours; channels over
    (16, 12, 32, 44, 78, 2, 3, 1, 0, 0.7),    # ... a filter that is not square
    (7, 12, 40, 39, 150, 3, 3, 2, 1, 0.8),    # ... short rows, stride 2
    (16, 130, 44, 44, 33, 1, 1, 1, 0, 0.7),   # images dealt to the XCDs
]


@gpu
@pytest.mark.parametrize("order", ["sorted", "shuffled"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_forms_of_the_general_kernel(oracle, shape, order):
    """Against the oracle, to n roundings of a row's n products; rows 0..34 hold 0..34 nonzeros (as far as they have them)."""
    N, C, H, W, M, R, S, stride, pad, sparsity = shape
    L = wl.custom_layer(N, C, H, W, M, R, S, stride, pad, sparsity, seed=23, dist="normal")
    keep = np.concatenate([np.arange(b) < a if i < 35 else np.ones(b, bool)
                           for i, (a, b) in enumerate(zip(range(M), np.diff(L.rowptr)))])
    rows = np.add.reduceat(np.append(keep, 0), np.minimum(L.rowptr[:-1], keep.size)) * (np.diff(L.rowptr) > 0)
    L.colidx, L.value = L.colidx[keep], L.value[keep]
    L.rowptr = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    dl = DeviceLayer(esc, L)
    if order == "shuffled":
        mix = np.concatenate([a + np.random.default_rng(a).permutation(b - a) for a, b in zip(L.rowptr, L.rowptr[1:])]).astype(int)
        dl.d_colidx, dl.d_value = to_dev(dl.stretched[mix]), to_dev(L.value[mix])
    for flags in (0, esc.F_BIAS | esc.F_RELU):
        ref, bound = oracle_full(oracle, L, flags)
        got = dl.forward(flags)
        limit = (np.maximum(np.diff(L.rowptr), 1)[:, None, None] + 1) * 2.0 ** -24 * (bound + np.abs(ref))
        assert (np.abs(got.astype(np.float64) - ref) <= limit).all()  # a NaN fails
