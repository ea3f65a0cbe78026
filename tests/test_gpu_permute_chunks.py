"""The two maps of moe_permute where its workgroups end: pairs around one wavefront (64), one chunk (1024) and the number of chunks
(8) above which the chunks are counted by a launch of their own, the number of counters (65536) above which another one scans
them; expert counts around powers of two (the ids are matched bit by
bit); every pair on one expert, and experts without pairs.  Whole numbers: the maps equal the oracle's stable counting sort."""
import numpy as np
import pytest

from oracle import moe_oracle as O
from tests.util import to_dev, to_np

pytestmark = pytest.mark.gpu

# (T, k, E)
SIZES = [(1, 1, 1), (1, 8, 128), (21, 3, 5), (64, 1, 16), (1023, 1, 1), (512, 2, 60), (1025, 1, 1024), (1023, 8, 128), (1024, 8, 128),
         (1025, 8, 128), (16385, 1, 16), (9001, 4, 1000), (5000, 7, 65),
         (65536, 1, 1024), (65537, 1, 1024), (32768, 4, 513), (131073, 4, 65), (524289, 2, 5)]


@pytest.mark.parametrize("spread", ["even", "one", "skewed"])
@pytest.mark.parametrize("T,k,E", SIZES)
def test_maps_equal_the_stable_sort(T, k, E, spread):
    from paper_2508_02317_amd import libmoe as L
    r = np.random.default_rng(T * 31 + E)
    if spread == "one":
        idx = np.full((T, k), E - 1, dtype=np.int32)
    else:
        u = r.random((T, k))
        idx = np.minimum((u if spread == "even" else u ** 6) * E, E - 1).astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(np.bincount(idx.ravel(), minlength=E))]).astype(np.int32)
    row_of_pair, pair_of_row = O.permute_maps(idx, offsets)
    _, rows, pairs = L.moe_permute(None, to_dev(idx), to_dev(offsets), E)
    assert np.array_equal(to_np(rows).ravel(), np.asarray(row_of_pair).ravel())
    assert np.array_equal(to_np(pairs), pair_of_row)
