"""Kernels at the sizes where their tiling can go wrong, against the CPU oracle: edges of tiles,
remainders, the smallest and largest shapes of a variant.  Bit-exact like every result of the library."""
import numpy as np
import pytest
import torch

from oracle import st_oracle as O
from paper_2511_14881_amd import binding as st

pytestmark = pytest.mark.gpu


def _u64(t):
    return t.detach().cpu().numpy().view(np.uint64)


# row blocks of 32, passes of 512 rows, 1 to 8 tiles per workgroup of the export; last tile full, one item, one missing
@pytest.mark.parametrize("m", [1, 33, 64, 65, 192, 257, 511, 512, 513, 1024, 1100])
@pytest.mark.parametrize("n", [1, 1023, 8 * 1024, 9 * 1024 + 1])
def test_index_build_and_export_at_tile_edges(n, m):
    print(f"[edges] build/export n={n} m={m}", flush=True)
    rng = np.random.default_rng(n * 7919 + m)
    lens = rng.integers(0, 20, n)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ids = rng.integers(0, 1 << 62, int(off[-1])).astype(np.int64)
    bloom = st.st_bloom_build(torch.from_numpy(off).cuda(), torch.from_numpy(ids).cuda(), n, m, 3)
    got = _u64(st.st_bloom_export_signatures(bloom))
    assert np.array_equal(got, O.bloom_build(off, ids.view(np.uint64), m, 3))
