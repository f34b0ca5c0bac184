"""Pooled forward at bag lengths around the number of rows a lane group keeps in flight (4, 8 and 16, chosen by the mean bag
length and the number of bags).  The sum runs in fp32 in ascending lookup order, so a sequential fp32 sum in numpy gives the
same bits whichever form runs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import gpu_helpers
    return gpu_helpers


# mean below 8; around 8 to 32; 32 and more with few bags; the same with many bags
LENGTHS = {"short": [0, 1, 2, 3, 4, 5, 7, 9, 12], "middle": [0, 1, 7, 8, 9, 15, 16, 17, 31, 33], "long": [15, 16, 17, 31, 32, 33, 63, 64, 65, 130]}


@pytest.mark.parametrize("table", ["float32", "bfloat16", "float16"])
@pytest.mark.parametrize("dim", [8, 20, 64, 128])
@pytest.mark.parametrize("lengths,repeat", [("short", 3), ("middle", 3), ("long", 2), ("long", 1700)])
def test_pooled_sums_match_a_sequential_fp32_sum(H, table, dim, lengths, repeat):
    import torch
    if repeat > 100 and dim != 64:
        pytest.skip("the many-bag form once per table type")
    rng = np.random.default_rng(dim + repeat)
    R = 500
    lens = np.tile(np.array(LENGTHS[lengths]), repeat)
    rng.shuffle(lens)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    keys = rng.integers(0, R, size=int(off[-1])).astype(np.int64)
    t = torch.from_numpy(rng.standard_normal((R, dim)).astype(np.float32)).to(getattr(torch, table))
    rows = t.float().numpy()
    got, _ = H.B.np_lookup_fwd_t(t.cuda(), H.dev(keys), None, H.dev(off), keys.size, H.B.POOL_SUM)
    got = H.host(got)
    want = np.zeros((lens.size, dim), np.float32)
    for k in range(int(lens.max())):       # the k-th lookup of every bag that has one
        has = lens > k
        want[has] += rows[keys[off[:-1][has] + k]]
    assert np.array_equal(got, want)
