"""np_dedup and np_route at the sizes where their kernels change: tile edges, the largest input of every form and the next one,
against the oracle (whole numbers, so exact)."""
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


def _keys(n, bits, skew, seed):
    rng = np.random.default_rng(seed)
    keys = rng.integers(0, 1 << bits, size=n)
    if skew:   # one key takes half of the lookups, a hundred take a quarter
        u = rng.random(n)
        keys[u < 0.5] = (1 << bits) - 1
        few = rng.integers(0, 1 << bits, size=100)
        mid = (u >= 0.5) & (u < 0.75)
        keys[mid] = few[rng.integers(0, 100, size=int(mid.sum()))]
    return keys.astype(np.int64)


SIZES = [1, 2, 63, 64, 65, 2047, 2048, 2049, 24575, 24576, 24577, 65535, 65536, 65537, 131072, 131073, 262144, 262145]


@pytest.mark.parametrize("skew", [False, True])
@pytest.mark.parametrize("bits", [9, 17, 20, 22, 33])
def test_dedup_at_the_edges_of_its_forms(H, bits, skew):
    for n in SIZES:
        H.progress(f"np_dedup n={n} bits={bits} skew={skew}")
        keys = _keys(n, bits, skew, n + bits)
        g, _ = H.gpu_dedup(keys, bits)
        H.assert_dedup_equal(g, keys)


CAPS = [1, 2048, 24576, 24577, 65536, 65537, 300000]


@pytest.mark.parametrize("S,cap", [(S, cap) for S in (1, 37, 1536, 2048, 2049) for cap in CAPS] +
                         [(S, cap) for S in (1, 64, 65) for cap in (1 << 21, (1 << 21) + 1)])  # the largest two-launch form, and past it
def test_route_at_the_edges_of_its_forms(H, S, cap):
    rng = np.random.default_rng(cap + S)
    for U in sorted({0, 1, cap // 3, cap}):      # the bound is the batch size, the count a part of it
        H.progress(f"np_route cap={cap} S={S} U={U}")
        unique = np.sort(rng.choice(1 << 22, size=U, replace=False)).astype(np.int64)
        buf = np.zeros(cap, np.int64)
        buf[:U] = unique
        r = H.B.np_route(H.dev(buf), H.dev(np.array([U], np.int32)), cap, S, 1)
        send_keys, splits, send_offsets, sfu, uts = H.O.route(unique, S, 1)
        for name, want, k in (("send_keys", send_keys, U), ("splits", splits, S), ("send_offsets", send_offsets, S + 1),
                              ("send_from_unique", sfu, U), ("unique_to_send", uts, U)):
            assert np.array_equal(H.host(r[name])[:k], want), (name, cap, S, U)
