"""Export and import of bf16 layers: the conversion to half and back and the transposition, bit for bit
against numpy, over every bf16 pattern and where a layer passes through the staging area in parts."""
import numpy as np
import pytest

from paper_2603_05959_amd import binding as B

pytestmark = pytest.mark.gpu


def through_half(bits):
    """bf16 bits -> half (saturating, one NaN) -> bf16 bits, round to nearest even both times."""
    f = (bits.astype(np.uint32) << 16).view(np.float32)
    h = np.clip(f, -65504.0, 65504.0).astype(np.float16).astype(np.float32)
    u = h.view(np.uint32)
    r = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    return np.where(np.isnan(f), np.uint16(0x7FC0), r)


@pytest.mark.parametrize("n,H,hybrid", [(1024, 1, None), (341, 3, None), (64, 16, 0.5), (3400, 64, None),
                                        (1, 1, None), (1, 5, 0.5), (64, 1, None), (65, 1, None)])   # around 16 KB: one copy, and two
def test_round_trip_is_bf16_through_half(n, H, hybrid):
    cache = B.Cache(2, H, 64, 7, 64, max(n, 7), "bf16", hybrid_beta=hybrid)
    rng = np.random.default_rng(n)
    # every pattern once where the layer is large enough, finite ones only where a centroid is built
    k = np.resize(rng.permutation(65536).astype(np.uint16), (n, H, 64))
    if hybrid is not None:
        k = np.where((k & 0x7F80) == 0x7F80, np.uint16(0x3F80), k)
    v = k[::-1].copy()
    ids, ss, flags = np.arange(n, dtype=np.uint32), rng.random(n).astype(np.float32), (rng.random(n) < 0.2).astype(np.uint8)
    B.ovggt_cache_import(cache.h, 1, n, n, ids, k, v, ss, flags, cache.stream)
    ke, ve, ie, se, fe = np.zeros_like(k), np.zeros_like(v), np.zeros_like(ids), np.zeros_like(ss), np.zeros_like(flags)
    B.ovggt_cache_export(cache.h, 1, ie, ke, ve, se, fe, cache.stream)
    assert np.array_equal(ke, through_half(k)) and np.array_equal(ve, through_half(v))
    assert np.array_equal(ie, ids) and np.array_equal(se, ss) and np.array_equal(fe, flags)
    only_v = np.zeros_like(v)
    B.ovggt_cache_export(cache.h, 1, None, None, only_v, None, None, cache.stream)
    assert np.array_equal(only_v, ve)
    assert cache.size(0) == 0
    cache.close()
