"""Bands of more than 32 words in the strip form, against the CPU oracle: 64
lanes per pair down to as many as the band needs, several strips, 2, 5 and 8 bit
planes.  Integers: equality."""
import numpy as np
import pytest

import synthdata as sd
from tests._gpu_util import to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ej.lib()
    return ej.Context(0)


# Thresholds per pair: those are verified in strips whatever their number.  The
# first strip ends at 2 K + 95 columns (up to 4 letters) or 5 K / 4 + 95, and the
# texts go on behind it; 8,192 pairs and fewer are one strip.
@pytest.mark.parametrize("letters,K,length", [
    (b"ACGT", 800, 2200), (b"ACGT", 1023, 2700), (b"ACGT", 1100, 2900), (b"ACGT", 1500, 3700),
    (b"ACGT", 2046, 4900), (bytes(range(65, 90)), 1100, 2300), (bytes(range(65, 90)), 2046, 3300),
    (bytes(range(40, 90)), 1030, 2200), (bytes(range(40, 90)), 2046, 3300)])
def test_wide_bands(ctx, oracle_lib, letters, K, length):
    import torch
    rng = np.random.default_rng(K)
    col = sd.clusters(K, 5, lambda r, b: 4, lambda r: r.integers(length - 400, length),
                      lambda r, L: r.poisson(K // 2), letters=letters)
    a = rng.integers(0, col.n, size=36)
    b = np.where(rng.random(36) < 0.6, (a + 1) % col.n, rng.integers(0, col.n, size=36))
    # similar pairs: strings of one cluster
    same = np.array([rng.choice(np.flatnonzero(col.labels == col.labels[i])) for i in a])
    b = np.where(rng.random(36) < 0.5, same, b)
    codes = (a.astype(np.uint64) << np.uint64(32)) | b.astype(np.uint64)
    low = np.where(np.arange(36) % 2 == 0, K, rng.integers(0, K + 1, size=36))
    low[0] = K
    want = np.array([oracle_lib.verify_pairs(col.chars, col.offsets, codes[i:i + 1], int(k))[0]
                     for i, k in enumerate(low)], dtype=np.uint32)
    chars, offs = to_device(col)
    for count in (1, 36, 500, 1024, 1025, 4000, 8193, 20000, 135000):
        pick = np.arange(count) % 36
        print(f"[gpu-case] wide K={K} letters={len(letters)} pairs={count}", flush=True)
        got = ctx.verify(chars, offs, torch.from_numpy(codes[pick].astype(np.int64)).cuda(), 0,
                         d_Kq=torch.from_numpy(low[pick].astype(np.int32)).cuda())
        assert np.array_equal(got.cpu().numpy().astype(np.uint32), want[pick])
