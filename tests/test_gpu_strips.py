"""The strip form of the verification at its edges, against the CPU oracle:
word edges of the band, every number of lanes per pair, alphabets of 2, 5 and 8
bit planes, thresholds per pair, several strips.  Integers: equality."""
import numpy as np
import pytest

import synthdata as sd
from tests._gpu_util import to_device

pytestmark = pytest.mark.gpu

BYTES = bytes(range(40, 90))  # 50 letters: 8 planes


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ej.lib()
    return ej.Context(0)


def _check(ctx, oracle_lib, col, codes, K, Kq=None, times=(1,)):
    import torch
    if Kq is None:
        want = oracle_lib.verify_pairs(col.chars, col.offsets, codes, K)
    else:
        want = np.array([oracle_lib.verify_pairs(col.chars, col.offsets, codes[i:i + 1], int(k))[0]
                         for i, k in enumerate(Kq)], dtype=np.uint32)
    chars, offs = to_device(col)
    for t in times:
        print(f"[gpu-case] strips K={K} pairs={len(codes) * t} per-pair={Kq is not None}",
              flush=True)
        pairs = torch.from_numpy(np.tile(codes, t).astype(np.int64)).cuda()
        kq = None if Kq is None else torch.from_numpy(np.tile(Kq, t).astype(np.int32)).cuda()
        got = ctx.verify(chars, offs, pairs, K, d_Kq=kq).cpu().numpy().astype(np.uint32)
        assert np.array_equal(got.reshape(t, -1), np.tile(want, (t, 1)))


def _pairs(rng, n, count):
    # half neighbours in a cluster's order, half any two
    a = rng.integers(0, n, size=count)
    b = np.where(rng.random(count) < 0.5, (a + 1) % n, rng.integers(0, n, size=count))
    return (a.astype(np.uint64) << np.uint64(32)) | b.astype(np.uint64)


@pytest.mark.parametrize("letters,K", [(sd.DNA, 30), (sd.DNA, 31), (sd.DNA, 94), (sd.DNA, 95),
                                       (sd.DNA, 255), (sd.DNA, 510), (sd.DNA, 511),
                                       (BYTES[:25], 63), (BYTES[:25], 286), (BYTES, 127),
                                       (BYTES, 530), (sd.DNA, 2046)])
def test_lanes_per_pair(ctx, oracle_lib, letters, K):
    """500 pairs, repeated: 16 lanes per pair down to one (131,072 lanes fill
    the chip), the last strip of each at other lane counts than the first."""
    rng = np.random.default_rng(K)
    long = min(6 * K, 1500) + 40  # several strips
    col = sd.clusters(K, 8, lambda r, b: 4, lambda r: r.integers(long // 2, long),
                      lambda r, L: r.poisson(max(1, K // 3)), letters=letters)
    _check(ctx, oracle_lib, col, _pairs(rng, col.n, 500), K, times=(1, 17, 35, 70, 140, 280))


@pytest.mark.parametrize("letters", [sd.DNA, BYTES[:25], BYTES])
def test_per_pair_thresholds(ctx, oracle_lib, letters):
    rng = np.random.default_rng(5)
    col = sd.clusters(9, 10, lambda r, b: 4, lambda r: r.integers(0, 1500),
                      lambda r, L: r.poisson(20), letters=letters)
    codes = _pairs(rng, col.n, 400)
    _check(ctx, oracle_lib, col, codes, 0, Kq=rng.integers(0, 300, size=400), times=(1, 90, 400))


def test_long_strings(ctx, oracle_lib):
    """Strips past the first two: texts of 7,000 letters at small thresholds."""
    rng = np.random.default_rng(3)
    col = sd.clusters(4, 6, lambda r, b: 4, lambda r: r.integers(3000, 7000),
                      lambda r, L: r.poisson(40))
    _check(ctx, oracle_lib, col, _pairs(rng, col.n, 200), 150, times=(1, 40, 700))
