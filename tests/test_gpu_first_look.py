"""The first look at a string set (lengths, alphabet, length order) and the
drawing of the randomness at the edges of their launches: joins against the
oracle, bit for bit."""
import numpy as np
import pytest

import synthdata as sd
from tests._gpu_util import pairs_to_codes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ej.lib()
    return ej.Context(0)


def _check(ctx, oracle_lib, chars, offsets, K, r, z, m, L):
    ref = oracle_lib.join(chars, offsets, K, r, z, m, seed=2, L=L)
    print(f"[gpu-case] first look n={len(offsets) - 1} base={offsets[0]} out={len(ref.out)}",
          flush=True)
    res = ctx.join(chars, offsets, K, r, z, m, seed=2, L=L)
    assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
    assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()
    assert res.n_candidates == len(ref.cand) and res.sigma == len(np.unique(
        chars[int(offsets[0]):int(offsets[-1])]))


@pytest.mark.parametrize("letters", [b"ACGT", b"acgtn", b"AZaz@_`{", bytes(range(0, 255)),
                                     b"\x00\x3f\x40\x5f\x60\x7f\x80\xff"])
def test_byte_classes(ctx, oracle_lib, letters):
    col = sd.clusters(5, 30, lambda r, b: 3, lambda r: r.integers(1, 120),
                      lambda r, L: r.poisson(2), letters=letters)
    for cut in (0, 1, 3, 17):  # the text's first byte at any alignment
        _check(ctx, oracle_lib, col.chars, col.offsets[cut:].copy(), 6, 3, 4, 3, 40)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1024, 8191, 8192, 8193, 20000])
def test_length_order(ctx, oracle_lib, n):
    rng = np.random.default_rng(n)
    lens = rng.integers(0, 30, size=n)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
    chars = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, size=int(offsets[-1]))]
    if chars.size == 0:
        chars = np.frombuffer(b"A", np.uint8).copy()
        offsets[-1] = 1
    _check(ctx, oracle_lib, chars, offsets, 2, 2, 3, 10, 25)


@pytest.mark.parametrize("z,m,L,letters", [(64, 64, 30, b"ACGT"), (65, 64, 30, b"ACGT"),
                                           (3, 5, 300, bytes(range(60, 92))),
                                           (3, 5, 300, bytes(range(60, 93)))])
def test_randomness(ctx, oracle_lib, z, m, L, letters):
    """4,096 and 4,160 samples per seed; 32 and 33 letters."""
    col = sd.clusters(6, 20, lambda r, b: 4, lambda r: r.integers(80, 200),
                      lambda r, L: r.poisson(2), letters=letters)
    _check(ctx, oracle_lib, col.chars, col.offsets, 5, 2, z, m, L)
