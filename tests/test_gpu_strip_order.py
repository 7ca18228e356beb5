"""Pairs of texts of unlike lengths verified in length order, against the CPU
oracle.  Integers: equality."""
import numpy as np
import pytest

import synthdata as sd
from tests._gpu_util import pairs_to_codes, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ej.lib()
    return ej.Context(0)


def _strings(letters, seed):
    """Near copies of short strings of several lengths, and of one long string:
    21,800 pairs of close lengths, whose longest text counts for the rule."""
    rng = np.random.default_rng(seed)
    let = np.frombuffer(letters, np.uint8)
    out = []
    for length, copies in ((60, 105), (120, 105), (200, 105), (300, 105), (17000, 3)):
        base = let[rng.integers(0, len(let), size=length)]
        out += [bytes(sd.mutate(rng, base, int(rng.integers(0, 12)), let)) for _ in range(copies)]
    return sd.from_strings([out[i] for i in rng.permutation(len(out))])


@pytest.mark.parametrize("letters", [b"ACGT", bytes(range(65, 90)), bytes(range(40, 90))])
def test_join_of_unlike_lengths(ctx, oracle_lib, letters):
    import paper_1702_00093_amd as ej
    col = _strings(letters, len(letters))
    ref = oracle_lib.join(col.chars, col.offsets, 40, 4, 6, 1, seed=3, L=32)
    assert len(ref.cand) > 16400  # 2 band words x 16,400 pairs x 17,000 columns: ordered
    chars, offs = to_device(col)
    for flags in (ej.FLAG_TIMING, ej.FLAG_GRAPH, ej.FLAG_GRAPH, ej.FLAG_GRAPH):
        print(f"[gpu-case] ordered join letters={len(letters)} cand={len(ref.cand)} flags={flags}",
              flush=True)
        res = ctx.join(chars, offs, 40, 4, 6, 1, seed=3, L=32, flags=flags)
        assert flags != ej.FLAG_TIMING or res.verify_form == 6
        assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
        assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()


@pytest.mark.parametrize("letters", [b"ACGT", bytes(range(65, 90))])
@pytest.mark.parametrize("count", [8192, 8193, 20011])
def test_thresholds_per_pair(ctx, oracle_lib, letters, count):
    """Order and width classes together; several strips."""
    import torch
    rng = np.random.default_rng(count)
    col = sd.clusters(count, 6, lambda r, b: 4, lambda r: int(60 * 25 ** r.random()),
                      lambda r, L: r.poisson(8), letters=letters)
    col = sd.from_strings([col.string(i) for i in range(col.n)] +
                          [bytes(letters[:4]) * 5000, bytes(letters[:4]) * 4990])
    a = rng.integers(0, col.n - 2, size=400)
    b = np.where(rng.random(400) < 0.7, (a + 1) % (col.n - 2), rng.integers(0, col.n - 2, size=400))
    codes = (a.astype(np.uint64) << np.uint64(32)) | b.astype(np.uint64)
    Kq = rng.integers(0, 200, size=400)
    want = np.array([oracle_lib.verify_pairs(col.chars, col.offsets, codes[i:i + 1], int(k))[0]
                     for i, k in enumerate(Kq)], dtype=np.uint32)
    pick = np.arange(count) % 400
    chars, offs = to_device(col)
    print(f"[gpu-case] ordered pairs={count} letters={len(letters)}", flush=True)
    got = ctx.verify(chars, offs, torch.from_numpy(codes[pick].astype(np.int64)).cuda(), 0,
                     d_Kq=torch.from_numpy(Kq[pick].astype(np.int32)).cuda())
    assert np.array_equal(got.cpu().numpy().astype(np.uint32), want[pick])
