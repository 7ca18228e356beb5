"""Candidates that lie in few large groups (near copies in a row among unrelated
strings): within the limit of the sort in LDS and past it, against the oracle.
Integers: equality."""
import numpy as np
import pytest

from tests._gpu_util import pairs_to_codes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ej.lib()
    return ej.Context(0)


# groups of n / 2,048 first strings: of up to 8,000, 34,000 and 250,000 codes,
# the last two above 16,384 and a 256th of all
@pytest.mark.parametrize("n,copies,r,z", [(3000, 1100, 2, 2), (12000, 1300, 2, 2),
                                          (20000, 2200, 2, 5)])
@pytest.mark.parametrize("plus", [False, True])
def test_copies_in_a_row(ctx, oracle_lib, n, copies, r, z, plus):
    rng = np.random.default_rng(n)
    let = np.frombuffer(b"ACGT", np.uint8)
    X = let[rng.integers(0, 4, size=(n, 24))]
    X[:copies] = X[0]
    k = np.arange(0, copies, 4)
    X[k, rng.integers(0, 24, size=len(k))] = let[rng.integers(0, 4, size=len(k))]
    offs = np.arange(n + 1, dtype=np.uint64) * np.uint64(24)
    args = (X.reshape(-1).copy(), offs, 2, r, z, 12)
    if plus:
        ref = oracle_lib.join_plus(*args, delta=2, T=1, seed=1, L=20)
        res = ctx.join_plus(*args, delta=2, T=1, seed=1, L=20)
    else:
        ref = oracle_lib.join(*args, seed=1, L=20)
        res = ctx.join(*args, seed=1, L=20)
    print(f"[gpu-case] copies in a row n={n} raw={ref.n_raw} cand={len(ref.cand)}", flush=True)
    assert res.n_raw == ref.n_raw and res.n_candidates == len(ref.cand)
    assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
    assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()
