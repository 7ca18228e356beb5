"""De-duplication of candidates whose groups hold many distinct codes: sorted in
LDS, or all together when a group is too large, against the oracle.  Integers:
equality."""
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


def _alike(n, length, every, seed):
    """n copies of one string, every `every`-th with one edit."""
    rng = np.random.default_rng(seed)
    let = np.frombuffer(b"ACGT", np.uint8)
    base = let[rng.integers(0, 4, size=length)]
    return sd.from_strings([bytes(sd.mutate(rng, base, 1, let)) if i % every == 0 else bytes(base)
                            for i in range(n)])


def _equal(res, ref):
    assert res.n_raw == ref.n_raw and res.n_candidates == len(ref.cand)
    assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
    assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()


# groups (of one first string each) of up to n distinct codes, z * r times over:
# within the hash table, sorted at 1, 8 and 16 rounds, and past the LDS
@pytest.mark.parametrize("n,r,z", [(900, 2, 2), (1030, 1, 1), (1100, 2, 4), (1500, 2, 5),
                                   (1500, 4, 5), (2049, 2, 3)])
def test_join(ctx, oracle_lib, n, r, z):
    col = _alike(n, 24, 5, n)
    ref = oracle_lib.join(col.chars, col.offsets, 2, r, z, 2, seed=1, L=20)
    print(f"[gpu-case] group sort n={n} raw={ref.n_raw} cand={len(ref.cand)}", flush=True)
    _equal(ctx.join(col.chars, col.offsets, 2, r, z, 2, seed=1, L=20), ref)


@pytest.mark.parametrize("n,T,delta", [(40, 1, 1), (300, 2, 1), (700, 2, 2), (700, 3, 2),
                                       (1300, 2, 1)])
def test_plus(ctx, oracle_lib, n, T, delta):
    """Runs of at least T equal tuples, and one of each pair: with K = 4, 4 or 2
    suffixes per string."""
    col = _alike(n, 24, 3, n)
    ref = oracle_lib.join_plus(col.chars, col.offsets, 4, 2, 3, 3, delta=delta, T=T, seed=1, L=20)
    print(f"[gpu-case] tuple groups n={n} T={T} raw={ref.n_raw} cand={len(ref.cand)}", flush=True)
    _equal(ctx.join_plus(col.chars, col.offsets, 4, 2, 3, 3, delta=delta, T=T, seed=1, L=20), ref)


@pytest.mark.parametrize("n", [2, 3, 1030, 2100])
def test_union_with_short_pairs(ctx, oracle_lib, n):
    """The union of the tables' candidates and all short pairs, in groups of up to
    n codes and by the device-wide sort."""
    col = _alike(n, 24, 5, n)
    ref = oracle_lib.join(col.chars, col.offsets, 2, 2, 2, 4, seed=1, L=20, exact_len=24)
    print(f"[gpu-case] union n={n} cand={len(ref.cand)}", flush=True)
    for knob in (0, 1):
        ctx.tune_set("dedup_sort", knob)
        try:
            _equal(ctx.join(col.chars, col.offsets, 2, 2, 2, 4, seed=1, L=20, exact_len=24), ref)
        finally:
            ctx.tune_set("dedup_sort", 0)
