"""Calls that reach the caps of a batch: more pairs than one batch of strips
holds, length groups of more entries, samples or lengths than one front end
takes.  Against the CPU oracle; integers: equality."""
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


# 2^24 pairs a batch up to 16 band words, 2^23 above; a pair of long texts among
# them makes it several strips, in length order
@pytest.mark.parametrize("K,count,per_pair", [(5, (1 << 24) + 1000, False),
                                              (40, (1 << 24) + 1000, True),
                                              (530, (1 << 23) + 1000, False),
                                              (530, (1 << 24) + 1000, True)])
def test_batches_of_pairs(ctx, oracle_lib, K, count, per_pair):
    import torch
    rng = np.random.default_rng(K)
    short = sd.clusters(K, 20, lambda r, b: 4, lambda r: r.integers(12, 40),
                        lambda r, L: r.poisson(3))
    let = np.frombuffer(b"ACGT", np.uint8)
    base = let[rng.integers(0, 4, size=2500)]
    col = sd.from_strings(short.strings() + [bytes(base), bytes(sd.mutate(rng, base, 4, let))])
    a = rng.integers(0, short.n, size=997)
    b = rng.integers(0, short.n, size=997)
    a[500], b[500] = short.n, short.n + 1
    codes = (a.astype(np.uint64) << np.uint64(32)) | b.astype(np.uint64)
    Kq = rng.integers(0, K + 1, size=997) if per_pair else np.full(997, K)
    Kq[500] = K
    want = np.array([oracle_lib.verify_pairs(col.chars, col.offsets, codes[i:i + 1], int(k))[0]
                     for i, k in enumerate(Kq)], dtype=np.int32)
    pick = torch.arange(count, device="cuda") % 997
    # the long pair a few hundred times, in every batch
    pick = torch.where((pick == 500) & (torch.arange(count, device="cuda") % 50 != 0), 0, pick)
    chars, offs = to_device(col)
    print(f"[gpu-case] batches K={K} pairs={count} per-pair={per_pair}", flush=True)
    got = ctx.verify(chars, offs, torch.from_numpy(codes.astype(np.int64)).cuda()[pick],
                     0 if per_pair else K,
                     d_Kq=torch.from_numpy(Kq.astype(np.int32)).cuda()[pick] if per_pair else None)
    assert torch.equal(got.int(), torch.from_numpy(want).cuda()[pick])


def _equal(res, ref):
    assert res.n_raw == ref.n_raw and res.n_candidates == len(ref.cand)
    assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
    assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()


def test_group_entries(ctx, oracle_lib):
    """More than 2^25 table entries: 1,024 tables, 34,000 strings counted once
    per group."""
    col = sd.clusters(5, 4300, lambda r, b: 4, lambda r: r.integers(12, 60),
                      lambda r, L: r.poisson(1))
    ref = oracle_lib.join_grouped(col.chars, col.offsets, 4, 32, 32, 14, seed=1, L=24)
    print(f"[gpu-case] group entries n={col.n} cand={len(ref.cand)}", flush=True)
    _equal(ctx.join_grouped(col.chars, col.offsets, 4, 32, 32, 14, seed=1, L=24), ref)


@pytest.mark.parametrize("long,r,z,m", [(0, 32, 16, 64), (4200000, 2, 3, 4)])
def test_groups(ctx, oracle_lib, long, r, z, m):
    """600 groups (K = 0: one per length): more than 2^24 samples, or lengths that
    pass 31 bits set one behind the other."""
    rng = np.random.default_rng(r)
    let = np.frombuffer(b"ACGT", np.uint8)
    strings = []
    for length in range(8, 608):
        s = bytes(let[rng.integers(0, 4, size=length)])
        strings += [b"ACGT" + s, b"ACGT" + s]
    if long:
        s = bytes(let[rng.integers(0, 4, size=long)])
        strings += [s, s]
    col = sd.from_strings([strings[i] for i in rng.permutation(len(strings))])
    ref = oracle_lib.join_grouped(col.chars, col.offsets, 0, r, z, m, seed=3, L=16)
    assert len(ref.out) == len(strings) // 2
    print(f"[gpu-case] groups n={col.n} long={long}", flush=True)
    _equal(ctx.join_grouped(col.chars, col.offsets, 0, r, z, m, seed=3, L=16), ref)
