"""The probe of a query batch where its search can go wrong: runs of equal
keys (duplicates), keys far from evenly spread, tables of 1 to a few entries,
and codes of more than 32 bits.  Against the oracle, or against the same
queries in small batches: equality."""
import numpy as np
import pytest

import synthdata as sd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ej():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ej.lib()
    return ej


@pytest.mark.parametrize("case", ["one", "few", "copies", "two_letters"])
def test_probe_matches_oracle(ej, oracle_lib, case):
    rng = np.random.default_rng(3)

    def rand(n, k=4):
        return bytes(b"ACGT"[:k][i] for i in rng.integers(0, k, size=n))

    if case == "one":
        strings = [rand(50)]
    elif case == "few":
        strings = [rand(int(n)) for n in (0, 1, 40, 41, 41, 60, 60)]
    elif case == "copies":  # long runs of one key among others
        base = [rand(80) for _ in range(4)]
        strings = [base[i % 4] for i in range(900)] + [rand(80) for _ in range(300)]
    else:  # short walks on two letters: few distinct keys, some very frequent
        strings = [rand(int(n), 2) for n in rng.integers(1, 12, size=1500)]
    col = sd.from_strings(strings)
    q = sd.from_strings([strings[i % len(strings)] for i in range(0, 90, 2)] +
                        [rand(int(n), 2 if case == "two_letters" else 4)
                         for n in rng.integers(1, 90, size=20)])
    if case == "one":
        q = sd.from_strings([strings[0]] * 3)
    Kq = rng.integers(0, 6, size=q.n).astype(np.uint32)
    r, z, m, L = 4, 4, 3, 24
    ref = oracle_lib.query(col.chars, col.offsets, q.chars, q.offsets, Kq, r, z, m, seed=5, L=L)
    ix = ej.Index(ej.Context(0), col.chars, col.offsets, r, z, m, seed=5, L=L)
    print(f"[gpu-case] probe {case} n={col.n} nq={q.n} hits={len(ref[1])}", flush=True)
    res = ix.query(q.chars, q.offsets, Kq)
    assert res.offsets.astype(np.uint64).tolist() == ref[0].tolist()
    assert res.ids.astype(np.uint32).tolist() == ref[1].tolist()
    assert res.dist.astype(np.int64).tolist() == ref[2].astype(np.int64).tolist()
    ix.close()


def test_codes_above_32_bits(ej):
    """70,000 queries on 70,000 strings (34-bit codes) and the same queries 1,000
    at a time (27 bits)."""
    rng = np.random.default_rng(8)
    n = 70000
    chars = np.frombuffer(b"ACGT", np.uint8)[rng.integers(0, 4, size=40 * n)]
    offs = np.arange(0, 40 * n + 1, 40, dtype=np.uint64)
    ix = ej.Index(ej.Context(0), chars, offs, 2, 2, 8, seed=1, L=40)
    q = chars.reshape(n, 40).copy()
    q[:, 39] = ord("A")
    Kq = np.full(n, 1, np.uint32)
    print("[gpu-case] probe with 34-bit codes", flush=True)
    whole = ix.query(q.reshape(-1), offs, Kq)
    assert len(whole.ids) >= n // 2
    for a in (0, 31000, 69000):
        part = ix.query(q[a:a + 1000].reshape(-1), offs[:1001], Kq[:1000])
        lo, hi = int(whole.offsets[a]), int(whole.offsets[a + 1000])
        assert np.array_equal(part.ids, whole.ids[lo:hi])
        assert np.array_equal(part.dist, whole.dist[lo:hi])
        assert np.array_equal(part.offsets + lo, whole.offsets[a:a + 1001])
    ix.close()


def test_index_memory_is_reused(ej, oracle_lib):
    """Indexes of other sizes built in the memory of freed ones, one grown by an
    insert, two alive at a time: every one answers as the oracle does."""
    ctx = ej.Context(0)
    r, z, m, L = 3, 4, 4, 32
    held = []
    for i, (bases, letters) in enumerate([(60, b"ACGT"), (50, b"ACGT"), (58, sd.DNA), (9, b"ACGT"),
                                          (60, bytes(range(65, 85))), (61, b"ACGT")]):
        col = sd.clusters(30 + i, bases, lambda rr, b: 4, lambda rr: rr.integers(60, 200),
                          lambda rr, LL: rr.poisson(3), letters=letters)
        Kq = np.full(20, 8, np.uint32)
        q, qo = col.chars[:int(col.offsets[20])], col.offsets[:21]
        print(f"[gpu-case] index memory {i} n={col.n}", flush=True)
        ix = ej.Index(ctx, col.chars, col.offsets, r, z, m, seed=i, L=L)
        ref = oracle_lib.query(col.chars, col.offsets, q, qo, Kq, r, z, m, seed=i, L=L)
        if i % 2:
            ix.insert(col.chars, col.offsets)  # (queries below find both copies)
        held.append((ix, q, qo, Kq, ref, i % 2, col.n))
        if len(held) > 2:
            held.pop(0)[0].close()
        for jx, jq, jqo, jK, (ro, ri, rd), twice, n in held:
            res = jx.query(jq, jqo, jK)
            if twice:
                for k in range(len(jqo) - 1):
                    got = res.ids[int(res.offsets[k]):int(res.offsets[k + 1])]
                    want = ri[int(ro[k]):int(ro[k + 1])]
                    assert sorted(got.tolist()) == sorted([*want, *(want.astype(np.int64) + n)])
            else:
                assert res.offsets.astype(np.uint64).tolist() == ro.tolist()
                assert res.ids.astype(np.uint32).tolist() == ri.tolist()
                assert res.dist.astype(np.int64).tolist() == rd.astype(np.int64).tolist()
    for jx, *_ in held:
        jx.close()
