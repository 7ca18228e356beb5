"""What the admission of a query batch counts: the index strings' match masks,
which the first batch under another verification form than the strips builds,
and the strips' own state per pair."""
import numpy as np
import pytest

import synthdata as sd

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ej.lib()
    return ej.Context(0)


def _mask_words(total, n, sigma):
    return sigma * (total // 32 + n + 1)


def _tail(col, k):
    t = sd.from_strings([col.string(i) for i in range(col.n - k, col.n)])
    return t.chars, t.offsets


@pytest.mark.parametrize("letters", [sd.DNA, sd.PROTEIN25])
def test_index_masks_are_admitted(ctx, oracle_lib, letters):
    """A limit that the masks alone exceed refuses the batch before they are
    requested; the index answers on, and under a limit with room for them."""
    import paper_1702_00093_amd as ej
    col = sd.clusters(41, 60, lambda r, b: 5, lambda r: r.integers(3000, 3400),
                      lambda r, L: r.poisson(20), letters=letters)
    q = sd.from_strings([col.string(i) for i in range(4)])
    Kq = np.full(4, 60, dtype=np.uint32)
    prm = (3, 4, 6)
    ref = oracle_lib.query(col.chars, col.offsets, q.chars, q.offsets, Kq, *prm, seed=1, L=64)
    ix = ej.Index(ctx, col.chars, col.offsets, *prm, seed=1, L=64)
    masks = 4 * _mask_words(int(col.offsets[-1]), col.n, len(letters))
    print(f"[gpu-case] admission of masks letters={len(letters)} bytes={masks}", flush=True)

    def check(res):
        assert res.offsets.astype(np.int64).tolist() == ref[0].astype(np.int64).tolist()
        assert res.ids.tolist() == ref[1].tolist()
        assert res.dist.tolist() == ref[2].astype(np.int32).tolist()

    base = ix.query(q.chars, q.offsets, Kq)
    check(base)
    try:
        ctx.tune_set("verify_mode", 1)
        ix.set_hbm_limit(base.workspace_bytes + masks // 2)
        for _ in range(2):
            with pytest.raises(ej.EmbedJoinError) as e:
                ix.query(q.chars, q.offsets, Kq)
            assert e.value.status == ej.EJ_ENOMEM and "verification" in str(e.value)
        ctx.tune_set("verify_mode", 0)
        check(ix.query(q.chars, q.offsets, Kq))
        ctx.tune_set("verify_mode", 1)
        ix.set_hbm_limit(base.workspace_bytes + masks + 16 * (col.n + 100))
        first = ix.query(q.chars, q.offsets, Kq)
        check(first)
        assert first.workspace_bytes >= masks
        ix.set_hbm_limit(base.workspace_bytes)  # the masks are there now
        check(ix.query(q.chars, q.offsets, Kq))
        ctx.tune_set("verify_mode", 2)
        check(ix.query(q.chars, q.offsets, Kq))
        # a grown index takes them along
        ix.set_hbm_limit(0)
        ix.insert(*_tail(col, 3))
        assert ix.size() == col.n + 3
        grown = ix.query(q.chars, q.offsets, Kq)
        ctx.tune_set("verify_mode", 0)
        strips = ix.query(q.chars, q.offsets, Kq)
        assert grown.ids.tolist() == strips.ids.tolist()
        assert grown.dist.tolist() == strips.dist.tolist()
    finally:
        ctx.tune_set("verify_mode", 0)
        ix.close()


def test_strip_state_is_admitted(ctx):
    """64 band words per pair: 8 bytes each, 8 for the pair, two sets of 9 lists
    and the order, beside the output and the one table's raw candidates."""
    import paper_1702_00093_amd as ej
    col = sd.clusters(43, 1, lambda r, b: 300, lambda r: r.integers(2200, 2201),
                      lambda r, L: r.poisson(4))
    q = sd.from_strings([col.string(i) for i in range(40)])
    Kq = np.full(q.n, 2046, dtype=np.uint32)
    ix = ej.Index(ctx, col.chars, col.offsets, 1, 1, 1, seed=1, L=16)
    print("[gpu-case] admission of strips", flush=True)
    try:
        res = ix.query(q.chars, q.offsets, Kq)
        c = res.n_candidates
        assert c > 2000
        qb = int(q.offsets[-1])
        masks = 4 * _mask_words(qb, q.n, 4) + 24 * (q.n + 1)
        known = ix.workspace_estimate(q.offsets, Kq) + masks + c * (44 + 20)
        assert res.workspace_bytes - known >= c * (8 * 64 + 8 + 2 * 4 * 9 + 4)
    finally:
        ix.close()
