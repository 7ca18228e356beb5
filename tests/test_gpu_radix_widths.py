"""The general radix sort (segments of more than 8,192 entries) at every digit
width the knob takes: odd, even and merged numbers of passes, values gathered
and generated, long runs of one digit.  Against numpy's stable sort and the
oracle's join."""
import numpy as np
import pytest

import synthdata as sd
from tests._gpu_util import pairs_to_codes

pytestmark = pytest.mark.gpu

WIDTHS = (4, 5, 6, 7, 8, 9, 10, 11)


@pytest.fixture()
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ctx = ej.Context(0)
    yield ctx
    ctx.close()


@pytest.mark.parametrize("n", [8193, 10000, 20481])
def test_bucket_order(ctx, n):
    import torch
    rng = np.random.default_rng(n)
    T = 3
    keys = rng.integers(0, (1 << 61) - 1, size=(T, n), dtype=np.int64)
    keys[0, : n // 2] = keys[0, 0]              # one run of half the segment
    keys[1] &= ~np.int64((1 << 57) - 1)         # 16 buckets
    lens = rng.integers(0, 50, size=n).astype(np.int32)
    d_keys, d_len = torch.from_numpy(keys).cuda(), torch.from_numpy(lens).cuda()
    for width in WIDTHS:
        ctx.tune_set("radix_bits", width)
        for bits in (0, 1, 5, 8, 9, 13, 16, 17, 22, 24, 27, 32):   # 0: whole keys
            print(f"[gpu-case] radix n={n} width={width} bits={bits}", flush=True)
            ids, _ = ctx.lsh_bucket(d_keys, d_len, key_bits=bits)
            ids = ids.cpu().numpy().reshape(T, n)
            for t in range(T):
                top = keys[t] >> (61 - bits) if bits else keys[t]
                assert np.array_equal(ids[t], np.lexsort((np.arange(n), lens, top)))


def test_join(ctx, oracle_lib):
    """More than 8,192 strings: the first pass makes the ranks itself."""
    col = sd.clusters(8, 3001, lambda r, b: 3, lambda r: r.integers(24, 40),
                      lambda r, L: r.poisson(1))
    ref = oracle_lib.join(col.chars, col.offsets, 3, 2, 3, 6, seed=4, L=24)
    assert len(ref.out) > 3000
    for width in WIDTHS:
        for key_bits in (0, 7, 16, 21, 32):
            for dedup in (0, 1):
                print(f"[gpu-case] radix join width={width} key bits={key_bits} sort={dedup}",
                      flush=True)
                ctx.tune_set("radix_bits", width)
                ctx.tune_set("bucket_key_bits", key_bits)
                ctx.tune_set("dedup_sort", dedup)
                res = ctx.join(col.chars, col.offsets, 3, 2, 3, 6, seed=4, L=24)
                assert res.n_raw == ref.n_raw and res.n_candidates == len(ref.cand)
                assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
                assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()
