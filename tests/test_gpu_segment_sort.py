"""The bucketing sort at the sizes where its form changes: members of a table in
(key bits, length, position) order, against numpy's stable sort."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ej.lib()
    return ej.Context(0)


@pytest.mark.parametrize("n", [1, 2, 63, 65, 511, 512, 513, 2047, 2048, 2049, 4096, 4097, 8191,
                               8192, 8193, 20000])
def test_bucket_order(ctx, n):
    import torch
    rng = np.random.default_rng(n)
    T = 3
    keys = rng.integers(0, (1 << 61) - 1, size=(T, n), dtype=np.int64)
    keys[0] = keys[0, 0]                        # one bucket
    keys[1] &= ~np.int64((1 << 57) - 1)         # 16 buckets
    lens = rng.integers(0, 50, size=n).astype(np.int32)
    d_keys, d_len = torch.from_numpy(keys).cuda(), torch.from_numpy(lens).cuda()
    for bits in (0, 1, 7, 8, 13, 22, 28, 32):   # 0: whole keys
        print(f"[gpu-case] bucket sort n={n} bits={bits}", flush=True)
        ids, _ = ctx.lsh_bucket(d_keys, d_len, key_bits=bits)
        ids = ids.cpu().numpy().reshape(T, n)
        for t in range(T):
            top = keys[t] >> (61 - bits) if bits else keys[t]
            assert np.array_equal(ids[t], np.lexsort((np.arange(n), lens, top)))
