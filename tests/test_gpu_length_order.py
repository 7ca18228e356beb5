"""The length order at the size where it passes from counting to the sort: joins
against the CPU oracle."""
import numpy as np
import pytest

import synthdata as sd
from tests._gpu_util import pairs_to_codes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4095, 4096, 4097, 8192, 8193])
def test_join(oracle_lib, n):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ctx = ej.Context(0)
    rng = np.random.default_rng(n)
    let = np.frombuffer(b"ACGT", np.uint8)
    out = []
    while len(out) < n:
        s = let[rng.integers(0, 4, size=int(rng.integers(0, 60)))]
        out += [bytes(s), bytes(sd.mutate(rng, s, 1, let))]
    col = sd.from_strings([out[i] for i in rng.permutation(n)])
    ref = oracle_lib.join(col.chars, col.offsets, 2, 2, 3, 8, seed=4, L=24)
    print(f"[gpu-case] length order n={n} cand={len(ref.cand)}", flush=True)
    res = ctx.join(col.chars, col.offsets, 2, 2, 3, 8, seed=4, L=24)
    assert res.n_raw == ref.n_raw and res.n_candidates == len(ref.cand)
    assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
    assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()
    ctx.close()
