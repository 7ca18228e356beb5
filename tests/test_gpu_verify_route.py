"""Which verification form a join's candidates take: strips, or the two-pass
form where that is the faster one; the result against the CPU oracle."""
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


@pytest.mark.parametrize("letters,K,n,form", [
    (b"ACGT", 60, 230, 6),                   # two words: always strips
    (b"ACGT", 100, 200, 6),                  # 4 words x 19,900 pairs: not a lane each
    (b"ACGT", 200, 220, 6),                  # 7 words x 24,000 pairs
    (b"ACGT", 200, 290, 5),                  # 7 words x 42,000 pairs
    (b"ACGT", 300, 110, 6),                  # few pairs
    (b"ACGTN", 100, 200, 6),                 # 5 planes, 4 words x 20,000 pairs
    (b"ACGTN", 100, 245, 5),                 # 4 words x 30,000 pairs
    (b"ACGTN", 100, 120, 6),
    (bytes(range(65, 85)), 300, 220, 5),     # 20 letters
    (bytes(range(65, 90)), 300, 200, 5),     # 25 letters: up to 32,768 pairs
    (bytes(range(65, 90)), 300, 270, 6),
    (bytes(range(40, 80)), 300, 220, 6),     # 8 planes
])
def test_join_form(ctx, oracle_lib, letters, K, n, form):
    import paper_1702_00093_amd as ej
    rng = np.random.default_rng(K + n)
    let = np.frombuffer(letters, np.uint8)
    base = let[rng.integers(0, len(let), size=120)]
    col = sd.from_strings([bytes(sd.mutate(rng, base, int(rng.integers(0, 14)), let))
                           for _ in range(n)] + [(bytes(letters) * 30)[:120]])
    ref = oracle_lib.join(col.chars, col.offsets, K, 4, 6, 1, seed=5, L=60)
    assert len(ref.cand) >= 0.98 * n * (n - 1) / 2
    chars, offs = to_device(col)
    for flags in (ej.FLAG_TIMING, ej.FLAG_GRAPH, ej.FLAG_GRAPH, ej.FLAG_GRAPH):
        print(f"[gpu-case] route letters={len(letters)} K={K} cand={len(ref.cand)} flags={flags}",
              flush=True)
        res = ctx.join(chars, offs, K, 4, 6, 1, seed=5, L=60, flags=flags)
        assert flags != ej.FLAG_TIMING or res.verify_form == form
        assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
        assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()
