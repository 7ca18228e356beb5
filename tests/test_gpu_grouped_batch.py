"""Length groups that go through one front end together, and those that may
not: against the oracle's grouped join, bit for bit."""
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


def _strings(rng, letters, lens):
    let = np.frombuffer(letters, np.uint8)
    out = []
    for L in lens:
        s = let[rng.integers(0, len(let), size=L)]
        out += [bytes(s), bytes(sd.mutate(rng, s, 2, let)) if L > 4 else bytes(s)]
    return out


@pytest.mark.parametrize("K,L,lens,letters", [
    # walks of 3 x 20 to 3 x 400 steps: with and without a record of all steps
    (8, 0, range(20, 400, 3), b"ACGT"),
    # groups of 63, 64, 65, 128 and 130 strings (chunks of 64 entries)
    (10, 0, [15] * 31 + [35] * 32 + [55] * 33 + [75] * 64 + [95] * 65, b"ACGT"),
    # one group per length
    (0, 0, [0, 0, 1, 1, 5, 40, 90, 90, 130, 200], b"ACGT"),
    # a caller's truncation shorter than some groups' 3 x longest
    (20, 150, range(10, 300, 7), b"ACGT"),
    # 40 letters: short groups lack some and keep a front end of their own
    (6, 0, range(3, 300, 2), bytes(range(48, 88))),
])
def test_groups_together(ctx, oracle_lib, K, L, lens, letters):
    rng = np.random.default_rng(K + len(letters))
    strings = _strings(rng, letters, lens)
    if letters == b"ACGT":  # a run of lengths without the letter T
        strings += _strings(rng, b"ACG", range(500, 520, 2))
    col = sd.from_strings([strings[i] for i in rng.permutation(len(strings))])
    ref = oracle_lib.join_grouped(col.chars, col.offsets, K, 3, 5, 4, seed=7, L=L)
    print(f"[gpu-case] grouped K={K} L={L} n={col.n} cand={len(ref.cand)}", flush=True)
    for _ in range(2):
        res = ctx.join_grouped(col.chars, col.offsets, K, 3, 5, 4, seed=7, L=L)
        assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
        assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()
        assert res.n_candidates == len(ref.cand) and res.n_raw == ref.n_raw
