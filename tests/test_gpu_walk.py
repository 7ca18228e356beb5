"""Walks longer than the recorded ones: sampled steps at the edges of pairs,
groups and staged windows, every code width, strings used up early.  Keys through
the join against the oracle: equality."""
import numpy as np
import pytest

import synthdata as sd
from tests._gpu_util import to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1702_00093_amd as ej
    ej.lib()
    return ej.Context(0)


@pytest.mark.parametrize("sigma", [1, 2, 4, 5, 16, 17, 32, 33])
@pytest.mark.parametrize("L,z,m", [(257, 1, 1), (272, 7, 9), (300, 1, 64), (515, 13, 5),
                                   (2000, 16, 20), (4001, 2, 3)])
def test_keys(ctx, oracle_lib, sigma, L, z, m):
    rng = np.random.default_rng(sigma * 10000 + L)
    letters = bytes(range(50, 50 + sigma))
    lens = np.concatenate([rng.integers(0, 1500, size=120), [0, 1, 2, 15, 16, 17, 4100]])
    col = sd.from_strings([bytes(np.frombuffer(letters, np.uint8)[
        rng.integers(0, sigma, size=int(n))]) for n in lens] + [letters])
    r = 3
    ref = oracle_lib.join(col.chars, col.offsets, 5, r, z, m, seed=4, L=L)
    chars, offs = to_device(col)
    print(f"[gpu-case] walk sigma={sigma} L={L} samples={z * m}", flush=True)
    keys, _, _, _ = ctx.embed(chars, offs, r, z, m, seed=4, L=L)
    got = keys.cpu().numpy().astype(np.uint64).reshape(r * z, col.n)
    assert np.array_equal(got, np.asarray(ref.keys, dtype=np.uint64).reshape(r * z, col.n))
