"""The whole join as a graph where the same buffers come to hold strings of
unlike lengths, which are verified in another order: contents of either kind are
captured and replayed, with the results of the joins without a graph."""
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


def _strings(short):
    """20 clusters of 40 copies, 15,600 pairs in bands of 8 words, and nine
    strings alone: all of 4,500 to 5,000 letters, or one of 1,500; as many
    letters and the same longest string either way."""
    rng = np.random.default_rng(11)
    let = np.frombuffer(b"ACGT", np.uint8)
    out = []
    for c in range(20):
        base = let[rng.integers(0, 4, size=5000 if c == 0 else 4500)]
        for _ in range(40):
            s = base.copy()
            at = rng.integers(0, len(s), size=20)
            s[at] = let[rng.integers(0, 4, size=20)]
            out.append(bytes(s))
    for i in range(9):
        length = 4500 if not short else 1500 if i == 0 else 4875
        out.append(bytes(let[rng.integers(0, 4, size=length)]))
    return sd.from_strings(out)


def test_lengths_change_in_the_buffers(ctx):
    import paper_1702_00093_amd as ej
    sets = [_strings(False), _strings(True)]
    assert sets[0].offsets[-1] == sets[1].offsets[-1]
    chars, offs = to_device(sets[0])
    other = [to_device(s) for s in sets]
    args = dict(K=250, r=4, z=6, m=10, seed=5, L=64)
    want = []
    for c, o in other:
        res = ctx.join(c, o, **args)
        assert res.n_candidates > 15000
        want.append((pairs_to_codes(res.pairs), np.asarray(res.dist)))

    def run(kind, times):
        chars.copy_(other[kind][0])
        offs.copy_(other[kind][1])
        ran = []
        for _ in range(times):
            print(f"[gpu-case] graph of changing lengths kind={kind}", flush=True)
            res = ctx.join(chars, offs, flags=ej.FLAG_GRAPH, **args)
            assert np.array_equal(pairs_to_codes(res.pairs), want[kind][0])
            assert np.array_equal(np.asarray(res.dist), want[kind][1])
            ran.append(res.graph)
        return ran

    # sized by the host, then on the device; then unlike lengths, anew
    assert run(0, 2) == [0, 1]
    assert run(1, 4) == [0, 1, 2, 2]
    assert run(0, 3)[-1] == 2
    assert run(1, 3)[-1] == 2
