"""The memory kept of a freed index is gone with the context that gave it."""
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


def _index(ej, ctx, n):
    col = sd.random_strings(n, n, 180, 220)
    return col, ej.Index(ctx, col.chars, col.offsets, 8, 8, 6, seed=1, L=64)


def _kept(n):
    return 64 * n * 20  # the tables' 20 bytes per string and table


def test_index_freed_after_its_context(ej):
    import torch
    ctx = ej.Context(0)
    print("[gpu-case] index freed after its context", flush=True)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    _, first = _index(ej, ctx, 40000)
    _, second = _index(ej, ctx, 40000)
    first.close()                          # kept by the context ...
    ctx.close()                            # ... and freed with it
    used = before - torch.cuda.mem_get_info()[0]
    assert used >= _kept(40000)
    second.close()
    assert before - torch.cuda.mem_get_info()[0] <= used - _kept(40000)
