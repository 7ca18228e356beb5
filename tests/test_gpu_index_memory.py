"""The memory kept of a freed index: counted, of the last index only, one piece
per device, and gone with the context that gave it."""
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


def _index(ej, ctx, n):
    col = sd.random_strings(n, n, 180, 220)
    return col, ej.Index(ctx, col.chars, col.offsets, 8, 8, 6, seed=1, L=64)


def _kept(n):
    return 64 * n * 20  # the tables' 20 bytes per string and table


def _answers(ej, oracle_lib, ctx, col, ix):
    q = sd.from_strings([col.string(i) for i in range(5)])
    Kq = np.full(5, 20, dtype=np.uint32)
    ref = oracle_lib.query(col.chars, col.offsets, q.chars, q.offsets, Kq, 8, 8, 6, seed=1, L=64)
    res = ix.query(q.chars, q.offsets, Kq)
    assert res.ids.tolist() == ref[1].tolist()


def test_only_the_last_index_is_kept(ej, oracle_lib):
    ctx = ej.Context(0)
    print("[gpu-case] kept index memory", flush=True)
    _index(ej, ctx, 20000)[1].close()
    _index(ej, ctx, 20000)[1].close()      # reuses it, and has grown the workspace
    held = ctx.workspace_bytes
    col, ix = _index(ej, ctx, 20000)
    assert ctx.workspace_bytes <= held - _kept(20000)  # in use, not kept
    _answers(ej, oracle_lib, ctx, col, ix)
    ix.close()
    held = ctx.workspace_bytes
    col, ix = _index(ej, ctx, 500)         # too small for it: the large piece goes
    assert ctx.workspace_bytes <= held - _kept(20000)
    _answers(ej, oracle_lib, ctx, col, ix)
    ix.close()
    assert ctx.workspace_bytes <= held - _kept(20000) + 2 * _kept(500) + 1000000
    ctx.close()


def test_one_piece_for_two_contexts(ej, oracle_lib):
    a, b = ej.Context(0), ej.Context(0)
    print("[gpu-case] kept index memory, two contexts", flush=True)
    _index(ej, a, 20000)[1].close()
    _index(ej, b, 20000)[1].close()        # a's piece, given by b now
    held_a, held_b = a.workspace_bytes, b.workspace_bytes
    col, ix = _index(ej, a, 20000)
    assert a.workspace_bytes == held_a     # a kept nothing
    assert b.workspace_bytes <= held_b - _kept(20000)
    _answers(ej, oracle_lib, a, col, ix)
    ix.close()
    assert a.workspace_bytes >= held_a + _kept(20000)
    a.close()
    col, ix = _index(ej, b, 20000)
    _answers(ej, oracle_lib, b, col, ix)
    ix.close()
    b.close()


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
