"""The autotuner leaves alone what the form in use does not read."""
import numpy as np
import pytest

import synthdata as sd
from tests._gpu_util import pairs_to_codes, to_device

pytestmark = pytest.mark.gpu


def test_knobs_of_other_forms_stay(oracle_lib):
    import paper_1702_00093_amd as ej
    ctx = ej.Context(0)
    col = sd.clusters(3, 40, lambda r, b: 5, lambda r: r.integers(300, 500),
                      lambda r, L: r.poisson(8))
    prm = dict(K=25, r=4, z=6, m=6, seed=2, L=48)
    ref = oracle_lib.join(col.chars, col.offsets, 25, 4, 6, 6, seed=2, L=48)
    chars, offs = to_device(col)
    default = ctx.knobs()
    strips = ("verify_mode", "verify_wpl", "verify_ring", "verify_pass1_cols", "verify_lds_budget",
              "verify_blocks_per_cu", "verify_len_order")
    for trial in range(6):
        print(f"[gpu-case] autotune {trial}", flush=True)
        _, knobs = ctx.autotune(chars, offs, reps=1, **prm)
        if all(knobs[k] == default[k] for k in strips):
            assert knobs["verify_order"] == default["verify_order"]
            assert knobs["verify_split"] == default["verify_split"]
        res = ctx.join(chars, offs, **prm)
        assert pairs_to_codes(res.pairs).tolist() == ref.out.tolist()
        assert res.dist.tolist() == ref.out_dist.astype(np.int32).tolist()
        for k, v in default.items():
            ctx.tune_set(k, v)
    ctx.close()
