"""The attention sums the K ranges' slices of the q|k|v projection: in one, two, four, eight and sixteen ranges, trees of one and two query
tiles, alone and in a batch (whose kernel loads them in larger groups) with the same bits, and against the oracle."""
import numpy as np
import pytest
import torch

import goose_inputs as gi
from util import device_cache_as_oracle, gpu_model, oracle_model, torch_model
from test_gpu_batched import _alone, _batched, _requests, _rows
from test_gpu_parity import _compare_step, _gpu_prefill, tol_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,kv,norm,dtype", [(512, 4, False, "bf16"), (1024, 2, False, "f16"), (2048, 2, True, "bf16"), (2056, 1, False, "bf16"),
                                                  (4096, 2, True, "f16"), (8192, 4, False, "bf16")])
def test_slices_of_every_number_of_ranges(hidden, kv, norm, dtype):
    shape = gi.ModelShape("slices", 1, hidden, 4, 128, 264, 512, dtype=dtype, n_kv_heads=kv, qk_norm=norm)
    tm = torch_model(shape, seed=6, gain_jitter=0.1)
    gm = gpu_model(shape, tm, max_B=64, cap=512, max_rows=192)
    reqs = _requests(gm, shape, [32, 5, 33, 64], [70, 33, 131, 64], [90, 50, 140, 80])
    alone = _alone(gm, reqs)
    _batched(gm, reqs)
    for q, a in zip(reqs, alone):
        assert torch.equal(q["argmax"], a["argmax"]) and torch.equal(q["succ_ids"], a["ids"]) and torch.equal(q["succ_scores"], a["scores"])
        k_b, v_b = _rows(gm, q["kcache"], q["vcache"], 0, a["P"])
        k_a, v_a = _rows(gm, a["k"], a["v"], 0, a["P"])
        assert torch.equal(k_b, k_a) and torch.equal(v_b, v_a)
    om = oracle_model(shape, tm)
    for tree in (gi.tree_random(29, seed=3, spine_len=8), gi.tree_random(64, seed=4, spine_len=8)):
        gm.set_P(0)
        root = int(_gpu_prefill(gm, gi.prefix_tokens(3, 90, shape.vocab), 64)["argmax"][-1].item())
        tokens = gi.draft_tokens_uniform(5, tree.parent, shape.vocab, root)
        _compare_step(shape, gm, om, device_cache_as_oracle(gm, gm.P), np.asarray(tokens, np.int32), tree, tol_for(shape))
    gm.ctx.close()
