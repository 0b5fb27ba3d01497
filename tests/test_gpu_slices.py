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


@pytest.mark.parametrize("kv,dtype", [(8, "bf16"), (32, "f16")])
def test_contexts_of_more_rows_give_the_same_bits(kv, dtype):
    """A K range's sum is part of a result, so the O product (eight ranges here) has the same ones in contexts of 128, 256 and 512 rows."""
    shape = gi.ModelShape("context", 1, 4096, 32, 128, 512, 512, dtype=dtype, n_kv_heads=kv)
    tm = torch_model(shape, seed=9, gain_jitter=0.1)
    first = None
    for max_rows in (128, 256, 512):
        gm = gpu_model(shape, tm, max_B=128, cap=256, max_rows=max_rows)
        got = []
        for B in (40, 1):
            gm.set_P(0)
            root = int(_gpu_prefill(gm, gi.prefix_tokens(3, 90, shape.vocab), 64)["argmax"][-1].item())
            tree = gi.tree_random(B, seed=3, spine_len=8) if B > 1 else gi.tree_single()
            tokens = np.asarray(gi.draft_tokens_uniform(5, tree.parent, shape.vocab, root), np.int32)
            got.append(gm.verify_step_calls(tokens, tree.parent, tree.is_spine, want_logits=True)["logits"].clone())
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first))
        gm.ctx.close()
