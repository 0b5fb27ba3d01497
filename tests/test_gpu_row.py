"""Passes of a single row: the projections form their operand row themselves (norm, merge of the attention's key splits), with the same bits as
the separate launches that a row takes beside other requests."""
import dataclasses

import numpy as np
import pytest
import torch

import goose_inputs as gi
from paper_2604_02047_amd import ModelDesc
from paper_2604_02047_amd.runner import GooseModel
from util import device_cache_as_oracle, gpu_model, oracle_model, torch_model
from test_gpu_batched import _alone, _batched, _requests, _rows
from test_gpu_parity import _compare_step, _gpu_prefill, tol_for

pytestmark = pytest.mark.gpu


# rows of up to 1024, 4096 and 8192 columns, no multiple of 128; head sizes, grouped queries and q/k norm; prefixes of one key split, two and
# three (merged in the O projection); both types and operand modes; K in one, two and four ranges; workgroups of five wavefronts (1120 gate/up
# tiles; 516 of q|k|v and 137 of O in contexts of more than 64 rows), whose rows gather four slices, eight, or none; contexts of more than 64 rows,
# where O has eight ranges; O and down in 17 ranges together, which is one too many for the row kernels
@pytest.mark.parametrize("hidden,heads,head_dim,ffn,kv,norm,dtype,act_mode,P,max_rows,own", [
    (256, 4, 64, 688, 4, False, "bf16", 0, 40, 64, True), (1032, 8, 128, 264, 2, True, "f16", 0, 600, 64, True),
    (1024, 8, 64, 1000, 8, False, "bf16", 1, 300, 64, True), (4096, 32, 128, 512, 8, False, "bf16", 0, 300, 64, True),
    (4360, 34, 128, 360, 34, False, "bf16", 0, 550, 64, True), (256, 4, 64, 17920, 4, False, "f16", 1, 20, 64, False),
    (4360, 4, 64, 17920, 2, False, "bf16", 0, 300, 64, True), (2560, 4, 64, 17920, 4, False, "f16", 1, 20, 64, True),
    (4360, 34, 128, 17920, 2, False, "f16", 0, 300, 64, True), (1024, 43, 128, 264, 43, False, "bf16", 0, 40, 128, True),
    (4096, 32, 128, 512, 8, True, "bf16", 0, 300, 128, True), (4360, 40, 128, 17920, 2, False, "bf16", 1, 300, 128, True),
    (4096, 32, 128, 512, 32, False, "f16", 0, 550, 512, True)])
def test_one_row_alone_and_beside_another_request(hidden, heads, head_dim, ffn, kv, norm, dtype, act_mode, P, max_rows, own):
    shape = gi.ModelShape("row", 1 if ffn > 10000 else 2, hidden, heads, head_dim, ffn, 512, dtype=dtype, n_kv_heads=kv, qk_norm=norm)
    tm = torch_model(shape, seed=4, gain_jitter=0.1)
    gm = GooseModel(dataclasses.replace(ModelDesc.from_shape(shape), act_mode=act_mode), 64, 768, lambda l: tm["layers"][l], tm["embed"],
                    tm["lm_head"], tm["final_norm"], max_rows=max_rows)
    reqs = _requests(gm, shape, [1, 5], [P, 33], [P + 8, max(P, 33) + 8])
    alone = _alone(gm, reqs)
    _batched(gm, reqs)
    for q, a in zip(reqs, alone):
        assert torch.equal(q["argmax"], a["argmax"]) and torch.equal(q["succ_ids"], a["ids"]) and torch.equal(q["succ_scores"], a["scores"])
        k_b, v_b = _rows(gm, q["kcache"], q["vcache"], 0, a["P"])
        k_a, v_a = _rows(gm, a["k"], a["v"], 0, a["P"])
        assert torch.equal(k_b, k_a) and torch.equal(v_b, v_a)
    # the row was verified by its own kernels: the only norm left a launch is the one behind the down projection
    gm.ctx.goose_profile_enable(True)
    _alone(gm, reqs[:1])
    assert gm.ctx.goose_profile_read()["rmsnorm_residual"][1] == (shape.n_layers if own else 2 * shape.n_layers + 1)
    gm.ctx.close()


@pytest.mark.parametrize("shape_name", ["small_bf16", "small_gqa_qknorm_f16"])
def test_one_row_against_the_oracle(shape_name):
    shape = gi.SHAPES[shape_name]
    tm = torch_model(shape, seed=7, gain_jitter=0.1)
    om = oracle_model(shape, tm)
    gm = gpu_model(shape, tm, max_B=64, cap=768)
    root = int(_gpu_prefill(gm, gi.prefix_tokens(3, 530, shape.vocab), 64)["argmax"][-1].item())   # (three key splits)
    for _ in range(3):
        g, _, _ = _compare_step(shape, gm, om, device_cache_as_oracle(gm, gm.P), np.array([root], np.int32), gi.tree_single(), tol_for(shape))
        root = g["bonus"]
    gm.ctx.close()


def test_range_flag_of_one_row():
    from paper_2604_02047_amd.binding import GOOSE_FLAG_RANGE
    shape = dataclasses.replace(gi.SHAPES["tiny_bf16"], n_layers=1)
    tm = torch_model(shape, seed=13)
    w = tm["layers"][0]
    w["wo"][0] = 0                                      # component 0 of the row: nothing but what the embedding holds
    w["wg"][7, 0], w["wu"][7, 0] = 250.0, -250.0
    tm["embed"][5] = 0
    tm["embed"][5, 0] = 16.0                            # normalised about 16: gate 4000, up -4000
    tm["embed"][6, 0] = 0
    gm = gpu_model(shape, tm, max_B=32, cap=256)
    for token, flags in ((6, 0), (5, GOOSE_FLAG_RANGE)):
        gm.set_P(0)
        gm.verify_step_calls([token], [-1], None, commit=False)
        assert gm.ctx.goose_device_flags() == flags
    gm.ctx.close()
