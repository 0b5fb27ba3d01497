"""fp32 models: a step of five launches a layer.  The projections take in the norms, the rotation, SwiGLU and the residual adds, the
first launch of a step the mask and the embedding, the last one the walk and the commit."""
import numpy as np
import pytest
import torch

import goose_inputs as gi
from oracle import goose_oracle as orc
from util import gpu_model, oracle_model, torch_model
from test_gpu_parity import TOL, _compare_step

pytestmark = pytest.mark.gpu


def _cached(shape, P, seed):
    """A random prefix as the oracle holds it (fp32 values)."""
    rng = np.random.RandomState(seed)
    return [tuple(rng.randn(shape.n_heads, P, shape.head_dim).astype(np.float32).astype(np.float64) for _ in range(2))
            for _ in range(shape.n_layers)]


# inputs of 256 (one round of a wavefront) and around it, single and split over four wavefronts; heads shorter than the 64 columns of a
# round of the attention, longer, and of the largest size; trees at the edges of groups of eight rows and of mask words; lengths around
# the 64 keys of a round; the last two keep more scores in LDS than a launch has by default
@pytest.mark.parametrize("hidden,heads,head_dim,ffn,vocab,B,P", [
    (256, 4, 64, 688, 1024, 8, 64), (256, 1, 8, 256, 64, 1, 1), (260, 2, 72, 260, 1000, 65, 61), (1024, 2, 128, 257, 511, 128, 0),
    (64, 3, 256, 64, 33, 9, 130), (36, 2, 136, 1030, 77, 17, 63), (8, 1, 8, 12, 40, 64, 16300), (16, 2, 16, 20, 40, 3, 16360)])
def test_steps_of_odd_sizes(hidden, heads, head_dim, ffn, vocab, B, P):
    """Against the oracle through the separate entry points; then the whole step, which must give the same bits."""
    shape = gi.ModelShape("f32", 2, hidden, heads, head_dim, ffn, vocab, dtype="f32")
    tm = torch_model(shape, seed=5, gain_jitter=0.1)
    cap = (P + B + 127) // 64 * 64
    gm = gpu_model(shape, tm, max_B=B, cap=min(cap, 16384))
    cache = _cached(shape, P, 8)
    for l, (k, v) in enumerate(cache):
        if P:
            gm.write_rows(l, torch.from_numpy(k), torch.from_numpy(v))
    gm.set_P(P)
    tree = gi.tree_random(B, seed=3, spine_len=max(1, B // 3)) if B > 1 else gi.tree_single()
    tokens = np.random.RandomState(1).randint(0, vocab, B).astype(np.int32)
    before = gm.kcache.clone(), gm.vcache.clone()
    g, _, _ = _compare_step(shape, gm, oracle_model(shape, tm), cache, tokens, tree, TOL["f32"])
    want = gm.kcache.clone(), gm.vcache.clone(), gm.P
    gm.kcache.copy_(before[0])
    gm.vcache.copy_(before[1])
    gm.set_P(P)
    logits, margin = torch.zeros(B, vocab, device=gm.device), torch.zeros(B, device=gm.device)
    nxt = torch.zeros(1, dtype=torch.int32, device=gm.device)
    t, p, s = gm.stage_tree(tokens, tree.parent, tree.is_spine)
    gm.verify_step_fused(t, p, s, B, min(cap, 16384) - B if P < 16000 else P, next_root=nxt, logits=logits, margin=margin)
    torch.cuda.synchronize()
    assert gm.ctx.goose_device_flags() == 0
    assert torch.equal(logits, g["logits"]) and torch.equal(margin, g["margin"])
    assert torch.equal(gm.argmax[:B], g["argmax"]) and gm.path[:B].tolist() == g["path"].tolist()
    assert int(gm.accept_len.item()) == g["accept_len"] and int(gm.bonus.item()) == g["bonus"] == int(nxt.item())
    assert int(gm.d_P.item()) == want[2]
    assert torch.equal(gm.kcache, want[0]) and torch.equal(gm.vcache, want[1])
    gm.ctx.close()


def test_a_node_without_finite_values_stays_alone():
    """The embedding of one node is infinite: nodes that do not descend from it get the same bits as beside a finite one."""
    shape = gi.SHAPES["tiny"]
    tm = torch_model(shape, seed=2)
    gm = gpu_model(shape, tm, max_B=16, cap=256)
    tree = gi.tree_star(9)
    out = []
    for value in (1.0, float("inf")):
        gm.embed[5] = value
        gm.set_P(0)
        gm.kcache.zero_()
        gm.vcache.zero_()
        out.append(gm.verify_step_calls(np.array([1, 2, 3, 5, 6, 7, 8, 9, 10], np.int32), tree.parent, tree.is_spine, want_logits=True,
                                        commit=False)["logits"])
    rest = [i for i in range(9) if i != 3]
    assert torch.equal(out[0][rest], out[1][rest]) and torch.isfinite(out[1][rest]).all()
    gm.ctx.close()


@pytest.mark.parametrize("hidden", [256, 260])
def test_rows_beyond_the_range_of_a_sum(hidden):
    """Squares of a finite row that overflow scale it to zeros; sums that would overflow before they are scaled do not; an infinity gives NaN."""
    shape = gi.ModelShape("f32", 2, hidden, 4, 64, 516, 300, dtype="f32")
    tm = torch_model(shape, seed=4, gain_jitter=0.1)
    tm["lm_head"][7] *= 1e25
    tm["embed"][5] = tm["embed"][50] * 1e22     # (embedding values are about 0.02)
    tm["embed"][6] = tm["embed"][50] * 1e18
    tm["embed"][8, 3] = float("inf")
    gm = gpu_model(shape, tm, max_B=16, cap=256)
    om = oracle_model(shape, tm)
    for at in (1, 9):                           # in both groups of eight rows
        tokens = np.arange(20, 31, dtype=np.int32)
        tokens[at] = 5
        tokens[at - 1] = 6
        gm.set_P(0)
        gm.kcache.fill_(float("nan"))
        gm.vcache.fill_(float("nan"))
        tree = gi.tree_star(11)
        logits = gm.verify_step_calls(tokens, tree.parent, tree.is_spine, want_logits=True, commit=False)["logits"]
        k, v = gm.k_rows(0, 11), gm.v_rows(0, 11)
        zero = [at]
        rest = [i for i in range(11) if i != at]
        assert not logits[zero].any() and not k[:, :, zero].any() and not v[:, :, zero].any()
        assert torch.isfinite(logits).all() and torch.isfinite(k).all() and torch.isfinite(v).all()
        ref = orc.tree_logits(om, orc.empty_cache(om), tokens[rest], gi.tree_star(10).parent)[0]
        assert np.abs(logits[rest].cpu().numpy() - ref).max(0)[7] <= TOL["f32"] * np.abs(ref[:, 7]).max()
        small = [c for c in range(300) if c != 7]
        assert np.abs(logits[rest].cpu().numpy() - ref)[:, small].max() <= TOL["f32"] * np.abs(ref[:, small]).max()
    tokens[9] = 8
    assert torch.isnan(gm.verify_step_calls(tokens, tree.parent, tree.is_spine, want_logits=True, commit=False)["logits"][9]).all()
    gm.ctx.close()


def test_workspace_of_an_fp32_context():
    """No partial sums, operand rows or attention splits: those are of 16-bit models (250 MB at this size)."""
    from paper_2604_02047_amd import ModelDesc
    from paper_2604_02047_amd.binding import GooseContext
    torch.zeros(1, device="cuda:0")
    before = torch.cuda.mem_get_info()[0]
    ctx = GooseContext(ModelDesc(1, 4096, 32, 128, 11008, 32000, 10000.0, 1e-5, "f32"), 128, 256)
    assert before - torch.cuda.mem_get_info()[0] < 64 << 20
    ctx.close()
