"""Logit harvest into the unigram successor tables (Sec. 4 stage 2; App. C "adjacency table" tier 1,
"logit harvesting"): the HIP kernel against the oracle on the same logits -- ids bit-exact (also
under ties and repeated tokens), scores to fp32 round-off -- alone and inside the fused step."""
import ctypes

import numpy as np
import pytest
import torch

import goose_inputs as gi
from oracle import goose_oracle as orc
from paper_2604_02047_amd.binding import load_library
from util import gpu_model, torch_model

pytestmark = pytest.mark.gpu


def _ctx(vocab):
    from paper_2604_02047_amd import GooseContext, ModelDesc
    shape = gi.ModelShape("h", 1, 256, 4, 64, 688, vocab, dtype="bf16")
    return GooseContext(ModelDesc.from_shape(shape), 128, 128)


@pytest.mark.parametrize("V,B,K,quant", [(1000, 1, 10, 0), (1000, 37, 10, 0.25), (32000, 64, 10, 0),
                                         (32000, 128, 16, 0.5), (4093, 128, 1, 0), (50, 9, 10, 1.0)])
def test_harvest_kernel_matches_the_oracle(V, B, K, quant):
    dev = "cuda:0"
    c = _ctx(V)
    rng = np.random.default_rng(V + B)
    logits = rng.normal(size=(B, V)).astype(np.float32) * 4
    if quant:
        logits = (np.round(logits / quant) * quant).astype(np.float32)      # many exact ties
    tokens = rng.integers(0, V, size=B).astype(np.int32)
    if B > 4:
        tokens[B // 2] = tokens[1]                                          # repeated tokens: the later node wins
        tokens[B - 1] = tokens[0]
    ld = V + 24                                                             # a padded row length
    d_logits = torch.full((B, ld), float("nan"), dtype=torch.float32, device=dev)
    d_logits[:, :V] = torch.from_numpy(logits)
    ids0 = rng.integers(0, V, size=(V, K)).astype(np.int32)
    sc0 = rng.random(size=(V, K)).astype(np.float32)
    d_ids, d_sc = torch.from_numpy(ids0).to(dev), torch.from_numpy(sc0).to(dev)
    c.goose_harvest_topk(d_logits, ld, torch.from_numpy(tokens).to(dev), B, K, d_ids, d_sc)
    torch.cuda.synchronize()
    ref_ids, ref_sc = orc.harvest_topk(logits.astype(np.float64), tokens, K, table_ids=ids0, table_scores=sc0)
    assert np.array_equal(d_ids.cpu().numpy(), ref_ids)
    np.testing.assert_allclose(d_sc.cpu().numpy(), ref_sc, rtol=2e-5, atol=1e-9)
    c.close()


def test_harvest_row_that_defeats_the_prefilter():
    """More than a thousand large logits sitting in nine residue classes of the column index: the
    kernel's short candidate list overflows and it must take its plain route; results unchanged."""
    dev = "cuda:0"
    V, B, K = 32000, 3, 10
    c = _ctx(V)
    rng = np.random.default_rng(9)
    logits = rng.normal(size=(B, V)).astype(np.float32)
    cols = np.arange(V)
    logits[1, cols % 256 < 9] += 50.0
    logits[2, :] = 1.5                                            # all equal: ids 0..K-1 in order
    tokens = np.array([5, 6, 7], np.int32)
    d_ids = torch.full((V, K), -1, dtype=torch.int32, device=dev)
    d_sc = torch.zeros((V, K), dtype=torch.float32, device=dev)
    c.goose_harvest_topk(torch.from_numpy(logits).to(dev), V, torch.from_numpy(tokens).to(dev), B, K, d_ids, d_sc)
    torch.cuda.synchronize()
    ref_ids, ref_sc = orc.harvest_topk(logits.astype(np.float64), tokens, K)
    assert np.array_equal(d_ids.cpu().numpy(), ref_ids)
    np.testing.assert_allclose(d_sc.cpu().numpy(), ref_sc, rtol=2e-5, atol=1e-12)
    assert ref_ids[7].tolist() == list(range(K))
    c.close()


@pytest.mark.parametrize("V,K", [(16, 16), (8191, 10), (8192, 16), (8193, 16), (24577, 3), (600000, 16)])
def test_harvest_chunk_edges(V, K):
    """A row is cut into chunks of 8192 columns: vocabularies around the cut (the last chunk may hold one column), and one whose
    chunks give more pairs than one merge round ranks.  Rows: ordinary; every large logit in the share of four neighbouring
    threads; all -inf but a few; the winners spread over the chunk borders; equal everywhere."""
    dev = "cuda:0"
    c = _ctx(V)
    rng = np.random.default_rng(V)
    logits = (rng.normal(size=(5, V)) * 3).astype(np.float32)
    cols = np.arange(V)
    logits[1, (cols % 256) < 4] += 40.0
    logits[2] = -np.inf
    logits[2, rng.permutation(V)[:5]] = [1.0, 2.0, 2.0, -3.0, 0.5]
    logits[3, np.unique(np.clip([0, 8190, 8191, 8192, 8193, 16383, 16384, V - 2, V - 1], 0, V - 1))] = 30.0
    logits[4] = -0.25
    tokens = rng.permutation(V)[:5].astype(np.int32)
    d_ids = torch.full((V, K), -1, dtype=torch.int32, device=dev)
    d_sc = torch.zeros((V, K), dtype=torch.float32, device=dev)
    c.goose_harvest_topk(torch.from_numpy(logits).to(dev), V, torch.from_numpy(tokens).to(dev), 5, K, d_ids, d_sc)
    torch.cuda.synchronize()
    ref_ids, ref_sc = orc.harvest_topk(logits.astype(np.float64), tokens, K)
    assert np.array_equal(d_ids.cpu().numpy(), ref_ids)
    np.testing.assert_allclose(d_sc.cpu().numpy(), ref_sc, rtol=2e-5, atol=1e-12)
    c.close()


@pytest.mark.parametrize("V", [7, 1023, 1024, 1025, 4096, 4097, 8192])
def test_harvest_of_one_chunk(V):
    """Vocabularies of one chunk: 4, 16 or 32 logits a thread, on both sides of each; the smallest and the largest K."""
    for K in (1, min(V, 16)):
        test_harvest_chunk_edges(V, K)


@pytest.mark.parametrize("V,launches", [(1000, 1), (8192, 1), (8193, 2)])
def test_harvest_launches(V, launches):
    """A row of one chunk has nothing to merge: a second launch would double the time of a small vocabulary."""
    dev = "cuda:0"
    c = _ctx(V)
    logits, tokens = torch.zeros((4, V), device=dev), torch.zeros(4, dtype=torch.int32, device=dev)
    ids, sc = torch.zeros((V, 1), dtype=torch.int32, device=dev), torch.zeros((V, 1), device=dev)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        c.goose_harvest_topk(logits, V, tokens, 4, 1, ids, sc)
    n = ctypes.c_size_t(0)
    assert load_library().hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    assert n.value == launches
    c.close()


@pytest.mark.parametrize("V", [100, 8192, 20000])
def test_harvest_of_infinite_logits(V):
    """Softmax is undefined where a row's largest logit is infinite: its scores are NaN, as in the oracle, and its ids still
    ordered.  Logits of -inf under a finite largest one have probability 0, also where they fill a whole chunk of the row."""
    dev, K = "cuda:0", 10
    c = _ctx(V)
    logits = np.random.default_rng(V).normal(size=(5, V)).astype(np.float32)
    logits[0, V - 3] = np.inf
    logits[1, [2, V // 2, V - 1]] = np.inf
    logits[2] = -np.inf
    logits[3, :V // 2] = -np.inf
    logits[4] = -np.inf
    logits[4, [5, V - 2]] = [0.5, 1.5]
    tokens = np.arange(5, dtype=np.int32)
    d_ids = torch.full((V, K), -1, dtype=torch.int32, device=dev)
    d_sc = torch.zeros((V, K), dtype=torch.float32, device=dev)
    c.goose_harvest_topk(torch.from_numpy(logits).to(dev), V, torch.from_numpy(tokens).to(dev), 5, K, d_ids, d_sc)
    torch.cuda.synchronize()
    with np.errstate(invalid="ignore"):
        ref_ids, ref_sc = orc.harvest_topk(logits.astype(np.float64), tokens, K)
    assert np.isnan(ref_sc[:3]).all() and np.isfinite(ref_sc[3:]).all()
    assert np.array_equal(d_ids.cpu().numpy(), ref_ids)
    np.testing.assert_allclose(d_sc.cpu().numpy(), ref_sc, rtol=2e-5, atol=1e-12)
    c.close()


def test_harvest_inside_the_fused_step():
    shape = gi.SHAPES["small_bf16"]
    tm = torch_model(shape, seed=2, gain_jitter=0.1)
    gm = gpu_model(shape, tm, max_B=128, cap=256)
    dev = gm.device
    tree = gi.tree_spine_7b(3)
    B, K = tree.B, 10
    tokens = gi.draft_tokens_uniform(5, tree.parent, shape.vocab, 11)
    tokens[40] = tokens[3]                                                  # a repeated token
    t, p, s = gm.stage_tree(tokens, tree.parent, tree.is_spine)
    results = []
    for want_logits in (True, False):
        gm.set_P(0)
        ids = torch.full((shape.vocab, K), -1, dtype=torch.int32, device=dev)
        sc = torch.zeros((shape.vocab, K), dtype=torch.float32, device=dev)
        logits = torch.empty((B, shape.vocab), dtype=torch.float32, device=dev) if want_logits else None
        gm.verify_step_fused(t, p, s, B, 128, logits=logits, succ_ids=ids, succ_scores=sc)
        torch.cuda.synchronize()
        results.append((ids.cpu().numpy(), sc.cpu().numpy(), None if logits is None else logits.cpu().numpy()))
    ids_a, sc_a, gl = results[0]
    ref_ids, ref_sc = orc.harvest_topk(gl.astype(np.float64), tokens, K)
    assert np.array_equal(ids_a, ref_ids)
    np.testing.assert_allclose(sc_a, ref_sc, rtol=2e-5, atol=1e-9)
    # the tables do not depend on whether the caller also asked for the logits
    assert np.array_equal(results[1][0], ids_a) and np.array_equal(results[1][1], sc_a)
    # every node's first successor is its greedy prediction
    am = gm.argmax[:B].cpu().numpy()
    last = {int(tok): i for i, tok in enumerate(tokens)}
    for tok, i in last.items():
        assert ids_a[tok, 0] == am[i]
    gm.ctx.close()
