"""The norms of 16-bit models round in one fixed order: every result equals, bit for bit, the same steps in NumPy's float32."""
import dataclasses

import numpy as np
import pytest
import torch

import goose_inputs as gi
from paper_2604_02047_amd import ModelDesc
from paper_2604_02047_amd.runner import GooseModel
from util import torch_model

pytestmark = pytest.mark.gpu

f32 = np.float32


def _fma(a, b, c):
    """float32 fma (the product is exact in 64 bits, the sum nearly always in the 80-bit type)."""
    return (a.astype(np.longdouble) * b.astype(np.longdouble) + c.astype(np.longdouble)).astype(f32)


def _bf16(a):
    return torch.from_numpy(a).to(torch.bfloat16).float().numpy()


def _norm(x, g, eps):
    """RMSNorm(x) * g in two terms: four neighbouring columns y, x, z, w a step, steps of a thread in order, lanes in halves, wavefronts in order."""
    rows, H = x.shape
    threads = 256 if H <= 1024 else 1024
    q = np.zeros((rows, -(-H // (4 * threads)), threads, 4), f32)
    q.reshape(rows, -1)[:, :H] = x
    ss = np.zeros((rows, threads), f32)
    for i in range(q.shape[1]):
        a = q[:, i]
        sq = a[..., 1] * a[..., 1]
        for e in (0, 2, 3):
            sq = _fma(a[..., e], a[..., e], sq)
        ss = ss + sq
    ss = ss.reshape(rows, threads // 64, 64)
    for off in (32, 16, 8, 4, 2, 1):
        ss = ss + ss[..., np.arange(64) ^ off]
    tot = np.zeros(rows, f32)
    for w in range(threads // 64):
        tot = tot + ss[:, w, 0]
    t = x * (f32(1) / np.sqrt(tot / f32(H) + f32(eps)))[:, None]
    hi = _bf16(t * g)
    return hi + _bf16(_fma(t, np.broadcast_to(g, t.shape), -hi))


@pytest.mark.parametrize("hidden", [256, 1024, 1032, 4104])
def test_every_bit_of_a_norm(hidden):
    """The output head is the identity and the operands are two bf16 terms, so the logits are the normalised rows to 16 bits."""
    shape = gi.ModelShape("norm", 1, hidden, 1, 64, 64, hidden, dtype="bf16")
    tm = torch_model(shape, seed=3, gain_jitter=0.1)
    gm = GooseModel(dataclasses.replace(ModelDesc.from_shape(shape), act_mode=1), 64, 128, lambda l: tm["layers"][l], tm["embed"],
                    torch.eye(hidden, dtype=torch.bfloat16), tm["final_norm"])
    x = gi.gen_normal(11, 11, (64, hidden), 1.0, torch.float32, "cpu")
    logits = torch.zeros((64, hidden), dtype=torch.float32, device=gm.device)
    argmax = torch.zeros(64, dtype=torch.int32, device=gm.device)
    gm.ctx.goose_lm_head_argmax(gm.packed_head, x.to(gm.device), 64, argmax, logits)
    torch.cuda.synchronize()
    assert np.array_equal(logits.cpu().numpy(), _norm(x.numpy(), tm["final_norm"].float().numpy(), shape.rms_eps))
    gm.ctx.close()
