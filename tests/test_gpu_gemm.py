"""The skinny-M projection kernel alone against an fp64 product of the same bf16 inputs."""
import numpy as np
import pytest
import torch

import paper_2604_02047_amd as g

pytestmark = pytest.mark.gpu


def _a_rows(B):
    """Rows of the operand buffer: the whole 32-row tiles that the product must be able to read, and more beyond 128 rows."""
    return (B + 31) // 32 * 32 if B <= 128 else (B + 127) // 128 * 128


def _operand(a32, rows, Kp, dt, terms, dev):
    """fp32 rows [B][K] -> (device operand in `terms` terms with `rows` rows, the exact values it carries as fp64)."""
    B, K = a32.shape
    if terms == 1:
        a = torch.zeros((rows, Kp), dtype=dt)
        a[:B, :K] = a32.to(dt)
        return a.to(dev), a[:B, :K].double().numpy()
    src = torch.zeros((rows, Kp), dtype=torch.float32, device=dev)
    src[:B, :K] = a32.to(dev)
    a2 = torch.full((rows, 2 * Kp), float("nan"), dtype=dt, device=dev)
    g.goose_split_operand(src, rows, Kp, Kp, a2, 2 * Kp)
    torch.cuda.synchronize()
    groups = a2.view(rows, Kp // 8, 2, 8).double().cpu()      # [row][group][hi|lo][8]
    carried = (groups[:, :, 0] + groups[:, :, 1]).reshape(rows, Kp)
    hi = groups[:, :, 0].reshape(rows, Kp)
    assert torch.equal(hi[:B, :K].to(dt), a32.to(dt))                       # hi is the plain rounding
    assert (carried[:B, :K] - a32.double()).abs().max() <= 2.0 ** -15 * a32.abs().max()   # hi + lo: 16 more bits
    return a2, carried[:B, :K].numpy()


def _run(B, N, K, nw, ks, seed=0, dt=torch.bfloat16, terms=1, guard=0):
    """guard > 0: that many rows behind the last slab, which must stay as they were, like the rows B.. of every slab."""
    dev = "cuda:0"
    gen = torch.Generator(device="cpu").manual_seed(seed)
    Kp, Np, rows = (K + 127) // 128 * 128, (N + 31) // 32 * 32, (B + 31) // 32 * 32
    a, a_exact = _operand(torch.randn((B, K), generator=gen), _a_rows(B), Kp, dt, terms, dev)
    w = (torch.randn((N, K), generator=gen) * 0.05).to(dt)
    ref = a_exact @ w.double().numpy().T
    packed = torch.zeros(g.goose_packed_matrix_bytes(N, K), dtype=torch.uint8, device=dev)
    g.goose_pack_matrix(w.to(dev), N, K, packed)
    whole = torch.full((ks * rows + guard, Np), float("nan"), dtype=torch.float32, device=dev)
    part = whole[:ks * rows].view(ks, rows, Np)
    if terms == 1:
        g.goose_gemm_packed(a, Kp, packed, N, K, B, nw, ks, part)
    else:
        g.goose_gemm_packed_ex(a, Kp * terms, terms, packed, N, K, B, nw, ks, part)
    torch.cuda.synchronize()
    out = part[:, :B, :N].double().sum(0).cpu().numpy()
    scale = np.abs(ref).max()
    err = np.abs(out - ref).max()
    # fp32 accumulation of exact bf16 products: only summation-order rounding remains
    assert err <= 2e-5 * scale * max(1.0, np.sqrt(K) / 16), (B, N, K, nw, ks, err, scale)
    if guard:
        assert torch.isnan(part[:, B:]).all() and torch.isnan(whole[ks * rows:]).all(), (B, N, K, nw, ks)


@pytest.mark.parametrize("B", [1, 16, 33, 64, 80, 128])
def test_gemm_row_tiles(B):
    _run(B, 256, 512, 2, 1)
    _run(B, 288, 1024, 4, 2)


@pytest.mark.parametrize("B", [129, 200, 256, 300, 512])
def test_gemm_row_chunks(B):
    """More than 128 rows: chunks of a workgroup's rows (128 in these grids), dealt so that the chunks of a
    column group share an XCD; grids that are no multiple of 8 workgroups, ragged last chunk."""
    _run(B, 256, 512, 2, 1)
    _run(B, 288, 1024, 4, 2)
    _run(B, 1000, 1000, 4, 3)
    _run(B, 4096, 2048, 4, 4)


@pytest.mark.parametrize("B", [129, 191, 193, 256, 257, 384, 385, 449])
def test_gemm_many_rows_edges(B):
    """The many-row kernel with fewer columns than one workgroup, a ragged last one, and ranges of 2 to 6 stages.  Grids as small
    as these always take workgroups of 128 rows x 256 columns; test_gemm_tall_workgroups has the others."""
    for K in (128, 256, 384):
        _run(B, 40, K, 4, 1, dt=torch.float16)
        _run(B, 288, K, 4, 1, terms=2)
    _run(B, 2080, 640, 4, 5)
    _run(B, 2080, 896, 2, 3, dt=torch.float16)


# The rows of a workgroup (128, 192 or 256) follow from the grid: the least rounds of 256 workgroups x (height / 64 + 1).  With
# 86 .. 128 (groups of 256 columns) x (K ranges), as here, 257 .. 384 rows take 192 and 385 .. 512 rows take 256.
@pytest.mark.parametrize("B", [257, 288, 320, 383, 384, 385, 448, 449, 512])
@pytest.mark.parametrize("terms", [1, 2])
def test_gemm_tall_workgroups(B, terms):
    """Workgroups of 192 and 256 rows: row counts on both sides of a workgroup's end and of the rows that one of its wavefronts
    copies, ranges of two to four stages of 64 inputs (four to eight of 32 in two terms), K ranges, a ragged last column group.
    Nothing is written outside rows < B."""
    dt = torch.bfloat16 if B & 1 else torch.float16
    _run(B, 22016, 256, 4, 1, dt=dt, terms=terms, guard=512)
    _run(B, 22100, 128, 4, 1, terms=terms, guard=512)
    _run(B, 5504, 512, 4, 4, terms=terms, guard=512)


@pytest.mark.parametrize("B", [1, 33, 63, 100, 127, 129, 161, 191, 255])
def test_gemm_writes_only_its_rows(B):
    """Row tiles that end inside a tile or lie wholly beyond B, column tiles beyond the last: every other row keeps its contents."""
    _run(B, 288, 512, 4, 2, guard=512)
    _run(B, 1000, 384, 2, 3, guard=512, terms=2)


@pytest.mark.parametrize("stages,ks", [(1, 1), (2, 1), (2, 2), (3, 1), (3, 3), (4, 2), (5, 1), (5, 2), (6, 3),
                                       (8, 2), (9, 2), (22, 5), (32, 1), (32, 4), (86, 8)])
def test_gemm_stage_counts_and_splits(stages, ks):
    for nw in (2, 4):
        for B in (64, 16, 96):
            _run(B, 160, stages * 128, nw, ks, seed=stages)


@pytest.mark.parametrize("B", [16, 80, 128, 300])
def test_gemm_fp16_operands(B):
    """The same kernels on fp16 operands (exact products, fp32 accumulation: the same bound)."""
    _run(B, 288, 1024, 4, 2, dt=torch.float16)
    _run(B, 1000, 1000, 2, 1, dt=torch.float16)


@pytest.mark.parametrize("B", [1, 16, 33, 64, 80, 128, 200, 512])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
def test_gemm_two_term_operand(B, dt):
    """The activation operand as hi + lo (the layout the decoder layers use): the product must be that of
    the sum of both terms, i.e. of the fp32 activations to 2^-17."""
    _run(B, 288, 1024, 4, 2, dt=dt, terms=2)
    _run(B, 256, 512, 2, 1, dt=dt, terms=2)
    _run(B, 1000, 1000, 4, 3, dt=dt, terms=2)


def test_gemm_ragged_shapes():
    _run(50, 1000, 1000, 4, 2)   # N not a multiple of the 4-tile group, K padded to 1024
    _run(7, 40, 200, 2, 1)
    _run(64, 4096, 4096, 4, 8)


@pytest.mark.parametrize("B,F,K,nw", [(16, 96, 256, 2), (16, 2752, 1024, 2), (64, 2752, 1024, 4), (80, 352, 640, 2),
                                       (80, 17920, 256, 4),
                                       (128, 704, 256, 4), (33, 64, 4096, 2), (300, 704, 256, 4), (512, 352, 640, 2),
                                       (160, 2752, 1024, 4)])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float16])
@pytest.mark.parametrize("terms", [1, 2])
def test_gemm_swiglu_epilogue(B, F, K, nw, dt, terms):
    _run_swiglu(B, F, K, nw, dt, terms)


@pytest.mark.parametrize("B", [257, 320, 384, 385, 449, 512])
@pytest.mark.parametrize("terms", [1, 2])
def test_gemm_swiglu_tall_workgroups(B, terms):
    """The same epilogue in workgroups of 192 and 256 rows (see test_gemm_tall_workgroups), the last column group ragged."""
    _run_swiglu(B, 11008, 256, 4, torch.float16 if B & 1 else torch.bfloat16, terms, guard=512)
    _run_swiglu(B, 11104, 128, 4, torch.bfloat16, terms, guard=512)


@pytest.mark.parametrize("B", [1, 50, 127, 129, 200])
def test_gemm_swiglu_writes_only_its_rows(B):
    _run_swiglu(B, 352, 640, 4, torch.bfloat16, 1, guard=512)
    _run_swiglu(B, 352, 640, 2, torch.float16, 2, guard=512)


def _run_swiglu(B, F, K, nw, dt, terms, guard=0, pad=0):
    """guard > 0: that many rows behind the result, pad > 0: that many elements behind each row, which must stay as they were."""
    dev = "cuda:0"
    gen = torch.Generator(device="cpu").manual_seed(F)
    Kp, rows = (K + 127) // 128 * 128, (B + 31) // 32 * 32
    a, a_exact = _operand(torch.randn((B, K), generator=gen), _a_rows(B), Kp, dt, terms, dev)
    wg = (torch.randn((F, K), generator=gen) * 0.05).to(dt)
    wu = (torch.randn((F, K), generator=gen) * 0.05).to(dt)
    assert F % 16 == 0
    inter = torch.stack([wg.view(F // 16, 16, K), wu.view(F // 16, 16, K)], dim=1).reshape(2 * F, K).contiguous()
    gd, ud = torch.from_numpy(a_exact) @ wg.double().T, torch.from_numpy(a_exact) @ wu.double().T
    ref = (gd / (1 + torch.exp(-gd)) * ud).numpy()
    packed = torch.zeros(g.goose_packed_matrix_bytes(2 * F, K), dtype=torch.uint8, device=dev)
    g.goose_pack_matrix(inter.to(dev), 2 * F, K, packed)
    whole = torch.full((rows + guard, F * terms + pad), float("nan"), dtype=dt, device=dev)
    if terms == 1:
        g.goose_gemm_swiglu_packed(a, Kp, packed, 2 * F, K, B, nw, whole, F + pad)
    else:
        g.goose_gemm_swiglu_packed_ex(a, Kp * terms, terms, packed, 2 * F, K, B, nw, whole, F * terms + pad)
    torch.cuda.synchronize()
    h = whole[:, :F * terms]
    if terms == 1:
        out = h[:B].double().cpu().numpy()
        # one rounding of the result to the storage type (relative to the element, hence to the largest)
        tol = 6e-3 if dt == torch.bfloat16 else 8e-4
    else:   # the result keeps two terms as well: hi + lo carries it to 2^-17 (the silu itself is fp32)
        pair = h[:B].reshape(B, F // 8, 2, 8).double().cpu()
        out = (pair[:, :, 0] + pair[:, :, 1]).reshape(B, F).numpy()
        tol = 2e-5
    assert np.abs(out - ref).max() <= tol * np.abs(ref).max()
    if guard or pad:
        assert torch.isnan(h[B:]).all() and torch.isnan(whole[:, F * terms:]).all()


@pytest.mark.parametrize("B,F,nw", [(1, 352, 2), (33, 352, 4), (128, 352, 2), (128, 704, 4), (80, 17920, 4), (150, 352, 4),
                                    (300, 11104, 4), (400, 11008, 4)])
@pytest.mark.parametrize("terms", [1, 2])
@pytest.mark.parametrize("pad", [2, 6])
def test_gemm_swiglu_pitch_against_the_reference(B, F, nw, terms, pad):
    """Both kernels, result rows that start at odd multiples of four bytes, against the fp64 product."""
    _run_swiglu(B, F, 256, nw, torch.float16 if B & 1 else torch.bfloat16, terms, guard=64, pad=pad)


@pytest.mark.parametrize("B,F,nw", [(1, 352, 2), (33, 352, 4), (64, 352, 2), (128, 704, 4), (80, 17920, 4), (150, 352, 4),
                                    (300, 11104, 4), (400, 11008, 4)])
@pytest.mark.parametrize("terms", [1, 2])
def test_gemm_swiglu_beyond_fp16(B, F, nw, terms):
    """Results beyond fp16 become +-65504 exactly; the others of their columns stay what they are, and those of the other columns
    keep the bits that they have without any large ones beside them."""
    dev, K, dt = "cuda:0", 128, torch.float16
    gen = torch.Generator(device="cpu").manual_seed(B)
    a, exact = _operand(torch.randn((B, K), generator=gen), _a_rows(B), K, dt, terms, dev)
    wg, wu = ((torch.randn((F, K), generator=gen) * 0.05).to(dt) for _ in range(2))
    big = torch.zeros(F, dtype=torch.bool)
    big[[0, 7, 8, 15, 16, 85, F // 2 + 3, F - 17, F - 1]] = True           # first and last columns of groups of 8 and of tiles
    out = []
    for scale in (1.0, 2000.0):                                             # gate and up around 1100 in the large columns
        s = torch.where(big, scale, 1.0).view(F, 1)
        inter = torch.stack([(w.float() * s).to(dt).view(F // 16, 16, K) for w in (wg, wu)], dim=1).reshape(2 * F, K)
        packed = torch.zeros(g.goose_packed_matrix_bytes(2 * F, K), dtype=torch.uint8, device=dev)
        g.goose_pack_matrix(inter.contiguous().to(dev), 2 * F, K, packed)
        h = torch.full(((B + 31) // 32 * 32, F * terms), float("nan"), dtype=dt, device=dev)
        g.goose_gemm_swiglu_packed_ex(a, K * terms, terms, packed, 2 * F, K, B, nw, h, F * terms)
        torch.cuda.synchronize()
        assert torch.isnan(h[B:]).all()
        out.append(h[:B].view(B, F // 8, terms, 8).transpose(1, 2).reshape(B, terms, F).cpu())   # [row][hi|lo][column]
    assert torch.equal(out[0][:, :, ~big], out[1][:, :, ~big])
    gate, up = (torch.from_numpy(exact) @ (w[big].float() * 2000.0).to(dt).double().T for w in (wg, wu))
    ref = gate / (1 + torch.exp(-gate)) * up
    got = out[1][:, :, big].double().sum(1)
    over = ref.abs() > 65504 * 1.001
    assert over.any() and (~over).any() and (B == 1 or ((ref[over] > 0).any() and (ref[over] < 0).any()))
    assert torch.equal(got[over], ref[over].sign() * 65504)
    # fp32 sums of 128 exact products (2^-24 a step) in both factors, one rounding of the result to fp16
    err = (got - ref.clamp(-65504, 65504)).abs()
    assert (err <= 2.0 ** -10 * ref.abs() + 2.0 ** -16 * gate.abs().max() * up.abs().max()).all()


def test_gemm_more_tiles_than_one_round_of_four_tile_workgroups():
    """Beyond 1024 column tiles the launcher switches to five-wavefront workgroups (one round of 256)."""
    _run(80, 33024, 256, 4, 1)            # 1032 tiles
    _run(64, 20000, 512, 4, 2, seed=3)    # 625 tiles x 2 K ranges
    _run(33, 40960, 128, 4, 1, seed=4)    # 1280 tiles: the last five-wide grid that fits


def test_gemm_repeated_large_launches_are_stable():
    """The weight stream is hand scheduled (asynchronous loads awaited by count): hammer the
    big shapes of the 7B model, where memory latency is longest, and check every launch."""
    for rep in range(6):
        _run(64, 4096, 4096, 4, 8, seed=rep)
        _run(64, 4096, 11008, 4, 8, seed=rep)
        _run(64, 2048, 4096, 2, 1, seed=rep)
        _run(16, 4096, 4096, 2, 4, seed=rep)
        _run(128, 1024, 4096, 4, 2, seed=rep)


# Workgroups of 128, 192 and 256 rows over ranges of 6, 10 and 18 stages of 64 inputs: the unrolled loop of four stages once, twice
# and more often, each with two stages left over (12, 20 and 36 stages in two terms: none left).
@pytest.mark.parametrize("B,N", [(200, 2080), (320, 22016), (500, 22016)])
@pytest.mark.parametrize("K", [384, 640, 1152])
@pytest.mark.parametrize("terms", [1, 2])
def test_gemm_many_rows_stage_remainders(B, N, K, terms):
    _run(B, N, K, 4, 1, dt=torch.float16 if K == 640 else torch.bfloat16, terms=terms, guard=512)


@pytest.mark.parametrize("B,F", [(150, 352), (300, 11104), (400, 11008)])
@pytest.mark.parametrize("terms", [1, 2])
def test_gemm_swiglu_rows_at_any_even_pitch(B, F, terms):
    """Result rows that start at odd multiples of four bytes (16-byte stores of the many-row kernel); nothing between them is written."""
    dev, K, dt = "cuda:0", 256, torch.float16
    gen = torch.Generator(device="cpu").manual_seed(F)
    a, _ = _operand(torch.randn((B, K), generator=gen), _a_rows(B), K, dt, terms, dev)
    packed = torch.zeros(g.goose_packed_matrix_bytes(2 * F, K), dtype=torch.uint8, device=dev)
    g.goose_pack_matrix((torch.randn((2 * F, K), generator=gen) * 0.05).to(dt).to(dev), 2 * F, K, packed)
    out = []
    for ldh in (F * terms, F * terms + 2):
        h = torch.full((B, ldh), float("nan"), dtype=dt, device=dev)
        g.goose_gemm_swiglu_packed_ex(a, K * terms, terms, packed, 2 * F, K, B, 4, h, ldh)
        torch.cuda.synchronize()
        out.append(h[:, :F * terms].cpu())
        assert torch.isnan(h[:, F * terms:]).all()
    assert not torch.isnan(out[0]).any() and torch.equal(out[0], out[1])


@pytest.mark.parametrize("swiglu", [False, True])
@pytest.mark.parametrize("terms", [1, 2])
def test_gemm_many_rows_far_apart(swiglu, terms):
    """129 rows of 128 inputs, 168 MB from one to the next: 32-bit byte offsets reach the first 26 only."""
    dev, B, N, K, lda = "cuda:0", 129, 288 if not swiglu else 320, 128, 80 << 20
    gen = torch.Generator(device="cpu").manual_seed(terms)
    near, exact = _operand(torch.randn((B, K), generator=gen), B, K, torch.float16, terms, dev)
    a = torch.empty(B * lda, dtype=torch.float16, device=dev)
    a.view(B, lda)[:, :K * terms] = near
    w = (torch.randn((N, K), generator=gen) * 0.05).half()
    packed = torch.zeros(g.goose_packed_matrix_bytes(N, K), dtype=torch.uint8, device=dev)
    g.goose_pack_matrix(w.to(dev), N, K, packed)
    rows = 160
    if swiglu:
        out = torch.full((rows, N // 2 * terms), float("nan"), dtype=torch.float16, device=dev)
        g.goose_gemm_swiglu_packed_ex(a, lda, terms, packed, N, K, B, 4, out, N // 2 * terms)
        same = torch.empty_like(out)
        g.goose_gemm_swiglu_packed_ex(near, K * terms, terms, packed, N, K, B, 4, same, N // 2 * terms)
        torch.cuda.synchronize()
        assert torch.equal(out[:B], same[:B])
    else:
        out = torch.full((rows, N), float("nan"), dtype=torch.float32, device=dev)
        g.goose_gemm_packed_ex(a, lda, terms, packed, N, K, B, 4, 1, out)
        torch.cuda.synchronize()
        ref = exact @ w.double().numpy().T
        assert np.abs(out[:B].double().cpu().numpy() - ref).max() <= 2e-5 * np.abs(ref).max()
    assert torch.isnan(out[B:]).all()


def test_gemm_more_column_groups_than_a_grid_is_high():
    """65538 groups of two column tiles: the grid of a split product takes its groups in two layers."""
    dev, N, K = "cuda:0", 32 * (2 * 65535 + 5), 256
    gen = torch.Generator(device=dev).manual_seed(1)
    w = (torch.randn((N, K), generator=gen, device=dev) * 0.05).half()
    a = torch.zeros((32, K), dtype=torch.float16, device=dev)
    a[0] = torch.randn(K, generator=gen, device=dev).half()
    packed = torch.zeros(g.goose_packed_matrix_bytes(N, K), dtype=torch.uint8, device=dev)
    g.goose_pack_matrix(w, N, K, packed)
    part = torch.full((2, 32, N), float("nan"), dtype=torch.float32, device=dev)
    g.goose_gemm_packed(a, K, packed, N, K, 1, 2, 2, part)
    torch.cuda.synchronize()
    ref = torch.cat([c.double() @ a[0].double() for c in w.split(1 << 19)])
    assert (part[:, 0].double().sum(0) - ref).abs().max() <= 2e-5 * ref.abs().max()
    assert torch.isnan(part[:, 1:]).all()
