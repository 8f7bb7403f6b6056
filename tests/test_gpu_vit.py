"""GPU parity of the Vision Transformer path (include/cnnk_vit.h) against oracle/vit.py: every
operator on seeded tensors, whole tensors element by element, and the whole training step (every
activation, activation gradient, parameter gradient, updated parameter and momentum buffer)."""
import numpy as np
import pytest
import torch

import workloads as WL
from util import (JITTER_REL, JITTER_SEEDS, SCALE_TO_EXACT, SCALE_TO_MEMBER, dev, dev_f32, ensemble_bound, host,
                  max_rel_err, rep)

pytestmark = pytest.mark.gpu

from oracle import vit as V  # noqa: E402
from oracle.step import _q as oracle_quantiser  # noqa: E402


@pytest.fixture(scope="module")
def K():
    assert torch.cuda.is_available(), "the GPU tests need a GPU"
    from paper_2503_23186_amd import vit
    return vit


def dt_of(K, dtype):
    return K.BF16 if dtype == "bf16" else K.F32


def ws_for(nbytes):
    n = max(int(nbytes), 256)
    return torch.empty(n, dtype=torch.uint8, device="cuda:0"), n


# one unit in the last place of the largest element for bf16 outputs; fp32 sums of bf16-sized terms
OUT_TOL = {"f32": 2e-6, "bf16": 4e-3}
SUM_TOL = {"f32": 2e-5, "bf16": 2e-5}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,C,stride", [(37, 32, 0), (394, 768, 0), (101, 128, 0), (50, 1024, 0), (9, 4096, 0),
                                           (13, 768, 197 * 768), (1, 4, 0), (5, 260, 0)])
def test_layernorm(K, rows, C, stride, dtype):
    rng = np.random.default_rng(rows * 1000 + C)
    xs = stride or C
    xfull = rep(rng.standard_normal((rows, xs)) * 2.0 + 0.7, dtype)
    x = xfull[:, :C]
    g = rep(1.0 + 0.2 * rng.standard_normal(C), "f32")
    b = rep(0.3 * rng.standard_normal(C), "f32")
    dy = rep(rng.standard_normal((rows, C)), dtype)
    dresfull = rep(rng.standard_normal((rows, xs)), dtype)
    y, mean, rstd = V.layernorm_fwd(x, g, b)
    dx, dg, db = V.layernorm_bwd(dy, x, g, mean, rstd)
    d = K.ln_desc(rows, C, dt_of(K, dtype), 1e-6, stride)
    gx, gy = dev(xfull, dtype), dev(np.zeros((rows, C)), dtype)
    stats = torch.zeros((rows, 2), device="cuda:0")
    K.cnnk_layernorm_fwd(d, gx, dev_f32(g), dev_f32(b), gy, stats)
    torch.cuda.synchronize()
    assert max_rel_err(host(gy), y) <= OUT_TOL[dtype]
    assert max_rel_err(host(stats)[:, 0], mean) <= 1e-5 and max_rel_err(host(stats)[:, 1], rstd) <= 1e-5
    ws, nb = ws_for(K.cnnk_layernorm_workspace_bytes(d))
    for with_res in (False, True):
        gdx = dev(np.full((rows, xs), 7.0), dtype)
        gdg, gdb = torch.zeros(C, device="cuda:0"), torch.zeros(C, device="cuda:0")
        K.cnnk_layernorm_bwd(d, dev(dy, dtype), gx, dev_f32(g), stats, dev(dresfull, dtype) if with_res else None, gdx, gdg,
                             gdb, ws, nb)
        torch.cuda.synchronize()
        want = dx + (dresfull[:, :C] if with_res else 0.0)
        got = host(gdx)
        assert max_rel_err(got[:, :C], want) <= OUT_TOL[dtype] * (2 if with_res else 1)
        assert (got[:, C:] == 7.0).all()                     # nothing outside the rows' C elements is touched
        assert max_rel_err(host(gdg), dg) <= SUM_TOL[dtype] and max_rel_err(host(gdb), db) <= SUM_TOL[dtype]


# rows on either side of each change in the number of rows of a wavefront, with the widths on either side of each
# change of kernel and of resident workgroups
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,C", [(1600, 520), (1601, 768), (1602, 772), (4097, 64), (8193, 512), (3073, 1024), (6145, 776), (2049, 1032),
                                    (3, 640), (5, 516)])
def test_layernorm_row_splits(K, rows, C, dtype):
    test_layernorm(K, rows, C, 0, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,C", [(37, 32), (394, 3072), (100, 2304), (1000, 768), (3, 8), (129, 264)])
def test_bias_activation_residual(K, rows, C, dtype):
    rng = np.random.default_rng(rows + C)
    z = rep(rng.standard_normal((rows, C)) * 1.5, dtype)
    bias = rep(0.5 * rng.standard_normal(C), "f32")
    res = rep(rng.standard_normal((rows, C)), dtype)
    dy = rep(rng.standard_normal((rows, C)), dtype)
    dt = dt_of(K, dtype)
    ws, nb = ws_for(K.cnnk_bias_act_workspace_bytes(rows, C))
    # bias only, bias + residual
    for r in (None, res):
        gy = dev(np.zeros((rows, C)), dtype)
        K.cnnk_bias_act_fwd(rows, C, dt, K.ACT_NONE, dev(z, dtype), dev_f32(bias), None if r is None else dev(r, dtype), None, gy)
        torch.cuda.synchronize()
        assert max_rel_err(host(gy), z + bias + (0.0 if r is None else r)) <= OUT_TOL[dtype]
    gdb = torch.zeros(C, device="cuda:0")
    K.cnnk_bias_act_bwd(rows, C, dt, K.ACT_NONE, dev(dy, dtype), None, None, gdb, ws, nb)
    torch.cuda.synchronize()
    assert max_rel_err(host(gdb), dy.sum(0)) <= SUM_TOL[dtype]
    # bias + GELU: the stored pre-activation, the activation of the STORED value, and the gradient
    gu, gy = dev(np.zeros((rows, C)), dtype), dev(np.zeros((rows, C)), dtype)
    K.cnnk_bias_act_fwd(rows, C, dt, K.ACT_GELU, dev(z, dtype), dev_f32(bias), None, gu, gy)
    torch.cuda.synchronize()
    u = host(gu)
    assert max_rel_err(u, z + bias) <= OUT_TOL[dtype]
    assert max_rel_err(host(gy), V.gelu(u)) <= OUT_TOL[dtype]
    gdz = dev(np.zeros((rows, C)), dtype)
    K.cnnk_bias_act_bwd(rows, C, dt, K.ACT_GELU, dev(dy, dtype), gu, gdz, gdb, ws, nb)
    torch.cuda.synchronize()
    want = dy * V.gelu_grad(u)
    assert max_rel_err(host(gdz), want) <= OUT_TOL[dtype]
    assert max_rel_err(host(gdb), want.sum(0)) <= SUM_TOL[dtype]
    # in place: u over z
    gz = dev(z, dtype)
    K.cnnk_bias_act_fwd(rows, C, dt, K.ACT_GELU, gz, dev_f32(bias), None, gz, gy)
    torch.cuda.synchronize()
    assert (host(gz) == u).all()


# bf16 runs on the dense matrix-core kernels (256 x 128 tiles, 32 reduction elements per stage: ragged
# row and column tiles, ragged last stages, one to many stages, split and unsplit weight gradients);
# fp32 and "bf16-conv" on the 1 x 1 convolution kernels.  The last shapes are ViT-B/16's at batch 64.
LINEAR_SHAPES = [(64, 32, 32), (288, 64, 160), (1056, 768, 96), (68, 128, 256), (100, 40, 24), (512, 3072, 128),
                 (12608, 768, 2304), (12608, 3072, 768), (12544, 768, 768)]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "bf16-rows64", "bf16-rows128", "bf16-conv"])
@pytest.mark.parametrize("rows,Kd,N", LINEAR_SHAPES)
def test_linear_layers(K, rows, Kd, N, dtype):
    from paper_2503_23186_amd import cnnk
    if dtype == "f32" and rows > 2000:
        pytest.skip("the fp32 mode is a small-shape validation mode")
    if dtype == "bf16-conv":
        if rows > 2000:
            pytest.skip("covered by the convolution tests")
        cnnk.cnnk_tune(15, -1)
    if dtype in ("bf16-rows64", "bf16-rows128"):
        # the matrix-core kernels with 64-byte / 128-byte operand rows in LDS whatever the shape
        cnnk.cnnk_tune(15, 1 if dtype == "bf16-rows64" else 2)
    try:
        _linear_case(K, rows, Kd, N, "bf16" if dtype.startswith("bf16-") else dtype)
    finally:
        cnnk.cnnk_tune(15, 0)


# The tile shapes for small problems (64 x 64, 64 x 128 and 128 x 128 tiles, one or two groups of wavefronts
# that split the reduction), each forced: single ragged tiles, a reduction shorter than one stage, stage
# counts that the groups share unevenly (1, 3, 13 stages), and several tiles in both directions.
@pytest.mark.parametrize("shape", range(5))
@pytest.mark.parametrize("rows,Kd,N", [(1, 8, 8), (65, 72, 136), (130, 192, 64), (197, 776, 264), (788, 384, 1152)])
def test_linear_small_tiles(K, rows, Kd, N, shape):
    from paper_2503_23186_amd import cnnk
    cnnk.cnnk_tune(15, 16 + shape)
    try:
        _linear_case(K, rows, Kd, N, "bf16")
    finally:
        cnnk.cnnk_tune(15, 0)


# One workgroup on each of the eight XCDs (tuning key 18), so that each walks several tiles: reductions shorter than the
# pipeline (one stage), of its length and longer, ragged tiles in the middle and at the end of a walk, fewer tiles than
# XCDs.  Shapes: 16, 18 and 20 are the small ones with one group of wavefronts, 1 and 2 the large ones.
@pytest.mark.parametrize("shape", [16, 18, 20, 1, 2])
@pytest.mark.parametrize("rows,Kd,N", [(1600, 64, 264), (1090, 128, 200), (2500, 200, 136), (777, 392, 648), (300, 72, 136)])
def test_linear_workgroups_that_walk_several_tiles(K, rows, Kd, N, shape):
    from paper_2503_23186_amd import cnnk
    cnnk.cnnk_tune(15, shape)
    cnnk.cnnk_tune(18, 1)
    try:
        _linear_case(K, rows, Kd, N, "bf16")
    finally:
        cnnk.cnnk_tune(15, 0)
        cnnk.cnnk_tune(18, 0)


# The step's own products among them (GELU's derivative and column sums in the data gradient of the second linear layer, residuals,
# GELU) with one workgroup on each XCD: the bits of one tile to a workgroup.
@pytest.mark.parametrize("shape", [18, 20, 1, 2])
@pytest.mark.parametrize("batch,dim,mlp", [(9, 128, 512), (21, 192, 328)])
def test_steps_whose_workgroups_walk_several_tiles(K, shape, batch, dim, mlp):
    from paper_2503_23186_amd import cnnk
    net = WL.vit_mini(batch=batch, dtype="bf16", image=32, patch=4, dim=dim, heads=dim // 64, layers=2, mlp=mlp)
    inp = WL.make_vit_inputs(net, 6)
    runs = []
    for walk in (-1, 1):
        cnnk.cnnk_tune(15, shape)
        cnnk.cnnk_tune(18, walk)
        try:
            r = K.VitRunner(net)
            r.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
            r.step(0.1, 0.9, 0.0)
            torch.cuda.synchronize()
        finally:
            cnnk.cnnk_tune(15, 0)
            cnnk.cnnk_tune(18, 0)
        runs.append(r)
    a, b = runs
    assert torch.isfinite(a.loss).all() and torch.equal(a.loss, b.loss)
    for k, name in enumerate(a.names):
        assert torch.isfinite(a.grad[k]).all() and torch.equal(a.grad[k], b.grad[k]) and torch.equal(a.param[k], b.param[k]), name


def _linear_case(K, rows, Kd, N, dtype):
    rng = np.random.default_rng(rows + Kd + N)
    x = rep(rng.standard_normal((rows, Kd)), dtype)
    w = rep(rng.standard_normal((N, Kd)) / np.sqrt(Kd), dtype)
    bias = rep(0.5 * rng.standard_normal(N), "f32")
    dy = rep(rng.standard_normal((rows, N)), dtype)
    dt = dt_of(K, dtype)
    ws, nb = ws_for(K.cnnk_linear_workspace_bytes(rows, Kd, N, dt))
    gx, gw, gdy = dev(x, dtype), dev(w, dtype), dev(dy, dtype)
    tol = OUT_TOL[dtype] if dtype == "bf16" else 2e-5
    z = x @ w.T
    for b in (None, bias):
        gy = dev(np.zeros((rows, N)), dtype)
        K.cnnk_linear_fwd(rows, Kd, N, dt, gx, gw, None if b is None else dev_f32(b), K.ACT_NONE, None, gy, ws, nb)
        torch.cuda.synchronize()
        # convolution path in bf16: the product is rounded before the bias is added, and again after
        assert max_rel_err(host(gy), z + (0.0 if b is None else b)) <= tol * (2 if (dtype == "bf16" and b is not None) else 1)
    # residual connection: the sum of the stored product and the residual
    res = rep(rng.standard_normal((rows, N)), dtype)
    gy = dev(np.zeros((rows, N)), dtype)
    K.cnnk_linear_fwd(rows, Kd, N, dt, gx, gw, dev_f32(bias), K.ACT_NONE, None, gy, ws, nb, res=dev(res, dtype))
    torch.cuda.synchronize()
    assert max_rel_err(host(gy), z + bias + res) <= tol * (2 if dtype == "bf16" else 1)
    gu, gy = dev(np.zeros((rows, N)), dtype), dev(np.zeros((rows, N)), dtype)
    K.cnnk_linear_fwd(rows, Kd, N, dt, gx, gw, dev_f32(bias), K.ACT_GELU, gu, gy, ws, nb)
    torch.cuda.synchronize()
    u = host(gu)
    assert max_rel_err(u, z + bias) <= tol * (2 if dtype == "bf16" else 1)
    assert max_rel_err(host(gy), V.gelu(u)) <= tol
    gdx = dev(np.zeros((rows, Kd)), dtype)
    K.cnnk_linear_dgrad(rows, Kd, N, dt, gdy, gw, gdx, ws, nb)
    torch.cuda.synchronize()
    assert max_rel_err(host(gdx), dy @ w) <= tol
    gdw = torch.full((N, Kd), 3.0, device="cuda:0")
    K.cnnk_linear_wgrad(rows, Kd, N, dt, gx, gdy, gdw, ws, nb)
    torch.cuda.synchronize()
    assert max_rel_err(host(gdw), dy.T @ x) <= 2e-5
    # bit-reproducible
    gdw2 = torch.zeros((N, Kd), device="cuda:0")
    K.cnnk_linear_wgrad(rows, Kd, N, dt, gx, gdy, gdw2, ws, nb)
    torch.cuda.synchronize()
    assert torch.equal(gdw, gdw2)


# bf16 with head size 64 runs on the matrix cores (one 32-token block per wavefront: 17, 197, 256, 33
# tokens = 1, 7, 8, 2 blocks with ragged and full last blocks); "bf16-valu" forces the general kernels
@pytest.mark.parametrize("dtype", ["f32", "bf16", "bf16-valu"])
@pytest.mark.parametrize("B,T,heads,dh", [(2, 17, 2, 64), (1, 197, 3, 64), (2, 5, 2, 16), (1, 50, 4, 32), (1, 300, 1, 32),
                                          (3, 1, 2, 16), (1, 256, 1, 64), (2, 33, 12, 64), (1, 1, 1, 64)])
def test_attention(K, B, T, heads, dh, dtype):
    from paper_2503_23186_amd import cnnk
    if dtype == "bf16-valu":
        if dh != 64:
            pytest.skip("already on the general kernels")
        cnnk.cnnk_tune(10, -1)
        try:
            _attention_case(K, B, T, heads, dh, "bf16")
        finally:
            cnnk.cnnk_tune(10, 0)
    else:
        _attention_case(K, B, T, heads, dh, dtype)


# five to eight blocks of tokens, in one or two parts to a head; 128 heads in all and more, not a multiple of eight.  rise: scores
# that climb (or fall) by that much over the keys, so that the sums' reference is raised in several tiles, by little and by much
@pytest.mark.parametrize("B,T,heads,rise", [(1, 129, 3, 0), (1, 160, 2, 0), (3, 161, 1, 0), (2, 192, 5, 0), (1, 225, 1, 0), (11, 129, 12, 0),
                                            (43, 130, 3, 0), (2, 197, 2, 12), (2, 197, 2, 60), (2, 197, 2, -60), (1, 65, 3, 30)])
def test_attention_in_parts(K, B, T, heads, rise):
    _attention_case(K, B, T, heads, 64, "bf16", rise)


# so many heads that the backward pass takes each as a whole: one to eight blocks of tokens, the first count of heads past the line
# and one more round
@pytest.mark.parametrize("B,T,heads,rise", [(205, 20, 5, 0), (57, 33, 9, 0), (103, 64, 5, 0), (257, 65, 1, 0), (52, 96, 5, 60), (257, 97, 1, 0), (64, 128, 8, 0),
                                            (19, 65, 41, 0), (43, 129, 3, -60), (32, 160, 8, 0), (13, 161, 10, 0), (9, 197, 50, 0), (15, 256, 9, 0)])
def test_attention_as_a_whole(K, B, T, heads, rise):
    _attention_case(K, B, T, heads, 64, "bf16", rise)


# scores that all lie far from zero, at lengths that are no multiple of 32: a key past the end has score 0, and its exponential
# relative to the others' log-sum-exp is beyond every float
@pytest.mark.parametrize("B,T,heads,shift", [(2, 33, 3, -110), (1, 65, 6, -128), (3, 101, 2, -200), (40, 65, 6, -128), (1, 130, 2, -128), (2, 197, 2, -150),
                                             (16, 197, 12, -128), (22, 129, 12, -128), (44, 65, 6, -128), (1, 65, 2, 128), (1, 197, 2, 200)])
def test_attention_scores_far_from_zero(K, B, T, heads, shift):
    _attention_case(K, B, T, heads, 64, "bf16", 0, shift)


# values near the largest float: the result is an average of them and finite, undivided sums of it are not
@pytest.mark.parametrize("B,T,heads,rise", [(1, 65, 2, 0), (2, 197, 3, 0), (1, 256, 2, 0), (1, 197, 2, 60), (3, 40, 2, -30)])
def test_attention_of_values_near_the_largest_float(K, B, T, heads, rise):
    rng = np.random.default_rng(T)
    d = heads * 64
    qkv = rng.standard_normal((B, T, 3 * d))
    qkv[:, :, 0:d:64] = 8.0
    qkv[:, :, d:2 * d:64] = (rise * np.arange(T) / T)[None, :, None]
    qkv[:, :, 2 * d + 5::64] = 3e38                                  # one feature of every head, the others as they are
    qkv[:, :, 2 * d + 9::64] = -1e36 * rng.random((B, T, heads))
    qkv = rep(qkv, "bf16")
    O, A = V.attention_fwd(qkv, heads)
    go, lse = dev(np.zeros((B, T, d)), "bf16"), torch.zeros((B, heads, T), device="cuda:0")
    K.cnnk_attention_fwd(K.attn_desc(B, T, heads, 64, dt_of(K, "bf16")), dev(qkv, "bf16"), go, lse)
    torch.cuda.synchronize()
    got = host(go)
    weight = (A @ np.abs(qkv[:, :, 2 * d:].reshape(B, T, heads, 64).transpose(0, 2, 1, 3))).transpose(0, 2, 1, 3).reshape(B, T, d)
    worst = (np.abs(got - O) / (2.0 ** -8 * 1.01 * (np.abs(O) + weight))).max()
    assert np.isfinite(got).all() and worst <= 1, worst


def _attention_case(K, B, T, heads, dh, dtype, rise=None, shift=0):
    rng = np.random.default_rng(B * 7 + T * 13 + heads + dh)
    d = heads * dh
    qkv = rng.standard_normal((B, T, 3 * d)) * 1.3
    if rise or shift:        # one feature carries it: 8 of every query times shift + rise * t / T of key t, over the scale of 8
        qkv[:, :, 0:d:dh] = 8.0
        qkv[:, :, d:2 * d:dh] = (shift + (rise or 0) * np.arange(T) / T)[None, :, None]
    qkv = rep(qkv, dtype)
    dO = rep(rng.standard_normal((B, T, d)), dtype)
    O, A = V.attention_fwd(qkv, heads)
    ad = K.attn_desc(B, T, heads, dh, dt_of(K, dtype))
    gq, go = dev(qkv, dtype), dev(np.zeros((B, T, d)), dtype)
    lse = torch.zeros((B, heads, T), device="cuda:0")
    K.cnnk_attention_fwd(ad, gq, go, lse)
    torch.cuda.synchronize()
    split = lambda t, n: [t[:, :, i * d:(i + 1) * d].reshape(B, T, heads, dh).transpose(0, 2, 1, 3) for i in range(n)]
    join = lambda t: t.transpose(0, 2, 1, 3).reshape(B, T, d)
    q, k, v = split(qkv, 3)
    if rise is None:
        assert max_rel_err(host(go), O) <= (OUT_TOL[dtype] if dtype == "bf16" else 5e-5)
    else:           # the probabilities are rounded to bf16 in front of their product, its result in storage: 2^-8 of either
        assert np.all(np.abs(host(go) - O) <= 2.0 ** -8 * 1.01 * (np.abs(O) + join(A @ np.abs(v))))
    S = q @ k.transpose(0, 1, 3, 2) / np.sqrt(dh)
    want_lse = np.log(np.exp(S - S.max(-1, keepdims=True)).sum(-1)) + S.max(-1)
    assert np.abs(host(lse) - want_lse).max() <= 1e-4
    # backward from the oracle's own output (both sides differentiate at the same point)
    Oq = rep(O, dtype)
    want = V.attention_bwd(dO, qkv, A, heads)
    gd = dev(np.zeros((B, T, 3 * d)), dtype)
    K.cnnk_attention_bwd(ad, gq, dev(Oq, dtype), dev(dO, dtype), lse, gd)
    torch.cuda.synchronize()
    got = host(gd)
    assert np.isfinite(got).all()
    if rise or shift:
        # The large feature's products cancel in the sums, so the bound is made of the terms: half an ulp of bf16 (2^-8) for the
        # probabilities, for ds = p (dp - D) / 8 and for the result; D is taken of the rounded output; 2e-4 for the exponent (scores of
        # up to 200 in fp32, five roundings of 2^-24 of 300) and 1e-5 of its operands for the difference.
        g, o = split(dO, 1)[0], split(O, 1)[0]
        dA = g @ v.transpose(0, 1, 3, 2)
        D = (dA * A).sum(-1, keepdims=True)
        h = 2.0 ** -8 * 1.01
        e_ds = (A * np.abs(dA - D) * (h + 2e-4) + A * (h * (np.abs(g) * np.abs(o)).sum(-1, keepdims=True) + 1e-5 * (np.abs(dA) + np.abs(D)))) / np.sqrt(dh)
        e_p = A * (h + 2e-4)
        T_ = lambda t: t.transpose(0, 1, 3, 2)
        for i, (name, bound) in enumerate((("q", e_ds @ np.abs(k)), ("k", T_(e_ds) @ np.abs(q)), ("v", T_(e_p) @ np.abs(g)))):
            part, ref = got[:, :, i * d:(i + 1) * d], want[:, :, i * d:(i + 1) * d]
            worst = (np.abs(part - ref) / (join(bound) + h * (np.abs(ref) + join(bound)) + 1e-30)).max()
            assert worst <= 1, (name, worst)
        return
    for i, name in enumerate("qkv"):
        # D = do . o is taken of the stored (rounded) output: one more rounding than the oracle's exact D.
        # With a single key the query and key gradients are exactly zero: the error is then measured
        # against the size of the value gradient.
        part, ref = got[:, :, i * d:(i + 1) * d], want[:, :, i * d:(i + 1) * d]
        scale = max(np.abs(ref).max(), 1e-2 * np.abs(want).max())
        assert np.abs(part - ref).max() / scale <= (OUT_TOL[dtype] * 2 if dtype == "bf16" else 5e-5), name


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,image,patch,dim", [(2, 16, 4, 32), (3, 32, 8, 128), (1, 224, 16, 768), (2, 24, 8, 64)])
def test_patches_and_tokens(K, B, image, patch, dim, dtype):
    rng = np.random.default_rng(image + dim)
    n = (image // patch) ** 2
    x = rep(rng.standard_normal((B, image, image, 3)), dtype)
    ed = K.embed_desc(B, image, patch, dim, dt_of(K, dtype))
    gp = dev(np.zeros((B, n, patch * patch * 3)), dtype)
    K.cnnk_vit_patchify(ed, dev(x, dtype), gp)
    torch.cuda.synchronize()
    assert (host(gp) == V.patchify(x, patch)).all()
    z = rep(rng.standard_normal((B, n, dim)), dtype)
    be, cls, pos = (rep(rng.standard_normal(s), "f32") for s in ((dim,), (dim,), (n + 1, dim)))
    gt = dev(np.zeros((B, n + 1, dim)), dtype)
    K.cnnk_vit_embed_fwd(ed, dev(z, dtype), dev_f32(be), dev_f32(cls), dev_f32(pos), gt)
    torch.cuda.synchronize()
    want = np.empty((B, n + 1, dim))
    want[:, 0] = cls + pos[0]
    want[:, 1:] = z + be + pos[1:]
    assert max_rel_err(host(gt), want) <= OUT_TOL[dtype]
    dtok = rep(rng.standard_normal((B, n + 1, dim)), dtype)
    gdz = dev(np.zeros((B, n, dim)), dtype)
    gdbe, gdcls, gdpos = (torch.zeros(s, device="cuda:0") for s in ((dim,), (dim,), (n + 1, dim)))
    K.cnnk_vit_embed_bwd(ed, dev(dtok, dtype), gdz, gdbe, gdcls, gdpos)
    torch.cuda.synchronize()
    assert (host(gdz) == dtok[:, 1:]).all()
    assert max_rel_err(host(gdpos), dtok.sum(0)) <= SUM_TOL[dtype]
    assert max_rel_err(host(gdcls), dtok[:, 0].sum(0)) <= SUM_TOL[dtype]
    assert max_rel_err(host(gdbe), dtok[:, 1:].sum((0, 1))) <= SUM_TOL[dtype]


# ---- the whole step -------------------------------------------------------------------------------------
ACTS = {"TOK": "X0", "H": "H", "QKV": "QKV", "O": "O", "XMID": "Xmid", "H2": "H2", "U": "U", "G": "G", "F": "F"}
DACTS = {"DH": "H", "DQKV": "QKV", "DO": "O", "DXMID": "Xmid", "DH2": "H2", "DU": "U", "DG": "G", "DF": "F"}


def run_hip(net, inp, lr, momentum, wd, two_streams=True):
    from paper_2503_23186_amd.vit import VitRunner
    r = VitRunner(net, two_streams=two_streams)
    r.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
    r.step(lr, momentum, wd)
    torch.cuda.synchronize()
    return r


def hip_tensors(r, net):
    """The HIP step's tensors by the oracle's names: (acts, dacts, grads, params, mom)."""
    B, T, L = net.batch, net.tokens, net.layers
    acts, dacts = {}, {}
    for name, on in ACTS.items():
        if name in ("TOK", "F"):
            acts[on] = host(r.tensor(name))
        else:
            for l in range(L):
                acts["%s.%d" % (on, l)] = host(r.tensor(name, l))
    for l in range(L):
        acts["Xout.%d" % l] = host(r.tensor("XOUT", l))
    for name, on in DACTS.items():
        if name == "DF":
            dacts[on] = host(r.tensor(name))
        else:
            for l in range(L):
                dacts["%s.%d" % (on, l)] = host(r.tensor(name, l))
    for l in range(L):
        dacts["Xin.%d" % l] = host(r.tensor("DXOUT", l - 1)) if l else host(r.tensor("DTOK"))
    dacts["Xout"] = host(r.tensor("DXOUT", L - 1))
    grads = {n: host(r.grad[k]) for k, n in enumerate(r.names)}
    params = {n: host(r.param[k]) for k, n in enumerate(r.names)}
    mom = {n: host(r.mom[k]) for k, n in enumerate(r.names)}
    return acts, dacts, grads, params, mom


def oracle_tensors(out, net):
    c, L = out["cache"], net.layers
    acts = {k: v for k, v in c.items() if k.split(".")[0] in ("X0", "H", "QKV", "O", "Xmid", "H2", "U", "G", "F")}
    for l in range(L):
        acts["Xout.%d" % l] = c["Xin.%d" % (l + 1)] if l + 1 < L else c["Xout"]
    return acts, out["dacts"], out["grads"], out["params"], out["mom"]


def compare(got, want, metric):
    """Worst figure per tensor class over all tensors of the class."""
    worst = {}
    for cls, g, w in zip(("acts", "dacts", "grads", "params", "mom"), got, want):
        assert set(g) == set(w), (cls, set(g) ^ set(w))
        worst[cls] = max(metric(g[k].reshape(w[k].shape), w[k]) for k in w)
    return worst


def l2_rel(got, ref):
    return float(np.linalg.norm((got - ref).ravel()) / max(np.linalg.norm(ref.ravel()), 1e-30))


STEP_NETS = {
    "b16": dict(batch=2, image=224, patch=16, dim=768, heads=12, layers=2, mlp=3072),  # ViT-B/16's geometry, two blocks
    "b16-full-depth": dict(batch=8, image=224, patch=16, dim=768, heads=12, layers=12, mlp=3072),  # ViT-B/16 itself, batch 8
    "mini": dict(batch=4, image=32, patch=8, dim=128, heads=2, layers=2, mlp=256),
    "tall": dict(batch=2, image=64, patch=8, dim=64, heads=4, layers=3, mlp=192),     # 65 tokens, dh 16
    "wide": dict(batch=3, image=32, patch=16, dim=256, heads=4, layers=1, mlp=1024),  # 5 tokens, dh 64
}


@pytest.mark.parametrize("name", [n for n in STEP_NETS if not n.startswith("b16")])
def test_step_fp32(K, name):
    net = WL.vit_mini(dtype="f32", **STEP_NETS[name])
    inp = WL.make_vit_inputs(net, config_id=62)
    lr, mu, wd = 0.05, 0.9, 1e-3
    r = run_hip(net, inp, lr, mu, wd)
    out = V.train_step(net.cfg(), inp["x"], inp["labels"], inp["params"], inp["mom"], lr, mu, wd)
    assert abs(r.loss.item() - out["loss"]) <= 1e-4 * abs(out["loss"])
    assert (host(r.pred) == out["pred"]).all()
    assert np.abs(host(r.probs) - out["probs"]).max() <= 1e-5
    worst = compare(hip_tensors(r, net), oracle_tensors(out, net), max_rel_err)
    assert all(v <= 1e-4 for v in worst.values()), worst


@pytest.mark.parametrize("name", list(STEP_NETS))
def test_step_bf16_against_the_ensemble_of_legal_walks(K, name):
    """The free-running bf16 step against the float64 walk and against the oracle's own bf16 walks
    (plain and seeded, as for the convolutional networks): per tensor class the L2 distance to the
    float64 walk and the mean distance to the members must lie inside the band that the members
    themselves span; loss within 2e-2; predictions equal wherever the oracle's margin is clear."""
    net = WL.vit_mini(dtype="bf16", **STEP_NETS[name])
    inp = WL.make_vit_inputs(net, config_id=63)
    lr, mu, wd = 0.05, 0.9, 1e-3
    r = run_hip(net, inp, lr, mu, wd)
    cfg = net.cfg()
    exact = V.train_step(cfg, inp["x"], inp["labels"], inp["params"], inp["mom"], lr, mu, wd)
    members = [V.train_step(cfg, inp["x"], inp["labels"], inp["params"], inp["mom"], lr, mu, wd, storage="bf16")]
    members += [V.train_step(cfg, inp["x"], inp["labels"], inp["params"], inp["mom"], lr, mu, wd,
                             q=oracle_quantiser("bf16", (s, JITTER_REL))) for s in JITTER_SEEDS]
    assert abs(r.loss.item() - exact["loss"]) <= 2e-2
    got = hip_tensors(r, net)
    ex = oracle_tensors(exact, net)
    mem = [oracle_tensors(m, net) for m in members]
    d_exact = compare(got, ex, l2_rel)
    m_exact = [compare(m, ex, l2_rel) for m in mem]
    d_mem = [compare(got, m, l2_rel) for m in mem]
    m_mem = [compare(mem[i], mem[j], l2_rel) for i in range(len(mem)) for j in range(i + 1, len(mem))]
    for cls in d_exact:
        tol = 1e-6 if cls in ("params", "mom") else 2e-2
        assert d_exact[cls] <= ensemble_bound([m[cls] for m in m_exact], tol, SCALE_TO_EXACT), (cls, d_exact, m_exact)
        assert np.mean([d[cls] for d in d_mem]) <= ensemble_bound([m[cls] for m in m_mem], tol, SCALE_TO_MEMBER), (cls, d_mem, m_mem)
    logits = exact["cache"]["logits"]
    top2 = np.sort(logits, axis=1)[:, -2:]
    clear = (top2[:, 1] - top2[:, 0]) > 5e-2
    assert (host(r.pred)[clear] == exact["pred"][clear]).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_second_stream_changes_no_bit(K, dtype):
    """The weight and bias gradients forked onto a second stream: same kernels, same order of every
    sum, so two consecutive steps give bit-identical parameters, momentum buffers and gradients."""
    net = WL.vit_mini(dtype=dtype, **STEP_NETS["mini"])
    inp = WL.make_vit_inputs(net, config_id=64)
    runs = []
    for two in (False, True):
        r = run_hip(net, inp, 0.05, 0.9, 1e-3, two_streams=two)
        r.step(0.05, 0.9, 1e-3)
        torch.cuda.synchronize()
        runs.append(r)
    a, b = runs
    assert a.loss.item() == b.loss.item()
    for k in range(len(a.names)):
        assert torch.equal(a.param[k], b.param[k]) and torch.equal(a.mom[k], b.mom[k]) and torch.equal(a.grad[k], b.grad[k]), a.names[k]


# ragged groups: two and one blocks left over on two streams, two on one; rows split over workgroups (64 columns); a group
# that one stream makes large and two streams small
@pytest.mark.parametrize("batch,image,patch,dim,layers,mlp", [(24, 32, 4, 384, 8, 1536), (40, 32, 4, 192, 9, 768), (70, 32, 4, 64, 9, 256),
                                                              (3, 32, 8, 768, 9, 3072)])
def test_second_stream_changes_no_bit_of_grouped_gradients(batch, image, patch, dim, layers, mlp):
    net = WL.ViT("vit", batch, "bf16", image, patch, dim, dim // 64, layers, mlp)
    inp = WL.make_vit_inputs(net, 29)
    a, b = (run_hip(net, inp, 0.05, 0.9, 1e-3, two_streams=two) for two in (False, True))
    torch.cuda.synchronize()
    for k, name in enumerate(a.names):
        assert torch.equal(a.grad[k], b.grad[k]) and torch.equal(a.param[k], b.param[k]), name


# ---- the epoch loop around the step ---------------------------------------------------------------------
def _loop_case(dtype):
    net = WL.vit_mini(batch=4, dtype=dtype, image=32, patch=8, dim=128, heads=2, layers=2, mlp=256, classes=10)
    inp = WL.make_vit_inputs(net, config_id=66)
    ds = WL.make_vit_dataset(net, 66, n_train=24, n_val=8, signal=1.0)
    return net, inp, ds


def test_eval_step_matches_the_oracle_and_touches_no_training_state(K):
    from paper_2503_23186_amd.vit import VitRunner
    for dtype in ("f32", "bf16"):
        net, inp, ds = _loop_case(dtype)
        r = VitRunner(net)
        r.load(ds["val_x"][:4], ds["val_y"][:4], inp["params"], inp["mom"])
        before = [t.clone() for t in r.param + r.mom + r.grad]
        nc = torch.full((1,), 5, dtype=torch.int32, device="cuda:0")
        K.cnnk_vit_eval_step(r.desc, r.buffers, nc)
        torch.cuda.synchronize()
        loss, c = V.forward(net.cfg(), ds["val_x"][:4], ds["val_y"][:4], inp["params"], storage=None)
        tol = 1e-5 if dtype == "f32" else 2e-2
        assert abs(r.loss.item() - loss) <= tol * max(1.0, abs(loss))
        assert np.abs(host(r.probs) - c["probs"]).max() <= tol
        top2 = np.sort(c["logits"], axis=1)[:, -2:]
        clear = (top2[:, 1] - top2[:, 0]) > (1e-4 if dtype == "f32" else 5e-2)
        assert (host(r.pred)[clear] == c["pred"][clear]).all()
        assert nc.item() == 5 + int(np.sum(host(r.pred) == ds["val_y"][:4]))
        assert all(torch.equal(a, b) for a, b in zip(before, r.param + r.mom + r.grad))


def test_fit_matches_the_oracle_loop_fp32(K, tmp_path):
    from paper_2503_23186_amd.trainer import VitTrainer, cosine_lr
    net, inp, ds = _loop_case("f32")
    epochs, nb = 3, 24 // 4
    orders = WL.epoch_orders(66, 24, 4, epochs)
    lrs = cosine_lr(0.05, epochs * nb, warmup_steps=3)
    want = V.fit(net.cfg(), 4, ds["train_x"], ds["train_y"], ds["val_x"], ds["val_y"], inp["params"], inp["mom"], orders, lrs,
                 momentum=0.9, weight_decay=1e-3)
    t = VitTrainer(net)
    t.load_state(inp["params"], inp["mom"])
    tx, ty = t.to_device(ds["train_x"], ds["train_y"])
    vx, vy = t.to_device(ds["val_x"], ds["val_y"])
    ck = str(tmp_path / "best.safetensors")
    hist = t.fit(tx, ty, vx, vy, orders, lrs, 0.9, 1e-3, ckpt_path=ck)
    for (gl, ga, gv), (wl, wa, wv) in zip(hist, want["history"]):
        assert abs(gl - wl) <= 1e-4 * abs(wl) and ga == wa and abs(gv - wv) <= 1e-4 * abs(wv)
    for k, name in enumerate(t.run.names):
        assert max_rel_err(host(t.run.param[k]), want["params"][name].reshape(t.run.param[k].shape)) <= 1e-4, name
        assert max_rel_err(host(t.run.mom[k]), want["mom"][name].reshape(t.run.mom[k].shape)) <= 1e-4, name
    assert t.best_epoch == want["best"]["epoch"] and t.best_acc == want["best"]["acc"]
    # the checkpoint holds the best epoch's parameters and reproduces its accuracy
    t2 = VitTrainer(net)
    t2.load_checkpoint(ck)
    assert t2.epoch == want["best"]["epoch"] + 1
    for k, name in enumerate(t2.run.names):
        assert max_rel_err(host(t2.run.param[k]), want["best"]["params"][name].reshape(t2.run.param[k].shape)) <= 1e-4, name
    assert t2.evaluate(vx, vy)[0] == want["best"]["acc"]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_resume_from_checkpoint_is_bit_identical(K, tmp_path, dtype):
    from paper_2503_23186_amd.trainer import VitTrainer, step_lr
    net, inp, ds = _loop_case(dtype)
    nb = 24 // 4
    orders = WL.epoch_orders(67, 24, 4, 4)
    lrs = step_lr(0.05, nb, 4, milestones=[2])
    full = VitTrainer(net)
    full.load_state(inp["params"], inp["mom"])
    tx, ty = full.to_device(ds["train_x"], ds["train_y"])
    vx, vy = full.to_device(ds["val_x"], ds["val_y"])
    h_full = full.fit(tx, ty, vx, vy, orders, lrs, 0.9, 1e-3)
    a = VitTrainer(net)
    a.load_state(inp["params"], inp["mom"])
    h_a = a.fit(tx, ty, vx, vy, orders[:2], lrs, 0.9, 1e-3)
    ck = str(tmp_path / "mid.safetensors")
    a.save_checkpoint(ck)
    b = VitTrainer(net)
    b.load_checkpoint(ck)
    h_b = b.fit(tx, ty, vx, vy, orders[2:], lrs, 0.9, 1e-3)
    assert h_a + h_b == h_full
    for k in range(len(full.run.names)):
        assert torch.equal(full.run.param[k], b.run.param[k]) and torch.equal(full.run.mom[k], b.run.mom[k])
    # the per-call profile leaves the training state alone
    before = [t.clone() for t in b.run.param + b.run.mom]
    prof = b.profile(steps=2)
    assert len(prof) == b.run.n_calls and all(ms >= 0 for _, ms in prof)
    assert all(torch.equal(x, y) for x, y in zip(before, b.run.param + b.run.mom))


# The backward pass with its weight gradients in groups (the default) against the same step call by call (per-call
# timing makes it so): one block and one token row tile; rows split over workgroups (>= 512 rows, few tiles); several
# blocks a group with a ragged last group; a width whose products fill the device unsplit.
@pytest.mark.parametrize("two_streams", [True, False])
@pytest.mark.parametrize("batch,image,patch,dim,layers,mlp", [(1, 16, 16, 64, 1, 72), (9, 64, 8, 128, 2, 200), (40, 32, 4, 192, 9, 768),
                                                              (3, 32, 8, 768, 3, 3072)])
def test_grouped_backward_matches_call_by_call(batch, image, patch, dim, layers, mlp, two_streams):
    from paper_2503_23186_amd.vit import VitRunner
    net = WL.ViT("vit", batch, "bf16", image, patch, dim, dim // 64, layers, mlp)
    inp = WL.make_vit_inputs(net, 11)
    got = []
    for timed in (False, True):
        run = VitRunner(net, two_streams=two_streams)
        run.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
        run.enable_timing(timed)
        run.step(0.05, 0.9, 1e-3)
        torch.cuda.synchronize()
        got.append(dict(zip(run.names, zip(run.grad, run.param, run.mom))))
    for name in got[0]:
        for a, b in zip(got[0][name], got[1][name]):
            a, b = a.double(), b.double()
            # the two differ in the order of fp32 sums and in gelu's derivative (1e-7 each): where that moves a stored
            # bf16 gradient by a unit (2^-8), the layers below see an error of that size in few elements
            assert (a - b).norm() <= 1e-2 * b.norm() + 1e-12, (name, ((a - b).norm() / b.norm()).item())


# every tile shape of the data gradient that takes GELU's gradient (tuning key 15), ragged in rows and columns, and the
# shapes that the sizes choose (0) for one tile and for several
@pytest.mark.parametrize("batch,image,patch,dim,mlp,shape", [(9, 64, 8, 128, 200, s) for s in (0, 1, 2, 16, 17, 18, 19, 20)] +
                         [(1, 16, 16, 64, 72, 0), (40, 32, 4, 192, 768, 0)])
def test_grouped_step_sums_the_unrounded_products_for_the_bias_of_the_activation(batch, image, patch, dim, mlp, shape):
    """dc1 = column sums of dg * gelu'(u) before the products are stored: fp32 sums of fp32 products, so within some
    units of 2^-24 of the sums' terms (the stored bf16 products are off by 2^-9 each)."""
    from paper_2503_23186_amd import cnnk
    from paper_2503_23186_amd.vit import VitRunner
    net = WL.ViT("vit", batch, "bf16", image, patch, dim, dim // 64, 2, mlp)
    inp = WL.make_vit_inputs(net, 13)
    cnnk.cnnk_tune(15, shape)
    try:
        run = VitRunner(net)
        run.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
        run.step(0.05, 0.9, 1e-3)
        torch.cuda.synchronize()
    finally:
        cnnk.cnnk_tune(15, 0)
    for l in range(2):
        dg, u, du = (run.tensor(n, l).view(-1, mlp).double() for n in ("DG", "U", "DU"))
        terms = dg * (0.5 * torch.erfc(-u / 2 ** 0.5) + u * torch.exp(-0.5 * u * u) / (2 * torch.pi) ** 0.5)
        assert bool(((du - terms).abs() <= 2 ** -8 * terms.abs() + 1e-6 * dg.abs()).all())
        err = (run.grad[run.names.index("c1.%d" % l)].double() - terms.sum(0)).abs()
        assert bool((err <= 2 ** -20 * terms.abs().sum(0) + 1e-30).all()), (l, (err / terms.abs().sum(0)).max().item())


# A sum of `rows` products runs in steps of 16; two chains of about the root of the steps each leave a relative error of
# about 2^-24 times the fourth root of the steps / 2 to 3 (1.8e-7 at 12608 rows), one chain of them all four times that.
def wgrad_bound(rows):
    return 0.75 * 2.0 ** -24 * (rows / 16) ** 0.25


@pytest.mark.parametrize("rows,K,N,shape", [(6240, 384, 1536, 0), (788, 768, 3072, 0), (1576, 768, 768, 0), (1576, 3072, 768, 0), (4097, 200, 72, 0)] +
                         [(5003, 136, 200, s) for s in (16, 17, 18, 19)])
def test_linear_weight_gradient_keeps_its_chains_of_sums_short(rows, K, N, shape):
    from paper_2503_23186_amd import cnnk, vit
    g = torch.Generator(device="cuda:0")
    g.manual_seed(17)
    x, dy = (torch.randn((rows, c), generator=g, device="cuda:0").bfloat16() for c in (K, N))
    dw = torch.zeros((N, K), device="cuda:0")
    cnnk.cnnk_tune(15, shape)
    try:
        need = max(256, vit.cnnk_linear_workspace_bytes(rows, K, N, cnnk.BF16))
        ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
        vit.cnnk_linear_wgrad(rows, K, N, cnnk.BF16, x, dy, dw, ws, need, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        cnnk.cnnk_tune(15, 0)
    want = dy.double().T @ x.double()
    assert ((dw.double() - want).norm() / want.norm()).item() <= wgrad_bound(rows)


@pytest.mark.parametrize("batch,image,patch,dim,mlp", [(64, 224, 16, 768, 3072), (15, 60, 4, 768, 3072), (40, 32, 4, 192, 768)])
def test_grouped_weight_and_bias_gradients_keep_their_chains_of_sums_short(batch, image, patch, dim, mlp):
    from paper_2503_23186_amd.vit import VitRunner
    net = WL.ViT("vit", batch, "bf16", image, patch, dim, dim // 64, 2, mlp)
    inp = WL.make_vit_inputs(net, 19)
    run = VitRunner(net)
    run.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
    run.step(0.05, 0.9, 1e-3)
    torch.cuda.synchronize()
    rows, grad = batch * net.tokens, dict(zip(run.names, run.grad))
    for dy, x, w, b in (("DXOUT", "G", "W2", "c2"), ("DU", "H2", "W1", None), ("DXMID", "O", "Wo", "bo"), ("DQKV", "H", "Wqkv", "bqkv")):
        d, x = run.tensor(dy, 0).view(rows, -1).double(), run.tensor(x, 0).view(rows, -1).double()
        want = d.T @ x
        assert ((grad[w + ".0"].double() - want).norm() / want.norm()).item() <= wgrad_bound(rows), w
        if b:           # a compensated sum: the roundings of sixteen terms at a time and of the result
            want = d.sum(0)
            assert ((grad[b + ".0"].double() - want).norm() / want.norm()).item() <= 2.0 ** -23, b


def test_infinite_gradient_makes_an_infinite_bias_gradient():
    """One image, so that one row of the last block's output has a gradient: the gradient of that block's last bias is
    this row, also where it overflows (a huge scale of the final norm on one channel)."""
    from paper_2503_23186_amd.vit import VitRunner
    net = WL.ViT("vit", 1, "bf16", 16, 16, 64, 1, 1, 72)
    inp = WL.make_vit_inputs(net, 29)
    p = inp["params"]
    for name in ("cls", "pos", "Wo.0", "bo.0", "W2.0", "c2.0"):
        p[name] = p[name] * 2.0 ** -6
    p["gf"][7] = 2.0 ** 119
    p["bf"][7] = 0
    p["Wh"][:, 7] = np.where(np.arange(len(p["Wh"])) == inp["labels"][0], 1.0, -1.0)
    p["cls"][7], p["pos"][0, 7] = -2.0 ** -10, -2.0 ** -10      # below the mean: the label's logit is the lowest
    run = VitRunner(net)
    run.load(inp["x"], inp["labels"], p, inp["mom"])
    run.step(0.05, 0.9, 1e-3)
    torch.cuda.synchronize()
    dx = run.tensor("DXOUT", 0).view(2, 64).float()
    assert bool(dx[0, 7].isinf()) and bool(dx[0].isfinite().any()) and not bool(dx.isnan().any()) and not bool(dx[1].any())
    assert torch.equal(run.grad[run.names.index("c2.0")], dx[0])


@pytest.mark.parametrize("two_streams", [True, False])
@pytest.mark.parametrize("batch,image,patch,dim,layers,mlp", [(3, 32, 8, 768, 5, 3072), (9, 64, 8, 128, 9, 200)])
def test_step_needs_nothing_of_its_workspace_but_the_room(batch, image, patch, dim, layers, mlp, two_streams):
    """Same bits from a workspace of the size that the library asks for, whatever it holds, and no byte behind it."""
    from paper_2503_23186_amd.vit import VitRunner
    net = WL.ViT("vit", batch, "bf16", image, patch, dim, dim // 64, layers, mlp)
    inp = WL.make_vit_inputs(net, 23)
    out = []
    for fill in (0x00, 0xff):
        run = VitRunner(net, two_streams=two_streams)
        room = run.ws.numel()
        assert room == run.ws_bytes * (2 if two_streams else 1)
        guarded = torch.full((room + 4096,), fill, dtype=torch.uint8, device="cuda:0")
        run.buffers.ws = guarded.data_ptr()
        run.load(inp["x"], inp["labels"], inp["params"], inp["mom"])
        for _ in range(2):
            run.step(0.05, 0.9, 1e-3)
        torch.cuda.synchronize()
        assert bool((guarded[room:] == fill).all())
        out.append([t.clone() for t in run.param + run.mom + run.grad])
    for name, a, b in zip(3 * run.names, *out):
        assert torch.equal(a, b), name
