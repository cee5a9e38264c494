"""The fp32 matrix-core kernels at the edges of their tiles, every tile shape forced, against 64-bit products.

Tolerance: a product over K terms of unit-variance operands, summed in fp32 in any order, is off by at most about
eps * sqrt(K) of its own spread sqrt(K) per rounding, i.e. a few times 2^-24 * sqrt(K) relative to the largest element;
2e-5 leaves that a factor of ten at the largest K here.
"""
import numpy as np
import pytest

from oracle import stage_oracle as so
from paper_2507_00217_amd import synth
from tests.gpu_util import to_dev, to_np
from tests.test_gpu_kernels import L, P

pytestmark = pytest.mark.gpu
TOL = 2e-5

# one tile and less, one past a tile edge in M, reductions below / at / past a 16-deep slice, W slices and their double buffer
SHAPES = [(1, 4, 4), (16, 16, 16), (17, 20, 20), (33, 36, 132), (65, 68, 260), (63, 64, 1028), (130, 196, 524),
          (2052, 2048, 63), (2052, 2048, 65)]      # on either side of the rule for short reductions of large outputs (K is rounded up to 64 and 66 or 68)


@pytest.mark.parametrize("shape", [0, 2, 3, 4])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_products(mode, shape, M, N, K):
    import torch
    if mode == 2:
        M = (M + 3) // 4 * 4
        K = K + 1                                   # a slow reduction index has no alignment
    else:
        K = (K + 3) // 4 * 4
    A = synth.normal(31, 1, (K, M) if mode == 2 else (M, K)); B = synth.normal(31, 2, (N, K) if mode == 1 else (K, N))
    C0 = synth.normal(31, 3, (M, N))
    ref = (A.astype(np.float64).T if mode == 2 else A.astype(np.float64)) @ (B.astype(np.float64).T if mode == 1 else B.astype(np.float64))
    Ad, Bd, Rd = to_dev(A, "fp32"), to_dev(B, "fp32"), to_dev(C0, "fp32")
    if mode == 2:
        Cd = Rd.clone()
        rc = L().stage_kernel_gemm(0, 2, M, N, K, P(Ad), M, P(Bd), N, P(Cd), N, None, 0, 1, shape, None)
    else:
        Cd = torch.full((M, N), float("nan"), device="cuda:0")
        rc = L().stage_kernel_gemm(0, mode, M, N, K, P(Ad), K, P(Bd), Bd.shape[1], P(Cd), N, P(Rd), N, 0, shape, None)
    assert rc == 0
    assert so.max_rel_err(to_np(Cd), ref + C0) <= TOL


@pytest.mark.parametrize("shape", [0, 2, 3, 4])
@pytest.mark.parametrize("act", [0, 1])
@pytest.mark.parametrize("M,f,K", [(1, 4, 4), (17, 20, 36), (65, 36, 132), (130, 100, 524)])
def test_fused_activations(act, shape, M, f, K):
    """FFN-in with its activation, FFN-out's input gradient with the activation backward (da is kept in the scratch too)."""
    import torch
    fin = (1 + act) * f
    sh = so.Shape(1, 64, 1, 1, f, 1, 1, act="swiglu" if act else "gelu")
    X, W = synth.normal(32, 1, (M, K)), synth.normal(32, 2, (K, fin), std=K ** -0.5)
    dY, V = synth.normal(32, 3, (M, K)), synth.normal(32, 4, (f, K), std=K ** -0.5)
    z = X.astype(np.float64) @ W.astype(np.float64)
    a = z[:, :f] * so.sigmoid(z[:, :f]) * z[:, f:] if act else so.gelu(z)
    da = dY.astype(np.float64) @ V.astype(np.float64).T
    Zd, Aout, DA = (torch.full((M, n), float("nan"), device="cuda:0") for n in (fin, f, f))
    Xd, Wd, dYd, Vd = (to_dev(t, "fp32") for t in (X, W, dY, V))
    assert L().stage_kernel_gemm_act(0, act, M, f, K, P(Xd), K, P(Wd), fin, P(Zd), fin, P(Aout), f, shape, None) == 0
    assert so.max_rel_err(to_np(Zd), z) <= TOL and so.max_rel_err(to_np(Aout), a) <= TOL
    assert L().stage_kernel_gemm_act_bwd(0, act, M, f, K, P(dYd), K, P(Vd), K, P(Zd), fin, P(DA), shape, None) == 0
    assert so.max_rel_err(to_np(DA), da) <= TOL
    assert so.max_rel_err(to_np(Zd), so.act_backward(sh, z, da)) <= TOL


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("b,s,h,hkv,hd", [(1, 1, 1, 1, 64), (2, 16, 2, 1, 128), (1, 17, 3, 3, 64), (2, 129, 4, 2, 128), (1, 275, 6, 2, 64)])
def test_attention_against_64_bits(b, s, h, hkv, hd, causal):
    """Blocks of 16 queries and keys, eight wavefronts over them: one block, one past it, one past a full round of wavefronts."""
    import torch
    width = (h + 2 * hkv) * hd
    g = torch.Generator().manual_seed(33)
    qkv, do = torch.randn((b * s, width), generator=g), torch.randn((b * s, h * hd), generator=g)
    x = qkv.double().requires_grad_()
    outs, lses = [], []
    for t in x.split(s, 0):
        for j in range(h):
            q, k, v = (t[:, o * hd:(o + 1) * hd] for o in (j, h + j // (h // hkv), h + hkv + j // (h // hkv)))
            sc = q @ k.t() / hd ** 0.5
            if causal:
                sc = sc.masked_fill(torch.ones_like(sc, dtype=torch.bool).triu(1), -float("inf"))
            lse = torch.logsumexp(sc, -1)
            outs.append(torch.exp(sc - lse[:, None]) @ v); lses.append(lse)
    o = torch.stack([torch.cat(outs[i * h:(i + 1) * h], 1) for i in range(b)]).view(b * s, h * hd)
    o.backward(do.double())
    dev = lambda t: t.to("cuda:0")
    qkvd, dod = dev(qkv), dev(do)
    od, dqkv = torch.full_like(dod, float("nan")), torch.full_like(qkvd, float("nan"))
    lse, delta = (torch.full((b, h, s), float("nan"), device="cuda:0") for _ in range(2))
    assert L().stage_kernel_attention_fwd(0, b, s, h, hkv, hd, causal, P(qkvd), P(od), P(lse), 0, None) == 0
    assert L().stage_kernel_attention_bwd(0, b, s, h, hkv, hd, causal, P(qkvd), P(od), P(lse), P(dod), P(dqkv), P(delta), 0, None) == 0
    assert so.max_rel_err(to_np(od), o.detach().numpy()) <= TOL
    assert so.max_rel_err(to_np(lse), torch.stack(lses).view(b, h, s).detach().numpy()) <= TOL
    assert so.max_rel_err(to_np(dqkv), x.grad.numpy()) <= TOL


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("mode,M,N,K,lda,ldb", [(2, 24, 40, 50, 0, 0), (2, 64, 64, 33, 8, 16), (2, 24, 40, 50, 24, 8), (2, 24, 40, 50, -24, -40),
                                                (0, 24, 40, 64, 64, 0), (0, 24, 40, 64, 8, 8), (0, 24, 40, 64, -64, -40), (1, 24, 40, 64, 0, 64),
                                                (1, 24, 40, 64, 8, 8), (1, 24, 40, 64, -64, -64)])
def test_products_of_overlapping_rows(dtype, mode, M, N, K, lda, ldb):
    """Row strides smaller than a row (a broadcast row, a sliding window) or negative (rows in reverse): the sums of the rows written
    out.  Tolerance as above; bf16 outputs (modes 0 and 1): one rounding, 2^-8."""
    import ctypes as C
    import torch
    a_shape, b_shape = ((K, M) if mode == 2 else (M, K)), ((N, K) if mode == 1 else (K, N))
    bufs, ptrs, mats = [], [], []
    for i, (r, c), ld in ((1, a_shape, lda), (2, b_shape, ldb)):
        buf = to_dev(synth.normal(34, i, ((r - 1) * abs(ld) + c,)), dtype)
        first = (r - 1) * -ld if ld < 0 else 0                       # element at which row 0 starts
        rows = buf.as_strided((r, c), (abs(ld), 1)).double()
        bufs.append(buf); ptrs.append(P(buf) + first * buf.element_size()); mats.append(rows.flip(0) if ld < 0 else rows)
    A, B = mats
    C0 = torch.from_numpy(synth.normal(34, 3, (M, N))).to("cuda:0") if mode == 2 else torch.zeros((M, N), device="cuda:0", dtype=bufs[0].dtype)
    ref = C0.double() + (A.t() if mode == 2 else A) @ (B.t() if mode == 1 else B)
    dt, tol = {"fp32": 0, "bf16": 1}[dtype], TOL if dtype == "fp32" or mode == 2 else 2.0 ** -8
    Cd = C0.clone()
    assert L().stage_kernel_gemm(dt, mode, M, N, K, ptrs[0], lda, ptrs[1], ldb, P(Cd), N, None, 0, int(mode == 2), 0, None) == 0
    assert so.max_rel_err(to_np(Cd), ref.cpu().numpy()) <= tol
    if mode == 2:
        Cg = C0.clone()
        i1, l1, p1 = (lambda v: (C.c_int * 1)(v)), (lambda v: (C.c_int64 * 1)(v)), (lambda p: (C.c_void_p * 1)(p))
        assert L().stage_kernel_wgrad_group(dt, 1, i1(M), i1(N), i1(K), p1(ptrs[0]), l1(lda), p1(ptrs[1]), l1(ldb), p1(P(Cg)), l1(N), 0, None) == 0
        assert torch.equal(Cg, Cd)


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
@pytest.mark.parametrize("part", ["q", "k", "v", "do"])
@pytest.mark.parametrize("s,hd,causal,at", [(16, 64, 1, 9), (37, 128, 1, 20), (37, 64, 1, 36), (37, 64, 0, 36), (150, 128, 1, 0), (150, 64, 1, 141)])
def test_attention_keeps_a_position_to_those_that_see_it(part, value, s, hd, causal, at):
    """An infinity or NaN in q, k, v or dO of one position: what the plain kernels, which never read a key behind its query nor a row
    past the end, leave finite stays finite and right, and the rest is the same kind of non-finite."""
    import torch
    h, hkv = 2, 1
    g = torch.Generator().manual_seed(35)
    qkv, do = torch.randn((s, (h + 2 * hkv) * hd), generator=g), torch.randn((s, h * hd), generator=g)
    if part == "do":
        do[at, hd + 3] = value
    else:
        qkv[at, {"q": hd, "k": h * hd, "v": (h + hkv) * hd}[part] + 5] = value
    qkv, do = qkv.to("cuda:0"), do.to("cuda:0")
    outs = []
    for ks in (0, 1):
        o, dqkv = torch.zeros_like(do), torch.zeros_like(qkv)
        lse, delta = (torch.zeros((h, s), device="cuda:0") for _ in range(2))
        assert L().stage_kernel_attention_fwd(0, 1, s, h, hkv, hd, causal, P(qkv), P(o), P(lse), ks, None) == 0
        assert L().stage_kernel_attention_bwd(0, 1, s, h, hkv, hd, causal, P(qkv), P(o), P(lse), P(do), P(dqkv), P(delta), ks, None) == 0
        outs.append((o, lse, delta, dqkv))
    for name, x, y in zip(("o", "lse", "delta", "dqkv"), *outs):
        assert torch.equal(torch.isnan(x), torch.isnan(y)), name
        inf = torch.isinf(y)
        assert torch.equal(torch.isinf(x), inf) and torch.equal(x[inf], y[inf]), name
        fin = torch.isfinite(y)
        if fin.any():
            assert so.max_rel_err(to_np(x[fin]), to_np(y[fin])) <= TOL, name
