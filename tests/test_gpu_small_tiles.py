"""The small tiles of the bf16 products at their edges."""
import ctypes as C
import re

import numpy as np
import pytest

from oracle import stage_oracle as so
from paper_2507_00217_amd import synth
from tests.gpu_util import SMALL, TOL, launches, rnd, to_dev, to_np
from tests.test_gpu_kernels import KTOL, L, P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (64, 64, 128), (65, 72, 448), (129, 136, 512), (200, 264, 576), (400, 1736, 1088),
                                   (24, 5720, 64), (6000, 136, 64), (4352, 4096, 64), (4600, 4096, 64)])
def test_small_tiles_agree_bitwise(mode, M, N, K):
    """64 x 64 (5), 128 x 64 (6) and 128 x 128 tiles (4) against full ones (2) and the rule (0): one row, one past a tile, reductions
    from one K tile over the ring's depth of eight to two rounds of it; products a fraction of a full tile high or wide, and last
    rounds of 16 and 32 full tiles behind a complete one, which the rule gives to 64 x 64 and 128 x 64 tiles."""
    import torch
    A, Bm = rnd(synth.normal(43, 1, (M, K)), "bf16"), rnd(synth.normal(43, 2, (N, K) if mode else (K, N)), "bf16")
    R = rnd(synth.normal(43, 3, (M, N)), "bf16")
    Ad, Bd, Rd = to_dev(A, "bf16"), to_dev(Bm, "bf16"), to_dev(R, "bf16")
    outs = []
    for ks in (2, 4, 5, 6, 0):
        Cd = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        assert L().stage_kernel_gemm(1, mode, M, N, K, P(Ad), K, P(Bd), Bd.shape[1], P(Cd), N, None if mode else P(Rd), N, 0, ks, None) == 0
        outs.append(Cd)
    ref = A.astype(np.float64) @ (Bm.astype(np.float64).T if mode else Bm.astype(np.float64)) + (0 if mode else R)
    assert so.max_rel_err(to_np(outs[0]), ref) <= KTOL["bf16"]
    assert all(torch.equal(outs[0], o) for o in outs[1:])


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_reductions_around_the_ring(mode):
    """One to 20 K tiles on small tiles whose operands other wavefronts load, four (128 x 128, 128 x 64) or eight (64 x 64) K tiles ahead: the start-up,
    the steady state and the end of the ring with every remainder, against full tiles; a ragged last K tile for weight gradients."""
    import torch
    M, N = 136, 72
    A, B = torch.randn((M, 1280), device="cuda:0").bfloat16(), torch.randn((N, 1280), device="cuda:0").bfloat16()
    for K in [64 * i for i in range(1, 21)] + ([57, 185, 313] if mode == 2 else []):
        a = A[:, :K].t().contiguous() if mode == 2 else A[:, :K].contiguous()
        b = B[:, :K].contiguous() if mode == 1 else B[:, :K].t().contiguous()
        outs = []
        for ks in (2, 4, 5, 6):
            c = torch.ones((M, N), dtype=torch.float32 if mode == 2 else torch.bfloat16, device="cuda:0")
            assert L().stage_kernel_gemm(1, mode, M, N, K, P(a), a.shape[1], P(b), b.shape[1], P(c), N, None, 0, int(mode == 2), ks, None) == 0
            outs.append(c)
        ref = A[:, :K].double() @ B[:, :K].double().t() + (1 if mode == 2 else 0)
        # one bf16 rounding of the output, or fp32 sums of K products
        assert ((outs[0].double() - ref).abs().max() / ref.abs().max()).item() <= (1e-5 * K ** 0.5 if mode == 2 else KTOL["bf16"])
        assert all(torch.equal(outs[0], o) for o in outs[1:]), K


@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (96, 64, 128), (97, 72, 192), (193, 136, 256), (129, 200, 320), (200, 392, 448), (400, 1736, 1088),
                                   (1000, 1280, 64), (1000, 5120, 192), (4096, 1536, 192)])
def test_tiles_between_the_powers_of_two(M, N, K):
    """96 x 64 (7), 192 x 128 (8) and 128 x 192 tiles (9) against full ones (2) and the rule (0), every epilogue that an entry
    point reaches with bf16 operands alone (bias, fp32 residual and fp32 output: test_stage_epilogues_between_the_powers_of_two): one row, one past a
    tile, reductions around the ring's depths of two and four; the last three shapes are what the rule gives to each of them."""
    import torch
    P0, R = P, lambda i, *sh: to_dev(rnd(synth.normal(45, i, sh, std=1.0 if i != 2 else 1.5 * K ** -0.5), "bf16"), "bf16")
    A, B, Bt, Rd, Z = R(1, M, K), R(2, K, N), R(2, N, K), R(3, M, N), R(4, M, N)
    outs = []
    for ks in (2, 7, 8, 9, 0):
        Cs = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(5)]
        dz = Z.clone()
        for c, mode, w, r in ((Cs[0], 0, B, None), (Cs[1], 0, B, Rd), (Cs[2], 1, Bt, None)):
            assert L().stage_kernel_gemm(1, mode, M, N, K, P0(A), K, P0(w), w.shape[1], P0(c), N, None if r is None else P0(r), N, 0, ks, None) == 0
        assert L().stage_kernel_gemm_act(1, 0, M, N, K, P0(A), K, P0(B), N, P0(Cs[3]), N, P0(Cs[4]), N, ks, None) == 0
        assert L().stage_kernel_gemm_act_bwd(1, 0, M, N, K, P0(A), K, P0(Bt), K, P0(dz), N, None, ks, None) == 0
        outs.append(Cs + [dz])
    ref = A.double() @ B.double()
    assert ((outs[0][0].double() - ref).abs().max() / ref.abs().max()).item() <= KTOL["bf16"]          # one bf16 rounding of the output
    for i, o in enumerate(outs[1:]):
        assert all(torch.equal(x, y) for x, y in zip(outs[0], o)), i


@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (31, 64, 128), (33, 72, 448), (64, 136, 512), (65, 56, 576), (130, 200, 1088), (512, 1024, 64), (513, 1024, 64)])
def test_tiles_of_32_rows(M, N, K):
    """32 x 64 tiles (10) against full ones (2) and the rule (0), every epilogue that an entry point reaches: one row, on either side of a tile, reductions from one
    K tile over the ring's depth of eight to two rounds of it; the last two are the largest that the rule gives to them and one past it."""
    import torch
    P0, R = P, lambda i, *sh: to_dev(rnd(synth.normal(46, i, sh, std=1.0 if i != 2 else 1.5 * K ** -0.5), "bf16"), "bf16")
    A, B, Bt, Rd, Z = R(1, M, K), R(2, K, N), R(2, N, K), R(3, M, N), R(4, M, 2 * N)
    outs = []
    for ks in (2, 10, 0):
        Cs = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(5)]
        for c, mode, w, r in ((Cs[0], 0, B, None), (Cs[1], 0, B, Rd), (Cs[2], 1, Bt, None)):
            assert L().stage_kernel_gemm(1, mode, M, N, K, P0(A), K, P0(w), w.shape[1], P0(c), N, None if r is None else P0(r), N, 0, ks, None) == 0
        assert L().stage_kernel_gemm_act(1, 0, M, N, K, P0(A), K, P0(B), N, P0(Cs[3]), N, P0(Cs[4]), N, ks, None) == 0
        dz = [Z[:, :N].contiguous().clone(), Z.clone()]      # (a single row is contiguous already)
        for act in (0, 1):
            assert L().stage_kernel_gemm_act_bwd(1, act, M, N, K, P0(A), K, P0(Bt), K, P0(dz[act]), (1 + act) * N, None, ks, None) == 0
        outs.append(Cs + dz)
    ref = A.double() @ B.double()
    assert ((outs[0][0].double() - ref).abs().max() / ref.abs().max()).item() <= KTOL["bf16"]          # one bf16 rounding of the output
    for i, o in enumerate(outs[1:]):
        assert all(torch.equal(x, y) for x, y in zip(outs[0], o)), i


@pytest.mark.parametrize("act", [0, 1])
@pytest.mark.parametrize("M,f,K", [(1, 8, 64), (127, 64, 64), (129, 72, 128), (128, 136, 320), (257, 200, 384),
                                   (1100, 72, 128), (300, 2000, 192),
                                   (1100, 1736, 64), (1100, 3000, 64), (1100, 4200, 64)])
def test_fused_activations_on_small_products(act, M, f, K):
    """The tiles that the rule picks on 256 compute units, one round of which is enough: 32 x 64 or 64 x 64 (SwiGLU forward: 128 x 64, of 32 features)
    up to (300, 2000); then 128 x 64, 128 x 128 and two 128 x 128 workgroups to a compute unit (SwiGLU forward: the last of these twice, then
    full ones; SwiGLU backward: half-height ones at the end).  One row, one past a tile in each dimension, reductions from one K tile to past the ring.  Tolerance: one
    bf16 rounding of the output and of z, as for the larger tiles."""
    import torch
    fin = (1 + act) * f
    sh = so.Shape(1, 64, 1, 1, f, 1, 1, act="swiglu" if act else "gelu")
    X, W = rnd(synth.normal(41, 1, (M, K)), "bf16"), rnd(synth.normal(41, 2, (K, fin), std=1.5 * K ** -0.5), "bf16")
    dY, V = rnd(synth.normal(41, 3, (M, K)), "bf16"), rnd(synth.normal(41, 4, (f, K), std=1.5 * K ** -0.5), "bf16")
    z = X.astype(np.float64) @ W.astype(np.float64)
    a = z[:, :f] * so.sigmoid(z[:, :f]) * z[:, f:] if act else so.gelu(z)
    Xd, Wd, dYd, Vd = (to_dev(t, "bf16") for t in (X, W, dY, V))
    Zd, Aout = (torch.full((M, n), float("nan"), dtype=torch.bfloat16, device="cuda:0") for n in (fin, f))
    assert L().stage_kernel_gemm_act(1, act, M, f, K, P(Xd), K, P(Wd), fin, P(Zd), fin, P(Aout), f, 0, None) == 0
    assert so.max_rel_err(to_np(Zd), z) <= KTOL["bf16"] and so.max_rel_err(to_np(Aout), a) <= KTOL["bf16"]
    zr = to_np(Zd)
    da = dY.astype(np.float64) @ V.astype(np.float64).T
    assert L().stage_kernel_gemm_act_bwd(1, act, M, f, K, P(dYd), K, P(Vd), K, P(Zd), fin, None, 0, None) == 0
    assert so.max_rel_err(to_np(Zd), so.act_backward(sh, zr, da)) <= KTOL["bf16"]


@pytest.mark.parametrize("act", [0, 1])
@pytest.mark.parametrize("M,f,K", [(1, 8, 64), (65, 72, 448), (129, 136, 512), (200, 264, 576), (400, 1736, 192), (1100, 3400, 64), (24, 5720, 64), (4352, 4096, 64)])
def test_fused_tiles_agree_bitwise(act, M, f, K):
    """64 x 64 (5), 128 x 64 (6) and 128 x 128 tiles (4) of the fused products, and half-height ones (3, SwiGLU backward), against full ones (2) and the rule (0):
    z, the activation and its backward, with rows and features past every tile's edge and reductions around the rings' depths;
    1100 x 3400 has more than 256 tiles of 128 x 128, which (except the SwiGLU backward's) then go out two to a compute unit; the last shape
    has a last round of 16 (SwiGLU forward: 32) full tiles."""
    import torch
    fin = (1 + act) * f
    X, W = rnd(synth.normal(44, 1, (M, K)), "bf16"), rnd(synth.normal(44, 2, (K, fin), std=1.5 * K ** -0.5), "bf16")
    dY, V = rnd(synth.normal(44, 3, (M, K)), "bf16"), rnd(synth.normal(44, 4, (f, K), std=1.5 * K ** -0.5), "bf16")
    Xd, Wd, dYd, Vd = (to_dev(t, "bf16") for t in (X, W, dY, V))
    outs = []
    for ks in (2, 3, 4, 5, 6, 0):
        Zd, Aout = (torch.full((M, n), float("nan"), dtype=torch.bfloat16, device="cuda:0") for n in (fin, f))
        assert L().stage_kernel_gemm_act(1, act, M, f, K, P(Xd), K, P(Wd), fin, P(Zd), fin, P(Aout), f, ks, None) == 0
        z = Zd.clone()
        assert L().stage_kernel_gemm_act_bwd(1, act, M, f, K, P(dYd), K, P(Vd), K, P(Zd), fin, None, ks, None) == 0
        outs.append((z, Aout, Zd))
    assert not any(bool(torch.isnan(o).any()) for o in outs[0])
    for o in outs[1:]:
        assert all(torch.equal(x, y) for x, y in zip(outs[0], o))


@pytest.mark.parametrize("kernel_set", [0, 2])
def test_fused_gelu_is_the_plain_gelu(kernel_set):
    """Every finite bf16 value through the fused GELU epilogues (products with the identity, so the accumulators hold the value itself, and
    with da = 1): the same bits as the plain activation kernels, which evaluate 0.5 u (1 + erf(u / sqrt 2)) and its derivative."""
    import torch
    u = (torch.arange(65536, dtype=torch.int32) << 16).view(torch.float32)
    u = torch.where(torch.isfinite(u), u, torch.zeros_like(u)).view(1024, 64).bfloat16().to("cuda:0")
    eye = torch.eye(64, device="cuda:0").bfloat16()
    one = torch.ones((1024, 64), device="cuda:0").bfloat16()
    outs = []
    for ks in (kernel_set, 1):
        Z, A = torch.empty_like(u), torch.empty_like(u)
        assert L().stage_kernel_gemm_act(1, 0, 1024, 64, 64, P(u), 64, P(eye), 64, P(Z), 64, P(A), 64, ks, None) == 0
        assert torch.equal(Z, u)
        da = torch.empty_like(u)
        assert L().stage_kernel_gemm_act_bwd(1, 0, 1024, 64, 64, P(one), 64, P(eye), 64, P(Z), 64, P(da), ks, None) == 0
        outs.append((A.view(torch.int16), Z.view(torch.int16)))
    for x, y in zip(*outs):
        assert torch.equal(x, y), "%d of 65536 differ" % int((x != y).sum())


# full tiles of the lists: 1, 1, 7, 256 + 35, 48, 90, 256 + 54, 151
@pytest.mark.parametrize("shapes", [[(8, 8, 1)], [(128, 136, 65)], [(264, 520, 200), (136, 8, 64)],
                                    [(4096, 4096, 72), (2560, 264, 320), (520, 1032, 129)],
                                    [(1800, 1288, 520)], [(2056, 2312, 584)], [(4096, 4096, 64), (1288, 2056, 600)],
                                    [(2048, 4104, 40), (1032, 520, 136)]])      # 151 tiles: more than half a round, full tiles
def test_weight_gradients_of_a_short_last_round(shapes):
    """Lists whose last round keeps at most half of the CUs busy go out (partly) in smaller tiles: 64 x 64 (reductions of at most 512, or at most 32
    tiles), 128 x 128 with a deep ring (at most 64 tiles) or two to a compute unit.  The same bits as full tiles, whether the
    rule picks the tiles (0) or they are forced on the whole list (4, 5)."""
    import torch
    n = len(shapes)
    g = torch.Generator().manual_seed(42)
    A, B, Cs = [], [], []
    for M, N, K in shapes:
        A.append(torch.randn((K, M), generator=g).bfloat16().to("cuda:0")); B.append(torch.randn((K, N), generator=g).bfloat16().to("cuda:0"))
        Cs.append(torch.randn((M, N), generator=g).to("cuda:0"))
    Ms, Ns, Ks = zip(*shapes)
    ia, la, pa = (lambda v: (C.c_int * n)(*v)), (lambda v: (C.c_int64 * n)(*v)), (lambda t: (C.c_void_p * n)(*[u.data_ptr() for u in t]))

    def run(ks):
        out = [c.clone() for c in Cs]
        assert L().stage_kernel_wgrad_group(1, n, ia(Ms), ia(Ns), ia(Ks), pa(A), la(Ms), pa(B), la(Ns), pa(out), la(Ns), ks, None) == 0
        return out
    full = run(2)
    for (M, N, K), a, b, c, got in zip(shapes, A, B, Cs, full):
        ref = c.double() + a.double().t() @ b.double()
        assert ((got.double() - ref).abs().max() / ref.abs().max()).item() <= 1e-5 * max(1.0, K ** 0.5)
        one = c.clone()
        assert L().stage_kernel_gemm(1, 2, M, N, K, P(a), M, P(b), N, P(one), N, None, 0, 1, 2, None) == 0
        assert torch.equal(one, got)
    for ks in (0, 4, 5):
        assert all(torch.equal(x, y) for x, y in zip(run(ks), full)), ks


@pytest.mark.parametrize("hidden,ffn", [(512, 1408), (768, 2048)])
def test_merged_weight_gradients_in_small_tiles(hidden, ffn):
    """W ops at the end of the list reduce over all microbatches in one pass: 3 x 300 tokens in 40 (128 x 128 tiles, deep ring) and 84
    full tiles (two to a compute unit), the same bits as W right behind each B, whose reductions of 300 take 64 x 64 tiles."""
    import torch
    from paper_2507_00217_amd import stage as S
    cfg = dict(n_layers=1, hidden=hidden, n_heads=hidden // 128, n_kv_heads=hidden // 128, head_dim=128, ffn=ffn, seq=300, mb_size=1, n_microbatches=3,
               norm="layernorm", act="gelu", dtype="bf16", stash_cap=3, enforce_mb_order=1)
    params, X, G = synth.make_weights(cfg, 71), synth.make_boundary(cfg, 72), synth.make_boundary(cfg, 73)
    grads = []
    for ops in ([(o, m) for m in range(3) for o in (0, 1, 2)], [(o, m) for m in range(3) for o in (0, 1)] + [(2, m) for m in range(3)]):
        st = S.Stage(cfg)
        st.load_weights(params)
        Xd, Gd = to_dev(X, "bf16"), to_dev(G, "bf16")
        st.run_schedule(ops, Xd, Gd, torch.zeros_like(Xd), torch.zeros_like(Xd))
        torch.cuda.synchronize()
        grads.append(st.grads())
        st.close()
    for a, b in zip(*grads):
        assert all(np.array_equal(a[k], b[k]) for k in a)


@pytest.mark.parametrize("M,N,K,paced", [(65, 8000, 5248, True), (104, 8000, 5248, True), (105, 8000, 5248, False), (65, 8000, 5184, False), (129, 5120, 8256, True)])
@pytest.mark.parametrize("form", ["forward", "residual", "input gradient"])
def test_last_tile_row_keeps_pace(form, M, N, K, paced):
    """64 x 64 tiles over a B of more than 80 MiB with 1 to 40 rows in the last row of tiles: the wavefronts that multiply load as well (four per
    workgroup, not eight), with the bits of the other form; on either side of the lines."""
    import torch
    torch.manual_seed(47)
    A, B = torch.randn((M, K), device="cuda:0").bfloat16(), torch.randn((N, K) if form == "input gradient" else (K, N), device="cuda:0").bfloat16()
    R = torch.randn((M, N), device="cuda:0").bfloat16() if form == "residual" else None
    outs = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(2)]

    def run(out, ks, stream=None):
        return L().stage_kernel_gemm(1, int(form == "input gradient"), M, N, K, P(A), K, P(B), B.shape[1], P(out), N, None if R is None else P(R), N, 0, ks, stream)
    for o, ks in zip(outs, (0, 5)):
        assert run(o, ks) == 0
    assert torch.equal(outs[0], outs[1])
    (name, _, threads), = launches(lambda stream: run(outs[0], 0, stream))
    assert "gemm_tiny_kernel" in name and threads == (256 if paced else 512)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("M,N", [(1000, 5120), (4096, 1536)])
def test_short_reductions_with_a_plain_store(mode, M, N):
    """192 x 128 and 128 x 192 tiles from 192 terms on; below, two 128 x 128 workgroups to a compute unit.  With a residual at any length."""
    import torch
    for K in (64, 128, 192):
        A, B, R = (torch.randn(sh, device="cuda:0").bfloat16() for sh in ((M, K), (N, K) if mode else (K, N), (M, N)))
        outs = [torch.empty((M, N), dtype=torch.bfloat16, device="cuda:0") for _ in range(2)]

        def run(out, ks, stream=None, res=None):
            return L().stage_kernel_gemm(1, mode, M, N, K, P(A), K, P(B), B.shape[1], P(out), N, res, N, 0, ks, stream)
        for o, ks in zip(outs, (0, 2)):
            assert run(o, ks) == 0
        assert torch.equal(outs[0], outs[1])
        (name, _, _), = launches(lambda stream: run(outs[0], 0, stream))
        assert ("gemm_mid_kernel" if K >= 192 else "gemm_quarter_kernel") in name
        if mode == 0:
            (name, _, _), = launches(lambda stream: run(outs[0], 0, stream, P(R)))
            assert "gemm_mid_kernel" in name


@pytest.mark.parametrize("M,N,K", [(400, 1736, 1088), (1100, 2048, 128), (2048, 4096, 256)])
def test_shapes_that_a_product_lacks_leave_the_rule(M, N, K):
    """kernel_set 7 to 10 where there is no such tile: the kernels of kernel_set 0 (captures: nothing runs)."""
    import torch
    t = P(torch.zeros(256, dtype=torch.uint8, device="cuda:0"))
    ints, longs, ptrs = (C.c_int * 1), (C.c_int64 * 1), (C.c_void_p * 1)
    calls = {
        "weight gradient": lambda ks, s: L().stage_kernel_gemm(1, 2, M, N, K, t, M, t, N, t, N, None, 0, 1, ks, s),
        "weight gradients": lambda ks, s: L().stage_kernel_wgrad_group(1, 1, ints(M), ints(N), ints(K), ptrs(t), longs(M), ptrs(t), longs(N), ptrs(t), longs(N), ks, s),
        "SwiGLU": lambda ks, s: L().stage_kernel_gemm_act(1, 1, M, N, K, t, K, t, 2 * N, t, 2 * N, t, N, ks, s),
        "SwiGLU backward": lambda ks, s: L().stage_kernel_gemm_act_bwd(1, 1, M, N, K, t, K, t, K, t, 2 * N, None, ks, s),
    }
    for name, call in calls.items():
        for ks in (7, 8, 9) if name == "SwiGLU backward" else (7, 8, 9, 10):
            assert launches(lambda s: call(ks, s)) == launches(lambda s: call(0, s)), (name, ks)


@pytest.mark.parametrize("T,mb,hidden,ffn,tiles", [(1000, 2, 1280, 5120, {(1280, 1280): 0, (1280, 5120): 0, (5120, 1280): 1}), (4096, 8, 1536, 512, {(1536, 1536): 2}),
                                                   (2016, 4, 2560, 512, {(2560, 2560): 1})])
def test_stage_epilogues_between_the_powers_of_two(T, mb, hidden, ffn, tiles):
    """Bias, fp32 residual and fp32 output on 96 x 64 (0), 192 x 128 (1) and 128 x 192 tiles (2), which only a stage asks for: one GPT-style layer with
    biases against the oracle, whose products of (outputs, reduction) over T tokens the rule gives to those tiles."""
    import torch
    from tests.test_gpu_stage import compare, inputs, run_gpu, run_oracle
    for (N, K), shape in tiles.items():
        t = P(torch.zeros(256, dtype=torch.uint8, device="cuda:0"))
        # (a residual gives the tiles of both residual products; the product with GELU is launched by its own entry)
        call = (lambda s: L().stage_kernel_gemm_act(1, 0, T, N, K, t, K, t, N, t, N, t, N, 0, s)) if N == ffn else \
               (lambda s: L().stage_kernel_gemm(1, 0, T, N, K, t, K, t, N, t, N, t, N, 0, 0, s))
        (name, _, _), = launches(call)
        assert re.search(rf"gemm_mid_kernelILb0ELi\d+ELi{shape}E", name), name
    cfg = dict(SMALL["cfg4s"], n_layers=1, hidden=hidden, n_heads=hidden // 128, n_kv_heads=hidden // 128, ffn=ffn, mb_size=mb, seq=T // mb, n_microbatches=1,
               stash_cap=1, bias=1, norm="layernorm", act="gelu")
    params, X, G = inputs(cfg, 4600)
    ops = [(0, 0), (1, 0), (2, 0)]
    compare(cfg, run_gpu(cfg, params, X, G, ops), run_oracle(cfg, params, X, G, ops), TOL["bf16"])


@pytest.mark.parametrize("M,N,K,loaders", [(2048, 2048, 1536, False), (2048, 2048, 1600, True), (1900, 2000, 256, False), (4864, 4096, 64, True)])
def test_short_reductions_of_the_gelu_backward(M, N, K, loaders):
    """Whole products in 128 x 128 tiles up to 1536 terms without wavefronts that only load (256 threads, not 512), a last round with them; the
    bits of full tiles."""
    import torch
    torch.manual_seed(48)
    dY, W, Z = (torch.randn(sh, device="cuda:0").bfloat16() for sh in ((M, K), (N, K), (M, N)))

    def run(z, ks, stream=None):
        return L().stage_kernel_gemm_act_bwd(1, 0, M, N, K, P(dY), K, P(W), K, P(z), N, None, ks, stream)
    outs = [Z.clone() for _ in range(3)]
    for z, ks in zip(outs, (0, 2, 4)):
        assert run(z, ks) == 0
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    name, _, threads = launches(lambda stream: run(outs[0], 0, stream))[-1]
    assert "gemm_quarter_kernel" in name and threads == (512 if loaders else 256)
