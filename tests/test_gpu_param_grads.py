"""Row-wise kernels and the parameter gradients summed behind them, at the sizes where their shape changes."""
import numpy as np
import pytest

from oracle import stage_oracle as so
from paper_2507_00217_amd import synth
from tests.gpu_util import SMALL, rnd, to_dev, to_np
from tests.test_gpu_kernels import DT, KTOL, L, P

pytestmark = pytest.mark.gpu
F, B, W = 0, 1, 2


# bf16 widths of one to four wavefronts with up to eight rows side by side, two and more pieces per thread (one row); fp32 twice the
# pieces.  Rows: one, fewer than the row groups, one past a full round of the workgroups
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("norm", ["layernorm", "rmsnorm"])
@pytest.mark.parametrize("rows,d", [(1, 8), (3, 512), (5, 520), (513, 1032), (2049, 264), (1025, 2056), (515, 2560), (2, 4096),
                                    (2561, 512), (1281, 1032), (768, 2568), (514, 2048), (130, 64)])      # two to eight rows side by side, 32 KiB of column sums
def test_norm_backward_row_shapes(dtype, norm, rows, d):
    import torch
    kind = {"layernorm": 0, "rmsnorm": 1}[norm]
    x, dout, resid = (rnd(synth.normal(51, i, (rows, d)), dtype) for i in (1, 2, 3))
    gamma = rnd(synth.normal(51, 4, (d,), mean=1.0, std=0.1), dtype)
    _, stats = so.norm_forward(norm, x.astype(np.float64), gamma.astype(np.float64), np.zeros(d), 1e-5)
    dx_ref, dg_ref, db_ref = so.norm_backward(norm, stats, gamma.astype(np.float64), dout.astype(np.float64))
    mu = x.astype(np.float64).mean(1, keepdims=True) if norm == "layernorm" else np.zeros((rows, 1))
    st = to_dev(np.concatenate([mu, stats[1]], 1), "fp32")
    xd, gd, dd, rd = to_dev(x, dtype), to_dev(gamma, dtype), to_dev(dout, dtype), to_dev(resid, dtype)
    dg, db = torch.zeros(d, device="cuda:0"), torch.zeros(d, device="cuda:0")
    part = torch.full((L().stage_kernel_norm_partial_bytes(d) // 4,), float("nan"), device="cuda:0")      # only what is written is read
    assert L().stage_kernel_norm_bwd(DT[dtype], kind, rows, d, P(xd), P(st), P(gd), P(dd), P(rd), P(xd), P(dg), P(db), P(part), None) == 0
    assert so.max_rel_err(to_np(xd), dx_ref + resid) <= KTOL[dtype]
    # fp32 sums of `rows` products of exact bf16 / fp32 inputs; xhat itself is off by eps * |mean| / std of the row
    assert so.max_rel_err(to_np(dg), dg_ref) <= 2e-5
    if norm == "layernorm":
        assert so.max_rel_err(to_np(db), db_ref) <= 1e-5


@pytest.mark.parametrize("rows", [3, 700])
@pytest.mark.parametrize("d", [64, 520, 1024, 2052, 3000, 4096])
def test_norm_backward_row_sum_order(rows, d):
    """dx from a row sum taken in one order whatever shape the workgroups have: 256 threads of 4 elements at a time, one running sum each, a
    butterfly over 64 threads, then the four 64s.  Emulated in fp32; a sum in another order changes a tenth of the elements, the
    emulation itself (fused multiply-adds rounded twice) next to none."""
    import torch
    f32 = np.float32
    fma = lambda a, b, c: (a.astype(np.float64) * b + c).astype(f32)
    x, dout = synth.normal(52, 1, (rows, d)), synth.normal(52, 2, (rows, d))
    gamma = synth.normal(52, 3, (d,), mean=1.0, std=0.1)
    rstd = (1.0 / np.sqrt((x.astype(np.float64) ** 2).mean(1, keepdims=True) + 1e-5)).astype(f32)
    xhat, dxhat = x * rstd, dout * gamma
    pad = lambda v: np.pad(v, ((0, 0), (0, 4096 - d))).reshape(rows, 4, 256, 4)
    px, pd, s = pad(xhat), pad(dxhat), np.zeros((rows, 256), f32)
    for c in range(4):
        for e in range(4):
            s = fma(pd[:, c, :, e], px[:, c, :, e], s)
    s = s.reshape(rows, 4, 64)
    for o in (32, 16, 8, 4, 2, 1):
        s = s + s[:, :, np.arange(64) ^ o]
    tot = ((s[:, 0, 0] + s[:, 1, 0]) + s[:, 2, 0]) + s[:, 3, 0]
    m2 = (tot * f32(1.0 / d))[:, None]
    ref = fma(-xhat, m2, dxhat) * rstd
    xd, dd, gd = (torch.from_numpy(v).to("cuda:0") for v in (x, dout, gamma))
    st = torch.from_numpy(np.concatenate([np.zeros_like(rstd), rstd], 1)).to("cuda:0")
    dx, dg = torch.empty_like(xd), torch.zeros(d, device="cuda:0")
    part = torch.empty(L().stage_kernel_norm_partial_bytes(d) // 4, device="cuda:0")
    assert L().stage_kernel_norm_bwd(0, 1, rows, d, P(xd), P(st), P(gd), P(dd), None, P(dx), P(dg), None, P(part), None) == 0
    assert np.mean(dx.cpu().numpy() != ref) <= 1e-3


def test_unaligned_gradient_input():
    """A dY 8 bytes past a 16-byte boundary: the same bits as the aligned one."""
    import torch
    from paper_2507_00217_amd import stage as S
    cfg = dict(SMALL["cfg2s"], n_microbatches=1, stash_cap=1, enforce_mb_order=1, bias=1)
    params, X, G = synth.make_weights(cfg, 61), synth.make_boundary(cfg, 62), synth.make_boundary(cfg, 63)
    outs = []
    for shift in (0, 4):
        st = S.Stage(cfg)
        st.load_weights(params)
        Xd, Gd = to_dev(X, "bf16"), to_dev(G, "bf16")
        buf = torch.zeros(Gd.numel() + 8, dtype=torch.bfloat16, device="cuda:0")
        dy = buf[shift:shift + Gd.numel()].view(Gd.shape)
        dy.copy_(Gd)
        Y, dX = torch.zeros_like(Xd), torch.zeros_like(Xd)
        st.run_schedule([(F, 0), (B, 0), (W, 0)], Xd, dy, Y, dX)
        torch.cuda.synchronize()
        outs.append((to_np(dX), st.grads()))
        st.close()
    assert np.array_equal(outs[0][0], outs[1][0])
    for a, b in zip(outs[0][1], outs[1][1]):
        assert all(np.array_equal(a[k], b[k]) for k in a)
