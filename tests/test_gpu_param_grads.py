"""Row-wise kernels and the parameter gradients summed behind them, at the sizes where their shape changes."""
import numpy as np
import pytest

from oracle import stage_oracle as so
from paper_2507_00217_amd import synth
from tests.gpu_util import SMALL, rnd, to_dev, to_np
from tests.test_gpu_kernels import DT, KTOL, L, P

pytestmark = pytest.mark.gpu
F, B, W = 0, 1, 2


# bf16 widths: one wavefront with 4 / 3 rows side by side, two with 2, three (one row), five, eight; fp32 twice the pieces.  Rows:
# one, fewer than the row groups, one past a full round of 512 workgroups
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("norm", ["layernorm", "rmsnorm"])
@pytest.mark.parametrize("rows,d", [(1, 8), (3, 512), (5, 520), (513, 1032), (2049, 264), (1025, 2056), (515, 2560), (2, 4096),
                                    (2561, 512), (1281, 1032), (768, 2568)])      # ten, five and three rows side by side, 80 KiB of column sums
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
