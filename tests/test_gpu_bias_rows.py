"""Bias gradients on both sides of the row count up to which one launch sums the gradient rows directly.  Needs a GPU."""
import numpy as np
import pytest

from tests import test_gpu_kernels as T
from tests.gpu_util import SMALL, launches, rnd, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("rows,n,ld", [(1, 8, 8), (127, 64, 64), (129, 72, 80), (511, 200, 200), (513, 136, 136), (1023, 64, 72),
                                       (1025, 1000, 1000), (2047, 192, 192), (2048, 328, 336), (2049, 328, 336), (2048, 320, 320), (2049, 320, 320)])
def test_direct_and_two_step_sums(dtype, rows, n, ld):
    """Edges of the rows in flight (512 / 1024 per step), of the 64 columns of a workgroup, and of the rule; dbias is added to.

    Tolerance: the longest chain of fp32 additions is at most rows / 128 * 2 + 40 in either form, so the error is at most that
    many half-ulps (2^-24) of the sum of magnitudes."""
    import torch
    lib = T.L()
    x = rnd(np.random.default_rng(rows + n).standard_normal((rows, ld)), dtype)
    start = np.linspace(-1, 1, n, dtype=np.float32)
    xd, db = to_dev(x, dtype), torch.from_numpy(start).to("cuda:0")
    scr = torch.zeros(lib.stage_kernel_bias_grad_scratch_bytes(n) // 4, dtype=torch.float32, device="cuda:0")
    assert lib.stage_kernel_bias_grad(T.DT[dtype], rows, n, T.P(xd), ld, T.P(db), T.P(scr), None) == 0
    torch.cuda.synchronize()
    ref = start.astype(np.float64) + x[:, :n].astype(np.float64).sum(0)
    bound = (rows / 128 * 2 + 40) * 2.0 ** -24 * (np.abs(x[:, :n]).astype(np.float64).sum(0) + np.abs(start))
    assert np.all(np.abs(to_np(db) - ref) <= bound)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("rows,n,ld,kernels", [(1024, 328, 336, 1), (1025, 328, 336, 2), (2048, 320, 320, 1), (2049, 320, 320, 2),
                                               (2048, 16384, 16384, 1), (1024, 16448, 16448, 1), (1025, 16448, 16448, 2), (512, 8200, 8200, 1),
                                               (513, 8200, 8200, 2)])
def test_launches_on_either_side_of_the_line(dtype, rows, n, ld, kernels):
    """One launch up to 2048 rows on 128-byte lines and 16384 columns, up to 1024 of others, 512 of more than 8192 columns off the lines (a capture: nothing runs)."""
    import torch
    t = torch.zeros(4096, dtype=torch.uint8, device="cuda:0")
    got = launches(lambda s: T.L().stage_kernel_bias_grad(T.DT[dtype], rows, n, T.P(t), ld, T.P(t), T.P(t), s))
    assert len(got) == kernels


@pytest.mark.parametrize("seq", [200, 2056])
def test_profile_counts_bias_gradients_with_the_copies(seq):
    """One launch or two, the bytes of the bias gradients are not the norms'."""
    import torch
    from paper_2507_00217_amd import stage as S
    from paper_2507_00217_amd import synth
    cfg, prof = dict(SMALL["cfg4s"], n_layers=1, seq=seq, n_microbatches=2, stash_cap=0, norm="layernorm", act="gelu"), {}
    ops = synth.schedule_1f1b(2, 1)
    for b in (0, 1):
        c = dict(cfg, bias=b)
        X = to_dev(synth.make_boundary(c, 8), c["dtype"])
        st = S.Stage(c)
        st.load_weights(synth.make_weights(c, 7))
        st.profile(True)
        st.run_schedule(ops, X, X.clone(), torch.zeros_like(X), torch.zeros_like(X))
        prof[b] = st.profile_read()
        st.close()
    rows, dq = cfg["mb_size"] * seq, cfg["hidden"] // cfg["n_heads"] * (cfg["n_heads"] + 2 * cfg["n_kv_heads"])
    assert prof[1]["norm_bwd"]["work"] == prof[0]["norm_bwd"]["work"] > 0
    assert prof[1]["copy"]["work"] - prof[0]["copy"]["work"] == 2 * rows * (2 * cfg["hidden"] + cfg["ffn"] + dq) * 2
