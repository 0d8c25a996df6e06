"""The surrogate kernels at the edges of their tiles: sample counts around the
training tile, the sliced weight gradients and the query tiles, with odd
member counts; against the FP64 reference network (the bars of
test_gpu_mlp.py for FP32 models)."""
import numpy as np
import pytest

import workloads as W
from oracle import mlp

from test_gpu_mlp import gpu, make_norm, ref_forward, setup  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 31, 32, 33, 355, 356, 515, 2051])
def test_fp32_gradient_at_tile_edges(gpu, n):  # noqa: F811
    import torch
    members = 3
    model, X, t, norm, params = setup(gpu, members, n, seed=n, precision=gpu.IT_MLP_FP32)
    grad, loss = gpu.it_mlp_grad(model, members, torch.tensor(X, device="cuda"), torch.tensor(t, device="cuda"))
    g = grad.cpu().numpy()
    _, Z = ref_forward(params, X, norm, members, cast=False)
    ts = (t.astype(np.float64) - float(norm[24])) / float(norm[25])
    for m in range(members):
        rl, rg = mlp.loss_and_grad(params[m].astype(np.float64), Z, ts, cast=False)
        assert loss[m] == pytest.approx(rl, rel=1e-5)
        off = 0
        for name, shape in mlp.SIZES:
            k = int(np.prod(shape))
            a, b = g[m, off:off + k], rg[off:off + k]
            assert np.linalg.norm(a - b) <= 1e-4 * np.linalg.norm(b) + 1e-8, (m, name)
            off += k


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("n", [1, 15, 17, 64, 1024, 1025, 8192, 8193, 64 * 4096 + 65])
def test_query_at_tile_edges(gpu, n, precision):  # noqa: F811
    """Answers and flagged indices on both sides of the rules that choose the
    tile and the compaction; some queries leave the box."""
    import torch
    prec = gpu.IT_MLP_FP32 if precision == "fp32" else gpu.IT_MLP_BF16
    model, X, t, norm, params = setup(gpu, 3, 512, precision=prec)
    Q = np.resize(X, (n, 6)).copy()
    Q[::7, 2] *= 100.0
    mean, spread, fb, idx, cnt = gpu.it_mlp_query(model, torch.tensor(Q, device="cuda"), 1e30)
    flags = np.arange(n) % 7 == 0
    assert np.array_equal(fb.cpu().numpy().astype(bool), flags)
    assert cnt == flags.sum() and np.array_equal(idx.cpu().numpy()[:cnt], np.nonzero(flags)[0])
    if precision == "fp32":
        k = min(n, 2000)
        ys, _ = ref_forward(params, Q[-k:], norm, 3, cast=False)
        ref = ys.mean(axis=0)
        assert np.max(np.abs(mean.cpu().numpy()[-k:] - ref) / (1 + np.abs(ref))) < 2e-5


@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_an_answer_does_not_depend_on_the_call(gpu, precision):  # noqa: F811
    """The same queries in calls of other sizes (other tiles), and alone, have
    the same answers bit for bit, with the analytic baseline in them."""
    import torch
    from paper_1610_06749_amd import surrogate
    X = W.surrogate_inputs(5, 9000).astype(np.float32)
    X[::2, [0, 4]] *= np.float32(1e-7)  # a baseline of 1e-8, which shows the order of its sums
    norm = make_norm(X.astype(np.float64), np.linspace(0.0, 1e-3, 9000))
    prec = gpu.IT_MLP_FP32 if precision == "fp32" else gpu.IT_MLP_BF16
    Q = torch.tensor(X, device="cuda")
    norm[24] = 0.0
    for t_sigma in (1e-30, 0.1):  # the baseline alone, and the network with it
        norm[25] = t_sigma
        model = torch.empty(gpu.it_mlp_model_bytes(3), dtype=torch.uint8, device="cuda")
        gpu.it_mlp_init(model, 3, W.mlp_init(7, 3), norm, phys=surrogate.phys_constants(), precision=prec)
        mean, spread, fb, _, _ = gpu.it_mlp_query(model, Q, 1e-3)
        for first, n in ((0, 8192), (8000, 1000), (17, 100), (8999, 1)):
            few = gpu.it_mlp_query(model, Q[first:first + n].contiguous(), 1e-3)
            for a, b in zip(few[:3], (mean, spread, fb)):
                assert torch.equal(a, b[first:first + n]), (t_sigma, first, n)


@pytest.mark.parametrize("n", [16, 61, 64, 65, 128, 129, 499, 500, 513, 628, 629, 1000])
def test_fp32_gradient_at_group_edges(gpu, n):  # noqa: F811
    """Samples around the groups in flight: 64 where a block adds the slices,
    512 and then 128 where each block has its own."""
    test_fp32_gradient_at_tile_edges(gpu, n)
