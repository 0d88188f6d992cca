"""Networks on hidden states at the edges of their tiling: groups of 16 output units, batches of 64 columns, column splits of narrow
layers, four rows per workgroup, stop flags settled in the launch (up to 256 rows) or by a second one."""
import numpy as np
import pytest
import torch

from workloads import mlp_weights

pytestmark = pytest.mark.gpu


def _reference(ws, bs, x):
    for l, (w, b) in enumerate(zip(ws, bs)):
        x = x @ w.astype(np.float64).T + b
        if l + 1 < len(ws):
            x = np.maximum(x, 0.0)
    return 1.0 / (1.0 + np.exp(-x[..., 0]))


@pytest.mark.parametrize("B,W", [(1, 1), (1, 5), (16, 16), (13, 20)])
@pytest.mark.parametrize("widths", [(4, 1), (60, 15, 1), (64, 16, 20, 1), (68, 17, 64, 1), (252, 20, 33, 1), (256, 64, 512, 1), (260, 65, 1),
                                    (1000, 129, 16, 1), (2048, 512, 65, 1), (2048, 128, 1), (320, 48, 7, 1), (576, 1, 1, 1)])
def test_layer_and_row_edges(widths, B, W):
    from paper_2409_10644_amd import binding
    rng = np.random.default_rng(sum(widths) + B)
    ws, bs = mlp_weights(widths, seed=len(widths) + widths[0])
    x = rng.standard_normal((B, W, widths[0])).astype(np.float32)
    mlp = binding.make_mlp([torch.from_numpy(w).cuda() for w in ws], [torch.from_numpy(b).cuda() for b in bs])
    d = torch.from_numpy(x).cuda()
    want = _reference(ws, bs, x.astype(np.float64))
    beta = float(np.float32(np.median(want)))
    for _ in range(2):
        prob = torch.full((B, W), -7.0, device="cuda")
        stop = torch.full((B,), -7, dtype=torch.int32, device="cuda")
        binding.early_stop_hidden(mlp, B, W, d, W * widths[0], widths[0], beta, prob, stop)
        got = prob.cpu().numpy()
        # a logit of magnitude up to ~10 from at most 2048 + 512 fp32 products in sums of depth < 100: below 1e-5 of a probability
        assert np.abs(got - want).max() <= 1e-5
        assert np.array_equal(stop.cpu().numpy(), (got < np.float32(beta)).all(axis=1).astype(np.int32))
