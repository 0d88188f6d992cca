"""Networks on hidden states at the edges of their tiling: groups of 16 output units, batches of 64 columns, column splits of narrow
layers, four rows per workgroup, stop flags settled in the launch (up to 160 rows) or by a second one.  The threshold lies
between the trees' largest probabilities, so that some trees stop and some do not, and the flags are right whatever the
probabilities were before: all below the threshold, or all above it."""
import numpy as np
import pytest
import torch

from workloads import mlp_weights

pytestmark = pytest.mark.gpu

WIDTHS = [(4, 1), (60, 15, 1), (64, 16, 20, 1), (68, 17, 64, 1), (252, 20, 33, 1), (256, 64, 512, 1), (260, 65, 1), (1000, 129, 16, 1),
          (2048, 512, 65, 1), (2048, 128, 1), (320, 48, 7, 1), (576, 1, 1, 1)]
# one tree, a few, as many rows as are settled in the launch, the next ones, 256; trees of four rows per workgroup and across them
TREES = [(1, 1), (1, 5), (7, 6), (26, 6), (8, 20), (32, 5), (33, 5), (41, 4), (16, 16), (13, 20)]


def _reference(ws, bs, x):
    for l, (w, b) in enumerate(zip(ws, bs)):
        x = x @ w.astype(np.float64).T + b
        if l + 1 < len(ws):
            x = np.maximum(x, 0.0)
    return 1.0 / (1.0 + np.exp(-x[..., 0]))


def _case(widths, B, W):
    """Weights, inputs, probabilities, and a threshold in the middle of the widest gap between the trees' largest probabilities;
    one above and one below them all where there is one tree, or a clipped unit makes them equal."""
    rng = np.random.default_rng(sum(widths) + B)
    ws, bs = mlp_weights(widths, seed=len(widths) + widths[0])
    x = rng.standard_normal((B, W, widths[0])).astype(np.float32)
    want = _reference(ws, bs, x.astype(np.float64))
    top = np.sort(want.max(axis=1))
    if top[-1] - top[0] < 1e-4:
        betas = [float(top[-1]) + 0.01, float(top[0]) - 0.01]
    else:
        k = int(np.argmax(np.diff(top)))
        betas = [float(top[k] + top[k + 1]) / 2]
    flags = [(want < beta).all(axis=1) for beta in betas]
    assert np.any(flags) and not np.all(flags)              # of both kinds, and not where fp32 and binary64 might differ
    assert min(np.abs(want.max(axis=1) - beta).min() for beta in betas) > 2e-5
    return ws, bs, x, want, list(zip(betas, flags))


@pytest.mark.parametrize("B,W", TREES)
@pytest.mark.parametrize("widths", WIDTHS)
def test_layer_and_row_edges(widths, B, W):
    from paper_2409_10644_amd import binding
    ws, bs, x, want, thresholds = _case(widths, B, W)
    mlp = binding.make_mlp([torch.from_numpy(w).cuda() for w in ws], [torch.from_numpy(b).cuda() for b in bs])
    d = torch.from_numpy(x).cuda()
    for beta, flags in thresholds:
        for before in (-7.0, 2.0):
            prob = torch.full((B, W), before, device="cuda")
            stop = torch.full((B,), -7, dtype=torch.int32, device="cuda")
            binding.early_stop_hidden(mlp, B, W, d, W * widths[0], widths[0], beta, prob, stop)
            got = prob.cpu().numpy()
            # a logit of magnitude up to ~10 from at most 2048 + 512 fp32 products in sums of depth < 100: below 1e-5 of a probability
            assert np.abs(got - want).max() <= 1e-5
            assert np.array_equal(stop.cpu().numpy(), flags.astype(np.int32)), (beta, before)


def _sums_in_order(w, x, chains):
    """fp32 sums in the order of the kernel, of the first 16 columns of each batch of 64: four columns one after the other, a tree
    of four such sums, batch after batch in `chains` alternating sums."""
    acc = np.zeros((chains, x.shape[0]), np.float32)
    for t in range(x.shape[1] // 64):
        a = np.zeros((4, x.shape[0]), np.float32)
        for c in range(4):
            for col in range(64 * t + 4 * c, 64 * t + 4 * c + 4):
                a[c] = (x[:, col].astype(np.float64) * w[col] + a[c]).astype(np.float32)
        acc[t % chains] += (a[0] + a[1]) + (a[2] + a[3])
    return acc.sum(0, dtype=np.float32)


def test_error_of_long_sums():
    """Terms of one sign, whose error grows most with the additions one after the other: a row of 32 batches leaves what two sums
    of 16 leave, half of what one sum of 32 does.  (Only one quarter of the columns counts here: what the tree over the quarters
    rounds would hide it.)"""
    from paper_2409_10644_amd import binding
    rng = np.random.default_rng(7)
    n, units, rows = 2048, 128, 2048
    w = np.zeros((units, n), np.float32)
    w[5] = np.where(np.arange(n) % 64 < 16, rng.uniform(0.47, 0.51, n), 0.0)
    last = np.zeros((1, units), np.float32)
    last[0, 5] = 1.0
    x = rng.uniform(0.47, 0.51, (rows, n)).astype(np.float32)
    exact = x.astype(np.float64) @ w[5].astype(np.float64)
    bias = -float(np.float32(exact.mean()))
    mlp = binding.make_mlp([torch.from_numpy(w).cuda(), torch.from_numpy(last).cuda()],
                           [torch.zeros(units, device="cuda"), torch.full((1,), bias, device="cuda")])
    prob, stop = torch.zeros((rows, 1), device="cuda"), torch.zeros((rows,), dtype=torch.int32, device="cuda")
    binding.early_stop_hidden(mlp, rows, 1, torch.from_numpy(x).cuda(), n, n, 0.5, prob, stop)
    p = prob.cpu().numpy()[:, 0].astype(np.float64)
    rms = lambda sums: float(np.sqrt(np.mean((sums - exact) ** 2)))
    two, one = rms(_sums_in_order(w[5], x, 2)), rms(_sums_in_order(w[5], x, 1))
    # the sum read back from the probability: the logit is exact (a difference of close numbers), |logit| < 1, and a probability
    # within 4 units of its last place, 2^-24 below 1, moves it by 4 * 2^-24 / (p (1 - p)) < 24 * 2^-24
    slack = 24 * 2.0 ** -24
    assert np.abs(exact + bias).max() < 1.0 and two + slack < 0.8 * one
    got = rms(np.log(p) - np.log1p(-p) - bias)
    assert got <= two + slack, (got, two, one)
