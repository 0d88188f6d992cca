"""Update after acceptance where the pieces of the work end: rows of one chunk to more than a round of chunks per workgroup, more
places for ids than a workgroup has threads, nodes and lengths outside their range.  Bit-exact against a plain copy."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,d,n_append", [(1, 8, 0), (17, 120, 1), (16, 128, 61), (1, 2056, 62), (32, 128, 63), (33, 128, 200), (65, 72, 5)])
def test_edges(H, d, n_append):
    from paper_2409_10644_amd import binding
    rng = np.random.default_rng(H * d)
    br, B, layers = (2, 2, 1), 5, 2
    gamma, view = 3, binding.slice_mask(binding.build_mask(br), 3)
    n, max_prefix = view.n_nodes, 12
    cap = max_prefix + gamma
    path = rng.integers(0, n, (B, gamma)).astype(np.int32)
    path[1, 0], path[3, 2] = -1, n                                # skipped
    alen = np.array([0, 3, 2, 7, -1], np.int32)                   # the last two clamped
    lens = np.array([0, 12, 5, 99, 4], np.int32)
    tokens, new = (rng.integers(0, 1000, s).astype(np.int32) for s in ((B, n), (B, n_append + 2)))
    tree = torch.randn((2, layers, B, H, n, d), device="cuda").bfloat16()
    cache = torch.randn((2, layers, B, H, cap, d), device="cuda").bfloat16()
    want, want_lens = cache.clone(), lens.copy()
    want_ids, want_n = np.full((B, gamma + n_append), -1, np.int32), np.zeros(B, np.int32)
    for b in range(B):
        a, L = min(max(alen[b], 0), gamma), min(max(lens[b], 0), max_prefix)
        for j in range(a):
            node = path[b, j]
            if 0 <= node < n:
                want[:, :, b, :, L + j] = tree[:, :, b, :, int(node)]
                want_ids[b, j] = tokens[b, node]
        want_ids[b, a:a + n_append] = new[b, :n_append]
        want_n[b], want_lens[b] = a + n_append, L + a
    dev = lambda x: torch.from_numpy(x).cuda()
    base = torch.arange(B, dtype=torch.int64, device="cuda") * (H * cap * d)
    d_lens, ids, n_ids = dev(lens), torch.full((B, gamma + n_append), -9, dtype=torch.int32, device="cuda"), dev(np.zeros(B, np.int32))
    binding.commit_path(view, 1, B, H, d, list(tree[0]), list(tree[1]), n, list(cache[0]), list(cache[1]), base, cap * d, max_prefix, cap,
                        dev(path), dev(alen), dev(tokens), dev(new), n_append + 2, n_append, d_lens, ids, n_ids)
    torch.cuda.synchronize()
    assert torch.equal(cache.view(torch.int16), want.view(torch.int16))
    assert np.array_equal(d_lens.cpu().numpy(), want_lens) and np.array_equal(n_ids.cpu().numpy(), want_n)
    assert np.array_equal(ids.cpu().numpy(), want_ids)
