"""What the workspace queries promise (no GPU needed): the size for a call serves the same batch and heads with fewer query
rows, fewer tree nodes or a shorter prefix, and is what the plan of each of these calls needs, in either element type."""
import numpy as np
import pytest

from paper_2409_10644_amd import binding as b

KINDS = ("attention", "gqa", "fp8")


def _query(kind, B, Hq, Hkv, d, n, row0, L):
    if kind == "fp8":
        return b.tree_attention_fp8kv_workspace(B, Hq, Hkv, n, row0, L)
    if kind == "gqa":
        return b.tree_attention_gqa_workspace(B, Hq, Hkv, d, n, row0, L)
    return b.tree_attention_rows_workspace(B, Hq, d, n, row0, L) if row0 else b.tree_attention_workspace(B, Hq, d, n, L)


def _need(kind, dtype, B, Hq, Hkv, d, n, row0, L):
    """Bytes that the plan of this call asks for: tag, counters, then per partial result maxima, denominators and outputs."""
    p = b.tree_attention_plan(None, dtype, int(kind == "fp8"), B, Hq, Hkv, d, n, row0, L)
    if p.key_splits == 1:
        return 0
    if dtype == b.MCSD_F32:
        rows = (n - row0 + 15) // 16 * 16
        slots = B * Hq * p.key_splits
        size = 4
    else:
        grp, qb = Hq // Hkv, (n - row0 + 31) // 32
        bph = 1 if qb <= 1 else 2 if qb == 2 else 4
        if kind == "fp8" and bph == 1 and grp % 2:
            bph = 2
        hpw = p.query_blocks // bph
        rows, slots, size = 32 * p.query_blocks, p.workgroups, 2
        assert slots >= B * Hq // hpw * p.key_splits
        # (a grid rounded up to whole dies has empty slots, without partial results)
        units = B * Hq // hpw
        slots = min(slots, units * (slots // units))
        keys = 128 if p.query_blocks == 1 else 64
        if (L + keys - 1) // keys * keys < 512 and slots // units <= 7:     # short prefixes: partial outputs in fp32
            size = 4
    up = lambda x: (x + 255) // 256 * 256
    return 256 + 65536 + 2 * up(slots * rows * 4) + up(slots * rows * d * size)


def _shape(rng, kind):
    Hkv = int(rng.choice((1, 2, 4, 8, 12, 16, 32)))
    Hq = Hkv if kind == "attention" else Hkv * int(rng.choice((1, 2, 3, 4, 8)))
    n = int(rng.integers(1, 129))
    row0 = int(rng.integers(0, n)) if rng.random() < 0.5 else 0
    L = int(np.exp(rng.uniform(0, np.log(16384))))
    return int(np.exp(rng.uniform(0, np.log(64)))), Hq, Hkv, 128 if kind == "fp8" or rng.random() < 0.5 else 64, n, row0, L


@pytest.mark.parametrize("kind", KINDS)
def test_a_larger_call_serves_the_smaller_ones(kind):
    rng = np.random.default_rng(KINDS.index(kind))
    for _ in range(6000):
        B, Hq, Hkv, d, n, row0, L = _shape(rng, kind)
        whole = _query(kind, B, Hq, Hkv, d, n, 0, L)
        rows = _query(kind, B, Hq, Hkv, d, n, row0, L)
        assert rows <= whole, (kind, B, Hq, Hkv, d, n, row0, L)
        n2 = int(rng.integers(1, n + 1))
        r2 = int(rng.integers(0, n2))
        L2 = int(rng.integers(0, L + 1))
        assert _query(kind, B, Hq, Hkv, d, n2, r2, L2) <= whole, (kind, B, Hq, Hkv, d, n, L, n2, r2, L2)
        for dtype in (b.MCSD_BF16,) if kind == "fp8" else (b.MCSD_BF16, b.MCSD_F32):
            assert _need(kind, dtype, B, Hq, Hkv, d, n, row0, L) <= rows, (kind, dtype, B, Hq, Hkv, d, n, row0, L)
            assert _need(kind, dtype, B, Hq, Hkv, d, n2, r2, L2) <= whole, (kind, dtype, B, Hq, Hkv, d, n, L, n2, r2, L2)


def test_newest_level_in_fp32_of_a_tree_that_is_not_split():
    assert b.tree_attention_rows_workspace(9, 32, 64, 87, 79, 243) <= b.tree_attention_workspace(9, 32, 64, 87, 243)
