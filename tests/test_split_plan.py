"""Calls whose plan leaves a member much shorter than the bound in one piece (no GPU needed): it is then rounded to bf16 once."""
import pytest

from paper_2409_10644_amd import binding as b

# sequences, query heads, key/value heads, head size, tree nodes, prefix bound, keys of the short member, fp8 cache
WHOLE = [(7, 12, 12, 128, 81, 2768, 800, 0), (4, 32, 32, 64, 44, 639, 300, 0), (29, 8, 4, 128, 4, 861, 322, 0), (1, 32, 32, 128, 28, 803, 224, 0),
         (7, 16, 16, 128, 81, 550, 256, 0), (1, 4, 4, 128, 20, 522, 165, 0), (3, 32, 4, 64, 88, 529, 292, 0), (3, 64, 32, 128, 44, 1030, 391, 1),
         (42, 16, 4, 128, 28, 495, 495, 1), (14, 16, 8, 128, 81, 2118, 2118, 1)]


def partial_results(B, Hq, Hkv, d, n, bound, L, fp8):
    """Of a sequence of L keys, by the plan of its call."""
    p = b.tree_attention_plan(None, b.MCSD_BF16, fp8, B, Hq, Hkv, d, n, 0, bound)
    T = 128 if p.query_blocks == 1 else 64
    blocks = -(-n // 32)
    blocks = 4 if blocks > 2 else 2 if blocks == 2 or (fp8 and Hq // Hkv % 2) else 1
    units = B * Hq * blocks // p.query_blocks
    tiles = lambda keys: -(-keys // T)
    per_split = -(-tiles(bound) // p.key_splits)
    return max(1, -(-tiles(L) // per_split)) + (p.workgroups // units > p.key_splits)


@pytest.mark.parametrize("B,Hq,Hkv,d,n,bound,L,fp8", WHOLE)
def test_short_members_stay_whole(B, Hq, Hkv, d, n, bound, L, fp8):
    assert partial_results(B, Hq, Hkv, d, n, bound, L, fp8) == 1
