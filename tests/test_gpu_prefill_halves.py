"""Prefill work items walked by two workgroups each (half of the item's rows, or of its eight heads; the upper waves take the
upper 32 keys of every KV tile and meet the lower ones in LDS) against the oracle: every group size and way an item is shared
out, rows that end on and around the edges of halves and tiles, prefixes that put the diagonal in either half of a tile, walks
cut into partitions (some of which the first half of an item does not reach), next to decode requests, and batches on both
sides of the line where the items get one workgroup again."""
import numpy as np
import pytest

from oracle import attention as A
from paper_2512_12928_amd import binding as B
from paper_2512_12928_amd import workloads as W
from gpu_harness import check_close, oracle_cache, run_prefilled

pytestmark = pytest.mark.gpu


def check(Hq, Hkv, items, seed, **kw):
    """items: (l_q, prefix)."""
    rng = np.random.default_rng(seed)
    b = W.build_batch(W.LayerShape(Hq, Hkv), [(n, p + n) for n, p in items], [1] * len(items), rng, seed=seed)
    t = W.make_tensors(b)
    want = A.paged_attention(t.q, oracle_cache(b, t), b.q_start, b.kv_len, b.bt_start, b.block_ids)
    got, _ = run_prefilled(b, t, **kw)
    check_close(got, want, False)
    return B.ps_plan_launch(Hq, Hkv, b.n_device_blocks, b, **kw)


@pytest.mark.parametrize("prefix", [0, 17, 40, 96, 130])
@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (2, 1), (3, 1), (8, 2), (8, 1), (16, 1), (12, 2)])
def test_edges_of_rows_and_tiles(Hq, Hkv, prefix):
    lens = [2, 31, 32, 33, 64, 65, 100]
    p = check(Hq, Hkv, [(n, prefix) for n in lens], seed=700 + Hq + prefix)
    assert 2 * p["prefill_workgroups"] <= 256


@pytest.mark.parametrize("Hq,Hkv,items", [
    (8, 2, [(64, 1984)]), (8, 1, [(70, 1000)]), (4, 4, [(256, 900), (33, 0)]), (8, 2, [(128, 1000), (40, 7)]), (64, 8, [(64, 1984)])])
def test_partitions(Hq, Hkv, items):
    p = check(Hq, Hkv, items, seed=720 + Hq)
    assert p["prefill_split_tiles"] > 0 and 2 * p["prefill_workgroups"] <= 256


@pytest.mark.parametrize("split", [1, 2, 3])
def test_first_half_that_reaches_nothing(split):
    """Given partition lengths: the last partition of an item starts behind what its first rows see."""
    check(4, 2, [(70, 60), (128, 1), (64, 65)], seed=740, prefill_split_tiles=split)
    check(8, 8, [(300, 60), (256, 1)], seed=741, prefill_split_tiles=split)


@pytest.mark.parametrize("n", [960, 1024, 1088])
def test_around_one_workgroup_per_unit(n):
    check(32, 8, [(n, 0)], seed=750 + n)


def test_next_to_decode_requests():
    check(32, 8, [(1, 200), (300, 100), (1, 7), (1, 1000)], seed=760)
