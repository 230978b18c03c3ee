"""Decode-only batches laid out by request (a workgroup of 4 or 8 waves per segment and kv-head, the waves meeting in LDS;
the wave with a request's last tile appends this step's row) against the oracle: context lengths on and around the edges of
blocks, tiles and of the waves' shares, every group size, requests whole and cut, 4 and 8 waves, with and without new rows.
The append of every decode path (this one, the slot walk, the waves of a mixed launch) has to leave the oracle's pool."""
import numpy as np
import pytest

from oracle import attention as A
from paper_2512_12928_amd import binding as B
from paper_2512_12928_amd import workloads as W
from gpu_harness import Layer, check_close, dev_to_u16, oracle_cache, run_prefilled, u16_to_dev
from paper_2512_12928_amd.kvlayout import from_device_layout, to_device_layout

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 127, 128, 129, 224, 255, 256, 257, 288, 289]


def batch_of(Hq, Hkv, items, seed):
    rng = np.random.default_rng(seed)
    b = W.build_batch(W.LayerShape(Hq, Hkv), items, [1] * len(items), rng, seed=seed)
    return b, W.make_tensors(b)


def check(b, t, append=True, **kw):
    full = oracle_cache(b, t)
    want = A.paged_attention(t.q, full, b.q_start, b.kv_len, b.bt_start, b.block_ids)
    if not append:
        got, _ = run_prefilled(b, t, **kw)
        check_close(got, want, False)
        return
    cache = u16_to_dev(to_device_layout(oracle_cache(b, t, upto_prefix=True).pool))
    k_new, v_new = t.new_rows(b)
    lay = Layer(b, **kw)
    out = lay.step(b, u16_to_dev(t.q), cache, u16_to_dev(k_new), u16_to_dev(v_new))
    lay.close()
    check_close(out.cpu().numpy().astype(np.float64), want, False)
    assert np.array_equal(from_device_layout(dev_to_u16(cache), b.shape.n_kv_heads), full.pool)


def plan(b):
    s = b.shape
    p = B.ps_plan_launch(s.n_q_heads, s.n_kv_heads, b.n_device_blocks, b)
    assert p["decode_workgroups"] == p["decode_slots"] * s.n_kv_heads      # laid out by request
    return p


@pytest.mark.parametrize("append", [True, False])
@pytest.mark.parametrize("Hq,Hkv", [(1, 1), (4, 2), (12, 4), (32, 8), (64, 8), (16, 1)])
def test_edges_of_blocks_tiles_and_shares(Hq, Hkv, append):
    b, t = batch_of(Hq, Hkv, [(1, L) for L in EDGES], seed=500 + Hq)
    assert plan(b)["decode_slots"] >= len(EDGES)
    check(b, t, append)


@pytest.mark.parametrize("lens", [[3000], [5000, 40, 700], [L for L in EDGES for _ in range(3)], [1300] * 5 + [900] * 11])
def test_whole_and_cut_requests(lens):
    """One long request (more than 8 partials), a long one next to short ones, more workgroups than compute units (4 waves
    each), equal requests."""
    b, t = batch_of(32, 8, [(1, L) for L in lens], seed=600 + len(lens))
    assert plan(b)["partial_slots"] > 8 or max(lens) < 3000
    check(b, t)


def test_nothing_of_a_stale_slot_reaches_the_output():
    """The slot of this step's token and those behind it hold NaN when the launch starts."""
    b, t = batch_of(16, 8, [(1, L) for L in (1, 16, 17, 32, 33, 200, 1025)], seed=77)
    check(b, t)


@pytest.mark.parametrize("kw", [dict(decode_waves=64), dict(decode_chunk=64), dict(mixed_launch=1), dict(mixed_launch=2)])
def test_every_decode_path_appends(kw):
    items = [(1, L) for L in EDGES] + ([(40, 90), (70, 70)] if "mixed_launch" in kw else [])
    b, t = batch_of(8, 2, items, seed=88)
    check(b, t, **kw)


@pytest.mark.parametrize("dead", [(0, 64), (32, 550), (0, 599)])
def test_a_run_of_keys_without_weight(dead):
    """Keys at minus infinity have weight 0, also where they are all that a wave, or a partition, has seen so far."""
    b, t = batch_of(8, 2, [(1, 600)] * 3 + [(1, 1700)], seed=91)
    t.q[:, :, 0] = 0x3F80                       # 1.0
    for k in t.k:
        k[dead[0]:dead[1], :, 0] = 0xFF80       # -inf
    check(b, t)


def test_a_row_that_another_request_reads():
    """The second request's context runs over the block that the first one's row completes in this step."""
    b, t = batch_of(8, 2, [(1, 48), (1, 80), (1, 20)], seed=92)
    b.block_ids[b.bt_start[1]:b.bt_start[1] + 3] = b.table(0)
    for x in (t.k, t.v):
        x[1][:48] = x[0]
    full = oracle_cache(b, t)
    want = A.paged_attention(t.q, full, b.q_start, b.kv_len, b.bt_start, b.block_ids)
    start = oracle_cache(b, t, upto_prefix=True)
    start.append(b.table(0)[2:], 15, *(np.full_like(x[0][:1], W.BF16_NAN) for x in (t.k, t.v)))
    cache = u16_to_dev(to_device_layout(start.pool))
    k_new, v_new = t.new_rows(b)
    lay = Layer(b)
    out = lay.step(b, u16_to_dev(t.q), cache, u16_to_dev(k_new), u16_to_dev(v_new))
    lay.close()
    check_close(out.cpu().numpy().astype(np.float64), want, False)
    assert np.array_equal(from_device_layout(dev_to_u16(cache), 2), full.pool)
