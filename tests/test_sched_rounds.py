"""Branches of the batch former that the step-by-step parity runs do not single out: a pool's duplicate check (a table of
marks or a sort, by the span of its ids), and the rounds of ps_sched_simulate, which leave the batch's tables out, against
the same rounds formed one by one.  Host only."""
import numpy as np
import pytest

from paper_2512_12928_amd import binding as B
from paper_2512_12928_amd import tdg_sim
from paper_2512_12928_amd import workloads as W


@pytest.mark.parametrize("stride", [1, 15, 1000])     # dense ids, the widest span of the table, beyond it
@pytest.mark.parametrize("base", [0, -7, 2 ** 31 - 1 - 1000 * 300])
def test_a_pool_that_names_a_block_twice_is_refused(stride, base):
    ids = (np.random.default_rng(3).permutation(300).astype(np.int64) * stride + base).astype(np.int32)
    B.ps_sched_destroy(B.ps_sched_create(tdg_sim.default_cfg(), ids, ids))
    for twice in (0, 299):
        bad = ids.copy()
        bad[150] = bad[twice]
        for pools in ((bad, ids), (ids, bad)):
            with pytest.raises(B.PsError) as e:
                B.ps_sched_create(tdg_sim.default_cfg(), *pools)
            assert e.value.code == B.PS_EINVAL


@pytest.mark.parametrize("pool,policy,gamma", [(40_000, 0, 9), (300, 0, 9), (300, 0, 0), (300, 1, 9), (300, 0, 10 ** 7)])
def test_simulated_rounds_are_the_rounds_formed_one_by_one(pool, policy, gamma):
    """No offload is ever reported complete here, so the two runs need no copy clock in common: t_block is so large that the
    simulated copy thread finishes nothing either."""
    cfg = tdg_sim.default_cfg(gamma_num=gamma, gamma_den=10, order_policy=policy, t_block_ps=10 ** 15, tau_ps=4 * 10 ** 12)
    trace = W.make_trace(2, 60, rate_per_s=400.0, seed=11, prompt_mean=500.0, prompt_max=2000, out_mean=40.0, out_max=120)
    order = np.random.default_rng(4).permutation(pool).astype(np.int32)
    sim = B.ps_sched_simulate(cfg, order, order, trace, 3000)
    s = B.ps_sched_create(cfg, order, order)
    pending, now, steps, evicted = list(trace), 0, 0, 0
    times = {p.rid: [] for p in trace}
    arrival = {p.rid: p.arrival_ps for p in trace}
    while steps < 3000:
        while pending and pending[0].arrival_ps <= now:
            p = pending.pop(0)
            B.ps_sched_add_request(s, p.rid, p.arrival_ps, p.prio, p.prompt_len, p.out_len)
        if B.ps_sched_counts(s)[0] == 0:
            if not pending:
                break
            now = pending[0].arrival_ps
            continue
        fb = B.ps_form_batch(s, now)
        steps += 1
        evicted += len(fb["evicted"])
        assert len(fb["order"]) == len(set(fb["order"].tolist()))
        for rid in fb["emitted_req"].tolist():
            times[rid].append(now + fb["t_batch"] - arrival[rid])
        now += fb["t_batch"] if fb["t_batch"] > 0 else cfg["eta_ps"]
    B.ps_sched_destroy(s)
    assert steps == sim["steps"] and now == sim["end_ps"]
    assert (evicted > 0) == (pool < 1000)
    for p, t in zip(trace, sim["token_times"]):
        assert t.tolist() == times[p.rid]
