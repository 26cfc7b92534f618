"""The device bytes that a batch plan states for its waves: those of the records it
counts with, no less than it holds, and within the budget."""
import pytest

import paper_2505_04431_amd as kc

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def torch_first():
    import torch
    torch.zeros(1, device="cuda:0")


def _sets(n, nbytes):
    return [nbytes // 150] * n, [nbytes // 150 * 150] * n


def _plan_bytes(ks, n, nbytes, **opts):
    sr, sb = _sets(n, nbytes)
    plan = kc.BatchPlan(sr, sb, ks, P=1, opts=kc.options(**opts) if opts else None)
    need = [w["device_bytes"] for w in plan.waves]
    plan.close()
    return need


@pytest.mark.parametrize("n", [2, 8, 100, 1500])
@pytest.mark.parametrize("k", [27, 31, 32])
def test_one_word_records(n, k):
    # k = 21 has one-word records whatever the number of sets; so have these, cut to
    # 64 bits where the set id does not fit beside the k-mer
    assert _plan_bytes([k] * n, n, 300_000) == _plan_bytes([21] * n, n, 300_000)


def test_two_word_records():
    # two shard bits do not hold the ids of eight sets: two-word records
    one, two = (_plan_bytes([k] * 8, 8, 3_000_000, shard_bits=2)[0] for k in (21, 32))
    assert two > 1.3 * one


@pytest.mark.parametrize("k,opts", [(21, {}), (31, {}), (32, {}), (32, dict(shard_bits=2))])
def test_plan_holds_no_more(k, opts):
    import torch
    sr, sb = _sets(24, 8_000_000)
    torch.cuda.synchronize()
    free0, _ = torch.cuda.mem_get_info()
    plan = kc.BatchPlan(sr, sb, [k] * 24, P=1, opts=kc.options(**opts) if opts else None)
    held = free0 - torch.cuda.mem_get_info()[0]
    need = plan.waves[0]["device_bytes"]
    plan.close()
    assert held <= need + (64 << 20), (held, need)  # (each array in whole pages)


@pytest.mark.parametrize("k", [21, 31])
def test_waves_within_the_budget(k):
    sr, sb = _sets(40, 2_000_000)
    whole = _plan_bytes([k] * 40, 40, 2_000_000)[0]
    plan = kc.BatchPlan(sr, sb, [k] * 40, P=1, hbm_budget=whole // 3)
    assert len(plan.waves) >= 3
    assert all(w["device_bytes"] <= whole // 3 for w in plan.waves)
    plan.close()
