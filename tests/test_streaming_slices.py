"""K slices of FP64 streaming plans: what ppl_plan_query reports is what a contraction runs. Stream-K,
which upper-triangle steps have no form of, is reported as the slices taken in its place."""
import pytest

from paper_2603_20912_amd import _lib


@pytest.mark.parametrize("o,v,naux,budget", [(20, 200, 600, 1 << 30), (9, 97, 61, 150 << 20), (4, 32, 19, 3 << 20)])
def test_reported_slices(tmp_path, o, v, naux, budget):
    plans = []

    def plan(tune):
        path = tmp_path / f"tune{len(plans)}.txt"
        path.write_text(f"ppl-tune 1 0 {o} {v} {tune}\n" if tune else "")
        plans.append(_lib.ppl_plan(o, v, naux, hbm_budget=budget, stream=False, tune_cache=str(path)))
        info = _lib.ppl_plan_query(plans[-1])
        assert info["resident"] == 0 and info["workspace_bytes"] <= budget
        return plans[-1], (info["splits_contract"], info["splits_contract_minus"])

    try:
        _, own = plan(None)
        p, eight = plan("8 8 8 8")
        _, streamk = plan("8 0 8 0")
        _, one = plan("8 1 8 1")
        assert min(own) >= 1 and one == (1, 1)
        # as many as the workspace holds sums for
        assert streamk == eight and 1 <= eight[0] == eight[1] <= 8
        _lib.ppl_set_contract_config(p, 8, 0, 5, 0)
        info = _lib.ppl_plan_query(p)
        assert (info["splits_contract"], info["splits_contract_minus"]) == eight
        for sp in range(1, 9):
            _lib.ppl_set_contract_config(p, 8, sp, 5, 9 - sp)
            info = _lib.ppl_plan_query(p)
            assert (info["splits_contract"], info["splits_contract_minus"]) == (sp, 9 - sp)
    finally:
        for p in plans:
            _lib.ppl_destroy(p)
