"""A streaming plan cuts K into the slices asked for, also where its workspace holds fewer sums:
every count rounds the results in its own way (the same bits for two counts would mean the same
decomposition), and all agree with the oracle as the other FP64 contractions do."""
import sys

import numpy as np
import pytest

import oracle as O
import ppl_synth as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2603_20912_amd as P
    return P


@pytest.mark.parametrize("slices", [1, 3])
def test_slices_asked_for(P, tmp_path, slices):
    """slices: what the plan is made with, so that it holds one or three sums."""
    o, v, naux = 5, 97, 31
    s = S.make_system(o, v, naux, 140)
    t = S.make_amplitudes(o, v, 141)
    ref = O.ppl(s["L"], o, t)
    L, t = (torch.from_numpy(x).cuda() for x in (s["L"], t))
    path = tmp_path / "tune.txt"
    path.write_text(f"ppl-tune 1 0 {o} {v} 6 {slices} 6 {slices}\n")
    res = P.PPL(o, v, naux)
    budget = int(res.info["workspace_bytes"]) // 2
    res.close()
    eng = P.PPL(o, v, naux, hbm_budget=budget, tune_cache=str(path))
    assert eng.info["resident"] == 0 and eng.contract_config() == (6, slices, 6, slices)
    eng.workspace.fill_(255)
    P.ppl_bind_workspace(eng.plan, eng.workspace)
    eng.build(L)
    out = []
    for sp in range(1, 9):
        print(f"[gpu-case] streaming ({o},{v},{naux}) made with {slices} slices, asked for {sp}", flush=True)
        sys.stdout.flush()
        eng.set_contract_config(6, sp, 6, sp)
        assert eng.contract_config() == (6, sp, 6, sp)
        R = eng.contract(t).cpu().numpy()
        assert np.linalg.norm(R - ref) < 1e-12 * np.linalg.norm(ref)
        assert np.array_equal(eng.contract(t).cpu().numpy(), R)
        out.append(R)
    assert all(not np.array_equal(out[i], out[j]) for i in range(8) for j in range(i))
    eng.close()
