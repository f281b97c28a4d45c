"""R+ and R- of a small problem run in one launch on tiles of their own; the results must equal,
bit for bit, those of two launches (which a plan uses while its launches are timed). Sizes put
N+ and N- below, at and past 32, 48 and 64 rows, and the workgroups of both below and above the
512 up to which one launch is used."""
import sys

import numpy as np
import pytest

import ppl_synth as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("o,v,naux", [(2, 9, 8), (7, 33, 20), (10, 40, 24), (11, 75, 30)])
def test_two_tiles_in_one_launch(prec, o, v, naux):
    import paper_2603_20912_amd as P
    L = torch.from_numpy(S.make_system(o, v, naux, 50)["L"]).cuda()
    t = torch.from_numpy(S.make_amplitudes(o, v, 51)).cuda()
    eng = P.PPL(o, v, naux, prec=prec)
    eng.build(L)
    for tp in (6, 7, 8):
        for tm in (6, 7, 8):
            for sp, sm in ((1, 1), (4, 2), (8, 8)):
                print(f"[gpu-case] pair {prec} ({o},{v}) tiles {tp} {tm} splits {sp} {sm}")
                sys.stdout.flush()
                eng.set_contract_config(tp, sp, tm, sm)
                one = eng.contract(t).cpu().numpy()
                P.ppl_profile_enable(eng.plan, True)
                two = eng.contract(t).cpu().numpy()
                P.ppl_profile_enable(eng.plan, False)
                assert np.isfinite(one).all() and np.array_equal(one, two)
    eng.close()
