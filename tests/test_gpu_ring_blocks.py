"""Ring terms and (ia|jb) start at sizes around the 32 x 32 blocks and the GEMM tiles that their
passes work in: v below, at and past 32 and 64, o v below, at and past a multiple of 64 (row
padding up to 63 columns), scratch and workspace filled with NaN. FP64, 1e-12 as for the
other terms."""
import sys

import numpy as np
import pytest

import oracle as O
import ppl_synth as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("o,v,naux", [(1, 2, 3), (2, 31, 10), (2, 32, 16), (3, 33, 40), (5, 51, 17), (13, 65, 33)])
def test_ring_and_ov_blocks(o, v, naux):
    import paper_2603_20912_amd as P
    print(f"[gpu-case] ring and (ia|jb) ({o},{v},{naux})")
    sys.stdout.flush()
    s = S.make_system(o, v, naux, 70)
    t2 = S.make_amplitudes(o, v, 71)
    L = torch.from_numpy(s["L"]).cuda()
    scratch = torch.full((P.ppl_ring_scratch_bytes(o, v, naux),), 255, dtype=torch.uint8, device="cuda")
    R0 = np.random.default_rng(72).standard_normal(t2.shape)
    R = torch.from_numpy(R0.copy()).cuda()
    P.ring(L, torch.from_numpy(t2).cuda(), R, alpha=2.0, beta=0.5, scratch=scratch)
    ref = 0.5 * R0 + 2.0 * O.ring(s["L"], o, t2)
    assert np.linalg.norm(R.cpu().numpy() - ref) < 1e-12 * np.linalg.norm(ref)
    eng = P.PPL(o, v, naux)
    eng.workspace.fill_(255)
    P.ppl_bind_workspace(eng.plan, eng.workspace)
    e_occ, e_vir = (torch.from_numpy(s[k]).cuda() for k in ("e_occ", "e_vir"))
    t = torch.full((o, o, v, v), float("nan"), dtype=torch.float64, device="cuda")
    eng.mp2(L, e_occ, e_vir, t)
    mp2 = O.mp2_amplitudes(s["L"], o, s["e_occ"], s["e_vir"])
    assert np.linalg.norm(t.cpu().numpy() - mp2) < 1e-12 * np.linalg.norm(mp2)
    eng.close()
