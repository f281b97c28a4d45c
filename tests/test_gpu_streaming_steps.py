"""Streaming plans of upper-triangle steps: every step adds S' V_step and its mirror image in one
launch per sign, from rows stored between zero rows and with zeros before their own pair.
Every workspace byte starts as 0xff (NaN), so a read of an entry that no step writes shows.
Sizes put steps at odd first pairs, shorter than a K chunk, wider than a column tile, and (P+, P-)
just below, at and past tile and block edges. V = U + U^T only reorders each sum: FP64 rounding of
sums of up to 4753 terms, bounded here as for the other FP64 contractions (1e-12)."""
import sys

import numpy as np
import pytest

import oracle as O
import ppl_synth as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2603_20912_amd as P
    return P


def streaming(P, o, v, naux, div):
    """The smallest budget above 1/div of a resident plan's workspace that is accepted."""
    res = P.PPL(o, v, naux)
    full = int(res.info["workspace_bytes"])
    res.close()
    budget = full // div
    while True:
        try:
            eng = P.PPL(o, v, naux, hbm_budget=budget)
        except P.PPLError:
            budget += full // 16
            continue
        assert eng.info["resident"] == 0 and budget < full
        eng.workspace.fill_(255)
        P.ppl_bind_workspace(eng.plan, eng.workspace)
        return eng


@pytest.mark.parametrize("o,v,naux,div", [(1, 31, 12, 3), (4, 32, 19, 3), (5, 45, 17, 2), (2, 64, 33, 9), (9, 97, 61, 4)])
def test_every_tile_and_slice_count(P, o, v, naux, div):
    s = S.make_system(o, v, naux, 60)
    t = S.make_amplitudes(o, v, 61)
    ref = O.ppl(s["L"], o, t)
    eng = streaming(P, o, v, naux, div)
    say(f"streaming ({o},{v},{naux}): {eng.info['n_batches']} steps of up to {eng.info['max_step_pairs']} pairs")
    L = torch.from_numpy(s["L"]).cuda()
    td = torch.from_numpy(t).cuda()
    eng.build(L)
    for tile in range(P.ppl_tile_count()):
        for splits in (1, 3, 8, 0):
            say(f"  tile {tile} slices {splits}")
            eng.set_contract_config(tile, splits, tile, splits)
            R = eng.contract(td).cpu().numpy()
            assert np.linalg.norm(R - ref) < 1e-12 * np.linalg.norm(ref)
    eng.close()
