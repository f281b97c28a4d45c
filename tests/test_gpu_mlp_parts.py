"""Guesses whose 16 x 16 tiles are dealt whole and in parts of 8, 4, 2 and 1 rows (the fewer tiles, the
smaller the parts), with a ragged last tile: every entry written, pair-symmetric, and sampled entries
against the FP64 reference within the bound of the BF16 hidden layer."""
import sys

import numpy as np
import pytest

from oracle import mlp_oracle as M
import ppl_synth as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


@pytest.mark.parametrize("o,v", [(12, 121), (8, 121), (6, 121), (4, 121), (2, 37)])
def test_guess_in_parts(o, v):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2603_20912_amd as P
    print(f"[gpu-case] mlp guess ({o},{v})", flush=True)
    sys.stdout.flush()
    s = S.make_system(o, v, 4, 26, "contractive")
    p = M.init_params(128, seed=27)
    mlp = P.MLP(max_batch=64)
    mlp.set_params(M.flatten(p).astype(np.float32))
    eng = P.PPL(o, v, 4, contract_only=True)
    tm = S.make_amplitudes(o, v, 28)
    out = torch.full((o, o, v, v), float("nan"), dtype=torch.float64, device="cuda")
    X, sigma = M.features(tm, s["e_occ"], s["e_vir"])
    mlp.guess(eng, dev(tm), dev(s["e_occ"]), dev(s["e_vir"]), sigma, out)
    got = out.cpu().numpy()
    assert np.isfinite(got).all()
    assert np.array_equal(got, got.transpose(1, 0, 3, 2))
    rng = np.random.default_rng(29)
    pick = rng.integers(0, o * o * v * v, 20000)
    i, j, a, b = np.unravel_index(pick, (o, o, v, v))
    own = (i < j) | ((i == j) & (a <= b))              # the element whose features a pair takes
    idx = np.where(own, pick, np.ravel_multi_index((j, i, b, a), (o, o, v, v)))
    fref, _ = M.forward(p, X[idx])
    d = (got.reshape(-1)[pick] - tm.reshape(-1)[idx]) / sigma - fref.reshape(-1)
    assert np.max(np.abs(d)) < 2e-2 * (1.0 + np.abs(fref).max())
    eng.close()
    mlp.close()
