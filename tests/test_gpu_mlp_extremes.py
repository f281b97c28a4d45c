"""Guesses with hidden units far out: SiLU is zero to FP32 for large negative arguments (to -0 or
within 1.1e-36 of it), +inf for +inf, and NaN only for NaN and -inf."""
import sys

import numpy as np
import pytest

from oracle import mlp_oracle as M
import ppl_synth as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

O_, V = 2, 19


def say(msg):
    print(f"[gpu-case] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2603_20912_amd as P
    return P


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def guess(P, p, tm=None):
    s = S.make_system(O_, V, 3 * V, 21, "contractive")
    if tm is None:
        tm = S.make_amplitudes(O_, V, 23)
    mlp = P.MLP(max_batch=64)
    mlp.set_params(M.flatten(p).astype(np.float32))
    eng = P.PPL(O_, V, 3 * V)
    out = mlp.guess(eng, dev(tm), dev(s["e_occ"]), dev(s["e_vir"]), 0.1).cpu().numpy()
    eng.close()
    mlp.close()
    return out


@pytest.mark.parametrize("z", [-95.0, -700.0, -1e4, -1e30, -3e38])
def test_large_negative_arguments_give_nothing(P, z):
    """The units' outgoing weights are large enough to show 1e-35: the same bits with and
    without them."""
    say(f"silu at {z}")
    p = M.init_params(128, seed=22)
    k = [0, 7, 77, 127]
    p["W1"][k] = 0.0
    p["b1"][k] = z
    p["W2"][k] = 0.0
    p["b2"][k] = z
    p["W2"][:, k] = 0.0
    p["W3"].reshape(-1)[k] = 0.0
    ref = guess(P, p)
    p["W2"][:, k] = 1e35
    p["W2"][k] = 0.0
    p["W3"].reshape(-1)[k] = 1e35
    assert np.isfinite(ref).all() and np.array_equal(guess(P, p), ref)


@pytest.mark.parametrize("layer", [1, 2])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_infinite_units(P, layer, sign):
    say(f"silu at +inf, layer {layer}")
    p = M.init_params(128, seed=24)
    p["W2"] = np.abs(p["W2"]) + 1e-3
    p["W3"] = sign * (np.abs(p["W3"]) + 1e-3)
    p["b1" if layer == 1 else "b2"][5] = np.inf
    assert (guess(P, p) == sign * np.inf).all()


def test_nan_amplitudes_stay_where_they_are(P):
    say("guess with a NaN amplitude")
    p = M.init_params(128, seed=25)
    tm = S.make_amplitudes(O_, V, 23)
    ref = guess(P, p, tm)
    bad = tm.copy()
    bad[0, 1, 3, 17] = bad[1, 0, 17, 3] = np.nan
    got = guess(P, p, bad)
    nan = np.isnan(got)
    assert nan.sum() == 2 and nan[0, 1, 3, 17] and nan[1, 0, 17, 3]
    assert np.array_equal(got[~nan], ref[~nan])
