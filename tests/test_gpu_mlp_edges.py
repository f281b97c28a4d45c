"""The learned start's kernels at the edges of their blocks: training launches whose last block
of 32 rows is ragged or whose workgroups take several blocks (more than 8192 rows), and guesses
whose 16 x 16 tiles of virtual pairs are ragged, against the FP64 reference."""
import sys

import numpy as np
import pytest

from oracle import mlp_oracle as M
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


def dev(x, dtype=torch.float64):
    return torch.from_numpy(np.ascontiguousarray(x)).to(dtype).to("cuda")


@pytest.mark.parametrize("n", [1, 31, 33, 8193, 20011])
def test_gradient_of_ragged_batches(P, n):
    """FP32 sums of at most 128 + n products of order one: 1e-4 relative per parameter array."""
    say(f"mlp gradient n={n}")
    p = M.init_params(128, seed=17)
    rng = np.random.default_rng(18)
    X = (rng.standard_normal((n, 4)) * np.array([1.0, 3.0, 1.0, 2.0])).astype(np.float32)
    Y = (rng.standard_normal(n) * 0.3).astype(np.float32)
    mlp = P.MLP(max_batch=32768)
    flat = M.flatten(p).astype(np.float32)
    mlp.set_params(flat)
    g, loss = mlp.grad(dev(X, torch.float32), dev(Y, torch.float32))
    p32 = M.unflatten(flat.astype(np.float64), 128)
    X, Y = X.astype(np.float64), Y.astype(np.float64)
    gref = M.flatten(M.grad(p32, X, Y))
    assert abs(loss - M.loss(p32, X, Y)) < 1e-5 * M.loss(p32, X, Y)
    off = 0
    for k in M.PARAM_ORDER:
        sz = p32[k].size
        a, b = g[off:off + sz].astype(np.float64), gref[off:off + sz]
        assert np.linalg.norm(a - b) < 1e-4 * np.linalg.norm(b), k
        off += sz
    mlp.close()


@pytest.mark.parametrize("o,v", [(1, 2), (2, 15), (3, 16), (2, 17), (3, 33)])
def test_guess_at_tile_edges(P, o, v):
    """BF16 operands of the hidden layer: 2^-8 per operand over 128 terms (the bound of the whole
    network's guess test); every entry written once from its own features, pair-symmetric."""
    say(f"mlp guess ({o},{v})")
    s = S.make_system(o, v, 3 * v, 21, "contractive")
    p = M.init_params(128, seed=22)
    mlp = P.MLP(max_batch=64)
    mlp.set_params(M.flatten(p).astype(np.float32))
    eng = P.PPL(o, v, 3 * v)
    tm = S.make_amplitudes(o, v, 23)
    out = torch.full((o, o, v, v), float("nan"), dtype=torch.float64, device="cuda")
    X, sigma = M.features(tm, s["e_occ"], s["e_vir"])
    mlp.guess(eng, dev(tm), dev(s["e_occ"]), dev(s["e_vir"]), sigma, out)
    got = out.cpu().numpy()
    fref, _ = M.forward(p, X)
    i, j, a, b = np.indices((o, o, v, v))
    fref = fref.reshape(o, o, v, v)
    own = (i < j) | ((i == j) & (a <= b))           # the element whose features a pair takes
    fref = np.where(own, fref, fref.transpose(1, 0, 3, 2))
    base = np.where(own, tm, tm.transpose(1, 0, 3, 2))
    assert np.isfinite(got).all()
    assert np.max(np.abs((got - base) / sigma - fref)) < 2e-2 * (1.0 + np.abs(fref).max())
    assert np.array_equal(got, got.transpose(1, 0, 3, 2))
    eng.close()
    mlp.close()
