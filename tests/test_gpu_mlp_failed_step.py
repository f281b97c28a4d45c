"""A training step that fails before its update does not count: the next one takes the first
step's bias correction."""
import ctypes
import sys

import numpy as np
import pytest

from oracle import mlp_oracle as M

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_failed_step_is_not_counted():
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2603_20912_amd as P
    print("[gpu-case] training step behind a failed host call", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(31)
    X = torch.from_numpy(rng.standard_normal((64, 4)).astype(np.float32)).cuda()
    Y = torch.from_numpy(rng.standard_normal(64).astype(np.float32)).cuda()
    start = M.flatten(M.init_params(128, seed=32)).astype(np.float32)
    mlp = P.MLP(max_batch=64)
    mlp.set_params(start)
    mlp.train_step(X, Y, lr=1e-2)
    ref = mlp.get_params()
    mlp.set_params(start)
    torch.cuda.synchronize()
    # an invalid device number is refused by the host runtime, which keeps the error for the next
    # query: the step finds it behind its first launch
    hip = ctypes.CDLL(P._lib.load()._name)      # (the HIP runtime that the library is linked to)
    assert hip.hipSetDevice(9999) != 0
    try:
        mlp.train_step(X, Y, lr=1e-2)
        failed = False
    except P.PPLError:
        failed = True
    torch.cuda.synchronize()
    if not failed:                # a runtime whose launches clear the error
        assert np.array_equal(mlp.get_params(), ref)
        mlp.set_params(start)
    else:
        assert np.array_equal(mlp.get_params(), start)
    mlp.train_step(X, Y, lr=1e-2)
    assert np.array_equal(mlp.get_params(), ref)
    mlp.close()
