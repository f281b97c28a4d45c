"""The ring operands of low-precision sweeps are rounded through FP32: amplitudes whose FP32 value lies
halfway between two bf16 numbers, while they themselves lie a little below, go to the even one of
the two. The workspace of a sweep holds the rows B[(i,a)][(k,c)] = t_ik^ca as bf16 planes."""
import sys

import numpy as np
import pytest

import ppl_synth as S

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def to_bf16(x):
    """FP32 -> bf16 bits, to nearest even."""
    u = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)


def from_bf16(h):
    return (h.astype(np.uint32) << 16).view(np.float32)


@pytest.mark.parametrize("prec", ["bf16x3", "bf16x6"])
def test_ring_operands_round_through_fp32(prec):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2603_20912_amd as P
    o, v, naux = 3, 7, 9
    print(f"[gpu-case] ring operands {prec} ({o},{v},{naux})", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(150)
    t = np.zeros((o, o, v, v))
    for i in range(o):
        for j in range(i, o):
            for a in range(v):
                for b in range(v):
                    if i == j and a > b:
                        continue
                    h = int(rng.integers(0x3C00, 0x3D00)) | 1          # odd bf16 numbers near 0.01
                    x = float(from_bf16(np.array([h], dtype=np.uint16))[0])
                    ulp = float(from_bf16(np.array([h + 1], dtype=np.uint16))[0]) - x
                    t[i, j, a, b] = t[j, i, b, a] = x + ulp / 2 - ulp * 2.0 ** -30
    s = S.make_system(o, v, naux, 151, "contractive")
    eng = P.PPL(o, v, naux, prec=prec, ring=True)
    t2 = dev(t)
    eng.iterate(dev(s["L"]), dev(s["e_occ"]), dev(s["e_vir"]), t2, max_sweeps=1, tol=0.0, start="given", ring=True,
                fail_on_noconv=False, diverge_factor=0.0)
    ws = eng.workspace.cpu().numpy().tobytes()
    eng.close()
    x32 = t.transpose(0, 3, 1, 2).reshape(o * v, o * v).astype(np.float32)
    hi = to_bf16(x32)
    rest = x32 - from_bf16(hi)
    lo = to_bf16(rest)
    assert (rest < 0).all()                                              # every value went up to the even number
    for row in range(o * v):
        assert ws.find(hi[row].tobytes()) >= 0 and ws.find(lo[row].tobytes()) >= 0, row
