"""Resident plans hold V+- as upper triangles with whole 256 x 256 diagonal
blocks. Every workspace byte is set to 0xff (NaN in every type) before the build, so a read
of an entry that is not stored shows in the result; the results must equal, bit for bit,
those of a plan that builds and stores every row in full (the same products summed in the
same order), and the oracle's. Sizes put P+ and P- just below, at and past block and
tile edges: (P+, P-) = (276, 253), (528, 496), (1035, 990)."""
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


def rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def plan(P, monkeypatch, sym, o, v, naux, **kw):
    monkeypatch.setenv("PPL_SYM_BUILD", sym)
    eng = P.PPL(o, v, naux, **kw)
    assert eng.info["resident"] == 1
    eng.workspace.fill_(255)
    P.ppl_bind_workspace(eng.plan, eng.workspace)
    return eng


SIZES = [(4, 23, 19), (3, 32, 40), (5, 45, 17)]


@pytest.mark.parametrize("prec,bound", [("fp64", 1e-12), ("fp32", 2e-6)])
@pytest.mark.parametrize("o,v,naux", SIZES)
def test_triangle_equals_full_rows_in_every_configuration(P, monkeypatch, prec, bound, o, v, naux):
    s = S.make_system(o, v, naux, 80)
    t = S.make_amplitudes(o, v, 81)
    ref = O.ppl(s["L"], o, t)
    L, t = dev(s["L"]), dev(t)
    tri = plan(P, monkeypatch, "1", o, v, naux, prec=prec, build_scratch=1 << 20)
    full = plan(P, monkeypatch, "0", o, v, naux, prec=prec)
    tri.build(L)
    full.build(L)
    for tile in range(P.ppl_tile_count()):
        for splits in (1, 3, 8, 0):
            say(f"triangle {prec} ({o},{v},{naux}) tile {tile} splits {splits}")
            out = []
            for eng in (tri, full):
                eng.set_contract_config(tile, splits, tile, splits)
                out.append(eng.contract(t).cpu().numpy())
            assert np.array_equal(out[0], out[1])
            assert rel(out[0], ref) < bound
    tri.close()
    full.close()


@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "bf16x6"])
@pytest.mark.parametrize("o,v,naux", SIZES)
def test_low_precision_copy_of_a_triangle(P, monkeypatch, prec, o, v, naux):
    """The low-precision V+- of a mixed plan, rounded from the FP64 triangle."""
    say(f"mixed operands from a triangle {prec} ({o},{v},{naux})")
    s = S.make_system(o, v, naux, 82)
    t = dev(S.make_amplitudes(o, v, 83))
    out = []
    for sym in ("1", "0"):
        eng = plan(P, monkeypatch, sym, o, v, naux, prec=prec, keep_fp64=True)
        eng.build(dev(s["L"]))
        out.append(eng.contract(t).cpu().numpy())
        eng.close()
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("prec,bound", [("fp64", 1e-12), ("fp32", 2e-6)])
def test_grouped_launch_reads_triangles(P, prec, bound):
    say(f"grouped triangles {prec}")
    b = P.Batch(SIZES, prec=prec)
    b.workspace.fill_(255)
    P.ppl_batch_bind_workspace(b.h, b.workspace)
    systems = [S.make_system(o, v, naux, 90 + k) for k, (o, v, naux) in enumerate(SIZES)]
    ts = [S.make_amplitudes(o, v, 95 + k) for k, (o, v, _) in enumerate(SIZES)]
    b.build([dev(s["L"]) for s in systems])
    Rs = [torch.empty(t.shape, dtype=torch.float64, device="cuda") for t in ts]
    b.contract([dev(t) for t in ts], Rs)
    torch.cuda.synchronize()
    for s, t, R in zip(systems, ts, Rs):
        assert rel(R.cpu().numpy(), O.ppl(s["L"], s["o"], t)) < bound
    b.close()


@pytest.mark.parametrize("prec,bound", [("bf16x3", 4e-5), ("bf16x6", 2e-6)])
@pytest.mark.parametrize("o,v,naux", SIZES)
def test_bf16_triangles(P, monkeypatch, prec, bound, o, v, naux):
    """BF16 triangles: every entry that is read is written (poisoned workspace), steps give the
    same rows in any order, and every tile (64, 128 and 256 columns, K chunks of 32 and 64) the
    same sums for a number of slices."""
    say(f"bf16 triangles {prec} ({o},{v},{naux})")
    s = S.make_system(o, v, naux, 84)
    t = S.make_amplitudes(o, v, 85)
    L = dev(s["L"])
    out = []
    for order in (None, 1, -1):
        eng = plan(P, monkeypatch, "1", o, v, naux, prec=prec, build_scratch=1 << 20)
        nb = int(eng.info["n_batches"])
        if order is None:
            eng.build(L)
        else:
            for k in list(range(nb))[::order] + [nb - 1]:
                eng.build(L, k)
        out.append(eng.contract(dev(t)).cpu().numpy())
        if order != -1:
            eng.close()
    ref = O.ppl(s["L"], o, t)
    assert rel(out[0], ref) < bound
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    for splits in (1, 3, 8, 0):
        res = []
        for tile in range(P.ppl_tile_count()):
            say(f"  tile {tile} splits {splits}")
            eng.set_contract_config(tile, splits, tile, splits)
            res.append(eng.contract(dev(t)).cpu().numpy())
            assert rel(res[-1], ref) < bound
            if splits == 1:
                assert np.array_equal(res[-1], res[0])
    eng.close()


@pytest.mark.parametrize("kw", [dict(prec="fp64"), dict(prec="bf16x6"), dict(prec="fp32", keep_fp64=True)])
def test_refused_vectors_leave_the_operands(P, kw):
    """The staging of a build runs while the host waits for the symmetry check: a refused L must
    leave V+- as they were."""
    o, v, naux = SIZES[0]
    say(f"refused vectors {kw}")
    s = S.make_system(o, v, naux, 86)
    t = dev(S.make_amplitudes(o, v, 87))
    eng = P.PPL(o, v, naux, **kw)
    eng.build(dev(s["L"]))
    before = eng.contract(t).cpu().numpy()
    bad = s["L"].copy()
    bad[0, o, o + 1] += 1.0
    with pytest.raises(P.PPLError):
        eng.build(dev(bad))
    assert np.array_equal(eng.contract(t).cpu().numpy(), before)
    eng.close()


@pytest.mark.parametrize("prec,bound", [("fp32", 2e-6), ("bf16x3", 4e-5), ("bf16x6", 2e-6)])
@pytest.mark.parametrize("v,naux", [(110, 33), (111, 31)])
def test_builds_on_both_sides_of_the_tile_rule(P, prec, bound, v, naux):
    """FP32 builds change their tile at v = 110; one chunk of vectors, and one more vector."""
    say(f"builds {prec} (2,{v},{naux})")
    s = S.make_system(2, v, naux, 88)
    t = S.make_amplitudes(2, v, 89)
    eng = P.PPL(2, v, naux, prec=prec)
    eng.workspace.fill_(255)
    P.ppl_bind_workspace(eng.plan, eng.workspace)
    eng.build(dev(s["L"]))
    assert rel(eng.contract(dev(t)).cpu().numpy(), O.ppl(s["L"], 2, t)) < bound
    eng.close()
