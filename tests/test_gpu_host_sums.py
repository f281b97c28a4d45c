"""Sums that the host reads live in memory of the library. What a call only enqueues must not
depend on it: such work can outlive the plan."""
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


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda")


def test_captured_mp2_outlives_its_plan(P):
    """ppl_mp2 without an energy is kernel launches only: a graph of it replays after
    ppl_destroy, on the workspace that the caller still owns."""
    o, v, naux = 3, 17, 23
    say(f"mp2 graph replayed without its plan ({o},{v},{naux})")
    systems = [S.make_system(o, v, naux, 120 + k) for k in range(3)]
    eo, ev = dev(systems[0]["e_occ"]), dev(systems[0]["e_vir"])
    ref = []
    eng = P.PPL(o, v, naux)
    for s in systems:
        ref.append(eng.mp2(dev(s["L"]), eo, ev)[0].cpu().numpy())
    eng.close()
    L = dev(systems[0]["L"])
    t = torch.empty((o, o, v, v), dtype=torch.float64, device="cuda")
    st = torch.cuda.Stream()
    eng = P.PPL(o, v, naux, stream=st)
    st.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        P.ppl_mp2(eng.plan, L, eo, ev, t, want_energy=False)
    plan, eng.plan = eng.plan, None
    P.ppl_destroy(plan)
    for k, s in enumerate(systems):
        L.copy_(dev(s["L"]))
        t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(t.cpu().numpy(), ref[k])
    del graph
    eng.close()


def solve(P, s, o, v, naux, **kw):
    eng = P.PPL(o, v, naux, hbm_budget=1 << 30, diis_max=4, **kw)
    t = torch.zeros((o, o, v, v), dtype=torch.float64, device="cuda")
    rep = eng.iterate(dev(s["L"]), dev(s["e_occ"]), dev(s["e_vir"]), t, max_sweeps=8, tol=0.0,
                      fail_on_noconv=False, diis=4)
    return eng, t.cpu().numpy(), rep


def test_plans_beyond_the_pinned_slots(P):
    """A plan that finds no free slot copies its sums from the workspace: the same numbers (start
    energy, symmetry check, residuals, DIIS products); a slot given back serves a later plan."""
    o, v, naux = 3, 12, 36
    s = S.make_system(o, v, naux, 7, "contractive")
    bad = s["L"].copy()
    bad[0, o, o + 1] += 1.0
    first = solve(P, s, o, v, naux)
    say(f"plans beyond the slots ({o},{v},{naux}), {first[0].info['workspace_bytes']} B each")
    _, hist, _ = O.jacobi_diis(s["L"], o, s["e_occ"], s["e_vir"], m=4, max_sweeps=8, tol=0.0)
    h, hr = np.array(first[2]["history"]), np.array(hist)
    big = hr > 1e-8                      # residuals agree to rounding until they approach it
    assert big.sum() >= 4 and np.all(np.abs(h[big] - hr[big]) <= 1e-6 * hr[big])
    held = [first[0]] + [P.PPL(o, v, naux, hbm_budget=1 << 30) for _ in range(300)]
    for k in range(2):
        eng, t, rep = solve(P, s, o, v, naux)
        assert np.array_equal(t, first[1]) and rep == first[2]
        e2, em = eng.mp2(dev(s["L"]), dev(s["e_occ"]), dev(s["e_vir"]))
        assert em == rep["energy_start"] and np.isfinite(e2.cpu().numpy()).all()
        with pytest.raises(P.PPLError):
            eng.build(dev(bad))
        eng.close()
        for h in held:
            h.close()
        held = []


def test_destroy_waits_for_no_other_work(P):
    """ppl_destroy frees host metadata: work of other streams is still running when it returns."""
    o, v, naux = 2, 8, 6
    say("destroy beside a busy stream")
    eng = P.PPL(o, v, naux)
    eng.build(dev(S.make_system(o, v, naux, 131)["L"]))
    a = torch.randn(6144, 6144, dtype=torch.float64, device="cuda")
    c = torch.empty_like(a)
    torch.mm(a, a, out=c)
    torch.cuda.synchronize()
    busy = torch.cuda.Stream()
    with torch.cuda.stream(busy):
        for _ in range(60):              # about 6.5 ms each
            torch.mm(a, a, out=c)
    plan, eng.plan = eng.plan, None
    P.ppl_destroy(plan)
    running = not busy.query()
    torch.cuda.synchronize()
    assert running
    eng.close()


def test_bind_and_destroy_beside_a_capture(P):
    """Plans come and go while another stream records a graph."""
    o, v, naux = 3, 9, 7
    say("destroy inside a capture")
    s = S.make_system(o, v, naux, 132)
    t = dev(S.make_amplitudes(o, v, 133))
    st = torch.cuda.Stream()
    eng = P.PPL(o, v, naux, stream=st)
    other = P.PPL(o, v, naux)
    eng.build(dev(s["L"]))
    other.build(dev(s["L"]))
    torch.cuda.synchronize()
    R = torch.empty_like(t)
    eng.contract(t, R)
    torch.cuda.synchronize()
    ref = R.cpu().numpy()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        plan, other.plan = other.plan, None
        P.ppl_destroy(plan)
        eng.contract(t, R)
    for _ in range(3):
        R.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(R.cpu().numpy(), ref)
    del graph
    other.close()
    eng.close()


def test_plans_of_several_threads(P):
    """Slots are taken and given back by several host threads at once: every solve reads its own."""
    import threading

    o, v, naux = 3, 12, 36
    say(f"solves in six threads ({o},{v},{naux})")
    systems = [S.make_system(o, v, naux, 140 + k, "contractive") for k in range(6)]
    ref = []
    for s in systems:
        eng, t, rep = solve(P, s, o, v, naux)
        eng.close()
        ref.append((t, rep))
    wrong = []

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(8):
                eng, t, rep = solve(P, systems[k], o, v, naux)
                torch.cuda.current_stream().synchronize()
                eng.close()
                if not np.array_equal(t, ref[k][0]) or rep != ref[k][1]:
                    wrong.append(k)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not wrong
