"""Sums that the host reads live in memory of the library. What a call only enqueues must not
depend on it: such work can outlive the plan."""
import sys

import numpy as np
import pytest

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
