"""Batched calls of one plan that follow each other without a synchronisation:
on another stream (each call's workspace and staging are the plan's), with
another graph while the last call's is still replayed, and a plan that ends
behind its last call.  Each against the same calls with the device idle in
between, bit for bit."""
import numpy as np
import pytest

from paper_2602_13385_amd import inputs as I

pytestmark = pytest.mark.gpu

HOST = (I.CONFIG4_HOST, 1.0)
SIZES = [3_000, 1, 40_000, 700]


def _inputs(torch, seed):
    off = np.concatenate([[0], np.cumsum(SIZES)]).astype(np.int64)
    st = np.concatenate([I.plummer(max(n, 2), seed + i).state()[:, :n]
                         for i, n in enumerate(SIZES)], axis=1).astype(np.float32)
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda")
    cen = np.array([[18.0 + i, -4.0, 2.5, 0.3, 1.2, 0.2] for i in range(len(SIZES))])
    return off, [dev(st[i]) for i in range(6)], dev(np.full(st.shape[1], 1e-4, np.float32)), cen


def _calls(torch, plan, streams, graphs, idle):
    """One call per stream on inputs of its own: (steps, dt) differ from call to call."""
    out = []
    args = [(_inputs(torch, 7500 + 10 * k), 60 + 7 * k, 1e-3 * (1 + k)) for k in range(len(streams))]
    torch.cuda.synchronize()
    for (inp, nsteps, dt), s, g in zip(args, streams, graphs):
        off, st, m, cen = inp
        with torch.cuda.stream(s):
            c, acc = plan.step_batched(off, st, m, dt, nsteps, host=HOST, centres=cen, graph=g)
        if idle:
            torch.cuda.synchronize()
        out.append((st, acc, c))
    torch.cuda.synchronize()
    return [(np.stack([t.cpu().numpy() for t in st + acc]), c) for st, acc, c in out]


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("same_stream", [False, True])
def test_calls_in_a_row(graph, same_stream):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13385_amd import scf as S
    print(f"[batched streams] graph={graph} same_stream={same_stream}", flush=True)
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    streams = [a, a, a, a] if same_stream else [a, b, a, b]
    graphs = [graph] * 4
    plan = S.Plan(6, 4)
    _calls(torch, plan, streams, graphs, True)  # code loaded, buffers allocated
    ref = _calls(torch, S.Plan(6, 4), streams, graphs, True)
    for _ in range(3):
        got = _calls(torch, plan, streams, graphs, False)
        for (x, c), (y, d) in zip(got, ref):
            assert np.array_equal(x, y) and np.array_equal(c, d)


def test_a_plan_ends_behind_its_last_call():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_13385_amd import scf as S
    print("[batched streams] plan destroyed", flush=True)
    off, st0, m, cen = _inputs(torch, 7600)
    out = []
    for idle in (True, False):
        plan, st = S.Plan(6, 4), [t.clone() for t in st0]
        _, acc = plan.step_batched(off, st, m, 1e-3, 60, host=HOST, centres=cen, graph=True)
        if idle:
            torch.cuda.synchronize()
        del plan
        torch.cuda.synchronize()
        out.append(np.stack([t.cpu().numpy() for t in st + acc]))
    assert np.array_equal(*out)
