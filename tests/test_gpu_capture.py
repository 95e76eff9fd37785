"""Steps of a run or batch on a stream that is being captured: refused unless the run was
made with UBQP_NO_GRAPH or UBQP_TIMING, and then every replay of the graph is one more
generation, up to G; later replays change neither the results nor memory behind them
(the rows of the dump past G keep their fill).  All values are integers and equal the
oracle's."""
import numpy as np
import pytest

import oracle
from paper_1706_00037_amd.inputs import make_instance

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
G = 3


@pytest.fixture(scope="module")
def ub():
    from paper_1706_00037_amd import ubqp
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return ubqp


def case(n, M, lo=-100, hi=100):
    return make_instance(n, 0.4, lo, hi, 300 + n), dict(M=M, H=4, lam_num=1, lam_den=2, G=G, run_seed=n)


def check(r, want, g):
    done = min(g, G)
    assert r["generations"] == done
    assert np.array_equal(r["stats"], want["stats"][:done])
    assert np.isnan(r["gen_ms"]).all()
    if g >= G:
        assert r["best_f"] == want["best_f"] and np.array_equal(r["best_x"], want["best_x"])


def eager_work():
    assert int(torch.arange(1 << 18, device="cuda").sum()) == (1 << 18) * ((1 << 18) - 1) // 2
    torch.cuda.synchronize()


def test_capture_is_refused_without_the_flag(ub):
    Q, kw = case(150, 300)
    want = oracle.multistart(Q, threads=8, **kw)
    ctx = ub.Context(0)
    prob = ctx.problem(Q)
    run, batch = ctx.run(prob, **kw), ctx.batch([prob, prob], [kw, kw])
    y = torch.zeros(4, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y += 1
        for h in (run, batch):
            with pytest.raises(ub.UbqpError) as e:
                h.step(1)
            assert e.value.code == ub.UBQP_EDEVICE
    graph.replay()
    torch.cuda.synchronize()
    run.step(G)
    batch.step(G)
    for r in (run.result(), batch.result(0), batch.result(1)):
        assert np.array_equal(r["stats"], want["stats"]) and r["best_f"] == want["best_f"]
        assert np.isfinite(r["gen_ms"]).all()


@pytest.mark.parametrize("flag", ["UBQP_NO_GRAPH", "UBQP_TIMING"])
@pytest.mark.parametrize("n,M,lo,hi", [(150, 300, -100, 100), (3200, 100, -100, 100), (90, 16500, -30000, 30000)])
def test_replays_of_a_captured_run(ub, n, M, lo, hi, flag):
    Q, kw = case(n, M, lo, hi)
    want = oracle.multistart(Q, dump=True, threads=8, **kw)
    ctx = ub.Context(0)
    dump = torch.full((G + 2, M), -7, dtype=torch.int64, device="cuda")
    run = ctx.run(ctx.problem(Q), f_dump=dump, flags=getattr(ub, flag), **kw)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run.step(1)
    check(run.result(), want, 0)
    for g in range(1, G + 3):
        graph.replay()
        torch.cuda.synchronize()
        check(run.result(), want, g)
        eager_work()
    got = dump.cpu().numpy()
    assert np.array_equal(got[:G], want["f_all"]) and (got[G:] == -7).all()


def test_replays_of_a_captured_batch(ub):
    """Lane ranges of one to four blocks, so the captured generation forks to side streams."""
    cases = [case(200, 300), case(1100, 200), case(2100, 120, -30000, 30000), case(3200, 64)]
    want = [oracle.multistart(Q, threads=8, **kw) for Q, kw in cases]
    ctx = ub.Context(0)
    batch = ctx.batch([ctx.problem(Q) for Q, _ in cases], [dict(kw, flags=ub.UBQP_NO_GRAPH) for _, kw in cases])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        batch.step(1)
    for g in range(1, G + 3):
        graph.replay()
        torch.cuda.synchronize()
        for k, w in enumerate(want):
            check(batch.result(k), w, g)
        eager_work()
