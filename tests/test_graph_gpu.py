"""The hot path captured in a HIP graph replays bit for bit.

After one call with the same problem on the same stream (which sizes the
workspace and stages the offsets), class_quantile, dro_cost_eval and
dro_argmin_reservation enqueue kernels only: no allocation, no host copy and
no memset node, so the step can be captured (torch.cuda.graph) and replayed.
Every replay is checked against the eager results, with eager calls of the
same step between replays: a one-class workload, ragged aliased segments
(one block per sample slice) and ratios-8x250k (the persistent grid that
claims slices, whose claim counters a fill kernel in the graph clears).

dro_cost_eval_noalloc enqueues kernels only on its first call too, and its
replays depend on no host memory: it is captured without an earlier call on
segments of unequal sizes (which are counted through a row table), and replayed
after other unequal segments were evaluated on the same context, after the
caller's host arrays were overwritten and after the context was closed.
"""
import pytest

from workloads import make_workload, random_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["lognormal-1x1k", "random", "ratios-8x250k"])
def test_captured_step_replays_bit_for_bit(dev, name):
    import torch
    import paper_2607_16892_amd as dro
    w = (make_workload(name) if name != "random" else
         random_workload(seed=61, C=5, N=(700, 33, 1500), alias=True, L=2000, K=97, M=40, E=3))
    print(f"[gpu] graph {w.name}: C={w.C} K={w.K} M={w.M} E={w.E}", flush=True)
    with dro.Context(dev.index or 0) as ctx:
        prob = dro.Problem.from_workload(w, dev)
        eps = torch.from_numpy(w.eps.copy()).to(dev)
        out = dict(S=torch.empty((w.C, w.K, w.M), dtype=torch.float64, device=dev),
                   W=torch.empty((w.E, w.C, w.K), dtype=torch.float64, device=dev),
                   m_star=torch.empty((w.E, w.C, w.K), dtype=torch.int32, device=dev),
                   q_value=torch.empty(w.C, dtype=torch.int32, device=dev),
                   q_rank=torch.empty(w.C, dtype=torch.int64, device=dev),
                   k_star=torch.empty((w.E, w.C), dtype=torch.int32, device=dev),
                   W_star=torch.empty((w.E, w.C), dtype=torch.float64, device=dev),
                   m_at_star=torch.empty((w.E, w.C), dtype=torch.int32, device=dev))

        def step():
            dro.class_quantile(ctx, prob, q_value=out["q_value"], q_rank=out["q_rank"])
            dro.dro_cost_eval(ctx, prob, eps, W=out["W"], m_star=out["m_star"], S=out["S"])
            dro.dro_argmin_reservation(ctx, prob, eps, out["S"], k_star=out["k_star"],
                                       W_star=out["W_star"], m_at_star=out["m_at_star"])

        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            step()  # sizes the workspace and stages the offsets for this stream
        torch.cuda.current_stream().wait_stream(s)
        torch.cuda.synchronize()
        ref = {k: v.clone() for k, v in out.items()}
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            step()
        torch.cuda.synchronize()

        def bits(t):
            return t.view(torch.int64) if t.dtype == torch.float64 else t

        for rep in range(3):
            for t in out.values():
                t.fill_(-7)
            g.replay()
            torch.cuda.synchronize()
            for k in out:
                assert torch.equal(bits(out[k]), bits(ref[k])), f"replay {rep}: {k} differs"
            with torch.cuda.stream(s):
                step()  # eager work between replays
            torch.cuda.synchronize()
            for k in out:
                assert torch.equal(bits(out[k]), bits(ref[k])), f"eager after replay {rep}: {k}"


@pytest.mark.parametrize("C,alias", [(3, False), (5, True), (4500, True)])
def test_captured_noalloc_replays_without_its_host_arrays(dev, C, alias):
    import torch
    import paper_2607_16892_amd as dro
    # three segments of 3, 1 and 5 parts, and others whose parts are 1, 13 and 1
    w = random_workload(seed=62, C=C, N=(40_000, 3, 70_000), alias=alias, L=2000, K=13, M=7, E=2)
    other = random_workload(seed=63, C=3, N=(90, 200_000, 1), L=2000, K=9, M=4, E=1)
    print(f"[gpu] no-alloc graph: C={w.C} S={w.offsets.size - 1}", flush=True)

    def outputs(w):
        return dict(S=torch.empty((w.C, w.K, w.M), dtype=torch.float64, device=dev),
                    W=torch.empty((w.E, w.C, w.K), dtype=torch.float64, device=dev),
                    m_star=torch.empty((w.E, w.C, w.K), dtype=torch.int32, device=dev))

    def run(ctx, prob, eps, out):
        dro.dro_cost_eval_noalloc(ctx, prob, eps, out["S"], out["W"], out["m_star"])

    ctx = dro.Context(dev.index or 0)
    prob, prob2 = dro.Problem.from_workload(w, dev), dro.Problem.from_workload(other, dev)
    eps, eps2 = (torch.from_numpy(x.eps.copy()).to(dev) for x in (w, other))
    ref, ref2 = dro.dro_cost_eval(ctx, prob, eps), dro.dro_cost_eval(ctx, prob2, eps2)
    out, out2 = outputs(w), outputs(other)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        run(ctx, prob, eps, out)
    torch.cuda.synchronize()

    def replay(when):
        for t in out.values():
            t.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        for k in out:
            assert torch.equal(out[k], ref[k]), f"{when}: {k} differs"

    replay("first replay")
    for _ in range(2):
        run(ctx, prob2, eps2, out2)  # eager, with another row table
        torch.cuda.synchronize()
        for k in out2:
            assert torch.equal(out2[k], ref2[k]), f"eager: {k} differs"
        replay("after another problem")
    prob.offsets_h[1:] = 1
    if prob.seg_h is not None:
        prob.seg_h[:] = 0
    replay("after the host arrays changed")
    ctx.close()
    replay("after the context was closed")
