"""The entry points are plain asynchronous launches on the caller's stream, so a whole step can be
recorded into a HIP graph and replayed.  Checked here: every replay reproduces the eager results
bit for bit (the kernels are deterministic), with eager work and synchronisations between replays."""
import numpy as np
import pytest

from paper_2501_13986_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_step_replays_from_a_hip_graph():
    from paper_2501_13986_amd import binding as b
    irr = (synth.MACE_X, synth.MACE_Y, synth.MACE_Z)
    plan = b.Plan(*irr, dtype=b.CGTP_F32, device=0)
    DX, DY, DZ, NW = plan.dim_x, plan.dim_y, plan.dim_z, plan.n_w
    B, V = 777, 300
    recv, send, unit = synth.periodic_graph(11, V, 20.0)
    E = recv.shape[0]
    print(f"graph capture: B={B} V={V} E={E} entries=tp_forward/tp_backward/conv_forward/conv_backward", flush=True)
    dev = "cuda"
    row_ptr, col, perm, t_row_ptr, t_perm = b.cgtp_csr_from_coo(torch.from_numpy(recv).to(dev), torch.from_numpy(send).to(dev), V)
    g = torch.Generator(device=dev)
    g.manual_seed(5)
    rnd = lambda *shape: torch.randn(shape, generator=g, device=dev, dtype=torch.float32)
    x, y, W, gz = rnd(B, DX), rnd(B, DY), rnd(B, NW), rnd(B, DZ)
    xn, ye, We, gzn = rnd(V, DX), rnd(E, DY), rnd(E, NW), rnd(V, DZ)
    outs = {"z": torch.empty(B, DZ, device=dev), "gx": torch.empty(B, DX, device=dev), "gy": torch.empty(B, DY, device=dev),
            "gW": torch.empty(B, NW, device=dev), "zn": torch.empty(V, DZ, device=dev), "gxn": torch.empty(V, DX, device=dev),
            "gye": torch.empty(E, DY, device=dev), "gWe": torch.empty(E, NW, device=dev)}

    def step():
        b.tp_forward(plan, x, y, W, outs["z"])
        b.tp_backward(plan, x, y, W, gz, outs["gx"], outs["gy"], outs["gW"])
        b.conv_forward(plan, xn, ye, We, outs["zn"], row_ptr, col)
        b.conv_backward(plan, xn, ye, We, gzn, outs["gxn"], outs["gye"], outs["gWe"], row_ptr, col, t_row_ptr, t_perm)

    step()                       # eager: also sizes the plan's workspace, which must not grow during capture
    torch.cuda.synchronize()
    eager = {k: v.clone() for k, v in outs.items()}
    side = torch.cuda.Stream()   # default priority
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        step()                   # warm-up on the capture stream
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for rep in range(3):
        for v in outs.values():
            v.fill_(float("nan"))            # eager work between replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for k in outs:
            assert torch.equal(outs[k], eager[k]), (rep, k)


def test_second_order_pass_captured_on_a_larger_graph():
    """The workspace of a smaller graph's call serves the larger graph (two rows for each of at most 16 384 workers and 44 000
    receiver ids), and what the one-walk form needs beyond it is part of the captured graph's own memory: the same bits as
    eager, and whatever the plan was used for before."""
    from paper_2501_13986_amd import binding as b
    new_plan = lambda: b.Plan("32x0e+32x1o", "1x0e+1x1o", "32x0e+32x1o", dtype=b.CGTP_F32, device=0)
    plan = new_plan()
    DX, DY, DZ, NW = plan.dim_x, plan.dim_y, plan.dim_z, plan.n_w

    def problem(E, V=500):
        g = torch.Generator(device="cuda")
        g.manual_seed(E)
        rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda")
        recv, send = (torch.randint(0, V, (E,), generator=g, device="cuda") for _ in range(2))
        row_ptr, col, _, t_row_ptr, t_perm = b.cgtp_csr_from_coo(recv, send, V)
        ins = [rnd(V, DX), rnd(E, DY), rnd(E, NW), rnd(V, DZ), rnd(V, DX), rnd(E, DY), rnd(E, NW)]
        outs = [torch.full(s, float("nan"), device="cuda") for s in ((V, DX), (E, DY), (E, NW), (V, DZ))]
        return ins, outs, (row_ptr, col, t_row_ptr, t_perm)

    small, large = problem(40000), problem(44000)
    call = lambda p, plan: b.conv_double_backward(plan, *p[0], *p[1], *p[2])
    assert b.lib().cgtp_conv_double_workspace_bytes(plan._h, 500, 44000) >= 44000 * DX * 4
    print("capture of conv_double_backward E=44000 after E=40000", flush=True)
    call(large, new_plan())
    torch.cuda.synchronize()
    eager = [v.clone() for v in large[1]]
    side = torch.cuda.Stream()   # default priority
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        call(small, plan)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            call(large, plan)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    for rep in range(3):
        for v in large[1]:
            v.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, e) for a, e in zip(large[1], eager)), rep
        call(small, plan)        # eager work between the replays: leaves the graph's memory alone
        torch.cuda.synchronize()


# larger and smaller graph: either side of a doubling of the windows (513 and 1 024 of them), and the backward by rows (15 000 of
# them) against the one by edge ranges, which leave more pieces
@pytest.mark.parametrize("large,small", [((500, 131073), (500, 131072)), ((15000, 420000), (500, 400000))])
def test_a_larger_graphs_workspace_serves_a_smaller_one(large, small):
    """A capture of the smaller graph after an eager call on the larger one allocates nothing; an eager call on the smaller
    one leaves the buffer that a captured step on the larger one uses."""
    from paper_2501_13986_amd import binding as b
    plan = b.Plan("32x0e+32x1o", "1x0e+1x1o", "32x0e+32x1o", dtype=b.CGTP_F32, device=0)
    DX, DY, DZ, NW = plan.dim_x, plan.dim_y, plan.dim_z, plan.n_w
    print(f"capture and eager calls of conv_forward/conv_backward {large} {small}", flush=True)

    def problem(V, E):
        g = torch.Generator(device="cuda")
        g.manual_seed(E)
        rnd = lambda *shape: torch.randn(shape, generator=g, device="cuda")
        recv, send = (torch.randint(0, V, (E,), generator=g, device="cuda") for _ in range(2))
        row_ptr, col, _, t_row_ptr, t_perm = b.cgtp_csr_from_coo(recv, send, V)
        ins, gz = [rnd(V, DX), rnd(E, DY), rnd(E, NW)], rnd(V, DZ)
        outs = [torch.full(s, float("nan"), device="cuda") for s in ((V, DZ), (V, DX), (E, DY), (E, NW))]

        def step():
            b.conv_forward(plan, *ins, outs[0], row_ptr, col)
            b.conv_backward(plan, *ins, gz, *outs[1:], row_ptr, col, t_row_ptr, t_perm)
        return step, outs

    def clear(outs):
        for v in outs:
            v.fill_(float("nan"))
        torch.cuda.synchronize()

    (step_l, out_l), (step_s, out_s) = problem(*large), problem(*small)
    step_l()
    torch.cuda.synchronize()
    want_l = [v.clone() for v in out_l]
    side = torch.cuda.Stream()   # default priority
    side.wait_stream(torch.cuda.current_stream())
    graph_s, graph_l = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph_s, stream=side):
        step_s()
    with torch.cuda.graph(graph_l, stream=side):
        step_l()
    torch.cuda.synchronize()
    clear(out_s)
    step_s()
    torch.cuda.synchronize()
    want_s = [v.clone() for v in out_s]
    assert all(bool(torch.isfinite(v).all()) for v in want_l + want_s)
    for rep in range(3):
        for graph, out, want in ((graph_l, out_l, want_l), (graph_s, out_s, want_s)):
            clear(out)
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, w) for a, w in zip(out, want)), rep
        step_s()      # eager work between the replays
