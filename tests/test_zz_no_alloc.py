"""sr_frame_step_static, the entry point that allocates nothing (K-split partial sums in the
library's static device array): through the C ABI, against sr_frame_step on the graph's own
scratch, bit for bit, every node after every frame -- on two graphs in a row, the second smaller
than the first (the array keeps the first one's contents)."""
import numpy as np
import pytest

import workloads as W
from workloads.graphs import Node, Graph
from gpu_util import to_device

pytestmark = pytest.mark.gpu


def hires_at(size, frames):
    g = W.hires_sr(batch=1, frames=frames)
    f = 256 // size
    nodes = [n if n.name == "out" else Node(n.name, n.channels, n.height // f, n.width // f, n.act) for n in g.nodes]
    return Graph(f"hires_sr@{size}", nodes, g.edges, 1, frames, "bf16", g.out_node)


def run_pair(g, seed, T, options=None):
    """T frames through sr_frame_step (own scratch) and through sr_frame_step_static; returns the
    number of tiles with and without K-split."""
    import paper_1806_04965_amd as sr
    w, b, x = W.make_case(g, seed=seed, bias_scale=0.1, frames=T)
    ins = g.input_nodes()
    xd = [to_device(x[v], g.dtype) for v in ins]
    own = sr.SrGraph(g, options=options)
    stat = sr.SrGraph(g, options=options)
    nosplit = sr.SrGraph(g, options={**(options or {}), 3: 0})
    for d in (own, stat, nosplit):
        d.set_parameters(w, b)
    tiles, tiles_nosplit = own.work()["mfma_tiles"], nosplit.work()["mfma_tiles"]
    nosplit.close()
    with pytest.raises(sr.SrError) as ei:          # not planned / reset yet
        stat.frame_step_static([xi[1] for xi in xd])
    assert ei.value.name == "SR_ERR_STATE"
    own.reset([xi[0] for xi in xd])
    stat.reset([xi[0] for xi in xd])
    for t in range(1, T + 1):
        own.frame_step([xi[t] for xi in xd])
        stat.frame_step_static([xi[t] for xi in xd])
        own.synchronize()
        stat.synchronize()
        for v in range(len(g.nodes)):
            a = own.get_state(v).float().cpu().numpy()
            s = stat.get_state(v).float().cpu().numpy()
            assert np.isfinite(s).all()
            np.testing.assert_array_equal(s, a, err_msg=f"{g.name} node {v} frame {t}")
        assert float(np.abs(stat.get_state(g.out_node).float().cpu().numpy()).max()) > 0
    assert stat.frame_index() == T
    own.close()
    stat.close()
    return tiles, tiles_nosplit


def test_static_scratch_matches_own_scratch_two_graphs_second_smaller():
    # first the full 256x256 high-resolution graph (about 300 parts, 38 MiB of partial sums), then
    # the same graph at 64x64 and the CIFAR-shaped one at batch 4, both much smaller
    t_big, t_big_ns = run_pair(W.hires_sr(batch=1, frames=3), seed=3, T=3)
    assert t_big > t_big_ns, "the first graph must have K-split tiles"
    t_small, t_small_ns = run_pair(hires_at(64, 3), seed=4, T=3)
    assert t_small > t_small_ns, "the second graph must have K-split tiles"
    assert t_small < t_big
    t_c, t_c_ns = run_pair(W.cifar_sr(batch=4, frames=4), seed=5, T=4)
    assert t_c > t_c_ns


def test_static_scratch_with_a_dependency_driven_graph():
    # sequential pattern: all update steps of a frame in one launch, ordered by completion counters
    import paper_1806_04965_amd as sr
    g0 = W.cifar_sr(batch=4, frames=3)
    g = g0.with_pattern(W.sequential_pattern(g0))
    dev = sr.SrGraph(g)
    w, b, _ = W.make_case(g, seed=7)
    dev.set_parameters(w, b)
    assert dev.health()["dependency_driven"]
    dev.close()
    run_pair(g, seed=7, T=3)


def test_static_scratch_with_the_eight_wave_kernel():
    run_pair(hires_at(64, 2), seed=6, T=2, options={4: 2})


def test_static_scratch_refuses_what_does_not_fit():
    # 200 nodes of 4x4 pixels, each fed by four 512-channel inputs through 3x3 edges: 200 one-tile nodes
    # with a contraction of 18432, every one cut into parts -- more partial sums than the array holds.
    # The call must say so, leave the graph as it was, and sr_frame_step must still serve it.
    import paper_1806_04965_amd as sr
    from workloads.graphs import Edge, ACT_IDENTITY
    n_in, n_hidden = 4, 200
    nodes = [Node(f"in{i}", 512, 4, 4, ACT_IDENTITY) for i in range(n_in)]
    nodes += [Node(f"h{i}", 32, 4, 4) for i in range(n_hidden)]
    nodes.append(Node("out", 10, 1, 1, ACT_IDENTITY))
    edges = [Edge(i, n_in + h) for h in range(n_hidden) for i in range(n_in)]
    edges.append(Edge(n_in, n_in + n_hidden, "gap_dense", 1, 1, 1, 0))
    g = Graph("many_deep_nodes", nodes, edges, 1, 1, "bf16", out_node=n_in + n_hidden)
    w, b, x = W.make_case(g, seed=7, frames=1)
    xd = [to_device(x[v], g.dtype) for v in g.input_nodes()]
    dev = sr.SrGraph(g)
    dev.set_parameters(w, b)
    dev.reset([xi[0] for xi in xd])
    with pytest.raises(sr.SrError) as ei:
        dev.frame_step_static([xi[1] for xi in xd])
    assert ei.value.name == "SR_ERR_ARG" and "static scratch holds" in str(ei.value), str(ei.value)
    assert dev.frame_index() == 0
    dev.frame_step([xi[1] for xi in xd])
    dev.synchronize()
    assert dev.frame_index() == 1
    assert float(dev.get_state(n_in + 1).float().abs().max()) > 0
    dev.close()


GRAPHS = {
    "bf16 streaming": lambda: W.cifar_sr(batch=2, frames=9),
    "bf16 sequential, dependency-driven": lambda: _with(W.cifar_sr(batch=2, frames=9), W.sequential_pattern),
    "bf16 hybrid, a launch per update step": lambda: _with(W.cifar_sr(batch=2, frames=9), W.hybrid_pattern),
    "f32 streaming": lambda: W.tiny_sr(batch=2, frames=9),
    "f32 sequential": lambda: _with(W.tiny_sr(batch=2, frames=9), W.sequential_pattern),
}


def _with(g, pattern):
    return g.with_pattern(pattern(g))


@pytest.mark.parametrize("hidden_node_recorded", [False, True])
@pytest.mark.parametrize("calls", [1, 2])
@pytest.mark.parametrize("name", list(GRAPHS))
def test_replays_of_recorded_calls_go_on_with_the_stream(name, calls, hidden_node_recorded):
    # `calls` frames recorded once and replayed, the caller's input buffer refilled before each replay, with frames of
    # ordinary calls and other GPU work between the replays: every node after every frame as without recording, bit for bit
    import torch
    import paper_1806_04965_amd as sr
    g = GRAPHS[name]()
    T = 9
    w, b, x = W.make_case(g, seed=21, bias_scale=0.1, frames=T)
    xd = [to_device(x[v], g.dtype) for v in g.input_nodes()]
    options = {5: 0} if "launch per" in name else None
    ref, dev = sr.SrGraph(g, options=options), sr.SrGraph(g, options=options)
    for d in (ref, dev):
        d.set_parameters(w, b)
        if hidden_node_recorded:     # leaves the graph with a copy launch behind every frame
            out = torch.empty((1, g.batch, g.nodes[1].height, g.nodes[1].width, g.nodes[1].channels), dtype=d.tdtype, device="cuda")
            d.rollout([t[:2].contiguous() for t in xd], 1, 1, out)
            d.synchronize()
        d.reset([t[0] for t in xd])
    buf = [[t[0].clone() for t in xd] for _ in range(calls)]
    recording = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(recording, stream=dev.stream):
        for k in range(calls):
            dev.frame_step_static(buf[k])
    t = 0

    def same(t):
        for v in range(len(g.nodes)):
            assert torch.equal(dev.get_state(v), ref.get_state(v)), (name, t, v)

    def eager(t):
        ref.frame_step([xi[t] for xi in xd])

    while t + calls < T:
        for k in range(calls):
            for dst, src in zip(buf[k], xd):
                dst.copy_(src[t + 1 + k])
        torch.cuda.synchronize()
        with torch.cuda.stream(dev.stream):
            recording.replay()
        torch.cuda.synchronize()
        for _ in range(calls):
            t += 1
            eager(t)
        ref.synchronize()
        same(t)
        torch.ones(1 << 20, device="cuda").cumsum(0)
        if t in (3, 4, 7):            # an ordinary call between two replays
            t += 1
            (dev.frame_step if t % 2 else dev.frame_step_static)([xi[t] for xi in xd])
            eager(t)
            ref.synchronize()
            dev.synchronize()
            same(t)
    state = ref.get_state(1)          # set_state goes to the copy the next frame reads
    dev.set_state(1, state)
    ref.set_state(1, state)
    same(t)
    assert dev.health()["dependency_timeouts"] == 0
    dev.reset([xi[0] for xi in xd])
    ref.reset([xi[0] for xi in xd])
    dev.frame_step([xi[1] for xi in xd])
    eager(1)
    ref.synchronize()
    dev.synchronize()
    same(1)
    ref.close()
    dev.close()


@pytest.mark.parametrize("what", ["reset and a frame", "rollout"])
@pytest.mark.parametrize("name", ["bf16 streaming", "bf16 sequential, dependency-driven", "f32 sequential"])
def test_replays_that_start_again_from_frame_0(name, what):
    # a recording that resets: a replay puts the stream back to frame 1 (rollout: 2) whatever has been computed since, and
    # ordinary frames go on from there
    import torch
    import paper_1806_04965_amd as sr
    g = GRAPHS[name]()
    w, b, x = W.make_case(g, seed=22, bias_scale=0.1, frames=9)
    xd = [to_device(x[v], g.dtype) for v in g.input_nodes()]
    ref, dev = sr.SrGraph(g), sr.SrGraph(g)
    for d in (ref, dev):
        d.set_parameters(w, b)
        d.reset([t[0] for t in xd])
    recorded = 1 if what == "reset and a frame" else 2
    out = torch.zeros((2, g.batch, 1, 1, g.nodes[g.out_node].channels), dtype=dev.tdtype, device="cuda")
    head = [t[:3].contiguous() for t in xd]
    dev.rollout(head, 2, g.out_node, out)     # (the recorded node is set: a rollout that changes it copies a table)
    dev.synchronize()
    recording = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(recording, stream=dev.stream):
        if recorded == 1:
            dev.reset([t[0] for t in xd])
            dev.frame_step_static([t[1] for t in xd])
        else:
            dev.rollout(head, 2, g.out_node, out)
    for more in (0, 1, 2, 3):
        out.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(dev.stream):
            recording.replay()
        torch.cuda.synchronize()
        ref.reset([t[0] for t in xd])
        for t in range(1, recorded + more + 1):
            ref.frame_step([xi[t] for xi in xd])
            if t > recorded:
                dev.frame_step([xi[t] for xi in xd])
            if t <= 2 and recorded == 2:
                ref.synchronize()
                assert torch.equal(out[t - 1].flatten(), ref.get_state(g.out_node).flatten()), (name, more, t)
        ref.synchronize()
        dev.synchronize()
        for v in range(len(g.nodes)):
            assert torch.equal(dev.get_state(v), ref.get_state(v)), (name, more, v)
    assert dev.health()["dependency_timeouts"] == 0
    ref.close()
    dev.close()


@pytest.mark.parametrize("pattern", [W.sequential_pattern, W.hybrid_pattern])
def test_replays_of_recorded_rollouts_between_rollouts_of_other_lengths(pattern):
    # a dependency-driven launch of several frames takes its work items in an order that is written for its number of frames:
    # recordings of two lengths bring their own along, and ordinary rollouts between the replays write theirs again.  All equal
    # one launch per update step, bit for bit.
    import torch
    import paper_1806_04965_amd as sr
    g0 = W.cifar_sr(batch=2, frames=70)
    g = g0.with_pattern(pattern(g0))
    w, b, x = W.make_case(g, seed=23, bias_scale=0.1, frames=70)
    xd = [to_device(x[v], g.dtype) for v in g.input_nodes()]
    classes = g.nodes[g.out_node].channels
    ref, dev = sr.SrGraph(g, options={5: 0}), sr.SrGraph(g)
    want = torch.zeros((70, g.batch, 1, 1, classes), dtype=dev.tdtype, device="cuda")
    for d in (ref, dev):
        d.set_parameters(w, b)
    ref.rollout(xd, 70, g.out_node, want)
    ref.synchronize()
    assert float(want[-1].abs().max()) > 0

    def ordinary(T):
        out = torch.zeros((T, g.batch, 1, 1, classes), dtype=dev.tdtype, device="cuda")
        dev.rollout([t[:T + 1].contiguous() for t in xd], T, g.out_node, out)
        dev.synchronize()
        assert torch.equal(out, want[:T]), T

    ordinary(20)                       # the order of the first recording's length is there when it is recorded
    recordings = []
    for T in (20, 7):
        out, head = torch.zeros((T, g.batch, 1, 1, classes), dtype=dev.tdtype, device="cuda"), [t[:T + 1].contiguous() for t in xd]
        recording = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(recording, stream=dev.stream):
            dev.rollout(head, T, g.out_node, out)
        recordings.append((recording, out, head))
    for turn, lengths in enumerate([(), (70,), (20,), (7, 3), (64, 2, 20), (1,), (33, 70)]):
        for T in lengths:
            ordinary(T)
        for recording, out, _ in recordings if turn % 2 else recordings[::-1]:
            out.zero_()
            torch.ones(1 << 20, device="cuda").cumsum(0)
            torch.cuda.synchronize()
            with torch.cuda.stream(dev.stream):
                recording.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want[:out.shape[0]]), (turn, out.shape[0])
    h = dev.health()
    assert h["dependency_driven"] and h["dependency_timeouts"] == 0
    ref.close()
    dev.close()
