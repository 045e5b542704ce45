"""GPU parity: the HIP library (through its C ABI) against the CPU oracle, element by element, on
the same seeded inputs.  Tolerances: max-abs-rel <= 1e-4 for fp32 graphs (oracle in float64),
<= 2e-2 for bf16 graphs (oracle emulating the bf16 storage points)."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from workloads.graphs import Node, Edge, Graph, ACT_IDENTITY, ACT_RELU
from gpu_util import (gpu_states_by_steps, gpu_rollout, oracle_states, compare_all, max_abs_rel,
                      to_device as to_device_)

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}
MODE = {"f32": "f64", "bf16": "bf16"}
OPT_DIRECT = {1: 1}
OPT_EAGER = {0: 0}
OPT_WIDE = {4: 2}     # 8-wave tile kernel (both operands through LDS, stages loaded one ahead)


def check(g, seed=0, T=None, options=None, bias_scale=0.1, label=None):
    T = g.frames if T is None else T
    w, b, x = W.make_case(g, seed=seed, bias_scale=bias_scale, frames=T)
    got, info, work = gpu_states_by_steps(g, w, b, x, T, options)
    ref = oracle_states(g, w, b, x, T, MODE[g.dtype])
    worst = compare_all(got, ref, TOL[g.dtype], label or g.name)
    print(f"[parity] {label or g.name}: worst max-abs-rel {worst:.3e} (tol {TOL[g.dtype]}), "
          f"F(R)={info['inference_factor']}, mfma tiles={work['mfma_tiles']}", flush=True)
    return info, work


def test_tiny_sr_fp32_streaming_all_nodes_all_frames():
    g = W.tiny_sr()
    info, _ = check(g)
    assert info["inference_factor"] == 1


@pytest.mark.parametrize("pattern", ["sequential", "hybrid"])
def test_tiny_sr_fp32_other_patterns(pattern):
    g = W.tiny_sr()
    bits = W.sequential_pattern(g) if pattern == "sequential" else W.hybrid_pattern(g)
    check(g.with_pattern(bits), label=f"tiny_sr/{pattern}")


def test_mnist_sr_net_fp32_conv7_stride4_and_dense_edges():
    check(W.mnist_net("SR", batch=3, frames=5))


def test_cifar_small_bf16_direct_kernel():
    g = W.cifar_sr(batch=2, frames=4)
    _, work = check(g, options=OPT_DIRECT, label="cifar_sr/direct")
    assert work["mfma_tiles"] == 0


def test_cifar_small_bf16_mfma_streaming():
    g = W.cifar_sr(batch=4, frames=6)
    info, work = check(g)
    assert work["mfma_tiles"] > 0 and info["inference_factor"] == 1


def test_cifar_ragged_batch_bf16_mfma():
    # B=3: nodes 5 and 6 have 192 pixels, less than one 256-pixel tile; nodes 3, 4 end in a partial tile
    check(W.cifar_sr(batch=3, frames=4), seed=3, label="cifar_sr/B3")


@pytest.mark.parametrize("pattern", ["sequential", "hybrid"])
def test_cifar_patterns_bf16_mfma(pattern):
    g = W.cifar_patterns(batch=4, frames=5)[pattern]
    info, work = check(g, label=g.name)
    assert work["mfma_tiles"] > 0
    assert info["inference_factor"] == (7 if pattern == "sequential" else info["inference_factor"])


def test_gtsrb_small_bf16_mfma_feedback_and_long_skips():
    check(W.gtsrb_sr(batch=2, frames=4), seed=1)


def test_dsr2_bf16_conv5_and_stride4():
    check(W.dsr_net(2, batch=2, frames=5), seed=2)


def test_hires_reduced_bf16_mfma():
    # the high-resolution graph at 64x64 input (same nodes, edges and channel schedule)
    g = W.hires_sr(batch=1, frames=3)
    nodes = []
    for n in g.nodes:
        if n.name == "out":
            nodes.append(n)
        else:
            nodes.append(Node(n.name, n.channels, n.height // 4, n.width // 4, n.act))
    g2 = Graph("hires_sr", nodes, g.edges, 1, 3, "bf16", g.out_node)
    check(g2, seed=4, label="hires_sr/64x64")


def test_gap_head_with_several_pixel_slabs():
    # 24x24 source -> 576 pixels per image: the head sums 9 slabs, the last one to finish combines them
    nodes = [Node("in", 3, 24, 24, ACT_IDENTITY), Node("a", 32, 24, 24), Node("out", 7, 1, 1, ACT_IDENTITY)]
    edges = [Edge(0, 1), Edge(1, 1), Edge(1, 2, "gap_dense", 1, 1, 1, 0)]
    for dtype in ("bf16", "f32"):
        g = Graph("gap", nodes, edges, batch=3, frames=4, dtype=dtype, out_node=2)
        check(g, seed=8, label=f"gap_head/{dtype}")
        check(g.with_pattern([0, 1, 0]), seed=8, label=f"gap_head/{dtype}/sequential")


def test_k_split_on_and_off_agree_with_the_oracle():
    # deep nodes with few pixels are cut along the contraction; with the option off they are not
    g = W.cifar_sr(batch=4, frames=5)
    _, work_on = check(g, seed=11, label="cifar_sr/k-split on")
    _, work_off = check(g, seed=11, options={3: 0}, label="cifar_sr/k-split off")
    assert work_on["mfma_tiles"] > work_off["mfma_tiles"]


def test_recording_a_hidden_node():
    g = W.cifar_sr(batch=2, frames=5)
    w, b, x = W.make_case(g, seed=9)
    got = gpu_rollout(g, w, b, x, 5, out_node=3)
    ref = oracle_states(g, w, b, x, 5, "bf16", nodes=[3])[3]
    for t in range(5):
        assert max_abs_rel(got[t], ref[t]) <= 2e-2


def test_rollout_equals_frame_steps_and_hipgraph_equals_eager():
    # one launch a frame: launched plainly, with and without HIP graphs (frames of more launches: the test below)
    g = W.cifar_sr(batch=2, frames=11)
    w, b, x = W.make_case(g, seed=5, bias_scale=0.1)
    T = g.frames
    a = gpu_rollout(g, w, b, x, T)
    c = gpu_rollout(g, w, b, x, T, options=OPT_EAGER)
    steps, _, _ = gpu_states_by_steps(g, w, b, x, T, nodes=[g.out_node])
    np.testing.assert_array_equal(a, c)
    np.testing.assert_array_equal(a, np.stack(steps[g.out_node]))
    ref = oracle_states(g, w, b, x, T, "bf16", nodes=[g.out_node])[g.out_node]
    for t in range(T):
        assert max_abs_rel(a[t], ref[t]) <= 2e-2


@pytest.mark.parametrize("out_node", [7, 3])
@pytest.mark.parametrize("T", [8, 11])
def test_recorded_bf16_frames_equal_plain_launches(T, out_node):
    # a launch per update step (dataflow off), seven a frame: eight frames replayed from a recording and three launched
    # plainly, against plain launches only; the head records itself, a hidden node has a copy launch behind every frame and,
    # recorded, the frame counter a launch of its own
    g = W.cifar_sr(batch=2, frames=T)
    g = g.with_pattern(W.sequential_pattern(g))
    assert g.out_node == 7
    w, b, x = W.make_case(g, seed=5, bias_scale=0.1, frames=T)
    a, dev = gpu_rollout(g, w, b, x, T, out_node=out_node, options={0: 1, 5: 0}, return_dev=True)
    assert dev.info()["launches_per_frame"] > 4 and not dev.health()["dependency_driven"]
    again = gpu_rollout(g, w, b, x, T, out_node=out_node, options={0: 0, 5: 0})
    np.testing.assert_array_equal(a, again)
    ref = oracle_states(g, w, b, x, T, "bf16", nodes=[out_node])[out_node]
    for t in range(T):
        assert np.abs(ref[t]).max() > 0
        assert max_abs_rel(a[t], ref[t]) <= 2e-2
    # one graph object: the other node recorded next, then single frames go on
    n = g.nodes[10 - out_node]
    import torch
    xd = [to_device_(x[v], g.dtype) for v in g.input_nodes()]
    out = torch.empty((T, g.batch, n.height, n.width, n.channels), dtype=dev.tdtype, device="cuda")
    dev.rollout([t[:T + 1] for t in xd], T, 10 - out_node, out)
    dev.synchronize()
    np.testing.assert_array_equal(out.float().cpu().numpy(), gpu_rollout(g, w, b, x, T, out_node=10 - out_node, options={0: 0, 5: 0}))
    dev.reset([t[0] for t in xd])
    for t in range(1, T + 1):
        dev.frame_step([xi[t] for xi in xd])
        np.testing.assert_array_equal(dev.get_state(out_node).float().cpu().numpy(), a[t - 1])
    dev.close()


@pytest.mark.parametrize("per_graph", [1, 2, 8])
@pytest.mark.parametrize("T", [1, 8, 19])
def test_recorded_frames_equal_plain_launches(per_graph, T):
    # a sequential fp32 net of more than four launches a frame: recorded where per_graph > 1 frames fit, any remainder
    # launched plainly; the same kernels on the same operands either way, so the same bits
    g = dataclasses.replace(W.dsr_net(2, batch=1, frames=T), dtype="f32")
    g = g.with_pattern(W.sequential_pattern(g))
    w, b, x = W.make_case(g, seed=8, bias_scale=0.1, frames=T)
    a, dev = gpu_rollout(g, w, b, x, T, options={0: 1, 2: per_graph}, return_dev=True)
    assert dev.info()["launches_per_frame"] > 4
    dev.close()
    np.testing.assert_array_equal(a, gpu_rollout(g, w, b, x, T, options=OPT_EAGER))
    steps, _, _ = gpu_states_by_steps(g, w, b, x, T, nodes=[g.out_node])
    np.testing.assert_array_equal(a, np.stack(steps[g.out_node]))


def test_checkpoint_restore_continues_bit_exactly():
    import paper_1806_04965_amd as sr
    from gpu_util import to_device
    g = W.cifar_sr(batch=2, frames=6)
    w, b, x = W.make_case(g, seed=6)
    xd = to_device(x[0], "bf16")
    full, _, _ = gpu_states_by_steps(g, w, b, x, 6, nodes=range(len(g.nodes)))
    dev = sr.SrGraph(g)
    dev.set_parameters(w, b)
    dev.reset([xd[0]])
    for t in range(1, 4):
        dev.frame_step([xd[t]])
    saved = [dev.get_state(v) for v in range(len(g.nodes))]
    dev.close()
    dev2 = sr.SrGraph(g)
    dev2.set_parameters(w, b)
    dev2.reset(None)
    for v, s in enumerate(saved):
        dev2.set_state(v, s)
    for t in range(4, 7):
        dev2.frame_step([xd[t]])
    for v in range(1, len(g.nodes)):
        np.testing.assert_array_equal(dev2.get_state(v).float().cpu().numpy(), full[v][-1])
    dev2.close()


def test_first_response_frame_on_gpu():
    # exact zeros at the output until shortest-path-many frames have passed (zero bias)
    g = W.cifar_sr(batch=2, frames=7)
    w, b, x = W.make_case(g, seed=7)
    out = gpu_rollout(g, w, b, x, 7)
    for t in range(1, 5):
        assert np.all(out[t - 1] == 0.0)
    assert np.any(out[4] != 0.0)


def test_two_inputs_and_unordered_node_ids():
    # node ids in no particular order: outputs first, two input nodes last
    nodes = [Node("out", 5, 1, 1, ACT_IDENTITY), Node("b", 32, 8, 8), Node("a", 32, 16, 16),
             Node("in2", 4, 16, 16, ACT_IDENTITY), Node("in1", 3, 16, 16, ACT_IDENTITY)]
    edges = [Edge(4, 2), Edge(3, 2), Edge(2, 1, stride=2), Edge(1, 1), Edge(1, 0, "gap_dense", 1, 1, 1, 0),
             Edge(3, 1, stride=2)]
    for dtype in ("bf16", "f32"):
        g = Graph("two_in", nodes, edges, batch=3, frames=4, dtype=dtype, out_node=0)
        assert g.input_nodes() == [3, 4]
        check(g, seed=12, label=f"two_in/{dtype}")
        check(g.with_pattern([0, 1, 0, 1, 0, 1]), seed=12, label=f"two_in/{dtype}/hybrid")


def test_zero_frames_and_single_sample():
    import torch
    import paper_1806_04965_amd as sr
    from gpu_util import to_device
    g = W.cifar_sr(batch=1, frames=3)
    w, b, x = W.make_case(g, seed=13)
    dev = sr.SrGraph(g)
    dev.set_parameters(w, b)
    xd = to_device(x[0], "bf16")
    dev.rollout([xd], 0, g.out_node, None)          # T = 0: only the initial state
    dev.synchronize()
    assert dev.frame_index() == 0
    np.testing.assert_array_equal(dev.get_state(0).float().cpu().numpy(), xd[0].float().cpu().numpy())
    for v in range(1, len(g.nodes)):
        assert float(dev.get_state(v).float().abs().max()) == 0.0
    dev.close()
    check(g, seed=13, label="cifar_sr/B1")


def test_errors_on_the_device_path():
    import paper_1806_04965_amd as sr
    from gpu_util import to_device
    g = W.tiny_sr()
    w, b, x = W.make_case(g, seed=14)
    dev = sr.SrGraph(g)
    xd = to_device(x[0], "f32")
    with pytest.raises(sr.SrError) as ei:
        dev.frame_step([xd[1]])
    assert ei.value.name == "SR_ERR_STATE"          # no sr_reset yet
    with pytest.raises(sr.SrError) as ei:
        dev.reset([xd[0]])
    assert ei.value.name == "SR_ERR_STATE"          # weights missing
    dev.set_parameters(w, b)
    dev.reset([xd[0]])
    dev.frame_step([xd[1]])
    dev.synchronize()
    with pytest.raises(sr.SrError) as ei:
        dev.set_weights(0, np.zeros(5, np.float32))
    assert ei.value.name == "SR_ERR_ARG"
    dev.close()


@pytest.mark.parametrize("name", ["cifar", "cifar_ragged", "gtsrb", "hires"])
def test_eight_wave_tile_kernel_streaming(name):
    g = {"cifar": lambda: W.cifar_sr(batch=4, frames=4), "cifar_ragged": lambda: W.cifar_sr(batch=3, frames=3),
         "gtsrb": lambda: W.gtsrb_sr(batch=3, frames=3), "hires": lambda: W.hires_sr(batch=1, frames=2)}[name]()
    info, work = check(g, seed=21, options=OPT_WIDE, label=f"{name}/8-wave kernel")
    assert work["mfma_tiles"] > 0 and info["inference_factor"] == 1


def test_eight_wave_tile_kernel_sequential_pattern_and_no_split():
    g = W.cifar_sr(batch=4, frames=3)
    check(g.with_pattern(W.sequential_pattern(g)), seed=22, options=OPT_WIDE, label="cifar_sr/sequential/8-wave kernel")
    check(W.hires_sr(batch=1, frames=2), seed=23, options={4: 2, 3: 0}, label="hires_sr/8-wave kernel, no K-split")


def test_eight_wave_tile_kernel_rollout_in_hipgraph_matches_steps():
    g = W.gtsrb_sr(batch=2, frames=5)
    w, b, x = W.make_case(g, seed=24, bias_scale=0.1, frames=5)
    a = gpu_rollout(g, w, b, x, 5, options=OPT_WIDE)
    c = gpu_rollout(g, w, b, x, 5, options={4: 2, 0: 0})
    assert np.array_equal(a, c)
    ref = oracle_states(g, w, b, x, 5, "bf16", nodes=[g.out_node])
    for t in range(5):
        assert max_abs_rel(a[t], ref[g.out_node][t]) <= TOL["bf16"]


def test_tile_kernel_choice_is_reported():
    import paper_1806_04965_amd as sr
    # CIFAR-shaped: every patch fits the 4-wave kernel; DSR0 at its batch of 64: the stride-4 edges into the 4x4 node
    # fit as phase planes; fp32 graphs have no MFMA node; an explicit choice is reported back
    for g, options, want in ((W.cifar_sr(batch=2, frames=2), None, 1), (W.dsr_net(0, batch=64, frames=2), None, 1),
                             (W.tiny_sr(), None, 0), (W.cifar_sr(batch=2, frames=2), OPT_WIDE, 2)):
        dev = sr.SrGraph(g, options=options)
        w, b, _ = W.make_case(g, seed=1)
        dev.set_parameters(w, b)
        assert dev.tile_kernel() == want, (g.name, options)
        dev.close()


OPT_FLOW_ON, OPT_FLOW_OFF = {5: 1}, {5: 0}


@pytest.mark.parametrize("pattern", ["streaming", "hybrid", "sequential"])
def test_dependency_driven_execution_equals_one_launch_per_update_step(pattern):
    # The same rollout dependency-driven (one launch for every update step of up to 8 frames; a work item
    # waits for the nodes it reads) and with one launch per update step: bit-identical outputs over
    # 19 frames (two 8-frame launches + 3 single frames), every node's final state too, and no
    # dependency wait may have given up.  K-split tiles, head and input-staging items all take part.
    import paper_1806_04965_amd as sr
    g0 = W.cifar_sr(batch=6, frames=19)
    g = g0.with_pattern({"streaming": W.streaming_pattern, "hybrid": W.hybrid_pattern,
                         "sequential": W.sequential_pattern}[pattern](g0))
    w, b, x = W.make_case(g, seed=41, bias_scale=0.1)
    outs, finals = {}, {}
    for name, opt in (("flow", OPT_FLOW_ON), ("steps", OPT_FLOW_OFF)):
        res, dev = gpu_rollout(g, w, b, x, g.frames, options=opt, return_dev=True)
        health, info = dev.health(), dev.info()
        assert health["dependency_driven"] == (name == "flow")
        assert health["dependency_timeouts"] == 0
        assert info["launches_per_frame"] == (1 if name == "flow" else max(1, info["inference_factor"]))
        outs[name] = res
        finals[name] = [dev.get_state(v).float().cpu().numpy() for v in range(len(g.nodes))]
        dev.close()
    np.testing.assert_array_equal(outs["flow"], outs["steps"])
    for a, c in zip(finals["flow"], finals["steps"]):
        np.testing.assert_array_equal(a, c)
    ref = oracle_states(g, w, b, x, g.frames, "bf16", nodes=[g.out_node])[g.out_node]
    for t in range(g.frames):
        assert np.abs(ref[t]).max() > 0
        assert max_abs_rel(outs["flow"][t], ref[t]) <= TOL["bf16"]


def test_dependency_driven_default_and_larger_graphs():
    # default: dependency-driven exactly when a frame has more than one update step
    import paper_1806_04965_amd as sr
    for g, want in ((W.cifar_sr(batch=2, frames=2), False),
                    (W.cifar_patterns(batch=2, frames=2)["sequential"], True), (W.tiny_sr(), False)):
        dev = sr.SrGraph(g)
        w, b, _ = W.make_case(g, seed=1)
        dev.set_parameters(w, b)
        assert dev.health()["dependency_driven"] == want, g.name
        dev.close()
    # forced on for streaming graphs with feedback, long skips and K-split tiles: against the oracle
    for g, seed in ((W.gtsrb_sr(batch=3, frames=10), 43), (W.hires_sr(batch=1, frames=3), 44)):
        if g.name == "hires_sr":
            g = Graph("hires_sr", [n if n.name == "out" else Node(n.name, n.channels, n.height // 4, n.width // 4, n.act)
                                   for n in g.nodes], g.edges, 1, 3, "bf16", g.out_node)
        check(g, seed=seed, options=OPT_FLOW_ON, label=f"{g.name}/dependency-driven")
        hy = g.with_pattern(W.hybrid_pattern(g))
        check(hy, seed=seed, label=f"{g.name}/hybrid (dependency-driven by default)")


def test_tile_spanning_more_than_127_images():
    # a 1x3 node at batch 160: one 512-pixel tile would span 170 images, more than the tile kernels'
    # packed image offset holds; the planner has to choose a shape (or kernel) that stays within it
    nodes = [Node("in", 16, 1, 3, ACT_IDENTITY), Node("a", 32, 1, 3), Node("out", 5, 1, 1, ACT_IDENTITY)]
    edges = [Edge(0, 1, "conv", 3, 3, 1, 1), Edge(1, 1, "conv", 3, 3, 1, 1), Edge(1, 2, "gap_dense", 1, 1, 1, 0)]
    g = Graph("thin", nodes, edges, batch=160, frames=3, dtype="bf16", out_node=2)
    for options in (None, OPT_WIDE):
        check(g, seed=17, options=options, label=f"thin/B160/{options}")


def test_mfma_nodes_of_the_benchmark_configurations():
    # which kernel the planner gives every node: all convolution nodes of the three bf16 benchmark
    # configurations run on matrix-core tiles (4-wave kernel), their heads as head items
    import paper_1806_04965_amd as sr
    for g in (W.cifar_sr(), W.gtsrb_sr(), W.hires_sr()):
        dev = sr.SrGraph(g)
        w, b, _ = W.make_case(g, seed=1, frames=0)
        dev.set_parameters(w, b)
        kinds = dev.node_kernels()
        assert dev.tile_kernel() == 1
        dev.close()
        for v, n in enumerate(g.nodes):
            want = 0 if v in g.input_nodes() else (4 if v == g.out_node else 1)
            assert kinds[v] == want, (g.name, n.name, kinds)


def test_two_graphs_alive_interleaved_and_recreated():
    # Two graphs with K-split nodes live side by side, stepped alternately; then both are destroyed and
    # created again (the partial-sum scratch of the first pair is handed to the second).  Every
    # graph's output must match its own single-graph run bit for bit and the oracle within tolerance.
    import paper_1806_04965_amd as sr
    ga = W.cifar_sr(batch=4, frames=5)
    gb = W.gtsrb_sr(batch=2, frames=5)
    cases = []
    for g, seed in ((ga, 21), (gb, 22)):
        w, b, x = W.make_case(g, seed=seed)
        alone, _, work = gpu_states_by_steps(g, w, b, x, g.frames, nodes=[g.out_node])
        ref = oracle_states(g, w, b, x, g.frames, "bf16", nodes=[g.out_node])[g.out_node]
        cases.append((g, w, b, x, alone[g.out_node], ref))
    for round_ in range(2):
        devs = []
        for g, w, b, x, _, _ in cases:
            d = sr.SrGraph(g)
            d.set_parameters(w, b)
            ins = g.input_nodes()
            xd = {v: to_device_(x[v], g.dtype) for v in ins}
            d.reset([xd[v][0] for v in ins])
            devs.append((d, xd, ins))
        for t in range(1, 6):
            for (d, xd, ins), (g, _, _, _, alone, ref) in zip(devs, cases):
                d.frame_step([xd[v][t] for v in ins])
            for (d, xd, ins), (g, _, _, _, alone, ref) in zip(devs, cases):
                got = d.get_state(g.out_node).float().cpu().numpy().astype(np.float64)
                np.testing.assert_array_equal(got, alone[t - 1])
                assert max_abs_rel(got, ref[t - 1]) <= 2e-2
        for d, _, _ in devs:
            d.close()


def test_dependency_wait_that_gives_up_is_counted_and_every_kernel_ends():
    # failure path of the dependency-driven launch, forced from the host: with a spin limit of 0 a wait
    # gives up at its first unsatisfied poll; the work item goes on (results undefined), the kernels
    # end normally, and the graph reports the waits that gave up.  sr_reset clears the count.
    import paper_1806_04965_amd as sr
    g0 = W.cifar_sr(batch=4, frames=4)
    g = g0.with_pattern(W.sequential_pattern(g0))
    w, b, x = W.make_case(g, seed=3, bias_scale=0.1, frames=4)
    dev = sr.SrGraph(g, options={6: 0})
    dev.set_parameters(w, b)
    xd = [to_device_(x[v], g.dtype) for v in g.input_nodes()]
    dev.rollout(xd, 4)
    dev.synchronize()
    h = dev.health()
    assert h["dependency_driven"] and h["dependency_timeouts"] > 0, h
    dev.reset([xi[0] for xi in xd])
    assert dev.health()["dependency_timeouts"] == 0
    dev.close()
    with pytest.raises(sr.SrError):
        sr.SrGraph(g, options={6: -1})


@pytest.mark.parametrize("name", ["cifar_seq", "cifar_hybrid", "dsr2_seq", "hires_seq"])
def test_depth_ordered_multi_frame_launch_equals_frame_after_frame(name):
    # a dependency-driven rollout dispatches the work items of 8 frames in the order of their depth in the rollout
    # window of those frames (Eq. 5 over update steps); the arithmetic of every item is the same as when the frames
    # are dispatched one after the other, so the outputs are bit-identical -- and both match the oracle
    g0 = {"cifar_seq": lambda: W.cifar_sr(batch=4, frames=19), "cifar_hybrid": lambda: W.cifar_sr(batch=4, frames=19),
          "dsr2_seq": lambda: W.dsr_net(2, batch=8, frames=17), "hires_seq": lambda: W.hires_sr(batch=1, frames=16)}[name]()
    pat = W.hybrid_pattern if name.endswith("hybrid") else W.sequential_pattern
    g = g0.with_pattern(pat(g0))
    T = g.frames
    w, b, x = W.make_case(g, seed=61, bias_scale=0.1, frames=T)
    a, dev = gpu_rollout(g, w, b, x, T, return_dev=True)
    h = dev.health()
    dev.close()
    assert h["dependency_driven"] and h["dependency_timeouts"] == 0
    c = gpu_rollout(g, w, b, x, T, options={7: 0})
    assert np.array_equal(a, c)
    ref = oracle_states(g, w, b, x, T, "bf16", nodes=[g.out_node])
    for t in range(T):
        assert np.abs(ref[g.out_node][t]).max() > 0
        assert max_abs_rel(a[t], ref[g.out_node][t]) <= TOL["bf16"], (name, t)


@pytest.mark.parametrize("frames_per_launch", [1, 2, 5, 16])
def test_depth_ordered_launches_of_other_lengths(frames_per_launch):
    # launches of at most the configured number of frames, of equal length or one apart (13 frames: 13 of 1; 6 of 2 and 1; 5, 4, 4;
    # one of 13); the pairs are written for each length.  All of them equal one launch per update step.
    g0 = W.cifar_sr(batch=3, frames=13)
    g = g0.with_pattern(W.sequential_pattern(g0))
    w, b, x = W.make_case(g, seed=62, bias_scale=0.1, frames=13)
    a = gpu_rollout(g, w, b, x, 13, options={2: frames_per_launch})
    c = gpu_rollout(g, w, b, x, 13, options={5: 0})
    assert np.array_equal(a, c)
    assert np.abs(a[-1]).max() > 0


@pytest.mark.parametrize("pattern", [W.sequential_pattern, W.hybrid_pattern])
def test_depth_ordered_launches_follow_the_rollouts_length(pattern):
    # one launch for up to 64 frames, launches of equal length beyond (65: 33 + 32, 130: 44 + 43 + 43); rollouts of other
    # lengths in between, whose launches take other (frame, item) pairs.  All equal one launch per update step.
    import torch
    import paper_1806_04965_amd as sr
    from gpu_util import to_device
    g0 = W.cifar_sr(batch=2, frames=130)
    g = g0.with_pattern(pattern(g0))
    w, b, x = W.make_case(g, seed=64, bias_scale=0.1, frames=130)
    want = gpu_rollout(g, w, b, x, 130, options={5: 0})
    dev = sr.SrGraph(g)
    dev.set_parameters(w, b)
    xd = [to_device(x[v], g.dtype) for v in g.input_nodes()]
    for T in (130, 2, 64, 65, 1, 64, 3, 130):
        out = torch.empty((T, 2, 1, 1, 10), dtype=torch.bfloat16, device="cuda")
        dev.rollout([t[:T + 1] for t in xd], T, g.out_node, out)
        dev.synchronize()
        assert np.array_equal(out.float().cpu().numpy(), want[:T]), T
    h = dev.health()
    dev.close()
    assert h["dependency_driven"] and h["dependency_timeouts"] == 0


@pytest.mark.parametrize("wanted", [100, 255, 1024])
def test_launches_of_more_than_64_frames(wanted):
    # frames from 128 on set the sign bit of a (frame, item) pair; 255 in one launch at most (260 frames: 3 of 87, 87, 86; 2 of 130)
    g0 = W.cifar_sr(batch=1, frames=260)
    g = g0.with_pattern(W.sequential_pattern(g0))
    w, b, x = W.make_case(g, seed=65, bias_scale=0.1, frames=260)
    a = gpu_rollout(g, w, b, x, 260, options={2: wanted})
    c = gpu_rollout(g, w, b, x, 260, options={5: 0})
    assert np.array_equal(a, c)
    assert np.abs(a[-1]).max() > 0


@pytest.mark.parametrize("batch", [1, 4, 37])
def test_pooled_slabs_of_several_frames_in_one_launch(batch):
    # a GAP read-out over 12 x 12 pixels is summed in three slabs whose arrival counter is reset by the last one:
    # in a launch that covers several frames the next frame's slabs, on other XCDs, must see the reset
    from workloads.graphs import Node, Edge, Graph, ACT_IDENTITY
    nodes = [Node("in", 3, 24, 24, ACT_IDENTITY), Node("a", 40, 24, 24), Node("b", 64, 12, 12), Node("out", 43, 1, 1, ACT_IDENTITY)]
    edges = [Edge(0, 1), Edge(1, 1), Edge(1, 2, "conv", 3, 3, 2, 1), Edge(2, 2), Edge(2, 3, "gap_dense", 1, 1, 1, 0)]
    g0 = Graph("slabs", nodes, edges, batch, 16, "bf16", out_node=3)
    g = g0.with_pattern(W.sequential_pattern(g0))
    w, b, x = W.make_case(g, seed=63, bias_scale=0.1, frames=16)
    a, dev = gpu_rollout(g, w, b, x, 16, return_dev=True, options={6: 4096})
    h = dev.health()
    dev.close()
    assert h["dependency_driven"] and h["dependency_timeouts"] == 0
    assert np.array_equal(a, gpu_rollout(g, w, b, x, 16, options={5: 0}))
    assert np.abs(a[-1]).max() > 0


@pytest.mark.parametrize("tall_from", [0, 2048, 1 << 30])
@pytest.mark.parametrize("channels", [(4, 32, 64), (31, 33, 65), (36, 100, 130)])
def test_fp32_row_tiles_at_tile_edges(channels, tall_from):
    # fp32 nodes run as row tiles: channel counts at, below and above the 32- / 64- / 128-wide column tiles, with
    # 16-byte and 4-byte gathers; 17 x 17 images (ragged row tiles over several images), a stride-2 edge, up-sampling,
    # a dense edge whose long sum is cut into parts.  tall_from (option 8) picks the tile shapes: 0 the tall ones.
    # Bound: a sum of K terms in float32 is off by about sqrt(K) * 2^-24 of the sum of magnitudes, which for these
    # inputs is a few times the tensor's largest element; K <= 5780: 5e-6 a frame, fed back over three frames.
    from workloads.graphs import Node, Edge, Graph, ACT_IDENTITY
    ca, cb, cc = channels
    nodes = [Node("in", 3, 17, 17, ACT_IDENTITY), Node("a", ca, 17, 17), Node("b", cb, 9, 9), Node("c", cc, 9, 9),
             Node("d", 20, 17, 17), Node("out", 7, 1, 1, ACT_IDENTITY)]
    edges = [Edge(0, 1, "conv", 5, 5, 1, 2), Edge(1, 1), Edge(1, 2, "conv", 3, 3, 2, 1), Edge(2, 3), Edge(3, 2, "conv", 1, 1, 1, 0),
             Edge(1, 4), Edge(3, 3), Edge(4, 5, "dense", 17, 17, 1, 0)]
    g0 = Graph("edges", nodes, edges, 5, 3, "f32", out_node=5)
    g = g0.with_pattern(W.hybrid_pattern(g0))
    w, b, x = W.make_case(g, seed=71, bias_scale=0.1, frames=3, recipe="uniform")
    got, _, _ = gpu_states_by_steps(g, w, b, x, 3, {8: tall_from})
    compare_all(got, oracle_states(g, w, b, x, 3, "f64"), 2e-5, f"row tiles {channels} tall_from={tall_from}")
    rec = gpu_rollout(g, w, b, x, 3, options={8: tall_from})
    assert np.array_equal(rec, np.stack(got[5]))     # recorded by the tiles themselves


@pytest.mark.parametrize("channels", [(32, 64), (20, 64), (16, 40)])
def test_fp32_64x64_tiles_in_pairs_of_steps(channels):
    # enough rows for the 64 x 64 and 128 x 32 tiles of a launch without 128 x 128 tiles (four workgroups per CU): sums of
    # 32 k channels (two steps share their addresses) beside 20, 16 and 3 (step by step, odd numbers of steps).
    # Bound: as in test_fp32_row_tiles_at_tile_edges, K <= 864.
    from workloads.graphs import Node, Edge, Graph, ACT_IDENTITY
    ca, cb = channels
    nodes = [Node("in", 3, 40, 40, ACT_IDENTITY), Node("a", ca, 40, 40), Node("b", cb, 40, 40), Node("out", 5, 1, 1, ACT_IDENTITY)]
    edges = [Edge(0, 1), Edge(1, 1, "conv", 1, 1, 1, 0), Edge(1, 2), Edge(2, 2, "conv", 1, 1, 1, 0), Edge(2, 3, "dense", 40, 40, 1, 0)]
    g0 = Graph("pairs", nodes, edges, 21, 3, "f32", out_node=3)
    g = g0.with_pattern(W.streaming_pattern(g0))
    w, b, x = W.make_case(g, seed=73, bias_scale=0.1, frames=3, recipe="uniform")
    got, _, _ = gpu_states_by_steps(g, w, b, x, 3)
    compare_all(got, oracle_states(g, w, b, x, 3, "f64"), 2e-5, f"pairs {channels}")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("channels", [1, 3, 5, 16, 33, 40])
def test_reset_copies_frame_0_of_an_input(channels, dtype):
    # whole pieces of 16 bytes, ragged ones, more than one chunk of a workgroup, and input frames that begin at any
    # element; frame 0 comes back bit for bit
    import torch
    import paper_1806_04965_amd as sr
    from workloads.graphs import Node, Edge, Graph, ACT_IDENTITY
    nodes = [Node("in", channels, 23, 31, ACT_IDENTITY), Node("a", 7, 23, 31)]
    g0 = Graph("reset", nodes, [Edge(0, 1)], 3, 1, dtype, out_node=1)
    g = g0.with_pattern(W.streaming_pattern(g0))
    w, b, _ = W.make_case(g, seed=5, frames=1, recipe="uniform")
    dev = sr.SrGraph(g)
    dev.set_parameters(w, b)
    n = 3 * 23 * 31 * channels
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    for start in (0, 1, 2):
        x = torch.randn(n + 2, device="cuda").to(tdt)[start:start + n].view(3, 23, 31, channels)
        dev.reset([x])
        assert torch.equal(dev.get_state(0), x)
    dev.close()


def set_frame_index(dev, index, tmp_path):
    """Count `index` frames as computed: the graph object's own counter, found by the offset that a C++ compiler gives it."""
    import ctypes
    import os
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src, exe = tmp_path / "at.cpp", tmp_path / "at"
    src.write_text('#include <cstddef>\n#include <cstdio>\n#include "sr_graph.h"\n'
                   'int main() { std::printf("%zu", offsetof(sr_graph, host_frame)); }\n')
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", f"{root}/paper_1806_04965_amd/csrc",
                    str(src), "-o", str(exe)], check=True, timeout=60)
    at = int(subprocess.run([str(exe)], check=True, capture_output=True, timeout=10).stdout)
    counter = ctypes.c_int64.from_address(dev.h.value + at)
    assert counter.value == dev.frame_index()
    counter.value = index


@pytest.mark.parametrize("net", ["f32 streaming", "f32 sequential", "bf16 streaming"])
def test_frames_past_the_32_bit_frame_counter(net, tmp_path):
    # a stream that has run for 2^31 - 3 frames (17 hours at 29 us) goes on as one that has just begun: the kernels' 32-bit
    # frame numbers wrap, inputs are still taken and both copies of a state still alternate
    import paper_1806_04965_amd as sr
    dtype, pattern = net.split()
    g = dataclasses.replace(W.tiny_sr(batch=2, frames=8), dtype=dtype)
    g = g.with_pattern((W.streaming_pattern if pattern == "streaming" else W.sequential_pattern)(g))
    w, b, x = W.make_case(g, seed=17, bias_scale=0.1, frames=8)
    ins = g.input_nodes()
    xd = [to_device_(x[v], dtype) for v in ins]
    runs = []
    for start in (0, 2 ** 31 - 4, 2 ** 32 - 4):     # even: frame 0 of the reset lies in copy 0
        dev = sr.SrGraph(g, options={5: 0})
        dev.set_parameters(w, b)
        dev.reset([t[0] for t in xd])
        set_frame_index(dev, start, tmp_path)
        states = []
        for t in range(1, 9):
            (dev.frame_step_static if t % 3 == 2 else dev.frame_step)([xi[t] for xi in xd])
            states += [dev.get_state(v).float().cpu().numpy() for v in range(len(g.nodes))]
        assert dev.frame_index() == start + 8
        dev.close()
        runs.append(states)
    for other in runs[1:]:
        for a, c in zip(runs[0], other):
            np.testing.assert_array_equal(a, c)
