"""Row tiles of fp32 graphs where the steps of whole segments follow one another: channel counts that make taps of one step, of
an odd number of steps and of pairs of steps, segments shorter than what is on the way at a time, gathered channel counts
that have a table of lines (1, 3, 6) and read-outs of few columns, over every tile shape, frames and windows.

Frames: float32 sums of at most 2000 products against the float64 oracle, held to the 1e-4 of every fp32 graph (measured
below 2e-6).  Windows: GRAD_TOL of test_gpu_training.py."""
import numpy as np
import pytest

import workloads as W
from workloads.graphs import Node, Edge, Graph, ACT_IDENTITY
from gpu_util import gpu_states_by_steps, oracle_states, compare_all, to_device
from test_gpu_training import check_against_oracle, run_case

pytestmark = pytest.mark.gpu


def net(cin, ca, cb, cc, classes=10, batch=5, size=13):
    half = (size + 1) // 2
    nodes = [Node("in", cin, size, size, ACT_IDENTITY), Node("a", ca, size, size), Node("b", cb, half, half), Node("c", cc, half, half),
             Node("out", classes, 1, 1, ACT_IDENTITY)]
    edges = [Edge(0, 1, "conv", 5, 5, 1, 2), Edge(1, 1, "conv", 1, 1, 1, 0), Edge(1, 2, "conv", 3, 3, 2, 1), Edge(0, 2, "conv", 7, 7, 2, 3),
             Edge(2, 3, "conv", 3, 3, 1, 1), Edge(3, 3, "conv", 1, 1, 1, 0), Edge(3, 4, "dense", half, half, 1, 0),
             Edge(2, 4, "dense", half, half, 1, 0)]
    g = Graph("rows", nodes, edges, batch, 3, "f32", out_node=4)
    return g.with_pattern(W.hybrid_pattern(g))


CHANNELS = [(1, 16, 32, 48), (3, 32, 64, 16), (6, 48, 16, 80), (16, 64, 160, 32), (3, 20, 130, 34)]


@pytest.mark.parametrize("tall_from", [0, 2048, 1 << 30])
@pytest.mark.parametrize("channels", CHANNELS)
def test_frames_and_windows(channels, tall_from):
    import paper_1806_04965_amd as sr
    g = net(*channels)
    w, b, x = W.make_case(g, seed=17, bias_scale=0.1, frames=g.frames, recipe="uniform")
    ref = oracle_states(g, w, b, x, g.frames, "f64")
    got, _, _ = gpu_states_by_steps(g, w, b, x, g.frames, {8: tall_from})
    worst = compare_all(got, ref, 1e-4, f"rows {channels} tall_from={tall_from}")
    print(f"[parity] rows {channels} tall_from={tall_from}: worst {worst:.3e}", flush=True)
    dev = sr.SrGraph(g, options={8: tall_from})
    dev.set_parameters(w, b)
    out, data = run_case(g, 3, seed=17, dev=dev)
    check_against_oracle(g, 3, out, data, f"rows {channels} tall_from={tall_from}")
    dev.close()


@pytest.mark.parametrize("tall_from", [0, 1 << 30])
def test_window_over_an_input_that_is_not_16_byte_aligned(tall_from):
    # a multiple of 16 channels whose addresses take 4-byte loads; GRAD_TOL as between any two correct windows
    import torch
    import paper_1806_04965_amd as sr
    g = net(16, 32, 64, 48)
    w, b, x = W.make_case(g, seed=5, bias_scale=0.1, frames=3, recipe="uniform")
    dev = sr.SrGraph(g, options={8: tall_from})
    dev.set_parameters(w, b)
    labels = torch.from_numpy(np.arange(g.batch, dtype=np.int32)).to("cuda")
    xa = to_device(x[0], "f32")
    flat = torch.empty(xa.numel() + 4, device="cuda")
    shifted = flat[1:1 + xa.numel()].view(xa.shape)
    shifted.copy_(xa)
    assert xa.data_ptr() % 16 == 0 and shifted.data_ptr() % 16 == 4
    a, b2 = (dev.window_gradients([t], labels, 3) for t in (xa, shifted))
    dev.synchronize()
    for p, q in zip([a[0], *a[1], *[t for t in a[2] if t is not None]], [b2[0], *b2[1], *[t for t in b2[2] if t is not None]]):
        assert float((p - q).abs().max()) <= 2e-5 * float(p.abs().max())
    dev.close()
