"""The planner of the tiled fp32 kernels (csrc/sr_f32_plan.cpp), compiled for the host: what its tables hold and how its work
items are spread."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1806_04965_amd", "csrc")

COMMON = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include "sr_f32.h"
#include "sr_graph.h"

#define CHECK(c, ...) do { if (!(c)) { std::printf(__VA_ARGS__); std::printf("  (%s)\n", #c); std::exit(1); } } while (0)

struct N { int channels, size; };
struct E { int src, dst, kind, k, stride, pad; };
static sr_graph* graph(int batch, std::vector<N> nodes, std::vector<E> edges) {   // every edge bridges
  sr_graph* g = new sr_graph();
  g->batch = batch;
  g->n_nodes = (int)nodes.size();
  g->n_edges = (int)edges.size();
  for (const N& n : nodes) {
    NodeRt r;
    r.d.channels = n.channels; r.d.height = r.d.width = n.size; r.d.act = 1;
    g->nodes.push_back(r);
  }
  g->an.is_input.assign(nodes.size(), 1);
  for (const E& e : edges) {
    EdgeRt r;
    r.d.src = e.src; r.d.dst = e.dst; r.d.kind = e.kind; r.d.bridge = 1; r.d.upsample = 1;
    r.d.stride = e.stride; r.d.pad = e.pad;
    r.kh = r.kw = e.kind == SR_EDGE_DENSE ? nodes[e.src].size : (e.kind == SR_EDGE_CONV ? e.k : 1);
    r.w_count = (size_t)r.kh * r.kw * nodes[e.src].channels * nodes[e.dst].channels;
    g->edges.push_back(r);
    g->an.is_input[e.dst] = 0;
  }
  return g;
}
// tensor numbers of a window with its loss at node `out`
static SrTrainIds train_ids(const sr_graph* g, int out) {
  SrTrainIds ids;
  ids.grad0 = g->n_nodes; ids.mask0 = 2 * g->n_nodes; ids.seed = -1; ids.out_node = out;
  int n = 3 * g->n_nodes + 1;
  ids.mean.assign(g->n_edges, -1);
  for (int e = 0; e < g->n_edges; ++e)
    if (g->edges[e].d.kind == SR_EDGE_GAP_DENSE) ids.mean[e] = n++;
  ids.dist.assign(g->n_nodes, -1);
  ids.dist[out] = 0;
  for (bool changed = true; changed;) {
    changed = false;
    for (const EdgeRt& e : g->edges)
      if (ids.dist[e.d.dst] >= 0 && (ids.dist[e.d.src] < 0 || ids.dist[e.d.src] > ids.dist[e.d.dst] + 1)) {
        ids.dist[e.d.src] = ids.dist[e.d.dst] + 1;
        changed = true;
      }
  }
  return ids;
}
"""

TILE_RECORD = COMMON + r"""
int main() {
  // Planned by the ten thousands in the first window of a graph, sorted, and copied to the device: a record has what tells a
  // workgroup its part, not the descriptors that many of them share.
  CHECK(sizeof(SrRowTile) <= 32, "a tile's record has %zu bytes", sizeof(SrRowTile));
  std::printf("ok\n");
}
"""

LINE_TABLES = COMMON + r"""
static long checked = 0;
// every segment's table against the indices decoded one by one
static void compare(const SrRowPlan& p, bool in_turn) {
  for (const SrSeg& s : p.segs) {
    if (s.lines < 0) continue;
    CHECK((s.R + 15) / 16 * 16 + (size_t)s.lines <= p.lines.size(), "a table past the end");
    for (int k = 0; k < (s.R + 15) / 16 * 16; ++k) {
      const int r = k / 16 * 16 + (in_turn ? sr_in_turn(k % 16) : k % 16);
      const SrLine& x = p.lines[s.lines + k];
      const SrTapAt t = sr_tap_at(s, r);
      ++checked;
      if (r >= s.R) CHECK(x.dh == SR_NO_ROW && x.dw == SR_NO_ROW, "an index that does not exist");
      else CHECK(x.off == sr_gather_off(s, t) && x.dh == s.dir * t.vi && x.dw == s.dir * t.vj, "index %d of %d", r, s.R);
    }
  }
}
int main() {
  // 96 x 96 pixels of 43 channels, read by two convolutions (stride 1 and 3) and a dense edge: a phase per pixel backwards
  sr_graph* g = graph(2, {{3, 96}, {43, 96}, {43, 96}, {43, 32}, {10, 1}},
                      {{0, 1, SR_EDGE_CONV, 5, 1, 2}, {1, 2, SR_EDGE_CONV, 3, 1, 1}, {1, 3, SR_EDGE_CONV, 3, 3, 0}, {1, 4, SR_EDGE_DENSE, 0, 1, 0},
                       {2, 4, SR_EDGE_GAP_DENSE, 0, 1, 0}, {3, 4, SR_EDGE_GAP_DENSE, 0, 1, 0}, {2, 2, SR_EDGE_CONV, 3, 1, 1}, {3, 3, SR_EDGE_CONV, 7, 1, 3}});
  const SrTrainIds ids = train_ids(g, 4);
  for (int train = 0; train < 2; ++train) {
    SrRowPlan f;
    for (int v = 1; v < 4; ++v) sr_rows_forward(&f, g, v, train ? &ids : nullptr);
    compare(f, train == 1);
    std::printf("forward %zu segments, %zu lines\n", f.segs.size(), f.lines.size());
  }
  SrRowPlan b;
  for (int v = 1; v < 4; ++v) sr_rows_backward(&b, g, v, ids);
  compare(b, false);
  std::printf("backwards %zu phases, %zu segments, %zu lines, %ld checked\n", b.phases.size(), b.segs.size(), b.lines.size(), checked);
  // tables of 3 x 3, 1 x 1 (stride 3: its only tap row and column), 7 x 7 taps of 43 channels and of 10: 400, 48 and 2112 lines and 16
  CHECK(b.segs.size() > 9216 * 2, "as many segments as expected");
  CHECK(b.lines.size() <= 8192, "%zu lines", b.lines.size());
  std::printf("ok\n");
}
"""

LITTLE_MEMORY = COMMON + r"""
int main() {
  // deep sums of large edges: as many slices as there are work items to make
  sr_graph* g = graph(64, {{64, 16}, {256, 16}, {256, 16}, {512, 8}, {10, 1}},
                      {{0, 1, SR_EDGE_CONV, 3, 1, 1}, {1, 2, SR_EDGE_CONV, 3, 1, 1}, {2, 3, SR_EDGE_CONV, 3, 2, 1}, {3, 3, SR_EDGE_CONV, 3, 1, 1},
                       {1, 1, SR_EDGE_CONV, 3, 1, 1}, {3, 4, SR_EDGE_GAP_DENSE, 0, 1, 0}});
  const SrTrainIds ids = train_ids(g, 4);
  const int W = 8;
  auto part_bytes = [&](const SrTrainRoom& r) {   // the largest chunk's, as a plan allocates them
    long long most = 0;
    for (int hi = W; hi >= 1; hi -= r.frames) {
      SrGradPlan p;
      sr_grad_plan(&p, g, ids, W, std::max(1, hi - r.frames + 1), hi, hi == W, 2048, r.items);
      most = std::max(most, p.part_floats * 4);
    }
    return most;
  };
  // a room whose memory is not to be had is followed by a smaller one: partial sums for half as many work items before any frame is
  // given up and with every number of frames after that, and for one a compute unit at the very end
  SrTrainRoom r{W, SR_GRAD_ITEMS};
  long long before = part_bytes(r);
  const long long full = before;
  int turns = 0, last_frames = W;
  while (r.shrink(r.frames)) {
    const long long now = part_bytes(r);
    std::printf("%d frames, %d items: %lld bytes of partial sums\n", r.frames, r.items, now);
    CHECK(r.frames <= last_frames && r.items < SR_GRAD_ITEMS, "%d frames, %d items", r.frames, r.items);
    CHECK(turns > 0 || (r.frames == W && now <= full * 5 / 8), "the first turn: %d frames, %lld of %lld bytes", r.frames, now, full);
    CHECK(r.frames < last_frames || now < before, "no less than before");
    last_frames = r.frames;
    before = now;
    CHECK(++turns < 20, "no end");
  }
  CHECK(r.frames == 1 && r.items == 1 && before <= full / 6, "%d frames, %d items, %lld of %lld bytes at the end", r.frames, r.items, before, full);
  std::printf("ok\n");
}
"""

SPREAD = COMMON + r"""
// cycles of the weight gradients' work items per XCD (workgroup i runs on XCD i % 8), by the planner's own measure
static double spread(const char* name, sr_graph* g, int out, int W, double limit) {
  const SrTrainIds ids = train_ids(g, out);
  SrGradPlan p;
  sr_grad_plan(&p, g, ids, W, 1, W, true, 2048, SR_GRAD_ITEMS);
  double load[8] = {}, all = 0, longest = 0;
  int items = 0;
  for (size_t k = 0; k < p.tiles.size(); ++k) {
    const SrGradTile& t = p.tiles[k];
    if (t.kind == 2) continue;
    int ti, tj;
    sr_f32_shape(t.shape, &ti, &tj);
    const double c = t.kind == 1 ? (t.step_end - t.step_begin) * 8.0
                                 : std::max(ti * tj / 8.0, 900.0) * (p.edges[t.edge].quads_in ? 1.0 : 1.6) * (t.step_end - t.step_begin);
    load[k % 8] += c;
    all += c;
    longest = std::max(longest, c);
    ++items;
  }
  const double most = *std::max_element(load, load + 8), mean = all / 8;
  std::printf("%s: %d items in %zu workgroups, most / mean %.3f, longest / mean %.3f\n", name, items, p.tiles.size(), most / mean, longest / mean);
  // no XCD has more than the limit, unless a single item is that long
  CHECK(most <= std::max(limit * mean, longest * 1.001), "%s", name);
  CHECK(p.tiles.size() <= items * 3 / 2 + 16, "%s: %zu workgroups for %d items", name, p.tiles.size(), items);
  return most / mean;
}
static sr_graph* mnist(int batch) {
  return graph(batch, {{1, 28}, {16, 7}, {128, 1}, {10, 1}},
               {{0, 1, SR_EDGE_CONV, 7, 4, 3}, {1, 2, SR_EDGE_DENSE, 0, 1, 0}, {2, 3, SR_EDGE_DENSE, 0, 1, 0}, {1, 3, SR_EDGE_DENSE, 0, 1, 0},
                {1, 1, SR_EDGE_CONV, 3, 1, 1}});
}
static sr_graph* chain(int batch, int size, int width) {
  return graph(batch, {{3, size}, {width, size}, {2 * width, size / 2}, {2 * width, size / 2}, {4 * width, size / 4}, {10, 1}},
               {{0, 1, SR_EDGE_CONV, 3, 1, 1}, {1, 2, SR_EDGE_CONV, 3, 2, 1}, {2, 3, SR_EDGE_CONV, 3, 1, 1}, {1, 3, SR_EDGE_CONV, 3, 2, 1},
                {3, 4, SR_EDGE_CONV, 3, 2, 1}, {2, 4, SR_EDGE_CONV, 3, 2, 1}, {2, 2, SR_EDGE_CONV, 3, 1, 1}, {4, 4, SR_EDGE_CONV, 3, 1, 1},
                {4, 5, SR_EDGE_GAP_DENSE, 0, 1, 0}});
}
int main() {
  spread("mnist_sr B=1", mnist(1), 3, 4, 1.3);
  spread("mnist_sr B=16", mnist(16), 3, 8, 1.15);
  spread("mnist_sr B=128", mnist(128), 3, 8, 1.1);
  for (int width : {8, 24, 64})
    for (int batch : {1, 5, 64}) spread("chain", chain(batch, 32, width), 5, 6, batch == 1 ? 1.25 : 1.15);
  std::printf("ok\n");
}
"""


def run(tmp_path, program):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(program)
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=undefined", "-D__HIP_PLATFORM_AMD__",
                    "-I/opt/rocm/include", "-I", CSRC, str(src), os.path.join(CSRC, "sr_f32_plan.cpp"), "-o", str(exe)],
                   check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.endswith("ok\n"), r.stdout + r.stderr
    return r.stdout


def test_tile_records_are_small(tmp_path):
    run(tmp_path, TILE_RECORD)


def test_segments_share_tables_of_lines(tmp_path):
    print(run(tmp_path, LINE_TABLES))


def test_a_window_that_does_not_fit_takes_fewer_partial_sums(tmp_path):
    print(run(tmp_path, LITTLE_MEMORY))


def test_weight_gradients_are_spread_over_the_chip(tmp_path):
    print(run(tmp_path, SPREAD))
