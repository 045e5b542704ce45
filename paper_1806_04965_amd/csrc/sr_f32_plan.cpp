// Planner of the tiled fp32 contractions (sr_f32.h): descriptors of a node's incoming edges and the tiles of a launch.
#include <algorithm>
#include <cmath>

#include "sr_f32.h"
#include "sr_graph.h"

namespace {

int64_t image_floats(const sr_node_desc& d) { return (int64_t)d.height * d.width * d.channels; }

struct Geometry {   // an edge as a convolution from a (H, W, Cin) image to a (Ho, Wo, Cout) one, up-sampled by `up`
  int H, W, Cin, Ho, Wo, Cout, kh, kw, stride, pad, up;
};
Geometry geometry(const sr_graph* g, const EdgeRt& e) {
  const sr_node_desc& s = g->nodes[e.d.src].d;
  const sr_node_desc& d = g->nodes[e.d.dst].d;
  if (e.d.kind == SR_EDGE_CONV)
    return Geometry{s.height, s.width, s.channels, d.height / e.d.upsample, d.width / e.d.upsample, d.channels, e.kh, e.kw,
                    e.d.stride, e.d.pad, e.d.upsample};
  // dense: a 1x1 map on a 1x1 image whose channels are all the source's elements (the memory layouts coincide);
  // GAP + dense: a 1x1 map on the channel means
  const int cin = e.d.kind == SR_EDGE_DENSE ? s.height * s.width * s.channels : s.channels;
  return Geometry{1, 1, cin, 1, 1, d.channels, 1, 1, 1, 0, 1};
}

int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

}  // namespace

bool sr_rows_take_forward(const sr_graph* g, int v) {
  const sr_node_desc& d = g->nodes[v].d;
  const int64_t pixels = (int64_t)d.height * d.width;
  if ((int64_t)g->batch * pixels >= ((int64_t)1 << 30) || pixels * d.channels * 4 >= ((int64_t)1 << 31)) return false;
  const int64_t images = std::min<int64_t>(g->batch, 128 / pixels + 2);   // that the rows of a tile can touch
  for (const EdgeRt& e : g->edges) {
    if (e.d.dst != v) continue;
    if (e.d.kind == SR_EDGE_GAP_DENSE) return false;
    if (images * image_floats(g->nodes[e.d.src].d) * 4 >= ((int64_t)1 << 31)) return false;
    if ((int64_t)e.w_count * 4 >= ((int64_t)1 << 31)) return false;
  }
  return true;
}

void sr_rows_forward(SrRowPlan* p, const sr_graph* g, int v) {
  const NodeRt& n = g->nodes[v];
  SrRowNode node{};
  node.out = v;
  node.x = node.seed = node.mask = -1;
  node.bias = n.bias_dev;
  node.C = n.d.channels;
  node.H = n.d.height;
  node.W = n.d.width;
  node.act = n.d.act;
  node.gnode = v;
  SrPhase ph{};
  ph.node = (int)p->nodes.size();
  ph.seg_begin = ph.seg_image = (int)p->segs.size();
  ph.I = g->batch * n.d.height * n.d.width;
  ph.Hp = n.d.height;
  ph.Wp = n.d.width;
  ph.S = 1;
  ph.image_scale = 1.f;
  ph.d_wp = sr_div_for(ph.Wp);
  ph.d_hpwp = sr_div_for(ph.Hp * ph.Wp);
  for (const EdgeRt& e : g->edges) {
    if (e.d.dst != v) continue;
    const Geometry q = geometry(g, e);
    SrSeg s{};
    s.w = e.w_dev;
    s.tensor = e.d.src;
    s.flags = (e.d.bridge ? SR_SEG_LAG : 0) | (g->an.is_input[e.d.src] ? 0 : SR_SEG_ZERO0) | (q.Cin % 4 == 0 ? SR_SEG_QUADS : 0);
    s.GH = q.H; s.GW = q.W; s.GC = q.Cin;
    s.rs = q.stride; s.r0h = s.r0w = -q.pad;
    s.dir = 1;
    s.ntj = q.kw;
    s.R = q.kh * q.kw * q.Cin;
    s.ldw = q.Cout;
    s.step0 = ph.steps;
    s.d_gc = sr_div_for(q.Cin);
    s.d_ntj = sr_div_for(q.kw);
    s.d_up = sr_div_for(q.up);
    ph.steps += ceil_div(s.R, SR_F32_KS);
    p->segs.push_back(s);
  }
  ph.seg_end = (int)p->segs.size();
  p->nodes.push_back(node);
  p->phases.push_back(ph);
}

double sr_rows_work(const SrRowPlan& p, int phase) {
  const SrPhase& ph = p.phases[phase];
  const int C = p.nodes[ph.node].C;
  // a CU does 256 fp32 operations per cycle on its matrix cores
  return 2.0 * ph.I * ((C + 31) / 32 * 32) * ph.steps * SR_F32_KS / 256.0;
}

// Tile shape of a phase.  Taller tiles fetch fewer operand bytes per product and pass fewer barriers; smaller ones
// give the launch more workgroups and shorter chains of dependent steps.  A tile may take as long as an even share of
// the launch's work per compute unit (or some microseconds), else the next smaller shape is tried; below that the
// reduction is cut into parts.
void sr_rows_tiles(const SrRowPlan& p, const std::vector<int>& phases, double work_cycles, int tall_from, bool split,
                   int* split_slots, std::vector<SrRowTile>* out, int* lds_bytes) {
  double work = 0;
  int64_t n_short = 0;
  for (int f : phases) {
    const SrPhase& ph = p.phases[f];
    const int C = p.nodes[ph.node].C;
    work += sr_rows_work(p, f);
    n_short += C <= 32 ? ceil_div(ph.I, 128) : (int64_t)ceil_div(ph.I, 64) * ceil_div(C, 64);
  }
  const double share = std::max(work, work_cycles) / SR_CUS;
  if (work_cycles > work && work > 0) n_short = (int64_t)(n_short * (work_cycles / work));
  // cycles from a tile's start to its end on a moderately busy compute unit
  auto latency = [&](int shape, double steps) {
    int ti, tj;
    sr_f32_shape(shape, &ti, &tj);
    if (shape == SR_F32_SMALL) return steps / 4 * 750.0 + 5000.0;
    return steps * std::max(ti * tj / 8.0, 700.0) + 5000.0;
  };
  struct Keyed { double cost; SrRowTile t; };
  std::vector<std::vector<Keyed>> per_xcd(SR_XCDS);
  for (int f : phases) {
    const SrPhase& ph = p.phases[f];
    const int C = p.nodes[ph.node].C;
    int tall, mid;
    if (C <= 32) { tall = SR_F32_128x32; mid = SR_F32_128x32; }
    else if (C <= 64 || (C + 127) / 128 * 128 - C >= 64) { tall = SR_F32_128x64; mid = SR_F32_64x64; }
    else { tall = SR_F32_128x128; mid = SR_F32_64x64; }
    int shape = SR_F32_SMALL, parts = 1;
    if (tall_from == 0 || (n_short >= tall_from && latency(tall, ph.steps) <= std::max(share, 20000.0))) {
      shape = tall;
    } else if (n_short >= 2 * SR_CUS && latency(mid, ph.steps) <= std::max(share, 12000.0)) {
      shape = mid;
    } else {
      const double lat = latency(SR_F32_SMALL, ph.steps), want = std::max(share, 10000.0);
      if (split && lat > want) parts = std::max(1, std::min(std::min(ceil_div((int64_t)lat, (int64_t)want), 16), ph.steps / 16));
    }
    int ti, tj;
    sr_f32_shape(shape, &ti, &tj);
    *lds_bytes = std::max(*lds_bytes, sr_f32_lds_bytes(shape));
    const int n_i = ceil_div(ph.I, ti), n_j = ceil_div(C, tj);
    const int64_t total = (int64_t)n_i * n_j * parts;
    int64_t k = 0;
    for (int a = 0; a < n_i; ++a)
      for (int b = 0; b < n_j; ++b) {
        int slot = -1;
        if (parts > 1) {
          slot = *split_slots;
          *split_slots += parts * (shape == SR_F32_SMALL ? 1 : ti * tj / 1024);
        }
        for (int part = 0; part < parts; ++part, ++k) {
          SrRowTile t{};
          t.phase = f;
          t.shape = shape;
          t.i0 = a * ti;
          t.j0 = b * tj;
          t.step_begin = (int)((int64_t)ph.steps * part / parts);
          t.step_end = (int)((int64_t)ph.steps * (part + 1) / parts);
          t.split_slot = slot;
          t.part = part | (parts << 16);
          per_xcd[k * SR_XCDS / total].push_back(Keyed{latency(shape, (double)ph.steps / parts), t});
        }
      }
  }
  // workgroup i runs on XCD i % 8: every XCD takes an eighth of each node's pixels, longest tiles first
  size_t longest = 0;
  for (auto& v : per_xcd) {
    std::stable_sort(v.begin(), v.end(), [](const Keyed& a, const Keyed& b) { return a.cost > b.cost; });
    longest = std::max(longest, v.size());
  }
  SrRowTile none{};
  none.phase = -1;
  for (size_t k = 0; k < longest; ++k)
    for (int x = 0; x < SR_XCDS; ++x) out->push_back(k < per_xcd[x].size() ? per_xcd[x][k].t : none);
}
