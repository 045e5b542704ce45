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

constexpr int64_t kRows = ((int64_t)1 << 31) - 256;   // rows, columns and reduction indices are ints, some past the last one

// rows of the node, and the rows and columns of its images, are counted in ints
bool rows_fit(const sr_graph* g, const sr_node_desc& d) {
  return (int64_t)g->batch * d.height * d.width < kRows && std::max(d.height, d.width) < (1 << 30) && d.channels < (1 << 27);
}

// theta: offsets in 32 bits; one edge's reduction over (tap, channel) in an int, and a dense edge's source as a row of one
bool weights_fit(const EdgeRt& e, const Geometry& q) {
  return (int64_t)e.w_count < ((int64_t)1 << 32) && (int64_t)e.kh * e.kw * std::max(q.Cin, q.Cout) < kRows;
}

// The lines of segment s, in the order in which a step's indices lie in LDS.  Segments that differ in nothing that a line holds
// share a table: a node that a convolution and a dense edge read has a phase, and a segment of either, per pixel.
void add_lines(SrRowPlan* p, SrSeg* s, bool in_turn) {
  s->lines = -1;
  if ((s->flags & SR_SEG_QUADS) || s->R > SR_LINES_MAX) return;
  const auto known = p->line_tables.emplace(std::array<int, 6>{s->GC, s->GW, s->ntj, s->R, s->dir, in_turn}, -1);
  int& at = known.first->second;
  if (!known.second) {
    s->lines = at;
    return;
  }
  const int first = (int)p->lines.size();
  for (int r0 = 0; r0 < s->R; r0 += SR_F32_KS)
    for (int l = 0; l < SR_F32_KS; ++l) {
      const int r = r0 + (in_turn ? sr_in_turn(l) : l);
      SrLine x{0, SR_NO_ROW, SR_NO_ROW, 0};
      if (r < s->R) {
        const SrTapAt t = sr_tap_at(*s, r);
        const long long off = sr_gather_off(*s, t);
        if (off != (int32_t)off) {   // taps of an image of 2^31 floats a row apart and more
          p->lines.resize(first);
          return;
        }
        x = SrLine{(int32_t)off, s->dir * t.vi, s->dir * t.vj, 0};
      }
      p->lines.push_back(x);
    }
  at = s->lines = first;
}

}  // namespace

bool sr_rows_take_forward(const sr_graph* g, int v) {
  for (const EdgeRt& e : g->edges) {
    if (e.d.dst != v) continue;
    const sr_node_desc& s = g->nodes[e.d.src].d;
    if (e.d.kind == SR_EDGE_GAP_DENSE || (e.d.kind == SR_EDGE_DENSE && image_floats(s) >= kRows)) return false;
    if (!rows_fit(g, g->nodes[v].d) || !rows_fit(g, s) || !weights_fit(e, geometry(g, e))) return false;
  }
  return true;
}

bool sr_rows_take_training(const sr_graph* g) {
  for (const EdgeRt& e : g->edges) {
    const sr_node_desc &s = g->nodes[e.d.src].d, &d = g->nodes[e.d.dst].d;
    if (e.d.kind == SR_EDGE_DENSE && image_floats(s) >= kRows) return false;
    const Geometry q = geometry(g, e);
    if (!rows_fit(g, d) || !rows_fit(g, s) || !weights_fit(e, q)) return false;
    // a gradient tile's step: 16 pixels of the target, whose windows lie in this many images of the source
    const int64_t images = std::min<int64_t>(g->batch, 15 / ((int64_t)d.height * d.width) + 2);
    if (images * q.H * q.W * q.Cin >= ((int64_t)1 << 32)) return false;
  }
  return true;
}

int sr_rows_forward(SrRowPlan* p, const sr_graph* g, int v, const SrTrainIds* ids) {
  const NodeRt& n = g->nodes[v];
  // a window's values that a rectifier may yet read have one order of sums whatever the batch and the tiles, also inside a step
  const bool free_order = !ids || (v == ids->out_node && ids->seed < 0);
  SrRowNode node{};
  node.out = v;
  node.x = node.seed = -1;
  node.mask = ids ? ids->mask0 + v : -1;
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
  for (int ei = 0; ei < g->n_edges; ++ei) {
    const EdgeRt& e = g->edges[ei];
    if (e.d.dst != v) continue;
    const Geometry q = geometry(g, e);
    SrSeg s{};
    s.w = e.w_dev;
    if (e.d.kind == SR_EDGE_GAP_DENSE) {
      s.tensor = ids->mean[ei];   // of the frame the rows belong to: the lag was applied when the means were taken
    } else {
      s.tensor = e.d.src;
      s.flags = (e.d.bridge ? SR_SEG_LAG : 0) | (g->an.is_input[e.d.src] ? 0 : SR_SEG_ZERO0);
    }
    if (q.Cin % 4 == 0 && (free_order || q.Cout % 4 == 0)) s.flags |= SR_SEG_QUADS;
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
    s.d_wup = sr_div_for(1);
    ph.steps += ceil_div(s.R, SR_F32_KS);
    add_lines(p, &s, ids != nullptr);
    p->segs.push_back(s);
  }
  ph.seg_end = (int)p->segs.size();
  p->nodes.push_back(node);
  p->phases.push_back(ph);
  return (int)p->phases.size() - 1;
}

// State gradient of node v from the gradients of all its readers.  A stride-s edge pairs a source pixel only with the
// taps of its own residues, so the pixels are cut into S x S phases, S the common multiple of the strides of v's
// outgoing convolutions, each with its own tap lists.  A dense edge pairs a pixel with a slice of theta of its own: a
// node all of whose outgoing edges are dense is one row per image over all its elements, and one that has convolutions
// as well gets a phase per pixel.
int sr_rows_backward(SrRowPlan* p, const sr_graph* g, int v, const SrTrainIds& ids) {
  const NodeRt& n = g->nodes[v];
  const int H = n.d.height, W = n.d.width, C = n.d.channels;
  std::vector<int> gap, dense, conv;
  int64_t S = 1;
  for (int ei = 0; ei < g->n_edges; ++ei) {
    const EdgeRt& e = g->edges[ei];
    if (e.d.src != v || ids.dist[e.d.dst] < 0) continue;
    if (e.d.kind == SR_EDGE_GAP_DENSE) gap.push_back(ei);
    else if (e.d.kind == SR_EDGE_DENSE) dense.push_back(ei);
    else {
      conv.push_back(ei);
      int64_t a = S, b = e.d.stride;
      while (b) { const int64_t t = a % b; a = b; b = t; }
      S = S / a * e.d.stride;
    }
  }
  const bool flat = !dense.empty() && conv.empty() && gap.empty();
  if (!flat && !dense.empty()) S = std::max(H, W);
  S = std::min<int64_t>(S, std::max(H, W));   // from there on every phase is a single pixel
  // (a single pixel pairs through stride s with the taps of its residue whatever S is)
  SrRowNode node{};
  node.out = ids.grad0 + v;
  node.x = v;
  node.seed = v == ids.out_node ? ids.seed : -1;
  node.mask = ids.mask0 + v;
  node.C = flat ? H * W * C : C;
  node.H = flat ? 1 : H;
  node.W = flat ? 1 : W;
  node.act = n.d.act;
  node.gnode = v;
  const int node_index = (int)p->nodes.size(), first = (int)p->phases.size();
  p->nodes.push_back(node);
  for (int phh = 0; phh < (flat ? 1 : std::min<int64_t>(S, H)); ++phh)
    for (int pww = 0; pww < (flat ? 1 : std::min<int64_t>(S, W)); ++pww) {
      SrPhase ph{};
      ph.node = node_index;
      ph.S = flat ? 1 : (int)S;
      ph.ph = phh;
      ph.pw = pww;
      ph.Hp = flat ? 1 : ceil_div(H - phh, S);
      ph.Wp = flat ? 1 : ceil_div(W - pww, S);
      ph.I = g->batch * ph.Hp * ph.Wp;
      ph.image_scale = 1.f / (float)(H * W);
      ph.d_wp = sr_div_for(ph.Wp);
      ph.d_hpwp = sr_div_for(ph.Hp * ph.Wp);
      ph.seg_begin = (int)p->segs.size();
      auto add = [&](const EdgeRt& e, SrSeg s, int nti, int ntj) {
        s.w = e.w_dev;
        s.tensor = ids.grad0 + e.d.dst;
        s.flags |= (e.d.bridge ? SR_SEG_LAG : 0) | (s.GC % 4 == 0 ? SR_SEG_QUADS : 0);
        s.dir = -1;
        s.ntj = ntj;
        s.R = nti * ntj * s.GC;
        s.ldw = node.C;
        s.dist = ids.dist[e.d.dst];
        s.step0 = ph.steps;
        s.d_gc = sr_div_for(s.GC);
        s.d_ntj = sr_div_for(ntj);
        s.d_up = sr_div_for(1);
        ph.steps += ceil_div(s.R, SR_F32_KS);
        add_lines(p, &s, false);
        p->segs.push_back(s);
      };
      for (int ei : gap) {
        const EdgeRt& e = g->edges[ei];
        SrSeg s{};
        s.flags = SR_SEG_IMAGE;
        s.GH = s.GW = 1;
        s.GC = g->nodes[e.d.dst].d.channels;
        s.d_wup = sr_div_for(1);
        add(e, s, 1, 1);
      }
      ph.seg_image = (int)p->segs.size();
      for (int ei : dense) {
        const EdgeRt& e = g->edges[ei];
        SrSeg s{};
        s.GH = s.GW = 1;
        s.GC = g->nodes[e.d.dst].d.channels;
        s.wt0 = flat ? 0 : phh * W + pww;   // the pixel's slice of theta
        s.d_wup = sr_div_for(1);
        add(e, s, 1, 1);
      }
      for (int ei : conv) {
        const EdgeRt& e = g->edges[ei];
        const Geometry q = geometry(g, e);
        const int ti0 = (phh + q.pad) % q.stride, tj0 = (pww + q.pad) % q.stride;
        const int nti = ti0 < q.kh ? ceil_div(q.kh - ti0, q.stride) : 0, ntj = tj0 < q.kw ? ceil_div(q.kw - tj0, q.stride) : 0;
        if (nti * ntj == 0) continue;
        // pixel (hh S + ph) pairs through the tap ti0 + a s with row (hh S + ph + pad - ti0) / s - a of the edge's
        // result, each row of which stands for `up` rows of the target
        SrSeg s{};
        s.GH = g->nodes[e.d.dst].d.height;
        s.GW = g->nodes[e.d.dst].d.width;
        s.GC = q.Cout;
        s.rs = ph.Hp > 1 || ph.Wp > 1 ? (int)(S / q.stride) * q.up : 0;
        s.r0h = (phh + q.pad - ti0) / q.stride * q.up + q.up - 1;
        s.r0w = (pww + q.pad - tj0) / q.stride * q.up + q.up - 1;
        s.wt0 = ti0 * q.kw + tj0;
        s.wti = q.stride * q.kw;
        s.wtj = q.stride;
        s.d_wup = sr_div_for(q.up);
        add(e, s, nti * q.up, ntj * q.up);
      }
      ph.seg_end = (int)p->segs.size();
      p->phases.push_back(ph);
    }
  return first;
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
// What the constants are worth (us; clips of MNIST SR B=128 T=16, DSR2 B=64 T=16, DSR2 sequential B=1 T=16, MNIST S B=9 T=32, DSR6 B=4 T=8,
// windows of MNIST SR B=128 W=8, DSR2 B=16 W=4, DSR5 B=1 W=4; as they are 208 1306 1019 321 264 324 225 181) --
//   6000 cycles a 32 x 32 tile may take uncut    5000: all within noise; 10000: 221 1305 1057 354 265 327 227 184
//   750 per four steps of 32 x 32 tiles          500: 207 1724 1037 325 257 325 220 183; 1100: 208 1306 1019 321 278 325 224 180
// The reverse launches alone, of 10000 cycles for 6000: MNIST SR B=128 11.0-11.8 -> 11.2-12.7 each, DSR2 B=64 and GTSRB-shaped equal.
// Measured when the kernels were slower:
//   12000 of a middle one, 512 of them           24000, 256: noise
//   700 a step of middle tiles                   600, 900: noise
//   20000 cycles a tall tile may take, 5000 fixed, at most 16 parts   measured when the kernels were slower: noise within 4 %
void sr_rows_tiles(const SrRowPlan& p, const std::vector<int>& phases, double work_cycles, int tall_from, bool split, bool ordered,
                   int* split_slots, std::vector<SrRowTile>* out, int* shapes) {
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
  struct Keyed { double cost; int tile; };
  std::vector<SrRowTile> tiles;
  std::vector<std::vector<Keyed>> per_xcd(SR_XCDS);
  for (int f : phases) {
    const SrPhase& ph = p.phases[f];
    const int C = p.nodes[ph.node].C;
    int tall, mid;
    if (C <= 32) { tall = SR_F32_128x32; mid = SR_F32_128x32; }
    // (ordered tiles: a lane would hold 64 accumulators and 64 sums of an 128 x 128 tile, which leaves two workgroups per CU;
    // GTSRB-shaped window 6181 us with them, 6125 without)
    else if (ordered || C <= 64 || (C + 127) / 128 * 128 - C >= 64) { tall = SR_F32_128x64; mid = SR_F32_64x64; }
    else { tall = SR_F32_128x128; mid = SR_F32_64x64; }
    int shape = SR_F32_SMALL, parts = 1;
    if (tall_from == 0 || (n_short >= tall_from && latency(tall, ph.steps) <= std::max(share, 20000.0))) {
      shape = tall;
    } else if (n_short >= 2 * SR_CUS && latency(mid, ph.steps) <= std::max(share, 12000.0)) {
      shape = mid;
    } else {
      const double lat = latency(SR_F32_SMALL, ph.steps), want = std::max(share, 6000.0);
      if (split && lat > want) parts = std::max(1, std::min(std::min(ceil_div((int64_t)lat, (int64_t)want), 16), ph.steps / 16));
    }
    int ti, tj;
    sr_f32_shape(shape, &ti, &tj);
    *shapes |= 1 << shape;
    const int n_i = ceil_div(ph.I, ti), n_j = ceil_div(C, tj);
    const int64_t total = (int64_t)n_i * n_j * parts;
    int64_t k = 0;
    for (int a = 0; a < n_i; ++a)
      for (int b = 0; b < n_j; ++b) {
        int slot = -1;
        if (parts > 1) {
          slot = *split_slots;
          *split_slots += parts;   // 32 x 32 floats each
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
          per_xcd[k * SR_XCDS / total].push_back(Keyed{latency(shape, (double)ph.steps / parts), (int)tiles.size()});
          tiles.push_back(t);
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
    for (int x = 0; x < SR_XCDS; ++x) out->push_back(k < per_xcd[x].size() ? tiles[per_xcd[x][k].tile] : none);
}

void sr_grad_plan(SrGradPlan* p, const sr_graph* g, const SrTrainIds& ids, int W, int lo, int hi, bool first, int tall_from, int items_per_cu) {
  // columns of work: per edge its shape, tiles, steps
  struct Item { int edge, shape, n_i, n_j, steps; double step_cycles; };
  std::vector<Item> items;
  double work = 0;
  int64_t n_short = 0;
  for (int ei = 0; ei < g->n_edges; ++ei) {
    const EdgeRt& e = g->edges[ei];
    const int w = e.d.dst;
    // frames in which the target has a gradient and the source is not the window's zero initial state
    const int f0 = std::max(lo, e.d.bridge && !g->an.is_input[e.d.src] ? 2 : 1);
    const int f1 = ids.dist[w] < 0 ? 0 : std::min(hi, W - ids.dist[w]);
    if (f1 < f0) {
      if (first) {
        p->sums.push_back(SrGradSum{0, (long long)e.w_count, 0, ei, p->sum_blocks, 0});
        p->sum_blocks += ceil_div(e.w_count, 64);
      }
      continue;
    }
    const Geometry q = geometry(g, e);
    SrGradEdge d{};
    d.x = e.d.kind == SR_EDGE_GAP_DENSE ? ids.mean[ei] : e.d.src;
    d.dy = ids.grad0 + w;
    d.lag = e.d.kind == SR_EDGE_GAP_DENSE ? 0 : (int)e.d.bridge;
    d.frame0 = f0;
    d.H = q.H; d.W = q.W; d.Cin = q.Cin;
    d.Ho = q.Ho * q.up; d.Wo = q.Wo * q.up; d.Cout = q.Cout;
    d.kw = q.kw; d.stride = q.stride; d.pad = q.pad;
    d.I = q.kh * q.kw * q.Cin;
    d.M = g->batch * d.Ho * d.Wo;
    d.quads_in = q.Cin % 4 == 0;
    d.quads_out = q.Cout % 4 == 0;
    d.dst = ei;
    d.steps_per_frame = ceil_div(d.M, SR_F32_KS);
    d.d_cin = sr_div_for(q.Cin);
    d.d_kw = sr_div_for(q.kw);
    d.d_wo = sr_div_for(d.Wo);
    d.d_howo = sr_div_for(d.Ho * d.Wo);
    d.d_up = sr_div_for(q.up);
    d.d_steps = sr_div_for(d.steps_per_frame);
    d.along = q.up == 1 && d.M >= SR_F32_KS && (int64_t)g->batch * q.H * q.W * q.Cin < ((int64_t)1 << 31) && q.Cout < (1 << 22) &&
              std::max(q.Ho, q.Wo) < (1 << 24) / std::max(q.stride, 1);
    Item it{(int)p->edges.size(), 0, 0, 0, d.steps_per_frame * (f1 - f0 + 1), 0};
    p->edges.push_back(d);
    items.push_back(it);
    n_short += (int64_t)ceil_div(d.I, 64) * ceil_div(d.Cout, 64) * std::max(1, it.steps / 64);
  }
  const bool tall = n_short >= tall_from;
  for (Item& it : items) {
    const SrGradEdge& d = p->edges[it.edge];
    if (d.Cout <= 32) it.shape = SR_F32_128x32;
    else if (!tall || d.I <= 64) it.shape = SR_F32_64x64;
    else it.shape = (d.Cout <= 64 || (d.Cout + 127) / 128 * 128 - d.Cout >= 64) ? SR_F32_128x64 : SR_F32_128x128;
    int ti, tj;
    sr_f32_shape(it.shape, &ti, &tj);
    it.n_i = ceil_div(d.I, ti);
    it.n_j = ceil_div(d.Cout, tj);
    // (measured, us a step of three workgroups on a compute unit: 128 x 32 1.55, fetched element by element 2.56; 128 x 64 1.82; 128 x 128 2.8)
    it.step_cycles = std::max(ti * tj / 8.0, 900.0) * (d.quads_in ? 1.0 : 1.6);
    work += it.step_cycles * it.steps * it.n_i * it.n_j;
    p->shapes |= 1 << it.shape;
  }
  // The pixel sums are cut into slices so that the launch has about items_per_cu (SR_GRAD_ITEMS: 12) work items of equal length per compute unit,
  // none shorter than 16 steps: shorter ones are dominated by filling the pipeline and by their partial sums.  (Six, two
  // generations on the three places of a compute unit, left a fifth of the DSR2 window's launch to the last ones:
  // 1480 us with 6, 1430 with 12, 1440 with 16; GTSRB-shaped 5630, 5550, 5555.)
  const double item_cycles = work / (SR_CUS * (double)items_per_cu);
  struct Keyed { double cost; int tile; };
  std::vector<SrGradTile> tiles;
  // Every XCD takes an eighth of each edge's tiles, slice by slice: the tiles of a slice read the same pixels, which then come
  // through one L2 (workgroup i runs on XCD i % 8).  Where that cannot be even, of few tiles each goes to the XCD with the least
  // work so far, and of many the first eighth does.  (All of them from XCD 0 on: it had 3.0 times the mean of an MNIST SR window of
  // one image, 1.5 times of 16.)
  std::vector<std::vector<Keyed>> per_xcd(SR_XCDS);
  std::vector<double> load(SR_XCDS, 0.0);
  int first_xcd = 0;
  auto least = [&]() { return (int)(std::min_element(load.begin(), load.end()) - load.begin()); };
  auto place = [&](int64_t k, int64_t total, double cost, const SrGradTile& t) {   // the k-th of `total` that belong together
    if (k == 0 || total < 4 * SR_XCDS) first_xcd = least();
    const int x = total < 4 * SR_XCDS ? first_xcd : (int)((first_xcd + k * SR_XCDS / total) % SR_XCDS);
    load[x] += cost;
    per_xcd[x].push_back(Keyed{cost, (int)tiles.size()});
    tiles.push_back(t);
  };
  for (const Item& it : items) {
    SrGradEdge& d = p->edges[it.edge];
    const int64_t most = std::max(1, it.steps / 16);
    const int64_t want = (int64_t)std::ceil(it.step_cycles * it.steps / std::max(item_cycles, 1.0));
    d.slices = (int)std::max<int64_t>(1, std::min<int64_t>(std::min(want, most), 1024));
    if (d.slices > 1) {
      d.part_at = p->part_floats;
      p->part_floats += ((long long)d.I * d.Cout * d.slices + 63) / 64 * 64;
      p->sums.push_back(SrGradSum{d.part_at, (long long)d.I * d.Cout, d.slices, d.dst, p->sum_blocks, 0});
      p->sum_blocks += ceil_div((int64_t)d.I * d.Cout, 64);
    }
    int ti, tj;
    sr_f32_shape(it.shape, &ti, &tj);
    const int64_t total = (int64_t)d.slices * it.n_i * it.n_j;
    int64_t k = 0;
    for (int s = 0; s < d.slices; ++s)
      for (int a = 0; a < it.n_i; ++a)
        for (int b = 0; b < it.n_j; ++b, ++k) {
          SrGradTile t{};
          t.edge = it.edge;
          t.shape = it.shape;
          t.i0 = a * ti;
          t.j0 = b * tj;
          t.step_begin = (int)((int64_t)it.steps * s / d.slices);
          t.step_end = (int)((int64_t)it.steps * (s + 1) / d.slices);
          t.slice = s;
          place(k, total, it.step_cycles * (t.step_end - t.step_begin), t);
        }
  }
  for (int v = 0; v < g->n_nodes; ++v) {
    if (g->an.is_input[v]) continue;
    const sr_node_desc& d = g->nodes[v].d;
    const int f1 = ids.dist[v] < 0 ? 0 : std::min(hi, W - ids.dist[v]);
    SrGradSum sum{0, d.channels, 0, g->n_edges + v, p->sum_blocks, 0};
    if (f1 >= lo) {
      SrGradBias b{};
      b.dy = ids.grad0 + v;
      b.C = d.channels;
      b.M = g->batch * d.height * d.width;
      b.frame0 = lo;
      b.d_m = sr_div_for(b.M);
      const int64_t rows = (int64_t)b.M * (f1 - lo + 1);
      const int slices = (int)std::max<int64_t>(1, std::min<int64_t>(512, rows / 256));
      b.part_at = p->part_floats;
      p->part_floats += ((long long)d.channels * slices + 63) / 64 * 64;
      sum.part_at = b.part_at;
      sum.slices = slices;
      const int64_t total = (int64_t)slices * ceil_div(d.channels, 64);
      int64_t k = 0;
      for (int s = 0; s < slices; ++s)
        for (int j = 0; j < d.channels; j += 64, ++k) {
          SrGradTile t{};
          t.edge = (int)p->biases.size();
          t.j0 = j;
          t.step_begin = (int)(rows * s / slices);
          t.step_end = (int)(rows * (s + 1) / slices);
          t.slice = s;
          t.kind = 1;
          place(k, total, (t.step_end - t.step_begin) * 8.0, t);
        }
      p->biases.push_back(b);
    } else if (!first) {
      continue;
    }
    p->sums.push_back(sum);
    p->sum_blocks += ceil_div(d.channels, 64);
  }
  size_t longest = 0;
  for (auto& v : per_xcd) {
    std::stable_sort(v.begin(), v.end(), [](const Keyed& a, const Keyed& b) { return a.cost > b.cost; });
    longest = std::max(longest, v.size());
  }
  SrGradTile none{};
  none.kind = 2;
  for (size_t k = 0; k < longest; ++k)
    for (int x = 0; x < SR_XCDS; ++x) p->tiles.push_back(k < per_xcd[x].size() ? tiles[per_xcd[x][k].tile] : none);
}
