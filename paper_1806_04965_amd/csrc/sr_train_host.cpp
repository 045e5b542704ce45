// Host side of one training window (Sec. 3: rollout window of size W; Sec. 2: backpropagation through the rolled-out
// network; App. A2: loss): plans the window's launches and runs them.
//
// A window is a directed graph over (frame, node).  Its forward pass runs launch by launch in the order of the depth of
// the pairs in that graph (the inference tableau of Eq. 5 over the whole window), one launch for all pairs of a depth,
// whatever their frame; the reverse sweep likewise in the order of the depth from the loss terms.  Every frame's states
// and state gradients are kept, so that all weight and bias gradients are one launch behind the sweep.
//
// Measured (launch per edge and per elementwise pass on four streams, state gradients accumulated in memory -> launch
// per depth, everything fused): MNIST SR B=128 W=8 sequential 250 launches, 1.98 ms -> 22, 0.33; DSR2 B=64 W=8 485,
// 5.1 -> 18, 1.4; GTSRB-shaped B=128 W=4 52.7 -> 10, 5.5 (a window
// shorter than the network is deep: an eighth of its nominal operations reach the loss; 107 TFLOP/s on those).
//
// Values that cannot reach a loss term are not computed: node v is at least dist(v) bridging edges away from the out
// node, so its states and gradients of the frames after W - dist(v) have no reader.  Nor are the products with the
// window's initial state, which is zero.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <memory>
#include <string>
#include <vector>

#include "../../include/sr.h"
#include "sr_f32.h"
#include "sr_graph.h"
#include "sr_internal.h"

// The plan of windows of W frames with the loss at node `out`: device tables in one allocation, offsets into the arena.
struct SrTrainPlan {
  struct Key {   // what it was made for, and the options that it went by
    int W, out, tall_from, frames_kept;
    bool split;
    bool operator==(const Key& o) const {
      return W == o.W && out == o.out && tall_from == o.tall_from && frames_kept == o.frames_kept && split == o.split;
    }
  };
  struct Launch {
    int run0 = 0, n_runs = 0, blocks = 0, shapes = 0;
    std::vector<std::pair<SrPool, std::pair<int, int>>> pools;   // before it: means of (first frame, number of frames)
  };
  struct Chunk {   // frames lo..hi of the reverse sweep
    int lo = 0, hi = 0;
    std::vector<Launch> back;
    SrGradPlan grad;
    const SrGradEdge* edges = nullptr;
    const SrGradBias* biases = nullptr;
    const SrGradTile* tiles = nullptr;
    const SrGradSum* sums = nullptr;
  };
  Key key{};
  int ring = 0;
  std::vector<Launch> fwd;
  std::vector<Chunk> chunks;
  SrTrainIds ids;
  bool out_is_sink = false;
  float* terms = nullptr;
  float* part = nullptr;
  void* tables = nullptr;
  SrTensor* tensors = nullptr;
  float** dst = nullptr;
  const SrRun* runs = nullptr;
  SrRowArgs rows_fwd{}, rows_back{};
  SrTrainPlan() = default;
  SrTrainPlan(const SrTrainPlan&) = delete;
  ~SrTrainPlan() {
    if (tables) hipFree(tables);
  }
};

// what a graph keeps for its training windows between calls
struct SrTrainState {
  // one arena: the states of the frames 1..W, the state gradients of a chunk of frames, and scratch
  float* arena = nullptr;
  size_t arena_floats = 0;
  std::vector<float*> rms_w, rms_b;   // RMSprop's running mean of the squared gradient, per edge / node (on first use)
  // Plans, the last one used first; all work in the one arena, one window at a time.  Making a plan takes up to some
  // milliseconds of the host; programs that alternate window sizes or out nodes use a few.
  std::vector<std::unique_ptr<SrTrainPlan>> plans;
};
constexpr size_t kTrainPlans = 4;

void sr_train_state_release(SrTrainState* t) {
  if (!t) return;
  t->plans.clear();
  if (t->arena) hipFree(t->arena);
  delete t;
}

namespace {

SrTrainState& train_state(sr_graph* g) {
  if (!g->train) g->train = new SrTrainState();
  return *g->train;
}

// device tables gathered on the host and uploaded in one copy
struct Blob {
  std::vector<unsigned char> bytes;
  template <typename T>
  size_t add(const std::vector<T>& v) {
    bytes.resize((bytes.size() + 255) / 256 * 256);
    const size_t at = bytes.size();
    bytes.resize(at + std::max<size_t>(v.size(), 1) * sizeof(T));
    if (!v.empty()) std::memcpy(&bytes[at], v.data(), v.size() * sizeof(T));
    return at;
  }
};

constexpr size_t kGradRingBytes = (size_t)16 << 30;   // state gradients kept at a time: a longer window is swept in chunks

size_t node_floats(const sr_graph* g, int v) {
  const sr_node_desc& d = g->nodes[v].d;
  return (size_t)g->batch * d.height * d.width * d.channels;
}

// (frame, node) pairs of one depth as runs over the nodes' tile lists, longest tiles first
struct NodeTiles { int tile0 = 0, n = 0, slots = 0, shapes = 0; double length = 0; };

// the launches of pairs[depth]; returns the split slots the largest one needs
int make_launches(const std::vector<std::vector<std::pair<int, int>>>& pairs, const std::vector<NodeTiles>& tiles,
                  std::vector<SrRun>* runs, std::vector<SrTrainPlan::Launch>* out) {
  int most = 0;
  for (auto level : pairs) {   // (frame, node)
    std::stable_sort(level.begin(), level.end(), [&](const std::pair<int, int>& a, const std::pair<int, int>& b) {
      return tiles[a.second].length > tiles[b.second].length;
    });
    SrTrainPlan::Launch l;
    l.run0 = (int)runs->size();
    int slots = 0;
    for (const auto& fv : level) {
      const NodeTiles& t = tiles[fv.second];
      runs->push_back(SrRun{l.blocks, t.tile0, fv.first, slots});
      l.blocks += t.n;
      l.shapes |= t.shapes;
      slots += t.slots;
    }
    l.n_runs = (int)level.size();
    most = std::max(most, slots);
    out->push_back(l);
  }
  return most;
}

// The plan for `key` within `room`; *kept receives the number of frames whose state gradients it keeps at a time.
sr_status make_plan(sr_graph* g, SrTrainState& S, SrTrainPlan& T, const SrTrainPlan::Key& key, const SrTrainRoom& room, int* kept) {
  const int N = g->n_nodes, E = g->n_edges, B = g->batch, W = key.W, out_node = key.out;
  SrTrainIds ids;
  ids.grad0 = N;
  ids.mask0 = 2 * N;
  ids.seed = 3 * N;
  ids.out_node = out_node;
  ids.mean.assign(E, -1);
  int n_tensors = 3 * N + 1;
  for (int e = 0; e < E; ++e)
    if (g->edges[e].d.kind == SR_EDGE_GAP_DENSE) ids.mean[e] = n_tensors++;
  ids.dist.assign(N, -1);
  ids.dist[out_node] = 0;
  for (bool changed = true; changed;) {
    changed = false;
    for (const EdgeRt& e : g->edges) {
      if (ids.dist[e.d.dst] < 0) continue;
      const int d = ids.dist[e.d.dst] + (int)e.d.bridge;
      int& s = ids.dist[e.d.src];
      if (s < 0 || d < s) { s = d; changed = true; }
    }
  }
  auto last = [&](int v) { return ids.dist[v] < 0 ? 0 : W - ids.dist[v]; };   // last frame of v that a loss term depends on
  T.out_is_sink = true;
  for (const EdgeRt& e : g->edges)
    if (e.d.src == out_node && ids.dist[e.d.dst] >= 0) T.out_is_sink = false;
  if (T.out_is_sink) ids.seed = -1;
  std::vector<int> order;   // sources of R = 0 edges before their targets
  for (int v = 0; v < N; ++v)
    if (!g->an.is_input[v] && ids.dist[v] >= 0) order.push_back(v);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return g->an.level[a] < g->an.level[b]; });

  // arena
  size_t at = 0;
  auto take = [&](size_t n) { size_t r = at; at += (n + 63) / 64 * 64; return r; };
  std::vector<size_t> in_frame(N, 0);
  size_t frame_floats = 0;
  int64_t most_pixels = 1;
  for (int v = 0; v < N; ++v) {
    if (g->an.is_input[v]) continue;
    in_frame[v] = frame_floats;
    frame_floats += (node_floats(g, v) + 63) / 64 * 64;
    most_pixels = std::max<int64_t>(most_pixels, (int64_t)B * g->nodes[v].d.height * g->nodes[v].d.width);
  }
  int chunk = (int)std::max<int64_t>(1, std::min<int64_t>(W, std::min<int64_t>(kGradRingBytes / 4 / frame_floats, ((int64_t)1 << 30) / most_pixels)));
  if (key.frames_kept > 0) chunk = std::min(chunk, key.frames_kept);
  chunk = std::min(chunk, room.frames);
  *kept = chunk;
  const int ring = chunk + 1;
  const size_t x_at = take(frame_floats * W), dx_at = take(frame_floats * ring);
  const size_t seed_at = take((size_t)W * B * g->nodes[out_node].d.channels);
  std::vector<size_t> mean_at(E, 0);
  for (int e = 0; e < E; ++e)
    if (ids.mean[e] >= 0) mean_at[e] = take((size_t)W * B * g->nodes[g->edges[e].d.src].d.channels);
  const size_t terms_at = take((size_t)W * B);

  // forward: depth of (frame, node)
  std::vector<std::vector<int>> depth(W + 2, std::vector<int>(N, 0));
  int deepest = 0;
  std::vector<std::vector<std::pair<int, int>>> pairs;
  auto put = [&](int d, int i, int v) {
    if ((int)pairs.size() <= d) pairs.resize(d + 1);
    pairs[d].push_back({i, v});
  };
  for (int i = 1; i <= W; ++i)
    for (int v : order) {
      if (i > last(v) || (v == out_node && T.out_is_sink)) continue;
      int d = 0;
      for (const EdgeRt& e : g->edges) {
        const int j = i - (int)e.d.bridge;
        if (e.d.dst == v && !g->an.is_input[e.d.src] && j >= 1) d = std::max(d, depth[j][e.d.src] + 1);
      }
      depth[i][v] = d;
      deepest = std::max(deepest, d + 1);
      put(d, i, v);
    }
  if (T.out_is_sink)   // nothing waits for the scores but the loss: all frames at once, last
    for (int i = 1; i <= W; ++i) put(deepest, i, out_node);

  SrRowPlan rf, rb;
  std::vector<SrRowTile> tf, tb;
  std::vector<NodeTiles> nf(N), nb(N);
  {
    std::vector<int> ph(N, -1);
    double work = 0;
    for (int v : order) {
      ph[v] = sr_rows_forward(&rf, g, v, &ids);
      work += sr_rows_work(rf, ph[v]) * std::max(last(v), 0);
    }
    for (int v : order) {
      NodeTiles& t = nf[v];
      t.tile0 = (int)tf.size();
      // a launch's work: the average one's; scores that nothing but the loss reads have a launch of their own (DSR2: 64 x 10
      // scores of 8192 products each, alone 75 us uncut, 23 in parts)
      const bool scores = v == out_node && T.out_is_sink;
      const double launch = scores ? sr_rows_work(rf, ph[v]) * W : work / std::max<size_t>(1, pairs.size());
      // the sums of all others have one order, so they are not cut into parts (SR_ROWS_ORDERED)
      sr_rows_tiles(rf, {ph[v]}, launch, key.tall_from, scores && key.split, true, &t.slots, &tf, &t.shapes);
      t.n = (int)tf.size() - t.tile0;
      t.length = rf.phases[ph[v]].steps * (tf[t.tile0].shape <= SR_F32_128x64 ? 2.0 : 1.0);
    }
  }
  std::vector<SrRun> runs;
  int slots = make_launches(pairs, nf, &runs, &T.fwd);
  // channel means: ahead of the launch that reads them
  for (int e = 0; e < E; ++e) {
    const EdgeRt& ed = g->edges[e];
    const int v = ed.d.dst;
    if (ids.mean[e] < 0 || ids.dist[v] < 0) continue;
    const sr_node_desc& sd = g->nodes[ed.d.src].d;
    const SrPool pool{ed.d.src, ids.mean[e], (int)ed.d.bridge, sd.height * sd.width, sd.channels, g->an.is_input[ed.d.src] ? 0 : 1};
    if (v == out_node && T.out_is_sink) {
      T.fwd[deepest].pools.push_back({pool, {1, W}});
    } else {
      for (int i = 1; i <= last(v); ++i) T.fwd[depth[i][v]].pools.push_back({pool, {i, 1}});
    }
  }

  // reverse sweep
  {
    std::vector<std::vector<int>> phs(N);
    double work = 0;
    for (int v : order) {
      if (v == out_node && T.out_is_sink) continue;
      const int first = sr_rows_backward(&rb, g, v, ids);
      for (int f = first; f < (int)rb.phases.size(); ++f) {
        phs[v].push_back(f);
        work += sr_rows_work(rb, f) * std::max(last(v), 0);
      }
    }
    const double per_launch = work / std::max<size_t>(1, pairs.size());
    for (int v : order) {
      if (phs[v].empty()) continue;
      NodeTiles& t = nb[v];
      t.tile0 = (int)tb.size();
      sr_rows_tiles(rb, phs[v], per_launch, key.tall_from, key.split, false, &t.slots, &tb, &t.shapes);
      t.n = (int)tb.size() - t.tile0;
      for (int f : phs[v]) t.length = std::max(t.length, rb.phases[f].steps * (tb[t.tile0].shape <= SR_F32_128x64 ? 2.0 : 1.0));
    }
    std::vector<int> rev(order.rbegin(), order.rend());   // readers of the same frame first
    for (int hi = W; hi >= 1; hi -= chunk) {
      SrTrainPlan::Chunk c;
      c.hi = hi;
      c.lo = std::max(1, hi - chunk + 1);
      std::vector<std::vector<int>> db(c.hi - c.lo + 2, std::vector<int>(N, 0));
      pairs.clear();
      for (int i = c.hi; i >= c.lo; --i)
        for (int v : rev) {
          if (i > last(v) || (v == out_node && T.out_is_sink)) continue;
          int d = 0;
          for (const EdgeRt& e : g->edges) {
            const int w = e.d.dst, j = i + (int)e.d.bridge;
            if (e.d.src != v || ids.dist[w] < 0 || j > last(w) || j > c.hi || (w == out_node && T.out_is_sink)) continue;
            d = std::max(d, db[j - c.lo][w] + 1);
          }
          db[i - c.lo][v] = d;
          put(d, i, v);
        }
      slots = std::max(slots, make_launches(pairs, nb, &runs, &c.back));
      sr_grad_plan(&c.grad, g, ids, W, c.lo, c.hi, hi == W, key.tall_from, room.items);
      T.chunks.push_back(std::move(c));
    }
  }
  long long part_floats = 0;
  for (const SrTrainPlan::Chunk& c : T.chunks) part_floats = std::max(part_floats, c.grad.part_floats);
  const size_t part_at = take((size_t)part_floats);
  const size_t slab_at = take((size_t)slots * 1024);

  if (at > S.arena_floats) {
    // what is in flight still uses the arena, and the tables of the other plans hold its address
    SR_HIP(g, hipStreamSynchronize(g->stream));
    S.plans.clear();
    if (S.arena) SR_HIP(g, hipFree(S.arena));
    S.arena = nullptr;
    S.arena_floats = 0;
    void* p = nullptr;
    SR_HIP(g, hipMalloc(&p, at * sizeof(float)));
    S.arena = (float*)p;
    S.arena_floats = at;
  }
  float* A = S.arena;
  auto tensor = [&](size_t offset, size_t floats_per_frame, int frame_of_slot0) {
    const long long stride = (long long)floats_per_frame * 4;
    return SrTensor{(char*)(A + offset) - stride * frame_of_slot0, stride};
  };
  std::vector<SrTensor> tensors(n_tensors, SrTensor{nullptr, 0});
  for (int v = 0; v < N; ++v) {
    if (g->an.is_input[v]) continue;   // the call's
    tensors[v] = tensor(x_at + in_frame[v], frame_floats, 1);        // slot = frame
    tensors[N + v] = tensor(dx_at + in_frame[v], frame_floats, 0);   // slot = frame % ring
  }
  tensors[3 * N] = tensor(seed_at, (size_t)B * g->nodes[out_node].d.channels, 1);
  for (int e = 0; e < E; ++e)
    if (ids.mean[e] >= 0) tensors[ids.mean[e]] = tensor(mean_at[e], (size_t)B * g->nodes[g->edges[e].d.src].d.channels, 1);

  Blob blob;
  const size_t o_tensors = blob.add(tensors), o_dst = blob.add(std::vector<float*>(E + N, nullptr)), o_runs = blob.add(runs);
  const size_t o_fn = blob.add(rf.nodes), o_fp = blob.add(rf.phases), o_fl = blob.add(rf.lines), o_fs = blob.add(rf.segs), o_ft = blob.add(tf);
  const size_t o_bn = blob.add(rb.nodes), o_bp = blob.add(rb.phases), o_bl = blob.add(rb.lines), o_bs = blob.add(rb.segs), o_bt = blob.add(tb);
  std::vector<std::vector<size_t>> o_chunk;
  for (const SrTrainPlan::Chunk& c : T.chunks)
    o_chunk.push_back({blob.add(c.grad.edges), blob.add(c.grad.biases), blob.add(c.grad.tiles), blob.add(c.grad.sums)});
  const size_t o_counters = blob.add(std::vector<int32_t>(slots, 0));   // zero between launches
  SR_HIP(g, hipMalloc(&T.tables, blob.bytes.size()));
  SR_HIP(g, hipMemcpy(T.tables, blob.bytes.data(), blob.bytes.size(), hipMemcpyHostToDevice));
  unsigned char* base = (unsigned char*)T.tables;
  T.tensors = (SrTensor*)(base + o_tensors);
  T.dst = (float**)(base + o_dst);
  SrSplitScratch split{A + slab_at, (int32_t*)(base + o_counters)};
  SrRowArgs a{};
  a.tensors = T.tensors;
  a.window = W;
  a.ring = ring;
  a.rec_node = -1;
  a.split = split;
  T.runs = (const SrRun*)(base + o_runs);
  T.rows_fwd = a;
  T.rows_fwd.nodes = (const SrRowNode*)(base + o_fn);
  T.rows_fwd.phases = (const SrPhase*)(base + o_fp);
  T.rows_fwd.lines = (const SrLine*)(base + o_fl);
  T.rows_fwd.segs = (const SrSeg*)(base + o_fs);
  T.rows_fwd.tiles = (const SrRowTile*)(base + o_ft);
  T.rows_back = a;
  T.rows_back.nodes = (const SrRowNode*)(base + o_bn);
  T.rows_back.phases = (const SrPhase*)(base + o_bp);
  T.rows_back.lines = (const SrLine*)(base + o_bl);
  T.rows_back.segs = (const SrSeg*)(base + o_bs);
  T.rows_back.tiles = (const SrRowTile*)(base + o_bt);
  for (size_t k = 0; k < T.chunks.size(); ++k) {
    SrTrainPlan::Chunk& c = T.chunks[k];
    c.edges = (const SrGradEdge*)(base + o_chunk[k][0]);
    c.biases = (const SrGradBias*)(base + o_chunk[k][1]);
    c.tiles = (const SrGradTile*)(base + o_chunk[k][2]);
    c.sums = (const SrGradSum*)(base + o_chunk[k][3]);
  }
  T.terms = A + terms_at;
  T.part = A + part_at;
  T.ring = ring;
  T.ids = ids;
  T.key = key;
  return SR_OK;
}

// The plan of a call: one that is kept, or a new one.  A window whose memory is not to be had gets by with fewer partial
// sums and the gradients of fewer frames at a time: at the least W + 2 frames of states.
sr_status plan_for(sr_graph* g, SrTrainState& S, const SrTrainPlan::Key& key, SrTrainPlan** out) {
  for (size_t k = 0; k < S.plans.size(); ++k)
    if (S.plans[k]->key == key) {
      std::rotate(S.plans.begin(), S.plans.begin() + k, S.plans.begin() + k + 1);
      *out = S.plans[0].get();
      return SR_OK;
    }
  if (S.plans.size() >= kTrainPlans) {
    SR_HIP(g, hipStreamSynchronize(g->stream));   // its tables may still be in use
    S.plans.pop_back();
  }
  for (SrTrainRoom room{key.W, SR_GRAD_ITEMS};;) {
    std::unique_ptr<SrTrainPlan> p(new SrTrainPlan());
    int kept = 1;
    const sr_status st = make_plan(g, S, *p, key, room, &kept);
    if (st == SR_OK) {
      S.plans.insert(S.plans.begin(), std::move(p));
      *out = S.plans[0].get();
      return SR_OK;
    }
    if (st != SR_ERR_OOM) return st;
    (void)hipGetLastError();   // of the allocation: the next launch would report it
    if (!room.shrink(kept)) return st;
  }
}

}  // namespace

extern "C" {

sr_status sr_window_gradients(sr_graph* g, int32_t W, const void* const* inputs, const float* const* masks,
                              const int32_t* labels, int32_t out_node, float* loss, float* const* dtheta,
                              float* const* dbias) {
  if (!g || !inputs || !labels || !loss || !dtheta || W < 1)
    return sr_gfail(g, SR_ERR_ARG, "bad argument to sr_window_gradients");
  if (g->dtype != SR_F32) return sr_gfail(g, SR_ERR_ARG, "sr_window_gradients: training windows take SR_F32 graphs only");
  if (out_node < 0 || out_node >= g->n_nodes || g->an.is_input[out_node] || g->nodes[out_node].d.height != 1 ||
      g->nodes[out_node].d.width != 1)
    return sr_gfail(g, SR_ERR_ARG, "sr_window_gradients: out_node must be a 1x1 node with incoming edges (the logits)");
  for (int e = 0; e < g->n_edges; ++e)
    if (!dtheta[e]) return sr_gfail(g, SR_ERR_ARG, "sr_window_gradients: dtheta[" + std::to_string(e) + "] is null");
  for (size_t i = 0; i < g->inputs.size(); ++i)
    if (!inputs[i]) return sr_gfail(g, SR_ERR_ARG, "input " + std::to_string(i) + " is null");
  for (int e = 0; e < g->n_edges; ++e)
    if (!g->edges[e].has_w) return sr_gfail(g, SR_ERR_STATE, "edge " + std::to_string(e) + " has no weights");
  if (W > 4096) return sr_gfail(g, SR_ERR_ARG, "sr_window_gradients: window size above 4096");
  if (!sr_rows_take_training(g))
    return sr_gfail(g, SR_ERR_ARG, "sr_window_gradients: a tensor past the limits of sr_window_gradients (sr.h)");
  SrTrainPlan* plan = nullptr;
  sr_status st = plan_for(g, train_state(g), SrTrainPlan::Key{W, out_node, g->train_tall_from, g->train_frames_kept, g->allow_split}, &plan);
  if (st != SR_OK) return st;
  SrTrainPlan& T = *plan;
  hipStream_t s = g->stream;
  const int B = g->batch, N = g->n_nodes, E = g->n_edges, C = g->nodes[out_node].d.channels;

  // the call's own tensors and destinations
  SrPatch patch{};
  auto set = [&](int index, const void* p, size_t floats_per_frame) -> sr_status {
    patch.index[patch.n] = index;
    patch.value[patch.n] = SrTensor{(char*)p, (long long)floats_per_frame * 4};
    if (++patch.n == SR_PATCH_MAX) {
      SR_HIP(g, sr_launch_patch(s, T.tensors, T.dst, patch));
      patch.n = 0;
    }
    return SR_OK;
  };
  for (size_t k = 0; k < g->inputs.size() && st == SR_OK; ++k) st = set(g->inputs[k], inputs[k], node_floats(g, g->inputs[k]));
  for (int v = 0; v < N && st == SR_OK; ++v)
    if (!g->an.is_input[v]) st = set(T.ids.mask0 + v, masks ? masks[v] : nullptr, node_floats(g, v));
  for (int e = 0; e < E && st == SR_OK; ++e) st = set(-1 - e, dtheta[e], 0);
  for (int v = 0; v < N && st == SR_OK; ++v)
    if (!g->an.is_input[v]) st = set(-1 - (E + v), dbias ? dbias[v] : nullptr, 0);
  if (st != SR_OK) return st;
  SR_HIP(g, sr_launch_patch(s, T.tensors, T.dst, patch));

  auto run = [&](const SrRowArgs& rows, const SrTrainPlan::Launch& l, int backward) -> sr_status {
    for (const auto& p : l.pools) SR_HIP(g, sr_launch_pool(s, T.tensors, p.first, B, p.second.first, p.second.second));
    SrRowArgs a = rows;
    a.runs = T.runs + l.run0;
    a.n_runs = l.n_runs;
    a.n_tiles = l.blocks;
    SR_HIP(g, sr_launch_rows_train(s, a, backward, l.shapes));
    return SR_OK;
  };
  for (const SrTrainPlan::Launch& l : T.fwd)
    if ((st = run(T.rows_fwd, l, 0)) != SR_OK) return st;
  const float scale = 1.0f / ((float)B * (float)W);
  for (size_t k = 0; k < T.chunks.size(); ++k) {
    const SrTrainPlan::Chunk& c = T.chunks[k];
    SrLossArgs l{};
    l.tensors = T.tensors;
    l.labels = labels;
    l.terms = T.terms;
    l.frame0 = c.lo;
    l.frames = c.hi - c.lo + 1;
    l.B = B;
    l.C = C;
    l.act = g->nodes[out_node].d.act;
    l.x = out_node;
    l.out = T.out_is_sink ? T.ids.grad0 + out_node : T.ids.seed;
    l.mask = T.ids.mask0 + out_node;
    l.ring = T.ring;
    l.gate = T.out_is_sink ? 1 : 0;
    l.scale = scale;
    SR_HIP(g, sr_launch_loss(s, l));
    for (const SrTrainPlan::Launch& b : c.back)
      if ((st = run(T.rows_back, b, 1)) != SR_OK) return st;
    SrGradArgs ga{};
    ga.tensors = T.tensors;
    ga.edges = c.edges;
    ga.biases = c.biases;
    ga.tiles = c.tiles;
    ga.dst = T.dst;
    ga.part = T.part;
    ga.n_tiles = (int)c.grad.tiles.size();
    ga.ring = T.ring;
    ga.accumulate = k > 0;
    SR_HIP(g, sr_launch_grad(s, ga, c.grad.shapes));
    const bool final = k + 1 == T.chunks.size();
    SR_HIP(g, sr_launch_grad_sum(s, c.sums, (int)c.grad.sums.size(), c.grad.sum_blocks, T.part, T.dst, k > 0, T.terms, (long long)W * B, scale,
                                 final ? loss : nullptr));
  }
  return SR_OK;
}

sr_status sr_rmsprop_step(sr_graph* g, float lr, float rho, float eps, const float* const* dtheta,
                          const float* const* dbias) {
  if (!g || !dtheta || !(lr >= 0.f) || !(rho >= 0.f && rho <= 1.f) || !(eps > 0.f))
    return sr_gfail(g, SR_ERR_ARG, "bad argument to sr_rmsprop_step");
  if (g->dtype != SR_F32) return sr_gfail(g, SR_ERR_ARG, "sr_rmsprop_step: SR_F32 graphs only");
  for (int e = 0; e < g->n_edges; ++e) {
    if (!dtheta[e]) return sr_gfail(g, SR_ERR_ARG, "sr_rmsprop_step: dtheta[" + std::to_string(e) + "] is null");
    if (!g->edges[e].has_w) return sr_gfail(g, SR_ERR_STATE, "edge " + std::to_string(e) + " has no weights");
  }
  SrTrainState& T = train_state(g);
  if (T.rms_w.empty()) {
    T.rms_w.assign(g->n_edges, nullptr);
    T.rms_b.assign(g->n_nodes, nullptr);
  }
  SrRmsBatch b{};
  auto flush = [&]() -> sr_status {
    SR_HIP(g, sr_launch_rmsprop(g->stream, b, lr, rho, eps));
    b.count = 0;
    return SR_OK;
  };
  auto add = [&](float* theta, float** mean, const float* grad, size_t n) -> sr_status {
    if (!*mean) {
      void* p = nullptr;
      SR_HIP(g, hipMalloc(&p, std::max<size_t>(n, 4) * sizeof(float)));
      g->dev_allocs.push_back(p);
      *mean = (float*)p;
      SR_HIP(g, sr_launch_fill_zero(g->stream, p, n * sizeof(float)));
    }
    const long long blocks = ((long long)n + 255) / 256;
    if (b.count > 0 && b.block0[b.count] + blocks > SR_F32_PIECE) {
      const sr_status st = flush();
      if (st != SR_OK) return st;
    }
    const int k = b.count++;
    b.theta[k] = theta;
    b.mean[k] = *mean;
    b.grad[k] = grad;
    b.n[k] = (long long)n;
    if (k == 0) b.block0[0] = 0;
    b.block0[k + 1] = b.block0[k] + (int)blocks;
    return b.count == SR_RMS_MAX ? flush() : SR_OK;
  };
  sr_status st = SR_OK;
  for (int e = 0; e < g->n_edges && st == SR_OK; ++e) st = add(g->edges[e].w_dev, &T.rms_w[e], dtheta[e], g->edges[e].w_count);
  for (int v = 0; dbias && v < g->n_nodes && st == SR_OK; ++v)
    if (!g->an.is_input[v] && dbias[v]) st = add(g->nodes[v].bias_dev, &T.rms_b[v], dbias[v], (size_t)g->nodes[v].d.channels);
  return st == SR_OK && b.count > 0 ? flush() : st;
}

sr_status sr_graph_get_weights(sr_graph* g, int32_t edge, float* host_w, size_t count) {
  if (!g || !host_w || edge < 0 || edge >= g->n_edges) return sr_gfail(g, SR_ERR_ARG, "bad argument to sr_graph_get_weights");
  const EdgeRt& e = g->edges[edge];
  if (count != e.w_count) return sr_gfail(g, SR_ERR_ARG, "edge " + std::to_string(edge) + ": expected " + std::to_string(e.w_count) + " weights");
  if (!e.has_w) return sr_gfail(g, SR_ERR_STATE, "edge " + std::to_string(edge) + " has no weights");
  SR_HIP(g, hipStreamSynchronize(g->stream));
  SR_HIP(g, hipMemcpy(host_w, e.w_dev, count * sizeof(float), hipMemcpyDeviceToHost));
  return SR_OK;
}

sr_status sr_graph_get_bias(sr_graph* g, int32_t node, float* host_b, size_t count) {
  if (!g || !host_b || node < 0 || node >= g->n_nodes) return sr_gfail(g, SR_ERR_ARG, "bad argument to sr_graph_get_bias");
  if (count != (size_t)g->nodes[node].d.channels) return sr_gfail(g, SR_ERR_ARG, "bias length differs from the node's channels");
  SR_HIP(g, hipStreamSynchronize(g->stream));
  SR_HIP(g, hipMemcpy(host_b, g->nodes[node].bias_dev, count * sizeof(float), hipMemcpyDeviceToHost));
  return SR_OK;
}

}  // extern "C"
