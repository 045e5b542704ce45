// Tiled fp32 contractions of whole update steps (fp32 graphs): descriptor tables, the index arithmetic shared by
// the kernels (sr_f32.hip) and their planner (sr_f32_plan.cpp), and the launchers.
//
// Two kernels.  A ROW tile computes a rectangle (pixels x channels) of one node's tensor as the sum over all
// contributing edges ("segments") of a contraction whose left operand is gathered from another tensor:
//   forward         x_v = m * sigma(b_v + sum_e f_e(x_u)):    rows = pixels of v, columns = channels of v,
//                   reduction = (tap, source channel) of every incoming edge
//   state gradient  da_u = m * sigma' * sum_e f_e^T(da_w):    rows = pixels of u (of one stride phase), columns =
//                   channels of u, reduction = (tap, target channel) of every outgoing edge
// A GRADIENT tile computes a rectangle of dtheta_e: rows = (tap, source channel), columns = target channels,
// reduction = (frame, pixel).  Work items of many nodes, edges and frames ride in one launch.
#ifndef SR_F32_H_
#define SR_F32_H_

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include <array>
#include <map>
#include <vector>

#include "sr_internal.h"

#ifdef __HIPCC__
#define SR_HD __host__ __device__ __forceinline__
#else
#define SR_HD inline
#endif

// n / d for n < 2^31 with the pair made for d (Granlund & Montgomery: l = ceil(log2 d),
// m = floor(2^32 (2^l - d) / d) + 1, q = (mulhi(m, n) + n) >> l; no overflow while n < 2^31)
struct SrDiv { uint32_t mul, sh; };
inline SrDiv sr_div_for(uint32_t d) {
  SrDiv q;
  q.sh = 0;
  while ((1ull << q.sh) < d) ++q.sh;
  q.mul = (uint32_t)((((1ull << q.sh) - d) << 32) / d + 1);
  return q;
}
SR_HD int sr_divide(int n, SrDiv d) {
  const uint32_t hi = (uint32_t)(((uint64_t)(uint32_t)n * d.mul) >> 32);
  return (int)((hi + (uint32_t)n) >> d.sh);
}

// A tensor that has a copy per frame (or per parity of the frame): copy s starts at base + s * stride bytes.
// base = null: the tensor does not exist (no dropout mask, no loss term).
struct SrTensor {
  char* base;
  long long stride;
};

#define SR_SEG_LAG 1      // reads the gathered tensor one frame away from the rows' own frame
#define SR_SEG_ZERO0 2    // forward, with SR_SEG_LAG: the tensor's frame 0 is all zero (the window's initial state)
#define SR_SEG_IMAGE 4    // the gathered row depends on the image only (mean over pixels + dense, backwards)
#define SR_SEG_QUADS 8    // channel counts are multiples of four: 16-byte gathers
struct SrSeg {
  const float* w;         // weights theta_e
  int32_t tensor, flags;
  int32_t GH, GW, GC;     // gathered image and its channels
  int32_t rs, r0h, r0w;   // first gathered row / column of a pixel: (hh / up) * rs + r0
  int32_t dir;            // gathered row of tap row vi: first + dir * vi
  int32_t ntj, R;         // taps per tap row; length of the reduction: taps * GC
  int32_t wt0, wti, wtj;  // backwards: tap of theta = wt0 + (vi / wup) * wti + (vj / wup) * wtj
  int32_t ldw;            // forward: columns of theta (= J); backwards: rows of theta per tap (= J)
  int32_t step0;          // first reduction step of this segment in the phase
  SrDiv d_gc, d_ntj, d_up;
  SrDiv d_wup;            // backwards: gathered positions per tap of an up-sampled edge
  int32_t dist;           // backwards: the gathered node's gradient is zero after frame W - dist
  int32_t lines;          // first SrLine of the segment's reduction indices; -1: no table
};
// A reduction index of a segment without SR_SEG_QUADS (a channel count that is no multiple of four): where it is from tap (0, 0), and its tap.
// Sixteen per step, in the order of the lines of a stage; past the end: a tap outside every image.  (Decoded from the index, 25
// scalar instructions a line, the five steps of a 5x5x3 edge took a 128 x 32 tile 30 us of 58.)
SR_HD int sr_in_turn(int line) { return 2 * (line & 7) + (line >> 3); }   // the index of a step that line `line` of its stage holds, if in turn
#define SR_LINES_MAX 4096   // reduction indices of an edge that gets a table
struct SrLine { int32_t off, dh, dw, pad_; };

// What a row tile's rows are: the pixels h = hh * S + ph, w = ww * S + pw of a node (S = 1: all of them).
struct SrPhase {
  int32_t node;                   // SrRowNode
  int32_t seg_begin, seg_image, seg_end;   // segments; [seg_begin, seg_image) are the SR_SEG_IMAGE ones
  int32_t steps;                  // reduction steps of all segments
  int32_t I, Hp, Wp;              // rows, and the phase's pixel grid
  int32_t S, ph, pw;
  float image_scale;              // 1 / pixels: factor of the SR_SEG_IMAGE segments
  SrDiv d_wp, d_hpwp;
};

struct SrRowNode {
  int32_t out, x, seed, mask;     // tensors: result; state (backwards: gate of the rectifier); term added to the sum; dropout
  const float* bias;              // forward
  int32_t C, H, W, act;
  int32_t gnode;                  // graph node (recording of rollout outputs)
  int32_t pad_[3];
};

// tile shapes: TI x TJ, of four waves; SR_F32_SMALL: each wave takes every fourth reduction step of a 32 x 32 tile
enum { SR_F32_128x128 = 0, SR_F32_128x64 = 1, SR_F32_64x64 = 2, SR_F32_128x32 = 3, SR_F32_SMALL = 4 };
// (With its phase in it, 128 bytes, a tile's start saved a round trip and a launch nothing that could be measured; the first window
// of a graph, which plans and copies them, took longer: MNIST SR 571 -> 606 us, DSR2 1842 -> 1858, GTSRB-shaped 7160 -> 7790.)
struct SrRowTile {
  int32_t phase;                  // < 0: empty slot
  int32_t shape, i0, j0;
  int32_t step_begin, step_end;   // part of the phase's reduction steps
  int32_t split_slot, part;       // K-split as in SrMfmaTile: slot of part 0 (-1: none), part index | parts << 16
};

// A launch over several (tile list, frame) pairs: pair k takes the workgroups from block0 on.
struct SrRun {
  int32_t block0, tile0, frame;
  int32_t slot0;          // added to the split slots of its tiles
};

#define SR_F32_KS 16              // reduction indices per step
// Variants of the tile kernels, by the shapes that a launch holds (bits 1 << shape):
//   WIDE    some 128 x 128 tiles: 64 accumulator registers a lane (weight gradients: 128), 48 KiB of LDS, three workgroups per CU
//           (not in the forward pass of a window: see sr_rows_tiles)
//   NARROW  none: at most 128 registers and 40 KiB of LDS, four workgroups per CU
//   DEEP    32 x 32 tiles only: few workgroups and a chain of loads per wave, so three steps ahead instead of two
// DSR2 window (B=64, W=8) with the weight gradients' tiles all narrow 1557 us, as planned 1575; GTSRB-shaped window without
// 128 x 128 tiles 6640, with them 6150: the wide tiles stay where they are most of the work.  MNIST SR frame 17.5 -> 17 us (DEEP).
enum { SR_F32_WIDE = 0, SR_F32_NARROW = 1, SR_F32_DEEP = 2 };
inline int sr_f32_variant(int shapes) {
  return shapes == 1 << SR_F32_SMALL ? SR_F32_DEEP : ((shapes >> SR_F32_128x128) & 1 ? SR_F32_WIDE : SR_F32_NARROW);
}
// steps of operands in LDS at a time (NARROW: two for the 32 x 32 tiles, whose four waves have LDS of their own)
#define SR_F32_PAIRS 104   // four, in pairs
SR_HD constexpr int sr_f32_stages(int variant, int shape) {
  return shape == SR_F32_64x64 || shape == SR_F32_128x32 ? 4 : shape != SR_F32_SMALL || variant == SR_F32_WIDE ? 3 : (variant == SR_F32_DEEP ? 4 : 2);
}

// k-th group of four reduction indices of row `row` of an operand that lies in LDS row by row (64 bytes a row):
// sixteen rows read together hit sixteen different 16-byte columns of the 256-byte LDS line
SR_HD int sr_f32_piece(int row, int k4) { return k4 ^ ((row >> 2) & 3); }

// Rows and taps that do not exist: whatever is added to them (images have fewer than 2^30 rows; sums wrap), the result is
// outside every image
#define SR_NO_ROW (-(1 << 30))
#define SR_NO_TAP 0x7fffffff

// A row of a row tile, seen by one segment: where tap (0, 0) lands in the gathered tensor.  A tile's 128 rows may lie in as
// many images (a phase of a strided edge has few pixels of each), so the offset takes 64 bits; lanes make it once a segment.
struct SrRowAt { int h, w; long long off; };   // off in floats; h = SR_NO_ROW: no such row
SR_HD SrRowAt sr_row_at(const SrPhase& p, const SrSeg& g, int i) {
  SrRowAt r;
  const int b = sr_divide(i, p.d_hpwp), rem = i - b * (p.Hp * p.Wp);
  const int hh = sr_divide(rem, p.d_wp), ww = rem - hh * p.Wp;
  if (g.flags & SR_SEG_IMAGE) {
    r.h = 0;
    r.w = 0;
    r.off = (long long)b * g.GC;
  } else {
    r.h = sr_divide(hh, g.d_up) * g.rs + g.r0h;
    r.w = sr_divide(ww, g.d_up) * g.rs + g.r0w;
    r.off = (((long long)b * g.GH + r.h) * g.GW + r.w) * g.GC;
  }
  if (i >= p.I) r.h = SR_NO_ROW;
  return r;
}

// Reduction index r of a segment: tap row and column, channel
struct SrTapAt { int vi, vj, c; };
SR_HD SrTapAt sr_tap_at(const SrSeg& g, int r) {
  SrTapAt t;
  const int tap = sr_divide(r, g.d_gc);
  t.c = r - tap * g.GC;
  t.vi = sr_divide(tap, g.d_ntj);
  t.vj = tap - t.vi * g.ntj;
  if (r >= g.R) t.vi = SR_NO_TAP;   // past the end
  return t;
}
SR_HD bool sr_gather_ok(const SrSeg& g, const SrRowAt& a, const SrTapAt& t) {
  return (unsigned)a.h + (unsigned)g.dir * (unsigned)t.vi < (unsigned)g.GH && (unsigned)(a.w + g.dir * t.vj) < (unsigned)g.GW;
}
SR_HD long long sr_gather_off(const SrSeg& g, const SrTapAt& t) {   // added to SrRowAt::off
  return (long long)(int)((unsigned)g.dir * ((unsigned)t.vi * (unsigned)g.GW + (unsigned)t.vj)) * g.GC + t.c;
}
// weights, backwards: theta[tap][j][c]
SR_HD uint32_t sr_weight_off(const SrSeg& g, const SrTapAt& t, int j) {
  const int tap = g.wt0 + sr_divide(t.vi, g.d_wup) * g.wti + sr_divide(t.vj, g.d_wup) * g.wtj;
  return ((uint32_t)tap * (uint32_t)g.ldw + (uint32_t)j) * (uint32_t)g.GC + (uint32_t)t.c;
}

// ---------------------------------------------------------------------------
// gradient tiles
// ---------------------------------------------------------------------------
struct SrGradEdge {
  int32_t x, dy;                  // tensors: source state, target gradient
  int32_t lag, frame0;            // the source is read at frame - lag; first frame that contributes
  int32_t H, W, Cin, Ho, Wo, Cout;   // Ho, Wo: the target's own (up-sampled) image
  int32_t kw, stride, pad;
  int32_t I, M;                   // rows = taps * Cin; pixels per frame
  int32_t quads_in, quads_out;    // channel counts that are multiples of four
  int32_t slices;                 // parts the reduction is cut into (1: straight to the destination)
  int32_t dst;                    // destination pointer
  long long part_at;              // first float of this edge's partial sums
  SrDiv d_cin, d_kw, d_wo, d_howo, d_up, d_steps;   // d_steps: steps per frame, ceil(M / SR_F32_KS)
  int32_t steps_per_frame;
  int32_t along;                  // a step's pixels can be had from those of the step before (no up-sampling, a frame within 2^31 floats)
};
// From a pixel of a gradient tile's reduction to the one 16 further on, in the coordinates of its window: the digits of 16 in
// (image, row, column), in steps of the stride, and the floats that they and the two carries stand for (modulo 2^32)
struct SrPixStep { int32_t w, h, n_w, n_h; uint32_t off, off_w, off_h; };
SR_HD SrPixStep sr_pix_step(const SrGradEdge& e, int pixels) {
  const int rows = sr_divide(pixels, e.d_wo), images = sr_divide(pixels, e.d_howo);
  const int dw = pixels - rows * e.Wo, dh = rows - images * e.Ho;
  const uint32_t line = (uint32_t)e.W * (uint32_t)e.Cin, image = (uint32_t)e.H * line;
  SrPixStep s;
  s.w = dw * e.stride;
  s.h = dh * e.stride;
  s.n_w = e.Wo * e.stride;
  s.n_h = e.Ho * e.stride;
  s.off = (uint32_t)s.w * (uint32_t)e.Cin + (uint32_t)s.h * line + (uint32_t)images * image;
  s.off_w = (uint32_t)e.stride * line - (uint32_t)s.n_w * (uint32_t)e.Cin;
  s.off_h = image - (uint32_t)s.n_h * line;
  return s;
}
// ... to the next pixel, of a step's own terms: one column on, whose carry is the same
SR_HD SrPixStep sr_pix_one(const SrGradEdge& e, const SrPixStep& s) {
  return SrPixStep{e.stride, 0, s.n_w, s.n_h, (uint32_t)e.stride * (uint32_t)e.Cin, s.off_w, s.off_h};
}
// ... the step: (w, h) is a tap of the pixel's window, lim_w and lim_h what they reach one column or row past the target's last
SR_HD void sr_pix_go(const SrPixStep& s, int stride, int lim_w, int lim_h, int* w, int* h, uint32_t* off) {
  const int w1 = *w + s.w;
  const bool cw = w1 >= lim_w;
  *w = cw ? w1 - s.n_w : w1;
  const int h1 = *h + s.h + (cw ? stride : 0);
  const bool ch = h1 >= lim_h;
  *h = ch ? h1 - s.n_h : h1;
  *off += s.off + (cw ? s.off_w : 0u) + (ch ? s.off_h : 0u);
}
// kind 0: gradient tile; 1: column sums of a gradient tensor (bias gradient), 64 channels x a range of rows; 2: empty slot
struct SrGradTile {
  int32_t edge, shape, i0, j0;
  int32_t step_begin, step_end;   // steps counted over the edge's frames (kind 1: rows counted over the frames)
  int32_t slice, kind;
};
struct SrGradBias {
  int32_t dy, C, M, frame0;       // rows per frame; first frame
  SrDiv d_m;
  long long part_at;
};
// dst[k] (+)= sum over the slices of part[s][k], in slice order; no slices: zero
struct SrGradSum {
  long long part_at, n;
  int32_t slices, dst;            // dst: index into the launch's destination pointers
  int32_t block0, pad_;           // first workgroup (64 elements each)
};

// pixel of a gradient tile's reduction: first row and column of its window in the source image
struct SrPixAt { int b, h, w; };
SR_HD SrPixAt sr_pix_at(const SrGradEdge& e, int m) {
  SrPixAt p;
  p.b = sr_divide(m, e.d_howo);
  const int rem = m - p.b * (e.Ho * e.Wo);
  const int ho = sr_divide(rem, e.d_wo), wo = rem - ho * e.Wo;
  p.h = sr_divide(ho, e.d_up) * e.stride - e.pad;
  p.w = sr_divide(wo, e.d_up) * e.stride - e.pad;
  if (m >= e.M) p.h = SR_NO_ROW;
  return p;
}
// ... does the tap at row ti, column tj of the window exist, and where is it (floats from the image of the step's first
// pixel, b0; below 2^32: sr_rows_take_training)?  aoff: of the tap and channel from the window's first element
SR_HD bool sr_pix_ok(const SrGradEdge& e, const SrPixAt& p, int ti, int tj) {
  return (unsigned)p.h + (unsigned)ti < (unsigned)e.H && (unsigned)(p.w + tj) < (unsigned)e.W;
}
SR_HD uint32_t sr_pix_off(const SrGradEdge& e, const SrPixAt& p, int b0, uint32_t aoff) {
  return (((uint32_t)(p.b - b0) * (uint32_t)e.H + (uint32_t)p.h) * (uint32_t)e.W + (uint32_t)p.w) * (uint32_t)e.Cin + aoff;
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
struct SrRowArgs {
  const SrTensor* tensors;
  const SrRowNode* nodes;
  const SrPhase* phases;
  const SrSeg* segs;
  const SrLine* lines;
  const SrRowTile* tiles;
  const SrRun* runs;              // training: (tile list, frame) pairs of the launch
  int32_t n_runs, n_tiles;        // n_tiles: workgroups
  int32_t first;                  // training: workgroup that the grid's first one is
  int32_t frame0;                 // training: frame of a run = frame0 + run.frame
  int32_t window;                 // training: W
  int32_t ring;                   // training: gradient tensors keep `ring` frames (slot = frame % ring)
  int32_t rec_node;               // frame path: node whose values also go to the rollout output (-1: none)
  SrSplitScratch split;
};
struct SrGradArgs {
  const SrTensor* tensors;
  const SrGradEdge* edges;
  const SrGradBias* biases;
  const SrGradTile* tiles;
  float* const* dst;
  float* part;
  int32_t n_tiles, ring, accumulate;
};
struct SrLossArgs {
  const SrTensor* tensors;
  const int32_t* labels;
  float* terms;                   // [W][B]
  int32_t frame0, frames;         // of the window, and of this launch
  int32_t B, C, act;
  int32_t x, out, mask;           // tensors: scores, where their gradient goes, dropout (out of the node itself)
  int32_t first;                  // (frame, sample) pair of the first wave
  int32_t ring, gate;             // gate: `out` is the node's own gradient (apply rectifier and dropout)
  float scale;
};
#define SR_PATCH_MAX 96
struct SrPatch {                  // entries of the tensor / destination tables that a call brings along
  int32_t index[SR_PATCH_MAX];    // >= 0: tensor; < 0: destination -1 - index
  SrTensor value[SR_PATCH_MAX];
  int32_t n;
};
struct SrPool {                   // channel means of a node's state
  int32_t x, mean, lag, HW, C, zero0;
};
#define SR_RMS_MAX 64
struct SrRmsBatch {
  float *theta[SR_RMS_MAX], *mean[SR_RMS_MAX];
  const float* grad[SR_RMS_MAX];
  long long n[SR_RMS_MAX];
  int32_t block0[SR_RMS_MAX + 1];
  int32_t count;
};

// frame path: the level's tiles and the auxiliary items in one launch
hipError_t sr_launch_rows_frame(hipStream_t s, const SrFrame& f, const SrRowArgs& a, int shapes, const SrAux* aux, int n_aux,
                                const SrHead* heads, const SrHeadEdge* head_edges, const SrStageNode* stage_nodes,
                                int aux_smem_bytes);
// training window
hipError_t sr_launch_rows_train(hipStream_t s, const SrRowArgs& a, int backward, int shapes);
hipError_t sr_launch_grad(hipStream_t s, const SrGradArgs& a, int shapes);
// destination sums, and (loss != null) loss = scale * sum of the n_terms loss terms
// (launches of more workgroups than a grid may have -- 2^32 threads, here 2^23 workgroups -- go in pieces)
#define SR_F32_PIECE (1 << 23)
hipError_t sr_launch_grad_sum(hipStream_t s, const SrGradSum* sums, int n_sums, int n_blocks, const float* part, float* const* dst,
                              int accumulate, const float* terms, long long n_terms, float scale, float* loss);
hipError_t sr_launch_loss(hipStream_t s, const SrLossArgs& a);
hipError_t sr_launch_patch(hipStream_t s, SrTensor* tensors, float** dst, const SrPatch& p);
hipError_t sr_launch_pool(hipStream_t s, const SrTensor* tensors, const SrPool& p, int B, int frame0, int frames);
hipError_t sr_launch_rmsprop(hipStream_t s, const SrRmsBatch& b, float lr, float rho, float eps);

// ---------------------------------------------------------------------------
// planner (sr_f32_plan.cpp)
// ---------------------------------------------------------------------------
inline void sr_f32_shape(int shape, int* ti, int* tj) {
  static const int t[5][2] = {{128, 128}, {128, 64}, {64, 64}, {128, 32}, {32, 32}};
  *ti = t[shape][0];
  *tj = t[shape][1];
}
inline int sr_f32_lds_bytes(int shapes) {   // of a workgroup of a launch with these shapes
  int most = 0;
  for (int shape = 0; shape < 5; ++shape) {
    if (!((shapes >> shape) & 1)) continue;
    int ti, tj;
    sr_f32_shape(shape, &ti, &tj);
    const int bytes = sr_f32_stages(sr_f32_variant(shapes), shape) * (ti + tj) * SR_F32_KS * 4 * (shape == SR_F32_SMALL ? 4 : 1);
    if (bytes > most) most = bytes;
  }
  return most;
}
struct sr_graph;
struct SrRowPlan {
  std::vector<SrSeg> segs;
  std::vector<SrLine> lines;
  std::map<std::array<int, 6>, int> line_tables;   // gathered channels, columns, taps per row, indices, direction, in turn -> its first line
  std::vector<SrPhase> phases;
  std::vector<SrRowNode> nodes;
};
// Tensor numbers of a training window: node v's state is v, its gradient grad0 + v, its dropout multipliers mask0 + v;
// mean[e]: channel means that the GAP edge e reads; seed: loss term of the out node (-1: stored as its gradient)
struct SrTrainIds {
  int grad0, mask0, seed, out_node;
  std::vector<int> mean;
  std::vector<int> dist;   // per node: fewest bridging edges on a path to the out node (-1: no path, the loss does not see it)
};
// can node v be computed by row tiles (no incoming GAP edge, offsets in 32 bits)?
bool sr_rows_take_forward(const sr_graph* g, int v);
// are all tensors of the graph within the index arithmetic of a training window's kernels?
bool sr_rows_take_training(const sr_graph* g);
// Append node v's descriptors; returns its first phase (a forward node has one).  ids = null: frame path, tensors
// numbered like the nodes.
int sr_rows_forward(SrRowPlan* p, const sr_graph* g, int v, const SrTrainIds* ids);
int sr_rows_backward(SrRowPlan* p, const sr_graph* g, int v, const SrTrainIds& ids);
// Tiles of phases that one launch covers, in the order of the list (workgroup i runs on XCD i % 8; padded to a
// multiple of 8 with empty tiles).  work_cycles: compute-unit cycles of the whole launch if it covers more than
// these phases (0: just these).  tall_from: SR_OPT_TRAIN_TALL_TILES_FROM; split: SR_OPT_K_SPLIT; ordered: forward pass of a
// training window.
void sr_rows_tiles(const SrRowPlan& p, const std::vector<int>& phases, double work_cycles, int tall_from, bool split, bool ordered,
                   int* split_slots, std::vector<SrRowTile>* out, int* shapes);
double sr_rows_work(const SrRowPlan& p, int phase);   // compute-unit cycles of a phase at the fp32 matrix rate
// Weight and bias gradients of the frames lo..hi of a window of W frames: descriptors, tiles, partial sums.  Destination
// pointers: edge e is e, node v's bias n_edges + v.  first: the first chunk of the window that is worked on (it
// overwrites the destinations, later ones add).
struct SrGradPlan {
  std::vector<SrGradEdge> edges;
  std::vector<SrGradBias> biases;
  std::vector<SrGradTile> tiles;
  std::vector<SrGradSum> sums;
  int sum_blocks = 0, shapes = 0;
  long long part_floats = 0;
};
// items: work items per compute unit that the pixel sums are cut for
void sr_grad_plan(SrGradPlan* p, const sr_graph* g, const SrTrainIds& ids, int W, int lo, int hi, bool first, int tall_from, int items);
// What a window's plan may take: state gradients of so many frames at a time, and partial sums for so many work items per compute unit.
#define SR_GRAD_ITEMS 12
struct SrTrainRoom {
  int frames, items;
  // less than a plan that kept `kept` frames and whose memory was not to be had; false: there is nothing to take back
  bool shrink(int kept) {
    if (items == SR_GRAD_ITEMS) items /= 2;   // (cheapest: half the partial sums for 1.5 % of a GTSRB-shaped window)
    else if (kept > 1) frames = kept / 2;
    else if (items > 1) items = 1;
    else return false;
    return true;
  }
};

#endif  // SR_F32_H_
