// Tiled contractions of fp32 graphs on the fp32 matrix cores (v_mfma_f32_32x32x2_f32): whole update steps of the
// frame path, and the forward pass, state gradients and weight gradients of a training window (see sr_f32.h).
//
// A workgroup of four waves owns a TI x TJ tile and walks its reduction in steps of 16 indices.  The operands of a
// step are brought into LDS by direct-to-LDS loads whose lane addresses do the gathering (taps, strides, padding;
// elements that do not exist are read from a line of zeros), ahead of the step being multiplied: no registers between
// global memory and LDS.  fp32 matrix instructions are slow (a 32x32x2 product takes 64 cycles of its SIMD); a step's
// operand traffic is 8 bytes per cycle of its products and CU for 128 x 128 tiles, 12 for 128 x 64, 16 for 64 x 64, 20 for
// 128 x 32 and 32 for 32 x 32.  What bounds a tile is the fp32 matrix rate, 157 TFLOP/s, for 128 x 128 tiles, whose waves have
// 32 products a step (GTSRB-shaped windows: matrix cores 86 % busy in the reverse sweep, 76 % in the weight gradients, 81 %
// in the forward pass with its 128 x 64 tiles; 77, 74 and 71 % before the loop below).  64 x 64 and 128 x 32 tiles have 8: there a step's fixed
// costs take as long as its products.  So these fetch steps in pairs, a barrier per pair; launches without 128 x 128 tiles run
// four workgroups per CU (see the variants in sr_f32.h); and the steps of whole segments go through a loop that holds nothing
// but their loads and products (run_along below: 155 instructions a pair, 16 of them products, where the code that takes any
// step of any segment has 400).  DSR2 frame: matrix cores 54 % busy before, 58 % since at 0.8 of the time.  Pairs are of consecutive
// steps, whatever their segments (but for ordered sums, whose pairs end with a segment): behind a segment of an odd number of steps
// the next one's pairs lie across the loop's, and none of them goes through it.  DSR2's largest node is such a one (5 steps of a
// 5x5x3 edge, then 18 of its self edge: a quarter of a frame's operations), so what the loop is worth to a frame is not known from
// a frame of DSR2; beside it a 128 x 32 tile of 18 steps spends 12 us of 28 in its tables, first operands and stores, while its
// compute unit's other three do the same.
//
// Measured, DSR2 as an fp32 graph (batch 64, 6.4 GFLOP per frame): 1350 us per frame with a thread per output (weights
// and taps through global loads, no matrix cores), 104 with row tiles (62 TFLOP/s), 100 with pairs, 82 with segments' steps back
// to back; MNIST SR, batch 128: 31 -> 17 -> 13 us.  Training windows, pairs and variants -> now, on one card: DSR2 B=64 W=8
// 1479 -> 1380 us, GTSRB-shaped B=128 W=4 6174 -> 5492, MNIST SR B=128 W=8 362 -> 330.
//
// In the loop a wave's priority is raised but for its products: loads, addresses and set-up of one wave then go ahead of the
// others' products, which the matrix cores take 64 cycles each for (GTSRB-shaped window 5690 -> 5620 us, DSR2 1437 -> 1423).
//
// Every sum has a fixed order (reduction index by index within a part, parts in order, waves in order): the same call
// gives the same bits.  The forward pass of a training window has one order for all sizes and tiles (SR_ROWS_ORDERED);
// against tiles that take theirs as it comes, and cut long sums, that costs DSR2 1459 -> 1480 us, GTSRB-shaped 5990 -> 6180,
// MNIST SR 302 -> 358.
#include <algorithm>

#include "sr_device.h"
#include "sr_f32.h"

namespace {

typedef int sr_i32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
#define SR_CONST4(T) const __attribute__((address_space(4))) T*
template <typename T>
__device__ __forceinline__ SR_CONST4(T) sr_k(const T* p) { return (SR_CONST4(T))(unsigned long long)p; }
#define SR_UNI(x) __builtin_amdgcn_readfirstlane(x)
__device__ __forceinline__ const char* sr_uni_ptr(const char* p) {
  const unsigned long long v = (unsigned long long)p;
  return (const char*)(((unsigned long long)(unsigned)SR_UNI((int)(v >> 32)) << 32) | (unsigned)SR_UNI((int)v));
}

__device__ __align__(128) const float sr_zero_line[32] = {};   // a lane reads 16 bytes of it, or 64 bytes further on (second step of a pair)

// One direct-to-LDS load: lane l's 16 (4) bytes go to lds + 16 l (4 l).
__device__ __forceinline__ void sr_to_lds16(const char* g, unsigned lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)(unsigned long long)lds, 16, 0, 0);
}
__device__ __forceinline__ void sr_to_lds4(const char* g, unsigned lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)(unsigned long long)lds, 4, 0, 0);
}
// this wave's loads but the newest N have landed, and its LDS reads are done
template <int N>
__device__ __forceinline__ void sr_wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory");
}
// a barrier that LDS accesses are not moved across (the waits stand before it)
__device__ __forceinline__ void sr_step_barrier() {
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ unsigned sr_lds_at(const void* p) {
  return (unsigned)(unsigned long long)(const __attribute__((address_space(3))) char*)p;
}

// the same address, but values read from it are not kept from earlier reads
template <typename T>
__device__ __forceinline__ SR_CONST4(T) sr_again(SR_CONST4(T) p) {
  asm volatile("" : "+s"(p));
  return p;
}

__device__ __forceinline__ SrDiv sr_load_div(SR_CONST4(SrDiv) d) { return SrDiv{d->mul, d->sh}; }
__device__ __forceinline__ SrSeg sr_load_seg(SR_CONST4(SrSeg) s) {
  SrSeg g;
  g.w = s->w;
  g.tensor = s->tensor; g.flags = s->flags;
  g.GH = s->GH; g.GW = s->GW; g.GC = s->GC;
  g.rs = s->rs; g.r0h = s->r0h; g.r0w = s->r0w;
  g.dir = s->dir; g.ntj = s->ntj; g.R = s->R;
  g.wt0 = s->wt0; g.wti = s->wti; g.wtj = s->wtj;
  g.ldw = s->ldw; g.step0 = s->step0;
  g.d_gc = sr_load_div(&s->d_gc); g.d_ntj = sr_load_div(&s->d_ntj); g.d_up = sr_load_div(&s->d_up);
  g.d_wup = sr_load_div(&s->d_wup); g.dist = s->dist; g.lines = s->lines;
  return g;
}
__device__ __forceinline__ SrPhase sr_load_phase(SR_CONST4(SrPhase) s) {
  SrPhase p;
  p.node = s->node; p.seg_begin = s->seg_begin; p.seg_image = s->seg_image; p.seg_end = s->seg_end; p.steps = s->steps;
  p.I = s->I; p.Hp = s->Hp; p.Wp = s->Wp; p.S = s->S; p.ph = s->ph; p.pw = s->pw;
  p.image_scale = s->image_scale;
  p.d_wp = sr_load_div(&s->d_wp); p.d_hpwp = sr_load_div(&s->d_hpwp);
  return p;
}

// float `off` of the tensor at p
__device__ __forceinline__ const char* sr_at(const char* p, uint32_t off) { return p + ((unsigned long long)off << 2); }

// which copies of its tensors a tile works on
struct SrSlots {
  int lag0, lag1;      // gathered tensors, without and with SR_SEG_LAG
  int own;             // result
  int frame;           // state, mask, loss term
  int left;            // training, backwards: frames from here to the window's last (W - frame); forward: frame; else large
};
// Does a segment contribute?  Forward: not if it reads the window's initial state, which is zero.  Backwards: not if
// it reads a gradient that no loss term of the window depends on.
template <bool BACK>
__device__ __forceinline__ bool sr_seg_counts(const SrSeg& g, const SrSlots& sl) {
  const int lag = (g.flags & SR_SEG_LAG) ? 1 : 0;
  return BACK ? sl.left >= lag + g.dist : !(lag && (g.flags & SR_SEG_ZERO0) && sl.left == 1);
}

// What a row tile is computed for.  SR_ROWS_ORDERED: the forward pass of a training window, whose sums are taken in one
// order whatever the sizes, so that the sign of a rectifier's input, and with it the path a gradient takes, does not hang
// on which tile shape a launch has.  Every edge's sum starts from zero and runs through its reduction indices step by step,
// the edges' sums are added in edge order; inside a step the products go 0, 8, 1, 9, .. where all channel counts are
// multiples of four (SR_SEG_QUADS), else 0, 1, 2, .. (line 8 h + k of its stage then holds index 2 k + h).
enum { SR_ROWS_FRAME = 0, SR_ROWS_BACK = 1, SR_ROWS_ORDERED = 2 };

// The operands of a tile of four waves: a TI x 16 and a 16 x TJ piece per step, the waves fetching them together.
//   rows:  TI (TJ) rows of 16 reduction indices, 64 bytes a row, pieces of four permuted (sr_f32_piece)
//   k-major: 16 lines of TI (TJ) elements
// A is rows when the gathered channel count is a multiple of four (16-byte loads), else k-major (4-byte loads); B is
// k-major in the forward direction, where theta's columns are contiguous, and like A backwards.
template <int TI, int TJ, int FOR>
struct SrRowOperands {
  static constexpr bool BACK = FOR == SR_ROWS_BACK;
  static constexpr int NW = 4;
  static constexpr int NA = TI / (16 * NW);                        // 16-byte loads of A per wave and step
  static constexpr int NB = TJ / (16 * NW) > 0 ? TJ / (16 * NW) : 1;   // ... of B (TJ = 32 of four waves: half the lanes)
  static constexpr int STAGE = (TI + TJ) * 64;                     // bytes of one step in LDS
  static constexpr int LOADS = NA + NB;                            // fewest loads a wave issues per step
  static constexpr bool HALF_B = TJ / (16 * NW) == 0;

  // Of the segment: what every step needs.  The rest is read again where it is needed (sr_again): with all of it in registers
  // the kernels of many shapes kept 150 scalar registers in lanes of vector registers, read back step by step.
  SR_CONST4(SrSeg) seg;
  int GH, GW, GC, dir, ntj, R, ldw;
  int wt0, wti, wtj;         // backwards
  SrDiv d_wup;
  int row_h[NA], row_w[NA];  // this lane's rows: where tap (0, 0) lands ...
  const char* row_at[NA];    // ... and its address
  int wv, lane, i0, j0;
  int quads, quads_w;
  int turn;                  // ordered: the products of a step go in turn
  // A step whose indices lie in one tap (channel counts that are multiples of 16) has addresses that go on from those of the
  // step before: a lane's gathered address by the channels passed, theta by a scalar base under lane offsets that stay for
  // the segment; only a new tap looks at the image's edges again.
  const SrLine* lines;       // null: no table
  int along;                 // A goes that way
  int at_r, vi, vj, c;       // step that the addresses are for; its tap and first channel
  const char* cur[NA];
  unsigned go[NA];           // 4, or 0 where the line of zeros is read: bytes per channel passed
  const char* wbase;         // theta at column j0, first index (backwards: tap 0, channel 0)
  const char* wcur;          // backwards: theta at column j0 of the tap and channel
  uint32_t woff[BACK ? NB : 1];
  uint32_t wpair;            // a pair's theta by full waves where a step's takes half of each (HALF_B)
  int wide_w;                // ... whose lane offsets fit 32 bits

  // a new segment, whose first step will be the one at r0: where this lane's rows are in its image
  __device__ __forceinline__ void enter(const SrSeg& g, SR_CONST4(SrSeg) at_seg, SR_CONST4(SrPhase) phase, const SrTensor* tensors,
                                        const SrLine* line_table, const SrSlots& sl, int r0) {
    const SrPhase p = sr_load_phase(sr_again(phase));
    seg = at_seg;
    GH = g.GH; GW = g.GW; GC = g.GC; dir = g.dir; ntj = g.ntj; R = g.R; ldw = g.ldw;
    if (BACK) { wt0 = g.wt0; wti = g.wti; wtj = g.wtj; d_wup = g.d_wup; }
    SR_CONST4(SrTensor) t = sr_k(tensors) + g.tensor;
    const int slot = sl.lag0 + ((g.flags & SR_SEG_LAG) ? sl.lag1 - sl.lag0 : 0);   // (a select between the fields would go through memory)
    const char* src = sr_uni_ptr((const char*)(unsigned long long)t->base + slot * t->stride);
    quads = SR_UNI((g.flags & SR_SEG_QUADS) && ((unsigned)(unsigned long long)src & 15u) == 0);
    quads_w = SR_UNI((g.ldw & 3) == 0);
    lines = g.lines >= 0 ? line_table + g.lines : nullptr;
    if (FOR == SR_ROWS_ORDERED) turn = !(g.flags & SR_SEG_QUADS);
#pragma unroll
    for (int n = 0; n < NA; ++n) {
      const int r = quads ? n * 16 * NW + wv * 16 + (lane >> 2)
                          : (TI == 128 ? (wv & 1) * 64 + lane : lane);
      const SrRowAt at = sr_row_at(p, g, i0 + r);
      row_h[n] = at.h;
      row_w[n] = at.w;
      row_at[n] = src + at.off * 4;
    }
    along = quads && (g.GC & 15) == 0;
    if (along) {
      const SrTapAt t0 = sr_tap_at(g, SR_UNI(r0));
      at_r = r0;
      vi = t0.vi;
      vj = t0.vj;
      c = t0.c;
      const int k4 = sr_f32_piece(lane >> 2, lane & 3);
#pragma unroll
      for (int n = 0; n < NA; ++n) row_at[n] += 16 * k4;
    }
    if (BACK) {
      wide_w = g.GC < (1 << 22);
      wbase = (const char*)g.w + (unsigned long long)(unsigned)j0 * (unsigned)g.GC * 4;
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int row = HALF_B ? wv * 8 + (lane >> 2) : n * 16 * NW + wv * 16 + (lane >> 2);
        // (a half-filled wave's rows start at a multiple of eight: its pieces are permuted differently from A's; columns that
        // the node does not have read its last one)
        woff[n] = ((uint32_t)min(row, g.ldw - 1 - j0) * (uint32_t)g.GC + 4u * (uint32_t)sr_f32_piece(row, lane & 3)) * 4u;
      }
    } else {
      wide_w = g.ldw < (1 << 22);
      wbase = (const char*)g.w + (unsigned long long)(unsigned)j0 * 4;
      const int id = HALF_B ? wv * 32 + lane : wv * 64 + lane;
      if (quads_w) woff[0] = ((uint32_t)(id / (TJ / 4)) * (uint32_t)g.ldw + (uint32_t)min(4 * (id % (TJ / 4)), g.ldw - 4 - j0)) * 4u;
      else woff[0] = ((uint32_t)((wv * 64 + lane) / TJ) * (uint32_t)g.ldw + (uint32_t)min((wv * 64 + lane) % TJ, g.ldw - 1 - j0)) * 4u;
    }
    if (HALF_B) {
      const int row = (wv & 1) * 16 + (lane >> 2), id = wv * 64 + lane;
      if (BACK) wpair = ((uint32_t)min(row, ldw - 1 - j0) * (uint32_t)GC + 4u * (uint32_t)sr_f32_piece(row, lane & 3) + 16u * (uint32_t)(wv >> 1)) * 4u;
      else wpair = ((uint32_t)(id / (TJ / 4)) * (uint32_t)ldw + (uint32_t)min(4 * (id % (TJ / 4)), max(ldw - 4 - j0, 0))) * 4u;
    }
    if (along) look();
  }
  // the fields above as a descriptor
  __device__ __forceinline__ SrSeg hot() const {
    SrSeg g{};
    g.GH = GH; g.GW = GW; g.GC = GC; g.dir = dir; g.ntj = ntj; g.R = R; g.ldw = ldw;
    if (BACK) { g.wt0 = wt0; g.wti = wti; g.wtj = wtj; g.d_wup = d_wup; }
    return g;
  }

  // the gathered addresses at tap (vi, vj), channel c
  __device__ __forceinline__ void look() {
    const SrSeg g = hot();
    const SrTapAt t{vi, vj, c};
    const long long toff = sr_gather_off(g, t) * 4;
#pragma unroll
    for (int n = 0; n < NA; ++n) {
      const bool ok = sr_gather_ok(g, SrRowAt{row_h[n], row_w[n], 0}, t);
      cur[n] = ok ? row_at[n] + toff : (const char*)sr_zero_line;
      go[n] = ok ? 4u : 0u;
    }
    if (BACK) wcur = wbase + (unsigned long long)sr_weight_off(g, t, 0) * 4;
  }
  // ... D channels further on
  template <int D>
  __device__ __forceinline__ void advance() {
    at_r += D;
    c += D;
    if (c < GC) {
#pragma unroll
      for (int n = 0; n < NA; ++n) cur[n] += D * go[n];
      if (BACK) wcur += 4 * D;
      return;
    }
    do {
      c -= GC;
      if (++vj == ntj) { vj = 0; ++vi; }
    } while (c >= GC);
    look();
  }
  // ... of the step at r0
  __device__ __forceinline__ void go_on(int r0) {
    while (at_r < r0) advance<SR_F32_KS>();
  }

  // Do this segment's steps (PAIR: at r0 even pairs of steps) take the loads of issue_along?
  template <bool PAIR>
  __device__ __forceinline__ bool all_along(int r0) const {
    return along && wide_w && (!PAIR || ((GC & 31) == 0 && (r0 & 31) == 0 && (BACK || quads_w)));
  }
  // loads of a step all of whose indices exist (PAIR: two of them, in one tap), its gathered addresses at hand; forward: w is theta
  // at its first index
  template <bool PAIR>
  __device__ __forceinline__ void issue_along(unsigned at, const char* w) const {
    const unsigned bt = at + TI * 64;
#pragma unroll
    for (int n = 0; n < NA; ++n) {
      sr_to_lds16(cur[n], at + (n * NW + wv) * 1024);
      if (PAIR) sr_to_lds16(cur[n] + 64, at + STAGE + (n * NW + wv) * 1024);
    }
    w = sr_uni_ptr(BACK ? wcur : w);
    const unsigned line = (unsigned)ldw * 4u;
    if (PAIR && HALF_B) {
      uint32_t o = wpair;
      asm volatile("" : "+v"(o));   // keeps the offset 32-bit: scalar base + lane offset addressing
      sr_to_lds16(w + o, bt + (wv >> 1) * STAGE + (wv & 1) * 1024);
    } else if (BACK || quads_w) {
#pragma unroll
      for (int n = 0; n < NB; ++n) {   // forward: 256 NW / TJ lines further on each time
        uint32_t o = woff[BACK ? n : 0];
        asm volatile("" : "+v"(o));
        const char* wn = BACK ? w : w + (unsigned long long)(n * (256 * NW / TJ)) * line;
        if (HALF_B) {
          if (lane < 32) sr_to_lds16(wn + o, bt + wv * 512);
        } else {
          sr_to_lds16(wn + o, bt + (n * NW + wv) * 1024);
          if (PAIR) sr_to_lds16((BACK ? wn + 64 : wn + (unsigned long long)SR_F32_KS * line) + o, bt + STAGE + (n * NW + wv) * 1024);
        }
      }
    } else {
      uint32_t o = woff[0];
      asm volatile("" : "+v"(o));
#pragma unroll
      for (int q = 0; q < TJ / 4 / NW; ++q)
        sr_to_lds4(w + (unsigned long long)(q * (64 * NW) / TJ) * line + o, bt + (q * NW + wv) * 256);
    }
  }
  __device__ __forceinline__ const char* theta(int r0) const { return wbase + (unsigned long long)(unsigned)r0 * ((unsigned)ldw * 4u); }

  // this lane's row at an SrLine
  __device__ __forceinline__ const char* lined(int off, int dh, int dw) const {
    const bool ok = (unsigned)row_h[0] + (unsigned)dh < (unsigned)GH && (unsigned)row_w[0] + (unsigned)dw < (unsigned)GW;
    return ok ? row_at[0] + (long long)off * 4 : (const char*)sr_zero_line;
  }
  __device__ __forceinline__ const char* gathered(const SrSeg& g, int n, const SrTapAt& t, long long tap_bytes) const {
    return sr_gather_ok(g, SrRowAt{row_h[n], row_w[n], 0}, t) ? row_at[n] + tap_bytes : (const char*)sr_zero_line;
  }

  // loads of the 16 reduction indices from r0 on, into LDS at `at`
  __device__ __forceinline__ void issue(int r0, unsigned at) {
    const char* zero = (const char*)sr_zero_line;
    const unsigned bt = at + TI * 64;
    const bool all = r0 + SR_F32_KS <= R;   // all sixteen indices exist
    if (all && all_along<false>(r0)) {
      go_on(r0);
      issue_along<false>(at, theta(r0));
      return;
    }
    if (along && all) {
      go_on(r0);
#pragma unroll
      for (int n = 0; n < NA; ++n) sr_to_lds16(cur[n], at + (n * NW + wv) * 1024);
    } else if (quads) {   // (past the end: of the rows' addresses, which may include k4, none is read)
      const SrSeg g = sr_load_seg(sr_again(seg));
      const SrTapAt t = sr_tap_at(g, r0 + 4 * sr_f32_piece(lane >> 2, lane & 3));
      const long long toff = sr_gather_off(g, t) * 4;
#pragma unroll
      for (int n = 0; n < NA; ++n) sr_to_lds16(gathered(g, n, t, toff), at + (n * NW + wv) * 1024);
    } else if (lines != nullptr) {
      SR_CONST4(sr_i32x16) step = (SR_CONST4(sr_i32x16))(unsigned long long)(lines + r0);
      const int l0 = TI == 128 ? 8 * (wv >> 1) : 4 * wv;   // this wave's lines, 64 of a line's rows
#pragma nounroll
      for (int k = 0; k < TI / 64; ++k) {   // (four lines in scalar registers at a time)
        const sr_i32x16 x = step[l0 / 4 + k];
#pragma unroll
        for (int q = 0; q < 4; ++q) sr_to_lds4(lined(x[4 * q], x[4 * q + 1], x[4 * q + 2]), at + (l0 + 4 * k + q) * (TI * 4) + (TI == 128 ? (wv & 1) * 256 : 0));
      }
    } else {
      const SrSeg g = sr_load_seg(sr_again(seg));
#pragma unroll
      for (int q = 0; q < TI / 4 / NW; ++q) {
        const int id = q * NW + wv;
        const int line = id * 64 / TI;
        const int k = FOR == SR_ROWS_ORDERED && turn ? sr_in_turn(line) : line;
        const SrTapAt t = sr_tap_at(g, SR_UNI(r0 + k));
        const char* p = gathered(g, 0, t, sr_gather_off(g, t) * 4);
        sr_to_lds4(p, at + id * 256);
      }
    }
    if (BACK) {
      if (quads) {
        // (a half-filled wave's rows start at a multiple of eight: its pieces are permuted differently from A's)
        const SrSeg g = sr_load_seg(sr_again(seg));
        const SrTapAt t = sr_tap_at(g, r0 + 4 * sr_f32_piece((HALF_B ? wv * 8 : 0) + (lane >> 2), lane & 3));
        const bool r_ok = t.vi != SR_NO_TAP;
        const uint32_t off = sr_weight_off(g, t, 0);
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const int j = j0 + (HALF_B ? wv * 8 + (lane >> 2) : n * 16 * NW + wv * 16 + (lane >> 2));
          const char* p = (r_ok && j < g.ldw) ? sr_at((const char*)g.w, off + (uint32_t)j * (uint32_t)g.GC) : zero;
          if (HALF_B) {
            if (lane < 32) sr_to_lds16(p, bt + wv * 512);
          } else {
            sr_to_lds16(p, bt + (n * NW + wv) * 1024);
          }
        }
      } else {
        const SrSeg g = sr_load_seg(sr_again(seg));
#pragma unroll
        for (int q = 0; q < TJ / 4 / NW; ++q) {
          const int id = q * NW + wv;
          const int k = TJ >= 64 ? id * 64 / TJ : 2 * id + (lane >> 5);
          const int j = j0 + (TJ >= 64 ? (TJ == 128 ? (id & 1) * 64 + lane : lane) : (lane & 31));
          const SrTapAt t = sr_tap_at(g, TJ >= 64 ? SR_UNI(r0 + k) : r0 + k);
          const char* p = (t.vi != SR_NO_TAP && j < g.ldw) ? sr_at((const char*)g.w, sr_weight_off(g, t, j)) : zero;
          sr_to_lds4(p, bt + id * 256);
        }
      }
      return;
    }
    // forward: 16 lines of theta
    if (all && wide_w && !(FOR == SR_ROWS_ORDERED && turn)) {
      const unsigned line = (unsigned)ldw * 4u;
      const char* w = sr_uni_ptr(theta(r0));
      uint32_t o = woff[0];
      asm volatile("" : "+v"(o));
      if (quads_w) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const char* wn = w + (unsigned long long)(n * (256 * NW / TJ)) * line;
          if (HALF_B) {
            if (lane < 32) sr_to_lds16(wn + o, bt + wv * 512);
          } else {
            sr_to_lds16(wn + o, bt + (n * NW + wv) * 1024);
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < TJ / 4 / NW; ++q)
          sr_to_lds4(w + (unsigned long long)(q * (64 * NW) / TJ) * line + o, bt + (q * NW + wv) * 256);
      }
      return;
    }
    const SrSeg g = sr_load_seg(sr_again(seg));
    if (FOR == SR_ROWS_ORDERED && turn) {
      if (quads_w) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const int id = HALF_B ? wv * 32 + lane : (n * NW + wv) * 64 + lane;
          const int r = r0 + sr_in_turn((id / (TJ / 4)) & 15), j = j0 + 4 * (id % (TJ / 4));
          const char* p = (r < g.R && j < g.ldw) ? sr_at((const char*)g.w, (uint32_t)r * (uint32_t)g.ldw + (uint32_t)j) : zero;
          if (HALF_B) {
            if (lane < 32) sr_to_lds16(p, bt + wv * 512);
          } else {
            sr_to_lds16(p, bt + (n * NW + wv) * 1024);
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < TJ / 4 / NW; ++q) {
          const int id = q * NW + wv;
          const int r = r0 + sr_in_turn((id * 64 + lane) / TJ), j = j0 + (id * 64 + lane) % TJ;
          const char* p = (r < g.R && j < g.ldw) ? sr_at((const char*)g.w, (uint32_t)r * (uint32_t)g.ldw + (uint32_t)j) : zero;
          sr_to_lds4(p, bt + id * 256);
        }
      }
    } else if (quads_w) {
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int id = HALF_B ? wv * 32 + lane : (n * NW + wv) * 64 + lane;
        const int r = r0 + id / (TJ / 4), j = j0 + 4 * (id % (TJ / 4));
        const char* p = (r < g.R && j < g.ldw) ? sr_at((const char*)g.w, (uint32_t)r * (uint32_t)g.ldw + (uint32_t)j) : zero;
        if (HALF_B) {
          if (lane < 32) sr_to_lds16(p, bt + wv * 512);
        } else {
          sr_to_lds16(p, bt + (n * NW + wv) * 1024);
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < TJ / 4 / NW; ++q) {
        const int id = q * NW + wv;
        const int r = r0 + (id * 64 + lane) / TJ, j = j0 + (id * 64 + lane) % TJ;
        const char* p = (r < g.R && j < g.ldw) ? sr_at((const char*)g.w, (uint32_t)r * (uint32_t)g.ldw + (uint32_t)j) : zero;
        sr_to_lds4(p, bt + id * 256);
      }
    }
  }
};

// The operands of a 32 x 32 tile, laid out as above and fetched by one wave.  A launch of such tiles is one generation of them, a
// wave takes one to ten steps of a segment, and the instructions in a row from a tile's start to its end are what it takes: a
// scalar one 5 to 8 cycles.  So a segment's descriptor stays in registers, a step is decoded from its number, and addresses that
// go on from step to step (as above) are set up where the loop that uses them starts.  (Set up with every segment, 270 more
// scalar instructions a tile: windows MNIST SR 343 -> 327 us, DSR1 B=3 273 -> 255, DSR5 B=1 486 -> 454; 16 frames of the
// CIFAR-shaped graph B=7 514 -> 494, of 33x33 images in 16 channels 224 -> 214.  Segments and steps as two loops, or filling,
// running and draining the stages as one, made the kernels a third smaller and 3 to 10 % slower: copies of accumulators and
// descriptors between the parts.)
template <int FOR>
struct SrSmallOperands {
  static constexpr bool BACK = FOR == SR_ROWS_BACK;
  static constexpr int N = 2;                // 16-byte loads of A, and of B, per step
  static constexpr int STAGE = 64 * 64, LOADS = 2 * N;

  SrSeg g;
  int row_h[N], row_w[N];    // this lane's rows: where tap (0, 0) lands ...
  const char* row_at[N];     // ... and its address
  int lane, i0, j0;
  int quads, quads_w;
  int turn;                  // ordered: the products of a step go in turn

  // a new segment: where this lane's rows are in its image
  __device__ __forceinline__ void enter(const SrPhase& p, const SrTensor* tensors, const SrSlots& sl) {
    SR_CONST4(SrTensor) t = sr_k(tensors) + g.tensor;
    const int slot = sl.lag0 + ((g.flags & SR_SEG_LAG) ? sl.lag1 - sl.lag0 : 0);   // (a select between the fields would go through memory)
    const char* src = sr_uni_ptr((const char*)(unsigned long long)t->base + slot * t->stride);
    quads = SR_UNI((g.flags & SR_SEG_QUADS) && ((unsigned)(unsigned long long)src & 15u) == 0);
    quads_w = SR_UNI((g.ldw & 3) == 0);
    if (FOR == SR_ROWS_ORDERED) turn = !(g.flags & SR_SEG_QUADS);
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const SrRowAt at = sr_row_at(p, g, i0 + (quads ? n * 16 + (lane >> 2) : (lane & 31)));
      row_h[n] = at.h;
      row_w[n] = at.w;
      row_at[n] = src + at.off * 4;
    }
  }

  __device__ __forceinline__ const char* gathered(int n, const SrTapAt& t, long long tap_bytes) const {
    return sr_gather_ok(g, SrRowAt{row_h[n], row_w[n], 0}, t) ? row_at[n] + tap_bytes : (const char*)sr_zero_line;
  }
  // theta at row r, column j (forward)
  __device__ __forceinline__ const char* theta(int r, int j) const {
    const bool ok = (r < g.R) & (j < g.ldw);   // (&& is a branch here: 2 % of a frame)
    return ok ? sr_at((const char*)g.w, (uint32_t)r * (uint32_t)g.ldw + (uint32_t)j) : (const char*)sr_zero_line;
  }

  // loads of the 16 reduction indices from r0 on, into LDS at `at`
  __device__ __forceinline__ void issue(int r0, unsigned at) {
    const char* zero = (const char*)sr_zero_line;
    const unsigned bt = at + 32 * 64;
    if (quads) {
      const int k4 = sr_f32_piece(lane >> 2, lane & 3);
      SrTapAt t;
      if ((g.GC & 15) == 0) {   // the step lies inside one tap: its decoding runs on the scalar unit
        t = sr_tap_at(g, SR_UNI(r0));
        t.c += 4 * k4;
      } else {
        t = sr_tap_at(g, r0 + 4 * k4);
      }
      const long long toff = sr_gather_off(g, t) * 4;
#pragma unroll
      for (int n = 0; n < N; ++n) sr_to_lds16(gathered(n, t, toff), at + n * 1024);
      if (BACK) {
        const bool r_ok = t.vi != SR_NO_TAP;
        const uint32_t woff = sr_weight_off(g, t, 0);
#pragma unroll
        for (int n = 0; n < N; ++n) {
          const int j = j0 + n * 16 + (lane >> 2);
          sr_to_lds16(r_ok && j < g.ldw ? sr_at((const char*)g.w, woff + (uint32_t)j * (uint32_t)g.GC) : zero, bt + n * 1024);
        }
        return;
      }
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int line = 2 * q + (lane >> 5);
        const SrTapAt t = sr_tap_at(g, r0 + (FOR == SR_ROWS_ORDERED && turn ? sr_in_turn(line) : line));
        sr_to_lds4(gathered(0, t, sr_gather_off(g, t) * 4), at + q * 256);
      }
      if (BACK) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int j = j0 + (lane & 31);
          const SrTapAt t = sr_tap_at(g, r0 + 2 * q + (lane >> 5));
          sr_to_lds4(t.vi != SR_NO_TAP && j < g.ldw ? sr_at((const char*)g.w, sr_weight_off(g, t, j)) : zero, bt + q * 256);
        }
        return;
      }
    }
    // forward: 16 lines of theta
    if (FOR == SR_ROWS_ORDERED && turn) {
      if (quads_w) {
#pragma unroll
        for (int n = 0; n < N; ++n) sr_to_lds16(theta(r0 + sr_in_turn(n * 8 + lane / 8), j0 + 4 * (lane % 8)), bt + n * 1024);
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) sr_to_lds4(theta(r0 + sr_in_turn(q * 2 + lane / 32), j0 + lane % 32), bt + q * 256);
      }
    } else if (quads_w) {
#pragma unroll
      for (int n = 0; n < N; ++n) sr_to_lds16(theta(r0 + n * 8 + lane / 8, j0 + 4 * (lane % 8)), bt + n * 1024);
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) sr_to_lds4(theta(r0 + q * 2 + lane / 32, j0 + lane % 32), bt + q * 256);
    }
  }

  // Addresses that go on from one of a wave's steps to the next, each in one tap.
  int vi, vj, c;             // tap and first channel of the step that the addresses are for
  const char* row_k[N];      // row_at, at this lane's channels of a step
  const char* cur[N];
  unsigned go[N];            // 4, or 0 where the line of zeros is read: bytes per channel passed
  const char* w;             // forward: theta at the step's first index, column j0; backwards: at its tap and channel, row j0
  uint32_t woff[BACK ? N : 1];

  // can the segment's steps go that way? (channels in sixteens; theta's lane offsets fit 32 bits)
  __device__ __forceinline__ bool goes_along() const { return quads && (g.GC & 15) == 0 && (BACK ? g.GC : g.ldw) < (1 << 22); }
  __device__ __forceinline__ void begin_along(int r0) {
    const SrTapAt t = sr_tap_at(g, SR_UNI(r0));
    vi = t.vi;
    vj = t.vj;
    c = t.c;
#pragma unroll
    for (int n = 0; n < N; ++n) row_k[n] = row_at[n] + 16 * sr_f32_piece(lane >> 2, lane & 3);
    if (BACK) {   // (columns that the node does not have read its last one)
#pragma unroll
      for (int n = 0; n < N; ++n)
        woff[n] = ((uint32_t)min(n * 16 + (lane >> 2), g.ldw - 1 - j0) * (uint32_t)g.GC + 4u * (uint32_t)sr_f32_piece(lane >> 2, lane & 3)) * 4u;
    } else {
      w = (const char*)g.w + ((unsigned long long)(unsigned)r0 * (unsigned)g.ldw + (unsigned)j0) * 4;
      woff[0] = quads_w ? ((uint32_t)(lane / 8) * (uint32_t)g.ldw + (uint32_t)min(4 * (lane % 8), g.ldw - 4 - j0)) * 4u
                        : ((uint32_t)(lane / 32) * (uint32_t)g.ldw + (uint32_t)min(lane % 32, g.ldw - 1 - j0)) * 4u;
    }
    look();
  }
  // the addresses at tap (vi, vj), channel c
  __device__ __forceinline__ void look() {
    const SrTapAt t{vi, vj, c};
    const long long toff = sr_gather_off(g, t) * 4;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const bool ok = sr_gather_ok(g, SrRowAt{row_h[n], row_w[n], 0}, t);
      cur[n] = ok ? row_k[n] + toff : (const char*)sr_zero_line;
      go[n] = ok ? 4u : 0u;
    }
    if (BACK) w = (const char*)g.w + (unsigned long long)(unsigned)j0 * (unsigned)g.GC * 4 + (unsigned long long)sr_weight_off(g, t, 0) * 4;
  }
  // ... four steps further on
  __device__ __forceinline__ void advance() {
    constexpr int D = 4 * SR_F32_KS;
    if (!BACK) w += (unsigned long long)((unsigned)g.ldw * (4u * D));
    c += D;
    if (c < g.GC) {
#pragma unroll
      for (int n = 0; n < N; ++n) cur[n] += D * go[n];
      if (BACK) w += 4 * D;
      return;
    }
    do {
      c -= g.GC;
      if (++vj == g.ntj) { vj = 0; ++vi; }
    } while (c >= g.GC);
    look();
  }
  // loads of a step all of whose indices exist, at the addresses in hand
  __device__ __forceinline__ void issue_along(unsigned at) const {
    const unsigned bt = at + 32 * 64;
#pragma unroll
    for (int n = 0; n < N; ++n) sr_to_lds16(cur[n], at + n * 1024);
    const char* wu = sr_uni_ptr(w);
    const unsigned line = (unsigned)g.ldw * 4u;
    if (BACK || quads_w) {
#pragma unroll
      for (int n = 0; n < N; ++n) {   // forward: eight lines further on each time
        uint32_t o = woff[BACK ? n : 0];
        asm volatile("" : "+v"(o));   // keeps the offset 32-bit: scalar base + lane offset addressing
        sr_to_lds16((BACK ? wu : wu + (unsigned long long)(n * 8) * line) + o, bt + n * 1024);
      }
    } else {
      uint32_t o = woff[0];
      asm volatile("" : "+v"(o));
#pragma unroll
      for (int q = 0; q < 8; ++q) sr_to_lds4(wu + (unsigned long long)(q * 2) * line + o, bt + q * 256);
    }
  }
};

// operand fragments of one 32-row (32-column) block for the eight products of a step: reduction index 8 (lane / 32) + kk
__device__ __forceinline__ void sr_frag_rows(const unsigned char* lds, int row, int half, float (&f)[8]) {
  const unsigned char* p = lds + row * 64;
  const f32x4_t lo = *(const f32x4_t*)(p + sr_f32_piece(row, 2 * half) * 16);
  const f32x4_t hi = *(const f32x4_t*)(p + sr_f32_piece(row, 2 * half + 1) * 16);
  f[0] = lo.x; f[1] = lo.y; f[2] = lo.z; f[3] = lo.w;
  f[4] = hi.x; f[5] = hi.y; f[6] = hi.z; f[7] = hi.w;
}
template <int T>
__device__ __forceinline__ void sr_frag_lines(const unsigned char* lds, int row, int half, float (&f)[8]) {
  const float* p = (const float*)lds + half * 8 * T + row;
#pragma unroll
  for (int k = 0; k < 8; ++k) f[k] = p[k * T];
}

template <int TI, int TJ, int MI, int MJ>
__device__ __forceinline__ void sr_step_products(const unsigned char* st, int iw, int jw, int lane, bool a_rows, bool b_rows,
                                                 f32x16_t (&acc)[MI][MJ]) {
  const int l = lane & 31, half = lane >> 5;
  float a[MI][8], b[MJ][8];
  if (a_rows) {
#pragma unroll
    for (int x = 0; x < MI; ++x) sr_frag_rows(st, iw + 32 * x + l, half, a[x]);
  } else {
#pragma unroll
    for (int x = 0; x < MI; ++x) sr_frag_lines<TI>(st, iw + 32 * x + l, half, a[x]);
  }
  if (b_rows) {
#pragma unroll
    for (int y = 0; y < MJ; ++y) sr_frag_rows(st + TI * 64, jw + 32 * y + l, half, b[y]);
  } else {
#pragma unroll
    for (int y = 0; y < MJ; ++y) sr_frag_lines<TJ>(st + TI * 64, jw + 32 * y + l, half, b[y]);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int x = 0; x < MI; ++x)
#pragma unroll
      for (int y = 0; y < MJ; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[x][k], b[y][k], acc[x][y], 0, 0, 0);
}

// The products of four steps for a 16 x 16 quarter of a 32 x 32 tile, four reduction indices per instruction, in the order
// in which the 32x32x2 products take them: 0, 8, 1, 9, ...  Both instructions add their products one after the other, each
// rounded like a fused multiply-add (300 000 sums compared bit for bit, products below the normal range among them).
struct SrQuarter { float a[4][4], b[4][4]; };   // operands of four steps
template <bool A_ROWS>
__device__ __forceinline__ void sr_quarter_read(const unsigned char* st, int iw, int jw, int lane, SrQuarter& f4) {
  constexpr int STAGE = 64 * 64;
  auto &a = f4.a, &b = f4.b;
  const int l = lane & 15, q = lane >> 4;
  const int k0 = 8 * (q & 1) + (q >> 1);   // this lane's index of product m: k0 + 2 m
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (A_ROWS) {
      float f[8];
      sr_frag_rows(st + s * STAGE, iw + l, q & 1, f);
#pragma unroll
      for (int m = 0; m < 4; ++m) a[s][m] = (q >> 1) ? f[2 * m + 1] : f[2 * m];
    } else {
      const float* p = (const float*)(st + s * STAGE) + k0 * 32 + iw + l;
#pragma unroll
      for (int m = 0; m < 4; ++m) a[s][m] = p[m * 64];
    }
    const float* p = (const float*)(st + s * STAGE + 32 * 64) + k0 * 32 + jw + l;
#pragma unroll
    for (int m = 0; m < 4; ++m) b[s][m] = p[m * 64];
  }
}
__device__ __forceinline__ void sr_quarter_products(const SrQuarter& f, f32x4_t& acc) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int m = 0; m < 4; ++m) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[s][m], f.b[s][m], acc, 0, 0, 0);
}

// K-split: every part leaves its registers in its slab, the part that arrives last adds them up in part order.
// Agent-scope accesses throughout: the parts run on different XCDs.
template <int N>
__device__ __forceinline__ bool sr_row_split(float (&o)[N], const SrSplitScratch& split, int slot, int part_info, int tid, int* flag) {
  const int n_parts = part_info >> 16;
  float* mine = split.slabs + ((size_t)slot + (size_t)(part_info & 0xffff)) * 1024 + tid;
#pragma unroll
  for (int q = 0; q < N; ++q)
    __hip_atomic_store((unsigned*)(mine + q * 256), __float_as_uint(o[q]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    int* counter = split.counters + slot;
    const int old = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *flag = (old == n_parts - 1);
    if (old == n_parts - 1) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!*flag) return false;
#pragma unroll
  for (int q = 0; q < N; ++q) o[q] = 0.f;
  const float* all = split.slabs + (size_t)slot * 1024 + tid;
  for (int p = 0; p < n_parts; ++p) {
#pragma unroll
    for (int q = 0; q < N; ++q)
      o[q] += __uint_as_float(__hip_atomic_load((const unsigned*)(all + (size_t)p * 1024 + q * 256), __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT));
  }
  return true;
}

// Where a tile's sums go and what is applied to them on the way: open() reads the node, locate() the tensors, a round trip each.
template <int FOR, int YB>
struct SrRowEnd {
  static constexpr bool BACK = FOR == SR_ROWS_BACK;
  float* out;
  const float *mask, *gate, *seed;
  int C, act, id_out, id_mask, id_x, id_seed;
  const float* biases;
  float bias[BACK ? 1 : YB];   // of this lane's columns j0, j0 + 32, ..
  __device__ __forceinline__ void open(SR_CONST4(SrRowNode) nd) {
    C = nd->C;
    act = nd->act;
    id_out = nd->out;
    id_mask = nd->mask;
    id_x = nd->x;
    id_seed = nd->seed;
    biases = nd->bias;
  }
  __device__ __forceinline__ void locate(const SrRowArgs& A, const SrSlots& sl, int j0) {
    auto tensor_at = [&](int id, int slot) -> float* {   // (tensor 0 stands in for one that is not there: no branch, so one round trip for all)
      SR_CONST4(SrTensor) t = sr_k(A.tensors) + max(id, 0);
      char* b = (char*)(unsigned long long)t->base;
      return (float*)(id < 0 || b == nullptr ? nullptr : b + slot * t->stride);
    };
    out = tensor_at(id_out, sl.own);
    mask = FOR == SR_ROWS_FRAME ? nullptr : tensor_at(id_mask, sl.frame);
    gate = BACK && act == 1 ? tensor_at(id_x, sl.frame) : nullptr;
    seed = BACK ? tensor_at(id_seed, sl.frame) : nullptr;
    if constexpr (!BACK) {
#pragma unroll
      for (int y = 0; y < YB; ++y) bias[y] = biases && j0 + y * 32 < C ? biases[j0 + y * 32] : 0.f;
    }
  }
};

// Bias, loss term, rectifier, gate and mask over a tile's sums o, and their store.  A lane has XB x YB blocks 32 rows and columns
// apart, in each VB values of column j0, from row row0 on (VB = 16: rows 8 (v / 4) + v % 4 further on).  i_end: the tile's end.
template <int FOR, int XB, int YB, int VB>
__device__ __forceinline__ void sr_row_store(const SrRowArgs& A, const SrRowEnd<FOR, YB>& end, SR_CONST4(SrPhase) ph, float* record, int rec_node,
                                             const float* o, int row0, int j0, int i_end) {
  constexpr bool BACK = FOR == SR_ROWS_BACK;
  SR_CONST4(SrRowNode) nd = sr_k(A.nodes) + ph->node;
  const int I = ph->I, S = ph->S, C = end.C;
  if (rec_node < 0 || nd->gnode != rec_node) record = nullptr;
  const bool whole = i_end <= I;   // all rows exist
  auto further = [](int q) { return VB == 4 ? q : 8 * (q >> 2) + (q & 3); };
#pragma unroll
  for (int x = 0; x < XB; ++x) {
    const int row = row0 + x * 32;
    size_t at[VB];
    if (S == 1) {
      const size_t at0 = (size_t)row * C;
#pragma unroll
      for (int q = 0; q < VB; ++q) at[q] = whole || row + further(q) < I ? at0 + (size_t)further(q) * C : 0;
    } else {
      const SrPhase p = sr_load_phase(ph);
      const int H = nd->H, W = nd->W;
#pragma unroll
      for (int q = 0; q < VB; ++q) {
        const int i = row + further(q) < I ? row + further(q) : 0;
        const int b = sr_divide(i, p.d_hpwp), rem = i - b * (p.Hp * p.Wp);
        const int hh = sr_divide(rem, p.d_wp), ww = rem - hh * p.Wp;
        at[q] = (((size_t)b * H + hh * p.S + p.ph) * W + ww * p.S + p.pw) * C;
      }
    }
#pragma unroll
    for (int y = 0; y < YB; ++y) {
      const int j = j0 + y * 32;
      if (j >= C) continue;
      float val[VB];
#pragma unroll
      for (int q = 0; q < VB; ++q) val[q] = o[(x * YB + y) * VB + q] + (BACK ? 0.f : end.bias[BACK ? 0 : y]);
      if (end.seed) {
#pragma unroll
        for (int q = 0; q < VB; ++q) val[q] += end.seed[at[q] + j];
      }
      if (BACK) {
        if (end.gate) {
#pragma unroll
          for (int q = 0; q < VB; ++q) val[q] = end.gate[at[q] + j] > 0.f ? val[q] : 0.f;
        }
      } else if (end.act == 1) {
#pragma unroll
        for (int q = 0; q < VB; ++q) val[q] = fmaxf(val[q], 0.f);
      }
      if (end.mask) {
#pragma unroll
        for (int q = 0; q < VB; ++q) val[q] *= end.mask[at[q] + j];
      }
      if (whole) {
#pragma unroll
        for (int q = 0; q < VB; ++q) end.out[at[q] + j] = val[q];
      } else {
#pragma unroll
        for (int q = 0; q < VB; ++q)
          if (row + further(q) < I) end.out[at[q] + j] = val[q];
      }
      if (record) {
#pragma unroll
        for (int q = 0; q < VB; ++q)
          if (row + further(q) < I) record[at[q] + j] = val[q];
      }
    }
  }
}

// A 32 x 32 tile.  Every wave takes every fourth step through LDS of its own (no barriers); the four waves' sums are added in order
// at the end.  Ordered, four steps go at a time: wave w fetches the w-th, then every wave multiplies all four for a 16 x 16
// quarter of the tile -- as long a chain of products per wave.
template <int FOR, int STAGES>
__device__ __forceinline__ void sr_small_tile(const SrRowArgs& A, SR_CONST4(SrPhase) phase, int i0, int j0, int step_begin, int step_end,
                                              int split_slot, int part_info, const SrSlots& sl, float* record, int rec_node,
                                              unsigned char* lds) {
  constexpr bool BACK = FOR == SR_ROWS_BACK, QUARTERS = FOR == SR_ROWS_ORDERED;
  typedef SrSmallOperands<FOR> Ops;
  const int tid = threadIdx.x, lane = tid & 63, wave = SR_UNI(tid >> 6);
  constexpr int PITCH = (QUARTERS ? 4 : 1) * Ops::STAGE;   // from one stage to the next
  unsigned char* base = QUARTERS ? lds : lds + wave * (STAGES * Ops::STAGE);
  const unsigned at0 = sr_lds_at(base) + (QUARTERS ? wave * Ops::STAGE : 0);
  const SrPhase p = sr_load_phase(phase);

  Ops op;
  op.lane = lane; op.i0 = i0; op.j0 = j0;
  f32x16_t acc[1][1];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[0][0][v] = 0.f;
  f32x4_t quarter{0.f, 0.f, 0.f, 0.f}, quarter_sum{0.f, 0.f, 0.f, 0.f};   // ordered: of the segment, of those that are done

  // two groups of segments: those that depend on the image only (backwards), whose sum is scaled, then the others
#pragma nounroll
  for (int group = BACK && p.seg_image > p.seg_begin ? 0 : 1; group < 2; ++group) {
    int seg = (group == 0 ? p.seg_begin : p.seg_image) - 1;
    const int seg_end = group == 0 ? p.seg_image : p.seg_end;
    constexpr int INC = 4 * SR_F32_KS, AHEAD = STAGES - 1;
    int r = 0, r_stop = 0;   // next step's first index, end of the segment's share
    // r: the next step of this wave (quarters: four steps), in the next segment where this one's share is done; false when there is none
    auto settle = [&]() -> bool {
      while (r >= r_stop) {
        if (++seg >= seg_end) return false;
        op.g = sr_load_seg(sr_k(A.segs) + seg);
        if (!sr_seg_counts<BACK>(op.g, sl)) continue;
        const int n = (op.g.R + SR_F32_KS - 1) / SR_F32_KS;
        int lo = max(step_begin - op.g.step0, 0);
        const int hi = min(step_end - op.g.step0, n);
        if (!QUARTERS) lo += (wave - (op.g.step0 + lo)) & 3;
        r = lo * SR_F32_KS;
        r_stop = hi * SR_F32_KS;
        if (r < r_stop) op.enter(p, A.tensors, sl);
      }
      return true;
    };
    auto next = [&]() -> bool {
      r += INC;
      return settle();
    };
    int issued = 0, done = 0, wr = 0, rd = 0;
    unsigned rows = 0;   // per stage: the gathered operand (backwards: both) lies row by row
    unsigned ends = 0;   // ordered, per stage: it is the last one of its segment
    auto issue = [&]() {
      const unsigned bit = 1u << wr;
      rows = op.quads ? rows | bit : rows & ~bit;
      if constexpr (QUARTERS) ends = r + INC >= r_stop ? ends | bit : ends & ~bit;
      // (quarters: the steps of the four that are past the end of the share are zero)
      op.issue(!QUARTERS ? r : (r + wave * SR_F32_KS < r_stop ? r + wave * SR_F32_KS : op.g.R), at0 + wr * PITCH);
      wr = wr == STAGES - 1 ? 0 : wr + 1;
      ++issued;
    };
    auto multiply = [&](bool a_rows) {   // the stage at rd
      const unsigned char* st = base + rd * PITCH;
      if constexpr (QUARTERS) {
        SrQuarter f;
        if (a_rows) sr_quarter_read<true>(st, 16 * (wave >> 1), 16 * (wave & 1), lane, f);
        else sr_quarter_read<false>(st, 16 * (wave >> 1), 16 * (wave & 1), lane, f);
        sr_quarter_products(f, quarter);
      } else {
        sr_step_products<32, 32, 1, 1>(st, 0, 0, lane, a_rows, BACK && a_rows, acc);
      }
    };
    auto fold = [&]() {   // a segment is done
      quarter_sum += quarter;
      quarter = f32x4_t{0.f, 0.f, 0.f, 0.f};
    };
    bool more = next();
    // The steps of whole segments back to back, from r on, nothing but their loads and products: as long as there are
    // such steps, AHEAD of them on the way at a time.
    auto run_along = [&]() {
      int n = 0;   // passes to go
      auto begin = [&](int least) -> bool {
        n = (r_stop - r + (QUARTERS ? 0 : INC - SR_F32_KS)) / INC;
        if (!more || n < least || !op.goes_along()) return false;
        op.begin_along(QUARTERS ? r + wave * SR_F32_KS : r);
        return true;
      };
      if (!begin(1)) return;
      bool folding = false;
      for (;;) {
        if constexpr (QUARTERS && STAGES > 3) {
          // A quarter's sixteen products are a chain of 512 cycles; the reads of the next four steps' operands go under it.
          SrQuarter f, g;
          auto read = [&](SrQuarter& q) {
            if (!op.quads_w) sr_wait_loads<(AHEAD - 1) * (Ops::N + 8)>();
            else sr_wait_loads<(AHEAD - 1) * Ops::LOADS>();
            sr_step_barrier();   // as below
            op.issue_along(at0 + wr * PITCH);
            op.advance();
            sr_quarter_read<true>(base + rd * PITCH, 16 * (wave >> 1), 16 * (wave & 1), lane, q);
            r += INC;
            rd = rd == STAGES - 1 ? 0 : rd + 1;
            wr = wr == STAGES - 1 ? 0 : wr + 1;
            --n;
          };
          read(f);
          for (;;) {
            if (n == 0) { sr_quarter_products(f, quarter); break; }
            read(g);
            sr_quarter_products(f, quarter);
            if (n == 0) { sr_quarter_products(g, quarter); break; }
            read(f);
            sr_quarter_products(g, quarter);
          }
        } else {
          do {
            if (!BACK && !op.quads_w) sr_wait_loads<(AHEAD - 1) * (Ops::N + 8)>();
            else sr_wait_loads<(AHEAD - 1) * Ops::LOADS>();
            if (QUARTERS) sr_step_barrier();   // everybody's loads of the steps in hand; and the ones before have been read by all
            op.issue_along(at0 + wr * PITCH);
            op.advance();
            multiply(true);
            r += INC;
            rd = rd == STAGES - 1 ? 0 : rd + 1;
            wr = wr == STAGES - 1 ? 0 : wr + 1;
          } while (--n > 0);
        }
        ends = 0;
        if (QUARTERS && folding) {
          fold();   // the segment before: its last steps were multiplied while this one's first were on the way
          folding = false;
          n = (r_stop - r) / INC;
          if (n > 0) continue;
        }
        if (r < r_stop) break;   // what is less than four steps
        if (QUARTERS) ends = 1u << (wr == 0 ? STAGES - 1 : wr - 1);
        more = settle();
        if (!begin(QUARTERS ? AHEAD : 1)) break;
        if (QUARTERS) {
          folding = true;
          n = AHEAD;
        }
      }
      rows = (1u << STAGES) - 1u;
    };
#pragma nounroll
    for (int k = 0; k < AHEAD && more; ++k) {
      issue();
      more = next();
    }
    while (done < issued) {
      bool end;   // of the loop: ordered, of a segment
      do {
        if (issued - done == AHEAD && r < r_stop) {
          const unsigned others = ((1u << STAGES) - 1u) & ~(1u << wr);   // the stages on the way: row by row, and none ends a segment?
          if ((rows & others) == others && !(QUARTERS && (ends & others))) run_along();
        }
        if (STAGES > 3 && issued - done >= 3) sr_wait_loads<2 * Ops::LOADS>();
        else if (issued - done >= 2) sr_wait_loads<Ops::LOADS>();
        else sr_wait_loads<0>();
        if (QUARTERS) sr_step_barrier();   // everybody's loads of this step; and the step before has been read by all
        end = QUARTERS && ((ends >> rd) & 1);
        if (more) {
          issue();
          more = next();
        }
        multiply((rows >> rd) & 1);
        rd = rd == STAGES - 1 ? 0 : rd + 1;
        ++done;
        if (!QUARTERS) end = done == issued;
      } while (!end);
      if (QUARTERS) fold();
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (QUARTERS) sr_step_barrier();   // the stages are free again
    if (BACK && group == 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[0][0][v] *= p.image_scale;
    }
  }

  // register v of lane l holds row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 (a quarter: row 4 (l / 16) + v, column l % 16)
  float o[4];
  if constexpr (QUARTERS) {
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = quarter_sum[q];
  } else {
    __syncthreads();
    float* red = (float*)lds;   // [wave][register][lane]
#pragma unroll
    for (int v = 0; v < 16; ++v) red[(wave * 16 + v) * 64 + lane] = acc[0][0][v];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float* s = red + (4 * wave + q) * 64 + lane;
      o[q] = ((s[0] + s[16 * 64]) + s[32 * 64]) + s[48 * 64];
    }
  }
  if ((part_info >> 16) > 1) {
    __syncthreads();
    if (!sr_row_split<4>(o, A.split, split_slot, part_info, tid, (int*)lds)) return;
  }
  const int row = i0 + (QUARTERS ? 16 * (wave >> 1) + 4 * (lane >> 4) : 8 * wave + 4 * (lane >> 5));
  const int column = j0 + (QUARTERS ? 16 * (wave & 1) + (lane & 15) : (lane & 31));
  SrRowEnd<FOR, 1> end;
  end.open(sr_k(A.nodes) + p.node);
  end.locate(A, sl, column);
  sr_row_store<FOR, 1, 1, 4>(A, end, phase, record, rec_node, o, row, column, i0 + 32);
}

// A tile of four waves.
template <int TI, int TJ, int WJN, int FOR, int STAGES>
__device__ __forceinline__ void sr_row_tile(const SrRowArgs& A, SR_CONST4(SrPhase) phase, int i0, int j0, int step_begin, int step_end,
                                            const SrSlots& sl, float* record, int rec_node, unsigned char* lds) {
  constexpr bool BACK = FOR == SR_ROWS_BACK, ORDERED = FOR == SR_ROWS_ORDERED;
  constexpr bool PAIRS = STAGES == SR_F32_PAIRS;
  constexpr int WIN = 4 / WJN, MI = TI / (32 * WIN), MJ = TJ / (32 * WJN);
  typedef SrRowOperands<TI, TJ, FOR> Ops;
  const int tid = threadIdx.x, lane = tid & 63, wave = SR_UNI(tid >> 6);
  const int iw = (wave / WJN) * 32 * MI, jw = (wave % WJN) * 32 * MJ;
  const unsigned at0 = sr_lds_at(lds);

  Ops op;
  op.wv = wave; op.lane = lane; op.i0 = i0; op.j0 = j0;
  f32x16_t acc[MI][MJ];
#pragma unroll
  for (int x = 0; x < MI; ++x)
#pragma unroll
    for (int y = 0; y < MJ; ++y)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[x][y][v] = 0.f;
  f32x16_t sum[ORDERED ? MI : 1][ORDERED ? MJ : 1];   // of the segments that are done
  if constexpr (ORDERED) {
#pragma unroll
    for (int x = 0; x < MI; ++x)
#pragma unroll
      for (int y = 0; y < MJ; ++y) sum[x][y] = acc[x][y];
  }

  __builtin_amdgcn_s_setprio(2);
  const int seg_begin = phase->seg_begin, seg_image = phase->seg_image, seg_last = phase->seg_end;
  // Located while the first operands are on their way (24x24 frames of 40 channels 995 -> 965 us; DSR6 571 -> 567), but at the end in the
  // forward pass of a window: there it took registers that its sums need (a first depth of 2 to 5 steps a tile: GTSRB-shaped 59 -> 47
  // us, DSR2 31 -> 28)
  constexpr bool EARLY = !ORDERED;
  SrRowEnd<FOR, MJ> end;
  const int column = j0 + jw + (lane & 31);
  if (EARLY) end.open(sr_k(A.nodes) + phase->node);
  // two groups of segments: those that depend on the image only (backwards), whose sum is scaled, then the others
  const int first = BACK && seg_image > seg_begin ? 0 : 1;
  for (int group = first; group < 2; ++group) {
    int seg = (group == 0 ? seg_begin : seg_image) - 1;
    const int seg_end = group == 0 ? seg_image : seg_last;
    int r = 0, r_stop = 0;   // next step's first index, end of the segment's share
    // r: the next step of this workgroup (wave), in the next segment where this one's share is done; false when there is none
    auto settle = [&]() -> bool {
      while (r >= r_stop) {
        if (++seg >= seg_end) return false;
        const SrSeg g = sr_load_seg(sr_k(A.segs) + seg);
        if (!sr_seg_counts<BACK>(g, sl)) continue;
        const int n = (g.R + SR_F32_KS - 1) / SR_F32_KS;
        const int lo = max(step_begin - g.step0, 0);
        const int hi = min(step_end - g.step0, n);
        r = lo * SR_F32_KS;
        r_stop = hi * SR_F32_KS;
        if (r < r_stop) op.enter(g, sr_k(A.segs) + seg, phase, A.tensors, A.lines, sl, r);
      }
      return true;
    };
    auto next = [&]() -> bool {
      r += SR_F32_KS;
      return settle();
    };
    int issued = 0, done = 0, wr = 0, rd = 0;
    unsigned rows = 0;   // per stage: the gathered operand (backwards: both) lies row by row
    unsigned ends = 0;   // ordered, per stage: it is the last one of its segment
    auto mark = [&](int stage) {   // what the step at r, about to be fetched into `stage`, is
      const unsigned bit = 1u << stage;
      rows = op.quads ? rows | bit : rows & ~bit;
      if constexpr (ORDERED)
        ends = r + SR_F32_KS >= r_stop ? ends | bit : ends & ~bit;
    };
    auto issue = [&]() {
      mark(wr);
      op.issue(r, at0 + wr * Ops::STAGE);
      if (!PAIRS) wr = wr == STAGES - 1 ? 0 : wr + 1;
      ++issued;
    };
    auto multiply = [&](int stage, bool a_rows) {
      __builtin_amdgcn_s_setprio(0);
      sr_step_products<TI, TJ, MI, MJ>(lds + stage * Ops::STAGE, iw, jw, lane, a_rows, BACK && a_rows, acc);
      __builtin_amdgcn_s_setprio(2);
    };
    // do these stages hold steps that lie row by row, and none that ends a segment?
    auto plain = [&](unsigned stages) { return (rows & stages) == stages && !(ORDERED && (ends & stages)); };
    auto fold = [&]() {   // a segment is done
      if constexpr (ORDERED) {
#pragma unroll
        for (int x = 0; x < MI; ++x)
#pragma unroll
          for (int y = 0; y < MJ; ++y)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
              sum[x][y][v] += acc[x][y][v];
              acc[x][y][v] = 0.f;
            }
      }
    };
    // The steps (pairs) of whole segments back to back, from r on, nothing but their loads and products: as long as there are
    // such steps, AHEAD of them on the way at a time.  (Every step through the code that takes any step of any segment cost 130
    // instructions around a pair's 16 products: 98 us of a DSR2 frame of batch 64; the same without them 67.)
    constexpr int INC = (PAIRS ? 2 : 1) * SR_F32_KS, AHEAD = PAIRS ? 1 : STAGES - 1;
    bool more = next();
    auto run_along = [&]() {
      int n = 0;   // passes to go
      const char* w = nullptr;
      auto begin = [&](int least) -> bool {
        if (!more || !op.template all_along<PAIRS>(r)) return false;
        n = (r_stop - r) / INC;
        if (n < least) return false;
        op.go_on(r);
        if (!BACK) w = op.theta(r);
        return true;
      };
      if (!begin(1)) return;
      bool folding = false;
      unsigned w_step = (unsigned)op.ldw * (4u * INC);
      for (;;) {
        do {
          sr_wait_loads<PAIRS ? 0 : (AHEAD - 1) * Ops::LOADS>();
          sr_step_barrier();   // everybody's loads of the steps in hand; and the ones before have been read by all
          op.template issue_along<PAIRS>(at0 + wr * Ops::STAGE, w);
          op.template advance<INC>();
          if (!BACK) w += w_step;
          multiply(rd, true);
          if (PAIRS) multiply(rd + 1, true);
          r += INC;
          if (PAIRS) {
            rd ^= 2;
            wr ^= 2;
          } else {
            rd = rd == STAGES - 1 ? 0 : rd + 1;
            wr = wr == STAGES - 1 ? 0 : wr + 1;
          }
        } while (--n > 0);
        ends = 0;
        if (ORDERED && folding) {
          fold();   // the segment before: its last steps were multiplied while this one's first were on the way
          folding = false;
          n = (r_stop - r) / INC;
          if (n > 0) continue;
        }
        if (r < r_stop) break;   // what is less than a pair
        if (ORDERED) ends = 1u << (PAIRS ? rd + 1 : (wr == 0 ? STAGES - 1 : wr - 1));
        more = settle();
        if (!begin(ORDERED ? AHEAD : 1)) break;
        w_step = (unsigned)op.ldw * (4u * INC);
        if (ORDERED) {
          folding = true;
          n = AHEAD;
        }
      }
      rows = (1u << (PAIRS ? 4 : STAGES)) - 1u;
    };
    if constexpr (PAIRS) {
      // two steps per barrier: a pair is fetched while the one before it is multiplied
      auto issue_pair = [&](int to) -> int {
        int n = 0;
#pragma nounroll
        for (bool last = false; n < 2 && more && !last; ++n) {
          wr = to + n;
          issue();
          last = ORDERED && ((ends >> (to + n)) & 1);   // a pair lies in one segment
          more = next();
        }
        return n;
      };
      int cur = issue_pair(0);
      if (EARLY && group == first) end.locate(A, sl, column);
      while (cur > 0) {
        bool end;   // of the loop: ordered, of a segment
        do {
          if (cur == 2 && plain(3u << rd)) {
            wr = rd ^ 2;
            run_along();
          }
          sr_wait_loads<0>();
          sr_step_barrier();   // everybody's loads of this pair; and the pair before has been read by all
          end = ORDERED && ((ends >> (rd + cur - 1)) & 1);
          const int following = issue_pair(rd ^ 2);
          multiply(rd, (rows >> rd) & 1);
          if (cur == 2) multiply(rd + 1, (rows >> (rd + 1)) & 1);
          rd ^= 2;
          cur = following;
          if (!ORDERED) end = cur == 0;
        } while (!end);
        fold();
      }
      issued = 0;
    } else {
#pragma nounroll
      for (int k = 0; k < STAGES - 1 && more; ++k) {
        issue();
        more = next();
      }
      if (EARLY && group == first) end.locate(A, sl, column);
      while (done < issued) {
        bool end;
        do {
          if (issued - done == AHEAD && plain(((1u << STAGES) - 1u) & ~(1u << wr))) run_along();
          if (issued - done >= 2) sr_wait_loads<Ops::LOADS>();
          else sr_wait_loads<0>();
          sr_step_barrier();   // everybody's loads of this step; and the step before has been read by all
          end = ORDERED && ((ends >> rd) & 1);
          if (more) {
            issue();
            more = next();
          }
          multiply(rd, (rows >> rd) & 1);
          rd = rd == STAGES - 1 ? 0 : rd + 1;
          ++done;
          if (!ORDERED) end = done == issued;
        } while (!end);
        fold();
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    sr_step_barrier();   // the stages are free again
    if (BACK && group == 0) {
      const float image_scale = sr_again(phase)->image_scale;
#pragma unroll
      for (int x = 0; x < MI; ++x)
#pragma unroll
        for (int y = 0; y < MJ; ++y)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[x][y][v] *= image_scale;
    }
  }

  // register v of lane l holds row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 of its block
  float o[MI * MJ * 16];
#pragma unroll
  for (int x = 0; x < MI; ++x)
#pragma unroll
    for (int y = 0; y < MJ; ++y)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[(x * MJ + y) * 16 + v] = ORDERED ? sum[ORDERED ? x : 0][ORDERED ? y : 0][v] : acc[x][y][v];
  if (!EARLY) {
    end.open(sr_k(A.nodes) + sr_again(phase)->node);
    end.locate(A, sl, column);
  }
  sr_row_store<FOR, MI, MJ, 16>(A, end, sr_again(phase), record, rec_node, o, i0 + iw + 4 * (lane >> 5), column, i0 + TI);
}

template <int FOR, int VARIANT>
__device__ __forceinline__ void sr_row_item(const SrRowArgs& A, SR_CONST4(SrRowTile) t, int slot0, const SrSlots& sl, float* record,
                                            int rec_node, unsigned char* lds) {
  const int phase = t->phase;
  if (phase < 0) return;
  SR_CONST4(SrPhase) p = sr_k(A.phases) + phase;
  const int shape = t->shape, i0 = t->i0, j0 = t->j0, sb = t->step_begin, se = t->step_end, slot = slot0 + t->split_slot, part = t->part;
  if constexpr (VARIANT != SR_F32_DEEP) {
    if constexpr (VARIANT == SR_F32_WIDE)
      if (shape == SR_F32_128x128) sr_row_tile<128, 128, 2, FOR, 3>(A, p, i0, j0, sb, se, sl, record, rec_node, lds);
    if (shape == SR_F32_128x64) sr_row_tile<128, 64, 2, FOR, 3>(A, p, i0, j0, sb, se, sl, record, rec_node, lds);
    else if (shape == SR_F32_64x64) sr_row_tile<64, 64, 2, FOR, SR_F32_PAIRS>(A, p, i0, j0, sb, se, sl, record, rec_node, lds);
    else if (shape == SR_F32_128x32) sr_row_tile<128, 32, 1, FOR, SR_F32_PAIRS>(A, p, i0, j0, sb, se, sl, record, rec_node, lds);
  }
  if (shape == SR_F32_SMALL)
    sr_small_tile<FOR, sr_f32_stages(VARIANT, SR_F32_SMALL)>(A, p, i0, j0, sb, se, slot, part, sl, record, rec_node, lds);
}

}  // namespace

template <int VARIANT>
__global__ __launch_bounds__(256, VARIANT == SR_F32_NARROW ? 4 : 2) void sr_rows_frame_kernel(SrFrame f, SrRowArgs A,
                                                               const SrAux* __restrict__ aux, int n_aux, int aux_at,
                                                               const SrHead* __restrict__ heads,
                                                               const SrHeadEdge* __restrict__ head_edges,
                                                               const SrStageNode* __restrict__ stage_nodes, int vec_floats) {
  extern __shared__ __align__(1024) unsigned char sr_rows_lds[];
  const int item = blockIdx.x;
  const sr_call_t call = sr_call(f);
  const int frame = call->frame + f.offset;
  if (item >= aux_at && item < aux_at + n_aux) {
    sr_aux_item<float>(f.ctx, call, aux[item - aux_at], heads, head_edges, stage_nodes, (float*)sr_rows_lds, vec_floats, frame,
                       SrFlow{nullptr, nullptr, 0, 0, nullptr});
  } else {
    const int cur = frame & 1;
    const SrSlots sl{cur, cur ^ 1, cur, 0, 1 << 30};
    char* rec = A.rec_node >= 0 ? (char*)(unsigned long long)call->out_ptr : nullptr;
    if (rec) rec += (int64_t)(frame - call->out_base) * call->out_stride;
    sr_row_item<SR_ROWS_FRAME, VARIANT>(A, sr_k(A.tiles) + (item < aux_at ? item : item - n_aux), 0, sl, (float*)rec, rec ? A.rec_node : -1, sr_rows_lds);
  }
  sr_block_done(f, gridDim.x);
}

hipError_t sr_launch_rows_frame(hipStream_t s, const SrFrame& f, const SrRowArgs& a, int shapes, const SrAux* aux, int n_aux,
                                const SrHead* heads, const SrHeadEdge* head_edges, const SrStageNode* stage_nodes,
                                int aux_smem_bytes) {
  if (a.n_tiles + n_aux == 0) return hipSuccess;
  const int variant = sr_f32_variant(shapes), tile_lds = sr_f32_lds_bytes(shapes);
  const auto kernel = variant == SR_F32_WIDE ? sr_rows_frame_kernel<SR_F32_WIDE>
                                             : (variant == SR_F32_NARROW ? sr_rows_frame_kernel<SR_F32_NARROW> : sr_rows_frame_kernel<SR_F32_DEEP>);
  hipLaunchKernelGGL(kernel, dim3(a.n_tiles + n_aux), dim3(256), tile_lds > aux_smem_bytes ? tile_lds : aux_smem_bytes, s, f, a, aux, n_aux, a.n_tiles / 2, heads,
                     head_edges, stage_nodes, (aux_smem_bytes - 16 - 4096) / 4);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// training window
// ---------------------------------------------------------------------------
template <bool BACK, int VARIANT>
__global__ __launch_bounds__(256, VARIANT == SR_F32_NARROW ? 4 : 2) void sr_rows_train_kernel(SrRowArgs A) {
  extern __shared__ __align__(1024) unsigned char sr_rows_lds[];
  // the run (tile list, frame) this workgroup belongs to: runs are in order of their first workgroup
  const int lane = threadIdx.x & 63, block = (int)blockIdx.x + A.first;
  // (a lane reads a whole run, so the one found needs no second round trip)
  SrRun mine{0x7fffffff, 0, 0, 0}, run{0, 0, 0, 0};
  for (int base = 0; base < A.n_runs; base += 64) {
    mine = SrRun{0x7fffffff, 0, 0, 0};
    if (base + lane < A.n_runs) mine = A.runs[base + lane];
    const unsigned long long m = __builtin_amdgcn_ballot_w64(mine.block0 <= block);
    if (m == 0) break;   // the last one of the 64 before
    const int k = __popcll(m) - 1;
    run.block0 = __builtin_amdgcn_readlane(mine.block0, k);
    run.tile0 = __builtin_amdgcn_readlane(mine.tile0, k);
    run.frame = __builtin_amdgcn_readlane(mine.frame, k);
    run.slot0 = __builtin_amdgcn_readlane(mine.slot0, k);
    if (m != ~0ull) break;
  }
  const int frame = A.frame0 + run.frame;
  SrSlots sl;
  if (BACK) {
    sl.lag0 = frame % A.ring;
    sl.lag1 = (frame + 1) % A.ring;
    sl.own = sl.lag0;
    sl.left = A.window - frame;
  } else {
    sl.lag0 = frame;
    sl.lag1 = frame - 1;
    sl.own = frame;
    sl.left = frame;
  }
  sl.frame = frame;
  sr_row_item<BACK ? SR_ROWS_BACK : SR_ROWS_ORDERED, VARIANT>(A, sr_k(A.tiles) + run.tile0 + (block - run.block0), run.slot0, sl, nullptr, -1, sr_rows_lds);
}

namespace {

// The operands of a weight gradient tile: 16 lines of TI (source channels of the taps' pixels) and of TJ (target
// channels) elements per step; a pixel's channels are contiguous.
template <int TI, int TJ>
struct SrGradOperands {
  static constexpr int NA = TI / 64, NB = TJ >= 64 ? TJ / 64 : 1, STAGE = (TI + TJ) * 64, LOADS = NA + NB;
  static constexpr bool HALF_B = TJ < 64;
  SrGradEdge e;
  const char *xb0, *yb0;
  long long xs, ys, image;
  int quads_a, quads_b, ring;
  int wv, lane, j0;
  int ti, tj;          // this lane's row (rows i .. i + 3) of A: tap and ...
  uint32_t aoff;       // ... offset from the window's first element
  // The pixels of the next step, if its frame's steps go on from one another (SrGradEdge::along): where this lane's tap lies in
  // the source image, and floats from the frame's start.  (Decoded from the step's number, a load cost ten multiplications, at a
  // quarter of the rate each: windows of DSR2 1480 us, with the pixels so 1443; GTSRB-shaped 5620, 5540.)
  static constexpr int LINES = TI == 128 ? 8 : 4;   // 4-byte loads: pixels per wave and step, one after the other, 64 rows of each
  SrPixStep go;                      // 16-byte loads: 16 pixels on
  int at_h[NA], at_w[NA], lim_h, lim_w;
  int tap_h;                         // tap row, and how many rows of the image it may lie in: none for a row of theta past the last
  unsigned in_h;
  uint32_t at_off[NA], ob;
  int px_h, px_w;                    // 4-byte loads: the wave's next pixel (scalar)
  uint32_t px_off;
  int along, fi, m0, fresh;
  const char *xf, *yf;

  // pixel m's window, at this lane's tap
  __device__ __forceinline__ void look(int n, int m) {
    const int b = sr_divide(m, e.d_howo), rem = m - b * (e.Ho * e.Wo), ho = sr_divide(rem, e.d_wo), wo = rem - ho * e.Wo;
    const int h = ho * e.stride - e.pad, w = wo * e.stride - e.pad;
    at_off[n] = (((uint32_t)b * (uint32_t)e.H + (uint32_t)h) * (uint32_t)e.W + (uint32_t)w) * (uint32_t)e.Cin + aoff;
    at_h[n] = h + tap_h;
    at_w[n] = w + tj;
  }
  __device__ __forceinline__ const char* looked(int n) const {
    return (unsigned)at_h[n] < in_h && (unsigned)at_w[n] < (unsigned)e.W ? sr_at(xf, at_off[n]) : (const char*)sr_zero_line;
  }
  // ... that of a later one
  __device__ __forceinline__ void step_on(int n) {
    sr_pix_go(go, e.stride, lim_w, lim_h, &at_w[n], &at_h[n], &at_off[n]);
  }

  // the tile's first step
  __device__ __forceinline__ void begin(int step) {
    fi = sr_divide(step, e.d_steps);
    m0 = (step - fi * e.steps_per_frame) * SR_F32_KS;
    fresh = 0;
    if (!along) return;
    go = sr_pix_step(e, SR_F32_KS);
    tap_h = ti == SR_NO_TAP ? 0 : ti;
    in_h = ti == SR_NO_TAP ? 0u : (unsigned)e.H;
    lim_h = e.Ho * e.stride - e.pad + tap_h;
    lim_w = e.Wo * e.stride - e.pad + tj;
    const int id = HALF_B ? wv * 32 + lane : wv * 64 + lane;
    if (quads_b) ob = ((uint32_t)(id / (TJ / 4)) * (uint32_t)e.Cout + (uint32_t)min(4 * (id % (TJ / 4)), e.Cout - 4 - j0)) * 4u;
    else ob = ((uint32_t)((wv * 64 + lane) / TJ) * (uint32_t)e.Cout + (uint32_t)min((wv * 64 + lane) % TJ, e.Cout - 1 - j0)) * 4u;
    fresh = 1;
  }
  __device__ __forceinline__ void frame_begin() {
    const int frame = e.frame0 + fi;
    xf = sr_uni_ptr(xb0 + (frame - e.lag) * xs);
    yf = sr_uni_ptr(yb0 + (frame % ring) * ys + ((long long)m0 * e.Cout + j0) * 4);
    if (quads_a) {
#pragma unroll
      for (int n = 0; n < NA; ++n) look(n, m0 + (n * 4 + wv) * (256 / TI) + lane / (TI / 4));
    } else {
      const SrPixAt p = sr_pix_at(e, SR_UNI(m0 + LINES * (TI == 128 ? wv >> 1 : wv)));
      px_h = p.h;
      px_w = p.w;
      px_off = sr_pix_off(e, p, 0, 0);
    }
  }
  // loads of the next step
  __device__ __forceinline__ void issue_next(unsigned at) {
    const char* zero = (const char*)sr_zero_line;
    if (fresh) {
      frame_begin();
      fresh = 0;
    }
    if (!along || m0 + SR_F32_KS > e.M) {
      issue(fi * e.steps_per_frame + m0 / SR_F32_KS, at);
    } else {
      if (quads_a) {
#pragma unroll
        for (int n = 0; n < NA; ++n) {
          sr_to_lds16(looked(n), at + (n * 4 + wv) * 1024);
          step_on(n);
        }
      } else {
        const SrPixStep one = sr_pix_one(e, go);
        int h = px_h, w = px_w;   // the wave's pixels one after the other
        uint32_t off = px_off;
        const unsigned line = at + LINES * (TI == 128 ? wv >> 1 : wv) * (TI * 4) + (TI == 128 ? (wv & 1) * 256 : 0);
#pragma nounroll
        for (int q = 0; q < LINES; ++q) {
          const bool ok = (unsigned)(h + tap_h) < in_h && (unsigned)(w + tj) < (unsigned)e.W;
          sr_to_lds4(ok ? sr_at(xf, off + aoff) : zero, line + q * (TI * 4));
          sr_pix_go(one, e.stride, one.n_w - e.pad, one.n_h - e.pad, &w, &h, &off);
        }
        sr_pix_go(go, e.stride, go.n_w - e.pad, go.n_h - e.pad, &px_w, &px_h, &px_off);
      }
      const unsigned bt = at + TI * 64, line = (unsigned)e.Cout * 4u;
      const char* y = sr_uni_ptr(yf);
      uint32_t o = ob;
      asm volatile("" : "+v"(o));   // keeps the offset 32-bit: scalar base + lane offset addressing
      if (quads_b) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const char* yn = y + (unsigned long long)(n * (1024 / TJ)) * line;
          if (HALF_B) {
            if (lane < 32) sr_to_lds16(yn + o, bt + wv * 512);
          } else {
            sr_to_lds16(yn + o, bt + (n * 4 + wv) * 1024);
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < TJ / 16; ++q) sr_to_lds4(y + (unsigned long long)(q * 256 / TJ) * line + o, bt + (q * 4 + wv) * 256);
      }
      yf = y + (unsigned long long)SR_F32_KS * line;
    }
    m0 += SR_F32_KS;
    if (m0 >= e.M) {
      m0 = 0;
      ++fi;
      fresh = along;
    }
  }

  __device__ __forceinline__ void enter(SR_CONST4(SrGradEdge) ek, const SrTensor* tensors, int ring_, int i0, int j0_) {
    e.x = ek->x; e.dy = ek->dy; e.lag = ek->lag; e.frame0 = ek->frame0;
    e.H = ek->H; e.W = ek->W; e.Cin = ek->Cin; e.Ho = ek->Ho; e.Wo = ek->Wo; e.Cout = ek->Cout;
    e.kw = ek->kw; e.stride = ek->stride; e.pad = ek->pad; e.I = ek->I; e.M = ek->M;
    e.d_cin = sr_load_div(&ek->d_cin); e.d_kw = sr_load_div(&ek->d_kw); e.d_wo = sr_load_div(&ek->d_wo);
    e.d_howo = sr_load_div(&ek->d_howo); e.d_up = sr_load_div(&ek->d_up); e.d_steps = sr_load_div(&ek->d_steps);
    e.steps_per_frame = ek->steps_per_frame;
    SR_CONST4(SrTensor) tx = sr_k(tensors) + e.x;
    SR_CONST4(SrTensor) ty = sr_k(tensors) + e.dy;
    xb0 = (const char*)(unsigned long long)tx->base;
    yb0 = (const char*)(unsigned long long)ty->base;
    xs = tx->stride;
    ys = ty->stride;
    image = (long long)e.H * e.W * e.Cin * 4;
    quads_a = SR_UNI(ek->quads_in && (((unsigned)(unsigned long long)xb0 | (unsigned)xs | (unsigned)image) & 15u) == 0);
    quads_b = SR_UNI(ek->quads_out && (((unsigned)(unsigned long long)yb0 | (unsigned)ys) & 15u) == 0);
    ring = ring_;
    j0 = j0_;
    const int i = quads_a ? i0 + 4 * (lane % (TI / 4)) : i0 + (TI == 128 ? (wv & 1) * 64 + lane : lane);
    const int tap = sr_divide(i, e.d_cin), ci = i - tap * e.Cin;
    ti = sr_divide(tap, e.d_kw);
    tj = tap - ti * e.kw;
    aoff = (uint32_t)(ti * e.W + tj) * (uint32_t)e.Cin + (uint32_t)ci;
    if (i >= e.I) ti = SR_NO_TAP;
    along = ek->along;
  }

  __device__ __forceinline__ void issue(int step, unsigned at) {
    const char* zero = (const char*)sr_zero_line;
    const int fi = sr_divide(step, e.d_steps), m0 = (step - fi * e.steps_per_frame) * SR_F32_KS;
    const int frame = e.frame0 + fi;
    const int b0 = sr_divide(m0, e.d_howo);
    const char* xb = xb0 + (frame - e.lag) * xs + b0 * image;
    const char* yb = yb0 + (frame % ring) * ys + (long long)m0 * e.Cout * 4;
    if (quads_a) {
#pragma unroll
      for (int n = 0; n < NA; ++n) {
        const SrPixAt p = sr_pix_at(e, m0 + (n * 4 + wv) * (256 / TI) + lane / (TI / 4));
        sr_to_lds16(sr_pix_ok(e, p, ti, tj) ? sr_at(xb, sr_pix_off(e, p, b0, aoff)) : zero, at + (n * 4 + wv) * 1024);
      }
    } else {
#pragma unroll
      for (int q = 0; q < TI / 16; ++q) {
        const int id = q * 4 + wv;
        const SrPixAt p = sr_pix_at(e, SR_UNI(m0 + id * 64 / TI));
        sr_to_lds4(sr_pix_ok(e, p, ti, tj) ? sr_at(xb, sr_pix_off(e, p, b0, aoff)) : zero, at + id * 256);
      }
    }
    const unsigned bt = at + TI * 64;
    if (quads_b) {
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int id = HALF_B ? wv * 32 + lane : (n * 4 + wv) * 64 + lane;
        const int k = id / (TJ / 4), j = j0 + 4 * (id % (TJ / 4));
        const char* p = (m0 + k < e.M && j < e.Cout) ? sr_at(yb, (uint32_t)k * (uint32_t)e.Cout + (uint32_t)j) : zero;
        if (HALF_B) {
          if (lane < 32) sr_to_lds16(p, bt + wv * 512);
        } else {
          sr_to_lds16(p, bt + (n * 4 + wv) * 1024);
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < TJ / 16; ++q) {
        const int id = (q * 4 + wv) * 64 + lane;
        const int k = id / TJ, j = j0 + id % TJ;
        sr_to_lds4((m0 + k < e.M && j < e.Cout) ? sr_at(yb, (uint32_t)k * (uint32_t)e.Cout + (uint32_t)j) : zero, bt + (q * 4 + wv) * 256);
      }
    }
  }
};

// Weight gradient: rows i = (tap, source channel), columns j = target channel, reduction over the pixels of the
// edge's frames, 16 pixels of one frame per step.  The sum over a tile's steps is taken in blocks of 128 steps, so that
// it stays as accurate as the sums of short slices that a second pass would add up.
template <int TI, int TJ, int WJN>
__device__ __forceinline__ void sr_grad_tile(const SrGradArgs& A, SR_CONST4(SrGradEdge) ek, int i0, int j0, int step_begin, int step_end,
                                             int slice, unsigned char* lds) {
  constexpr int WIN = 4 / WJN, MI = TI / (32 * WIN), MJ = TJ / (32 * WJN);
  constexpr int STAGES = TI * TJ == 4096 ? 4 : 3;   // 64 x 64 and 128 x 32 tiles: a step is 512 cycles of products, so three on the way
  typedef SrGradOperands<TI, TJ> Ops;
  const int tid = threadIdx.x, lane = tid & 63, wv = SR_UNI(tid >> 6);
  const unsigned at0 = sr_lds_at(lds);
  Ops op;
  op.wv = wv;
  op.lane = lane;
  op.enter(ek, A.tensors, A.ring, i0, j0);

  f32x16_t acc[MI][MJ], sum[MI][MJ];
#pragma unroll
  for (int x = 0; x < MI; ++x)
#pragma unroll
    for (int y = 0; y < MJ; ++y)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[x][y][v] = sum[x][y][v] = 0.f;
  const int iw = (wv / WJN) * 32 * MI, jw = (wv % WJN) * 32 * MJ;
  int wr = 0, rd = 0, next = step_begin;
  op.begin(step_begin);
#pragma nounroll
  for (int k = 0; k < STAGES - 1 && next < step_end; ++k, ++next) {
    op.issue_next(at0 + wr * Ops::STAGE);
    wr = wr == STAGES - 1 ? 0 : wr + 1;
  }
  for (int s = step_begin; s < step_end;) {
    const int block_end = min(s + 128, step_end);
    for (; s < block_end; ++s) {
      if (STAGES > 3 && s + 2 < step_end) sr_wait_loads<2 * Ops::LOADS>();
      else if (s + 1 < step_end) sr_wait_loads<Ops::LOADS>();
      else sr_wait_loads<0>();
      sr_step_barrier();
      if (next < step_end) {
        ++next;
        op.issue_next(at0 + wr * Ops::STAGE);
        wr = wr == STAGES - 1 ? 0 : wr + 1;
      }
      sr_step_products<TI, TJ, MI, MJ>(lds + rd * Ops::STAGE, iw, jw, lane, false, false, acc);
      rd = rd == STAGES - 1 ? 0 : rd + 1;
    }
    // (a loop of its own: a fold that a step may or may not do costs it a move per accumulator)
#pragma unroll
    for (int x = 0; x < MI; ++x)
#pragma unroll
      for (int y = 0; y < MJ; ++y)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          sum[x][y][v] += acc[x][y][v];
          acc[x][y][v] = 0.f;
        }
  }
  const int slices = ek->slices;
  const int I = op.e.I, J = op.e.Cout;
  float* out = slices == 1 ? A.dst[ek->dst] : A.part + ek->part_at + (size_t)slice * I * J;
  const bool add = slices == 1 && A.accumulate;
#pragma unroll
  for (int x = 0; x < MI; ++x)
#pragma unroll
    for (int y = 0; y < MJ; ++y)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = i0 + iw + x * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3), j = j0 + jw + y * 32 + (lane & 31);
        if (i < I && j < J) {
          float* d = out + (size_t)i * J + j;
          const float r = sum[x][y][v];
          *d = add ? *d + r : r;
        }
      }
}

// Column sums of a gradient tensor over a range of rows (frame, pixel): 64 channels, four row lanes per channel (each
// adds every fourth row in order, eight loads in flight, then the four in order)
__device__ __forceinline__ void sr_grad_bias(const SrGradArgs& A, SR_CONST4(SrGradBias) bk, int j0, int row_begin, int row_end, int slice,
                                             float* lds) {
  const int C = bk->C, M = bk->M, frame0 = bk->frame0;
  const SrDiv d_m = sr_load_div(&bk->d_m);
  SR_CONST4(SrTensor) t = sr_k(A.tensors) + bk->dy;
  const char* base = (const char*)(unsigned long long)t->base;
  const long long stride = t->stride;
  const int c = j0 + (threadIdx.x & 63), rl = threadIdx.x >> 6;
  float acc = 0.f;
  if (c < C)
    for (int r = row_begin + rl; r < row_end; r += 32) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int q = min(r + 4 * u, row_end - 1);
        const int fi = sr_divide(q, d_m), m = q - fi * M;
        v[u] = *(const float*)(base + ((frame0 + fi) % A.ring) * stride + ((size_t)m * C + c) * 4);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += r + 4 * u < row_end ? v[u] : 0.f;
    }
  lds[rl * 64 + (threadIdx.x & 63)] = acc;
  __syncthreads();
  if (rl == 0 && c < C)
    A.part[bk->part_at + (size_t)slice * C + c] =
        ((lds[threadIdx.x] + lds[64 + threadIdx.x]) + lds[128 + threadIdx.x]) + lds[192 + threadIdx.x];
}

}  // namespace

// (WIDE: 168 registers, four spilled, and three workgroups per CU; two with 172.  All variants together took the GTSRB-shaped
// window from 6270 to 6150 us.)
template <int VARIANT>
__global__ __launch_bounds__(256, VARIANT == SR_F32_NARROW ? 4 : 3) void sr_grad_kernel(SrGradArgs A) {
  extern __shared__ __align__(1024) unsigned char sr_rows_lds[];
  SR_CONST4(SrGradTile) t = sr_k(A.tiles) + blockIdx.x;
  const int kind = t->kind, shape = t->shape, i0 = t->i0, j0 = t->j0, sb = t->step_begin, se = t->step_end, slice = t->slice;
  if (kind == 2) return;
  if (kind == 1) {
    sr_grad_bias(A, sr_k(A.biases) + t->edge, j0, sb, se, slice, (float*)sr_rows_lds);
    return;
  }
  SR_CONST4(SrGradEdge) e = sr_k(A.edges) + t->edge;
  if constexpr (VARIANT == SR_F32_WIDE)
    if (shape == SR_F32_128x128) sr_grad_tile<128, 128, 2>(A, e, i0, j0, sb, se, slice, sr_rows_lds);
  if (shape == SR_F32_128x64) sr_grad_tile<128, 64, 2>(A, e, i0, j0, sb, se, slice, sr_rows_lds);
  else if (shape == SR_F32_64x64) sr_grad_tile<64, 64, 2>(A, e, i0, j0, sb, se, slice, sr_rows_lds);
  else if (shape == SR_F32_128x32) sr_grad_tile<128, 32, 1>(A, e, i0, j0, sb, se, slice, sr_rows_lds);
}

// The partial sums of gradients cut into slices, added in slice order: a workgroup takes 64 elements, four slice lanes
// per element (each adds every fourth slice in order, eight loads in flight; then the four in order).  The last
// workgroup adds up the loss.
__global__ __launch_bounds__(256) void sr_grad_sum_kernel(const SrGradSum* __restrict__ sums, int n_sums, const float* __restrict__ part,
                                                          float* const* __restrict__ dst, int accumulate, int first, int last,
                                                          const float* __restrict__ terms, long long n_terms, float scale,
                                                          float* __restrict__ loss) {
  __shared__ float lanes[256];
  const int t = threadIdx.x, block = (int)blockIdx.x + first;
  if (block == last) {
    float acc = 0.f;
    for (long long i = t; i < n_terms; i += 256) acc += terms[i];
    lanes[t] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
      if (t < s) lanes[t] += lanes[t + s];
      __syncthreads();
    }
    if (t == 0) loss[0] = lanes[0] * scale;
    return;
  }
  int k = 0;
  for (int base = 0; base < n_sums; base += 64) {
    const int q = base + (t & 63);
    const int b0 = q < n_sums ? sums[q].block0 : 0x7fffffff;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(b0 <= block);
    k += __popcll(m);
    if (m != ~0ull) break;
  }
  SR_CONST4(SrGradSum) s = sr_k(sums) + SR_UNI(k - 1);
  const long long n = s->n, e = (long long)(block - s->block0) * 64 + (t & 63);
  const int slices = s->slices, sl = t >> 6;
  const float* p = part + s->part_at;
  float acc = 0.f;
  if (e < n)
    for (int s0 = sl; s0 < slices; s0 += 32) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(size_t)min(s0 + 4 * u, slices - 1) * n + e];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += s0 + 4 * u < slices ? v[u] : 0.f;
    }
  lanes[t] = acc;
  __syncthreads();
  if (sl == 0 && e < n) {
    const float r = ((lanes[t] + lanes[64 + t]) + lanes[128 + t]) + lanes[192 + t];
    float* d = dst[s->dst];
    if (!d) return;   // a gradient the caller did not ask for
    d += e;
    *d = accumulate ? *d + r : r;
  }
}

// Softmax cross-entropy of every frame of the window (App. A2), a wave per (frame, sample): its term of the loss and
// the gradient of the scores, (softmax - [class == label]) * scale
__global__ __launch_bounds__(256) void sr_loss_kernel(SrLossArgs A) {
  const int lane = threadIdx.x & 63, idx = A.first + (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6);
  if (idx >= A.frames * A.B) return;   // a whole wave
  const int fi = idx / A.B, frame = A.frame0 + fi, b = idx - fi * A.B, C = A.C;
  auto at = [&](int id, int slot) -> float* {
    const SrTensor t = A.tensors[id];
    return t.base ? (float*)(t.base + slot * t.stride) + (size_t)b * C : nullptr;
  };
  const float* z = at(A.x, frame);
  float* d = at(A.out, A.gate ? frame % A.ring : frame);
  const float* mask = A.gate ? at(A.mask, frame) : nullptr;
  float zmax = -INFINITY;
  for (int c = lane; c < C; c += 64) zmax = fmaxf(zmax, z[c]);
  for (int m = 32; m > 0; m >>= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, m, 64));
  float sum = 0.f;
  for (int c = lane; c < C; c += 64) sum += expf(z[c] - zmax);
  for (int m = 32; m > 0; m >>= 1) sum += __shfl_xor(sum, m, 64);
  const float lse = zmax + logf(sum);
  int lab = A.labels[b];
  lab = lab < 0 ? 0 : (lab >= C ? C - 1 : lab);   // the host checks nothing on the device: stay in bounds
  if (lane == 0) A.terms[(size_t)(frame - 1) * A.B + b] = lse - z[lab];
  for (int c = lane; c < C; c += 64) {
    float v = (expf(z[c] - lse) - (c == lab ? 1.f : 0.f)) * A.scale;
    if (A.gate) {
      if (A.act == 1 && !(z[c] > 0.f)) v = 0.f;
      if (mask) v *= mask[c];
    }
    d[c] = v;
  }
}

__global__ void sr_patch_kernel(SrTensor* __restrict__ tensors, float** __restrict__ dst, SrPatch p) {
  for (int k = threadIdx.x; k < p.n; k += blockDim.x) {
    const int i = p.index[k];
    if (i >= 0) tensors[i] = p.value[k];
    else dst[-1 - i] = (float*)p.value[k].base;
  }
}

// channel means of a node's state at the frames frame0 .. (the mean read at frame f is that of frame f - lag), a
// workgroup per 64 channels of one image: four pixel lanes per channel, eight loads in flight
__global__ __launch_bounds__(256) void sr_pool_kernel(const SrTensor* __restrict__ tensors, SrPool q, int frame0, int image0) {
  __shared__ float lanes[256];
  const int frame = frame0 + blockIdx.z, b = image0 + blockIdx.y, t = threadIdx.x, c = blockIdx.x * 64 + (t & 63), pl = t >> 6;
  const SrTensor x = tensors[q.x], mean = tensors[q.mean];
  float acc = 0.f;
  if (c < q.C && !(q.zero0 && frame - q.lag == 0)) {
    const float* p = (const float*)(x.base + (frame - q.lag) * x.stride) + (size_t)b * q.HW * q.C + c;
    for (int i = pl; i < q.HW; i += 32) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[(size_t)min(i + 4 * u, q.HW - 1) * q.C];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += i + 4 * u < q.HW ? v[u] : 0.f;
    }
  }
  lanes[t] = acc;
  __syncthreads();
  if (pl == 0 && c < q.C)
    ((float*)(mean.base + frame * mean.stride))[(size_t)b * q.C + c] =
        (((lanes[t] + lanes[64 + t]) + lanes[128 + t]) + lanes[192 + t]) / (float)q.HW;
}

// RMSprop of many parameters in one launch: a <- rho a + (1 - rho) g^2;  theta <- theta - lr g / (sqrt(a) + eps)
__global__ __launch_bounds__(256) void sr_rmsprop_kernel(SrRmsBatch b, float lr, float rho, float eps) {
  int k = 0;
  while (k + 1 < b.count && (int)blockIdx.x >= b.block0[k + 1]) ++k;
  const long long i = (long long)(blockIdx.x - b.block0[k]) * 256 + threadIdx.x;
  if (i >= b.n[k]) return;
  const float gi = b.grad[k][i];
  const float ai = rho * b.mean[k][i] + (1.f - rho) * gi * gi;
  b.mean[k][i] = ai;
  b.theta[k][i] -= lr * gi / (sqrtf(ai) + eps);
}

hipError_t sr_launch_rows_train(hipStream_t s, const SrRowArgs& a, int backward, int shapes) {
  if (a.n_tiles == 0) return hipSuccess;
  if (!backward && sr_f32_variant(shapes) == SR_F32_WIDE) return hipErrorInvalidValue;   // not planned: see sr_rows_tiles
  static void (*const kernels[2][3])(SrRowArgs) = {
      {nullptr, sr_rows_train_kernel<false, SR_F32_NARROW>, sr_rows_train_kernel<false, SR_F32_DEEP>},
      {sr_rows_train_kernel<true, SR_F32_WIDE>, sr_rows_train_kernel<true, SR_F32_NARROW>, sr_rows_train_kernel<true, SR_F32_DEEP>}};
  SrRowArgs piece = a;
  for (piece.first = 0; piece.first < a.n_tiles; piece.first += SR_F32_PIECE) {
    hipLaunchKernelGGL(kernels[backward ? 1 : 0][sr_f32_variant(shapes)], dim3(std::min(SR_F32_PIECE, a.n_tiles - piece.first)), dim3(256),
                       sr_f32_lds_bytes(shapes), s, piece);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t sr_launch_grad(hipStream_t s, const SrGradArgs& a, int shapes) {
  if (a.n_tiles == 0) return hipSuccess;
  const int lds = sr_f32_lds_bytes(shapes);
  const auto kernel = sr_f32_variant(shapes) == SR_F32_WIDE ? sr_grad_kernel<SR_F32_WIDE> : sr_grad_kernel<SR_F32_NARROW>;
  hipLaunchKernelGGL(kernel, dim3(a.n_tiles), dim3(256), lds > 1024 ? lds : 1024 /* column sums */, s, a);
  return hipGetLastError();
}

hipError_t sr_launch_grad_sum(hipStream_t s, const SrGradSum* sums, int n_sums, int n_blocks, const float* part, float* const* dst,
                              int accumulate, const float* terms, long long n_terms, float scale, float* loss) {
  const int blocks = n_blocks + (loss ? 1 : 0);   // the last one adds up the loss
  for (int first = 0; first < blocks; first += SR_F32_PIECE) {
    hipLaunchKernelGGL(sr_grad_sum_kernel, dim3(std::min(SR_F32_PIECE, blocks - first)), dim3(256), 0, s, sums, n_sums, part, dst, accumulate, first,
                       n_blocks, terms, n_terms, scale, loss);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t sr_launch_loss(hipStream_t s, const SrLossArgs& a) {
  SrLossArgs piece = a;
  const long long n = (long long)a.frames * a.B;   // below 2^31
  for (long long first = 0; first < n; first += 4ll * SR_F32_PIECE) {
    piece.first = (int)first;
    hipLaunchKernelGGL(sr_loss_kernel, dim3((unsigned)((std::min(n - first, 4ll * SR_F32_PIECE) + 3) / 4)), dim3(256), 0, s, piece);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t sr_launch_patch(hipStream_t s, SrTensor* tensors, float** dst, const SrPatch& p) {
  if (p.n == 0) return hipSuccess;
  hipLaunchKernelGGL(sr_patch_kernel, dim3(1), dim3(64), 0, s, tensors, dst, p);
  return hipGetLastError();
}

hipError_t sr_launch_pool(hipStream_t s, const SrTensor* tensors, const SrPool& p, int B, int frame0, int frames) {
  // images and frames as grid rows, some thousands at a time (grid y and z are limited to 65535)
  for (int f = 0; f < frames; f += 4096)
    for (int b = 0; b < B; b += 32768) {
      hipLaunchKernelGGL(sr_pool_kernel, dim3((p.C + 63) / 64, B - b < 32768 ? B - b : 32768, frames - f < 4096 ? frames - f : 4096), dim3(256),
                         0, s, tensors, p, frame0 + f, b);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

hipError_t sr_launch_rmsprop(hipStream_t s, const SrRmsBatch& b, float lr, float rho, float eps) {
  if (b.count == 0 || b.block0[b.count] == 0) return hipSuccess;
  hipLaunchKernelGGL(sr_rmsprop_kernel, dim3(b.block0[b.count]), dim3(256), 0, s, b, lr, rho, eps);
  return hipGetLastError();
}
