// Device code shared by the kernel files: bf16 conversion, agent-scope accesses, dependency waits, the end of a
// frame, and the auxiliary work items (input staging, dense / GAP+dense heads) that ride along in a level's launch.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>
#include "sr_internal.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4_t;

// ---------------------------------------------------------------------------
// bfloat16 <-> float (round to nearest even)
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf16_bits_to_float(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

template <typename T> struct Store;
#define SR_GLOBAL __attribute__((address_space(1)))
// load / store: ordinary accesses.  aload / astore: agent-scope accesses (a store goes through to
// memory, a load does not take a stale line from this XCD's L2) for node states, which in a
// dependency-driven launch are produced and consumed by workgroups on different XCDs.
template <> struct Store<float> {
  static __device__ __forceinline__ float aload(const float* p) {
    return __uint_as_float(__hip_atomic_load((const unsigned*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  }
  static __device__ __forceinline__ void astore(float* p, float v) {
    __hip_atomic_store((unsigned*)p, __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  static __device__ __forceinline__ float load(const float* p) { return *p; }
  static __device__ __forceinline__ float gload(const SR_GLOBAL float* p) { return *p; }
  static __device__ __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Store<uint16_t> {
  static __device__ __forceinline__ float aload(const uint16_t* p) {
    return bf16_bits_to_float(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
  }
  static __device__ __forceinline__ void astore(uint16_t* p, float v) {
    __hip_atomic_store(p, float_to_bf16_bits(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  static __device__ __forceinline__ float load(const uint16_t* p) { return bf16_bits_to_float(*p); }
  static __device__ __forceinline__ float gload(const SR_GLOBAL uint16_t* p) { return bf16_bits_to_float(*p); }
  static __device__ __forceinline__ void store(uint16_t* p, float v) { *p = float_to_bf16_bits(v); }
};

// The call's values (see SrFrame): in the launch's own arguments, of which the SrFrame is the first, or in memory.
// Read with scalar loads; constant while the launch runs (the last workgroup advances the frame counter when all others
// have read it).
typedef const __attribute__((address_space(4))) SrCtx* sr_call_t;
// A plain launch, which does not read the counter in memory, puts it right here (at its end, the values that this needs cost
// the tile kernel registers: CIFAR-shaped frames 28.3 -> 32 us).
__device__ __forceinline__ sr_call_t sr_call(const SrFrame& f) {
  if (f.advance < 0 && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) f.ctx->frame = f.here.frame - f.advance;
  return f.plain ? (sr_call_t)__builtin_amdgcn_kernarg_segment_ptr() : (sr_call_t)(unsigned long long)f.ctx;
}

// Called by every workgroup of a launch once its work is stored.  If the launch advances the frame counter, the
// workgroup that arrives last does so (all others have read it long before).
__device__ __forceinline__ void sr_block_done(const SrFrame& f, int n_blocks) {
  // no fence: the counter only orders "everyone has read the frame counter" (done at kernel start)
  // before its update, and the next launch sees the update through the kernel boundary
  if (f.advance <= 0) return;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int old = __hip_atomic_fetch_add(&f.ctx->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old == n_blocks - 1) {
      f.ctx->done = 0;
      f.ctx->frame = f.ctx->frame + f.advance;
    }
  }
}

// Dependency-driven launches: wait until every node this work item depends on has completed the
// frames it needs.  The first wave polls, one dependency per lane, sleeping between polls; the other
// waves wait at the barrier.  Counters wrap, so they are compared by signed difference.  The wait is
// bounded: past the spin limit it gives up and reports itself (results are then undefined, the
// launch still ends).
struct SrDepPoll {   // a dependency wait whose first poll is in flight
  const int* counter;
  int need, first, count;
};

// first poll goes out (the caller has other things to do before it needs the answer)
__device__ __forceinline__ SrDepPoll sr_deps_begin(const SrFlow& flow, int begin, int count, int frame) {
  SrDepPoll w;
  w.counter = flow.done;
  w.need = 0;
  w.first = 0;
  w.count = (flow.deps == nullptr) ? 0 : count;
  if (w.count > 0 && threadIdx.x < (unsigned)w.count) {
    const SrDep d = flow.deps[begin + threadIdx.x];
    w.counter = flow.done + d.node * SR_DONE_STRIDE;
    w.need = d.units * (frame - d.lag);
    w.first = __hip_atomic_load(w.counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  return w;
}

// ... and the wait itself
__device__ __forceinline__ void sr_deps_finish(const SrFlow& flow, const SrDepPoll& w, SrCtx* ctx) {
  if (w.count == 0) return;
  if (threadIdx.x < 64) {
    const int lane = threadIdx.x;
    int seen = w.first;
    int spins = 0;
    for (;;) {
      const int ok = (lane >= w.count) || (seen - w.need) >= 0;
      if (__builtin_amdgcn_ballot_w64(!ok) == 0) break;
      // give up at the spin limit -- or at once if any wait of this graph has given up before, so that
      // a broken dependency costs one limit, not one per work item
      int failed = 0;
      if ((spins & 63) == 63) failed = __hip_atomic_load(&ctx->dep_timeouts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (++spins > flow.spin_limit || failed > 0) {
        if (lane == 0) __hip_atomic_fetch_add(&ctx->dep_timeouts, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      // back off: the counters are shared by every waiting workgroup of the chip
      if (spins < 16) __builtin_amdgcn_s_sleep(8);
      else if (spins < 64) __builtin_amdgcn_s_sleep(32);
      else __builtin_amdgcn_s_sleep(127);
      if (lane < w.count) seen = __hip_atomic_load(w.counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
}

__device__ __forceinline__ void sr_wait_deps(const SrFlow& flow, int begin, int count, int frame, SrCtx* ctx) {
  const SrDepPoll w = sr_deps_begin(flow, begin, count, frame);
  sr_deps_finish(flow, w, ctx);
}

// ... and tell the dependants: this work item's results are in memory (its stores were agent-scope
// and have completed when each thread's wait for them ends; the barrier collects the workgroup's).
__device__ __forceinline__ void sr_signal_done(const SrFlow& flow, int gnode) {
  if (flow.deps == nullptr) return;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_fetch_add(flow.done + gnode * SR_DONE_STRIDE, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 16-byte agent-scope store of node-state data (see Store<T>::astore)
__device__ __forceinline__ void sr_store16_agent(void* p, u32x4_t v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1" ::"v"((__attribute__((address_space(1))) u32x4_t*)(unsigned long long)p), "v"(v) : "memory");
}

// ---------------------------------------------------------------------------
// auxiliary work items that ride along in a level's launch
// ---------------------------------------------------------------------------
// input staging: state[frame & 1] of an input node := this frame's input, channel pitch C -> Cp;
// one item covers SR_STAGE_CHUNK pixels, one pixel per thread and pass, 16-byte stores when the
// stored pixel is a whole number of them
// `ahead` = 1 stages the NEXT frame's input (into the copy that frame will be read from) while the
// current frame's last launch runs: a pattern whose input edges do not bridge needs frame t's input
// in place before frame t's first launch.  Frames the caller has given no input for are skipped
// (the item still counts as completed for its dependants).
template <typename T>
__device__ __forceinline__ void sr_stage_item(SrCtx* __restrict__ ctx, sr_call_t call, const SrStageNode& nd, int chunk, int ahead,
                                              int frame_now, const SrFlow& flow) {
  const int frame = frame_now + ahead;
  const char* base = (const char*)(unsigned long long)call->in_ptr[nd.input_slot];
  // the copy written was last read two frames ago (one frame ago, by bridging edges): wait for those readers
  sr_wait_deps(flow, nd.dep_begin, nd.dep_count, frame, ctx);
  if (base != nullptr && frame <= call->in_last) {
    const T* in = (const T*)(base + (int64_t)(frame - call->in_base) * call->in_stride[nd.input_slot]);
    T* out = (T*)nd.state[frame & 1];
    const int end = min(nd.elems_px, (chunk + 1) * SR_STAGE_CHUNK);
    constexpr int V = 16 / sizeof(T);
    if ((nd.Cp == V || nd.Cp == 2 * V) && nd.C <= V && SR_AUX_THREADS * 4 == SR_STAGE_CHUNK) {
      // few channels (an image): one 16-byte piece of data per pixel (and one of zeros if the pitch is two),
      // four pixels per thread, all loads first
      const int p0 = chunk * SR_STAGE_CHUNK + threadIdx.x;
      T v[4][V];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int p = min(p0 + j * SR_AUX_THREADS, nd.elems_px - 1);
        const T* ip = in + (size_t)p * nd.C;
#pragma unroll
        for (int i = 0; i < V; ++i) v[j][i] = (i < nd.C) ? ip[i] : (T)0;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int p = p0 + j * SR_AUX_THREADS;
        if (p < end) {
          sr_store16_agent(out + (size_t)p * nd.Cp, *(const u32x4_t*)v[j]);
          if (nd.Cp == 2 * V) sr_store16_agent(out + (size_t)p * nd.Cp + V, u32x4_t{0u, 0u, 0u, 0u});
        }
      }
    } else if ((nd.Cp % V) == 0) {
      for (int p = chunk * SR_STAGE_CHUNK + threadIdx.x; p < end; p += SR_AUX_THREADS) {
        const T* ip = in + (size_t)p * nd.C;
        for (int c0 = 0; c0 < nd.Cp; c0 += V) {
          T v[V];
#pragma unroll
          for (int i = 0; i < V; ++i) v[i] = (c0 + i < nd.C) ? ip[c0 + i] : (T)0;
          sr_store16_agent(out + (size_t)p * nd.Cp + c0, *(const u32x4_t*)v);
        }
      }
    } else {
      for (int p = chunk * SR_STAGE_CHUNK + threadIdx.x; p < end; p += SR_AUX_THREADS)
        for (int c = 0; c < nd.Cp; ++c)
          Store<T>::astore(out + (size_t)p * nd.Cp + c, (c < nd.C) ? Store<T>::load(in + (size_t)p * nd.C + c) : 0.f);
    }
  }
  sr_signal_done(flow, nd.gnode);
}

// Head node (App. A2: fully connected layers, optionally after global average pooling): a 1x1 node
// whose incoming edges are all dense or GAP+dense.  One item per image (and, for a single pooled
// edge over many pixels, per pixel slab: the slab sums go to `partial` and the item that finishes
// last for an image adds them in slab order).  For every edge the input vector (pooled means or the
// flattened source) is put into LDS, then each of the 4 waves multiplies a quarter of it into up to
// 256 outputs (with at most 64 outputs: 256 / CO slices of it into CO = 16, 32 or 64 output columns);
// the parts are added in a fixed order, then bias, activation, store and, if this node is being
// recorded, the rollout output.  smem: SR_HEAD_MAX_K floats, one int, 4*64*4 floats.
template <typename T>
__device__ __forceinline__ bool sr_head_body(sr_call_t call, const SrHead& h,
                                             const SrHeadEdge* __restrict__ head_edges, int b, int split,
                                             float* smem, int vec_floats, int frame) {
  const int cur = frame & 1;
  int* flag = (int*)(smem + vec_floats);
  float* red = smem + vec_floats + 4;
  const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
  float acc[4] = {0.f, 0.f, 0.f, 0.f};     // outputs lane, lane+64, lane+128, lane+192: this wave's share
  // up to 64 outputs: CO = 16, 32 or 64 output columns, 256 / CO slices of the input vector
  const bool narrow = h.Cout <= 64;
  const int CO = h.Cout <= 16 ? 16 : (h.Cout <= 32 ? 32 : 64);
  const int n_slices = 256 / CO;
  const int co_n = threadIdx.x & (CO - 1), slice = threadIdx.x / CO;
  for (int ei = 0; ei < h.edge_count; ++ei) {
    const SrHeadEdge e = head_edges[h.edge_begin + ei];
    const T* src = (const T*)((e.bridge ? (cur ^ 1) : cur) ? e.src[1] : e.src[0]) + (size_t)b * e.HW * e.Csp;
    int K;
    __syncthreads();   // the previous edge's vector is no longer needed
    if (e.pooled) {
      K = e.Cin;
      const int per = (e.HW + h.splits - 1) / h.splits;
      const int p0 = split * per, p1 = min(e.HW, p0 + per);
      const float inv = 1.0f / (float)e.HW;
      for (int c = threadIdx.x; c < e.Cin; c += SR_AUX_THREADS) {
        float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
        int p = p0;
        for (; p + 12 <= p1; p += 12) {   // twelve loads in flight
          float v[12];
#pragma unroll
          for (int u = 0; u < 12; ++u) v[u] = Store<T>::aload(src + (size_t)(p + u) * e.Csp + c);
          s0 += (v[0] + v[4]) + v[8];
          s1 += (v[1] + v[5]) + v[9];
          s2 += (v[2] + v[6]) + v[10];
          s3 += (v[3] + v[7]) + v[11];
        }
        for (; p + 4 <= p1; p += 4) {
          s0 += Store<T>::aload(src + (size_t)p * e.Csp + c);
          s1 += Store<T>::aload(src + (size_t)(p + 1) * e.Csp + c);
          s2 += Store<T>::aload(src + (size_t)(p + 2) * e.Csp + c);
          s3 += Store<T>::aload(src + (size_t)(p + 3) * e.Csp + c);
        }
        for (; p < p1; ++p) s0 += Store<T>::aload(src + (size_t)p * e.Csp + c);
        const float sum = (s0 + s1) + (s2 + s3);
        if (h.splits == 1) smem[c] = sum * inv;
        else   // device-coherent (write-through) store, read back below by whichever slab finishes last
          __hip_atomic_store(&h.partial[((size_t)b * h.splits + split) * e.Cin + c], sum, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      }
      if (h.splits > 1) {   // only single-edge heads are cut into slabs
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) {
          const int old = __hip_atomic_fetch_add(&h.counters[b], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          *flag = (old == h.splits - 1);
          // an agent-scope store: a launch may cover several frames, whose slabs count on from here on other XCDs
          if (old == h.splits - 1) __hip_atomic_store(&h.counters[b], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (!*flag) return false;
        for (int c = threadIdx.x; c < e.Cin; c += SR_AUX_THREADS) {
          float sum = 0.f;
          for (int s = 0; s < h.splits; ++s)
            sum += __hip_atomic_load(&h.partial[((size_t)b * h.splits + s) * e.Cin + c], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
          smem[c] = sum * inv;
        }
      }
    } else {
      K = e.HW * e.Cin;
      for (int k = threadIdx.x; k < K; k += SR_AUX_THREADS) {
        const int p = k / e.Cin, c = k - p * e.Cin;
        smem[k] = Store<T>::aload(src + (size_t)p * e.Csp + c);
      }
    }
    __syncthreads();
    if (narrow) {
      // few outputs: the threads are arranged (slice of the vector) x (output)
      const int kper = (K + n_slices - 1) / n_slices;
      const int k_lo = slice * kper, k_hi = min(K, k_lo + kper);
      if (co_n < h.Cout) {
        // sixteen independent chains keep sixteen weight loads in flight
        float a[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) a[u] = 0.f;
        int k = k_lo;
        for (; k + 16 <= k_hi; k += 16) {
          float wv[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) wv[u] = e.w[(size_t)(k + u) * h.Cout + co_n];
#pragma unroll
          for (int u = 0; u < 16; ++u) a[u] += smem[k + u] * wv[u];
        }
        for (; k < k_hi; ++k) a[0] += smem[k] * e.w[(size_t)k * h.Cout + co_n];
        const float a0 = (a[0] + a[1]) + (a[2] + a[3]), a1 = (a[4] + a[5]) + (a[6] + a[7]);
        const float a2 = (a[8] + a[9]) + (a[10] + a[11]), a3 = (a[12] + a[13]) + (a[14] + a[15]);
        acc[0] += (a0 + a1) + (a2 + a3);
      }
    } else {
      const int kper = (K + 3) / 4;
      const int k_lo = part * kper, k_hi = min(K, k_lo + kper);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int co = lane + 64 * j;
        if (co < h.Cout) {
          float p8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};   // eight weight loads in flight
          int k = k_lo;
          for (; k + 8 <= k_hi; k += 8) {
            float wv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) wv[u] = e.w[(size_t)(k + u) * h.Cout + co];
#pragma unroll
            for (int u = 0; u < 8; ++u) p8[u] += smem[k + u] * wv[u];
          }
          for (; k < k_hi; ++k) p8[0] += smem[k] * e.w[(size_t)k * h.Cout + co];
          acc[j] += ((p8[0] + p8[1]) + (p8[2] + p8[3])) + ((p8[4] + p8[5]) + (p8[6] + p8[7]));
        }
      }
    }
  }
  char* rec = h.record ? (char*)(unsigned long long)call->out_ptr : nullptr;
  T* recp = rec ? (T*)(rec + (int64_t)(frame - call->out_base) * call->out_stride) : nullptr;
  if (narrow) {
    red[slice * CO + co_n] = acc[0];
    __syncthreads();
    for (int co = threadIdx.x; co < h.Cout; co += SR_AUX_THREADS) {
      float v = 0.f;
      for (int sl = 0; sl < n_slices; ++sl) v += red[sl * CO + co];   // slice order: deterministic
      v += h.bias[co];
      if (h.act == 1) v = fmaxf(v, 0.f);
      Store<T>::astore((T*)h.out[cur] + (size_t)b * h.Cp + co, v);
      if (recp) Store<T>::store(recp + (size_t)b * h.Cout + co, v);
    }
    return true;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) red[(part * 4 + j) * 64 + lane] = acc[j];
  __syncthreads();
  for (int co = threadIdx.x; co < h.Cout; co += SR_AUX_THREADS) {
    const int j = co >> 6, l = co & 63;
    float v = h.bias[co] + ((red[(0 * 4 + j) * 64 + l] + red[(1 * 4 + j) * 64 + l]) +
                            (red[(2 * 4 + j) * 64 + l] + red[(3 * 4 + j) * 64 + l]));
    if (h.act == 1) v = fmaxf(v, 0.f);
    Store<T>::astore((T*)h.out[cur] + (size_t)b * h.Cp + co, v);
    if (recp) Store<T>::store(recp + (size_t)b * h.Cout + co, v);
  }
  return true;
}

// ... as a work item: wait for the source nodes (and for the readers of the copy about to be
// overwritten), compute, and count the image as done once its outputs are in memory
template <typename T>
__device__ __forceinline__ void sr_head_item(SrCtx* __restrict__ ctx, sr_call_t call, const SrHead& h,
                                             const SrHeadEdge* __restrict__ head_edges, int b, int split,
                                             float* smem, int vec_floats, int frame, const SrFlow& flow) {
  sr_wait_deps(flow, h.dep_begin, h.dep_count, frame, ctx);
  const bool wrote = sr_head_body<T>(call, h, head_edges, b, split, smem, vec_floats, frame);
  if (wrote) sr_signal_done(flow, h.gnode);
}


template <typename T>
__device__ __forceinline__ void sr_aux_item(SrCtx* __restrict__ ctx, sr_call_t call, const SrAux& it,
                                            const SrHead* __restrict__ heads,
                                            const SrHeadEdge* __restrict__ head_edges,
                                            const SrStageNode* __restrict__ stage_nodes, float* smem, int vec_floats,
                                            int frame, const SrFlow& flow) {
  if (it.kind == SR_AUX_HEAD) sr_head_item<T>(ctx, call, heads[it.a], head_edges, it.b, it.c, smem, vec_floats, frame, flow);
  else if (it.kind == SR_AUX_STAGE) sr_stage_item<T>(ctx, call, stage_nodes[it.a], it.b, it.c, frame, flow);
}
