// Backward pass of the shortest-path costs with respect to edge weights.
//
// With cost_i[x] the weight sum along the pred-tree path from instance i's
// source to x, L = sum_i sum_x g_i[x] * cost_i[x] has
//   dL/dw[e] = sum_i [e == pred_i[head(e)]] * acc_i[head(e)],
//   acc_i[y] = g_i[y] + sum over tree children c of y of acc_i[c].
// The children of y are the heads of y's out-edges e with pred[head(e)] == e,
// added in edge order, and the instances of a graph are summed in instance
// order, so every sum has a fixed order and the result is deterministic.
//
// The source of an instance is the root of its tree whatever its pred entry
// says: it is never taken as a child, and no edge into it gets a gradient.
// Only vertices whose parents lead to the root contribute (a pred array that
// the solver did not write may hold parent cycles and stray trees).
//
// There are no levels and no barriers.  A vertex's sum is complete when its
// last child's is, so every leaf starts a walk towards the root and each
// vertex is carried on by the child that arrives last; the work is one walk
// over the tree, in whatever order its parts are ready, and only the deepest
// path is serial.  A level list with a barrier per level spends most of its
// time in the barriers (a 512 x 512 grid has 1000 levels of 260 vertices):
// whole pass of 16 trees of 30011 vertices 1.05 -> 0.20 ms, 64 of 512 x 512
// 4.33 -> 2.1, a skewed tree of 2^18 vertices 26.9 -> 0.7, 64 of 150001 7.1 ->
// 1.5.  What bounds it now: the latency of each iteration's dependent accesses
// (returning atomics, performed on the memory side: 4 M in the grid case) times
// the iterations, and for few deep trees the deepest path, about 1200 cycles a
// vertex.
#include "sssp_dev.h"
#include "sssp_kernels.h"
#include "team.h"

namespace sssp {

constexpr int BBS = kBackBlock;
constexpr int kBackIn = 8;      // in-edges of a vertex held in registers
// instances per block of the parent pass (16 on 30011 vertices: 2, 4, 8 take 29,
// 31, 38 us; 64 on 512 x 512: 181, 174, 174)
constexpr int kBackChunk = 4;
constexpr int kGradAhead = 8;   // instances whose entries the gradient pass reads together
constexpr int kBackScan = 16;   // out-edges one lane looks through by itself
constexpr int kWalkBlocks = 2048;  // of the walk: every wave slot of the chip

// BackArgs::ctl: a flag, and the number of vertices walked in kBackSums parts
// (then the XCDs' words and the instance queue)
constexpr int kBackSums = kBackCtl / kBackStride - 10;
constexpr int kSweep = 64;    // vertices a wave starts from at a time
constexpr int kClaim = 64;    // the same, where an XCD's waves share an instance

// BackArgs::par of a vertex without a parent
enum : int32_t {
  kNoParent = -1,     // not the source: its subtree counts for nothing
  kUnderRoot = -2,    // a child of the source (whose own sum nobody needs)
  kRoot = -3,
};

__global__ __launch_bounds__(BBS) void bw_zero_kernel(BackArgs a) {
  const int64_t step = (int64_t)gridDim.x * BBS, i0 = (int64_t)blockIdx.x * BBS + threadIdx.x;
  for (int64_t i = i0; i < a.total; i += step) a.word[i] = 0ull;
  for (int64_t i = i0; i < a.total_m; i += step) a.grad_w[i] = 0.0f;
  for (int64_t i = i0; i < kBackCtl; i += step) a.ctl[i] = 0u;
}

// The graph whose vertices block b of the per-vertex passes covers.
__device__ __forceinline__ int32_t block_graph(const BackArgs &a, int32_t b) {
  int32_t lo = 0, hi = a.num_graphs;  // bbase[lo] <= b < bbase[hi]
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (a.bbase[mid] <= b) lo = mid;
    else hi = mid;
  }
  return lo;
}

// A vertex's first in-edges (id and tail); slots past the list's end hold an
// id that no entry names.
struct InEdges {
  int32_t deg, eid[kBackIn], src[kBackIn];
  __device__ __forceinline__ void load(const GraphDev &G, int32_t y, bool tails) {
    const int32_t o = G.u_in_off[y];
    deg = G.u_in_off[y + 1] - o;
#pragma unroll
    for (int q = 0; q < kBackIn; ++q) {
      eid[q] = q < deg ? G.u_in_eid[o + q] : -1;
      src[q] = tails && q < deg ? G.u_in_src[o + q] : -1;
    }
  }
};

// the tail of edge e
__device__ __forceinline__ int32_t edge_tail(const GraphDev &G, int32_t e) {
  int32_t lo = 0, hi = G.n;  // u_out_off[lo] <= e < u_out_off[hi]
  while (hi - lo > 1) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if (G.u_out_off[mid] <= e) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Each vertex's parent and, in the low half of its word, its number of
// children.  A block holds the in-edges of its vertices in registers and
// looks the entries of up to kBackChunk instances up in them.
__global__ __launch_bounds__(BBS) void bw_parent_kernel(BackArgs a) {
  for (int32_t b = blockIdx.x; b < a.blocks; b += gridDim.x) {
    const int32_t g = block_graph(a, b);
    const GraphDev &G = a.graphs[g];
    const int32_t y = (b - a.bbase[g]) * BBS + (int32_t)threadIdx.x;
    const int32_t j1 = a.goff[g + 1];
    int32_t j = a.goff[g] + (int32_t)blockIdx.y * kBackChunk;
    if (j >= j1 || y >= G.n) continue;
    InEdges in;
    in.load(G, y, true);
    for (; j < j1; j += (int32_t)gridDim.y * kBackChunk) {
#pragma unroll 4
      for (int32_t jj = j; jj < (j + kBackChunk < j1 ? j + kBackChunk : j1); ++jj) {
        const InstDev id = a.insts[a.ginst[jj]];
        const int32_t e = a.pred[id.sbase + y];
        int32_t t = -1;
        if (e >= 0) {
#pragma unroll
          for (int q = 0; q < kBackIn; ++q) t = in.eid[q] == e ? in.src[q] : t;
          if (in.deg > kBackIn && t < 0 && e < G.m && G.u_out_dst[e] == y) t = edge_tail(G, e);
        }
        int32_t up = id.sbase + t;
        if (y == id.source) up = kRoot;
        else if (t < 0) up = kNoParent;
        else if (t == id.source) up = kUnderRoot;
        else atomicAdd((unsigned int *)&a.word[up], 1u);
        a.par[id.sbase + y] = up;
      }
    }
  }
}

// The walk.  The word of a vertex p holds the number of its children (low
// half) and, with three or more, how many have arrived (high half).  The
// first of two children swaps its edge id and sum into the word and leaves;
// the second finds them there.  Of more children, each stores its sum, waits
// until the store is done and counts itself; the last reads the sums in edge
// order, alone or (long out-lists) with its whole wave.  An only child just
// goes on, so a chain costs one load's latency a vertex.
//
// A lane whose walk has ended takes the wave's next vertex in the same
// iteration, and its loads are the walkers' loads, so lanes stay busy beside
// a long walk.

// Vertices to start from, over the whole chip: wave wid of `waves` takes every
// waves-th chunk of [at, end).
struct SweepSource {
  static constexpr bool kOneL2 = false;
  int64_t at, end, step;
  __device__ __forceinline__ bool grab(const BackArgs &, int64_t *pos, int64_t *lim) {
    if (at >= end) return false;
    *pos = at;
    *lim = at + kSweep < end ? at + kSweep : end;
    at += step;
    return true;
  }
};

// Vertices to start from, each instance on one XCD: the XCD's word holds the
// instance it is at (plus one) and the chunks of it that are taken; the wave
// that finds the last one taken claims the next instance.
struct XcdSource {
  static constexpr bool kOneL2 = true;
  unsigned long long *cur;
  unsigned int *queue;
  __device__ __forceinline__ bool grab(const BackArgs &a, int64_t *pos, int64_t *lim) {
    unsigned long long t = 0;
    if (lane_id() == 0)
      t = __hip_atomic_fetch_add(cur, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    int32_t ins = __builtin_amdgcn_readfirstlane((int)(t >> 32)) - 1;
    int32_t c = __builtin_amdgcn_readfirstlane((int)t);
    if (ins == -2) return false;
    const int32_t chunks = ins < 0 ? 0 : (a.insts[ins].n + kClaim - 1) / kClaim;
    if (c > chunks) return true;  // another wave is claiming
    if (c == chunks) {
      unsigned int i = 0;
      if (lane_id() == 0)
        i = __hip_atomic_fetch_add(queue, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ins = __builtin_amdgcn_readfirstlane((int)i);
      const bool over = ins >= a.num_inst;
      if (lane_id() == 0)
        put64(cur, over ? 0xffffffffull << 32 : (unsigned long long)(ins + 1) << 32 | 1ull, true);
      if (over) return false;
      c = 0;
    }
    const InstDev id = a.insts[ins];
    *pos = (int64_t)id.sbase + (int64_t)c * kClaim;
    *lim = (c + 1) * (int64_t)kClaim < id.n ? *pos + kClaim : (int64_t)id.sbase + id.n;
    return true;
  }
};

// Returns the number of vertices this lane completed.
template <typename SOURCE>
__device__ __forceinline__ int32_t walk(const BackArgs &a, SOURCE source) {
  const int l = lane_id();
  int64_t pos = 0, lim = 0;
  bool more = true;
  int32_t v = 0, up = kNoParent, steps = 0;
  bool act = false;
  float acc = 0.0f;
  // the instance of the lane's last scan of an out-list (looked up for every
  // scan, the walk takes 2.0 against 1.8 ms on 64 trees of 512 x 512, 132
  // against 118 us on 16 of 30011; out-lists read ahead of the count 1.9 and 125)
  int32_t sb = 0, sn = 0, root = -1;
  const int32_t *off = nullptr, *dst = nullptr;
  for (;;) {
    // v's sum is complete: on to its parent, or to a new vertex
    if (act && up < 0) {
      a.acc[v] = acc;
      act = false;
    }
    const unsigned long long idle = __ballot(!act);
    if (pos >= lim && more && idle) more = source.grab(a, &pos, &lim);
    const int64_t at = act ? up : pos + __popcll(idle & ((1ull << l) - 1ull));
    const bool fresh = !act && at < lim;
    if (!__ballot(act || fresh)) {
      if (!more) break;
      __builtin_amdgcn_s_sleep(4);
      continue;
    }
    pos += __popcll(idle);
    bool many = false;
    if (act || fresh) {
      const int32_t p = (int32_t)at;
      const int32_t e = a.pred[act ? v : p];
      unsigned long long w = ld_relaxed64(&a.word[p]);
      const float g = a.gcost[p];
      up = a.par[p];
      if (fresh) {
        if (w == 0ull) {
          act = true;
          acc = g;
        } else if (up == kNoParent) {
          a.ctl[0] = 1u;  // a stray tree
        }
      } else if ((long long)w < 0 || (uint32_t)w <= 2u) {
        a.acc[v] = acc;
        if ((long long)w >= 0 && (uint32_t)w == 2u)
          w = __hip_atomic_exchange(&a.word[p],
                                    ((unsigned long long)(0x80000000u | (uint32_t)e) << 32) |
                                        (unsigned long long)__float_as_uint(acc),
                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((long long)w < 0) {
          const int32_t e2 = (int32_t)((uint32_t)(w >> 32) & 0x7fffffffu);
          const float s = __uint_as_float((uint32_t)w);
          acc = __fadd_rn(__fadd_rn(g, e < e2 ? acc : s), e < e2 ? s : acc);
        } else if ((uint32_t)w == 1u) {
          acc = __fadd_rn(g, acc);
        } else {
          act = false;
        }
      } else {
        put((int32_t *)&a.acc[v], __float_as_int(acc), SOURCE::kOneL2);
        stores_done();
        w = __hip_atomic_fetch_add(&a.word[p], 1ull << 32, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("" ::: "memory");  // nothing below is read before the count
        if ((uint32_t)(w >> 32) + 1u == (uint32_t)w) many = true;
        else act = false;
        acc = g;
      }
      v = p;
      if (act) ++steps;
    }
    unsigned long long left = __ballot(many);
    if (left) {
      int32_t k0 = 0, k1 = 0;
      if (many) {
        if (v < sb || v - sb >= sn) {
          int32_t lo = 0, hi = a.num_inst;  // insts[lo].sbase <= v < insts[hi].sbase
          while (hi - lo > 1) {
            const int32_t mid = (lo + hi) >> 1;
            if (a.insts[mid].sbase <= v) lo = mid;
            else hi = mid;
          }
          const InstDev id = a.insts[lo];
          sb = id.sbase;
          sn = id.n;
          root = id.source;
          off = a.graphs[id.graph].u_out_off;
          dst = a.graphs[id.graph].u_out_dst;
        }
        k0 = off[v - sb];
        k1 = off[v - sb + 1];
        if (k1 - k0 <= kBackScan) {
          // four out-edges at a time, each step's loads issued together
          // (past the list's end a lane reads edge kb again and its test
          // fails)
          for (int32_t kb = k0; kb < k1; kb += 4) {
            int32_t c[4], pr[4];
            float av[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) c[q] = dst[kb + q < k1 ? kb + q : kb];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              pr[q] = a.pred[sb + c[q]];
              av[q] = __hip_atomic_load(&a.acc[sb + c[q]], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (kb + q < k1 && c[q] != root && pr[q] == kb + q) acc = __fadd_rn(acc, av[q]);
          }
          many = false;
        }
      }
      left = __ballot(many);
      while (left) {
        const int o = __ffsll(left) - 1;
        left &= left - 1;
        const int32_t ob = __shfl(k0, o), oe = __shfl(k1, o), osb = __shfl(sb, o);
        const int32_t ort = __shfl(root, o);
        const int32_t *od = (const int32_t *)(((unsigned long long)(uint32_t)__shfl(
                                                   (int)((unsigned long long)dst >> 32), o)
                                               << 32) |
                                              (uint32_t)__shfl((int)(unsigned long long)dst, o));
        float s = __shfl(acc, o);
        int32_t c = ob + l < oe ? od[ob + l] : -1;
        for (int32_t kb = ob; kb < oe; kb += SSSP_WAVE) {
          const int32_t cn = kb + SSSP_WAVE + l < oe ? od[kb + SSSP_WAVE + l] : -1;
          bool ch = false;
          float av = 0.0f;
          if (c >= 0) {
            ch = c != ort && a.pred[osb + c] == kb + l;
            if (ch)
              av = __hip_atomic_load(&a.acc[osb + c], __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
          }
          unsigned long long cm = __ballot(ch);
          while (cm) {
            const int q = __ffsll(cm) - 1;
            cm &= cm - 1;
            s = __fadd_rn(s, __uint_as_float((uint32_t)__builtin_amdgcn_readlane(
                                 (int)__float_as_uint(av), q)));
          }
          c = cn;
        }
        if (l == o) acc = s;
      }
    }
  }
  return steps;
}

// (no barrier: a wave on a long path would hold the block's other waves)
__device__ __forceinline__ void add_steps(const BackArgs &a, int32_t steps, int64_t wid) {
  steps = (int32_t)wave_sum64(steps);
  if (lane_id() == 0 && steps)
    atomicAdd(&a.ctl[(1 + wid % kBackSums) * kBackStride], (unsigned int)steps);
}

// Blocks b with the same b mod 8 (one XCD) sweep the same eighth of the vertices.
__global__ __launch_bounds__(BBS) void bw_walk_kernel(BackArgs a) {
  const int64_t part = blockIdx.x & 7, waves = (int64_t)(gridDim.x >> 3) * (BBS / SSSP_WAVE);
  const int64_t wid = (int64_t)(blockIdx.x >> 3) * (BBS / SSSP_WAVE) +
                      __builtin_amdgcn_readfirstlane((int)(threadIdx.x / SSSP_WAVE));
  const SweepSource from = {((part * a.total) >> 3) + wid * kSweep, ((part + 1) * a.total) >> 3,
                            waves * kSweep};
  add_steps(a, walk(a, from), part * waves + wid);
}

__global__ __launch_bounds__(BBS) void bw_walk_xcd_kernel(BackArgs a) {
  const int64_t wid = (int64_t)blockIdx.x * (BBS / SSSP_WAVE) +
                      __builtin_amdgcn_readfirstlane((int)(threadIdx.x / SSSP_WAVE));
  const XcdSource from = {
      (unsigned long long *)(a.ctl + (1 + kBackSums + (xcd_id() & 7)) * kBackStride),
      a.ctl + (1 + kBackSums + 8) * kBackStride};
  add_steps(a, walk(a, from), wid);
}

// Only for a pred array with stray trees or parent cycles (the walk does not
// reach every vertex): each vertex's parent moves up to its parent's parent
// until it is one of the three ends or, after log2(n) rounds, still on a
// cycle; the sums of vertices that do not end under the root are cleared.
__global__ __launch_bounds__(1024) void bw_prune_kernel(BackArgs a) {
  int32_t reached = 0;
  for (int q = lane_id(); q < kBackSums; q += SSSP_WAVE)
    reached += (int32_t)a.ctl[(1 + q) * kBackStride];
  if (a.ctl[0] == 0u && wave_sum64(reached) == a.total) return;
  for (int32_t ins = blockIdx.x; ins < a.num_inst; ins += gridDim.x) {
    const InstDev id = a.insts[ins];
    for (int64_t far = 1; far < 2 * (int64_t)id.n; far <<= 1) {
      for (int32_t x = (int32_t)threadIdx.x; x < id.n; x += 1024) {
        int32_t *at = &a.par[id.sbase + x];
        const int32_t up = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (up >= 0)
          __hip_atomic_store(at,
                             __hip_atomic_load(&a.par[up], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      stores_done();
      __syncthreads();
    }
    for (int32_t x = (int32_t)threadIdx.x; x < id.n; x += 1024)
      if (__hip_atomic_load(&a.par[id.sbase + x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) !=
          kUnderRoot)
        a.acc[id.sbase + x] = 0.0f;
  }
}

// grad_w[ebase[g] + e] = sum over instances i of graph g (instance order) of
// acc_i[head(e)] if pred_i[head(e)] == e: a thread per vertex, whose entries
// are read once, coalesced, and added to the sums of its in-edges in
// registers; past kBackIn in-edges the thread, which alone touches them, adds
// in memory.  The order of the sums leaves a graph of few vertices only few
// threads, each with a chain of reads per instance: the instances' places come
// from LDS and kGradAhead of them are read at once (3000 instances of 200 vertices,
// whole pass 3.26 -> 2.27 ms, 20000 of 30 14.7 -> 6.7, 1000 of 900 0.93 -> 0.53; 64 of
// 512 x 512 as before).
__global__ __launch_bounds__(BBS) void bw_grad_kernel(BackArgs a) {
  __shared__ int2 tab[BBS];  // the instances' bases and sources
  for (int32_t b = blockIdx.x; b < a.blocks; b += gridDim.x) {
    const int32_t g = block_graph(a, b);
    const GraphDev &G = a.graphs[g];
    const int32_t y = (b - a.bbase[g]) * BBS + (int32_t)threadIdx.x;
    const bool on = y < G.n;
    InEdges in;
    in.deg = 0;
    if (on) in.load(G, y, false);
    float *grad = a.grad_w + a.ebase[g];
    float sum[kBackIn];
#pragma unroll
    for (int q = 0; q < kBackIn; ++q) sum[q] = 0.0f;
    const int32_t j1 = a.goff[g + 1];
    for (int32_t j = a.goff[g]; j < j1; j += BBS) {
      const int32_t cnt = j1 - j < BBS ? j1 - j : BBS;
      __syncthreads();
      if ((int32_t)threadIdx.x < cnt) {
        const InstDev id = a.insts[a.ginst[j + (int32_t)threadIdx.x]];
        tab[threadIdx.x] = make_int2(id.sbase, id.source);
      }
      __syncthreads();
      if (!on) continue;
      for (int32_t k = 0; k < cnt; k += kGradAhead) {
        int32_t e[kGradAhead];
        float v[kGradAhead];
#pragma unroll
        for (int u = 0; u < kGradAhead; ++u) {  // (past the end: the last one again, unused)
          const int2 id = tab[k + u < cnt ? k + u : cnt - 1];
          e[u] = k + u < cnt && y != id.y ? a.pred[id.x + y] : -1;
          v[u] = a.acc[id.x + y];
        }
#pragma unroll
        for (int u = 0; u < kGradAhead; ++u) {
          if (e[u] < 0) continue;
          if (in.deg <= kBackIn) {
#pragma unroll
            for (int q = 0; q < kBackIn; ++q)
              sum[q] = in.eid[q] == e[u] ? __fadd_rn(sum[q], v[u]) : sum[q];
          } else if (e[u] < G.m && G.u_out_dst[e[u]] == y) {
            grad[e[u]] = __fadd_rn(grad[e[u]], v[u]);
          }
        }
      }
    }
    if (on && in.deg <= kBackIn) {
#pragma unroll
      for (int q = 0; q < kBackIn; ++q)
        if (q < in.deg) grad[in.eid[q]] = sum[q];
    }
  }
}

hipError_t launch_backward(const BackArgs &a, int32_t max_inst, int32_t max_n,
                           hipStream_t stream) {
  const auto grid = [](int64_t items, int64_t most) {
    const int64_t b = (items + BBS - 1) / BBS;
    return dim3((unsigned int)(b < 1 ? 1 : b > most ? most : b));
  };
  const int64_t z = a.total > a.total_m ? a.total : a.total_m;
  hipLaunchKernelGGL(bw_zero_kernel, grid(z, 8192), dim3(BBS), 0, stream, a);
  dim3 vg((unsigned int)(a.blocks < 65536 ? a.blocks : 65536));
  const int chunks = (max_inst + kBackChunk - 1) / kBackChunk;
  dim3 pg(vg.x, (unsigned int)(chunks < 64 ? chunks : 64));
  hipLaunchKernelGGL(bw_parent_kernel, pg, dim3(BBS), 0, stream, a);
  // Each instance on one XCD keeps what its walkers read in that XCD's L2, but
  // takes its vertices from a counter and needs instances enough to go round:
  // 64 trees of 512 x 512 (16.8 M vertices) 3.2 -> 1.8 ms, 256 of 30011 2.05 ->
  // 1.57 (the whole pass), 8 of 10^6 1.60 -> 1.65, 64 of 30011 0.49 -> 0.54, 16
  // of 30011 0.13 -> 0.18.
  if (a.total >= (1 << 22) && (int64_t)max_n * 16 <= a.total) {
    hipLaunchKernelGGL(bw_walk_xcd_kernel, grid(a.total, kWalkBlocks), dim3(BBS), 0, stream, a);
  } else {
    dim3 wg = grid(a.total, kWalkBlocks);
    wg.x = (wg.x + 7u) & ~7u;
    hipLaunchKernelGGL(bw_walk_kernel, wg, dim3(BBS), 0, stream, a);
  }
  hipLaunchKernelGGL(bw_prune_kernel, dim3((unsigned int)(a.num_inst < 256 ? a.num_inst : 256)),
                     dim3(1024), 0, stream, a);
  hipLaunchKernelGGL(bw_grad_kernel, vg, dim3(BBS), 0, stream, a);
  return hipGetLastError();
}

}  // namespace sssp
