// The rounds of solves on small graphs (n <= kSmallN), each in one workgroup
// with the whole per-vertex state in LDS: the (D, parent) keys, both C
// buffers, the relax set, the D of each vertex's last relax and the
// out-offsets.  Only the edges are read from global memory (through this CU's
// L2), and of a vertex's in-edges the kRegEdges lightest stay in registers.
// Instance i of a batch runs on block i.  Results and counters are those of
// the persistent kernel, round for round (Section VI's rounds in the adopted
// order: relax, minD and the threshold, the lower bounds of Eq. 1, fix).  The
// block writes the costs and parents itself, so a solve is one launch.
//
// What bounds it: latency.  A round is three block barriers, one global read
// per relaxed edge, an LDS atomic, two block minima and the in-edges' LDS
// gathers; a solve has tens of rounds.  1003 vertices of degree 8: 17 rounds,
// 80 -> 48 us against a block scan and a window search per relax, separate
// bound and fix passes, one register edge, a launch of its own for the costs;
// 4096 vertices: 21 rounds, 205 -> 140 us.  A batch of 64 solves on 4001
// vertices takes 154 us here and 1.6 ms on the persistent kernel, whose every
// round waits for all the instances.
#include "sssp_dev.h"
#include "sssp_kernels.h"

namespace sssp {

constexpr int kRegEdges = 4;   // a vertex's lightest in-edges kept in registers
constexpr int kItemLanes = 8;  // lanes that share a relax item's out-list
// Longer out-lists are relaxed by a wave each, these by the whole block.  All
// of them one after another by the whole block, 4096 vertices of degree 64,
// 256 and 1000 take 1766, 4852 and 4493 us, this way 542, 1021 and 2913 (with four
// reads in flight a lane instead of two 542, 805 and 2478, but then solves without
// such lists take 1 % longer).  The line at 32 or 16: 212 and 230 us at degree 32
// (174 at 64), 500 at degree 64.
constexpr int32_t kLongOut = 64, kHugeOut = 1024;

// The open set O is implicit: y is open iff it is discovered (D < INF) and
// not fixed (C < INF; fixed vertices carry C = INF, and a discovered vertex
// never has C = INF otherwise, as C <= D).
template <int N, int NW>
struct SmallLds {
  unsigned long long D[N];  // (D << 32) | equal-cost flag << 31 | edge id
  int32_t C[2][N];          // lower bounds by round parity (INF: fixed)
  int32_t DR[N];            // D of the last relax, or of the coming one (INF: never)
  int32_t off[N + 1];       // out-offsets
  uint16_t F[N];            // relax set
  uint16_t L[N];            // its members with long out-lists, the huge ones from the end
  int32_t red[2][2 * NW];   // by round parity
  int32_t nF, nL, target_hit, ndegen;  // nL: of the long lists, and (<< 16) the huge ones
  unsigned long long relaxed, scanned, visits, settled;
};

// Levels of float32 equal-cost vertices (the rule at the emit pass): the
// block's queue q[0, nd) of caller ids, all of one instance whose costs and
// parents (-2: queued) start at D and pred.
template <class V>
__device__ int small_degen(const GraphDev &G, const int32_t *D, int32_t *pred, const int32_t *q,
                           int nd, int32_t *lvl, int32_t *flag) {
  int bad = 0;
  for (int lv = 0;; ++lv) {
    for (int i = threadIdx.x; i < nd; i += blockDim.x) {
      flag[i] = 0;
      const int32_t y = q[i];
      if (lvl[y] != -1) continue;
      const int32_t dy = D[y];
      for (int32_t j = G.u_in_off[y]; j < G.u_in_off[y + 1]; ++j) {
        const int32_t v = G.u_in_src[j], dv = D[v];
        if (dv == dy && V::add(dv, G.u_in_w[j]) == dy &&
            (pred[v] == -2 ? lvl[v] : 0) == lv) {
          flag[i] = 1;
          break;
        }
      }
    }
    __syncthreads();
    int changed = 0;
    for (int i = threadIdx.x; i < nd; i += blockDim.x) {
      if (flag[i]) {
        lvl[q[i]] = lv + 1;
        changed = 1;
      }
    }
    if (!__syncthreads_or(changed)) break;
  }
  for (int i = threadIdx.x; i < nd; i += blockDim.x) {
    const int32_t y = q[i], dy = D[y], ly = lvl[y];
    int32_t best = -1;
    if (ly >= 1) {
      for (int32_t j = G.u_in_off[y]; j < G.u_in_off[y + 1]; ++j) {
        const int32_t v = G.u_in_src[j], dv = D[v];
        if (dv == dy && V::add(dv, G.u_in_w[j]) == dy &&
            (pred[v] == -2 ? lvl[v] : 0) == ly - 1) {
          best = G.u_in_eid[j];
          break;
        }
      }
    }
    flag[i] = best;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nd; i += blockDim.x) {
    pred[q[i]] = flag[i];
    if (flag[i] < 0) bad = 1;
  }
  return __syncthreads_or(bad);
}

// T threads, each owning the vertices tid + k * T, k < SLOTS.  pred nullable;
// fault: the device's fault flag.
template <class V, bool BATCH, int T, int SLOTS>
__global__ __launch_bounds__(T) void small_rounds_kernel(RoundArgs a, int32_t *pred,
                                                         int32_t *fault) {
  constexpr int N = T * SLOTS, NW = T / SSSP_WAVE;
  static_assert(N <= 65536, "vertex ids fit 16 bits");
  __shared__ SmallLds<N, NW> s;
  const int tid = threadIdx.x;
  int32_t sb = 0, gi = 0, usrc = a.source;
  if constexpr (BATCH) {
    const InstDev id = a.insts[blockIdx.x];
    sb = id.sbase;
    gi = id.graph;
    usrc = id.source;
  }
  const GraphDev G = graph_of<BATCH>(a, gi);  // by value: its fields stay in registers
  const int n = G.n;
  const bool lc = G.lc != 0, all = G.all != 0;
  int32_t src = usrc, tgt = BATCH ? -1 : a.target;
  if (G.rank) {
    src = G.rank[src];
    if (tgt >= 0) tgt = G.rank[tgt];
  }
  // this thread's vertices: in-degree, in-list offset, out_wmin, the lightest
  // in-edges (INF weights past the list's end)
  int32_t id[SLOTS], ib[SLOTS], owm[SLOTS];
  uint32_t es[SLOTS][(kRegEdges + 1) / 2];  // tails, two to a word
  int32_t ew[SLOTS][kRegEdges];
#pragma unroll
  for (int k = 0; k < SLOTS; ++k) {
    const int y = tid + k * T;
    id[k] = ib[k] = 0;
    owm[k] = V::INF;
    if (y < n) {
      const int4 rec = G.vin[y];  // in_off, in_degree, the lightest in-edge's tail and weight
      ib[k] = rec.x;
      id[k] = rec.y;
      owm[k] = G.out_wmin[y];
      s.off[y] = G.out_off[y];
      const bool is_s = y == src;
      s.D[y] = make_key(is_s ? 0 : V::INF, -1, false);
      s.C[0][y] = s.C[1][y] = is_s ? V::INF : 0;  // the source is fixed from the start
      s.DR[y] = is_s ? 0 : V::INF;
    }
  }
#pragma unroll
  for (int k = 0; k < SLOTS; ++k) {
#pragma unroll
    for (int q = 0; q < kRegEdges; ++q) {
      ew[k][q] = V::INF;
      if (q % 2 == 0) es[k][q / 2] = 0u;
      if (q < id[k]) {
        const int2 e = G.in_sw[ib[k] + q];
        es[k][q / 2] |= (uint32_t)e.x << (16 * (q % 2));
        ew[k][q] = e.y;
      }
    }
  }
  if (tid == 0) {
    s.off[n] = G.out_off[n];
    s.F[0] = (uint16_t)src;
    s.nF = 1;
    s.nL = 0;
    s.ndegen = 0;
    s.target_hit = (tgt >= 0 && tgt == src) ? 1 : 0;
    s.relaxed = s.scanned = s.visits = 0ull;
    s.settled = 1ull;  // the source
  }
  // per-thread counts, summed at the end
  unsigned long long nrel = 0, nscan = 0;
  uint32_t nfix = 0, nvis = 0;
  __syncthreads();
  int r = 0, status = 0;
  for (;;) {
    if (tgt >= 0 && s.target_hit) break;  // the frontier that fixed it is not relaxed
    ++r;
    if (r > n + 1 || r > a.max_rounds) {
      status = 7;
      break;
    }
    const int cur = r & 1;  // the bound step reads C[cur] and writes C[cur ^ 1]
    // (A) relax the relax set's out-edges, each vertex from the D it had when
    // it joined the set (first discoveries join O by getting a finite D):
    // kItemLanes lanes to an item, two items at a time
    const int nF = s.nF;
    auto relax_edge = [&](int32_t dx, const int4 &er) {
      // er: head, weight, edge id, the head's out_wmin
      const int32_t cand = V::add(dx, er.y);
      atomicMin(&s.D[er.x], make_key(cand, er.z, cand == dx));
    };
    {
      constexpr int GR = T / kItemLanes;
      const int g = tid / kItemLanes, l = tid % kItemLanes;
      for (int i = g; i < nF; i += 2 * GR) {
        int32_t b[2], e[2], dx[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int iu = i + u * GR;
          b[u] = e[u] = dx[u] = 0;
          if (iu < nF) {
            const int x = s.F[iu];
            b[u] = s.off[x];
            e[u] = s.off[x + 1];
            dx[u] = s.DR[x];
            if (l == 0) {
              nrel += (unsigned long long)(e[u] - b[u]);
              if (__builtin_expect(e[u] - b[u] > kLongOut, 0)) {
                const bool huge = e[u] - b[u] > kHugeOut;
                const int at = atomicAdd(&s.nL, huge ? 1 << 16 : 1);
                s.L[huge ? N - 1 - (at >> 16) : at & 0xffff] = (uint16_t)x;
              }
            }
            if (e[u] - b[u] > kLongOut) e[u] = b[u];
          }
        }
        for (int32_t k = l; b[0] + k < e[0] || b[1] + k < e[1]; k += kItemLanes) {
          int4 er[2];
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (b[u] + k < e[u]) er[u] = G.out_rec[b[u] + k];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            if (b[u] + k < e[u]) relax_edge(dx[u], er[u]);
          }
        }
      }
    }
    __syncthreads();
    const int lists = s.nL;
    if (__builtin_expect(lists > 0, 0)) {
      constexpr int U = 2;
      const int nL = lists & 0xffff, nH = lists >> 16;
      for (int i = tid / SSSP_WAVE; i < nL; i += NW) {
        const int x = s.L[i];
        const int4 *rec = G.out_rec + s.off[x];
        const int32_t deg = s.off[x + 1] - s.off[x], dx = s.DR[x];
        for (int32_t k = lane_id(); k < deg; k += U * SSSP_WAVE) {
          int4 er[U];
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (k + u * SSSP_WAVE < deg) er[u] = rec[k + u * SSSP_WAVE];
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (k + u * SSSP_WAVE < deg) relax_edge(dx, er[u]);
        }
      }
      for (int i = 0; i < nH; ++i) {
        const int x = s.L[N - 1 - i];
        const int4 *rec = G.out_rec + s.off[x];
        const int32_t deg = s.off[x + 1] - s.off[x], dx = s.DR[x];
        for (int32_t k = tid; k < deg; k += T) relax_edge(dx, rec[k]);
      }
      __syncthreads();
    }
    if (tid == 0) s.nF = 0;  // (read by all before the barrier above)
    const int32_t *Cold = s.C[cur];
    int32_t *Cnew = s.C[cur ^ 1];
    // (B) minD and the threshold over O
    int32_t md = V::INF, th = V::INF;
    int32_t dy[SLOTS], c[SLOTS];
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
      const int y = tid + k * T;
      dy[k] = c[k] = V::INF;
      if (y < n) {
        dy[k] = (int32_t)(s.D[y] >> 32);
        c[k] = Cold[y];
        if (dy[k] != V::INF && c[k] != V::INF) {
          md = kmin(md, dy[k]);
          th = kmin(th, V::add(dy[k], owm[k]));
        }
      }
    }
    md = wave_min(md);
    th = wave_min(th);
    {
      int32_t *red = s.red[cur];
      if (lane_id() == 0) {
        red[tid / SSSP_WAVE] = md;
        red[NW + tid / SSSP_WAVE] = th;
      }
      __syncthreads();
      md = red[0];
      th = red[NW];
#pragma unroll
      for (int i = 1; i < NW; ++i) {
        md = kmin(md, red[i]);
        th = kmin(th, red[NW + i]);
      }
    }
    if (md == V::INF) break;  // (A) left nothing open
    if (tid == 0) s.nL = 0;
    // (C) lower bounds (Eq. 1), Jacobi over C[cur]; SP_4's scope also
    // raises C of undiscovered vertices (an unreachable one, C = INF, keeps
    // it).  In-lists ascend by weight and every term max(C[v], minD) + w is
    // at least minD + w, so a scan stops at the first edge with
    // minD + w >= min(D[y], m_y) (D = INF for undiscovered ones); the slots'
    // register edges go side by side.  The counters take whole in-degrees.
    int32_t m[SLOTS];
    bool on[SLOTS];
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
      m[k] = V::INF;
      on[k] = c[k] != V::INF && (dy[k] != V::INF || all);
    }
#pragma unroll
    for (int q = 0; q < kRegEdges; ++q) {
      int32_t cv[SLOTS];
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        on[k] = on[k] && V::add(md, ew[k][q]) < kmin(dy[k], m[k]);
        cv[k] = Cold[on[k] ? (es[k][q / 2] >> (16 * (q % 2))) & 0xffffu : 0u];
      }
#pragma unroll
      for (int k = 0; k < SLOTS; ++k)
        if (on[k] && cv[k] != V::INF) m[k] = kmin(m[k], V::add(kmax(cv[k], md), ew[k][q]));
    }
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
      if (on[k] && id[k] > kRegEdges) {
        for (int32_t j = kRegEdges; j < id[k]; ++j) {
          const int2 e = G.in_sw[ib[k] + j];  // tail, weight
          if (V::add(md, e.y) >= kmin(dy[k], m[k])) break;
          const int32_t cv = Cold[e.x];
          if (cv != V::INF) m[k] = kmin(m[k], V::add(kmax(cv, md), e.y));
        }
      }
    }
    // (These chains of global reads are the longest part of a round at 4096
    // vertices, 2.8 of 6.7 us.  Other ways measured there, at 140 us a solve:
    // 6 or 8 register edges 140 and 160; the slots' chains side by side 166;
    // four edges a step 157; the lists scanned by groups of 8 lanes from an
    // LDS queue 155.)
    // (D) fix: C' >= D or D <= thr.  The next relax set is the newly fixed
    // vertices (label-correcting: those and, in the first bucket above minD,
    // the survivors whose D fell since their last relax, the fixed ones only
    // if it fell); its places come from one LDS atomic per wave
    uint64_t push[SLOTS];
    int npush = 0;
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
      const int y = tid + k * T;
      const bool disc = dy[k] != V::INF, live = c[k] != V::INF;
      const bool open = disc && live, step = open || (!disc && all);  // step (C) covers y
      // a fixed or unreachable vertex keeps C = INF
      const int32_t cn = live ? kmax(kmax(c[k], md), kmin(dy[k], m[k])) : V::INF;
      const bool fix = open && (cn >= dy[k] || dy[k] <= th);
      bool p = false;
      if (y < n) {
        if (step) nscan += (unsigned long long)id[k];
        if (step || !live) Cnew[y] = fix ? V::INF : cn;
        nvis += open ? 1u : 0u;
        nfix += fix ? 1u : 0u;
        if (fix && y == tgt) s.target_hit = 1;
        p = open && (fix || (lc && dy[k] < V::add(md, G.delta)));
        if (lc && p) p = dy[k] < s.DR[y];
        if (p) s.DR[y] = dy[k];
      }
      push[k] = __ballot(p);
      npush += __popcll(push[k]);
    }
    if (npush) {  // (wave-uniform)
      int at = 0;
      if (lane_id() == 0) at = atomicAdd(&s.nF, npush);
      at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        const uint64_t mine = push[k];
        if ((mine >> lane_id()) & 1ull)
          s.F[at + __builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u))] =
              (uint16_t)(tid + k * T);
        at += __popcll(mine);
      }
    }
    __syncthreads();
  }
  __syncthreads();
  // costs and parents (the emit pass's rule), in the caller's numbering
  int32_t *cost = a.D + sb, *queue = a.degen + sb, *lvl = a.lvl + sb;
  int32_t *par = pred ? pred + sb : nullptr;
#pragma unroll
  for (int k = 0; k < SLOTS; ++k) {
    const int y = tid + k * T;
    if (y < n) {
      const int32_t uy = G.vid ? G.vid[y] : y;
      const unsigned long long key = s.D[y];
      const int32_t d = (int32_t)(key >> 32);
      cost[uy] = d;
      if (par) {
        int32_t p = -1;
        if (uy != usrc && d != V::INF) {
          if (key & kKeyEqualCost) {
            p = -2;
            queue[atomicAdd(&s.ndegen, 1)] = uy;
            lvl[uy] = -1;
          } else {
            p = (int32_t)(key & kKeyEidMask);
          }
        }
        par[uy] = p;
      }
    }
  }
  {
    const long long v0 = wave_sum64((long long)nrel), v1 = wave_sum64((long long)nscan);
    const long long v2 = wave_sum64((long long)nvis), v3 = wave_sum64((long long)nfix);
    if (lane_id() == 0) {
      if (v0) atomicAdd(&s.relaxed, (unsigned long long)v0);
      if (v1) atomicAdd(&s.scanned, (unsigned long long)v1);
      if (v2) atomicAdd(&s.visits, (unsigned long long)v2);
      if (v3) atomicAdd(&s.settled, (unsigned long long)v3);
    }
  }
  __syncthreads();
  const int nd = s.ndegen;
  if (nd > 0 && small_degen<V>(G, cost, par, queue, nd, lvl, a.flag + sb)) status = 7;
  if (tid != 0) return;
  if (status) atomicOr(fault, 1);
  Ctl *ctl = a.ctl;
  if constexpr (BATCH) {
    const int inst = blockIdx.x;
    a.irounds[inst] = r;
    a.iscanned[3 * inst] = s.scanned;
    a.iscanned[3 * inst + 1] = s.visits;
    a.iscanned[3 * inst + 2] = s.relaxed;
    if (a.idead) a.idead[2 * inst] = a.idead[2 * inst + 1] = 0ull;  // counted round by round
    if (a.istat) {
      a.istat[4 * inst] = a.istat[4 * inst + 3] = 0;
      a.istat[4 * inst + 1] = (long long)s.settled;
      a.istat[4 * inst + 2] = (long long)s.relaxed;
    }
    if (status) atomicMax(&ctl->status, status);
  } else {
    ctl->front_ctr[0] = ctl->front_ctr[1] = 0ull;
    ctl->open_ctr[0] = ctl->open_ctr[1] = 0ull;
    ctl->live_ctr[0] = ctl->live_ctr[1] = 0ull;
    ctl->go = 0u;
    ctl->deg_count = nd;
    ctl->solo_phases = 0;
    ctl->dead_deg = ctl->dead_deg_r = 0ull;
    ctl->rounds = r;
    ctl->status = status;
    ctl->settled = (long long)s.settled;
    ctl->relaxed = (long long)s.relaxed;
    ctl->scanned = (long long)s.scanned;
    ctl->open_visits = (long long)s.visits;
    ctl->target_id = tgt;
    ctl->target_hit = s.target_hit;
  }
}

// A batch's control block (its instances raise the status).
__global__ void small_reset_kernel(Ctl *ctl) {
  ctl->status = 0;
  ctl->rounds = 0;
  ctl->deg_count = 0;
  ctl->solo_phases = 0;
}

template <class V, bool BATCH>
static hipError_t launch_small_t(const RoundArgs &a, int32_t *pred, int32_t max_n,
                                 const KernelTimer *timer, Launcher &L) {
  hipError_t e;
  if (max_n > kSmallN || (!BATCH && a.num_inst != 1)) return hipErrorInvalidValue;
  RoundArgs arg = a;
  int32_t *p = pred, *fault = nullptr;
  if ((e = fault_flag_address(&fault)) != hipSuccess) return e;
  Ctl *ctl = a.ctl;
  void *params[] = {&arg, &p, &fault};
  void *reset[] = {&ctl};
  if (BATCH && (e = launch_kernel(L, (const void *)small_reset_kernel, dim3(1), dim3(1), reset,
                                  false)) != hipSuccess)
    return e;
  if (L.graph) timer = nullptr;
  if (timer && (e = hipEventRecord(timer->start, L.stream)) != hipSuccess) return e;
  const dim3 grid(BATCH ? (unsigned)a.num_inst : 1u);
  // 1024 threads also where 256 or 512 would own several vertices each:
  // 1003 vertices take 48 us, against 58 (512 x 2) and 91 (256 x 4)
  if (max_n <= 1024)
    e = launch_kernel(L, (const void *)small_rounds_kernel<V, BATCH, 1024, 1>, grid, dim3(1024),
                      params, false);
  else if (max_n <= 2048)
    e = launch_kernel(L, (const void *)small_rounds_kernel<V, BATCH, 1024, 2>, grid, dim3(1024),
                      params, false);
  else
    e = launch_kernel(L, (const void *)small_rounds_kernel<V, BATCH, 1024, 4>, grid, dim3(1024),
                      params, false);
  if (e != hipSuccess) return e;
  if (timer && (e = hipEventRecord(timer->stop, L.stream)) != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_small(bool f32, bool batch, const RoundArgs &a, int32_t *pred, int32_t max_n,
                        const KernelTimer *timer, Launcher &L) {
  if (f32)
    return batch ? launch_small_t<KeyF32, true>(a, pred, max_n, timer, L)
                 : launch_small_t<KeyF32, false>(a, pred, max_n, timer, L);
  return batch ? launch_small_t<KeyI32, true>(a, pred, max_n, timer, L)
               : launch_small_t<KeyI32, false>(a, pred, max_n, timer, L);
}

}  // namespace sssp
