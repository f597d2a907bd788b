// The rounds of solves under C scope ALL on graphs without hubs (random
// digraphs), each by a team of K workgroups on one XCD.  Under that scope a
// round visits every vertex that is not fixed, so the lists, windows and
// stagers of the grid-wide kernel buy nothing there: every thread owns
// vertices for the whole solve and loops over those still live (a bit mask in
// a register).  Its own D, C and vertex records are read coalesced, only the
// tails' C are gathered, and there is no list but the relax set, which stays
// in the workgroup's LDS.  D and C of a solve fit the XCD's L2; a batch runs
// its instances one after another on each team, so their working sets stay
// there too instead of sweeping all instances every round (those that make up
// much of the batch first: 240 graphs of 300 to 700 vertices and one of 200000
// take 2.1 ms wherever it stands among them; last in the queue it took 3.5.  All by
// size, 256 graphs of 1 to 200 thousand vertices take 23.4 ms, 22.9 as they come:
// the largest then contend for memory).  A single large
// solve takes all XCDs as one team.
//
// What bounds it: on one XCD the gathers of the bound step, 52 of 81 thousand
// cycles a round at 150001 vertices of degree 8 (eight such solves: 0.49 M L2
// requests a round and XCD, reads of 455 cycles against 234 in the mesh kernel,
// 70 % of them hits; waves wait 75 % of their time and issue 13 %); on all XCDs the
// step takes 9 of 35 thousand and the two barriers, with the wait for the slowest
// block, 8 and 11.  Against the grid-wide kernel: 150001 vertices 1.70 -> 0.51
// ms, 400003 x 6 2.24 -> 0.81, 10^6 x 8 3.62 -> 1.83, 5000 0.84 -> 0.19; 256
// graphs of up to 200000 vertices 58.6 -> 22.9 ms; 16 sources on 30011
// vertices 2.53 -> 0.46.
//
// A round: relax the block's relax set (returning atomics: the offers to minD
// and thr); team barrier, whose words carry the offers; bound and fix (Eq. 1,
// then the fix rule, for the thread's own vertices); team barrier.
#include <atomic>

#include "sssp_dev.h"
#include "sssp_kernels.h"
#include "team.h"

namespace sssp {

constexpr int DBS = 1024;
constexpr int kDenseItems = 4096;   // relax items in LDS; the rest is relaxed by its owner
constexpr int kDenseLanes = 8;      // lanes that share a relax item's out-list
constexpr int kMaxTeamBlocks = 32;  // one per compute unit of an XCD
constexpr int kMaxWide = 256;       // blocks of a team over all XCDs
constexpr int kDenseSlots = 32;     // vertices per thread: bits of the live mask

// two in-list entries (tail, weight), read at once
typedef int32_t edge_pair __attribute__((ext_vector_type(4), aligned(8)));

struct DenseArgs {
  int32_t K, teams;
  unsigned long long *words;  // [teams][2 K + 1]: offers, round ends, the next instance
  int32_t *queue;             // instances taken beyond the first of each team
};

__global__ __launch_bounds__(256) void dense_init_kernel(RoundArgs a, DenseArgs q) {
  for (int i = threadIdx.x; i < q.teams * (2 * q.K + 1); i += 256) q.words[i] = 0ull;
  if (threadIdx.x == 0) {
    *q.queue = 0;
    Ctl *c = a.ctl;
    c->front_ctr[0] = c->front_ctr[1] = 0ull;
    c->open_ctr[0] = c->open_ctr[1] = 0ull;
    c->live_ctr[0] = c->live_ctr[1] = 0ull;
    c->go = 0u;
    c->deg_count = 0;
    c->solo_phases = 0;
    c->dead_deg = c->dead_deg_r = 0ull;
    c->status = 0;
    c->rounds = 0;
    c->settled = c->relaxed = c->scanned = c->open_visits = 0;
    c->target_id = -1;
    c->target_hit = 0;
  }
}

struct DenseLds {
  int4 rel[kDenseItems];  // relax set: vertex, D to relax from, out-offset, out-degree
  int32_t red[2][DBS / SSSP_WAVE];
  int32_t md, th, nF, lost, next;
  unsigned long long relaxed, scanned, visits, settled;
};

// a pointer all lanes hold alike, in scalar registers
template <class T>
__device__ __forceinline__ T *scalar_ptr(T *p) {
  return (T *)(uintptr_t)readlane64((int64_t)(uintptr_t)p, 0);
}

// WIDE: the instances one after another, by one team of q.K blocks (up to
// kMaxWide) over all XCDs.  Every wait reads as many words as the widest team of
// its form has blocks: one a lane, four where WIDE.  That is the team's width and
// nothing else: a batch may be as wide as a single solve.
template <class V, bool BATCH, bool WIDE>
__global__ __launch_bounds__(DBS) void dense_rounds_kernel(RoundArgs a, DenseArgs q) {
  __shared__ DenseLds s;
  const int tid = threadIdx.x, wv = tid / SSSP_WAVE, l = lane_id();
  const int tb = blockIdx.x >> 3, K = q.K;
  const int j = WIDE ? (int)blockIdx.x : tb % K;
  const int team = WIDE ? 0 : (tb / K) * 8 + (int)(blockIdx.x & 7u);
  if (team >= q.teams) return;
  unsigned long long *pub = q.words + (size_t)team * (2 * K + 1);
  unsigned long long *fin = pub + K, *nxt = fin + K;
  unsigned ep = 1;
  bool same = false, lost = false;
  // Team barrier on `words`, with the minima of md and th over the team (the
  // words of round ep).  Every store made before it is seen after it.
  auto team_min = [&](unsigned long long *words, int32_t &md, int32_t &th, bool reset) {
    md = wave_min(md);
    th = wave_min(th);
    stores_done();
    if (l == 0) {
      s.red[0][wv] = md;
      s.red[1][wv] = th;
    }
    __syncthreads();
    if (wv == 0) {
      constexpr int NW = DBS / SSSP_WAVE;
      md = wave_min(s.red[0][l % NW]);
      th = wave_min(s.red[1][l % NW]);
      if (l == 0) put64(&words[j], offers(ep, md, th), same);
      bool lo = false;
      md = th = 0x7fffffff;
      if constexpr (!WIDE) {
        static_assert(kMaxTeamBlocks <= SSSP_WAVE, "a word a lane");
        const unsigned long long x = await_offers(words, l < K ? l : 0, ep, &lo);
        md = offers_md(x);
        th = offers_th(x);
      } else {  // up to four words a lane, read together
        static_assert(kMaxWide <= 4 * SSSP_WAVE, "four words a lane");
        unsigned long long x[4];
        int spins = 0;
        bool wait;
        do {
          wait = false;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int b = i * SSSP_WAVE + l;
            x[i] = ld_relaxed64(&words[b < K ? b : 0]);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) wait |= (unsigned)(x[i] >> 62) != (ep & 3u);
          lo = ++spins > kSpinLimit;
        } while (!lo && __ballot(wait));
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          md = kmin(md, offers_md(x[i]));
          th = kmin(th, offers_th(x[i]));
        }
      }
      md = wave_min(md);
      th = wave_min(th);
      if (l == 0) {
        s.md = md;
        s.th = th;
        s.lost = lo ? 1 : 0;
        if (reset) s.nF = 0;
      }
    }
    __syncthreads();
    md = __builtin_amdgcn_readfirstlane(s.md);
    th = __builtin_amdgcn_readfirstlane(s.th);
    lost = __builtin_amdgcn_readfirstlane(s.lost) != 0;
  };
  {
    // round 1 of the words: whether the team shares an XCD, and so an L2
    int32_t lo = xcd_id() + 1, hi = 0x7fffffff - lo;
    const int32_t mine = lo;
    team_min(pub, lo, hi, false);
    const bool eq = lo == mine && 0x7fffffff - hi == mine;
    int32_t d0 = 0, d1 = 0;
    team_min(fin, d0, d1, false);
    same = eq;
  }
  int turn = team;  // in the batch's order
  while (turn < a.num_inst && !lost) {
    int32_t sb = 0, gi = 0, src = a.source, inst = 0;
    if constexpr (BATCH) {
      inst = ((const int32_t *)(a.insts + a.num_inst))[turn];
      const InstDev id = a.insts[inst];
      sb = id.sbase;
      gi = id.graph;
      src = id.source;
    }
    GraphDev G = graph_of<BATCH>(a, gi);
    if constexpr (BATCH) {
      // read from a table, so in vector registers, though alike in all lanes
      sb = __builtin_amdgcn_readfirstlane(sb);
      src = __builtin_amdgcn_readfirstlane(src);
      G.n = __builtin_amdgcn_readfirstlane(G.n);
      G.lc = __builtin_amdgcn_readfirstlane(G.lc);
      G.delta = __builtin_amdgcn_readfirstlane(G.delta);
      G.out_rec = scalar_ptr(G.out_rec);
      G.vrec = scalar_ptr(G.vrec);
      G.vin = scalar_ptr(G.vin);
      G.in_sw = scalar_ptr(G.in_sw);
      G.out_wmin = scalar_ptr(G.out_wmin);
      G.out_off = scalar_ptr(G.out_off);
      G.rank = scalar_ptr(G.rank);
    }
    const int n = G.n;
    const bool lc = G.lc != 0;
    int32_t tgt = BATCH ? -1 : a.target;
    if (G.rank) {
      src = G.rank[src];
      if (tgt >= 0) tgt = G.rank[tgt];
    }
    unsigned long long *D = a.D64 + sb;
    int32_t *C[2] = {a.C0 + sb, a.C1 + sb};
    int32_t *DR = lc ? a.DR + sb : nullptr;
    // per vertex: how many of its lightest in-edges have tails fixed for good
    int32_t *SK = a.mtmp + sb;
    // slot k of this thread: vertex y0 + k * ystep (64 neighbours to a wave,
    // neighbouring 64s to different blocks)
    const int32_t y0 = (wv * K + j) * SSSP_WAVE + l, ystep = K * DBS;
    const int S = (n + ystep - 1) / ystep;
    uint32_t live = 0;   // slots neither fixed nor known unreachable
    // relax items that found no place in LDS (pmark: those with no edges)
    uint32_t pend = 0, pmark = 0;
    for (int k = 0; k < S; ++k) {
      const int64_t y = y0 + (int64_t)k * ystep;
      if (y < n) {
        const bool is_s = y == src;
        put64(&D[y], make_key(is_s ? 0 : V::INF, -1, false), same);
        put(&C[0][y], is_s ? V::INF : 0, same);  // the source is fixed from the start
        put(&C[1][y], is_s ? V::INF : 0, same);
        if (DR) DR[y] = is_s ? 0 : V::INF;
        SK[y] = 0;
        if (!is_s) live |= 1u << k;
      }
    }
    if (tid == 0) {
      s.nF = 0;
      if (j == 0) {
        const int32_t o0 = G.out_off[src];
        s.rel[0] = make_int4(src, 0, o0, G.out_off[src + 1] - o0);
        s.nF = 1;
      }
      s.relaxed = s.scanned = s.visits = s.settled = 0ull;
    }
    ++ep;
    {
      int32_t d0 = 0, d1 = 0;
      team_min(pub, d0, d1, false);  // D is set everywhere
      if (!lost) team_min(fin, d0, d1, false);
    }
    unsigned long long nrel = 0, nscan = 0, ddeg = 0, ddeg_r = 0;
    uint32_t nvis = 0, nfix = 0;
    int32_t smd = V::INF, sth = V::INF;
    int r = 0, bounds = 0, status = 0;
    bool hit = tgt >= 0 && tgt == src;
    while (!lost) {
      if (hit) break;  // the frontier that fixed the target is not relaxed
      ++r;
      ++ep;
      if (r > n + 1 || r > a.max_rounds) {  // (every block alike)
        status = 7;
        break;
      }
      const int cur = r & 1;  // the bound step reads C[cur] and writes C[cur ^ 1]
      int32_t *Cold = C[cur], *Cnew = C[cur ^ 1];
      // (A) relax, each item from its D at the start of the step (bit 31: an
      // open vertex, label-correcting; INF: already relaxed at this D).  A
      // fixed item also marks its C in the buffer this round writes.
      int32_t md = smd, th = sth;
      const int nF = s.nF < kDenseItems ? s.nF : kDenseItems;
      auto offer = [&](const int4 &e, int32_t dx) {
        // e: head, weight, edge id, the head's out_wmin
        const int32_t cand = V::add(dx, e.y);
        const unsigned long long old = atomicMin(&D[e.x], make_key(cand, e.z, cand == dx));
        if (cand < (int32_t)(old >> 32)) {
          md = kmin(md, cand);
          th = kmin(th, V::add(cand, e.w));
        }
      };
      {
        constexpr int GR = DBS / kDenseLanes;
        const int g = tid / kDenseLanes, e0 = tid % kDenseLanes;
        for (int i = g; i < nF; i += 2 * GR) {
          int4 f[2];
          int32_t dx[2], deg[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const bool in = i + u * GR < nF;
            f[u] = in ? s.rel[i + u * GR] : make_int4(0, kOpenRelax, 0, 0);
            dx[u] = f[u].y & 0x7fffffff;
            deg[u] = in && dx[u] != V::INF ? f[u].w : 0;
            if (e0 == 0) {
              nrel += (unsigned long long)deg[u];
              if (f[u].y >= 0) put(&Cnew[f[u].x], V::INF, same);
            }
          }
          for (int32_t k = e0; k < deg[0] || k < deg[1]; k += kDenseLanes) {
            int4 e[2];
#pragma unroll
            for (int u = 0; u < 2; ++u)
              if (k < deg[u]) e[u] = G.out_rec[f[u].z + k];
#pragma unroll
            for (int u = 0; u < 2; ++u)
              if (k < deg[u]) offer(e[u], dx[u]);
          }
        }
      }
      while (pend) {  // (per thread) items without a place: the owner's own
        const int k = __ffs((int)pend) - 1;
        pend &= pend - 1u;
        const int32_t y = y0 + k * ystep;
        const bool fixed = !((live >> k) & 1u);
        const int32_t dx = lc ? DR[y] : (int32_t)(ld_relaxed64(&D[y]) >> 32);
        const int4 rec = G.vrec[2 * y];  // out_off, out_degree, in_off, in_degree
        if (fixed) put(&Cnew[y], V::INF, same);
        nrel += (unsigned long long)rec.y;
        for (int32_t e = 0; e < rec.y; ++e) offer(G.out_rec[rec.x + e], dx);
      }
      while (pmark) {
        const int k = __ffs((int)pmark) - 1;
        pmark &= pmark - 1u;
        put(&Cnew[y0 + k * ystep], V::INF, same);
      }
      team_min(pub, md, th, true);
      if (lost) break;
      if (md == V::INF) {  // (A) left nothing open
        // the words are rewritten by the team's next instance: only after
        // every block has read them
        int32_t z0 = 0, z1 = 0;
        if (BATCH) team_min(fin, z0, z1, false);
        break;
      }
      ++bounds;
      // (C) lower bounds (Eq. 1), Jacobi over C[cur], and (D) fix, for the
      // thread's live vertices, two at a time.  In-lists ascend by weight and
      // every term max(C[v], minD) + w is at least minD + w, so a scan stops
      // at the first edge with minD + w >= min(D[y], m_y) (D = INF for
      // undiscovered ones); the counters take whole in-degrees.
      smd = sth = V::INF;
      bool hit_now = false;
      constexpr int U = 2;  // (three or four spill: a batch takes 28 or 36 ms instead of 23)
      for (int k0 = 0; k0 < S; k0 += U) {
        if (!__ballot((live >> k0) & ((1u << U) - 1u))) continue;
        bool on[U];
        int32_t y[U], c[U], cz[U], owm[U], sk[U], sk0[U];
        unsigned long long dk[U];
        int4 rec[U];  // in_off, in_degree, lightest in-edge's tail and weight
#pragma unroll
        for (int u = 0; u < U; ++u) {
          on[u] = (live >> (k0 + u)) & 1u;
          y[u] = on[u] ? y0 + (k0 + u) * ystep : 0;
          dk[u] = ld_relaxed64(&D[y[u]]);
          c[u] = ld_relaxed(&Cold[y[u]]);
          rec[u] = G.vin[y[u]];
          owm[u] = G.out_wmin[y[u]];
          sk[u] = sk0[u] = SK[y[u]];
        }
        // The scan starts behind the lightest in-edges whose tails are known
        // to be fixed (or unreachable), for good: an open vertex's tails are
        // mostly fixed ones, and reading them again every round was most of
        // the step's L2 requests.
        // Then two edges at a time of both vertices, in one read each.
        int32_t dy[U], m[U], p[U];
        bool act[U], lead[U];  // lead: every edge before p has a fixed tail
#pragma unroll
        for (int u = 0; u < U; ++u) {
          dy[u] = (int32_t)(dk[u] >> 32);
          act[u] = on[u] & (c[u] != V::INF) & (sk[u] < rec[u].y) &
                   (V::add(md, rec[u].w) < dy[u]);
          cz[u] = ld_relaxed(&Cold[act[u] && sk[u] == 0 ? rec[u].z : 0]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          m[u] = V::INF;
          p[u] = sk[u];
          lead[u] = true;
          if (act[u] && sk[u] == 0) {
            if (cz[u] != V::INF) {
              m[u] = V::add(kmax(cz[u], md), rec[u].w);
              lead[u] = false;
            } else {
              sk[u] = 1;
            }
            p[u] = 1;
            act[u] = rec[u].y > 1 && V::add(md, rec[u].w) < m[u];
          }
        }
        for (;;) {
          bool any = false;
#pragma unroll
          for (int u = 0; u < U; ++u) any |= act[u];
          if (!__ballot(any)) break;
          int2 e[U][2];
          int32_t cv[U][2];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            // entries p and p + 1 (p - 1 and p at the list's end; p >= 1)
            const bool two = p[u] + 1 < rec[u].y;
            edge_pair x = {0, V::INF, 0, V::INF};
            if (act[u]) x = *(const edge_pair *)&G.in_sw[rec[u].x + p[u] - (two ? 0 : 1)];
            e[u][0] = two ? make_int2(x[0], x[1]) : make_int2(x[2], x[3]);
            e[u][1] = two ? make_int2(x[2], x[3]) : make_int2(0, V::INF);
          }
          bool use[U][2];
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              use[u][t] = act[u] && V::add(md, e[u][t].y) < kmin(dy[u], m[u]);
              cv[u][t] = V::INF;
              if (use[u][t]) cv[u][t] = ld_relaxed(&Cold[e[u][t].x]);
            }
#pragma unroll
          for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
              if (cv[u][t] != V::INF) m[u] = kmin(m[u], V::add(kmax(cv[u][t], md), e[u][t].y));
              lead[u] = lead[u] && use[u][t] && cv[u][t] == V::INF;
              if (lead[u]) sk[u] = p[u] + t + 1;
            }
            p[u] += 2;
            act[u] = act[u] && p[u] < rec[u].y && V::add(md, e[u][1].y) < kmin(dy[u], m[u]);
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (!on[u]) continue;
          const int32_t deg = rec[u].y;
          const bool disc = dy[u] != V::INF;
          if (sk[u] != sk0[u]) SK[y[u]] = sk[u];
          nscan += (unsigned long long)deg;
          if (c[u] == V::INF) {  // unreachable: C = INF in both buffers now
            put(&Cnew[y[u]], V::INF, same);
            ddeg += (unsigned long long)deg;
            ddeg_r += (unsigned long long)deg * (unsigned long long)bounds;
            live &= ~(1u << (k0 + u));
            continue;
          }
          const int32_t cn = kmax(kmax(c[u], md), kmin(dy[u], m[u]));
          if (!disc) {
            put(&Cnew[y[u]], cn, same);
            continue;
          }
          ++nvis;
          const int32_t dr = lc ? DR[y[u]] : V::INF;
          const bool relax_again = !lc || dy[u] < dr;
          const bool fix = cn >= dy[u] || dy[u] <= th;
          put(&Cnew[y[u]], fix ? V::INF : cn, same);
          bool push = false;
          int32_t fd = dy[u];
          if (fix) {
            ++nfix;
            hit_now |= y[u] == tgt;
            live &= ~(1u << (k0 + u));
            push = true;  // (with no edges, to mark its C, if relaxed at this D)
            if (!relax_again) fd = V::INF;
          } else {
            smd = kmin(smd, dy[u]);
            sth = kmin(sth, V::add(dy[u], owm[u]));
            // label-correcting: relaxed again from its lower D (while in the
            // first bucket above minD)
            if (lc && relax_again && dy[u] < V::add(md, G.delta)) {
              push = true;
              fd = dy[u] | kOpenRelax;
            }
          }
          if (push) {
            if (lc && fd != V::INF) DR[y[u]] = dy[u];
            const int p = atomicAdd(&s.nF, 1);
            if (p < kDenseItems) {
              const int4 ra = G.vrec[2 * y[u]];  // out_off, out_degree
              s.rel[p] = make_int4(y[u], fd, ra.x, ra.y);
            } else if (fd != V::INF) {
              pend |= 1u << (k0 + u);
            } else {
              pmark |= 1u << (k0 + u);
            }
          }
        }
      }
      int32_t h = hit_now ? 0 : 1, z = 0;
      team_min(fin, h, z, false);
      hit = h == 0;
    }
    if (lost) break;
    // ---- the instance's counts
    nscan += ddeg * (unsigned long long)bounds - ddeg_r;
    const long long v0 = wave_sum64((long long)nrel), v1 = wave_sum64((long long)nscan);
    const long long v2 = wave_sum64((long long)nvis), v3 = wave_sum64((long long)nfix);
    if (l == 0) {
      if (v0) atomicAdd(&s.relaxed, (unsigned long long)v0);
      if (v1) atomicAdd(&s.scanned, (unsigned long long)v1);
      if (v2) atomicAdd(&s.visits, (unsigned long long)v2);
      if (v3) atomicAdd(&s.settled, (unsigned long long)v3);
    }
    __syncthreads();
    if (tid == 0) {
      if constexpr (BATCH) {
        atomicAdd(&a.iscanned[3 * inst], s.scanned);
        atomicAdd(&a.iscanned[3 * inst + 1], s.visits);
        atomicAdd(&a.iscanned[3 * inst + 2], s.relaxed);
        if (j == 0) {
          a.irounds[inst] = r;
          if (status) atomicMax(&a.ctl->status, status);
        }
      } else {
        Ctl *c = a.ctl;
        atomicAdd((unsigned long long *)&c->relaxed, s.relaxed);
        atomicAdd((unsigned long long *)&c->scanned, s.scanned);
        atomicAdd((unsigned long long *)&c->open_visits, s.visits);
        // the source is settled too
        atomicAdd((unsigned long long *)&c->settled, s.settled + (j == 0 ? 1ull : 0ull));
        if (j == 0) {
          c->rounds = hit ? r : (status ? a.max_rounds : r);
          c->status = status;
          c->target_id = tgt;
          c->target_hit = hit ? 1 : 0;
        }
      }
    }
    // ---- the next instance: the team's first block takes it from the queue
    ++ep;
    if (!BATCH) break;
    if (wv == 0) {
      int32_t next = 0;
      if (j == 0) {
        if (l == 0) {
          next = q.teams + atomicAdd(q.queue, 1);
          put64(nxt, tagged(ep, next), same);
        }
        next = __builtin_amdgcn_readfirstlane(next);
      } else {
        unsigned long long x = 0;
        int spins = 0;
        do {
          x = ld_relaxed64(nxt);
          lost = ++spins > kSpinLimit;
        } while (!lost && (unsigned)(x >> 32) != ep);
        next = (int32_t)(uint32_t)x;
      }
      if (l == 0) {
        s.next = next;
        s.lost = lost ? 1 : 0;
      }
    }
    __syncthreads();
    // (uniform: the graph's fields then sit in scalar registers)
    turn = __builtin_amdgcn_readfirstlane(s.next);
    lost = __builtin_amdgcn_readfirstlane(s.lost) != 0;
    __syncthreads();
  }
  if (lost && tid == 0) atomicMax(&a.ctl->status, 7);
}

// per-instance counters of a batch
__global__ void dense_counts_kernel(RoundArgs a) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= a.num_inst) return;
  a.irounds[i] = 0;
  for (int k = 0; k < 3; ++k) a.iscanned[3 * i + k] = 0ull;
  if (a.idead) a.idead[2 * i] = a.idead[2 * i + 1] = 0ull;  // counted in the kernel
  if (a.istat)
    for (int k = 0; k < 4; ++k) a.istat[4 * i + k] = 0;
}

// From here one instance, two or three run, one after another, on one team over
// all XCDs (agent-scope stores, 256 words a barrier), below each on an XCD: one of
// 30000 vertices of degree 8 takes 0.30 ms on one, 0.33 on all; 40000 0.38 and
// 0.37; 150001 0.93 and 0.51.  Two of 150000 1.01 and 1.02, 200000 1.30 and 1.19,
// 10^6 7.6 and 3.7 (7.2 on the grid-wide kernel); three of 300000 1.88 and 2.2,
// 500000 2.98 and 2.9, 10^6 7.9 and 5.5.
constexpr int32_t kWideFrom[3] = {36864, 163840, 491520};
// Blocks per team: one per 1024 vertices where the instances then all run at
// once; else smaller teams, more of them, down to one block per 8192 vertices
// (and at most 16 where instances queue): 256 instances of 5 to 6 thousand
// vertices take 1.4 ms on teams of 2, 1.8 on 4, 2.7 on 8; of 5 to 30 thousand
// 4.8 on 4, 5.5 on 8, 7.3 on 16; of 1 to 200 thousand 26.8 on 8, 23.1 on 16,
// 25.2 on 32.
constexpr int32_t kDensePerBlock = 1024, kDenseMostPerBlock = 8192;
constexpr int kDenseQueueBlocks = 16;

// Co-resident blocks per compute unit (0: none).
template <class V, bool BATCH, bool WIDE>
static hipError_t dense_occupancy(int *occ) {
  static std::atomic<int> known{0};
  hipError_t e = hipSuccess;
  if ((*occ = known.load()) == 0) {
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        occ, (const void *)dense_rounds_kernel<V, BATCH, WIDE>, DBS, 0);
    if (e == hipSuccess) known.store(*occ);
  }
  return e;
}

template <class V, bool BATCH>
static hipError_t launch_dense_t(const RoundArgs &a, const LaunchGeom &geo, int32_t max_n,
                                 const KernelTimer *timer, Launcher &L, bool *done) {
  *done = false;
  hipError_t e;
  const bool wide = a.num_inst <= 3 && max_n > kWideFrom[a.num_inst - 1];
  int occ = 0;
  if ((e = wide ? dense_occupancy<V, BATCH, true>(&occ)
                : dense_occupancy<V, BATCH, false>(&occ)) != hipSuccess)
    return e;
  if (occ < 1) return hipSuccess;
  const int blocks = geo.blocks < geo.cus ? geo.blocks : geo.cus;  // one per compute unit
  int K = blocks / 8 < kMaxTeamBlocks ? blocks / 8 : kMaxTeamBlocks;
  if (wide) K = blocks < kMaxWide ? blocks : kMaxWide;
  if (K < 1 || (int64_t)max_n > (int64_t)K * DBS * kDenseSlots) return hipSuccess;
  if (!wide) {
    int least = 1;  // where instances queue
    while (least < kDenseQueueBlocks && (int64_t)least * kDenseMostPerBlock < max_n) least *= 2;
    while (K > 1 && (int64_t)(K / 2) * kDensePerBlock >= max_n) K /= 2;
    while (K > least && K > 1 && blocks / (8 * K) * 8 < a.num_inst &&
           (int64_t)max_n <= (int64_t)(K / 2) * DBS * kDenseSlots)
      K /= 2;
  }
  int teams = wide ? 1 : blocks / (8 * K) * 8;
  if (teams > a.num_inst) teams = a.num_inst;
  if ((size_t)teams * (2 * K + 1) * 8 + 64 > (size_t)kMaxBlocks * kFlagStride * 4)
    return hipSuccess;
  DenseArgs q;
  q.K = K;
  q.teams = teams;
  q.words = (unsigned long long *)a.flags;
  q.queue = a.part;
  RoundArgs arg = a;
  void *params[] = {&arg, &q};
  if ((e = launch_kernel(L, (const void *)dense_init_kernel, dim3(1), dim3(256), params, false)) !=
      hipSuccess)
    return e;
  if (BATCH) {
    void *cargs[] = {&arg};
    if ((e = launch_kernel(L, (const void *)dense_counts_kernel,
                           dim3((unsigned)((a.num_inst + 255) / 256)), dim3(256), cargs,
                           false)) != hipSuccess)
      return e;
  }
  if (L.graph) timer = nullptr;
  if (timer && (e = hipEventRecord(timer->start, L.stream)) != hipSuccess) return e;
  const unsigned grid = wide ? (unsigned)K : (unsigned)((teams + 7) / 8) * 8u * (unsigned)K;
  const void *fn = wide ? (const void *)dense_rounds_kernel<V, BATCH, true>
                        : (const void *)dense_rounds_kernel<V, BATCH, false>;
  if ((e = launch_kernel(L, fn, dim3(grid), dim3(DBS), params, true)) != hipSuccess) return e;
  if (timer && (e = hipEventRecord(timer->stop, L.stream)) != hipSuccess) return e;
  *done = true;
  return hipSuccess;
}

hipError_t launch_dense(bool f32, bool batch, const RoundArgs &a, const LaunchGeom &geo,
                        int32_t max_n, const KernelTimer *timer, Launcher &L, bool *done) {
  if (f32)
    return batch ? launch_dense_t<KeyF32, true>(a, geo, max_n, timer, L, done)
                 : launch_dense_t<KeyF32, false>(a, geo, max_n, timer, L, done);
  return batch ? launch_dense_t<KeyI32, true>(a, geo, max_n, timer, L, done)
               : launch_dense_t<KeyI32, false>(a, geo, max_n, timer, L, done);
}

}  // namespace sssp
