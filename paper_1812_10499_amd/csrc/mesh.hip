// The rounds of solves on graphs of low degree spread (meshes, grids) under C
// scope OPEN, each by a team of W single-wave workgroups.  Such a solve has
// thousands of rounds of a few hundred relaxed vertices and a few thousand
// open ones: one workgroup is bound by its compute unit's memory pipeline
// (13 of 18 us a round on a 1024 x 1024 grid), the grid-wide kernel by its
// barriers and list windows.  Here a round takes 4.8 us: the chain of atomic,
// mailbox, word, D, vertex record, in-edges and C, each through the L2 or the
// Infinity Cache, one after another in some wave of every round (relax 2.2,
// waiting for the words 2.7, D and C 1.9, newcomers 2.6, fix 2.5, last wait
// 0.5 thousand cycles).  1024 x 1024 grid 80 -> 22.4 ms, 2048 x 2048 372 ->
// 78, 64 solves of a 512 x 512 grid 9.7 -> 7.5.
//
// Every vertex belongs to one wave of the team (a hash of its id).  An open
// vertex lives in a seat in its wave's registers from its discovery to its
// fix, with its lower bound, offsets and lightest in-edges, so a round reads
// only D and the tails' C for it.  What the waves share (D, C, the mailboxes,
// the words below) goes through agent-scope relaxed loads and atomics and the
// stores of team.h and nothing else, so no cache is written back or invalidated,
// wherever the waves run; the blocks are numbered so that a team shares an XCD's L2.
//
// A round of wave w:
//   relax the edges of its relax set; a first discovery goes to the owner's
//     mailbox for (w, owner), tagged with the round;
//   wait for its own stores, then publish (round, its minD and thr offers);
//   read all waves' words until all carry the round: the barrier, minD and
//     thr in one read (mailboxes are complete, and so is every D);
//   read D and the tails' C for the open seats and the mailboxes together,
//     seat the discoveries, publish "D read" (round);
//   bound and fix each seat (write C, build the next relax set);
//   read the "D read" words until all carry the round: only then may the
//     next relax change D.  C is double-buffered by round parity, as in the
//     other kernels, and every wave's reads of a buffer end before its next
//     publication, so its rewriting a round later needs no barrier of its
//     own.
// A mailbox or a wave's seats can fill up (large open sets).  The wave says so
// with its next word, the whole team leaves, and the one-workgroup kernel,
// launched behind this one, goes on with that instance at the bound step of
// the round that did not fit; it skips the others.  It finds nearly all it needs
// in memory.  What else a team left there as it goes (the counts before each
// bound step, the D of each relax) cost a 1024 x 1024 grid 2 to 4 % of its time,
// and so did the same exits without the hints on their likelihood: a wave is
// alone on its SIMD, and every jump on its way counts.
#include <atomic>

#include "sssp_dev.h"
#include "sssp_kernels.h"
#include "team.h"

namespace sssp {

constexpr int kMeshEdges = 4;  // lightest in-edges kept with a seat
constexpr int kBox = 16;       // mailbox entries per pair of waves and round
constexpr int kMeshLanes = 4;  // lanes that share a relax item's out-list
constexpr int32_t kGiveUp = 0;  // as minD: below every open vertex's D
constexpr int32_t kReadHit = 1, kReadFull = 2;  // target fixed; seats full

// The wave of the team that owns vertex y (W = 1 << lw): Murmur3's 32-bit
// finalizer (Appleby), low bits.  A plain multiplicative hash sends all the
// grid neighbours of one wave's vertices to a few waves and their mailboxes
// fill up.
__device__ __forceinline__ int mesh_owner(int32_t y, int lw) {
  uint32_t h = (uint32_t)y;
  h = (h ^ (h >> 16)) * 0x85EBCA6Bu;
  h = (h ^ (h >> 13)) * 0xC2B2AE35u;
  return (int)((h ^ (h >> 16)) & ((1u << lw) - 1u));
}

// Team words and mailboxes.  words: [teams][2][W]: offers, D read (round,
// flags).  box: [parity][teams][owner][entry][sender] of (round, vertex).
struct MeshArgs {
  int32_t lw, teams;
  unsigned long long *words, *box0, *box1;
  // per instance: the round the one-workgroup kernel goes on with (a mailbox was
  // full; negative: the seats were, and the round's bound step has run for the
  // vertices that had one), or 0
  int32_t *redo;
};

// D = INF, C = 0, the sources, empty words and mailboxes, the control block
// and the instances' counters.  Grid y: the instance.
template <class V, bool BATCH>
__global__ __launch_bounds__(256) void mesh_init_kernel(RoundArgs a, MeshArgs q) {
  const int inst = blockIdx.y;
  int32_t sb = 0, gi = 0, src = a.source, n = a.g.n;
  if constexpr (BATCH) {
    const InstDev id = a.insts[inst];
    sb = id.sbase;
    gi = id.graph;
    src = id.source;
    n = id.n;
  }
  const GraphDev &G = graph_of<BATCH>(a, gi);
  if (G.rank) src = G.rank[src];
  const int t0 = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
  for (int64_t y = t0; y < n; y += step) {
    const bool is_s = y == src;
    a.D64[sb + y] = make_key(is_s ? 0 : V::INF, -1, false);
    a.C0[sb + y] = a.C1[sb + y] = is_s ? V::INF : 0;  // the source is fixed from the start
    if (G.lc) a.DR[sb + y] = V::INF;
  }
  if (t0 == 0) {
    q.redo[inst] = 0;
    if constexpr (BATCH) {
      a.irounds[inst] = 0;
      for (int k = 0; k < 3; ++k) a.iscanned[3 * inst + k] = 0ull;
      if (a.istat)
        for (int k = 0; k < 4; ++k) a.istat[4 * inst + k] = 0;
    }
  }
  if (inst != 0) return;
  const int64_t W = (int64_t)1 << q.lw, words = 2 * W * q.teams, box = W * W * kBox * q.teams;
  for (int64_t i = t0; i < words; i += step) q.words[i] = 0ull;
  for (int64_t i = t0; i < box; i += step) q.box0[i] = q.box1[i] = 0ull;
  if (t0 == 0) {
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

template <int kSeatMax>
struct MeshLds {
  int4 rel[kSeatMax];  // relax set: vertex, D to relax from, out-offset, out-degree
  int32_t msg[kSeatMax];
  int32_t sent[SSSP_WAVE];  // mailbox entries written this round, by owner
};

// kSeats: open vertices per lane.
template <class V, bool BATCH, int kSeats>
__global__ __launch_bounds__(SSSP_WAVE) void mesh_rounds_kernel(RoundArgs a, MeshArgs q) {
  constexpr int kSeatMax = SSSP_WAVE * kSeats;
  __shared__ MeshLds<kSeatMax> s;
  const int l = lane_id(), lw = q.lw, W = 1 << lw;
  // team t runs on the blocks of one residue mod 8: blocks go round-robin to
  // the XCDs
  const int tb = blockIdx.x >> 3, team = (tb >> lw) * 8 + (int)(blockIdx.x & 7u);
  const int w = tb & (W - 1);
  if (team >= q.teams) return;
  unsigned long long *pub = q.words + (size_t)team * 2 * W, *read_d = pub + W;
  const size_t box_team = (size_t)W * W * kBox * team;
  unsigned long long *const box0 = q.box0 + box_team, *const box1 = q.box1 + box_team;
  const int lp = l < W ? l : 0;  // the wave whose words this lane reads
  unsigned ep = 1;               // rounds over all of the team's instances: the tag
  bool lost = false;
  // all "D read" words of this round: the union of their flags
  auto await_read = [&]() -> int32_t {
    unsigned long long x = 0;
    int spins = 0;
    do {
      x = ld_relaxed64(&read_d[lp]);
      lost = ++spins > kSpinLimit;
    } while (!lost && __ballot((int)((unsigned)(x >> 32) - ep) < 0));
    asm volatile("" ::: "memory");
    int32_t f = 0;
    if (__ballot((uint32_t)x & (uint32_t)kReadHit)) f |= kReadHit;
    if (__ballot((uint32_t)x & (uint32_t)kReadFull)) f |= kReadFull;
    return f;
  };
  // round 1 of the words: whether the team shares an XCD, and so an L2
  bool same = false;
  {
    const int32_t xcc = xcd_id();
    if (l == 0) put64(&pub[w], offers(ep, xcc + 1, 0), false);
    const unsigned long long x = await_offers(pub, lp, ep, &lost);
    same = __ballot(offers_md(x) != xcc + 1) == 0ull;
    if (l == 0) put64(&read_d[w], tagged(ep, 0), false);
    await_read();
    if (lost) {
      if (l == 0) atomicMax(&a.ctl->status, 7);
      return;
    }
  }
  for (int inst = team; inst < a.num_inst; inst += q.teams) {
    int32_t sb = 0, gi = 0, src = a.source, n = a.g.n;
    if constexpr (BATCH) {
      const InstDev id = a.insts[inst];
      sb = id.sbase;
      gi = id.graph;
      src = id.source;
      n = id.n;
    }
    const GraphDev G = graph_of<BATCH>(a, gi);
    const bool lc = G.lc != 0;
    int32_t tgt = BATCH ? -1 : a.target;
    if (G.rank) {
      src = G.rank[src];
      if (tgt >= 0) tgt = G.rank[tgt];
    }
    unsigned long long *D = a.D64 + sb;
    int32_t *C[2] = {a.C0 + sb, a.C1 + sb};
    // the seats: vertex (-1: free), C, D of the last relax, out_wmin, offsets
    // and degrees, the lightest in-edges
    int32_t y[kSeats], cy[kSeats], dr[kSeats], owm[kSeats], ioff[kSeats], ideg[kSeats];
    int32_t ooff[kSeats], odeg[kSeats], et[kSeats][kMeshEdges], ew[kSeats][kMeshEdges];
#pragma unroll
    for (int u = 0; u < kSeats; ++u) {
      y[u] = -1;
      cy[u] = dr[u] = owm[u] = ioff[u] = ideg[u] = ooff[u] = odeg[u] = 0;
#pragma unroll
      for (int e = 0; e < kMeshEdges; ++e) et[u][e] = ew[u][e] = 0;
    }
    int nF = 0;
    if (w == 0) {
      const int32_t o0 = G.out_off[src];
      if (l == 0) s.rel[0] = make_int4(src, 0, o0, G.out_off[src + 1] - o0);
      nF = 1;
    }
    __syncthreads();
    // this lane's counts, and its survivors' offers to minD and thr
    unsigned long long nrel = 0, nscan = 0;
    uint32_t nvis = 0, nfix = 0;
    int32_t smd = V::INF, sth = V::INF;
    bool full = false, hit = tgt >= 0 && tgt == src;
    int r = 0, status = 0, gave_up = 0;
    // the first edge of this lane's first relax item, read ahead
    int4 er = make_int4(0, 0, 0, 0);
    bool ahead = false;
    for (;;) {
      if (__builtin_expect(hit, 0)) break;  // the frontier that fixed the target is not relaxed
      ++r;
      ++ep;
      if (__builtin_expect(r > n + 1 || r > a.max_rounds, 0)) {  // (every wave alike)
        status = 7;
        break;
      }
      const int cur = r & 1;  // the bound step reads C[cur] and writes C[cur ^ 1]
      int32_t *Cold = C[cur], *Cnew = C[cur ^ 1];
      unsigned long long *box = cur ? box1 : box0;
      // (A) relax, each item from its D at the start of the step (bit 31: an
      // open vertex, label-correcting; INF: already relaxed at this D)
      int32_t md = smd, th = sth;
      if (nF) {
        s.sent[l] = 0;
        __syncthreads();
        for (int i0 = 0; i0 < nF; i0 += SSSP_WAVE / kMeshLanes) {
          const int i = i0 + l / kMeshLanes, e0 = l % kMeshLanes;
          int4 f = make_int4(0, V::INF, 0, 0);
          if (i < nF) f = s.rel[i];
          const int32_t dx = f.y & 0x7fffffff;
          const int32_t deg = i < nF && dx != V::INF ? f.w : 0;
          if (e0 == 0) nrel += (unsigned long long)deg;
          for (int32_t k = e0; k < deg; k += kMeshLanes) {
            // head, weight, edge id, the head's out_wmin
            if (__builtin_expect(i0 > 0 || k != e0 || !ahead, 0)) er = G.out_rec[f.z + k];
            const int32_t cand = V::add(dx, er.y);
            const unsigned long long old =
                atomicMin(&D[er.x], make_key(cand, er.z, cand == dx));
            const int32_t od = (int32_t)(old >> 32);
            if (cand < od) {  // D fell: offer it to minD and thr
              md = kmin(md, cand);
              th = kmin(th, V::add(cand, er.w));
            }
            if (od == V::INF) {  // a first discovery
              const int o = mesh_owner(er.x, lw);
              const int p = atomicAdd(&s.sent[o], 1);
              if (__builtin_expect(p < kBox, 1))
                put64(&box[((size_t)o * kBox + p) * W + w], tagged(ep, er.x), same);
              else full = true;
            }
          }
        }
      }
      md = __ballot(full) ? kGiveUp : wave_min(md);
      th = wave_min(th);
      stores_done();
      if (l == 0) put64(&pub[w], offers(ep, md, th), same);
      {
        const unsigned long long x = await_offers(pub, lp, ep, &lost);
        md = wave_min(offers_md(x));
        th = wave_min(offers_th(x));
      }
      if (__builtin_expect(lost, 0)) break;
      if (__builtin_expect(md == kGiveUp || md == V::INF, 0)) {  // (every wave alike)
        gave_up = md == kGiveUp ? r : 0;
        // the words are rewritten by the team's next instance: only after
        // every wave has read them
        if (l == 0) put64(&read_d[w], tagged(ep, 0), same);
        await_read();
        break;
      }
      // (B) done: md and th are minD and the threshold.  D and the tails' C
      // of the open seats, and the first two entries of every mailbox
      unsigned long long dk[kSeats], m0, m1;
      int32_t cv[kSeats][kMeshEdges];
      {
        const size_t at = (size_t)w * kBox * W + lp;
        m0 = ld_relaxed64(&box[at]);
        m1 = ld_relaxed64(&box[at + W]);
      }
#pragma unroll
      for (int u = 0; u < kSeats; ++u) {
        dk[u] = 0;
#pragma unroll
        for (int e = 0; e < kMeshEdges; ++e) cv[u][e] = V::INF;
        if (__ballot(y[u] >= 0)) {
          dk[u] = ld_relaxed64(&D[y[u] >= 0 ? y[u] : 0]);
#pragma unroll
          for (int e = 0; e < kMeshEdges; ++e) cv[u][e] = ld_relaxed(&Cold[et[u][e]]);
        }
      }
      // the discoveries, gathered in LDS
      int nmsg = 0;
      {
        bool v0 = l < W && (unsigned)(m0 >> 32) == ep, v1 = l < W && (unsigned)(m1 >> 32) == ep;
        const uint64_t b0 = __ballot(v0), b1 = __ballot(v1);
        const uint64_t lt = (1ull << l) - 1ull;
        if (v0) s.msg[__popcll(b0 & lt)] = (int32_t)(uint32_t)m0;
        nmsg = __popcll(b0);
        if (v1) s.msg[nmsg + __popcll(b1 & lt)] = (int32_t)(uint32_t)m1;
        nmsg += __popcll(b1);
        for (int k = 2; k < kBox && __builtin_expect(__ballot(v1) != 0ull, 0); ++k) {
          const unsigned long long m = ld_relaxed64(&box[((size_t)w * kBox + k) * W + lp]);
          v1 = v1 && (unsigned)(m >> 32) == ep;
          const uint64_t b = __ballot(v1);
          const int p = nmsg + __popcll(b & lt);
          if (v1 && p < kSeatMax) s.msg[p] = (int32_t)(uint32_t)m;
          nmsg += __popcll(b);
        }
      }
      bool fresh[kSeats];
      {
        __syncthreads();
        int taken = 0;
#pragma unroll
        for (int u = 0; u < kSeats; ++u) {
          fresh[u] = false;
          const uint64_t fm = __ballot(y[u] < 0);
          if (taken < nmsg && fm) {  // (wave-uniform)
            const int p = taken + __popcll(fm & ((1ull << l) - 1ull));
            fresh[u] = y[u] < 0 && p < nmsg && p < kSeatMax;
            if (fresh[u]) {
              y[u] = s.msg[p];
              dk[u] = ld_relaxed64(&D[y[u]]);
              const int4 ra = G.vrec[2 * y[u]], rb = G.vrec[2 * y[u] + 1];
              ooff[u] = ra.x;
              odeg[u] = ra.y;
              ioff[u] = ra.z;
              ideg[u] = ra.w;
              owm[u] = rb.x;
              et[u][0] = rb.y;
              ew[u][0] = ra.w > 0 ? rb.z : V::INF;
              cy[u] = 0;       // C of an undiscovered vertex
              dr[u] = V::INF;  // never relaxed
            }
            taken += __popcll(fm);
          }
        }
        full = taken < nmsg;
      }
      // the rest of the newcomers' lightest in-edges, then their tails' C
#pragma unroll
      for (int u = 0; u < kSeats; ++u) {
        if (fresh[u]) {
#pragma unroll
          for (int e = 1; e < kMeshEdges; ++e) {
            const int2 x = e < ideg[u] ? G.in_sw[ioff[u] + e] : make_int2(0, V::INF);
            et[u][e] = x.x;
            ew[u][e] = x.y;
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kSeats; ++u) {
        if (fresh[u]) {
#pragma unroll
          for (int e = 0; e < kMeshEdges; ++e) cv[u][e] = ld_relaxed(&Cold[et[u][e]]);
        }
      }
#pragma unroll
      for (int u = 0; u < kSeats; ++u) asm volatile("" : "+v"(dk[u]));  // every D has arrived
      if (tgt < 0 && l == 0) put64(&read_d[w], tagged(ep, full ? kReadFull : 0), same);
      // vertices fixed last round: C = INF in this round's buffer too
      for (int i = l; i < nF; i += SSSP_WAVE) {
        const int4 f = s.rel[i];
        if (f.y >= 0) put(&Cnew[f.x], V::INF, same);
      }
      __syncthreads();
      // (C) lower bounds (Eq. 1), Jacobi, and (D) fix, seat by seat.  An
      // in-edge with minD + w >= D[y] cannot lower C'[y]; in-lists ascend by
      // weight.
      smd = sth = V::INF;
      nF = 0;
      bool hit_now = false;
#pragma unroll
      for (int u = 0; u < kSeats; ++u) {
        if (!__ballot(y[u] >= 0)) continue;
        bool push = false;
        int32_t fd = 0;
        const int32_t x = y[u];
        if (x >= 0) {
          const int32_t dy = (int32_t)(dk[u] >> 32);
          int32_t m = V::INF;
#pragma unroll
          for (int e = 0; e < kMeshEdges; ++e)
            if (cv[u][e] != V::INF && V::add(md, ew[u][e]) < dy)
              m = kmin(m, V::add(kmax(cv[u][e], md), ew[u][e]));
          if (__builtin_expect(ideg[u] > kMeshEdges, 0) &&
              V::add(md, ew[u][kMeshEdges - 1]) < kmin(dy, m)) {
            for (int32_t j = kMeshEdges; j < ideg[u]; ++j) {
              const int2 e = G.in_sw[ioff[u] + j];  // tail, weight
              if (V::add(md, e.y) >= kmin(dy, m)) break;
              const int32_t c = ld_relaxed(&Cold[e.x]);
              if (c != V::INF) m = kmin(m, V::add(kmax(c, md), e.y));
            }
          }
          const int32_t cn = kmax(kmax(cy[u], md), kmin(dy, m));
          nscan += (unsigned long long)ideg[u];
          ++nvis;
          const bool relax_again = !lc || dy < dr[u];
          if (cn >= dy || dy <= th) {
            put(&Cnew[x], V::INF, same);
            ++nfix;
            hit_now |= x == tgt;
            push = true;
            fd = relax_again ? dy : V::INF;
            y[u] = -1;
          } else {
            put(&Cnew[x], cn, same);
            cy[u] = cn;
            smd = kmin(smd, dy);
            sth = kmin(sth, V::add(dy, owm[u]));
            // label-correcting: relaxed again from its lower D (while in the
            // first bucket above minD)
            if (lc && relax_again && dy < V::add(md, G.delta)) {
              push = true;
              fd = dy | kOpenRelax;
              dr[u] = dy;
            }
          }
        }
        const uint64_t pm = __ballot(push);
        if (push)
          s.rel[nF + __popcll(pm & ((1ull << l) - 1ull))] = make_int4(x, fd, ooff[u], odeg[u]);
        nF += __popcll(pm);
      }
      __syncthreads();
      // the next relax's first edges, on their way during the wait below
      {
        const int i = l / kMeshLanes, e = l % kMeshLanes;
        ahead = false;
        if (i < nF) {
          const int4 f = s.rel[i];
          ahead = (f.y & 0x7fffffff) != V::INF && e < f.w;
          if (ahead) er = G.out_rec[f.z + e];
        }
      }
      if (tgt >= 0) {
        const bool h = __ballot(hit_now) != 0ull;
        if (l == 0)
          put64(&read_d[w], tagged(ep, (h ? kReadHit : 0) | (full ? kReadFull : 0)), same);
      }
      const int32_t flags = await_read();
      if (__builtin_expect(lost, 0)) break;
      if (__builtin_expect((flags & kReadFull) != 0, 0)) {
        gave_up = -r;
        break;
      }
      hit = (flags & kReadHit) != 0;
    }
    if (lost) {
      if (l == 0) atomicMax(&a.ctl->status, 7);
      return;
    }
    if (w == 0 && l == 0) q.redo[inst] = gave_up;
    if (__builtin_expect(gave_up != 0 && lc, 0)) {
      // DR: the D that each open vertex was last relaxed with.  The seats have
      // it, and for a vertex that this round's bound step put into the relax set,
      // which is to decide again, INF or 0 (above its D, or not) does.
      // (its address is read from the kernel's arguments here: kept over the
      // rounds in scalar registers it would push the loop's own out of them)
      const RoundArgs *args = (const RoundArgs *)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(args));
      int32_t *DR = args->DR + sb;
#pragma unroll
      for (int u = 0; u < kSeats; ++u)
        if (y[u] >= 0) put(&DR[y[u]], dr[u], same);
      stores_done();
      if (gave_up < 0) {
        for (int i = l; i < nF; i += SSSP_WAVE) {
          const int4 f = s.rel[i];
          put(&DR[f.x], f.y != V::INF ? V::INF : 0, same);
        }
      }
    }
    const long long v0 = wave_sum64((long long)nrel), v1 = wave_sum64((long long)nscan);
    const long long v2 = wave_sum64((long long)nvis), v3 = wave_sum64((long long)nfix);
    if (l == 0) {
      if constexpr (BATCH) {
        atomicAdd(&a.iscanned[3 * inst], (unsigned long long)v1);
        atomicAdd(&a.iscanned[3 * inst + 1], (unsigned long long)v2);
        atomicAdd(&a.iscanned[3 * inst + 2], (unsigned long long)v0);
        if (w == 0) {
          a.irounds[inst] = r;
          if (status) atomicMax(&a.ctl->status, status);
        }
      } else {
        Ctl *c = a.ctl;
        atomicAdd((unsigned long long *)&c->relaxed, (unsigned long long)v0);
        atomicAdd((unsigned long long *)&c->scanned, (unsigned long long)v1);
        atomicAdd((unsigned long long *)&c->open_visits, (unsigned long long)v2);
        // the source is settled too
        atomicAdd((unsigned long long *)&c->settled, (unsigned long long)(v3 + (w == 0 ? 1 : 0)));
        if (w == 0) {
          c->rounds = r;
          c->status = status;
          c->target_id = tgt;
          c->target_hit = hit ? 1 : 0;
        }
      }
    }
  }
}

// Waves per team: one per kMeshPerWave vertices, and more while all teams
// together have at most kMeshRoomy (six a compute unit): they hold wider open
// sets, and cost little.  Single solves on 8, 16, 32 waves and in one
// workgroup: 70 x 70 grid 733, 694, 675, 883 us; 20^3 mesh 936 (gives up), 564,
// 482, 723; random 3-regular on 5000 vertices 333 (gives up), 352 (gives up),
// 165, 244.  48 solves: 66 x 66 grid 973, 965, 998, 1104, 96 x 96 1500, 1476,
// 1505, 1730, 3-regular on 5000 vertices 369, 355, 299, 303, on 9000 556, 534, 493,
// 484.  64: 977, 1002, 1060, 1116; 1515, 1524, 1566, 1736; 369, 356, 316, 304; 570,
// 558, 518, 500.  (Whether an open set will fit cannot be told beforehand: small
// graphs without a planar grid's structure lose up to a fourth from 49 instances
// on, grids gain a tenth to a third.)  Wide graphs get all there is room for: 32
// solves of 5000 vertices 8-regular on 16 and 32 waves 437 and 303, 395 in one
// workgroup each.
// At most 64 (a lane reads one wave's words; a 1024 x 1024 grid takes 22.4 ms on
// 64, 27.8 on 32).  All teams together kMeshWavesPerCu waves per compute unit: 64
// solves of a 384 x 384 grid take 4.8 ms at 8, 5.3 at 4 and 11.5 at 2 (seats fill
// up), 5.8 in one workgroup each.
constexpr int32_t kMeshPerWave = 512;
constexpr int kMeshRoomy = 1536;
// Wide graphs: four seats a lane, and beyond this many instances, whose teams
// would be small, a workgroup each.  Against one workgroup each (and two seats):
// one 50^3 mesh 11.3 -> 3.4 ms (6.9), 15^4 5.3 -> 1.4 (4.5), 5000 vertices
// 8-regular 364 -> 221 us (378), 20000 5-regular 1.15 -> 0.32 ms (1.04), a 128 x
// 128 grid with diagonals 2.5 -> 2.0 (1.9); sets that do not fit either way, an
// 80^3 mesh 60.7 -> 43.6 (56.6), 100000 6-regular 8.6 -> 8.5 (8.7).  32 of them
// 14.9 -> 4.8, 7.2 -> 2.1, 0.40 -> 0.30, 1.76 -> 1.1, 2.5 -> 2.2, 75.8 -> 65.8 and
// 11.1 -> 10.8 ms.  64 and 128: 50^3 mesh 16.6 -> 17.9 and 21.1 -> 21.9, 32^3 3.6 ->
// 2.2 and 4.0 -> 5.2.  Graphs of more than 16 edges a vertex (MESH_NONE): 5000
// vertices of degree 40 1.31 -> 0.57, but 32 of them 1.46 -> 2.17, and 4 of
// degree 256 7.3 -> 9.7.
constexpr int kMeshWideMost = 32;
constexpr int kMeshWavesPerCu = 8;

// Teams for this solve, or false: the one-workgroup kernel takes it.
template <class V, bool BATCH>
static bool mesh_plan(const RoundArgs &a, const LaunchGeom &geo, int32_t max_n, MeshArgs &q,
                      int *seats, hipError_t *err) {
  static std::atomic<int> known{0};  // co-resident blocks per compute unit
  int occ = known.load();
  if (occ == 0) {
    *err = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &occ, (const void *)mesh_rounds_kernel<V, BATCH, 4>, SSSP_WAVE, 0);
    if (*err != hipSuccess || occ < 1) return false;
    known.store(occ);
  }
  // More instances than half the compute units: a workgroup each fills the
  // chip with less traffic (256 solves of a 256 x 256 grid: 4.4 ms there, 7.7
  // in teams; 128 of them: 3.6 and 3.3).
  if (2 * a.num_inst > geo.cus) return false;
  if (a.mesh == MESH_NONE || (a.mesh == MESH_WIDE && a.num_inst > kMeshWideMost)) return false;
  const int per_cu = occ < kMeshWavesPerCu ? occ : kMeshWavesPerCu;
  const int64_t blocks = (int64_t)per_cu * (geo.blocks < geo.cus ? geo.blocks : geo.cus);
  // the redo words lie in the per-block partials, the team words in the
  // barrier flags, the mailboxes in the open lists' payload
  if (a.num_inst > kParts * kMaxBlocks) return false;
  if (max_n < 2 * kMeshPerWave) return false;
  int lw = 0;
  while (lw < 6 && (a.mesh == MESH_WIDE || ((int64_t)2 << lw) * kMeshPerWave <= (int64_t)max_n ||
                    ((int64_t)2 << lw) * a.num_inst <= kMeshRoomy))
    ++lw;
  for (; lw >= 1; --lw) {
    const int64_t W = (int64_t)1 << lw;
    int64_t teams = blocks / (8 * W) * 8;  // whole sets of eight teams
    if (teams > a.num_inst) teams = a.num_inst;
    if (teams < a.num_inst) continue;  // smaller teams, one per instance
    if (teams * W * W * kBox * 8 > (int64_t)kOXMem * 4 * a.total) continue;
    if (2 * W * teams * 8 > (int64_t)kMaxBlocks * kFlagStride * 4) continue;
    q.lw = lw;
    q.teams = (int32_t)teams;
    q.words = (unsigned long long *)a.flags;
    q.box0 = (unsigned long long *)a.open_x0[0];
    q.box1 = (unsigned long long *)a.open_x1[0];
    q.redo = a.part;
    // two seats a lane where a wavefront of about 4 sqrt(n) open vertices fills at
    // most 3/5 of them (four: a 1024 x 1024 grid takes 26.7 ms, not 25.6).  Where
    // four would not hold the estimate, the team still gains until it is outgrown:
    // 4096 x 4096 (16384 estimated, 64 x 256 seats) fits and takes 0.25 s, 1.56 in
    // one workgroup, 8192 x 8192 4.73 before, 4.80 with the team's work lost.
    const double room = 0.6 * 2 * SSSP_WAVE * W;
    *seats = a.mesh == MESH_FLAT && 16.0 * max_n <= room * room ? 2 : 4;
    return true;
  }
  return false;
}

template <class V, bool BATCH>
static hipError_t launch_mesh_t(const RoundArgs &a, const LaunchGeom &geo, int32_t max_n,
                                const KernelTimer *timer, Launcher &L, const int32_t **redo) {
  *redo = nullptr;
  hipError_t e = hipSuccess;
  MeshArgs q;
  int seats = 4;
  if (a.scope_all || !mesh_plan<V, BATCH>(a, geo, max_n, q, &seats, &e)) return e;
  RoundArgs arg = a;
  void *params[] = {&arg, &q};
  int bx = (max_n + 1023) / 1024;
  if (bx > 2048) bx = 2048;
  if ((e = launch_kernel(L, (const void *)mesh_init_kernel<V, BATCH>,
                         dim3((unsigned)bx, (unsigned)a.num_inst), dim3(256), params, false)) !=
      hipSuccess)
    return e;
  if (L.graph) timer = nullptr;
  if (timer && (e = hipEventRecord(timer->start, L.stream)) != hipSuccess) return e;
  const unsigned grid = (unsigned)(((q.teams + 7) / 8) << q.lw) * 8u;
  const void *fn = seats == 2 ? (const void *)mesh_rounds_kernel<V, BATCH, 2>
                              : (const void *)mesh_rounds_kernel<V, BATCH, 4>;
  if ((e = launch_kernel(L, fn, dim3(grid), dim3(SSSP_WAVE), params, true)) != hipSuccess)
    return e;
  *redo = q.redo;
  return hipSuccess;
}

// (the timer is stopped behind launch_wg, which may have a part of the rounds)
hipError_t launch_mesh(bool f32, bool batch, const RoundArgs &a, const LaunchGeom &geo,
                       int32_t max_n, const KernelTimer *timer, Launcher &L,
                       const int32_t **redo) {
  if (f32)
    return batch ? launch_mesh_t<KeyF32, true>(a, geo, max_n, timer, L, redo)
                 : launch_mesh_t<KeyF32, false>(a, geo, max_n, timer, L, redo);
  return batch ? launch_mesh_t<KeyI32, true>(a, geo, max_n, timer, L, redo)
               : launch_mesh_t<KeyI32, false>(a, geo, max_n, timer, L, redo);
}

}  // namespace sssp
