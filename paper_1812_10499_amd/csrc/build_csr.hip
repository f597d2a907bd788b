// Graph builder on gfx950: COO edges -> CSR by tail (stable: the edges of a
// tail keep their input order; edge id = CSR position) and CSC by head over
// edge ids in increasing order (so every in-list is ascending by edge id).
// This is the incoming-edge access the method assumes, built once per
// graph; out_wmin is the per-vertex minimum out-edge weight (outWeight of
// Figs. 5 and 6).
//
// The solver's working copy: an optional renumbering by descending total
// degree (CSR copy, vid/rank), and always a CSC whose in-lists are ascending
// by weight.  The lower-bound step only needs the in-edges (v, y, w) with
// minD + w < D[y]; with weight-ordered in-lists they are a prefix of y's
// list whose length one binary search finds.
//
// Sorting: LSD radix sort of rows of up to four int32 columns, one of them
// the key (sort_rows below).  No atomics decide any order.
#include "sssp_dev.h"
#include "sssp_kernels.h"

namespace sssp {

constexpr int SCAN_BS = 256;
constexpr int SCAN_PT = 16;
constexpr int SCAN_TILE = SCAN_BS * SCAN_PT;

enum : int32_t { BAD_GRAPH = 1, BAD_WEIGHT = 2 };

static inline int grid_for(int64_t work) {
  int64_t b = (work + 255) / 256;
  if (b < 1) b = 1;
  if (b > 16384) b = 16384;
  return (int)b;
}

// -------------------------------------------------------------- validate
// status: [0] error flags, [1] largest weight key, [2] largest total degree,
// [3] INT32_MAX minus the smallest weight key (a maximum, so the zeroed word
// is its identity), [4] largest in-degree
// One atomic per block and word, and few blocks: every thread issuing its own
// on the same words took 763 us at 16.8 M edges, a block of 256 threads each
// 99 us (27 us at 0.8 M, most of it those atomics).
constexpr int kCheckThreads = 1024;
constexpr int kCheckBlocks = 512;

struct CheckAcc {
  int32_t bad = 0, wmax = 0, wmin_c = 0, ideg = 0;
};

template <bool ENDS>
__device__ __forceinline__ void check_edges(CheckAcc &c, int32_t n, int64_t m, int f32,
                                            const int32_t *src, const int32_t *dst,
                                            const int32_t *w, int64_t t0, int64_t stride) {
  constexpr int U = 4;
  for (int64_t i0 = t0; i0 < m; i0 += U * stride) {
    int32_t k[U], s[U], d[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // past the end: the thread's first edge again
      const int64_t i = i0 + u * stride < m ? i0 + u * stride : i0;
      k[u] = w[i];
      s[u] = ENDS ? src[i] : 0;
      d[u] = ENDS ? dst[i] : 0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (ENDS && (s[u] < 0 || s[u] >= n || d[u] < 0 || d[u] >= n)) c.bad |= BAD_GRAPH;
      // int32: w >= 1.  float32 key: w > 0 and finite  <=>  0 < bits < 0x7f800000
      if (f32 ? (k[u] <= 0 || k[u] >= 0x7f800000) : (k[u] < 1)) {
        c.bad |= BAD_WEIGHT;
      } else {
        c.wmax = kmax(c.wmax, k[u]);
        c.wmin_c = kmax(c.wmin_c, 0x7fffffff - k[u]);
      }
    }
  }
}

__global__ __launch_bounds__(kCheckThreads) void validate_kernel(int32_t n, int32_t m, int f32,
                                                                 const int32_t *src,
                                                                 const int32_t *dst,
                                                                 const int32_t *w,
                                                                 const int32_t *in_off,
                                                                 int32_t *status) {
  constexpr int NW = kCheckThreads / SSSP_WAVE;
  __shared__ int32_t red[4][NW];
  CheckAcc c;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (src) check_edges<true>(c, n, m, f32, src, dst, w, t0, stride);
  else check_edges<false>(c, n, m, f32, src, dst, w, t0, stride);
  if (in_off)
    for (int64_t v = t0; v < n; v += stride) c.ideg = kmax(c.ideg, in_off[v + 1] - in_off[v]);
  // whole waves arrive here together; bad is a set of two flags
  const int32_t bad = (__ballot(c.bad & BAD_GRAPH) ? BAD_GRAPH : 0) |
                      (__ballot(c.bad & BAD_WEIGHT) ? BAD_WEIGHT : 0);
  const int32_t wmax = wave_max(c.wmax), wmin_c = wave_max(c.wmin_c), ideg = wave_max(c.ideg);
  const int wv = threadIdx.x / SSSP_WAVE;
  if (lane_id() == 0) {
    red[0][wv] = bad;
    red[1][wv] = wmax;
    red[2][wv] = wmin_c;
    red[3][wv] = ideg;
  }
  __syncthreads();
  if (threadIdx.x < 4) {  // one word each
    const int q = threadIdx.x;
    int32_t x = red[q][0];
    for (int k = 1; k < NW; ++k) x = q == 0 ? (x | red[q][k]) : kmax(x, red[q][k]);
    const int32_t slot = q == 0 ? 0 : (q == 1 ? 1 : (q == 2 ? 3 : 4));
    if (q == 0 && x) atomicOr(&status[slot], x);
    if (q != 0 && x > ld_relaxed(&status[slot])) atomicMax(&status[slot], x);
  }
}

hipError_t launch_validate(int32_t n, int32_t m, bool f32, const int32_t *src,
                           const int32_t *dst, const int32_t *w, const int32_t *in_off,
                           int32_t *status, hipStream_t stream) {
  const int64_t work = in_off && n > m ? n : m;
  int64_t blocks = (work + 4 * kCheckThreads - 1) / (4 * kCheckThreads);
  if (blocks < 1) blocks = 1;
  if (blocks > kCheckBlocks) blocks = kCheckBlocks;
  hipLaunchKernelGGL(validate_kernel, dim3((unsigned)blocks), dim3(kCheckThreads), 0, stream, n,
                     m, f32 ? 1 : 0, src, dst, w, in_off, status);
  return hipGetLastError();
}

// ------------------------------------------------------------------ scan
// exclusive prefix sum of int32 data[L] in place, three passes
__global__ void scan_reduce_kernel(const int32_t *data, int32_t L, int32_t *sums) {
  __shared__ uint64_t sc[SCAN_BS / SSSP_WAVE + 1];
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
  int32_t s = 0;
  for (int j = 0; j < SCAN_PT; ++j) {
    const int64_t i = base + (int64_t)j * SCAN_BS + threadIdx.x;
    if (i < L) s += data[i];
  }
  uint64_t tot;
  block_excl_scan64<SCAN_BS>((uint64_t)(uint32_t)s, sc, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = (int32_t)tot;
}

__global__ void scan_sums_kernel(int32_t *sums, int32_t ns) {
  __shared__ uint64_t sc[SCAN_BS / SSSP_WAVE + 1];
  uint64_t run = 0;
  for (int b0 = 0; b0 < ns; b0 += SCAN_BS) {
    const int i = b0 + threadIdx.x;
    const uint32_t v = i < ns ? (uint32_t)sums[i] : 0u;
    uint64_t tot;
    const uint64_t ex = block_excl_scan64<SCAN_BS>((uint64_t)v, sc, &tot);
    if (i < ns) sums[i] = (int32_t)(run + ex);
    run += tot;
  }
}

__global__ void scan_apply_kernel(int32_t *data, int32_t L, const int32_t *sums) {
  __shared__ uint64_t sc[SCAN_BS / SSSP_WAVE + 1];
  const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
  // each thread owns SCAN_PT consecutive elements
  int32_t v[SCAN_PT];
  int32_t s = 0;
  const int64_t mine = base + (int64_t)threadIdx.x * SCAN_PT;
  for (int j = 0; j < SCAN_PT; ++j) {
    const int64_t i = mine + j;
    v[j] = i < L ? data[i] : 0;
    s += v[j];
  }
  uint64_t tot;
  const uint64_t ex = block_excl_scan64<SCAN_BS>((uint64_t)(uint32_t)s, sc, &tot);
  int32_t run = sums[blockIdx.x] + (int32_t)ex;
  for (int j = 0; j < SCAN_PT; ++j) {
    const int64_t i = mine + j;
    if (i < L) data[i] = run;
    run += v[j];
  }
}

static hipError_t exclusive_scan(int32_t *data, int32_t L, int32_t *sums, hipStream_t stream) {
  const int nb = (L + SCAN_TILE - 1) / SCAN_TILE;
  hipLaunchKernelGGL(scan_reduce_kernel, dim3(nb), dim3(SCAN_BS), 0, stream, data, L, sums);
  hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(SCAN_BS), 0, stream, sums, nb);
  hipLaunchKernelGGL(scan_apply_kernel, dim3(nb), dim3(SCAN_BS), 0, stream, data, L, sums);
  return hipGetLastError();
}

// ------------------------------------------------------------ radix sort
// One pass sorts m rows of NC int32 columns stably by one digit of the key
// column: a histogram of the digit per tile, an exclusive scan of every
// digit's counts over the tiles, and a scatter.  The scatter block ranks its
// tile's rows (64-lane ballots per digit bit, per-wave digit counts in LDS),
// sorts each column through LDS and writes runs of equal digits, so a row's
// columns travel with it and nothing is gathered afterwards.
//
// What bounds it: the memory traffic, 8 NC bytes per row and pass plus 4 for
// the histogram, and how well the scattered runs meet in the L2s.  Digits of
// up to 11 bits (2048 bins) sort any vertex id below 2^22 in two passes; a
// tile of 16384 rows leaves runs of 8 to 16 rows per bin.  One block per
// compute unit: two (half the registers) leave twice as many lines open, and
// a pass over 16.8 M rows of four columns takes 322 us instead of 156 (3.4
// TB/s; a tile of 8192 rows: 167 us, and twice the counts to scan).  The same
// rows carried as (key, row number) pairs and gathered at the end took 175 us
// a pass and 0.6 to 0.9 ms for each gather.  Below 4 M rows tiles of 4096
// keep the chip's 256 compute units busy (13 us a pass at 0.8 M rows).
constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / SSSP_WAVE;
constexpr int kMaxDigit = 11;
constexpr int32_t kBigSort = 1 << 22;  // from here tiles of kBigRows rows per thread
constexpr int kBigRows = 16;

static inline int sort_rows_per_thread(int32_t m) { return m >= kBigSort ? kBigRows : 4; }
static inline int64_t sort_tiles(int32_t m) {
  const int64_t tile = (int64_t)kSortThreads * sort_rows_per_thread(m);
  return ((int64_t)m + tile - 1) / tile;
}

size_t build_hist_entries(int32_t n, int32_t m) {
  // rows of m edges or n vertices (a large m may have fewer, larger tiles)
  const size_t tm = (size_t)sort_tiles(m > 0 ? m : 1), tn = (size_t)sort_tiles(n > 0 ? n : 1);
  const size_t t = tm > tn ? tm : tn;
  const size_t sums = ((size_t)n + 1 + SCAN_TILE - 1) / SCAN_TILE + 64;
  return (t + 1) * (1u << kMaxDigit) + sums;
}

template <int NC>
struct SortCols {
  const int32_t *in[NC];  // null: the row number
  int32_t *out[NC];       // null: not written
};

// hist[tile * bins + digit]
template <int RK>
__global__ __launch_bounds__(kSortThreads) void sort_hist_kernel(const int32_t *keys, int32_t m,
                                                                 int shift, int bits,
                                                                 int32_t *hist) {
  __shared__ int32_t h[1 << kMaxDigit];
  const int bins = 1 << bits;
  for (int b = threadIdx.x; b < bins; b += kSortThreads) h[b] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * (kSortThreads * RK);
  int32_t k[RK];
#pragma unroll
  for (int j = 0; j < RK; ++j) {
    const int64_t i = base + j * kSortThreads + threadIdx.x;
    k[j] = i < m ? keys[i] : 0;
  }
#pragma unroll
  for (int j = 0; j < RK; ++j) {
    const int64_t i = base + j * kSortThreads + threadIdx.x;
    if (i < m) atomicAdd(&h[(k[j] >> shift) & (bins - 1)], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < bins; b += kSortThreads)
    hist[(int64_t)blockIdx.x * bins + b] = h[b];
}

// Exclusive prefix of every digit's counts over the tiles, in place, and the
// digit totals: block b takes 16 digits, 64 threads share a digit's tiles.
__global__ __launch_bounds__(1024) void sort_scan_kernel(int32_t *hist, int bins, int64_t tiles,
                                                         int32_t *totals) {
  __shared__ int32_t part[64][16];
  const int c = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int b = blockIdx.x * 16 + c;
  const int64_t per = (tiles + 63) / 64, t0 = g * per;
  const int64_t t1 = t0 + per < tiles ? t0 + per : tiles;
  int32_t s = 0;
  if (b < bins)
    for (int64_t t = t0; t < t1; ++t) s += hist[t * bins + b];
  part[g][c] = s;
  __syncthreads();
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t v = g >= d ? part[g - d][c] : 0;
    __syncthreads();
    part[g][c] += v;
    __syncthreads();
  }
  int32_t run = part[g][c] - s;
  if (b >= bins) return;
  if (g == 63) totals[b] = run + s;
  for (int64_t t = t0; t < t1; ++t) {
    const int32_t v = hist[t * bins + b];
    hist[t * bins + b] = run;
    run += v;
  }
}

// Blocks go round-robin to the 8 XCDs; each XCD takes a contiguous range of
// the tiles, so that the runs neighbouring tiles append to one digit meet in
// one L2 and leave it as whole lines.
constexpr unsigned kXcds = 8;
__device__ __forceinline__ int64_t sort_tile_of(unsigned b, unsigned tiles) {
  const unsigned x = b % kXcds, q = b / kXcds, per = tiles / kXcds, more = tiles % kXcds;
  return (int64_t)x * per + (x < more ? x : more) + q;
}

// KC: the key column.
template <int RK, int NC, int KC>
__global__ __launch_bounds__(kSortThreads) void sort_scatter_kernel(SortCols<NC> cols, int32_t m,
                                                                    int shift, int bits,
                                                                    const int32_t *hist,
                                                                    const int32_t *totals) {
  constexpr int TILE = kSortThreads * RK;
  constexpr int kBins = 1 << kMaxDigit;
  // per-wave digit counts while ranking, then the column being reordered
  __shared__ union {
    uint16_t wcnt[kSortWaves][kBins];
    int32_t buf[TILE];
  } u;
  // where a digit's rows start in the sorted tile, and their global position
  // minus that place (the scan's scratch lies there before)
  __shared__ union {
    int32_t at[2][kBins];
    uint64_t scan[kSortWaves + 1];
  } dg;
  int32_t *lstart = dg.at[0], *gshift = dg.at[1];
  const int bins = 1 << bits, tid = threadIdx.x, w = tid / SSSP_WAVE, l = lane_id();
  const int64_t tile = sort_tile_of(blockIdx.x, gridDim.x);
  const int64_t base = tile * TILE;
  const int cnt = (int)(m - base < TILE ? m - base : TILE);
  // wave w holds rows [w * 64 * RK, (w + 1) * 64 * RK) of the tile, row
  // j * 64 + lane of them in slot j, so that order is (wave, slot, lane)
  const int first = w * (SSSP_WAVE * RK) + l;
  int32_t key[RK], pos[RK];  // key: then the column being moved
  const int32_t *const in = cols.in[KC] + base;
#pragma unroll
  for (int j = 0; j < RK; ++j) {
    const int i = first + j * SSSP_WAVE;
    key[j] = in[i < cnt ? i : 0];
  }
  for (int b = l; b < bins; b += SSSP_WAVE) u.wcnt[w][b] = 0;
  const uint64_t lt = (1ull << l) - 1ull;
#pragma unroll
  for (int j = 0; j < RK; ++j) {
    const bool valid = first + j * SSSP_WAVE < cnt;
    const int d = (key[j] >> shift) & (bins - 1);
    uint64_t mask = __ballot(valid);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bb = __ballot(bit);
      mask &= bit ? bb : ~bb;
    }
    // a wave's LDS accesses are performed in order: every lane reads its
    // digit's count before the digit's first lane raises it
    __builtin_amdgcn_wave_barrier();
    const int before = u.wcnt[w][d];
    __builtin_amdgcn_wave_barrier();
    const int mine = __popcll(mask & lt);
    if (valid && mine == 0) u.wcnt[w][d] = (uint16_t)(before + __popcll(mask));
    __builtin_amdgcn_wave_barrier();
    pos[j] = before + mine;
  }
  // (the digits are taken from the keys again below: kept, they spill)
#pragma unroll
  for (int j = 0; j < RK; ++j) asm volatile("" : "+v"(key[j]));
  __syncthreads();
  {
    // digits 2 tid and 2 tid + 1: their rows over the waves, then over the
    // digits (the tile's places and the digits' global starts in one scan)
    constexpr int BPT = kBins / kSortThreads > 0 ? kBins / kSortThreads : 1;
    uint64_t v[BPT] = {};
    uint64_t sum = 0;
#pragma unroll
    for (int q = 0; q < BPT; ++q) {
      const int b = BPT * tid + q;
      if (b < bins) {
        int run = 0;
        for (int x = 0; x < kSortWaves; ++x) {
          const int t = u.wcnt[x][b];
          u.wcnt[x][b] = (uint16_t)run;
          run += t;
        }
        v[q] = ((uint64_t)(uint32_t)totals[b] << 32) | (uint32_t)run;
        sum += v[q];
      }
    }
    uint64_t tot;
    uint64_t ex = block_excl_scan64<kSortThreads>(sum, dg.scan, &tot);
#pragma unroll
    for (int q = 0; q < BPT; ++q) {
      const int b = BPT * tid + q;
      if (b < bins) {
        const int32_t ls = (int32_t)(uint32_t)ex;
        lstart[b] = ls;
        gshift[b] = (int32_t)(ex >> 32) + hist[tile * bins + b] - ls;
      }
      ex += v[q];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < RK; ++j) {
    const int d = (key[j] >> shift) & (bins - 1);
    pos[j] += lstart[d] + u.wcnt[w][d];
  }
  __syncthreads();
  int32_t gp[RK];  // where sorted row tid + j * kSortThreads goes
  // the key column, then the others, one at a time (all of them in registers
  // at once spill: 217 us a pass at 16.8 M rows, 156 this way)
#pragma unroll
  for (int cc = 0; cc < NC; ++cc) {
    const int c = (KC + cc) % NC;
    if (cc > 0 && !cols.out[c]) continue;
    if (cc > 0) {
      const int32_t *const from = cols.in[c] ? cols.in[c] + base : nullptr;
#pragma unroll
      for (int j = 0; j < RK; ++j) {
        const int i = first + j * SSSP_WAVE;
        const int ic = i < cnt ? i : 0;
        key[j] = from ? from[ic] : (int32_t)base + ic;
      }
    }
#pragma unroll
    for (int j = 0; j < RK; ++j)
      if (first + j * SSSP_WAVE < cnt) u.buf[pos[j]] = key[j];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < RK; ++j) {
      const int i = tid + j * kSortThreads;
      if (i < cnt) {
        const int32_t x = u.buf[i];
        if (cc == 0) gp[j] = gshift[(x >> shift) & (bins - 1)] + i;
        if (cols.out[c]) cols.out[c][gp[j]] = x;
      }
    }
    __syncthreads();
  }
}

template <int RK, int NC>
static void sort_pass(const SortCols<NC> &cols, int kc, int32_t m, int shift, int bits,
                      int32_t *hist, hipStream_t stream) {
  const int64_t tiles = sort_tiles(m);
  const int bins = 1 << bits;
  int32_t *totals = hist + tiles * bins;
  hipLaunchKernelGGL(sort_hist_kernel<RK>, dim3((unsigned)tiles), dim3(kSortThreads), 0, stream,
                     cols.in[kc], m, shift, bits, hist);
  hipLaunchKernelGGL(sort_scan_kernel, dim3((bins + 15) / 16), dim3(1024), 0, stream, hist, bins,
                     tiles, totals);
  if (kc == 0)
    hipLaunchKernelGGL((sort_scatter_kernel<RK, NC, 0>), dim3((unsigned)tiles),
                       dim3(kSortThreads), 0, stream, cols, m, shift, bits, hist, totals);
  else
    hipLaunchKernelGGL((sort_scatter_kernel<RK, NC, 1>), dim3((unsigned)tiles),
                       dim3(kSortThreads), 0, stream, cols, m, shift, bits, hist, totals);
}

// Sorts the m rows of `in` stably by column kc (0 or 1; not null), whose
// values lie in [0, 2^bits) (other bits are ignored), into `out` (null
// columns are dropped).  in_a: `in` is the column set t.a; out_a: `out` is
// (never both).  t.a and t.b are overwritten.
template <int NC>
static hipError_t sort_rows(const int32_t *const (&in)[NC], int32_t *const (&out)[NC], int kc,
                            int32_t m, int bits, bool in_a, bool out_a, const BuildTemps &t,
                            hipStream_t stream) {
  if (m <= 0) return hipSuccess;
  if (bits < 1) bits = 1;
  const int passes = (bits + kMaxDigit - 1) / kMaxDigit;
  const int digit = (bits + passes - 1) / passes;
  // intermediate p goes to t.a or t.b in turn, so that no pass writes what
  // it reads
  bool to_b = in_a || (out_a && passes % 2 == 0);
  SortCols<NC> c;
  for (int q = 0; q < NC; ++q) c.in[q] = in[q];
  for (int p = 0; p < passes; ++p) {
    const int shift = p * digit, width = bits - shift < digit ? bits - shift : digit;
    for (int q = 0; q < NC; ++q) c.out[q] = p == passes - 1 ? out[q] : (to_b ? t.b[q] : t.a[q]);
    if (sort_rows_per_thread(m) == kBigRows) sort_pass<kBigRows, NC>(c, kc, m, shift, width, t.hist, stream);
    else sort_pass<4, NC>(c, kc, m, shift, width, t.hist, stream);
    for (int q = 0; q < NC; ++q) c.in[q] = c.out[q];
    to_b = !to_b;
  }
  return hipGetLastError();
}

// bits that hold the values 0 .. count - 1
static int bits_of(int64_t count) {
  int b = 0;
  while (b < 31 && ((int64_t)1 << b) < count) ++b;
  return b;
}

// ---------------------------------------------------------- assembling
// off[v] = the number of sorted keys below v (v = 0 .. n): one binary search
// per vertex, so a long run of vertices with no edges costs no thread more
// than the others
__global__ void offsets_kernel(const int32_t *skeys, int32_t m, int32_t n, int32_t *off) {
  for (int64_t v = blockIdx.x * blockDim.x + threadIdx.x; v <= n; v += gridDim.x * blockDim.x) {
    int32_t lo = 0, hi = m;
    while (lo < hi) {
      const int32_t mid = lo + ((hi - lo) >> 1);
      if (skeys[mid] < v) lo = mid + 1;
      else hi = mid;
    }
    off[v] = lo;
  }
}

// The list positions [0, m) in tiles of kTile per block, so that a hub's list
// costs no block more than its share (lists shared out by vertex left the
// hubs, neighbours under degree order, to one block: 3.3 ms for one copy of
// 16.8 M entries, 0.2 this way).  The block finds the vertices that own its
// tile's two ends; an entry's owner is then searched between them.
constexpr int kTileThreads = 256;
constexpr int kTilePT = 8;
constexpr int kTile = kTileThreads * kTilePT;

// the vertex in [lo, hi] whose list holds position p: the last with off <= p
// (lists before it may be empty)
__device__ __forceinline__ int32_t owner_between(const int32_t *off, int32_t lo, int32_t hi,
                                                 int32_t p) {
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo + 1) >> 1);
    if (off[mid] <= p) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// item(v, p, on) for every position p of this block's tile, whole waves
// together over 64 neighbouring positions (on: p < m; owner: the vertices by
// position where they are known, else null)
template <class Item>
__device__ __forceinline__ void for_tile(const int32_t *off, int32_t n, int32_t m,
                                         const int32_t *owner, Item item) {
  __shared__ int32_t ends[2];
  const int64_t p0 = (int64_t)blockIdx.x * kTile;
  int32_t lo = 0, hi = 0;
  if (!owner) {
    const int wv = threadIdx.x / SSSP_WAVE, l = lane_id();
    if (wv < 2) {  // wave 0: the first position's owner, wave 1: the last's
      const int64_t pe = wv == 0 ? p0 : p0 + kTile - 1;
      const int32_t p = (int32_t)(pe < m ? pe : m - 1);
      int32_t a = 0, b = n;  // off[a] <= p < off[b]
      while (b - a > 1) {    // 64 samples a step
        const int64_t span = (int64_t)b - a;
        const int32_t x = a + (int32_t)(span * l / SSSP_WAVE);
        const int t = __popcll(__ballot(off[x] <= p)) - 1;  // they form a prefix
        const int32_t nb = t == SSSP_WAVE - 1 ? b : a + (int32_t)(span * (t + 1) / SSSP_WAVE);
        a += (int32_t)(span * t / SSSP_WAVE);
        b = nb;
      }
      if (l == 0) ends[wv] = a;
    }
    __syncthreads();
    lo = ends[0];
    hi = ends[1];
  }
#pragma unroll
  for (int j = 0; j < kTilePT; ++j) {
    const int64_t p = p0 + j * kTileThreads + threadIdx.x;
    const bool on = p < m;
    const int32_t pc = (int32_t)(on ? p : m - 1);
    item(owner ? owner[pc] : owner_between(off, lo, hi, pc), pc, on);
  }
}

static inline dim3 tile_grid(int32_t m) {
  return dim3((unsigned)(((int64_t)m + kTile - 1) / kTile));
}

// Minimum out-weight per vertex into out_wmin (INF before; weights are
// positive, so float bits order like int32): a segmented minimum over each
// wave's 64 positions, one atomic per list and wave.  A thread per 256
// positions took 621 us at 16.8 M edges.
__global__ __launch_bounds__(kTileThreads) void wmin_kernel(const int32_t *out_off,
                                                            const int32_t *out_w, int32_t n,
                                                            int32_t m, const int32_t *owner,
                                                            int32_t *out_wmin) {
  for_tile(out_off, n, m, owner, [&](int32_t v, int32_t p, bool on) {
    // (positions past m repeat the last one: their weight is a true one)
    int32_t x = out_w[p];
    const int l = lane_id();
#pragma unroll
    for (int d = 1; d < SSSP_WAVE; d <<= 1) {
      const int32_t y = __shfl_up(x, d), u = __shfl_up(v, d);
      if (l >= d && u == v) x = kmin(x, y);
    }
    const int32_t next = __shfl_down(v, 1);
    if (l == SSSP_WAVE - 1 || next != v) atomicMin(&out_wmin[v], x);
  });
}

__global__ void fill_kernel(int32_t n, int32_t value, int32_t *out) {
  for (int64_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
    out[v] = value;
}

// The same with 8 lanes to a vertex, for graphs without long lists: no fill,
// no search for the owners (4.7 us against 16 at 0.1 M vertices of degree 8).
constexpr int kShortLanes = 8;
constexpr int32_t kShortList = 128;

__global__ __launch_bounds__(256) void wmin_short_kernel(const int32_t *out_off,
                                                         const int32_t *out_w, int32_t n,
                                                         int32_t inf, int32_t *out_wmin) {
  const int64_t v = ((int64_t)blockIdx.x * 256 + threadIdx.x) / kShortLanes;
  const int l = threadIdx.x % kShortLanes;
  int32_t mn = inf;
  if (v < n) {
    const int32_t e = out_off[v + 1];
    for (int32_t k = out_off[v] + l; k < e; k += kShortLanes) mn = kmin(mn, out_w[k]);
  }
  mn = lanes8_min(mn);
  if (v < n && l == 0) out_wmin[v] = mn;
}

// deg_max: at least the largest out-degree; owner: the tails by edge id, or
// null
static void launch_wmin(bool f32, int32_t n, int32_t m, int32_t deg_max, const int32_t *out_off,
                        const int32_t *out_w, const int32_t *owner, int32_t *out_wmin,
                        hipStream_t stream) {
  const int32_t inf = f32 ? KeyF32::INF : KeyI32::INF;
  if (deg_max <= kShortList) {
    hipLaunchKernelGGL(wmin_short_kernel,
                       dim3((unsigned)(((int64_t)n * kShortLanes + 255) / 256)), dim3(256), 0,
                       stream, out_off, out_w, n, inf, out_wmin);
    return;
  }
  hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(256), 0, stream, n, inf, out_wmin);
  if (m > 0)
    hipLaunchKernelGGL(wmin_kernel, tile_grid(m), dim3(kTileThreads), 0, stream, out_off, out_w,
                       n, m, owner, out_wmin);
}

// owner[p] = the vertex whose list holds position p
__global__ __launch_bounds__(kTileThreads) void owner_kernel(const int32_t *off, int32_t n,
                                                             int32_t m, int32_t *owner) {
  for_tile(off, n, m, nullptr, [&](int32_t v, int32_t p, bool on) {
    if (on) owner[p] = v;
  });
}

// total degree per vertex, its maximum and the largest in-degree
__global__ __launch_bounds__(kCheckThreads) void degree_kernel(const int32_t *out_off,
                                                               const int32_t *in_off, int32_t n,
                                                               int32_t *deg, int32_t *status) {
  constexpr int NW = kCheckThreads / SSSP_WAVE;
  __shared__ int32_t red[2][NW];
  int32_t mx = 0, mi = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
    const int32_t i = in_off[v + 1] - in_off[v], d = (out_off[v + 1] - out_off[v]) + i;
    deg[v] = d;
    mx = kmax(mx, d);
    mi = kmax(mi, i);
  }
  mx = wave_max(mx);
  mi = wave_max(mi);
  if (lane_id() == 0) {
    red[0][threadIdx.x / SSSP_WAVE] = mx;
    red[1][threadIdx.x / SSSP_WAVE] = mi;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    int32_t x = 0;
    for (int k = 0; k < NW; ++k) x = kmax(x, red[threadIdx.x][k]);
    int32_t *word = &status[threadIdx.x == 0 ? 2 : 4];
    if (x > ld_relaxed(word)) atomicMax(word, x);
  }
}

// Nothing here indexes by an endpoint's value, so it may run before the
// caller has seen launch_validate's verdict (on bad endpoints the outputs
// are of no use, but no access is out of range).
hipError_t launch_build(int32_t n, int32_t m, const int32_t *src, const int32_t *dst,
                        const int32_t *w, int32_t *out_off, int32_t *out_dst, int32_t *out_w,
                        int32_t *in_off, int32_t *in_src, int32_t *in_eid, int32_t *in_w,
                        int32_t *perm, const BuildTemps &t, hipStream_t stream) {
  hipError_t e;
  const int gn = grid_for((int64_t)n + 1), bits = bits_of(n);
  // CSR: rows (tail, head, weight, input index) by tail
  {
    const int32_t *const in[4] = {src, dst, w, nullptr};
    int32_t *const out[4] = {t.tail, out_dst, out_w, perm};
    if ((e = sort_rows<4>(in, out, 0, m, bits, false, false, t, stream)) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(offsets_kernel, dim3(gn), dim3(256), 0, stream, t.tail, m, n, out_off);
  // CSC: rows (tail, head, weight, edge id) by head; the heads by CSC
  // position are left in t.head
  {
    const int32_t *const in[4] = {t.tail, out_dst, out_w, nullptr};
    int32_t *const out[4] = {in_src, t.head, in_w, in_eid};
    if ((e = sort_rows<4>(in, out, 1, m, bits, false, false, t, stream)) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(offsets_kernel, dim3(gn), dim3(256), 0, stream, t.head, m, n, in_off);
  if (m > 0) {
    const int64_t gd = ((int64_t)n + kCheckThreads - 1) / kCheckThreads;
    hipLaunchKernelGGL(degree_kernel, dim3((unsigned)(gd < kCheckBlocks ? gd : kCheckBlocks)),
                       dim3(kCheckThreads), 0, stream, out_off, in_off, n, t.deg,
                       t.status);
  }
  return hipGetLastError();
}

hipError_t launch_out_wmin(bool f32, int32_t n, int32_t m, int32_t deg_max,
                           const int32_t *out_off, const int32_t *out_w, int32_t *out_wmin,
                           const BuildTemps &t, hipStream_t stream) {
  launch_wmin(f32, n, m, deg_max, out_off, out_w, t.tail, out_wmin, stream);
  return hipGetLastError();
}

// --------------------------------------------------- the working copy
// sort key for descending degree: dmax - deg
__global__ void degree_key_kernel(int32_t *key, int32_t n, int32_t dmax) {
  for (int64_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x)
    key[v] = dmax - key[v];
}

// the inverse numbering, and the degrees by solver id (entry n: 0)
__global__ void rank_kernel(const int32_t *vid, int32_t n, const int32_t *out_off,
                            const int32_t *in_off, int32_t *rank, int32_t *s_out_deg,
                            int32_t *s_in_deg) {
  for (int64_t k = blockIdx.x * blockDim.x + threadIdx.x; k <= n; k += gridDim.x * blockDim.x) {
    if (k == n) {
      s_out_deg[k] = s_in_deg[k] = 0;
      continue;
    }
    const int32_t v = vid[k];
    rank[v] = (int32_t)k;
    s_out_deg[k] = out_off[v + 1] - out_off[v];
    s_in_deg[k] = in_off[v + 1] - in_off[v];
  }
}

// The in-lists in solver order of their heads: rows (head, tail, weight,
// edge id) in solver ids, each list as in the CSC.
__global__ __launch_bounds__(kTileThreads) void copy_lists_kernel(
    const int32_t *s_in_off, int32_t n, int32_t m, const int32_t *vid, const int32_t *rank,
    const int32_t *in_off, const int32_t *in_src, const int32_t *in_w, const int32_t *in_eid,
    int32_t *head, int32_t *tail, int32_t *w, int32_t *eid) {
  for_tile(s_in_off, n, m, nullptr, [&](int32_t k, int32_t p, bool on) {
    const int32_t j = in_off[vid[k]] + (p - s_in_off[k]);
    const int32_t t = rank[in_src[j]], x = in_w[j], e = in_eid[j];
    if (on) {
      head[p] = k;
      tail[p] = t;
      w[p] = x;
      eid[p] = e;
    }
  });
}

__global__ void copy_wmin_kernel(const int32_t *vid, const int32_t *out_wmin, int32_t n,
                                 int32_t *s_out_wmin) {
  for (int64_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x)
    s_out_wmin[k] = out_wmin[vid[k]];
}

hipError_t launch_renumber(int32_t n, int32_t m, int32_t dmax, const int32_t *out_off,
                           const int32_t *in_off, const int32_t *in_src, const int32_t *in_w,
                           const int32_t *in_eid, const int32_t *out_wmin, const SolverCopy &c,
                           const BuildTemps &t, hipStream_t stream) {
  hipError_t e;
  // vertex order: stable sort by dmax - degree (t.deg holds the degrees)
  hipLaunchKernelGGL(degree_key_kernel, dim3(grid_for(n)), dim3(256), 0, stream, t.deg, n, dmax);
  {
    const int32_t *const in[2] = {t.deg, nullptr};
    int32_t *const out[2] = {nullptr, c.vid};
    if ((e = sort_rows<2>(in, out, 0, n, bits_of((int64_t)dmax + 1), false, false, t, stream)) !=
        hipSuccess)
      return e;
  }
  hipLaunchKernelGGL(rank_kernel, dim3(grid_for((int64_t)n + 1)), dim3(256), 0, stream, c.vid, n,
                     out_off, in_off, c.rank, c.out_off, c.in_off);
  if ((e = exclusive_scan(c.out_off, n + 1, t.hist, stream)) != hipSuccess) return e;
  if ((e = exclusive_scan(c.in_off, n + 1, t.hist, stream)) != hipSuccess) return e;
  if (m > 0) {
    // CSR: the in-lists in head order are rows by (head, edge id); sorted by
    // tail they are by (tail, head, edge id).  The tails stay in t.tail.
    hipLaunchKernelGGL(copy_lists_kernel, tile_grid(m), dim3(kTileThreads), 0, stream,
                       c.in_off, n, m, c.vid, c.rank, in_off, in_src, in_w, in_eid, t.a[1], t.a[0],
                       t.a[2], t.a[3]);
    const int32_t *const in[4] = {t.a[0], t.a[1], t.a[2], t.a[3]};
    int32_t *const out[4] = {t.tail, c.out_dst, c.out_w, c.out_eid};
    if ((e = sort_rows<4>(in, out, 0, m, bits_of(n), true, false, t, stream)) != hipSuccess)
      return e;
  }
  hipLaunchKernelGGL(copy_wmin_kernel, dim3(grid_for(n)), dim3(256), 0, stream, c.vid, out_wmin,
                     n, c.out_wmin);
  return hipGetLastError();
}

// Weight order within the CSC's in-lists, a thread per entry: an entry's
// place is the number of entries of its list that precede it by (weight,
// position).  Lists are read through the caches; the work is the sum of the
// squared in-degrees, so it serves graphs whose largest in-degree is at most
// kRankList (a grid's 4, a random digraph's 30) and replaces the radix
// passes over the whole weight (four for float32) and the head.  New weights
// this way and sorted, float32 and (sorted) int32: 0.1 M vertices of in-degree 8
// 83, 199 and 144 us, 50000 of 64 226 and 417, of 128 559, 801 and 633, 20000 of
// 256 600, 696 and 539, of 400 1377 and 906.
// head: by CSC position, or null (then out_dst of the entry's edge id).
constexpr int32_t kRankList = 128;

__global__ void rank_lists_kernel(int32_t m, const int32_t *in_off, const int32_t *in_src,
                                  const int32_t *in_eid, const int32_t *in_w,
                                  const int32_t *head, const int32_t *out_dst, int32_t *s_in_src,
                                  int32_t *s_in_eid, int32_t *s_in_w, int2 *s_in_sw) {
  for (int64_t j = blockIdx.x * blockDim.x + threadIdx.x; j < m; j += gridDim.x * blockDim.x) {
    const int32_t eid = in_eid[j], src = in_src[j], w = in_w[j];
    const int32_t y = head ? head[j] : out_dst[eid];
    const int32_t b = in_off[y], e = in_off[y + 1];
    int32_t p = b;
    for (int32_t k = b; k < e; ++k) {
      const int32_t x = in_w[k];
      p += (x < w || (x == w && k < j)) ? 1 : 0;
    }
    s_in_src[p] = src;
    s_in_eid[p] = eid;
    s_in_w[p] = w;
    s_in_sw[p] = make_int2(src, w);
  }
}

// heads by CSC position
__global__ void head_kernel(int32_t m, const int32_t *in_eid, const int32_t *out_dst,
                            int32_t *head) {
  for (int64_t j = blockIdx.x * blockDim.x + threadIdx.x; j < m; j += gridDim.x * blockDim.x)
    head[j] = out_dst[in_eid[j]];
}

__global__ void pair_kernel(int32_t m, const int32_t *in_src, const int32_t *in_w, int2 *in_sw) {
  for (int64_t j = blockIdx.x * blockDim.x + threadIdx.x; j < m; j += gridDim.x * blockDim.x)
    in_sw[j] = make_int2(in_src[j], in_w[j]);
}

hipError_t launch_in_lists(int32_t n, int32_t m, int32_t wkey_max, int32_t ideg_max,
                           const int32_t *out_dst, const int32_t *in_off, const int32_t *in_src,
                           const int32_t *in_eid, const int32_t *in_w, bool fresh,
                           const SolverCopy &c, const BuildTemps &t, hipStream_t stream) {
  hipError_t e;
  const int gm = grid_for(m);
  if (!c.vid && (e = hipMemcpyAsync(c.in_off, in_off, sizeof(int32_t) * ((size_t)n + 1),
                                    hipMemcpyDeviceToDevice, stream)) != hipSuccess)
    return e;
  if (m <= 0) return hipSuccess;
  if (!c.vid && ideg_max <= kRankList) {
    hipLaunchKernelGGL(rank_lists_kernel, dim3(gm), dim3(256), 0, stream, m, in_off, in_src,
                       in_eid, in_w, fresh ? t.head : nullptr, out_dst, c.in_src, c.in_eid,
                       c.in_w, (int2 *)c.in_sw);
    return hipGetLastError();
  }
  // Rows (weight, head, tail, edge id), in degree order those of the copy's
  // CSR (by tail, head, edge id), else of the CSC (by head, edge id; an edge
  // id orders the tails): by weight, then by head, which leaves each head's
  // list by (weight, tail, edge id).
  if (!fresh) {
    if (c.vid)
      hipLaunchKernelGGL(owner_kernel, tile_grid(m), dim3(kTileThreads), 0, stream, c.out_off,
                         n, m, t.tail);
    else
      hipLaunchKernelGGL(head_kernel, dim3(gm), dim3(256), 0, stream, m, in_eid, out_dst,
                         t.head);
  }
  const int32_t *const in[4] = {c.vid ? c.out_w : in_w, c.vid ? c.out_dst : t.head,
                                c.vid ? t.tail : in_src, c.vid ? c.out_eid : in_eid};
  int32_t *const mid[4] = {t.a[0], t.a[1], t.a[2], t.a[3]};
  const int32_t *const mid_in[4] = {t.a[0], t.a[1], t.a[2], t.a[3]};
  int32_t *const out[4] = {c.in_w, nullptr, c.in_src, c.in_eid};
  if ((e = sort_rows<4>(in, mid, 0, m, bits_of((int64_t)wkey_max + 1), false, true, t,
                        stream)) != hipSuccess)
    return e;
  if ((e = sort_rows<4>(mid_in, out, 1, m, bits_of(n), true, false, t, stream)) != hipSuccess)
    return e;
  hipLaunchKernelGGL(pair_kernel, dim3(gm), dim3(256), 0, stream, m, c.in_src, c.in_w,
                     (int2 *)c.in_sw);
  return hipGetLastError();
}

// The record also carries the head of the weight-ordered in-list (tail and
// weight of the lightest in-edge; 0, 0 with no in-edges), so that a pass
// over many vertices reads its first in-edge from the record's line instead
// of one line of in_src and one of in_w per vertex.
__global__ void vrec_kernel(int32_t n, const int32_t *out_off, const int32_t *in_off,
                            const int32_t *in_src, const int32_t *in_w,
                            const int32_t *out_wmin, int4 *vrec, int4 *vin) {
  for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gridDim.x * blockDim.x) {
    const int32_t o = out_off[v], i = in_off[v], ideg = in_off[v + 1] - i;
    const int32_t s0 = ideg ? in_src[i] : 0, w0 = ideg ? in_w[i] : 0;
    vrec[2 * v] = make_int4(o, out_off[v + 1] - o, i, ideg);
    vrec[2 * v + 1] = make_int4(out_wmin[v], s0, w0, 0);
    vin[v] = make_int4(i, ideg, s0, w0);
  }
}

hipError_t launch_vrec(int32_t n, const SolverCopy &c, hipStream_t stream) {
  hipLaunchKernelGGL(vrec_kernel, dim3(grid_for(n)), dim3(256), 0, stream, n, c.out_off,
                     c.in_off, c.in_src, c.in_w, c.out_wmin, (int4 *)c.vrec, (int4 *)c.vin);
  return hipGetLastError();
}

// Entry p of the working copy's out-lists as one record: head, weight, edge
// id (the position when the copy is the CSR itself), the head's out_wmin.
__global__ void out_rec_kernel(int32_t m, const int32_t *out_dst, const int32_t *out_w,
                               const int32_t *out_eid, const int32_t *out_wmin, int4 *rec) {
  for (int32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < m; p += gridDim.x * blockDim.x) {
    const int32_t y = out_dst[p];
    rec[p] = make_int4(y, out_w[p], out_eid ? out_eid[p] : p, out_wmin[y]);
  }
}

hipError_t launch_out_rec(int32_t m, const SolverCopy &c, hipStream_t stream) {
  if (m > 0)
    hipLaunchKernelGGL(out_rec_kernel, dim3(grid_for(m)), dim3(256), 0, stream, m, c.out_dst,
                       c.out_w, c.out_eid, c.out_wmin, (int4 *)c.out_rec);
  return hipGetLastError();
}

// ---------------------------------------------------------- reweighting
__global__ void set_weights_kernel(const int32_t *w, const int32_t *in_eid, int32_t m,
                                   int32_t *out_w, int32_t *in_w, const int32_t *s_out_eid,
                                   int32_t *s_out_w) {
  for (int64_t j = blockIdx.x * blockDim.x + threadIdx.x; j < m; j += gridDim.x * blockDim.x) {
    out_w[j] = w[j];
    in_w[j] = w[in_eid[j]];
    if (s_out_eid) s_out_w[j] = w[s_out_eid[j]];
  }
}

hipError_t launch_set_weights(int32_t n, int32_t m, bool f32, int32_t deg_max,
                              const int32_t *w, const int32_t *out_off, const int32_t *in_eid, int32_t *out_w,
                              int32_t *in_w, int32_t *out_wmin, const SolverCopy &c,
                              hipStream_t stream) {
  hipLaunchKernelGGL(set_weights_kernel, dim3(grid_for(m)), dim3(256), 0, stream, w, in_eid, m,
                     out_w, in_w, c.out_eid, c.out_w);
  launch_wmin(f32, n, m, deg_max, out_off, out_w, nullptr, out_wmin, stream);
  if (c.vid)
    hipLaunchKernelGGL(copy_wmin_kernel, dim3(grid_for(n)), dim3(256), 0, stream, c.vid,
                       out_wmin, n, c.out_wmin);
  return hipGetLastError();
}

// ------------------------------------------------- COO <-> edge-id order
// out[k] = in[perm[k]] (gather into edge-id order) or out[perm[k]] = in[k]
// (scatter into COO order): consecutive k read perm and one side
// coalesced; the other side follows the permutation.
__global__ void permute_edges_kernel(const int32_t *perm, int64_t m, const int32_t *in,
                                     int32_t *out, bool to_coo) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < m; k += stride) {
    const int32_t p = perm[k];
    if (to_coo) out[p] = in[k];
    else out[k] = in[p];
  }
}

hipError_t launch_permute_edges(const int32_t *perm, int64_t m, const int32_t *in, int32_t *out,
                                bool to_coo, hipStream_t stream) {
  hipLaunchKernelGGL(permute_edges_kernel, dim3(grid_for(m)), dim3(256), 0, stream, perm, m, in,
                     out, to_coo);
  return hipGetLastError();
}

}  // namespace sssp
