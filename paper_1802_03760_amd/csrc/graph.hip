// Forward and reverse CSR indexes of the edge relation (Sec. 4.1: one forward
// and one reverse index serve every atom).  Built by sorting (src, dst) keys,
// dropping repeats and self-loops, and deriving row pointers.
#include <algorithm>

#include "gj_internal.h"
#include "prim.h"

namespace gj {

__global__ void k_make_keys(const uint32_t* __restrict__ src, const uint32_t* __restrict__ dst, uint64_t m,
                            uint32_t n, uint64_t* __restrict__ keys, uint32_t* __restrict__ bad) {
  uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
    uint32_t s = src[i], d = dst[i];
    if (s >= n || d >= n) atomicOr(bad, 1u);
    keys[i] = ((uint64_t)s << 32) | d;
  }
}

// Sorted keys become edges: the first of equal keys, no self-loops.  Two
// passes over tiles of kEdgeTile keys, counts then edges at their offsets
// (flags and 64-bit offsets per key in memory between them cost as much again
// as both passes: 67.5e6 keys, 0.93 -> 0.45 ms).
constexpr int kEdgeItems = 8;
constexpr int kEdgeTile = kBlock * kEdgeItems;

__device__ __forceinline__ bool edge_key(const uint64_t* __restrict__ keys, uint64_t i, uint64_t k) {
  return (uint32_t)(k >> 32) != (uint32_t)k && (i == 0 || keys[i - 1] != k);
}

__global__ void __launch_bounds__(kBlock) k_count_edges(const uint64_t* __restrict__ keys, uint64_t m,
                                                        uint32_t* __restrict__ cnt) {
  const uint64_t base = (uint64_t)blockIdx.x * kEdgeTile;
  uint64_t t = 0;
#pragma unroll
  for (int i = 0; i < kEdgeItems; ++i) {
    const uint64_t at = base + (uint64_t)i * kBlock + threadIdx.x;
    if (at < m) t += edge_key(keys, at, keys[at]) ? 1 : 0;
  }
  t = block_sum<kBlock>(t);
  if (threadIdx.x == 0) cnt[blockIdx.x] = (uint32_t)t;
}

__global__ void __launch_bounds__(kBlock) k_compact_edges(const uint64_t* __restrict__ keys, uint64_t m,
                                                          const uint64_t* __restrict__ off,
                                                          uint32_t* __restrict__ row, uint32_t* __restrict__ col,
                                                          uint64_t* __restrict__ swapped) {
  // a wave takes kEdgeItems x 64 consecutive keys of the tile
  __shared__ uint32_t wcnt[kBlock / 64];
  const int lane = lane_id(), wave = wave_id();
  const uint64_t base = (uint64_t)blockIdx.x * kEdgeTile + (uint64_t)wave * (64 * kEdgeItems);
  uint64_t k[kEdgeItems], b[kEdgeItems];
  uint32_t t = 0;
#pragma unroll
  for (int i = 0; i < kEdgeItems; ++i) {
    const uint64_t at = base + (uint64_t)i * 64 + lane;
    k[i] = at < m ? keys[at] : 0;
    b[i] = __ballot(at < m && edge_key(keys, at, k[i]));
    t += (uint32_t)__popcll(b[i]);
  }
  if (lane == 0) wcnt[wave] = t;
  __syncthreads();
  uint64_t p = off[blockIdx.x];
  for (int w = 0; w < wave; ++w) p += wcnt[w];
#pragma unroll
  for (int i = 0; i < kEdgeItems; ++i) {
    if ((b[i] >> lane) & 1) {
      const uint64_t o = p + (uint64_t)__popcll(b[i] & lanemask_lt());
      const uint32_t s = (uint32_t)(k[i] >> 32), d = (uint32_t)k[i];
      row[o] = s;
      col[o] = d;
      swapped[o] = ((uint64_t)d << 32) | s;
    }
    p += (uint64_t)__popcll(b[i]);
  }
}

// the number of edges among the sorted keys; tile offsets left in `off`
static uint64_t count_edges(gj_ctx* c, const uint64_t* keys, uint64_t m, uint64_t*& off) {
  const uint64_t tiles = (m + kEdgeTile - 1) / kEdgeTile;
  uint32_t* cnt = (uint32_t*)ws_get(c, "gb_cnt", (tiles + 1) * sizeof(uint32_t));
  off = (uint64_t*)ws_get(c, "gb_off", (tiles + 1) * sizeof(uint64_t));
  if (m) k_count_edges<<<(unsigned)tiles, kBlock, 0, c->stream>>>(keys, m, cnt);
  scan_u32_to_u64(c, cnt, off, tiles);
  return read_u64(c, off + tiles);
}

static void compact_edges(gj_ctx* c, const uint64_t* keys, uint64_t m, const uint64_t* off, uint32_t* row,
                          uint32_t* col, uint64_t* swapped) {
  if (m)
    k_compact_edges<<<(unsigned)((m + kEdgeTile - 1) / kEdgeTile), kBlock, 0, c->stream>>>(keys, m, off, row, col,
                                                                                          swapped);
  GJ_HIP(hipGetLastError());
}

__global__ void k_split_keys(const uint64_t* __restrict__ keys, uint64_t m, uint32_t* __restrict__ row,
                             uint32_t* __restrict__ col) {
  uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
    uint64_t k = keys[i];
    row[i] = (uint32_t)(k >> 32);
    col[i] = (uint32_t)k;
  }
}

// first e in [0, m) with row[e] >= x (row ascending), else m; by the whole wave
__device__ __forceinline__ uint64_t wave_lower(const uint32_t* __restrict__ row, uint64_t m, uint64_t x) {
  uint64_t lo = 0, len = m;
  while (len > 0) {
    const uint64_t step = (len + 63) / 64, at = lane_id() * step;
    const uint64_t below = __ballot(at < len && row[lo + at] < x);  // lanes 0..k-1
    const uint64_t k = (uint64_t)__popcll(below);
    if (!k) break;
    const uint64_t next = k * step < len ? k * step : len;  // not below, or the end
    lo += (k - 1) * step + 1;
    len = next - ((k - 1) * step + 1);
  }
  return lo;
}

// rp[v] = first entry of row v in a row-sorted entry list (rp[n] = m): entry
// e starts the rows after its predecessor's up to its own (and entry m those
// up to n).  Runs of empty rows longer than a few are filled by the whole
// wave, but for the chunks of kRowChunk rows that lie inside one run: those
// have a wave each, the workgroups from `entries` on, so that a wave fills at
// most two chunks of a run.  Builds of 4.2e6 vertices without edges: 92 us
// with a search per vertex, 4.05 ms where one wave fills a run, 97 us so; of
// as many with 1,000 edges 264, 562 and 242 (399 at chunks of 4,096 rows),
// with 6.4e7 edges 5.06, 5.02 and 5.02 ms.
constexpr uint64_t kRowChunk = 512;

__global__ void __launch_bounds__(kBlock) k_rowptr(const uint32_t* __restrict__ row, uint64_t m, uint32_t n,
                                                   unsigned entries, uint32_t* __restrict__ rp) {
  constexpr uint64_t kAlone = 8;
  const uint64_t rows = (uint64_t)n + 1;
  if (blockIdx.x >= entries) {
    const uint64_t waves = (uint64_t)(gridDim.x - entries) * (kBlock / 64);
    for (uint64_t a = ((uint64_t)(blockIdx.x - entries) * (kBlock / 64) + wave_id()) * kRowChunk; a < rows;
         a += waves * kRowChunk) {
      const uint64_t b = a + kRowChunk < rows ? a + kRowChunk : rows;
      const uint64_t e = wave_lower(row, m, a);
      if (e == m || (uint64_t)row[e] + 1 >= b)
        for (uint64_t v = a + lane_id(); v < b; v += 64) rp[v] = (uint32_t)e;
    }
    return;
  }
  const uint64_t stride = (uint64_t)entries * kBlock;
  for (uint64_t b = (uint64_t)blockIdx.x * kBlock; b <= m; b += stride) {  // whole waves take every step
    const uint64_t e = b + threadIdx.x;
    uint64_t lo = 0, hi = 0;  // rows [lo, hi) start at e
    if (e <= m) {
      lo = e ? (uint64_t)row[e - 1] + 1 : 0;
      hi = e < m ? (uint64_t)row[e] + 1 : rows;
    }
    const bool big = hi > lo + kAlone;
    if (!big)
      for (; lo < hi; ++lo) rp[lo] = (uint32_t)e;
    for (uint64_t left = __ballot(big); left; left &= left - 1) {
      const int src = __ffsll((unsigned long long)left) - 1;
      const uint64_t l = shfl_u64(lo, src), h = shfl_u64(hi, src), x = shfl_u64(e, src);
      // the whole chunks in [l, h): from c0 to c1 (the last chunk ends at rows)
      uint64_t c0 = (l + kRowChunk - 1) / kRowChunk * kRowChunk;
      uint64_t c1 = h == rows ? rows : h / kRowChunk * kRowChunk;
      if (c0 > c1 || c0 >= rows) c0 = c1 = h;
      for (uint64_t v = l + lane_id(); v < c0; v += 64) rp[v] = (uint32_t)x;
      for (uint64_t v = c1 + lane_id(); v < h; v += 64) rp[v] = (uint32_t)x;
    }
  }
}

static void row_pointers(gj_ctx* c, const uint32_t* row, uint64_t m, uint32_t n, uint32_t* rp) {
  const unsigned entries = grid_for(m + 1, kBlock, 1u << 16);
  const unsigned chunks = grid_for((uint64_t)n + 1, kRowChunk * (kBlock / 64), 1u << 16);
  k_rowptr<<<entries + chunks, kBlock, 0, c->stream>>>(row, m, n, entries, rp);
}

// Largest degrees of both directions, the sums over the vertices of out^2,
// in^2 and out x in, and how many have more than kBigDegree edges: a few
// atomics per workgroup, into one of kDegreeSlots lines (a thousand workgroups'
// on one address are some 25 us), which the host adds up.
constexpr int kDegreeSlots = 32;
struct alignas(64) DegreeStats {
  uint32_t most[2];
  unsigned long long two[4];  // the last: the vertices of many edges
};

__global__ void __launch_bounds__(kBlock) k_degrees(const uint32_t* __restrict__ rp0,
                                                    const uint32_t* __restrict__ rp1, uint32_t n,
                                                    DegreeStats* __restrict__ out) {
  __shared__ uint32_t wbest[2][kBlock / 64];
  out += blockIdx.x % kDegreeSlots;
  uint32_t best[2] = {0, 0};
  uint64_t two[4] = {0, 0, 0, 0};
  uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
    const uint32_t d0 = rp0[v + 1] - rp0[v], d1 = rp1[v + 1] - rp1[v];
    best[0] = d0 > best[0] ? d0 : best[0];
    best[1] = d1 > best[1] ? d1 : best[1];
    two[0] += (uint64_t)d0 * d0;
    two[1] += (uint64_t)d1 * d1;
    two[2] += (uint64_t)d0 * d1;
    two[3] += (uint64_t)d0 + d1 > kBigDegree ? 1 : 0;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint64_t t = block_sum<kBlock>(two[i]);
    if (threadIdx.x == 0 && t) atomicAdd(&out->two[i], (unsigned long long)t);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    best[i] = wave_max(best[i]);
    if (lane_id() == 0) wbest[i][wave_id()] = best[i];
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    uint32_t b = 0;
    for (int w = 0; w < kBlock / 64; ++w) b = wbest[threadIdx.x][w] > b ? wbest[threadIdx.x][w] : b;
    if (b) atomicMax(&out->most[threadIdx.x], b);
  }
}

void version_alloc(gj_ctx* c, Version& v, uint32_t n, uint64_t cap) {
  if (cap < 1) cap = 1;
  ++v.gen;  // the slot is about to be rewritten
  for (int d = 0; d < 2; ++d) {
    if (!v.d[d].rp) v.d[d].rp = (uint32_t*)dev_alloc(c, ((uint64_t)n + 1) * sizeof(uint32_t));
    if (cap > v.cap) {
      // a failure part-way leaves this direction without arrays and the
      // slot's capacity at 0, so the next call allocates them again
      dev_free(c, v.d[d].col);
      dev_free(c, v.d[d].row);
      v.d[d].col = nullptr;
      v.d[d].row = nullptr;
      if (d == 0) v.cap = 0;
      v.d[d].col = (uint32_t*)dev_alloc(c, cap * sizeof(uint32_t));
      v.d[d].row = (uint32_t*)dev_alloc(c, cap * sizeof(uint32_t));
    }
  }
  if (cap > v.cap) v.cap = cap;
}

void version_free(gj_ctx* c, Version& v) {
  for (int d = 0; d < 2; ++d) {
    dev_free(c, v.d[d].rp);
    dev_free(c, v.d[d].col);
    dev_free(c, v.d[d].row);
    v.d[d] = CsrDir{};
  }
  v.cap = v.m = 0;
}

int bits_for(uint32_t n) {
  int b = 0;
  while (b < 32 && ((uint64_t)1 << b) < n) ++b;
  return b;
}

void version_finish(gj_ctx* c, Version& v, uint32_t n) {
  ++v.gen;
  DegreeStats h[kDegreeSlots];
  DegreeStats* stats = (DegreeStats*)ws_get(c, "degrees", sizeof(h));
  GJ_HIP(hipMemsetAsync(stats, 0, sizeof(h), c->stream));
  for (int d = 0; d < 2; ++d) row_pointers(c, v.d[d].row, v.m, n, v.d[d].rp);
  k_degrees<<<grid_for(n, kBlock * 16, 1024), kBlock, 0, c->stream>>>(v.d[0].rp, v.d[1].rp, n, stats);
  GJ_HIP(hipGetLastError());
  read_bytes(c, h, stats, sizeof(h));
  v.blur = ~0ull;
  v.max_deg[0] = v.max_deg[1] = 0;
  v.two[0] = v.two[1] = v.two[2] = v.big = 0;
  for (const DegreeStats& x : h) {
    for (int d = 0; d < 2; ++d) v.max_deg[d] = std::max(v.max_deg[d], x.most[d]);
    for (int i = 0; i < 3; ++i) v.two[i] += x.two[i];
    v.big += x.two[3];
  }
}

void graph_build(gj_ctx* c, gj_graph* g, const uint32_t* d_src, const uint32_t* d_dst, uint64_t m) {
  uint32_t n = g->n;
  int bits = bits_for(n);
  uint64_t* keys = (uint64_t*)ws_get(c, "gb_keys", (m + 1) * sizeof(uint64_t));
  uint64_t* alt = (uint64_t*)ws_get(c, "gb_alt", (m + 1) * sizeof(uint64_t));
  uint32_t* bad = (uint32_t*)ws_get(c, "gb_bad", sizeof(uint32_t));
  GJ_HIP(hipMemsetAsync(bad, 0, sizeof(uint32_t), c->stream));
  unsigned gr = grid_for(m, kBlock, 1u << 16);
  if (m) k_make_keys<<<gr, kBlock, 0, c->stream>>>(d_src, d_dst, m, n, keys, bad);
  GJ_HIP(hipGetLastError());
  uint32_t hbad = 0;
  read_bytes(c, &hbad, bad, sizeof(hbad));
  GJ_CHECK(!hbad, GJ_EINVAL, "vertex id >= num_vertices");
  uint64_t* sorted = sort_u64(c, keys, alt, m, bits, bits);
  uint64_t* other = sorted == keys ? alt : keys;
  uint64_t* off = nullptr;
  uint64_t mu = count_edges(c, sorted, m, off);
  Version& v = g->ver[g->cur];
  // the same growth room as the versions updates write, so that no slot is
  // reallocated when updates come back round to it
  version_alloc(c, v, n, mu + mu / 16 + (1ull << 20));
  v.m = mu;
  compact_edges(c, sorted, m, off, v.d[0].row, v.d[0].col, other);
  uint64_t* other_alt = sorted;  // free for reuse now
  // the swapped keys come in ascending order of their low half (the source),
  // so a stable sort by the high half finishes them
  uint64_t* rsorted = sort_u64(c, other, other_alt, mu, 0, bits);
  if (mu) k_split_keys<<<grid_for(mu, kBlock, 1u << 16), kBlock, 0, c->stream>>>(rsorted, mu, v.d[1].row, v.d[1].col);
  GJ_HIP(hipGetLastError());
  version_finish(c, v, n);
}

// ---------------------------------------------------------------- renaming by degree (Sec. 5.4)
// Both directions of every input edge as (src, dst) keys.
__global__ void k_make_sym_keys(const uint32_t* __restrict__ src, const uint32_t* __restrict__ dst, uint64_t m,
                                uint32_t n, uint64_t* __restrict__ keys, uint32_t* __restrict__ bad) {
  uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
    uint32_t s = src[i], d = dst[i];
    if (s >= n || d >= n) atomicOr(bad, 1u);
    keys[i] = ((uint64_t)s << 32) | d;
    keys[m + i] = ((uint64_t)d << 32) | s;
  }
}

// (degree, id) of every vertex; the degree is its row length in the
// symmetric edge set, i.e. the number of distinct neighbours
__global__ void k_degree_keys(const uint32_t* __restrict__ rp, uint32_t n, uint64_t* __restrict__ vkeys) {
  uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride)
    vkeys[v] = ((uint64_t)(rp[v + 1] - rp[v]) << 32) | v;
}

// new id = rank in (degree, id) order
__global__ void k_rank_ids(const uint64_t* __restrict__ vkeys, uint32_t n, uint32_t* __restrict__ old_of_new,
                           uint32_t* __restrict__ new_of_old) {
  uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    uint32_t o = (uint32_t)vkeys[i];
    old_of_new[i] = o;
    new_of_old[o] = (uint32_t)i;
  }
}

// Renames both ends; with `up_only` an edge that does not go from a lower new
// id to a higher one is written as a self-loop, which the build drops.
__global__ void k_rename_edges(const uint32_t* __restrict__ row, const uint32_t* __restrict__ col, uint64_t m,
                               const uint32_t* __restrict__ new_of_old, int up_only, uint32_t* __restrict__ osrc,
                               uint32_t* __restrict__ odst) {
  uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
    uint32_t u = new_of_old[row[i]], v = new_of_old[col[i]];
    osrc[i] = u;
    odst[i] = (up_only && !(u < v)) ? u : v;
  }
}

void graph_build_sym(gj_ctx* c, gj_graph* g, const uint32_t* d_src, const uint32_t* d_dst, uint64_t m,
                     bool degree_order, bool undirected) {
  uint32_t n = g->n;
  int bits = bits_for(n);
  uint64_t m2 = 2 * m;
  struct Temps {  // freed on every exit, errors included
    gj_ctx* c;
    std::vector<void*> p;
    ~Temps() {
      for (void* x : p) dev_free(c, x);
    }
  } tmp{c, {}};
  auto alloc = [&](size_t bytes) {
    void* p = dev_alloc(c, bytes ? bytes : 1);
    tmp.p.push_back(p);
    return p;
  };
  uint64_t* keys = (uint64_t*)alloc((m2 + 1) * sizeof(uint64_t));
  uint64_t* alt = (uint64_t*)alloc((m2 + 1) * sizeof(uint64_t));
  uint32_t* bad = (uint32_t*)alloc(sizeof(uint32_t));
  GJ_HIP(hipMemsetAsync(bad, 0, sizeof(uint32_t), c->stream));
  unsigned gr = grid_for(m, kBlock, 1u << 16);
  if (m) k_make_sym_keys<<<gr, kBlock, 0, c->stream>>>(d_src, d_dst, m, n, keys, bad);
  GJ_HIP(hipGetLastError());
  uint32_t hbad = 0;
  read_bytes(c, &hbad, bad, sizeof(hbad));
  GJ_CHECK(!hbad, GJ_EINVAL, "vertex id >= num_vertices");
  // the symmetric edge set: both directions of every distinct pair, no loops
  uint64_t* sorted = sort_u64(c, keys, alt, m2, bits, bits);
  uint64_t* other = sorted == keys ? alt : keys;
  uint64_t* off = nullptr;
  uint64_t ms = count_edges(c, sorted, m2, off);
  uint32_t* srow = (uint32_t*)alloc((ms + 1) * sizeof(uint32_t));
  uint32_t* scol = (uint32_t*)alloc((ms + 1) * sizeof(uint32_t));
  compact_edges(c, sorted, m2, off, srow, scol, other);
  const uint32_t *es = srow, *ed = scol;
  if (degree_order) {
    uint32_t* rp = (uint32_t*)alloc(((uint64_t)n + 1) * sizeof(uint32_t));
    uint64_t* vk = (uint64_t*)alloc((uint64_t)n * sizeof(uint64_t));
    uint64_t* vk2 = (uint64_t*)alloc((uint64_t)n * sizeof(uint64_t));
    uint32_t* new_of_old = (uint32_t*)alloc((uint64_t)n * sizeof(uint32_t));
    unsigned gn = grid_for((uint64_t)n + 1, kBlock, 1u << 16);
    row_pointers(c, srow, ms, n, rp);
    k_degree_keys<<<gn, kBlock, 0, c->stream>>>(rp, n, vk);
    uint64_t* vs = sort_u64(c, vk, vk2, n, 0, bits);  // stable: equal degrees by id
    g->old_of_new = (uint32_t*)dev_alloc(c, (uint64_t)n * sizeof(uint32_t));
    k_rank_ids<<<gn, kBlock, 0, c->stream>>>(vs, n, g->old_of_new, new_of_old);
    uint32_t* osrc = (uint32_t*)alloc((ms + 1) * sizeof(uint32_t));
    uint32_t* odst = (uint32_t*)alloc((ms + 1) * sizeof(uint32_t));
    if (ms)
      k_rename_edges<<<grid_for(ms, kBlock, 1u << 16), kBlock, 0, c->stream>>>(srow, scol, ms, new_of_old,
                                                                               undirected ? 0 : 1, osrc, odst);
    es = osrc;
    ed = odst;
  }
  GJ_HIP(hipGetLastError());
  graph_build(c, g, es, ed, ms);
  if (degree_order) g->ver[g->cur].blur = 0;
  GJ_HIP(hipStreamSynchronize(c->stream));
}

}  // namespace gj
