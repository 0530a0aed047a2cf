// Whole counts of the transitive 4-clique and 5-clique (every atom from an
// earlier attribute of the order to a later one) without inequalities, on bit
// matrices.
//
// Vertices are renamed by descending degree (hub.h), and a match is counted at
// its greatest vertex v (the one of least degree): its other vertices lie in
// N = the neighbours of v below it in either direction, at most a few hundred
// even where degrees reach 10^5.  O marks the members that v has an edge to,
// I those with an edge to v, F the edges among them as a bit matrix in LDS.  v
// may stand at any position of the order, with members of I before it and of
// O behind it, so for the 4-clique the others b0 -> b1 -> b2 (b0 -> b2 too)
// are OOO, IOO, IIO or III; for each edge (i, j) of F the third is a population
// count of row i & row j & O (or I).  The 5-clique fixes a third member k of
// row i & row j the same way.  On a graph oriented by degree I is empty.
//
// The matrix costs one walk of the members' own prefixes, the sum over edges
// of the hub-side degree (4.4e9 entries at R-MAT-20 undirected), against
// 5.8e10 candidates of the depth-first evaluation there; members among the
// hubs take bit reads instead (k_cb_bits).  The counts read LDS only.  Counters
// are the depth-first ones: prefixes are cliques, and extensions sum the least
// out-degree of a prefix's vertices.
//
// Measured (MI355X): R-MAT-20 oriented 4-clique 177 -> 7.9 ms, oriented 5-clique
// of a 300,007-vertex R-MAT graph 20.4 -> 5.7 ms, directed R-MAT-17 4-clique
// 90.6 -> 1.1 ms, against a wave per seed edge that probes rows in memory for
// every a2 (clique.hip, still there for inequalities, for light graphs
// (choose_order) and where a vertex has more than 1,056 neighbours of higher
// degree).  Bound by the build's probes
// and bit reads, then by the counts' LDS reads and popcounts.
#include <algorithm>

#include "gj_internal.h"
#include "hub.h"
#include "prim.h"

namespace gj {

// matches, then pre and ext per stage: kCb + 2 (j - 2) and + 1 for |P_j|, j >= 3
enum { kCbMatches, kCbExt2, kCbPre3, kCbExt3, kCbPre4, kCbExt4, kCbAcc };
constexpr int kCbClasses = 4;
constexpr uint32_t kCbCap[kCbClasses] = {64, 256, 512, kBigDegree};
// Edges from which the hubs' adjacency bits are built, where some vertex has
// more than kCbCap[0] neighbours below it.  Their build is some 40 us: R-MAT-15
// (3.2e5 edges) 4-clique 795 -> 729 us and 5-clique 1,481 -> 1,487, R-MAT-16
// 1,008 -> 857 and 1,835 -> 1,853, R-MAT-17 1,628 -> 1,080 and 4,047 -> 3,437;
// uniform random graphs, whose members have short rows, lose (5.2e5 edges: 367
// -> 430 us).
constexpr uint64_t kCbBitsEdges = 500000;

// Which kernels count the cliques, and in which order of the vertices.  Any
// order counts every clique once; any of the three ways is right for any graph.
//
// As they are: graphs of at most kCbAsIs vertices without hubs (largest out-
// and in-degree together at most kCbAsIsDeg), and larger ones where no vertex
// can have more than kCbAsIsAny members.  Renaming costs 110 us, 5 us per
// 10^5 edges and 40 per 10^6 ids, and saves nothing there: uniform graphs,
// 4-clique, edge-grouped kernels / as they are / renamed: 16,385 vertices and
// 65,536 edges 255 / 91 / 280 us, 2.6e5 and 2.6e5 398 / 145 / 396, 4.2e6 and
// 1.7e7 12.9 / 4.4 / 6.3 ms.
//
// The edge-grouped kernels (clique.hip) where the graph is too light to repay
// the preparation: two = sum of out^2, which bounds their first step, against
// 36 for every edge (64 with more than 24 ids to each) and a sixth for every
// id.  R-MAT, 4-clique, edge-grouped / renamed: 16,384 vertices, 16,073 edges
// (two = 4.2e5) 222 / 274 us, 65,536 and 32,000 (7.5e5) 229 / 298, 1,024 and
// 9,500 (1.2e6) 1017 / 257, 65,536 and 65,000 (2.6e6) 510 / 402; 2.6e5 and
// 1.3e5 (4.7e6) 463 / 497.  From
// 2^19 edges and one per eight ids on no graph is light: an edge costs them 0.8
// ns at least, and 0.4 to rename (1.0e6 vertices and 3.4e7 edges, uniform: 25.8
// / 14 ms).  In id spaces of 6.7e7 with 20,000 edges 275 us / 3.4 ms, with 2e5
// (two = 117 an edge) 12.3 / 3.9 ms; of 3.4e7 with 1.0e6 (48) 1.1 / 2.5 ms.
// A 5-clique pays one workgroup's chain for its largest vertex, so light
// graphs go there from kCbAsIsAny on (1,024 vertices, 3,600 edges: 228 us, as
// they are 296).  Uniform graphs stay as they are up to kCbIds ids and 32 per
// edge (4.2e6 ids, 84,000 edges 139 us / 232; 1.7e7 ids, 2,000 edges 390 /
// 199).  Graphs built with ids ascending by degree are reversed, at a third of
// the renaming's cost, but for small ones where nothing lies two edges deep (a
// star of 2,000 edges 99 / 132 us, of 20,000 124 / 127, of 200,000 293 / 129).
constexpr uint32_t kCbAsIs = 16384, kCbAsIsDeg = 512, kCbAsIsAny = 128;
constexpr uint64_t kCbLightEdge = 36, kCbLightApart = 64, kCbLightIds = 6, kCbLightMost = 1ull << 19;
constexpr uint64_t kCbIds = 1ull << 21, kCbFlat = 16384;

static bool choose_order(const Version& v, uint32_t n, int q, HubOrder& order) {
  const uint64_t most = (uint64_t)v.max_deg[0] + v.max_deg[1];
  const uint64_t two = std::min(v.two[0], v.m * std::min(v.max_deg[0], v.max_deg[1]));
  const uint64_t each = n > 24 * v.m ? kCbLightApart : kCbLightEdge;
  const bool light = two < each * v.m + n / kCbLightIds && v.m < kCbLightMost + n / 8;
  const bool apart = n > kCbIds + 32 * v.m;
  if (v.ranked()) {
    order = HubOrder::kReversed;
    return (two > v.m || v.m > kCbFlat) && !(apart && light);
  }
  if (most <= (n <= kCbAsIs ? kCbAsIsDeg : kCbAsIsAny)) {
    order = HubOrder::kAsIs;
    return !(light && (apart || (q == 5 && most > kCbAsIsAny)));
  }
  order = HubOrder::kDegree;
  return !light;
}

// extensions[2]: the lesser out-degree of every edge's ends
__global__ void __launch_bounds__(kBlock) k_cb_ext2(HubGraph g, const uint32_t* __restrict__ row, uint64_t m,
                                                    unsigned long long* __restrict__ acc) {
  uint64_t s = 0;
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += gs) {
    const uint32_t a = g.deg(0, row[e]), b = g.deg(0, g.col[0][e]);
    s += a < b ? a : b;
  }
  s = block_sum<kBlock>(s);
  if (threadIdx.x == 0 && s) atomicAdd(acc + kCbExt2, (unsigned long long)s);
}

// Vertices with two or more neighbours below them, by how many; len[kCbClasses]
// counts those beyond the last class.  A neighbour both ways counts twice, but
// for the last class: R-MAT-22 has 380 vertices of more than 1,056 neighbours
// so counted, none of more than 1,049 (its 4-clique: 16.4 s on the
// edge-grouped kernels, 0.12 s here).  fits: none is beyond, as is known; else
// the two rows of such a vertex are merged, by one thread (0.4 ms for rows of
// 1,040 entries each).
__global__ void __launch_bounds__(kBlock) k_cb_classes(HubGraph g, int fits, unsigned int* __restrict__ len,
                                                       uint32_t* __restrict__ lists) {
  __shared__ uint32_t cnt[kCbClasses + 1], base[kCbClasses + 1];
  for (uint64_t b = (uint64_t)blockIdx.x * kBlock; b < g.n; b += (uint64_t)gridDim.x * kBlock) {
    if (threadIdx.x <= kCbClasses) cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t v = b + threadIdx.x;
    int c = -1;
    uint32_t at = 0;
    if (v < g.n) {
      const uint64_t d = (uint64_t)(g.end[0][v] - g.rp[0][v]) + (g.end[1][v] - g.rp[1][v]);
      if (d >= 2) {
        c = 0;
        while (c < kCbClasses && d > kCbCap[c]) ++c;
        if (fits && c == kCbClasses) {
          --c;
        } else if (c == kCbClasses && d <= 2 * kCbCap[c - 1]) {
          uint64_t i = g.rp[0][v], j = g.rp[1][v], both = 0;  // rows ascend
          while (i < g.end[0][v] && j < g.end[1][v]) {
            const uint32_t x = g.col[0][i], y = g.col[1][j];
            both += x == y;
            i += x <= y;
            j += y <= x;
          }
          if (d - both <= kCbCap[c - 1]) --c;
        }
        at = atomicAdd(&cnt[c], 1u);
      }
    }
    __syncthreads();
    if (threadIdx.x <= kCbClasses && cnt[threadIdx.x])
      base[threadIdx.x] = atomicAdd(len + threadIdx.x, cnt[threadIdx.x]);
    __syncthreads();
    if (c >= 0 && c < kCbClasses) lists[(uint64_t)c * g.n + base[c] + at] = (uint32_t)v;
    __syncthreads();
  }
}

// Adjacency of the hubs: bit x of row u (kCbTop / 32 words) of bits[s] is set
// for x in the prefix of u's row in direction s, for u below kCbTop.  null:
// not built (bits[1] also where no vertex has an in-prefix).  Most members of
// the larger v are such hubs, and a member's edges to the ones below it are
// then bit reads, members' pairs of v only, instead of a walk of its whole
// prefix against v's hash table (oriented R-MAT-20, 4-clique: 22.6 -> 7.9
// ms, 5-clique at 300,007 vertices 6.9 -> 5.7 ms).
constexpr uint32_t kCbTop = 32768;
struct CbBits {
  const uint32_t* bits[2];
};

// a wave per hub and direction
__global__ void __launch_bounds__(kBlock) k_cb_bits(HubGraph g, uint32_t top, uint32_t* __restrict__ b0,
                                                    uint32_t* __restrict__ b1) {
  const uint32_t w = blockIdx.x * (kBlock / 64) + wave_id(), u = w >> 1, s = w & 1;
  uint32_t* b = s ? b1 : b0;
  if (u >= top || !b) return;
  const uint32_t lo = g.rp[s][u], n = g.end[s][u] - lo;
  for (uint32_t i = lane_id(); i < n; i += 64) {
    const uint32_t x = g.col[s][(uint64_t)lo + i];
    atomicOr(b + (uint64_t)u * (kCbTop / 32) + (x >> 5), 1u << (x & 31));
  }
}

// LDS of one v: its members' table (open addressing, about half full at most, ~0 =
// free) with their positions, ids and out-degrees, the masks O and I, and the
// matrix F: bit (i, j) is bit j & 31 of mat[(j / 32) * kStride + i], so that
// lanes on consecutive rows read one word of each without bank conflicts (and
// a lane per word reads a row without any: the stride is odd).
template <uint32_t CAP, uint32_t SLOTS>
struct CbLds {
  static constexpr uint32_t kWords = CAP / 32, kStride = CAP + 1;
  uint32_t key[SLOTS];
  uint16_t pos[SLOTS];
  uint32_t id[CAP], deg[CAP];
  uint32_t O[kWords], I[kWords];
  uint32_t n;
  uint32_t mat[kWords * kStride + 64];
};

template <uint32_t CAP, uint32_t SLOTS>
__device__ __forceinline__ uint32_t cb_home(uint32_t x) {
  return (x * 0x9E3779B1u) >> (32 - __builtin_ctz(SLOTS));
}

// position of x, or ~0
template <uint32_t CAP, uint32_t SLOTS>
__device__ __forceinline__ uint32_t cb_find(const CbLds<CAP, SLOTS>& s, uint32_t x) {
  for (uint32_t h = cb_home<CAP, SLOTS>(x);; h = (h + 1) & (SLOTS - 1)) {
    const uint32_t k = s.key[h];
    if (k == ~0u) return ~0u;
    if (k == x) return s.pos[h];
  }
}

template <uint32_t CAP, uint32_t SLOTS>
__device__ __forceinline__ void cb_insert(CbLds<CAP, SLOTS>& s, uint32_t x, uint32_t p) {
  uint32_t h = cb_home<CAP, SLOTS>(x);
  while (atomicCAS(&s.key[h], ~0u, x) != ~0u) h = (h + 1) & (SLOTS - 1);
  s.pos[h] = (uint16_t)p;
  s.id[p] = x;
}

// Builds v's members and matrix with NT threads (nw waves, this one wave);
// sync separates their phases.  Returns the number of members.
template <uint32_t CAP, uint32_t SLOTS, class Sync>
__device__ __forceinline__ uint32_t cb_build(CbLds<CAP, SLOTS>& s, const HubGraph& g, const CbBits& hb, uint32_t v,
                                             uint32_t tid, uint32_t nt, Sync sync) {
  const uint32_t lane = lane_id(), wave = tid / 64, nw = nt / 64;
  const uint32_t b0 = g.rp[0][v], n0 = g.end[0][v] - b0, b1 = g.rp[1][v], n1 = g.end[1][v] - b1;
  const uint32_t most_words = (n0 + n1 + 31) / 32, words = most_words < CAP / 32 ? most_words : CAP / 32;
  sync();  // the previous v is done with
  for (uint32_t i = tid; i < SLOTS; i += nt) s.key[i] = ~0u;
  for (uint32_t i = tid; i < words * CbLds<CAP, SLOTS>::kStride; i += nt) s.mat[i] = 0;
  for (uint32_t i = tid; i < words; i += nt) {
    const uint32_t left = n0 > 32 * i ? n0 - 32 * i : 0;
    s.O[i] = left >= 32 ? ~0u : (1u << left) - 1;
    s.I[i] = 0;
  }
  if (tid == 0) s.n = n0;
  sync();
  for (uint32_t i = tid; i < n0; i += nt) cb_insert(s, g.col[0][(uint64_t)b0 + i], i);
  sync();
  for (uint32_t i = tid; i < n1; i += nt) {
    const uint32_t x = g.col[1][(uint64_t)b1 + i];
    uint32_t p = cb_find(s, x);  // a reciprocal neighbour has its place already
    if (p == ~0u) {
      p = atomicAdd(&s.n, 1u);
      cb_insert(s, x, p);
    }
    atomicOr(&s.I[p >> 5], 1u << (p & 31));
  }
  sync();
  const uint32_t n = s.n;
  for (uint32_t i = tid; i < n; i += nt) s.deg[i] = g.deg(0, s.id[i]);
  // the hubs among the members: 64 / P of them at a time, P lanes of members
  // each, tested for the members below
  constexpr uint32_t kStride = CbLds<CAP, SLOTS>::kStride;
  const uint32_t top = hb.bits[0] ? kCbTop : 0;
  if (top) {
    const uint32_t lg = n > 32 ? 6 : n > 16 ? 5 : n > 8 ? 4 : 3, P = 1u << lg;
    const uint32_t sub = lane & (P - 1), first = lane >> lg;
    for (uint32_t i0 = wave << (6 - lg); i0 < n; i0 += nw << (6 - lg)) {
      const uint32_t i = i0 + first, u = i < n ? s.id[i] : ~0u;
      const uint64_t at = (uint64_t)u * (kCbTop / 32);
      const uint32_t most = n1 || lg < 6 ? n : i0;  // without in-neighbours the members ascend
      for (uint32_t j0 = 0; j0 < most; j0 += P) {
        const uint32_t j = j0 + sub, x = j < n ? s.id[j] : ~0u;
        const bool below = u < top && x < u;
        const uint64_t b = __ballot(below && (hb.bits[0][at + (x >> 5)] >> (x & 31) & 1));
        if (lg == 6) {
          if (lane < 2 && (uint32_t)(b >> (32 * lane)))
            atomicOr(&s.mat[((j0 >> 5) + lane) * kStride + i0], (uint32_t)(b >> (32 * lane)));
        } else if (sub == 0) {
          const uint32_t mine = (uint32_t)(b >> (first << lg)) & (uint32_t)((1ull << P) - 1);
          if (mine) atomicOr(&s.mat[i], mine);
        }
        if (hb.bits[1] && below && (hb.bits[1][at + (x >> 5)] >> (x & 31) & 1))
          atomicOr(&s.mat[(i >> 5) * kStride + j], 1u << (i & 31));
      }
    }
  }
  // the other members' prefixes, out- and in-, as rows tagged with member and
  // side
  for (uint32_t r0 = wave * 64; r0 < 2 * n; r0 += nw * 64) {
    const uint32_t r = r0 + lane, i = r >> 1, side = r & 1;
    uint32_t p = 0, q = 0;
    if (r < 2 * n) {
      const uint32_t u = s.id[i];
      if (u >= top) {
        const uint32_t* pq = side ? g.pq[1] : g.pq[0];
        p = pq[u];
        q = pq[(uint64_t)u + 1] - p;
      }
    }
    const uint64_t some = __ballot(q != 0), lt = lanemask_lt();
    const uint32_t cn = (uint32_t)__popcll(some);
    const uint32_t to = q ? (uint32_t)__popcll(some & lt) : cn + (uint32_t)__popcll(~some & lt);
    p = (uint32_t)__builtin_amdgcn_ds_permute(to * 4, (int)p);
    // quads in the low half: a member, as any vertex here, has at most kBigDegree
    // entries in a prefix; r < 2 CAP in the high one
    static_assert(kBigDegree / 4 + 1 < 1 << 16 && 2 * CAP < 1 << 16, "a row's quads and its tag in one word");
    q = (uint32_t)__builtin_amdgcn_ds_permute(to * 4, (int)(q | r << 16));
    walk_batch<2, 16>(g.pre, p, q, cn, v, [&](uint32_t x, uint32_t tag) {
      const uint32_t j = cb_find(s, x);  // ~0 is not found
      if (j == ~0u) return;
      const uint32_t i = tag >> 1, a = tag & 1 ? j : i, b = tag & 1 ? i : j;  // side 0: i -> x, side 1: x -> i
      atomicOr(&s.mat[(b >> 5) * kStride + a], 1u << (b & 31));
    });
  }
  sync();
  return n;
}

struct CbSums {
  uint64_t v[kCbAcc] = {};
};

__device__ __forceinline__ bool bit_of(uint32_t lo, uint32_t hi, uint32_t lane) {
  return ((lane < 32 ? lo >> lane : hi >> (lane - 32)) & 1) != 0;
}

// The 5-cliques through v and member i whose row (lane w: word w) has L <= 64 R
// members: that row's members alone, renumbered 0..L-1 in order, with the edges
// among them as bit rows in registers, R rows of 2 R words to a lane.  The
// words of the full matrix hold mostly members outside the row, and every
// pair (i, j) would go through all of them (R-MAT, 300,007 vertices, oriented:
// 9.2 -> 5.2 ms for the counts).  sel: 64 R LDS entries of this wave.
template <bool IN, int R, uint32_t CAP, uint32_t SLOTS>
__device__ __forceinline__ void cb_count5(const CbLds<CAP, SLOTS>& s, uint16_t* sel, uint32_t row, uint64_t rows,
                                          uint32_t L, uint32_t di, uint32_t iO, uint32_t iI, CbSums& t) {
  constexpr uint32_t kStride = CbLds<CAP, SLOTS>::kStride;
  const uint32_t lane = lane_id();
  uint32_t at = 0;
  for (uint64_t jw = rows; jw; jw &= jw - 1) {
    const uint32_t w = (uint32_t)__builtin_ctzll(jw), x = lane_value(row, w);
    if (lane < 32 && (x >> lane & 1)) sel[at + (uint32_t)__popc(x & ((1u << lane) - 1))] = (uint16_t)(w * 32 + lane);
    at += (uint32_t)__popc(x);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  uint32_t j[R], d[R], B[R][2 * R] = {};
  uint32_t mO[2 * R], mI[2 * R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool live = r * 64 + lane < L;
    j[r] = live ? sel[r * 64 + lane] : 0;
    d[r] = live ? min(di, s.deg[j[r]]) : 0;
    const uint64_t o = IN ? __ballot(live && (s.O[j[r] >> 5] >> (j[r] & 31) & 1)) : ~0ull;
    const uint64_t n = IN ? __ballot(live && (s.I[j[r] >> 5] >> (j[r] & 31) & 1)) : 0;
    mO[2 * r] = (uint32_t)o;
    mO[2 * r + 1] = (uint32_t)(o >> 32);
    mI[2 * r] = (uint32_t)n;
    mI[2 * r + 1] = (uint32_t)(n >> 32);
  }
  // bit kk of every row, member by member in order
  uint32_t cur[R] = {}, kk = 0;
  auto flush = [&](uint32_t q) {
#pragma unroll
    for (int z = 0; z < 2 * R; ++z)
      if (q == (uint32_t)z)
#pragma unroll
        for (int r = 0; r < R; ++r) B[r][z] = cur[r];
#pragma unroll
    for (int r = 0; r < R; ++r) cur[r] = 0;
  };
  for (uint64_t jw = rows; jw; jw &= jw - 1) {
    const uint32_t w = (uint32_t)__builtin_ctzll(jw);
    uint32_t x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = r * 64 + lane < L ? s.mat[w * kStride + j[r]] : 0;
    for (uint32_t left = lane_value(row, w); left; left &= left - 1) {
      const uint32_t b = (uint32_t)__builtin_ctz(left);
#pragma unroll
      for (int r = 0; r < R; ++r) cur[r] |= (x[r] >> b & 1) << (kk & 31);
      if ((++kk & 31) == 0) flush((kk >> 5) - 1);
    }
  }
  if (kk & 31) flush(kk >> 5);
#pragma unroll
  for (int jr = 0; jr < R; ++jr) {
    if (!IN && jr * 64 + lane < L) {
      t.v[kCbPre3] += 1;
      t.v[kCbExt3] += d[jr];
    }
    const uint32_t nj = L <= jr * 64u ? 0 : L - jr * 64u < 64 ? L - jr * 64u : 64;
    for (uint32_t jj = 0; jj < nj; ++jj) {
      uint32_t a = 1, b = 0;
      const uint32_t dj = lane_value(d[jr], jj);
      if (IN) {
        const uint32_t q = jj >> 5, bit = jj & 31;
        const uint32_t jO = (q ? mO[2 * jr + 1] : mO[2 * jr]) >> bit & 1, jI = (q ? mI[2 * jr + 1] : mI[2 * jr]) >> bit & 1;
        b = jI * iI;
        a = jO * (iO + iI) + b;
        if (!a) continue;
        if (lane == 0) {
          t.v[kCbPre3] += a;
          t.v[kCbExt3] += (uint64_t)a * dj;
        }
      }
      uint32_t m[2 * R], any = 0;
#pragma unroll
      for (int z = 0; z < 2 * R; ++z) any |= m[z] = lane_value(B[jr][z], jj);
      if (!any) continue;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        uint32_t cO = 0, cI = 0;
#pragma unroll
        for (int z = 0; z < 2 * R; ++z) {
          cO += (uint32_t)__popc(B[r][z] & m[z] & mO[z]);
          if (IN) cI += (uint32_t)__popc(B[r][z] & m[z] & mI[z]);
        }
        if (bit_of(m[2 * r], m[2 * r + 1], lane)) {
          const uint32_t dk = min(dj, d[r]);
          if (!IN) {
            t.v[kCbMatches] += cO;
            t.v[kCbPre4] += 1;
            t.v[kCbExt4] += dk;
          } else {
            const uint32_t kO = bit_of(mO[2 * r], mO[2 * r + 1], lane), kI = bit_of(mI[2 * r], mI[2 * r + 1], lane);
            const uint32_t f = kO * a + kI * b;
            t.v[kCbMatches] += (uint64_t)(kO * a) * cO + (uint64_t)(kI * b) * (cO + cI);
            t.v[kCbPre4] += f;
            t.v[kCbExt4] += (uint64_t)f * dk;
          }
        }
      }
    }
  }
}

// The cliques of v in rows wave, wave + nw, ... of its matrix (n members).
// Q: 4 or 5; IN: some member is in I (else O is all of them).
template <int Q, bool IN, uint32_t CAP, uint32_t SLOTS>
__device__ __forceinline__ void cb_count(const CbLds<CAP, SLOTS>& s, uint16_t* sel, uint32_t n, uint32_t dv,
                                         uint32_t wave, uint32_t nw, CbSums& t) {
  constexpr uint32_t kStride = CbLds<CAP, SLOTS>::kStride;
  const uint32_t lane = lane_id(), words = (n + 31) / 32;
  const uint32_t Ow = IN && lane < words ? s.O[lane] : ~0u, Iw = IN && lane < words ? s.I[lane] : 0;
  auto word = [&](uint32_t x, uint32_t w) { return w < words ? lane_value(x, w) : 0u; };
  for (uint32_t i = wave; i < n; i += nw) {
    const uint32_t row = lane < words ? s.mat[lane * kStride + i] : 0;
    const uint64_t rows = __ballot(row != 0);
    if (!rows) continue;
    const uint32_t di = min(dv, s.deg[i]);
    const uint32_t iO = IN ? lane_value(Ow, i >> 5) >> (i & 31) & 1 : 1, iI = IN ? lane_value(Iw, i >> 5) >> (i & 31) & 1 : 0;
    if (Q == 4) {
      const uint32_t rowO = row & Ow, rowI = row & Iw;
      for (uint32_t j0 = 0; j0 < n; j0 += 64) {
        const uint32_t lo = word(row, j0 / 32), hi = word(row, j0 / 32 + 1);
        if (!(lo | hi)) continue;
        const uint32_t j = j0 + lane;  // rows at n and beyond are masked by the bit
        uint32_t cO = 0, cI = 0;
        for (uint64_t left = rows; left; left &= left - 1) {
          const uint32_t w = (uint32_t)__builtin_ctzll(left);
          const uint32_t x = s.mat[w * kStride + j];
          cO += (uint32_t)__popc(x & lane_value(rowO, w));
          if (IN) cI += (uint32_t)__popc(x & lane_value(rowI, w));
        }
        if (bit_of(lo, hi, lane)) {
          const uint32_t dij = min(di, s.deg[j]);
          if (!IN) {
            t.v[kCbMatches] += cO;
            t.v[kCbPre3] += 1;
            t.v[kCbExt3] += dij;
          } else {
            const uint32_t jO = s.O[j >> 5] >> (j & 31) & 1, jI = s.I[j >> 5] >> (j & 31) & 1;
            const uint32_t a = jO * (iO + iI), b = jI * iI;
            t.v[kCbMatches] += (uint64_t)a * cO + (uint64_t)b * (cO + cI);
            t.v[kCbPre3] += a + b;
            t.v[kCbExt3] += (uint64_t)(a + b) * dij;
          }
        }
      }
    } else {
      const uint32_t L = (uint32_t)wave_sum((uint64_t)__popc(row));
      if (L <= 64) {
        cb_count5<IN, 1>(s, sel, row, rows, L, di, iO, iI, t);
        continue;
      }
      if (L <= 128) {
        cb_count5<IN, 2>(s, sel, row, rows, L, di, iO, iI, t);
        continue;
      }
      for (uint64_t jw = rows; jw; jw &= jw - 1) {
        const uint32_t w0 = (uint32_t)__builtin_ctzll(jw);
        for (uint32_t js = lane_value(row, w0); js; js &= js - 1) {
          const uint32_t j = w0 * 32 + (uint32_t)__builtin_ctz(js);
          const uint32_t jO = IN ? lane_value(Ow, w0) >> (j & 31) & 1 : 1, jI = IN ? lane_value(Iw, w0) >> (j & 31) & 1 : 0;
          const uint32_t a = jO * (iO + iI) + jI * iI, b = jI * iI;  // prefixes (v, i, j); those all in I
          if (IN && !a) continue;
          const uint32_t dij = min(di, s.deg[j]);
          if (lane == 0) {
            t.v[kCbPre3] += a;
            t.v[kCbExt3] += (uint64_t)a * dij;
          }
          const uint32_t m = lane < words ? row & s.mat[lane * kStride + j] : 0;
          const uint64_t ms = __ballot(m != 0);
          const uint32_t mO = m & Ow, mI = m & Iw;
          for (uint64_t kw = ms; kw;) {
            const uint32_t k0 = (uint32_t)__builtin_ctzll(kw) & ~1u;
            kw &= ~(3ull << k0);
            const uint32_t lo = word(m, k0), hi = word(m, k0 + 1);
            const uint32_t k = k0 * 32 + lane;
            uint32_t cO = 0, cI = 0;
            for (uint64_t left = ms; left; left &= left - 1) {
              const uint32_t w = (uint32_t)__builtin_ctzll(left);
              const uint32_t x = s.mat[w * kStride + k];
              cO += (uint32_t)__popc(x & lane_value(mO, w));
              if (IN) cI += (uint32_t)__popc(x & lane_value(mI, w));
            }
            if (bit_of(lo, hi, lane)) {
              const uint32_t dk = min(dij, s.deg[k]);
              if (!IN) {
                t.v[kCbMatches] += cO;
                t.v[kCbPre4] += 1;
                t.v[kCbExt4] += dk;
              } else {
                const uint32_t kO = s.O[k >> 5] >> (k & 31) & 1, kI = s.I[k >> 5] >> (k & 31) & 1;
                const uint32_t f = kO * a + kI * b;
                t.v[kCbMatches] += (uint64_t)(kO * a) * cO + (uint64_t)(kI * b) * (cO + cI);
                t.v[kCbPre4] += f;
                t.v[kCbExt4] += (uint64_t)f * dk;
              }
            }
          }
        }
      }
    }
  }
}

// One v per workgroup (CAP above 64) or per wave.
template <int Q, uint32_t CAP, uint32_t SLOTS, int NT>
__global__ void __launch_bounds__(NT) k_cb_cliques(HubGraph g, CbBits hb, const uint32_t* __restrict__ list,
                                                   const unsigned int* __restrict__ len,
                                                   unsigned long long* __restrict__ acc) {
  constexpr bool kWave = CAP <= 64;
  constexpr uint32_t kGroups = kWave ? NT / 64 : 1, kNT = kWave ? 64 : NT;
  __shared__ CbLds<CAP, SLOTS> lds[kGroups];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(wave_id());
  const uint32_t grp = kWave ? wave : 0, tid = kWave ? lane_id() : threadIdx.x;
  CbLds<CAP, SLOTS>& s = lds[grp];
  const unsigned int total = *len;
  CbSums t;
  uint16_t* sel = (uint16_t*)s.key + (kWave ? 0 : wave) * 128;  // the table is done with once the matrix is built
  static_assert(SLOTS * 2 >= kNT / 64 * 128, "room for every wave's list");
  auto sync = [] {
    if (kWave) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  };
  for (uint64_t k = (uint64_t)blockIdx.x * kGroups + grp; k < total; k += (uint64_t)gridDim.x * kGroups) {
    const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[k]);
    const uint32_t n = cb_build(s, g, hb, v, tid, kNT, sync), dv = g.deg(0, v);
    const uint32_t w = kWave ? 0 : wave, nw = kNT / 64;
    if (g.end[1][v] == g.rp[1][v])
      cb_count<Q, false>(s, sel, n, dv, w, nw, t);
    else
      cb_count<Q, true>(s, sel, n, dv, w, nw, t);
  }
#pragma unroll
  for (int i = 0; i < kCbAcc; ++i) {
    const uint64_t x = wave_sum(t.v[i]);
    if (lane_id() == 0 && x) atomicAdd(acc + i, (unsigned long long)x);
  }
}

// most: the greatest number of neighbours a vertex may have below it
template <int Q>
static void launch(gj_ctx* c, const HubGraph& g, const CbBits& hb, const uint32_t* lists, const unsigned int* len,
                   uint64_t most, unsigned long long* acc) {
  const unsigned cus = (unsigned)c->num_cus;
  const uint64_t n = g.n;
  if (most > kCbCap[2])
    k_cb_cliques<Q, kCbCap[3], 2048, 1024><<<cus, 1024, 0, c->stream>>>(g, hb, lists + 3 * n, len + 3, acc);
  if (most > kCbCap[1])
    k_cb_cliques<Q, kCbCap[2], 1024, 512><<<cus * 3, 512, 0, c->stream>>>(g, hb, lists + 2 * n, len + 2, acc);
  if (most > kCbCap[0])
    k_cb_cliques<Q, kCbCap[1], 512, 256><<<cus * 8, 256, 0, c->stream>>>(g, hb, lists + n, len + 1, acc);
  k_cb_cliques<Q, kCbCap[0], 128, 256><<<cus * 8, 256, 0, c->stream>>>(g, hb, lists, len, acc);
}

bool clique_bits_count(gj_ctx* c, const Version& v, uint32_t n, int q, KernelTimer& timer, uint64_t out[6]) {
  for (int i = 0; i < 6; ++i) out[i] = 0;
  if (!v.m) return true;
  HubOrder order;
  if (!choose_order(v, n, q, order)) return false;
  constexpr size_t kCtl = kCbAcc * 8 + (kCbClasses + 2) * 4;
  unsigned long long* acc = (unsigned long long*)ws_get(c, "cb_ctl", kCtl);
  unsigned int* len = (unsigned int*)(acc + kCbAcc);
  uint32_t* lists = (uint32_t*)ws_get(c, "cb_lists", (uint64_t)kCbClasses * n * sizeof(uint32_t));
  const unsigned cus = (unsigned)c->num_cus;
  const uint64_t most = (uint64_t)v.max_deg[0] + v.max_deg[1];
  const uint32_t* row = nullptr;
  HubGraph g;
  auto prepare = [&](HubOrder o) {
    if (!hub_graph(c, v, n, o, true, g, row)) return false;
    GJ_HIP(hipMemsetAsync(acc, 0, kCtl, c->stream));
    const bool fits = o != HubOrder::kReversed || (!v.blur && !hub_limit_open(v));
    k_cb_classes<<<grid_for(n, kBlock, cus * 8), kBlock, 0, c->stream>>>(g, fits ? 1 : 0, len, lists);
    GJ_HIP(hipGetLastError());
    if (fits) return true;
    unsigned int beyond = 0;
    read_bytes(c, &beyond, len + kCbClasses, sizeof(beyond));
    return beyond == 0;
  };
  // reversed ids that changes have blurred may say too little of who is a hub
  if (!prepare(order) && (order != HubOrder::kReversed || !v.blur || !prepare(HubOrder::kDegree))) return false;
  CbBits hb{};
  if (v.m >= kCbBitsEdges && most > kCbCap[0]) {
    // quads of the two directions end to end: does any vertex have an in-prefix?
    uint32_t h[2];
    read_u32s(c, {g.pq[1], g.pq[1] + n}, h);
    const uint32_t top = std::min(n, kCbTop);
    const uint64_t words = (uint64_t)top * (kCbTop / 32);
    const int dirs = h[0] == h[1] ? 1 : 2;
    uint32_t* b = (uint32_t*)ws_get(c, "cb_bits", dirs * words * sizeof(uint32_t));
    GJ_HIP(hipMemsetAsync(b, 0, dirs * words * sizeof(uint32_t), c->stream));
    hb.bits[0] = b;
    hb.bits[1] = dirs == 2 ? b + words : nullptr;
    k_cb_bits<<<(2 * top + kBlock / 64 - 1) / (kBlock / 64), kBlock, 0, c->stream>>>(g, top, b,
                                                                                    dirs == 2 ? b + words : nullptr);
  }
  timer.start();
  k_cb_ext2<<<grid_for(v.m, kBlock * 4, cus * 16), kBlock, 0, c->stream>>>(g, row, v.m, acc);
  if (q == 4)
    launch<4>(c, g, hb, lists, len, most, acc);
  else
    launch<5>(c, g, hb, lists, len, most, acc);
  timer.stop();
  GJ_HIP(hipGetLastError());
  unsigned long long h[kCbAcc];
  read_bytes(c, h, acc, sizeof(h));
  for (int i = 0; i < kCbAcc; ++i) out[i] = h[i];
  return true;
}

}  // namespace gj
