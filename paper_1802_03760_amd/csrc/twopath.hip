// Whole counts of the diamond edge(a0,a1), edge(a0,a2), edge(a1,a3),
// edge(a2,a3) and of the 4-cycle edge(a0,a1), edge(a1,a2), edge(a2,a3),
// edge(a3,a0), without inequalities, from the numbers of 2-paths between
// pairs of vertices.
//
// Vertices are renamed by descending degree (in + out), so a small id is a
// hub.  A match is counted at its least vertex v: with w > v the vertex
// opposite to v in the 4-cycle of the query, the two others are mid vertices
// u > v of 2-paths between v and w.  Per pair (v, w), v < w, with u > v:
//   A = #{v -> u -> w}     B = #{w -> u -> v}
//   O = #{u -> v, u -> w}  I = #{v -> u, w -> u}
// Diamond (join semantics: a1 = a2 and a0 = a3 allowed):
//   v = a0 or v = a3, a0 != a3:  sum A^2 + B^2
//   v = a1 or v = a2, a1 != a2, a0 != a3:  2 (sum O I - sum K), K = #{u: u
//     both ways connected to v and to w} (the pairs with a0 = a3)
//   v = a1 = a2, a0 != a3:  per v, in>(v) out>(v) - r>(v)
//   a0 = a3 = x:  r(x)^2
// 4-cycle (the four rotations of v at a0, a0 != a2; and a0 = a2 or a1 = a3):
//   4 sum A B + 2 sum r>(v)^2
// where r(x) counts x's reciprocal neighbours and > restricts a set to ids
// above the vertex.
//
// The pairs are grouped by w: v ranges over the entries below min(u, w) of
// u's sorted row, a prefix, for u in w's row.  That is Chiba and Nishizeki's
// order (the work is the sum over edges of the hub-side degree, not over all
// 2-paths: 6.7e9 instead of 2.1e10 entries for the diamond at R-MAT-20), and
// v is nearly always a hub, so a counter array over [0, 32768) in LDS takes
// 99% of them.  A (or O) and B (or I) share one word per v.
//
// Measured (MI355X): R-MAT-18 diamond 128.3 -> 3.4 ms, 4-cycle of a
// 600,011-vertex R-MAT graph (8.4e6 edges) 404 -> 3.8 ms, against one walk of
// all 2-paths of an a0 with atomics on a dense array of counters in HBM, which
// were its bound (1.8e10 atomics/s).  Now the walks (k_hub_dense, k_hub_small,
// k_hub_wave) are 70% of the time and issue-bound, the renaming's sorts 12%.
#include <algorithm>

#include "gj_internal.h"
#include "hub.h"
#include "prim.h"

namespace gj {

// Accumulators of one call.
enum { kTpAB, kTpOI, kTpRec2, kTpBoth, kTpMid, kTpRecUp2, kTpPaths, kTpMin, kTpWalk, kTpSegs, kTpAcc };

// ---------------------------------------------------------------- reciprocal pairs
// Per vertex, its reciprocal neighbours (rec) and those below it (rec_lo):
// one thread per edge x -> y looks for x among the shorter of out(y) and for
// y among in(x).  Lanes of a wave that share x add once.
__global__ void __launch_bounds__(kBlock) k_hub_recip(HubGraph g, const uint32_t* __restrict__ row, uint64_t m,
                                                      uint32_t* __restrict__ rec, uint32_t* __restrict__ rec_lo) {
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t b = (uint64_t)blockIdx.x * blockDim.x; b < m; b += gs) {  // whole waves take every step
    const uint64_t e = b + threadIdx.x;
    bool hit = false, lo = false;
    uint32_t x = 0;
    if (e < m) {
      x = row[e];
      const uint32_t y = g.col[0][e];
      const uint32_t yn = g.deg(0, y), xn = g.deg(1, x);
      hit = yn <= xn ? contains_u32(g.row(0, y), 0, yn, x) : contains_u32(g.row(1, x), 0, xn, y);
      lo = hit && y < x;
    }
    uint64_t left = __ballot(hit);
    while (left) {
      const int first = __ffsll((unsigned long long)left) - 1;
      const uint32_t fx = __shfl(x, first, 64);
      const uint64_t same = __ballot(hit && x == fx);
      const uint64_t same_lo = __ballot(lo && x == fx);
      if (lane_id() == first) {
        atomicAdd(&rec[fx], (uint32_t)__popcll(same));
        if (same_lo) atomicAdd(&rec_lo[fx], (uint32_t)__popcll(same_lo));
      }
      left &= ~same;
    }
  }
}

// The terms of the header that depend on one vertex.
__global__ void __launch_bounds__(kBlock) k_hub_terms(HubGraph g, const uint32_t* __restrict__ rec,
                                                      const uint32_t* __restrict__ rec_lo, int cycle,
                                                      unsigned long long* __restrict__ acc) {
  uint64_t rec2 = 0, both = 0, mid = 0, up2 = 0, paths = 0, walk = 0;
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < g.n; v += gs) {
    const uint64_t r = rec[v], lo = rec_lo[v];
    const uint64_t out = g.deg(0, v), in = g.deg(1, v);
    const uint64_t out_up = g.rp[0][v + 1] - g.end[0][v], in_up = g.rp[1][v + 1] - g.end[1][v];
    rec2 += r * r;
    if (lo) both += lo * (r - 1) - lo * (lo - 1) / 2;  // pairs v' < w' of its reciprocal row with v' below it
    mid += in_up * out_up - (r - lo);
    up2 += (r - lo) * (r - lo);
    paths += cycle ? in * out : out * out;
    walk += in * out;
  }
  const uint64_t t[6] = {rec2, both, mid, up2, paths, walk};
  const int at[6] = {kTpRec2, kTpBoth, kTpMid, kTpRecUp2, kTpPaths, kTpWalk};
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const uint64_t s = block_sum<kBlock>(t[i]);
    if (threadIdx.x == 0 && s) atomicAdd(acc + at[i], (unsigned long long)s);
  }
}

// ---------------------------------------------------------------- classes of w
// Classes by the entries w's walk reads (an upper bound: whole quads, and
// rows' prefixes up to u, not min(u, w)), those of them from the first quad
// with an id of kTpHubs on, and w's degrees:
//  0 one wave, hash table of 1,024 slots          at most 512 entries
//  1 256 threads, 8-bit counters below kTpHubs     both degrees at most 255,
//                                                  none above
//  2 the same, and a hash table for those above    at most 1,024 above
//  3 1,024 threads, array of 2 x 16 bits           both degrees at most 65,535
//  4 1,024 threads, array of 2 x 32 bits           the rest
// A count of mid vertices is at most w's degree in either direction, so no
// field overflows.  Rows beyond kTpProbe entries go to the last two
// without being measured.  A w without neighbours on one side has no A B and
// no O I; one with a single neighbour has A + B = 1 at every entry of its
// walk and is summed here.
// A w of the last two takes a step for every kTpSeg3 or kTpSeg4 ids below it,
// whatever its entries: count_2path adds the steps up (kTpSegs) against the
// 2-paths (kTpWalk).
constexpr int kTpClasses = 5;
constexpr uint32_t kTpWave = 512, kTpAbove = 1024, kTpProbe = 512;
constexpr int kTpSeg3 = 32768, kTpSeg4 = 16384;

// A workgroup classes 64 vertices, 16 lanes to each for its walk's length,
// and takes its places in the lists with one atomic per pass and class.
// pass 0 walks in-prefixes of in-neighbours and out-prefixes of
// out-neighbours (A, B), pass 1 the crossed ones (O, I).
__global__ void __launch_bounds__(kBlock) k_hub_classes(HubGraph g, int cycle, unsigned int* __restrict__ cnt,
                                                        uint32_t* __restrict__ lists, uint64_t stride,
                                                        unsigned long long* __restrict__ acc) {
  __shared__ int8_t cls_s[2][64];
  const uint32_t sub = threadIdx.x & 15, grp = threadIdx.x / 16;
  const int passes = cycle ? 1 : 2;
  uint64_t ones = 0, segs = 0;
  for (uint64_t b = (uint64_t)blockIdx.x * 64; b < g.n; b += (uint64_t)gridDim.x * 64) {
    for (uint32_t k = 0; k < 4; ++k) {
      const uint32_t slot = k * 16 + grp;
      const uint64_t w = b + slot;
      uint32_t deg[2] = {0, 0};
      uint64_t work[2] = {0, 0};  // entries, and those above kTpHubs << 32
      if (w < g.n) {
        for (int s = 0; s < 2; ++s) deg[s] = g.deg(s, w);
        if (deg[0] + (uint64_t)deg[1] <= kTpProbe) {
          for (int s = 0; s < 2; ++s)
            for (uint32_t i = sub; i < deg[s]; i += 16) {
              const uint32_t u = g.row(s, w)[i];
              for (int p = 0; p < passes; ++p) {
                const int d = p ? 1 - s : s;
                const uint32_t e = g.pq[d][u + 1], all = e - g.pq[d][u], above = e - g.mq[d][u];
                // capped, so that no field of a sum over 512 rows overflows
                work[p] += 4 * min(all, 1u << 18) | (uint64_t)(4 * min(above, 1u << 18)) << 32;
              }
            }
        } else {
          work[0] = work[1] = 1ull << 52 | 1u << 20;
        }
      }
      for (int p = 0; p < passes; ++p) {
        uint32_t t = (uint32_t)work[p], above = (uint32_t)(work[p] >> 32);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
          t += __shfl_xor(t, o, 16);
          above += __shfl_xor(above, o, 16);
        }
        if (w <= kTpHubs) above = 0;
        if (sub == 0) {
          int cls = -1;
          const bool product = cycle || p;
          if (t && w && w < g.n && !(product && (!deg[0] || !deg[1]))) {  // w = 0 has no v below it
            if (deg[0] + (uint64_t)deg[1] == 1) {
              // its one neighbour u: the entries below min(u, w)
              const int s = deg[1] ? 1 : 0;
              const uint32_t u = g.row(s, w)[0];
              const uint32_t len = g.end[s][u] - g.rp[s][u];
              ones += u < w ? len : lower_bound_u32(g.row(s, u), 0, len, (uint32_t)w);
            }
            else if (t <= kTpWave) cls = 0;
            else if (deg[0] <= 255 && deg[1] <= 255 && above <= kTpAbove) cls = above ? 2 : 1;
            else if (deg[0] <= 65535 && deg[1] <= 65535) cls = 3;
            else cls = 4;
            if (cls >= 3) segs += (w + (cls == 3 ? kTpSeg3 : kTpSeg4) - 1) / (cls == 3 ? kTpSeg3 : kTpSeg4);
          }
          cls_s[p][slot] = (int8_t)cls;
        }
      }
    }
    __syncthreads();
    const int p = wave_id();  // a wave per pass
    if (p < passes) {
      const int c = cls_s[p][lane_id()];
      uint32_t rank = 0, mine_n = 0;
#pragma unroll
      for (int q = 0; q < kTpClasses; ++q) {
        const uint64_t mine = __ballot(c == q);
        if (c == q) rank = (uint32_t)__popcll(mine & lanemask_lt());
        if (lane_id() == q) mine_n = (uint32_t)__popcll(mine);
      }
      uint32_t at = 0;
      if (mine_n) at = atomicAdd(cnt + p * kTpClasses + lane_id(), mine_n);
      at = __shfl(at, c < 0 ? 0 : c, 64);
      if (c >= 0) lists[(uint64_t)(p * kTpClasses + c) * stride + at + rank] = (uint32_t)(b + lane_id());
    }
    __syncthreads();
  }
  ones = block_sum<kBlock>(ones);
  if (threadIdx.x == 0 && ones) atomicAdd(acc + kTpAB, (unsigned long long)ones);
  segs = block_sum<kBlock>(segs);
  if (threadIdx.x == 0 && segs) atomicAdd(acc + kTpSegs, (unsigned long long)segs);
}

// ---------------------------------------------------------------- the walk
// w's neighbours: the first nin of the walk's rows belong to in-neighbours
// (fields A, O), the other nout to out-neighbours (B, I).
struct HubRow {
  uint32_t w, nin, nout;
  uint32_t in, out;  // where its rows start, per direction
};

__device__ __forceinline__ HubRow hub_row(const HubGraph& g, uint32_t w) {
  return HubRow{w, g.deg(1, w), g.deg(0, w), g.rp[1][w], g.rp[0][w]};
}

// The walk of w: the entries x in [s0, lim) of the prefix of every neighbour
// u's row (pass 0: u's row in the direction of w's own row, pass 1: in the
// other).  Neighbours are dealt to the waves in batches of up to 64, one to a
// lane.  load(), bounds() and pack() are apart so that what each loads can
// arrive while another walk runs.
struct HubBatch {
  uint32_t u;         // lane's neighbour
  bool live, out;     // there is one; it is an out-neighbour
  uint32_t b, e;      // its quads to read, in its direction
  uint32_t p;         // packed: its first quad of pre
  uint32_t len;       // their number, and the side in the top bit
};

__device__ __forceinline__ uint32_t batch_size(const HubRow& h, uint32_t nwaves) {
  const uint64_t per = ((uint64_t)h.nin + h.nout + nwaves - 1) / nwaves;
  return per > 64 ? 64 : (uint32_t)per;
}

__device__ __forceinline__ HubBatch batch_load(const HubGraph& g, const HubRow& h, uint64_t i0, uint32_t G) {
  HubBatch t{};
  const uint64_t i = i0 + lane_id();
  t.live = (uint32_t)lane_id() < G && i < (uint64_t)h.nin + h.nout;
  t.out = t.live && i >= h.nin;
  if (t.live) t.u = t.out ? g.col[0][h.out + (i - h.nin)] : g.col[1][h.in + i];
  return t;
}

// from: 0 the whole prefix, 1 its part at ids of kTpHubs and above
__device__ __forceinline__ void batch_bounds(const HubGraph& g, int pass, int from, HubBatch& t) {
  if (!t.live) return;
  const bool fwd = t.out != (pass != 0);  // the direction of u's row
  t.b = from ? (fwd ? g.mq[0] : g.mq[1])[t.u] : (fwd ? g.pq[0] : g.pq[1])[t.u];
  t.e = (fwd ? g.pq[0] : g.pq[1])[(uint64_t)t.u + 1];
}

// Leaves out the quads below s0 and moves the rows that have any to the
// lowest lanes.
__device__ __forceinline__ void batch_pack(const HubGraph& g, uint32_t s0, HubBatch& t) {
  uint32_t n = 0;
  t.p = 0;
  if (t.live) {
    uint32_t b = t.b, len = t.e - t.b;
    if (s0)
      while (len > 0) {
        const uint32_t half = len >> 1;
        if (g.pre[(uint64_t)b + half].w < s0) {
          b += half + 1;
          len -= half + 1;
        } else {
          len = half;
        }
      }
    t.p = b;
    n = t.e - b;
  }
  const uint64_t some = __ballot(n != 0);
  const uint32_t cn = (uint32_t)__popcll(some);
  // lane i's row goes to the rank of i among the rows kept; the others fill up
  // the lanes behind, so that every lane receives one
  const uint64_t lt = lanemask_lt();
  const uint32_t to = n ? (uint32_t)__popcll(some & lt) : cn + (uint32_t)__popcll(~some & lt);
  t.p = (uint32_t)__builtin_amdgcn_ds_permute(to * 4, (int)t.p);
  t.len = (uint32_t)__builtin_amdgcn_ds_permute(to * 4, (int)(n | (t.out ? 0x80000000u : 0)));
  t.live = (uint32_t)lane_id() < cn;
}

// The walk of w's batches from its first, t (packed from s0).
template <int DEPTH, class F>
__device__ __forceinline__ void walk_pairs(const HubGraph& g, int pass, int from, const HubRow& h, HubBatch t,
                                           uint32_t s0, uint32_t lim, uint32_t wave, uint32_t nwaves, F add) {
  const uint64_t d = (uint64_t)h.nin + h.nout;
  const uint32_t G = batch_size(h, nwaves);
  const uint64_t step = (uint64_t)nwaves * G;
  uint64_t i0 = (uint64_t)wave * G;
  HubBatch n{};
  if (i0 + step < d) {
    n = batch_load(g, h, i0 + step, G);
    batch_bounds(g, pass, from, n);
  }
  for (; i0 < d; i0 += step) {
    HubBatch f{};
    if (i0 + 2 * step < d) f = batch_load(g, h, i0 + 2 * step, G);
    walk_batch<DEPTH, 31>(g.pre, t.p, t.len, (uint32_t)__popcll(__ballot(t.live)), lim, add);
    if (i0 + step < d) batch_pack(g, s0, n);
    t = n;
    batch_bounds(g, pass, from, f);
    n = f;
  }
}

// What a pair with fields (a, b) contributes: op 0 a^2 + b^2, op 1 a b.
__device__ __forceinline__ uint64_t pair_term(int op, uint64_t a, uint64_t b) { return op ? a * b : a * a + b * b; }

// The w of a list taken by one workgroup or wave, every step-th from k: the
// walk of one overlaps the loads of the next ones' ids, row bounds, neighbours
// and neighbours' rows, a stage per step.  Without that the chain of five
// dependent loads before each walk, about 7 us, was most of the time of the
// small classes.
template <int NW>
struct HubFeed {
  const HubGraph& g;
  const uint32_t* ws;
  uint64_t total, step, k;
  int pass;
  uint32_t wave;
  HubRow cur, n1, n2;
  uint32_t w3;
  HubBatch t, b1;

  __device__ __forceinline__ uint32_t id(uint64_t i) const {
    return i < total ? (uint32_t)__builtin_amdgcn_readfirstlane((int)ws[i]) : 0;
  }
  __device__ __forceinline__ HubRow row(uint64_t i, uint32_t w) const { return i < total ? hub_row(g, w) : HubRow{}; }
  __device__ __forceinline__ HubBatch first(const HubRow& r) const {
    const uint32_t G = batch_size(r, NW);
    return batch_load(g, r, (uint64_t)wave * G, G);
  }
  __device__ __forceinline__ HubFeed(const HubGraph& g_, int pass_, const uint32_t* ws_, uint64_t total_,
                                     uint64_t step_, uint64_t k_, uint32_t wave_)
      : g(g_), ws(ws_), total(total_), step(step_), k(k_), pass(pass_), wave(wave_) {
    cur = row(k, id(k));
    n1 = row(k + step, id(k + step));
    n2 = row(k + 2 * step, id(k + 2 * step));
    w3 = id(k + 3 * step);
    t = first(cur);
    batch_bounds(g, pass, 0, t);
    batch_pack(g, 0, t);
    b1 = first(n1);
  }
  __device__ __forceinline__ bool more() const { return k < total; }
  // walk(cur, t) with the loads of the later ones in flight, then on to the next
  template <class F>
  __device__ __forceinline__ void next(F walk) {
    const uint32_t w4 = id(k + 4 * step);
    const HubRow n3 = row(k + 3 * step, w3);
    HubBatch b2 = first(n2);
    batch_bounds(g, pass, 0, b1);
    walk();
    batch_pack(g, 0, b1);
    t = b1;
    b1 = b2;
    cur = n1;
    n1 = n2;
    n2 = n3;
    w3 = w4;
    k += step;
  }
};

__device__ __forceinline__ uint64_t pair_terms8(int op, uint32_t c) {
  return pair_term(op, c & 0xFF, (c >> 8) & 0xFF) + pair_term(op, (c >> 16) & 0xFF, c >> 24);
}
__device__ __forceinline__ uint64_t pair_terms16(int op, uint32_t c) { return pair_term(op, c & 0xFFFF, c >> 16); }

// Sum of term over q[0, n) and all of it cleared, by nt threads.
template <class F>
__device__ __forceinline__ uint64_t take_counts(uint4* q, uint32_t n, uint32_t tid, uint32_t nt, F term) {
  uint64_t s = 0;
  for (uint32_t i = tid; i < n; i += nt) {
    const uint4 c = q[i];
    if (c.x | c.y | c.z | c.w) {
      q[i] = make_uint4(0, 0, 0, 0);
      s += term(c);
    }
  }
  return s;
}

// Hash table of SLOTS (zeroed) keys, v + 1, and as many 2 x 16-bit counters;
// linear probing.  Callers put in at most half as many v as there are slots,
// so an insertion always ends.
template <int SLOTS>
__device__ __forceinline__ void hash_add(uint32_t* key, uint32_t* cnt, uint32_t x, uint32_t side) {
  uint32_t p = (x * 0x9E3779B1u) >> (32 - __builtin_ctz(SLOTS));
  for (;;) {
    uint32_t o = key[p];
    if (o == 0) o = atomicCAS(&key[p], 0u, x + 1);
    if (o == 0 || o == x + 1) break;
    p = (p + 1) & (SLOTS - 1);
  }
  atomicAdd(&cnt[p], 1u << (16 * side));
}

// One w per workgroup: two counters of BITS bits per v over [s0, s0 + SEG) in
// LDS, s0 in steps of SEG below w (one step for nearly every entry, see the
// header; a later one costs a search per row and the scan of its counters).
// Bound by the LDS adds and the latency of the rows' loads, which come from
// L2 (every row is read once per neighbour).
template <int BITS, int SEG>
__global__ void __launch_bounds__(1024) k_hub_dense(HubGraph g, int pass, int op, const uint32_t* __restrict__ ws,
                                                    const unsigned int* __restrict__ nws,
                                                    unsigned long long* __restrict__ acc) {
  constexpr int kNW = 16;
  constexpr int kWords = SEG / 32 * (2 * BITS);  // 32-bit words
  __shared__ __align__(16) uint32_t cnt[kWords + 64];
  const uint32_t idle = kWords + lane_id();
  const uint32_t tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(wave_id());
  const unsigned int total = *nws;
  if (blockIdx.x >= total) return;
  for (uint32_t i = tid; i < kWords; i += 1024) cnt[i] = 0;
  __syncthreads();
  uint64_t sum = 0;
  HubFeed<kNW> f(g, pass, ws, total, gridDim.x, blockIdx.x, wave);
  while (f.more())
    f.next([&] {
      const uint32_t w = f.cur.w;
      for (uint32_t s0 = 0; s0 < w; s0 += SEG) {
        const uint32_t lim = w - s0 < (uint32_t)SEG ? w : s0 + SEG;
        if (s0) {
          f.t = f.first(f.cur);
          batch_bounds(g, pass, 0, f.t);
          batch_pack(g, s0, f.t);
        }
        walk_pairs<4>(g, pass, 0, f.cur, f.t, s0, lim, wave, kNW, [&](uint32_t x, uint32_t side) {
          const bool in = x - s0 < lim - s0;  // else the lane's own idle word
          if (BITS == 16)
            atomicAdd(&cnt[in ? x - s0 : idle], 1u << (16 * side));
          else
            atomicAdd(&cnt[in ? 2 * (x - s0) + side : idle], 1u);
        });
        __syncthreads();
        // 16-byte steps; entries of the last one at lim and beyond are zero
        sum += take_counts((uint4*)cnt, ((lim - s0) * (2 * BITS / 8) + 15) / 16, tid, 1024, [&](const uint4& c) {
          return BITS == 16 ? pair_terms16(op, c.x) + pair_terms16(op, c.y) + pair_terms16(op, c.z) + pair_terms16(op, c.w)
                            : pair_term(op, c.x, c.y) + pair_term(op, c.z, c.w);
        });
        __syncthreads();
      }
    });
  sum = block_sum<1024>(sum);
  if (tid == 0 && sum) atomicAdd(acc, (unsigned long long)sum);
}

// One w of small degree per workgroup of 256: a pair of 8-bit counters for
// every v below kTpHubs, and (ABOVE) then a hash table of 2,048 slots in the
// same LDS for the entries from there on, 1.6% of all at R-MAT-20.  32 KiB
// keep four workgroups on a CU, against two with counters for 32,768 v.
template <bool ABOVE>
__global__ void __launch_bounds__(kBlock) k_hub_small(HubGraph g, int pass, int op, const uint32_t* __restrict__ ws,
                                                      const unsigned int* __restrict__ nws,
                                                      unsigned long long* __restrict__ acc) {
  constexpr int kNW = kBlock / 64;
  constexpr int kSlots = 2 * kTpAbove;
  // the counters, and a word per lane for what does not count
  __shared__ __align__(16) uint32_t cnt[kTpHubs / 2 + 64];
  const uint32_t idle = kTpHubs + 2 * lane_id();
  const uint32_t tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(wave_id());
  const unsigned int total = *nws;
  if (blockIdx.x >= total) return;
  for (uint32_t i = tid; i < kTpHubs / 2; i += kBlock) cnt[i] = 0;
  __syncthreads();
  uint64_t sum = 0;
  HubFeed<kNW> f(g, pass, ws, total, gridDim.x, blockIdx.x, wave);
  while (f.more())
    f.next([&] {
      const uint32_t lim = min(f.cur.w, kTpHubs);
      HubBatch a{};
      if (ABOVE) {
        a = f.first(f.cur);
        batch_bounds(g, pass, 1, a);
      }
      walk_pairs<2>(g, pass, 0, f.cur, f.t, 0, lim, wave, kNW, [&](uint32_t x, uint32_t side) {
        const uint32_t y = x < lim ? x : idle;
        atomicAdd(&cnt[y >> 1], (1u << (8 * side)) << (16 * (y & 1)));
      });
      __syncthreads();
      sum += take_counts((uint4*)cnt, (lim + 7) / 8, tid, kBlock, [&](const uint4& c) {
        return pair_terms8(op, c.x) + pair_terms8(op, c.y) + pair_terms8(op, c.z) + pair_terms8(op, c.w);
      });
      __syncthreads();
      if (ABOVE) {
        batch_pack(g, 0, a);
        const uint32_t w = f.cur.w;
        walk_pairs<2>(g, pass, 1, f.cur, a, 0, w, wave, kNW, [&](uint32_t x, uint32_t side) {
          if (x >= kTpHubs && x < w) hash_add<kSlots>(cnt, cnt + kSlots, x, side);
        });
        __syncthreads();
        sum += take_counts((uint4*)(cnt + kSlots), kSlots / 4, tid, kBlock, [&](const uint4& c) {
          return pair_terms16(op, c.x) + pair_terms16(op, c.y) + pair_terms16(op, c.z) + pair_terms16(op, c.w);
        });
        take_counts((uint4*)cnt, kSlots / 4, tid, kBlock, [](const uint4&) { return 0ull; });
        __syncthreads();
      }
    });
  sum = wave_sum(sum);
  if (lane_id() == 0 && sum) atomicAdd(acc, (unsigned long long)sum);
}

// One w per wave, all its entries in a hash table of 1,024 slots: the
// low-degree w are most of the vertices and few of the entries, and the scan
// of an array of counters would cost them more than their walk.
__global__ void __launch_bounds__(kBlock) k_hub_wave(HubGraph g, int pass, int op, const uint32_t* __restrict__ ws,
                                                     const unsigned int* __restrict__ nws,
                                                     unsigned long long* __restrict__ acc) {
  constexpr int kWaves = kBlock / 64, kSlots = 2 * kTpWave;
  __shared__ __align__(16) uint32_t key_s[kWaves][kSlots], cnt_s[kWaves][kSlots];
  const uint32_t wave = __builtin_amdgcn_readfirstlane(wave_id()), lane = lane_id();
  uint32_t *key = key_s[wave], *cnt = cnt_s[wave];
  const unsigned int total = *nws;
  for (uint32_t i = lane; i < kSlots; i += 64) key[i] = cnt[i] = 0;
  auto sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  sync();
  uint64_t sum = 0;
  HubFeed<1> f(g, pass, ws, total, (uint64_t)gridDim.x * kWaves, (uint64_t)blockIdx.x * kWaves + wave, 0);
  while (f.more())
    f.next([&] {
      const uint32_t w = f.cur.w;
      walk_pairs<2>(g, pass, 0, f.cur, f.t, 0, w, 0, 1, [&](uint32_t x, uint32_t side) {
        if (x < w) hash_add<kSlots>(key, cnt, x, side);
      });
      sync();
      for (uint32_t i = lane; i < kSlots / 4; i += 64) {
        uint4* q = (uint4*)cnt + i;
        const uint4 c = *q;
        if (c.x | c.y | c.z | c.w) {
          *q = make_uint4(0, 0, 0, 0);
          ((uint4*)key)[i] = make_uint4(0, 0, 0, 0);
          sum += pair_terms16(op, c.x) + pair_terms16(op, c.y) + pair_terms16(op, c.z) + pair_terms16(op, c.w);
        }
      }
      sync();
    });
  sum = wave_sum(sum);
  if (lane == 0 && sum) atomicAdd(acc, (unsigned long long)sum);
}

// ---------------------------------------------------------------- the stage-3 counter
// extensions[3] of the depth-first evaluation: over the centre c of a pair of
// edges, the sum over x in its first row and y in its second of min(f(x),
// s(y)).  Diamond: c = a0, both rows out(c), f = s = out-degree.  4-cycle:
// c = a1, rows in(c) and out(c), f = in-degree, s = out-degree.
//
// Rows of at most kMinRow entries: one wave per centre, the first row's
// values in registers, the second's broadcast lane by lane.  Longer rows: a
// workgroup per centre counts the values of both rows, capped at kMinBins,
// in LDS histograms; min(a, b) = #{t >= 1: a >= t and b >= t}, so the part up
// to the cap is a sum over t of products of suffix counts, and the values
// above the cap (few vertices have that degree) are compared pair by pair on
// what exceeds it.  That replaces d^2 comparisons of a hub row by d
// increments: 1.5e11 of them at R-MAT-22.
constexpr uint32_t kMinRow = 512, kMinBins = 4096;

// T: 32 bits while 8 x 64 values below 2^22 add up in it
template <int R, typename T>
__device__ __forceinline__ uint64_t min_pairs(const uint32_t (&a)[8], uint32_t y, uint32_t nb) {
  T s = 0;
  for (uint32_t j = 0; j < nb; ++j) {
    const uint32_t b = lane_value(y, j);
#pragma unroll
    for (int r = 0; r < R; ++r) s += a[r] < b ? a[r] : b;
  }
  return s;
}

// The sum over the centres with short rows, by the grid's waves; the others
// are listed in big.
template <typename T>
__device__ __forceinline__ uint64_t min_rows(const HubGraph& g, int first, uint64_t wave, uint64_t waves,
                                             uint32_t* __restrict__ big, unsigned int* __restrict__ nbig) {
  const uint32_t lane = lane_id();
  uint64_t sum = 0;
  for (uint64_t c = wave; c < g.n; c += waves) {
    const uint32_t na = g.deg(first, c), nb = g.deg(0, c);
    if (!na || !nb) continue;
    if (na > kMinRow || nb > kMinRow) {
      if (lane == 0) big[atomicAdd(nbig, 1u)] = (uint32_t)c;
      continue;
    }
    const uint32_t *ra = g.row(first, c), *rb = g.row(0, c);
    uint32_t a[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) a[r] = r * 64 + lane < na ? g.deg(first, ra[r * 64 + lane]) : 0;
    for (uint32_t t = 0; t < nb; t += 64) {
      const uint32_t cn = nb - t < 64 ? nb - t : 64;
      const uint32_t y = lane < cn ? g.deg(0, rb[t + lane]) : 0;
      sum += na <= 64 ? min_pairs<1, T>(a, y, cn) : na <= 128 ? min_pairs<2, T>(a, y, cn)
             : na <= 256 ? min_pairs<4, T>(a, y, cn) : min_pairs<8, T>(a, y, cn);
    }
  }
  return sum;
}

template <typename T>
__global__ void __launch_bounds__(kBlock) k_hub_min_rows(HubGraph g, int first, uint32_t* __restrict__ big,
                                                         unsigned int* __restrict__ nbig,
                                                         unsigned long long* __restrict__ acc) {
  const uint64_t sum = block_sum<kBlock>(min_rows<T>(g, first, (uint64_t)blockIdx.x * (kBlock / 64) + wave_id(),
                                                     (uint64_t)gridDim.x * (kBlock / 64), big, nbig));
  if (threadIdx.x == 0 && sum) atomicAdd(acc, (unsigned long long)sum);
}

__global__ void __launch_bounds__(kBlock) k_hub_min_big(HubGraph g, int first, const uint32_t* __restrict__ big,
                                                        const unsigned int* __restrict__ nbig,
                                                        unsigned int* __restrict__ claim,
                                                        uint32_t* __restrict__ over_all, uint64_t over_cap,
                                                        unsigned long long* __restrict__ acc) {
  constexpr uint32_t kPer = kMinBins / kBlock;
  __shared__ uint32_t H[2][kMinBins + 1];  // bin t: values capped to t
  __shared__ unsigned int next, nover[2];
  const uint32_t tid = threadIdx.x;
  uint32_t* over[2] = {over_all + (uint64_t)blockIdx.x * 2 * over_cap,
                       over_all + (uint64_t)blockIdx.x * 2 * over_cap + over_cap};
  uint64_t sum = 0;
  const unsigned int total = *nbig;
  for (;;) {
    __syncthreads();
    if (tid == 0) {
      next = atomicAdd(claim, 1u);
      nover[0] = nover[1] = 0;
    }
    for (uint32_t i = tid; i < 2 * (kMinBins + 1); i += kBlock) (&H[0][0])[i] = 0;
    __syncthreads();
    if (next >= total) break;
    const uint32_t c = big[next];
    for (int s = 0; s < 2; ++s) {
      const int dir = s ? 0 : first;
      const uint32_t* r = g.row(dir, c);
      const uint32_t n = g.deg(dir, c);
      for (uint32_t i = tid; i < n; i += kBlock) {
        const uint32_t x = g.deg(dir, r[i]);
        atomicAdd(&H[s][x < kMinBins ? x : kMinBins], 1u);
        if (x > kMinBins) over[s][atomicAdd(&nover[s], 1u)] = x - kMinBins;
      }
    }
    __threadfence_block();
    __syncthreads();
    // suffix counts over bins 1..kMinBins: thread tid holds bins
    // kMinBins - kPer * tid - i, i < kPer, so a running sum goes downwards
    uint32_t run[2];
    for (int s = 0; s < 2; ++s) {
      uint32_t t = 0;
      for (uint32_t i = 0; i < kPer; ++i) t += H[s][kMinBins - kPer * tid - i];
      uint32_t all = 0;
      run[s] = block_excl_scan<kBlock>(t, all);
    }
    for (uint32_t i = 0; i < kPer; ++i) {
      const uint32_t t = kMinBins - kPer * tid - i;
      run[0] += H[0][t];
      run[1] += H[1][t];
      sum += (uint64_t)run[0] * run[1];
    }
    const uint32_t n0 = nover[0], n1 = nover[1];
    for (uint32_t i = tid; i < n0; i += kBlock) {
      const uint32_t x = over[0][i];
      for (uint32_t j = 0; j < n1; ++j) {
        const uint32_t y = over[1][j];
        sum += x < y ? x : y;
      }
    }
  }
  sum = block_sum<kBlock>(sum);
  if (tid == 0 && sum) atomicAdd(acc, (unsigned long long)sum);
}

// ---------------------------------------------------------------- small graphs
// At most kTpDirect vertices, of degree at most kTpDirectDeg: a workgroup per
// a0 counts the ends of its 2-paths in an LDS counter per vertex, on the graph
// as it is.  Diamond: the sum of squares.  4-cycle: the backward 2-paths a2 ->
// a3 -> a0 add up the counters they end at.  The renaming's sorts take about
// 0.3 ms whatever the size, which small graphs do not get back (measured,
// renamed -> direct: 16,000 vertices, 256,000 edges, uniform, diamond 526 ->
// 115 us, 4-cycle 417 -> 126 us; R-MAT-13 595 -> 204, 468 -> 359 us); but a hub's
// 2-paths are one workgroup's (R-MAT-14, degrees to 2,440: 662 -> 502, 512 ->
// 938 us), so graphs with hubs are renamed.
constexpr uint32_t kTpDirect = 16384, kTpDirectDeg = 2048;
constexpr int kTpDirectNT = 1024;

// f(x) for the entries of the rows (direction dir) of list[0, d), 16 lanes a row
template <class F>
__device__ __forceinline__ void walk_rows16(const HubGraph& g, int dir, const uint32_t* __restrict__ list, uint32_t d,
                                            F f) {
  const uint32_t sub = threadIdx.x & 15;
  for (uint32_t i = threadIdx.x / 16; i < d; i += kTpDirectNT / 16) {
    const uint32_t u = list[i], n = g.deg(dir, u);
    const uint32_t* r = g.row(dir, u);
    for (uint32_t t = sub; t < n; t += 16) f(r[t]);
  }
}

template <bool CYCLE>
__global__ void __launch_bounds__(kTpDirectNT) k_tp_direct(HubGraph g, uint32_t* __restrict__ big,
                                                           unsigned int* __restrict__ nbig,
                                                           unsigned long long* __restrict__ acc) {
  __shared__ uint32_t cnt[kTpDirect];
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = tid; i < g.n; i += kTpDirectNT) cnt[i] = 0;
  uint64_t sum = 0, paths = 0;
  for (uint32_t a0 = blockIdx.x; a0 < g.n; a0 += gridDim.x) {
    const uint32_t out = g.deg(0, a0), in = g.deg(1, a0);
    if (!out) continue;
    if (tid == 0) paths += (uint64_t)out * (CYCLE ? in : out);
    if (CYCLE && !in) continue;
    __syncthreads();
    walk_rows16(g, 0, g.row(0, a0), out, [&](uint32_t x) { atomicAdd(&cnt[x], 1u); });
    __syncthreads();
    if (CYCLE) {
      walk_rows16(g, 1, g.row(1, a0), in, [&](uint32_t x) { sum += cnt[x]; });
      __syncthreads();
    }
    for (uint32_t i = tid; i < g.n; i += kTpDirectNT) {
      const uint64_t k = cnt[i];
      if (!CYCLE) sum += k * k;
      cnt[i] = 0;
    }
  }
  const uint64_t mins = min_rows<uint32_t>(g, CYCLE ? 1 : 0, (uint64_t)blockIdx.x * (kTpDirectNT / 64) + wave_id(),
                                           (uint64_t)gridDim.x * (kTpDirectNT / 64), big, nbig);
  const uint64_t t[3] = {sum, paths, mins};
  const int at[3] = {kTpAB, kTpPaths, kTpMin};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const uint64_t v = block_sum<kTpDirectNT>(t[i]);
    if (tid == 0 && v) atomicAdd(acc + at[i], (unsigned long long)v);
  }
}

// ---------------------------------------------------------------- host
// Large graphs without hubs have many w of hundreds of thousands of ids below
// them and a few thousand entries each: a step of k_hub_dense is 4.2 us of one
// of 256 CUs however few of them it counts.  The dense counters of clique.hip
// take a 2-path in 0.11 ns and an id in 70, or for the 4-cycle, which walks
// them twice, 200; so they count where the steps, in 2-paths, are more.
// Uniform graphs, diamond, here / dense counters: 1.0e6 vertices of 48 edges
// 541 / 311 ms, 2.1e6 of 64 2,206 / 959, 4.2e6 of 32 2,401 / 781; 1.0e6 of 96
// 781 / 1,002; 4-cycle: 2.1e6 of 64 1,072 / 1,688, 4.2e6 of 32 1,095 / 1,869.
// Up to kTpFewIds there are two steps to a w at most, and nobody asks.
constexpr uint64_t kTpStep = 145, kTpId = 640, kTpIdCycle = 1800;
constexpr uint32_t kTpFewIds = 65536;

// force: whatever the dense counters would take; else false, and nothing
// counted, where they are the sooner
static bool count_2path(gj_ctx* c, const Version& v, uint32_t n, bool cycle, bool force, KernelTimer& timer,
                        uint64_t out[3]) {
  for (int i = 0; i < 3; ++i) out[i] = 0;
  if (!v.m) return true;
  // control words: the accumulators, the lists' lengths per pass and class,
  // then the long rows of the stage-3 counter and their claim counter
  constexpr int kLists = 2 * kTpClasses;
  unsigned long long* acc = (unsigned long long*)ws_get(c, "tp_ctl", kTpAcc * 8 + (kLists + 2) * 4);
  unsigned int* len = (unsigned int*)(acc + kTpAcc);
  unsigned int* nbig = len + kLists;
  uint32_t* big = (uint32_t*)ws_get(c, "tp_big", (uint64_t)n * sizeof(uint32_t));
  const unsigned cus = (unsigned)c->num_cus;
  const int first = cycle ? 1 : 0;
  const uint64_t over = std::min<uint64_t>(std::max(v.max_deg[0], v.max_deg[first]), v.m / kMinBins + 1);
  uint32_t* overs = (uint32_t*)ws_get(c, "tp_over", (uint64_t)cus * 4 * 2 * over * sizeof(uint32_t));
  GJ_HIP(hipMemsetAsync(acc, 0, kTpAcc * 8 + (kLists + 2) * 4, c->stream));
  const bool long_rows = std::max(v.max_deg[0], v.max_deg[1]) > kMinRow;
  unsigned long long h[kTpAcc];
  if (n <= kTpDirect && std::max(v.max_deg[0], v.max_deg[1]) <= kTpDirectDeg) {
    const HubGraph g{{v.d[0].rp, v.d[1].rp}, {}, {}, {}, {v.d[0].col, v.d[1].col}, nullptr, n};
    const unsigned grid = std::min<unsigned>(n, cus * 2);
    timer.start();
    if (cycle)
      k_tp_direct<true><<<grid, kTpDirectNT, 0, c->stream>>>(g, big, nbig, acc);
    else
      k_tp_direct<false><<<grid, kTpDirectNT, 0, c->stream>>>(g, big, nbig, acc);
    if (long_rows)
      k_hub_min_big<<<cus * 4, kBlock, 0, c->stream>>>(g, first, big, nbig, nbig + 1, overs, over, acc + kTpMin);
    timer.stop();
    GJ_HIP(hipGetLastError());
    read_bytes(c, h, acc, sizeof(h));
    out[0] = h[kTpAB];
    out[1] = h[kTpPaths];
    out[2] = h[kTpMin];
    return true;
  }
  const uint32_t* row = nullptr;
  HubGraph g;
  hub_graph(c, v, n, v.ranked() ? HubOrder::kReversed : HubOrder::kDegree, false, g, row);
  hub_above(c, g);
  const int passes = cycle ? 1 : 2;
  uint32_t* lists = (uint32_t*)ws_get(c, "tp_lists", (uint64_t)passes * kTpClasses * n * sizeof(uint32_t));
  uint32_t* rec = (uint32_t*)ws_get(c, "tp_rec", 2 * (uint64_t)n * sizeof(uint32_t));
  GJ_HIP(hipMemsetAsync(rec, 0, 2 * (uint64_t)n * sizeof(uint32_t), c->stream));
  timer.start();
  const unsigned gn = grid_for(n, kBlock, cus * 8);
  k_hub_recip<<<grid_for(v.m, kBlock, cus * 32), kBlock, 0, c->stream>>>(g, row, v.m, rec, rec + n);
  k_hub_terms<<<gn, kBlock, 0, c->stream>>>(g, rec, rec + n, cycle ? 1 : 0, acc);
  k_hub_classes<<<grid_for(n, 64, cus * 16), kBlock, 0, c->stream>>>(g, cycle ? 1 : 0, len, lists, n, acc);
  const bool ask = n > kTpFewIds && !force;
  HostEvent asked;
  unsigned long long* now = (unsigned long long*)c->pinned;
  if (ask) {  // the stage-3 counter's kernels run while the host waits
    GJ_HIP(hipMemcpyAsync(now, acc + kTpWalk, 2 * sizeof(*now), hipMemcpyDeviceToHost, c->stream));
    asked.record(c->stream);
  }
  if (std::max(v.max_deg[0], v.max_deg[1]) < (1u << 22))
    k_hub_min_rows<uint32_t><<<cus * 8, kBlock, 0, c->stream>>>(g, first, big, nbig, acc + kTpMin);
  else
    k_hub_min_rows<uint64_t><<<cus * 8, kBlock, 0, c->stream>>>(g, first, big, nbig, acc + kTpMin);
  if (long_rows)
    k_hub_min_big<<<cus * 4, kBlock, 0, c->stream>>>(g, first, big, nbig, nbig + 1, overs, over, acc + kTpMin);
  if (ask) {
    asked.wait();
    if ((cycle ? 2 * now[0] + kTpIdCycle * n : now[0] + kTpId * n) < kTpStep * now[1]) {
      timer.stop();
      return false;
    }
  }
  for (int p = 0; p < passes; ++p) {
    const int op = cycle || p ? 1 : 0;
    unsigned long long* a = acc + (p ? kTpOI : kTpAB);
    const uint32_t* l = lists + (uint64_t)p * kTpClasses * n;
    const unsigned int* ln = len + p * kTpClasses;
    k_hub_dense<32, kTpSeg4><<<cus, 1024, 0, c->stream>>>(g, p, op, l + 4ull * n, ln + 4, a);
    k_hub_dense<16, kTpSeg3><<<cus, 1024, 0, c->stream>>>(g, p, op, l + 3ull * n, ln + 3, a);
    k_hub_small<true><<<cus * 4, kBlock, 0, c->stream>>>(g, p, op, l + 2ull * n, ln + 2, a);
    k_hub_small<false><<<cus * 4, kBlock, 0, c->stream>>>(g, p, op, l + 1ull * n, ln + 1, a);
    k_hub_wave<<<cus * 4, kBlock, 0, c->stream>>>(g, p, op, l, ln, a);
  }
  timer.stop();
  GJ_HIP(hipGetLastError());
  read_bytes(c, h, acc, sizeof(h));
  out[0] = cycle ? 4 * h[kTpAB] + 2 * h[kTpRecUp2] : h[kTpAB] + 2 * (h[kTpOI] - h[kTpBoth]) + h[kTpRec2] + h[kTpMid];
  out[1] = h[kTpPaths];
  out[2] = h[kTpMin];
  return true;
}

bool diamond2p_count(gj_ctx* c, const Version& v, uint32_t n, bool force, KernelTimer& timer, uint64_t out[3]) {
  return count_2path(c, v, n, false, force, timer, out);
}

bool cycle4_2p_count(gj_ctx* c, const Version& v, uint32_t n, bool force, KernelTimer& timer, uint64_t out[3]) {
  return count_2path(c, v, n, true, force, timer, out);
}

}  // namespace gj
