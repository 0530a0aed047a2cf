// The renaming by descending degree (hub.h).
#include <algorithm>

#include "gj_internal.h"
#include "hub.h"
#include "prim.h"

namespace gj {

__global__ void k_hub_keys(const uint32_t* __restrict__ rp0, const uint32_t* __restrict__ rp1, uint32_t n,
                           uint32_t top, uint64_t* __restrict__ keys) {
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += gs) {
    const uint32_t d = (rp0[v + 1] - rp0[v]) + (rp1[v + 1] - rp1[v]);  // at most top
    keys[v] = ((uint64_t)(top - d) << 32) | v;
  }
}

// new id = position in descending degree order; degrees in the new order;
// lim[0]: the vertices of more than cap edges
__global__ void k_hub_ids(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ rp0,
                          const uint32_t* __restrict__ rp1, uint32_t n, uint32_t* __restrict__ new_of_old,
                          uint32_t* __restrict__ d0, uint32_t* __restrict__ d1, uint64_t cap,
                          unsigned int* __restrict__ lim) {
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gs) {
    const uint32_t o = (uint32_t)keys[i];
    new_of_old[o] = (uint32_t)i;
    const uint32_t a = rp0[o + 1] - rp0[o], b = rp1[o + 1] - rp1[o];
    d0[i] = a;
    d1[i] = b;
    if (lim && (uint64_t)a + b > cap) {  // the last of these says how many they are
      const uint32_t next = i + 1 < n ? (uint32_t)keys[i + 1] : 0;
      if (i + 1 == n || (uint64_t)(rp0[next + 1] - rp0[next]) + (rp1[next + 1] - rp1[next]) <= cap)
        lim[0] = (unsigned int)i + 1;
    }
  }
}

// LIMIT: below[v], for v in (cap, lim[0]), counts the edges between v and
// vertices below it (the others have no more than cap of either); a row's own
// by one atomic per wave, rows being sorted.
template <bool LIMIT>
__global__ void __launch_bounds__(kBlock) k_hub_edges(const uint32_t* __restrict__ row,
                                                      const uint32_t* __restrict__ col, uint64_t m,
                                                      const uint32_t* __restrict__ new_of_old,
                                                      uint64_t* __restrict__ keys,
                                                      uint32_t cap, const unsigned int* __restrict__ lim,
                                                      uint32_t* __restrict__ below) {
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  const uint32_t big = LIMIT ? lim[0] : 0;
  for (uint64_t b = (uint64_t)blockIdx.x * blockDim.x; b < m; b += gs) {  // whole waves take every step
    const uint64_t i = b + threadIdx.x;
    uint32_t u = ~0u, v = ~0u;
    if (i < m) {
      u = new_of_old[row[i]];
      v = new_of_old[col[i]];
      keys[i] = ((uint64_t)u << 32) | v;
    }
    if (LIMIT) {
      if (v < big && v > cap && u < v) atomicAdd(below + v, 1u);
      const bool mine = u < big && u > cap && v < u;
      for (uint64_t left = __ballot(mine); left;) {
        const int first = __ffsll((unsigned long long)left) - 1;
        const uint32_t fu = __shfl(u, first, 64);
        const uint64_t same = __ballot(mine && u == fu);
        if (lane_id() == first) atomicAdd(below + fu, (uint32_t)__popcll(same));
        left &= ~same;
      }
    }
  }
}

// lim[1]: the vertices with more than cap different neighbours below them.
// One that is a neighbour both ways was counted twice, so a workgroup looks
// those of v's row up in the other, where that can make the difference.
__global__ void __launch_bounds__(kBlock) k_hub_limit(const uint64_t* __restrict__ keys,
                                                      const uint32_t* __restrict__ rp0,
                                                      const uint32_t* __restrict__ col0,
                                                      const uint32_t* __restrict__ rp1,
                                                      const uint32_t* __restrict__ col1,
                                                      const uint32_t* __restrict__ new_of_old,
                                                      const uint32_t* __restrict__ below, uint32_t cap,
                                                      unsigned int* __restrict__ lim) {
  const uint32_t big = lim[0];
  for (uint32_t v = cap + 1 + blockIdx.x; v < big; v += gridDim.x) {
    const uint32_t b = below[v];
    if (b <= cap) continue;
    uint64_t both = 0;
    if (b <= 2 * cap) {
      const uint32_t o = (uint32_t)keys[v], lo = rp1[o], hi = rp1[o + 1];
      for (uint64_t i = (uint64_t)rp0[o] + threadIdx.x; i < rp0[o + 1]; i += kBlock) {
        const uint32_t x = col0[i];
        if (new_of_old[x] < v && contains_u32(col1, lo, hi, x)) ++both;
      }
      both = block_sum<kBlock>(both);
    }
    if (threadIdx.x == 0 && b - both > cap) atomicAdd(lim + 1, 1u);
  }
}

// rows and columns of the sorted keys, and the swapped keys for the other
// direction (null: none)
__global__ void k_hub_split(const uint64_t* __restrict__ keys, uint64_t m, uint32_t* __restrict__ row,
                            uint32_t* __restrict__ col, uint64_t* __restrict__ swapped) {
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gs) {
    const uint64_t k = keys[i];
    row[i] = (uint32_t)(k >> 32);
    col[i] = (uint32_t)k;
    if (swapped) swapped[i] = (k << 32) | (k >> 32);
  }
}

// The same graph with id v renamed to n - 1 - v: every array backwards.
__global__ void k_hub_reverse(const uint32_t* __restrict__ rp, const uint32_t* __restrict__ row,
                              const uint32_t* __restrict__ col, uint64_t m, uint32_t n, uint32_t* __restrict__ orp,
                              uint32_t* __restrict__ orow, uint32_t* __restrict__ ocol) {
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x, t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (uint64_t i = t; i < m; i += gs) {
    orow[m - 1 - i] = n - 1 - row[i];
    ocol[m - 1 - i] = n - 1 - col[i];
  }
  for (uint64_t v = t; v <= n; v += gs) orp[v] = (uint32_t)m - rp[n - v];
}

// end of every row's prefix, and its quads; both directions
__global__ void k_hub_prefix(HubGraph g, uint32_t* __restrict__ end, uint32_t* __restrict__ quads) {
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 2ull * g.n; i += gs) {
    const int s = i >= g.n;
    const uint32_t u = (uint32_t)(s ? i - g.n : i);
    const uint32_t b = g.rp[s][u], e = lower_bound_u32(g.col[s], b, g.rp[s][(uint64_t)u + 1], u);
    end[i] = e;
    quads[i] = (e - b + 3) / 4;
  }
}

// The prefixes' entries into their quads, the last one of a prefix padding its
// quad; both directions.
__global__ void k_hub_quads(HubGraph g, const uint32_t* __restrict__ row0, const uint32_t* __restrict__ row1,
                            uint64_t m, uint32_t* __restrict__ pre) {
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  for (int s = 0; s < 2; ++s)
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gs) {
      const uint32_t x = (s ? row1 : row0)[i], y = g.col[s][i];
      if (y >= x) continue;
      uint64_t at = (uint64_t)g.pq[s][x] * 4 + (i - g.rp[s][x]);
      pre[at] = y;
      if (i + 1 == g.end[s][x])
        while (++at & 3) pre[at] = ~0u;
    }
}

// first quad with an id of kTpHubs or above; both directions
__global__ void k_hub_above(HubGraph g, uint32_t* __restrict__ mq) {
  const uint64_t gs = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 2ull * g.n; i += gs) {
    const uint64_t u = i >= g.n ? i - g.n : i;
    uint32_t lo = g.pq[0][i], len = g.pq[0][i + 1] - lo;  // the directions' arrays follow each other
    if (u <= kTpHubs) {
      lo += len;
    } else {
      const uint32_t e = lo + len;
      while (len > 0) {
        const uint32_t half = len >> 1;
        if (g.pre[(uint64_t)lo + half].w < kTpHubs) {
          lo += half + 1;
          len -= half + 1;
        } else {
          len = half;
        }
      }
      if (lo < e) {  // the last quad may hold padding only beyond its ids below
        const uint4 t = g.pre[lo];
        const auto above = [](uint32_t x) { return x >= kTpHubs && x != ~0u; };
        if (!(above(t.x) || above(t.y) || above(t.z) || above(t.w))) lo = e;
      }
    }
    mq[i] = lo;
  }
}

void hub_above(gj_ctx* c, HubGraph& g) {
  uint32_t* mq = (uint32_t*)ws_get(c, "tp_mq", 2 * (uint64_t)g.n * sizeof(uint32_t));
  k_hub_above<<<grid_for(2ull * g.n, kBlock, 1u << 14), kBlock, 0, c->stream>>>(g, mq);
  GJ_HIP(hipGetLastError());
  g.mq[0] = mq;
  g.mq[1] = mq + g.n;
}

bool hub_graph(gj_ctx* c, const Version& v, uint32_t n, HubOrder order, bool limit, HubGraph& g,
               const uint32_t*& row) {
  const uint64_t m = v.m;
  g = HubGraph{};
  g.n = n;
  const unsigned gn = grid_for(n, kBlock, 1u << 14), ge = grid_for(m, kBlock * 4, 1u << 14);
  auto words = [&](const std::string& name, uint64_t count) {
    return (uint32_t*)ws_get(c, "tp_" + name, count * sizeof(uint32_t));
  };
  const uint32_t* rows[2];
  if (order == HubOrder::kAsIs) {
    for (int s = 0; s < 2; ++s) {
      g.rp[s] = v.d[s].rp;
      g.col[s] = v.d[s].col;
      rows[s] = v.d[s].row;
    }
  } else {
    uint32_t *rp[2], *orow[2], *ocol[2];
    auto copies = [&] {
      for (int s = 0; s < 2; ++s) {
        const std::string z = s ? "1" : "0";
        g.rp[s] = rp[s] = words("rp" + z, (uint64_t)n + 1);
        g.col[s] = ocol[s] = words("col" + z, m + 1);
        rows[s] = orow[s] = words("row" + z, m + 1);
      }
    };
    if (order == HubOrder::kReversed) {
      copies();
      for (int s = 0; s < 2; ++s)
        k_hub_reverse<<<ge, kBlock, 0, c->stream>>>(v.d[s].rp, v.d[s].row, v.d[s].col, m, n, rp[s], orow[s], ocol[s]);
    } else {
      uint64_t* vk = (uint64_t*)ws_get(c, "tp_vk", (uint64_t)n * sizeof(uint64_t));
      uint64_t* vk2 = (uint64_t*)ws_get(c, "tp_vk2", (uint64_t)n * sizeof(uint64_t));
      uint64_t* keys = (uint64_t*)ws_get(c, "tp_keys", (m + 1) * sizeof(uint64_t));
      uint64_t* alt = (uint64_t*)ws_get(c, "tp_alt", (m + 1) * sizeof(uint64_t));
      uint32_t* ids = words("ids", n);
      uint32_t* deg = words("deg", 2 * (uint64_t)n);
      const uint32_t top = v.max_deg[0] + v.max_deg[1];
      k_hub_keys<<<gn, kBlock, 0, c->stream>>>(v.d[0].rp, v.d[1].rp, n, top, vk);
      const uint64_t* vs = sort_u64(c, vk, vk2, n, 0, bits_for(top + 1));  // stable: equal degrees by id
      constexpr uint32_t cap = kBigDegree;
      limit = limit && hub_limit_open(v);
      unsigned int* lim = nullptr;
      if (limit) {
        const uint64_t most = std::min<uint64_t>(n, 2 * m / cap);  // vertices of more than cap edges
        lim = words("lim", 2 + most);
        GJ_HIP(hipMemsetAsync(lim, 0, (2 + most) * sizeof(uint32_t), c->stream));
      }
      k_hub_ids<<<gn, kBlock, 0, c->stream>>>(vs, v.d[0].rp, v.d[1].rp, n, ids, deg, deg + n, cap, lim);
      if (limit) {
        k_hub_edges<true><<<ge, kBlock, 0, c->stream>>>(v.d[0].row, v.d[0].col, m, ids, keys, cap, lim, lim + 2);
        k_hub_limit<<<c->num_cus * 8, kBlock, 0, c->stream>>>(vs, v.d[0].rp, v.d[0].col, v.d[1].rp, v.d[1].col, ids,
                                                              lim + 2, cap, lim);
        GJ_HIP(hipGetLastError());
        unsigned int beyond = 0;
        read_bytes(c, &beyond, lim + 1, sizeof(beyond));
        if (beyond) return false;
      } else {
        k_hub_edges<false><<<ge, kBlock, 0, c->stream>>>(v.d[0].row, v.d[0].col, m, ids, keys, 0, nullptr, nullptr);
      }
      copies();
      const int bits = bits_for(n);
      for (int s = 0; s < 2; ++s) {
        scan_u32(c, deg + (uint64_t)s * n, rp[s], n);
        // the reverse keys come out of the forward order, already ascending in
        // their low half: a stable sort by the high half finishes them
        uint64_t* sorted = sort_u64(c, keys, alt, m, s ? 0 : bits, bits);
        uint64_t* other = sorted == keys ? alt : keys;
        k_hub_split<<<ge, kBlock, 0, c->stream>>>(sorted, m, orow[s], ocol[s], s ? nullptr : other);
        keys = other;
        alt = sorted;
      }
    }
  }
  // every edge is in one prefix, of at most 2 min(n, m) that are not empty
  const uint64_t quads = (m + 6 * std::min<uint64_t>(n, m)) / 4 + 2;
  uint4* pre = (uint4*)ws_get(c, "tp_pre", quads * sizeof(uint4));
  uint32_t* qn = words("qn", 2 * (uint64_t)n);
  uint32_t* end = words("end", 2 * (uint64_t)n);
  uint32_t* pq = words("pq", 2 * (uint64_t)n + 1);
  g.pre = pre;
  k_hub_prefix<<<grid_for(2ull * n, kBlock, 1u << 14), kBlock, 0, c->stream>>>(g, end, qn);
  scan_u32(c, qn, pq, 2 * (uint64_t)n);
  for (int s = 0; s < 2; ++s) {
    g.end[s] = end + (uint64_t)s * n;
    g.pq[s] = pq + (uint64_t)s * n;
  }
  k_hub_quads<<<ge, kBlock, 0, c->stream>>>(g, rows[0], rows[1], m, (uint32_t*)pre);
  GJ_HIP(hipGetLastError());
  row = rows[0];
  return true;
}

}  // namespace gj
