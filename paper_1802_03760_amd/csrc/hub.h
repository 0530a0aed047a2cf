// A graph renamed so that small ids are hubs, for the whole counts that
// attribute a match to its least or greatest vertex (twopath.hip,
// cliquebits.hip), and the walk over prefixes of its rows.
#pragma once

#include "gj_internal.h"
#include "prim.h"

namespace gj {

// The renamed graph: per direction (0 out-, 1 in-neighbours) rows sorted by
// new id, row u at col[rp[u] .. rp[u + 1]); end[u] closes the prefix of ids
// below u.  The prefixes are stored again on their own, in quads of four
// entries padded with ~0: direction s's of u at quads [pq[s][u], pq[s][u + 1])
// of pre, so that a walk loads 16 aligned bytes a lane and an entry's value
// alone says whether it counts.  mq[s][u] (hub_above): the first of those quads
// with an id of kTpHubs or above.
struct HubGraph {
  const uint32_t* rp[2];
  const uint32_t* end[2];
  const uint32_t* pq[2];
  const uint32_t* mq[2];
  const uint32_t* col[2];
  const uint4* pre;
  uint32_t n;
  __device__ __forceinline__ uint32_t deg(int s, uint64_t v) const { return rp[s][v + 1] - rp[s][v]; }
  __device__ __forceinline__ const uint32_t* row(int s, uint64_t v) const { return col[s] + rp[s][v]; }
};

constexpr uint32_t kTpHubs = 16384;  // ids below it: 8-bit counter pairs for all of them take 32 KiB

// How a version's ids become hub-first: sorted by degree; reversed, where they
// ascend by degree (Version::ranked(); the order decides work, never results); or
// left as they are, for graphs whose sorts would cost more than the order
// saves.
enum class HubOrder { kDegree, kReversed, kAsIs };

// May some vertex have more than kBigDegree different neighbours below it, by
// degree?  It and they have more than kBigDegree edges each, so a graph with
// one has more such vertices than that, and 559,153 edges or more.
inline bool hub_limit_open(const Version& v) {
  return v.big > kBigDegree && (uint64_t)v.max_deg[0] + v.max_deg[1] > kBigDegree &&
         v.m >= (kBigDegree + 1ull) * (kBigDegree + 2) / 2;
}

// hub.hip: version v (m > 0, fewer than 2^31 edges) under `order`, in
// workspace of the context; row receives the row of every out-entry.  limit,
// looked at when sorting by degree only: false, before the edges are sorted,
// where some vertex has more than kBigDegree different neighbours below it.
bool hub_graph(gj_ctx* c, const Version& v, uint32_t n, HubOrder order, bool limit, HubGraph& g,
               const uint32_t*& row);
void hub_above(gj_ctx* c, HubGraph& g);  // fills g.mq

__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

// Sixteen lanes to a row, a quad to a lane, so a wave walks four rows side by
// side and a group that finishes one takes the batch's next; DEPTH loads are
// in flight.  Row i < cn is lane i's: rlen & (2^LB - 1) quads from pre[rp] on,
// with rlen >> LB as its tag.  Calls add(x, tag) for every entry and for
// fillers (~0), so that it can do without a branch per entry.  A row ends at its
// first quad beyond lim.  Issue-bound (about 60 instructions for 256 entries): addressing is
// per lane, since a row to a wave kept the scalar unit busy with row
// bookkeeping, and lengths are tested per quad, not per entry.
template <int DEPTH, int LB, class F>
__device__ __forceinline__ void walk_batch(const uint4* __restrict__ pre, uint32_t rp, uint32_t rlen, uint32_t cn, uint32_t lim,
                                           F add) {
  const uint32_t lane = lane_id(), sub = lane & 15;
  const uint64_t group = 0xFFFFull << (lane & 48), below = (1ull << (lane & 48)) - 1;
  if (!cn) return;
  uint32_t next = 4, row = lane >> 4;  // the batch's rows taken; this group's
  uint32_t p = 0, left = 0, tag = 0;  // left: quads of the row from p on; 0 once the batch has no more
  auto take = [&](bool mine) {  // all lanes
    const uint32_t a = __shfl(rp, row & 63, 64), l = __shfl(rlen, row & 63, 64);
    if (mine) {
      p = a + sub;
      left = row < cn ? l & ((1u << LB) - 1) : 0;
      tag = l >> LB;
    }
  };
  uint4 q[DEPTH];
  uint32_t qtag[DEPTH], qrow[DEPTH];
  uint64_t qlive[DEPTH];
  auto issue = [&](int d) {
    q[d] = make_uint4(~0u, ~0u, ~0u, ~0u);
    qlive[d] = __ballot(left != 0);
    qtag[d] = tag;
    qrow[d] = row;
    if (sub < left) q[d] = pre[p];
    // the group's next 64 entries, of the row or of another
    const bool more = left > 16;
    const uint64_t ask = qlive[d] & ~__ballot(more) & 0x0001000100010001ull;  // a bit per group
    if (ask) {
      const bool mine = left && !more;
      if (mine) row = next + (uint32_t)__popcll(ask & below);
      next += (uint32_t)__popcll(ask);
      if (more) left -= 16;
      p += 16;
      take(mine);
    } else {
      left -= more ? 16 : 0;
      p += 16;
    }
  };
  take(true);
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) issue(d);
  for (;;) {
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
      if (!qlive[d]) return;  // issued in order: none behind it either
      // the rest of a row whose quads reach lim lies beyond it: one more step ends it
      const uint64_t stop = __ballot(q[d].w >= lim);
      add(q[d].x, qtag[d]);
      add(q[d].y, qtag[d]);
      add(q[d].z, qtag[d]);
      add(q[d].w, qtag[d]);
      if ((stop & group) && row == qrow[d] && left > 1) left = 1;
      issue(d);
    }
  }
}

}  // namespace gj
