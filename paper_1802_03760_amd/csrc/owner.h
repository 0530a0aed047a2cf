// Owner-grouped first-stage intersection (see owner.hip).
#pragma once

#include "gj_internal.h"

namespace gj {

// Seed edges (x0, x1); LA = extension set of the atom on x0, LB = of the atom
// on x1; S0 = seed index (partners x1 of x0), S1 = its transpose (partners x0
// of x1).  Each pair (rp, adj) is a CSR row-pointer and column array.
struct OwnerArgs {
  const uint32_t *rpA, *adjA;
  const uint32_t *rpB, *adjB;
  const uint32_t *rpS0, *adjS0;
  const uint32_t *rpS1, *adjS1;
  uint32_t n;
  // optional signs of the seed edges (null: all +1), in S0 order (seed-index
  // order, as seed_row/seed_col) and in S1 order (transposed order)
  const int8_t* sg0 = nullptr;
  const int8_t* sg1 = nullptr;
};

// matches = sum over all seed edges of |LA(x0) ∩ LB(x1)|;
// extensions = sum of min(|LA(x0)|, |LB(x1)|); wsum = the same sum as
// matches with each edge's term times its sign.  seed_row/seed_col: the E
// seed edges as (x0, x1) in seed-index order; t_row/t_col: the same edges in
// transposed-index order as (x1, x0).
// plan (with gen, the version's generation, and pc, the context that owns
// the graph's memory): a static count's plan kept with the version, reused
// while valid, else built and stored there; null: planned for this call only.
void owner_count(gj_ctx* c, const OwnerArgs& a, const uint32_t* seed_row, const uint32_t* seed_col,
                 const uint32_t* t_row, const uint32_t* t_col, uint64_t E, KernelTimer& timer, uint64_t& matches,
                 uint64_t& extensions, int64_t* wsum = nullptr, OwnerPlan* plan = nullptr, uint64_t gen = 0,
                 gj_ctx* pc = nullptr);

// Listing: a bit per value of every seed edge's proposing set.
struct OwnerMask {
  unsigned long long* mask = nullptr;
  const uint32_t* woff = nullptr;     // E + 1: an edge's first word
  const uint32_t* seed_of = nullptr;  // E: transposed entry -> seed edge
};
constexpr uint64_t kOwnerMaskMax = 4ull << 30;  // bytes of mask

// The pairs of owner_count's sets, for listing: marks every match, counts and
// numbers the rows of every seed edge, in workspace (`words` of mask); matches
// and extensions as owner_count (its plan, too).  False, and nothing marked,
// when extensions are below `least` or the mask would take more than
// most_words.  Until the context's next
// owner_mask, owner_mask_counts are the matches per seed edge, and owner_rows
// writes the `matches` rows in seed and value order, with their columns placed
// by map.
bool owner_mask(gj_ctx* c, const OwnerArgs& a, const uint32_t* seed_row, const uint32_t* seed_col,
                const uint32_t* t_row, const uint32_t* t_col, uint64_t E, uint64_t least,
                uint64_t most_words, KernelTimer& timer, OwnerPlan* plan, uint64_t gen, gj_ctx* pc,
                uint64_t& words, uint64_t& matches, uint64_t& extensions);
void owner_rows(gj_ctx* c, const OwnerArgs& a, const uint32_t* seed_row, const uint32_t* seed_col, uint64_t E,
                uint64_t words, const RowMap& map, uint32_t* rows);
const uint32_t* owner_mask_counts(gj_ctx* c);
// acc[0] += cnt[position of edge x[p] -> y[p]] over the n prefixes p (every
// pair is an edge of the forward index rp, col)
void owner_pair_sum(gj_ctx* c, const uint32_t* x, const uint32_t* y, uint64_t n, const uint32_t* rp,
                    const uint32_t* col, const uint32_t* cnt, unsigned long long* acc);

}  // namespace gj
