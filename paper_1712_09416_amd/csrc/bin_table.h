// Where a pad row's bin offsets stand in the slot's table.  Plain C++, so that
// the arithmetic can be checked at its limits without a GPU.
#pragma once

#include <cstdint>

namespace tpc {

constexpr int kBinsPerHit = 2;            // a row has at most this many bins per hit

// A row of n hits has at most kBinsPerHit * max(n, 1) bins and one end entry:
// 2 n + 4 entries hold them.  Row sr (of all the slot's rows), `first` hits
// before it, starts where the rows before it would end if all were as long as
// they can be, at an even entry: the place is counted in pairs of entries,
// which 32 bits hold for every slot (2^31 - 1 clusters, 4096 events of 5724
// rows); the entry itself is past 2^32 there.
constexpr uint32_t bin_table_pair(uint32_t first, uint32_t sr) { return first + 2u * sr; }
constexpr int64_t bin_table_entries(int64_t clusters, int64_t rows) { return 2 * (clusters + 2 * rows); }

static_assert(bin_table_entries(0x7FFFFFFFll, 4096ll * 36 * 159) / 2 <= 0xFFFFFFFFll,
              "the largest slot's table");

}  // namespace tpc
