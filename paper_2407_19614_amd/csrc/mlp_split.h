// How the row sum of g_W2 = h1^T dz2 is split (host code without HIP types, so
// that it can be checked for every row count on a machine without a GPU).
#pragma once

#include <algorithm>
#include <cstdint>

namespace ri {

// Most splits: 16 tiles x 32 = two workgroups per CU.  The workspace holds this
// many partial products.
constexpr int GW2_SPLITS = 32;

struct Gw2Split {
    int64_t per;   // rows of each of a split's four waves: a multiple of 16, at least 64
    int splits;    // at most GW2_SPLITS
};

// rows is a multiple of 32.  The quotient is rounded up before it goes to a
// multiple of 16: rounded down, a remainder that fills no wave's share would
// become one split too many.
inline Gw2Split gw2_split(int64_t rows) {
    const int64_t waves = 4 * GW2_SPLITS, per = std::max<int64_t>(64, ((rows + waves - 1) / waves + 15) / 16 * 16);
    return {per, (int)((rows + 4 * per - 1) / (4 * per))};
}

}  // namespace ri
