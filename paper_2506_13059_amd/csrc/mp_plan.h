// Sizes that the value pass's launch is planned with: plain host functions of the call's sizes, so that they can be checked
// without a GPU.
#pragma once

#include <algorithm>

namespace mp {

// Upper bound of the keys a decode call selects per unit: the selected clusters fit the key budget, and with two levels
// they are children of the promising clusters, which fit the coarse budget.  (The launch is cut by this bound: by the key
// budget alone, a coarse budget of an eighth of it left seven of eight workgroups without rows -- 128 units, budgets
// 32768 / 4096, 4 heads, whole step 153 us, now 66; 64 units 95, now 43.)
inline int most_selected(int levels, int key_budget, int coarse_budget, int n_tokens)
{
    const int most = std::min(key_budget, n_tokens);
    return levels == 2 ? std::min(most, coarse_budget) : most;
}

}  // namespace mp
