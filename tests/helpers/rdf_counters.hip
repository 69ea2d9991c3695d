// The pair-count kernel's 32-bit counters: whatever the number of ions the
// library takes (1 to 2^24), the items between two flushes cannot carry an
// entry past 2^32, and at least one item is always taken.  Compiled, never run.
#include "../../paper_1602_05716_amd/csrc/mc_sweep_kernel.hpp"
#include "../../paper_1602_05716_amd/csrc/mc_aux_kernels.hpp"

constexpr bool safe(int n) {
    const int items = mcdev::rdf_items_per_flush(n);
    return items >= 1 && 64ull * (unsigned long long)n * (unsigned long long)items < (1ull << 32);
}
static_assert(safe(1) && safe(2000) && safe(131072) && safe(1 << 20) && safe((1 << 20) + 1));
static_assert(safe(12000000) && safe((1 << 24) - 1) && safe(1 << 24));
