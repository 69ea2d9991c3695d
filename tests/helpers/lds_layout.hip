// Alignment of the LDS fields that the kernels access in pieces wider than
// their element type, for every instantiation of the sweep kernels and for
// the training kernel.  Compiled, never run: each line is a static_assert.
#include <cstddef>

#include "../../paper_1602_05716_amd/csrc/mc_train.hip"
#include "../../paper_1602_05716_amd/csrc/mc_sweep_kernel.hpp"

#pragma clang diagnostic ignored "-Winvalid-offsetof"
#define ALIGNED(S, field, bytes) \
    static_assert(offsetof(S, field) % bytes == 0 && alignof(S) % bytes == 0, #S "::" #field)

template <typename T, int M, bool DA>
struct Sweep {
    using S = mcdev::SweepShared<T, M, DA>;
    // rows of corrections and their factors, 16 bytes at a time
    ALIGNED(S, c_own, 16);
    ALIGNED(S, c_b, 16);
    ALIGNED(S, fac, 16);
    static_assert(S::LC == 1 || offsetof(S, fac_h) % 16 == 0, "fac_h");
    static_assert(sizeof(T) * S::CS % 16 == 0, "row stride");
    // words of overlap bits
    ALIGNED(S, ovo_own, 8);
    ALIGNED(S, ovt_own, 8);
    ALIGNED(S, ovo_b, 8);
    ALIGNED(S, ovt_b, 8);
    // the network's biases, 16 bytes, and its weights, 8 bytes at a time
    ALIGNED(S, bias, 16);
    static_assert(!S::kWtsLds || (offsetof(S, wts) % 8 == 0 && sizeof(S::wts[0]) % 8 == 0), "wts");
};
template struct Sweep<float, 4, false>;
template struct Sweep<float, 8, false>;
template struct Sweep<double, 4, false>;
template struct Sweep<double, 8, false>;
template struct Sweep<float, 4, true>;
template struct Sweep<double, 4, true>;

ALIGNED(RowsShared, x, 8);
ALIGNED(RowsShared, h, 8);
ALIGNED(RowsShared, w1t, 8);
ALIGNED(RowsShared, w2t, 8);
ALIGNED(RowsShared, w2, 8);
static_assert(sizeof(row_t) % 8 == 0, "row stride");
