// Lean instantiations (plain GEMMs) of the Stream-K GEMM kernel for one
// input type, and its workgroup sizes.
#include "kernel_tables.hpp"

namespace skg {

const void* kernel_fn_f16(bool akc, bool bkc, int v) { return kernel_table<DT_F16, false>(akc, bkc, v); }

int kernel_threads_f16(int v) {
    constexpr int n[] = {kThreadsOf<DT_F16, 0>, kThreadsOf<DT_F16, 1>, kThreadsOf<DT_F16, 2>, kThreadsOf<DT_F16, 3>,
                         kThreadsOf<DT_F16, 4>, kThreadsOf<DT_F16, 5>, kThreadsOf<DT_F16, 6>, kThreadsOf<DT_F16, 7>,
                         kThreadsOf<DT_F16, 8>, kThreadsOf<DT_F16, 9>, kThreadsOf<DT_F16, 10>, kThreadsOf<DT_F16, 11>,
                         kThreadsOf<DT_F16, 12>};
    static_assert(sizeof(n) / sizeof(n[0]) == kVariants, "one entry per variant");
    return v >= 0 && v < kVariants ? n[v] : 0;
}

}  // namespace skg
