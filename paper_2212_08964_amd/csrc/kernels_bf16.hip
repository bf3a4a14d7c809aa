// Lean instantiations (plain GEMMs) of the Stream-K GEMM kernel for one
// input type, and its workgroup sizes.
#include "kernel_tables.hpp"

namespace skg {

const void* kernel_fn_bf16(bool akc, bool bkc, int v) { return kernel_table<DT_BF16, false>(akc, bkc, v); }

int kernel_threads_bf16(int v) {
    constexpr int n[] = {kThreadsOf<DT_BF16, 0>, kThreadsOf<DT_BF16, 1>, kThreadsOf<DT_BF16, 2>, kThreadsOf<DT_BF16, 3>,
                         kThreadsOf<DT_BF16, 4>, kThreadsOf<DT_BF16, 5>, kThreadsOf<DT_BF16, 6>, kThreadsOf<DT_BF16, 7>,
                         kThreadsOf<DT_BF16, 8>, kThreadsOf<DT_BF16, 9>, kThreadsOf<DT_BF16, 10>, kThreadsOf<DT_BF16, 11>,
                         kThreadsOf<DT_BF16, 12>};
    static_assert(sizeof(n) / sizeof(n[0]) == kVariants, "one entry per variant");
    return v >= 0 && v < kVariants ? n[v] : 0;
}

}  // namespace skg
