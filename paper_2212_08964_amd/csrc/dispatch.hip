// Kernel lookup, occupancy query and launch for the Stream-K GEMM kernels.
#include <hip/hip_runtime.h>

#include "skgemm_internal.h"

namespace skg {

const void* kernel_fn_f32(bool akc, bool bkc, int v);
const void* kernel_fn_f16(bool akc, bool bkc, int v);
const void* kernel_fn_bf16(bool akc, bool bkc, int v);
const void* kernel_fn_f8(bool akc, bool bkc, int v);
const void* kernel_fn_f64(bool akc, bool bkc, int v);
const void* kernel_fn_f32_full(bool akc, bool bkc, int v);
const void* kernel_fn_f16_full(bool akc, bool bkc, int v);
const void* kernel_fn_bf16_full(bool akc, bool bkc, int v);
const void* kernel_fn_f8_full(bool akc, bool bkc, int v);
const void* kernel_fn_f64_full(bool akc, bool bkc, int v);
int kernel_threads_f32(int v);
int kernel_threads_f16(int v);
int kernel_threads_bf16(int v);
int kernel_threads_f8(int v);
int kernel_threads_f64(int v);

// Instantiations of one plan's kernel.
enum Form {
    FORM_FULL = 1,       // with the group table, batch, trace and timestamp paths
    FORM_OUT32 = 2,      // for FP32 results
    FORMS = 4
};

static const void* kernel_for(int dtype, bool akc, bool bkc, int v, int form) {
    const bool half = dtype == DT_F16 || dtype == DT_BF16, full = form & FORM_FULL;
    if (half && (form & FORM_OUT32)) v = with_block_sums(v);
    switch (dtype) {
        case DT_F32: return full ? kernel_fn_f32_full(akc, bkc, v) : kernel_fn_f32(akc, bkc, v);
        case DT_F16: return full ? kernel_fn_f16_full(akc, bkc, v) : kernel_fn_f16(akc, bkc, v);
        case DT_BF16: return full ? kernel_fn_bf16_full(akc, bkc, v) : kernel_fn_bf16(akc, bkc, v);
        case DT_F8: return full ? kernel_fn_f8_full(akc, bkc, v) : kernel_fn_f8(akc, bkc, v);
        case DT_F64: return full ? kernel_fn_f64_full(akc, bkc, v) : kernel_fn_f64(akc, bkc, v);
        default: return nullptr;
    }
}

static bool needs_full(const KArgs& a) { return a.G || a.batch > 1 || a.trace || a.times; }

bool kernel_exists(int dtype, bool akc, bool bkc, int v) {
    for (int form = 0; form < FORMS; ++form)
        if (!kernel_for(dtype, akc, bkc, v, form)) return false;
    return true;
}

int kernel_threads(int dtype, int v) {
    switch (dtype) {
        case DT_F32: return kernel_threads_f32(v);
        case DT_F16: return kernel_threads_f16(v);
        case DT_BF16: return kernel_threads_bf16(v);
        case DT_F8: return kernel_threads_f8(v);
        case DT_F64: return kernel_threads_f64(v);
        default: return 0;
    }
}

// The smallest of the forms' occupancies: a plan's grid must be co-resident
// whichever form runs it.
int kernel_occupancy(int dtype, bool akc, bool bkc, int v) {
    int occ = 0;
    for (int form = 0; form < FORMS; ++form) {
        const void* f = kernel_for(dtype, akc, bkc, v, form);
        if (!f) return 0;
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, kernel_threads(dtype, v), 0) != hipSuccess) return 0;
        occ = form ? (n < occ ? n : occ) : n;
    }
    return occ;
}

int launch_gemm(int dtype, bool akc, bool bkc, int v, const KArgs& args, int grid, void* stream) {
    const int form = (needs_full(args) ? FORM_FULL : 0) | (args.out_dtype == DT_F32 ? FORM_OUT32 : 0);
    const void* f = kernel_for(dtype, akc, bkc, v, form);
    if (!f) return int(hipErrorInvalidDeviceFunction);
    KArgs copy = args;
    void* params[] = {&copy};
    return int(hipLaunchKernel(f, dim3(grid), dim3(kernel_threads(dtype, v)), params, 0,
                               reinterpret_cast<hipStream_t>(stream)));
}

}  // namespace skg
