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
    FORM_RAGGED = 4,     // for operands whose rows do not start on 4 bytes
    FORM_SHORT = 8,      // for short products
    FORMS = 16
};

static const void* kernel_for(int dtype, bool akc, bool bkc, int v, int form) {
    const bool half = dtype == DT_F16 || dtype == DT_BF16, full = form & FORM_FULL;
    if (half && (form & FORM_OUT32)) v = with_block_sums(v);
    if ((form & FORM_RAGGED) && ((half && v == 2) || (dtype == DT_F8 && v == 1))) v = kKernelRagged;
    if (dtype == DT_F32 && v == 1 && (form & FORM_SHORT)) v = kKernelShort;
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

// Rows that do not start on 4 bytes, in launches whose workgroups run one tile or
// share at most.  The 16-bit tile where B's do not (A's alone: 2176x2048x2047 37.8 us
// on the seam loop, 40.5 without) and a workgroup runs more than 16 slabs (fewer:
// mean 1.00): of 130 such launches the time goes from the seam loop's to 0.96 (0.91-1.03)
// for shares and 0.99 (0.95-1.05) for whole tiles; of 48 with B's rows on 4 or 8 bytes
// to 1.05 (0.99-1.15), of 11 whose workgroups go on to a second tile to 1.04.  The FP8 tile
// where either operand's do not and more than one workgroup on a CU runs a share:
// 0.99 (0.96-1.04) of 19; rows on 4 or 8 bytes 1.02, one workgroup on a CU 1.01, whole
// tiles 1.02.
static bool ragged(int dtype, const KArgs& a, int cus) {
    if (a.G || a.t > a.grid) return false;              // (a table's operands are not known here)
    if (dtype == DT_F8 ? a.dp_only || a.grid <= cus : (a.dp_only ? a.ipt : a.sk_q) <= 16) return false;
    const int eb = dtype == DT_F8 ? 1 : 2;
    const auto off = [&](const void* x, int64_t ld, int64_t stride) {
        return ((reinterpret_cast<uintptr_t>(x) | uint64_t(ld * eb) | uint64_t(a.batch > 1 ? stride : 0)) & 3) != 0;
    };
    return off(a.B, a.ldb, a.stride_b) || (dtype == DT_F8 && off(a.A, a.lda, a.stride_a));
}

// Up to eight slabs of the FP32 quarter-size tile (a group's products any number).
static bool short_product(int dtype, const KArgs& a) { return dtype == DT_F32 && (a.G || a.ipt <= 8); }

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

int launch_gemm(int dtype, bool akc, bool bkc, int v, const KArgs& args, int grid, int cus, void* stream) {
    const int form = (needs_full(args) ? FORM_FULL : 0) | (args.out_dtype == DT_F32 ? FORM_OUT32 : 0) |
                     (ragged(dtype, args, cus) ? FORM_RAGGED : 0) | (short_product(dtype, args) ? FORM_SHORT : 0);
    const void* f = kernel_for(dtype, akc, bkc, v, form);
    if (!f) return int(hipErrorInvalidDeviceFunction);
    KArgs copy = args;
    void* params[] = {&copy};
    return int(hipLaunchKernel(f, dim3(grid), dim3(kernel_threads(dtype, v)), params, 0,
                               reinterpret_cast<hipStream_t>(stream)));
}

}  // namespace skg
