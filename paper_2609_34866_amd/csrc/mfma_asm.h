// mfma_asm.h -- a matrix product written as inline assembly, for the attention kernels whose output
// accumulators fill the 256 accumulation registers.
#pragma once

#include "device_common.h"

namespace jab {
namespace {

// S^T += K Q^T with the result in architectural registers, for the kernels whose output
// accumulators fill the 256 accumulation registers (the compiler would place this product's
// result in accumulation registers too and shuffle output blocks out and back every block).
// The compiler does not see the product inside the asm, so the hazards it would cover are covered
// here: two wait states before each product (a vector write of an operand), and 19 after the last
// product of a chain (LAST), inside the same asm, so that no instruction the compiler places after
// it (a copy of the result included) reads or writes the result too early.  Between the products
// of a chain the result passes from one asm to the next as a tied operand; the build checks the
// generated code for any other access within the window.
template <int DT>
__device__ inline f32x16 mma_v(typename Mma<DT>::operand a, typename Mma<DT>::operand b, f32x16 c, bool first,
                               bool last) {
    static_assert(DT == BF16 || DT == F16, "16-bit operands");
#define JAB_MMA_V(OP, C, TAIL, CON)                                                             \
    asm volatile("s_nop 1\n\t" OP " %0, %1, %2, " C TAIL : CON(d) : "v"(a), "v"(b))
#define JAB_DRAIN "\n\ts_nop 7\n\ts_nop 7\n\ts_nop 2"
#define JAB_MMA_V_ALL(OP)                                                                       \
    if (first && last) JAB_MMA_V(OP, "0", JAB_DRAIN, "=&v");                                    \
    else if (first) JAB_MMA_V(OP, "0", "", "=&v");                                              \
    else if (last) JAB_MMA_V(OP, "%0", JAB_DRAIN, "+v");                                        \
    else JAB_MMA_V(OP, "%0", "", "+v")
    f32x16 d = c;
    if constexpr (DT == BF16) {
        JAB_MMA_V_ALL("v_mfma_f32_32x32x16_bf16");
    } else {
        JAB_MMA_V_ALL("v_mfma_f32_32x32x16_f16");
    }
#undef JAB_MMA_V_ALL
#undef JAB_DRAIN
#undef JAB_MMA_V
    return d;
}

}  // namespace
}  // namespace jab
