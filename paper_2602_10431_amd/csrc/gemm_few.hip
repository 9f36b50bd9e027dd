// 4-bit forms of the few-row GEMM and its dispatch (the kernel is in gemm_few.h; the other code widths, which take as long
// to compile, are in gemm_few_low.hip).
#include "gemm_few.h"

namespace qtale {

hipError_t launch_gemm_few_low(const GemmDev& d, int epilogue, const FewPrologue* pro, int cus, hipStream_t stream);

bool few_prologue_fits(int T, int max_rows, int hidden) {
    // one 8-column piece of every row per thread of the smallest workgroup (8 waves); the normalised rows fit the 64 KB of
    // LDS that a kernel gets without asking (with a little static LDS beside them)
    return max_rows > 0 && T <= kFewFuseT && hidden <= 8 * 512 * kFewPasses && static_cast<size_t>(max_rows) * (hidden + 8) * 2 <= 60 * 1024;
}

hipError_t launch_gemm_few(const GemmDev& d, int epilogue, const FewPrologue* pro, int cus, hipStream_t stream) {
    if (d.bits != 4) return launch_gemm_few_low(d, epilogue, pro, cus, stream);
    FewDev a{};
    a.g = d;
    if (pro) a.pro = *pro;
    return d.gshift == 5 ? few_shape<4, 2>(a, epilogue, cus, stream) : few_shape<4, 1>(a, epilogue, cus, stream);
}

}  // namespace qtale
