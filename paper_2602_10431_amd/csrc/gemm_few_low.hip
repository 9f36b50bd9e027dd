// 3- and 2-bit forms of the few-row GEMM (gemm_few.h).
#include "gemm_few.h"

namespace qtale {

hipError_t launch_gemm_few_low(const GemmDev& d, int epilogue, const FewPrologue* pro, int cus, hipStream_t stream) {
    FewDev a{};
    a.g = d;
    if (pro) a.pro = *pro;
    if (d.bits == 3) return d.gshift == 5 ? few_shape<3, 2>(a, epilogue, cus, stream) : few_shape<3, 1>(a, epilogue, cus, stream);
    return d.gshift == 5 ? few_shape<2, 2>(a, epilogue, cus, stream) : few_shape<2, 1>(a, epilogue, cus, stream);
}

}  // namespace qtale
