// The weight-gradient products whose operands are both token-contiguous.
#include "epilogues.h"
#include "launch.h"

namespace ee {

hipError_t gemm_weight_grad_kk(bool f32, const void *g_t, const void *xhat_t, int m, int h, int ldn,
                               const void *gain, const void *w, float *dw, float *part, int accumulate,
                               hipStream_t stream, const float *gsum, const void *bias, float *part_b) {
  EE_DISPATCH(f32, {
    typename EpiWeightGrad<T>::Params ep{dw,   h,         static_cast<const T *>(gain), static_cast<const T *>(w),
                                         part, accumulate, gsum, static_cast<const T *>(bias), part_b};
    return run_gemm<T, true, true, EpiWeightGrad<T>>(Operand{xhat_t, ldn}, Operand{g_t, ldn},
                                                        GemmShape{h, m, ldn}, ep, stream);
  });
  return hipSuccess;
}

hipError_t gemm_weight_grad_kk_pair(bool f32, const void *g1_t, const void *g2_t, const void *xhat_t, int m, int h,
                                    int ldn, const void *gain, const void *w1, const void *w2, float *dw1, float *dw2,
                                    float *part1, float *part2, int accumulate, hipStream_t stream) {
  EE_DISPATCH(f32, {
    const T *gn = static_cast<const T *>(gain);
    typename EpiWeightGrad<T>::Params e1{dw1, h, gn, static_cast<const T *>(w1), part1, accumulate};
    typename EpiWeightGrad<T>::Params e2{dw2, h, gn, static_cast<const T *>(w2), part2, accumulate};
    return run_gemm_pair<T, true, true, EpiWeightGrad<T>, true, true, EpiWeightGrad<T>>(
        Operand{xhat_t, ldn}, Operand{g1_t, ldn}, GemmShape{h, m, ldn}, e1, Operand{xhat_t, ldn},
        Operand{g2_t, ldn}, GemmShape{h, m, ldn}, e2, stream);
  });
  return hipSuccess;
}

}  // namespace ee
