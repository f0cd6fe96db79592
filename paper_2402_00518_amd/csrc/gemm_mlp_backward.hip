// The backward products of the MLP exit that read an operand MN-major.
#include "epilogues.h"
#include "launch.h"

namespace ee {

hipError_t gemm_dz(bool f32, const void *g_t, const void *w_out, int n, int ldn, int h, int vocab, float *dz,
                   hipStream_t stream, SplitTail sp) {
  EE_DISPATCH(f32, {
    const T *gt = static_cast<const T *>(g_t), *wo = static_cast<const T *>(w_out);
    // Tiles: tokens (padded to ldn; rows past n are not stored) as rows,
    // features as columns, both operands read MN-major.  Split region:
    // tokens [t0, n) x features [f0, h); the rest takes all of K: tokens
    // [0, t0) (f0 == 0) or features [0, f0) (t0 == 0).
    if (sp.splits <= 1) {
      typename EpiStoreF32<T>::Params ep{dz, h, n, 0, 0};
      return run_gemm<T, false, false, EpiStoreF32<T>>(Operand{gt, ldn}, Operand{wo, h}, GemmShape{ldn, h, vocab}, ep,
                                                        stream);
    }
    const int t0 = sp.tok0, f0 = sp.feat0;
    if (t0 < 0 || t0 > n || t0 % 64 != 0 || f0 < 0 || f0 > h || (t0 > 0 && f0 > 0)) return hipErrorInvalidValue;
    const int m1 = t0 > 0 ? t0 : ldn, n1 = t0 > 0 ? h : f0;
    typename EpiStoreF32<T>::Params e1{dz, h, t0 > 0 ? t0 : n, 0, 0};
    typename EpiStoreF32<T>::Params e2{dz + static_cast<int64_t>(t0) * h + f0, h, n - t0, 0,
                                       static_cast<int64_t>(n) * h};
    GemmShape s2{ldn - t0, h - f0, vocab};
    s2.kchunk = split_kchunk(vocab, sp.splits);
    if (cdiv(vocab, s2.kchunk) != sp.splits) return hipErrorInvalidValue;  // dZ holds sp.splits slices
    return run_gemm_pair<T, false, false, EpiStoreF32<T>, false, false, EpiStoreF32<T>>(
        Operand{gt, ldn}, Operand{wo, h}, GemmShape{m1, n1, vocab}, e1, Operand{gt + t0, ldn}, Operand{wo + f0, h}, s2,
        e2, stream);
  });
  return hipSuccess;
}

hipError_t gemm_da_swiglu_dw_down(bool f32, const void *dy, const void *w_down, int n, int inter, int h,
                                 const void *hgu, void *dhg_t, void *dhu_t, int ldn, const void *act, float *dwd,
                                 int accumulate, hipStream_t stream) {
  EE_DISPATCH(f32, {
    typename EpiSwiGLUBwd<T>::Params e1{static_cast<const typename GatePair<T>::type *>(hgu),
                                        static_cast<T *>(dhg_t), static_cast<T *>(dhu_t), inter, ldn};
    typename EpiStoreF32<T>::Params e2{dwd, inter, h, accumulate};
    return run_gemm_pair<T, true, false, EpiSwiGLUBwd<T>, false, false, EpiStoreF32<T>>(
        Operand{dy, h}, Operand{w_down, inter}, GemmShape{n, inter, h}, e1, Operand{dy, h}, Operand{act, inter},
        GemmShape{h, inter, n}, e2, stream);
  });
  return hipSuccess;
}

}  // namespace ee
