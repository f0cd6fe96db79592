// The output-matrix product of the exit head with its softmax-partials epilogue.
#include "epilogues.h"
#include "launch.h"

namespace ee {

static_assert(CfgBig::WN == 64 && CfgMid::WN == 64 && CfgF32::WN == 64 && CfgF32Small::WN == 64, "one slice width");
bool gemm_mid_tile(int64_t big_tiles) { return big_tiles <= kLoopBlocks / 2; }

int gemm_part_cols(bool) { return CfgBig::WN; }

hipError_t gemm_logits(bool f32, const void *w_out, const void *z, int vocab, int n, int h, void *P, int ldn,
                       float *part_m, float *part_l, float *tgt, const int32_t *targets, hipStream_t stream,
                       int shift0, const int *run_if) {
  EE_DISPATCH(f32, {
    typename EpiLogits<T>::Params ep{static_cast<T *>(P), ldn, part_m, part_l, tgt, targets, shift0};
    const Operand A{z, h}, B{w_out, h};
    const GemmShape sh{n, vocab, h};
    if (run_if != nullptr) {
      if constexpr (std::is_same<T, bf16_t>::value)
        return launch_gemm_gated<T, true, true, EpiLogits<T>, CfgBig>(A, B, sh, ep, run_if, stream);
      else
        return launch_gemm_gated<T, true, true, EpiLogits<T>, CfgF32>(A, B, sh, ep, run_if, stream);
    }
    return run_gemm<T, true, true, EpiLogits<T>>(A, B, sh, ep, stream);
  });
  return hipSuccess;
}

}  // namespace ee
