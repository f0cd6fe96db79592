// The output-matrix product of the exit head with its softmax-partials epilogue.
#include "epilogues.h"
#include "launch.h"

namespace ee {

static_assert(CfgBig::WN == 64 && CfgMid::WN == 64 && CfgF32::WN == 64 && CfgF32Small::WN == 64, "one slice width");
bool gemm_mid_tile(int64_t big_tiles) { return big_tiles <= kLoopBlocks / 2; }

int gemm_f32_parts(int64_t tiles, int64_t small_tiles) {
  return 3 * cdiv(small_tiles, kLoopBlocks) < 10 * cdiv(tiles, kLoopBlocks) ? 4 : 1;
}
bool gemm_f32_small(int64_t tiles, int64_t small_tiles, int K) {
  constexpr int kPair = 2 * kLoopBlocks;  // blocks of a round, two a CU
  const int64_t rounds = cdiv(tiles, kLoopBlocks);
  double big = (rounds / 2) * (10.7 + 0.1165 * K) + (rounds % 2) * (4.5 + 0.068 * K);
  if (gemm_f32_parts(tiles, small_tiles) > 1) big *= 1.03;  // what the parts cost
  const double one = 5.3 + 0.0188 * K, two = 6.0 + 0.0313 * K;  // a round of small tiles, one and two a CU
  const int64_t rest = small_tiles % kPair;
  double small = static_cast<double>(small_tiles / kPair) * two;
  if (rest > kLoopBlocks)
    small += two;
  else if (rest > 0)  // after a full round, some CUs take two of the rest
    small += one + (small_tiles > kPair ? 0.7 * (two - one) * static_cast<double>(rest) / kLoopBlocks : 0.0);
  return small < big;
}
bool gemm_f32_loops(int64_t tiles) {
  const int64_t rest = tiles % (2 * kLoopBlocks);
  return tiles > 2 * kLoopBlocks && rest > 0 && rest <= kLoopBlocks;
}

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
