// The forward products of the MLP exit, and the split-K tail its token-by-feature products share.
#include <algorithm>
#include <functional>
#include <queue>
#include <vector>

#include "epilogues.h"
#include "launch.h"

namespace ee {

hipError_t gemm_gate_up_swiglu(bool f32, const void *u, const void *w_gate, const void *w_up, int n, int inter,
                               int h, void *hgu, void *act, hipStream_t stream) {
  EE_DISPATCH(f32, {
    typename EpiGateUp<T>::Params ep{static_cast<typename GatePair<T>::type *>(hgu), static_cast<T *>(act)};
    const int64_t pair = static_cast<const char *>(w_up) - static_cast<const char *>(w_gate);
    return run_gemm<T, true, true, EpiGateUp<T>>(Operand{u, h}, Operand{w_gate, h, pair},
                                                    GemmShape{n, 2 * inter, h}, ep, stream);
  });
  return hipSuccess;
}

hipError_t gemm_down_residual(bool f32, const void *act, const void *w_down, const void *x, int n, int h,
                              int inter, float *y, hipStream_t stream, SplitTail sp) {
  EE_DISPATCH(f32, {
    const T *xt = static_cast<const T *>(x), *at = static_cast<const T *>(act), *wd = static_cast<const T *>(w_down);
    // Tiles: tokens as rows, features as columns.  Split region: tokens
    // [t0, n) x features [f0, h).  The rest takes all of K: tokens [0, t0)
    // (f0 == 0) or features [0, f0) (t0 == 0).
    const bool split = sp.splits > 1;
    const int t0 = split ? sp.tok0 : n, f0 = split ? sp.feat0 : 0;
    if (t0 < 0 || t0 > n || f0 < 0 || f0 > h || (t0 > 0 && f0 > 0)) return hipErrorInvalidValue;
    const int m1 = t0 > 0 ? t0 : n, n1 = t0 > 0 ? h : f0;
    const int64_t o = static_cast<int64_t>(t0) * h + f0;
    typename EpiResidual<T>::Params e1{y, xt, h, 0};
    typename EpiResidual<T>::Params e2{y + o, xt + o, h, static_cast<int64_t>(n) * h};
    GemmShape s2{n - t0, h - f0, inter};
    if (split) {
      s2.kchunk = split_kchunk(inter, sp.splits);
      if (cdiv(inter, s2.kchunk) != sp.splits) return hipErrorInvalidValue;  // Y holds sp.splits slices
    }
    return run_gemm_pair<T, true, true, EpiResidual<T>, true, true, EpiResidual<T>>(
        Operand{at, inter}, Operand{wd, inter}, GemmShape{m1, n1, inter}, e1,
        Operand{at + static_cast<int64_t>(t0) * inter, inter}, Operand{wd + static_cast<int64_t>(f0) * inter, inter},
        s2, e2, stream);
  });
  return hipSuccess;
}

namespace {

constexpr int kCus = 256;           // compute units the launch shapes are planned for
constexpr double kEpilogueK = 1024;  // prologue and epilogue of a 256 x 256 tile, in K values of its main loop
constexpr double kBytesPerK = 1.2e5;  // HBM bytes moved while a CU runs one such K value

// Duration, in K values, of `full` whole-K tiles followed by `parts` blocks
// of kchunk K values each, dispatched in order to the first free of kCus
// compute units.
double launch_span(int64_t full, int64_t parts, int K, int kchunk) {
  const double D = K + kEpilogueK, d = kchunk + kEpilogueK;
  const int64_t rest = full % kCus;
  std::priority_queue<double, std::vector<double>, std::greater<double>> q;
  double end = rest > 0 ? D : 0.0;
  for (int i = 0; i < kCus; ++i) q.push(i < rest ? D : 0.0);
  for (int64_t p = 0; p < parts; ++p) {
    const double t = q.top() + d;
    q.pop();
    q.push(t);
    end = std::max(end, t);
  }
  return static_cast<double>(full / kCus) * D + end;
}

}  // namespace

int split_kchunk(int K, int splits) { return cdiv(cdiv(K, splits), 64) * 64; }

SplitTail split_tail(bool f32, int n, int h, int K, int most) {
  SplitTail best{n, 0, 1};
  if (n <= 0) return best;
  if (f32) {
    // every output as up to `most` partial sums of at least 256 values of K, as
    // long as the 64 x 64 tiles leave two blocks a CU unfilled
    const int s = static_cast<int>(std::min<int64_t>({most, 2 * kCus / (static_cast<int64_t>(cdiv(n, 64)) * cdiv(h, 64)), K / 256}));
    return s > 1 ? SplitTail{0, 0, cdiv(K, split_kchunk(K, s))} : best;
  }
  // the last few shapes asked for (a layout asks for two per call)
  struct Memo {
    int n = -1, h = -1, K = -1;
    SplitTail sp{0, 0, 1};
  };
  static thread_local Memo memo[4];
  static thread_local int next = 0;
  for (const Memo &m : memo)
    if (m.n == n && m.h == h && m.K == K) return m.sp;
  const int tm = cdiv(h, CfgBig::BM), tn = cdiv(n, CfgBig::BN);
  const int64_t tiles = static_cast<int64_t>(tm) * tn;
  if (tiles < 4 * kCus) {
    const int64_t rounds = tiles / kCus;
    double best_span = 0.9 * launch_span(tiles, 0, K, K);
    for (int s = 2; s <= 4; s *= 2) {
      if (K / s < 4 * 64) break;
      const int kc = split_kchunk(K, s), slices = cdiv(K, kc);
      // Split the last c token blocks (dim 0) or feature blocks (dim 1):
      // all of them, or the fewest that leave the whole-K tiles one or two
      // rounds short of the current count.
      for (int dim = 0; dim < 2; ++dim) {
        const int blocks = dim == 0 ? tn : tm, across = dim == 0 ? tm : tn;
        int cand[3] = {blocks, 0, 0};
        for (int r = 0; r < 2; ++r)
          if (rounds - r >= 0) cand[r + 1] = static_cast<int>((tiles - (rounds - r) * kCus + across - 1) / across);
        for (int c : cand) {
          if (c < 1 || c > blocks) continue;
          const SplitTail sp = dim == 0 ? SplitTail{(tn - c) * CfgBig::BN, 0, slices}
                                        : SplitTail{0, (tm - c) * CfgBig::BM, slices};
          // extra HBM traffic: slices 1.. written and read back, their sum written
          const double outs = static_cast<double>(n - sp.tok0) * (h - sp.feat0);
          const double extra = outs * 4 * (2 * (slices - 1) + 1) / kBytesPerK;
          const double span = launch_span(static_cast<int64_t>(blocks - c) * across,
                                          static_cast<int64_t>(c) * across * slices, K, kc) + extra;
          if (span < best_span) {
            best_span = span;
            best = sp;
          }
        }
      }
    }
  }
  memo[next] = Memo{n, h, K, best};
  next = (next + 1) % 4;
  return best;
}

}  // namespace ee
