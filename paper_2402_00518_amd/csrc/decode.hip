// Decode-time exit head (Sec. 3 "Inference": greedy decoding with a
// confidence-based exit): a handful of rows through one exit, forward only.
//
// At decode the products are skinny, C[r][j] = sum_k W[r][k] Z[j][k] with a
// weight W of R rows and B token rows Z, bound by streaming W from HBM once.
//
// bf16: ring_kernel, W and Z through LDS (see launch_ring); skinny_kernel where
// W has few rows (see decode_skinny_logits).
//
// fp32, and those: skinny_kernel, 32 tokens a pass.  A block owns 32 rows of W (64 for a
// wide W past 8 token rows, so that each token fragment serves two row groups
// and the token rows' share of the loads halves); each of its waves takes a
// share of K and reads its rows straight into MFMA A fragments (16 bytes of K
// per lane), 12 fragments per row group in flight per lane; the token rows
// come from L2 as B fragments (tokens past B re-read row B-1 and their outputs
// are dropped).  The waves' partial sums meet in LDS in a fixed order and the
// first wave runs the epilogue.
//
// Epilogues: SwiGLU (gate and up projections), residual (down projection)
// and, for the output matrix, softmax partials of 32 rows at a time:
// for each token the maximum logit over the wave's rows, the lowest row
// reaching it and sum exp(S - max).  decide_kernel combines the partials
// of all waves into the greedy token, its probability and the exit flag.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ee_device.h"
#include "launch.h"
#include "ring.h"

namespace ee {

namespace {

constexpr int cdiv64(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

constexpr int kDecRows = 32;    // rows of W per row group (one MFMA tile)
constexpr int kDecTokens = 32;  // token rows per pass (grid.y walks more)
// Waves per block (each a share of K): 4 when the rows give at least two
// blocks per CU of a 256-CU GPU, else 8 or 16, so that narrow products (the
// MLP's down projection: 5120 rows, K = 13824) still keep enough loads in
// flight.  A shape-only rule, so results do not depend on the device.
constexpr int kDecWavesMax = 16;
__host__ __device__ constexpr int dec_waves(int row_blocks) {
  return row_blocks >= 512 ? 4 : (row_blocks >= 256 ? 8 : 16);
}
constexpr int kDecGroup = 12;   // fragment loads per operand per lane in flight (8 and 16 measured slower)

template <typename T> struct DecFrag;
// bf16: a 16-byte load holds 8 values of K; one MFMA consumes 16 (two lane halves).
template <> struct DecFrag<bf16_t> {
  static constexpr int K_PER_LOAD = 16;  // values of K covered by one load across the wave
  __device__ __forceinline__ static void mma(const u32x4_t &a, const u32x4_t &b, f32x16_t &acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b),
                                                  acc, 0, 0, 0);
  }
};
// fp32: a 16-byte load holds 4 values of K; four MFMAs of K = 2 (lane halves
// hold K offsets 0-3 and 4-7 of the same 8, in the same order for A and B).
template <> struct DecFrag<float> {
  static constexpr int K_PER_LOAD = 8;
  __device__ __forceinline__ static void mma(const u32x4_t &a, const u32x4_t &b, f32x16_t &acc) {
    static_for<4>([&](auto e) EE_ALWAYS_INLINE {
      constexpr int E = decltype(e)::value;
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[E]), __uint_as_float(b[E]), acc, 0, 0, 0);
    });
  }
};

// acc[v] of lane l: row r0 + (v/4)*8 + (l/32)*4 + v%4, token j0 + l%32.
__device__ __forceinline__ int dec_row(int r0, int lane, int v) {
  return r0 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
}

template <typename T, class Epi, int kDecWaves, int RG>
__global__ __launch_bounds__(64 * kDecWaves) void skinny_kernel(const T *__restrict__ W, int64_t ldw, int R,
                                                                const T *__restrict__ Z, int64_t ldz, int B, int K,
                                                                typename Epi::Params ep) {
  constexpr int KL = DecFrag<T>::K_PER_LOAD;
  constexpr int PER_LOAD = 16 / sizeof(T);  // elements of one 16-byte load
  __shared__ f32x16_t red[kDecWaves - 1][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r0 = blockIdx.x * kDecRows * RG, j0 = blockIdx.y * kDecTokens;
  const int zr = min(j0 + (lane & 31), B - 1);
  const int koff = (lane >> 5) * PER_LOAD;
  const char *wp[RG];
  static_for<RG>([&](auto g) EE_ALWAYS_INLINE {
    constexpr int G = decltype(g)::value;
    const int wr = min(r0 + G * kDecRows + (lane & 31), R - 1);
    wp[G] = reinterpret_cast<const char *>(W + static_cast<int64_t>(wr) * ldw + koff);
  });
  const char *zp = reinterpret_cast<const char *>(Z + static_cast<int64_t>(zr) * ldz + koff);
  f32x16_t acc[RG];
  static_for<RG>([&](auto g) EE_ALWAYS_INLINE {
    static_for<16>([&](auto v) EE_ALWAYS_INLINE { acc[decltype(g)::value][decltype(v)::value] = 0.0f; });
  });

  // This wave's share of K, in whole groups of 4 loads (K is a multiple of
  // 4 KL): groups [g0, g1) of the K / (4 KL) groups.  Each token fragment
  // serves the RG row groups of the block.
  constexpr int KG4 = 4 * KL;
  const int groups = K / KG4;
  const int g0 = wave * groups / kDecWaves, g1 = (wave + 1) * groups / kDecWaves;
  int k = g0 * KG4;
  const int kend = g1 * KG4;
  auto step = [&](auto nq) EE_ALWAYS_INLINE {
    constexpr int NQ = decltype(nq)::value;
    u32x4_t a[RG][NQ], b[NQ];
    static_for<NQ>([&](auto q) EE_ALWAYS_INLINE {
      constexpr int Q = decltype(q)::value;
      const int64_t off = (static_cast<int64_t>(k) + Q * KL) * sizeof(T);
      static_for<RG>([&](auto g) EE_ALWAYS_INLINE {
        a[decltype(g)::value][Q] = *reinterpret_cast<const u32x4_t *>(wp[decltype(g)::value] + off);
      });
      b[Q] = *reinterpret_cast<const u32x4_t *>(zp + off);
    });
    // Keep every load of the group ahead of the MFMAs: left alone, the
    // scheduler would trade loads in flight for registers.
    __builtin_amdgcn_sched_barrier(0);
    static_for<NQ>([&](auto q) EE_ALWAYS_INLINE {
      static_for<RG>([&](auto g) EE_ALWAYS_INLINE {
        DecFrag<T>::mma(a[decltype(g)::value][decltype(q)::value], b[decltype(q)::value], acc[decltype(g)::value]);
      });
    });
  };
  constexpr int KG = kDecGroup * KL;
  for (; k + KG <= kend; k += KG) step(std::integral_constant<int, kDecGroup>{});
  for (; k < kend; k += KG4) step(std::integral_constant<int, 4>{});
  // Per row group: partial sums of waves 1.. to LDS; wave 0 adds them in
  // order and finishes.
  static_for<RG>([&](auto g) EE_ALWAYS_INLINE {
    constexpr int G = decltype(g)::value;
    if (G > 0) __syncthreads();  // wave 0 has read the previous group
    if (wave > 0) red[wave - 1][lane] = acc[G];
    __syncthreads();
    if (wave == 0 && r0 + G * kDecRows < R) {  // a second group may lie past the last row
      f32x16_t c = acc[G];
      static_for<kDecWaves - 1>([&](auto w) EE_ALWAYS_INLINE { c += red[decltype(w)::value][lane]; });
      Epi::apply(ep, c, r0 + G * kDecRows, j0, lane, R, B);
    }
  });
}

// Four consecutive rows of one token as fp32 (bf16 or fp32 storage).
template <typename T> __device__ __forceinline__ f32x4_t dload4(const T *p);
template <> __device__ __forceinline__ f32x4_t dload4<float>(const float *p) {
  return *reinterpret_cast<const f32x4_t *>(p);
}
template <> __device__ __forceinline__ f32x4_t dload4<bf16_t>(const bf16_t *p) {
  const u32x2_t u = *reinterpret_cast<const u32x2_t *>(p);
  return f32x4_t{__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xFFFF0000u), __uint_as_float(u[1] << 16),
                 __uint_as_float(u[1] & 0xFFFF0000u)};
}
template <typename T> __device__ __forceinline__ void dstore4(T *p, f32x4_t v);
template <> __device__ __forceinline__ void dstore4<float>(float *p, f32x4_t v) {
  *reinterpret_cast<f32x4_t *>(p) = v;
}
template <> __device__ __forceinline__ void dstore4<bf16_t>(bf16_t *p, f32x4_t v) {
  const u32x2_t u = {static_cast<uint32_t>(f32_to_bf16(v[0])) | (static_cast<uint32_t>(f32_to_bf16(v[1])) << 16),
                     static_cast<uint32_t>(f32_to_bf16(v[2])) | (static_cast<uint32_t>(f32_to_bf16(v[3])) << 16)};
  *reinterpret_cast<u32x2_t *>(p) = u;
}

// f(row0, token, vals) for each group of 4 consecutive rows of the lane
// (rows are feature indices, a multiple of 4 apart from the tile origin;
// R is a multiple of 64 for the MLP products that use this).
template <class F>
__device__ __forceinline__ void for_rows4(const f32x16_t &acc, int r0, int j0, int lane, int R, int B, F &&f) {
  const int j = j0 + (lane & 31);
  if (j >= B) return;
  static_for<4>([&](auto q) EE_ALWAYS_INLINE {
    constexpr int Q = decltype(q)::value;
    const int row0 = dec_row(r0, lane, 4 * Q);
    if (row0 < R) f(row0, j, f32x4_t{acc[4 * Q], acc[4 * Q + 1], acc[4 * Q + 2], acc[4 * Q + 3]});
  });
}

struct DecStore {  // out[j][r] = C[r][j]  (fp32)
  struct Params {
    float *out;
    int64_t ld;
  };
  __device__ __forceinline__ static void apply(const Params &p, const f32x16_t &acc, int r0, int j0, int lane, int R,
                                               int B) {
    for_rows4(acc, r0, j0, lane, R, B, [&](int row0, int j, f32x4_t c) EE_ALWAYS_INLINE {
      dstore4<float>(p.out + static_cast<int64_t>(j) * p.ld + row0, c);
    });
  }
};

struct DecSwiGLU {  // A[j][r] = silu(Hg[j][r]) * C[r][j]  (fp32)
  struct Params {
    const float *hg;
    float *act;
    int64_t ld;
  };
  __device__ __forceinline__ static void apply(const Params &p, const f32x16_t &acc, int r0, int j0, int lane, int R,
                                               int B) {
    for_rows4(acc, r0, j0, lane, R, B, [&](int row0, int j, f32x4_t hu) EE_ALWAYS_INLINE {
      const int64_t o = static_cast<int64_t>(j) * p.ld + row0;
      const f32x4_t hg = dload4<float>(p.hg + o);
      f32x4_t a;
      static_for<4>([&](auto e) EE_ALWAYS_INLINE {
        constexpr int E = decltype(e)::value;
        a[E] = silu_f(hg[E]) * hu[E];
      });
      dstore4<float>(p.act + o, a);
    });
  }
};

// Y[j][r] = X[j][r] + C[r][j]  (fp32 out).  With split K, slice 0 does so and
// slice z > 0 stores its partial sum at extra + (z - 1) zstride (the exit norm
// adds the slices).
template <typename T>
struct DecResidual {
  static constexpr bool kSplit = true;
  struct Params {
    const T *x;
    float *y;
    int64_t ld;
    float *extra;
    int64_t zstride;
  };
  __device__ __forceinline__ static void slice(Params &p, int z) {
    if (z > 0) {
      p.x = nullptr;
      p.y = p.extra + (z - 1) * p.zstride;
    }
  }
  __device__ __forceinline__ static void apply(const Params &p, const f32x16_t &acc, int r0, int j0, int lane, int R,
                                               int B) {
    for_rows4(acc, r0, j0, lane, R, B, [&](int row0, int j, f32x4_t c) EE_ALWAYS_INLINE {
      const int64_t o = static_cast<int64_t>(j) * p.ld + row0;
      dstore4<float>(p.y + o, p.x != nullptr ? c + dload4<T>(p.x + o) : c);
    });
  }
};

// Softmax partials of the output-matrix product over 32 rows (vocabulary
// ids), per token: m = max, arg = lowest id reaching m, l = sum exp(S - m).
// Stored at [32-row tile][token].
struct DecLogits {
  static constexpr bool kSplit = false;
  struct Params {
    float *part_m;
    float *part_l;
    int32_t *part_arg;
    int ld;  // tokens per partial row (B)
  };
  __device__ __forceinline__ static void apply(const Params &p, const f32x16_t &acc, int r0, int j0, int lane, int R,
                                               int B) {
    float m = -INFINITY;
    int arg = r0;  // a valid id even if no logit compares (NaN)
    static_for<16>([&](auto v) EE_ALWAYS_INLINE {
      constexpr int Vv = decltype(v)::value;
      const int row = dec_row(r0, lane, Vv);
      const float s = acc[Vv];
      if (row < R && (s > m || (s == m && row < arg))) {
        m = s;
        arg = row;
      }
    });
    const float om = __shfl_xor(m, 32);
    const int oa = __shfl_xor(arg, 32);
    if (om > m || (om == m && oa < arg)) {
      m = om;
      arg = oa;
    }
    float l = 0.0f;
    static_for<16>([&](auto v) EE_ALWAYS_INLINE {
      constexpr int Vv = decltype(v)::value;
      if (dec_row(r0, lane, Vv) < R) l += __expf(acc[Vv] - m);
    });
    l += __shfl_xor(l, 32);
    const int j = j0 + lane;
    if (lane < 32 && j < B) {
      const int64_t o = static_cast<int64_t>(r0 / kDecRows) * p.ld + j;
      p.part_m[o] = m;
      p.part_l[o] = l;
      p.part_arg[o] = arg;
    }
  }
};

// One block of 256 threads per token: combine the tiles' partials.  Each
// thread scans every 256th tile, then the waves combine by shuffles and the
// four waves through LDS (two barriers per reduction).
__device__ __forceinline__ void argmax_merge(float &m, int &t, float om, int ot) {
  // the larger maximum, the lower tile on a tie; a thread that saw no tile
  // (t < 0) takes any other, and a NaN never displaces a tile already seen
  if (ot >= 0 && (t < 0 || om > m || (om == m && ot < t))) {
    m = om;
    t = ot;
  }
}

constexpr int kDecideTiles = 8;  // tiles a thread keeps: every load is issued at once

__global__ __launch_bounds__(256) void decide_kernel(const float *part_m, const float *part_l,
                                                     const int32_t *part_arg, int tiles, int B, float threshold,
                                                     int32_t *token, float *confidence, int32_t *exit_flag) {
  __shared__ float sm[4];
  __shared__ int st[4];
  __shared__ float sl[4];
  __shared__ int sa[4];
  const int j = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // max over tiles, and the lowest tile reaching it; the first tile a thread
  // sees is always taken, so the result is a valid tile even when no maximum
  // compares (NaN)
  float m = -INFINITY;
  int t_best = -1, arg = 0;
  const bool kept = tiles <= kDecideTiles * 256;
  float pm[kDecideTiles], pl[kDecideTiles];
  int pa[kDecideTiles];
  if (kept) {
#pragma unroll
    for (int q = 0; q < kDecideTiles; ++q) {
      const int64_t o = static_cast<int64_t>(min(tid + 256 * q, tiles - 1)) * B + j;
      pm[q] = part_m[o];
      pl[q] = part_l[o];
      pa[q] = part_arg[o];
    }
#pragma unroll
    for (int q = 0; q < kDecideTiles; ++q) {
      const int t = tid + 256 * q;
      if (t < tiles && (t_best < 0 || pm[q] > m)) {  // t increases, so the first tile reaching the maximum is kept
        m = pm[q];
        t_best = t;
        arg = pa[q];
      }
    }
  } else {
    for (int t = tid; t < tiles; t += 256) {
      const float v = part_m[static_cast<int64_t>(t) * B + j];
      if (t_best < 0 || v > m) {
        m = v;
        t_best = t;
      }
    }
  }
  const int mine = t_best;
  for (int o = 1; o < 64; o <<= 1) argmax_merge(m, t_best, __shfl_xor(m, o), __shfl_xor(t_best, o));
  if (mine >= 0 && mine == t_best) {  // one thread of the wave
    if (!kept) arg = part_arg[static_cast<int64_t>(mine) * B + j];
    sa[wave] = arg;
  }
  if (lane == 0) {
    sm[wave] = m;
    st[wave] = t_best;
  }
  __syncthreads();
  float mx = sm[0];
  int tb = st[0];
  for (int w = 1; w < 4; ++w) argmax_merge(mx, tb, sm[w], st[w]);
  float l = 0.0f;
  if (kept) {
#pragma unroll
    for (int q = 0; q < kDecideTiles; ++q)
      if (tid + 256 * q < tiles) l += pl[q] * __expf(pm[q] - mx);
  } else {
    for (int t = tid; t < tiles; t += 256) {
      const int64_t o = static_cast<int64_t>(t) * B + j;
      l += part_l[o] * __expf(part_m[o] - mx);
    }
  }
  l = warp_sum(l);
  if (lane == 0) sl[wave] = l;
  __syncthreads();
  if (tid == 0) {
    const float conf = 1.0f / ((sl[0] + sl[1]) + (sl[2] + sl[3]));
    token[j] = sa[tb % 256 / 64];  // the tile's thread is tile mod 256
    confidence[j] = conf;
    exit_flag[j] = conf > threshold ? 1 : 0;
  }
}

// Gate and up projections as one product (W's rows interleaved in blocks of
// 32; bf16): A[j][r] = silu(Hg[j][r]) * Hu[j][r], Hg rounded to bf16 first.
struct DecGateUp {
  static constexpr bool kSplit = false;
  struct Params {
    bf16_t *act;
    int64_t ld;
  };
  __device__ __forceinline__ static void apply(const Params &p, const f32x16_t &hg, const f32x16_t &hu, int r0, int j0,
                                               int lane, int R, int B) {
    const int j = j0 + (lane & 31);
    if (j >= B) return;
    static_for<4>([&](auto q) EE_ALWAYS_INLINE {
      constexpr int Q = decltype(q)::value;
      const int row0 = dec_row(r0, lane, 4 * Q);
      if (row0 >= R) return;
      f32x4_t a;
      static_for<4>([&](auto e) EE_ALWAYS_INLINE {
        constexpr int E = decltype(e)::value;
        a[E] = silu_f(to_f32(from_f32<bf16_t>(hg[4 * Q + E]))) * hu[4 * Q + E];
      });
      dstore4<bf16_t>(p.act + static_cast<int64_t>(j) * p.ld + row0, a);
    });
  }
};

// bf16: the products from LDS.  A block takes BM
// rows of W (PAIR: BM / 2 of each matrix) and BN tokens through the ring of
// ring.h; blocks of one row tile and several token groups are neighbours on
// one XCD, so W comes from memory once.  blockIdx.y: split-K slice; blockIdx.z:
// token groups past the first `groups`.
template <class Epi, int BM, int BN, int WN, int NS, int Q, bool PAIR, int SEQ>
__global__ __launch_bounds__(BM / 64 * (BN / WN) * 64) void ring_kernel(Operand W, int R, Operand Z, int B, int K,
                                                                        int kchunk, int groups,
                                                                        typename Epi::Params ep) {
  using Rg = Ring<BM, BN, 64, WN, NS, true, true, PAIR, false, Q, SEQ>;
  __shared__ __attribute__((aligned(16))) char smem[NS * Rg::STAGE_BYTES];
  const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  const int tile = (idx / groups) * 8 + xcd, rows = PAIR ? 2 * R : R;
  const int j0 = (static_cast<int>(blockIdx.z) * groups + idx % groups) * BN;
  if (tile * BM >= rows || j0 >= B) return;
  const int kbeg = blockIdx.y * kchunk;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  f32x4_t acc[4][WN / 16];
  Rg::run(W, tile * BM, rows, Z, j0, B, kbeg, min(kchunk, K - kbeg), tid, smem, acc);
  if constexpr (Epi::kSplit) Epi::slice(ep, blockIdx.y);
  f32x16_t blk[2][WN / 32];
  to_blocks32<2, WN / 32>(acc, blk);
  const int r0 = tile * BM + (wave / Rg::WAVES_N) * 64, t0 = j0 + (wave % Rg::WAVES_N) * WN;
  static_for<WN / 32>([&](auto j) EE_ALWAYS_INLINE {
    constexpr int J = decltype(j)::value;
    if constexpr (PAIR) {
      Epi::apply(ep, blk[0][J], blk[1][J], r0 / 2, t0 + 32 * J, lane, R, B);
    } else {
      static_for<2>([&](auto i) EE_ALWAYS_INLINE {
        constexpr int I = decltype(i)::value;
        if (r0 + 32 * I < R) Epi::apply(ep, blk[I][J], r0 + 32 * I, t0 + 32 * J, lane, R, B);
      });
    }
  });
}

template <class Epi, int BM, int BN, int WN, int NS, int Q, bool PAIR, int SEQ = 1>
hipError_t launch_ring_cfg(Operand W, int R, Operand Z, int B, int K, int splits, const typename Epi::Params &ep,
                           hipStream_t stream) {
  const int rows = PAIR ? 2 * R : R;
  const int tiles = (rows + BM - 1) / BM, all = (B + BN - 1) / BN, groups = std::min(all, 64);
  const int kchunk = ((K / 64 + splits - 1) / splits) * 64;
  hipLaunchKernelGGL((ring_kernel<Epi, BM, BN, WN, NS, Q, PAIR, SEQ>),
                     dim3(static_cast<unsigned>((tiles + 7) / 8 * 8 * groups), static_cast<unsigned>(splits),
                          static_cast<unsigned>((all + groups - 1) / groups)),
                     dim3(BM / 64 * (BN / WN) * 64), 0, stream, W, R, Z, B, K, kchunk, groups, ep);
  return hipGetLastError();
}

// Shapes, from us per call of the whole decision (7B Norm exit: h 4096, V 32000;
// 70B: h 8192; 13B MLP: h 5120, I 13824; the former path, K split over the
// waves of a block and 32 tokens a pass, in brackets):
//   8 tokens: 7B 61 (62), 70B 111 (119), 13B MLP 162 (203);
//   64 tokens: 7B 63 (135), 70B 110 (267), 13B MLP 180 (473);
//   230 tokens: 7B 100 (448), 70B 177 (967), 13B MLP 306 (1439).
// W's rows come 128 a block, and the tokens in groups of 32, 64 or, past 64
// tokens, 128.  Two blocks share a CU (4 x 20, 3 x 24 or 2 x 32 KB of LDS)
// except where 128-token blocks are at most one per CU, which take 4 stages (70
// against 92 us for 7B at 128 tokens; at 230 tokens, two a CU, 100 against 110).
// Rows a multiple of 8 KB apart are taken in parts (see Ring: 70B at 32 tokens
// 140 -> 111 us, 7B 74 -> 62; h 1024, 2048 and 5120 gain nothing), where the
// registers allow it.  A narrow product (the down projection) is split over K
// and takes 64 rows a block (13B MLP at 64 tokens: 248 us unsplit, 189 split,
// 180 with 64 rows) as long as 128-row blocks would leave half of the CUs idle
// (us a call, V 8000 or 32000, 64 rows against 128: h 5120, I 13824, 120 blocks of
// 128, 64 tokens 180/190; h 8192, I 22016, 128 blocks, 100 tokens 378/396; h 6144,
// I 16384, 144 blocks, 100 tokens 298/261; h 8192, 192 blocks, 100 tokens 434/395).
constexpr int kCampBytes = 8192;
template <class Epi, bool PAIR>
hipError_t launch_ring(Operand W, int R, Operand Z, int B, int K, int splits, const typename Epi::Params &ep,
                       hipStream_t stream, bool exact = false) {
  if (R <= 0 || B <= 0) return hipSuccess;
  if (K % 64 != 0) return hipErrorInvalidValue;
  const bool camp = W.ld * 2 % kCampBytes == 0 && splits == 1;
  const int64_t blocks = (static_cast<int64_t>(PAIR ? 2 * R : R) + 127) / 128 * ((B + 127) / 128) * splits;
  if constexpr (Epi::kSplit) {
    if (B <= 128 && blocks <= 136) {
      if (B <= 32) return launch_ring_cfg<Epi, 64, 32, 32, 4, 1, PAIR>(W, R, Z, B, K, splits, ep, stream);
      if (B <= 64) return launch_ring_cfg<Epi, 64, 64, 32, 4, 1, PAIR>(W, R, Z, B, K, splits, ep, stream);
      return launch_ring_cfg<Epi, 64, 128, 64, 4, 1, PAIR>(W, R, Z, B, K, splits, ep, stream);
    }
  }
  if constexpr (std::is_same<Epi, DecLogits>::value) {
    // Sums as short as the parts of camping rows give, so that the error against
    // 64 bits is that of K shared by skinny_kernel's waves (confidences: h 5120, V
    // 20000, 128 tokens 8.3e-7 in one sum, 2.1e-7 in parts and in skinny_kernel; h
    // 2048, V 32000, 400 tokens 5.2e-7, 2.0e-7, 1.8e-7), for up to 8% more time.
    if (exact && K > 512 && !(camp && (B <= 64 || blocks <= 256))) {
      if (B <= 32) return launch_ring_cfg<Epi, 128, 32, 32, 4, 1, PAIR, 8>(W, R, Z, B, K, splits, ep, stream);
      if (B <= 64) return launch_ring_cfg<Epi, 128, 64, 32, 3, 1, PAIR, 8>(W, R, Z, B, K, splits, ep, stream);
      if (blocks > 256) return launch_ring_cfg<Epi, 128, 128, 64, 2, 1, PAIR, 8>(W, R, Z, B, K, splits, ep, stream);
      return launch_ring_cfg<Epi, 128, 128, 64, 4, 1, PAIR, 8>(W, R, Z, B, K, splits, ep, stream);
    }
  }
  if (B <= 32) {
    if (camp) return launch_ring_cfg<Epi, 128, 32, 32, 4, 8, PAIR>(W, R, Z, B, K, splits, ep, stream);
    return launch_ring_cfg<Epi, 128, 32, 32, 4, 1, PAIR>(W, R, Z, B, K, splits, ep, stream);
  }
  if (B <= 64) {
    if (camp) return launch_ring_cfg<Epi, 128, 64, 32, 3, 8, PAIR>(W, R, Z, B, K, splits, ep, stream);
    return launch_ring_cfg<Epi, 128, 64, 32, 3, 1, PAIR>(W, R, Z, B, K, splits, ep, stream);
  }
  if (blocks > 256) return launch_ring_cfg<Epi, 128, 128, 64, 2, 1, PAIR>(W, R, Z, B, K, splits, ep, stream);
  if (camp) return launch_ring_cfg<Epi, 128, 128, 64, 4, 4, PAIR>(W, R, Z, B, K, splits, ep, stream);
  return launch_ring_cfg<Epi, 128, 128, 64, 4, 1, PAIR>(W, R, Z, B, K, splits, ep, stream);
}

template <typename T, class Epi, int RG>
hipError_t launch_skinny_rg(const T *w, int64_t ldw, int R, const T *z, int64_t ldz, int B, int K,
                            const typename Epi::Params &ep, hipStream_t stream) {
  const int row_blocks = (R + kDecRows * RG - 1) / (kDecRows * RG);
  const dim3 grid(static_cast<unsigned>(row_blocks), static_cast<unsigned>((B + kDecTokens - 1) / kDecTokens));
  // 16 waves of 1024 threads leave 128 registers a lane: too few for two row groups
  const int waves = RG > 1 ? std::min(dec_waves(row_blocks), 8) : dec_waves(row_blocks);
  switch (waves) {
    case 4:
      hipLaunchKernelGGL((skinny_kernel<T, Epi, 4, RG>), grid, dim3(64 * 4), 0, stream, w, ldw, R, z, ldz, B, K, ep);
      break;
    case 8:
      hipLaunchKernelGGL((skinny_kernel<T, Epi, 8, RG>), grid, dim3(64 * 8), 0, stream, w, ldw, R, z, ldz, B, K, ep);
      break;
    default:
      if constexpr (RG == 1)
        hipLaunchKernelGGL((skinny_kernel<T, Epi, kDecWavesMax, RG>), grid, dim3(64 * kDecWavesMax), 0, stream, w, ldw,
                           R, z, ldz, B, K, ep);
  }
  return hipGetLastError();
}

// Past 8 token rows, a wide W (at least 12288 rows) is read by blocks of two
// 32-row groups per token fragment, halving the token rows' share of the
// loads (at 8 waves a block: measured 11% faster at 32 tokens for 13824 and
// 32000 rows; with 5120 rows the 80 blocks kept too few loads in flight).
template <typename T, class Epi>
hipError_t launch_skinny(const void *W, int64_t ldw, int R, const void *Z, int64_t ldz, int B, int K,
                         const typename Epi::Params &ep, hipStream_t stream) {
  if (R <= 0 || B <= 0) return hipSuccess;
  if (K % (4 * DecFrag<T>::K_PER_LOAD) != 0) return hipErrorInvalidValue;
  const T *w = static_cast<const T *>(W);
  const T *z = static_cast<const T *>(Z);
  if (B > 8 && R >= 12288) return launch_skinny_rg<T, Epi, 2>(w, ldw, R, z, ldz, B, K, ep, stream);
  return launch_skinny_rg<T, Epi, 1>(w, ldw, R, z, ldz, B, K, ep, stream);
}

}  // namespace

// Which bf16 products skinny_kernel takes.  It has 32 rows of W a block and up
// to 16 waves that share K, where a block of the ring has 128 rows (64 for
// the split down projection) and two or four waves that walk all of K: few
// rows of W leave the ring a latency chain on a few CUs.  But skinny_kernel
// reads W once for every 32 tokens, so it loses past one round of 16 waves a
// CU (two rounds past 64 tokens, where the ring has a 128-token block).  us a
// call, ring against skinny, W from memory (Embedding exit, h 4096):
//   1 token: V 2000 36.5 against 17.1, 8192 36.8/20.1, 16384 38.3/29.7, 24000
//   42.9/41.7;
//   32 tokens: 2000 37.8/24.7, 8192 38.9/26.1, 10000 39.1/40.0, 20000 45.6/71.2;
//   64 tokens: 4096 39.9/25.6, 6000 40.6/42.7 (48 tokens 40.0/38.9, and with h
//   2048 23.7/24.6); 128: 4096 53.2/42.4, 6000 54.1/61.0; 256: 2000 52.8/42.8,
//   3000 53.2/59.8; 96 tokens, V 8192: 53.9/53.5, h 1024 22.4/20.0.
// Past a block a CU (8192 rows) it depends on the tokens' share of the loads (h
// 5120, V 10000: 16 tokens 44.0/44.6, 32 46.3/54.3), on the stride of the rows (a
// multiple of 8 KB, or of 4 KB with long rows, favours waves spread over K: 24
// tokens, V 14000, h 4096 39.9/38.7, h 5120 47.4/49.2; the ring takes no parts at
// an odd multiple of 4 KB: h 2048, V 48000, 8 tokens 51.1/45.4) and on whether the
// ring's 128-row blocks are a few more than the CUs, so that some CUs take two
// (h 4096, 1 token, ring time over skinny's: V 28000 0.95, 33000 1.16, 38111
// 1.17, 48000 1.06, 58000 0.97; 8 tokens 0.88, 1.13, 1.11, 1.02, 0.91).
constexpr int kWavesRound = 16 * 256;  // 16 waves a CU
bool decode_skinny_logits(int rows, int n, int k) {
  const int64_t rb = cdiv64(rows, kDecRows), passes = cdiv64(n, kDecTokens), waves = rb * passes * dec_waves(rb);
  if (n > 64) return rb < 256 ? waves <= 2 * kWavesRound : (k <= 2048 && 2 * waves <= 3 * kWavesRound);
  if (n > 32) return (n <= 48 && k >= 4096 && rb <= 192) || (rb <= 256 && waves <= kWavesRound);
  if (rb <= 256 || (rb < 384 && n <= 16)) return true;
  const int stride = k * 2;
  if (rb <= 512) return n <= 8 || (n <= 24 && k >= 4096 && stride % 4096 == 0);
  if (n > 8) return false;
  if (k <= 512 || stride % kCampBytes == kCampBytes / 2 || (n <= 4 && k <= 1536)) return true;
  return rb > 1024 && (rb <= 1216 || (rb <= 1536 && n <= 4 && k < 8192));
}
// The ring splits K here and keeps up except where K is short (us a call of the
// whole MLP exit, V 8000, ring against skinny: h 512, I 1344: 1 token 31/30, 250
// tokens 49/43; h = I = 4096: 1 token 92/89; h 2048, I 5504: 1 token 58/59) and,
// past 64 tokens, skinny_kernel takes one round (h = I = 2048: 128 tokens 77/73,
// 250 tokens 80/83).  From 9 to 64 tokens the two are within 2 us.
bool decode_skinny_down(int rows, int n, int k) {
  const bool short_k = 4 * static_cast<int64_t>(k) <= 11 * static_cast<int64_t>(rows);
  if (n <= 8) return k <= rows || (rows <= 512 && short_k);
  const int64_t rb = cdiv64(rows, kDecRows), passes = cdiv64(n, kDecTokens);
  return n > 64 && (k <= rows || (rows <= 1024 && short_k)) && rb * passes * dec_waves(rb) <= kWavesRound;
}

int decode_tiles(int rows) { return (rows + kDecRows - 1) / kDecRows; }

hipError_t decode_gate_up(bool f32, const void *w_gate, const void *w_up, int rows, const void *z, int n, int k,
                          void *hg, void *act, hipStream_t stream) {
  if (!f32) {
    const int64_t pair = static_cast<const char *>(w_up) - static_cast<const char *>(w_gate);
    return launch_ring<DecGateUp, true>(Operand{w_gate, k, pair}, rows, Operand{z, k}, n, k, 1,
                                        {static_cast<bf16_t *>(act), rows}, stream);
  }
  const hipError_t e =
      launch_skinny<float, DecStore>(w_gate, k, rows, z, k, n, k, {static_cast<float *>(hg), rows}, stream);
  if (e != hipSuccess) return e;
  return launch_skinny<float, DecSwiGLU>(w_up, k, rows, z, k, n, k,
                                         {static_cast<const float *>(hg), static_cast<float *>(act), rows}, stream);
}

// Slices of the down projection's K: enough for two 64-row blocks a CU (two
// 128-row blocks past 128 tokens), at most `most`, and 512 values of K each.  (One
// block a CU: h 5120, I 13824, 400 tokens 351 -> 375 us a call, h 4096, I 11008,
// 500 tokens 272 -> 255; three or four: the same within 1%, h 8192, I 22016, 400
// tokens 873 -> 915.)
int decode_residual_splits(bool f32, int rows, int n, int k, int most) {
  if (f32 || decode_skinny_down(rows, n, k)) return 1;
  const int64_t bm = n <= 128 ? 64 : 128, blocks = (rows + bm - 1) / bm * ((n + 127) / 128);
  const int s = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>({most, 512 / blocks, k / 512})));
  return cdiv64(k / 64, cdiv64(k / 64, s));  // slices of whole stages, none empty
}

hipError_t decode_residual(bool f32, const void *w, int rows, const void *z, int n, int k, const void *x,
                           float *y, int splits, float *extra, hipStream_t stream) {
  const bool skinny = f32 || decode_skinny_down(rows, n, k);
  if (splits < 1 || (splits > 1 && (skinny || extra == nullptr))) return hipErrorInvalidValue;
  if (skinny)
    EE_DISPATCH(f32, return (launch_skinny<T, DecResidual<T>>(w, k, rows, z, k, n, k,
                                                              {static_cast<const T *>(x), y, rows, nullptr, 0}, stream)));
  return launch_ring<DecResidual<bf16_t>, false>(
      Operand{w, k}, rows, Operand{z, k}, n, k, splits,
      {static_cast<const bf16_t *>(x), y, rows, extra, static_cast<int64_t>(n) * rows}, stream);
}

hipError_t decode_logits(bool f32, const void *w_out, int vocab, const void *z, int n, int h, float *part_m,
                         float *part_l, int32_t *part_arg, hipStream_t stream, bool exact) {
  const DecLogits::Params ep{part_m, part_l, part_arg, n};
  if (f32 || decode_skinny_logits(vocab, n, h))
    EE_DISPATCH(f32, return (launch_skinny<T, DecLogits>(w_out, h, vocab, z, h, n, h, ep, stream)));
  return launch_ring<DecLogits, false>(Operand{w_out, h}, vocab, Operand{z, h}, n, h, 1, ep, stream, exact);
}

hipError_t decode_decide(const float *part_m, const float *part_l, const int32_t *part_arg, int tiles, int n,
                         float threshold, int32_t *token, float *confidence, int32_t *exit_flag,
                         hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(decide_kernel, dim3(static_cast<unsigned>(n)), dim3(256), 0, stream, part_m, part_l, part_arg,
                     tiles, n, threshold, token, confidence, exit_flag);
  return hipGetLastError();
}

}  // namespace ee
