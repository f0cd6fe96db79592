// Tiled MFMA GEMM for gfx950 with fused epilogues.
//
//   C[m][n] = sum_k A(m, k) * B(n, k)
//
// Each operand is either K-major (element (r, k) at ptr[r*ld + k], K
// contiguous) or MN-major (element (r, k) at ptr[k*ld + r], rows
// contiguous).  Operand tiles go from memory straight into LDS
// (global_load_lds_dwordx4), as they are: K-major tiles as rows of K, MN-major
// tiles as k-rows, which bf16 fragment reads transpose (ds_read_b64_tr_b16), so
// neither side spends ALU work or registers on the way.
//
// bf16 products (v_mfma_f32_16x16x32_bf16) run a 256 x 256 tile on 8 wave64
// waves of 128 x 64, the two waves of a SIMD taking turns, one in its MFMAs
// while the other reads its fragments; where few such tiles exist, a 128 x 128
// tile on 4 waves of 64 x 64 with a ring of stages (ring.h).  fp32 products
// (v_mfma_f32_32x32x2_f32) run the ring on 128 x 128 or 64 x 64.  All
// accumulate in fp32 and hand their epilogue 32 x 32 blocks (TileCtx).
//
// Blocks are ordered for the L2 of each XCD: the hardware hands block b to
// XCD b % 8, so consecutive logical tiles are given to the same XCD, and
// logical tiles walk GROUP_M tile rows at a time (the concurrent tiles of an
// XCD then share a few A and B panels).
#pragma once

#include <algorithm>

#include "ee_device.h"
#include "launch.h"
#include "ring.h"

namespace ee {

struct GemmShape {
  int M, N, K;
  int kchunk = 0;  // split-K: blockIdx.z covers K values [z kchunk, (z + 1) kchunk); 0 = all of K
  int parts = 1;   // fp32, 128 x 128 tiles: K is summed in this many parts (see RingF32)
};

constexpr int kRowBytes = 128;
constexpr int kNumXcd = 8;
constexpr int kGroupM = 4;
constexpr int kLoopBlocks = 256;  // grid of the looping kernels: one block per CU of a 256-CU GPU (a multiple of kNumXcd)

template <int BM_, int BN_, int WM_, int WN_, int MIN_BLOCKS_, int STAGES_ = 2, int KW_ = 1>
struct TileCfg {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int MIN_BLOCKS = MIN_BLOCKS_;  // workgroups per CU the registers must allow
  static constexpr int WAVES_M = BM / WM, WAVES_N = BN / WN;
  static constexpr int THREADS = WAVES_M * WAVES_N * 64;
  static constexpr int KW = KW_;                 // waves that share a wave's tile, each a part of K (fp32)
  static constexpr int BLOCK = THREADS * KW;     // threads of a workgroup
  static constexpr int MB = WM / 32, NB = WN / 32;
  static constexpr int STAGE_BYTES = (BM + BN) * kRowBytes;
  static constexpr int STAGES = STAGES_;  // LDS stages
  static constexpr int SMEM_BYTES = STAGES * STAGE_BYTES;
};
// 256 x 256 tile, 8 waves of 128 x 64 (two waves per SIMD), for bf16 products
// with enough of them: 1.5x the MFMA work per byte read from LDS of the small
// tile, and a second wave per SIMD to issue while the other waits.
using CfgBig = TileCfg<256, 256, 128, 64, 1>;
// 128 x 128 tile, 64 x 64 per wave, a ring of 2 stages: bf16 products with too
// few 256 x 256 tiles to fill the chip.
using CfgMid = TileCfg<128, 128, 64, 64, 2, 2>;
// fp32: 128 x 128 on 4 waves of 64 x 64, or 64 x 64 on 4 waves that share K.
using CfgF32 = TileCfg<128, 128, 64, 64, 2, 2>;
using CfgF32Small = TileCfg<64, 64, 64, 64, 2, 4, 4>;

template <typename T> struct Elem;
template <> struct Elem<bf16_t> {
  static constexpr int CH = 8;  // elements per 16-byte chunk
};
template <> struct Elem<float> {
  static constexpr int CH = 4;
};

__host__ __device__ constexpr int cdiv(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

// Epilogues that take the B operand as an interleaved pair declare
// kPairB = true.
template <class E, class = void> struct EpiPairB : std::false_type {};
template <class E> struct EpiPairB<E, std::void_t<decltype(E::kPairB)>> : std::bool_constant<E::kPairB> {};
// Epilogues whose GEMMs run as one block per CU looping over the tiles.
template <class E, class = void> struct EpiPersistent : std::false_type {};
template <class E>
struct EpiPersistent<E, std::void_t<decltype(E::kPersistent)>> : std::bool_constant<E::kPersistent> {};

// Barriers an epilogue passes (kBarriers; waves without a tile of their own
// pass them too).
template <class E, class = void> struct EpiBarriers : std::integral_constant<int, 0> {};
template <class E>
struct EpiBarriers<E, std::void_t<decltype(E::kBarriers)>> : std::integral_constant<int, E::kBarriers> {};

// Position of accumulator element (i, j, v) of a lane:
//   row = m0 + wave_m*WM + i*32 + (v/4)*8 + (lane/32)*4 + v%4
//   col = n0 + wave_n*WN + j*32 + lane%32
template <class Cfg>
struct TileCtx {
  static constexpr int MB = Cfg::MB, NB = Cfg::NB;
  int M, N;            // problem bounds of C
  int m0, n0;          // tile origin
  int tile_m, tile_n;  // tile indices
  int wave_m, wave_n, lane;
  char *smem;          // the tile's LDS (two stages), free for the epilogue after a barrier
  int kz = 0;          // split-K slice of this block (epilogues that support splits offset by it)

  __device__ __forceinline__ int row(int i, int v) const {
    return m0 + wave_m * Cfg::WM + i * 32 + (v >> 2) * 8 + (lane >> 5) * 4 + (v & 3);
  }
  __device__ __forceinline__ int col(int j) const { return n0 + tcol(j); }
  // column index inside the tile
  __device__ __forceinline__ int tcol(int j) const { return wave_n * Cfg::WN + j * 32 + (lane & 31); }
};

// Logical tile of this block (XCD-aware, grouped order).  Blocks that run
// together on one XCD take consecutive logical tiles; the logical order
// walks groups of kGroupM tiles along the dimension with more tiles, sweeping
// the other dimension inside a group, so the operand with more panels is
// streamed once while the few panels of the other stay cache-resident.
__device__ __forceinline__ void tile_of_block(int b, int nblk, int tiles_m, int tiles_n, int &tile_m, int &tile_n) {
  const int per = nblk / kNumXcd, rem = nblk % kNumXcd;
  const int xcd = b % kNumXcd, idx = b / kNumXcd;
  const int logical = xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
  const bool swap = tiles_n > tiles_m;
  const int ta = swap ? tiles_n : tiles_m, tb = swap ? tiles_m : tiles_n;  // grouped, swept
  const int in_group = kGroupM * tb;
  const int first = (logical / in_group) * kGroupM;
  const int g = min(ta - first, kGroupM);
  const int r = logical % in_group;
  const int a = first + r % g, c = r / g;
  tile_m = swap ? c : a;
  tile_n = swap ? a : c;
}

// ----------------------------------------------------------------- kernel
// Block b of nblk (b mod 8 = the XCD it runs on) of one GEMM problem, split-K
// slice kz: main loop and epilogue of its tile.  LOOP: the caller loops over
// tiles; the thread index is then opaque to the compiler, so that no address
// it derives is hoisted out of the loop and kept live through the epilogue
// (which spilled registers).
template <typename T, bool AK, bool BKM, class Epi, class Cfg, bool LOOP>
struct GemmBlock;

// fp32.
template <bool AK, bool BKM, class Epi, class Cfg, bool LOOP>
struct GemmBlock<float, AK, BKM, Epi, Cfg, LOOP> {
  static __device__ __forceinline__ void run(const Operand &A, const Operand &B, const GemmShape &s,
                                             const typename Epi::Params &ep, int b, int nblk, int kz, char *smem) {
    using R = RingF32<Cfg::BM, Cfg::BN, Cfg::KW, Cfg::STAGES, AK, BKM, EpiPairB<Epi>::value>;
    static_assert(R::THREADS == Cfg::BLOCK && (!LOOP || Cfg::KW == 1), "waves of 64 x 64");
    int tid_v = threadIdx.x;
    if constexpr (LOOP) asm volatile("" : "+v"(tid_v));
    const int tid = tid_v, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tile_m, tile_n;
    tile_of_block(b, nblk, cdiv(s.M, Cfg::BM), cdiv(s.N, Cfg::BN), tile_m, tile_n);
    const int m0 = tile_m * Cfg::BM, n0 = tile_n * Cfg::BN;
    const int kbeg = s.kchunk > 0 ? kz * s.kchunk : 0;
    const int K = (s.kchunk > 0 ? min(s.K, kbeg + s.kchunk) : s.K) - kbeg;
    f32x16_t acc[2][2];
    R::run(A, m0, s.M, B, n0, s.N, kbeg, K, s.parts, tid, smem, acc);
    if (Cfg::KW > 1 && wave > 0) {  // the first wave holds the tile
      static_for<EpiBarriers<Epi>::value>([&](auto) EE_ALWAYS_INLINE { __syncthreads(); });
      return;
    }
    const int w = Cfg::KW > 1 ? 0 : wave;
    TileCtx<Cfg> ctx{s.M, s.N, m0, n0, tile_m, tile_n, w / Cfg::WAVES_N, w % Cfg::WAVES_N, lane, smem, kz};
    Epi::template apply<Cfg>(ep, acc, ctx);
  }
};

// ------------------------------------------------------------ bf16 main loop
// One operand of a 256-row tile, in two halves of 128 rows.  Half q holds,
// for each wave that owns rows of this operand, the wave's 16-row blocks q *
// WR / 2 .. : WR rows a wave (128 for A, 64 for B), WR / 2 of them per half.
//
// K-major: a half is 128 LDS rows of 64 values of K (128 bytes), 16-byte
// chunk c of row r at chunk c ^ ((r / 2) mod 8): 16 lanes of a fragment read, served
// at a time from 256 bytes of banks (two LDS rows), read one chunk of 16
// consecutive rows, and the XOR puts rows of equal parity on distinct chunks.  The load writes LDS linearly, so the XOR is applied to the address a lane
// reads from; it stays inside the row's 128-byte line.
// MN-major: a half is 64 LDS k-rows of 128 operand rows (256 bytes), chunk c of
// k-row k at c ^ (2 (k mod 4) + 8 (k / 8 mod 2)).  ds_read_b64_tr_b16 gives lane
// 4 a + b of each 16-lane group element b of the 8-byte pieces that lanes a,
// a + 4, a + 8, a + 12 of the group address, so lane j of group g addresses
// k-row 8 g + j / 4 (+ 4 for the second read) at 4 rows and receives row j at
// 8 consecutive k; the XOR spreads the 8 k-rows of two groups over all banks.
template <bool KM, int WR, bool PERM, bool PAIR>
struct TileOperandB16 {
  static constexpr int BLK = WR / 2 / 16;  // 16-row blocks per half
  uint32_t off[PAIR ? 1 : 2][2];           // byte offsets of this thread's two chunks of each half
  uint32_t ld2, kr;                        // MN-major: bytes per k-row; k-row of the thread's first chunk
  const char *rd[KM ? 2 : BLK];            // fragment addresses of stage 0, half 0: K-major per 32 values of K; else per block
  const char *base;
  int64_t pair, step;

  __device__ __forceinline__ static int tile_row(int q, int lr) { return (lr / (WR / 2)) * WR + q * (WR / 2) + lr % (WR / 2); }

  // row0: first tile row, rows: rows of the operand (PAIR: of both matrices);
  // wave: which WR rows of the tile the wave owns; lds: LDS of stage 0.
  __device__ __forceinline__ void init(const Operand &O, int row0, int rows, int kbeg, int tid, int wave, int lane,
                                       const char *lds) {
    const bf16_t *p = static_cast<const bf16_t *>(O.ptr);
    ld2 = static_cast<uint32_t>(O.ld * 2);
    pair = O.pair;
    const int r0 = PAIR ? row0 / 2 : row0, nrows = PAIR ? rows / 2 : rows;
    if constexpr (KM) {
      base = reinterpret_cast<const char *>(p + static_cast<int64_t>(r0) * O.ld + kbeg);
      step = 128;
      static_for<2>([&](auto e) EE_ALWAYS_INLINE {
        const int c = decltype(e)::value * 512 + tid, lr = c >> 3, ch = (c & 7) ^ ((lr >> 1) & 7);
        static_for<PAIR ? 1 : 2>([&](auto q) EE_ALWAYS_INLINE {
          const int r = PAIR ? lr : tile_row(decltype(q)::value, lr);
          off[q][e] = static_cast<uint32_t>(min(r0 + r, nrows - 1) - r0) * ld2 + ch * 16;
        });
      });
      const int r = PERM ? acc_row(lane & 15) : lane & 15, x = (r >> 1) & 7;
      static_for<2>([&](auto ks) EE_ALWAYS_INLINE {
        rd[ks] = lds + (wave * (WR / 2) + r) * 128 + (((decltype(ks)::value * 4 + (lane >> 4)) ^ x) << 4);
      });
    } else {
      base = reinterpret_cast<const char *>(p + static_cast<int64_t>(kbeg) * O.ld + row0);
      step = static_cast<int64_t>(ld2) * 64;
      kr = tid >> 4;
      static_for<2>([&](auto e) EE_ALWAYS_INLINE {
        const int k = decltype(e)::value * 32 + (tid >> 4), ch = (tid & 15) ^ swz(k);
        static_for<2>([&](auto q) EE_ALWAYS_INLINE {
          off[q][e] = static_cast<uint32_t>(min(row0 + tile_row(decltype(q)::value, ch * 8), rows - 8) - row0) * 2;
        });
      });
      const int k = 8 * (lane >> 4) + ((lane >> 2) & 3), j = lane & 3;
      const int m = PERM ? (j & 1) * 8 + (j >> 1) * 4 : 4 * j;
      static_for<BLK>([&](auto i) EE_ALWAYS_INLINE {
        const int row = wave * (WR / 2) + decltype(i)::value * 16 + m;
        rd[i] = lds + k * 256 + (((row >> 3) ^ swz(k)) << 4) + (row & 7) * 2;
      });
    }
  }
  __device__ __forceinline__ static int swz(int k) { return 2 * (k & 3) + 8 * ((k >> 3) & 1); }

  // Load half Q of stage t (of K values left from this stage on: MN-major
  // k-rows past them re-read the last one).
  template <int Q>
  __device__ __forceinline__ void load(int t, int left, uint32_t lds_wave) const {
    const char *p = base + static_cast<int64_t>(t) * step;
    if constexpr (PAIR) p += Q * pair;
    static_for<2>([&](auto e) EE_ALWAYS_INLINE {
      constexpr int E = decltype(e)::value;
      uint32_t o = off[PAIR ? 0 : Q][E];
      if constexpr (!KM) o += __umul24(min(static_cast<int>(kr) + 32 * E, left - 1), ld2);
      load_lds16(p, o, lds_wave + Q * 16384 + E * 8192);
    });
  }
  // Zero the chunks this thread loads whose k-rows lie past K (MN-major).
  __device__ __forceinline__ void zero_tail(int left, int tid, char *lds) const {
    static_for<2>([&](auto e) EE_ALWAYS_INLINE {
      if (static_cast<int>(kr) + 32 * decltype(e)::value >= left) {
        static_for<2>([&](auto q) EE_ALWAYS_INLINE {
          *reinterpret_cast<u32x4_t *>(lds + decltype(q)::value * 16384 + decltype(e)::value * 8192 + tid * 16) = u32x4_t{0, 0, 0, 0};
        });
      }
    });
  }
  // Fragments of half Q of the stage in buffer BUF, both 32-value K steps.
  template <int BUF, int Q>
  __device__ __forceinline__ void read(bf16x8_t (&f)[BLK][2]) const {
    static_for<BLK>([&](auto i) EE_ALWAYS_INLINE {
      constexpr int I = decltype(i)::value;
      static_for<2>([&](auto ks) EE_ALWAYS_INLINE {
        constexpr int KS = decltype(ks)::value;
        if constexpr (KM) {
          f[I][KS] = *reinterpret_cast<const bf16x8_t *>(rd[KS] + BUF * 65536 + Q * 16384 + I * 2048);
        } else {
          const char *p = rd[I] + BUF * 65536 + Q * 16384 + KS * 8192;
          const s16x4_t both[2] = {__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(p)),
                                   __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(p + 1024))};
          f[I][KS] = __builtin_bit_cast(bf16x8_t, both);
        }
      });
    });
  }
};

// bf16.  The wave's 128 x 64 outputs are 8 x 4 blocks of 16 x 16; a stage is
// four phases, one per quadrant (half of A, half of B), 16 MFMAs each:
//   read the fragments that are new (8, 4, 8 and 4 of them: the last phase
//   reads the next stage's first half of B, so the order of B's halves
//   alternates), start loading the half of two stages ahead whose LDS every
//   wave has read by now, wait for the half that the next phase reads;
//   barrier; MFMAs; barrier.
// Waves 4..7 run one barrier behind waves 0..3 (a SIMD holds one of each),
// so one wave's MFMAs cover the other's reads (in step, the same code takes
// 22% longer); a half is read by waves 0..3 in one interval, by waves 4..7 in
// the next, in which waves 0..3 compute, and overwritten from the one after.
// Six halves (12 loads a thread) stay in flight.
//
// What bounds it is power: with random operands the chip holds its clock
// down, and at its limit 16 x 16 x 32 MFMAs on registers alone run at 2143
// TFLOP/s where 32 x 32 x 16 reach 1867; loads that bypass the registers
// lower it further.  4096 x 32000 x 4096 with nothing stored: 1540 TFLOP/s,
// where 32 x 32 x 16 staged through registers and interleaved MFMA by MFMA
// reached 1340 (12, 4, 8 and no fragment reads a phase: 1525; with a raised
// wave priority around the MFMAs: 1530).
template <bool AK, bool BKM, class Epi, class Cfg, bool LOOP>
struct GemmBlockBig {
  static __device__ __forceinline__ void run(const Operand &A, const Operand &B, const GemmShape &s,
                                             const typename Epi::Params &ep, int b, int nblk, int kz, char *smem) {
    static_assert(Cfg::BM == 256 && Cfg::BN == 256 && Cfg::WM == 128 && Cfg::WN == 64, "8 waves of 128 x 64");
    constexpr bool kPair = EpiPairB<Epi>::value;
    static_assert(!kPair || BKM, "an interleaved pair is read K-major");
    int tid_v = threadIdx.x;
    if constexpr (LOOP) asm volatile("" : "+v"(tid_v));
    const int tid = tid_v, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave / Cfg::WAVES_N, wave_n = wave % Cfg::WAVES_N;
    int tile_m, tile_n;
    tile_of_block(b, nblk, cdiv(s.M, Cfg::BM), cdiv(s.N, Cfg::BN), tile_m, tile_n);
    const int m0 = tile_m * Cfg::BM, n0 = tile_n * Cfg::BN;
    const int kbeg = s.kchunk > 0 ? kz * s.kchunk : 0;
    const int K = (s.kchunk > 0 ? min(s.K, kbeg + s.kchunk) : s.K) - kbeg;
    const int nk = cdiv(K, 64);

    // LDS: per stage the halves A0, A1, B0, B1 of 16 KB.
    constexpr int B_OFF = 32768;
    TileOperandB16<AK, 128, true, false> ta;
    TileOperandB16<BKM, 64, false, kPair> tb;
    ta.init(A, m0, s.M, kbeg, tid, wave_m, lane, smem);
    tb.init(B, n0, s.N, kbeg, tid, wave_n, lane, smem + B_OFF);
    const uint32_t lds_wave =
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char *)smem)) + wave * 1024;
    // Stages past the last re-read it (into halves nobody reads again).
    auto load_a = [&](auto q, auto buf, int t) EE_ALWAYS_INLINE {
      const int u = min(t, nk - 1);
      ta.template load<decltype(q)::value>(u, K - u * 64, lds_wave + decltype(buf)::value * 65536);
    };
    auto load_b = [&](auto q, auto buf, int t) EE_ALWAYS_INLINE {
      const int u = min(t, nk - 1);
      tb.template load<decltype(q)::value>(u, K - u * 64, lds_wave + decltype(buf)::value * 65536 + B_OFF);
    };
    f32x4_t acc[8][4];
    static_for<8>([&](auto i) EE_ALWAYS_INLINE {
      static_for<4>([&](auto j) EE_ALWAYS_INLINE { acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}; });
    });
    bf16x8_t fa[4][2], fb[2][2][2];
    auto mma = [&](auto qa, auto qb) EE_ALWAYS_INLINE {
      static_for<2>([&](auto ks) EE_ALWAYS_INLINE {
        static_for<4>([&](auto i) EE_ALWAYS_INLINE {
          static_for<2>([&](auto j) EE_ALWAYS_INLINE {
            constexpr int I = decltype(qa)::value * 4 + decltype(i)::value, J = decltype(qb)::value * 2 + decltype(j)::value;
            acc[I][J] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i][ks], fb[qb][j][ks], acc[I][J], 0, 0, 0);
          });
        });
      });
    };
    using H0 = std::integral_constant<int, 0>;
    using H1 = std::integral_constant<int, 1>;
    load_b(H0{}, H0{}, 0);
    load_a(H0{}, H0{}, 0);
    load_b(H1{}, H0{}, 0);
    load_a(H1{}, H0{}, 0);
    load_b(H1{}, H1{}, 1);
    load_a(H0{}, H1{}, 1);
    load_b(H0{}, H1{}, 1);
    load_a(H1{}, H1{}, 1);
    wait_vm<12>();  // stage 0's first halves of B and A
    phase_barrier();
    tb.template read<0, 0>(fb[0]);
    wait_lgkm();
    phase_barrier();  // every wave has read the half that the first phase overwrites
    if (wave_m == 1) phase_barrier();  // waves 4..7 run one barrier behind
    auto stage = [&](auto buf, int t) EE_ALWAYS_INLINE {
      constexpr int BUF = decltype(buf)::value;
      using Cur = std::integral_constant<int, BUF>;
      using First = Cur;  // the half of B this stage starts and ends with
      using Second = std::integral_constant<int, BUF ^ 1>;
      if constexpr (!AK) {
        // The last stage of an MN-major product whose K is no multiple of 64:
        // zero A's k-rows past K, each thread the chunks it loaded itself.
        if (t == nk - 1 && K % 64 != 0) {
          wait_vm<0>();
          ta.zero_tail(K - t * 64, tid, smem + BUF * 65536);
          wait_lgkm();
          phase_barrier();
          phase_barrier();
        }
      }
      ta.template read<BUF, 0>(fa);
      load_b(First{}, Cur{}, t + 2);
      wait_vm<12>();
      wait_lgkm();
      phase_barrier();
      mma(H0{}, First{});
      phase_barrier();
      tb.template read<BUF, BUF ^ 1>(fb[BUF ^ 1]);
      load_a(H0{}, Cur{}, t + 2);
      wait_vm<12>();
      wait_lgkm();
      phase_barrier();
      mma(H0{}, Second{});
      phase_barrier();
      ta.template read<BUF, 1>(fa);
      load_b(Second{}, Cur{}, t + 2);
      wait_vm<12>();
      wait_lgkm();
      phase_barrier();
      mma(H1{}, Second{});
      phase_barrier();
      tb.template read<BUF ^ 1, BUF ^ 1>(fb[BUF ^ 1]);
      load_a(H1{}, Cur{}, t + 2);
      wait_vm<12>();
      wait_lgkm();
      phase_barrier();
      mma(H1{}, First{});
      phase_barrier();
    };
    int t = 0;
    for (; t + 1 < nk; t += 2) {
      stage(H0{}, t);
      stage(H1{}, t + 1);
    }
    if (t < nk) stage(H0{}, t);
    if (wave_m == 0) phase_barrier();
    wait_vm<0>();  // the epilogue's first barrier then frees the tile's LDS

    f32x16_t blk[Cfg::MB][Cfg::NB];
    to_blocks32<Cfg::MB, Cfg::NB>(acc, blk);
    TileCtx<Cfg> ctx{s.M, s.N, m0, n0, tile_m, tile_n, wave_m, wave_n, lane, smem, kz};
    Epi::template apply<Cfg>(ep, blk, ctx);
  }
};

// bf16 on the small tile.
template <bool AK, bool BKM, class Epi, class Cfg, bool LOOP>
struct GemmBlockMid {
  static __device__ __forceinline__ void run(const Operand &A, const Operand &B, const GemmShape &s,
                                             const typename Epi::Params &ep, int b, int nblk, int kz, char *smem) {
    using R = Ring<Cfg::BM, Cfg::BN, Cfg::WM, Cfg::WN, Cfg::STAGES, AK, BKM, false, EpiPairB<Epi>::value>;
    int tid_v = threadIdx.x;
    if constexpr (LOOP) asm volatile("" : "+v"(tid_v));
    const int tid = tid_v, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tile_m, tile_n;
    tile_of_block(b, nblk, cdiv(s.M, Cfg::BM), cdiv(s.N, Cfg::BN), tile_m, tile_n);
    const int m0 = tile_m * Cfg::BM, n0 = tile_n * Cfg::BN;
    const int kbeg = s.kchunk > 0 ? kz * s.kchunk : 0;
    const int K = (s.kchunk > 0 ? min(s.K, kbeg + s.kchunk) : s.K) - kbeg;
    f32x4_t acc[2 * Cfg::MB][2 * Cfg::NB];
    R::run(A, m0, s.M, B, n0, s.N, kbeg, K, tid, smem, acc);
    f32x16_t blk[Cfg::MB][Cfg::NB];
    to_blocks32<Cfg::MB, Cfg::NB>(acc, blk);
    TileCtx<Cfg> ctx{s.M, s.N, m0, n0, tile_m, tile_n, wave / Cfg::WAVES_N, wave % Cfg::WAVES_N, lane, smem, kz};
    Epi::template apply<Cfg>(ep, blk, ctx);
  }
};

template <bool AK, bool BKM, class Epi, class Cfg, bool LOOP>
struct GemmBlock<bf16_t, AK, BKM, Epi, Cfg, LOOP>
    : std::conditional_t<Cfg::BM == 256, GemmBlockBig<AK, BKM, Epi, Cfg, LOOP>, GemmBlockMid<AK, BKM, Epi, Cfg, LOOP>> {};

template <typename T, bool AK, bool BKM, class Epi, class Cfg, bool LOOP = false>
__device__ __forceinline__ void gemm_block(const Operand &A, const Operand &B, const GemmShape &s,
                                           const typename Epi::Params &ep, int b, int nblk, int kz, char *smem) {
  GemmBlock<T, AK, BKM, Epi, Cfg, LOOP>::run(A, B, s, ep, b, nblk, kz, smem);
}

template <typename T, bool AK, bool BKM, class Epi, class Cfg>
__global__ __launch_bounds__(Cfg::BLOCK, Cfg::MIN_BLOCKS) void gemm_kernel(Operand A, Operand B, GemmShape s,
                                                                typename Epi::Params ep) {
  __shared__ __attribute__((aligned(128))) char smem[Cfg::SMEM_BYTES];
  gemm_block<T, AK, BKM, Epi, Cfg>(A, B, s, ep, blockIdx.x, gridDim.x, blockIdx.z, smem);
}

// The same product for a launch that usually has nothing to do: it runs
// only if *run_if is non-zero (a flag an earlier kernel of the stream set),
// one block per CU looping over the tiles.  The grid is a multiple of the
// XCD count, so tile t still runs on XCD t mod 8 and keeps its place in the
// XCD-aware order; when the flag is clear the launch costs one round of
// blocks that read it and return.
template <typename T, bool AK, bool BKM, class Epi, class Cfg>
__global__ __launch_bounds__(Cfg::BLOCK, Cfg::MIN_BLOCKS) void gemm_gated_kernel(Operand A, Operand B, GemmShape s,
                                                                      typename Epi::Params ep, const int *run_if) {
  __shared__ __attribute__((aligned(128))) char smem[Cfg::SMEM_BYTES];
  if (*run_if == 0) return;  // the same word for every thread
  const int tiles = cdiv(s.M, Cfg::BM) * cdiv(s.N, Cfg::BN);
  for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
    gemm_block<T, AK, BKM, Epi, Cfg, true>(A, B, s, ep, t, tiles, 0, smem);
    __syncthreads();  // the next tile's first stage overwrites what the epilogue used
  }
}

// One block per CU looping over the tiles, tile t on block t mod gridDim.x
// (a multiple of 8, so on XCD t mod 8 as in the one-block-per-tile launch):
// a CU starts its next tile's loads right after the epilogue's barrier,
// without waiting for a new block to be dispatched (measured at 2.6 us
// between one weight-gradient tile's end and the next one's start on the
// freed CU).  fp32: two blocks a CU, see gemm_f32_loops.
template <typename T, bool AK, bool BKM, class Epi, class Cfg>
__global__ __launch_bounds__(Cfg::BLOCK, Cfg::MIN_BLOCKS) void gemm_persistent_kernel(Operand A, Operand B,
                                                                           GemmShape s,
                                                                           typename Epi::Params ep) {
  __shared__ __attribute__((aligned(128))) char smem[Cfg::SMEM_BYTES];
  const int tiles = cdiv(s.M, Cfg::BM) * cdiv(s.N, Cfg::BN);
  for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
    gemm_block<T, AK, BKM, Epi, Cfg, true>(A, B, s, ep, t, tiles, 0, smem);
    __syncthreads();  // the next tile's first stage overwrites what the epilogue used
  }
}

// Two independent problems in one grid: blocks [0, blocks1) take problem 1,
// blocks [base2, gridDim.x) problem 2, where base2 = blocks1 rounded up to a
// multiple of 8 (the blocks in between do nothing), so that both keep the
// XCD-aware tile order.  The hardware dispatches blocks in order, so the
// problems share the GPU only where the first one's last round of tiles
// leaves CUs idle.  Problem 2 may be split along K (s2.kchunk > 0): its
// blocks then run slice by slice, each slice over all of its tiles.
template <typename T, bool AK1, bool BKM1, class Epi1, bool AK2, bool BKM2, class Epi2, class Cfg>
__global__ __launch_bounds__(Cfg::BLOCK, Cfg::MIN_BLOCKS) void gemm_pair_kernel(
    Operand A1, Operand B1, GemmShape s1, typename Epi1::Params ep1, Operand A2, Operand B2, GemmShape s2,
    typename Epi2::Params ep2, int blocks1, int base2) {
  __shared__ __attribute__((aligned(128))) char smem[Cfg::SMEM_BYTES];
  const int b = blockIdx.x;
  if (b < blocks1)
    gemm_block<T, AK1, BKM1, Epi1, Cfg>(A1, B1, s1, ep1, b, blocks1, 0, smem);
  else if (b >= base2) {
    const int tiles2 = cdiv(s2.M, Cfg::BM) * cdiv(s2.N, Cfg::BN), b2 = b - base2;
    gemm_block<T, AK2, BKM2, Epi2, Cfg>(A2, B2, s2, ep2, b2 % tiles2, tiles2, b2 / tiles2, smem);
  }
}

// The pair as one block per CU looping over the same block order (logical
// block t on block t mod gridDim.x, a multiple of 8), for two
// weight-gradient products.
template <typename T, bool AK1, bool BKM1, class Epi1, bool AK2, bool BKM2, class Epi2, class Cfg>
__global__ __launch_bounds__(Cfg::BLOCK, Cfg::MIN_BLOCKS) void gemm_pair_persistent_kernel(
    Operand A1, Operand B1, GemmShape s1, typename Epi1::Params ep1, Operand A2, Operand B2, GemmShape s2,
    typename Epi2::Params ep2, int blocks1, int base2, int total) {
  __shared__ __attribute__((aligned(128))) char smem[Cfg::SMEM_BYTES];
  const int tiles2 = cdiv(s2.M, Cfg::BM) * cdiv(s2.N, Cfg::BN);
  for (int t = blockIdx.x; t < total; t += gridDim.x) {
    if (t < blocks1) {
      gemm_block<T, AK1, BKM1, Epi1, Cfg, true>(A1, B1, s1, ep1, t, blocks1, 0, smem);
    } else if (t >= base2) {
      const int b2 = t - base2;
      gemm_block<T, AK2, BKM2, Epi2, Cfg, true>(A2, B2, s2, ep2, b2 % tiles2, tiles2, b2 / tiles2, smem);
    }
    __syncthreads();  // the next tile's first stage overwrites what the epilogue used
  }
}

// Shapes the loaders handle.
template <typename T, bool AK, bool BKM>
bool gemm_shape_ok(const Operand &A, const Operand &B, const GemmShape &s) {
  constexpr int BK = 8 * Elem<T>::CH;
  if (((AK || BKM) && s.K % BK != 0) || (!AK && s.M % 8 != 0) || (!BKM && s.N % 8 != 0)) return false;
  // MN-major loaders multiply by the k-row stride in bytes as an unsigned 24-bit
  // number: 2^22 fp32 values are 2^24 bytes
  return !((!AK && A.ld >= (int64_t{1} << 22)) || (!BKM && B.ld >= (int64_t{1} << 22)));
}

template <typename T, bool AK, bool BKM, class Epi, class Cfg>
hipError_t launch_gemm(Operand A, Operand B, GemmShape s, const typename Epi::Params &ep,
                       hipStream_t stream) {
  const int64_t blocks = static_cast<int64_t>(cdiv(s.M, Cfg::BM)) * cdiv(s.N, Cfg::BN);
  if (blocks <= 0) return hipSuccess;
  constexpr int BK = 8 * Elem<T>::CH;
  if (!gemm_shape_ok<T, AK, BKM>(A, B, s)) return hipErrorInvalidValue;
  int splits = 1;
  if (s.kchunk > 0) {
    if (s.kchunk % BK != 0) return hipErrorInvalidValue;  // slices start on stage boundaries
    splits = cdiv(s.K, s.kchunk);
  }
  if constexpr (EpiPersistent<Epi>::value && std::is_same<T, bf16_t>::value) {
    if (splits == 1 && blocks > 2 * kLoopBlocks) {
      hipLaunchKernelGGL((gemm_persistent_kernel<T, AK, BKM, Epi, Cfg>), dim3(kLoopBlocks), dim3(Cfg::BLOCK), 0,
                         stream, A, B, s, ep);
      return hipGetLastError();
    }
  }
  if constexpr (std::is_same<T, float>::value && Cfg::KW == 1) {
    if (splits == 1 && gemm_f32_loops(blocks)) {
      hipLaunchKernelGGL((gemm_persistent_kernel<T, AK, BKM, Epi, Cfg>), dim3(2 * kLoopBlocks), dim3(Cfg::BLOCK), 0,
                         stream, A, B, s, ep);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((gemm_kernel<T, AK, BKM, Epi, Cfg>), dim3(static_cast<unsigned>(blocks), 1, splits),
                     dim3(Cfg::BLOCK), 0, stream, A, B, s, ep);
  return hipGetLastError();
}

constexpr int kGatedBlocks = kLoopBlocks;

template <typename T, bool AK, bool BKM, class Epi, class Cfg>
hipError_t launch_gemm_gated(Operand A, Operand B, GemmShape s, const typename Epi::Params &ep, const int *run_if,
                             hipStream_t stream) {
  const int64_t tiles = static_cast<int64_t>(cdiv(s.M, Cfg::BM)) * cdiv(s.N, Cfg::BN);
  if (tiles <= 0) return hipSuccess;
  if (s.kchunk != 0 || run_if == nullptr || !gemm_shape_ok<T, AK, BKM>(A, B, s)) return hipErrorInvalidValue;
  const int64_t blocks = std::min<int64_t>(kGatedBlocks, (tiles + kNumXcd - 1) / kNumXcd * kNumXcd);
  hipLaunchKernelGGL((gemm_gated_kernel<T, AK, BKM, Epi, Cfg>), dim3(static_cast<unsigned>(blocks)),
                     dim3(Cfg::BLOCK), 0, stream, A, B, s, ep, run_if);
  return hipGetLastError();
}

template <typename T, bool AK1, bool BKM1, class Epi1, bool AK2, bool BKM2, class Epi2, class Cfg>
hipError_t launch_gemm_pair(Operand A1, Operand B1, GemmShape s1, const typename Epi1::Params &ep1, Operand A2,
                            Operand B2, GemmShape s2, const typename Epi2::Params &ep2, hipStream_t stream) {
  const int64_t b1 = static_cast<int64_t>(cdiv(s1.M, Cfg::BM)) * cdiv(s1.N, Cfg::BN);
  const int64_t b2 = static_cast<int64_t>(cdiv(s2.M, Cfg::BM)) * cdiv(s2.N, Cfg::BN);
  constexpr int BK = 8 * Elem<T>::CH;
  if (s1.kchunk != 0) return hipErrorInvalidValue;
  if (b1 <= 0) return launch_gemm<T, AK2, BKM2, Epi2, Cfg>(A2, B2, s2, ep2, stream);
  if (b2 <= 0) return launch_gemm<T, AK1, BKM1, Epi1, Cfg>(A1, B1, s1, ep1, stream);
  if (!gemm_shape_ok<T, AK1, BKM1>(A1, B1, s1) || !gemm_shape_ok<T, AK2, BKM2>(A2, B2, s2))
    return hipErrorInvalidValue;
  int64_t splits2 = 1;
  if (s2.kchunk > 0) {
    if (s2.kchunk % BK != 0) return hipErrorInvalidValue;
    splits2 = cdiv(s2.K, s2.kchunk);
  }
  const int64_t base2 = (b1 + kNumXcd - 1) / kNumXcd * kNumXcd;
  if constexpr (EpiPersistent<Epi1>::value && EpiPersistent<Epi2>::value && std::is_same<T, bf16_t>::value) {
    if (base2 + b2 * splits2 > 2 * kLoopBlocks) {
      hipLaunchKernelGGL((gemm_pair_persistent_kernel<T, AK1, BKM1, Epi1, AK2, BKM2, Epi2, Cfg>), dim3(kLoopBlocks),
                         dim3(Cfg::BLOCK), 0, stream, A1, B1, s1, ep1, A2, B2, s2, ep2, static_cast<int>(b1),
                         static_cast<int>(base2), static_cast<int>(base2 + b2 * splits2));
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((gemm_pair_kernel<T, AK1, BKM1, Epi1, AK2, BKM2, Epi2, Cfg>),
                     dim3(static_cast<unsigned>(base2 + b2 * splits2)), dim3(Cfg::BLOCK), 0, stream, A1, B1, s1, ep1, A2,
                     B2, s2, ep2, static_cast<int>(b1), static_cast<int>(base2));
  return hipGetLastError();
}

// Tile choice: gemm_mid_tile (bf16) and gemm_f32_small.
template <class Cfg> int64_t tiles_of(const GemmShape &s) {
  return static_cast<int64_t>(cdiv(s.M, Cfg::BM)) * cdiv(s.N, Cfg::BN) * (s.kchunk > 0 ? cdiv(s.K, s.kchunk) : 1);
}

inline int depth_of(const GemmShape &s) { return s.kchunk > 0 ? std::min(s.kchunk, s.K) : s.K; }

template <class... S> int parts_of(const S &...shapes) {
  return gemm_f32_parts((tiles_of<CfgF32>(shapes) + ...), (tiles_of<CfgF32Small>(shapes) + ...));
}

// f(configuration) for the tiles that these products take together.
template <typename T, class F, class... S>
hipError_t with_tile(F &&f, const S &...shapes) {
  if constexpr (std::is_same<T, bf16_t>::value) {
    if (gemm_mid_tile((tiles_of<CfgBig>(shapes) + ...))) return f(CfgMid{});
    return f(CfgBig{});
  } else {
    if (gemm_f32_small((tiles_of<CfgF32>(shapes) + ...), (tiles_of<CfgF32Small>(shapes) + ...), std::max({depth_of(shapes)...})))
      return f(CfgF32Small{});
    return f(CfgF32{});
  }
}

template <typename T, bool AK, bool BKM, class Epi>
hipError_t run_gemm(Operand A, Operand B, GemmShape s, const typename Epi::Params &ep, hipStream_t stream) {
  s.parts = parts_of(s);
  return with_tile<T>([&](auto c) { return launch_gemm<T, AK, BKM, Epi, decltype(c)>(A, B, s, ep, stream); }, s);
}

template <typename T, bool AK1, bool BKM1, class Epi1, bool AK2, bool BKM2, class Epi2>
hipError_t run_gemm_pair(Operand A1, Operand B1, GemmShape s1, const typename Epi1::Params &ep1, Operand A2,
                         Operand B2, GemmShape s2, const typename Epi2::Params &ep2, hipStream_t stream) {
  s1.parts = s2.parts = parts_of(s1, s2);
  return with_tile<T>(
      [&](auto c) {
        return launch_gemm_pair<T, AK1, BKM1, Epi1, AK2, BKM2, Epi2, decltype(c)>(A1, B1, s1, ep1, A2, B2, s2, ep2,
                                                                                  stream);
      },
      s1, s2);
}

}  // namespace ee
