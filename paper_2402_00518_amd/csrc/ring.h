// Building blocks of the products whose operands go straight from memory into
// LDS, and their ring main loops: bf16 on v_mfma_f32_16x16x32_bf16, shared by the
// small tiles and the decode-time products, and fp32 on v_mfma_f32_32x32x2_f32.
#pragma once

#include "ee_device.h"

// (load_lds16 names m0, which the compiler warns is a register it reserves)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"

namespace ee {

struct Operand {
  const void *ptr;
  int64_t ld;         // elements between consecutive rows of the stored matrix
  int64_t pair = 0;   // interleaved pair of matrices: bytes from the first matrix to the second
};

// 16 bytes a lane from base + off (off per lane) to LDS: lane l's bytes land
// at lds + 16 l.  The compiler does not count these loads: whoever reads what
// they bring waits with wait_vm, and a barrier makes it visible to the block.
// (Only inputs, so nothing of the load in flight sits in a register.)
__device__ __forceinline__ void load_lds16(const char *base, uint32_t off, uint32_t lds) {
  // base and lds are the same in every lane; say so, as the asm takes them in scalar registers
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  base = reinterpret_cast<const char *>(
      static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b)))) |
      static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(b >> 32)))) << 32);
  lds = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(lds)));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base)
               : "memory", "m0");
}
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lgkm() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
// A barrier without a wait for loads in flight (as __syncthreads would have).
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

// Accumulator rows of a 16 x 16 MFMA block: lanes 16 g .. 16 g + 15 hold rows
// 4 g .. 4 g + 3 of the block, which stand for rows 0, 8, 4, 12 (+ 0..3) of
// the tile's 16, so that one lane swap per register pair turns two column
// blocks into the 32 x 32 layout of TileCtx.
__device__ __forceinline__ int acc_row(int r) { return ((r >> 2) & 1) * 8 + ((r >> 3) & 1) * 4 + (r & 3); }

// Two 16-column blocks side by side -> the 32 x 32 layout: the swap hands
// lanes 16..31 (48..63) the right block's columns of the rows that lanes 0..15
// (32..47) keep of the left one, and the other way round.
template <int MB, int NB>
__device__ __forceinline__ void to_blocks32(const f32x4_t (&acc)[2 * MB][2 * NB], f32x16_t (&blk)[MB][NB]) {
  static_for<2 * MB>([&](auto i) EE_ALWAYS_INLINE {
    static_for<NB>([&](auto j) EE_ALWAYS_INLINE {
      static_for<4>([&](auto e) EE_ALWAYS_INLINE {
        constexpr int I = decltype(i)::value, J = decltype(j)::value, E = decltype(e)::value;
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[I][2 * J][E]),
                                                        __float_as_uint(acc[I][2 * J + 1][E]), false, false);
        blk[I / 2][J][(I % 2) * 8 + E] = __uint_as_float(r[0]);
        blk[I / 2][J][(I % 2) * 8 + 4 + E] = __uint_as_float(r[1]);
      });
    });
  });
}

// One operand of a ring stage: ROWS rows by 128 bytes of K (64 bf16 or 32 fp32
// values), loaded by THREADS threads, 16 bytes each a load.
// K-major: LDS rows of 128 bytes, 16-byte chunk c of row r at c ^ ((r / 2) mod
// 8); PAIR: rows of two matrices of F rows each in alternating blocks of 32,
// tile row r being row (r / 64) * 32 + r % 32 of the first matrix when (r / 32)
// is even, else of the second (row0 and rows count the interleaved rows).
// MN-major: the stage's k-rows as they are in memory.  bf16 (128 rows: k-rows of
// 256 bytes): chunk c of k-row k at c ^ (2 (k mod 4) + 8 (k / 8 mod 2)), read with
// ds_read_b64_tr_b16, which gives lane 4 a + b of each 16-lane group element b
// of the 8-byte pieces that lanes a, a + 4, a + 8, a + 12 of the group address.
// fp32: an MFMA takes one value a lane, so 32 lanes read 32 rows of a k-row.
template <typename T, bool KM, int ROWS, int THREADS, bool PERM, bool PAIR>
struct RingOperand {
  static constexpr bool kB16 = sizeof(T) == 2;
  static constexpr int KS = 128 / sizeof(T);  // values of K per stage
  static constexpr int LOADS = ROWS * 8 / THREADS;
  static constexpr int BYTES = ROWS * 128;
  static constexpr int KROW = ROWS * sizeof(T);   // MN-major: bytes of a k-row in LDS
  static constexpr int KCH = KROW / 16;           // and its chunks
  static constexpr int KSTEP = THREADS / KCH;     // k-rows between a thread's chunks
  static_assert(LOADS * THREADS == ROWS * 8, "every thread loads the same number of chunks");
  static_assert(KM || (!PAIR && (!kB16 || ROWS == 128)), "bf16 MN-major k-rows are 256 bytes");
  static_assert(!PAIR || THREADS / 8 <= 32, "a load's rows come from one matrix");
  uint32_t off[LOADS];
  uint32_t ldb, kr;  // MN-major: bytes between k-rows; k-row of the thread's first chunk
  const char *rd[kB16 ? (KM ? 2 : ROWS / 16) : 4];
  const char *base;
  int64_t pair, step;

  __device__ __forceinline__ static int swz(int k) { return kB16 ? 2 * (k & 3) + 8 * ((k >> 3) & 1) : 0; }

  // row0: first (interleaved) row of the tile, rows: rows of the operand;
  // wrow: the wave's first row in the tile; lds: the operand's LDS in stage 0;
  // kw (fp32): the 8 values of K of each stage from 8 kw on are the wave's, or
  // -1: all 32.
  __device__ __forceinline__ void init(const Operand &O, int row0, int rows, int kbeg, int tid, int wrow, int lane,
                                       const char *lds, int kw = -1) {
    const T *p = static_cast<const T *>(O.ptr);
    ldb = static_cast<uint32_t>(O.ld * sizeof(T));
    pair = O.pair;
    if constexpr (KM) {
      const int r0 = PAIR ? row0 / 2 : row0, last = (PAIR ? rows / 2 : rows) - 1;
      base = reinterpret_cast<const char *>(p + static_cast<int64_t>(r0) * O.ld + kbeg);
      step = 128;
      static_for<LOADS>([&](auto e) EE_ALWAYS_INLINE {
        const int c = decltype(e)::value * THREADS + tid, lr = c >> 3, ch = (c & 7) ^ ((lr >> 1) & 7);
        const int r = PAIR ? (lr >> 6) * 32 + (lr & 31) : lr;
        off[e] = static_cast<uint32_t>(min(r0 + r, last) - r0) * ldb + ch * 16;
      });
      if constexpr (kB16) {
        const int r = PERM ? acc_row(lane & 15) : lane & 15, x = (r >> 1) & 7;
        static_for<2>([&](auto ks) EE_ALWAYS_INLINE {
          rd[ks] = lds + (wrow + r) * 128 + (((decltype(ks)::value * 4 + (lane >> 4)) ^ x) << 4);
        });
      } else {
        const int r = lane & 31, x = (r >> 1) & 7;
        static_for<4>([&](auto g) EE_ALWAYS_INLINE {
          rd[g] = lds + (wrow + r) * 128 + (((2 * (kw < 0 ? decltype(g)::value : kw) + (lane >> 5)) ^ x) << 4);
        });
      }
    } else {
      base = reinterpret_cast<const char *>(p + static_cast<int64_t>(kbeg) * O.ld + row0);
      step = static_cast<int64_t>(ldb) * KS;
      kr = tid / KCH;
      constexpr int V = 16 / sizeof(T);
      static_for<LOADS>([&](auto e) EE_ALWAYS_INLINE {
        const int c = decltype(e)::value * THREADS + tid, k = c / KCH, ch = (c % KCH) ^ swz(k);
        off[e] = static_cast<uint32_t>(min(row0 + ch * V, rows - V) - row0) * sizeof(T);
      });
      if constexpr (kB16) {
        const int k = 8 * (lane >> 4) + ((lane >> 2) & 3), j = lane & 3;
        const int m = PERM ? (j & 1) * 8 + (j >> 1) * 4 : 4 * j;
        static_for<ROWS / 16>([&](auto i) EE_ALWAYS_INLINE {
          const int row = (wrow + decltype(i)::value * 16 + m) & (ROWS - 1);  // (blocks past the wave's rows are not read)
          rd[i] = lds + k * KROW + (((row >> 3) ^ swz(k)) << 4) + (row & 7) * 2;
        });
      } else {
        rd[0] = lds + (8 * (kw < 0 ? 0 : kw) + 4 * (lane >> 5)) * KROW + (wrow + (lane & 31)) * 4;
      }
    }
  }
  // Stage t into LDS from lds_wave on (the wave's first chunk of the operand);
  // left: values of K from this stage on (MN-major k-rows past them re-read the
  // last one).
  __device__ __forceinline__ void load(int t, int left, uint32_t lds_wave) const {
    const char *p = base + static_cast<int64_t>(t) * step;
    static_for<LOADS>([&](auto e) EE_ALWAYS_INLINE {
      constexpr int E = decltype(e)::value;
      uint32_t o = off[E];
      if constexpr (!KM) o += __umul24(min(static_cast<int>(kr) + E * KSTEP, left - 1), ldb);
      load_lds16(PAIR && ((E * THREADS / 8) >> 5) % 2 == 1 ? p + pair : p, o, lds_wave + E * THREADS * 16);
    });
  }
  // Zero the chunks this thread loads whose k-rows lie past K (MN-major).
  __device__ __forceinline__ void zero_tail(int left, int tid, char *lds) const {
    static_for<LOADS>([&](auto e) EE_ALWAYS_INLINE {
      constexpr int E = decltype(e)::value;
      if (static_cast<int>(kr) + E * KSTEP >= left)
        *reinterpret_cast<u32x4_t *>(lds + E * THREADS * 16 + tid * 16) = u32x4_t{0, 0, 0, 0};
    });
  }
  // bf16: fragments of NBLK 16-row blocks at the KS-th 32 values of K of the
  // stage `stage` bytes from stage 0.
  template <int KSI, int NBLK>
  __device__ __forceinline__ void read(int stage, bf16x8_t (&f)[NBLK]) const {
    static_for<NBLK>([&](auto i) EE_ALWAYS_INLINE {
      constexpr int I = decltype(i)::value;
      if constexpr (KM) {
        f[I] = *reinterpret_cast<const bf16x8_t *>(rd[KSI] + stage + I * 2048);
      } else {
        const char *p = rd[I] + stage + KSI * 8192;
        const s16x4_t both[2] = {__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(p)),
                                 __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(p + 1024))};
        f[I] = __builtin_bit_cast(bf16x8_t, both);
      }
    });
  }
  // fp32: values K = 8 (kw + G) + 4 (lane / 32) + 0..3 of the lane's row in NBLK
  // 32-row blocks.
  template <int G, int NBLK>
  __device__ __forceinline__ void read4(int stage, f32x4_t (&f)[NBLK]) const {
    static_for<NBLK>([&](auto i) EE_ALWAYS_INLINE {
      constexpr int I = decltype(i)::value;
      if constexpr (KM) {
        f[I] = *reinterpret_cast<const f32x4_t *>(rd[G] + stage + I * 4096);
      } else {
        static_for<4>([&](auto e) EE_ALWAYS_INLINE {
          f[I][decltype(e)::value] =
              *reinterpret_cast<const float *>(rd[0] + stage + (8 * G + decltype(e)::value) * KROW + I * 128);
        });
      }
    });
  }
};

// Ring of NS stages of 64 values of K: the stage NS - 1 further on is loaded
// while one is consumed, one barrier per stage.  A BM x BN tile on waves of
// WM x WN.  On return acc holds the wave's outputs, every load has landed and
// every wave has read what it needs (a barrier was passed since).
//
// PARTS = 4 or 8: K is summed in that many consecutive parts, as a balanced tree,
// (0 + 1) + (2 + 3) and for 8 that plus (4 + 5) + (6 + 7), and the tiles take them
// in PARTS different orders: row tile t starts at part o = t / 8 mod PARTS and
// takes part p ^ o as its p-th, which swaps the two sides of some sums (4
// parts: 0123, 1032, 2301, 3210).  Rows whose stride is a power of two lie in
// the same few memory channels at one K, and tiles that walk K in step all
// wait for those.  Every tile adds the same values in the same order up to
// swapped summands, so equal rows still give equal sums.
//
// SEQ > 1 (PARTS = 1): K is summed in up to that many consecutive parts, added up
// in order, for shorter chains of fp32 sums with half of the registers of 4 parts.
template <int BM_, int BN_, int WM_, int WN_, int NS_, bool AK, bool BKM, bool A_PAIR, bool B_PAIR, int PARTS = 1,
          int SEQ = 1>
struct Ring {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, NS = NS_;
  static constexpr int WAVES_M = BM / WM, WAVES_N = BN / WN, THREADS = WAVES_M * WAVES_N * 64;
  static constexpr int STAGE_BYTES = (BM + BN) * 128;
  using TA = RingOperand<bf16_t, AK, BM, THREADS, true, A_PAIR>;
  using TB = RingOperand<bf16_t, BKM, BN, THREADS, false, B_PAIR>;
  static constexpr int LOADS = TA::LOADS + TB::LOADS;
  using Acc = f32x4_t[WM / 16][WN / 16];
  static_assert((NS - 2) * LOADS <= 63, "loads in flight past the waited-for stage");
  static_assert(PARTS == 1 || SEQ == 1, "one way to take K in parts");
  static_assert(PARTS == 1 || ((PARTS == 4 || PARTS == 8) && AK), "parts: 1, or 4 or 8 of a K-major product");

  template <class F> __device__ __forceinline__ static void each(F &&f) {
    static_for<WM / 16>([&](auto i) EE_ALWAYS_INLINE {
      static_for<WN / 16>([&](auto j) EE_ALWAYS_INLINE { f(i, j); });
    });
  }

  // K values [kbeg, kbeg + K) of A's rows m0.. (of M) and B's rows n0.. (of N).
  __device__ __forceinline__ static void run(const Operand &A, int m0, int M, const Operand &B, int n0, int N, int kbeg,
                                             int K, int tid, char *smem, Acc &acc) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nk = (K + 63) / 64;
    TA ta;
    TB tb;
    ta.init(A, m0, M, kbeg, tid, (wave / WAVES_N) * WM, lane, smem);
    tb.init(B, n0, N, kbeg, tid, (wave % WAVES_N) * WN, lane, smem + TA::BYTES);
    const uint32_t lds_wave =
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char *)smem)) + wave * 1024;
    // the next stage to load, in the tile's order of parts
    const int order = PARTS > 1 ? m0 / BM / 8 % PARTS : 0;
    const int plen = (nk / PARTS) | 1;
    auto part_begin = [&](int p) EE_ALWAYS_INLINE { return PARTS > 1 ? (p < PARTS ? min(p * plen, nk) : nk) : p * nk; };
    int l_part = 0, l_t = part_begin(order), l_end = part_begin(order + 1), left = nk;  // left: stages not yet loaded
    auto load = [&](int buf) EE_ALWAYS_INLINE {
      if constexpr (PARTS > 1) {
        while (l_t == l_end && l_part < PARTS - 1) {  // (a part may be empty)
          ++l_part;
          l_t = part_begin(l_part ^ order);
          l_end = part_begin((l_part ^ order) + 1);
        }
      }
      ta.load(l_t, K - l_t * 64, lds_wave + buf * STAGE_BYTES);
      tb.load(l_t, K - l_t * 64, lds_wave + buf * STAGE_BYTES + TA::BYTES);
      ++l_t;
      --left;
    };
    static_for<NS - 1>([&](auto t) EE_ALWAYS_INLINE {
      if (decltype(t)::value < nk) load(decltype(t)::value);
    });
    int cur = 0;  // buffer of the stage to consume
    int todo = nk;
    auto consume = [&]() EE_ALWAYS_INLINE {
      // it has landed when at most the later stages' loads are in flight
      const int later = min(todo - 1, NS - 2);
      static_for<NS - 1>([&](auto l) EE_ALWAYS_INLINE {
        if (later == decltype(l)::value) wait_vm<decltype(l)::value * LOADS>();
      });
      if constexpr (!AK) {
        if (todo == 1 && K % 64 != 0) {  // zero A's k-rows past K, each thread the chunks it loaded itself
          ta.zero_tail(K - (nk - 1) * 64, tid, smem + cur * STAGE_BYTES);
          wait_lgkm();
        }
      }
      phase_barrier();
      if (left > 0) load(cur == 0 ? NS - 1 : cur - 1);  // over the last stage, which every wave has read
      const int stage = cur * STAGE_BYTES;
      static_for<2>([&](auto ks) EE_ALWAYS_INLINE {
        bf16x8_t fa[WM / 16], fb[WN / 16];
        tb.template read<decltype(ks)::value>(stage, fb);
        ta.template read<decltype(ks)::value>(stage, fa);
        each([&](auto i, auto j) EE_ALWAYS_INLINE {
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
        });
      });
      wait_lgkm();
      cur = cur == NS - 1 ? 0 : cur + 1;
      --todo;
    };
    constexpr int LEVELS = PARTS == 1 ? 1 : PARTS == 4 ? 2 : 3;
    Acc sum[LEVELS];  // sum[l]: the finished first half of a group of 2^(l+1) parts
    static_for<PARTS>([&](auto p_) EE_ALWAYS_INLINE {
      constexpr int P = decltype(p_)::value;
      each([&](auto i, auto j) EE_ALWAYS_INLINE { acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f}; });
      const int p = P ^ order, len = part_begin(p + 1) - part_begin(p);
      if constexpr (SEQ > 1) {
        const int slen = max((nk + SEQ - 1) / SEQ, 8);  // (512 values of K at least)
        Acc done;  // the parts before
        for (int t0 = 0; t0 < nk; t0 += slen) {
          const int t1 = min(t0 + slen, nk);
          for (int t = t0; t < t1; ++t) consume();
          each([&](auto i, auto j) EE_ALWAYS_INLINE {
            if (t0 > 0) acc[i][j] += done[i][j];
            done[i][j] = acc[i][j];
            if (t1 < nk) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
          });
        }
      } else {
        for (int t = 0; t < len; ++t) consume();
      }
      if constexpr (PARTS > 1) {
        constexpr int FULL = P == PARTS - 1 ? LEVELS : __builtin_ctz(~P);  // groups that end with this part
        each([&](auto i, auto j) EE_ALWAYS_INLINE {
          static_for<FULL>([&](auto l) EE_ALWAYS_INLINE { acc[i][j] += sum[l][i][j]; });
          if constexpr (FULL < LEVELS) sum[FULL][i][j] = acc[i][j];
        });
      }
    });
    phase_barrier();
  }
};

// The same ring for fp32 operands, 32 values of K a stage,
// v_mfma_f32_32x32x2_f32: a BM x BN tile on waves of 64 x 64.  KW = 4: the four
// waves of a 64 x 64 tile take 8 values of K each and their sums are added up,
// in order, in the first wave (the others' sums pass through LDS, 16 KB each).
// KW = 1 with parts = 4: K is summed in up to four consecutive parts, so that its
// sums are as short, and their error as small, as with KW = 4 (gradient of W_out,
// 340 tokens, h 384, V 7440: relative error 3.4e-7 in one sum, 1.9e-7 in four parts
// and with KW = 4).  Between parts the matrix cores wait for 128 VALU instructions
// a wave (504 tiles of K 512: 72.5 us in one sum, 77.6 in four parts).
template <int BM_, int BN_, int KW_, int NS_, bool AK, bool BKM, bool B_PAIR>
struct RingF32 {
  static constexpr int BM = BM_, BN = BN_, KW = KW_, NS = NS_;
  static constexpr int WAVES_N = BN / 64, THREADS = BM / 64 * WAVES_N * KW * 64;
  static constexpr int STAGE_BYTES = (BM + BN) * 128;
  using TA = RingOperand<float, AK, BM, THREADS, false, false>;
  using TB = RingOperand<float, BKM, BN, THREADS, false, B_PAIR>;
  static constexpr int LOADS = TA::LOADS + TB::LOADS;
  static_assert(KW == 1 || (KW == 4 && BM == 64 && BN == 64 && 3 * 16384 <= NS * STAGE_BYTES), "one 64 x 64 tile");

  // As Ring::run; with KW = 4 acc is whole in wave 0 only.
  __device__ __forceinline__ static void run(const Operand &A, int m0, int M, const Operand &B, int n0, int N, int kbeg,
                                             int K, int parts, int tid, char *smem, f32x16_t (&acc)[2][2]) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nk = (K + 31) / 32, kw = KW == 4 ? wave : -1;
    TA ta;
    TB tb;
    ta.init(A, m0, M, kbeg, tid, KW == 4 ? 0 : wave / WAVES_N * 64, lane, smem, kw);
    tb.init(B, n0, N, kbeg, tid, KW == 4 ? 0 : wave % WAVES_N * 64, lane, smem + TA::BYTES, kw);
    const uint32_t lds_wave =
        static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char *)smem)) + wave * 1024;
    auto load = [&](int t, int buf) EE_ALWAYS_INLINE {
      ta.load(t, K - t * 32, lds_wave + buf * STAGE_BYTES);
      tb.load(t, K - t * 32, lds_wave + buf * STAGE_BYTES + TA::BYTES);
    };
    f32x16_t sum[2][2];  // KW = 1: the finished parts, if any
    bool split = false;
    auto each = [&](auto &&f) EE_ALWAYS_INLINE {
      static_for<2>([&](auto i) EE_ALWAYS_INLINE { static_for<2>([&](auto j) EE_ALWAYS_INLINE { f(i, j); }); });
    };
    auto zero = [&](f32x16_t &a) EE_ALWAYS_INLINE {
      static_for<16>([&](auto v) EE_ALWAYS_INLINE { a[decltype(v)::value] = 0.0f; });
    };
    each([&](auto i, auto j) EE_ALWAYS_INLINE { zero(acc[i][j]); });
    static_for<NS - 1>([&](auto t) EE_ALWAYS_INLINE {
      if (decltype(t)::value < nk) load(decltype(t)::value, decltype(t)::value);
    });
    const int part = (nk + parts - 1) / parts;
    int part_end = part;
    int cur = 0;  // buffer of stage t
    for (int t = 0; t < nk; ++t) {
      if constexpr (KW == 1) {
        if (t == part_end) {
          each([&](auto i, auto j) EE_ALWAYS_INLINE {
            sum[i][j] = split ? sum[i][j] + acc[i][j] : acc[i][j];
            zero(acc[i][j]);
          });
          split = true;
          part_end += part;
        }
      }
      const int later = min(nk - 1 - t, NS - 2);
      static_for<NS - 1>([&](auto l) EE_ALWAYS_INLINE {
        if (later == decltype(l)::value) wait_vm<decltype(l)::value * LOADS>();
      });
      if constexpr (!AK) {
        if (t == nk - 1 && K % 32 != 0) {  // zero A's k-rows past K, each thread the chunks it loaded itself
          ta.zero_tail(K - t * 32, tid, smem + cur * STAGE_BYTES);
          wait_lgkm();
        }
      }
      phase_barrier();
      if (t + NS - 1 < nk) load(t + NS - 1, cur == 0 ? NS - 1 : cur - 1);  // over stage t - 1, which every wave has read
      const int stage = cur * STAGE_BYTES;
      static_for<KW == 4 ? 1 : 4>([&](auto g) EE_ALWAYS_INLINE {
        f32x4_t fa[2], fb[2];
        ta.template read4<decltype(g)::value>(stage, fa);
        tb.template read4<decltype(g)::value>(stage, fb);
        static_for<4>([&](auto e) EE_ALWAYS_INLINE {
          static_for<2>([&](auto i) EE_ALWAYS_INLINE {
            static_for<2>([&](auto j) EE_ALWAYS_INLINE {
              constexpr int E = decltype(e)::value;
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][E], fb[j][E], acc[i][j], 0, 0, 0);
            });
          });
        });
      });
      wait_lgkm();
      cur = cur == NS - 1 ? 0 : cur + 1;
    }
    phase_barrier();
    if constexpr (KW == 1) {
      if (split) each([&](auto i, auto j) EE_ALWAYS_INLINE { acc[i][j] += sum[i][j]; });
    }
    if constexpr (KW == 4) {
      // [wave - 1][block and quarter][lane] of 16 bytes
      f32x4_t *part = reinterpret_cast<f32x4_t *>(smem);
      if (wave > 0) {
        static_for<16>([&](auto q) EE_ALWAYS_INLINE {
          constexpr int Q = decltype(q)::value, I = Q / 8, J = Q / 4 % 2, E = Q % 4 * 4;
          part[((wave - 1) * 16 + Q) * 64 + lane] =
              f32x4_t{acc[I][J][E], acc[I][J][E + 1], acc[I][J][E + 2], acc[I][J][E + 3]};
        });
      }
      __syncthreads();
      if (wave == 0) {
        static_for<16>([&](auto q) EE_ALWAYS_INLINE {
          constexpr int Q = decltype(q)::value, I = Q / 8, J = Q / 4 % 2, E = Q % 4 * 4;
          static_for<3>([&](auto w) EE_ALWAYS_INLINE {
            const f32x4_t v = part[(decltype(w)::value * 16 + Q) * 64 + lane];
            static_for<4>([&](auto e) EE_ALWAYS_INLINE { acc[I][J][E + decltype(e)::value] += v[decltype(e)::value]; });
          });
        });
      }
    }
  }
};

}  // namespace ee

#pragma clang diagnostic pop
