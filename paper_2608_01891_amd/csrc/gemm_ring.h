// MFMA-bound tiles of up to 256 rows of the FFN GEMMs, gfx950 (the contract and
// the parameters of gemm_nt_kernel in gemm.h).
//
// What bounds these shapes: the matrix cores under the board's power limit (the
// clock falls from 2.4 to 1.7-1.9 GHz), so every LDS read and every idle cycle
// costs. Four waves, one per SIMD, each own 128 x 128 of the 256 x 256 outputs
// (of 256 x 128 of each of gate and up): a third fewer fragment reads per
// product than eight waves of 128 x 64. One wave per SIMD has nobody to hide
// its waits, so everything runs ahead: the fragments of a k-chunk of 32 are
// read while the previous chunk is multiplied, and loads go out one per eight
// products, evenly over the k-step (bursts of two: 6% slower).
//
// LDS is a ring of ten half tiles (128 rows x 64 k, 16 KiB) in the order A rows
// 0-127, B rows 0-127, B rows 128-255, A rows 128-255 of one k-step after the
// other. One barrier per k-step, where the wait leaves the two youngest half
// tiles in flight: 2.5 k-steps of loads, against one with two whole stages.
//
// Rows: 16-row block 2 i + wm of the tile is block i of the waves with row index
// wm, so a partly filled tile is shared evenly by the waves; only filled blocks
// are loaded and multiplied (in instances of 2 to 8 blocks per wave).
//
// Measured (dense SwiGLU, H = 5120, I = 25600; the eight-wave 32x32x16 tiles
// with two 64-wide stages before, both on one GPU): T = 4096 2854 -> 2384 us
// (1.13 -> 1.35 PFLOP/s), T = 512 423 -> 358 us; 8192^3 linear 885 -> 740 us.
// Bit-identical. (k-loops of few steps gain less or lose: kFewSteps in ffn_plan.h.)
// Tried and slower: a barrier after each quarter of the tile that frees half
// tiles earlier (eight waves; 13% less), two barriers per k-step (1-2%),
// persistent work-groups that load the next tile's first k-steps under the
// epilogue (no gain: the stores of a tile, 8 us when all CUs write at once,
// are what is left between tiles, and a wait for a load waits for them),
// buffer instead of global loads (no difference).
#pragma once
#include "gemm.h"

namespace aflex {

template <int N, class F, int I = 0>
__device__ __forceinline__ void unroll_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll_for<N, F, I + 1>(static_cast<F&&>(f));
  }
}

// Direct HBM -> LDS loads of 16 bytes per lane as lds_dma16, without restoring
// m0 (nothing else in the kernel that uses them reads it); the first takes a
// uniform base and a per-lane byte offset.
template <bool NT>
__device__ __forceinline__ void lds_dma16_s(const void* base, uint32_t voff, uint32_t lds) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0 nt" ::"s"(base), "v"(voff), "s"(lds) : "memory");
  else
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0" ::"s"(base), "v"(voff), "s"(lds) : "memory");
}
__device__ __forceinline__ void lds_dma16_v(const void* gptr, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr), "s"(lds) : "memory");
}

// acc += b . a on the matrix cores, the accumulator held in AGPRs.
__device__ __forceinline__ void mfma_acc(f32x4& acc, bf16x8 b, bf16x8 a) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}

constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8); }

template <bool DUAL, bool OUT_F32, bool NT_B = false>
__global__ __launch_bounds__(256, 1) void gemm_ring_kernel(GemmParams p) {
  constexpr int BN = DUAL ? 128 : 256;
  constexpr int HB = 128 * 64 * 2;  // bytes of a half tile: 128 rows x 64 k
  constexpr int RING = 10 * HB;
  // Weight rows of a wave's column block j (of four per B half): consecutive
  // ones for fp32 output, where a lane's 4 columns are one 16-byte store. For
  // bf16 output block pairs interleave in groups of 4 rows, so that a lane's
  // columns of both blocks are 8 consecutive ones, again one 16-byte store.
  constexpr bool PAIR = !OUT_F32;
  __shared__ __attribute__((aligned(16))) uint8_t sm[RING];

  GemmTile x;
  if (!gemm_tile_of(p, x)) return;
  const int n0 = x.nt * BN;
  const int kb = x.split * x.kps;
  const int nk = (min(p.K, kb + x.kps) - kb) / 64;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r = lane & 15, qg = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;

  // Sources of this wave's loads: wave-load j of a half tile covers its rows
  // 32 j + 8 wave + lane / 8, chunk lane % 8 of the LDS row holding chunk
  // (lane % 8) ^ swz(row). The swizzle puts the 16 rows of a fragment read on
  // distinct bank groups: (row / 2) % 8, for paired blocks (whose fragment rows
  // are 8 a + b, b < 4) 2 (row / 8 % 4) + row / 2 % 2. Rows past the tile's end
  // read its first row; weight rows past N read the last 8 (N is a multiple of
  // 64, so a wave-load's 8 rows are all inside or all past the end).
  const int lr = wave * 8 + (lane >> 3);
  const int ach = (lane & 7) ^ ((lr >> 1) & 7);
  const int bch = PAIR ? (lane & 7) ^ (wave * 2 + ((lane >> 4) & 1)) : ach;
  const uint32_t bvoff = ((lane >> 3) * p.ldb + bch * 8) * 2;
  const uint32_t wlds = __builtin_amdgcn_readfirstlane(lds_offset(sm)) + wave * 1024;
  const uint16_t* asrc[2][4];
  const uint16_t* bsrc[2][4];  // uniform
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = x.row0 + m * 128 + j * 32 + lr;
      const int g = row < x.row1 ? row : x.row0;
      const int srow = p.gather ? p.gather[g] / p.gather_div : g;
      asrc[m][j] = p.A + (size_t)srow * p.lda + kb + ach * 8;
      const int n = min(n0 + (DUAL ? 0 : m * 128) + j * 32 + wave * 8, p.N - 8);
      bsrc[m][j] = ((DUAL && m) ? p.B1 : p.B0) + (size_t)x.expert * p.b_expert_stride + (size_t)n * p.ldb + kb;
    }

  // Wave-load J of half tile Q of k-step `lk` into the ring at SLOT; the source
  // moves on with it. Loads past the last k-step re-read it.
  int lk = 0, step = 0;
  auto load_step = [&]() {  // before the first of a k-step's loads
    if (lk < nk) ++lk;
    step = lk < nk ? 64 : 0;
  };
#define RING_ISSUE(Q, SLOT, J)                                   \
  do {                                                          \
    const uint32_t d_ = wlds + (SLOT) + (J) * 4096;              \
    if constexpr ((Q) == 0 || (Q) == 3) {                        \
      if constexpr (((Q) / 3 * 4 + (J)) < N) {                   \
        lds_dma16_v(asrc[(Q) / 3][J], d_);                       \
        asrc[(Q) / 3][J] += step;                                \
      }                                                         \
    } else {                                                    \
      lds_dma16_s<NT_B>(bsrc[((Q) - 1) & 1][J], bvoff, d_);            \
      bsrc[((Q) - 1) & 1][J] += step;                            \
    }                                                           \
  } while (0)

  f32x4 acc[8][8];  // [row block][column block]

  // Byte offsets of this lane's fragments of k-chunk 0 and 1 in a half tile.
  const uint32_t off0 = r * 128 + ((qg ^ ((r >> 1) & 7)) << 4);
  const uint32_t offb = PAIR ? ((r >> 2) * 8 + (r & 3)) * 128 + ((qg ^ ((r >> 2) * 2 + ((r >> 1) & 1))) << 4) : off0;
  const uint32_t aoff[2] = {off0 + wm * 2048, (off0 ^ 64) + wm * 2048};
  const uint32_t boff[2] = {offb + wn * 8192, (offb ^ 64) + wn * 8192};

  auto kloop = [&](auto cn) {
    // Row blocks of each wave that are multiplied: N, 32 N rows of the tile, the
    // same for all waves; wave-loads of A rows past them are left out, so a
    // k-step takes 8 + N wave-loads, its first two half tiles 4 + min(N, 4).
    constexpr int N = decltype(cn)::value;
    bf16x8 fa[2][8], fb[2][8];
    // Fragment X of k-chunk C: X < 8 weight block X, else row block X - 8. U is
    // the ring offset of the k-step's first two half tiles, V of the other two.
#define RING_BOFF(J) (PAIR ? ((J) >> 1) * 4096 + ((J) & 1) * 512 : (J) * 2048)
#define RING_READ(C, X, U, V)                                                                          \
  do {                                                                                                 \
    if constexpr ((X) < 4)                                                                              \
      fb[C][X] = *reinterpret_cast<const bf16x8*>(sm + ((U) + boff[C]) + (HB + RING_BOFF(X)));            \
    else if constexpr ((X) < 8)                                                                         \
      fb[C][X] = *reinterpret_cast<const bf16x8*>(sm + ((V) + boff[C]) + RING_BOFF((X) - 4));             \
    else if constexpr ((X) < 12)                                                                        \
      fa[C][(X) - 8] = *reinterpret_cast<const bf16x8*>(sm + ((U) + aoff[C]) + ((X) - 8) * 4096);         \
    else                                                                                               \
      fa[C][(X) - 8] = *reinterpret_cast<const bf16x8*>(sm + ((V) + aoff[C]) + (HB + ((X) - 12) * 4096)); \
  } while (0)

    unroll_for<2>([&](auto s) {
      load_step();
      unroll_for<16>([&](auto l) {
        constexpr int L = decltype(l)::value, Q = L >> 2;
        RING_ISSUE(Q, (decltype(s)::value * 4 + Q) * HB, L & 3);
      });
    });
    // 256 accumulator registers of a wave, about a thousand cycles: behind the first
    // loads (the empty statements keep the compiler from moving it past the wait).
    // Before the loads and once more after the wait, k-loops of 8 and 16 steps
    // took 3 and 5% longer (MoE 512 x 4096, T = 940 86.4 -> 89.3 us; linear 7168 x
    // 9216, T = 256 59.4 -> 62.4).
#pragma unroll
    for (int i = 0; i < 8; ++i) {
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
      asm volatile("" : "+a"(acc[i][0]), "+a"(acc[i][1]), "+a"(acc[i][2]), "+a"(acc[i][3]), "+a"(acc[i][4]),
                        "+a"(acc[i][5]), "+a"(acc[i][6]), "+a"(acc[i][7]));
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(8 + N));
    __syncthreads();
    // Ring offsets: (u, v) of this k-step, vp = v of the one before (where the
    // third k-step's first half tiles go), (un, vn) of the next.
    int u = 0, v = 2 * HB, vp = 8 * HB, un = 4 * HB, vn = 6 * HB;
    unroll_for<8 + N>([&](auto f) { RING_READ(0, decltype(f)::value, 0, 2 * HB); });
    for (int kt = 0; kt < nk; ++kt) {
      load_step();
      // 16 slots (2 k-chunks of 32 x 8): a slot multiplies one row block, reads
      // up to 3 fragments of the next chunk and issues one wave-load of k-step
      // kt + 2 (its first two half tiles go where k-step kt - 1 ended, the
      // other two where k-step kt began).
      unroll_for<16>([&](auto ss) {
        constexpr int S = decltype(ss)::value, C = S >> 3, I = S & 7, Q = S >> 2;
        if constexpr (S == 8) {
          // Every fragment of k-step kt is in registers and k-step kt + 1 has
          // landed (the wave-loads since may be in flight), for all waves.
          __builtin_amdgcn_s_waitcnt(vmcnt_imm(4 + (N < 4 ? N : 4)));
          __syncthreads();
          __builtin_amdgcn_sched_barrier(0);
        }
        RING_ISSUE(Q, (C == 0 ? vp : u) + (Q & 1) * HB, S & 3);
        constexpr int XA = I < 4 ? I * 3 : 12 + (I - 4) * 2, XN = I < 4 ? 3 : (I < 6 ? 2 : 0);
        unroll_for<4>([&](auto gg) {
          constexpr int G = decltype(gg)::value, X = XA + G;
          if constexpr (I < N) {
            mfma_acc(acc[I][2 * G], fb[C][2 * G], fa[C][I]);
            mfma_acc(acc[I][2 * G + 1], fb[C][2 * G + 1], fa[C][I]);
          }
          if constexpr (G < XN && X < 8 + N) {
            if constexpr (C == 0)
              RING_READ(1, X, u, v);
            else
              RING_READ(0, X, un, vn);  // (past the last k-step: never used)
          }
          __builtin_amdgcn_sched_barrier(0);
        });
      });
      vp = v;
      u = un;
      v = vn;
      un = vn + 2 * HB == RING ? 0 : vn + 2 * HB;
      vn = un + 2 * HB == RING ? 0 : un + 2 * HB;
    }
    // No load may still target LDS when the work-group retires; the last
    // products are done before the accumulators are read (the compiler does
    // not see the matrix instructions and adds no wait states for them: the
    // empty statements tie every accumulator to a point after the wait).
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
    for (int i = 0; i < 8; ++i)
      asm volatile("" : "+a"(acc[i][0]), "+a"(acc[i][1]), "+a"(acc[i][2]), "+a"(acc[i][3]), "+a"(acc[i][4]),
                        "+a"(acc[i][5]), "+a"(acc[i][6]), "+a"(acc[i][7]));
  };
  const int rows = x.row1 - x.row0;  // (no split is without a k-step)
  if (rows > 224)
    kloop(std::integral_constant<int, 8>{});
  else if (rows > 192)
    kloop(std::integral_constant<int, 7>{});
  else if (rows > 160)
    kloop(std::integral_constant<int, 6>{});
  else if (rows > 128)
    kloop(std::integral_constant<int, 5>{});
  else if (rows > 96)
    kloop(std::integral_constant<int, 4>{});
  else if (rows > 64)
    kloop(std::integral_constant<int, 3>{});
  else
    kloop(std::integral_constant<int, 2>{});
#undef RING_ISSUE
#undef RING_READ
#undef RING_BOFF

  // Epilogue: accumulator elements 0..3 of a lane are four consecutive columns
  // of row r of the 16-row block.
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = x.row0 + (2 * i + wm) * 16 + r;
    if (row >= x.row1) continue;
    if constexpr (OUT_F32) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int col = n0 + (j >> 2) * 128 + wn * 64 + (j & 3) * 16 + qg * 4;
        if (col < p.N)
          *reinterpret_cast<f32x4*>(p.P + (size_t)x.split * p.p_split_stride + (size_t)row * p.ldp + col) = acc[i][j];
      }
    } else {
#pragma unroll
      for (int m = 0; m < (DUAL ? 2 : 4); ++m) {
        const int col = n0 + (m >> 1) * 128 + wn * 64 + (m & 1) * 32 + qg * 8;
        if (col >= p.N) continue;
        uint32_t o[4], rs[4] = {0, 0, 0, 0};
        if (!DUAL && p.R) *reinterpret_cast<uint4*>(rs) = *reinterpret_cast<const uint4*>(p.R + (size_t)row * p.ldc + col);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float w = acc[i][2 * m + (e >> 2)][e & 3];
          if (DUAL)
            w = w / (1.f + __expf(-w)) * acc[i][4 + 2 * (m & 1) + (e >> 2)][e & 3];
          else
            w += bf2f(static_cast<uint16_t>(rs[e >> 1] >> ((e & 1) * 16)));
          const uint32_t h = f2bf(w);
          if (e & 1)
            o[e >> 1] |= h << 16;
          else
            o[e >> 1] = h;
        }
        *reinterpret_cast<uint4*>(p.C + (size_t)row * p.ldc + col) = make_uint4(o[0], o[1], o[2], o[3]);
      }
    }
  }
}

}  // namespace aflex
