// KV-cache append of the current decode token, gfx950.
//
// Each decode step adds the new token's key and value to the growing cache
// before attention reads it (section 1; section 2, "LLM Serving"). The new
// token is the last cached one: position j = ctx_b - 1 of sequence b.
// One thread per (sequence, kv head, 8 elements of d): the key chunk is one
// 16-byte store into the token-major K tile, the value chunk eight 2-byte
// stores into the token-fastest V tile. Sequences with ctx_b <= 0 or a
// position past the table's capacity, and out-of-range block ids, write
// nothing.
#include "common.h"
#include "kernels.h"
#include "profile.h"

namespace aflex {

__global__ __launch_bounds__(256) void kv_append_kernel(aflex_kv_append_args a) {
  const int chunks = a.D / 8;
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long long)a.B * a.Hkv * chunks) return;
  const int c = (int)(idx % chunks);
  const int h = (int)((idx / chunks) % a.Hkv);
  const int b = (int)(idx / ((long long)chunks * a.Hkv));
  const int ctx = a.context_lens[b];
  if (ctx <= 0 || ctx > a.max_blocks_per_seq * 16) return;
  const int j = ctx - 1;
  const int blk = a.block_table[(size_t)b * a.max_blocks_per_seq + j / 16];
  if (blk < 0 || blk >= a.num_blocks) return;
  const int o = j % 16;
  const size_t src = ((size_t)b * a.Hkv + h) * a.D + c * 8;
  const uint4 kv = *reinterpret_cast<const uint4*>(a.k_new + src);
  *reinterpret_cast<uint4*>(a.k_cache + (((size_t)blk * a.Hkv + h) * 16 + o) * a.D + c * 8) = kv;
  const uint4 vv = *reinterpret_cast<const uint4*>(a.v_new + src);
  const uint32_t w[4] = {vv.x, vv.y, vv.z, vv.w};
  uint16_t* vdst = a.v_cache + (((size_t)blk * a.Hkv + h) * a.D + c * 8) * 16 + o;
#pragma unroll
  for (int e = 0; e < 8; ++e) vdst[e * 16] = static_cast<uint16_t>(w[e >> 1] >> ((e & 1) * 16));
}

__device__ __forceinline__ uint32_t chunk_word(const uint4& v, int i) {
  return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
}

// Packed multi-token write: one work-group per (cache block slot, sequence, K or
// V), one thread per (kv head, 8 elements of d). Slot jj of sequence b is logical
// block (max(start, 0) / 16) + jj with start = ctx_b - n_b; a thread moves the
// block's new positions: K rows as 16-byte stores, and V as whole 32-byte rows
// of the token-fastest tile when the block is entirely new (2-byte stores at a
// partial first or last block). Bound by memory latency: all 16 rows of a block
// are loaded before the first is stored (row by row, and K then V in one
// thread, 9500 tokens of 8 heads x 128 took 30 us for 78 MB). FEW: fewer than 16
// new tokens per sequence, so no block is whole, and only the rows a block has are
// loaded.
template <bool XCHG, bool FEW>
__global__ __launch_bounds__(XCHG ? 256 : 1024) void kv_write_kernel(aflex_kv_write_args a) {
  const int chunks = a.D / 8;
  const int g = threadIdx.x / chunks, c = threadIdx.x % chunks;
  if (g >= a.Hkv) return;
  const int b = blockIdx.y;
  int s1 = a.cu_seqlens[b + 1], s0 = a.cu_seqlens[b];
  s1 = min(max(s1, 0), a.T);
  s0 = min(max(s0, 0), s1);
  const int n = s1 - s0, ctx = a.context_lens[b];
  if (n <= 0 || ctx <= 0 || ctx > a.max_blocks_per_seq * 16) return;
  const int start = ctx - n;
  const int jb = max(start, 0) / 16 + (int)blockIdx.x;
  const int lo = max(jb * 16, max(start, 0)), hi = min(jb * 16 + 16, ctx);
  if (lo >= hi) return;
  const int blk = a.block_table[(size_t)b * a.max_blocks_per_seq + jb];
  if (blk < 0 || blk >= a.num_blocks) return;
  const size_t row_stride = (size_t)a.Hkv * a.D;
  // new token at cache position pos is row s0 + pos - start of k_new / v_new
  const long long shift = (long long)s0 - start;
  const uint16_t* src = (blockIdx.z ? a.v_new : a.k_new) + (size_t)g * a.D + c * 8;
  uint16_t* kc = a.k_cache + ((size_t)blk * a.Hkv + g) * 16 * a.D + c * 8;
  uint16_t* vc = a.v_cache + (((size_t)blk * a.Hkv + g) * a.D + c * 8) * 16;
  const int o0 = lo - jb * 16, o1 = hi - jb * 16;
  uint4 row[16];
#pragma unroll
  for (int o = 0; o < 16; ++o)  // (rows outside [o0, o1) repeat a row inside and are not stored)
    if (!FEW || (o >= o0 && o < o1))
      row[o] = *reinterpret_cast<const uint4*>(src + (size_t)(shift + jb * 16 + min(max(o, o0), o1 - 1)) * row_stride);
  if (blockIdx.z == 0) {
#pragma unroll
    for (int o = 0; o < 16; ++o)
      if (o >= o0 && o < o1) *reinterpret_cast<uint4*>(kc + (size_t)o * a.D) = row[o];
  } else if (!FEW && o1 - o0 == 16) {
    uint4 out[16];  // this thread's 8 rows of the V tile, 256 contiguous bytes
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
      uint32_t r[8];
#pragma unroll
      for (int o = 0; o < 8; ++o)
        r[o] = __builtin_amdgcn_perm(chunk_word(row[2 * o + 1], e >> 1), chunk_word(row[2 * o], e >> 1), sel);
      out[2 * e] = make_uint4(r[0], r[1], r[2], r[3]);
      out[2 * e + 1] = make_uint4(r[4], r[5], r[6], r[7]);
    }
    const int t = threadIdx.x & 15;
    if (XCHG && (int)(threadIdx.x | 15) < a.Hkv * chunks) {
      // 16 threads (4 KiB of contiguous V rows) exchange through LDS, so that
      // each store of theirs covers 256 contiguous bytes instead of 16 in every
      // 256. Piece x of thread t sits at x ^ t.
      extern __shared__ __attribute__((aligned(16))) uint8_t sm[];
      uint8_t* grp = sm + (threadIdx.x >> 4) * 4096;
#pragma unroll
      for (int x = 0; x < 16; ++x) *reinterpret_cast<uint4*>(grp + t * 256 + ((x ^ t) << 4)) = out[x];
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the 16 threads are lanes of one wave
      __builtin_amdgcn_wave_barrier();
      uint16_t* vt = vc - t * 128;  // the first thread's bytes
#pragma unroll
      for (int i = 0; i < 16; ++i)
        *reinterpret_cast<uint4*>(vt + i * 128 + t * 8) = *reinterpret_cast<const uint4*>(grp + i * 256 + ((t ^ i) << 4));
    } else {
#pragma unroll
      for (int x = 0; x < 16; ++x) *reinterpret_cast<uint4*>(vc + x * 8) = out[x];
    }
  } else {
#pragma unroll
    for (int o = 0; o < 16; ++o)
      if (o >= o0 && o < o1) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          vc[e * 16 + o] = static_cast<uint16_t>(chunk_word(row[o], e >> 1) >> ((e & 1) * 16));
      }
  }
}

hipError_t launch_kv_write(const aflex_kv_write_args& a, hipStream_t stream) {
  if (a.T == 0 || a.max_seqlen == 0) return hipSuccess;
  const int slots = (a.max_seqlen + 15) / 16 + 1;
  ProfScope ps("kv_write", stream);
  // The exchange of V rows takes 256 bytes of LDS per thread: up to 64 KiB. Wide
  // rows of few tokens: 64 sequences of one token, 64 heads x 128, 10.8 us with
  // only those rows loaded, 12.3 with 16; up to 256 threads no difference, and
  // whole blocks are 3-20% slower with the condition.
  const int threads = a.Hkv * (a.D / 8);
  const dim3 grid(slots, a.B, 2);
  if (threads <= 256)
    kv_write_kernel<true, false><<<grid, threads, (threads + 15) / 16 * 4096, stream>>>(a);
  else if (a.max_seqlen < 16)
    kv_write_kernel<false, true><<<grid, threads, 0, stream>>>(a);
  else
    kv_write_kernel<false, false><<<grid, threads, 0, stream>>>(a);
  return hipGetLastError();
}

hipError_t launch_kv_append(const aflex_kv_append_args& a, hipStream_t stream) {
  const long long n = (long long)a.B * a.Hkv * (a.D / 8);
  if (n == 0) return hipSuccess;
  ProfScope ps("kv_append", stream);
  kv_append_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(a);
  return hipGetLastError();
}

}  // namespace aflex
