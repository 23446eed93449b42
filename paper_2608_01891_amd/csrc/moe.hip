// Top-k mixture-of-experts SwiGLU FFN, gfx950.
//
// The FFN of the MoE model the paper evaluates (Mixtral-8x7B, section 6.1;
// section 6.2 "Generality" notes that sparse expert execution changes the
// FFN's computation and communication). Steps, all on the device and without
// a host synchronisation:
//   1. route: per token, top-k experts by logit (ties -> lower id) and the
//      softmax over the k selected logits; per-expert counts, their exclusive
//      prefix, the stable (expert, token, slot) order of the token/slot pairs,
//      each pair's position in that order, and the m-tile map of the grouped
//      GEMMs. One work-group up to 512 tokens, else two kernels over chunks of
//      64 tokens (and a scan of the chunks' counts between them where there are
//      very many); ranks count the expert's earlier tokens in bit masks, so the
//      order is deterministic (and the same for all paths).
//   2. grouped gate/up GEMM with fused SwiGLU; the A rows are gathered from x
//      through the pair order (no permuted copy of x is written).
//   3. grouped down GEMM into fp32 split-K partials, rows in pair order.
//   4. combine: y_t = sum_j w_t,j * (sum over splits of row pos(t,j)), fixed
//      order, bf16 out.
#include "ffn_plan.h"
#include "gemm.h"
#include "kernels.h"
#include "profile.h"

namespace aflex {

constexpr int kMaxK = 8;
constexpr int kMaxE = 64;
// Up to this many tokens one work-group routes the batch (a single launch);
// larger batches take two kernels over chunks of kChunk tokens.
constexpr int kSingleRouteMaxT = 512;
constexpr int kChunk = 64;
// Chunks above which a launch between the two adds up the chunks' counts.
constexpr int kMaxSummedChunks = 512;

// Workspace: a routing block (ids .. num_tiles, written by the route kernel)
// followed by the expert block (h, P). The two can live apart: the pipeline
// keeps one routing block per microbatch and one shared expert block.
struct MoeLayout {
  size_t ids, wts, offsets, sorted, pos, tile_map, num_tiles, blockcnt, route_total;
  size_t h, P, expert_total;
  int bm, max_tiles, down_splits, down_kps;
  bool once, nt;
};

static MoeLayout moe_layout(const aflex_ffn_args& f) {
  MoeLayout L;
  const size_t pairs = (size_t)f.T * f.k;
  const MoePlan pl = plan_moe((long long)pairs, f.H, f.I, f.E, f.k);
  L.bm = pl.bm;
  L.once = pl.once;
  L.nt = pl.nt;
  L.max_tiles = (int)((pairs + L.bm - 1) / L.bm) + f.E;
  const int ntiles = (f.H + down_bn(L.bm) - 1) / down_bn(L.bm);
  // The tile count is a worst case here (the routing stays on the device):
  // round filling only for the one-work-group-per-CU tiles, as measured.
  plan_splits(L.max_tiles * ntiles, f.I, down_target(L.bm), L.bm >= 128 ? concurrent_wgs(L.bm) : 0, 16,
              &L.down_splits, &L.down_kps);
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o += align_up(bytes, 256);
    return at;
  };
  L.ids = take(pairs * 4);
  L.wts = take(pairs * 4);
  L.offsets = take((size_t)(f.E + 1) * 4);
  L.sorted = take(pairs * 4);
  L.pos = take(pairs * 4);
  L.tile_map = take((size_t)L.max_tiles * 3 * 4);
  L.num_tiles = take(4);
  L.blockcnt = take((((size_t)f.T + kChunk - 1) / kChunk + 1) * f.E * 4);  // (and a row of totals)
  L.route_total = o;
  o = 0;
  L.h = take(pairs * f.I * 2);
  L.P = take((size_t)L.down_splits * pairs * f.H * 4);
  L.expert_total = o;
  return L;
}

size_t moe_route_bytes(const aflex_ffn_args& f) { return moe_layout(f).route_total; }
size_t moe_expert_bytes(const aflex_ffn_args& f) { return moe_layout(f).expert_total; }
size_t moe_workspace_bytes(const aflex_ffn_args& f) {
  const MoeLayout L = moe_layout(f);
  return L.route_total + L.expert_total;
}

// Top-k of one token's logits (descending, ties to the lower id) and the
// softmax over the selected ones.
__device__ __forceinline__ void topk_token(const float* l, int E, int k, int* sid, float* w) {
  uint64_t taken = 0;
  float sel[kMaxK];
  for (int j = 0; j < k; ++j) {
    int bi = -1;
    float bv = 0.f;
    for (int e = 0; e < E; ++e) {
      if ((taken >> e) & 1) continue;
      const float v = l[e];
      if (bi < 0 || v > bv) {
        bi = e;
        bv = v;
      }
    }
    taken |= 1ull << bi;
    sel[j] = bv;
    sid[j] = bi;
  }
  float z = 0.f, ex[kMaxK];
  for (int j = 0; j < k; ++j) {
    ex[j] = expf(sel[j] - sel[0]);
    z += ex[j];
  }
  for (int j = 0; j < k; ++j) w[j] = ex[j] / z;
}

// Copy the logits of `rows` tokens (rows of E floats, contiguous) into LDS rows
// of stride ls, eight independent loads per lane in flight at a time: the
// top-k then reads LDS instead of issuing one dependent global load per
// compared logit (about 16 serial memory round trips per token at E = 8,
// k = 2).
template <int NT>
__device__ __forceinline__ void stage_logits(const float* __restrict__ src, int rows, int E, int ls, float* s_log,
                                             int tid) {
  const int n = rows * E;
  for (int i0 = 0; i0 < n; i0 += NT * 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * NT + tid;
      v[u] = i < n ? src[i] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = i0 + u * NT + tid;
      if (i < n) {
        const int r = i / E;
        s_log[r * ls + (i - r * E)] = v[u];
      }
    }
  }
}

// Top-k of one token by the 8 lanes of its group (lane j of the group holds
// logits [8 j, 8 j + 8), E <= 64), the same choice as topk_token: the largest
// untaken logit, ties to the lower id (a NaN is only taken as the first untaken
// one). Lane j < k returns slot j's expert and weight. For many experts: with
// one thread per token the 8 x 64 dependent compares and LDS reads of E = 64,
// k = 8 made the whole routing of 24 tokens take 108 us; one round here is a
// tournament over 8 registers and three DPP exchanges.
__device__ __forceinline__ void topk_lanes(const float* __restrict__ row, bool valid, int E, int k, int j8, int lane,
                                           int* id_out, float* w_out) {
  float l[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) l[i] = (valid && j8 * 8 + i < E) ? row[j8 * 8 + i] : 0.f;
  const uint64_t all = E == 64 ? ~0ull : (1ull << E) - 1ull;
  uint64_t taken = ~all;
  int my_id = 0;
  float my_v = 0.f, v0 = 0.f;
  for (int s = 0; s < k; ++s) {
    float bv = kNegInf;
    int bi = 127;  // loses every tie
#pragma unroll
    for (int i = 7; i >= 0; --i) {  // (descending, so >= leaves ties to the lower id)
      const int e = j8 * 8 + i;
      const bool ok = !((taken >> e) & 1) && l[i] >= bv;
      bv = ok ? l[i] : bv;
      bi = ok ? e : bi;
    }
    const int f = __builtin_ctzll(~taken);
    if ((f >> 3) == j8) {
      float lf = l[0];
#pragma unroll
      for (int i = 1; i < 8; ++i) lf = (f & 7) == i ? l[i] : lf;
      if (lf != lf) {
        bv = -kNegInf;
        bi = f - 64;  // wins every tie
      }
    }
    auto meet = [&](float ov, int oi) {
      const bool t = ov > bv || (ov == bv && oi < bi);
      bv = t ? ov : bv;
      bi = t ? oi : bi;
    };
#define AFLEX_DPP(X, CTRL) __builtin_amdgcn_update_dpp(X, X, CTRL, 0xf, 0xf, false)
    meet(__int_as_float(AFLEX_DPP(__float_as_int(bv), 0xB1)), AFLEX_DPP(bi, 0xB1));    // lane ^ 1
    meet(__int_as_float(AFLEX_DPP(__float_as_int(bv), 0x4E)), AFLEX_DPP(bi, 0x4E));    // lane ^ 2
    meet(__int_as_float(AFLEX_DPP(__float_as_int(bv), 0x141)), AFLEX_DPP(bi, 0x141));  // the group's other four
#undef AFLEX_DPP
    if (bi < 0) {
      bi += 64;
      bv = __builtin_nanf("");
    }
    taken |= 1ull << bi;
    v0 = s == 0 ? bv : v0;
    if (s == j8) {
      my_id = bi;
      my_v = bv;
    }
  }
  const float ex = j8 < k ? expf(my_v - v0) : 0.f;
  float z = 0.f;
  for (int s = 0; s < k; ++s) z += __shfl(ex, (lane & ~7) + s);
  *id_out = my_id;
  *w_out = ex / z;
}

// Exclusive offsets of the experts' pair counts and the m-tile map (at most bm
// rows per tile, in expert order) by one wave, lane e for expert e: cnt is the
// lane's count (0 past E). Offsets go to `off`, and with `publish` to memory, where the map goes.
__device__ __forceinline__ void plan_tiles(int cnt, int lane, int E, int bm, bool publish, int* off, int32_t* offsets,
                                           int32_t* u_offsets, int32_t* tile_map, int32_t* num_tiles) {
  const int rows = tile_rows(cnt, bm), n = (cnt + rows - 1) / rows;
  int incl = cnt, tincl = n;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int a = __shfl_up(incl, o), t = __shfl_up(tincl, o);
    if (lane >= o) {
      incl += a;
      tincl += t;
    }
  }
  const int first = incl - cnt, nt = tincl - n;
  off[lane] = first;  // (off[E] is the total: lanes past E count nothing)
  if (lane == 63) off[64] = incl;
  if (publish && lane < E) {
    offsets[lane] = first;
    if (u_offsets) u_offsets[lane] = first;
    if (lane == E - 1) {
      offsets[E] = incl;
      if (u_offsets) u_offsets[E] = incl;
      *num_tiles = tincl;
    }
    for (int i = 0; i < n; ++i) {
      int32_t* m = tile_map + 3 * (nt + i);
      m[0] = lane;
      m[1] = first + i * rows;
      m[2] = first + min((i + 1) * rows, cnt);
    }
  }
}

// Experts above which a token's top-k is shared by 8 lanes (topk_lanes): up to
// 16 experts one thread per token has few compares and no exchanges.
constexpr int kThreadTopkMaxE = 16;

// The whole routing of up to kSingleRouteMaxT tokens in one work-group. What
// bounds it is the chain of dependent steps, so each is done by as many lanes as
// it has items: the top-k, then per expert a bit mask of its tokens in LDS; one
// wave scans the experts' counts for the offsets and the tile map; a pair's
// stable rank is the number of its expert's mask bits below its token.
// (One thread building offsets and map, and ranks by ballots over all experts:
// E = 64, k = 8, 24 tokens 108 us in all, E = 8, k = 2, 256 tokens 12.)
__global__ __launch_bounds__(512) void moe_route_kernel(const float* __restrict__ logits, int T, int E, int k,
                                                        int bm, int32_t* ids, float* wts, int32_t* offsets,
                                                        int32_t* sorted, int32_t* pos, int32_t* tile_map,
                                                        int32_t* num_tiles, int32_t* u_ids, float* u_w,
                                                        int32_t* u_offsets, int32_t* u_sorted) {
  constexpr int kWords = kSingleRouteMaxT / 32;
  static_assert(kSingleRouteMaxT == 512, "one thread per token");
  __shared__ int off[kMaxE + 1];
  __shared__ uint32_t mask[kMaxE * (kWords + 1)];             // tokens of each expert, rows of odd stride
  __shared__ float s_log[512 * (kThreadTopkMaxE + 1)];        // logits, rows of odd stride
  __shared__ uint8_t s_ids[kSingleRouteMaxT * kMaxK];         // selected experts, read back for the ranks
  const int tid = threadIdx.x, lane = tid & 63;
  const int nw = (T + 31) >> 5;
  for (int i = tid; i < E * (kWords + 1); i += 512) mask[i] = 0;

  // 1. top-k and softmax over the selected logits.
  if (E <= kThreadTopkMaxE) {
    const int ls = E | 1;
    stage_logits<512>(logits, T, E, ls, s_log, tid);
    __syncthreads();
    if (tid < T) {
      int sid[kMaxK];
      float w[kMaxK];
      topk_token(s_log + tid * ls, E, k, sid, w);
      for (int j = 0; j < k; ++j) {
        const int e = sid[j], i = tid * k + j;
        ids[i] = e;
        wts[i] = w[j];
        s_ids[i] = static_cast<uint8_t>(e);
        if (u_ids) u_ids[i] = e;
        if (u_w) u_w[i] = w[j];
        atomicOr(&mask[e * (kWords + 1) + (tid >> 5)], 1u << (tid & 31));
      }
    }
  } else {
    __syncthreads();
    for (int t0 = 0; t0 < T; t0 += 64) {
      const int t = t0 + (tid >> 3), j = tid & 7;
      int e;
      float w;
      topk_lanes(logits + (size_t)t * E, t < T, E, k, j, lane, &e, &w);
      if (t < T && j < k) {
        const int i = t * k + j;
        ids[i] = e;
        wts[i] = w;
        s_ids[i] = static_cast<uint8_t>(e);
        if (u_ids) u_ids[i] = e;
        if (u_w) u_w[i] = w;
        atomicOr(&mask[e * (kWords + 1) + (t >> 5)], 1u << (t & 31));
      }
    }
  }
  __syncthreads();

  // 2. offsets and the m-tile map.
  if (tid < 64) {
    int cnt = 0;
    if (lane < E)
      for (int w = 0; w < nw; ++w) cnt += __popc(mask[lane * (kWords + 1) + w]);
    plan_tiles(cnt, lane, E, bm, true, off, offsets, u_offsets, tile_map, num_tiles);
  }
  __syncthreads();

  // 3. stable ranks: pairs of expert e are ordered by token (a token holds e
  //    at most once).
  for (int i = tid; i < T * k; i += 512) {
    const int e = s_ids[i], t = i / k;
    const uint32_t* m = mask + e * (kWords + 1);
    int rank = __popc(m[t >> 5] & ((1u << (t & 31)) - 1u));
    for (int w = 0; w < (t >> 5); ++w) rank += __popc(m[w]);
    const int pidx = off[e] + rank;
    sorted[pidx] = i;
    pos[i] = pidx;
    if (u_sorted) u_sorted[pidx] = i;
  }
}

// Batches of more than kSingleRouteMaxT tokens, in two launches over chunks of
// kChunk tokens: this one selects each chunk's experts, counts its pairs per
// expert and ranks them within the chunk (as moe_route_kernel does); the next
// adds up the counts and places the pairs. (Three launches, with ranks from
// ballots over all experts: E = 64, k = 8, 700 tokens 122 us, now 13; E = 8, k = 2,
// 2048 tokens 18 us, now 12.)
__global__ __launch_bounds__(8 * kChunk) void moe_topk_kernel(const float* __restrict__ logits, int T, int E, int k,
                                                              int32_t* ids, float* wts, int32_t* u_ids, float* u_w,
                                                              int32_t* blockcnt, int32_t* rank) {
  constexpr int kWords = kChunk / 32;
  __shared__ uint32_t mask[kMaxE * (kWords + 1)];
  __shared__ float s_log[kChunk * (kThreadTopkMaxE + 1)];
  __shared__ uint8_t s_ids[kChunk * kMaxK];
  const int tid = threadIdx.x;
  const int t0 = blockIdx.x * kChunk, n = min(kChunk, T - t0);
  if (tid < E * (kWords + 1)) mask[tid] = 0;
  auto put = [&](int t, int j, int e, float w) {  // slot j of the chunk's token t
    const size_t i = (size_t)(t0 + t) * k + j;
    ids[i] = e;
    wts[i] = w;
    s_ids[t * k + j] = static_cast<uint8_t>(e);
    if (u_ids) u_ids[i] = e;
    if (u_w) u_w[i] = w;
    atomicOr(&mask[e * (kWords + 1) + (t >> 5)], 1u << (t & 31));
  };
  if (E <= kThreadTopkMaxE) {
    const int ls = E | 1;
    stage_logits<8 * kChunk>(logits + (size_t)t0 * E, n, E, ls, s_log, tid);
    __syncthreads();
    if (tid < n) {
      int sid[kMaxK];
      float w[kMaxK];
      topk_token(s_log + tid * ls, E, k, sid, w);
      for (int j = 0; j < k; ++j) put(tid, j, sid[j], w[j]);
    }
  } else {
    __syncthreads();
    const int t = tid >> 3, j = tid & 7;
    int e;
    float w;
    topk_lanes(logits + (size_t)(t0 + t) * E, t < n, E, k, j, tid & 63, &e, &w);
    if (t < n && j < k) put(t, j, e, w);
  }
  __syncthreads();
  if (tid < E) {
    int cnt = 0;
    for (int w = 0; w < kWords; ++w) cnt += __popc(mask[tid * (kWords + 1) + w]);
    blockcnt[(size_t)blockIdx.x * E + tid] = cnt;
  }
  if (tid < n * k) {
    const int t = tid / k;
    const uint32_t* m = mask + s_ids[tid] * (kWords + 1);
    int r = __popc(m[t >> 5] & ((1u << (t & 31)) - 1u));
    for (int w = 0; w < (t >> 5); ++w) r += __popc(m[w]);
    rank[(size_t)t0 * k + tid] = r;
  }
}

// Chunk counts of one expert per work-group into what the earlier chunks hold,
// and the total into the row past the last chunk. For more than kMaxSummedChunks
// chunks: every placing work-group reading all counts grows with the square of
// the chunks (all of the routing, E = 8, k = 2: 512 chunks 17 us either way, 1024
// 25 -> 18, 2048 65 -> 27, 8192 718 -> 75).
__global__ __launch_bounds__(1024) void moe_scan_kernel(int32_t* blockcnt, int nblk, int E) {
  __shared__ int wsum[16];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  int32_t* col = blockcnt + blockIdx.x;
  int base = 0;
  for (int b0 = 0; b0 < nblk; b0 += 1024) {
    const int b = b0 + tid;
    const int v = b < nblk ? col[(size_t)b * E] : 0;
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o);
      if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = base, all = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      before += w < wave ? wsum[w] : 0;
      all += wsum[w];
    }
    if (b < nblk) col[(size_t)b * E] = before + incl - v;
    base += all;
    __syncthreads();  // (wsum is written again)
  }
  if (tid == 0) col[(size_t)nblk * E] = base;
}

// Places a chunk's pairs: every work-group adds up all chunks' counts (8 groups
// of 64 lanes, lane e for expert e) or, with `scanned`, reads the sums of
// moe_scan_kernel; the first one writes offsets and tile map. `pos` holds the
// ranks within the chunk on entry.
__global__ __launch_bounds__(8 * kChunk) void moe_place_kernel(const int32_t* __restrict__ ids,
                                                               const int32_t* __restrict__ blockcnt, int nblk,
                                                               bool scanned, int T, int E, int k, int bm,
                                                               int32_t* offsets,
                                                               int32_t* u_offsets, int32_t* tile_map,
                                                               int32_t* num_tiles, int32_t* sorted, int32_t* pos,
                                                               int32_t* u_sorted) {
  constexpr int kParts = 8 * kChunk / 64;
  __shared__ int s_tot[kParts][64], s_pre[kParts][64];
  __shared__ int off[kMaxE + 1], base[kMaxE];
  const int tid = threadIdx.x, lane = tid & 63, part = tid >> 6, blk = blockIdx.x;
  const int n = min(kChunk, T - blk * kChunk) * k;
  const size_t i = (size_t)blk * kChunk * k + tid;
  const int e = tid < n ? ids[i] : 0, r = tid < n ? pos[i] : 0;
  int tot = 0, pre = 0;
  if (scanned) {
    if (part == 0 && lane < E) {
      tot = blockcnt[(size_t)nblk * E + lane];
      pre = blockcnt[(size_t)blk * E + lane];
    }
  } else if (lane < E) {
#pragma unroll 4
    for (int b = part; b < nblk; b += kParts) {
      const int v = blockcnt[(size_t)b * E + lane];
      tot += v;
      pre += b < blk ? v : 0;
    }
  }
  s_tot[part][lane] = tot;
  s_pre[part][lane] = pre;
  __syncthreads();
  if (tid < 64) {
    tot = pre = 0;
#pragma unroll
    for (int q = 0; q < kParts; ++q) {
      tot += s_tot[q][lane];
      pre += s_pre[q][lane];
    }
    plan_tiles(tot, lane, E, bm, blk == 0, off, offsets, u_offsets, tile_map, num_tiles);
    base[lane] = pre;
  }
  __syncthreads();
  if (tid < n) {
    const int pidx = off[e] + base[e] + r;
    sorted[pidx] = (int)i;
    pos[i] = pidx;
    if (u_sorted) u_sorted[pidx] = (int)i;
  }
}

// The loads are issued in two independent batches -- the token's pair
// positions and weights (and the routed tile count), then the partial rows of
// up to four splits for all k pairs -- so a token waits for two memory round
// trips instead of one per pair and per split (inside the two-stream step,
// where every round trip queues behind the attention stream's loads, the
// chained form took 44 us per 64-token call on average). Sums keep split order
// per pair, then pair order.
template <int KMAX>
__global__ __launch_bounds__(256) void moe_combine_kernel(const float* __restrict__ P, long long split_stride,
                                                          int splits, int split_slots,
                                                          const int32_t* __restrict__ num_tiles, int n_ntiles,
                                                          int ksteps, const int32_t* __restrict__ pos,
                                                          const float* __restrict__ w, int k, int H,
                                                          const uint16_t* __restrict__ residual,
                                                          uint16_t* __restrict__ y) {
  const int t = blockIdx.x;
  const int c = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (c >= H) return;
  const int routed = split_slots > 0 ? *num_tiles : 0;
  long long row[KMAX];
  float wt[KMAX];
#pragma unroll
  for (int j = 0; j < KMAX; ++j) {  // pairs past k re-read the last one and are not added
    const int jj = min(j, k - 1);
    row[j] = pos[t * k + jj];
    wt[j] = w[t * k + jj];
  }
  // Uses of the loaded values here keep the compiler from sinking these loads
  // below the split planning, which waits for the routed tile count: all of
  // them then share one round trip.
  asm volatile("" ::"s"(routed));
#pragma unroll
  for (int j = 0; j < KMAX; ++j) asm volatile("" ::"s"(row[j]), "s"(wt[j]));
  if (split_slots > 0) {  // the down GEMM planned its split count on the device
    int kps;
    split_plan_slots(routed * n_ntiles, ksteps, splits, split_slots, &splits, &kps);
  }
  // Splits past the last re-read it and are not added; sums start from -0,
  // which leaves the first split's value unchanged.
  constexpr int kBatch = 4;
  f32x4 s[KMAX];
#pragma unroll
  for (int j = 0; j < KMAX; ++j) s[j] = f32x4{-0.f, -0.f, -0.f, -0.f};
  for (int sp0 = 0; sp0 < splits; sp0 += kBatch) {
    f32x4 v[kBatch][KMAX];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int j = 0; j < KMAX; ++j)
        v[u][j] = *reinterpret_cast<const f32x4*>(P + min(sp0 + u, splits - 1) * split_stride + row[j] * H + c);
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
#pragma unroll
      for (int j = 0; j < KMAX; ++j)
        if (sp0 + u < splits) s[j] += v[u][j];
  }
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < KMAX; ++j)
    if (j < k) acc += wt[j] * s[j];
  if (residual) {
    const ushort4 rv = *reinterpret_cast<const ushort4*>(residual + (size_t)t * H + c);
    acc[0] += bf2f(rv.x);
    acc[1] += bf2f(rv.y);
    acc[2] += bf2f(rv.z);
    acc[3] += bf2f(rv.w);
  }
  ushort4 o;
  o.x = f2bf(acc[0]);
  o.y = f2bf(acc[1]);
  o.z = f2bf(acc[2]);
  o.w = f2bf(acc[3]);
  *reinterpret_cast<ushort4*>(y + (size_t)t * H + c) = o;
}

hipError_t launch_moe_route(const aflex_ffn_args& f, void* route_ws, hipStream_t stream) {
  const MoeLayout L = moe_layout(f);
  char* w = static_cast<char*>(route_ws);
  int32_t* ids = reinterpret_cast<int32_t*>(w + L.ids);
  float* wts = reinterpret_cast<float*>(w + L.wts);
  int32_t* offsets = reinterpret_cast<int32_t*>(w + L.offsets);
  int32_t* sorted = reinterpret_cast<int32_t*>(w + L.sorted);
  int32_t* pos = reinterpret_cast<int32_t*>(w + L.pos);
  int32_t* tile_map = reinterpret_cast<int32_t*>(w + L.tile_map);
  int32_t* num_tiles = reinterpret_cast<int32_t*>(w + L.num_tiles);
  ProfScope ps("moe_route", stream);
  if (f.T <= kSingleRouteMaxT) {
    moe_route_kernel<<<1, 512, 0, stream>>>(f.router_logits, f.T, f.E, f.k, L.bm, ids, wts, offsets, sorted, pos,
                                            tile_map, num_tiles, f.topk_ids, f.topk_w, f.expert_offsets,
                                            f.sorted_pairs);
    return hipGetLastError();
  }
  const int nblk = (f.T + kChunk - 1) / kChunk;
  int32_t* blockcnt = reinterpret_cast<int32_t*>(w + L.blockcnt);
  moe_topk_kernel<<<nblk, 8 * kChunk, 0, stream>>>(f.router_logits, f.T, f.E, f.k, ids, wts, f.topk_ids, f.topk_w,
                                                   blockcnt, pos);
  const bool scan = nblk > kMaxSummedChunks;
  if (scan) moe_scan_kernel<<<f.E, 1024, 0, stream>>>(blockcnt, nblk, f.E);
  moe_place_kernel<<<nblk, 8 * kChunk, 0, stream>>>(ids, blockcnt, nblk, scan, f.T, f.E, f.k, L.bm, offsets,
                                                    f.expert_offsets, tile_map, num_tiles, sorted, pos,
                                                    f.sorted_pairs);
  return hipGetLastError();
}

hipError_t launch_moe(const aflex_ffn_args& f, void* ws, hipStream_t stream, const uint16_t* residual) {
  const MoeLayout L = moe_layout(f);
  hipError_t e = launch_moe_route(f, ws, stream);
  if (e != hipSuccess) return e;
  return launch_moe_experts(f, ws, static_cast<char*>(ws) + L.route_total, stream, residual);
}

hipError_t launch_moe_experts(const aflex_ffn_args& f, void* route_ws, void* expert_ws, hipStream_t stream,
                              const uint16_t* residual) {
  const MoeLayout L = moe_layout(f);
  char* w = static_cast<char*>(route_ws);
  char* xw = static_cast<char*>(expert_ws);
  const float* wts = reinterpret_cast<const float*>(w + L.wts);
  const int32_t* sorted = reinterpret_cast<const int32_t*>(w + L.sorted);
  const int32_t* pos = reinterpret_cast<const int32_t*>(w + L.pos);
  const int32_t* tile_map = reinterpret_cast<const int32_t*>(w + L.tile_map);
  const int32_t* num_tiles = reinterpret_cast<const int32_t*>(w + L.num_tiles);
  uint16_t* h = reinterpret_cast<uint16_t*>(xw + L.h);
  float* P = reinterpret_cast<float*>(xw + L.P);
  hipError_t e;

  GemmParams g = {};
  g.A = f.x;
  g.lda = f.H;
  g.gather = sorted;
  g.gather_div = f.k;
  g.B0 = f.w_gate;
  g.B1 = f.w_up;
  g.ldb = f.H;
  g.b_expert_stride = (long long)f.I * f.H;
  g.N = f.I;
  g.K = f.H;
  g.k_per_split = f.H;
  g.splits = 1;
  g.tile_map = tile_map;
  g.num_mtiles = num_tiles;
  g.max_mtiles = L.max_tiles;
  g.n_ntiles = (f.I + gate_bn(L.bm) - 1) / gate_bn(L.bm);
  // Experts expected in one row tile each (their weights streamed once):
  // expert-major order over the device-side tile count, so each XCD takes
  // consecutive n-tiles of one or two experts and keeps their token rows in
  // its L2 (64 tokens: 452 -> 444 us; the down GEMM at 256 tokens 179 -> 174
  // us). Otherwise an expert's m-tiles stay adjacent, so its overflow tiles
  // re-read the weights from L2 (the expert-major order took 512 tokens from
  // 745 to 820 us).
  const int order = L.once;
  g.mt_major = order;
  g.C = h;
  g.ldc = f.I;
  e = launch_gate_up(L.bm, L.nt, g, stream);
  if (e != hipSuccess) return e;

  const long long pairs = (long long)f.T * f.k;
  GemmParams d = {};
  d.A = h;
  d.lda = f.I;
  d.B0 = f.w_down;
  d.ldb = f.I;
  d.b_expert_stride = (long long)f.H * f.I;
  d.N = f.H;
  d.K = f.I;
  d.k_per_split = L.down_kps;
  d.splits = L.down_splits;
  // One-work-group-per-CU tiles: the split count follows the routed tile
  // count (at most the worst-case plan's), so whole rounds stay filled
  // without fp32 partials the tile count does not need (2048 tokens: one
  // split instead of three).
  d.split_slots = L.bm >= 128 ? concurrent_wgs(L.bm) : 0;
  d.tile_map = tile_map;
  d.num_mtiles = num_tiles;
  d.max_mtiles = L.max_tiles;
  d.n_ntiles = (f.H + down_bn(L.bm) - 1) / down_bn(L.bm);
  d.mt_major = order;
  d.P = P;
  d.p_split_stride = pairs * f.H;
  d.ldp = f.H;
  e = launch_down(L.bm, true, L.nt, d, stream);
  if (e != hipSuccess) return e;

  dim3 grid(f.T, (f.H / 4 + 255) / 256);
  ProfScope ps("moe_combine", stream);
  if (f.k <= 2)
    moe_combine_kernel<2><<<grid, 256, 0, stream>>>(P, d.p_split_stride, L.down_splits, d.split_slots, num_tiles,
                                                    d.n_ntiles, f.I / 64, pos, wts, f.k, f.H, residual, f.y);
  else
    moe_combine_kernel<kMaxK><<<grid, 256, 0, stream>>>(P, d.p_split_stride, L.down_splits, d.split_slots,
                                                        num_tiles, d.n_ntiles, f.I / 64, pos, wts, f.k, f.H,
                                                        residual, f.y);
  return hipGetLastError();
}

}  // namespace aflex
