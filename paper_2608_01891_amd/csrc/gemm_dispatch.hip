// Instantiations of the FFN GEMM tiles and their launch helpers.
//
// Row-tile size selects the shape: 32- and 64-row tiles stream weights (4
// waves, 16x16x32 MFMA, 64-wide k-steps, two work-groups per CU, HBM-bound);
// 128-row tiles are an 8-wave 32x32x16 MFMA shape (wave tiles of 64 rows by 32
// columns of each gate/up matrix or 64 columns of the down matrix, one
// work-group per CU in the whole 160 KiB of LDS as a ring of three stages); both
// take 64-wide k-steps, so every k-step reads whole 128-byte lines of each row.
// 256-row tiles are the MFMA-bound kernel of gemm_ring.h; 320-row tiles, for MoE
// calls that fit one round with them (plan_moe), the eight-wave shape with wave
// tiles of 160 rows in two stages. Weights that one tile
// streams exactly once load non-temporally where they are too large to stay
// cached (128-row tiles, dense T = 128 of 786 MB: 188 -> 175 us).
#include "ffn_plan.h"
#include "gemm_ring.h"
#include "profile.h"

namespace aflex {

template <int BM, int BN, int WM, int WN, int BK, int MS, bool DUAL, bool F32, int LDS, bool NT = false>
static void go(const GemmParams& g, unsigned grid, hipStream_t stream) {
  gemm_nt_kernel<BM, BN, WM, WN, BK, MS, DUAL, F32, LDS, NT><<<grid, 64 * WM * WN, 0, stream>>>(g);
}

static unsigned grid_of(const GemmParams& g) {
  return (unsigned)((long long)g.max_mtiles * g.n_ntiles * g.splits);
}

hipError_t launch_gate_up(int bm, bool nt, const GemmParams& g, hipStream_t stream) {
  const unsigned grid = grid_of(g);
  if (grid == 0) return hipSuccess;
  ProfScope ps("gemm_gate_up", stream);
  auto with = [&](auto n) {
    constexpr bool NT = decltype(n)::value;
    switch (bm) {
      case 32: go<32, 64, 1, 4, 64, 16, true, false, 81920, NT>(g, grid, stream); break;
      case 64: go<64, 64, 2, 2, 64, 16, true, false, 81920, NT>(g, grid, stream); break;
      case 128: go<128, 128, 2, 4, 64, 32, true, false, 163840, NT>(g, grid, stream); break;
      case 320: go<320, 128, 2, 4, 64, 32, true, false, 163840>(g, grid, stream); break;
      default: gemm_ring_kernel<true, false, NT><<<grid, 256, 0, stream>>>(g); break;
    }
  };
  if (nt)
    with(std::true_type{});
  else
    with(std::false_type{});
  return hipGetLastError();
}

template <bool F32, bool NT>
static void down(int bm, const GemmParams& g, unsigned grid, hipStream_t stream) {
  switch (bm) {
    case 32: go<32, 128, 1, 4, 64, 16, false, F32, 81920, NT>(g, grid, stream); break;
    case 64: go<64, 128, 2, 2, 64, 16, false, F32, 81920, NT>(g, grid, stream); break;
    case 128: go<128, 256, 2, 4, 64, 32, false, F32, 163840, NT>(g, grid, stream); break;
    case 320: go<320, 256, 2, 4, 64, 32, false, F32, 163840>(g, grid, stream); break;
    default: gemm_ring_kernel<false, F32, NT><<<grid, 256, 0, stream>>>(g); break;
  }
}

hipError_t launch_down(int bm, bool f32_partials, bool nt, const GemmParams& g, hipStream_t stream) {
  const unsigned grid = grid_of(g);
  if (grid == 0) return hipSuccess;
  ProfScope ps("gemm_down", stream);
  if (f32_partials)
    nt ? down<true, true>(bm, g, grid, stream) : down<true, false>(bm, g, grid, stream);
  else
    nt ? down<false, true>(bm, g, grid, stream) : down<false, false>(bm, g, grid, stream);
  return hipGetLastError();
}

}  // namespace aflex
