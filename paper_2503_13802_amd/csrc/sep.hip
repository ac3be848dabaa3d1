// Launchers of the separable passes of run-time geometry.
#include <algorithm>

#include "sep.hpp"

namespace mh3d {

void sep_launch_plane_fwd(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const int2* tasks,
                          const float* a, int src) {
  k_sep_plane_fwd<<<grid, block, lds, s>>>(vd, tasks, a, src);
}

template <bool ANY>
static void launch_col(int mode, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const int2* tasks, int chk,
                       int fin) {
  switch (mode) {
    case NRM_RESID: k_sep_col<NRM_RESID, ANY><<<grid, block, lds, s>>>(vd, tasks, chk, fin); break;
    case NRM_PLAIN: k_sep_col<NRM_PLAIN, ANY><<<grid, block, lds, s>>>(vd, tasks, chk, fin); break;
    case NRM_STORE: k_sep_col<NRM_STORE, ANY><<<grid, block, lds, s>>>(vd, tasks, chk, fin); break;
    case COL_FWD: k_sep_col<COL_FWD, ANY><<<grid, block, lds, s>>>(vd, tasks, chk, fin); break;
    case COL_ADJ: k_sep_col<COL_ADJ, ANY><<<grid, block, lds, s>>>(vd, tasks, chk, fin); break;
    default: k_sep_col<COL_DATA, ANY><<<grid, block, lds, s>>>(vd, tasks, chk, fin); break;
  }
}

void sep_launch_col(bool any, int mode, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd,
                    const int2* tasks, int chk, int fin) {
  if (any) launch_col<true>(mode, grid, block, lds, s, vd, tasks, chk, fin);
  else launch_col<false>(mode, grid, block, lds, s, vd, tasks, chk, fin);
}

// Blocks that the 256 CUs hold at once: by registers `waves` waves on each of a CU's 4 SIMDs, by LDS
// 160 KiB per CU (512 bytes of a block's are static).
static unsigned step_blocks_at_once(dim3 block, size_t lds, int waves) {
  const unsigned by_regs = 4 * waves / ((block.x + 63) / 64), by_lds = (unsigned)(160 * 1024 / (lds + 512));
  return 256 * std::max(1u, std::min(by_regs, by_lds));
}

void sep_launch_plane_adj(int out, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const int2* tasks,
                          AdjOut ao) {
  if (out == OUT_STEP_NORMAL) k_sep_plane_adj<OUT_STEP_NORMAL, 6><<<grid, block, lds, s>>>(vd, tasks, ao);
  else if (out == OUT_STEP_FISTA) {
    // the form of 80 registers where it takes fewer rounds of the chip (see k_sep_plane_adj)
    const unsigned n5 = step_blocks_at_once(block, lds, 5), n6 = step_blocks_at_once(block, lds, 6);
    if ((grid.x + n6 - 1) / n6 < (grid.x + n5 - 1) / n5)
      k_sep_plane_adj<OUT_STEP_FISTA, 6><<<grid, block, lds, s>>>(vd, tasks, ao);
    else
      k_sep_plane_adj<OUT_STEP_FISTA, 5><<<grid, block, lds, s>>>(vd, tasks, ao);
  } else k_sep_plane_adj<OUT_SCALE_B, 6><<<grid, block, lds, s>>>(vd, tasks, ao);
}

void sep_launch_adj_and_store(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, AdjOut ao, float* d,
                              int nbp) {
  k_sep_adj_and_store<<<grid, block, lds, s>>>(vd, ao, d, nbp);
}

void sep_launch_small_inv(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const int2* tasks, float* d,
                          int epi) {
  k_sep_small_inv<<<grid, block, lds, s>>>(vd, tasks, d, epi);
}

void sep_launch_small_fwd(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const float* r, float2* out) {
  k_sep_small_fwd<<<grid, block, lds, s>>>(vd, r, out);
}

}  // namespace mh3d
