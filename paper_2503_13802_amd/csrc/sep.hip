// Launchers of the separable passes of run-time geometry.
#include "sep.hpp"

namespace mh3d {

void sep_launch_plane_fwd(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const int2* tasks,
                          const float* a, int src) {
  k_sep_plane_fwd<<<grid, block, lds, s>>>(vd, tasks, a, src);
}

void sep_launch_col(bool any, int mode, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd,
                    const int2* tasks, int chk, int fin) {
  if (any) k_sep_col<-1><<<grid, block, lds, s>>>(vd, tasks, mode, chk, fin);
  else switch (mode) {
    case NRM_RESID: k_sep_col<NRM_RESID><<<grid, block, lds, s>>>(vd, tasks, mode, chk, fin); break;
    case NRM_PLAIN: k_sep_col<NRM_PLAIN><<<grid, block, lds, s>>>(vd, tasks, mode, chk, fin); break;
    case NRM_STORE: k_sep_col<NRM_STORE><<<grid, block, lds, s>>>(vd, tasks, mode, chk, fin); break;
    case COL_FWD: k_sep_col<COL_FWD><<<grid, block, lds, s>>>(vd, tasks, mode, chk, fin); break;
    case COL_ADJ: k_sep_col<COL_ADJ><<<grid, block, lds, s>>>(vd, tasks, mode, chk, fin); break;
    default: k_sep_col<COL_DATA><<<grid, block, lds, s>>>(vd, tasks, mode, chk, fin); break;
  }
}

void sep_launch_plane_adj(int out, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const int2* tasks,
                          AdjOut ao) {
  if (out == OUT_STEP_NORMAL) k_sep_plane_adj<OUT_STEP_NORMAL, 6><<<grid, block, lds, s>>>(vd, tasks, ao);
  else if (out == OUT_STEP_FISTA && grid.x > 512) k_sep_plane_adj<OUT_STEP_FISTA, 6><<<grid, block, lds, s>>>(vd, tasks, ao);
  else if (out == OUT_STEP_FISTA) k_sep_plane_adj<OUT_STEP_FISTA, 5><<<grid, block, lds, s>>>(vd, tasks, ao);
  else k_sep_plane_adj<OUT_SCALE_B, 6><<<grid, block, lds, s>>>(vd, tasks, ao);
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
