// Launchers of the passes of plans with user PSFs.
#include "user.hpp"

namespace mh3d {

void user_launch_plane_fwd(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const float* a, int src) {
  if (src == SRC_RAW) k_user_plane_fwd<true><<<grid, block, lds, s>>>(vd, a, src);
  else k_user_plane_fwd<false><<<grid, block, lds, s>>>(vd, a, src);
}

template <bool ROUNDS>
static void plane_adj(int out, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, AdjOut ao) {
  if (out == OUT_STEP_NORMAL) k_user_plane_adj<OUT_STEP_NORMAL, ROUNDS><<<grid, block, lds, s>>>(vd, ao);
  else if (out == OUT_STEP_FISTA) k_user_plane_adj<OUT_STEP_FISTA, ROUNDS><<<grid, block, lds, s>>>(vd, ao);
  else k_user_plane_adj<OUT_SCALE_B, ROUNDS><<<grid, block, lds, s>>>(vd, ao);
}
void user_launch_plane_adj(bool rounds, int out, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, AdjOut ao) {
  if (rounds) plane_adj<true>(out, grid, block, lds, s, vd, ao);
  else plane_adj<false>(out, grid, block, lds, s, vd, ao);
}

void user_launch_step_and_fwd(bool rounds, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, AdjOut ao) {
  if (rounds) k_user_step_and_fwd<true><<<grid, block, lds, s>>>(vd, ao);
  else k_user_step_and_fwd<false><<<grid, block, lds, s>>>(vd, ao);
}

void user_launch_adj_and_store(bool rounds, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, AdjOut ao,
                               float* d) {
  if (rounds) k_user_adj_and_store<true><<<grid, block, lds, s>>>(vd, ao, d);
  else k_user_adj_and_store<false><<<grid, block, lds, s>>>(vd, ao, d);
}

// the class passes compile in units of their own
void user_launch_class(int E, int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk,
                       int mode, int fin) {
  switch (E) {
    case 1: user_launch_class1(cb, dir, grid, block, lds, s, vd, chk, mode, fin); break;
    case 2: user_launch_class2(cb, dir, grid, block, lds, s, vd, chk, mode, fin); break;
    case 4: user_launch_class4(cb, dir, grid, block, lds, s, vd, chk, mode, fin); break;
    default: user_launch_class3689(E, cb, dir, grid, block, lds, s, vd, chk, mode, fin); break;
  }
}

}  // namespace mh3d
