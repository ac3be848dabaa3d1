// The class passes with 3, 6, 8 or 9 spectrum elements per thread.
#include "user_class.hpp"

namespace mh3d {

void user_launch_class3689(int E, int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk,
                           int mode, int fin) {
  switch (E) {
    case 9: class_cb<9>(cb, dir, grid, block, lds, s, vd, chk, mode, fin); break;
    case 8: class_cb<8>(cb, dir, grid, block, lds, s, vd, chk, mode, fin); break;
    case 6: class_cb<6>(cb, dir, grid, block, lds, s, vd, chk, mode, fin); break;
    default: class_cb<3>(cb, dir, grid, block, lds, s, vd, chk, mode, fin); break;
  }
}

}  // namespace mh3d
