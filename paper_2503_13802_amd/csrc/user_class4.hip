// The class passes with 4 spectrum elements per thread.
#include "user_class.hpp"

namespace mh3d {

void user_launch_class4(int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk, int mode, int fin) {
  class_cb<4>(cb, dir, grid, block, lds, s, vd, chk, mode, fin);
}

}  // namespace mh3d
