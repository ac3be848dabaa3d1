// The class passes with 1 spectrum element per thread.
#include "user_class.hpp"

namespace mh3d {

void user_launch_class1(int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk, int mode, int fin) {
  class_cb<1>(cb, dir, grid, block, lds, s, vd, chk, mode, fin);
}

}  // namespace mh3d
