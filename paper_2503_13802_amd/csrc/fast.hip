// Compile-time-geometry passes: instantiations and their launchers.
#include <algorithm>

#include "fast.hpp"

namespace mh3d {

template <class G>
struct FastImpl {
  static void plane_fwd(hipStream_t s, const VolDesc* vd, int src, const float* a) {
    const dim3 grid(G::NBP), block(G::TPF);
    switch (src) {
      case SRC_PLAIN: k_fast_plane_fwd<G, SRC_PLAIN><<<grid, block, G::LDS_PLANE, s>>>(vd, a, 0); break;
      case SRC_FISTA_Y: k_fast_plane_fwd<G, SRC_FISTA_Y><<<grid, block, G::LDS_PLANE, s>>>(vd, a, 0); break;
      case SRC_FISTA_NEXT: k_fast_plane_fwd<G, SRC_FISTA_Y><<<grid, block, G::LDS_PLANE, s>>>(vd, a, 1); break;
      default: k_fast_plane_fwd<G, SRC_SCALED><<<grid, block, G::LDS_PLANE, s>>>(vd, a, 0); break;
    }
  }
  static void cls(hipStream_t s, const VolDesc* vd, int mode, int chk, int fin) {
    const dim3 grid(G::NCLS / G::CPC + fin), block(G::TC);
    switch (mode) {
      case NRM_RESID: k_fast_col<G, NRM_RESID><<<grid, block, G::LDS_COL, s>>>(vd, chk, fin); break;
      case NRM_PLAIN: k_fast_col<G, NRM_PLAIN><<<grid, block, G::LDS_COL, s>>>(vd, chk, fin); break;
      case COL_FWD: k_fast_col<G, COL_FWD><<<grid, block, G::LDS_COL, s>>>(vd, chk, fin); break;
      case COL_ADJ: k_fast_col<G, COL_ADJ><<<grid, block, G::LDS_COL, s>>>(vd, chk, fin); break;
      default: k_fast_col<G, NRM_STORE><<<grid, block, G::LDS_COL, s>>>(vd, chk, fin); break;
    }
  }
  static void plane_adj(hipStream_t s, const VolDesc* vd, int out, AdjOut ao) {
    const dim3 grid(G::NBP), block(G::TP);
    if (out == OUT_STEP_NORMAL) k_fast_plane_adj<G, OUT_STEP_NORMAL><<<grid, block, G::LDS_PLANE, s>>>(vd, ao);
    else if (out == OUT_STEP_FISTA) k_fast_plane_adj<G, OUT_STEP_FISTA><<<grid, block, G::LDS_PLANE, s>>>(vd, ao);
    else k_fast_plane_adj<G, OUT_SCALE_B><<<grid, block, G::LDS_PLANE, s>>>(vd, ao);
  }
  static void adj_and_store(hipStream_t s, const VolDesc* vd, AdjOut ao, float* d, int nsmall, int xb) {
    k_fast_adj_and_store<G><<<dim3(G::NBP + nsmall), dim3(G::TP), std::max(G::small_lds(xb), G::LDS_PLANE), s>>>(
        vd, ao, d);
  }
  static void small_inv(hipStream_t s, const VolDesc* vd, float* d, int nsmall, int xb) {
    k_fast_small_inv<G><<<dim3(nsmall), dim3(G::TP), G::small_lds(xb), s>>>(vd, d);
  }
  static void small_fwd(hipStream_t s, const VolDesc* vd, const float* r, float2* out, int nsmall, int xb) {
    k_fast_small_fwd<G><<<dim3(nsmall), dim3(G::TP), G::small_lds(xb), s>>>(vd, r, out);
  }
  static void adjoint_each(hipStream_t s, const VolDesc* vd, int nv, float* out) {
    k_fast_col<G, COL_ADJ><<<dim3(G::NCLS / G::CPC, nv), dim3(G::TC), G::LDS_COL, s>>>(vd, 0, 0);
    AdjOut ao;
    ao.out = out;
    ao.yin = nullptr;
    k_fast_plane_adj<G, OUT_SCALE_B><<<dim3(G::NBP, nv), dim3(G::TP), G::LDS_PLANE, s>>>(vd, ao);
  }
  static FastOps ops() {
    return FastOps{G::NX, G::NY, G::NZ, G::SX, G::SY, G::SZ, G::KMAX, G::NBP, G::NCLS / G::CPC, G::TC,
                   G::LDS_PLANE, G::LDS_COL, &plane_fwd, &cls, &plane_adj, &adj_and_store, &small_inv,
                   &adjoint_each, &small_fwd};
  }
};

// Grids with compile-time passes: (nx, ny, nz, sx, sy, sz, columns per column-pass block,
// largest harmonic count).
extern const FastOps kFast[] = {
    FastImpl<FastGeo<128, 128, 128, 2, 4, 4, 4, 12, 512, 512, 134>>::ops(),   // 128^3, k = 2..12
    FastImpl<FastGeo<96, 96, 64, 2, 2, 2, 4, 8, 512, 512>>::ops(),            // 96 x 96 x 64, k = 2..8
    // small grids of the parity tests: every y split (1 to 4), radix 3 along x and y
    FastImpl<FastGeo<32, 32, 32, 2, 4, 4, 4, 12>>::ops(),
    FastImpl<FastGeo<16, 24, 16, 2, 2, 2, 4, 8>>::ops(),
    FastImpl<FastGeo<16, 16, 16, 2, 1, 2, 4, 8>>::ops(),
    FastImpl<FastGeo<24, 24, 16, 2, 3, 2, 4, 8>>::ops(),
};
extern const int kFastCount = (int)(sizeof kFast / sizeof kFast[0]);

}  // namespace mh3d
