// Geometry of one MH3D plan, shared by host launch code and kernels.
//
// Spectra use an "alias-class" layout.  The decimated grid (mx, my, mz) has a
// Hermitian half along z, q'z in [0, mz/2].  A class is one pair (q'y, q'z),
// class id c = q'y * mzh + q'z, mzh = mz/2 + 1.  Its nmem = sy*sz members are the
// full-grid (qy, qz) = (q'y + jy*my, q'z + jz*mz), member id m = jy*sz + jz.  Folding
// the full spectrum onto the decimated grid (the Fourier form of the row selector
// P) sums exactly over the members of one class and over qx = q'x + jx*mx, so one
// workgroup can own a class end to end.  Members with qz > nz/2 are stored as the
// conjugate of the in-plane Hermitian partner (ny - qy, nz - qz), which is exact for
// the y-z spectrum of a real x-plane.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mh3d {

// Division by a per-plan constant d >= 1 for 0 <= n < 2^31 with one 32x64-bit
// multiply: q = (n * m) >> s, m = ceil(2^(31+l) / d), l = ceil(log2 d)
// (Granlund & Montgomery, PLDI 1994, round-up variant).
struct FastDiv {
  uint64_t m;
  uint32_t s, d;
  __host__ __device__ inline uint32_t div(uint32_t n) const { return (uint32_t)(((uint64_t)n * m) >> s); }
  __host__ __device__ inline uint32_t mod(uint32_t n) const { return n - div(n) * d; }
};

inline FastDiv make_fastdiv(uint32_t d) {
  uint32_t l = 0;
  while ((1ull << l) < d) ++l;
  FastDiv f;
  f.d = d;
  f.s = 31 + l;
  const unsigned __int128 one = 1;
  const unsigned __int128 p = one << (31 + l);
  f.m = (uint64_t)((p + d - 1) / d);
  return f;
}

// n / d for 0 <= n < 2^16 with n * d <= 2^24, by one 24-bit high multiply (full rate, where
// a 32-bit one takes four times as long): with m = ceil(2^24 / d) and e = m d - 2^24 < d
// the quotient (n 2^8)(m) / 2^32 is exact while n e < 2^24.  The passes stay within that: their axes,
// columns and blocks are few, and transforms with compiled stages have at least 4 points of the
// 10240 that an LDS buffer holds, so at most 2048 lines of fewer than 4096 butterflies
// (tests/test_divisors.py goes through all of them).  The small grid's y' lines of one to three
// points can be more: the run-time transforms, which take those, deal by div_any.
struct MDiv {
  uint32_t m, d;
  __host__ __device__ __forceinline__ int div(int n) const {
    const uint32_t a = ((uint32_t)n << 8) & 0xffffffu, b = m & 0xffffffu;
    const int q = (int)(uint32_t)(((uint64_t)a * b) >> 32);
    return d == 1 ? n : q;
  }
  // n / d and the remainder for any 0 <= n, d < 2^16: n m / 2^24 exceeds n / d by n e / (d 2^24) < 2^-8, so the
  // quotient above is at most one too large.
  __host__ __device__ __forceinline__ int div_any(int n, int& rem) const {
    int q = div(n);
    rem = n - q * (int)d;
    if (rem < 0) {
      --q;
      rem += (int)d;
    }
    return q;
  }
};

inline MDiv make_mdiv(int d) {
  MDiv r;
  r.d = (uint32_t)d;
  r.m = d == 1 ? 0u : (uint32_t)(((1u << 24) + (uint32_t)d - 1) / (uint32_t)d);
  return r;
}

// Launch shapes and divisors of the run-time separable and small-grid passes (sep.hpp).
struct SepGeo {
  int np;                  // row pairs of a plane block: (my + 1)/2
  int lsz, lsy;            // LDS line strides of its packed z lines and its y lines
  int pbuf;                // one of its two LDS buffers (complex values)
  int cpc, kg;             // columns per column block, harmonics per group of it
  int lsx, lsm;            // LDS line strides of its x and x' lines
  int lsmz;                // line stride of the small grid's packed z' lines
  int nxb;                 // x'-blocks: mx / xb
  // d_nzv, d_mzv: vectors (4 or 2 values) per row of the plane and of the small grid
  MDiv d_sy, d_np, d_nzh, d_mzh, d_nzv, d_mz, d_mzv, d_my, d_mx, d_cpc, d_cpcmx, d_cpcxb, d_xb, d_kgcpc, d_klcpc, d_spairs,
      d_xbmzh, d_nxb;
};

// Launch shapes and divisors of the user-PSF passes (user.hpp).
struct UserGeo {
  int pl;                  // one LDS buffer of a component's plane (complex values)
  int pcb;                 // components per round of the adjoint plane pass (1 or C)
  int cb;                  // components at once in the class passes: all C, or 0 for rounds of one
  int fls;                 // LDS line stride of the folded spectra
  // of the plane passes: npairs, alone and times pcb; the two column counts of a workgroup; pcb (nz/2 + 1); the two
  // counts of row pairs of a workgroup, times pcb and alone.  Of the class passes: cpw nmem, that
  // times the components at once, K cpw, cpw mx and cpw xb.
  MDiv d_np, d_cnp, d_qlo, d_qhi, d_ycols, d_jlo, d_jhi, d_j1lo, d_j1hi, d_w, d_cbw, d_kc, d_cm, d_cxb;
};

struct Geo {
  int nx, ny, nz, nzh;     // grid, nzh = nz/2 + 1
  int mx, my, mz, mzh;     // decimated grid, mzh = mz/2 + 1
  int sx, sy, sz, S;       // decimation factors, S = sx*sy*sz
  int nmem;                // members per class = sy*sz
  int ncls;                // classes = my*mzh
  int plane;               // complex values per x-plane of the class layout = ncls*nmem
  int K;                   // harmonics
  int C;                   // components of the vector model (1: scalar b and h_k)
  int cpw;                 // classes per class-kernel workgroup (divides ncls)
  int E;                   // spectrum elements per thread in the class kernel (divides S)
  int xb;                  // x' planes per small-grid workgroup (divides mx)
  int ps;                  // workgroups per x-plane in the plane passes (1 to 4)
  int npairs;              // (ny + 1)/2 row pairs of one full x-plane
  int spairs;              // (xb*my + 1)/2 row pairs of one small-grid workgroup
  int lsy;                 // LDS line stride of y-transforms in the plane kernels (ny + pad)
  int lsx;                 // LDS line stride of x-transforms in the class kernels (nx + pad)
  int lsmy;                // LDS line stride of y'-transforms in the small kernels (my + pad)
  long long N, M;          // nx*ny*nz, mx*my*mz
  int padded;              // boundary padding: the portraits cover only the field of view
  int pxs, pys, pzs;       // field-of-view offsets in decimated samples (padding / decimation)
  int mxf, myf, mzf;       // field-of-view portrait dims
  long long Mf;            // mxf*myf*mzf (= M without padding)
  long long hsz;           // spectrum elements per harmonic = ncls*mx*S = plane*nx
  SepGeo sep;
  UserGeo usr;
  FastDiv f_nmem, f_my, f_mz, f_W, f_S, f_mxS;
};

}  // namespace mh3d
