// Separable passes of run-time geometry: the operator of every analytic-PSF plan without
// passes of its own in fast.hpp (any 2^a 3^b grid, decimation and harmonic count, with or
// without boundary padding, single volumes and batches), and the small-grid passes of
// every plan.
//
// The factorisation and the intermediates are fast.hpp's: h_k(x, y, z) = c_k L^(k)(a x)
// E(y, z) (Sec. 3.3 eq. hkapprox), so a plane pass per (x-plane, y residue y0) applies the
// shared (y, z) factor and folds its aliases (P of Sec. 4.1 in Fourier form), and a column
// pass per decimated (y, z) frequency transforms along x and applies every harmonic's x
// factor.  Only the sizes are run-time values here: transform lengths come from a
// block-uniform switch over compile-time stages (lines.hpp), index divisions are one high
// multiply, and whatever fast.hpp keeps in registers of a fixed count is loaded in batches.
//
// What they replaced: per-harmonic 3-D spectra in the alias-class layout (K nx ny (nz/2 + 1)
// values read per application, against K nx + sy my (nz/2 + 1) here), x transforms of all
// sy sz members of a class (one column per class here) and plane passes that repeated
// their z transforms in every workgroup of a plane.
//
// What bounds them: up to about 96^3 each pass is one workgroup's chain of scalar reads, loads,
// LDS transform stages and stores (5 to 8 us a launch whatever its size; a wave alone on
// its SIMD issues one dependent instruction per 8 cycles), beyond that memory: at 256 x 128
// x 128, K = 8, s = (2,2,2) the plane passes move 42 and 38 MB in 15.3 and 18.5 us.
// Measured against the passes they replaced (microseconds per call, before and after):
// A then A^T at 32^3, K = 2: 20.9, 17.0; A and A^T as two calls at 72 x 108 x 48, K = 5, s =
// (2,3,2): 68.4, 35.5 and at 256 x 128 x 128: 243.9, 114; 25 padded updates at 64^3, K =
// 6: 1503, 1150; 16 updates of a batch of 48^3, 64^3, 96 x 96 x 64 and 128 x 128 x 96:
// 2630, 1040 (both solves with the finish riding along, see vol_finish).
#pragma once
#include "kernels.hpp"
#include "lines.hpp"
#include "passes.hpp"

namespace mh3d {

// Loads a block-uniform value into a scalar register here.  The descriptor's fields are read
// through a pointer, and the compiler reads each where it is first used: a dozen dependent
// scalar-cache misses in a row before a pass's first data load.  Each body pins what it uses
// at its start, so the reads are in flight together (with that and twice the threads the
// plane passes at 72 x 108 x 48 went from 9.7 and 9.2 us to 6.7 and 7.0).
template <typename T> __device__ __forceinline__ void pin(T& v) {
  static_assert(sizeof(T) == 4 || sizeof(T) == 8, "a word or a pointer");
  if constexpr (sizeof(T) == 4) {
    int w = __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v));
    asm volatile("" : "+s"(w));
    v = __builtin_bit_cast(T, w);
  } else {
    const uint64_t q = __builtin_bit_cast(uint64_t, v);
    int lo = __builtin_amdgcn_readfirstlane((int)q), hi = __builtin_amdgcn_readfirstlane((int)(q >> 32));
    asm volatile("" : "+s"(lo), "+s"(hi));
    v = __builtin_bit_cast(T, (uint64_t)(uint32_t)lo | ((uint64_t)(uint32_t)hi << 32));
  }
}
template <typename T, typename... R> __device__ __forceinline__ void pin(T& v, R&... r) {
  pin(v);
  pin(r...);
}
__device__ __forceinline__ void pin(MDiv& v) {
  pin(v.m);
  pin(v.d);
}

// Volume and local block of this workgroup: the task table of a batch, or descriptor
// blockIdx.y and block blockIdx.x.
__device__ __forceinline__ void sep_task(const int2* __restrict__ tasks, int& v, int& lb) {
  v = blockIdx.y;
  lb = blockIdx.x;
  if (tasks) {
    const int2 t = tasks[blockIdx.x];
    v = __builtin_amdgcn_readfirstlane(t.x);
    lb = __builtin_amdgcn_readfirstlane(t.y);
  }
}

// A table of n <= NU * blockDim complex values on its way from global memory into LDS: loads
// at construction, stores in commit, so that other loads can be issued in between.
template <int NU>
struct TableLoad {
  float2 r[NU];
  __device__ __forceinline__ TableLoad(const float2* src, int n, int T) {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int i = threadIdx.x + u * T;
      if (i < n) r[u] = ldg(src + i);
    }
  }
  __device__ __forceinline__ void commit(float2* dst, int n, int T) const {
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int i = threadIdx.x + u * T;
      if (i < n) dst[i] = r[u];
    }
  }
};

// V consecutive floats (V = 4 where the row length allows it, else 2: nz and mz are even)
template <int V> __device__ __forceinline__ void ldv(const float* p, float* v) {
  if constexpr (V == 4) {
    const float4 t = ldg(reinterpret_cast<const float4*>(p));
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  } else {
    const float2 t = ldg(reinterpret_cast<const float2*>(p));
    v[0] = t.x; v[1] = t.y;
  }
}
template <int V> __device__ __forceinline__ void stv(float* p, const float* v) {
  if constexpr (V == 4) stg(reinterpret_cast<float4*>(p), make_float4(v[0], v[1], v[2], v[3]));
  else stg(reinterpret_cast<float2*>(p), make_float2(v[0], v[1]));
}

// Plane-pass block b -> (x-plane, y0): the blocks of one XCD (b mod 8) take a run of
// consecutive planes with all their y0 (as fast_plane_of).
__device__ __forceinline__ void sep_plane_of(int nx, int sy, MDiv d_sy, int b, int& x, int& y0) {
  if (nx % 8 == 0) {
    const int i = b >> 3, q = d_sy.div(i);
    y0 = i - q * sy;
    x = (b & 7) * (nx >> 3) + q;
  } else {
    x = d_sy.div(b);
    y0 = b - x * sy;
  }
}

// ============================================================================ plane pass (forward)
// u = b . a on rows y = sy*y1 + y0 of plane x as packed pairs (rows 2j, 2j + 1 in the real
// and imaginary parts of line j of P).  mid() runs once, after the first loads are issued.
template <int V, class Mid>
__device__ __forceinline__ void sep_load_rows(const float* __restrict__ a, const float* __restrict__ bs, int np, int my,
                                              int sy, int y0, int nz, MDiv d_nv, int lsz, bool scaled, float coef,
                                              float2* __restrict__ P, int T, Mid mid) {
  const int nv = nz / V, items = np * nv;
  constexpr int U = 2;   // items in flight: 4 U vector loads
  bool first = true;
  for (int i0 = threadIdx.x; i0 < items || first; i0 += U * T) {
    float va[U][2][V], vb[U][2][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * T;
      if (i < items) {
        const int j = d_nv.div(i), c = i - j * nv;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (2 * j + h < my) {
            const int off = (sy * (2 * j + h) + y0) * nz + V * c;
            ldv<V>(a + off, va[u][h]);
            ldv<V>(bs + off, vb[u][h]);
          } else {
#pragma unroll
            for (int q = 0; q < V; ++q) va[u][h][q] = vb[u][h][q] = 0.f;
          }
        }
      }
    }
    if (first) mid();
    first = false;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * T;
      if (i < items) {
        const int j = d_nv.div(i), c = i - j * nv;
        float2* d2 = P + j * lsz + V * c;
#pragma unroll
        for (int q = 0; q < V; ++q) {
          const float r = scaled ? vb[u][0][q] * (coef * va[u][0][q]) : vb[u][0][q] * va[u][0][q];
          const float m = scaled ? vb[u][1][q] * (coef * va[u][1][q]) : vb[u][1][q] * va[u][1][q];
          d2[q] = make_float2(r, m);
        }
      }
    }
  }
}

// Block (x, y0): the rows' R2C along z, the length-my DFT along y1, then the share
// C(y0; x, q'y, q'z) of the folded plane into cp[y0][x][column].
__device__ __forceinline__ void sep_plane_fwd_body(const VolDesc& vd, int lb, const float* __restrict__ a, int src, int T) {
  int nx = vd.g.nx, ny = vd.g.ny, nz = vd.g.nz, nzh = vd.g.nzh, my = vd.g.my, mz = vd.g.mz, mzh = vd.g.mzh, sy = vd.g.sy,
      sz = vd.g.sz, ncls = vd.g.ncls, np = vd.g.sep.np, lsz = vd.g.sep.lsz, lsy = vd.g.sep.lsy, pbuf = vd.g.sep.pbuf;
  MDiv d_sy = vd.g.sep.d_sy, d_np = vd.g.sep.d_np, d_nzh = vd.g.sep.d_nzh, d_mzh = vd.g.sep.d_mzh;
  MDiv d_nv = vd.g.sep.d_nzv;
  const float* bs = vd.b;
  const float2 *tw = vd.tw, *set = vd.set;
  float2* cp = vd.cp;
  int offz = vd.off[2], offy = vd.off[4];
  pin(nx, ny, nz, nzh, my, mz, mzh, sy, sz, ncls, np, lsz, lsy, pbuf, d_sy, d_np, d_nzh, d_mzh, d_nv, bs, tw, set, cp, offz,
      offy);
  int x, y0;
  sep_plane_of(nx, sy, d_sy, lb, x, y0);
  extern __shared__ float2 lds[];
  float2* twz = lds;
  float2* twy = twz + nz;
  float2* B0 = twy + my;
  float2* B1 = B0 + pbuf;
  const int t = threadIdx.x;
  const float coef = src == SRC_SCALED ? (float)vd.st->scale : 1.f;
  // the first columns' table values (the whole table of a thread where sz <= 4 and the
  // block has at most 2 columns per thread): loaded behind the rows, before the transforms
  constexpr int PC = 2, PZ = 4;
  const float2* __restrict__ et = set + (long long)y0 * my * nzh;
  float2 ev[PC][PZ];
  auto mid = [&]() {
    const TableLoad<2> tz(tw + offz, nz, T), ty(tw + offy, my, T);
#pragma unroll
    for (int i = 0; i < PC; ++i) {
      const int c = t + T * i;
      if (c < ncls) {
        const int qyp = d_mzh.div(c), qzp = c - qyp * mzh;
#pragma unroll
        for (int jz = 0; jz < PZ; ++jz) {
          if (jz < sz) {
            const int qz = qzp + mz * jz;
            ev[i][jz] = ldg(et + qyp * nzh + (2 * qz <= nz ? qz : nz - qz));
          }
        }
      }
    }
    tz.commit(twz, nz, T);
    ty.commit(twy, my, T);
  };
  const long long pb = (long long)x * ny * nz;
  if (nz % 4 == 0) sep_load_rows<4>(a + pb, bs + pb, np, my, sy, y0, nz, d_nv, lsz, src == SRC_SCALED, coef, B0, T, mid);
  else sep_load_rows<2>(a + pb, bs + pb, np, my, sy, y0, nz, d_nv, lsz, src == SRC_SCALED, coef, B0, T, mid);
  __syncthreads();
  const Lines lz{np, lsz, T, d_np}, ly{nzh, lsy, T, d_nzh};
  float2* Z = line_fft<-1>(B0, B1, twz, nz, lz);
  float2* X = Z == B0 ? B1 : B0;
  // line qz, element y1: the half spectrum of a row, split from its packed pair
  auto split = [=](int q, int y1) {
    const float2* row = Z + (y1 >> 1) * lsz;
    const float2 zq = row[q], zm = row[q == 0 ? 0 : nz - q];
    return (y1 & 1) ? make_float2(0.5f * (zq.y + zm.y), -0.5f * (zq.x - zm.x))
                    : make_float2(0.5f * (zq.x + zm.x), 0.5f * (zq.y - zm.y));
  };
  const float2* Y = line_fft_ld<-1>(split, X, Z, twy, my, ly);
  float2* __restrict__ dst = cp + ((long long)y0 * nx + x) * ncls;
  auto column = [&](int c, auto tab) {
    const int qyp = d_mzh.div(c), qzp = c - qyp * mzh;
    const int qym = qyp == 0 ? 0 : my - qyp;
    float sx = 0.f, sy2 = 0.f;
    auto add = [&](int jz, float2 e) {
      const int qz = qzp + mz * jz;
      const bool up = 2 * qz > nz;     // beyond the half spectrum: the Hermitian partner
      float2 v = Y[(up ? nz - qz : qz) * lsy + (up ? qym : qyp)];
      if (up) v.y = -v.y;
      sx += e.x * v.x - e.y * v.y;
      sy2 += e.x * v.y + e.y * v.x;
    };
    tab(qyp, qzp, add);
    stg(dst + c, make_float2(sx, sy2));
  };
  auto from = [&](int qyp, int qzp, int jz0, auto& add) {
    for (int jz = jz0; jz < sz; ++jz) {
      const int qz = qzp + mz * jz;
      add(jz, ldg(et + qyp * nzh + (2 * qz <= nz ? qz : nz - qz)));
    }
  };
#pragma unroll
  for (int i = 0; i < PC; ++i) {
    const int c = t + T * i;
    if (c < ncls)
      column(c, [&](int qyp, int qzp, auto& add) {
#pragma unroll
        for (int jz = 0; jz < PZ; ++jz)
          if (jz < sz) add(jz, ev[i][jz]);
        from(qyp, qzp, PZ, add);
      });
  }
  for (int c = t + T * PC; c < ncls; c += T)
    column(c, [&](int qyp, int qzp, auto& add) { from(qyp, qzp, 0, add); });
}

// src: SRC_PLAIN, SRC_FISTA_Y / SRC_FISTA_NEXT (y^k, y^{k+1} of the volume, a ignored) or SRC_SCALED (a = NULL:
// rho[k & 1]); the solver's sources are skipped once the volume's solve is done.
static __global__ __launch_bounds__(512, 6) void k_sep_plane_fwd(const VolDesc* __restrict__ vds, const int2* __restrict__ tasks,
                                                       const float* __restrict__ a, int src) {
  int lb, v, T = blockDim.x;
  sep_task(tasks, v, lb);
  const VolDesc& vd = vds[v];
  if (src != SRC_PLAIN) {
    const bool fista = src != SRC_SCALED;
    const float *v0 = fista ? vd.y[0] : vd.rho[0], *v1 = fista ? vd.y[1] : vd.rho[1];
    DevState* st = vd.st;
    pin(v0, v1, st, T);
    const int done = st->done, k = st->k + (src == SRC_FISTA_NEXT);
    if (done) {
      set_skip(st, lb == 0);
      return;
    }
    if (fista || !a) a = (k & 1) ? v1 : v0;
  }
  sep_plane_fwd_body(vd, lb, a, src, T);
}

// ============================================================================ column pass
// The sums below are written as fused multiply-adds, so that every instantiation rounds alike
// (a batch and the volume's own solve may run different ones).
__device__ __forceinline__ void fma_acc(float2& q, float f, float2 R) {
  q.x = fmaf(f, R.x, q.x);
  q.y = fmaf(f, R.y, q.y);
}
__device__ __forceinline__ float2 col_resid(int mode, float Mf, float2 v, float2 D) {
  if (mode == NRM_RESID) return make_float2(fmaf(Mf, v.x, -D.x), fmaf(Mf, v.y, -D.y));
  return make_float2(Mf * v.x, Mf * v.y);
}

// The products of kn harmonics from k0 on for the aliases of one (column, q'x), sx = SX of
// them in registers: w the x transform, q the adjoint's sums.  F: this thread's entry of
// harmonic k0 (stride fst per harmonic); D: its data term (residual mode); fk: the x
// factors from harmonic k0.
template <int SX>
__device__ __forceinline__ void sep_products(int mode, int k0, int kn, const float* fk, int nx, int mx, uint32_t imag,
                                             float Mf, const float2* w, float2* q, float2* F, const float2* D, int fst) {
#pragma unroll 2
  for (int i = 0; i < kn; ++i) {
    const bool im = (imag >> (k0 + i)) & 1u;
    float f[SX];
#pragma unroll
    for (int jx = 0; jx < SX; ++jx) f[jx] = fk[i * nx + jx * mx];
    float2 R;
    if (mode != COL_ADJ) {
      float2 a = make_float2(0.f, 0.f);
#pragma unroll
      for (int jx = 0; jx < SX; ++jx) fma_acc(a, f[jx], w[jx]);
      const float2 v = im ? make_float2(-a.y, a.x) : a;
      if (mode == NRM_STORE || mode == COL_FWD) F[i * fst] = v;
      if (mode == COL_FWD) continue;
      R = col_resid(mode, Mf, v, mode == NRM_RESID ? D[i * fst] : v);
    } else {
      R = F[i * fst];
    }
    if (im) R = make_float2(R.y, -R.x);   // conj(i F) R = -i F R
#pragma unroll
    for (int jx = 0; jx < SX; ++jx) fma_acc(q[jx], f[jx], R);
  }
}

// The same for any sx: the aliases stay in LDS (W: the x transform, Q: the sums so far) and go
// through the registers four at a time, `parts` threads sharing a (column, q'x): harmonics part,
// part + parts, ... of the folded values F (between the runs of aliases F holds the sum so
// far), then, after a barrier, runs part, part + parts, ... of the adjoint's sums.  One thread that
// read every alias of every harmonic from LDS in turn was a chain of K sx reads.  Column pass
// of A, of A^T, of both in one, before and after (with a kernel per mode and up to four times the threads):
// 64 x 32 x 32, s = (16,1,1), K = 8: 12.7, 6.9; 16.3, 6.8; 28.4, 11.5 us; 256 x 16 x 16, s = (8,1,1),
// K = 20: 21.9, 12.2; 25.0, 12.8; 40.6, 20.3.
template <int N>
__device__ __forceinline__ void sep_fold_run(int j0, bool last, int k0, int kn, int part, int parts, const float* fk, int nx,
                                             int mx, uint32_t imag, const float2* W, float2* F, int fst) {
  float2 w[N];
#pragma unroll
  for (int j = 0; j < N; ++j) w[j] = W[(j0 + j) * mx];
  fk += j0 * mx;
#pragma unroll 2
  for (int i = part; i < kn; i += parts) {
    float2 a = j0 ? F[i * fst] : make_float2(0.f, 0.f);
#pragma unroll
    for (int j = 0; j < N; ++j) fma_acc(a, fk[i * nx + j * mx], w[j]);
    F[i * fst] = last && ((imag >> (k0 + i)) & 1u) ? make_float2(-a.y, a.x) : a;
  }
}
template <int N>
__device__ __forceinline__ void sep_spread_run(int mode, int j0, int k0, int kn, const float* fk, int nx, int mx, uint32_t imag,
                                               float Mf, float2* Q, const float2* F, const float2* D, int fst) {
  float2 q[N];
#pragma unroll
  for (int j = 0; j < N; ++j) q[j] = Q[(j0 + j) * mx];
  fk += j0 * mx;
#pragma unroll 2
  for (int i = 0; i < kn; ++i) {
    float2 R = F[i * fst];
    if (mode != COL_ADJ) R = col_resid(mode, Mf, R, mode == NRM_RESID ? D[i * fst] : R);
    if ((imag >> (k0 + i)) & 1u) R = make_float2(R.y, -R.x);
#pragma unroll
    for (int j = 0; j < N; ++j) fma_acc(q[j], fk[i * nx + j * mx], R);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) Q[(j0 + j) * mx] = q[j];
}
__device__ __forceinline__ void sep_fold_any(int k0, int kn, int sx, int part, int parts, const float* fk, int nx, int mx,
                                             uint32_t imag, const float2* W, float2* F, int fst) {
  const int s4 = sx & ~3;   // runs of four, then the other one to three
  for (int j0 = 0; j0 < s4; j0 += 4) sep_fold_run<4>(j0, j0 + 4 == sx, k0, kn, part, parts, fk, nx, mx, imag, W, F, fst);
  if (sx & 2) sep_fold_run<2>(s4, s4 + 2 == sx, k0, kn, part, parts, fk, nx, mx, imag, W, F, fst);
  if (sx & 1) sep_fold_run<1>(sx - 1, true, k0, kn, part, parts, fk, nx, mx, imag, W, F, fst);
}
__device__ __forceinline__ void sep_spread_any(int mode, int k0, int kn, int sx, int part, int parts, const float* fk, int nx,
                                               int mx, uint32_t imag, float Mf, float2* Q, const float2* F, const float2* D,
                                               int fst) {
  int r = part;   // runs of four, the last of one to three
  for (; 4 * r + 4 <= sx; r += parts) sep_spread_run<4>(mode, 4 * r, k0, kn, fk, nx, mx, imag, Mf, Q, F, D, fst);
  if (4 * r >= sx) return;
  if (sx & 2) sep_spread_run<2>(mode, 4 * r, k0, kn, fk, nx, mx, imag, Mf, Q, F, D, fst);
  if (sx & 1) sep_spread_run<1>(mode, sx - 1, k0, kn, fk, nx, mx, imag, Mf, Q, F, D, fst);
}

// Block: cpc columns, one thread per (column, q'x) owning the x aliases q'x + mx jx.
// Plain form: every harmonic's folded spectrum in LDS at once (kg = K) and at most 4 x aliases.
// kAny: harmonics in groups of kg, any sx, for the plans that need it (Launch::col_any).
template <int MODE, bool kAny>
__device__ __forceinline__ void sep_col_body(const VolDesc& vd, int lb, int T) {
  constexpr int mode = MODE;
  constexpr bool fwd = mode != COL_ADJ && mode != COL_DATA, adj = mode != COL_FWD && mode != COL_DATA;
  constexpr bool store_g = mode == NRM_STORE || mode == COL_FWD, load_g = mode == COL_ADJ || mode == COL_DATA;
  int nx = vd.g.nx, mx = vd.g.mx, sx = vd.g.sx, sy = vd.g.sy, K = vd.g.K, ncls = vd.g.ncls, xb = vd.g.xb, M = (int)vd.g.M;
  int cpc = vd.g.sep.cpc, lsx = vd.g.sep.lsx, lsm = vd.g.sep.lsm, nxb = vd.g.sep.nxb;
  int kg = kAny ? vd.g.sep.kg : K;
  MDiv d_mx = vd.g.sep.d_mx, d_cpc = vd.g.sep.d_cpc, d_cpcmx = vd.g.sep.d_cpcmx, d_cpcxb = vd.g.sep.d_cpcxb,
       d_xb = vd.g.sep.d_xb, d_kgcpc = vd.g.sep.d_kgcpc;
  const float2 *tw = vd.tw, *cp = vd.cp;
  const float* sfs = vd.sfs;
  float2 *qx = vd.qx, *Gv = vd.G, *Gpv = vd.Gp;
  uint32_t imag = vd.imag_mask;
  int offx = vd.off[0], offm = vd.off[3];
  pin(nx, mx, sx, K, ncls, cpc, lsx, lsm, d_mx, d_cpc, tw, sfs, imag, offx, offm);
  if (fwd) pin(sy, cp, M);
  if (adj) pin(qx);
  if (store_g || load_g) pin(xb, nxb, d_cpcmx, d_cpcxb, d_xb, d_kgcpc, Gv);
  if (load_g || mode == NRM_RESID) pin(Gpv);
  if constexpr (kAny) pin(kg);
  const int c0 = lb * cpc, nc = ncls - c0 < cpc ? ncls - c0 : cpc;
  extern __shared__ float2 lds[];
  float2* twx = lds;
  float2* twm = twx + nx;
  float2* U0 = twm + mx;
  float2* U1 = U0 + cpc * lsx;
  float* fs = reinterpret_cast<float*>(U1 + cpc * lsx);         // x factors [K][nx]
  float2* F1 = reinterpret_cast<float2*>(fs + ((K * nx + 1) & ~1));
  float2* F0 = F1 + kg * cpc * lsm;     // (only where the mode stores or reads them: Launch::lds_col_of)
  const int t = threadIdx.x;
  int tc = t, part = 0, parts = 1;   // kAny: the block's threads are `parts` for each (column, q'x)
  if constexpr (kAny) {
    part = vd.g.sep.d_cpcmx.div(t);
    parts = vd.g.sep.d_cpcmx.div(T);
    tc = t - part * cpc * mx;
  }
  const int cl = d_mx.div(tc), qxp = tc - __mul24(cl, mx);
  const bool act = cl < nc && part == 0;
  const int own = __mul24(cl, lsm) + qxp;   // this thread's entry of a harmonic in F0 / F1
  const int fst = cpc * lsm;                // one harmonic
  auto load_data = [&](int k0, int kn) {   // this thread's data terms into F1 (no barrier: its own entries)
    if (!act) return;
    const float2* __restrict__ Dt = Gpv + (k0 * ncls + c0 + cl) * mx + qxp;   // (at most 2^26 values)
    const int ks = ncls * mx;
    for (int i = 0; i < kn; i += 4) {
      float2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i + u < kn) v[u] = ldg(Dt + (i + u) * ks);
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i + u < kn) F1[own + (i + u) * fst] = v[u];
    }
  };
  // tables and x factors: issued behind the first loads of the data
  auto mid = [&]() {
    const TableLoad<2> tx(tw + offx, nx, T), tm(tw + offm, mx, T);
    if (mode != COL_DATA) {
      const int nf = K * nx;
      constexpr int U = 4;
      for (int i0 = t; i0 < nf; i0 += U * T) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (i0 + u * T < nf) v[u] = ldg(sfs + i0 + u * T);
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (i0 + u * T < nf) fs[i0 + u * T] = v[u];
      }
    }
    tx.commit(twx, nx, T);
    tm.commit(twm, mx, T);
    if (mode == NRM_RESID && kg >= K) load_data(0, K);
  };
  // element p of a group of harmonics from k0 in the order of G's runs -> its entry of F and of G
  auto g_index = [&](int p, int k0, int& fo, int& go) {
    const int k = d_cpcmx.div(p), r = p - __mul24(k, __mul24(cpc, mx));
    const int xbi = d_cpcxb.div(r), r2 = r - __mul24(xbi, __mul24(cpc, xb));
    const int c = d_xb.div(r2), xi = r2 - __mul24(c, xb);
    fo = __mul24(__mul24(k, cpc) + c, lsm) + __mul24(xbi, xb) + xi;
    go = c < nc ? (((k0 + k) * nxb + xbi) * ncls + c0 + c) * xb + xi : -1;
  };
  auto load_group = [&](int k0, int n) {
    const float2* __restrict__ src = mode == COL_DATA ? Gv : Gpv;
    constexpr int U = 4;
    for (int p0 = t; p0 < n; p0 += U * T) {
      float2 v[U];
      int fo[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = p0 + u * T;
        int go = -1;
        fo[u] = -1;
        if (p < n) g_index(p, k0, fo[u], go);
        v[u] = make_float2(0.f, 0.f);
        if (go >= 0) v[u] = ldg(src + go);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (fo[u] >= 0) F0[fo[u]] = v[u];
    }
  };
  if (fwd) {
    // the columns' shares, summed over y0: consecutive threads take the columns of one x
    const int items = cpc * nx;
    const float2* __restrict__ cb = cp + c0;
    const int ys = nx * ncls;
    constexpr int U = 2;
    bool first = true;
    for (int i0 = t; i0 < items || first; i0 += U * T) {
      float2 v[U], p[U][3];
      int at[U], go[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * T;
        const int xx = d_cpc.div(i), c = i - __mul24(xx, cpc);
        at[u] = i < items ? __mul24(c, lsx) + xx : -1;
        go[u] = i < items && c < nc ? xx * ncls + c : -1;
        v[u] = make_float2(0.f, 0.f);
        if (go[u] >= 0) v[u] = ldg(cb + go[u]);
      }
      // kAny: of more than sixteen residues eight shares in flight (32 x 128 x 8, s = (2,64,1), K = 3: A
      // 22.5 us with three, 20.0)
      const int sy3 = kAny && sy > 16 ? 4 : sy;
      for (int y0 = 1; y0 < sy3 || first; y0 += 3) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int h = 0; h < 3; ++h) {
            p[u][h] = make_float2(0.f, 0.f);
            if (y0 + h < sy && go[u] >= 0) p[u][h] = ldg(cb + (y0 + h) * ys + go[u]);
          }
        if (first) mid();
        first = false;
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = cadd(cadd(cadd(v[u], p[u][0]), p[u][1]), p[u][2]);
      }
      if constexpr (kAny) {
        for (int y0 = sy3; y0 < sy; y0 += 8) {
          float2 e[U][8];
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int h = 0; h < 8; ++h) {
              e[u][h] = make_float2(0.f, 0.f);
              if (y0 + h < sy && go[u] >= 0) e[u][h] = ldg(cb + (y0 + h) * ys + go[u]);
            }
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int h = 0; h < 8; ++h) v[u] = cadd(v[u], e[u][h]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (at[u] >= 0) U0[at[u]] = v[u];
    }
  } else {
    if constexpr (!kAny) load_group(0, K * cpc * mx);
    mid();
  }
  __syncthreads();
  const Lines lx{cpc, lsx, T, d_cpc};
  float2* U = U0;
  if (fwd) U = line_fft<-1>(U0, U1, twx, nx, lx);
  float2* Qb = U == U0 ? U1 : U0;      // free: the adjoint's sums
  const float Mf = (float)M;
  float2 w[SXR], q[SXR];
  const int ux = __mul24(cl, lsx) + qxp;
#pragma unroll
  for (int jx = 0; jx < SXR; ++jx) {
    w[jx] = q[jx] = make_float2(0.f, 0.f);
    if (fwd && act && jx < sx) w[jx] = U[ux + jx * mx];
  }
  if constexpr (kAny) {
    if (sx > SXR && act && adj)
      for (int jx = 0; jx < sx; ++jx) Qb[ux + jx * mx] = make_float2(0.f, 0.f);
  }
  auto group = [&](int k0, int kn, const Lines& lm) {
    const int n = kn * cpc * mx;
    float2* F = F0;
    if (load_g) {
      if constexpr (kAny) {
        load_group(k0, n);
        __syncthreads();
      }
      F = line_fft<-1>(F0, F1, twm, mx, lm);
      if (mode == COL_DATA) {
        for (int p = t; p < n; p += T) {
          const int k = d_cpcmx.div(p), r = p - k * cpc * mx, c = d_mx.div(r), qq = r - c * mx;
          if (c < nc) stg(Gpv + ((k0 + k) * ncls + c0 + c) * mx + qq, F[(k * cpc + c) * lsm + qq]);
        }
        return;
      }
    }
    if (mode == NRM_RESID && kg < K) load_data(k0, kn);
    if (act) {
      const float* fk = fs + k0 * nx + qxp;
      float2* Fo = F + own;
      const float2* Do = F1 + own;
      switch (sx) {
        case 1: sep_products<1>(mode, k0, kn, fk, nx, mx, imag, Mf, w, q, Fo, Do, fst); break;
        case 2: sep_products<2>(mode, k0, kn, fk, nx, mx, imag, Mf, w, q, Fo, Do, fst); break;
        case 3: sep_products<3>(mode, k0, kn, fk, nx, mx, imag, Mf, w, q, Fo, Do, fst); break;
        case 4: sep_products<4>(mode, k0, kn, fk, nx, mx, imag, Mf, w, q, Fo, Do, fst); break;
      }
    }
    if constexpr (kAny) {
      if (sx > SXR) {
        const bool live = cl < nc && part < parts;
        const float* fk = fs + k0 * nx + qxp;
        if (fwd && live) sep_fold_any(k0, kn, sx, part, parts, fk, nx, mx, imag, U + ux, F + own, fst);
        if (fwd && adj) __syncthreads();
        if (adj && live)
          sep_spread_any(mode, k0, kn, sx, part, parts, fk, nx, mx, imag, Mf, Qb + ux, F + own, F1 + own, fst);
      }
    }
    if (store_g) {
      if (!act && part == 0 && cl < cpc)   // columns past the last one of the grid: finite values for the transform
        for (int i = 0; i < kn; ++i) F0[own + i * fst] = make_float2(0.f, 0.f);
      __syncthreads();
      const float2* R = line_fft<+1>(F0, F1, twm, mx, lm);
      for (int p = t; p < n; p += T) {
        int fo, go;
        g_index(p, k0, fo, go);
        if (go >= 0) stg(Gv + go, R[fo]);
      }
    }
  };
  if constexpr (kAny) {
    const MDiv d_klcpc = vd.g.sep.d_klcpc;
    for (int k0 = 0; k0 < K; k0 += kg) {
      const int kn = K - k0 < kg ? K - k0 : kg;
      if (k0) __syncthreads();   // the groups share F0 / F1
      group(k0, kn, Lines{kn * cpc, lsm, T, kn == kg ? d_kgcpc : d_klcpc});
    }
  } else {
    group(0, K, Lines{K * cpc, lsm, T, d_kgcpc});
  }
  if (adj) {
    if (cl < cpc && part == 0) {
      if (!kAny || sx <= SXR) {
#pragma unroll
        for (int jx = 0; jx < SXR; ++jx)
          if (jx < sx) Qb[ux + jx * mx] = act ? q[jx] : make_float2(0.f, 0.f);
      } else if (!act) {
        for (int jx = 0; jx < sx; ++jx) Qb[ux + jx * mx] = make_float2(0.f, 0.f);
      }
    }
    __syncthreads();
    const float2* V = line_fft<+1>(Qb, Qb == U0 ? U1 : U0, twx, nx, lx);
    float2* __restrict__ qo = qx + c0;
    for (int i = t; i < cpc * nx; i += T) {
      const int xx = d_cpc.div(i), c = i - __mul24(xx, cpc);
      if (c < nc) stg(qo + xx * ncls + c, V[__mul24(c, lsx) + xx]);
    }
  }
}

// Column block of workgroup b of nb: the workgroups of one XCD (b mod 8) take a run of
// consecutive column blocks, whose short runs of the shares, of G and of Q share cache
// lines (the last nb mod 8 blocks keep their order).
__device__ __forceinline__ int sep_col_block(int b, int nb) {
  const int per = nb >> 3;
  return b < 8 * per ? (b & 7) * per + (b >> 3) : b;
}

// grid.y > 1 runs one descriptor per y-block (the back-projections of single harmonics).  fin: the
// last block (in a batch the tasks of local block -1) finishes the previous update.
template <int MODE, bool ANY>
static __global__ __launch_bounds__(512, ANY ? 4 : 6) void k_sep_col(const VolDesc* __restrict__ vds, const int2* __restrict__ tasks,
                                                                     int check_done, int fin) {
  int lb, v, T = blockDim.x;
  sep_task(tasks, v, lb);
  const VolDesc& vd = vds[v];
  if (fin && (tasks ? lb < 0 : lb == (int)gridDim.x - 1)) {
    extern __shared__ float2 lds[];
    vol_finish<UPD_FISTA>(vd, T, reinterpret_cast<double*>(lds));
    return;
  }
  if (!tasks) lb = sep_col_block(lb, gridDim.x - fin);
  if (check_done && solve_over(vd, fin)) return;
  pin(T);
  sep_col_body<MODE, ANY>(vd, lb, T);
}

// ============================================================================ solver step
// What a plane block ends with.
struct SepRows {
  int ny, nz, my, sy, lsz, y0, T;
  MDiv d_nv;               // divides by the vectors of a row
  const float* bs;         // the plane's sensitivity
};

// User PSFs: nc components in the block, whose packed rows lie zs apart and whose
// sensitivities bstride, added to the plane part (or NULL) of earlier components.
struct UserRows {
  int nc, zs;
  long long bstride;
  const float* part;
};

// The end of a solver step on the block's voxels (rows y = sy*y1 + y0 of plane x), with
// u = b . v from the packed rows Z in LDS: on V
// consecutive voxels along z.  FP64 block partials go to vd.partials[lb].
struct SepStep {
  const float *yv, *rk;    // y^k or w_{t-1}; rho^k
  float *out, *out2;       // rho^{k+1} (or the normal operator's result), y^{k+1}
  float s, lam, alpha, tau, beta1;
  int reg_kind, aw, nx;
};

template <int UPD>
__device__ __forceinline__ SepStep sep_step_of(const VolDesc& vd, const AdjOut& ao, int nx) {
  SepStep c;
  const float *r0 = vd.rho[0], *r1 = vd.rho[1], *y0 = vd.y[0], *y1 = vd.y[1];
  const DevState* st = vd.st;
  c.lam = vd.lam;
  c.alpha = vd.alpha;
  c.reg_kind = vd.reg_kind;
  c.aw = vd.aw;
  c.nx = nx;
  pin(r0, r1, y0, y1, st, c.lam, c.alpha, c.reg_kind, c.aw);
  const int kk = st->k;
  c.s = (UPD == UPD_NORMAL) ? (float)st->scale : 1.f;
  c.tau = (float)st->tau;
  c.beta1 = (float)((double)kk / (kk + 3.0));
  const float* rk = (kk & 1) ? r1 : r0;
  const float* rn = (kk & 1) ? r0 : r1;
  c.rk = rk;
  if constexpr (UPD == UPD_NORMAL) {
    c.yv = ao.yin ? ao.yin : rk;
    c.out = ao.out ? ao.out : const_cast<float*>(rn);
    c.out2 = nullptr;
  } else {
    c.yv = (kk & 1) ? y1 : y0;
    c.out = const_cast<float*>(rn);
    c.out2 = const_cast<float*>((kk & 1) ? y0 : y1);
  }
  return c;
}

// USER: user PSFs (u summed over the components; 2D grids, whose projection axis of length 1
// has no faces and no second differences: every neighbour along it is the voxel itself).
template <int UPD, int V, bool USER = false>
__device__ __forceinline__ void sep_step(const VolDesc& vd, const SepStep& cx, const SepRows& w, const float2* __restrict__ Z,
                                         int x, int lb, double* red, const UserRows& us = UserRows{}) {
  constexpr int NV = UPD == UPD_NORMAL ? 2 : 3;
  const int T = w.T, y0 = w.y0;
  const float s = cx.s, lam = cx.lam, alpha = cx.alpha, tau = cx.tau, beta1 = cx.beta1;
  const bool stencil = cx.reg_kind == 0;
  const int aw = cx.aw, nx = cx.nx, ny = w.ny, nz = w.nz;
  const int PL = ny * nz, pb = x * PL;   // voxel indices fit in 32 bits (at most 256^3)
  const float* __restrict__ yv = cx.yv;
  const float* __restrict__ rk = cx.rk;
  float* __restrict__ out = cx.out;
  float* __restrict__ y_next = cx.out2;
  double acc[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) acc[j] = 0.0;
  auto wrap = [](int q, int n) { return q < 0 ? q + n : (q >= n ? q - n : q); };
  const bool flat = USER && ny == 1;
  auto wrap_y = [&](int q) { return flat ? 0 : wrap(q, ny); };
  const int oxm2 = (wrap(x - 2, nx) - x) * PL, oxm1 = (wrap(x - 1, nx) - x) * PL;
  const int oxp1 = (wrap(x + 1, nx) - x) * PL, oxp2 = (wrap(x + 2, nx) - x) * PL;
  const int nv = nz / V, items = w.my * nv;
  const MDiv d_nv = w.d_nv;
  // items whose loads are in flight together: one (11 vector loads) keeps the pass within
  // 128 registers, two 512-thread blocks per CU
  constexpr int U = 1;
  for (int f0 = threadIdx.x; f0 < items; f0 += U * T) {
    float c[U][V], ym2[U][V], ym1[U][V], yp1[U][V], yp2[U][V], xm2[U][V], xm1[U][V], xp1[U][V], xp2[U][V], rv[U][V], bv[U][V];
    float zl2[U], zl1[U], zr1[U], zr2[U];
    float bx[U][2][V], pv[U][V];   // USER: the other components' sensitivities, the sum so far
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int f = f0 + q * T;
      if (f >= items) break;
      const int y1 = d_nv.div(f), z0 = V * (f - y1 * nv);
      const int y = w.sy * y1 + y0, row = pb + y * nz, i0 = row + z0;
      ldv<V>(yv + i0, c[q]);
      ldv<V>(w.bs + y * nz + z0, bv[q]);
      if constexpr (USER) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
          if (i + 1 < us.nc) ldv<V>(w.bs + (i + 1) * us.bstride + y * nz + z0, bx[q][i]);
        if (us.part) ldv<V>(us.part + y * nz + z0, pv[q]);
      }
      if (UPD == UPD_FISTA) ldv<V>(rk + i0, rv[q]);
      if (stencil) {
        zl2[q] = ldg(yv + row + wrap(z0 - 2, nz));
        zl1[q] = ldg(yv + row + wrap(z0 - 1, nz));
        zr1[q] = ldg(yv + row + wrap(z0 + V, nz));
        zr2[q] = ldg(yv + row + wrap(z0 + V + 1, nz));
        const int pz = pb + z0;
        ldv<V>(yv + pz + wrap_y(y - 2) * nz, ym2[q]);
        ldv<V>(yv + pz + wrap_y(y - 1) * nz, ym1[q]);
        ldv<V>(yv + pz + wrap_y(y + 1) * nz, yp1[q]);
        ldv<V>(yv + pz + wrap_y(y + 2) * nz, yp2[q]);
        ldv<V>(yv + i0 + oxm2, xm2[q]);
        ldv<V>(yv + i0 + oxm1, xm1[q]);
        ldv<V>(yv + i0 + oxp1, xp1[q]);
        ldv<V>(yv + i0 + oxp2, xp2[q]);
      }
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int f = f0 + q * T;
      if (f >= items) break;
      const int y1 = d_nv.div(f), z0 = V * (f - y1 * nv);
      const int y = w.sy * y1 + y0, i0 = pb + y * nz + z0;
      const float2* zr = Z + (y1 >> 1) * w.lsz + z0;
      float zrow[V + 4];
      zrow[0] = zl2[q]; zrow[1] = zl1[q]; zrow[V + 2] = zr1[q]; zrow[V + 3] = zr2[q];
#pragma unroll
      for (int e = 0; e < V; ++e) zrow[e + 2] = c[q][e];
      float o4[V], m4[V];
#pragma unroll
      for (int e = 0; e < V; ++e) {
#pragma clang fp contract(off)
        const int z = z0 + e;
        const float vz = (y1 & 1) ? zr[e].y : zr[e].x;
        float u = __fmul_rn(bv[q][e], vz);
        if constexpr (USER) {
          if (us.part) u += pv[q][e];
#pragma unroll
          for (int i = 0; i < 2; ++i)
            if (i + 1 < us.nc) {
              const float2 zi = zr[(i + 1) * us.zs + e];
              u += bx[q][i][e] * ((y1 & 1) ? zi.y : zi.x);
            }
        }
        float t;
        if (!stencil) {
          t = s * c[q][e];
        } else {
          t = 18.f * (s * c[q][e]);
          t += s * (zrow[e + 4] + zrow[e]) - 4.f * s * (zrow[e + 3] + zrow[e + 1]);
          t += s * (yp2[q][e] + ym2[q][e]) - 4.f * s * (yp1[q][e] + ym1[q][e]);
          t += s * (xp2[q][e] + xm2[q][e]) - 4.f * s * (xp1[q][e] + xm1[q][e]);
        }
        if (alpha > 0.f) {
          const bool shell = x < aw || x >= nx - aw || (!flat && (y < aw || y >= ny - aw)) || z < aw || z >= nz - aw;
          if (shell) t += alpha * (s * c[q][e]);
        }
        const float gr = u + lam * t;
        if constexpr (UPD == UPD_NORMAL) {
          o4[e] = gr;
          acc[0] += (double)(s * c[q][e]) * (double)gr;
          acc[1] += (double)gr * (double)gr;
        } else {
          const float yk = c[q][e];
          const float rn = fmaxf(yk - tau * gr, 0.f);
          o4[e] = rn;
          m4[e] = rn + beta1 * (rn - rv[q][e]);
          const double dd = (double)rn - (double)yk;
          acc[0] += dd * dd;
          acc[1] += (double)rn * (double)rn;
          if (!isfinite(gr) || !isfinite(yk)) acc[2] += 1.0;   // max(NaN, 0) would hide it
        }
      }
      if constexpr (UPD == UPD_NORMAL) {
        stv<V>(out + i0, o4);
      } else {
        stv<V>(out + i0, o4);
        stv<V>(y_next + i0, m4);
      }
    }
  }
  store_step_partials<NV>(vd, acc, red, lb);
}

// ============================================================================ plane pass (adjoint)
// out = b . v on the block's rows, from the packed rows Z (out: the plane).
template <int V, bool USER = false>
__device__ __forceinline__ void sep_store_rows(const SepRows& w, const float2* __restrict__ Z, float* __restrict__ out,
                                               const UserRows& us = UserRows{}) {
  const int nv = w.nz / V, items = w.my * nv;
  constexpr int U = 4;
  for (int i0 = threadIdx.x; i0 < items; i0 += U * w.T) {
    float bv[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * w.T;
      const int y1 = w.d_nv.div(i), c = i - y1 * nv;
      if (i < items) ldv<V>(w.bs + (w.sy * y1 + w.y0) * w.nz + V * c, bv[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * w.T;
      const int y1 = w.d_nv.div(i), c = i - y1 * nv;
      if (i < items) {
        const float2* zr = Z + (y1 >> 1) * w.lsz + V * c;
        float o[V];
#pragma unroll
        for (int q = 0; q < V; ++q) o[q] = bv[u][q] * ((y1 & 1) ? zr[q].y : zr[q].x);
        if constexpr (USER) {
          const int at = (w.sy * y1 + w.y0) * w.nz + V * c;
          if (us.part) {
            float pv[V];
            ldv<V>(us.part + at, pv);
#pragma unroll
            for (int q = 0; q < V; ++q) o[q] += pv[q];
          }
          for (int i = 1; i < us.nc; ++i) {
            float bx[V];
            ldv<V>(w.bs + i * us.bstride + at, bx);
#pragma unroll
            for (int q = 0; q < V; ++q) {
              const float2 zi = zr[i * us.zs + q];
              o[q] += bx[q] * ((y1 & 1) ? zi.y : zi.x);
            }
          }
        }
        stv<V>(out + (w.sy * y1 + w.y0) * w.nz + V * c, o);
      }
    }
  }
}

// Block (x, y0): the residue's half spectrum Q(x, q'y, qz mod mz) conj(Et(y0, q'y, qz)) (Q
// Hermitian over (q'y, q'z)), inverse length-my DFT along y1, C2R along z, then ao.out =
// b . v or the solver step with u = b . v (OUT_STEP_*; skipped once the solve is done).
template <int OUT>
__device__ __forceinline__ void sep_plane_adj_body(const VolDesc& vd, int lb, const AdjOut& ao, int T) {
  constexpr bool kStep = (OUT == OUT_STEP_NORMAL || OUT == OUT_STEP_FISTA);
  int nx = vd.g.nx, ny = vd.g.ny, nz = vd.g.nz, nzh = vd.g.nzh, my = vd.g.my, mz = vd.g.mz, mzh = vd.g.mzh, sy = vd.g.sy,
      ncls = vd.g.ncls, np = vd.g.sep.np, lsz = vd.g.sep.lsz, lsy = vd.g.sep.lsy, pbuf = vd.g.sep.pbuf;
  MDiv d_sy = vd.g.sep.d_sy, d_np = vd.g.sep.d_np, d_nzh = vd.g.sep.d_nzh, d_mz = vd.g.sep.d_mz, d_nv = vd.g.sep.d_nzv;
  const float* bs = vd.b;
  const float2 *tw = vd.tw, *set = vd.set, *qx = vd.qx;
  int offz = vd.off[2], offy = vd.off[4];
  const DevState* st = vd.st;
  pin(nx, ny, nz, nzh, my, mz, mzh, sy, ncls, np, lsz, lsy, pbuf, d_sy, d_np, d_nzh, d_mz, d_nv, bs, tw, set, qx, offz, offy,
      st);
  if constexpr (kStep) {
    if (st->done) return;
  }
  int x, y0;
  sep_plane_of(nx, sy, d_sy, lb, x, y0);
  extern __shared__ float2 lds[];
  __shared__ double red[64];
  float2* twz = lds;
  float2* twy = twz + nz;
  float2* B0 = twy + my;
  float2* B1 = B0 + pbuf;
  const float2* __restrict__ et = set + (long long)y0 * my * nzh;
  const float2* __restrict__ Q = qx + (long long)x * ncls;
  const int ne = my * nzh;
  constexpr int U = 8;
  bool first = true;
  for (int i0 = threadIdx.x; i0 < ne || first; i0 += U * T) {
    float2 ev[U], qv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * T;
      if (i < ne) {
        const int qyp = d_nzh.div(i), qz = i - qyp * nzh;
        const int qzr = qz - d_mz.div(qz) * mz;
        const bool up = 2 * qzr > mz;
        ev[u] = ldg(et + i);
        qv[u] = ldg(Q + (up ? (qyp == 0 ? 0 : my - qyp) * mzh + mz - qzr : qyp * mzh + qzr));
        if (up) qv[u].y = -qv[u].y;
      }
    }
    if (first) {   // the tables' loads go out behind the first batch
      const TableLoad<2> tz(tw + offz, nz, T), ty(tw + offy, my, T);
      tz.commit(twz, nz, T);
      ty.commit(twy, my, T);
      first = false;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * T;
      if (i < ne) {
        const int qyp = d_nzh.div(i), qz = i - qyp * nzh;
        B0[qz * lsy + qyp] = cmulcj(ev[u], qv[u]);   // conj(Et) Q
      }
    }
  }
  SepStep cx;
  if constexpr (OUT == OUT_STEP_NORMAL) cx = sep_step_of<UPD_NORMAL>(vd, ao, nx);
  if constexpr (OUT == OUT_STEP_FISTA) cx = sep_step_of<UPD_FISTA>(vd, ao, nx);
  __syncthreads();
  const Lines lz{np, lsz, T, d_np}, ly{nzh, lsy, T, d_nzh};
  float2* X = line_fft<+1>(B0, B1, twy, my, ly);
  float2* Zb = X == B0 ? B1 : B0;
  // line j = X[2j] + i X[2j+1] with the Hermitian extension beyond nz/2
  auto pack = [=](int j, int q) {
    const bool upper = 2 * q > nz;
    const int qq = upper ? nz - q : q;
    const float2* col = X + qq * lsy + 2 * j;
    float2 xv = col[0];
    float2 yv = 2 * j + 1 < my ? col[1] : make_float2(0.f, 0.f);
    if (qq == 0 || 2 * qq == nz) { xv.y = 0.f; yv.y = 0.f; }
    if (upper) { xv.y = -xv.y; yv.y = -yv.y; }
    return make_float2(xv.x - yv.y, xv.y + yv.x);
  };
  const float2* Z = line_fft_ld<+1>(pack, Zb, X, twz, nz, lz);
  const long long pl = (long long)x * ny * nz;
  const SepRows w{ny, nz, my, sy, lsz, y0, T, d_nv, bs + pl};
  if constexpr (kStep) {
    constexpr int UPD = OUT == OUT_STEP_NORMAL ? UPD_NORMAL : UPD_FISTA;
    if (nz % 4 == 0) sep_step<UPD, 4>(vd, cx, w, Z, x, lb, red);
    else sep_step<UPD, 2>(vd, cx, w, Z, x, lb, red);
  } else {
    if (nz % 4 == 0) sep_store_rows<4>(w, Z, ao.out + pl);
    else sep_store_rows<2>(w, Z, ao.out + pl);
  }
}

// grid.y > 1 (OUT_SCALE_B only): descriptor y and output volume y of consecutive volumes.
// W waves per SIMD: a solver step takes 85 registers, five waves per SIMD: two blocks of 512 threads,
// five of 256 or ten of 128 on a CU.  The form held to 80 (five of them spilled) lets three, six
// or twelve run and is the slower one otherwise, so it runs where it saves a round of blocks on
// the chip.  Microseconds per update with 85 and with 80 registers: 512 threads, 512 blocks (four
// volumes of 64^3) 33.8 and 36.7, 640 (five) 45.9 and 42.5, 1024 (eight) 59.8 and 61.1, 1536 (twelve) 80.5
// and 77.6; 256 threads, 1024 blocks (256 x 64 x 64) 30.7 and 32.9, 1536 (48 of 32^3) 117.7 and 115.8,
// 2048 149.2 and 153.5; 128 threads, 2560 blocks (40 of 32^3) 86.8 and 89.3, 3072 103.8 and 102.3.
template <int OUT, int W>
static __global__ __launch_bounds__(512, W) void k_sep_plane_adj(const VolDesc* __restrict__ vds, const int2* __restrict__ tasks,
                                                       AdjOut ao) {
  int lb, v, T = blockDim.x;
  sep_task(tasks, v, lb);
  const VolDesc& vd = vds[v];
  if constexpr (OUT == OUT_SCALE_B) ao.out += (long long)blockIdx.y * vd.g.N;
  pin(T);
  sep_plane_adj_body<OUT>(vd, lb, ao, T);
}

// ============================================================================ small grid
// Portrait samples are read and written V at a time; with boundary padding one at a time
// through SmallFov (the field of view's rows start at any offset).

// Field-of-view index of sample (row r = xi my + y', z) of x'-block xbi (relative to the
// harmonic's portrait), -1 for a sample of the padding.
struct SmallFov {
  int my, xb, xbi, pxs, pys, pzs, mxf, myf, mzf;
  MDiv d_my;
  __device__ __forceinline__ int at(int r, int z) const {
    const int xi = d_my.div(r), y = r - xi * my;
    const int xf = xbi * xb + xi - pxs, yf = y - pys, zf = z - pzs;
    if ((unsigned)xf >= (unsigned)mxf || (unsigned)yf >= (unsigned)myf || (unsigned)zf >= (unsigned)mzf) return -1;
    return (xf * myf + yf) * mzf + zf;
  }
};

// The block-uniform values of the small-grid passes.
struct SmallGeo {
  int my, mz, mzh, xb, nxb, ncls, spairs, lsmy, lsmz, padded, M, T;
  MDiv d_spairs, d_xbmzh, d_mzh, d_xb, d_mz, d_mzv, d_my, d_nxb;
  const float2* tw;
  int offy, offz;
  __device__ __forceinline__ SmallGeo(const VolDesc& vd, int threads) {
    const Geo& g = vd.g;
    my = g.my; mz = g.mz; mzh = g.mzh; xb = g.xb; nxb = g.sep.nxb; ncls = g.ncls; spairs = g.spairs; lsmy = g.lsmy;
    lsmz = g.sep.lsmz; padded = g.padded; M = (int)g.M; T = threads;
    d_spairs = g.sep.d_spairs; d_xbmzh = g.sep.d_xbmzh; d_mzh = g.sep.d_mzh; d_xb = g.sep.d_xb; d_mzv = g.sep.d_mzv;
    d_my = g.sep.d_my; d_nxb = g.sep.d_nxb; d_mz = g.sep.d_mz;
    tw = vd.tw; offy = vd.off[4]; offz = vd.off[5];
    pin(my, mz, mzh, xb, nxb, ncls, spairs, lsmy, lsmz, padded, M, d_spairs, d_xbmzh, d_mzh, d_xb, d_mz, d_mzv, d_my, d_nxb,
        tw, offy, offz);
  }
  // one LDS buffer: packed row pairs or half-spectrum columns (small_lds of kernels.hpp)
  __device__ __forceinline__ int buffer() const {
    const int a = spairs * lsmz, b = xb * mzh * lsmy;
    return a > b ? a : b;
  }
};

// The class layout G[k][x'-block][column][x'-in-block] of the packed rows in *a.
__device__ __forceinline__ void sep_small_r2c(const SmallGeo& s, float2* a, float2* b, const float2* twy, const float2* twz,
                                              float2* __restrict__ out, int k, int xbi) {
  const Lines lz{s.spairs, s.lsmz, s.T, s.d_spairs}, ly{s.xb * s.mzh, s.lsmy, s.T, s.d_xbmzh};
  float2* Z = line_fft<-1>(a, b, twz, s.mz, lz);
  float2* X = Z == a ? b : a;
  const int mz = s.mz, mzh = s.mzh, my = s.my, lsmz = s.lsmz;
  const MDiv d_mzh = s.d_mzh;
  auto split = [=](int l, int yp) {
    const int xi = d_mzh.div(l), q = l - xi * mzh, r = xi * my + yp;
    const float2* row = Z + (r >> 1) * lsmz;
    const float2 zq = row[q], zm = row[q == 0 ? 0 : mz - q];
    return (r & 1) ? make_float2(0.5f * (zq.y + zm.y), -0.5f * (zq.x - zm.x))
                   : make_float2(0.5f * (zq.x + zm.x), 0.5f * (zq.y - zm.y));
  };
  const float2* Y = line_fft_ld<-1, false, true>(split, X, Z, twy, my, ly);
  float2* __restrict__ dst = out + ((long long)k * s.nxb + xbi) * s.ncls * s.xb;
  const int n = s.ncls * s.xb;
  for (int p = threadIdx.x; p < n; p += s.T) {
    const int c = s.d_xb.div(p), xi = p - c * s.xb;
    const int qy = s.d_mzh.div(c), qz = c - qy * mzh;
    stg(dst + p, Y[(xi * mzh + qz) * s.lsmy + qy]);
  }
}

template <int V>
__device__ __forceinline__ void sep_small_load(const SmallGeo& s, const float* __restrict__ src, float* __restrict__ Pf) {
  const int mv = s.mz / V, items = s.xb * s.my * mv;
  batched<4, float4>(items,
                     [&](int f) {
                       float v[4] = {0.f, 0.f, 0.f, 0.f};
                       ldv<V>(src + V * f, v);
                       return make_float4(v[0], v[1], v[2], v[3]);
                     },
                     [&](int f, float4 v4) {
                       const float v[4] = {v4.x, v4.y, v4.z, v4.w};
                       const int r = s.d_mzv.div(f), c = f - r * mv;
                       float* o = Pf + 2 * ((r >> 1) * s.lsmz + V * c) + (r & 1);
#pragma unroll
                       for (int q = 0; q < V; ++q) o[2 * q] = v[q];
                     });
}

// The small-grid spectra of the portraits r into out (A^T's first pass; the solver's data).
static __global__ __launch_bounds__(512, 6) void k_sep_small_fwd(const VolDesc* __restrict__ vds, const float* __restrict__ r,
                                                       float2* __restrict__ out) {
  const VolDesc& vd = vds[0];
  const Geo& g = vd.g;
  const SmallGeo s(vd, blockDim.x);
  extern __shared__ float2 lds[];
  float2* twy = lds;
  float2* twz = twy + s.my;
  float2* P0 = twz + s.mz;
  const int k = s.d_nxb.div(blockIdx.x), xbi = blockIdx.x - k * s.nxb;
  const int rows = s.xb * s.my, n = rows * s.mz;
  float* Pf = reinterpret_cast<float*>(P0);
  const TableLoad<2> ty(s.tw + s.offy, s.my, s.T), tz(s.tw + s.offz, s.mz, s.T);
  if (!s.padded) {
    const float* src = r + (long long)k * s.M + (long long)xbi * n;
    if (s.mz % 4 == 0) sep_small_load<4>(s, src, Pf);
    else sep_small_load<2>(s, src, Pf);
  } else {   // C^T r is zero outside the field of view
    const SmallFov f{s.my, s.xb, xbi, g.pxs, g.pys, g.pzs, g.mxf, g.myf, g.mzf, s.d_my};
    const float* __restrict__ src = r + (long long)k * g.Mf;
    batched<8, float>(n, [&](int p) {
                        const int rr = s.d_mz.div(p), di = f.at(rr, p - rr * s.mz);
                        return di >= 0 ? ldg(src + di) : 0.f;
                      },
                      [&](int p, float v) {
                        const int rr = s.d_mz.div(p), z = p - rr * s.mz;
                        Pf[2 * ((rr >> 1) * s.lsmz + z) + (rr & 1)] = v;
                      });
  }
  if (rows & 1)
    for (int z = threadIdx.x; z < s.mz; z += s.T) Pf[2 * ((rows >> 1) * s.lsmz + z) + 1] = 0.f;
  ty.commit(twy, s.my, s.T);
  tz.commit(twz, s.mz, s.T);
  __syncthreads();
  sep_small_r2c(s, P0, P0 + s.buffer(), twy, twz, out, k, xbi);
}

template <int V>
__device__ __forceinline__ void sep_small_store(const SmallGeo& s, const float2* __restrict__ Z, float* __restrict__ dst) {
  const int mv = s.mz / V, items = s.xb * s.my * mv;
  for (int f = threadIdx.x; f < items; f += s.T) {
    const int r = s.d_mzv.div(f), c = f - r * mv;
    const float2* zr = Z + (r >> 1) * s.lsmz + V * c;
    float v[V];
#pragma unroll
    for (int q = 0; q < V; ++q) v[q] = (r & 1) ? zr[q].y : zr[q].x;
    stv<V>(dst + V * f, v);
  }
}

// Block (k, x'-block): the portraits of its planes from G, then by epi (kernels.hpp):
// EPI_STORE writes them to d; the padded volumes' EPI_STORE_BACK, EPI_RESID_BACK (minus the
// volume's data) and EPI_BACK also transform the field of view's crop back into G'.
__device__ __forceinline__ void sep_small_inv_body(const VolDesc& vd, int lb, float* __restrict__ d, int epi, int T) {
  const Geo& g = vd.g;
  if ((epi == EPI_RESID_BACK || epi == EPI_BACK) && vd.st->done) return;
  const float2* Gv = vd.G;
  pin(Gv);
  const SmallGeo s(vd, T);
  extern __shared__ float2 lds[];
  float2* twy = lds;
  float2* twz = twy + s.my;
  float2* P0 = twz + s.mz;
  float2* P1 = P0 + s.buffer();
  const int k = s.d_nxb.div(lb), xbi = lb - k * s.nxb;
  const int xb = s.xb, mzh = s.mzh, my = s.my, mz = s.mz, lsmy = s.lsmy, lsmz = s.lsmz;
  const float2* __restrict__ src = Gv + ((long long)k * s.nxb + xbi) * s.ncls * xb;
  const TableLoad<2> ty(s.tw + s.offy, my, T), tz(s.tw + s.offz, mz, T);
  batched<8, float2>(s.ncls * xb, [&](int p) { return ldg(src + p); },
                     [&](int p, float2 v) {
                       const int c = s.d_xb.div(p), xi = p - c * xb;
                       const int qy = s.d_mzh.div(c), qz = c - qy * mzh;
                       P0[(xi * mzh + qz) * lsmy + qy] = v;
                     });
  ty.commit(twy, my, T);
  tz.commit(twz, mz, T);
  __syncthreads();
  const Lines lz{s.spairs, lsmz, T, s.d_spairs}, ly{xb * mzh, lsmy, T, s.d_xbmzh};
  float2* X = line_fft<+1, false, true>(P0, P1, twy, my, ly);
  float2* Zb = X == P0 ? P1 : P0;
  const int rows = xb * my;
  const MDiv d_my = s.d_my;
  auto pack = [=](int j, int q) {
    const bool upper = 2 * q > mz;
    const int qq = upper ? mz - q : q;
    const int r0 = 2 * j, r1 = 2 * j + 1;
    const int x0 = d_my.div(r0), x1 = d_my.div(r1);
    float2 xv = X[(x0 * mzh + qq) * lsmy + r0 - x0 * my];
    float2 yv = r1 < rows ? X[(x1 * mzh + qq) * lsmy + r1 - x1 * my] : make_float2(0.f, 0.f);
    if (qq == 0 || 2 * qq == mz) { xv.y = 0.f; yv.y = 0.f; }
    if (upper) { xv.y = -xv.y; yv.y = -yv.y; }
    return make_float2(xv.x - yv.y, xv.y + yv.x);
  };
  float2* Z = line_fft_ld<+1>(pack, Zb, X, twz, mz, lz);
  const int n = rows * mz;
  if (!s.padded) {
    if (epi == EPI_STORE) {
      float* dst = d + (long long)k * s.M + (long long)xbi * n;
      if (mz % 4 == 0) sep_small_store<4>(s, Z, dst);
      else sep_small_store<2>(s, Z, dst);
    }
    return;
  }
  // boundary padding: only the field-of-view samples are data (C P); the padding's
  // samples of the residual are zero (C^T C P)
  float* Zf = reinterpret_cast<float*>(Z);
  const SmallFov f{my, xb, xbi, g.pxs, g.pys, g.pzs, g.mxf, g.myf, g.mzf, d_my};
  const float* __restrict__ dm = vd.d + (long long)k * g.Mf;
  float* __restrict__ dk = d + (long long)k * g.Mf;
  batched<8, float>(n, [&](int p) {
                      if (epi != EPI_RESID_BACK) return 0.f;
                      const int r = s.d_mz.div(p), di = f.at(r, p - r * mz);
                      return di >= 0 ? ldg(dm + di) : 0.f;
                    },
                    [&](int p, float m) {
                      const int r = s.d_mz.div(p), z = p - r * mz, di = f.at(r, z);
                      float& v = Zf[2 * ((r >> 1) * lsmz + z) + (r & 1)];
                      if (di >= 0 && (epi == EPI_STORE || epi == EPI_STORE_BACK)) stg(dk + di, v);
                      if (epi == EPI_RESID_BACK) v = v - m;
                      if (di < 0) v = 0.f;
                    });
  if (epi == EPI_STORE) return;
  if (rows & 1)
    for (int z = threadIdx.x; z < mz; z += T) Zf[2 * ((rows >> 1) * lsmz + z) + 1] = 0.f;
  __syncthreads();
  sep_small_r2c(s, Z, Z == P0 ? P1 : P0, twy, twz, vd.Gp, k, xbi);
}
static __global__ __launch_bounds__(512, 6) void k_sep_small_inv(const VolDesc* __restrict__ vds, const int2* __restrict__ tasks,
                                                       float* __restrict__ d, int epi) {
  int lb, v, T = blockDim.x;
  sep_task(tasks, v, lb);
  const VolDesc& vd = vds[v];
  pin(T);
  sep_small_inv_body(vd, lb, d, epi, T);
}

// A then A^T after the column pass (NRM_STORE): blocks [0, nbp = sy nx) run the adjoint plane
// pass (ao.out = b . v), the others the small-grid inverse pass that writes d.
static __global__ __launch_bounds__(512, 5) void k_sep_adj_and_store(const VolDesc* __restrict__ vds, AdjOut ao,
                                                           float* __restrict__ d, int nbp) {
  const VolDesc& vd = vds[0];
  int T = blockDim.x;
  pin(T);
  if ((int)blockIdx.x < nbp) sep_plane_adj_body<OUT_SCALE_B>(vd, blockIdx.x, ao, T);
  else sep_small_inv_body(vd, blockIdx.x - nbp, d, EPI_STORE, T);
}

}  // namespace mh3d
