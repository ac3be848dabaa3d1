// Passes of plans with user PSFs (scalar and vector model, 2D grids, with or without
// boundary padding): complex spectra in the class layout (geo.hpp), which no factorisation
// shortens.
//
//   plane pass   one x-plane (a share of its columns or rows): R2C along z, DFT along y,
//                into the class layout; and back
//   class pass   cpw classes: DFT along x of their members, the products with every
//                harmonic's spectrum summed over the alias members, and the transforms of the
//                folded spectra along x'; and back
//
// The transforms are those of the separable passes (lines.hpp), a class-layout position is
// looked up in a table instead of divided out, descriptor fields are pinned, and the
// components of the vector model go through a pass together where the LDS holds them: each
// pass is a chain of loads, transform stages and stores that one workgroup per CU (or less)
// cannot hide, and taking components one after another tripled it.
// Measured against the passes these replaced, microseconds per call: A and A^T as two calls at
// 96 x 96 x 64, K = 7, three components 126.2, 77.6 (forward plane pass 32.1, 13.0; adjoint 31.7,
// 12.8; class passes 25.6 and 22.0, 18.1 and 18.0); 30 updates of a 128 x 256 image of 7
// harmonics from two scans 1817, 965 (step and next forward pass 23.8, 12.3 in one launch; class
// passes 29.2 as two launches, 14.8 as one; the finish riding along, see vol_finish); a scalar
// 256 x 256 image 20.7, 20.2 (A) and 20.4, 18.0 (A^T).
#pragma once
#include "sep.hpp"

namespace mh3d {

// ============================================================================ plane pass (forward)
// u = b_i . a for the components i < nc (bs + i N) on every row of a plane, as packed pairs
// (rows 2j, 2j + 1 in the real and imaginary parts of line i np + j of P).  RAW: a alone.
// mid() runs once, after the first loads are issued.
template <int V, bool RAW, class Mid>
__device__ __forceinline__ void user_load_rows(const float* __restrict__ a, const float* __restrict__ bs, long long N, int nc,
                                               int np, int ny, int nz, MDiv d_np, MDiv d_nv, int lsz, bool scaled, float coef,
                                               float2* __restrict__ P, int T, Mid mid) {
  const int nv = nz / V, items = nc * np * nv;
  constexpr int U = 2;   // items in flight: 4 U vector loads
  bool first = true;
  for (int i0 = threadIdx.x; i0 < items || first; i0 += U * T) {
    float va[U][2][V], vb[U][2][V];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * T;
      if (i < items) {
        const int l = d_nv.div(i), z = V * (i - l * nv), c = nc == 1 ? 0 : d_np.div(l), y = 2 * (l - c * np);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int q = 0; q < V; ++q) va[u][h][q] = 0.f, vb[u][h][q] = 1.f;
          if (y + h < ny) {
            ldv<V>(a + (y + h) * nz + z, va[u][h]);
            if constexpr (!RAW) ldv<V>(bs + c * N + (y + h) * nz + z, vb[u][h]);
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
        const int l = d_nv.div(i), z = V * (i - l * nv);
        float2* d2 = P + l * lsz + z;
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

// cb components from comp on (one, or all C with one workgroup per plane) of workgroup h of
// x-plane x; a the volume.
template <bool RAW>
__device__ __forceinline__ void user_plane_fwd_body(const VolDesc& vd, int x, int h, int comp, int cb,
                                                    const float* __restrict__ a, bool scaled, int T) {
  int ny = vd.g.ny, nz = vd.g.nz, nzh = vd.g.nzh, np = vd.g.npairs, lsy = vd.g.lsy, lsz = vd.g.sep.lsz, plane = vd.g.plane,
      ps = vd.g.ps, pl = vd.g.usr.pl;
  MDiv d_np = vd.g.usr.d_np, d_nv = vd.g.sep.d_nzv, d_lo = vd.g.usr.d_qlo, d_hi = vd.g.usr.d_qhi;
  MDiv d_cnp = vd.g.usr.d_cnp, d_cq = vd.g.usr.d_ycols;   // of cb = C components and every column
  const float* b = vd.b;
  const float2* tw = vd.tw;
  const int* cidx = vd.cidx;
  float2* uperm = vd.uperm;
  int offz = vd.off[2], offy = vd.off[1];
  long long hsz = vd.g.hsz, N = vd.g.N;
  const DevState* st = vd.st;
  pin(ny, nz, nzh, np, lsy, lsz, plane, ps, pl, d_np, d_nv, d_lo, d_hi, d_cnp, d_cq, b, tw, cidx, uperm, offz, offy, hsz, N, st);
  extern __shared__ float2 lds[];
  float2* twz = lds;
  float2* twy = twz + nz;
  float2* B0 = twy + ny;
  float2* B1 = B0 + cb * pl;
  // ps workgroups per plane: all of them transform every row along z, workgroup h then takes
  // the y-transforms of the columns [q0, q1)
  const int q0 = h * nzh / ps, q1 = (h + 1) * nzh / ps, nq = q1 - q0;
  const float coef = scaled ? (float)st->scale : 1.f;
  const long long pb = (long long)x * ny * nz;
  const int t = threadIdx.x;
  constexpr int PC = 8;   // table entries held from the start
  int ce[PC];
  auto mid = [&]() {
    const TableLoad<2> tz(tw + offz, nz, T), ty(tw + offy, ny, T);
#pragma unroll
    for (int i = 0; i < PC; ++i) ce[i] = t + T * i < plane ? ldg(cidx + t + T * i) : 0;
    tz.commit(twz, nz, T);
    ty.commit(twy, ny, T);
  };
  const MDiv d_q = cb > 1 ? d_cq : nq == (int)d_lo.d ? d_lo : d_hi;   // divides by cb * nq
  {
    const float* bs = b + comp * N + pb;
    if (nz % 4 == 0) user_load_rows<4, RAW>(a + pb, bs, N, cb, np, ny, nz, d_np, d_nv, lsz, scaled, coef, B0, T, mid);
    else user_load_rows<2, RAW>(a + pb, bs, N, cb, np, ny, nz, d_np, d_nv, lsz, scaled, coef, B0, T, mid);
    __syncthreads();
    float2* Z = line_fft<-1>(B0, B1, twz, nz, Lines{cb * np, lsz, T, cb > 1 ? d_cnp : d_np});
    float2* X = Z == B0 ? B1 : B0;
    // line l = column q0 + l of a component (cb > 1: i nzh + column), element y: the half
    // spectrum of a row, split from its packed pair
    auto split = [=](int l, int y) {
      const int i = cb > 1 ? d_lo.div(l) : 0, q = q0 + l - i * nzh;   // cb > 1: ps = 1, d_lo divides by nzh
      const float2* row = Z + __mul24((y >> 1) + i * np, lsz);
      const float2 zq = row[q], zm = row[q == 0 ? 0 : nz - q];
      return (y & 1) ? make_float2(0.5f * (zq.y + zm.y), -0.5f * (zq.x - zm.x))
                     : make_float2(0.5f * (zq.x + zm.x), 0.5f * (zq.y - zm.y));
    };
    const float2* Y = line_fft_ld<-1>(split, X, Z, twy, ny, Lines{cb * nq, lsy, T, d_q});
    float2* __restrict__ dst = uperm + comp * hsz + (long long)x * plane;
    auto put = [&](int e, int c) {
      const int col = ((c >> 16) & 0xff) - q0;
      if ((unsigned)col >= (unsigned)nq) return;
      for (int i = 0; i < cb; ++i) {
        float2 v = Y[__mul24(col + i * nzh, lsy) + (c & 0xffff)];
        if (c & CIDX_CONJ) v.y = -v.y;
        stg(dst + i * hsz + e, v);
      }
    };
#pragma unroll
    for (int i = 0; i < PC; ++i)
      if (t + T * i < plane) put(t + T * i, ce[i]);
    for (int e = t + T * PC; e < plane; e += T) put(e, ldg(cidx + e));
  }
}

// grid = components x ps x nx (a raw source has one component).  SRC_FISTA_Y and
// SRC_FISTA_NEXT read y^k and y^{k+1} of the volume (a ignored); the solver's sources are skipped once the volume's solve is done.
template <bool RAW>
static __global__ __launch_bounds__(512, 4) void k_user_plane_fwd(const VolDesc* __restrict__ vds, const float* __restrict__ a,
                                                                  int src) {
  const VolDesc& vd = vds[0];
  int nx = vd.g.nx, per = vd.g.ps * nx, T = blockDim.x;
  const bool fista = src == SRC_FISTA_Y || src == SRC_FISTA_NEXT;
  const float *v0 = fista ? vd.y[0] : vd.rho[0], *v1 = fista ? vd.y[1] : vd.rho[1];
  DevState* st = vd.st;
  pin(nx, per, T, v0, v1, st);
  if (fista || src == SRC_SCALED) {
    const int done = st->done, k = st->k + (src == SRC_FISTA_NEXT);
    if (done) {
      set_skip(st, blockIdx.x == 0);
      return;
    }
    if (fista || !a) a = (k & 1) ? v1 : v0;
  }
  const int comp = blockIdx.x / per, r = blockIdx.x - comp * per, h = r / nx;
  user_plane_fwd_body<RAW>(vd, plane_of_block(r - h * nx, nx), h, comp, 1, a, src == SRC_SCALED, T);
}

// ============================================================================ plane pass (adjoint)
// Workgroup h of x-plane x: the class layout back into half planes, inverse DFT along y of
// every column, C2R along z of the row pairs [j0, j1), then sum_i b_i . v_i over the
// components: ao.out (OUT_SCALE_B) or the solver step (OUT_STEP_*; its FP64 sums in
// vd.partials[lb]).  pcb components at a time; what earlier rounds summed waits in the output
// (vd.u for a step), written and read by the same thread.
// One round, of the components from comp on.  ROUNDS: pcb < C, else a round holds them all.
template <int OUT, bool ROUNDS>
__device__ __forceinline__ void user_plane_adj_round(const VolDesc& vd, int lb, const AdjOut& ao, int T, int comp) {
  constexpr bool kStep = (OUT == OUT_STEP_NORMAL || OUT == OUT_STEP_FISTA);
  int nx = vd.g.nx, ny = vd.g.ny, nz = vd.g.nz, nzh = vd.g.nzh, np = vd.g.npairs, lsy = vd.g.lsy, lsz = vd.g.sep.lsz,
      plane = vd.g.plane, ps = vd.g.ps, pl = vd.g.usr.pl, pcb = vd.g.usr.pcb;
  MDiv d_y = vd.g.usr.d_ycols, d_nv = vd.g.sep.d_nzv;
  const float* b = vd.b;
  const float2 *tw = vd.tw, *uperm = vd.uperm;
  const int* cidx = vd.cidx;
  float* up = vd.u;
  int offz = vd.off[2], offy = vd.off[1];
  long long hsz = vd.g.hsz, N = vd.g.N;
  const DevState* st = vd.st;
  pin(nx, ny, nz, nzh, np, lsy, lsz, plane, ps, pl, pcb, d_y, d_nv, b, tw, uperm, cidx, up, offz, offy, hsz, N, st);
  if constexpr (kStep) {
    if (st->done) return;
  }
  const int h = lb / nx, x = plane_of_block(lb - h * nx, nx);
  const int j0 = h * np / ps, nj = (h + 1) * np / ps - j0;
  const bool more = nj == (int)vd.g.usr.d_j1hi.d;
  const MDiv d_nj = more ? vd.g.usr.d_jhi : vd.g.usr.d_jlo;     // divides by pcb * nj
  const MDiv d_j1 = more ? vd.g.usr.d_j1hi : vd.g.usr.d_j1lo;   // divides by nj
  extern __shared__ float2 lds[];
  __shared__ double red[64];
  float2* twz = lds;
  float2* twy = twz + nz;
  float2* B0 = twy + ny;
  float2* B1 = B0 + pcb * pl;
  const int ysz = nzh * lsy;
  const int rows = 2 * (j0 + nj) < ny ? 2 * nj : ny - 2 * j0;
  const long long pb = (long long)x * ny * nz;
  SepStep cx;
  if constexpr (OUT == OUT_STEP_NORMAL) cx = sep_step_of<UPD_NORMAL>(vd, ao, nx);
  if constexpr (OUT == OUT_STEP_FISTA) cx = sep_step_of<UPD_FISTA>(vd, ao, nx);
  {
    constexpr int U = 2;
    bool first = true;
    const float2* __restrict__ src = uperm + comp * hsz + (long long)x * plane;
    for (int e0 = threadIdx.x; e0 < plane || first; e0 += U * T) {
      int c[U];
      float2 v[U][3];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * T;
        if (e < plane) {
          c[u] = ldg(cidx + e);
#pragma unroll
          for (int i = 0; i < 3; ++i)
            if (i < pcb) v[u][i] = ldg(src + i * hsz + e);
        }
      }
      if (first) {
        const TableLoad<2> tz(tw + offz, nz, T), ty(tw + offy, ny, T);
        tz.commit(twz, nz, T);
        ty.commit(twy, ny, T);
        first = false;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = e0 + u * T;
        if (e < plane && (c[u] & CIDX_OWNER)) {
          const int pos = __mul24((c[u] >> 16) & 0xff, lsy) + (c[u] & 0xffff);
#pragma unroll
          for (int i = 0; i < 3; ++i)
            if (i < pcb) B0[i * ysz + pos] = make_float2(v[u][i].x, (c[u] & CIDX_CONJ) ? -v[u][i].y : v[u][i].y);
        }
      }
    }
    __syncthreads();
    float2* X = ny == 1 ? B0 : line_fft<+1>(B0, B1, twy, ny, Lines{pcb * nzh, lsy, T, d_y});
    float2* Zb = X == B0 ? B1 : B0;
    // line i nj + j of component comp + i: X[2j] + i X[2j + 1] with the Hermitian extension
    auto pack = [=](int l, int q) {
      const int i = pcb == 1 ? 0 : d_j1.div(l), j = l - i * nj + j0;
      const bool upper = 2 * q > nz;
      const int qq = upper ? nz - q : q;
      const float2* col = X + i * ysz + __mul24(qq, lsy) + 2 * j;
      float2 xv = col[0];
      float2 yv = 2 * j + 1 < ny ? col[1] : make_float2(0.f, 0.f);
      if (qq == 0 || 2 * qq == nz) { xv.y = 0.f; yv.y = 0.f; }
      if (upper) { xv.y = -xv.y; yv.y = -yv.y; }
      return make_float2(xv.x - yv.y, xv.y + yv.x);
    };
    const float2* Z = line_fft_ld<+1>(pack, Zb, X, twz, nz, Lines{pcb * nj, lsz, T, d_nj});
    const SepRows w{ny, nz, rows, 1, lsz, 2 * j0, T, d_nv, b + comp * N + pb};
    const bool last = !ROUNDS || comp + pcb == vd.ncomp;
    float* part = (kStep ? up : ao.out) + pb;   // the sum so far
    const UserRows us{pcb, nj * lsz, N, ROUNDS && comp ? part : nullptr};
    if (!kStep || !last) {
      if (nz % 4 == 0) sep_store_rows<4, true>(w, Z, part, us);
      else sep_store_rows<2, true>(w, Z, part, us);
    } else if constexpr (kStep) {
      constexpr int UPD = OUT == OUT_STEP_NORMAL ? UPD_NORMAL : UPD_FISTA;
      if (nz % 4 == 0) sep_step<UPD, 4, true>(vd, cx, w, Z, x, lb, red, us);
      else sep_step<UPD, 2, true>(vd, cx, w, Z, x, lb, red, us);
    }
  }
}

// The descriptor through a pointer that the compiler cannot see through: a round reads its
// fields anew instead of keeping forty scalars alive over the loop (they spilled).
__device__ __forceinline__ const VolDesc& reread(const VolDesc& vd) {
  const VolDesc* p = &vd;
  asm volatile("" : "+s"(p));
  return *p;
}
template <int OUT, bool ROUNDS>
__device__ __forceinline__ void user_plane_adj_body(const VolDesc& vd, int lb, const AdjOut& ao, int T) {
  if constexpr (!ROUNDS) {
    user_plane_adj_round<OUT, false>(vd, lb, ao, T, 0);
  } else {
    const int C = vd.ncomp, pcb = vd.g.usr.pcb;
    for (int comp = 0; comp < C; comp += pcb) {
      if (comp) __syncthreads();   // the last round's rows are still being read
      user_plane_adj_round<OUT, true>(reread(vd), lb, ao, T, comp);
    }
  }
}

// grid = ps * nx blocks
template <int OUT, bool ROUNDS>
static __global__ __launch_bounds__(1024) void k_user_plane_adj(const VolDesc* __restrict__ vds, AdjOut ao) {
  int T = blockDim.x;
  pin(T);
  user_plane_adj_body<OUT, ROUNDS>(vds[0], blockIdx.x, ao, T);
}

// A solver update's adjoint plane pass and step (OUT_STEP_FISTA), then, in the same
// workgroup, the next update's forward plane pass on the y^{k+1} the step just wrote: a
// plane's forward pass needs only that plane's y, so with one workgroup per x-plane (ps = 1) no
// other block is awaited, and the next update starts at its class pass.  If this step ends the
// solve, the extra forward pass is unused.  grid = nx blocks (ps must be 1).
template <bool ROUNDS>
static __global__ __launch_bounds__(1024) void k_user_step_and_fwd(const VolDesc* __restrict__ vds, AdjOut ao) {
  const VolDesc& vd = vds[0];
  int T = blockDim.x;
  pin(T);
  if (vd.st->done) {
    set_skip(vd.st, blockIdx.x == 0);   // (the next update's forward pass is in this launch)
    return;
  }
  const float* ynext = vd.y[(vd.st->k + 1) & 1];
  user_plane_adj_body<OUT_STEP_FISTA, ROUNDS>(vd, blockIdx.x, ao, T);
  __syncthreads();   // the block's stores of y^{k+1} are visible to it; the LDS is free
  if constexpr (!ROUNDS) {
    user_plane_fwd_body<false>(vd, plane_of_block(blockIdx.x, vd.g.nx), 0, 0, vd.g.usr.pcb, ynext, false, T);
  } else {
    const int x = plane_of_block(blockIdx.x, vd.g.nx), pcb = vd.g.usr.pcb;
    for (int comp = 0; comp < vd.ncomp; comp += pcb) {
      if (comp) __syncthreads();   // the last round's columns are still being read
      user_plane_fwd_body<false>(reread(vd), x, 0, comp, pcb, ynext, false, T);
    }
  }
}

// A then A^T after the fused class pass: both halves read only what that pass wrote, so
// blocks [0, ps nx) run the adjoint plane pass (ao.out = sum_i b_i . v_i) while the others run
// the small-grid inverse pass that writes the portraits d.  The plane blocks come first (their
// XCD-aware plane order assumes block ids 0 .. ps nx - 1).  Both bodies loop over blockDim
// (512 or 1024).
template <bool ROUNDS>
static __global__ __launch_bounds__(1024) void k_user_adj_and_store(const VolDesc* __restrict__ vds, AdjOut ao,
                                                                    float* __restrict__ d) {
  const VolDesc& vd = vds[0];
  const int nplane = vd.g.ps * vd.g.nx;
  int T = blockDim.x;
  pin(T);
  if ((int)blockIdx.x < nplane) user_plane_adj_body<OUT_SCALE_B, ROUNDS>(vd, blockIdx.x, ao, T);
  else sep_small_inv_body(vd, blockIdx.x - nplane, d, EPI_STORE, T);
}

}  // namespace mh3d
