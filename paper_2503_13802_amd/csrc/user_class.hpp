// The class passes of plans with user PSFs (see user.hpp).
#pragma once
#include "sep.hpp"

namespace mh3d {

// ============================================================================ class pass
// Position of class-layout element p of a (k, x'-block, class, x'-in-block) store, p over
// K * cpw * mx, as offsets into F (line k * cpw + c, element x') and G.
__device__ __forceinline__ void user_g_index(const Geo& g, int fls, int p, int c0, int& fo, int& go) {
  const int k = g.usr.d_cm.div(p), r = p - k * g.cpw * g.mx;
  const int xbi = g.usr.d_cxb.div(r), r2 = r - xbi * g.cpw * g.xb;
  const int c = g.sep.d_xb.div(r2), xi = r2 - c * g.xb;
  fo = (k * g.cpw + c) * fls + xbi * g.xb + xi;
  go = ((k * g.sep.nxb + xbi) * g.ncls + c0 + c) * g.xb + xi;   // K M values, below 2^31
}

// One block: cpw classes, of which a thread owns E consecutive alias members of one folded
// frequency (the members of S / E neighbouring lanes sum to it).  DIR:
//   CLS_FWD     the folded spectra, transformed along x' into G (the small-grid pass turns them
//               into portraits)
//   CLS_ADJ     G' transformed along x', times conj(Hhat), back along x
//   CLS_NORMAL  both (no boundary padding), for the solver's updates, the normal operator
//               and A then A^T.  The folded spectra Fhat_k stay in LDS and the adjoint starts
//               from them: the inverse x' transform, the small-grid inverse and forward
//               transforms and the forward x' transform between the two passes compose to
//               multiplication by M = mx my mz (up to rounding), so
//                 NRM_RESID  R_k = M Fhat_k - Dt_k, Dt = the x' transform of the measured
//                            portraits' small-grid spectra (COL_DATA, in G' as
//                            [k][class][qx'])
//                 NRM_PLAIN  R_k = M Fhat_k                       (normal operator)
//                 NRM_STORE  R_k = M Fhat_k, and G = the inverse x' transform of Fhat (the
//                            small-grid pass turns it into the portraits)
// CB components at once, all of the plan's (0: rounds of one, where the LDS holds no more or a
// thread's spectra of all would take too many registers); the spectra stream through a ring of RK
// harmonics.  With all of them in the ring (K <= RK) the adjoint half reuses it.

// The products are written as fused multiply-adds, so that every instantiation rounds alike (a
// stacked plan with zero blocks equals one plan per scan bitwise).
__device__ __forceinline__ void fma_mul(float2& q, float2 h, float2 u) {     // q += h u
  q.x = fmaf(-h.y, u.y, fmaf(h.x, u.x, q.x));
  q.y = fmaf(h.y, u.x, fmaf(h.x, u.y, q.y));
}
__device__ __forceinline__ void fma_mulcj(float2& q, float2 h, float2 r) {   // q += conj(h) r
  q.x = fmaf(h.y, r.y, fmaf(h.x, r.x, q.x));
  q.y = fmaf(-h.y, r.x, fmaf(h.x, r.y, q.y));
}

// Harmonics of the ring: up to 4, in about 24 registers (the transforms take 80 of the 128 that
// a 1024-thread block leaves a thread).
constexpr int user_ring(int e, int cb) {
  const int n = 12 / (e * cb);
  return n > 4 ? 4 : n < 2 ? 2 : n;
}

template <int E, int CBT, int DIR>
__device__ __forceinline__ void user_class_body(const VolDesc& vd, int lb, int mode, int T) {
  constexpr int CB = CBT ? CBT : 1;
  constexpr int RK = user_ring(E, CB);
  const Geo& g = vd.g;
  int nx = g.nx, mx = g.mx, S = g.S, K = g.K, cpw = g.cpw, nmem = g.nmem, lsx = g.lsx, plane = g.plane,
      fls = g.usr.fls;
  MDiv d_w = g.usr.d_w, d_cbw = g.usr.d_cbw;
  const float2* hs = reinterpret_cast<const float2*>(vd.hs);
  const float2* tw = vd.tw;
  float2* uperm = vd.uperm;
  int offx = vd.off[0], offm = vd.off[3];
  long long hsz = g.hsz, hcs = vd.hs_cstride;
  pin(nx, mx, S, K, cpw, nmem, lsx, plane, fls, d_w, d_cbw, hs, tw, uperm, offx, offm, hsz, hcs);
  // read where they are used
  float2 *G = vd.G, *Gp = vd.Gp;
  const int ncls = g.ncls, C = CBT ? CB : vd.ncomp, tc = vd.T_class;
  const MDiv d_kc = g.usr.d_kc;
  const long long M = g.M;
  extern __shared__ float2 lds[];
  const int W = cpw * nmem, LW = CB * W;
  float2* twx = lds;
  float2* twm = twx + nx;
  float2* U0 = twm + mx;
  float2* U1 = U0 + LW * lsx;
  float2* F0 = U1 + LW * lsx;
  float2* F1 = F0 + K * cpw * fls;
  const int c0 = lb * cpw;
  const bool act = (int)threadIdx.x < tc;
  // this thread's E spectrum elements: all share class cl and folded frequency qxp (a thread
  // beyond them repeats the first one's reads and writes nothing)
  const int e0 = act ? (int)threadIdx.x * E : 0;
  const int per_cls = mx * S;
  const int cl = (int)g.f_mxS.div((uint32_t)e0);
  const int rem = e0 - cl * per_cls;
  const int qxp = (int)g.f_S.div((uint32_t)rem);
  const int within = rem - qxp * S;
  const int LG = S / E;
  int uo[E];   // their places in the lines of a component
  {
    int jx = (int)g.f_nmem.div((uint32_t)within), m = within - jx * nmem;
#pragma unroll
    for (int i = 0; i < E; ++i) {
      uo[i] = (cl * nmem + m) * lsx + qxp + jx * mx;
      if (++m == nmem) { m = 0; ++jx; }
    }
  }
  const int fi0 = cl * fls + qxp, fstep = cpw * fls;   // F of harmonic k at fi0 + k * fstep
  const long long h0 = (long long)c0 * per_cls + e0;
  HLoad<E> hb[RK][CB];
  uint32_t pm[CB];
  auto load_h = [&](int i, int k, int comp) {
#pragma unroll
    for (int c = 0; c < CB; ++c)
      if (k < K && ((pm[c] >> k) & 1u)) hb[i][c].load(hs, (comp + c) * hcs + k * hsz + h0);
  };
  auto ring = [&](int comp) {
#pragma unroll
    for (int c = 0; c < CB; ++c) pm[c] = vd.cmask[comp + c];
#pragma unroll
    for (int i = 0; i < RK; ++i) load_h(i, i, comp);
  };
  const Lines lxs{LW, lsx, T, d_cbw}, lms{K * cpw, fls, T, d_kc};
  const int KCM = K * cpw * mx;
  ring(0);
  const TableLoad<4> tx(tw + offx, nx, T), tm(tw + offm, mx, T);
  const float2* F = F0;
  if constexpr (DIR == CLS_ADJ) {
    batched<8, float2>(KCM,
                       [&](int p) {
                         int fo, go;
                         user_g_index(g, fls, p, c0, fo, go);
                         return ldg(Gp + go);
                       },
                       [&](int p, float2 v) {
                         int fo, go;
                         user_g_index(g, fls, p, c0, fo, go);
                         F0[fo] = v;
                       });
    tx.commit(twx, nx, T);
    tm.commit(twm, mx, T);
    __syncthreads();
    F = line_fft<-1, true>(F0, F1, twm, mx, lms);
  } else {
    uint32_t before = 0;   // harmonics some earlier round has written to F0
    for (int comp = 0; comp < C; comp += CB) {
      if (comp) {
        __syncthreads();   // the last round's U is still being read
        ring(comp);
      }
      const float2* __restrict__ us = uperm + comp * hsz + c0 * nmem;
      batched<8, float2>(nx * LW,
                         [&](int p) {
                           const int xx = d_cbw.div(p), l = p - xx * LW;
                           const int c = CB == 1 ? 0 : d_w.div(l);
                           return ldg(us + c * hsz + (xx * plane + l - c * W));
                         },
                         [&](int p, float2 v) {
                           const int xx = d_cbw.div(p), l = p - xx * LW;
                           U0[__mul24(l, lsx) + xx] = v;
                         });
      if (comp == 0) {
        tx.commit(twx, nx, T);
        tm.commit(twm, mx, T);
        if (DIR == CLS_NORMAL && mode == NRM_RESID) {   // the data term of the block's classes
          batched<4, float2>(KCM,
                             [&](int p) {
                               const int k = g.usr.d_cm.div(p);
                               return ldg(Gp + (k * ncls + c0) * mx + (p - k * cpw * mx));
                             },
                             [&](int p, float2 v) {
                               const int k = g.usr.d_cm.div(p), r = p - k * cpw * mx, c = g.sep.d_mx.div(r);
                               F1[(k * cpw + c) * fls + r - c * mx] = v;
                             });
        }
      }
      __syncthreads();
      const float2* U = line_fft<-1, true>(U0, U1, twx, nx, lxs);
      float2 ur[CB][E];
#pragma unroll
      for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int i = 0; i < E; ++i) ur[c][i] = U[c * W * lsx + uo[i]];
      uint32_t pany = 0;
#pragma unroll
      for (int c = 0; c < CB; ++c) pany |= pm[c];
      // Fhat_k(cl, qx') = sum over the components and the S alias members of Hhat U
      // (a round's sums over the lanes go side by side: each is a chain of cross-lane reads)
      for (int k0 = 0; k0 < K; k0 += RK) {
        float2 acc[RK];
#pragma unroll
        for (int i = 0; i < RK; ++i) {
          acc[i] = make_float2(0.f, 0.f);
#pragma unroll
          for (int c = 0; c < CB; ++c)
            if (k0 + i < K && ((pm[c] >> (k0 + i)) & 1u)) {
#pragma unroll
              for (int t = 0; t < E; ++t) fma_mul(acc[i], hb[i][c].v[t], ur[c][t]);
            }
          if (DIR == CLS_FWD || k0 + i + RK < K) load_h(i, k0 + i + RK, comp);
        }
        for (int o = LG >> 1; o >= 1; o >>= 1) {
#pragma unroll
          for (int i = 0; i < RK; ++i) {
            acc[i].x += __shfl_xor(acc[i].x, o, 64);
            acc[i].y += __shfl_xor(acc[i].y, o, 64);
          }
        }
        if (act && (threadIdx.x & (LG - 1)) == 0) {
#pragma unroll
          for (int i = 0; i < RK; ++i) {
            const int k = k0 + i;
            if (k < K && ((pany >> k) & 1u)) {
              float2& f = F0[fi0 + k * fstep];
              f = ((before >> k) & 1u) ? cadd(f, acc[i]) : acc[i];
            }
          }
        }
      }
      before |= pany;
    }
    __syncthreads();   // Fhat complete; U0 / U1 free
  }
  if constexpr (DIR == CLS_FWD) {
    const float2* R = line_fft<+1, true>(F0, F1, twm, mx, lms);
    for (int p = threadIdx.x; p < KCM; p += T) {
      int fo, go;
      user_g_index(g, fls, p, c0, fo, go);
      stg(G + go, R[fo]);
    }
    return;
  }
  const float Mf = (float)M;
  for (int comp = 0; comp < C; comp += CB) {
    // the forward half's ring still holds the spectra of its last round's last harmonics
    if (comp || (DIR == CLS_NORMAL && (K > RK || CB < C))) {
      if (comp) __syncthreads();   // the last round's lines are still being stored
      ring(comp);
    }
    float2 acc[CB][E];
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
      for (int t = 0; t < E; ++t) acc[c][t] = make_float2(0.f, 0.f);
    for (int k0 = 0; k0 < K; k0 += RK) {
      float2 R[RK];
#pragma unroll
      for (int i = 0; i < RK; ++i) {
        R[i] = make_float2(0.f, 0.f);
        if (k0 + i < K) {
          R[i] = F[fi0 + (k0 + i) * fstep];
          if constexpr (DIR == CLS_NORMAL)
            R[i] = col_resid(mode, Mf, R[i], mode == NRM_RESID ? F1[fi0 + (k0 + i) * fstep] : R[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < RK; ++i) {
#pragma unroll
        for (int c = 0; c < CB; ++c)
          if (k0 + i < K && ((pm[c] >> (k0 + i)) & 1u)) {
#pragma unroll
            for (int t = 0; t < E; ++t) fma_mulcj(acc[c][t], hb[i][c].v[t], R[i]);
          }
        load_h(i, k0 + i + RK, comp);
      }
    }
    // every element of the lines is written exactly once
    if (act) {
#pragma unroll
      for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int t = 0; t < E; ++t) U0[c * W * lsx + uo[t]] = acc[c][t];
    }
    __syncthreads();
    const float2* V = line_fft<+1, true>(U0, U1, twx, nx, lxs);
    float2* __restrict__ vs = uperm + comp * hsz + c0 * nmem;
    for (int p = threadIdx.x; p < nx * LW; p += T) {
      const int xx = d_cbw.div(p), l = p - xx * LW;
      const int c = CB == 1 ? 0 : d_w.div(l);
      stg(vs + c * hsz + (xx * plane + l - c * W), V[__mul24(l, lsx) + xx]);
    }
  }
  if (DIR == CLS_NORMAL && mode == NRM_STORE) {
    // the portraits' small-grid spectra (F0 still holds Fhat: the adjoint only read it)
    const float2* R = line_fft<+1, true>(F0, F1, twm, mx, lms);
    for (int p = threadIdx.x; p < KCM; p += T) {
      int fo, go;
      user_g_index(g, fls, p, c0, fo, go);
      stg(G + go, R[fo]);
    }
  }
}

// grid = ncls / cpw blocks, fin: and one that finishes the previous update.  check_done skips the launch once the volume's solve is done.
// XCD-aware: consecutive class blocks run on one XCD, so the short runs of G, G' and the
// class-layout spectra that neighbouring blocks share are fetched into one L2.
template <int E, int CB, int DIR>
static __global__ __launch_bounds__(1024) void k_user_class(const VolDesc* __restrict__ vds, int check_done, int mode, int fin) {
  const VolDesc& vd = vds[0];
  int T = blockDim.x;
  if (fin && blockIdx.x == gridDim.x - 1) {
    extern __shared__ float2 lds[];
    vol_finish<UPD_FISTA>(vd, T, reinterpret_cast<double*>(lds));
    return;
  }
  if (check_done && solve_over(vd, fin)) return;
  pin(T);
  user_class_body<E, CB, DIR>(vd, plane_of_block(blockIdx.x, gridDim.x - fin), mode, T);
}

// The launchers of one split E (all its component counts and directions).
template <int E, int CB>
static void class_dir(int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk, int mode, int fin) {
  if (dir == CLS_FWD) k_user_class<E, CB, CLS_FWD><<<grid, block, lds, s>>>(vd, chk, mode, fin);
  else if (dir == CLS_ADJ) k_user_class<E, CB, CLS_ADJ><<<grid, block, lds, s>>>(vd, chk, mode, fin);
  else k_user_class<E, CB, CLS_NORMAL><<<grid, block, lds, s>>>(vd, chk, mode, fin);
}
template <int E>
static void class_cb(int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk, int mode, int fin) {
  if constexpr (user_all_at_once(E)) {
    if (cb == 2) return class_dir<E, 2>(dir, grid, block, lds, s, vd, chk, mode, fin);
    if (cb == 3) return class_dir<E, 3>(dir, grid, block, lds, s, vd, chk, mode, fin);
  }
  if (cb) class_dir<E, 1>(dir, grid, block, lds, s, vd, chk, mode, fin);
  else class_dir<E, 0>(dir, grid, block, lds, s, vd, chk, mode, fin);
}

}  // namespace mh3d
