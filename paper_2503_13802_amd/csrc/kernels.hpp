// HIP kernels of the MH3D operator A = P H B, its adjoint and the solver updates for plans
// with user PSF arrays (full spectra), and the pieces shared with the separable passes of
// analytic plans (sep.hpp, fast.hpp).
//
// Pipeline of one application of A (Sec. 4.1 eq. dN, Table tab:ops):
//   plane_fwd  one workgroup per x-plane: u = b . rho, 2-D R2C FFT over (y, z) in
//              LDS, written in the alias-class layout (see geo.hpp)            [B, F_yz]
//   class_fwd  one workgroup per group of classes: FFT along x, multiply by every
//              precomputed spectrum H_k, fold the aliases (P in Fourier form),
//              inverse FFT along the decimated x                                [F_x, H, P]
//   small_inv  (sep.hpp) one workgroup per (k, block of x'): 2-D C2R over (y', z') of the
//              decimated spectrum -> portrait d_k (optionally minus data)         [F^-1]
// The adjoint runs the same passes backwards (small_fwd, class_adj, plane_adj):
// F(P^T r) tiles the small spectrum, H_k^T multiplies by conj(H_k), and the sum
// over k happens in registers before the inverse x FFT.
//
// Spectra are scaled by 1/N at plan time, so every FFT here is unnormalised.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fft_lds.hpp"
#include "geo.hpp"
#include "langevin_dev.hpp"

namespace mh3d {

// ============================================================================ helpers
// Class-layout index of the full-grid half-plane position (qy, qz), qz <= nz/2,
// and whether the stored value is the conjugate.
__device__ __forceinline__ int class_index_of(const Geo& g, int qy, int qz, bool& cj) {
  const int qzr = (int)g.f_mz.mod((uint32_t)qz);
  int yy = qy, zz = qz;
  cj = false;
  if (2 * qzr > g.mz) {            // stored as the conjugate of (ny - qy, nz - qz)
    yy = qy == 0 ? 0 : g.ny - qy;
    zz = g.nz - qz;
    cj = true;
  }
  const int yq = (int)g.f_my.div((uint32_t)yy), zq = (int)g.f_mz.div((uint32_t)zz);
  const int c = (yy - yq * g.my) * g.mzh + (zz - zq * g.mz);
  const int m = yq * g.sz + zq;
  return c * g.nmem + m;
}

// LDS line strides: transforms run on contiguous lines padded to an odd length so
// that the transposing passes between them hit distinct banks.
__host__ __device__ inline int pad_odd(int n) { return (n & 1) ? n : n + 1; }

// Complex elements of one LDS buffer of the x-plane kernels: packed row pairs
// [npairs][lsz], half-spectrum columns [nzh][lsy], or a staged class-layout plane.
__host__ __device__ inline int plane_lds(const Geo& g) {
  const int a = g.npairs * pad_odd(g.nz), b = g.nzh * g.lsy, c = g.plane;
  const int m = a > b ? a : b;
  return m > c ? m : c;
}
// One LDS buffer of the small-grid kernels: row pairs [spairs][lsmz] or
// columns [xb*mzh][lsmy].
__host__ __device__ inline int small_lds(const Geo& g) {
  const int a = g.spairs * pad_odd(g.mz), b = g.xb * g.mzh * g.lsmy;
  return a > b ? a : b;
}

// Deterministic block reduction of NV doubles; result valid in thread 0.
template <int NV>
__device__ __forceinline__ void block_reduce_f64(double* v, double* sh) {
  // sh: >= NV * (blockDim.x / 64 + 1) doubles
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    double x = v[j];
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    v[j] = x;
  }
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < NV; ++j) sh[j * nw + wid] = v[j];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += sh[j * nw + w];
      v[j] = s;
    }
  }
  __syncthreads();
}

// Strided block loop with U independent loads in flight per thread: all loads of a
// batch are issued before any result is used (a plain strided loop would wait for
// each load in turn).
template <int U, typename T, typename LD, typename ST>
__device__ __forceinline__ void batched(int n, LD ld, ST st) {
  const int nt = blockDim.x;
  for (int p0 = threadIdx.x; p0 < n; p0 += U * nt) {
    T v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = p0 + u * nt;
      if (p < n) v[u] = ld(p);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = p0 + u * nt;
      if (p < n) st(p, v[u]);
    }
  }
}

// x-plane (or other unit) handled by block b of nx: consecutive units go to the same
// XCD (blocks are dealt round-robin over the 8 XCDs), so neighbours share an L2.
__device__ __forceinline__ int plane_of_block(int b, int nx) {
  if (nx % 8) return b;
  return (b & 7) * (nx >> 3) + (b >> 3);
}

// Solver / power-iteration state kept in device memory so that a captured
// sequence of launches can be replayed.
struct DevState {
  int k;            // FISTA iteration index of the current y^k
  int done;         // 1 once r_k <= tol or the iteration cap was reached
  int last_k;       // iteration of the last performed update
  int counter;      // arrivals for the last-block reduction
  double tau, lam, tol;
  int kmax;         // last iteration index allowed (k0 + max_iter - 1)
  int skip;         // `done` as the launch before a pass with a finish beside it saw it
  double rel_step;  // last r_k
  double scale;     // power iteration: 1/||w_{t-1}||
  double lmax;      // power iteration: latest Rayleigh quotient
  double nonfinite;
};

// Everything a pass needs about one volume, in device memory.  The solver's
// iterates rotate by the parity of the device-side iteration counter st->k, so a
// recorded sequence of launches stays valid on replay.
struct VolDesc {
  Geo g;
  const void* hs;          // user PSFs: spectra in the class layout (scaled by 1/N)
  uint32_t imag_mask;      // separable spectra: bit k set -> harmonic k's x factor is imaginary
  const float* b;          // sensitivity
  float2* uperm;           // class-layout yz spectra (forward) / adjoint spectra
  float2* G;               // decimated spectra (forward)
  float2* Gp;              // decimated spectra (adjoint)
  float* rho[2];           // FISTA iterates rho^k in rho[k & 1]
  float* y[2];             // FISTA extrapolated points y^k in y[k & 1]
  const float* d;          // FISTA data
  const float2* tw;        // FP32 twiddle tables, offsets off[] for nx, ny, nz, mx, my, mz
  int off[6];
  DevState* st;
  double* partials;        // per-block FP64 partial sums of the x-plane passes
  double* hist;            // FISTA r_k history, index k - k_first
  int hist_len, k_first;
  int reg_kind;
  float lam;
  int T_class;             // threads of the class passes doing element work
  float* u;                // A^T A part of the current step, summed over the components so far
  const int* cidx;         // user PSFs: the class layout's positions in a half plane (user.hpp)
  float alpha;             // boundary prior weight (eq. finalR), 0 = off
  int aw;                  // its shell depth in voxels
  int nb_upd;              // blocks whose sums a solver step leaves
  // Vector model (components i of the PSF vector and of the sensitivity): component
  // i's spectra at hs + i * hs_cstride elements, its sensitivity at b + i * N and its
  // class-layout spectra at uperm + i * hsz.  ncomp = 1 is the scalar model.
  int ncomp;
  long long hs_cstride;
  // bit k of cmask[i]: component i of harmonic k is present (a PSF block that is
  // identically zero is skipped: no spectrum load, no product)
  uint32_t cmask[3];
  // Separable analytic spectra (the passes of sep.hpp and fast.hpp): the x factors
  // sfs[k][qx], the y-residue table set[y0][q'y][qz], and their intermediates, both in
  // uperm's memory: cp[y0][x][column] (the plane pass's folded shares) and
  // qx[x][column] (the column pass's output for the adjoint plane pass).
  const float* sfs;
  const float2* set;
  float2* cp;
  float2* qx;
};

// Volume and local block index of this block: task table (batched launches) or
// the single volume vds[0].
__device__ __forceinline__ const VolDesc& vol_of(const VolDesc* __restrict__ vds, const int2* __restrict__ tasks,
                                                 int& lb) {
  if (tasks) {
    const int2 t = tasks[blockIdx.x];
    lb = t.y;
    return vds[t.x];
  }
  lb = blockIdx.x;
  return vds[0];
}

// ============================================================================ pass 1: x-plane R2C
// SRC_FISTA_NEXT: y^{k+1}, for a pass between an update's step and its finish (which advances k)
enum { SRC_PLAIN = 0, SRC_RAW = 1, SRC_FISTA_Y = 2, SRC_SCALED = 3, SRC_FISTA_NEXT = 4 };

// ============================================================================ pass 2: classes
// E consecutive spectrum elements.
template <int E>
struct HLoad {
  float2 v[E];
  __device__ __forceinline__ void load(const void* base, long long off) {
    const float2* p = reinterpret_cast<const float2*>(base) + off;
    if constexpr (E % 2 == 0) {
#pragma unroll
      for (int i = 0; i < E; i += 2) {
        const float4 t = ldg(reinterpret_cast<const float4*>(p + i));
        v[i] = make_float2(t.x, t.y); v[i + 1] = make_float2(t.z, t.w);
      }
    } else {
#pragma unroll
      for (int i = 0; i < E; ++i) v[i] = ldg(p + i);
    }
  }
};

// LDS of the class passes with cb components per round and line stride fls of the folded
// spectra: tables (nx + mx), two buffers of cb * cpw * nmem x lines, two of K * cpw x' lines.
__host__ __device__ inline size_t class_lds_elems(const Geo& g, int cb, int fls) {
  const size_t W = (size_t)g.cpw * g.nmem;
  return (size_t)g.nx + g.mx + 2 * cb * W * g.lsx + 2 * (size_t)g.K * g.cpw * fls;
}

// Destinations of the fused class (or column) pass: see user.hpp and sep.hpp.
enum { NRM_RESID = 0, NRM_PLAIN = 1, NRM_STORE = 2 };

// ============================================================================ pass 3: small grid
enum { EPI_STORE = 0, EPI_RESID_BACK = 1, EPI_BACK = 2, EPI_STORE_BACK = 3 };

// ============================================================================ pass 1 adjoint
enum { OUT_SCALE_B = 0, OUT_STEP_NORMAL = 2, OUT_STEP_FISTA = 3 };
enum { UPD_NORMAL = 1, UPD_FISTA = 2 };

struct AdjOut {
  float* out;              // OUT_SCALE_B / UPD_NORMAL: result (UPD_NORMAL: NULL -> rho[(k+1) & 1])
  const float* yin;        // UPD_NORMAL: w_{t-1} (v = scale * w_{t-1}); NULL -> rho[k & 1]
};

// The block's FP64 sums into vd.partials[NV * lb ...] (k_vol_finish reduces them).
template <int NV>
__device__ __forceinline__ void store_step_partials(const VolDesc& vd, double* acc, double* red, int lb) {
  block_reduce_f64<NV>(acc, red);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < NV; ++j) vd.partials[NV * lb + j] = acc[j];
  }
}

// Deterministic grid reduction: every block writes NV partials; the last block to
// arrive sums them in block order.  Returns true in thread 0 of the last block.
template <int NV>
__device__ __forceinline__ bool grid_reduce_last(double* v, double* partials, DevState* st, double* sh,
                                                 int blk, int nblk) {
  block_reduce_f64<NV>(v, sh);
  __shared__ int is_last;
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < NV; ++j) partials[blk * NV + j] = v[j];
    __threadfence();
    const int prev = atomicAdd(&st->counter, 1);
    is_last = (prev == nblk - 1);
  }
  __syncthreads();
  if (!is_last) return false;
  // the last block sums the partials: thread t takes blocks t, t + blockDim, ... in
  // order, then the fixed-order block reduction (the same result for any arrival order)
  __threadfence();
  double w[NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) w[j] = 0.0;
  const volatile double* vp = partials;
  for (int bidx = threadIdx.x; bidx < nblk; bidx += blockDim.x) {
#pragma unroll
    for (int j = 0; j < NV; ++j) w[j] += vp[bidx * NV + j];
  }
  block_reduce_f64<NV>(w, sh);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < NV; ++j) v[j] = w[j];
    st->counter = 0;
  }
  return threadIdx.x == 0;
}

// Sums the block partials of a solver step in a fixed order, the same for any block size T (a
// multiple of 64): 256 running sums over the blocks t, t + 256, ..., folded wave by wave;
// and advances the state.  One block per volume, sh: 12 doubles of its LDS.  A kernel
// boundary orders it after every partial store.
//
// An update's finish runs as one more block of the next update's column or class pass, which
// reads nothing it writes: the pass stops at `skip`, which the launch before it sets if the solve
// was done then (solve_over).  The pass of the update after the last fills scratch buffers, and
// the step after it, which reads `done`, ends.  The forward plane pass before it takes y^{k+1}
// (SRC_FISTA_NEXT).  As a launch of its own, which it still is before the host reads the state, it
// took 3.6 to 4.9 us: 30 updates at 128^3 1176 us with it, 1054 without; 25 padded ones at 64^3
// 1301, 1212; 16 of a batch of four 1164, 1106; 30 of a 128 x 256 image 1073, 971.
__device__ __forceinline__ bool solve_over(const VolDesc& vd, int fin) {
  const DevState* st = vd.st;
  return *(fin ? &st->skip : &st->done) != 0;
}
// The first block of a launch before such a pass, if it finds the solve done.  (Never in a launch that
// has work to do: a block that first stored `done` waited for that store, 1 us of an update of
// a batch.)
__device__ __forceinline__ void set_skip(DevState* st, bool first) {
  if (first && threadIdx.x == 0) st->skip = 1;
}
template <int UPD>
__device__ __forceinline__ void vol_finish(const VolDesc& vd, int T, double* sh) {
  DevState* st = vd.st;
  if (st->done) return;
  constexpr int NV = UPD == UPD_NORMAL ? 2 : 3;
  double acc[NV];
  for (int t = threadIdx.x; t < 256; t += T) {
#pragma unroll
    for (int j = 0; j < NV; ++j) acc[j] = 0.0;
    for (int b = t; b < vd.nb_upd; b += 256) {
#pragma unroll
      for (int j = 0; j < NV; ++j) acc[j] += vd.partials[b * NV + j];
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      for (int o = 32; o >= 1; o >>= 1) acc[j] += __shfl_xor(acc[j], o, 64);
      if ((t & 63) == 0) sh[j * 4 + (t >> 6)] = acc[j];
    }
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    acc[j] = 0.0;
    for (int w = 0; w < 4; ++w) acc[j] += sh[j * 4 + w];
  }
  const int kk = st->k;
  if constexpr (UPD == UPD_NORMAL) {
    st->lmax = acc[0];
    st->scale = 1.0 / sqrt(acc[1]);
    if (!(acc[0] == acc[0]) || !(acc[1] < 1e300)) st->nonfinite = 1.0;
    st->k = kk + 1;
    if (kk >= st->kmax) st->done = 1;
  } else {
    double r;
    if (acc[1] == 0.0) r = (acc[0] == 0.0) ? 0.0 : __builtin_inf();
    else r = sqrt(acc[0]) / sqrt(acc[1]);
    st->rel_step = r;
    st->last_k = kk;
    const int hi = kk - vd.k_first;
    if (vd.hist && hi >= 0 && hi < vd.hist_len) vd.hist[hi] = r;
    if (acc[2] != 0.0 || !(acc[0] == acc[0]) || !(acc[1] == acc[1]) || acc[1] > 1e300) {
      st->nonfinite = 1.0;
      st->done = 1;
    }
    // tol = 0 never stops early (not even at r_k = 0): the run takes max_iter updates
    if ((st->tol > 0.0 && r <= st->tol) || kk >= st->kmax) st->done = 1;
    st->k = kk + 1;
  }
}
template <int UPD>
static __global__ __launch_bounds__(256) void k_vol_finish(const VolDesc* __restrict__ vds, const int2* __restrict__ tasks) {
  __shared__ double sh[12];
  int lb;
  vol_finish<UPD>(vol_of(vds, tasks, lb), 256, sh);
}

// ============================================================================ MHAD
// Multi-harmonic anti-differentiation (App. D, eq. mhadM): the native image on the
// portrait grid from the portraits, per line along the drive axis (x'):
//   rho_N^(q) = sum_k c_k^{-1} conj(f^(q))^{k-1} d_k^(q) / (sum_k |f^(q)|^{2(k-1)} + lambda),
// f^(q) = 2i sin(2 pi q / m) (the central difference u[j+1] - u[j-1]).  A block takes
// CB lines (consecutive (y', z') columns, so the loads and stores are coalesced), FFTs
// each harmonic's lines in LDS and accumulates the weighted spectra, then divides and
// transforms back.  grid = ceil(C / CB), C = my' mz'; dynamic LDS (m + 3 CB ls) float2
// + m floats, ls = pad_odd(m).
struct MhadW {
  int ord[32];        // k - 1 per harmonic
  double cinv[32];    // 1 / c_k
};

static __global__ __launch_bounds__(256) void k_mhad(const float* __restrict__ d, int K, MhadW wk, double lam, int m,
                                              long long C, int CB, float* __restrict__ out) {
  extern __shared__ float2 sm[];
  const int ls = pad_odd(m);
  float2* tw = sm;
  float2* A0 = tw + m;
  float2* A1 = A0 + CB * ls;
  float2* acc = A1 + CB * ls;
  float* den = reinterpret_cast<float*>(acc + CB * ls);
  const long long c0 = (long long)blockIdx.x * CB;
  const int nc = (int)(C - c0 < CB ? C - c0 : CB);
  for (int t = threadIdx.x; t < m; t += blockDim.x) {
    double sn, cs;
    sincospi(2.0 * (double)t / (double)m, &sn, &cs);
    tw[t] = make_float2((float)cs, (float)-sn);
    double sum = lam;
    for (int i = 0; i < K; ++i) sum += pow(4.0 * sn * sn, (double)wk.ord[i]);
    den[t] = (float)sum;
  }
  for (int p = threadIdx.x; p < CB * ls; p += blockDim.x) acc[p] = make_float2(0.f, 0.f);
  for (int i = 0; i < K; ++i) {
    __syncthreads();
    for (int p = threadIdx.x; p < m * nc; p += blockDim.x) {
      const int x = p / nc, c = p - x * nc;
      A0[c * ls + x] = make_float2(d[(long long)i * m * C + (long long)x * C + c0 + c], 0.f);
    }
    const float2* F = fft_lines<-1>(A0, A1, tw, m, nc, ls);
    const int n = wk.ord[i];
    for (int p = threadIdx.x; p < m * nc; p += blockDim.x) {
      const int c = p / m, q = p - c * m;
      // c_k^{-1} (-2i sin)^n = c_k^{-1} (2 sin)^n (-i)^n
      const double mag = wk.cinv[i] * pow(2.0 * sinpi(2.0 * (double)q / (double)m), (double)n);
      float2 w;
      switch (n & 3) {
        case 0: w = make_float2((float)mag, 0.f); break;
        case 1: w = make_float2(0.f, (float)-mag); break;
        case 2: w = make_float2((float)-mag, 0.f); break;
        default: w = make_float2(0.f, (float)mag); break;
      }
      const float2 v = F[c * ls + q];
      float2& a = acc[c * ls + q];
      a.x += w.x * v.x - w.y * v.y;
      a.y += w.x * v.y + w.y * v.x;
    }
  }
  __syncthreads();
  for (int p = threadIdx.x; p < m * nc; p += blockDim.x) {
    const int c = p / m, q = p - c * m;
    const float inv = 1.f / den[q];
    A0[c * ls + q] = make_float2(acc[c * ls + q].x * inv, acc[c * ls + q].y * inv);
  }
  const float2* G = fft_lines<+1>(A0, A1, tw, m, nc, ls);
  const float invm = 1.f / (float)m;
  for (int p = threadIdx.x; p < m * nc; p += blockDim.x) {
    const int x = p / nc, c = p - x * nc;
    out[(long long)x * C + c0 + c] = G[c * ls + x].x * invm;
  }
}

// y^{k0} = rho^{k0} + (k0-1)/(k0+2) (rho^{k0} - rho^{k0-1}) for a (re)started solve.
// y^{k0} = rho^{k0} + beta (rho^{k0} - rho^{k0-1}), rounded as the step forms y^{k+1}
// (no contraction), so a resumed solve continues bitwise as the uninterrupted one.
static __global__ void k_fista_init(long long n, const float* __restrict__ rk, const float* __restrict__ rkm1,
                             float beta, float* __restrict__ y) {
#pragma clang fp contract(off)
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const float r = rk[i];
    y[i] = r + beta * (r - rkm1[i]);
  }
}

// ============================================================================ plan-time kernels
// Twiddle tables exp(-2 pi i t / n), FP64 evaluation, FP32 and FP64 copies.
static __global__ void k_twiddles(int n, float2* __restrict__ t32, double2* __restrict__ t64) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
    double s, c;
    sincospi(2.0 * (double)t / (double)n, &s, &c);
    if (t32) t32[t] = make_float2((float)c, (float)-s);
    if (t64) t64[t] = make_double2(c, -s);
  }
}

// Gaussian sensitivity, peak 1 at the geometric centre ((N-1)/2 voxel).
static __global__ void k_sensitivity(Geo g, double vox, double sx, double sy, double sz, float* __restrict__ b) {
  const long long n = g.N;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const int z = (int)(i % g.nz);
    const int y = (int)((i / g.nz) % g.ny);
    const int x = (int)(i / ((long long)g.ny * g.nz));
    const double ax = (x - 0.5 * (g.nx - 1)) * vox / sx;
    const double ay = (y - 0.5 * (g.ny - 1)) * vox / sy;
    const double az = (z - 0.5 * (g.nz - 1)) * vox / sz;
    b[i] = (float)exp(-0.5 * (ax * ax + ay * ay + az * az));
  }
}

__device__ __forceinline__ int signed_offset(int i, int n) { return (2 * i < n) ? i : i - n; }

// Drive-axis profiles f_k(x) = L^(order_k)(a vox w(x)) (symmetric mean at x = nx/2
// for even nx), their FFT along x in FP64, and ||f_k||^2.  grid = K blocks.
static __global__ __launch_bounds__(256) void k_psf_profile(int nx, const int* __restrict__ order, double a_vox,
                                                     const double2* __restrict__ tw64,
                                                     double* __restrict__ prof, double2* __restrict__ fhat,
                                                     double* __restrict__ fnorm2) {
  extern __shared__ double2 lds64[];
  double2* tw = lds64;
  double2* X = tw + nx;
  double2* X1 = X + nx;
  __shared__ double red[64];
  const int k = blockIdx.x;
  const int n = order[k];
  load_table(tw, tw64, nx);
  double acc[1] = {0.0};
  for (int i = threadIdx.x; i < nx; i += blockDim.x) {
    double f;
    if ((nx % 2 == 0) && 2 * i == nx) {
      const double u = a_vox * (nx / 2);
      f = 0.5 * (langevin_deriv_dev(n, u) + langevin_deriv_dev(n, -u));
    } else {
      f = langevin_deriv_dev(n, a_vox * signed_offset(i, nx));
    }
    prof[(long long)k * nx + i] = f;
    X[i] = make_double2(f, 0.0);
    acc[0] += f * f;
  }
  const double2* F = fft_lines<-1>(X, X1, tw, nx, 1, nx);
  for (int i = threadIdx.x; i < nx; i += blockDim.x) fhat[(long long)k * nx + i] = F[i];
  block_reduce_f64<1>(acc, red);
  if (threadIdx.x == 0) fnorm2[k] = acc[0];
}

// Transverse envelope E(y, z) = L'(a r)/r, E(0) = L'(0) 4 asinh(1)/vox, one row per
// block, then FFT along z (FP64).  Also per-row sum of E^2.  grid = ny blocks.
static __global__ __launch_bounds__(256) void k_psf_env_rows(int ny, int nz, double a, double vox,
                                                      const double2* __restrict__ tw64z,
                                                      double* __restrict__ env, double2* __restrict__ tmp,
                                                      double* __restrict__ rowsum) {
  extern __shared__ double2 lds64[];
  double2* tw = lds64;
  double2* X = tw + nz;
  double2* X1 = X + nz;
  __shared__ double red[64];
  const int y = blockIdx.x;
  load_table(tw, tw64z, nz);
  double acc[1] = {0.0};
  const double wy = signed_offset(y, ny) * vox;
  for (int z = threadIdx.x; z < nz; z += blockDim.x) {
    const double wz = signed_offset(z, nz) * vox;
    const double r = sqrt(wy * wy + wz * wz);
    double e;
    if (r > 0.0) e = langevin_deriv_dev(1, a * r) / r;
    else e = (1.0 / 3.0) * 4.0 * asinh(1.0) / vox;
    env[(long long)y * nz + z] = e;
    X[z] = make_double2(e, 0.0);
    acc[0] += e * e;
  }
  const double2* F = fft_lines<-1>(X, X1, tw, nz, 1, nz);
  for (int z = threadIdx.x; z < nz; z += blockDim.x) tmp[(long long)y * nz + z] = F[z];
  block_reduce_f64<1>(acc, red);
  if (threadIdx.x == 0) rowsum[y] = acc[0];
}

// FFT along y of the row-transformed envelope, one column per block (qz <= nz/2).
static __global__ __launch_bounds__(256) void k_psf_env_cols(int ny, int nz, const double2* __restrict__ tw64y,
                                                      const double2* __restrict__ tmp, double2* __restrict__ ehat) {
  extern __shared__ double2 lds64[];
  double2* tw = lds64;
  double2* X = tw + ny;
  double2* X1 = X + ny;
  const int qz = blockIdx.x;
  load_table(tw, tw64y, ny);
  for (int y = threadIdx.x; y < ny; y += blockDim.x) X[y] = tmp[(long long)y * nz + qz];
  const double2* F = fft_lines<-1>(X, X1, tw, ny, 1, ny);
  for (int y = threadIdx.x; y < ny; y += blockDim.x) ehat[(long long)y * (nz / 2 + 1) + qz] = F[y];
}

// scale[k] = 1 / (||f_k|| ||E|| N)   (unit-norm PSF, unnormalised FFTs downstream)
static __global__ void k_psf_scales(int K, int ny, long long N, const double* __restrict__ fnorm2,
                             const double* __restrict__ rowsum, double* __restrict__ scale) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double e2 = 0.0;
    for (int y = 0; y < ny; ++y) e2 += rowsum[y];
    for (int k = 0; k < K; ++k) scale[k] = 1.0 / (sqrt(fnorm2[k]) * sqrt(e2) * (double)N);
  }
}

// Plan-time tables of the separable passes (FP64 sums, FP32 storage):
//   sfs[k][qx]        scale_k F_k(qx) (its real part, or its imaginary part when bit k of
//                     imag_mask is set), the x factor of the stored spectra
//   set[y0][q'y][qz]  Et(y0, q'y, qz) = sum_jy w_ny^(y0 qy) Ehat(qy, qz), qz <= nz/2
static __global__ void k_sep_tables(Geo g, const double2* __restrict__ fhat, const double2* __restrict__ ehat,
                             const double* __restrict__ scale, uint32_t imag_mask,
                             const double2* __restrict__ tw64y, float* __restrict__ sfs, float2* __restrict__ set) {
  const int nf = g.K * g.nx;
  const int ne = g.sy * g.my * g.nzh;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < nf + ne; t += gridDim.x * blockDim.x) {
    if (t < nf) {
      const int k = t / g.nx;
      const double2 f = fhat[t];
      sfs[t] = (float)((((imag_mask >> k) & 1u) ? f.y : f.x) * scale[k]);
    } else {
      const int r = t - nf;
      const int y0 = r / (g.my * g.nzh), r2 = r - y0 * (g.my * g.nzh);
      const int qyp = r2 / g.nzh, qz = r2 - qyp * g.nzh;
      double sr = 0.0, si = 0.0;
      for (int jy = 0; jy < g.sy; ++jy) {
        const int qy = qyp + jy * g.my;
        const double2 w = tw64y[(long long)y0 * qy % g.ny];   // exp(-2 pi i y0 qy / ny)
        const double2 e = ehat[(long long)qy * g.nzh + qz];
        sr += w.x * e.x - w.y * e.y;
        si += w.x * e.y + w.y * e.x;
      }
      set[r] = make_float2((float)sr, (float)si);
    }
  }
}

// fft(h_k) of the analytic PSF, [k][nx][ny][nzh] complex, from its factors: F_k(qx) Ehat(qy,
// qz) scale_k N in FP64, rounded to FP32 once (its real part for odd orders, its imaginary
// part for even ones; tests and tools).  It shows the factors that the passes' tables are made
// of, not the tables: sfs and set each round their own sums, and what the passes multiply with
// is checked by the operator's parity with the oracle.
static __global__ void k_spectrum_analytic(Geo g, const double2* __restrict__ fhat, const double2* __restrict__ ehat,
                                    const double* __restrict__ scale, uint32_t imag_mask, float2* __restrict__ out) {
  const long long per_k = (long long)g.nx * g.ny * g.nzh, total = (long long)g.K * per_k;
  const float Nf = (float)g.N;
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total; t += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(t / per_k);
    const long long r = t % per_k;
    const double2 f = fhat[(long long)k * g.nx + r / ((long long)g.ny * g.nzh)];
    const double2 e = ehat[r % ((long long)g.ny * g.nzh)];
    const double s = scale[k];
    out[t] = ((imag_mask >> k) & 1u) ? make_float2(0.f, (float)((f.x * e.y + f.y * e.x) * s) * Nf)
                                     : make_float2((float)((f.x * e.x - f.y * e.y) * s) * Nf, 0.f);
  }
}

// User PSF spectra: FFT along x of the class-layout yz spectrum of h_k, scaled by
// 1/N, stored complex in the class layout.  grid = ncls/cpw blocks, cpw*nmem lines.
static __global__ __launch_bounds__(1024) void k_class_hcopy(Geo g, int k, const float2* __restrict__ uperm,
                                                      float2* __restrict__ hs, const float2* __restrict__ tw_x) {
  extern __shared__ float2 lds[];
  float2* twx = lds;
  const int W = g.cpw * g.nmem;
  float2* U0 = twx + g.nx;
  float2* U1 = U0 + W * g.lsx;
  load_table(twx, tw_x, g.nx);
  const int c0 = blockIdx.x * g.cpw;
  batched<8, float2>(g.nx * W,
                     [&](int p) {
                       const int xx = (int)g.f_W.div((uint32_t)p), e = p - xx * W;
                       return uperm[(long long)xx * g.plane + (long long)c0 * g.nmem + e];
                     },
                     [&](int p, float2 v) {
                       const int xx = (int)g.f_W.div((uint32_t)p), e = p - xx * W;
                       U0[e * g.lsx + xx] = v;
                     });
  const float2* Ul = fft_lines<-1>(U0, U1, twx, g.nx, W, g.lsx);
  const float invN = (float)(1.0 / (double)g.N);
  const int per_cls = g.mx * g.S;
  for (int t = threadIdx.x; t < g.cpw * per_cls; t += blockDim.x) {
    const int cl = (int)g.f_mxS.div((uint32_t)t), r2 = t - cl * per_cls;
    const int qxp = (int)g.f_S.div((uint32_t)r2), w = r2 - qxp * g.S;
    const int jx = (int)g.f_nmem.div((uint32_t)w), m = w - jx * g.nmem;
    const float2 v = Ul[(cl * g.nmem + m) * g.lsx + qxp + jx * g.mx];
    hs[(long long)k * g.hsz + (long long)c0 * per_cls + t] = make_float2(v.x * invN, v.y * invN);
  }
}

// Flags of the PSF blocks that are not identically zero: blockIdx.x = j selects the
// (component, harmonic) block psf + j * N, blockIdx.y = s one of gridDim.y strided
// shares of it; flags[j * gridDim.y + s] = any nonzero in the share.
static __global__ __launch_bounds__(256) void k_nonzero_blocks(const float* __restrict__ psf, long long N,
                                                        int* __restrict__ flags) {
  const float* p = psf + (long long)blockIdx.x * N;
  const long long step = (long long)gridDim.y * blockDim.x;
  int any = 0;
  for (long long i = (long long)blockIdx.y * blockDim.x + threadIdx.x; i < N; i += step) any |= (p[i] != 0.f);
  any = __syncthreads_or(any);
  if (threadIdx.x == 0) flags[blockIdx.x * gridDim.y + blockIdx.y] = any;
}

// Back from the class layout to [k][nx][ny][nzh] complex, times N (tests/tools).
static __global__ void k_spectrum_export(Geo g, const float2* __restrict__ hs, float2* __restrict__ out) {
  const long long per_k = (long long)g.nx * g.ny * g.nzh;
  const long long total = (long long)g.K * per_k;
  const int per_cls = g.mx * g.S;
  for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < total; t += (long long)gridDim.x * blockDim.x) {
    const int k = (int)(t / per_k);
    long long r = t % per_k;
    const int qz = (int)(r % g.nzh);
    const int qy = (int)((r / g.nzh) % g.ny);
    const int qx = (int)(r / ((long long)g.nzh * g.ny));
    bool cj;
    const int e = class_index_of(g, qy, qz, cj);  // member index in the plane layout
    const int c = e / g.nmem, m = e % g.nmem;
    const int qxs = cj ? (g.nx - qx) % g.nx : qx;   // conjugate partner also negates qx
    const int qxp = qxs % g.mx, jx = qxs / g.mx;
    const long long idx = (long long)k * g.hsz + (long long)c * per_cls + qxp * g.S + jx * g.nmem + m;
    float2 v = hs[idx];
    if (cj) v.y = -v.y;
    const float Nf = (float)g.N;
    out[t] = make_float2(v.x * Nf, v.y * Nf);
  }
}

// ============================================================================ small helpers
// Philox4x32-10 (Salmon et al., SC'11) uniform (w + 0.5)/2^32 start vector, and
// FP64 partials of its squared norm; last block stores 1/||x0|| in st->scale.
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u, W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) { k0 += W0; k1 += W1; }
    const uint32_t hi0 = __umulhi(M0, c[0]), lo0 = M0 * c[0];
    const uint32_t hi1 = __umulhi(M1, c[2]), lo1 = M1 * c[2];
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
  }
}

static __global__ void k_philox_uniform(long long n, uint64_t seed, uint32_t stream, float* __restrict__ out,
                                 double* __restrict__ partials, DevState* st) {
  __shared__ double red[64];
  double acc[1] = {0.0};
  const long long nblk = (n + 3) / 4;
  for (long long bi = blockIdx.x * (long long)blockDim.x + threadIdx.x; bi < nblk; bi += (long long)gridDim.x * blockDim.x) {
    uint32_t c[4] = {(uint32_t)bi, stream, 0u, 0u};
    philox4x32_10(c, (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32));
    for (int j = 0; j < 4; ++j) {
      const long long i = bi * 4 + j;
      if (i < n) {
        const double u = ((double)c[j] + 0.5) / 4294967296.0;
        out[i] = (float)u;
        acc[0] += (double)(float)u * (double)(float)u;
      }
    }
  }
  if (grid_reduce_last<1>(acc, partials, st, red, blockIdx.x, gridDim.x)) st->scale = 1.0 / sqrt(acc[0]);
}

// Raw Philox words for the known-answer test.
static __global__ void k_philox_words(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0, uint32_t k1,
                               uint32_t* __restrict__ out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    uint32_t c[4] = {c0, c1, c2, c3};
    philox4x32_10(c, k0, k1);
    for (int j = 0; j < 4; ++j) out[j] = c[j];
  }
}

}  // namespace mh3d
