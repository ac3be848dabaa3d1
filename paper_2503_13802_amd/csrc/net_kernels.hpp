// Warm-start 3D U-Net on gfx950: BF16 activations and weights, FP32 accumulation on
// MFMA (v_mfma_f32_16x16x32_bf16, two 16-deep reduction chunks per instruction; a
// trailing odd chunk uses v_mfma_f32_16x16x16_bf16), FP32 master weights, Adam.
//
// Tensors are channels-last BF16 [X][Y][Z][Cs] with the channel stride Cs a
// multiple of 4 (padding channels hold zeros).  Grid axes are powers of two so
// voxel decoding is shifts.  A 3x3x3 convolution is an implicit GEMM
//   out[n][co] = b[co] + sum_k W[co][k] in[n + d(tap(k))][ci(k)],  k = tap*Cs_in + ci,
// tap = (dx+1)*9 + (dy+1)*3 + (dz+1), zero outside the grid; K is padded to a
// multiple of 16 with zero weights.  One wavefront computes 16 voxels x all output
// channels (16-wide tiles); per MFMA the lane layout is
//   A[row = lane%16][k = 4*(lane/16) + j]   (voxel x reduction),
//   B[k = 4*(lane/16) + j][col = lane%16]   (reduction x channel),
//   D[row = 4*(lane/16) + j][col = lane%16].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mh3d {
namespace net {

typedef short s4v __attribute__((ext_vector_type(4)));
typedef short s8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));

// Two 16-deep reduction chunks in one 16x16x32 MFMA.  The instruction reads lane group g
// (lane / 16) element j as reduction index 8g + j of A and of B; placing chunk 0's
// slice (k = 4g + j) in elements 0..3 and chunk 1's (k = 16 + 4g + j) in 4..7 applies
// the same permutation of the 32 reduction indices to both operands, so the result is
// the sum of the two 16x16x16 products (in another order of the FP32 additions).
__device__ __forceinline__ f4v mfma2(s4v a0, s4v a1, s4v b0, s4v b1, f4v c) {
  const s8v a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
  const s8v b = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a), __builtin_bit_cast(bf8v, b), c, 0, 0, 0);
}

constexpr int NT_MAX = 7;   // output-channel tiles per wave (112 channels)

// FP32 -> BF16, round to nearest even (NaN kept quiet).
// Nearest BF16, ties to even (gfx950's v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// ReLU backward of a data gradient in the kernel that forms it: mask, the post-ReLU tensor
// the gradient belongs to (NULL: keep everything), zeroes the gradient where it is not > 0.
__device__ __forceinline__ bool keep(const uint16_t* mask, long long i) { return !mask || bf2f(mask[i]) > 0.f; }
template <typename V> __device__ __forceinline__ V masked(V g, V act) {
#pragma unroll
  for (int q = 0; q < (int)(sizeof(V) / 2); ++q) g[q] = bf2f((uint16_t)act[q]) > 0.f ? g[q] : (short)0;
  return g;
}

struct Dims {
  int lx, ly, lz;          // log2 of the axes
  __host__ __device__ __forceinline__ long long n() const { return 1ll << (lx + ly + lz); }
  __device__ __forceinline__ void decode(long long i, int& x, int& y, int& z) const {
    z = (int)(i & ((1ll << lz) - 1));
    y = (int)((i >> lz) & ((1ll << ly) - 1));
    x = (int)(i >> (ly + lz));
  }
  __device__ __forceinline__ long long encode(int x, int y, int z) const {
    return ((long long)x << (ly + lz)) | ((long long)y << lz) | z;
  }
  __device__ __forceinline__ bool inside(int x, int y, int z) const {
    return x >= 0 && y >= 0 && z >= 0 && x < (1 << lx) && y < (1 << ly) && z < (1 << lz);
  }
};

__device__ __forceinline__ void tap_offset(int tap, int ks, int& dx, int& dy, int& dz) {
  if (ks == 1) { dx = dy = dz = 0; return; }
  dx = tap / 9 - 1;
  dy = (tap / 3) % 3 - 1;
  dz = tap % 3 - 1;
}

// Convolution (ks = 3 or 1).  in: [N][cs_in]; W: [cout_tiles*16][kp] BF16; bias FP32
// [cout]; out: BF16 [N][cs_out].  Padding output
// channels cout..cs_out-1 are written as zeros.  block = 256 (4 waves, 64 voxels).
template <bool RELU>
__global__ __launch_bounds__(256) void k_conv(const uint16_t* __restrict__ in, Dims dm, int cs_in, int ks,
                                              const uint16_t* __restrict__ W, int kp,
                                              const float* __restrict__ bias, int cout, int cs_out,
                                              uint16_t* __restrict__ out, const uint16_t* __restrict__ mask) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long N = dm.n();
  const long long n0 = ((long long)blockIdx.x * 4 + wave) * 16;
  if (n0 >= N) return;                      // wave-uniform, no block barriers below
  const int r = lane & 15, g = lane >> 4;
  const long long n = n0 + r;
  const bool nvalid = n < N;
  int x = 0, y = 0, z = 0;
  if (nvalid) dm.decode(n, x, y, z);
  const int ntile = (cout + 15) >> 4;
  const int ntap = ks * ks * ks;
  f4v acc[NT_MAX];
#pragma unroll
  for (int t = 0; t < NT_MAX; ++t) acc[t] = f4v{0.f, 0.f, 0.f, 0.f};
  int tap = 0, ci = 4 * g;
  while (ci >= cs_in) { ci -= cs_in; ++tap; }
  // A slice of the current chunk (this lane's voxel, 4 reduction indices), then step
  auto a_next = [&]() {
    s4v a = s4v{0, 0, 0, 0};
    if (nvalid && tap < ntap) {
      int dx, dy, dz;
      tap_offset(tap, ks, dx, dy, dz);
      const int xx = x + dx, yy = y + dy, zz = z + dz;
      if (dm.inside(xx, yy, zz)) a = *reinterpret_cast<const s4v*>(in + dm.encode(xx, yy, zz) * cs_in + ci);
    }
    ci += 16;
    while (ci >= cs_in) { ci -= cs_in; ++tap; }
    return a;
  };
  const int nkc = kp >> 4;
  for (int kc = 0; kc < nkc; kc += 2) {
    const s4v a0 = a_next();
    const uint16_t* wr = W + (long long)r * kp + kc * 16 + 4 * g;
    if (kc + 1 < nkc) {
      const s4v a1 = a_next();
#pragma unroll
      for (int t = 0; t < NT_MAX; ++t) {
        if (t < ntile) {
          const s4v b0 = *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp);
          const s4v b1 = *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp + 16);
          acc[t] = mfma2(a0, a1, b0, b1, acc[t]);
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < NT_MAX; ++t) {
        if (t < ntile) {
          const s4v b = *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp);
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0, b, acc[t], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int t = 0; t < NT_MAX; ++t) {
    if (t >= ntile) break;
    const int co = t * 16 + r;
    const float bv = co < cout ? bias[co] : 0.f;   // once: the stores may alias bias for the compiler
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const long long nn = n0 + 4 * g + j;
      if (nn >= N) continue;
      if (co < cout) {
        float v = acc[t][j] + bv;
        if (RELU) v = fmaxf(v, 0.f);
        out[nn * cs_out + co] = keep(mask, nn * cs_out + co) ? f2bf(v) : (uint16_t)0;
      } else if (co < cs_out) {
        out[nn * cs_out + co] = 0;
      }
    }
  }
}

// Convolution with the reduction split over the 4 waves of a block (for deep K on
// small grids, where k_conv has too few waves to hide its load latency): the block
// owns 16 voxels, wave w takes the K chunks w, w+4, ..., the partial tiles are
// summed in LDS in wave order and wave 0 writes the result.  Same operands, output
// and padding rules as k_conv (BF16 output).  grid = ceil(N/16), block = 256.
template <bool RELU>
__global__ __launch_bounds__(256) void k_conv_splitk(const uint16_t* __restrict__ in, Dims dm, int cs_in, int ks,
                                                     const uint16_t* __restrict__ W, int kp,
                                                     const float* __restrict__ bias, int cout, int cs_out,
                                                     uint16_t* __restrict__ out, const uint16_t* __restrict__ mask) {
  __shared__ f4v part[3][NT_MAX][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long N = dm.n();
  const long long n0 = (long long)blockIdx.x * 16;
  const int r = lane & 15, g = lane >> 4;
  const long long n = n0 + r;
  const bool nvalid = n < N;
  int x = 0, y = 0, z = 0;
  if (nvalid) dm.decode(n, x, y, z);
  const int ntile = (cout + 15) >> 4;
  const int ntap = ks * ks * ks;
  f4v acc[NT_MAX];
#pragma unroll
  for (int t = 0; t < NT_MAX; ++t) acc[t] = f4v{0.f, 0.f, 0.f, 0.f};
  // k = kc*16 + 4g: start at chunk `wave`, step 4 chunks (64 k) at a time
  int tap = 0, ci = wave * 16 + 4 * g;
  while (ci >= cs_in) { ci -= cs_in; ++tap; }
  // A slice of this wave's current chunk, then step to its next chunk (4 chunks on)
  auto a_next = [&]() {
    s4v a = s4v{0, 0, 0, 0};
    if (nvalid && tap < ntap) {
      int dx, dy, dz;
      tap_offset(tap, ks, dx, dy, dz);
      const int xx = x + dx, yy = y + dy, zz = z + dz;
      if (dm.inside(xx, yy, zz)) a = *reinterpret_cast<const s4v*>(in + dm.encode(xx, yy, zz) * cs_in + ci);
    }
    ci += 64;
    while (ci >= cs_in) { ci -= cs_in; ++tap; }
    return a;
  };
  const int nkc = kp >> 4;
  for (int kc = wave; kc < nkc; kc += 8) {   // chunks kc and kc + 4 in one instruction
    const s4v a0 = a_next();
    const uint16_t* wr = W + (long long)r * kp + kc * 16 + 4 * g;
    if (kc + 4 < nkc) {
      const s4v a1 = a_next();
#pragma unroll
      for (int t = 0; t < NT_MAX; ++t) {
        if (t < ntile) {
          const s4v b0 = *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp);
          const s4v b1 = *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp + 64);
          acc[t] = mfma2(a0, a1, b0, b1, acc[t]);
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < NT_MAX; ++t) {
        if (t < ntile) {
          const s4v b = *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp);
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0, b, acc[t], 0, 0, 0);
        }
      }
    }
  }
  if (wave) {
#pragma unroll
    for (int t = 0; t < NT_MAX; ++t)
      if (t < ntile) part[wave - 1][t][lane] = acc[t];
  }
  __syncthreads();
  if (wave) return;
#pragma unroll
  for (int t = 0; t < NT_MAX; ++t) {
    if (t >= ntile) break;
    f4v v = acc[t];
#pragma unroll
    for (int w = 0; w < 3; ++w) v += part[w][t][lane];
    const int co = t * 16 + r;
    const float bv = co < cout ? bias[co] : 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const long long nn = n0 + 4 * g + j;
      if (nn >= N) continue;
      if (co < cout) {
        float o = v[j] + bv;
        if (RELU) o = fmaxf(o, 0.f);
        out[nn * cs_out + co] = keep(mask, nn * cs_out + co) ? f2bf(o) : (uint16_t)0;
      } else if (co < cs_out) {
        out[nn * cs_out + co] = 0;
      }
    }
  }
}

// The 6 x 6 x 18 input halo of a 4 x 4 x 16 output tile at (x0, y0, z0) into LDS
// ([voxel][cs_in], zero outside the volume), 4 channels (8 bytes) per item with z-runs
// contiguous in global memory.  A thread's items go in batches of 8 whose loads are all
// issued before the LDS writes (a load-then-write loop would wait on every load).
__device__ __forceinline__ void stage_halo(uint16_t* __restrict__ tile, const uint16_t* __restrict__ in, const Dims& dm,
                                           int cs_in, int x0, int y0, int z0) {
  const int cq = cs_in >> 2;
  const int nitem = 648 * cq;
  for (int q0 = threadIdx.x; q0 < nitem; q0 += 8 * 256) {
    s4v val[8];
    int dst[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = q0 + u * 256;
      val[u] = s4v{0, 0, 0, 0};
      dst[u] = -1;
      if (q < nitem) {
        const int v = q / cq, c4 = q - v * cq;
        const int zl = v % 18, yl = (v / 18) % 6, xl = v / 108;
        const int gx = x0 + xl - 1, gy = y0 + yl - 1, gz = z0 + zl - 1;
        dst[u] = v * cs_in + 4 * c4;
        if (dm.inside(gx, gy, gz)) val[u] = *reinterpret_cast<const s4v*>(in + dm.encode(gx, gy, gz) * cs_in + 4 * c4);
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (dst[u] >= 0) *reinterpret_cast<s4v*>(tile + dst[u]) = val[u];
  }
}

// k_conv_splitk for input channel strides divisible by 8: MFMA m takes the reduction
// indices 32 m .. 32 m + 31, lane group g the 8 consecutive channels 32 m + 8 g .. + 7 of
// one tap (one 16-byte gather of A, one 16-byte load of B per output tile); wave w takes
// m = w, w + 4, ..., U of them with all their loads issued before their MFMAs.  A block takes
// VG groups of 16 voxels, which share the weight loads: every block reads all of W, and
// with one group that is most of the traffic from L2 (32^3
// voxels, 112 -> 32 channels: 49 us with one group, 36 with two, 30 with four).
// grid.y splits the output tiles (NT per block) where the voxels alone give few blocks.
template <bool RELU, int NT, int VG>
__global__ __launch_bounds__(256) void k_conv_splitk8(const uint16_t* __restrict__ in, Dims dm, int cs_in, int ks,
                                                      const uint16_t* __restrict__ W, int kp,
                                                      const float* __restrict__ bias, int cout, int cs_out,
                                                      uint16_t* __restrict__ out, const uint16_t* __restrict__ mask) {
  constexpr int U = NT <= 2 && VG <= 2 ? 4 : 2;   // steps in flight per wave: U * VG gathers and U * NT weight slices
  __shared__ f4v part[3][VG * NT][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long N = dm.n();
  const long long n0 = (long long)blockIdx.x * (16 * VG);
  const int r = lane & 15, g = lane >> 4;
  int x[VG], y[VG], z[VG];
#pragma unroll
  for (int v = 0; v < VG; ++v) {
    const long long n = n0 + 16 * v + r;
    x[v] = y[v] = z[v] = 0;
    if (n < N) dm.decode(n, x[v], y[v], z[v]);
    else x[v] = -2;                    // every tap outside
  }
  const int ntap = ks * ks * ks;
  const int t0 = blockIdx.y * NT;   // first output tile of the block
  f4v acc[VG][NT];
#pragma unroll
  for (int v = 0; v < VG; ++v)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[v][t] = f4v{0.f, 0.f, 0.f, 0.f};
  // k = 32 m + 8 g for m = wave + 4 i: start, then step 128 reduction indices
  int tap = 0, ci = 32 * wave + 8 * g;
  while (ci >= cs_in) { ci -= cs_in; ++tap; }
  const int nm = (kp + 31) >> 5;
  const uint16_t* wr = W + (long long)(t0 * 16 + r) * kp + 8 * g;
  for (int m0 = wave; m0 < nm; m0 += 4 * U) {
    s8v a[U][VG], b[U][NT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int m = m0 + 4 * u;
      int dx = 0, dy = 0, dz = 0;
      const bool live = m < nm && tap < ntap;
      if (live) tap_offset(tap, ks, dx, dy, dz);
#pragma unroll
      for (int v = 0; v < VG; ++v) {
        a[u][v] = s8v{0, 0, 0, 0, 0, 0, 0, 0};
        const int xx = x[v] + dx, yy = y[v] + dy, zz = z[v] + dz;
        if (live && dm.inside(xx, yy, zz)) a[u][v] = *reinterpret_cast<const s8v*>(in + dm.encode(xx, yy, zz) * cs_in + ci);
      }
      const bool kin = m < nm && 32 * m + 8 * g < kp;
#pragma unroll
      for (int t = 0; t < NT; ++t)
        b[u][t] = kin ? *reinterpret_cast<const s8v*>(wr + (long long)t * 16 * kp + 32 * m) : s8v{0, 0, 0, 0, 0, 0, 0, 0};
      ci += 128;
      while (ci >= cs_in) { ci -= cs_in; ++tap; }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < VG; ++v)
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[v][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, a[u][v]),
                                                              __builtin_bit_cast(bf8v, b[u][t]), acc[v][t], 0, 0, 0);
  }
  if (wave) {
#pragma unroll
    for (int v = 0; v < VG; ++v)
#pragma unroll
      for (int t = 0; t < NT; ++t) part[wave - 1][v * NT + t][lane] = acc[v][t];
  }
  __syncthreads();
  if (wave) return;
#pragma unroll
  for (int v = 0; v < VG; ++v)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      f4v s = acc[v][t];
#pragma unroll
      for (int w = 0; w < 3; ++w) s += part[w][v * NT + t][lane];
      const int co = (t0 + t) * 16 + r;
      const float bv = co < cout ? bias[co] : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const long long nn = n0 + 16 * v + 4 * g + j;
        if (nn >= N) continue;
        if (co < cout) {
          float o = s[j] + bv;
          if (RELU) o = fmaxf(o, 0.f);
          out[nn * cs_out + co] = keep(mask, nn * cs_out + co) ? f2bf(o) : (uint16_t)0;
        } else if (co < cs_out) {
          out[nn * cs_out + co] = 0;
        }
      }
    }
}

// 3x3x3 convolution on an LDS-staged tile with the input channel stride CS fixed at
// compile time (the same implicit GEMM, tile and operands as k_conv_tiled, kp = 16
// NKC).  Every index the reduction needs is a constant or comes from a per-block table
// of the 4 lane groups' offsets per K chunk, so the reduction costs an LDS read of the
// offset, the operand reads at immediate offsets and the MFMA: no tap arithmetic per
// chunk.  The halo goes in per voxel (one contiguous CS-channel run), and the output
// tile leaves through LDS as contiguous 16- or 8-byte pieces of each z-run.
// C1 > 0: the input is the decoder's concatenation [skip, upsampled coarse] read in place
// (no concatenated copy): channels [0, C1) of voxel n from `in` (stride C1), the other
// CS - C1 from `in2` (stride CS - C1) at the coarse voxel (x/2, y/2, z/2), the halo
// tile holding the same values the concatenated tensor would.
// pool (or NULL): also the 2x2x2 average of the BF16 output (k_avgpool's sums), from the staged
// tile.
// PRE (NT = 1): for grids of few blocks, where a wave has a SIMD to itself and each weight
// load's latency shows: every weight fragment is loaded before the halo, and the output
// tiles go over grid.y.  The sums are the same.  16^3 voxels, 32 -> 32 channels: 13.2 us
// with one block for both output tiles and four loads in flight, 8.3 us so.
template <int CS, int NT, bool RELU, int C1 = 0, bool PRE = false>
__global__ __launch_bounds__(256) void k_conv_ct(const uint16_t* __restrict__ in, Dims dm,
                                                 const uint16_t* __restrict__ W, int kp,
                                                 const float* __restrict__ bias, int cout, int cs_out,
                                                 uint16_t* __restrict__ out, const uint16_t* __restrict__ in2,
                                                 const uint16_t* __restrict__ mask, uint16_t* __restrict__ pool) {
  static_assert(C1 % 4 == 0 && C1 < CS, "the skip channels are whole 4-channel groups");
  static_assert(!PRE || NT == 1, "one output tile per block");
  constexpr int NKC = (27 * CS + 15) / 16;
  constexpr int RS = 18 * CS;                       // one (x, y) row of the halo
  constexpr int HALO = 648 * CS;
  constexpr int STAGE = 256 * 16 * NT;              // output staging (elements), at most
  constexpr int TILE = ((HALO > STAGE ? HALO : STAGE) + 7) & ~7;
  extern __shared__ uint16_t sm[];
  uint16_t* tile = sm;
  int* toff = reinterpret_cast<int*>(sm + TILE);   // [NKC][4] element offsets
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, g = lane >> 4;
  const int nzt = dm.lz - 4, nyt = dm.ly - 2;
  const int tz = blockIdx.x & ((1 << nzt) - 1);
  const int rest = blockIdx.x >> nzt;
  const int ty = rest & ((1 << nyt) - 1);
  const int tx = rest >> nyt;
  const int x0 = tx * 4, y0 = ty * 4, z0 = tz * 16;
  // first channel of the block's output tiles, and how many of the stored channels they hold
  const int co0 = PRE ? 16 * blockIdx.y : 0, csl = PRE ? (cs_out - co0 < 16 ? cs_out - co0 : 16) : cs_out;
  if (PRE) W += (long long)co0 * kp;
  constexpr int KP = 16 * NKC, NM = (KP + 31) / 32;   // W's row length (kp), 32-deep steps
  // the weights of the steps, PRE only
  s8v bpre[PRE ? NM : 1];
  if constexpr (PRE && CS % 8 == 0) {
#pragma unroll
    for (int m = 0; m < NM; ++m)
      bpre[m] = (32 * m + 8 * g < KP) ? *reinterpret_cast<const s8v*>(W + (long long)r * KP + 8 * g + 32 * m)
                                      : s8v{0, 0, 0, 0, 0, 0, 0, 0};
  } else if constexpr (PRE) {
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      const uint16_t* p = W + (long long)r * KP + 4 * g + 32 * m;
      const s4v lo = *reinterpret_cast<const s4v*>(p), hi = 2 * m + 1 < NKC ? *reinterpret_cast<const s4v*>(p + 16) : s4v{0, 0, 0, 0};
      bpre[m] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
  }
  // reduction index k = 16 kc + 4 g + j -> (tap, channel) -> halo offset; the padding
  // columns (tap >= 27) meet zero rows of W and read any finite halo entry (offset 0)
  // (CS % 8 == 0: entry m * 4 + g holds k = 32 m + 8 g; else entry kc * 4 + g, k = 16 kc + 4 g)
  constexpr int NTAB = CS % 8 == 0 ? 4 * ((16 * NKC + 31) / 32) : 4 * NKC;
  for (int i = threadIdx.x; i < NTAB; i += 256) {
    const int k = (CS % 8 == 0 ? 8 : 4) * i;
    const int tap = k / CS, ci = k - (k / CS) * CS;
    toff[i] = tap < 27 ? ((tap / 9) * 108 + ((tap / 3) % 3) * 18 + tap % 3) * CS + ci : 0;
  }
  // halo: voxel v = threadIdx.x + 256 u, its CS channels as CS/4 8-byte loads, all of a
  // thread's loads issued before its LDS writes
  {
    constexpr int NQ = CS / 4, NQ1 = C1 / 4;
    const Dims dc{dm.lx - 1, dm.ly - 1, dm.lz - 1};
    s4v val[3][NQ];
    long long src[3], src2[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int v = threadIdx.x + 256 * u;
      src[u] = -1;
      src2[u] = 0;
      if (v < 648) {
        const int zl = v % 18, yl = (v / 18) % 6, xl = v / 108;
        const int gx = x0 + xl - 1, gy = y0 + yl - 1, gz = z0 + zl - 1;
        if (dm.inside(gx, gy, gz)) {
          src[u] = dm.encode(gx, gy, gz) * (C1 > 0 ? C1 : CS);
          if constexpr (C1 > 0) src2[u] = dc.encode(gx >> 1, gy >> 1, gz >> 1) * (CS - C1);
        }
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const uint16_t* p = (C1 > 0 && q >= NQ1) ? in2 + src2[u] + 4 * (q - NQ1) : in + src[u] + 4 * q;
        val[u][q] = src[u] >= 0 ? *reinterpret_cast<const s4v*>(p) : s4v{0, 0, 0, 0};
      }
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int v = threadIdx.x + 256 * u;
      if (v < 648) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) *reinterpret_cast<s4v*>(tile + v * CS + 4 * q) = val[u][q];
      }
    }
  }
  __syncthreads();
  const int lbase = (wave * 108 + r) * CS;
  f4v acc[4][NT];
#pragma unroll
  for (int yy = 0; yy < 4; ++yy)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[yy][t] = f4v{0.f, 0.f, 0.f, 0.f};
  if constexpr (CS % 8 == 0) {
    // lane group g takes the 8 consecutive reduction indices 32 m + 8 g .. + 7 of MFMA m:
    // 8 channels of one tap, one 16-byte LDS read of A and one 16-byte load of B (the
    // same index on both operands); W's padding columns (k >= 16 NKC) read as zeros
    const uint16_t* wr8 = W + (long long)r * KP + 8 * g;
#pragma unroll PRE ? NM : 4
    for (int m = 0; m < NM; ++m) {
      const int o = lbase + toff[m * 4 + g];
      s8v b[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t)
        b[t] = PRE ? bpre[PRE ? m : 0] : (32 * m + 8 * g < KP) ? *reinterpret_cast<const s8v*>(wr8 + t * 16 * KP + 32 * m)
                                     : s8v{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int yy = 0; yy < 4; ++yy) {
        const s8v av = *reinterpret_cast<const s8v*>(tile + o + yy * RS);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          acc[yy][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8v, av),
                                                               __builtin_bit_cast(bf8v, b[t]), acc[yy][t], 0, 0, 0);
      }
    }
  } else {
  const uint16_t* wr = W + (long long)r * kp + 4 * g;
  auto pair = [&](int kc, bool two) {
    const int o0 = lbase + toff[kc * 4 + g];
    const int o1 = two ? lbase + toff[(kc + 1) * 4 + g] : 0;
    s4v b0[NT], b1[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if constexpr (PRE) {
        b0[t] = __builtin_shufflevector(bpre[kc / 2], bpre[kc / 2], 0, 1, 2, 3);
        b1[t] = __builtin_shufflevector(bpre[kc / 2], bpre[kc / 2], 4, 5, 6, 7);
        continue;
      }
      b0[t] = *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp + kc * 16);
      b1[t] = two ? *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp + kc * 16 + 16) : s4v{0, 0, 0, 0};
    }
#pragma unroll
    for (int yy = 0; yy < 4; ++yy) {
      const s4v a0 = *reinterpret_cast<const s4v*>(tile + o0 + yy * RS);
      const s4v a1 = two ? *reinterpret_cast<const s4v*>(tile + o1 + yy * RS) : s4v{0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[yy][t] = mfma2(a0, a1, b0[t], b1[t], acc[yy][t]);
    }
  };
#pragma unroll PRE ? NKC : 4
  for (int kc = 0; kc + 1 < NKC; kc += 2) pair(kc, true);
  if constexpr (NKC & 1) pair(NKC - 1, false);
  }
  __syncthreads();   // every wave is done with the halo: its space stages the output
  // D[row = 4g + j][col = r]: voxel z0 + 4g + j of row (x0 + wave, y0 + yy), channel t*16 + r
  uint16_t* st = tile + wave * 64 * csl;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int co = t * 16 + r;
    const bool live = co0 + co < cout;
    const float bv = live ? bias[co0 + co] : 0.f;
    if (co < csl) {
      uint16_t* sl = st + 4 * g * csl + co;
#pragma unroll
      for (int yy = 0; yy < 4; ++yy)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float v = acc[yy][t][j] + bv;
          if (RELU) v = fmaxf(v, 0.f);
          const uint16_t h = f2bf(v);
          sl[(yy * 16 + j) * csl] = live ? h : (uint16_t)0;
        }
    }
  }
  __syncthreads();
  // each (x, y) row of 16 voxels is a contiguous run of 16 cs_out channels in memory (PRE: of
  // csl channels per voxel): the wave's 4 rows as 16-byte (8-byte) pieces, piece p of row
  // p / per_row
  const long long row0 = dm.encode(x0 + wave, y0, z0) * cs_out + co0;
  const long long ystride = (long long)cs_out << (dm.lz);   // one y step, in elements
  auto spread = [&](int e) { return PRE ? e / csl * cs_out + e % csl : e; };   // element of a row in memory
  if ((cs_out & 7) == 0) {
    const int per_row = 2 * csl;
    for (int p = lane; p < 4 * per_row; p += 64) {
      const int yy = p / per_row, q = p - yy * per_row;
      const long long o = row0 + yy * ystride + spread(8 * q);
      s8v v = *reinterpret_cast<const s8v*>(st + yy * 16 * csl + 8 * q);
      if (mask) v = masked(v, *reinterpret_cast<const s8v*>(mask + o));
      *reinterpret_cast<s8v*>(out + o) = v;
    }
  } else {
    const int per_row = 4 * csl;
    for (int p = lane; p < 4 * per_row; p += 64) {
      const int yy = p / per_row, q = p - yy * per_row;
      const long long o = row0 + yy * ystride + spread(4 * q);
      s4v v = *reinterpret_cast<const s4v*>(st + yy * 16 * csl + 4 * q);
      if (mask) v = masked(v, *reinterpret_cast<const s4v*>(mask + o));
      *reinterpret_cast<s4v*>(out + o) = v;
    }
  }
  if (pool) {
    // 2 x 2 x 8 coarse voxels, 4 channels per item
    const Dims dc{dm.lx - 1, dm.ly - 1, dm.lz - 1};
    const int cq = csl >> 2;
    for (int i = threadIdx.x; i < 32 * cq; i += 256) {
      const int v = i / cq, c = 4 * (i - v * cq), xc = v >> 4, yc = (v >> 3) & 1, zc = v & 7;
      float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const s4v e = *reinterpret_cast<const s4v*>(
            tile + (((2 * xc + (q >> 2)) * 4 + 2 * yc + ((q >> 1) & 1)) * 16 + 2 * zc + (q & 1)) * csl + c);
#pragma unroll
        for (int k = 0; k < 4; ++k) a[k] += bf2f((uint16_t)e[k]);
      }
      s4v o;
#pragma unroll
      for (int k = 0; k < 4; ++k) o[k] = (short)f2bf(0.125f * a[k]);
      *reinterpret_cast<s4v*>(pool + dc.encode((x0 >> 1) + xc, (y0 >> 1) + yc, (z0 >> 1) + zc) * cs_out + co0 + c) = o;
    }
  }
}

// LDS bytes of k_conv_ct<CS, NT, *>.
template <int CS, int NT>
constexpr size_t conv_ct_lds() {
  constexpr int NKC = (27 * CS + 15) / 16;
  constexpr int HALO = 648 * CS, STAGE = 256 * 16 * NT;
  constexpr int TILE = ((HALO > STAGE ? HALO : STAGE) + 7) & ~7;
  return sizeof(uint16_t) * TILE + sizeof(int) * NKC * 4;   // the table of either layout fits in NKC * 4
}

// 3x3x3 convolution on an LDS-staged input tile (the same implicit GEMM as k_conv).
// A workgroup of 4 waves computes a 4 (x) x 4 (y) x 16 (z) output tile: the input
// block with its one-voxel halo, 6 x 6 x 18 voxels x cs_in channels (zero outside
// the grid), is loaded once into LDS and every tap reads the A operand from there;
// wave w takes x = x0 + w and four 16-voxel z rows (y = y0 .. y0+3), so each weight
// fragment feeds 4 x NT MFMAs.  Needs lz >= 4, ly >= 2, lx >= 2 and NT*16 >= cout.
// grid = (X/4)(Y/4)(Z/16), block = 256, dynamic LDS = 648 cs_in BF16.
// grid.y splits the output tiles (NT per block).  ODD16: an odd last chunk as a 16-deep
// instruction, as k_conv does, whose layers of three output tiles this form takes.
template <bool RELU, int NT, bool ODD16 = false>
__global__ __launch_bounds__(256) void k_conv_tiled(const uint16_t* __restrict__ in, Dims dm, int cs_in,
                                                    const uint16_t* __restrict__ W, int kp,
                                                    const float* __restrict__ bias, int cout, int cs_out,
                                                    uint16_t* __restrict__ out, const uint16_t* __restrict__ mask) {
  extern __shared__ uint16_t tile[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nzt = dm.lz - 4, nyt = dm.ly - 2;
  const int tz = blockIdx.x & ((1 << nzt) - 1);
  const int rest = blockIdx.x >> nzt;
  const int ty = rest & ((1 << nyt) - 1);
  const int tx = rest >> nyt;
  const int x0 = tx * 4, y0 = ty * 4, z0 = tz * 16;
  stage_halo(tile, in, dm, cs_in, x0, y0, z0);
  __syncthreads();
  const int r = lane & 15, g = lane >> 4, co0 = 16 * NT * blockIdx.y;
  f4v acc[4][NT];
#pragma unroll
  for (int yy = 0; yy < 4; ++yy)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[yy][t] = f4v{0.f, 0.f, 0.f, 0.f};
  int tap = 0, ci = 4 * g;
  while (ci >= cs_in) { ci -= cs_in; ++tap; }
  const int row_stride = 18 * cs_in;            // one (x, y) row of the tile
  // LDS offset of the current chunk's A slice (taps past 26 only meet the zero padding
  // rows of W: their A values stay 0, offset -1), then step to the next chunk
  auto off_next = [&]() {
    int off = -1;
    if (tap < 27) {
      const int dx = tap / 9, dy = (tap / 3) % 3, dz = tap % 3;
      off = ((wave + dx) * 6 + dy) * row_stride + (r + dz) * cs_in + ci;
    }
    ci += 16;
    while (ci >= cs_in) { ci -= cs_in; ++tap; }
    return off;
  };
  auto a_at = [&](int off, int yy) {
    return off >= 0 ? *reinterpret_cast<const s4v*>(tile + off + yy * row_stride) : s4v{0, 0, 0, 0};
  };
  const int nkc = kp >> 4;
  const uint16_t* wr = W + (long long)(co0 + r) * kp + 4 * g;
  // B slices of the chunk pair (kc, kc + 1), loaded one pair ahead; an odd last chunk
  // pairs with zeros (its products add exact zeros)
  s4v nb0[NT], nb1[NT];
  auto load_b = [&](int kc) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      nb0[t] = *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp + kc * 16);
      nb1[t] = kc + 1 < nkc ? *reinterpret_cast<const s4v*>(wr + (long long)t * 16 * kp + kc * 16 + 16) : s4v{0, 0, 0, 0};
    }
  };
  load_b(0);
  for (int kc = 0; kc < nkc; kc += 2) {
    s4v b0[NT], b1[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) { b0[t] = nb0[t]; b1[t] = nb1[t]; }
    if (kc + 2 < nkc) load_b(kc + 2);
    const int off0 = off_next();
    if (ODD16 && kc + 1 >= nkc) {
#pragma unroll
      for (int yy = 0; yy < 4; ++yy) {
        const s4v a0 = a_at(off0, yy);
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[yy][t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0, b0[t], acc[yy][t], 0, 0, 0);
      }
      break;
    }
    const int off1 = kc + 1 < nkc ? off_next() : -1;
#pragma unroll
    for (int yy = 0; yy < 4; ++yy) {
      const s4v a0 = a_at(off0, yy), a1 = a_at(off1, yy);
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[yy][t] = mfma2(a0, a1, b0[t], b1[t], acc[yy][t]);
    }
  }
  // D[row = 4g + j][col = r]: voxel z0 + 4g + j of row (x0 + wave, y0 + yy), channel t*16 + r
#pragma unroll
  for (int yy = 0; yy < 4; ++yy) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int co = co0 + t * 16 + r;
      const float bv = co < cout ? bias[co] : 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const long long nn = dm.encode(x0 + wave, y0 + yy, z0 + 4 * g + j);
        if (co < cout) {
          float v = acc[yy][t][j] + bv;
          if (RELU) v = fmaxf(v, 0.f);
          out[nn * cs_out + co] = keep(mask, nn * cs_out + co) ? f2bf(v) : (uint16_t)0;
        } else if (co < cs_out) {
          out[nn * cs_out + co] = 0;
        }
      }
    }
  }
}

// Weight and bias gradients of every layer in one launch:
//   gW[co][tap][ci] = sum_n gout[n][co] in[n + d(tap)][ci],   gb[co] = sum_n gout[n][co].
// The reduction runs over voxels, so both MFMA operands need 8 voxels of one channel per
// lane while the tensors are channels-last: gfx950's transposing LDS read gives lane i of
// 16 the i-th of the 16 channels that the lanes read 4 at a time over 4 voxels, so an operand
// comes from the tensors' own layout, with no transposed copy and no gather of 2-byte values.
// A lane's 8 voxels are consecutive in z, and three reads (12 voxels) hold the operands of
// the three z taps, each one voxel on from the last.
//
// A task is (layer, up to WG_CC input channels, 16 output channels, a run of voxel tiles).  Per
// tile the block stages the input's halo [voxel][channels] and the gradients [voxel][16].  The
// columns (x and y tap, channel) go in groups of 16, each with its three z taps, over wc of
// the 4 waves, the voxels over the other 4 / wc: the sums stay in registers over the tiles.
// Each task writes its sums to a slice of its own and k_wgrad_sum adds the slices in a fixed
// order (the result is the same on every run, and no buffer has to be cleared).
// What bounds it: the LDS reads and the staging's latency.  It replaced a kernel per
// layer that gathered the operands 2 bytes at a time and added every block's sums with
// atomics, a kernel per layer for small grids and the head, one per layer for the bias and
// one to bring the sums into the flat layout: 610 us together for the 15 layers of the
// (8, 16, 32, 80) network on 64^3 voxels with 11 input channels, 60 us with k_wgrad_sum now.
constexpr int WG_CC = 32;    // input channels per task
constexpr int WG_KG = 5;     // column groups per wave: 9 * 32 / 16 over 4 waves
constexpr int WG_HALO = 648; // halo voxels of a tile at most (4 x 4 x 16)

struct WgLayer {
  const uint16_t* in;
  const uint16_t* gout;    // gradient of the layer's pre-activation output
  Dims dm;
  int cs_in, cs_g, cout, cin, ntap;
  int ltx, lty, ltz;       // log2 of the voxel tile (at most 256 voxels, halo <= WG_HALO; z at least 8)
  int ntx, nty, ntz;       // log2 of the tile counts
  // flat gradients, and the slices: chunk q (input channels), output tile u, split s at
  // base[q] + (u * nsplit + s) * 16 * wg_cols(q), the bias sums at bbase + (u * nsplit + s) * 16
  float* gw;
  float* gb;
  int nsplit, nchunk;
  int sb0, snb;            // blocks of k_wgrad_sum
  long long base[4], bbase;
};
struct WgTask {
  int layer, q, u, split, tile0, ntiles;
};
__host__ __device__ inline int wg_chunk(int cs, int q) { return cs - q * WG_CC < WG_CC ? cs - q * WG_CC : WG_CC; }
// Column groups of a chunk of cc channels, the columns of its slice (group, z tap, 16), and
// the waves that share the columns: enough that a wave's groups fit its registers.
__host__ __device__ inline int wg_groups(int ntap, int cc) { return ((ntap == 1 ? 1 : 9) * cc + 15) / 16; }
__host__ __device__ inline int wg_cols(int ntap, int cc) { return 48 * wg_groups(ntap, cc); }
__host__ __device__ inline int wg_waves(int groups) { return groups <= WG_KG ? 1 : groups <= 2 * WG_KG ? 2 : 4; }

typedef __attribute__((address_space(3))) s4v lds_s4v;
typedef __attribute__((ext_vector_type(2))) unsigned u2v;
typedef __attribute__((ext_vector_type(4))) unsigned u4v;
// 4 voxels of a lane's channel
__device__ __forceinline__ u2v tr_read(const uint16_t* p) {
  return __builtin_bit_cast(u2v, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v*)p));
}

__global__ __launch_bounds__(256) void k_wgrad(const WgLayer* __restrict__ layers, const WgTask* __restrict__ tasks,
                                               float* __restrict__ part) {
  extern __shared__ __align__(16) uint16_t sm[];
  const WgTask tk = tasks[blockIdx.x];
  const WgLayer& ly = layers[tk.layer];
  const Dims dm = ly.dm;
  const int cs_in = ly.cs_in, cs_g = ly.cs_g, ntap = ly.ntap;
  const int cc = wg_chunk(cs_in, tk.q), cq = cc >> 2;
  const int lty = ly.lty, ltz = ly.ltz, nty = ly.nty, ntz = ly.ntz, ltx = ly.ltx;
  const int HX = (1 << ltx) + 2, HY = (1 << lty) + 2, HZ = (1 << ltz) + 2, nh = HX * HY * HZ;
  const int nv = 1 << (ltx + lty + ltz), nvp = nv < 32 ? 32 : nv;
  const int ng = wg_groups(ntap, cc), wc = wg_waves(ng), wv = 4 / wc;
  const uint16_t* __restrict__ in = ly.in + tk.q * WG_CC;
  const uint16_t* __restrict__ gout = ly.gout + 16 * tk.u;
  const int gmax = cs_g - 16 * tk.u;
  uint16_t* gt = sm;                 // [nvp][16]
  uint16_t* halo = sm + 256 * 16;    // [nh][cc], two voxels more are read
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wcol = wave & (wc - 1), wvox = wave / wc;
  const int r = lane & 15, g4 = lane >> 4, rq = r & 3, rv = r >> 2;
  // halo offset of this lane's 4 columns of each of its groups (columns past the last tap
  // read offset 0 and are not summed)
  int off[WG_KG];
#pragma unroll
  for (int k = 0; k < WG_KG; ++k) {
    const int col = (wcol + wc * k) * 16 + 4 * rq, tap = col / cc, ci = col - tap * cc;
    const int dx = ntap == 1 ? 1 : tap / 3, dy = ntap == 1 ? 1 : tap - 3 * (tap / 3);
    off[k] = tap < (ntap == 1 ? 1 : 9) ? (dx * HY + dy) * HZ * cc + ci : 0;
  }
  f4v acc[WG_KG][3], accb = f4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < WG_KG; ++k)
#pragma unroll
    for (int t = 0; t < 3; ++t) acc[k][t] = f4v{0.f, 0.f, 0.f, 0.f};
  const bool bias = tk.q == 0 && wcol == wc - 1;   // the wave with the fewest columns
  s8v ones;
#pragma unroll
  for (int j = 0; j < 8; ++j) ones[j] = (short)0x3f80;
  constexpr int HI = (WG_HALO + 255) / 256;
  for (int it = 0; it < tk.ntiles; ++it) {
    const int tile = tk.tile0 + it;
    const int x0 = (tile >> (nty + ntz)) << ltx, y0 = ((tile >> ntz) & ((1 << nty) - 1)) << lty,
              z0 = (tile & ((1 << ntz) - 1)) << ltz;
    // every load of the tile before the first store
    s4v val[HI][WG_CC / 4], vg[4];
#pragma unroll
    for (int i = 0; i < HI; ++i) {
      const int h0 = threadIdx.x + 256 * i;
      const int hx = h0 / (HY * HZ), hr = h0 - hx * (HY * HZ), hy = hr / HZ, hz = hr - hy * HZ;
      const int gx = x0 + hx - 1, gy = y0 + hy - 1, gz = z0 + hz - 1;
      const bool in_grid = h0 < nh && dm.inside(gx, gy, gz);
      const uint16_t* src = in + dm.encode(in_grid ? gx : 0, in_grid ? gy : 0, in_grid ? gz : 0) * cs_in;
#pragma unroll
      for (int u = 0; u < WG_CC / 4; ++u) {
        val[i][u] = s4v{0, 0, 0, 0};
        if (u < cq && in_grid) val[i][u] = *reinterpret_cast<const s4v*>(src + 4 * u);
      }
    }
    {
      const int v = threadIdx.x;
      const int vx = x0 + (v >> (lty + ltz)), vy = y0 + ((v >> ltz) & ((1 << lty) - 1)), vz = z0 + (v & ((1 << ltz) - 1));
      const bool in_grid = v < nv && vz < (1 << dm.lz);
      const uint16_t* src = gout + dm.encode(in_grid ? vx : 0, in_grid ? vy : 0, in_grid ? vz : 0) * cs_g;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        vg[u] = s4v{0, 0, 0, 0};
        if (in_grid && 4 * u < gmax) vg[u] = *reinterpret_cast<const s4v*>(src + 4 * u);
      }
    }
    __syncthreads();      // the previous tile's reads are done
#pragma unroll
    for (int i = 0; i < HI; ++i) {
      const int h0 = threadIdx.x + 256 * i;
      if (h0 < nh) {
#pragma unroll
        for (int u = 0; u < WG_CC / 4; ++u)
          if (u < cq) *reinterpret_cast<s4v*>(halo + h0 * cc + 4 * u) = val[i][u];
      }
    }
    if ((int)threadIdx.x < nvp) {
#pragma unroll
      for (int u = 0; u < 4; ++u) *reinterpret_cast<s4v*>(gt + threadIdx.x * 16 + 4 * u) = vg[u];
    }
    __syncthreads();
    for (int vb = 32 * wvox; vb < nvp; vb += 32 * wv) {
      // this lane's 8 voxels along z; past the tile's last voxel the gradients are zero and
      // the input any finite entry
      const int v8 = vb + 8 * g4, vi = v8 & (nv - 1);
      const uint16_t* h = halo + (((vi >> (lty + ltz)) * HY + ((vi >> ltz) & ((1 << lty) - 1))) * HZ + (vi & ((1 << ltz) - 1)) + rv) * cc;
      const u2v al = tr_read(gt + (v8 + rv) * 16 + 4 * rq), ah = tr_read(gt + (v8 + 4 + rv) * 16 + 4 * rq);
      const bf8v a = __builtin_bit_cast(bf8v, u4v{al[0], al[1], ah[0], ah[1]});
      if (bias) accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf8v, ones), accb, 0, 0, 0);
#pragma unroll
      for (int k = 0; k < WG_KG; ++k) {
        if (wcol + wc * k < ng) {
          const u2v w0 = tr_read(h + off[k]), w1 = tr_read(h + off[k] + 4 * cc), w2 = tr_read(h + off[k] + 8 * cc);
          const u4v b0 = {w0[0], w0[1], w1[0], w1[1]}, b2 = {w0[1], w1[0], w1[1], w2[0]};
          u4v b1;
#pragma unroll
          for (int i = 0; i < 4; ++i) b1[i] = __builtin_amdgcn_alignbit(b2[i], b0[i], 16);
          acc[k][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf8v, b0), acc[k][0], 0, 0, 0);
          acc[k][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf8v, b1), acc[k][1], 0, 0, 0);
          acc[k][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf8v, b2), acc[k][2], 0, 0, 0);
        }
      }
    }
  }
  // the waves that share columns, added into the first in order
  f4v* red = reinterpret_cast<f4v*>(sm) + wcol * (3 * WG_KG + 1) * 64 + lane;
  for (int s = 1; s < wv; ++s) {
    __syncthreads();
    if (wvox == s) {
#pragma unroll
      for (int k = 0; k < WG_KG; ++k)
#pragma unroll
        for (int t = 0; t < 3; ++t) red[(3 * k + t) * 64] = acc[k][t];
      red[3 * WG_KG * 64] = accb;
    }
    __syncthreads();
    if (!wvox) {
#pragma unroll
      for (int k = 0; k < WG_KG; ++k)
#pragma unroll
        for (int t = 0; t < 3; ++t) acc[k][t] += red[(3 * k + t) * 64];
      accb += red[3 * WG_KG * 64];
    }
  }
  if (wvox) return;
  // D[row = 4 g4 + j][col = r]: output channel 4 g4 + j, column r of the group and z tap
  const int ncol = 48 * ng;
  const long long slice = tk.u * ly.nsplit + tk.split;
  float* __restrict__ dst = part + ly.base[tk.q] + slice * (16 * ncol);
#pragma unroll
  for (int k = 0; k < WG_KG; ++k) {
    if (wcol + wc * k < ng) {
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[(4 * g4 + j) * ncol + 48 * (wcol + wc * k) + 16 * t + r] = acc[k][t][j];
    }
  }
  if (bias && r == 0) *reinterpret_cast<f4v*>(part + ly.bbase + slice * 16 + 4 * g4) = accb;
}

// LDS bytes of k_wgrad for cc channels and nh halo voxels.
inline size_t wgrad_lds(int ntap, int cc, int nh) {
  const int wc = wg_waves(wg_groups(ntap, cc));
  const size_t stage = sizeof(uint16_t) * (256 * 16 + (size_t)(nh + 2) * cc), red = wc < 4 ? sizeof(f4v) * 64 * (3 * WG_KG + 1) * wc : 0;
  return stage > red ? stage : red;
}

// The slices of k_wgrad added up into the flat gradient, every layer in one launch (blocks
// [sb0, sb0 + snb) serve layer l).  Latency bounds it: the level-0 layers have few values of
// many slices, which one thread per value with four loads in flight added in 26 us for 15
// layers of up to 256 slices.  So a value of WS_MANY slices or more has 16 threads, each
// with eight loads in flight, whose sums are added in order: 9.9 us.
constexpr int WS_MANY = 32;
__host__ __device__ inline int ws_vals(int nsplit) { return nsplit >= WS_MANY ? 16 : 256; }   // values per block
struct WgBlocks {
  int sb0[24];   // first block of layers 1, 2, ... (23 layers at most), INT_MAX beyond the last
};
__global__ __launch_bounds__(256) void k_wgrad_sum(const WgLayer* __restrict__ layers, WgBlocks first, const float* __restrict__ part) {
  __shared__ float sums[256];
  int l = 0;
#pragma unroll
  for (int k = 0; k < 24; ++k) l += (int)blockIdx.x >= first.sb0[k];
  const WgLayer& ly = layers[l];
  const int nw = ly.cout * ly.ntap * ly.cin, n = nw + ly.cout, ns = ly.nsplit;
  const int vals = ws_vals(ns), ngrp = 256 / vals, grp = threadIdx.x / vals, v0 = threadIdx.x & (vals - 1);
  const int i = (blockIdx.x - ly.sb0) * vals + v0;
  float acc = 0.f;
  if (i < n) {
    const float* src;
    long long step;
    if (i < nw) {
      const int rest = i / ly.cin, ci = i - rest * ly.cin, co = rest / ly.ntap, tap = rest - co * ly.ntap;
      const int q = ci / WG_CC, cc = wg_chunk(ly.cs_in, q), ncol = wg_cols(ly.ntap, cc);
      const int xy = ly.ntap == 1 ? 0 : tap / 3, dz = ly.ntap == 1 ? 1 : tap - 3 * xy, col = xy * cc + ci - q * WG_CC;
      step = 16 * ncol;
      src = part + ly.base[q] + (long long)(co >> 4) * ns * step + (co & 15) * ncol + (3 * (col >> 4) + dz) * 16 + (col & 15);
    } else {
      const int co = i - nw;
      step = 16;
      src = part + ly.bbase + (long long)(co >> 4) * ns * step + (co & 15);
    }
    constexpr int U = 8;
    for (int s0 = grp; s0 < ns; s0 += ngrp * U) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = s0 + ngrp * u < ns ? src[(s0 + ngrp * u) * step] : 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u) acc += v[u];
    }
  }
  if (ngrp > 1) {
    sums[threadIdx.x] = acc;
    __syncthreads();
    if (!grp)
      for (int k = 1; k < 16; ++k) acc += sums[k * 16 + v0];
  }
  if (grp || i >= n) return;
  if (i < nw) ly.gw[i] = acc;
  else ly.gb[i - nw] = acc;
}

// FP32 channel-major volumes [C][src] / scale -> BF16 channels-last [N][cs] (crop
// window (o, dst) of the source; channels C..cs-1 zero).  The scale comes from k_absmax's
// slot; it is stored for the kernels after the network, and the loss is cleared.
__global__ void k_to_bf16_crop(const float* __restrict__ x, int C, Dims src, int ox, int oy, int oz, Dims dst,
                               const unsigned* __restrict__ slot, double* __restrict__ scale, double* __restrict__ loss, int cs,
                               uint16_t* __restrict__ out) {
  const long long N = dst.n(), ns = src.n();
  const float top = __uint_as_float(*slot);
  const double sc = top > 0.f ? (double)top : 1.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *scale = sc;
    *loss = 0.0;
  }
  const float inv = (float)(1.0 / sc);
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N; i += (long long)gridDim.x * blockDim.x) {
    int x0, y0, z0;
    dst.decode(i, x0, y0, z0);
    const long long j = src.encode(x0 + ox, y0 + oy, z0 + oz);
    for (int c4 = 0; c4 < cs; c4 += 4) {   // cs is a multiple of 4: 8-byte stores
      s4v v;
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = (short)(c4 + q < C ? f2bf(x[(c4 + q) * ns + j] * inv) : (uint16_t)0);
      *reinterpret_cast<s4v*>(out + i * cs + c4) = v;
    }
  }
}

// 2x2x2 average pooling (channels-last).
__global__ void k_avgpool(const uint16_t* __restrict__ in, Dims di, int cs, uint16_t* __restrict__ out, Dims dout) {
  const long long N = dout.n() * cs;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N; i += (long long)gridDim.x * blockDim.x) {
    const long long n = i / cs;
    const int c = (int)(i - n * cs);
    int x, y, z;
    dout.decode(n, x, y, z);
    float s = 0.f;
    for (int q = 0; q < 8; ++q) s += bf2f(in[di.encode(2 * x + (q >> 2), 2 * y + ((q >> 1) & 1), 2 * z + (q & 1)) * cs + c]);
    out[i] = f2bf(0.125f * s);
  }
}

// Gradient of an encoder output that feeds both the skip connection and the pool: the
// concatenation's gradient (its first cs channels, stride cs_cat) plus an eighth of the
// pooled voxel's, zeroed where the output act is not > 0.  Items of 4 channels.
__global__ void k_skip_pool_bwd(const uint16_t* __restrict__ gcat, int cs_cat, const uint16_t* __restrict__ gpool, Dims dp,
                                int cs, int c1, const uint16_t* __restrict__ act, uint16_t* __restrict__ out, Dims di) {
  const int cq = cs >> 2;
  const long long N = di.n() * cq;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N; i += (long long)gridDim.x * blockDim.x) {
    const long long n = i / cq;
    const int c = 4 * (int)(i - n * cq);
    int x, y, z;
    di.decode(n, x, y, z);
    const s4v gp = *reinterpret_cast<const s4v*>(gpool + dp.encode(x >> 1, y >> 1, z >> 1) * cs + c);
    const s4v av = *reinterpret_cast<const s4v*>(act + n * cs + c);
    // the skip channels of the concatenation end at c1, its padding is not part of them
    const s4v gc = *reinterpret_cast<const s4v*>(gcat + n * cs_cat + c);
    s4v v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float skip = c + q < c1 ? bf2f((uint16_t)gc[q]) : 0.f;
      v[q] = (short)f2bf(skip + 0.125f * bf2f((uint16_t)gp[q]));
    }
    *reinterpret_cast<s4v*>(out + n * cs + c) = masked(v, av);
  }
}

// out[n] = [skip[n][0:c1], coarse[n/2][0:c2], 0...] (nearest upsampling + concat).
// One thread per (fine voxel, group of 4 channels), 8-byte stores in memory order; a
// group that lies within one source at a 4-aligned offset is one 8-byte load (the
// channel strides are multiples of 4), any other group is gathered channel by channel.
__global__ void k_upcat(const uint16_t* __restrict__ skip, int cs1, int c1, const uint16_t* __restrict__ coarse, int cs2,
                        int c2, Dims df, Dims dc, int cs, uint16_t* __restrict__ out) {
  const int cq = cs >> 2;
  const long long N = df.n() * cq;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N; i += (long long)gridDim.x * blockDim.x) {
    const long long n = i / cq;
    const int c = 4 * (int)(i - n * cq);
    int x, y, z;
    df.decode(n, x, y, z);
    const uint16_t* sr = skip + n * cs1;
    const uint16_t* cr = coarse + dc.encode(x >> 1, y >> 1, z >> 1) * cs2;
    s4v v = s4v{0, 0, 0, 0};
    if (c + 4 <= c1) {
      v = *reinterpret_cast<const s4v*>(sr + c);
    } else if (c >= c1 && c + 4 <= c1 + c2 && ((c - c1) & 3) == 0) {
      v = *reinterpret_cast<const s4v*>(cr + (c - c1));
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int cc = c + q;
        v[q] = (short)(cc < c1 ? sr[cc] : (cc < c1 + c2 ? cr[cc - c1] : (uint16_t)0));
      }
    }
    *reinterpret_cast<s4v*>(out + 4 * i) = v;
  }
}

// Gradient of the coarse tensor of a concatenation: the sum over its 8 children of the
// channels c1 .. c1 + c2 - 1, zeroed where act (the coarse tensor) is not > 0.
__global__ void k_up_bwd(const uint16_t* __restrict__ g, int cs, int c1, int c2, Dims df, Dims dc,
                         const uint16_t* __restrict__ act, uint16_t* __restrict__ gcoarse, int cs2) {
  const long long Nc = dc.n() * cs2;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < Nc; i += (long long)gridDim.x * blockDim.x) {
    const long long m = i / cs2;
    const int c = (int)(i - m * cs2);
    float s = 0.f;
    if (c < c2) {
      int x, y, z;
      dc.decode(m, x, y, z);
      uint16_t v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = g[df.encode(2 * x + (q >> 2), 2 * y + ((q >> 1) & 1), 2 * z + (q & 1)) * cs + c1 + c];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += bf2f(v[q]);
    }
    gcoarse[i] = bf2f(act[i]) > 0.f ? f2bf(s) : (uint16_t)0;
  }
}

// Data gradient of the 1x1x1 head (one output channel, W the first row of its packed matrix):
// g[n][c] = gy[n] W[c], zeroed where act is not > 0.  gy is channel 0 of stride 4.
__global__ void k_head_bwd(const uint16_t* __restrict__ gy, long long N, int cs, int c, const uint16_t* __restrict__ W,
                           const uint16_t* __restrict__ act, uint16_t* __restrict__ g) {
  const int cq = cs >> 2;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N * cq; i += (long long)gridDim.x * blockDim.x) {
    const long long n = i / cq;
    const int c4 = 4 * (int)(i - n * cq);
    const float gv = bf2f(gy[4 * n]);
    s4v v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = (short)(c4 + q < c ? f2bf(gv * bf2f(W[c4 + q]) + 0.f) : (uint16_t)0);
    *reinterpret_cast<s4v*>(g + 4 * i) = masked(v, *reinterpret_cast<const s4v*>(act + 4 * i));
  }
}

// MSE on a crop: loss += sum (y - t/s)^2 / n (FP64 atomics); gy = 2 (y - t/s) / n as BF16 [N][4] (channel 0).
__global__ void k_mse(const float* __restrict__ y, const float* __restrict__ t, Dims src, int ox, int oy, int oz,
                      Dims dm, const double* __restrict__ scale, uint16_t* __restrict__ gy, double* __restrict__ loss) {
  __shared__ double part[4];   // 256 threads
  const long long N = dm.n();
  const float inv = (float)(1.0 / *scale);
  double acc = 0.0;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N; i += (long long)gridDim.x * blockDim.x) {
    int x, yy, z;
    dm.decode(i, x, yy, z);
    const float e = y[i] - t[src.encode(x + ox, yy + oy, z + oz)] * inv;
    acc += (double)e * (double)e;
    *reinterpret_cast<s4v*>(gy + 4 * i) = s4v{(short)f2bf(2.f * e / (float)N), 0, 0, 0};
  }
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(loss, (part[0] + part[1] + part[2] + part[3]) / (double)N);
}

// max_i |sum_c x[c][i]| over C channel-major volumes of n voxels: per-block maxima
// folded into *slot with an integer atomic max (the bit patterns of non-negative
// floats order like their values).  k_to_bf16_crop turns the slot into the scale (1 if the
// maximum is 0) and k_head1, the last kernel of the forward pass, clears it for the next call.
// Items of 4 consecutive voxels (n is a multiple of 4), channels summed in order.  128^3, 11
// channels: 35.2 us with the channels loaded one after another (2.6 TB/s) and an atomic from each of 2048 blocks,
// 23 us (4.0 TB/s) with six in flight and 1024 blocks.
__global__ void k_absmax(const float* __restrict__ x, long long n, int C, unsigned* __restrict__ slot) {
  __shared__ float part[4];   // 256 threads
  float m = 0.f;
  const long long n4 = n >> 2;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n4; i += (long long)gridDim.x * blockDim.x) {
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int U = 6;   // channels in flight
    for (int c0 = 0; c0 < C; c0 += U) {
      float4 a[U];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c0 + u < C) a[u] = reinterpret_cast<const float4*>(x + (c0 + u) * n)[i];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c0 + u < C) { v.x += a[u].x; v.y += a[u].y; v.z += a[u].z; v.w += a[u].w; }
    }
    m = fmaxf(fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w)));
  }
  for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) atomicMax(slot, __float_as_uint(fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]))));
}
// 1x1x1 convolution to one FP32 output channel (the head): y[n] = b + sum_c W[c] in[n][c],
// W the first row of the packed BF16 forward matrix, FP32 sums.
__global__ void k_head1(const uint16_t* __restrict__ in, long long N, int cs_in, int cin, const uint16_t* __restrict__ W,
                        const float* __restrict__ bias, float* __restrict__ y, unsigned* __restrict__ slot) {
  const float b = bias[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) *slot = 0u;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < N; i += (long long)gridDim.x * blockDim.x) {
    float acc = 0.f;
    for (int c4 = 0; c4 < cs_in; c4 += 4) {
      const s4v v = *reinterpret_cast<const s4v*>(in + i * cs_in + c4);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (c4 + q < cin) acc += bf2f((uint16_t)v[q]) * bf2f(W[c4 + q]);
    }
    y[i] = acc + b;
  }
}

// rho = s * max(y, 0)
__global__ void k_scale_relu(const float* __restrict__ y, long long n, const double* __restrict__ scale, float* __restrict__ rho) {
  const float s = (float)*scale;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x)
    rho[i] = s * fmaxf(y[i], 0.f);
}

// One layer's matrices for the packing kernels, and the range of the launch's blocks
// that serve it (every layer in one launch: blocks [b0, b0 + nb) take layer l).
struct PackDesc {
  const float* p;          // the layer's weights in the flat FP32 parameters
  uint16_t* Wf;
  uint16_t* Wt;
  int cin, cout, ks, cs_in, cs_out, kp, kpt, rows_f, rows_t;
  int pb0, pnb;            // blocks of k_pack_all
};

// Master FP32 layer parameters (flat layout W[co][tap][cin], bias) -> BF16 GEMM
// matrices: forward W[co_pad][kp] with k = tap*cs_in + ci, and the flipped,
// transposed matrix of the data gradient Wt[ci_pad][kpt] with k = tap'*cs_out + co,
// Wt[ci][tap'][co] = W[co][ntap-1-tap'][ci].  All nl layers in one launch.
__global__ void k_pack_all(const PackDesc* __restrict__ ds, int nl) {
  int l = 0;
  while (l + 1 < nl && (int)blockIdx.x >= ds[l + 1].pb0) ++l;
  const PackDesc& d = ds[l];
  const int ntap = d.ks * d.ks * d.ks;
  const long long nf = (long long)d.rows_f * d.kp, nt = (long long)d.rows_t * d.kpt;
  for (long long i = (blockIdx.x - d.pb0) * (long long)blockDim.x + threadIdx.x; i < nf + nt;
       i += (long long)d.pnb * blockDim.x) {
    if (i < nf) {
      const int co = (int)(i / d.kp), k = (int)(i - (long long)co * d.kp);
      const int tap = k / d.cs_in, ci = k - tap * d.cs_in;
      float v = 0.f;
      if (co < d.cout && tap < ntap && ci < d.cin) v = d.p[((long long)co * ntap + tap) * d.cin + ci];
      d.Wf[i] = f2bf(v);
    } else {
      const long long j = i - nf;
      const int ci = (int)(j / d.kpt), k = (int)(j - (long long)ci * d.kpt);
      const int tp = k / d.cs_out, co = k - tp * d.cs_out;
      float v = 0.f;
      if (ci < d.cin && tp < ntap && co < d.cout) v = d.p[((long long)co * ntap + (ntap - 1 - tp)) * d.cin + ci];
      d.Wt[j] = f2bf(v);
    }
  }
}

// Adam (Kingma & Ba 2015) on FP32 master parameters.
__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       long long n, float lr, float b1, float b2, float eps, float c1, float c2) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  }
}

__global__ void k_fill_f32(float* __restrict__ p, long long n, float v) {
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) p[i] = v;
}

}  // namespace net
}  // namespace mh3d
