// Transforms of groups of lines in LDS for passes whose line counts are known only at
// run time: the stages of fast.hpp's transforms (consecutive lanes on consecutive lines,
// odd line stride, out of place, a barrier after each stage) with the length a
// compile-time constant chosen by a block-uniform switch, and the line count and stride
// run-time values.
//
// Radices are chosen for few stages (every length that the switch knows takes at most two, but
// for 108 and 192, and for 96, 128, 144 and 256 in the class passes, see line_radix): a stage costs
// an LDS round trip and a barrier, and with the few lines of one workgroup that chain is most
// of a pass.  Other lengths (2, 3, 81, 162, 216, 243) take the run-time engine of fft_lds.hpp.
#pragma once
#include "fft_lds.hpp"
#include "geo.hpp"

namespace mh3d {

// radices 6, 9 and 12 as products of two smaller ones (decimation in time, the twiddles
// exp(SGN 2 pi i p / R) written out)
template <int SGN, typename C> __device__ __forceinline__ void dft6(C* v) {
  using R = typename real_of<C>::type;
  const R h = (R)0.86602540378443864676;
  C e[3] = {v[0], v[2], v[4]}, o[3] = {v[1], v[3], v[5]};
  dft3<SGN>(e);
  dft3<SGN>(o);
  const C t1 = cmul(o[1], cmk<C>((R)0.5, (R)SGN * h)), t2 = cmul(o[2], cmk<C>((R)-0.5, (R)SGN * h));
  v[0] = cadd(e[0], o[0]);
  v[3] = csub(e[0], o[0]);
  v[1] = cadd(e[1], t1);
  v[4] = csub(e[1], t1);
  v[2] = cadd(e[2], t2);
  v[5] = csub(e[2], t2);
}
template <int SGN, typename C> __device__ __forceinline__ void dft9(C* v) {
  using R = typename real_of<C>::type;
  // cos and sin of 2 pi / 9, 4 pi / 9, 8 pi / 9
  const R c1 = (R)0.76604444311897803520, s1 = (R)0.64278760968653932632;
  const R c2 = (R)0.17364817766693034885, s2 = (R)0.98480775301220805937;
  const R c4 = (R)-0.93969262078590838405, s4 = (R)0.34202014332566873304;
  C a[3][3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    a[r][0] = v[r]; a[r][1] = v[r + 3]; a[r][2] = v[r + 6];
    dft3<SGN>(a[r]);
  }
  a[1][1] = cmul(a[1][1], cmk<C>(c1, (R)SGN * s1));
  a[1][2] = cmul(a[1][2], cmk<C>(c2, (R)SGN * s2));
  a[2][1] = cmul(a[2][1], cmk<C>(c2, (R)SGN * s2));
  a[2][2] = cmul(a[2][2], cmk<C>(c4, (R)SGN * s4));
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    C t[3] = {a[0][p], a[1][p], a[2][p]};
    dft3<SGN>(t);
    v[p] = t[0]; v[p + 3] = t[1]; v[p + 6] = t[2];
  }
}
template <int SGN, typename C> __device__ __forceinline__ void dft12(C* v) {
  using R = typename real_of<C>::type;
  const R h = (R)0.86602540378443864676;
  C a[3][4];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
#pragma unroll
    for (int q = 0; q < 4; ++q) a[r][q] = v[3 * q + r];
    dft4<SGN>(a[r]);
  }
  // w^(r p), w = exp(SGN 2 pi i / 12)
  a[1][1] = cmul(a[1][1], cmk<C>(h, (R)SGN * (R)0.5));
  a[1][2] = cmul(a[1][2], cmk<C>((R)0.5, (R)SGN * h));
  a[1][3] = cmul_i<SGN>(a[1][3]);
  a[2][1] = cmul(a[2][1], cmk<C>((R)0.5, (R)SGN * h));
  a[2][2] = cmul(a[2][2], cmk<C>((R)-0.5, (R)SGN * h));
  a[2][3] = cscale(a[2][3], (R)-1);
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    C t[3] = {a[0][p], a[1][p], a[2][p]};
    dft3<SGN>(t);
    v[p] = t[0]; v[p + 4] = t[1]; v[p + 8] = t[2];
  }
}
template <int R, int SGN, typename C> __device__ __forceinline__ void dft_any(C* v) {
  if constexpr (R == 6) dft6<SGN>(v);
  else if constexpr (R == 9) dft9<SGN>(v);
  else if constexpr (R == 12) dft12<SGN>(v);
  else dft<R, SGN>(v);
}

// Radix of stage s for the lengths of the switch below.  few: of the class passes,
// whose workgroups have a few lines each.  A radix-16 stage is then one partly filled wave, and a wave
// alone takes about 5000 cycles for the two of a length-256 line against 2600 for three
// stages of radix 8 and 4 over four times the lanes (class pass of 256 x 256 images: 15.6 against
// 14.0 us).
__host__ __device__ constexpr int line_radix(int n, int s, bool few) {
  if (few) {
    constexpr int plan[][4] = {{96, 8, 4, 3}, {128, 8, 4, 4}, {144, 6, 6, 4}, {256, 8, 8, 4}};
    for (auto& p : plan)
      if (p[0] == n) return s < 3 ? p[1 + s] : 0;
  }
  constexpr int plan[][4] = {
      {4, 4, 0, 0},   {6, 6, 0, 0},   {8, 8, 0, 0},   {9, 9, 0, 0},
      {12, 4, 3, 0},  {16, 4, 4, 0},  {18, 6, 3, 0},  {24, 8, 3, 0},  {27, 9, 3, 0},  {32, 8, 4, 0},
      {36, 6, 6, 0},  {48, 8, 6, 0},  {54, 9, 6, 0},  {64, 8, 8, 0},  {72, 9, 8, 0},  {96, 12, 8, 0},
      {108, 6, 6, 3}, {128, 16, 8, 0}, {144, 12, 12, 0}, {192, 8, 6, 4}, {256, 16, 16, 0}};
  for (auto& p : plan)
    if (p[0] == n) return s < 3 ? p[1 + s] : 0;
  return 0;
}

// nl lines of one length, element p of line l at buffer[l * ls + p]
struct Lines {
  int nl, ls;
  int T;       // threads of the block
  MDiv md;     // divides by nl
};

// ld(l, p): element p of line l of the stage's input
template <int N, int R, int NS, int SGN, class Load>
__device__ __forceinline__ void line_stage(Load ld, float2* __restrict__ out, const float2* tw, const Lines& L) {
  constexpr int NB = N / R, TWS = N / (NS * R);
  const int total = L.nl * NB;
  for (int b = threadIdx.x; b < total; b += L.T) {
    const int j = L.md.div(b), l = b - __mul24(j, L.nl);
    __builtin_assume(j >= 0 && j < NB);
    const int k = j % NS;
    float2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = ld(l, j + r * NB);
    if constexpr (NS > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) {
        const float2 w = tw[k * r * TWS];
        v[r] = SGN < 0 ? cmul(v[r], w) : cmulcj(w, v[r]);
      }
    }
    dft_any<R, SGN>(v);
    float2* o = out + __mul24(l, L.ls) + (j / NS) * NS * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) o[r * NS] = v[r];
  }
}

template <int N, int S, int NS, int SGN, bool FEW>
__device__ __forceinline__ float2* line_stages(float2* a, float2* b, const float2* tw, const Lines& L) {
  constexpr int R = S < 3 ? line_radix(N, S, FEW) : 0;
  if constexpr (R == 0) {
    return a;
  } else {
    line_stage<N, R, NS, SGN>([&](int l, int p) { return a[__mul24(l, L.ls) + p]; }, b, tw, L);
    __syncthreads();
    return line_stages<N, S + 1, NS * R, SGN, FEW>(b, a, tw, L);
  }
}

// Length-n transforms (unnormalised) of L's lines, the inputs from ld (computed from
// memory that the first stage is the last to read): the first stage writes *a, the rest
// ping-pong between *a and *b.  Returns the buffer holding the result.  No leading
// barrier; ends with one.  Lengths that the switch does not know are copied to *a and
// take the run-time engine.  MANY: where thousands of lines of one to three points can come
// together (the small grid's y' lines), beyond the range of MDiv::div.
template <int SGN, bool FEW = false, bool MANY = false, class Load>
__device__ __forceinline__ float2* line_fft_ld(Load ld, float2* a, float2* b, const float2* tw, int n, const Lines& L) {
  switch (n) {
#define MH3D_LN(NN)                                                                       \
  case NN: {                                                                              \
    constexpr int R = line_radix(NN, 0, FEW);                                                \
    line_stage<NN, R, 1, SGN>(ld, a, tw, L);                                              \
    __syncthreads();                                                                      \
    return line_stages<NN, 1, R, SGN, FEW>(a, b, tw, L);                                  \
  }
    MH3D_LN(4) MH3D_LN(6) MH3D_LN(8) MH3D_LN(9) MH3D_LN(12) MH3D_LN(16) MH3D_LN(18) MH3D_LN(24) MH3D_LN(27)
    MH3D_LN(32) MH3D_LN(36) MH3D_LN(48) MH3D_LN(54) MH3D_LN(64) MH3D_LN(72) MH3D_LN(96) MH3D_LN(108) MH3D_LN(128)
    MH3D_LN(144) MH3D_LN(192) MH3D_LN(256)
#undef MH3D_LN
    default: {
      const int total = L.nl * n;
      for (int i = threadIdx.x; i < total; i += L.T) {
        int p = L.md.div(i), l = i - p * L.nl;
        if constexpr (MANY) p = L.md.div_any(i, l);
        a[l * L.ls + p] = ld(l, p);
      }
      return fft_lds<SGN>(a, b, tw, n, L.nl, LineMap{L.nl, 0, L.ls, 1}, true);
    }
  }
}

// The same for lines in *a: the stages ping-pong between *b and *a, starting from *a.
template <int SGN, bool FEW = false, bool MANY = false>
__device__ __forceinline__ float2* line_fft(float2* a, float2* b, const float2* tw, int n, const Lines& L) {
  const int ls = L.ls;
  return line_fft_ld<SGN, FEW, MANY>([=](int l, int p) { return a[__mul24(l, ls) + p]; }, b, a, tw, n, L);
}

}  // namespace mh3d
