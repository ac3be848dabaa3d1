// Launchers of the separable passes, defined in translation units of their own (sep.hip,
// fast.hip, user.hip): their kernels are most of the library's code, and the units compile side by
// side.
#pragma once
#include "kernels.hpp"

namespace mh3d {

// Column-pass modes beyond NRM_RESID, NRM_PLAIN and NRM_STORE (kernels.hpp): A alone, A^T
// alone, and COL_DATA, the x' transform of the measured portraits' small-grid spectra (G,
// as the small-grid pass left them) into G' as [k][column][q'x], the solver's data term.
enum { COL_FWD = 16, COL_ADJ = 17, COL_DATA = 18 };
constexpr int SXR = 4;   // x aliases that the column pass keeps in registers

// ---------------------------------------------------------------------------- fast passes
// Launchers of the compile-time-geometry passes (fast.hpp) of one grid, decimation and
// tile shape.  All passes of a fused sequence come from one entry (their slot layout is
// their own).
struct FastOps {
  int nx, ny, nz, sx, sy, sz, kmax;
  int nbp, ncls_blocks, tc;
  size_t lds_plane, lds_class;
  void (*plane_fwd)(hipStream_t, const VolDesc*, int src, const float* a);
  void (*cls)(hipStream_t, const VolDesc*, int mode, int chk, int fin);
  void (*plane_adj)(hipStream_t, const VolDesc*, int out, AdjOut ao);
  void (*adj_and_store)(hipStream_t, const VolDesc*, AdjOut ao, float* d, int nsmall, int xb);
  void (*small_inv)(hipStream_t, const VolDesc*, float* d, int nsmall, int xb);
  // A^T of nv single-harmonic descriptors at once (each with its own qx): out volumes
  // out + v N for v < nv
  void (*adjoint_each)(hipStream_t, const VolDesc*, int nv, float* out);
  // the portraits' small-grid spectra into G' (as k_sep_small_fwd)
  void (*small_fwd)(hipStream_t, const VolDesc*, const float* r, float2* out, int nsmall, int xb);
};

// The compiled grids.
extern const FastOps kFast[];
extern const int kFastCount;

// ---------------------------------------------------------------------------- run-time geometry
// tasks: the task table of a batch, or NULL (descriptor blockIdx.y, block blockIdx.x).
void sep_launch_plane_fwd(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const int2* tasks,
                          const float* a, int src);
// fin: with the finish of the previous update (one block more; in a batch the table's tasks of
// local block -1).  any: the general form (harmonics in groups, any number of x aliases and y
// residues)
void sep_launch_col(bool any, int mode, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd,
                    const int2* tasks, int chk, int fin = 0);
void sep_launch_plane_adj(int out, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const int2* tasks,
                          AdjOut ao);
void sep_launch_adj_and_store(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, AdjOut ao, float* d,
                              int nbp);
void sep_launch_small_inv(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const int2* tasks, float* d,
                          int epi);
void sep_launch_small_fwd(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const float* r, float2* out);

// ---------------------------------------------------------------------------- user PSFs
// Packed class-layout table: row in bits 0-15, column (qz <= nz/2) in bits 16-23
constexpr int CIDX_CONJ = 1 << 30;      // the element is the conjugate of that position
constexpr int CIDX_OWNER = 1 << 29;     // the position is read back from this element
enum { CLS_FWD = 0, CLS_ADJ = 1, CLS_NORMAL = 2 };   // see user_class.hpp
// splits for which the class passes are compiled with all components of a vector plan at once
constexpr bool user_all_at_once(int e) { return e == 1 || e == 2 || e == 4; }
void user_launch_plane_fwd(dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, const float* a, int src);
// rounds: a workgroup's LDS does not hold every component
void user_launch_plane_adj(bool rounds, int out, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, AdjOut ao);
void user_launch_step_and_fwd(bool rounds, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, AdjOut ao);
void user_launch_adj_and_store(bool rounds, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, AdjOut ao,
                               float* d);
void user_launch_class1(int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk, int mode, int fin);
void user_launch_class2(int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk, int mode, int fin);
void user_launch_class4(int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk, int mode, int fin);
void user_launch_class3689(int E, int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk,
                           int mode, int fin);
void user_launch_class(int E, int cb, int dir, dim3 grid, dim3 block, size_t lds, hipStream_t s, const VolDesc* vd, int chk,
                       int mode, int fin);

}  // namespace mh3d
