// Internal structures shared by the host plan (wvl_host.cpp) and the HIP
// kernels (wvl_kernels.hip).  Not part of the public ABI.
#pragma once

#include <stdint.h>

#include "../../include/wvl.h"

namespace wvl {

// Per support function, device resident.  Boxes use local indices:
// input coarse i in [0, n), fine real-space l in [-14, 2n+14] stored at
// l + 14, output coarse i in [-ext, n+ext) stored at i + ext.
struct SfDev {
  double c[3];        // localization centre (bohr), for the confining potential
  int32_t lo[3];
  int32_t n[3];
  int32_t ext;
  int32_t pad0;
  int64_t cin;        // input coefficient offset (elements)
  int64_t cout;       // output coefficient offset
  int64_t n_c, n_f, on_c, on_f;
  int64_t box_in;     // dense input box offset (wvl_uncompress)
  int64_t box_out;    // dense output box offset (wvl_compress)
  // row tables: for pattern p (0 in-coarse, 1 in-fine, 2 out-coarse,
  // 3 out-fine) entry rt[p] + r .. rt[p] + r + 1 bounds the segments of box
  // row r = (i3 - oz) * by + (i2 - oy), as indices into the segment array.
  int64_t rt[4];
  // tight bounding boxes (x0, x1, y0, y1, z0, z1) of the input and output
  // coarse patterns, global indices (empty pattern: x0 > x1).
  int32_t bb_in[6];
  int32_t bb_out[6];
  // compact row runs: for pattern p, RowRun entry rr[p] + r describes box
  // row r (same row numbering as rt)
  int64_t rr[4];
};

// One box row of a pattern: its single run [x0, x0 + len) starting at
// coefficient `off` of the pattern; len 0 = empty row, kMultiRun = several
// runs (walk the segments through the row table instead).
struct RowRun {
  uint16_t x0, len;
  int32_t off;
};
constexpr uint16_t kMultiRun = 0xFFFF;

// k_back_out: output rows (y', z') per block, 16 per wave (one wave per block
// measured fastest: the waves share no LDS, more blocks fit a CU)
constexpr int kBackOutRows = 16;

// Workspace offsets (elements of the compute type) of one support function
// in the workspace (R = 2N + 29, O = N + 2 ext).  The plan keeps these
// records in its processing order (functions sorted by box size, cut into
// chunks); kernels find the function's SfDev through `id`.
//   c8   dense input box, x fastest      [8][N2][N1][N0]
//   c8x  dense input box, y fastest      [8][N2][N0][N1]
//   g1   after the x, y up passes        [2][N2][R1][R0]
//   g2   after the z column pass         [2][O2][R1][R0]
//   q    after the y down pass           [4][O2][R0][O1]   (channel a2 + 2 a3)
//   ox   x part of the kinetic term      [8][N2][O0][N1]
//   oy   y part of the kinetic term      [8][N2][N0][O1]
//   oz   z part of the kinetic term      [8][O2][N0][N1]
//   gx   after the x up pass             [4][N2][N1][R0]   (channel a2 + 2 a3)
// and of the plane kernels:
//   p1   after the x, y up passes        [2][N2][R1][pad16(R0)]
//   p2   after the z column pass         [2][O2][R1][pad16(R0)]
//   pz   z part of the kinetic term      [8][O2][N1][N0]
// A function that takes the plane kernels in both types has the last three
// only; one that does so in one type has both sets in the same place.
struct SfWork {
  int64_t id;         // the function's index in the plan (SfDev array, outputs)
  int64_t c8, c8x, g1, g2, q, ox, oy, oz, gx;
  int64_t p1, p2, pz;
  int64_t epart;      // offset (in doubles) of its e_pot partials
  int64_t kpart;      // offset (in doubles) of its e_kin partials
  int64_t nkpart;     // number of e_kin partials: its own k_kin_col blocks
  int64_t nepart_pl[2], nkpart_pl;   // partials of the plane kernels (e_pot per type, e_kin)
};

// e_kin partial slots of one function: the blocks of k_kin_col along x, then
// y, then z, counted on the function's own box (so that the summation order
// does not depend on the other functions of the chunk)
// (the z part by k_kin_zmfma when zmfma: one block per 16 columns)
// row stride (elements) of Q[ch][z'][px][y'], the y analysis output: O1
// rounded up to 16, so that the 16-value chunks k_back_y writes (aligned by
// its window phase) are whole 64-byte (FP32) or 128-byte (FP64) pieces
__host__ __device__ inline int qrow_stride(int o1) { return (o1 + 15) & ~15; }
__host__ __device__ inline int kin_blocks(int axis, int n0, int n1, int n2, bool zmfma = false) {
  return axis == 0 ? (4 * n1 * n2 + 255) / 256
         : axis == 1 ? (4 * n0 * n2 + 63) / 64
         : zmfma ? (n0 * n1 + 15) / 16 : (4 * n0 * n1 + 255) / 256;
}

// Plane kernels (wvl_planes.hip).  LDS strides: see k_up_plane.
__host__ __device__ constexpr int pad16(int n) { return (n + 15) & ~15; }
__host__ __device__ constexpr int plane_ldx(int n0) { return ((n0 + 3) & ~7) + 4; }   // 4 (mod 8)
__host__ __device__ constexpr int plane_ych(int n0, int n1) {                          // 16 (mod 32)
  return ((n1 * (pad16(2 * n0 + 29) + 4) + 15) & ~31) + 16;
}
constexpr int kPlaneThreads = 256;   // k_kin_slab, k_up_kin
constexpr int64_t kPlaneLds = 160 * 1024 - 4096;   // dynamic LDS of a block at most
// dynamic LDS in elements of the compute type
constexpr int64_t plane_lds_up(int64_t n0, int64_t n1, bool both, int sz) {
  return sz == 4 ? 4 + 2 * n1 * (2 * n0 + 1) + n1 * (4 * n0 + 59)
                 : (both ? 4 : 2) * n1 * plane_ldx((int)n0) + 2 * (int64_t)plane_ych((int)n0, (int)n1);
}
__host__ __device__ constexpr int plane_kin_elems(int n0, int rows) {   // 4-aligned
  return (4 + rows * (4 * n0 + 1) + 3) & ~3;
}
constexpr int64_t plane_lds_kin(int64_t n0, int64_t n2) { return plane_kin_elems((int)n0, (int)n2); }
__host__ __device__ constexpr int64_t plane_lds_back(int64_t n0, int64_t n1, int64_t e, int64_t rows) {
  const int64_t q = 2 * rows * (pad16((int)(2 * n0 + 29)) + 4), x = plane_kin_elems((int)n0, (int)n1);
  return (q > x ? q : x) + 4 * rows * ((n0 + 2 * e) | 1);
}
// Output rows y' per k_back_plane block: 24; 32 where these are all (a second
// block for the last few rows costs as much as the first: a block's time is the
// latency of its phases), unless that takes the box past the LDS of a CU in a
// type.  300 boxes of 12^3 points: 1.00 -> 0.69 ms in FP32, 1.71 -> 1.20 in FP64;
// 40 of 96 x 10 x 30 in FP32 1.21 -> 0.59.
__host__ __device__ constexpr bool plane_strip_lds(int n0, int n1, int e, int rows, int sz) {
  return sz * plane_lds_back(n0, n1, e, rows) <= kPlaneLds;
}
__host__ __device__ constexpr int plane_strip(int n0, int n1, int e) {
  const int o1 = n1 + 2 * e;
  return o1 > 24 && o1 <= 32 &&
                 (plane_strip_lds(n0, n1, e, 32, 4) || !plane_strip_lds(n0, n1, e, 24, 4)) &&
                 (plane_strip_lds(n0, n1, e, 32, 8) || !plane_strip_lds(n0, n1, e, 24, 8))
             ? 32 : 24;
}
__host__ __device__ constexpr int plane_strips(int n0, int n1, int e) {
  return (n1 + 2 * e + plane_strip(n0, n1, e) - 1) / plane_strip(n0, n1, e);
}
constexpr int64_t plane_lds_back(int64_t n0, int64_t n1, int64_t e) {
  return plane_lds_back(n0, n1, e, plane_strip((int)n0, (int)n1, (int)e));
}
// Whether a function of this box takes the plane kernels in an element type
// of sz bytes: its planes fit the LDS of a CU (160 KiB, less the static
// part).  With ext 8, cubes of up to 49 points per axis do in FP64, of 66 in FP32;
// flatter boxes up to kPlaneMaxN points along any axis.  The rule looks at the function's own box only, so that results
// do not depend on the other functions of a plan.
constexpr int kPlaneMaxN = 96;    // bits of k_back_plane's row masks
constexpr bool plane_fits(int64_t n0, int64_t n1, int64_t n2, int64_t e, int sz) {
  return n0 <= kPlaneMaxN && n1 <= kPlaneMaxN && n2 <= kPlaneMaxN && sz * plane_lds_up(n0, n1, false, sz) <= kPlaneLds &&
         sz * plane_lds_kin(n0, n2) <= kPlaneLds && sz * plane_lds_back(n0, n1, e) <= kPlaneLds;
}

// Whether k_back_plane takes a function with more threads in FP32: where a block's LDS
// leaves room for one block per CU (58 points per axis and more, ext 8).
constexpr int kWideThreads = 1024;
constexpr bool plane_wide(int64_t n0, int64_t n1, int64_t e) {
  return 4 * plane_lds_back(n0, n1, e) > 80 * 1024 - 2048;
}

// per-chunk launch geometry of the fused kernels, for dtype d (0 f32, 1 f64)
struct ChunkDev {
  int32_t sf0, nsf;                // positions [sf0, sf0 + nsf) of the processing order
  int64_t maxbox_in;               // largest dense input box (elements)
  int32_t grid_u[2], group_u[2];   // k_unpack: (8 / group) blocks per input z
  int32_t grid_ux, grid_uy;        // k_up_x, k_up_y
  int64_t lds_u[2];
  int32_t grid_b;                  // k_pot_column
  int32_t grid_kx, grid_ky, grid_kz;   // k_kin_col (x, y, z)
  int32_t grid_by;                 // k_back_y
  int32_t grid_bx;                 // k_back_out
  int32_t nblk_pot, nblk_kin;      // partial slots per function
  // plane kernels, per type (0 f32, 1 f64): whether the chunk's functions take
  // them, dynamic LDS in bytes, both a2 at once in k_up_plane
  bool plane[2];
  bool wide;           // k_back_plane in FP32, see plane_wide
  int32_t strip;       // its rows per block, see plane_strip
  int32_t up_both[2];
  int64_t lds_up[2], lds_ks[2], lds_bp[2];
  int32_t grid_up, grid_ct, grid_ks, grid_bp;
};

// the apply of wvl_apply_local_ham on a workspace of `cap` bytes that the
// caller vouches for (wvl_host.cpp); rejects plans that need more
wvl_status apply_in_workspace(wvl_plan* plan, wvl_dtype dt, uint32_t terms, const void* psi_c,
                              const void* pot, void* hpsi_c, double* e_kin, double* e_pot,
                              void* workspace, size_t cap, const char* who);
// records an error on the plan's context (or the thread's, for a NULL plan)
wvl_status plan_error(wvl_plan* plan, wvl_status st, const char* msg);
// the HIP stream of the plan's context
void* plan_stream(const wvl_plan* plan);

// Loads every kernel's code object on the current device and sets the kernels'
// LDS limits there (hipError_t as int): at plan creation, and before a stream
// capture or anything else that must not load one
int preload_all();             // wvl_host.cpp: all of the following
int preload_kernels();         // wvl_kernels.hip
int preload_fused_kernels();   // wvl_fused.hip
int preload_plane_kernels();   // wvl_planes.hip

// launchers implemented in wvl_kernels.hip; all return hipError_t as int
int launch_gather(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                  const void* psi, void* box, int sf0, int nsf, int64_t maxvol);
int launch_scatter(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                   const void* box, void* out, int sf0, int nsf, int64_t maxvol);
int launch_fill(int f64, void* stream, void* ptr, int64_t n);
int launch_unpack(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                  const RowRun* rr, const void* psi, const SfWork* wk, int nsf, int gridx,
                  int group, size_t lds, void* ws);
int launch_up(int f64, void* stream, int axis, const SfWork* wk, const SfDev* sf, int nsf,
              int gridx, void* ws);
int launch_up_z(int f64, void* stream, const SfWork* wk, const SfDev* sf, int nsf, int gridx,
                const void* ws, const int64_t* fine_off, void* fine, int padded);
// density: tiles of 16 x 4 x 4 fine-grid points (a workgroup each) with the
// functions whose fine box meets them; at most kDensMaxCover functions may
// meet one plane (16 x 4 x 1 points) of a tile
constexpr int kDensTile[3] = {16, 4, 4};
constexpr int kDensMaxCover = 1024;
// a tile and the m functions that meet it, csf[c0 .. c0 + m); in launch order,
// first the nheavy tiles that more than kDensLight functions meet
struct DensTile {
  int32_t tile, m;
  int64_t c0;
};
constexpr int kDensLight = 32;
int launch_dens_tile(int f64, void* stream, const SfDev* sf, const int64_t* foff,
                     const void* fine, const int64_t* krow, const int32_t* kcol,
                     const double* kval, int64_t knnz, const DensTile* tiles, const int32_t* csf,
                     int64_t nheavy, int nsf, const int* gf, void* rho);
int launch_pot_column(int f64, void* stream, const SfDev* sf, const SfWork* wk, int sf0, int nsf,
                      int gridx, void* ws, const void* pot, int nf1, int nf2, double* epart,
                      const double* conf, double hh, int padded);
// the z part of the kinetic term on the FP64 matrix cores (banded Toeplitz)
int launch_kin_zmfma(int f64, void* stream, const SfDev* sf, const SfWork* wk, int sf0, int nsf,
                     int gridx, void* ws, double fac, double* kpart);
int launch_kin_col(int f64, void* stream, int axis, const SfDev* sf, const SfWork* wk, int sf0,
                   int nsf, int gridx, void* ws, double fac, double* kpart);
int launch_back_y(int f64, void* stream, const SfDev* sf, const SfWork* wk, int sf0, int nsf,
                  int gridx, void* ws);
int launch_back_out(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                    const RowRun* rr, const SfWork* wk, int sf0, int nsf, int gridx,
                    const void* ws, void* out, int pot_on, int kin_on, int accumulate);
// plane kernels (wvl_planes.hip)
int launch_up_plane(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                    const RowRun* rr, const void* psi, const SfWork* wk, int nsf, int gridx,
                    int both, size_t lds, void* ws);
// FP64: z passes on the matrix cores (FP32 takes k_pot_column, k_up_z)
int launch_col_tile(void* stream, const SfDev* sf, const SfWork* wk, int nsf, int gridx, void* ws,
                    const void* pot, int nf1, int nf2, double* epart, const double* conf,
                    double hh);
int launch_syn_tile(void* stream, const SfDev* sf, const SfWork* wk, int nsf, int gridx, void* ws,
                    const int64_t* fine_off, void* fine);
// both in one launch (lds: the larger of the two)
int launch_up_kin(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                  const RowRun* rr, const void* psi, const SfWork* wk, int nsf, int nup, int nkin,
                  int both, size_t lds, void* ws, double fac, double* kpart);
int launch_kin_slab(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                    const RowRun* rr, const void* psi, const SfWork* wk, int nsf, int gridx,
                    size_t lds, void* ws, double fac, double* kpart);
int launch_back_plane(int f64, void* stream, const SfDev* sf, const wvl_seg* seg,
                      const int32_t* rt, const RowRun* rr, const void* psi, const SfWork* wk,
                      int nsf, int gridx, int wide, int strip, size_t lds, const void* ws, void* out,
                      int pot_on, int kin_on, int accumulate, double fac, double* kpart);
int launch_plane_energies(int f64, void* stream, const SfWork* wk, int nsf, const double* parts,
                          double* e_kin, double* e_pot);
int launch_finalize(void* stream, const SfWork* wk, int sf0, int nsf, const double* parts,
                    int which, int nblk, double* out);
int launch_pattern(void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt, int nsf,
                   int ket_out, int64_t* count, const int64_t* rowptr, int32_t* col);
// Fermi operator expansion on a symmetric CSR pattern (row: row of each
// entry, tpos: position of the transposed entry).  foe_mm: one workgroup per
// row, 8 waves when no row has more than kFoeMaxDeg / 2 entries, else 4
// (and two rows of B a step when none has more than kFoeMaxDeg / 4);
// rows of at most kFoeMaxDeg entries, columns below kFoeMaxCol, entries
// addressed with 32-bit offsets; 2^lognb hash buckets of 16 bytes, at least
// as many as the longest row has entries (maxdeg) and at least 32 (at most
// 64 KiB of LDS in all).
constexpr int kFoeMaxDeg = 1024;
constexpr int kFoeMaxCol = 1 << 21;
int launch_foe_mm(void* stream, int nrow, const int32_t* rows, const int64_t* rowptr,
                  const int32_t* col, double alpha, const double* A, const double* B, double beta,
                  const double* D, double* C, int lognb, int maxdeg);
// C = alpha (R A)|_P + beta D (with tpos: stored transposed), A symmetric, from
// rows spread out in LDS: where the functions plus the longest row's entries
// number at most kFoeSpread (64 KiB of LDS; beyond it the launch is refused)
constexpr int kFoeSpread = 8192;
int launch_foe_rmul(void* stream, int nrow, const int32_t* rows, const int64_t* rowptr,
                    const int32_t* col, double alpha, const double* R, const double* A, double beta,
                    const double* D, const int64_t* tpos, double* C, int maxdeg);
int launch_foe_axpby(void* stream, int64_t nnz, double a, const double* X, double b,
                     const double* Y, const int32_t* row, const int32_t* col, double d,
                     double* out);
int launch_foe_sym(void* stream, int64_t nnz, const int64_t* tpos, const double* X, double* out);
int launch_foe_gather(void* stream, int64_t nnz, const int64_t* qpos, const double* X,
                      double* out);
// dot: part needs min(256, ceil(nnz / 2048)) doubles (at most nnz)
int launch_foe_dot(void* stream, int64_t nnz, const double* X, const double* Y, double* part,
                   double* out, int slot);
int launch_foe_trace(void* stream, int n, const int64_t* dpos, const double* X, int64_t stride,
                     int count, double* out, int slot);
int launch_foe_series(void* stream, int64_t nnz, int npl, const double* c, const double* T,
                      const int32_t* row, const int32_t* col, double* out);
// Gershgorin bounds: lo, hi hold nrow doubles each
int launch_foe_gersh(void* stream, int nrow, const int64_t* rowptr, const int32_t* col,
                     const double* X, double* lo, double* hi, double* out);
int launch_update(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                  double eta, const void* hpsi, const int64_t* hrow, const int32_t* hcol,
                  const double* hval, void* psi, int sf0, int nsf, int64_t maxsegs, int mode,
                  const double* shift, void* out);
// g_a = L^a [sum_d A_ad H phi_d - M_ad phi_d] over the rows of a CSR pattern
// (A and M in its order), one block per function a of [sf0, sf0 + nsf)
int launch_grad_rows(int f64, void* stream, const SfDev* sf, const wvl_seg* seg,
                     const int32_t* rt, const RowRun* rr, const int64_t* rowptr,
                     const int32_t* col, const double* av, const double* mv, const void* psi,
                     const void* hpsi, int sf0, int nsf, void* g);
int launch_sf_dot(int f64, void* stream, const SfDev* sf, const void* a, const void* b,
                  double* out, int sf0, int nsf);
int launch_cg_init(int f64, void* stream, const SfDev* sf, const void* g, void* x, void* r,
                   void* p, int sf0, int nsf);
int launch_cg_xr(int f64, void* stream, const SfDev* sf, const double* rr, const double* pap,
                 const void* p, const void* ap, void* x, void* r, int sf0, int nsf);
int launch_cg_p(int f64, void* stream, const SfDev* sf, double* rr, const double* rr_new,
                const void* r, void* p, int sf0, int nsf);
int launch_sparse_values(int f64, void* stream, const SfDev* sf, const wvl_seg* seg,
                         const int32_t* rt, const RowRun* rr, int ket_out, const void* bra,
                         const void* ket, const int32_t* row, const int32_t* col,
                         const int32_t* order, const int32_t* mirror, int64_t nnz, int64_t rows,
                         double* val);   // rows: mean rows of an input box (see the launch)

}  // namespace wvl
