// Plane kernels of the local Hamiltonian for gfx950 (MI355X): the apply of
// every function whose planes fit a CU's LDS (plane_fits; the column kernels
// of wvl_fused.hip take the others).
//
//   k_up_plane    (z, a3): uncompress one coarse plane into LDS, x up pass
//                 and y up pass -> G1 (FP32: k_up_plane_valu)
//   k_col_tile    FP64: 16 fine columns per wave, streaming along z: z up pass,
//                 times the potential, z down pass -> G2 (or, for the synthesis
//                 to real space, the fine values themselves); FP32 runs
//                 k_pot_column and k_up_z of wvl_fused.hip here
//   k_kin_slab    (y, a2): uncompress one x-z slab, z part of the kinetic
//                 term -> OZ
//   k_back_plane  (z', a3, 24 or 32 rows y'): y and x down passes, x and y parts of
//                 the kinetic term from the uncompressed plane, OZ, and the
//                 compression onto the output pattern, in LDS
//
// Against the column kernels a step writes and reads three arrays (G1, G2, OZ)
// instead of nine: 16 instead of 38 GB of traffic for 1,000 functions of radius
// 5-7 bohr in FP32 (13.0 -> 8.1 ms; FP64 25.3 -> 15.0 ms), and one launch of a
// single function waits for four short kernels instead of nine serial chains
// (FP64 442 -> 53 us).
//
// The down passes, and in FP64 the up passes, are products with banded Toeplitz
// matrices and run on the matrix cores (16x16x4): an output tile is 16 fine
// points (up) or 8 coarse points x 2 channels (down) of 16 rows, from a window
// of 48 inputs, 12 instructions of k = 4.  Every tile has the same 12 band
// operands (one register each), and neighbouring tiles share 8 of their 12 data
// operands, so a wave streams along the axis with four new operands per tile.
// 31 of 48 inputs per output carry a tap; the padding is paid on units that are
// otherwise idle (FP32: at twice the vector rate), with a twelfth of the
// instructions and a third of the registers of the vector form, and the vector
// units are left to the kinetic term of other waves.
//
// The FP32 up passes stay on the vector units: the column kernels round once
// more per tap pair than a multiply-add chain, the potential energies (double)
// show the difference at 1e-8, and both precisions keep the values they had.
// The kinetic term stays there too: its scaling channel is summed in double in
// both types, and FP64 runs at one rate on both units, without the band's
// padding on the vector unit.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "wvl_filters.h"
#include "wvl_internal.h"

namespace wvl {

namespace {

// kinetic taps as compile-time constants: they become scalar moves and
// literals, no memory is read for them
constexpr double kK64[2][2][29] = {{WVL_K00_F64, WVL_K01_F64}, {WVL_K10_F64, WVL_K11_F64}};
constexpr float kK32[2][2][29] = {{WVL_K00_F32, WVL_K01_F32}, {WVL_K10_F32, WVL_K11_F32}};

// 16x16x4 matrix instruction: lane l = 16 g + n supplies A[n][g] and B[g][n]
// and holds D[row(r, g)][n] in element r
template <typename T> struct Mma;
template <> struct Mma<float> {
  typedef float V __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ V mma(float a, float b, V c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int g) { return 4 * g + r; }
};
template <> struct Mma<double> {
  typedef double V __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ V mma(double a, double b, V c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int g) { return g + 4 * r; }
};

// Band operands, operand k of lane 16 g + n at v[kind][k][lane].
//   kUp, kUpPair: an up tile, fine points p0 + m, m = 0..15 (m = n), from coarse
//     points q = p0 / 2 - 16 + 4 ks + dq, ks = 0..5, of both channels a;
//     f_p = sum C_a[p - 2q] x_a(q).  Operand 2 ks + c holds in slot g
//     kUp: a = c, dq = g;  kUpPair: a = g & 1, dq = 2 c + (g >> 1).
//   kDown, kDownReg: a down tile, outputs m = 8 a + i (channel a, coarse point
//     i0 + i, i = 0..7; m = n) from fine points p = 2 i0 + 16 b + pk, b = 0..2.
//     Operand 4 b + r holds in slot g the point pk = 4 r + g (kDown) or the
//     one that element r of an up tile's result holds there (kDownReg), so
//     that such results are operands as they stand.
// An instruction adds its four products one after the other, slot 0 first, each
// with one rounding (checked on the device against fma chains).  With kDown's
// order the taps of an output therefore add up in ascending order, which in
// FP32 gives the bits of the column kernels' multiply-add chains (the operands
// outside the band are zeros and change nothing).
enum { kUp, kUpPair, kDown, kDownReg };
template <typename T> struct Bands {
  T v[4][12][64];
};
template <typename T> constexpr Bands<T> make_bands() {
  constexpr double c64[2][31] = {WVL_C0_F64, WVL_C1_F64};
  constexpr float c32[2][31] = {WVL_C0_F32, WVL_C1_F32};
  Bands<T> b{};
  for (int kind = 0; kind < 4; ++kind)
    for (int k = 0; k < 12; ++k)
      for (int l = 0; l < 64; ++l) {
        const int n = l & 15, g = l >> 4;
        int ch = 0, t = 0;
        if (kind == kUp || kind == kUpPair) {
          const int ks = k >> 1, c = k & 1;
          ch = kind == kUp ? c : g & 1;
          t = n + 32 - 8 * ks - 2 * (kind == kUp ? g : 2 * c + (g >> 1));
        } else {
          const int r = k & 3;
          const int pk = kind == kDown || sizeof(T) == 8 ? 4 * r + g : 4 * g + r;
          ch = n >> 3;
          t = 16 * (k >> 2) + pk - 2 * (n & 7);
        }
        b.v[kind][k][l] = t < 0 || t > 30 ? T(0) : sizeof(T) == 8 ? (T)c64[ch][t] : (T)c32[ch][t];
      }
  return b;
}
__device__ const Bands<float> gBands32 = make_bands<float>();
__device__ const Bands<double> gBands64 = make_bands<double>();
template <typename T>
__device__ __forceinline__ void load_band(T (&A)[12], int kind, int lane) {
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    if constexpr (sizeof(T) == 8)
      A[k] = gBands64.v[kind][k][lane];
    else
      A[k] = gBands32.v[kind][k][lane];
  }
}

// The products give every output the whole window, with zeros for the points
// that none of its taps meets, and zero times an infinity is NaN.  An output
// must not depend on such points: a wave whose products hold a value that is
// not finite (one value per lane and tile tells, since every point of a window
// enters every output of its row) runs its tiles once more with the outputs
// formed from the taps alone (operands B[at], B[at + 1], ..), in the order of
// the instructions.  The second run is code of its own (`again`), so that the
// first pays for a comparison per tile only.
template <typename T> __device__ __forceinline__ bool not_finite(T v) {
  return !__builtin_isfinite(v);
}
template <typename T, int NB>
__device__ __forceinline__ typename Mma<T>::V taps_only(const T (&B)[NB], int at, int kind,
                                                        int lane) {
  asm volatile("" : "+v"(lane));   // keeps what follows out of the loops around it
  const int n = lane & 15, g = lane >> 4;
  typename Mma<T>::V s = {T(0), T(0), T(0), T(0)};
#pragma unroll
  for (int k = 0; k < 12; ++k) {
#pragma unroll 1
    for (int h = 0; h < 4; ++h) {
      const T x = __shfl(B[at + k], 16 * h + n, 64);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        T c;
        if constexpr (sizeof(T) == 8)
          c = gBands64.v[kind][k][16 * h + Mma<T>::row(r, g)];
        else
          c = gBands32.v[kind][k][16 * h + Mma<T>::row(r, g)];
        if (c != T(0)) s[r] = __builtin_fma(c, x, s[r]);
      }
    }
  }
  return s;
}

// A buffer in global memory: loads beyond its bytes (negative offsets among
// them, which are large as unsigned) give 0, stores there are dropped.
// Offsets are in elements.
constexpr uint32_t kNone = 0xC0000000u;   // a byte offset beyond every buffer here
template <typename T> struct Buf {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ Buf(const T* p, int64_t n)
      : r(__builtin_amdgcn_make_buffer_rsrc((void*)p, 0,
                                            (int)(uint32_t)min(n * (int64_t)sizeof(T), (int64_t)0xBFFFFFF0),
                                            0x00020000)) {}
  __device__ __forceinline__ T at(uint32_t byte) const {
    if constexpr (sizeof(T) == 8) {
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, byte, 0, 0));
    } else {
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, byte, 0, 0));
    }
  }
  __device__ __forceinline__ T operator[](int i) const { return at((uint32_t)i * (uint32_t)sizeof(T)); }
  __device__ __forceinline__ void put(uint32_t byte, T v) const {
    if constexpr (sizeof(T) == 8) {
      typedef uint32_t U2 __attribute__((ext_vector_type(2)));
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), r, byte, 0, 0);
    } else {
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, byte, 0, 0);
    }
  }
};

// fixed-order sum over the block (valid in thread 0)
__device__ double plane_block_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __shared__ double part[16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) part[wv] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) r += part[k];
  return r;
}

// Uncompresses nrows rows of the input box: put(row j, x, v) gets the NC
// components cb + (k & 1) + cs (k >> 1) of every point; row j is box row
// r0 + j rstep.  Half a wave takes a row, four rows at a time: their run
// records are loaded together, then their values, so that a block waits for
// two load latencies per 4 x (block / 32) rows.  Rows of several runs walk
// their segments.
template <typename T, int NC, typename Put>
__device__ __forceinline__ void load_rows(int nrows, int cb, int cs, const SfDev& sf,
                                          const wvl_seg* __restrict__ seg,
                                          const int32_t* __restrict__ rt,
                                          const RowRun* __restrict__ rr,
                                          const T* __restrict__ psi, int r0, int rstep, Put put) {
  constexpr int U = 4;
  constexpr uint32_t SZ = sizeof(T);
  const int N0 = sf.n[0], lo = sf.lo[0];
  const int hw = blockDim.x >> 5, l = threadIdx.x & 31;
  const Buf<T> pc(psi + sf.cin, sf.n_c), pf(psi + sf.cin + sf.n_c, 7 * sf.n_f);
  const RowRun* const rrc = rr + sf.rr[0];
  const RowRun* const rrf = rr + sf.rr[1];
  for (int j0 = threadIdx.x >> 5; j0 < nrows; j0 += U * hw) {
    RowRun rc[U], rf[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t r = (uint32_t)(r0 + min(j0 + u * hw, nrows - 1) * rstep);
      rc[u] = RowRun{0, 0, 0};
      if (cb == 0) rc[u] = rrc[r];
      rf[u] = rrf[r];
    }
    for (int xb = 0; xb < N0; xb += 32) {
      const int x = xb + l, gx = lo + x;
      T v[U][NC];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int df = gx - (int)rf[u].x0, dc = gx - (int)rc[u].x0;
        const bool inf = rf[u].len != kMultiRun && (uint32_t)df < (uint32_t)rf[u].len;
        const bool inc = rc[u].len != kMultiRun && (uint32_t)dc < (uint32_t)rc[u].len;
        const uint32_t of = inf ? 7 * SZ * (uint32_t)(rf[u].off + df) : kNone;
        const uint32_t oc = inc ? SZ * (uint32_t)(rc[u].off + dc) : kNone;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
          const int c = cb + (k & 1) + cs * (k >> 1);
          v[u][k] = c == 0 ? pc.at(oc) : pf.at(of + SZ * (uint32_t)(c - 1));
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + u * hw;
        if (j >= nrows || x >= N0) continue;
        const int r = r0 + j * rstep;
        if (rf[u].len == kMultiRun)
          for (int q = rt[sf.rt[1] + r], q1 = rt[sf.rt[1] + r + 1]; q < q1; ++q) {
            const wvl_seg s = seg[q];
            if (gx < s.i1s || gx > s.i1e) continue;
#pragma unroll
            for (int k = 0; k < NC; ++k) {
              const int c = cb + (k & 1) + cs * (k >> 1);
              if (c > 0) v[u][k] = pf[7 * (int)(s.off + (gx - s.i1s)) + (c - 1)];
            }
          }
        if (rc[u].len == kMultiRun)
          for (int q = rt[sf.rt[0] + r], q1 = rt[sf.rt[0] + r + 1]; q < q1; ++q) {
            const wvl_seg s = seg[q];
            if (gx >= s.i1s && gx <= s.i1e) v[u][0] = pc[(int)(s.off + (gx - s.i1s))];
          }
        put(j, x, v[u]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// k_up_plane: block = (function, z, a3)
// ---------------------------------------------------------------------------
// X[a1][y][x] of the plane (both a2 at once, or one after the other when
// `both` is 0: the LDS of the larger planes) -> Y[a2][y][px] -> G1[a3][z][py][px]
// (rows pad16(R0) apart; the columns past R0 hold zeros).
// LDS strides: rows of X 4 (mod 8) apart and rows of Y 4 (mod 16) put the 16
// rows x 4 points of an operand on distinct banks; the channels of Y are
// 16 (mod 32) apart, so that the two channels of a y operand are too.
__device__ __forceinline__ void up_plane(int bx, const SfDev* __restrict__ sfs,
                                         const wvl_seg* __restrict__ seg,
                                         const int32_t* __restrict__ rt,
                                         const RowRun* __restrict__ rr,
                                         const double* __restrict__ psi,
                                         const SfWork* __restrict__ wk, double* __restrict__ ws,
                                         int both) {
  using T = double;
  extern __shared__ __align__(32) unsigned char smem_raw[];
  const SfWork& w = wk[blockIdx.y];
  const SfDev& sf = sfs[w.id];
  const int N0 = sf.n[0], N1 = sf.n[1], N2 = sf.n[2];
  const int z = bx >> 1, a3 = bx & 1;
  if (z >= N2) return;   // uniform over the block
  const int R1 = 2 * N1 + 29, P0 = pad16(2 * N0 + 29);
  const int ldx = plane_ldx(N0), ldy = P0 + 4, ych = plane_ych(N0, N1);
  T* X = reinterpret_cast<T*>(smem_raw);
  T* Y = X + (both ? 4 : 2) * N1 * ldx;
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  typedef typename Mma<T>::V V;
  const int nx = P0 >> 4;
  constexpr int NW = 4;
  {
    T A[12];
    load_band(A, kUp, lane);
    constexpr int NSP = NW / 2;   // px ranges a row tile is split into
    const int nrt = (N1 + 15) >> 4, len = (nx + NSP - 1) / NSP;
    for (int a2 = 0; a2 < 2; ++a2) {
      if (both) {
        if (a2 == 0)
          load_rows<T, 4>(N1, 4 * a3, 2, sf, seg, rt, rr, psi, z * N1, 1,
                          [&](int j, int x, const T* v) {
#pragma unroll
                            for (int k = 0; k < 4; ++k) X[(k * N1 + j) * ldx + x] = v[k];
                          });
      } else {
        load_rows<T, 2>(N1, 4 * a3 + 2 * a2, 2, sf, seg, rt, rr, psi, z * N1, 1,
                        [&](int j, int x, const T* v) {
#pragma unroll
                          for (int k = 0; k < 2; ++k) X[(k * N1 + j) * ldx + x] = v[k];
                        });
      }
      if (a2 == 0 || !both) __syncthreads();
      const T* const Xa = X + (both ? 2 * a2 * N1 * ldx : 0);
      auto pass = [&](auto again_) {
        constexpr bool again = decltype(again_)::value;
        bool bad = false;
        for (int job = wave; job < NSP * nrt; job += NW) {
          const int y = (job / NSP) * 16 + n;
          const T* const x0 = Xa + min(y, N1 - 1) * ldx;   // rows past N1: not stored
          const T* const x1 = x0 + N1 * ldx;
          T* const yo = Y + a2 * ych + y * ldy;
          const int t0 = (job % NSP) * len, t1 = min(nx, t0 + len);
          T B[12];
          auto fetch = [&](int ks, int t, int slot) {   // points 8 t - 16 + 4 ks + g
            const int q0 = 8 * t - 16 + 4 * ks, q = q0 + g;
            if (q0 >= 0 && q0 + 3 < N0) {
              B[2 * slot] = x0[q];
              B[2 * slot + 1] = x1[q];
            } else {
              const bool ok = q >= 0 && q < N0;
              const int k = ok ? q : 0;
              const T v0 = x0[k], v1 = x1[k];
              B[2 * slot] = ok ? v0 : T(0);
              B[2 * slot + 1] = ok ? v1 : T(0);
            }
          };
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) fetch(ks, t0, ks + 2);
          for (int t = t0; t < t1; ++t) {
#pragma unroll
            for (int k = 0; k < 8; ++k) B[k] = B[k + 4];
            fetch(4, t, 4);
            fetch(5, t, 5);
            V d = {T(0), T(0), T(0), T(0)};
#pragma unroll
            for (int ks = 0; !again && ks < 6; ++ks) {
              const int q = 8 * t - 16 + 4 * ks;
              if (q + 3 < 0 || q >= N0) continue;   // no input there
              d = Mma<T>::mma(A[2 * ks], B[2 * ks], d);
              d = Mma<T>::mma(A[2 * ks + 1], B[2 * ks + 1], d);
            }
            if (again) d = taps_only<T>(B, 0, kUp, lane);
            bad |= not_finite(d[0]);
            if (y < N1) {
#pragma unroll
              for (int r = 0; r < 4; ++r) yo[16 * t + Mma<T>::row(r, g)] = d[r];
            }
          }
        }
        return __any(bad) != 0;
      };
      if (__builtin_expect(pass(std::false_type{}), 0)) pass(std::true_type{});
      __syncthreads();
    }
  }
  // y pass: tiles (px tile, third of the py tiles)
  T A[12];
  load_band(A, kUpPair, lane);
  const int ny = (R1 + 15) >> 4, nch = (ny + 2) / 3;
  const Buf<T> o0(ws + w.p1 + ((int64_t)a3 * N2 + z) * ((int64_t)R1 * P0), R1 * P0);
  auto pass = [&](auto again_) {
    constexpr bool again = decltype(again_)::value;
    bool bad = false;
    for (int job = wave; job < nx * nch; job += NW) {
      const int tx = job % nx, t0 = 3 * (job / nx), t1 = min(ny, t0 + 3);
      const T* const yb = Y + (g & 1) * ych + 16 * tx + n;
      T B[12];
      auto fetch = [&](int ks, int t, int slot) {
        const int q0 = 8 * t - 16 + 4 * ks;
        if (q0 >= 0 && q0 + 3 < N1) {
          const T* const y = yb + (q0 + (g >> 1)) * ldy;
          B[2 * slot] = y[0];
          B[2 * slot + 1] = y[2 * ldy];
          return;
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int q = q0 + 2 * c + (g >> 1);
          const bool ok = q >= 0 && q < N1;
          const T v = yb[(ok ? q : 0) * ldy];
          B[2 * slot + c] = ok ? v : T(0);
        }
      };
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) fetch(ks, t0, ks + 2);
      for (int t = t0; t < t1; ++t) {
#pragma unroll
        for (int k = 0; k < 8; ++k) B[k] = B[k + 4];
        fetch(4, t, 4);
        fetch(5, t, 5);
        V d = {T(0), T(0), T(0), T(0)};
#pragma unroll
        for (int ks = 0; !again && ks < 6; ++ks) {
          const int q = 8 * t - 16 + 4 * ks;
          if (q + 3 < 0 || q >= N1) continue;
          d = Mma<T>::mma(A[2 * ks], B[2 * ks], d);
          d = Mma<T>::mma(A[2 * ks + 1], B[2 * ks + 1], d);
        }
        if (again) d = taps_only<T>(B, 0, kUpPair, lane);
        bad |= not_finite(d[0]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int py = 16 * t + Mma<T>::row(r, g);   // rows past R1: dropped
          o0.put((uint32_t)(py * P0 + 16 * tx + n) * (uint32_t)sizeof(T), d[r]);
        }
      }
    }
    return __any(bad) != 0;
  };
  if (__builtin_expect(pass(std::false_type{}), 0)) pass(std::true_type{});
}

// ---------------------------------------------------------------------------
// k_up_plane_valu: block = (function, z, a3), FP32
// ---------------------------------------------------------------------------
// The same passes on the vector units, each output as the column kernels add
// it (per tap pair one product, one multiply-add, one add), so that the values
// on the fine grid, and the potential energies made from them in double, keep
// their bits.  X[y][a2][x][a1] -> Y[y][px][a2] -> G1[a3][z][py][px].  An
// item is 8 coarse steps (16 outputs) of one row or column: 23 inputs of each
// channel in registers; items are dealt to lanes without gaps, rows and columns
// fastest.  Odd row strides of X and Y keep lanes along the rows off each
// other's banks.
struct UpTaps {
  float c[2][31];
};
constexpr UpTaps up_taps() {
  constexpr float c32[2][31] = {WVL_C0_F32, WVL_C1_F32};
  UpTaps t{};
  for (int b = 0; b < 2; ++b)
    for (int k = 0; k < 31; ++k) t.c[b][k] = c32[b][k];
  return t;
}
// coarse steps q0 .. q0 + 7 of a column S[lx + q st + b], 0 <= q < N (S[0]
// and S[1] hold zeros): fe[u], fo[u] at the fine points 2 (q0 + u), + 1
__device__ __forceinline__ void up_item(const float* S, int lx, int st, int q0, int N,
                                        float (&fe)[8], float (&fo)[8]) {
  constexpr UpTaps C = up_taps();
  float xs[23], xd[23];
#pragma unroll
  for (int k = 0; k < 23; ++k) {
    const int q = q0 - 15 + k;
    const int a = (uint32_t)q < (uint32_t)N ? lx + q * st : 0;
    xs[k] = S[a];
    xd[k] = S[a + 1];
  }
#pragma unroll
  for (int u = 0; u < 8; ++u) fe[u] = fo[u] = 0.f;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    // inputs q0 - k .. q0 - k + 7: nothing to add when all are zeros
    if (!__any(q0 - k + 7 >= 0 && q0 - k < N)) continue;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float a = xs[15 + u - k], b = xd[15 + u - k];
      fe[u] += __builtin_fmaf(C.c[0][2 * k], a, C.c[1][2 * k] * b);
      if (k < 15) fo[u] += __builtin_fmaf(C.c[0][2 * k + 1], a, C.c[1][2 * k + 1] * b);
    }
  }
}

__device__ __forceinline__ void up_plane(int bx, const SfDev* __restrict__ sfs,
                                         const wvl_seg* __restrict__ seg,
                                         const int32_t* __restrict__ rt,
                                         const RowRun* __restrict__ rr,
                                         const float* __restrict__ psi,
                                         const SfWork* __restrict__ wk, float* __restrict__ ws, int) {
  extern __shared__ __align__(32) unsigned char smem_raw[];
  const SfWork& w = wk[blockIdx.y];
  const SfDev& sf = sfs[w.id];
  const int N0 = sf.n[0], N1 = sf.n[1], N2 = sf.n[2];
  const int z = bx >> 1, a3 = bx & 1;
  if (z >= N2) return;   // uniform over the block
  const int R0 = 2 * N0 + 29, R1 = 2 * N1 + 29, P0 = pad16(R0);
  const int ldx = 2 * N0 + 1, ldy = 2 * R0 + 1;
  float* const X = reinterpret_cast<float*>(smem_raw);   // two zeros, then the rows
  float* const Y = X + 2 + 2 * N1 * ldx;                  // likewise
  const int tid = threadIdx.x;
  if (tid < 2) X[tid] = Y[tid] = 0.f;
  load_rows<float, 4>(N1, 4 * a3, 2, sf, seg, rt, rr, psi, z * N1, 1,
                      [&](int j, int x, const float* v) {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                          X[2 + (2 * j + (k >> 1)) * ldx + 2 * x + (k & 1)] = v[k];
                      });
  __syncthreads();
  const int nq0 = (R0 + 15) >> 4, nrow = 2 * N1;
  for (int it = tid & ~63; it < nrow * nq0; it += 256) {
    const int i = min(it + (tid & 63), nrow * nq0 - 1);   // the last lanes repeat the last item
    const int sg = i / nrow, row = i - sg * nrow;
    float fe[8], fo[8];
    up_item(X, 2 + row * ldx, 2, 8 * sg, N0, fe, fo);
    float* const o = Y + 2 + (row >> 1) * ldy + (row & 1) + 32 * sg;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (16 * sg + 2 * u < R0) o[4 * u] = fe[u];
      if (16 * sg + 2 * u + 1 < R0) o[4 * u + 2] = fo[u];
    }
  }
  __syncthreads();
  const int nq1 = (R1 + 15) >> 4;
  const Buf<float> o0(ws + w.p1 + ((int64_t)a3 * N2 + z) * ((int64_t)R1 * P0), R1 * P0);
  for (int it = tid & ~63; it < R0 * nq1; it += 256) {
    const int i = min(it + (tid & 63), R0 * nq1 - 1);
    const int sg = i / R0, px = i - sg * R0;
    float fe[8], fo[8];
    up_item(Y, 2 + 2 * px, ldy, 8 * sg, N1, fe, fo);
    uint32_t o = (uint32_t)(16 * sg * P0 + px) * 4u;
#pragma unroll
    for (int u = 0; u < 8; ++u) {   // rows past R1: dropped
      o0.put(o, fe[u]);
      o0.put(o + (uint32_t)P0 * 4u, fo[u]);
      o += (uint32_t)P0 * 8u;
    }
  }
}

// ---------------------------------------------------------------------------
// k_col_tile: wave = 16 fine columns (py, 16 px) of one function
// ---------------------------------------------------------------------------
// Tiles of 16 fine points p = 16 u - 2 sh .. along z (sh = ext, so that three
// tiles make the window of 8 outputs; 0 for SYN): z up pass from G1, and
//   SYN = false: times V + confinement (energy in double), z down pass -> G2
//   SYN = true:  the fine values themselves -> FINE
// The down pass takes the up pass' result registers as operands.
template <bool SYN>
__global__ __launch_bounds__(256) void k_col_tile(const SfDev* __restrict__ sfs,
                                                  const SfWork* __restrict__ wk,
                                                  double* __restrict__ ws, const double* __restrict__ pot,
                                                  int nf1, int nf2, double* __restrict__ epart,
                                                  const double* __restrict__ conf, double hh,
                                                  const int64_t* __restrict__ fine_off,
                                                  double* __restrict__ fine) {
  using T = double;
  const SfWork& w = wk[blockIdx.y];
  const SfDev& sf = sfs[w.id];
  const int N0 = sf.n[0], N1 = sf.n[1], N2 = sf.n[2], e = sf.ext;
  const int R0 = 2 * N0 + 29, R1 = 2 * N1 + 29, R2 = 2 * N2 + 29, P0 = pad16(R0);
  const int O2 = N2 + 2 * e;
  const int nx = P0 >> 4;
  const int items = nx * R1;
  if ((int)blockIdx.x * 4 >= items) return;   // uniform over the block
  const int lane = threadIdx.x & 63, n = lane & 15, g = lane >> 4;
  const int item = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  typedef typename Mma<T>::V V;
  constexpr uint32_t SZ = sizeof(T);
  double eacc = 0.0;
  if (item < items) {
    const int py = item / nx, px = 16 * (item - py * nx) + n;
    const int plane = R1 * P0, col = py * P0 + px;
    const Buf<T> in0(ws + w.p1, (int64_t)N2 * plane), in1(ws + w.p1 + (int64_t)N2 * plane,
                                                          (int64_t)N2 * plane);
    const bool pin = px < R0;
    const int sh = SYN ? 0 : e;
    // the lane's potential values of a tile: rows row(r, g), r = 0..3
    constexpr int kRow = 4;   // row(r + 1, g) - row(r, g)
    const int64_t vstride = (int64_t)nf1 * nf2;
    const bool von = !SYN && pot != nullptr;
    const T* const vcol = von ? pot + ((int64_t)(2 * sf.lo[2] - 2 * sh + Mma<T>::row(0, g)) * nf2 +
                                     (2 * sf.lo[1] + py)) * nf1 + (2 * sf.lo[0] + (pin ? px : 0))
                              : nullptr;
    const double ca = (!SYN && conf) ? conf[w.id] : 0.0;
    const double cdx = (double)(2 * sf.lo[0] + px - 14) * hh - sf.c[0];
    const double cdy = (double)(2 * sf.lo[1] + py - 14) * hh - sf.c[1];
    const double cxy = cdx * cdx + cdy * cdy;
    const double cz0 = (double)(2 * sf.lo[2] - 14) * hh - sf.c[2];
    T Au[12], Ad[12], B[12], G[12];
    load_band(Au, kUp, lane);
    if constexpr (!SYN) load_band(Ad, kDownReg, lane);
    // points q = 8 u - sh - 16 + 4 ks + g; 0 outside [0, N2)
    uint32_t inb;
    const uint32_t kstep = 4u * (uint32_t)plane * SZ;
    auto fetch = [&](int slot) {
      B[2 * slot] = in0.at(inb);
      B[2 * slot + 1] = in1.at(inb);
      inb += kstep;
    };
    const int nu = SYN ? (R2 + 15) >> 4 : ((O2 + 7) >> 3) + 2;
    const int fplane = R1 * R0;
    const Buf<T> out(SYN ? fine + fine_off[w.id] : ws + w.p2,
                     SYN ? (int64_t)fplane * R2 : 2ll * O2 * plane);
    auto pass = [&](auto again_) {
      constexpr bool again = decltype(again_)::value;
      bool bad = false;
      eacc = 0.0;
      const T* vq = vcol;
      inb = (uint32_t)((g - sh - 16) * plane + col) * SZ;   // of ks = 0, u = 0
      // of this lane's element 0
      uint32_t ob = SYN ? (uint32_t)(g * fplane + py * R0 + px) * SZ : (uint32_t)(g * plane + col) * SZ;
#pragma unroll
      for (int k = 0; k < 12; ++k) B[k] = G[k] = T(0);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) fetch(ks + 2);
      for (int u = 0; u < nu; ++u) {
        const int p0 = 16 * u - 2 * sh;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          B[k] = B[k + 4];
          G[k] = G[k + 4];
        }
        fetch(4);
        fetch(5);
        V d = {T(0), T(0), T(0), T(0)};
        if (p0 + 15 >= 0 && p0 < R2) {
          T v[4];
          if constexpr (!SYN) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int p = p0 + Mma<T>::row(r, g);
              T x = T(0);
              if (von && ((p0 >= 0 && p0 + 15 < R2) || (p >= 0 && p < R2)))
                x = vq[(int64_t)(r * kRow) * vstride];
              v[r] = pin ? x : T(0);
            }
            if (ca != 0.0) {
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const int p = p0 + Mma<T>::row(r, g);
                const double dz = cz0 + (double)p * hh, r2 = cxy + dz * dz;
                if (pin && p >= 0 && p < R2) v[r] = (T)((double)v[r] + ca * r2 * r2);
              }
            }
          }
#pragma unroll
          for (int ks = 0; !again && ks < 6; ++ks) {
            const int q = 8 * u - sh - 16 + 4 * ks;
            if (q + 3 < 0 || q >= N2) continue;
            d = Mma<T>::mma(Au[2 * ks], B[2 * ks], d);
            d = Mma<T>::mma(Au[2 * ks + 1], B[2 * ks + 1], d);
          }
          if (again) d = taps_only<T>(B, 0, kUp, lane);
          bad |= not_finite(d[0]);
          if constexpr (SYN) {
            if (pin) {   // rows past R2: dropped
#pragma unroll
              for (int r = 0; r < 4; ++r)
                out.put(ob + (uint32_t)(r * kRow * fplane) * SZ, d[r]);
            }
            ob += (uint32_t)(16 * fplane) * SZ;
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              eacc += (double)v[r] * (double)d[r] * (double)d[r];
              d[r] *= v[r];
            }
          }
        }
        if constexpr (!SYN) {
          vq += 16 * vstride;
#pragma unroll
          for (int r = 0; r < 4; ++r) G[8 + r] = d[r];
          if (u >= 2) {   // outputs 8 (u - 2) .. + 7 of both channels
            V o = {T(0), T(0), T(0), T(0)};
#pragma unroll
            for (int k = 0; !again && k < 12; ++k) o = Mma<T>::mma(Ad[k], G[k], o);
            if (again) o = taps_only<T>(G, 0, kDownReg, lane);
            bad |= not_finite(o[0]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              // m = 8 a + i: i = g + 4 (r & 1), a = r >> 1
              const int i = Mma<T>::row(r, g) & 7, or_ = 4 * (r & 1) + (r >> 1) * O2;
              if (8 * (u - 2) + 7 < O2 || 8 * (u - 2) + i < O2)
                out.put(ob + (uint32_t)(or_ * plane) * SZ, o[r]);
            }
            ob += (uint32_t)(8 * plane) * SZ;
          }
        }
      }
      return __any(bad) != 0;
    };
    if (__builtin_expect(pass(std::false_type{}), 0)) pass(std::true_type{});
  }
  if constexpr (!SYN) {
    const double b = plane_block_sum(eacc);
    if (threadIdx.x == 0) epart[w.epart + blockIdx.x] = b;
  }
}

// ---------------------------------------------------------------------------
// kinetic term along one axis
// ---------------------------------------------------------------------------
// SEG outputs per lane, i' = i0 + 14 .. i0 + 13 + SEG, of both channels:
//   r_a = fac sum_j sum_b K_ab[j] x_b(i' + j)
// from the LDS column x_b(i) = S[lx + i st + b D], 0 <= i < NA, zero
// elsewhere (S[0] and S[D] hold zeros); the lanes of a wave have i0 = ia .. ib.
// The taps run in the outer loop and a ring of inputs slides with them, so
// each tap is moved into scalar registers once for SEG outputs; the two
// channels of a point are one LDS read, issued two taps ahead, and pairs of
// taps that meet only zeros are left out.
// FP32: the scaling channel (exact as doubles) and the centre taps are summed
// in double with FP64 taps, the wavelet channel's other taps in FP32.
template <typename T, int SEG, int D>
__device__ __forceinline__ void kin_taps(const T* S, int lx, int st, int i0, int ia, int ib, int NA,
                                         double fac, double (&r0)[SEG], double (&r1)[SEG]) {
  constexpr int GT = 2, NG = (29 + GT - 1) / GT, RS = SEG + GT;
  double x0[RS], s0[SEG], s1[SEG];
  T x1[RS], w0[SEG], w1[SEG], n0[GT], n1[GT];
  int at = lx + i0 * st;
  int i = i0;
  auto fetch = [&](T& v0, T& v1) {   // the next input
    const int a = (uint32_t)i < (uint32_t)NA ? at : 0;
    v0 = S[a];
    v1 = S[a + D];
    ++i;
    at += st;
  };
#pragma unroll
  for (int k = 0; k < SEG + GT - 1; ++k) {
    T v0;
    fetch(v0, x1[k]);
    x0[k] = (double)v0;
  }
#pragma unroll
  for (int o = 0; o < SEG; ++o) {
    s0[o] = s1[o] = 0.0;
    w0[o] = w1[o] = T(0);
  }
#pragma unroll
  for (int gr = 0; gr < NG; ++gr) {
    if (gr + 1 < NG) {
#pragma unroll
      for (int k = 0; k < GT; ++k) fetch(n0[k], n1[k]);
    }
    if (ib + GT * gr + GT + SEG - 2 >= 0 && ia + GT * gr < NA) {   // not only zeros
#pragma unroll
      for (int t = GT * gr; t < GT * gr + GT; ++t) {
        if (t >= 29) continue;
#pragma unroll
        for (int o = 0; o < SEG; ++o) {
          const double a = x0[(t + o) % RS];
          const T b = x1[(t + o) % RS];
          s0[o] += kK64[0][0][t] * a;
          s1[o] += kK64[1][0][t] * a;
          if (sizeof(T) == 8 || t == 14) {
            s0[o] += kK64[0][1][t] * (double)b;
            s1[o] += kK64[1][1][t] * (double)b;
          } else {
            w0[o] += (T)kK32[0][1][t] * b;
            w1[o] += (T)kK32[1][1][t] * b;
          }
        }
      }
    }
    if (gr + 1 < NG) {
#pragma unroll
      for (int k = 0; k < GT; ++k) {
        const int sl = (GT * (gr + 1) + SEG - 1 + k) % RS;
        x0[sl] = (double)n0[k];
        x1[sl] = n1[k];
      }
    }
  }
#pragma unroll
  for (int o = 0; o < SEG; ++o) {
    r0[o] = fac * (sizeof(T) == 8 ? s0[o] : s0[o] + (double)w0[o]);
    r1[o] = fac * (sizeof(T) == 8 ? s1[o] : s1[o] + (double)w1[o]);
  }
}

// Kinetic planes in LDS: four zeros, then the point (row j, x) at
// 4 + j kin_row(N0) + 4 x: its components as [a1][a2 or a3].  The odd row
// stride puts lanes along x and lanes along the rows on distinct banks.
__device__ __forceinline__ int kin_row(int n0) { return 4 * n0 + 1; }
template <typename T>
__device__ __forceinline__ void put_kin(T* S, int n0, int j, int x, const T* v) {
  T* const o = S + 4 + j * kin_row(n0) + 4 * x;
  o[0] = v[0];
  o[1] = v[2];
  o[2] = v[1];
  o[3] = v[3];
}

// ---------------------------------------------------------------------------
// k_kin_slab: block = (function, y, a2): z part of the kinetic term
// ---------------------------------------------------------------------------
// The x-z slab of four components -> OZ[c][z'][y][x]; a wave takes 64 columns
// (x, a1) and 8 outputs z'.
template <typename T>
__device__ __forceinline__ void kin_slab(int bx, const SfDev* __restrict__ sfs,
                                         const wvl_seg* __restrict__ seg,
                                         const int32_t* __restrict__ rt,
                                         const RowRun* __restrict__ rr, const T* __restrict__ psi,
                                         const SfWork* __restrict__ wk, T* __restrict__ ws,
                                         double fac, double* __restrict__ kpart) {
  extern __shared__ __align__(32) unsigned char smem_raw[];
  const SfWork& w = wk[blockIdx.y];
  const SfDev& sf = sfs[w.id];
  const int N0 = sf.n[0], N1 = sf.n[1], N2 = sf.n[2], e = sf.ext;
  const int y = bx >> 1, a2 = bx & 1;
  if (y >= N1) return;   // uniform over the block
  const int O2 = N2 + 2 * e;
  T* const S = reinterpret_cast<T*>(smem_raw);
  if (threadIdx.x < 4) S[threadIdx.x] = T(0);
  load_rows<T, 4>(N2, 2 * a2, 4, sf, seg, rt, rr, psi, y, N1,
                  [&](int j, int x, const T* v) { put_kin(S, N0, j, x, v); });
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nseg = (O2 + 7) >> 3, ngrp = (2 * N0 + 63) >> 6;
  const int ocomp = O2 * N1 * N0, zst = N1 * N0;
  const Buf<T> oz(ws + w.pz, 8ll * ocomp);
  constexpr uint32_t SZ = sizeof(T);
  double eacc = 0.0;
  for (int job = wave; job < nseg * ngrp; job += kPlaneThreads / 64) {
    const int sg = job % nseg, ci = (job / nseg) * 64 + lane;
    const bool act = ci < 2 * N0;
    const int a1 = ci & 1, x = act ? ci >> 1 : 0;
    const int lx = 4 + 4 * x + 2 * a1, st = kin_row(N0);
    double r0[8], r1[8];
    const int ip = 8 * sg - e;   // first output
    kin_taps<T, 8, 1>(S, lx, st, ip - 14, ip - 14, ip - 14, N2, fac, r0, r1);
    if (!act) continue;
    const uint32_t o0 = (uint32_t)((a1 + 2 * a2) * ocomp + (8 * sg * N1 + y) * N0 + x) * SZ;
    const uint32_t o1 = o0 + 4u * (uint32_t)ocomp * SZ;
#pragma unroll
    for (int o = 0; o < 8; ++o) {
      if (8 * sg + o < O2) {
        oz.put(o0 + (uint32_t)(o * zst) * SZ, (T)r0[o]);
        oz.put(o1 + (uint32_t)(o * zst) * SZ, (T)r1[o]);
      }
      const int i = ip + o;
      if (i >= 0 && i < N2)
        eacc += (double)S[lx + i * st] * r0[o] + (double)S[lx + i * st + 1] * r1[o];
    }
  }
  const double b = plane_block_sum(eacc);
  if (threadIdx.x == 0) kpart[w.kpart + 2 * N2 * plane_strips(N0, N1, e) + bx] = b;
}

__global__ __launch_bounds__(256) void k_up_plane(
    const SfDev* __restrict__ sfs, const wvl_seg* __restrict__ seg, const int32_t* __restrict__ rt,
    const RowRun* __restrict__ rr, const double* __restrict__ psi, const SfWork* __restrict__ wk,
    double* __restrict__ ws, int both) {
  up_plane(blockIdx.x, sfs, seg, rt, rr, psi, wk, ws, both);
}
__global__ __launch_bounds__(256, 4) void k_up_plane_valu(
    const SfDev* __restrict__ sfs, const wvl_seg* __restrict__ seg, const int32_t* __restrict__ rt,
    const RowRun* __restrict__ rr, const float* __restrict__ psi, const SfWork* __restrict__ wk,
    float* __restrict__ ws) {
  up_plane(blockIdx.x, sfs, seg, rt, rr, psi, wk, ws, 1);
}
template <typename T>
__global__ __launch_bounds__(kPlaneThreads, sizeof(T) == 4 ? 4 : 2) void k_kin_slab(
    const SfDev* __restrict__ sfs, const wvl_seg* __restrict__ seg,
    const int32_t* __restrict__ rt, const RowRun* __restrict__ rr, const T* __restrict__ psi,
    const SfWork* __restrict__ wk, T* __restrict__ ws, double fac, double* __restrict__ kpart) {
  kin_slab<T>(blockIdx.x, sfs, seg, rt, rr, psi, wk, ws, fac, kpart);
}

// ---------------------------------------------------------------------------
// k_up_kin: both of the above, which only read psi, in one launch
// ---------------------------------------------------------------------------
// Blocks 0 .. nup - 1 of a function are those of the up pass, the others those
// of the z part.  For calls that leave the chip idle (see kUpKinBlocks).
template <typename T>
__global__ __launch_bounds__(kPlaneThreads, sizeof(T) == 4 ? 4 : 2) void k_up_kin(
    const SfDev* __restrict__ sfs, const wvl_seg* __restrict__ seg,
    const int32_t* __restrict__ rt, const RowRun* __restrict__ rr, const T* __restrict__ psi,
    const SfWork* __restrict__ wk, T* __restrict__ ws, int nup, int both, double fac,
    double* __restrict__ kpart) {
  if ((int)blockIdx.x < nup)
    up_plane(blockIdx.x, sfs, seg, rt, rr, psi, wk, ws, both);
  else
    kin_slab<T>(blockIdx.x - nup, sfs, seg, rt, rr, psi, wk, ws, fac, kpart);
}

// ---------------------------------------------------------------------------
// k_back_plane: block = (function, z', a3, strip of 24 or 32 rows y')
// ---------------------------------------------------------------------------
// G2 -> y down pass -> Q[a2][row][px] in LDS -> x down pass ->
// OUT[a1 + 2 a2][row][x'] in LDS; then the plane z = z' - ext is uncompressed
// into Q's place, the x kinetic part and then y + z parts are added (in this
// order: the sums of the column kernels), and the points of each row go to the
// compressed output.  One block holds four of the eight components of its
// points: 1 + 3 or 4 of the values a point has.  The blocks of a plane (a3,
// strips) run on one XCD, whose L2 joins their stores and serves their shared
// reads.  24 rows: three row tiles of the x pass, and LDS for four (FP32) or
// two (FP64) blocks per CU at the usual box sizes; the phases of one block are
// covered by the others.  32 where that is all of the box's rows (plane_strip).
// FP64 planes fill half a CU's LDS or more: twice the waves per block keep
// four per SIMD.  WIDE, FP32 where one block fills a CU's LDS (plane_wide): 1,024
// threads for 256, so that its phases are not four waves' on their own (60 boxes
// of 60^3 points: 4.59 -> 3.08 ms, one of 58^3 85 -> 60 us).
template <typename T> constexpr int back_threads(bool wide) {
  return sizeof(T) == 8 ? 512 : wide ? kWideThreads : 256;
}
constexpr int kRowWords = 2;   // O0 <= kPlaneMaxN + 32 points per row
template <typename T, bool WIDE, int kStrip>
__global__ __launch_bounds__(back_threads<T>(WIDE), 4) void k_back_plane(
    const SfDev* __restrict__ sfs, const wvl_seg* __restrict__ seg,
    const int32_t* __restrict__ rt, const RowRun* __restrict__ rr, const T* __restrict__ psi,
    const SfWork* __restrict__ wk, const T* __restrict__ ws, T* __restrict__ out, int pot_on,
    int kin_on, int accumulate, double fac, double* __restrict__ kpart) {
  extern __shared__ __align__(32) unsigned char smem_raw[];
  constexpr int NT = back_threads<T>(WIDE), NW = NT / 64;
  constexpr uint32_t SZ = sizeof(T);
  const SfWork& w = wk[blockIdx.y];
  const SfDev& sf = sfs[w.id];
  const int N0 = sf.n[0], N1 = sf.n[1], N2 = sf.n[2], e = sf.ext;
  const int R1 = 2 * N1 + 29, P0 = pad16(2 * N0 + 29);
  const int O0 = N0 + 2 * e, O1 = N1 + 2 * e, O2 = N2 + 2 * e;
  // blocks are dealt to the 8 XCDs in turn (gridDim.x is a multiple of 8)
  const int NS = (O1 + kStrip - 1) / kStrip, per = 2 * NS, bj = blockIdx.x >> 3;
  const int zp = 8 * (bj / per) + (blockIdx.x & 7);
  if (zp >= O2) return;   // uniform over the block
  const int a3 = (bj % per) & 1, strip = (bj % per) >> 1;
  const int s0 = kStrip * strip, ns = min(kStrip, O1 - s0);   // rows y' = s0 .. s0 + ns - 1
  const int z = zp - e;
  const bool kin = kin_on && z >= 0 && z < N2;
  const int ldo = O0 | 1, ldq = P0 + 4;
  const int och = kStrip * ldo;
  T* const Q = reinterpret_cast<T*>(smem_raw);   // Q[2][24][ldq], later the plane
  T* const OUT = Q + max(2 * kStrip * ldq, plane_kin_elems(N0, N1));
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the points of this strip's output rows (pattern, row): a bit per x' and
  // the index of the row's first point (the points of a row, also of one with
  // several runs, are consecutive in the output).  One wave per pattern, a
  // lane per segment.
  __shared__ uint64_t rmask[2][kStrip][kRowWords];
  __shared__ int32_t roff[2][kStrip];
  __shared__ uint8_t rank_x[NW][64];
  const int orow = zp * O1 + s0, xg0 = sf.lo[0] - e, nwd = (O0 + 63) >> 6;
  if (wave >= NW - 2) {
    const int pat = wave - (NW - 2);
    if (lane < kStrip) {
#pragma unroll
      for (int wd = 0; wd < kRowWords; ++wd) rmask[pat][lane][wd] = 0;
      roff[pat][lane] = INT32_MAX;
    }
    const int64_t grow = sf.rt[2 + pat] + orow;
    const int q1 = rt[grow + ns], y0 = sf.lo[1] - e + s0;
    for (int q = rt[grow] + lane; q < q1; q += 64) {
      const wvl_seg sg = seg[q];
      const int yl = sg.i2 - y0, xs = sg.i1s - xg0, xe = sg.i1e - xg0 + 1;
#pragma unroll
      for (int wd = 0; wd < kRowWords; ++wd) {
        const int lo = max(xs - 64 * wd, 0), hi = min(xe - 64 * wd, 64);
        if (lo < hi)
          atomicOr((unsigned long long*)&rmask[pat][yl][wd], (~0ull >> (64 - (hi - lo))) << lo);
      }
      atomicMin(&roff[pat][yl], (int)sg.off);
    }
  }
  if (pot_on) {
    typedef typename Mma<T>::V V;
    T A[12];
    load_band(A, kDown, lane);
    // y down pass: a wave takes 16 columns px, the fine rows p = 2 (s0 - e) ..
    // + 79 (0 outside the box; columns past R0 are not written in FP32), and
    // the outputs s0 .. s0 + 23 of both channels.  Q column of px: px + qs (qs
    // aligns the x pass' groups of four points for odd ext), zeros beside.
    const int qs = (2 * e) & 3;
    const Buf<T> g2(ws + w.p2 + (int64_t)(a3 * O2 + zp) * (R1 * P0), R1 * P0);
    auto y_pass = [&](auto again_) {
      constexpr bool again = decltype(again_)::value;
      bool bad = false;
      for (int tx = wave; tx < P0 >> 4; tx += NW) {
        constexpr int NB = 4 * (kStrip / 8 + 2);
        T B[NB];
        const uint32_t o = 16 * tx + n < 2 * N0 + 29
                               ? (uint32_t)((2 * (s0 - e) + g) * P0 + 16 * tx + n) * SZ : kNone;
#pragma unroll
        for (int k = 0; k < NB; ++k) B[k] = g2.at(o + (uint32_t)(4 * k * P0) * SZ);
        T* const qo = Q + (sizeof(T) == 4 ? (g >> 1) * kStrip + 4 * (g & 1) : g) * ldq + 16 * tx + n + qs;
#pragma unroll
        for (int t = 0; t < kStrip / 8; ++t) {
          V d = {T(0), T(0), T(0), T(0)};
#pragma unroll
          for (int k = 0; !again && k < 12; ++k) d = Mma<T>::mma(A[k], B[4 * t + k], d);
          if (again) d = taps_only<T>(B, 4 * t, kDown, lane);
          bad |= not_finite(d[0]);
          // m = 8 a2 + i: f32 i = 4 (g & 1) + r, a2 = g >> 1; f64 i = g + 4 (r & 1), a2 = r >> 1
#pragma unroll
          for (int r = 0; r < 4; ++r)
            qo[(8 * t + (sizeof(T) == 4 ? r : 4 * (r & 1) + (r >> 1) * kStrip)) * ldq] = d[r];
        }
      }
      return __any(bad) != 0;
    };
    if (__builtin_expect(y_pass(std::false_type{}), 0)) y_pass(std::true_type{});
    if (tid < 2 * kStrip) {
      for (int c = 0; c < qs; ++c) Q[tid * ldq + c] = T(0);
      for (int c = P0 + qs; c < ldq; ++c) Q[tid * ldq + c] = T(0);
    }
    __syncthreads();
    // x down pass: 16 rows (a2, y') per wave, half of the x' tiles
    const int T8 = (O0 + 7) >> 3, half = (T8 + 1) >> 1;
    auto x_pass = [&](auto again_) {
      constexpr bool again = decltype(again_)::value;
      bool bad = false;
      for (int job = wave; job < 2 * (2 * kStrip / 16); job += NW) {
        const int row = (job >> 1) * 16 + n;
        const T* const in = Q + row * ldq;
        const int t0 = (job & 1) * half, t1 = min(T8, t0 + half);
        const int a2 = row >= kStrip ? 1 : 0;
        T* const o = OUT + 2 * a2 * och + (row - a2 * kStrip) * ldo +
                     (sizeof(T) == 4 ? (g >> 1) * och + 4 * (g & 1) : g);
        T B[12];
        auto fetch = [&](int kb, int slot) {   // points 16 kb - 2 e + 4 r + g
          const int c = 16 * kb - 2 * e + g + qs;
#pragma unroll
          for (int r = 0; r < 4; ++r) {   // groups of four in or outside [0, ldq)
            const bool ok = (uint32_t)(c - g + 4 * r) < (uint32_t)ldq;
            const T v = in[ok ? c + 4 * r : 0];
            B[4 * slot + r] = ok ? v : T(0);
          }
        };
        fetch(t0, 1);
        fetch(t0 + 1, 2);
        for (int t = t0; t < t1; ++t) {
#pragma unroll
          for (int k = 0; k < 8; ++k) B[k] = B[k + 4];
          fetch(t + 2, 2);
          V d = {T(0), T(0), T(0), T(0)};
#pragma unroll
          for (int k = 0; !again && k < 12; ++k) d = Mma<T>::mma(A[k], B[k], d);
          if (again) d = taps_only<T>(B, 0, kDown, lane);
          bad |= not_finite(d[0]);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int xp = 8 * t + (Mma<T>::row(r, g) & 7);
            if (8 * t + 7 < O0 || xp < O0)
              o[8 * t + (sizeof(T) == 4 ? r : 4 * (r & 1) + (r >> 1) * och)] = d[r];
          }
        }
      }
      return __any(bad) != 0;
    };
    if (__builtin_expect(x_pass(std::false_type{}), 0)) x_pass(std::true_type{});
  } else {
    for (int k = tid; k < 4 * och; k += NT) OUT[k] = T(0);
  }
  __syncthreads();   // OUT written, Q no longer read
  double eacc = 0.0;
  if (kin) {
    if (tid < 4) Q[tid] = T(0);
    load_rows<T, 4>(N1, 4 * a3, 2, sf, seg, rt, rr, psi, z * N1, 1,
                    [&](int j, int x, const T* v) { put_kin(Q, N0, j, x, v); });
    __syncthreads();
    // x part: an item is a row (y, a2) of the strip inside the box and 8 outputs
    // x'.  FP32: the waves take 64 consecutive items, so that the usual 48 rows
    // x 5 segments are one round of four waves (two before: 4.02 -> 3.82 ms for
    // 700 functions); FP64, with eight waves, a segment each (items of several
    // segments cost registers: 8.24 -> 8.51 ms for 1,000).
    const int ya = max(0, s0 - e), nyb = max(0, min(N1, s0 + ns - e) - ya);
    const int nsx = (O0 + 7) >> 3;
    const int px = sizeof(T) == 4 ? 2 * nyb : nyb > 0 ? 64 : 0;   // items per segment
    for (int it = 64 * wave; it < nsx * px; it += 64 * NW) {
      const int ca = it / px, cb = sizeof(T) == 4 ? min(it + 63, nsx * px - 1) / px : ca;
      const int item = it + lane, job = sizeof(T) == 4 ? min(item / px, nsx - 1) : ca;
      const bool act = item - job * px < 2 * nyb;
      const int row = act ? item - job * px : 0;
      const int a2 = row & 1, y = ya + (row >> 1);
      const int lx = 4 + y * kin_row(N0) + a2;
      double r0[8], r1[8];
      const int ip = 8 * job - e;
      kin_taps<T, 8, 2>(Q, lx, 4, ip - 14, 8 * ca - e - 14, 8 * cb - e - 14, N0, fac, r0, r1);
      if (!act) continue;
      T* const o0 = OUT + 2 * a2 * och + (y + e - s0) * ldo + 8 * job;
#pragma unroll
      for (int o = 0; o < 8; ++o) {
        if (8 * job + o < O0) {
          o0[o] += (T)r0[o];
          o0[och + o] += (T)r1[o];
        }
        const int i = ip + o;
        if (i >= 0 && i < N0)
          eacc += (double)Q[lx + 4 * i] * r0[o] + (double)Q[lx + 4 * i + 2] * r1[o];
      }
    }
    __syncthreads();
  }
  if (kin_on) {
    // y + z parts: items of a column (x, a1) and 8 outputs y'
    const int nsy = (ns + 7) >> 3, ocomp = O2 * N1 * N0;
    const Buf<T> oz(ws + w.pz, 8ll * ocomp);
    const int py = sizeof(T) == 4 ? 2 * N0 : (2 * N0 + 63) & ~63;   // items per segment
    for (int it = 64 * wave; it < nsy * py; it += 64 * NW) {
      const int ca = it / py, cb = sizeof(T) == 4 ? min(it + 63, nsy * py - 1) / py : ca;
      const int item = it + lane, sg = sizeof(T) == 4 ? min(item / py, nsy - 1) : ca;
      const bool act = item - sg * py < 2 * N0;
      const int ci = act ? item - sg * py : 0;
      const int a1 = ci & 1, x = ci >> 1;
      const int ip = s0 + 8 * sg - e;
      const int zb = (4 * a3 + a1) * ocomp + (zp * N1 + ip) * N0 + x;   // oz of output 0, a2 = 0
      T z0[8], z1[8];
#pragma unroll
      for (int o = 0; o < 8; ++o) {
        const bool in = ip + o >= 0 && ip + o < N1;
        z0[o] = oz.at(in ? (uint32_t)(zb + o * N0) * SZ : kNone);
        z1[o] = oz.at(in ? (uint32_t)(zb + o * N0 + 2 * ocomp) * SZ : kNone);
      }
      double r0[8], r1[8];
      const int lx = 4 + 4 * x + 2 * a1, st = kin_row(N0);
      if (kin) {
        kin_taps<T, 8, 1>(Q, lx, st, ip - 14, s0 + 8 * ca - e - 14, s0 + 8 * cb - e - 14, N1, fac, r0,
                          r1);
      } else {
#pragma unroll
        for (int o = 0; o < 8; ++o) r0[o] = r1[o] = 0.0;
      }
      if (!act) continue;
      T* const o0 = OUT + a1 * och + 8 * sg * ldo + x + e;
#pragma unroll
      for (int o = 0; o < 8; ++o) {
        o0[o * ldo] += (T)r0[o] + z0[o];
        o0[2 * och + o * ldo] += (T)r1[o] + z1[o];
        const int i = ip + o;
        if (kin && i >= 0 && i < N1 && 8 * sg + o < ns)
          eacc += (double)Q[lx + i * st] * r0[o] + (double)Q[lx + i * st + 1] * r1[o];
      }
    }
    __syncthreads();
  }
  // compression: a wave per row; the values of its points are consecutive in
  // the output, so are the stores (wavelets: nc of every seven)
  const Buf<T> outc(out + sf.cout, sf.on_c), outf(out + sf.cout + sf.on_c, 7 * sf.on_f);
  auto put = [&](const Buf<T>& o, uint32_t at, T v) { o.put(at, accumulate ? o.at(at) + v : v); };
  const int nc = 3 + a3;   // wavelets per point here: components 1..3 or 4..7
  const T* const of = OUT + (a3 ? 0 : och);
  const uint64_t below = (1ull << lane) - 1ull;
  for (int yl = wave; yl < ns; yl += NW) {
    if (!a3) {
      int off = roff[0][yl];
      for (int wd = 0; wd < nwd; ++wd) {
        const uint64_t m = rmask[0][yl][wd];
        if ((m >> lane) & 1)
          put(outc, (uint32_t)(off + __popcll(m & below)) * SZ, OUT[yl * ldo + 64 * wd + lane]);
        off += __popcll(m);
      }
    }
    int off = roff[1][yl];
    for (int wd = 0; wd < nwd; ++wd) {
      const uint64_t m = rmask[1][yl][wd];
      if ((m >> lane) & 1) rank_x[wave][__popcll(m & below)] = (uint8_t)lane;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const T* const src = of + yl * ldo + 64 * wd;
      const int cnt = __popcll(m);
      for (int t = lane; t < nc * cnt; t += 64) {
        const int pt = a3 ? t >> 2 : (int)(((uint32_t)t * 43691u) >> 17), c = t - nc * pt;
        put(outf, (uint32_t)(7 * (off + pt) + 3 * a3 + c) * SZ, src[c * och + rank_x[wave][pt]]);
      }
      __builtin_amdgcn_wave_barrier();
      off += cnt;
    }
  }
  if (kin) {
    const double b = plane_block_sum(eacc);
    if (tid == 0) kpart[w.kpart + (2 * z + a3) * NS + strip] = b;
  }
}

// one block per function: fixed-order sums of its energy partials
__global__ __launch_bounds__(256) void k_plane_energies(const SfWork* __restrict__ wk,
                                                        const double* __restrict__ parts, int f64,
                                                        double* __restrict__ e_kin,
                                                        double* __restrict__ e_pot) {
  const SfWork& w = wk[blockIdx.x];
  for (int which = 0; which < 2; ++which) {
    double* const o = which ? e_pot : e_kin;
    if (o == nullptr) continue;
    const int64_t off = which ? w.epart : w.kpart;
    const int cnt = (int)(which ? w.nepart_pl[f64] : w.nkpart_pl);
    double v = 0.0;
    for (int i = threadIdx.x; i < cnt; i += 256) v += parts[off + i];
    const double b = plane_block_sum(v);
    if (threadIdx.x == 0) o[w.id] = b;
    __syncthreads();
  }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

// More than 64 KiB of dynamic LDS has to be asked for.  The limit belongs to the
// kernel on a device, not to a launch: it is set here to the most that any plan
// may use, and never to a launch's own size, which a launch of another thread
// (or a captured one) may exceed.
int preload_plane_kernels() {
  const void* fns[] = {(const void*)k_col_tile<false>, (const void*)k_col_tile<true>,
                       (const void*)k_plane_energies};
  const void* lds[] = {(const void*)k_up_plane_valu,     (const void*)k_up_plane,
                       (const void*)k_kin_slab<float>,   (const void*)k_kin_slab<double>,
                       (const void*)k_up_kin<float>,     (const void*)k_up_kin<double>,
                       (const void*)k_back_plane<float, false, 24>,
                       (const void*)k_back_plane<float, false, 32>,
                       (const void*)k_back_plane<float, true, 24>,
                       (const void*)k_back_plane<float, true, 32>,
                       (const void*)k_back_plane<double, false, 24>,
                       (const void*)k_back_plane<double, false, 32>};
  hipError_t e = hipSuccess;
  hipFuncAttributes a;
  for (const void* f : fns)
    if ((e = hipFuncGetAttributes(&a, f)) != hipSuccess) return (int)e;
  for (const void* f : lds) {
    if ((e = hipFuncGetAttributes(&a, f)) != hipSuccess) return (int)e;
    if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 (int)kPlaneLds)) != hipSuccess)
      return (int)e;
  }
  return 0;
}

int launch_up_plane(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                    const RowRun* rr, const void* psi, const SfWork* wk, int nsf, int gridx,
                    int both, size_t lds, void* ws) {
  if (nsf == 0 || gridx == 0) return 0;
  const dim3 g((unsigned)gridx, (unsigned)nsf);
  if (f64)
    hipLaunchKernelGGL(k_up_plane, g, dim3(256), lds, (hipStream_t)stream, sf, seg, rt, rr,
                       (const double*)psi, wk, (double*)ws, both);
  else
    hipLaunchKernelGGL(k_up_plane_valu, g, dim3(256), lds, (hipStream_t)stream, sf, seg, rt, rr,
                       (const float*)psi, wk, (float*)ws);
  return (int)hipGetLastError();
}

int launch_up_kin(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                  const RowRun* rr, const void* psi, const SfWork* wk, int nsf, int nup, int nkin,
                  int both, size_t lds, void* ws, double fac, double* kpart) {
  if (nsf == 0) return 0;
  const dim3 g((unsigned)(nup + nkin), (unsigned)nsf);
  if (f64)
    hipLaunchKernelGGL(k_up_kin<double>, g, dim3(kPlaneThreads), lds, (hipStream_t)stream, sf, seg,
                       rt, rr, (const double*)psi, wk, (double*)ws, nup, both, fac, kpart);
  else
    hipLaunchKernelGGL(k_up_kin<float>, g, dim3(kPlaneThreads), lds, (hipStream_t)stream, sf, seg,
                       rt, rr, (const float*)psi, wk, (float*)ws, nup, both, fac, kpart);
  return (int)hipGetLastError();
}

int launch_col_tile(void* stream, const SfDev* sf, const SfWork* wk, int nsf, int gridx, void* ws,
                    const void* pot, int nf1, int nf2, double* epart, const double* conf,
                    double hh) {
  if (nsf == 0 || gridx == 0) return 0;
  hipLaunchKernelGGL(k_col_tile<false>, dim3((unsigned)gridx, (unsigned)nsf), dim3(256), 0,
                     (hipStream_t)stream, sf, wk, (double*)ws, (const double*)pot, nf1, nf2, epart,
                     conf, hh, nullptr, nullptr);
  return (int)hipGetLastError();
}

int launch_syn_tile(void* stream, const SfDev* sf, const SfWork* wk, int nsf, int gridx, void* ws,
                    const int64_t* fine_off, void* fine) {
  if (nsf == 0 || gridx == 0) return 0;
  hipLaunchKernelGGL(k_col_tile<true>, dim3((unsigned)gridx, (unsigned)nsf), dim3(256), 0,
                     (hipStream_t)stream, sf, wk, (double*)ws, nullptr, 0, 0, nullptr, nullptr, 0.0,
                     fine_off, (double*)fine);
  return (int)hipGetLastError();
}

int launch_kin_slab(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                    const RowRun* rr, const void* psi, const SfWork* wk, int nsf, int gridx,
                    size_t lds, void* ws, double fac, double* kpart) {
  if (nsf == 0 || gridx == 0) return 0;
  const dim3 g((unsigned)gridx, (unsigned)nsf);
  if (f64)
    hipLaunchKernelGGL(k_kin_slab<double>, g, dim3(kPlaneThreads), lds, (hipStream_t)stream, sf,
                       seg, rt, rr, (const double*)psi, wk, (double*)ws, fac, kpart);
  else
    hipLaunchKernelGGL(k_kin_slab<float>, g, dim3(kPlaneThreads), lds, (hipStream_t)stream, sf,
                       seg, rt, rr, (const float*)psi, wk, (float*)ws, fac, kpart);
  return (int)hipGetLastError();
}

int launch_back_plane(int f64, void* stream, const SfDev* sf, const wvl_seg* seg,
                      const int32_t* rt, const RowRun* rr, const void* psi, const SfWork* wk,
                      int nsf, int gridx, int wide, int strip, size_t lds, const void* ws, void* out,
                      int pot_on, int kin_on, int accumulate, double fac, double* kpart) {
  if (nsf == 0 || gridx == 0) return 0;
  const dim3 g((unsigned)gridx, (unsigned)nsf);
  hipStream_t st = (hipStream_t)stream;
  auto go = [&](auto kernel, int threads, auto t) {
    using T = decltype(t);
    hipLaunchKernelGGL(kernel, g, dim3(threads), lds, st, sf, seg, rt, rr, (const T*)psi, wk,
                       (const T*)ws, (T*)out, pot_on, kin_on, accumulate, fac, kpart);
  };
  if (f64)
    strip == 24 ? go(k_back_plane<double, false, 24>, back_threads<double>(false), 0.0)
                : go(k_back_plane<double, false, 32>, back_threads<double>(false), 0.0);
  else if (wide)
    strip == 24 ? go(k_back_plane<float, true, 24>, back_threads<float>(true), 0.0f)
                : go(k_back_plane<float, true, 32>, back_threads<float>(true), 0.0f);
  else
    strip == 24 ? go(k_back_plane<float, false, 24>, back_threads<float>(false), 0.0f)
                : go(k_back_plane<float, false, 32>, back_threads<float>(false), 0.0f);
  return (int)hipGetLastError();
}

int launch_plane_energies(int f64, void* stream, const SfWork* wk, int nsf, const double* parts,
                          double* e_kin, double* e_pot) {
  if (nsf == 0 || (!e_kin && !e_pot)) return 0;
  hipLaunchKernelGGL(k_plane_energies, dim3(nsf), dim3(256), 0, (hipStream_t)stream, wk, parts,
                     f64, e_kin, e_pot);
  return (int)hipGetLastError();
}

}  // namespace wvl
