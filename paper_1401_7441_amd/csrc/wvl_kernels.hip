// HIP kernels for gfx950 (MI355X): the dense-box <-> compressed copies of the
// standalone uncompress / compress entry points, fixed-order energy sums, and
// the sparse overlap / Hamiltonian matrix elements.  The local Hamiltonian
// itself runs in the fused kernels of wvl_fused.hip.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "wvl_internal.h"

namespace wvl {

constexpr int TPB = 256;

// deterministic block sum of one double per thread: a fixed shuffle tree in
// each 64-lane wave, then the wave sums in order
__device__ double block_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  __shared__ double part[16];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  if (lane == 0) part[wv] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) r += part[k];
  __syncthreads();
  return r;
}

// ---------------------------------------------------------------------------
// compressed <-> dense
// ---------------------------------------------------------------------------

// Uncompress: thread per dense point of the input box [8][n2][n1][n0].
template <typename T>
__global__ __launch_bounds__(TPB) void k_gather(const SfDev* __restrict__ sfs,
                                                const wvl_seg* __restrict__ seg,
                                                const int32_t* __restrict__ rt,
                                                const T* __restrict__ psi, T* __restrict__ dst,
                                                int sf0) {
  const int s = blockIdx.y;
  const SfDev& sf = sfs[sf0 + s];
  const int n0 = sf.n[0], n1 = sf.n[1], n2 = sf.n[2];
  const int64_t vol = 8ll * n0 * n1 * n2;
  const int64_t idx = (int64_t)blockIdx.x * TPB + threadIdx.x;
  if (idx >= vol) return;
  const int x = (int)(idx % n0);
  int64_t t = idx / n0;
  const int y = (int)(t % n1);
  t /= n1;
  const int z = (int)(t % n2);
  const int c = (int)(t / n2);
  const int pat = c == 0 ? 0 : 1;
  const int64_t r = (int64_t)z * n1 + y;
  const int32_t s0 = rt[sf.rt[pat] + r], s1 = rt[sf.rt[pat] + r + 1];
  const int gx = sf.lo[0] + x;
  T v = T(0);
  for (int q = s0; q < s1; ++q) {
    const wvl_seg g = seg[q];
    if (gx >= g.i1s && gx <= g.i1e) {
      const int64_t k = g.off + (gx - g.i1s);
      v = c == 0 ? psi[sf.cin + k] : psi[sf.cin + sf.n_c + 7 * k + (c - 1)];
      break;
    }
  }
  dst[sf.box_in + idx] = v;
}

// Compress onto the output pattern: thread per dense point of the output box.
template <typename T>
__global__ __launch_bounds__(TPB) void k_scatter(const SfDev* __restrict__ sfs,
                                                 const wvl_seg* __restrict__ seg,
                                                 const int32_t* __restrict__ rt,
                                                 const T* __restrict__ src, T* __restrict__ out,
                                                 int sf0) {
  const int s = blockIdx.y;
  const SfDev& sf = sfs[sf0 + s];
  const int e = sf.ext;
  const int n0 = sf.n[0] + 2 * e, n1 = sf.n[1] + 2 * e, n2 = sf.n[2] + 2 * e;
  const int64_t vol = 8ll * n0 * n1 * n2;
  const int64_t idx = (int64_t)blockIdx.x * TPB + threadIdx.x;
  if (idx >= vol) return;
  const int x = (int)(idx % n0);
  int64_t t = idx / n0;
  const int y = (int)(t % n1);
  t /= n1;
  const int z = (int)(t % n2);
  const int c = (int)(t / n2);
  const int pat = c == 0 ? 2 : 3;
  const int64_t r = (int64_t)z * n1 + y;
  const int32_t s0 = rt[sf.rt[pat] + r], s1 = rt[sf.rt[pat] + r + 1];
  const int gx = sf.lo[0] - e + x;
  for (int q = s0; q < s1; ++q) {
    const wvl_seg g = seg[q];
    if (gx >= g.i1s && gx <= g.i1e) {
      const int64_t k = g.off + (gx - g.i1s);
      const int64_t o = c == 0 ? sf.cout + k : sf.cout + sf.on_c + 7 * k + (c - 1);
      out[o] = src[sf.box_out + idx];
      return;
    }
  }
}

// one block per function: fixed-order sum of its partials
__global__ __launch_bounds__(TPB) void k_finalize(const SfWork* __restrict__ wk, int sf0,
                                                  const double* __restrict__ parts, int which,
                                                  int nblk, double* __restrict__ out) {
  const int s = blockIdx.x;
  const int64_t off = which == 0 ? wk[s].epart : wk[s].kpart;
  if (which == 1) nblk = (int)wk[s].nkpart;   // only the function's own slots
  double v = 0.0;
  for (int i = threadIdx.x; i < nblk; i += TPB) v += parts[off + i];
  const double b = block_sum(v);
  if (threadIdx.x == 0) out[wk[s].id] = b;
}

template <typename T>
__global__ __launch_bounds__(TPB) void k_fill(T* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
  if (i < n) p[i] = T(0);
}

// ---------------------------------------------------------------------------
// sparse pattern and values
// ---------------------------------------------------------------------------

struct PatBox {
  int ox, oy, oz, bx, by;  // pattern box origin and row extents
};

__device__ __forceinline__ PatBox pat_box(const SfDev& s, int out) {
  const int e = out ? s.ext : 0;
  return PatBox{s.lo[0] - e, s.lo[1] - e, s.lo[2] - e, s.n[0] + 2 * e, s.n[1] + 2 * e};
}

__device__ __forceinline__ bool bb_meet(const int32_t* a, const int32_t* b) {
  return a[0] <= a[1] && b[0] <= b[1] && a[0] <= b[1] && b[0] <= a[1] && a[2] <= b[3] &&
         b[2] <= a[3] && a[4] <= b[5] && b[4] <= a[5];
}

// does the input coarse pattern of A share a point with B's pattern?
__device__ bool coarse_intersect(const SfDev& A, const SfDev& B, int ket_out,
                                 const wvl_seg* __restrict__ seg,
                                 const int32_t* __restrict__ rt) {
  const int32_t* bb = ket_out ? B.bb_out : B.bb_in;
  const int y0 = max(A.bb_in[2], bb[2]), y1 = min(A.bb_in[3], bb[3]);
  const int z0 = max(A.bb_in[4], bb[4]), z1 = min(A.bb_in[5], bb[5]);
  const PatBox pb = pat_box(B, ket_out);
  const int pB = ket_out ? 2 : 0;
  for (int z = z0; z <= z1; ++z) {
    for (int y = y0; y <= y1; ++y) {
      const int64_t ra = (int64_t)(z - A.lo[2]) * A.n[1] + (y - A.lo[1]);
      const int64_t rb = (int64_t)(z - pb.oz) * pb.by + (y - pb.oy);
      int qa = rt[A.rt[0] + ra], qa1 = rt[A.rt[0] + ra + 1];
      int qb = rt[B.rt[pB] + rb], qb1 = rt[B.rt[pB] + rb + 1];
      while (qa < qa1 && qb < qb1) {
        const wvl_seg sa = seg[qa], sb = seg[qb];
        if (sa.i1e < sb.i1s) {
          ++qa;
        } else if (sb.i1e < sa.i1s) {
          ++qb;
        } else {
          return true;
        }
      }
    }
  }
  return false;
}

// one 64-lane wavefront per row a; count (rowptr == NULL) or fill columns
__global__ __launch_bounds__(64) void k_pattern(const SfDev* __restrict__ sfs,
                                                const wvl_seg* __restrict__ seg,
                                                const int32_t* __restrict__ rt, int nsf,
                                                int ket_out, int64_t* __restrict__ count,
                                                const int64_t* __restrict__ rowptr,
                                                int32_t* __restrict__ col) {
  const int a = blockIdx.x;
  const int lane = threadIdx.x;
  const SfDev& A = sfs[a];
  int64_t n = 0;
  for (int b0 = 0; b0 < nsf; b0 += 64) {
    const int b = b0 + lane;
    bool hit = false;
    if (b < nsf) {
      const SfDev& B = sfs[b];
      if (bb_meet(A.bb_in, ket_out ? B.bb_out : B.bb_in))
        hit = coarse_intersect(A, B, ket_out, seg, rt);
    }
    const unsigned long long m = __ballot(hit);
    if (rowptr != nullptr && hit) {
      const int before = __popcll(m & ((1ull << lane) - 1ull));
      col[rowptr[a] + n + before] = b;
    }
    n += __popcll(m);
  }
  if (rowptr == nullptr && lane == 0) count[a] = n;
}

// One block of W waves per nonzero (a, b): batches of 64 rows of the box where
// both patterns may meet, dealt to the waves in turn.  Phase 1: lane r resolves
// row r (run records; the segment lists where a row holds several runs) to the
// first overlapping run of each kind (scaling / wavelet) and one further run of
// either; more, which sphere patterns hardly produce, are summed by that lane
// directly.  Phase 2: four 16-lane groups stream the coarse runs, four rows of
// each under way; then the whole wave takes the fine runs (seven wavelets per
// point: 70 values on average) and the further ones, four under way.  Every
// lane's partial sum and the final tree have an order fixed by the pair.
// Bound by the lines read from beyond L2, in FP64 by their bytes: H of 1,000
// functions of radius 5-7 bohr (301,162 entries) reads 31.4 GB there, 5.8 TB/s (a
// large copy: 4.8); in FP32 18.9 GB, 4.8 TB/s, but 14.7 GB with two waves per pair
// take no less time, so there the wait for a line counts as well.  Seven waves per
// SIMD are resident and wait for two thirds (FP64) and three quarters of their
// time; a SIMD issues 0.36 and 0.53 vector instructions in four cycles (the FP32
// up pass 1.3).  Registers stay below those that let eight waves run.  That H in FP64: 5.63 ms with one wave per pair and 16 lanes
// per fine run, 5.4 in this form; FP32, 4,000 functions: 9.46 and 7.92 ms; S of 56
// functions: 112 and 31 us.
// mirror (may be NULL): for the pair at processing position s, the CSR
// position that receives the same value as well (the transposed pair of a
// symmetric matrix), or -1.
template <typename T>
__device__ __forceinline__ double run_dot(const T* __restrict__ pa, const T* __restrict__ pk,
                                          int n) {
  double acc = 0.0;
  for (int x = 0; x < n; ++x) acc += (double)pa[x] * (double)pk[x];
  return acc;
}

// orders a wave's LDS writes before its other lanes' reads (and the reads
// before the next writes)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The runs of all lanes (starts a, b, length n; 0: none), one after the other
// by the whole wave: lane l takes the positions l, l + 64, ...
template <typename T>
__device__ __forceinline__ void fine_runs(const T* __restrict__ bra, const T* __restrict__ ket,
                                          int a, int b, int n, double& acc) {
  constexpr int R = 4;   // runs under way
  const int lane = threadIdx.x & 63;
  uint64_t m = __ballot(n > 0);
  while (m) {
    int l[R];
    const T *pa[R], *pk[R];
    T va[R], vk[R];
#pragma unroll
    for (int u = 0; u < R; ++u) {
      const int q = m ? __builtin_ctzll(m) : 0;
      l[u] = m ? __builtin_amdgcn_readlane(n, q) : 0;
      pa[u] = bra + __builtin_amdgcn_readlane(a, q);
      pk[u] = ket + __builtin_amdgcn_readlane(b, q);
      m &= m - 1;
      va[u] = vk[u] = T(0);
      if (lane < l[u]) {
        va[u] = pa[u][lane];
        vk[u] = pk[u][lane];
      }
    }
#pragma unroll
    for (int u = 0; u < R; ++u) acc += (double)va[u] * (double)vk[u];
#pragma unroll
    for (int u = 0; u < R; ++u)
      for (int x = lane + 64; x < l[u]; x += 64) acc += (double)pa[u][x] * (double)pk[u][x];
  }
}

template <typename T, int W>
__global__ __launch_bounds__(64 * W, 8) void k_sparse_values(const SfDev* __restrict__ sfs,
                                                      const wvl_seg* __restrict__ seg,
                                                      const int32_t* __restrict__ rt,
                                                      const RowRun* __restrict__ rr, int ket_out,
                                                      const T* __restrict__ bra,
                                                      const T* __restrict__ ket,
                                                      const int32_t* __restrict__ rowi,
                                                      const int32_t* __restrict__ coli,
                                                      const int32_t* __restrict__ order,
                                                      const int32_t* __restrict__ mirror,
                                                      int64_t nnz, double* __restrict__ val) {
  // coarse runs of a wave's rows: starts (bra, ket), lengths (0: none)
  __shared__ int32_t ea_[W][64], eb_[W][64], el_[W][64];
  // A batch of 64 rows adds to one of eight sums per lane, batch b to b mod 8,
  // whatever the number of waves: a pair has the same bits in every plan.
  __shared__ double lanes[512];
  // Workgroups are dealt to the 8 XCDs in turn: block b runs on XCD b % 8.
  // Each XCD walks its own contiguous eighth of the processing order, so the
  // pairs resident on one XCD share rows (and, rows being in spatial order,
  // most of their kets) in that XCD's L2.
  const int64_t per = (nnz + 7) / 8;
  const int64_t s = (int64_t)(blockIdx.x % 8) * per + blockIdx.x / 8;
  if (s >= nnz) return;
  const int64_t k = order[s];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int32_t *const ea = ea_[wv], *const eb = eb_[wv], *const el = el_[wv];
  const int grp = lane >> 4, gl = lane & 15;
  const SfDev& A = sfs[rowi[k]];
  const SfDev& B = sfs[coli[k]];
  const int32_t* bb = ket_out ? B.bb_out : B.bb_in;
  const int y0 = max(A.bb_in[2], bb[2]), y1 = min(A.bb_in[3], bb[3]);
  const int z0 = max(A.bb_in[4], bb[4]), z1 = min(A.bb_in[5], bb[5]);
  const PatBox pb = pat_box(B, ket_out);
  const int pc = ket_out ? 2 : 0, pf = ket_out ? 3 : 1;
  const T* const pbra = bra + A.cin;
  const T* const pket = ket + (ket_out ? B.cout : B.cin);
  const int bnc = (int)(ket_out ? B.on_c : B.n_c);
  const int ny = y1 - y0 + 1;
  const int nrows = (y1 >= y0 && z1 >= z0) ? ny * (z1 - z0 + 1) : 0;
  double acc = 0.0;
  for (int r0 = 64 * wv; r0 < nrows; r0 += 64 * W) {
    acc = 0.0;
    // phase 1
    const int r = r0 + lane;
    const bool in = r < nrows;
    const int y = y0 + (in ? r : 0) % ny, z = z0 + (in ? r : 0) / ny;
    const int64_t ra = (int64_t)(z - A.lo[2]) * A.n[1] + (y - A.lo[1]);
    const int64_t rb = (int64_t)(z - pb.oz) * pb.by + (y - pb.oy);
    // compact row runs: one 8-byte record per row, kind and side
    RowRun wa[2], wb[2];
#pragma unroll
    for (int fine = 0; fine < 2; ++fine) {
      wa[fine] = wb[fine] = RowRun{0, 0, 0};
      if (in) {
        wa[fine] = rr[A.rr[fine] + ra];
        wb[fine] = rr[B.rr[fine ? pf : pc] + rb];
      }
    }
    // coarse, fine and second run, from the functions' first coefficients
    int sa0[3] = {0, 0, 0}, sb0[3] = {0, 0, 0}, len[3] = {0, 0, 0};
#pragma unroll
    for (int fine = 0; fine < 2; ++fine) {
      if (wa[fine].len == 0 || wb[fine].len == 0) continue;
      // fine points hold their seven wavelets contiguously
      const int sc = fine ? 7 : 1;
      const int ba = fine ? (int)A.n_c : 0, bk = fine ? bnc : 0;
      if (wa[fine].len != kMultiRun && wb[fine].len != kMultiRun) {
        const int x0 = max((int)wa[fine].x0, (int)wb[fine].x0);
        const int x1 = min((int)wa[fine].x0 + wa[fine].len, (int)wb[fine].x0 + wb[fine].len) - 1;
        if (x0 <= x1) {
          sa0[fine] = ba + sc * (wa[fine].off + (x0 - wa[fine].x0));
          sb0[fine] = bk + sc * (wb[fine].off + (x0 - wb[fine].x0));
          len[fine] = sc * (x1 - x0 + 1);
        }
        continue;
      }
      // a row with several runs on either side: merge the segment lists
      int qa = rt[A.rt[fine] + ra];
      const int qa1 = rt[A.rt[fine] + ra + 1];
      int qb = rt[B.rt[fine ? pf : pc] + rb];
      const int qb1 = rt[B.rt[fine ? pf : pc] + rb + 1];
      while (qa < qa1 && qb < qb1) {
        const wvl_seg sa = seg[qa], sb = seg[qb];
        const int x0 = max(sa.i1s, sb.i1s), x1 = min(sa.i1e, sb.i1e);
        if (x0 <= x1) {
          const int oa = ba + sc * (sa.off + (x0 - sa.i1s));
          const int ob = bk + sc * (sb.off + (x0 - sb.i1s));
          const int n = sc * (x1 - x0 + 1);
          if (len[fine] == 0) {
            sa0[fine] = oa;
            sb0[fine] = ob;
            len[fine] = n;
          } else if (len[2] == 0) {
            sa0[2] = oa;
            sb0[2] = ob;
            len[2] = n;
          } else {
            acc += run_dot<T>(pbra + oa, pket + ob, n);
          }
        }
        if (sa.i1e < sb.i1e) ++qa; else ++qb;
      }
    }
    ea[lane] = sa0[0];
    eb[lane] = sb0[0];
    el[lane] = len[0];
    wave_sync();
    // phase 2, coarse runs
    const int nb = min(64, nrows - r0);
    constexpr int R = 4;   // rows under way
    for (int q0 = grp; q0 < nb; q0 += 4 * R) {
      T va[R], vk[R];
      int l[R];
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const int q = min(q0 + 4 * u, 63);
        l[u] = q0 + 4 * u < nb ? el[q] : 0;
        va[u] = vk[u] = T(0);
        if (gl < l[u]) {
          va[u] = pbra[ea[q] + gl];
          vk[u] = pket[eb[q] + gl];
        }
      }
#pragma unroll
      for (int u = 0; u < R; ++u) {
        acc += (double)va[u] * (double)vk[u];
        for (int x = gl + 16; x < l[u]; x += 16) {
          const int q = q0 + 4 * u;
          acc += (double)pbra[ea[q] + x] * (double)pket[eb[q] + x];
        }
      }
    }
    // fine runs, then the second runs: the whole wave takes a run
    fine_runs<T>(pbra, pket, sa0[1], sb0[1], len[1], acc);
    fine_runs<T>(pbra, pket, sa0[2], sb0[2], len[2], acc);
    wave_sync();
    if (r0 >= 512) acc += lanes[(r0 & 448) + lane];
    if (nrows > 64) lanes[(r0 & 448) + lane] = acc;
  }
  if (W > 1 && nrows > 64) __syncthreads();
  if (wv == 0) {
    if (nrows > 64) {
      acc = 0.0;
#pragma unroll
      for (int q = 0; q < 512; q += 64) acc += q < nrows ? lanes[q + lane] : 0.0;
    }
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) {
      val[k] = acc;
      if (mirror != nullptr && mirror[s] >= 0) val[mirror[s]] = acc;
    }
  }
}

// ---------------------------------------------------------------------------
// density rho(r) = sum_ab phi_a(r) K^ab phi_b(r) on the fine grid
// ---------------------------------------------------------------------------
// One workgroup per tile of 16 x 4 x 4 fine-grid points; a wave takes the
// 16 points along x of a (y, z).  The functions whose fine box meets the tile
// (its cover, increasing index) are taken in chunks of C, and the chunk pairs
// I <= J one after the other:
//   K block   the rows of both chunks are scanned (a wave per row, the next 256
//             entries loaded meanwhile) for columns in the pair's chunks (an
//             LDS hash), and the entries added into a dense block,
//             T[i][j] = K_ij + K_ji for i < j (i in I, j in J) and K_ii on the
//             diagonal: the density needs no more;
//   product   U_i(r) = sum_j T_ij phi_j(r) on the FP64 matrix cores
//             (16x16x4: 16 functions i x 16 points), the blocks below the
//             diagonal left out, and rho(r) += sum_i phi_i(r) U_i(r).
// Lane 16 g + n holds phi at point n of the functions 4 s + g of both chunks
// in registers: these are the product's operands as they stand, and the
// product's result has its rows in the same lanes.  The order of every sum is
// fixed by the tile's cover and K.  Columns outside [0, nsf) never match;
// positions outside [0, knnz) are skipped.  Values that are not finite enter the
// sums of the entries that name them only: a function that no entry of a pair
// names is left out of it, and where a sum is not finite all the same it is
// formed again entry by entry.
// 16 x 4 x 4 points: the rows of K are scanned once per tile and pair, the
// products cost m^2 / 2 multiply-adds per point for a cover of m (up to 340
// functions of radius 5-7 bohr at 0.037 per bohr^3, 37 in the middle of all
// tiles).  1,000 such functions in FP32: 16.8 ms with 16 x 4 x 1 points and the
// sums on the vector units; 8.0 ms in this form, of which the products take
// 2.7 (1.6 at the full FP64 matrix rate), the scans 2.5 and the values 1.0; 7.5
// with the tiles of the most chunks first, as long ones are not left for the end
// (400 functions of 6-7 bohr at 0.5 per bohr^3: 8.6 and 6.2 ms).
// Tiles of 16 x 4 x 2 points (two blocks per CU) took 9.6 ms, chunks of 128
// functions 9.4 (spilled registers).
// C: functions per chunk.  64: both chunks' values at a wave's points fit its
// registers.  kDensLight, for the tiles that at most so many functions meet: a
// third of the LDS and half of the registers, so that two blocks share a CU and
// the steps of one, of which there are as many for a few functions as for 64, are
// covered by the other's (same sums, same bits).  FP32, with blocks of K without an
// entry left out: 30 functions 0.28 -> 0.17 ms, one 0.117 -> 0.081 (an empty grid
// for the most part), a diagonal K of 1,000 6.8 -> 4.5.
constexpr int kDensChunk = 64;
constexpr int kDensThreads = 64 * 4 * kDensTile[2];
template <typename T, int C>
__global__ __launch_bounds__(kDensThreads, C == kDensLight ? 8 : 4) void k_dens_tile(
    const SfDev* __restrict__ sfs, const int64_t* __restrict__ foff, const T* __restrict__ fine,
    const int64_t* __restrict__ krow, const int32_t* __restrict__ kcol,
    const double* __restrict__ kval, int64_t knnz, const DensTile* __restrict__ tiles,
    const int32_t* __restrict__ csf, int nsf, int tx, int ty, int g0, int g1, int g2,
    T* __restrict__ rho) {
  constexpr int U = C == kDensLight ? 1 : 4;   // runs of 64 entries of K under way
  // blocks of 16 x 16 without an entry are left out (FP64 has no registers for it)
  constexpr bool kSkip = sizeof(T) == 4;
  constexpr int S = C / 4, LD = C + 4, NT = kDensThreads, NW = NT / 64;   // T's rows 4 (mod 16) apart: banks
  // hash of a pair's functions: at most 2 C in 32 C slots (function << 8 |
  // position), open addressing, so that one read settles most lookups
  constexpr int kDensSlots = 32 * C;
  auto dens_slot = [](int b) { return (int)(((uint64_t)((uint32_t)b * 2654435761u) * kDensSlots) >> 32); };
  typedef double V __attribute__((ext_vector_type(4)));
  // T: entries of the rows i, and of the rows j (each element then has one
  // wave that adds to it, so duplicated entries add up in their order)
  __shared__ __align__(16) double tk[2][C * LD];
  __shared__ uint32_t hslot[kDensSlots];
  // the pair's functions (I's, then J's): index, geometry on the fine grid
  // (origin, extents), first fine value, row of K
  __shared__ int32_t cov[2 * C];
  __shared__ int32_t geo[2 * C][6];
  __shared__ int64_t fo[2 * C], kq[2 * C];
  __shared__ int32_t kl[2 * C];
  __shared__ uint8_t used[2][C];      // the function has an entry in the pair's block
  __shared__ uint8_t blk[64];         // 16 x 16 blocks of T that hold entries
  static_assert(C <= 64, "a lane per function of a chunk");
  const DensTile dt = tiles[blockIdx.x];
  const int tile = dt.tile, m = dt.m;
  const int64_t c0 = dt.c0;
  const int ix = tile % tx, iy = (tile / tx) % ty, iz = tile / (tx * ty);
  const int tid = threadIdx.x, lane = tid & 63, n = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int gx = ix * kDensTile[0] + n;
  const int gy = iy * kDensTile[1] + (wave & 3);
  const int gz = iz * kDensTile[2] + (wave >> 2);
  const bool inside = gx < g0 && gy < g1 && gz < g2;
  if (m == 0) {   // uniform over the block
    if (inside && g == 0) rho[((int64_t)gz * g1 + gy) * g0 + gx] = T(0);
    return;
  }
  double acc = 0.0;
  T pi[S], pj[S];
  // stages a chunk's functions at half C (a barrier before and after)
  auto stage = [&](int half, int at, int cnt) {
    __syncthreads();   // the chunk before is no longer read
    if (tid < cnt) {
      const int h = half * C + tid;
      const int a = csf[c0 + at + tid];
      const SfDev& A = sfs[a];
      cov[h] = a;
      fo[h] = foff[a];
      const int64_t q0 = max((int64_t)0, krow[a]), q1 = min(knnz, krow[a + 1]);
      kq[h] = q0;
      kl[h] = (int)min(max((int64_t)0, q1 - q0), (int64_t)INT32_MAX);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        geo[h][d] = 2 * A.lo[d];
        geo[h][3 + d] = 2 * A.n[d] + 29;
      }
    }
    __syncthreads();
  };
  auto values = [&](int half, int cnt, T (&v)[S]) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      v[s] = T(0);
      if (4 * s >= cnt) continue;
      const int h = half * C + min(4 * s + g, cnt - 1);
      const int px = gx - geo[h][0], py = gy - geo[h][1], pz = gz - geo[h][2];
      const int R0 = geo[h][3], R1 = geo[h][4], R2 = geo[h][5];
      if (4 * s + g < cnt && inside && (uint32_t)px < (uint32_t)R0 &&
          (uint32_t)py < (uint32_t)R1 && (uint32_t)pz < (uint32_t)R2)
        v[s] = fine[fo[h] + ((int64_t)pz * R1 + py) * R0 + px];
      if (s % 2 == 1) __builtin_amdgcn_sched_barrier(0);   // few addresses at a time
    }
  };
  // The pair's sum at the lane's point again, over the entries of T alone (a
  // product with the other elements is zero times an infinity), where the
  // products gave one that is not finite.  Functions that do not meet the
  // tile's 16 x 4 x 1 points of this plane are left out, as their zeros are no
  // values of theirs.
  auto entries_only = [&](int jh, int ni, int nj) {
    auto meets = [&](int h) {
      const int x = ix * kDensTile[0] - geo[h][0], y = iy * kDensTile[1] - geo[h][1];
      return x > -kDensTile[0] && x < geo[h][3] && y > -kDensTile[1] && y < geo[h][4] &&
             gz >= geo[h][2] && gz < geo[h][2] + geo[h][5];
    };
    auto value = [&](int h) -> double {
      const int px = gx - geo[h][0], py = gy - geo[h][1], pz = gz - geo[h][2];
      const int R0 = geo[h][3], R1 = geo[h][4], R2 = geo[h][5];
      if (!inside || (uint32_t)px >= (uint32_t)R0 || (uint32_t)py >= (uint32_t)R1 ||
          (uint32_t)pz >= (uint32_t)R2)
        return 0.0;
      return (double)fine[fo[h] + ((int64_t)pz * R1 + py) * R0 + px];
    };
    double again = 0.0;
#pragma unroll 1
    for (int i = g; i < ni; i += 4) {   // the lane's rows
      if (!meets(i)) continue;
      double u = 0.0;
      bool any = false;
#pragma unroll 1
      for (int j = 0; j < nj; ++j) {
        const double t = tk[0][i * LD + j];
        if (t == 0.0 && __builtin_signbit(t)) continue;   // no entry
        if (!meets(jh * C + j)) continue;
        u += t * value(jh * C + j);
        any = true;
      }
      if (any) again += value(i) * u;
    }
    return again;
  };
  for (int ic = 0; ic < m; ic += C) {
    const int ni = min(C, m - ic);
    stage(0, ic, ni);
    values(0, ni, pi);
    for (int jc = ic; jc < m; jc += C) {
      const bool diag = jc == ic;
      const int nj = min(C, m - jc);
      const int jh = diag ? 0 : 1;
      if (!diag) {
        stage(1, jc, nj);
        values(1, nj, pj);
      } else {
#pragma unroll
        for (int s = 0; s < S; ++s) pj[s] = pi[s];
      }
      // the wave's rows to scan (I's, then J's), i = wave, wave + NW, ..: 64 U
      // entries at a time, the next ones loaded while these are looked up
      const int nrow = ni + (diag ? 0 : nj);
      int si = wave, sq = 0;   // the next row and its first entry
      auto slot = [&](int i) { return i < ni ? i : C + i - ni; };
      int b[U], bn[U], pa = 0, pan = 0;
      double kb[U], kn[U];
      auto fetch = [&](int (&bb)[U], double (&kk)[U], int& row) {
        row = -1;
#pragma unroll
        for (int u = 0; u < U; ++u) bb[u] = -1;
        while (si < nrow && sq >= kl[slot(si)]) {
          si += NW;
          sq = 0;
        }
        if (si >= nrow) return;
        row = slot(si);
        const int64_t q = kq[row] + sq;
        const int left = kl[row] - sq;
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (64 * u + lane < left) {
            bb[u] = kcol[q + 64 * u + lane];
            kk[u] = kval[q + 64 * u + lane];
          }
        sq += 64 * U;
      };
      fetch(b, kb, pa);
      // hash of the pair's functions and an empty T: -0 where there is no entry
      // (entries are added as kb + 0, never -0, so that a sum is never -0 either)
      for (int h = tid; h < kDensSlots; h += NT) hslot[h] = 0xFFFFFFFFu;
      if (tid < 2 * C) used[tid / C][tid % C] = 0;
      if (kSkip && tid < 64) blk[tid] = 0;
      const int nr = (ni + 15) & ~15;
      for (int h = tid; h < nr * (LD / 2); h += NT)
        reinterpret_cast<double2*>(tk[0])[h] = reinterpret_cast<double2*>(tk[1])[h] =
            make_double2(-0.0, -0.0);
      __syncthreads();
      if (tid < nrow) {
        const int h = slot(tid);
        const uint32_t key = ((uint32_t)cov[h] << 8) | (uint32_t)h;
        int at = dens_slot(cov[h]);
        while (atomicCAS(&hslot[at], 0xFFFFFFFFu, key) != 0xFFFFFFFFu) at = (at + 1) & (kDensSlots - 1);
      }
      __syncthreads();
      while (pa >= 0) {   // uniform over the wave
        fetch(bn, kn, pan);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (b[u] < 0 || b[u] >= nsf) continue;
          int at = dens_slot(b[u]);
          uint32_t v = hslot[at];
          while (v != 0xFFFFFFFFu && (v >> 8) != (uint32_t)b[u]) {
            at = (at + 1) & (kDensSlots - 1);
            v = hslot[at];
          }
          const int p = v == 0xFFFFFFFFu ? -1 : (int)(v & 255u);
          // an entry inside one chunk belongs to its diagonal pair
          if (p < 0 || (!diag && (p >= C) == (pa >= C))) continue;
          const int r = min(pa, p), c = max(pa, p) - (diag ? 0 : C);   // row in I, column in J
          unsafeAtomicAdd(&tk[pa > p][r * LD + c], kb[u] + 0.0);
          used[0][r] = 1;
          used[jh][c] = 1;
        }
        pa = pan;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          b[u] = bn[u];
          kb[u] = kn[u];
        }
      }
      __syncthreads();
      for (int h = tid; h < nr * (LD / 2); h += NT) {
        double2& t = reinterpret_cast<double2*>(tk[0])[h];
        const double2 v = reinterpret_cast<double2*>(tk[1])[h];
        t.x += v.x;
        t.y += v.y;
        if (kSkip && (!(__builtin_signbit(t.x) && t.x == 0.0) || !(__builtin_signbit(t.y) && t.y == 0.0)))
          blk[(h / (LD / 2) >> 4) * 4 + (2 * (h % (LD / 2)) >> 4)] = 1;
      }
      __syncthreads();
      // bit 4 s: function 4 s + g has an entry
      const uint64_t ui = __ballot(lane < C && used[0][lane % C]) >> g,
                     uj = __ballot(lane < C && used[jh][lane % C]) >> g;
      const uint64_t ub = kSkip ? __ballot(blk[lane]) : ~0ull;
#pragma unroll
      for (int s = 0; s < S; ++s) pj[s] = (uj >> (4 * s)) & 1u ? pj[s] : T(0);
      const double* const ta = tk[0] + n * LD + g;
      const double before = acc;
#pragma unroll
      for (int st = 0; st < C / 16; ++st) {
        if (16 * st >= ni || !((ub >> (4 * st)) & 15u)) continue;
        V d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int cb = 0; cb < C / 16; ++cb) {
          if (16 * cb >= nj || (diag && cb < st) || !((ub >> (4 * st + cb)) & 1u)) continue;
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int s = 4 * cb; s < 4 * cb + 4; ++s) {
            d = __builtin_amdgcn_mfma_f64_16x16x4f64(ta[16 * st * LD + 4 * s], (double)pj[s], d, 0,
                                                     0, 0);
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc += (ui >> (4 * (4 * st + j))) & 1u ? (double)pi[4 * st + j] * d[j] : 0.0;
      }
      if (__builtin_expect(__any(!__builtin_isfinite(acc)), 0)) {
        const double again = before + entries_only(jh, ni, nj);
        if (!__builtin_isfinite(acc)) acc = again;
      }
      __syncthreads();   // T, the hash and the flags no longer read
    }
  }
  acc += __shfl_xor(acc, 16, 64);
  acc += __shfl_xor(acc, 32, 64);
  if (inside && g == 0) rho[((int64_t)gz * g1 + gy) * g0 + gx] = (T)acc;
}

// ---------------------------------------------------------------------------
// Fermi operator expansion: matrices on one symmetric pattern P (CSR, sorted
// columns, diagonal present), values in double
// ---------------------------------------------------------------------------

// C = alpha (A B)|_P + beta D, one workgroup of W waves per row i of P,
// rows taken in the order `rows` gives (longest work first).  Row i's
// columns go into an LDS hash table of 2^lognb buckets of four 32-bit slots,
// each slot (column << 10 | position in the row); a bucket fills from its
// first slot, and a full one spills into the next.  Wave w takes the k of
// row i with index t = w, w + W, .. in increasing order; its lanes walk row
// k of B in parts of 256 / NH entries, NH parts a step, and add A_ik B_kj to
// the wave's accumulator of that part's slot when j is in row i.  The next
// step's entries of B are loaded while the current ones are added.  The
// accumulators are summed in (wave, slot) order at the end, so every entry's
// sum has a fixed order.  D may be NULL
// (beta ignored).  Needs columns below 2^21 and rows of at most 1024
// entries; LDS: W NH + 2 doubles per row entry (maxdeg) and 16 bytes per
// bucket.
constexpr uint32_t kFoeEmpty = 0xFFFFFFFFu;

__device__ __forceinline__ int foe_bucket(int j, int lognb) {
  return (int)(((uint32_t)j * 2654435761u) >> (32 - lognb));
}

// position of column j in a bucket, or -1
__device__ __forceinline__ int foe_match(uint4 v, int j) {
  const uint32_t uj = (uint32_t)j;
  int p = -1;
  if ((v.x >> 10) == uj) p = (int)(v.x & 1023u);
  if ((v.y >> 10) == uj) p = (int)(v.y & 1023u);
  if ((v.z >> 10) == uj) p = (int)(v.z & 1023u);
  if ((v.w >> 10) == uj) p = (int)(v.w & 1023u);
  return p;
}

template <int W, int NH>
__global__ __launch_bounds__(64 * W) void k_foe_mm(
    const int32_t* __restrict__ rows, const int64_t* __restrict__ rowptr,
    const int32_t* __restrict__ col, double alpha,
    const double* __restrict__ A, const double* __restrict__ B, double beta,
    const double* __restrict__ D, double* __restrict__ C, int lognb, int maxdeg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* acc = reinterpret_cast<double*>(smem_raw);   // [W][NH][maxdeg]
  double* av = acc + (size_t)W * NH * maxdeg;           // A_ik, [maxdeg]
  int* kst = reinterpret_cast<int*>(av + maxdeg);       // start of row k in B
  int* kdg = kst + maxdeg;                              // length of row k
  uint4* bucket = reinterpret_cast<uint4*>(kdg + maxdeg);   // [nb]
  uint32_t* slot = reinterpret_cast<uint32_t*>(bucket);
  constexpr int nt = 64 * W;
  constexpr int QW = 256 / NH;   // entries of a row k per part
  constexpr int UH = 4 / NH;     // 64-lane slots per part
  const int nb = 1 << lognb;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = rows[blockIdx.x];
  const int64_t r0 = rowptr[i];
  const int deg = (int)(rowptr[i + 1] - r0);
  for (int h = tid; h < 4 * nb; h += nt) slot[h] = kFoeEmpty;
  for (int p = tid; p < deg; p += nt) {
    const int k = col[r0 + p];
    const int64_t k0 = rowptr[k];
    kst[p] = (int)k0;
    kdg[p] = (int)(rowptr[k + 1] - k0);
    av[p] = A[r0 + p];
#pragma unroll
    for (int w = 0; w < W * NH; ++w) acc[(size_t)w * maxdeg + p] = 0.0;
  }
  __syncthreads();
  // 4 nb slots > deg: every insertion finds a free slot, every lookup a
  // bucket that is not full
  for (int p = tid; p < deg; p += nt) {
    const int j = col[r0 + p];
    const uint32_t key = ((uint32_t)j << 10) | (uint32_t)p;
    for (int b = foe_bucket(j, lognb);; b = (b + 1) & (nb - 1)) {
      int c = 0;
      while (c < 4 && atomicCAS(&slot[4 * b + c], kFoeEmpty, key) != kFoeEmpty) ++c;
      if (c < 4) break;
    }
  }
  __syncthreads();
  double* my = acc + (size_t)wave * NH * maxdeg;   // the wave's NH accumulators
  // the wave's parts in order: (t, q0) for t = wave, wave + W, .. and
  // q0 = 0, QW, .. below the length of row k; a step takes NH parts, part h
  // on the 64-lane slots h UH .. h UH + UH - 1 and into accumulator h
  int qt = wave, qq = 0;
  auto next = [&](int& k0, int& kd, int& q0, double& a) {
    if (qt >= deg) {
      k0 = 0;
      kd = 0;
      q0 = 0;
      a = 0.0;
      return;
    }
    k0 = kst[qt];
    kd = kdg[qt];
    q0 = qq;
    a = av[qt];
    qq += QW;
    if (qq >= kd) {
      qt += W;
      qq = 0;
    }
  };
  // column -1: none
  auto load = [&](const int (&k0)[NH], const int (&kd)[NH], const int (&q0)[NH], int (&jj)[4],
                  double (&bb)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int h = u / UH;
      const int q = q0[h] + 64 * (u % UH) + lane;
      jj[u] = q < kd[h] ? col[k0[h] + q] : -1;
      bb[u] = q < kd[h] ? B[k0[h] + q] : 0.0;
    }
  };
  // the four lookups, the four accumulator reads and the four writes are
  // issued together: within a part the columns (one row of B) are distinct,
  // and parts add into accumulators of their own
  auto add = [&](const int (&jj)[4], const double (&bb)[4], const double (&a)[NH]) {
    int b[4];
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      b[u] = foe_bucket(jj[u], lognb);
      v[u] = bucket[b[u]];
    }
    int p[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      p[u] = foe_match(v[u], jj[u]);
      while (p[u] < 0 && jj[u] >= 0 && v[u].w != kFoeEmpty) {
        b[u] = (b[u] + 1) & (nb - 1);
        v[u] = bucket[b[u]];
        p[u] = foe_match(v[u], jj[u]);
      }
    }
    double o[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = my[(size_t)(u / UH) * maxdeg + (p[u] >= 0 ? p[u] : 0)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (p[u] >= 0) my[(size_t)(u / UH) * maxdeg + p[u]] = o[u] + a[u / UH] * bb[u];
  };
  int steps = 0;
  for (int t = wave; t < deg; t += W) steps += (kdg[t] + QW - 1) / QW;
  steps = (steps + NH - 1) / NH;
  int k0[NH], kd[NH], q0[NH];
  double a[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) next(k0[h], kd[h], q0[h], a[h]);
  int jj[4];
  double bb[4];
  load(k0, kd, q0, jj, bb);
  // the next step's entries of B load while the current ones are added
  for (; steps > 0; --steps) {
    double an[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) next(k0[h], kd[h], q0[h], an[h]);
    int jn[4];
    double bn[4];
    load(k0, kd, q0, jn, bn);
    add(jj, bb, a);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      jj[u] = jn[u];
      bb[u] = bn[u];
    }
#pragma unroll
    for (int h = 0; h < NH; ++h) a[h] = an[h];
  }
  __syncthreads();
  for (int p = tid; p < deg; p += nt) {
    double v = acc[p];
#pragma unroll
    for (int w = 1; w < W * NH; ++w) v += acc[(size_t)w * maxdeg + p];
    C[r0 + p] = D ? alpha * v + beta * D[r0 + p] : alpha * v;
  }
}

// C = alpha (R A)|_P + beta D for a symmetric A on P (tpos: stored transposed,
// without D): a workgroup takes row r of P (longest work first), row r of R
// spread out in LDS (n doubles, zeros elsewhere); a group of 16 lanes takes an
// entry c of the row and adds up R_rk A_ck over row c of A, so that an entry costs
// one LDS read and no lookup.  Twelve loads of a row under way per lane cover the
// usual rows with one latency; the lanes' sums are added in a fixed tree.  Bound
// by the reads of A through L2 (12 bytes per product).  1,000 functions with 163
// entries a row (27M products): 70 us with k_foe_mm, 43 here (256 threads and four
// loads: 54); 4,000 with 72 entries: 54 and 34 us.
// LOOP: a block takes several rows (see the launch): the n zeros are written once,
// and only a row's own entries cleared after it.  A row's run starts are read
// before the first barrier with one row per block, after it with several: the other
// way round costs 2 and 10 %.
constexpr int kRmulThreads = 512;
template <bool LOOP>
__global__ __launch_bounds__(kRmulThreads) void k_foe_rmul(
    const int32_t* __restrict__ rows, const int64_t* __restrict__ rowptr,
    const int32_t* __restrict__ col, int n, double alpha, const double* __restrict__ R,
    const double* __restrict__ A, double beta, const double* __restrict__ D,
    const int64_t* __restrict__ tpos, double* __restrict__ C, int maxdeg) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* const x = reinterpret_cast<double*>(smem_raw);   // [n]
  int* const kst = reinterpret_cast<int*>(x + n);           // start and length of the rows c
  int* const kdg = kst + maxdeg;
  const int tid = threadIdx.x, l = tid & 15;
  for (int k = tid; k < n; k += kRmulThreads) x[k] = 0.0;
  for (int rq = blockIdx.x; rq < n; rq += gridDim.x) {
    const int i = rows[rq];
    const int64_t r0 = rowptr[i];
    const int deg = (int)(rowptr[i + 1] - r0);
    auto runs = [&](int p, int c) {
      const int64_t k0 = rowptr[c];
      kst[p] = (int)k0;
      kdg[p] = (int)(rowptr[c + 1] - k0);
    };
    if (!LOOP)   // meanwhile
      for (int p = tid; p < deg; p += kRmulThreads) runs(p, col[r0 + p]);
    __syncthreads();   // x is zero
    for (int p = tid; p < deg; p += kRmulThreads) {
      const int c = col[r0 + p];
      if (LOOP) runs(p, c);
      x[c] = R[r0 + p];
    }
    __syncthreads();
    for (int p = tid >> 4; p < deg; p += kRmulThreads / 16) {
      const int* const cc = col + kst[p];
      const double* const av = A + kst[p];
      const int kd = kdg[p];
      double s = 0.0;
      constexpr int U = 12;
      for (int q = l; q < kd; q += 16 * U) {
        int k[U];
        double a[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (q + 16 * u < kd) {
            k[u] = cc[q + 16 * u];
            a[u] = av[q + 16 * u];
          }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (q + 16 * u < kd) s += a[u] * x[k[u]];
      }
      for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
      if (l == 0) C[tpos ? tpos[r0 + p] : r0 + p] = D ? alpha * s + beta * D[r0 + p] : alpha * s;
    }
    if (!LOOP) return;
    if (rq + (int)gridDim.x < n) {
      __syncthreads();
      for (int p = tid; p < deg; p += kRmulThreads) x[col[r0 + p]] = 0.0;
    }
  }
}

// v = a x + b y (+ d on the diagonal), each term only when present; the one
// expression both k_foe_axpby and k_foe_series evaluate
__device__ __forceinline__ double foe_lin(bool hx, double a, double x, bool hy, double b,
                                          double y, bool diag, double d) {
  double v = 0.0;
  if (hx) v += a * x;
  if (hy) v += b * y;
  if (diag) v += d;
  return v;
}

// elementwise on P: out = a X + b Y (+ d on the diagonal when row != NULL)
__global__ __launch_bounds__(TPB) void k_foe_axpby(int64_t nnz, double a,
                                                   const double* __restrict__ X, double b,
                                                   const double* __restrict__ Y,
                                                   const int32_t* __restrict__ row,
                                                   const int32_t* __restrict__ col, double d,
                                                   double* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * TPB + threadIdx.x;
  if (p >= nnz) return;
  out[p] = foe_lin(X != nullptr, a, X ? X[p] : 0.0, Y != nullptr, b, Y ? Y[p] : 0.0,
                   row && row[p] == col[p], d);
}

// the Chebyshev series on P from the kept matrices T^0 .. T^npl (T^j at
// T + j nnz): out = c_0 / 2 I + c_1 T^1, then out += c_j T^j for j = 2 ..
// npl, term by term as k_foe_axpby adds them when the matrices are
// recomputed (same values, bit for bit)
__global__ __launch_bounds__(TPB) void k_foe_series(int64_t nnz, int npl,
                                                    const double* __restrict__ c,
                                                    const double* __restrict__ T,
                                                    const int32_t* __restrict__ row,
                                                    const int32_t* __restrict__ col,
                                                    double* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * TPB + threadIdx.x;
  if (p >= nnz) return;
  const bool diag = row[p] == col[p];
  double v = foe_lin(true, c[1], T[nnz + p], false, 0.0, 0.0, diag, 0.5 * c[0]);
  for (int j = 2; j <= npl; ++j)
    v = foe_lin(true, 1.0, v, true, c[j], T[(int64_t)j * nnz + p], diag, 0.0);
  out[p] = v;
}

// symmetric part on P: out = (X + X^T) / 2
__global__ __launch_bounds__(TPB) void k_foe_sym(int64_t nnz, const int64_t* __restrict__ tpos,
                                                 const double* __restrict__ X,
                                                 double* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * TPB + threadIdx.x;
  if (p >= nnz) return;
  out[p] = 0.5 * (X[p] + X[tpos[p]]);
}

// out = values of X (on pattern Q) at the positions qpos of P's entries
__global__ __launch_bounds__(TPB) void k_foe_gather(int64_t nnz, const int64_t* __restrict__ qpos,
                                                    const double* __restrict__ X,
                                                    double* __restrict__ out) {
  const int64_t p = (int64_t)blockIdx.x * TPB + threadIdx.x;
  if (p >= nnz) return;
  out[p] = X[qpos[p]];
}

// one block: out[slot] = sum_p X[p] Y[p] over P, in a fixed order
// block b of nblk: part[b] = sum of X[p] Y[p] over its contiguous chunk of
// the entries; then one block: out[slot] = part[0] + .. + part[nblk - 1]
// (both sums in fixed orders)
__global__ __launch_bounds__(TPB) void k_foe_dot(int64_t nnz, int64_t chunk,
                                                 const double* __restrict__ X,
                                                 const double* __restrict__ Y,
                                                 double* __restrict__ part) {
  const int64_t p0 = (int64_t)blockIdx.x * chunk;
  const int64_t p1 = min(nnz, p0 + chunk);
  double v = 0.0;
  for (int64_t p = p0 + threadIdx.x; p < p1; p += TPB) v += X[p] * Y[p];
  const double s = block_sum(v);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ __launch_bounds__(TPB) void k_foe_sum(int n, const double* __restrict__ part,
                                                 double* __restrict__ out, int slot) {
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += TPB) v += part[i];
  const double s = block_sum(v);
  if (threadIdx.x == 0) out[slot] = s;
}

// block b: out[slot + b] = trace of X + b stride, its diagonal entries at
// dpos[0..n), in a fixed order
__global__ __launch_bounds__(TPB) void k_foe_trace(int n, const int64_t* __restrict__ dpos,
                                                   const double* __restrict__ X, int64_t stride,
                                                   double* __restrict__ out, int slot) {
  const double* Xb = X + (int64_t)blockIdx.x * stride;
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += TPB) v += Xb[dpos[i]];
  const double s = block_sum(v);
  if (threadIdx.x == 0) out[slot + blockIdx.x] = s;
}

// Gershgorin discs of X: one wave per row i (four rows per block) sums
// r_i = sum_{j != i} |X_ij| over the lanes in a fixed tree and writes
// lo[i] = X_ii - r_i, hi[i] = X_ii + r_i
__global__ __launch_bounds__(TPB) void k_foe_gersh_rows(int nrow,
                                                        const int64_t* __restrict__ rowptr,
                                                        const int32_t* __restrict__ col,
                                                        const double* __restrict__ X,
                                                        double* __restrict__ lo,
                                                        double* __restrict__ hi) {
  const int i = blockIdx.x * (TPB / 64) + (int)(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (i >= nrow) return;
  double dgl = 0.0, r = 0.0;
  for (int64_t q = rowptr[i] + lane; q < rowptr[i + 1]; q += 64) {
    if (col[q] == i)
      dgl = X[q];
    else
      r += fabs(X[q]);
  }
  for (int o = 32; o > 0; o >>= 1) {
    r += __shfl_xor(r, o, 64);
    dgl += __shfl_xor(dgl, o, 64);   // one lane holds the diagonal, the others 0
  }
  if (lane == 0) {
    lo[i] = dgl - r;
    hi[i] = dgl + r;
  }
}

// one block: out[0] = min_i lo[i], out[1] = max_i hi[i]
__global__ __launch_bounds__(TPB) void k_foe_gersh(int nrow, const double* __restrict__ lo,
                                                   const double* __restrict__ hi,
                                                   double* __restrict__ out) {
  __shared__ double sl[TPB], sh[TPB];
  double l = 1e300, h = -1e300;
  for (int i = threadIdx.x; i < nrow; i += TPB) {
    l = fmin(l, lo[i]);
    h = fmax(h, hi[i]);
  }
  sl[threadIdx.x] = l;
  sh[threadIdx.x] = h;
  __syncthreads();
  for (int s = TPB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      sl[threadIdx.x] = fmin(sl[threadIdx.x], sl[threadIdx.x + s]);
      sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    out[0] = sl[0];
    out[1] = sh[0];
  }
}

// ---------------------------------------------------------------------------
// support-function update: psi <- psi - eta (P_L hpsi - H_aa psi)
// ---------------------------------------------------------------------------
// Block = 64 consecutive input segments of one function (coarse blocks, then
// fine).  Every input segment lies inside one maximal output segment (the
// input pattern is contained in the output pattern), so each segment maps
// affinely into H psi; the map is found once per segment and staged in LDS.
constexpr int kUpdSegs = 64;
// mode 0 (update):   psi <- psi - eta (P_L hpsi - H_aa psi)      (out = psi)
// mode 1 (restrict): out <- P_L hpsi - min(shift_a, 0) psi
template <typename T>
__global__ __launch_bounds__(256) void k_update(const SfDev* __restrict__ sfs,
                                                const wvl_seg* __restrict__ seg,
                                                const int32_t* __restrict__ rt, double eta,
                                                const T* __restrict__ hpsi,
                                                const int64_t* __restrict__ hrow,
                                                const int32_t* __restrict__ hcol,
                                                const double* __restrict__ hval,
                                                T* __restrict__ psi, int sf0, int mode,
                                                const double* __restrict__ shift,
                                                T* __restrict__ out) {
  __shared__ int s_in[kUpdSegs + 1];     // coefficient offset relative to the first segment
  __shared__ int64_t s_out[kUpdSegs];    // H psi index of the segment's first point
  __shared__ double s_diag;
  const int a = sf0 + blockIdx.y;
  const SfDev& sf = sfs[a];
  const int64_t nrows = (int64_t)sf.n[1] * sf.n[2];
  const int cb0 = rt[sf.rt[0]], ce0 = rt[sf.rt[0] + nrows];
  const int fb0 = rt[sf.rt[1]], fe0 = rt[sf.rt[1] + nrows];
  const int nbc = (ce0 - cb0 + kUpdSegs - 1) / kUpdSegs;
  const int nbf = (fe0 - fb0 + kUpdSegs - 1) / kUpdSegs;
  int bx = blockIdx.x;
  const bool fine = bx >= nbc;
  if (fine) bx -= nbc;
  if (bx >= (fine ? nbf : nbc)) return;   // uniform over the block
  const int sA = (fine ? fb0 : cb0) + bx * kUpdSegs;
  const int nseg = min(kUpdSegs, (fine ? fe0 : ce0) - sA);
  const int tid = threadIdx.x;
  const int64_t off0 = seg[sA].off;
  const PatBox ob = pat_box(sf, 1);
  if (tid < nseg) {
    const wvl_seg g = seg[sA + tid];
    s_in[tid] = (int)(g.off - off0);
    if (tid == nseg - 1) s_in[nseg] = (int)(g.off - off0) + (g.i1e - g.i1s + 1);
    const int64_t r = (int64_t)(g.i3 - ob.oz) * ob.by + (g.i2 - ob.oy);
    const int pat = fine ? 3 : 2;
    int64_t o = -1;
    for (int q = rt[sf.rt[pat] + r]; q < rt[sf.rt[pat] + r + 1]; ++q) {
      const wvl_seg h = seg[q];
      if (g.i1s >= h.i1s && g.i1s <= h.i1e) {
        o = h.off + (g.i1s - h.i1s);
        break;
      }
    }
    s_out[tid] = o;   // always found: the plan checks input inside output
  }
  if (tid == 0) {
    if (mode == 0) {  // H_aa: the diagonal entry of row a
      int64_t lo = hrow[a], hi = hrow[a + 1] - 1;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (hcol[mid] < a) lo = mid + 1; else hi = mid;
      }
      s_diag = hval[lo];
    } else {
      s_diag = shift ? fmin(shift[a], 0.0) : 0.0;
    }
  }
  __syncthreads();
  const int total = s_in[nseg];
  const double d = s_diag;
  const int cfirst = fine ? 1 : 0, clast = fine ? 7 : 0;
  for (int k = tid; k < total; k += 256) {
    int lo = 0, hi = nseg - 1;   // last segment with s_in <= k
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_in[mid] <= k) lo = mid; else hi = mid - 1;
    }
    if (s_out[lo] < 0) continue;   // not reached: the host checks input inside output
    const int64_t oi = s_out[lo] + (k - s_in[lo]);
    for (int c = cfirst; c <= clast; ++c) {
      const int64_t i = sf.cin + (c == 0 ? off0 + k : sf.n_c + 7 * (off0 + k) + (c - 1));
      const int64_t o = sf.cout + (c == 0 ? oi : sf.on_c + 7 * oi + (c - 1));
      const double x = (double)psi[i];
      if (mode == 0)
        psi[i] = (T)(x - eta * ((double)hpsi[o] - d * x));
      else
        out[i] = (T)((double)hpsi[o] - d * x);
    }
  }
}

// ---------------------------------------------------------------------------
// per-function vector algebra for the preconditioner (input layout: each
// function's coefficients are contiguous); one block per function, fixed
// summation order
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(TPB) void k_sf_dot(const SfDev* __restrict__ sfs,
                                                const T* __restrict__ a,
                                                const T* __restrict__ b, double* __restrict__ out,
                                                int sf0) {
  const SfDev& sf = sfs[sf0 + blockIdx.x];
  const int64_t n = sf.n_c + 7 * sf.n_f;
  double v = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += TPB) v += (double)a[sf.cin + i] * (double)b[sf.cin + i];
  const double r = block_sum(v);
  if (threadIdx.x == 0) out[sf0 + blockIdx.x] = r;
}

// one conjugate-gradient step after Ap and pAp = <p|Ap> are known:
//   al = rr / pAp (0 when pAp <= 0 or rr = 0);  x += al p;  r -= al Ap
template <typename T>
__global__ __launch_bounds__(TPB) void k_cg_xr(const SfDev* __restrict__ sfs,
                                               const double* __restrict__ rr,
                                               const double* __restrict__ pap,
                                               const T* __restrict__ p, const T* __restrict__ ap,
                                               T* __restrict__ x, T* __restrict__ r, int sf0) {
  const int a = sf0 + blockIdx.x;
  const SfDev& sf = sfs[a];
  const double al = (pap[a] > 0.0 && rr[a] > 0.0) ? rr[a] / pap[a] : 0.0;
  const int64_t n = sf.n_c + 7 * sf.n_f;
  for (int64_t i = threadIdx.x; i < n; i += TPB) {
    const int64_t k = sf.cin + i;
    x[k] = (T)((double)x[k] + al * (double)p[k]);
    r[k] = (T)((double)r[k] - al * (double)ap[k]);
  }
}

//   be = rr_new / rr (0 when rr = 0);  p = r + be p;  rr <- rr_new
template <typename T>
__global__ __launch_bounds__(TPB) void k_cg_p(const SfDev* __restrict__ sfs,
                                              double* __restrict__ rr,
                                              const double* __restrict__ rr_new,
                                              const T* __restrict__ r, T* __restrict__ p,
                                              int sf0) {
  const int a = sf0 + blockIdx.x;
  const SfDev& sf = sfs[a];
  const double be = rr[a] > 0.0 ? rr_new[a] / rr[a] : 0.0;
  const int64_t n = sf.n_c + 7 * sf.n_f;
  for (int64_t i = threadIdx.x; i < n; i += TPB) {
    const int64_t k = sf.cin + i;
    p[k] = (T)((double)r[k] + be * (double)p[k]);
  }
  __syncthreads();
  if (threadIdx.x == 0) rr[a] = rr_new[a];
}

// x = 0, r = p = -g over every function's coefficients
template <typename T>
__global__ __launch_bounds__(TPB) void k_cg_init(const SfDev* __restrict__ sfs,
                                                 const T* __restrict__ g, T* __restrict__ x,
                                                 T* __restrict__ r, T* __restrict__ p, int sf0) {
  const SfDev& sf = sfs[sf0 + blockIdx.x];
  const int64_t n = sf.n_c + 7 * sf.n_f;
  for (int64_t i = threadIdx.x; i < n; i += TPB) {
    const int64_t k = sf.cin + i;
    x[k] = T(0);
    r[k] = -g[k];
    p[k] = -g[k];
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

// ---------------------------------------------------------------------------
// gradient: g_a = L^a [ sum_d A_ad H|phi_d> - sum_d M_ad |phi_d> ] over row a
// of the overlap pattern (Eq. (gradient), Sec. IV.A, localized as Sec. III.A)
// ---------------------------------------------------------------------------
// Block = part of function a's rows (four waves), the neighbours d of row a
// staged in LDS, kGradNb at a time.  A wave takes a row of a's input box; for
// each segment of it (the scaling coefficients of the coarse pattern, then the
// seven wavelets of each point of the fine pattern) it works in two phases per
// 64 neighbours.  Phase 1: lane t looks up neighbour t's runs in this row (one
// record each for H|phi_d> and |phi_d>; rows of several runs walk their
// segments) and the runs that meet the segment go to a list in LDS, in CSR
// order.  Phase 2: lane j owns the elements j, j + 64, ... and adds the listed
// runs' values at its points, in double and in list order, several runs' loads
// under way at a time.  Each element of g_a is written once, by its owner.
// Bound by the latency of phase 2's loads and by its vector instructions.
// 500 functions of radius 5-7 bohr at 0.037 per bohr^3, FP32: 69.0 ms with one
// lookup and one value at a time, each waited for; 6.1 ms with the lists and 8
// or 4 runs under way; 4.6 ms with neighbour records of 72 instead of 144 bytes
// (five blocks per CU by LDS), 16 runs and multiply-adds under the lane mask.
constexpr int kGradNb = 256;
constexpr int kGradCap = 128;     // list entries per wave: 64 neighbours, two runs each
constexpr int kGradParts = 8;     // blocks per function (and rows 4 kGradParts apart per wave)

// a neighbour: its input box rows (origin, rows per plane, planes; the output
// box is ext wider on each side), the records of its input rows (those of the
// other patterns follow), its first coefficients, A_ad and M_ad
struct GradNb {
  int32_t y0, z0, by, nz, e, id;
  int32_t n_c, on_c;
  int64_t rr, cin, cout;
  double a, m;
};
static_assert(sizeof(GradNb) == 72);
// a run of |phi_d> or H|phi_d> in the row: points x0 .. x1, the value of
// component comp at p[per x + comp], its coefficient
template <typename T> struct GradRun {
  const T* p;
  int32_t x0, x1;
  double c;
};

// adds the runs list[0 .. n) to the lane's NS elements (element k at gx[k],
// offset lc[k] = per gx + comp)
template <typename T, int NS>
__device__ __forceinline__ void grad_add(const GradRun<T>* list, int n, const int (&gx)[4],
                                         const int (&lc)[4], double (&acc)[4]) {
  constexpr int U = sizeof(T) == 4 && NS == 1 ? 16 : 8 / NS;
  for (int i0 = 0; i0 < n; i0 += U) {
    T v[U][NS];
    double c[U];
    bool in[U][NS];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const GradRun<T> e = list[min(i0 + u, n - 1)];
      const int x1 = i0 + u < n ? e.x1 - e.x0 : -1;   // the last run repeated: no points
      c[u] = e.c;
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        in[u][k] = (uint32_t)gx[k] - (uint32_t)e.x0 <= (uint32_t)x1 && x1 >= 0;
        v[u][k] = T(0);
        if (in[u][k]) v[u][k] = e.p[lc[k]];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < NS; ++k)
        if (in[u][k]) acc[k] += c[u] * (double)v[u][k];
  }
}

template <typename T>
__global__ __launch_bounds__(256, 4) void k_grad_rows(const SfDev* __restrict__ sfs,
                                                   const wvl_seg* __restrict__ seg,
                                                   const int32_t* __restrict__ rt,
                                                   const RowRun* __restrict__ rr,
                                                   const int64_t* __restrict__ rowptr,
                                                   const int32_t* __restrict__ col,
                                                   const double* __restrict__ av,
                                                   const double* __restrict__ mv,
                                                   const T* __restrict__ psi,
                                                   const T* __restrict__ hpsi, int sf0,
                                                   T* __restrict__ g) {
  __shared__ GradNb nb[kGradNb];
  __shared__ GradRun<T> lists[4][kGradCap];
  const int a = sf0 + blockIdx.y;
  const SfDev& A = sfs[a];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  GradRun<T>* const list = lists[wv];
  const int N1 = A.n[1], N2 = A.n[2];
  const int nrows = N1 * N2;
  const int64_t q0 = rowptr[a], q1 = rowptr[a + 1];
  const uint64_t below = (1ull << lane) - 1ull;
  // neighbours in batches of kGradNb: each element's sum runs over the
  // batches in order, the first batch writing g and the next ones adding to
  // it (an element has the same owner, lane and wave, in every batch; rows of
  // more than kGradNb entries round once per batch)
  const int64_t nbatch = max((int64_t)1, (q1 - q0 + kGradNb - 1) / kGradNb);
  for (int64_t bi = 0; bi < nbatch; ++bi) {
    const int64_t b0 = q0 + bi * kGradNb;
    const int nn = (int)max((int64_t)0, min((int64_t)kGradNb, q1 - b0));
    __syncthreads();
    for (int t = threadIdx.x; t < nn; t += 256) {
      const int d = col[b0 + t];
      const SfDev& D = sfs[d];
      GradNb x;
      x.y0 = D.lo[1]; x.z0 = D.lo[2]; x.by = D.n[1]; x.nz = D.n[2]; x.e = D.ext;
      x.n_c = (int)D.n_c; x.on_c = (int)D.on_c;
      x.rr = D.rr[0]; x.cin = D.cin; x.cout = D.cout;
      x.a = av[b0 + t];
      x.m = mv[b0 + t];
      x.id = d;
      nb[t] = x;
    }
    __syncthreads();
    for (int r = blockIdx.x * 4 + wv; r < nrows; r += 4 * kGradParts) {
      const int y = A.lo[1] + r % N1, z = A.lo[2] + r / N1;
#pragma unroll
      for (int fine = 0; fine < 2; ++fine) {
        const int per = fine ? 7 : 1;
        const int64_t abase = A.cin + (fine ? A.n_c : 0);
        for (int q = rt[A.rt[fine] + r], qe = rt[A.rt[fine] + r + 1]; q < qe; ++q) {
          const int as = seg[q].i1s, ae = seg[q].i1e;
          const int64_t aoff = seg[q].off;
          const int len = per * (ae - as + 1);
          for (int j0 = 0; j0 < len; j0 += 256) {
            int gx[4], lc[4];
            double acc[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int j = j0 + 64 * k + lane;
              const int pt = j / per, comp = j - per * pt;
              gx[k] = j < len ? as + pt : INT32_MIN;   // meets no run (unsigned differences)
              lc[k] = per * (as + pt) + comp;
              acc[k] = 0.0;
            }
            const int ns = (min(len - j0, 256) + 63) >> 6;
            for (int t0 = 0; t0 < nn; t0 += 64) {
              // phase 1
              GradRun<T> e[2];
              bool has[2] = {false, false}, multi[2] = {false, false};
              int64_t row[2] = {0, 0};
              const int t = t0 + lane;
              const GradNb& x = nb[min(t, nn - 1)];
              if (t < nn) {
                RowRun w[2];
#pragma unroll
                for (int s = 0; s < 2; ++s) {   // 0: H phi_d, output pattern; 1: phi_d, input
                  const int o = s ? 0 : x.e, by = x.by + 2 * o, nz = x.nz + 2 * o;
                  const int ry = y - x.y0 + o, rz = z - x.z0 + o;
                  e[s].c = s ? -x.m : x.a;
                  w[s] = RowRun{0, 0, 0};
                  if (ry >= 0 && ry < by && rz >= 0 && rz < nz && e[s].c != 0.0) {
                    row[s] = (int64_t)rz * by + ry;
                    // the patterns' records follow each other: in-coarse,
                    // in-fine, out-coarse, out-fine
                    const int64_t nin = (int64_t)x.by * x.nz;
                    w[s] = rr[x.rr + (s ? 0 : 2 * nin) + (fine ? (s ? nin : (int64_t)by * nz) : 0) +
                              row[s]];
                  }
                }
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                  multi[s] = w[s].len == kMultiRun;
                  e[s].x0 = w[s].x0;
                  e[s].x1 = (int)w[s].x0 + (int)w[s].len - 1;
                  has[s] = w[s].len != 0 && (multi[s] || (e[s].x0 <= ae && e[s].x1 >= as));
                  e[s].p = (s ? psi + x.cin + (fine ? x.n_c : 0) : hpsi + x.cout + (fine ? x.on_c : 0)) +
                           (int64_t)per * ((int64_t)w[s].off - (int)w[s].x0);
                }
              }
              // the lane's runs in order: entry(run)
              const bool any_multi = __any(multi[0] || multi[1]);
              auto walk = [&](auto&& entry) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                  if (!has[s]) continue;
                  if (!multi[s]) {
                    entry(e[s]);
                    continue;
                  }
                  const int64_t tb = sfs[x.id].rt[(s ? 0 : 2) + fine] + row[s];
                  for (int p = rt[tb], pe = rt[tb + 1]; p < pe; ++p) {
                    const wvl_seg h = seg[p];
                    if (h.i1s > ae || h.i1e < as) continue;
                    GradRun<T> m;
                    m.x0 = h.i1s;
                    m.x1 = h.i1e;
                    m.c = e[s].c;
                    m.p = (s ? psi + x.cin + (fine ? x.n_c : 0) : hpsi + x.cout + (fine ? x.on_c : 0)) +
                          (int64_t)per * (h.off - h.i1s);
                    entry(m);
                  }
                }
              };
              int pos, n;   // first position of the lane's runs, runs in all
              if (!any_multi) {
                const uint64_t m0 = __ballot(has[0]), m1 = __ballot(has[1]);
                pos = __popcll(m0 & below) + __popcll(m1 & below);
                n = __popcll(m0) + __popcll(m1);
              } else {
                int cnt = 0;
                walk([&](const GradRun<T>&) { ++cnt; });
                pos = cnt;   // inclusive sum over the lanes
                for (int o = 1; o < 64; o <<= 1) {
                  const int up = __shfl_up(pos, o, 64);
                  if (lane >= o) pos += up;
                }
                n = __shfl(pos, 63, 64);
                pos -= cnt;
              }
              // the list in rounds of kGradCap (one unless rows have several runs)
              for (int base = 0; base < n; base += kGradCap) {
                int at = pos - base;
                walk([&](const GradRun<T>& m) {
                  if (at >= 0 && at < kGradCap) list[at] = m;
                  ++at;
                });
                wave_sync();
                const int nr = min(kGradCap, n - base);
                if (ns == 1) grad_add<T, 1>(list, nr, gx, lc, acc);
                else if (ns == 2) grad_add<T, 2>(list, nr, gx, lc, acc);
                else grad_add<T, 4>(list, nr, gx, lc, acc);
                wave_sync();
              }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              const int j = j0 + 64 * k + lane;
              if (j >= len) continue;
              T* o = g + abase + per * aoff + j;
              *o = bi == 0 ? (T)acc[k] : (T)((double)*o + acc[k]);
            }
          }
        }
      }
    }
  }
}

static inline dim3 grid2(int64_t maxvol, int nsf) {
  return dim3((unsigned)((maxvol + TPB - 1) / TPB), (unsigned)nsf);
}

// Loads the code objects of the kernels a captured step may launch.
int preload_kernels() {
  const void* fns[] = {(const void*)k_finalize, (const void*)k_sparse_values<float, 1>,
                       (const void*)k_sparse_values<double, 1>, (const void*)k_sparse_values<float, 2>,
                       (const void*)k_sparse_values<float, 4>, (const void*)k_sparse_values<float, 8>,
                       (const void*)k_sparse_values<double, 2>,
                       (const void*)k_sparse_values<double, 4>,
                       (const void*)k_sparse_values<double, 8>, (const void*)k_update<float>,
                       (const void*)k_update<double>, (const void*)k_sf_dot<float>,
                       (const void*)k_sf_dot<double>, (const void*)k_dens_tile<float, kDensChunk>,
                       (const void*)k_dens_tile<float, kDensLight>,
                       (const void*)k_dens_tile<double, kDensChunk>, (const void*)k_grad_rows<float>,
                       (const void*)k_grad_rows<double>};
  for (const void* f : fns) {
    hipFuncAttributes a;
    const hipError_t e = hipFuncGetAttributes(&a, f);
    if (e != hipSuccess) return (int)e;
  }
  return 0;
}

int launch_gather(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                  const void* psi, void* box, int sf0, int nsf, int64_t maxvol) {
  if (nsf == 0 || maxvol == 0) return 0;
  hipStream_t st = (hipStream_t)stream;
  if (f64)
    hipLaunchKernelGGL(k_gather<double>, grid2(maxvol, nsf), dim3(TPB), 0, st, sf, seg, rt,
                       (const double*)psi, (double*)box, sf0);
  else
    hipLaunchKernelGGL(k_gather<float>, grid2(maxvol, nsf), dim3(TPB), 0, st, sf, seg, rt,
                       (const float*)psi, (float*)box, sf0);
  return (int)hipGetLastError();
}

int launch_scatter(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                   const void* box, void* out, int sf0, int nsf, int64_t maxvol) {
  if (nsf == 0 || maxvol == 0) return 0;
  hipStream_t st = (hipStream_t)stream;
  if (f64)
    hipLaunchKernelGGL(k_scatter<double>, grid2(maxvol, nsf), dim3(TPB), 0, st, sf, seg, rt,
                       (const double*)box, (double*)out, sf0);
  else
    hipLaunchKernelGGL(k_scatter<float>, grid2(maxvol, nsf), dim3(TPB), 0, st, sf, seg, rt,
                       (const float*)box, (float*)out, sf0);
  return (int)hipGetLastError();
}

int launch_fill(int f64, void* stream, void* ptr, int64_t n) {
  if (n == 0) return 0;
  const dim3 g((unsigned)((n + TPB - 1) / TPB));
  if (f64)
    hipLaunchKernelGGL(k_fill<double>, g, dim3(TPB), 0, (hipStream_t)stream, (double*)ptr, n);
  else
    hipLaunchKernelGGL(k_fill<float>, g, dim3(TPB), 0, (hipStream_t)stream, (float*)ptr, n);
  return (int)hipGetLastError();
}

int launch_finalize(void* stream, const SfWork* wk, int sf0, int nsf, const double* parts,
                    int which, int nblk, double* out) {
  if (nsf == 0) return 0;
  hipLaunchKernelGGL(k_finalize, dim3(nsf), dim3(TPB), 0, (hipStream_t)stream, wk, sf0, parts,
                     which, nblk, out);
  return (int)hipGetLastError();
}

int launch_pattern(void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt, int nsf,
                   int ket_out, int64_t* count, const int64_t* rowptr, int32_t* col) {
  if (nsf == 0) return 0;
  hipLaunchKernelGGL(k_pattern, dim3(nsf), dim3(64), 0, (hipStream_t)stream, sf, seg, rt, nsf,
                     ket_out, count, rowptr, col);
  return (int)hipGetLastError();
}

int launch_sparse_values(int f64, void* stream, const SfDev* sf, const wvl_seg* seg,
                         const int32_t* rt, const RowRun* rr, int ket_out, const void* bra,
                         const void* ket, const int32_t* row, const int32_t* col,
                         const int32_t* order, const int32_t* mirror, int64_t nnz, int64_t rows,
                         double* val) {
  if (nnz == 0) return 0;
  const unsigned nblk = (unsigned)(8 * ((nnz + 7) / 8));
  auto go = [&](auto kernel, int w, auto t) {
    using T = decltype(t);
    hipLaunchKernelGGL(kernel, dim3(nblk), dim3(64 * w), 0, (hipStream_t)stream, sf, seg, rt, rr,
                       ket_out, (const T*)bra, (const T*)ket, row, col, order, mirror, nnz, val);
  };
  // Waves per pair: the chip holds 8,192 waves.  With fewer pairs than that
  // one wave's chain of loads is the time, so a pair's batches of 64 rows are
  // dealt to more: H of 56 functions (3,122 pairs, 724 rows per box, FP64) takes
  // 194 / 128 / 125 / 120 us with 1 / 2 / 4 / 8 waves, S of 100 (3,900, FP32) 139 /
  // 83 / 65 / 67.  With many pairs the waves of a pair read the same lines
  // together: H of 1,000 (301,162) FP64 5.62 / 5.37 / 5.38 / 7.14 ms, FP32 3.93 /
  // 4.04 / 4.39 / 7.03, S (82,000) 0.50 / 0.47 / 0.53 / 0.93.  A wave without a
  // batch of its own only costs: 33 rows per box, H of 4,000 (305,559), FP32 0.54 /
  // 0.94 / 1.69 / 3.61 ms; 95 rows, H of 9,000 (496,106), FP64 2.66 / 2.71 / 4.13 /
  // 8.59; 155 rows, H of 7,000 (566,476) FP64 4.72 / 4.65 / 6.04 / 12.0, FP32 3.09 /
  // 3.59.  The number of waves does not change a value.
  int w;
  if (rows <= 64) {
    w = 1;
  } else if (nnz <= 3584) {
    w = rows <= 128 ? 2 : rows <= 256 ? 4 : 8;
  } else if (nnz <= 32768) {
    w = rows <= 256 ? 2 : 4;
  } else if (f64) {
    w = rows <= 128 ? 1 : 2;
  } else {
    w = rows <= 256 || (ket_out && nnz > 131072) ? 1 : 2;
  }
  if (f64)
    w == 8   ? go(k_sparse_values<double, 8>, w, 0.0)
    : w == 4 ? go(k_sparse_values<double, 4>, w, 0.0)
    : w == 2 ? go(k_sparse_values<double, 2>, w, 0.0)
             : go(k_sparse_values<double, 1>, w, 0.0);
  else
    w == 8   ? go(k_sparse_values<float, 8>, w, 0.0f)
    : w == 4 ? go(k_sparse_values<float, 4>, w, 0.0f)
    : w == 2 ? go(k_sparse_values<float, 2>, w, 0.0f)
             : go(k_sparse_values<float, 1>, w, 0.0f);
  return (int)hipGetLastError();
}

int launch_dens_tile(int f64, void* stream, const SfDev* sf, const int64_t* foff,
                     const void* fine, const int64_t* krow, const int32_t* kcol,
                     const double* kval, int64_t knnz, const DensTile* tiles, const int32_t* csf,
                     int64_t nheavy, int nsf, const int* gf, void* rho) {
  const int tx = (gf[0] + kDensTile[0] - 1) / kDensTile[0];
  const int ty = (gf[1] + kDensTile[1] - 1) / kDensTile[1];
  const int tz = (gf[2] + kDensTile[2] - 1) / kDensTile[2];
  const int64_t ntile = (int64_t)tx * ty * tz;
  auto go = [&](auto kernel, const DensTile* list, int64_t n, auto t) {
    using T = decltype(t);
    if (n > 0)
      hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(kDensThreads), 0, (hipStream_t)stream, sf,
                         foff, (const T*)fine, krow, kcol, kval, knnz, list, csf, nsf, tx, ty, gf[0],
                         gf[1], gf[2], (T*)rho);
  };
  if (f64) {   // all tiles (the light form would spill)
    go(k_dens_tile<double, kDensChunk>, tiles, ntile, 0.0);
  } else {
    go(k_dens_tile<float, kDensChunk>, tiles, nheavy, 0.0f);
    go(k_dens_tile<float, kDensLight>, tiles + nheavy, ntile - nheavy, 0.0f);
  }
  return (int)hipGetLastError();
}

static inline dim3 grid1(int64_t n) { return dim3((unsigned)((n + TPB - 1) / TPB)); }

int launch_foe_mm(void* stream, int nrow, const int32_t* rows, const int64_t* rowptr,
                  const int32_t* col, double alpha, const double* A, const double* B, double beta,
                  const double* D, double* C, int lognb, int maxdeg) {
  if (nrow == 0) return 0;
  // rows of at most 256 entries: two rows of B (128 entries each) per step
  const int w = maxdeg <= kFoeMaxDeg / 2 ? 8 : 4;
  const int nh = maxdeg <= kFoeMaxDeg / 4 ? 2 : 1;
  const size_t lds = (size_t)maxdeg * 8 * (w * nh + 2) + ((size_t)16 << lognb);
  const dim3 g((unsigned)nrow), blk(64 * w);
  hipStream_t st = (hipStream_t)stream;
  if (nh == 2)
    hipLaunchKernelGGL((k_foe_mm<8, 2>), g, blk, lds, st, rows, rowptr, col, alpha, A, B, beta,
                       D, C, lognb, maxdeg);
  else if (w == 8)
    hipLaunchKernelGGL((k_foe_mm<8, 1>), g, blk, lds, st, rows, rowptr, col, alpha, A, B, beta,
                       D, C, lognb, maxdeg);
  else
    hipLaunchKernelGGL((k_foe_mm<4, 1>), g, blk, lds, st, rows, rowptr, col, alpha, A, B, beta,
                       D, C, lognb, maxdeg);
  return (int)hipGetLastError();
}

int launch_foe_rmul(void* stream, int nrow, const int32_t* rows, const int64_t* rowptr,
                    const int32_t* col, double alpha, const double* R, const double* A, double beta,
                    const double* D, const int64_t* tpos, double* C, int maxdeg) {
  if (nrow == 0) return 0;
  if ((int64_t)nrow + maxdeg > kFoeSpread) return (int)hipErrorInvalidValue;
  const size_t lds = (size_t)nrow * 8 + (size_t)maxdeg * 8;
  // one row per block while a CU's LDS holds four blocks (its 2,048 threads),
  // beyond that as many blocks as the 256 CUs hold, each with several rows: an
  // expansion of degree 50 of 7,900 functions with 6 entries a row 3.03 -> 2.38 ms, of
  // 6,000 with 50 3.03 -> 2.91, but of 4,000 with 72 2.70 -> 2.97
  const int fit = (int)(160 * 1024 / (lds + 256));
  const bool loop = fit < 2048 / kRmulThreads && 256 * fit < nrow;
  auto go = [&](auto kernel, int grid) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kRmulThreads), lds, (hipStream_t)stream,
                       rows, rowptr, col, nrow, alpha, R, A, beta, D, tpos, C, maxdeg);
  };
  loop ? go(k_foe_rmul<true>, 256 * fit) : go(k_foe_rmul<false>, nrow);
  return (int)hipGetLastError();
}

int launch_foe_axpby(void* stream, int64_t nnz, double a, const double* X, double b,
                     const double* Y, const int32_t* row, const int32_t* col, double d,
                     double* out) {
  if (nnz == 0) return 0;
  hipLaunchKernelGGL(k_foe_axpby, grid1(nnz), dim3(TPB), 0, (hipStream_t)stream, nnz, a, X, b, Y,
                     row, col, d, out);
  return (int)hipGetLastError();
}

int launch_foe_sym(void* stream, int64_t nnz, const int64_t* tpos, const double* X, double* out) {
  if (nnz == 0) return 0;
  hipLaunchKernelGGL(k_foe_sym, grid1(nnz), dim3(TPB), 0, (hipStream_t)stream, nnz, tpos, X, out);
  return (int)hipGetLastError();
}

int launch_foe_gather(void* stream, int64_t nnz, const int64_t* qpos, const double* X,
                      double* out) {
  if (nnz == 0) return 0;
  hipLaunchKernelGGL(k_foe_gather, grid1(nnz), dim3(TPB), 0, (hipStream_t)stream, nnz, qpos, X,
                     out);
  return (int)hipGetLastError();
}

int launch_foe_dot(void* stream, int64_t nnz, const double* X, const double* Y, double* part,
                   double* out, int slot) {
  const int nblk = (int)std::min<int64_t>(256, std::max<int64_t>(1, (nnz + 2047) / 2048));
  const int64_t chunk = (nnz + nblk - 1) / nblk;
  hipLaunchKernelGGL(k_foe_dot, dim3(nblk), dim3(TPB), 0, (hipStream_t)stream, nnz, chunk, X, Y,
                     part);
  hipLaunchKernelGGL(k_foe_sum, dim3(1), dim3(TPB), 0, (hipStream_t)stream, nblk, part, out, slot);
  return (int)hipGetLastError();
}

int launch_foe_trace(void* stream, int n, const int64_t* dpos, const double* X, int64_t stride,
                     int count, double* out, int slot) {
  if (count == 0) return 0;
  hipLaunchKernelGGL(k_foe_trace, dim3((unsigned)count), dim3(TPB), 0, (hipStream_t)stream, n,
                     dpos, X, stride, out, slot);
  return (int)hipGetLastError();
}

int launch_foe_series(void* stream, int64_t nnz, int npl, const double* c, const double* T,
                      const int32_t* row, const int32_t* col, double* out) {
  if (nnz == 0) return 0;
  hipLaunchKernelGGL(k_foe_series, grid1(nnz), dim3(TPB), 0, (hipStream_t)stream, nnz, npl, c, T,
                     row, col, out);
  return (int)hipGetLastError();
}

int launch_foe_gersh(void* stream, int nrow, const int64_t* rowptr, const int32_t* col,
                     const double* X, double* lo, double* hi, double* out) {
  if (nrow == 0) return 0;
  const int rows = TPB / 64;
  hipLaunchKernelGGL(k_foe_gersh_rows, dim3((unsigned)((nrow + rows - 1) / rows)), dim3(TPB), 0,
                     (hipStream_t)stream, nrow, rowptr, col, X, lo, hi);
  hipLaunchKernelGGL(k_foe_gersh, dim3(1), dim3(TPB), 0, (hipStream_t)stream, nrow, lo, hi, out);
  return (int)hipGetLastError();
}

int launch_update(int f64, void* stream, const SfDev* sf, const wvl_seg* seg, const int32_t* rt,
                  double eta, const void* hpsi, const int64_t* hrow, const int32_t* hcol,
                  const double* hval, void* psi, int sf0, int nsf, int64_t maxsegs, int mode,
                  const double* shift, void* out) {
  if (nsf == 0) return 0;
  const dim3 g((unsigned)(maxsegs / kUpdSegs + 2), (unsigned)nsf);
  if (f64)
    hipLaunchKernelGGL(k_update<double>, g, dim3(256), 0, (hipStream_t)stream, sf, seg, rt, eta,
                       (const double*)hpsi, hrow, hcol, hval, (double*)psi, sf0, mode, shift,
                       (double*)out);
  else
    hipLaunchKernelGGL(k_update<float>, g, dim3(256), 0, (hipStream_t)stream, sf, seg, rt, eta,
                       (const float*)hpsi, hrow, hcol, hval, (float*)psi, sf0, mode, shift,
                       (float*)out);
  return (int)hipGetLastError();
}

int launch_sf_dot(int f64, void* stream, const SfDev* sf, const void* a, const void* b,
                  double* out, int sf0, int nsf) {
  if (nsf == 0) return 0;
  if (f64)
    hipLaunchKernelGGL(k_sf_dot<double>, dim3(nsf), dim3(TPB), 0, (hipStream_t)stream, sf,
                       (const double*)a, (const double*)b, out, sf0);
  else
    hipLaunchKernelGGL(k_sf_dot<float>, dim3(nsf), dim3(TPB), 0, (hipStream_t)stream, sf,
                       (const float*)a, (const float*)b, out, sf0);
  return (int)hipGetLastError();
}

int launch_cg_init(int f64, void* stream, const SfDev* sf, const void* g, void* x, void* r,
                   void* p, int sf0, int nsf) {
  if (nsf == 0) return 0;
  if (f64)
    hipLaunchKernelGGL(k_cg_init<double>, dim3(nsf), dim3(TPB), 0, (hipStream_t)stream, sf,
                       (const double*)g, (double*)x, (double*)r, (double*)p, sf0);
  else
    hipLaunchKernelGGL(k_cg_init<float>, dim3(nsf), dim3(TPB), 0, (hipStream_t)stream, sf,
                       (const float*)g, (float*)x, (float*)r, (float*)p, sf0);
  return (int)hipGetLastError();
}

int launch_cg_xr(int f64, void* stream, const SfDev* sf, const double* rr, const double* pap,
                 const void* p, const void* ap, void* x, void* r, int sf0, int nsf) {
  if (nsf == 0) return 0;
  if (f64)
    hipLaunchKernelGGL(k_cg_xr<double>, dim3(nsf), dim3(TPB), 0, (hipStream_t)stream, sf, rr,
                       pap, (const double*)p, (const double*)ap, (double*)x, (double*)r, sf0);
  else
    hipLaunchKernelGGL(k_cg_xr<float>, dim3(nsf), dim3(TPB), 0, (hipStream_t)stream, sf, rr, pap,
                       (const float*)p, (const float*)ap, (float*)x, (float*)r, sf0);
  return (int)hipGetLastError();
}

int launch_cg_p(int f64, void* stream, const SfDev* sf, double* rr, const double* rr_new,
                const void* r, void* p, int sf0, int nsf) {
  if (nsf == 0) return 0;
  if (f64)
    hipLaunchKernelGGL(k_cg_p<double>, dim3(nsf), dim3(TPB), 0, (hipStream_t)stream, sf, rr,
                       rr_new, (const double*)r, (double*)p, sf0);
  else
    hipLaunchKernelGGL(k_cg_p<float>, dim3(nsf), dim3(TPB), 0, (hipStream_t)stream, sf, rr,
                       rr_new, (const float*)r, (float*)p, sf0);
  return (int)hipGetLastError();
}

int launch_grad_rows(int f64, void* stream, const SfDev* sf, const wvl_seg* seg,
                     const int32_t* rt, const RowRun* rr, const int64_t* rowptr,
                     const int32_t* col, const double* av, const double* mv, const void* psi,
                     const void* hpsi, int sf0, int nsf, void* g) {
  if (nsf == 0) return 0;
  if (f64)
    hipLaunchKernelGGL(k_grad_rows<double>, dim3(kGradParts, (unsigned)nsf), dim3(256), 0, (hipStream_t)stream,
                       sf, seg, rt, rr, rowptr, col, av, mv, (const double*)psi,
                       (const double*)hpsi, sf0, (double*)g);
  else
    hipLaunchKernelGGL(k_grad_rows<float>, dim3(kGradParts, (unsigned)nsf), dim3(256), 0, (hipStream_t)stream,
                       sf, seg, rt, rr, rowptr, col, av, mv, (const float*)psi,
                       (const float*)hpsi, sf0, (float*)g);
  return (int)hipGetLastError();
}

}  // namespace wvl
