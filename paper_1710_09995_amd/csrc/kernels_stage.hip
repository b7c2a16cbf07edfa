// Residual, time-stage update, time step and norm kernels.
//
// R_c = ((F_i+ - F_i-) + (F_j+ - F_j-) + (F_k+ - F_k-)) / V_c with
// F = (F_inv - F_vis) . S (Section 2.2, Eq. 3, dQ/dt = -R), and the stage
// update of Eqs. (4)-(6) with lambda = -dt:
//   stage 1: Q1   = Qn - dt R(Qn)
//   stage 2: Q2   = 3/4 Qn + 1/4 (Q1 - dt R(Q1))
//   stage 3: Qn+1 = 1/3 Qn + 2/3 (Q2 - dt R(Q2))
//
// All kernels run persistent over a tile work list that spans every block:
// workgroup w takes tiles w, w + G, w + 2G, ... (static round robin), so one
// launch covers all blocks of uneven sizes.  Reductions go wave64 butterfly
// -> LDS in fixed order -> one partial row per workgroup -> a single-workgroup
// finalize in fixed order, so results are bitwise reproducible.
//
// This file holds the simple per-cell kernel (every face read from global
// memory and computed by both of its cells); the tiled face-once kernel is in
// kernels_tiled.hip.
#include <hip/hip_runtime.h>
#include "cfd_internal.hpp"
#include "physics.hpp"
#include "stage_common.hpp"
#include "chunks.hpp"

namespace cfd {

// ------------------------------------------------- simple per-cell stage kernel
template <typename T, bool VISC, int MODE>
__global__ void __launch_bounds__(256) k_stage_simple(StageArgs A, const BlockDesc* __restrict__ blocks,
                                                      const TileDesc* __restrict__ tiles, Gas<T> gas) {
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int nty = blockDim.x >> 6;
  for (int tile = blockIdx.x; tile < A.ntiles; tile += gridDim.x) {
    const TileDesc td = tiles[tile];
    const BlockDesc B = blocks[td.blk];
    const int i = td.i0 + tx;
    int k0, kend;
    tile_run(B.n[2], A.tile_k, td.kp, k0, kend);
    const double* qb = A.qs + B.qoff;
    const double* mb = A.met + B.moff;
    const double* vb = VISC ? A.vmet + B.voff : nullptr;
    for (int j = td.j0 + ty; j < min(td.j0 + A.tile_j, B.n[1]); j += nty) {
      if (i >= B.n[0]) break;
      for (int k = k0; k < kend; ++k) {
        const int64_t c = (int64_t)(k + NG) * B.sk + (int64_t)(j + NG) * B.sj + (i + NG);
        double Fl[5], Fu[5], D[3][5];
        for (int d = 0; d < 3; ++d) {
          face_flux_global<T, VISC>(qb, mb, vb, B, c, d, gas, Fl);
          face_flux_global<T, VISC>(qb, mb, vb, B, c + dstride(d, B.sj, B.sk), d, gas, Fu);
          for (int q = 0; q < 5; ++q) D[d][q] = Fu[q] - Fl[q];
        }
        finish_cell<MODE>(A, B, c, D[0], D[1], D[2]);
      }
    }
  }
}

// ------------------------------------------------------------- time step
// dt_c = CFL V / (sum_d L_d + 4 sum_d Lv_d) with S_d averaged over the cell's
// two d-faces; per-workgroup partials: minimum dt (slot 12), sum V Q
// (slots 5-9) and the count of non-finite Q values (slot 11); local steps
// stored.  Without TOTALS the minimum alone (a step without a history).
template <bool TOTALS>
__global__ void __launch_bounds__(256) k_dt(const double* __restrict__ q, const double* __restrict__ met,
                                            double* __restrict__ dtcell, double* __restrict__ partials,
                                            const BlockDesc* __restrict__ blocks, int nblk, int64_t nchunks,
                                            StepParams P) {
  double acc[NPART];
  init_partials(acc);
  const int lane = threadIdx.x & 63;
  int64_t r0, r1;
  wave_rows(nchunks, r0, r1);
  ChunkWalk W;
  if (r0 < r1) W.start(blocks, nblk, r0);
  for (int64_t u = r0; u < r1; ++u) {
    int i, j, k;
    if (!W.cell(u, lane, i, j, k)) continue;
    const BlockDesc& B = W.B;
    const double* qb = q + B.qoff;
    const double* mb = met + B.moff;
    const int64_t c = (int64_t)(k + NG) * B.sk + (int64_t)(j + NG) * B.sj + (i + NG);
    const double qc[5] = {qb[c], qb[B.sv + c], qb[2 * B.sv + c], qb[3 * B.sv + c], qb[4 * B.sv + c]};
    const double vol = mb[9 * B.sv + c];
    const double dtc = cell_dt(qc, mb, c, B.sv, B.sj, B.sk, P);
    if (P.local_dt) dtcell[B.soff + c] = dtc;
    acc[12] = fmin(acc[12], dtc);
    if (TOTALS) {
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        acc[5 + v] += vol * qc[v];
        if (!finite(qc[v])) acc[11] += 1.0;
      }
    }
  }
  if (TOTALS) {
    wg_reduce_partials(acc, partials + (int64_t)blockIdx.x * NPART);
  } else {
    __shared__ double red[4];
    double m = acc[12];
    for (int off = 32; off > 0; off >>= 1) m = fmin(m, __shfl_xor(m, off, 64));
    if (lane == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0)
      partials[(int64_t)blockIdx.x * NPART + 12] = fmin(fmin(red[0], red[1]), fmin(red[2], red[3]));
  }
}

// ------------------------------------------------------------- norms
// Partials of sum R^2 (slots 0-4), max |R_rho| (10) and the non-finite count
// (11) of r, and of sum V Q (5-9) and the non-finite count of q; either of q
// (then met too) and r may be null.  Same cut of the grid as k_dt, so its
// sum V Q rows are bitwise k_dt's.
__global__ void __launch_bounds__(256) k_norms(const double* __restrict__ q, const double* __restrict__ r,
                                               const double* __restrict__ met, double* __restrict__ partials,
                                               const BlockDesc* __restrict__ blocks, int nblk, int64_t nchunks) {
  double acc[NPART];
  init_partials(acc);
  const int lane = threadIdx.x & 63;
  int64_t r0, r1;
  wave_rows(nchunks, r0, r1);
  ChunkWalk W;
  if (r0 < r1) W.start(blocks, nblk, r0);
  for (int64_t u = r0; u < r1; ++u) {
    int i, j, k;
    if (!W.cell(u, lane, i, j, k)) continue;
    const BlockDesc& B = W.B;
    const int64_t c = (int64_t)(k + NG) * B.sk + (int64_t)(j + NG) * B.sj + (i + NG);
    if (q) {
      double qv[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) qv[v] = q[B.qoff + v * B.sv + c];
      const double vol = met[B.moff + 9 * B.sv + c];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        acc[5 + v] += vol * qv[v];
        if (!finite(qv[v])) acc[11] += 1.0;
      }
    }
    if (r) {
      double rv[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) rv[v] = r[B.qoff + v * B.sv + c];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        acc[v] += rv[v] * rv[v];
        if (!finite(rv[v])) acc[11] += 1.0;
      }
      acc[10] = fmax(acc[10], fabs(rv[0]));
    }
  }
  wg_reduce_partials(acc, partials + (int64_t)blockIdx.x * NPART);
}

// ------------------------------------------------------------- finalize
// One workgroup reduces the rows in a fixed order.  mode 1 (history row [dt,
// L2 x5, sum VQ x5, max|R_rho|] and nonfinite count): 64 threads a slot read
// the rows as one array (thread t holds slot t % 13 of rows t / 13 + 64 m:
// coalesced), then a fixed tree over the 64.  A row's place in the order does
// not depend on the number of rows.  mode 2: the same with the minimum of slot
// 12 for dt.  mode 0: the minimum of slot 12 -> dt.
// Twelve loads of a thread are in flight (2048 rows 6 us, 13 rows 4; 10.5 and 6 with
// the slot's operation chosen for every value, 20 with one load after the other).
constexpr int FIN_T = 64 * NPART;

__device__ __forceinline__ double fin_op(int q, double a, double b) {
  return q == 10 ? fmax(a, b) : q == 12 ? fmin(a, b) : a + b;
}

__global__ void __launch_bounds__(FIN_T) k_finalize(const double* __restrict__ partials, int nrows, int mode,
                                                    double inv_ncells, double* __restrict__ dt,
                                                    double* __restrict__ hist, double* __restrict__ nonfinite) {
  __shared__ double sh[FIN_T];
  const int t = threadIdx.x;
  if (mode == 0) {
    double m = __builtin_inf();
#pragma unroll 4
    for (int row = t; row < nrows; row += FIN_T) m = fmin(m, partials[(int64_t)row * NPART + 12]);
    for (int off = 32; off > 0; off >>= 1) m = fmin(m, __shfl_xor(m, off, 64));
    if ((t & 63) == 0) sh[t >> 6] = m;
    __syncthreads();
    if (t == 0) {
      for (int w = 1; w < NPART; ++w) m = fmin(m, sh[w]);
      dt[0] = m;
    }
    return;
  }
  const int q = t % NPART;
  const double none = q == 12 ? __builtin_inf() : 0.0;
  const int total = nrows * NPART;
  // the slot's sum, and its largest value, of slot 12 the largest of the negated ones
  const uint64_t flip = q == 12 ? (uint64_t)1 << 63 : 0;
  auto negated = [&](double x) { return __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, x) ^ flip); };
  double sum = 0.0, most = negated(none);
  constexpr int U = 12;      // loads in flight
  for (int e0 = t; e0 < total; e0 += U * FIN_T) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = e0 + u * FIN_T;
      v[u] = partials[e < total ? e : t];
      if (e >= total) v[u] = none;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sum += v[u];
      most = fmax(most, negated(v[u]));
    }
  }
  const double acc = q == 10 || q == 12 ? negated(most) : sum;
  sh[t] = acc;
  __syncthreads();
  for (int s = 32; s > 0; s >>= 1) {
    if (t < s * NPART) sh[t] = fin_op(q, sh[t], sh[t + s * NPART]);
    __syncthreads();
  }
  if (t == 0) hist[0] = mode == 2 ? sh[12] : dt ? dt[0] : 0.0;
  if (t < 5) hist[1 + t] = sqrt(sh[t] * inv_ncells);
  else if (t < 10) hist[1 + t] = sh[t];
  else if (t == 10) hist[11] = sh[10];
  else if (t == 11 && nonfinite) nonfinite[0] = sh[11];
}

// ---------------------------------------------------------------- launchers

template <typename T, bool VISC, int MODE>
static void launch_simple_t(const StageArgs& A, const BlockDesc* blocks, const TileDesc* tiles,
                            const Gas<T>& gas, int nwg, hipStream_t s) {
  hipLaunchKernelGGL((k_stage_simple<T, VISC, MODE>), dim3(nwg), dim3(256), 0, s, A, blocks, tiles,
                     gas);
}

void launch_stage_simple(const StageArgs& A, int mode, bool visc, bool fp32, const BlockDesc* blocks,
                         const TileDesc* tiles, const Gas<double>& g64, const Gas<float>& g32, int nwg,
                         hipStream_t s) {
#define CFD_DISPATCH(T, G, V)                                                    \
  if (mode == 0) launch_simple_t<T, V, 0>(A, blocks, tiles, G, nwg, s);          \
  else if (mode == 1) launch_simple_t<T, V, 1>(A, blocks, tiles, G, nwg, s);     \
  else launch_simple_t<T, V, 2>(A, blocks, tiles, G, nwg, s);
  if (fp32) {
    if (visc) { CFD_DISPATCH(float, g32, true) } else { CFD_DISPATCH(float, g32, false) }
  } else {
    if (visc) { CFD_DISPATCH(double, g64, true) } else { CFD_DISPATCH(double, g64, false) }
  }
#undef CFD_DISPATCH
}

void launch_dt(const double* q, const double* met, double* dtcell, double* partials, const BlockDesc* blocks,
               int nblk, int64_t nchunks, const StepParams& P, int nwg, bool totals, hipStream_t s) {
  if (totals)
    hipLaunchKernelGGL(k_dt<true>, dim3(nwg), dim3(256), 0, s, q, met, dtcell, partials, blocks, nblk, nchunks, P);
  else
    hipLaunchKernelGGL(k_dt<false>, dim3(nwg), dim3(256), 0, s, q, met, dtcell, partials, blocks, nblk, nchunks, P);
}

void launch_norms(const double* q, const double* r, const double* met, double* partials, const BlockDesc* blocks,
                  int nblk, int64_t nchunks, int nwg, hipStream_t s) {
  hipLaunchKernelGGL(k_norms, dim3(nwg), dim3(256), 0, s, q, r, met, partials, blocks, nblk, nchunks);
}

void launch_finalize(const double* partials, int nrows, int mode, double inv_ncells, double* dt,
                     double* hist, double* nonfinite, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(FIN_T), 0, s, partials, nrows, mode, inv_ncells, dt, hist,
                     nonfinite);
}

}  // namespace cfd
