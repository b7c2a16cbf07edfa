// Brick residual / stage kernel for grids too small to fill the chip with
// marching tiles.
//
// On such a grid a launch is one short latency chain.  The marching kernels
// put five or six face fluxes of a plane one after the other in the same
// thread; here a workgroup of 512 threads takes a brick of 8 x 4 x 4 cells and
// every thread computes one face: 144 i-, 160 j- and 160 k-faces, 464 of the
// 512 threads.  The chain is one load of the brick's cells (with the halo of 2
// its faces read, 448 cells, no edges or corners for inviscid flow), one face,
// one cell update.  The price is 464 / 384 face fluxes per cell face and 3.5
// cells converted per cell, which is why grids that fill the chip march.
//
// Inviscid flow needs no ghost cells in memory: a brick at a block's face forms
// the ghost states as it reads them, from the neighbour's or its own interior
// cells (three ghost-fill launches a step less, each a latency of its own).
//
// A face flux gets the same bits as in the other stage kernels: the same
// primitives and expressions, with the direction as strides.
//
// 32^3 Euler, FP64: 7.5 us a launch against 11.5 with 64 x 4 x 1 marching tiles,
// 35 us a step with its history row against 77; the dispatch rule has the sizes
// at which either is faster.
#include <hip/hip_runtime.h>
#include "cfd_internal.hpp"
#include "physics.hpp"
#include "stage_common.hpp"
#include "ghosts.hpp"

namespace cfd {

namespace {

constexpr int BI = BRICK_I, BJ = BRICK_J, BK = BRICK_K;
constexpr int WI = BI + 4, WJ = BJ + 4, WK = BK + 4;
constexpr int NW3 = WI * WJ * WK;                 // cells of the brick with its halo
constexpr int FI = (BI + 1) * BJ * BK, FJ = BI * (BJ + 1) * BK, FK = BI * BJ * (BK + 1);
constexpr int NF = FI + FJ + FK;                  // faces
constexpr int CELLS = BI * BJ * BK;
constexpr int NT = 512;
static_assert(NF <= NT && CELLS == 128 && NT == 512 && BJ == 4 && BK == 4, "one face a thread, one wave a norm");

template <typename T, bool VISC, int MODE>
__global__ void __launch_bounds__(NT, sizeof(T) == 8 ? 2 : 4) k_stage_brick(StageArgs A, const BlockDesc* __restrict__ blocks,
                                                    const TileDesc* __restrict__ tiles, Gas<T> gas) {
  constexpr int NW = VISC ? 6 : 5;
  __shared__ T sW[NW][NW3];
  __shared__ double sF[5][NF];
  __shared__ double sdt[NT / 64];
  const int tid = threadIdx.x;
  // this thread's face: direction, cell above it, its place in sF and sW
  const int d = tid < FI ? 0 : tid < FI + FJ ? 1 : 2;
  const int e = tid - (d == 0 ? 0 : d == 1 ? FI : FI + FJ);
  const int ex = d == 0 ? BI + 1 : BI, ey = d == 1 ? BJ + 1 : BJ;
  const int fi = e % ex, fj = (e / ex) % ey, fk = e / (ex * ey);
  const int fp = ((fk + 2) * WJ + fj + 2) * WI + fi + 2;
  const int st = d == 0 ? 1 : d == 1 ? WI : WI * WJ;
  const int t1 = d == 0 ? WI : 1, t2 = d == 2 ? WI : WI * WJ;      // transverse, ascending
  // this thread's cell
  const int ci = tid % BI, cj = (tid / BI) % BJ, ck = tid / (BI * BJ);

  // norm partials of this thread's cells, kept in LDS (in registers they would
  // cost the face work its second workgroup per CU)
  constexpr int NP = 7;      // sum R^2 x5, max |R_rho|, non-finite count
  __shared__ double sacc[MODE == 1 ? NP : 1][MODE == 1 ? CELLS : 1];
  if (MODE == 1 && tid < CELLS)
    for (int q = 0; q < NP; ++q) sacc[q][tid] = 0.0;
  double dt_g = 0.0;
  if (MODE == 1 && A.rows) {
    double m = __builtin_inf();
    for (int r = tid; r < A.nrows; r += NT) m = fmin(m, A.rows[(int64_t)r * NPART + 12]);
    for (int off = 32; off > 0; off >>= 1) m = fmin(m, __shfl_xor(m, off, 64));
    if ((tid & 63) == 0) sdt[tid >> 6] = m;
    __syncthreads();
    dt_g = sdt[0];
    for (int w = 1; w < NT / 64; ++w) dt_g = fmin(dt_g, sdt[w]);
    if (blockIdx.x == 0 && tid == 0) A.dt_min[0] = dt_g;
  }

  for (int tile = blockIdx.x; tile < A.ntiles; tile += gridDim.x) {
    const TileDesc td = tiles[tile];
    const BlockDesc B = blocks[td.blk];
    const int i0 = td.i0, j0 = td.j0, k0 = td.kp * BK;
    const int64_t sv = B.sv;
    const double* qb = A.qs + B.qoff;
    const double* mb = A.met + B.moff;
    auto off = [&](int i, int j, int k) -> int64_t {
      return (int64_t)(k + NG) * B.sk + (int64_t)(j + NG) * B.sj + (i + NG);
    };
    const int fd = d == 0 ? 1 : 0, gd = d == 1 ? 1 : 0, hd = d == 2 ? 1 : 0;
    const bool fok = tid < NF && i0 + fi < B.n[0] + fd && j0 + fj < B.n[1] + gd && k0 + fk < B.n[2] + hd;
    const bool cok = tid < CELLS && i0 + ci < B.n[0] && j0 + cj < B.n[1] && k0 + ck < B.n[2];
    // metrics of the face, in flight over the fill
    const int64_t fc = off(i0 + fi, j0 + fj, k0 + fk), cc = off(i0 + ci, j0 + cj, k0 + ck);
    double sx = 1.0, sy = 0.0, sz = 0.0;
    if (fok) {
      sx = mb[(3 * d) * sv + fc];
      sy = mb[(3 * d + 1) * sv + fc];
      sz = mb[(3 * d + 2) * sv + fc];
    }
    // primitives of the brick and its halo
    auto fill = [&](int pi, int pj, int pk) {
      const int i = i0 + pi - 2, j = j0 + pj - 2, k = k0 + pk - 2;
      Prim<T> w;
      if (i > B.n[0] + 1 || j > B.n[1] + 1 || k > B.n[2] + 1) return;
      if (VISC) {
        w = ld_prim<T>(qb, off(i, j, k), sv, gas.gm1);
      } else {
        const int gi = i < 0 || i >= B.n[0], gj = j < 0 || j >= B.n[1], gk = k < 0 || k >= B.n[2];
        if (gi + gj + gk > 1) return;      // edges and corners: no inviscid face reads them
        double q[5];
        if (gi + gj + gk == 0 || !A.patches) {
          const int64_t o = off(i, j, k);
#pragma unroll
          for (int v = 0; v < 5; ++v) q[v] = qb[v * sv + o];
        } else if (!ghost_state(A.qs, A.met, blocks, A.patches, A.patch_first, td.blk, B, gi ? 0 : gj ? 1 : 2,
                                gi ? i : gj ? j : k, gi ? j : i, gk ? j : k, A.sp.gamma, q)) {
          return;
        }
        w = to_prim<T>(q[0], q[1], q[2], q[3], q[4], gas.gm1);
      }
      const int p = (pk * WJ + pj) * WI + pi;
      sW[0][p] = w.r;
      sW[1][p] = w.u;
      sW[2][p] = w.v;
      sW[3][p] = w.w;
      sW[4][p] = w.p;
      if (VISC) sW[NW - 1][p] = temp_of(w);
    };
    if (VISC) {
      for (int s = tid; s < NW3; s += NT) fill(s % WI, (s / WI) % WJ, s / (WI * WJ));
    } else {
      // the faces' own halo: BJ BK rows of WI cells, 4 j-layers and 4 k-layers of BI cells
      constexpr int RI = WI * BJ * BK, RJ = 4 * BI * BK, RK = 4 * BI * BJ;
      static_assert(RI + RJ + RK <= NT, "one cell a thread");
      int pi = tid % WI, pj = (tid / WI) % BJ + 2, pk = tid / (WI * BJ) + 2;
      if (tid >= RI) {
        const int s = tid < RI + RJ ? tid - RI : tid - RI - RJ;
        const int x = s % BI, y = (s / BI) % 4, z = s / (4 * BI);      // BJ = BK = 4
        const int l = tid < RI + RJ ? y : z, in = tid < RI + RJ ? z : y;
        const int out = l < 2 ? l : l + BJ;
        pi = x + 2;
        pj = tid < RI + RJ ? out : in + 2;
        pk = tid < RI + RJ ? in + 2 : out;
      }
      if (tid < RI + RJ + RK) fill(pi, pj, pk);
    }
    __syncthreads();
    if (fok) {
      auto prim = [&](int p) {
        Prim<T> w;
        w.r = sW[0][p];
        w.u = sW[1][p];
        w.v = sW[2][p];
        w.w = sW[3][p];
        w.p = sW[4][p];
        return w;
      };
      T f[5], n[3];
      const double area = face_inviscid<T>(prim(fp - 2 * st), prim(fp - st), prim(fp), prim(fp + st), sx, sy, sz, gas,
                                           f, n);
      if (VISC) {
        auto phi = [&](int p, T o[4]) {
          o[0] = sW[1][p];
          o[1] = sW[2][p];
          o[2] = sW[3][p];
          o[3] = sW[NW - 1][p];
        };
        T pl[4], pr[4], d1[4], d2[4], a[4], b[4], c[4], g[4];
        phi(fp - st, pl);
        phi(fp, pr);
        phi(fp - st + t1, a); phi(fp + t1, b); phi(fp - st - t1, c); phi(fp - t1, g);
        tdiff(a, b, c, g, d1);
        phi(fp - st + t2, a); phi(fp + t2, b); phi(fp - st - t2, c); phi(fp - t2, g);
        tdiff(a, b, c, g, d2);
        double St[2][3], vf;
        face_vmetrics(A.vmet + B.voff, sv, fc, d, St, vf);
        face_viscous<T>(pl, pr, sx, sy, sz, n, d1, d2, St, vf, gas, f);
      }
      double F[5];
      scale_flux_f64(f, area, F);
#pragma unroll
      for (int q = 0; q < 5; ++q) sF[q][tid] = F[q];
    }
    __builtin_amdgcn_sched_barrier(0);      // the cell's inputs are not live over the face
    CellIn cin;
    if (cok) {
      load_cell<MODE>(A, B, cc, cin);
      if (MODE == 1 && A.rows) cin.dt = dt_g;
    }
    __syncthreads();
    if (cok) {
      double D[3][5], Rc[5], Qo[5];
      const int xi = (ck * BJ + cj) * (BI + 1) + ci, xj = FI + (ck * (BJ + 1) + cj) * BI + ci,
                xk = FI + FJ + (ck * BJ + cj) * BI + ci;
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        D[0][q] = sF[q][xi + 1] - sF[q][xi];
        D[1][q] = sF[q][xj + BI] - sF[q][xj];
        D[2][q] = sF[q][xk + BI * BJ] - sF[q][xk];
      }
      update_cell<MODE>(A, B, cc, D[0], D[1], D[2], cin, Rc, Qo, A.force);
      if (MODE == 1 && A.partials) {
        double bad = 0.0;
#pragma unroll
        for (int q = 0; q < 5; ++q) {
          sacc[q][tid] += Rc[q] * Rc[q];
          if (!finite(Rc[q])) bad += 1.0;
          if (!finite(cin.qv[q])) bad += 1.0;
        }
        sacc[5][tid] = fmax(sacc[5][tid], fabs(Rc[0]));
        sacc[6][tid] += bad;
      }
    }
    __syncthreads();     // sW and sF are free for the next brick
  }
  // the workgroup's row: one wave a slot
  if (MODE == 1 && A.partials) {
    __syncthreads();
    const int w = tid >> 6, lane = tid & 63;
    double* row = A.partials + (int64_t)blockIdx.x * NPART;
    if (w < NP) {
      double v = w == 5 ? fmax(sacc[w][lane], sacc[w][lane + 64]) : sacc[w][lane] + sacc[w][lane + 64];
      for (int o = 32; o > 0; o >>= 1) {
        const double u = __shfl_xor(v, o, 64);
        v = w == 5 ? fmax(v, u) : v + u;
      }
      if (lane == 0) row[w < 5 ? w : w == 5 ? 10 : 11] = v;
    } else if (lane >= 5 && lane < 10) {
      row[lane] = 0.0;
    } else if (lane == 12) {
      row[lane] = __builtin_inf();
    }
  }
}

template <typename T, bool VISC, int MODE>
void brick_launch(const StageArgs& A, const BlockDesc* blocks, const TileDesc* tiles, const Gas<T>& gas, int nwg,
                  hipStream_t s, int* occ) {
  if (occ) {
    int n = 0;
    *occ = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_stage_brick<T, VISC, MODE>, NT, 0) == hipSuccess && n > 0
               ? n
               : 1;
    return;
  }
  hipLaunchKernelGGL((k_stage_brick<T, VISC, MODE>), dim3(nwg), dim3(NT), 0, s, A, blocks, tiles, gas);
}

template <typename T, bool VISC>
void brick_mode(const StageArgs& A, int mode, const BlockDesc* blocks, const TileDesc* tiles, const Gas<T>& gas,
                int nwg, hipStream_t s, int* occ) {
  if (mode == 0) brick_launch<T, VISC, 0>(A, blocks, tiles, gas, nwg, s, occ);
  else if (mode == 1) brick_launch<T, VISC, 1>(A, blocks, tiles, gas, nwg, s, occ);
  else brick_launch<T, VISC, 2>(A, blocks, tiles, gas, nwg, s, occ);
}

}  // namespace

// Launch (occ == nullptr) or query the resident workgroups per CU.
void stage_brick(const StageArgs& A, int mode, bool visc, bool fp32, const BlockDesc* blocks, const TileDesc* tiles,
                 const Gas<double>& g64, const Gas<float>& g32, int nwg, hipStream_t s, int* occ) {
  if (fp32) {
    if (visc) brick_mode<float, true>(A, mode, blocks, tiles, g32, nwg, s, occ);
    else brick_mode<float, false>(A, mode, blocks, tiles, g32, nwg, s, occ);
  } else {
    if (visc) brick_mode<double, true>(A, mode, blocks, tiles, g64, nwg, s, occ);
    else brick_mode<double, false>(A, mode, blocks, tiles, g64, nwg, s, occ);
  }
}

}  // namespace cfd
