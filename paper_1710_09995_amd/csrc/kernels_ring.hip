// Plane-ring face-once residual / stage kernel.  Tiles of TI x TJ columns,
// one thread each: 64 x 8 and 32 x 16 (tile_j 8), 32 x 8 and 16 x 16
// (tile_j 4), chosen by how the blocks' extents fill them.
//
// Same tile decomposition and per-face arithmetic as the tiled kernel, with a
// different plane pipeline.  LDS holds a ring of three primitive planes
// W(k-1), W(k), W(k+1), each with a halo of 2 cells (rho, u, v, w, p [, T]).
// The viscous face gradients take phi = (u, v, w, T) of the neighbouring
// planes straight from the ring, so every plane is loaded and converted once
// and no separate phi planes are kept or copied.
//
// Per k-plane, two barriers:
//   A. faces of plane k (W(k-1..k+1) ready): the lower i-face and lower
//      j-face of every column, the tile-edge faces, the upper k-face (cells
//      k-1..k+1 from the ring, k+2 from a one-cell register queue);
//   B. after the barrier: the cell update of plane k (its inputs were loaded
//      before the faces) together with the fill of W(k+2) into the slot of
//      W(k-1) and the queue load of W(k+3), so their memory latencies overlap.
// Stage 1 accumulates the norm partials of R(Qn) in registers (this kernel
// has the register room) instead of writing R for a separate norms kernel
// (the totals sum V Qn come from a row-chunk kernel whose cut of the grid
// does not depend on the tiles), and stage 3 (mode 3) evaluates the CFL time
// step of the state it writes (the next step's), instead of a separate
// time-step kernel.
// The i-face fluxes are exchanged between neighbouring lanes of the wave
// (shuffle) instead of through LDS; only the tile's edge i-faces and the
// j-faces go through LDS.  Every face flux gets the same bits as in the
// other stage kernels (same primitives, same expressions).
//
// With two waves a SIMD and barriers between them, what bounds it beside FP64
// issue is the latency of loads that sit right before their use.  So: a face's
// metrics are loaded together before its flux; W(k+2) and W(k+3) are loaded
// before the k-face, without branches (columns and planes clamped to the ghost
// layers; a load under a branch is waited for where the branch ends), but for
// W(k+2) in the FP32 Euler variants, four waves a SIMD, and in the FP64 stage 3,
// which would spill (256 x 128 x 128 NS, stage 3: 585 us before, 619 with it, 533
// without); and addresses are one 32-bit column offset beside scalar bases.  64-bit vector addresses per field,
// hoisted out of the plane loop, filled the registers and spilled: FP64
// Navier-Stokes stage 1 62 dwords, now none (stage 3 four).  256 x 128 x 128 NS
// 1577 -> 1500 us a step, 2 x 2 x (250 x 203 x 72) FP32 NS 5.07 -> 4.66 ms,
// 128 x (48 x 24 x 24) Euler V-cycles 5.50 -> 5.19 ms; FP32 Euler as before.
// FP64 Navier-Stokes on a grid past the caches runs at the rate of a copy (500 B
// a cell and stage); face metrics, Q^n and the output, used once, then carry the
// non-temporal hint (the face vectors not in stage 3, which reads them again)
// so that the caches keep the halos: 2 x 2 x (512 x 512 x 144)
// 55.6 -> 53.7 ms, 256 x 128 x 128 alike; FP32 NS would lose 2 % by it.
#include <hip/hip_runtime.h>
#include <type_traits>
#include "cfd_internal.hpp"
#include "physics.hpp"
#include "stage_common.hpp"

// Scheduling fence between face computations (register pressure), as in the
// tiled kernel.
#define CFD_FACE_FENCE_RING() __builtin_amdgcn_sched_barrier(0)

namespace cfd {

template <typename T, bool VISC, int TI_, int TJ_>
struct RingLds {
  static constexpr int TI = TI_, TJ = TJ_;
  static constexpr int WI = TI + 4, WJ = TJ + 4;   // halo 2
  static constexpr int NW = VISC ? 6 : 5;
  static constexpr int PLANE = NW * WJ * WI;   // elements of one plane
  static constexpr int W_BYTES = (3 * PLANE * (int)sizeof(T) + 15) / 16 * 16;
  static constexpr int FJ = 5 * (TJ + 1) * TI;  // doubles: lower j-faces, TJ+1 rows
  static constexpr int FE = 5 * TJ;             // doubles: i-faces at i0+TI
  static constexpr int TOTAL = W_BYTES + (FJ + FE) * 8;
  // stage 3 also keeps the area vectors of those faces for the time step
  static constexpr int SJ = 3 * (TJ + 1) * TI;  // doubles: S_j of the lower j-faces
  static constexpr int SE = 3 * TJ;             // doubles: S_i at i0+TI
  static constexpr int TOTAL_DT = TOTAL + (SJ + SE) * 8;
};

// Minimum waves per SIMD asked of the register allocator: the FP32 Euler
// variants fit 128 VGPRs (4 waves per SIMD), FP64 needs all 256 of two waves
// (without the bound its 256-column variants took 257 and ran one wave per
// SIMD: 256 x 128 x 128 NS 2.18 ms a step against 1.75), FP32 NS takes what it
// needs (two waves).
template <typename T, bool VISC>
constexpr int ring_min_waves() {
  return sizeof(T) == 8 ? 2 : VISC ? 1 : 4;
}

template <typename T, bool VISC, int MODE, int TI, int TJ>
__global__ void __launch_bounds__(TI * TJ, (ring_min_waves<T, VISC>())) k_stage_ring(
    StageArgs A, const BlockDesc* __restrict__ blocks, const TileDesc* __restrict__ tiles, Gas<T> gas) {
  using LD = RingLds<T, VISC, TI, TJ>;
  constexpr bool F64 = sizeof(T) == 8, EARLY = (F64 || VISC) && !(F64 && MODE == 3), STREAM = F64 && VISC;
  constexpr int NT = TI * TJ;
  constexpr int WI = LD::WI, WJ = LD::WJ;
  __shared__ __attribute__((aligned(16))) char smem[MODE == 3 ? LD::TOTAL_DT : LD::TOTAL];
  T* sW = reinterpret_cast<T*>(smem);                                   // [3][NW][WJ][WI]
  double* sFj = reinterpret_cast<double*>(smem + LD::W_BYTES);          // [5][TJ+1][TI]
  double* sFe = sFj + LD::FJ;                                           // [5][TJ]
  double* sSj = sFe + LD::FE;                                           // mode 3: [3][TJ+1][TI]
  double* sSe = sSj + LD::SJ;                                           // mode 3: [3][TJ]

  auto W = [&](int slot, int v, int p) -> T& { return sW[slot * LD::PLANE + v * (WJ * WI) + p]; };
  auto wprim = [&](int slot, int p) {
    Prim<T> w;
    w.r = W(slot, 0, p);
    w.u = W(slot, 1, p);
    w.v = W(slot, 2, p);
    w.w = W(slot, 3, p);
    w.p = W(slot, 4, p);
    return w;
  };
  auto wphi = [&](int slot, int p, T o[4]) {
    o[0] = W(slot, 1, p);
    o[1] = W(slot, 2, p);
    o[2] = W(slot, 3, p);
    o[3] = W(slot, VISC ? 5 : 4, p);
  };

  const int tid = threadIdx.x, tx = tid & (TI - 1), ty = tid / TI;
  // partials: stage 1 (mode 1) sum R^2, max |R_rho|, non-finite count;
  // stage 3 (mode 3) minimum time step of the new state
  double acc[NPART];
  init_partials(acc);

  for (int tile = blockIdx.x; tile < A.ntiles; tile += gridDim.x) {
    const TileDesc td = tiles[tile];
    BlockDesc B = blocks[td.blk];
    const int ni = B.n[0], nj = B.n[1], nk = B.n[2];
    const int i0 = td.i0, j0 = td.j0;
    int k0, kend;
    tile_run(nk, A.tile_k, td.kp, k0, kend);
    k0 = __builtin_amdgcn_readfirstlane(k0);
    kend = __builtin_amdgcn_readfirstlane(kend);
    const int i = i0 + tx, j = j0 + ty;
    const bool act = i < ni && j < nj;
    const bool fi_ok = i <= ni && j < nj;
    const bool fj_ok = j <= nj && i < ni;
    // faces on the tile's high edges: lanes [0, TI) the j-faces of row j0+TJ,
    // lanes [TI, TI+TJ) the i-faces of column i0+TI
    const bool e_j = tid < TI;
    const int e_ci = e_j ? tid : TI, e_rj = e_j ? TJ : tid - TI;
    const bool e_ok = tid < TI + TJ && (e_j ? j0 + TJ <= nj && i0 + e_ci < ni : i0 + TI <= ni && j0 + e_rj < nj);
    const double* qb = A.qs + B.qoff;
    const double* mb = A.met + B.moff;
    const double* vb = VISC ? A.vmet + B.voff : nullptr;
    const int64_t sj = B.sj, sk = B.sk;
    int64_t sv = B.sv;
    auto off = [&](int ii, int jj, int kk) -> int64_t {
      return (int64_t)(kk + NG) * sk + (int64_t)(jj + NG) * sj + (ii + NG);
    };
    // a column's byte offset, new to the compiler at each use: known to be the
    // same for every plane it would be added to each field's base outside the loop
    auto fresh = [](uint32_t c) {
      asm volatile("" : "+v"(c));
      return c;
    };
    auto col = [&](int ii, int jj) { return fresh((uint32_t)((jj + NG) * (int)sj + (ii + NG)) * 8u); };
    auto plane = [&](int kk) { return (int64_t)(__builtin_amdgcn_readfirstlane(kk) + NG) * sk; };
    const uint32_t own0 = col(min(i, ni + 1), min(j, nj + 1));
    // W(kk) with halo 2 into ring slot `slot`: a fixed trip count, unrolled,
    // so that all of a thread's loads are in flight together
    constexpr int NS = (WJ * WI + NT - 1) / NT;
    struct Raw {
      double q[5];
    };
    using Cell3 = std::conditional_t<F64, Raw, Prim<T>>;   // W(k + 2) of the column: converted late where that
                                                           // takes no more registers
    auto load_raw = [&](CellAt c, Raw& r) { load_fields<5>(qb, sv, c, r.q); };
    auto prim_of = [&](const auto& r) {
      if constexpr (std::is_same_v<std::decay_t<decltype(r)>, Raw>)
        return to_prim<T>(r.q[0], r.q[1], r.q[2], r.q[3], r.q[4], gas.gm1);
      else return r;
    };
    auto fill_load = [&](int kk, Raw raw[NS]) {
#pragma unroll
      for (int it = 0; it < NS; ++it) {
        const int s = min(tid + it * NT, WJ * WI - 1);
        const int pj = s / WI, pi = s - (s / WI) * WI;
        load_raw(CellAt{plane(kk), col(min(i0 - 2 + pi, ni + 1), min(j0 - 2 + pj, nj + 1))}, raw[it]);
      }
    };
    auto fill_store = [&](int slot, const Raw raw[NS]) {
#pragma unroll
      for (int it = 0; it < NS; ++it) {
        const int s = tid + it * NT;
        if (s >= WJ * WI) break;
        const Prim<T> w = prim_of(raw[it]);
        W(slot, 0, s) = w.r;
        W(slot, 1, s) = w.u;
        W(slot, 2, s) = w.v;
        W(slot, 3, s) = w.w;
        W(slot, 4, s) = w.p;
        if (VISC) W(slot, 5, s) = temp_of(w);
      }
    };
    auto fill = [&](int slot, int kk) {
      Raw raw[NS];
      fill_load(kk, raw);
      fill_store(slot, raw);
    };

    // lower k-face of the tile from global memory; queue cell W(k0+2)
    double Fklo[5] = {0, 0, 0, 0, 0};
    Cell3 q3{};
    if (act) {
      const int64_t c0 = off(i, j, k0);
      face_flux_global<T, VISC>(qb, mb, vb, B, c0, 2, gas, Fklo);
      Raw r;
      load_raw(CellAt{plane(k0 + 2), own0}, r);
      if constexpr (F64) q3 = r;
      else q3 = prim_of(r);
    }
    __syncthreads();   // the previous tile's LDS users are done
    int sm = 0, s0 = 1, sp = 2;   // ring slots of W(k-1), W(k), W(k+1)
    fill(sm, k0 - 1);
    fill(s0, k0);
    fill(sp, k0 + 1);
    __syncthreads();

    for (int k = k0; k < kend; ++k) {
      const uint32_t own = fresh(own0);
      // the field stride anew every plane: its multiples are cheap scalar
      // work, kept across the planes they filled the scalar registers
      asm volatile("" : "+s"(sv));
      B.sv = sv;
      // inputs of this plane's cell update, loaded before the face work
      CellIn cin;
      load_cell<MODE, STREAM>(A, B, CellAt{plane(k), own}, cin);
      // ---- A. faces of plane k
      // lower face, along direction d = 0 (i) or 1 (j), of cell (i0+ci, j0+rj):
      // flux F, area vector S.  One expression for both directions, so that
      // the tile-edge faces of either run in the same lanes.
      auto metrics = [&](int d, auto c, double S[3], double St[2][3], double& vf) {
        load_fields<3, STREAM && MODE != 3>(mb + (int64_t)(3 * d) * sv, sv, c, S);   // stage 3 reads them again
        if (VISC) face_vmetrics<STREAM>(vb, sv, c, d, St, vf);
      };
      auto face = [&](int d, int ci, int rj, const double S[3], const double St[2][3], double vf, double F[5]) {
        const int p = (rj + 2) * WI + ci + 2;             // the cell above the face
        const int st = d == 0 ? 1 : WI, tr = d == 0 ? WI : 1;   // along the face normal, across
        const double sx = S[0], sy = S[1], sz = S[2];
        T f[5], n[3];
        const double area = face_inviscid<T>(wprim(s0, p - 2 * st), wprim(s0, p - st), wprim(s0, p),
                                             wprim(s0, p + st), sx, sy, sz, gas, f, n);
        if (VISC) {
          T pl[4], pr[4], d1[4], d2[4], a[4], b[4], e[4], g[4];
          wphi(s0, p - st, pl);
          wphi(s0, p, pr);
          wphi(s0, p - st + tr, a); wphi(s0, p + tr, b); wphi(s0, p - st - tr, e); wphi(s0, p - tr, g);
          tdiff(a, b, e, g, d1);
          wphi(sp, p - st, a); wphi(sp, p, b); wphi(sm, p - st, e); wphi(sm, p, g);
          tdiff(a, b, e, g, d2);
          face_viscous<T>(pl, pr, sx, sy, sz, n, d1, d2, St, vf, gas, f);
        }
        scale_flux_f64(f, area, F);
      };
      auto keep_j = [&](int ci, int rj, const double F[5], const double S[3]) {   // a j-face -> LDS
        for (int q = 0; q < 5; ++q) sFj[(q * (TJ + 1) + rj) * TI + ci] = F[q];
        if (MODE == 3)
          for (int x = 0; x < 3; ++x) sSj[(x * (TJ + 1) + rj) * TI + ci] = S[x];
      };
      double Fi[5] = {0, 0, 0, 0, 0};
      double S[3], St[2][3], vf;
      if (fi_ok) {
        metrics(0, CellAt{plane(k), own}, S, St, vf);
        CFD_FACE_FENCE_RING();
        face(0, tx, ty, S, St, vf, Fi);
      }
      CFD_FACE_FENCE_RING();
      if (fj_ok) {
        metrics(1, CellAt{plane(k), own}, S, St, vf);
        CFD_FACE_FENCE_RING();
        double Fj[5];
        face(1, tx, ty, S, St, vf, Fj);
        keep_j(tx, ty, Fj, S);
      }
      CFD_FACE_FENCE_RING();
      if (e_ok) {
        double Fe[5];
        metrics(e_j ? 1 : 0, off(i0 + e_ci, j0 + e_rj, k), S, St, vf);
        face(e_j ? 1 : 0, e_ci, e_rj, S, St, vf, Fe);
        if (e_j) {
          keep_j(e_ci, TJ, Fe, S);
        } else {
          for (int q = 0; q < 5; ++q) sFe[q * TJ + e_rj] = Fe[q];
          if (MODE == 3)
            for (int x = 0; x < 3; ++x) sSe[x * TJ + e_rj] = S[x];
        }
      }
      CFD_FACE_FENCE_RING();
      const bool more = k + 1 < kend;
      Raw raw[NS], r3;
      metrics(2, CellAt{plane(k + 1), own}, S, St, vf);
      if (EARLY) {
        CFD_FACE_FENCE_RING();
        fill_load(k + 2, raw);
      }
      load_raw(CellAt{plane(min(k + 3, nk + 1)), own}, r3);
      CFD_FACE_FENCE_RING();
      double Fku[5] = {0, 0, 0, 0, 0};
      if (act) {   // upper k-face between (i, j, k) and (i, j, k+1)
        const int p = (ty + 2) * WI + tx + 2;
        const double sx = S[0], sy = S[1], sz = S[2];
        T f[5], n[3];
        const double area =
            face_inviscid<T>(wprim(sm, p), wprim(s0, p), wprim(sp, p), prim_of(q3), sx, sy, sz, gas, f, n);
        if (VISC) {
          T pl[4], pr[4], d1[4], d2[4], a[4], b[4], e[4], g[4];
          wphi(s0, p, pl);
          wphi(sp, p, pr);
          wphi(s0, p + 1, a); wphi(sp, p + 1, b); wphi(s0, p - 1, e); wphi(sp, p - 1, g);
          tdiff(a, b, e, g, d1);
          wphi(s0, p + WI, a); wphi(sp, p + WI, b); wphi(s0, p - WI, e); wphi(sp, p - WI, g);
          tdiff(a, b, e, g, d2);
          face_viscous<T>(pl, pr, sx, sy, sz, n, d1, d2, St, vf, gas, f);
        }
        scale_flux_f64(f, area, Fku);
      }
      // upper i-face flux of this cell = lower i-face flux of the next lane
      double Fiu[5];
      for (int q = 0; q < 5; ++q) Fiu[q] = __shfl_down(Fi[q], 1, 64);
      __syncthreads();   // j-face and edge fluxes stored; every read of W(k-1) done

      // ---- B. cell update of plane k; fill W(k+2) over W(k-1); queue W(k+3)
      Cell3 q3n = q3;
      if constexpr (F64) q3n = r3;
      else q3n = prim_of(r3);
      // mode 3: the cell's face-averaged area vectors b[d] = (S_d(c) + S_d(c + e_d)) / 2.
      // Upper faces from this plane's face work: S_i of the next lane
      // (shuffle; the tile-edge face from LDS for lane 63), S_j of the next
      // row (LDS), S_k from the k-face (registers).  The lower i- and k-faces
      // are loaded again (cheaper than keeping them live through the faces).
      double bdt[3][3];
      if (MODE == 3) {
        double Si[3] = {0, 0, 0}, Sk[3] = {0, 0, 0}, Sku[3] = {0, 0, 0};
        if (fi_ok) {
          load_fields<3>(mb, sv, CellAt{plane(k), own}, Si);
        }
        if (act) {
          load_fields<3>(mb + 6 * sv, sv, CellAt{plane(k), own}, Sk);
          load_fields<3>(mb + 6 * sv, sv, CellAt{plane(k + 1), own}, Sku);
        }
        double Siu[3];
        for (int x = 0; x < 3; ++x) Siu[x] = __shfl_down(Si[x], 1, 64);
        if (act)
          for (int x = 0; x < 3; ++x) {
            const double su = tx == TI - 1 ? sSe[x * TJ + ty] : Siu[x];
            bdt[0][x] = 0.5 * (Si[x] + su);
            bdt[1][x] = 0.5 * (sSj[(x * (TJ + 1) + ty) * TI + tx] + sSj[(x * (TJ + 1) + ty + 1) * TI + tx]);
            bdt[2][x] = 0.5 * (Sk[x] + Sku[x]);
          }
      }
      if (more) {
        if constexpr (EARLY) fill_store(sm, raw);
        else fill(sm, k + 2);
      }
      if (act) {
        double Di[5], Dj[5], Dk[5];
        for (int q = 0; q < 5; ++q) {
          const double fu = tx == TI - 1 ? sFe[q * TJ + ty] : Fiu[q];
          Di[q] = fu - Fi[q];
          Dj[q] = sFj[(q * (TJ + 1) + ty + 1) * TI + tx] - sFj[(q * (TJ + 1) + ty) * TI + tx];
          Dk[q] = Fku[q] - Fklo[q];
        }
        double Rc[5], Qo[5];
        update_cell<MODE, STREAM>(A, B, CellAt{plane(k), own}, Di, Dj, Dk, cin, Rc, Qo);
        if (MODE == 1) {
#pragma unroll
          for (int q = 0; q < 5; ++q) {
            acc[q] += Rc[q] * Rc[q];
            if (!finite(Rc[q])) acc[11] += 1.0;
            if (!finite(cin.qv[q])) acc[11] += 1.0;
          }
          acc[10] = fmax(acc[10], fabs(Rc[0]));
        }
        if (MODE == 3) {
          const double dtc = cell_dt_b(Qo, bdt, cin.vol, A.sp);
          if (A.sp.local_dt) A.dt_out[B.soff + off(i, j, k)] = dtc;
          acc[12] = fmin(acc[12], dtc);
        }
        for (int q = 0; q < 5; ++q) Fklo[q] = Fku[q];
      }
      q3 = q3n;
      const int t = sm;
      sm = s0;
      s0 = sp;
      sp = t;
      __syncthreads();   // W(k+2) filled; j-face and edge flux reads done
    }
  }
  // the j-face buffer is free once the tiles are done
  if (MODE == 1 || MODE == 3)
    wg_reduce_partials(acc, A.partials + (int64_t)blockIdx.x * NPART, reinterpret_cast<double(*)[16]>(sFj));
}

// ---------------------------------------------------------------- launchers

template <typename T, bool VISC, int MODE, int TI, int TJ>
static void ring_launch(const StageArgs& A, const BlockDesc* blocks, const TileDesc* tiles, const Gas<T>& gas,
                        int nwg, hipStream_t s, int* occ) {
  if (occ) {
    int n = 0;
    *occ = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_stage_ring<T, VISC, MODE, TI, TJ>, TI * TJ, 0) ==
                       hipSuccess && n > 0
               ? n
               : 1;
    return;
  }
  hipLaunchKernelGGL((k_stage_ring<T, VISC, MODE, TI, TJ>), dim3(nwg), dim3(TI * TJ), 0, s, A, blocks, tiles, gas);
}

template <typename T, bool VISC, int TI, int TJ>
static void ring_mode(const StageArgs& A, int mode, const BlockDesc* blocks, const TileDesc* tiles,
                      const Gas<T>& gas, int nwg, hipStream_t s, int* occ) {
  if (mode == 0) ring_launch<T, VISC, 0, TI, TJ>(A, blocks, tiles, gas, nwg, s, occ);
  else if (mode == 1) ring_launch<T, VISC, 1, TI, TJ>(A, blocks, tiles, gas, nwg, s, occ);
  else if (mode == 2) ring_launch<T, VISC, 2, TI, TJ>(A, blocks, tiles, gas, nwg, s, occ);
  else if constexpr (VISC) ring_launch<T, VISC, 3, TI, TJ>(A, blocks, tiles, gas, nwg, s, occ);
}

template <typename T, bool VISC>
static bool ring_shape(const StageArgs& A, int mode, const BlockDesc* blocks, const TileDesc* tiles, const Gas<T>& gas,
                       int nwg, hipStream_t s, int* occ) {
  if (mode == 3 && !VISC) return false;   // inviscid flow takes its time steps in a pass of their own
  if (A.tile_j == 8 && A.tile_i == 64) ring_mode<T, VISC, 64, 8>(A, mode, blocks, tiles, gas, nwg, s, occ);
  else if (A.tile_j == 8 && A.tile_i == 32) ring_mode<T, VISC, 32, 16>(A, mode, blocks, tiles, gas, nwg, s, occ);
  else if (A.tile_j == 4 && A.tile_i == 32) ring_mode<T, VISC, 32, 8>(A, mode, blocks, tiles, gas, nwg, s, occ);
  else if (A.tile_j == 4 && A.tile_i == 16) ring_mode<T, VISC, 16, 16>(A, mode, blocks, tiles, gas, nwg, s, occ);
  else return false;
  return true;
}

// Launch (occ == nullptr) or query the resident workgroups per CU.  Takes
// A.tile_j = 4 or 8, mode 3 for viscous flow; false otherwise.
bool stage_ring(const StageArgs& A, int mode, bool visc, bool fp32, const BlockDesc* blocks, const TileDesc* tiles,
                const Gas<double>& g64, const Gas<float>& g32, int nwg, hipStream_t s, int* occ) {
  if (fp32) {
    return visc ? ring_shape<float, true>(A, mode, blocks, tiles, g32, nwg, s, occ)
                : ring_shape<float, false>(A, mode, blocks, tiles, g32, nwg, s, occ);
  }
  return visc ? ring_shape<double, true>(A, mode, blocks, tiles, g64, nwg, s, occ)
              : ring_shape<double, false>(A, mode, blocks, tiles, g64, nwg, s, occ);
}

}  // namespace cfd
