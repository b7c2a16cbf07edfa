// Ghost-cell states shared by the ghost-fill kernels and by the stage kernel
// that takes its ghost cells straight from the cells they depend on.
#pragma once
#include <hip/hip_runtime.h>
#include "cfd_internal.hpp"
#include "physics.hpp"

namespace cfd {

// Offset (relative to the padded origin) of logical index (a along d, p1
// along t1, p2 along t2) with t1 < t2 the transverse directions.
__device__ __forceinline__ int64_t pos3(int d, int a, int p1, int p2, int64_t sj, int64_t sk) {
  int i, j, k;
  if (d == 0) { i = a; j = p1; k = p2; }
  else if (d == 1) { j = a; i = p1; k = p2; }
  else { k = a; i = p1; j = p2; }
  return (int64_t)(k + NG) * sk + (int64_t)(j + NG) * sj + (i + NG);
}

// Ghost state of a slip (momentum reflected about the boundary face's unit
// normal) or no-slip adiabatic wall (momentum negated) mirroring cell state w.
__device__ __forceinline__ void wall_state(int kind, const double w[NV], double nx, double ny, double nz,
                                           double g[NV]) {
  const double mx = w[1], my = w[2], mz = w[3];
  g[0] = w[0];
  if (kind == CFD_BC_KIND_SLIPWALL) {
    const double mn = mx * nx + my * ny + mz * nz;
    g[1] = mx - 2.0 * mn * nx;
    g[2] = my - 2.0 * mn * ny;
    g[3] = mz - 2.0 * mn * nz;
  } else {
    g[1] = -mx;
    g[2] = -my;
    g[3] = -mz;
  }
  g[4] = w[4];
}

// Ghost fill of the conserved state: thread t of a patch.
// One thread per transverse point, except on i-faces: there the NG ghost
// cells of a row are adjacent in memory while neighbouring points are a row
// apart, so a thread per (point, layer) puts a row's layers on adjacent lanes
// and halves the memory segments each access touches.
// With delta set, q is an update (the implicit step's dQ): connections copy it
// as they copy the state, and the ghost cells of physical patches get zero (1) or
// hold it already (2).
__device__ __forceinline__ void ghost_fill_point(double* __restrict__ q, const double* __restrict__ met,
                                                 const BlockDesc* __restrict__ blocks, const PatchDesc& P, int t,
                                                 const StepParams& SP, int delta) {
  const int d = P.face >> 1, side = P.face & 1;
  const int per = ghost_threads_per_point(P.kind, d);
  if (t >= P.count * per) return;
  const int pt = t / per;
  // transverse directions t1 < t2, selected without indexing (keeps P out of scratch)
  const int lo1 = d == 0 ? P.lo[1] : P.lo[0], hi1 = d == 0 ? P.hi[1] : P.hi[0];
  const int lo2 = d == 2 ? P.lo[1] : P.lo[2];
  const int w1 = hi1 - lo1;
  const int p1 = lo1 + pt % w1, p2 = lo2 + pt / w1;
  const BlockDesc& B = blocks[P.blk];
  const int n = d == 0 ? B.n[0] : (d == 1 ? B.n[1] : B.n[2]);
  double* qb = q + B.qoff;
  if (P.kind == 0) {
    const BlockDesc& N = blocks[P.nbr];
    const double* qn = q + N.qoff;
    const int nn = d == 0 ? N.n[0] : (d == 1 ? N.n[1] : N.n[2]);
    const int o1 = d == 0 ? P.noff[1] : P.noff[0], o2 = d == 2 ? P.noff[1] : P.noff[2];
    // Every load before the first store: source and destination share one
    // arena, so a load issued after a store would wait for it.
    if (per != 1) {     // this thread's layer only
      const int m = 1 + t % per;
      const int64_t od = pos3(d, side == 0 ? -m : n - 1 + m, p1, p2, B.sj, B.sk);
      const int64_t os = pos3(d, side == 0 ? nn - m : m - 1, p1 + o1, p2 + o2, N.sj, N.sk);
      double val[NV];
      for (int v = 0; v < NV; ++v) val[v] = qn[v * N.sv + os];
      for (int v = 0; v < NV; ++v) qb[v * B.sv + od] = val[v];
      return;
    }
    double val[NG][NV];
    int64_t od[NG];
    for (int m = 1; m <= NG; ++m) {
      const int gm = side == 0 ? -m : n - 1 + m;
      const int sm = side == 0 ? nn - m : m - 1;
      od[m - 1] = pos3(d, gm, p1, p2, B.sj, B.sk);
      const int64_t os = pos3(d, sm, p1 + o1, p2 + o2, N.sj, N.sk);
      for (int v = 0; v < NV; ++v) val[m - 1][v] = qn[v * N.sv + os];
    }
    for (int m = 0; m < NG; ++m)
      for (int v = 0; v < NV; ++v) qb[v * B.sv + od[m]] = val[m][v];
    return;
  }
  if (delta) {
    if (delta == 2) return;   // zero already
    if (per != 1) {     // this thread's layer only
      const int m = 1 + t % per;
      const int64_t od = pos3(d, side == 0 ? -m : n - 1 + m, p1, p2, B.sj, B.sk);
      for (int v = 0; v < NV; ++v) qb[v * B.sv + od] = 0.0;
      return;
    }
    for (int m = 1; m <= NG; ++m) {
      const int64_t od = pos3(d, side == 0 ? -m : n - 1 + m, p1, p2, B.sj, B.sk);
      for (int v = 0; v < NV; ++v) qb[v * B.sv + od] = 0.0;
    }
    return;
  }
  // boundary face vector at this transverse position
  const int fa = side == 0 ? 0 : n;
  const int64_t of = pos3(d, fa, p1, p2, B.sj, B.sk);
  const double* mb = met + B.moff;
  const double sx = mb[(3 * d) * B.sv + of], sy = mb[(3 * d + 1) * B.sv + of],
               sz = mb[(3 * d + 2) * B.sv + of];
  const double nrm = sqrt(sx * sx + sy * sy + sz * sz);
  const double nx = sx / nrm, ny = sy / nrm, nz = sz / nrm;
  const int a0 = side == 0 ? 0 : n - 1;
  if (P.kind == CFD_BC_KIND_FARFIELD || P.kind == CFD_BC_KIND_EXTRAP) {
    const int64_t o0 = pos3(d, a0, p1, p2, B.sj, B.sk);
    double qi[5], qg[5];
    for (int v = 0; v < NV; ++v) qi[v] = qb[v * B.sv + o0];
    if (P.kind == CFD_BC_KIND_FARFIELD) {
      const double s = side == 0 ? -1.0 : 1.0;
      farfield_state(qi, s * nx, s * ny, s * nz, SP.gamma, P.uinf, qg);
    } else {
      for (int v = 0; v < NV; ++v) qg[v] = qi[v];
    }
    if (per != 1) {     // this thread's layer only
      const int m = 1 + t % per;
      const int64_t od = pos3(d, side == 0 ? -m : n - 1 + m, p1, p2, B.sj, B.sk);
      for (int v = 0; v < NV; ++v) qb[v * B.sv + od] = qg[v];
      return;
    }
    for (int m = 1; m <= NG; ++m) {
      const int gm = side == 0 ? -m : n - 1 + m;
      const int64_t od = pos3(d, gm, p1, p2, B.sj, B.sk);
      for (int v = 0; v < NV; ++v) qb[v * B.sv + od] = qg[v];
    }
    return;
  }
  // walls: ghost layer m mirrors interior cell m - 1
  auto wall = [&](const double w[NV], int64_t od) {
    double g[NV];
    wall_state(P.kind, w, nx, ny, nz, g);
    for (int v = 0; v < NV; ++v) qb[v * B.sv + od] = g[v];
  };
  if (per != 1) {       // this thread's layer only
    const int m = 1 + t % per;
    const int64_t oi = pos3(d, side == 0 ? m - 1 : n - m, p1, p2, B.sj, B.sk);
    double w[NV];
    for (int v = 0; v < NV; ++v) w[v] = qb[v * B.sv + oi];
    wall(w, pos3(d, side == 0 ? -m : n - 1 + m, p1, p2, B.sj, B.sk));
    return;
  }
  double wv[NG][NV];       // the mirrored interior cells, all loaded before any store
  for (int m = 1; m <= NG; ++m) {
    const int im = side == 0 ? m - 1 : n - m;
    const int64_t oi = pos3(d, im, p1, p2, B.sj, B.sk);
    for (int v = 0; v < NV; ++v) wv[m - 1][v] = qb[v * B.sv + oi];
  }
  for (int m = 1; m <= NG; ++m) wall(wv[m - 1], pos3(d, side == 0 ? -m : n - 1 + m, p1, p2, B.sj, B.sk));
}

// The far-field state out of line: its two powers would set the register count
// of a kernel whose other paths need fewer.
struct FarState {
  double q[NV];
};
__device__ __attribute__((noinline)) inline FarState farfield_call(double r, double ru, double rv, double rw, double e,
                                                                   double nx, double ny, double nz, double gamma,
                                                                   double u0, double u1, double u2) {
  const double w[NV] = {r, ru, rv, rw, e}, uinf[3] = {u0, u1, u2};
  FarState s;
  farfield_state(w, nx, ny, nz, gamma, uinf, s.q);
  return s;
}

// State of the ghost cell at (a along d, p1, p2 across) of block b, from the
// interior cell it depends on: what ghost_fill_point would store there, for a
// kernel that reads no ghost cells (inviscid flow: ghosts beyond one face
// only).  patches: over the faces' own cells, grouped by block and face,
// first[6 nblk + 1] the groups' ranges.  False where no patch covers it.
__device__ __forceinline__ bool ghost_state(const double* __restrict__ q, const double* __restrict__ met,
                                            const BlockDesc* __restrict__ blocks,
                                            const PatchDesc* __restrict__ patches, const int32_t* __restrict__ first,
                                            int b, const BlockDesc& B, int d, int a, int p1, int p2, double gamma,
                                            double g[NV]) {
  const int side = a < 0 ? 0 : 1, n = d == 0 ? B.n[0] : d == 1 ? B.n[1] : B.n[2];
  const int m = side ? a - n + 1 : -a;      // ghost layer
  const int f = 6 * b + 2 * d + side;
  for (int r = first[f]; r < first[f + 1]; ++r) {
    const PatchDesc& P = patches[r];
    const int lo1 = d == 0 ? P.lo[1] : P.lo[0], hi1 = d == 0 ? P.hi[1] : P.hi[0];
    const int lo2 = d == 2 ? P.lo[1] : P.lo[2], hi2 = d == 2 ? P.hi[1] : P.hi[2];
    if (p1 < lo1 || p1 >= hi1 || p2 < lo2 || p2 >= hi2) continue;
    if (P.kind == 0) {
      const BlockDesc& N = blocks[P.nbr];
      const int nn = d == 0 ? N.n[0] : d == 1 ? N.n[1] : N.n[2];
      const int o1 = d == 0 ? P.noff[1] : P.noff[0], o2 = d == 2 ? P.noff[1] : P.noff[2];
      const int64_t os = N.qoff + pos3(d, side ? m - 1 : nn - m, p1 + o1, p2 + o2, N.sj, N.sk);
#pragma unroll
      for (int v = 0; v < NV; ++v) g[v] = q[v * N.sv + os];
      return true;
    }
    const double* mb = met + B.moff;
    const int64_t of = pos3(d, side ? n : 0, p1, p2, B.sj, B.sk);
    const double sx = mb[(3 * d) * B.sv + of], sy = mb[(3 * d + 1) * B.sv + of], sz = mb[(3 * d + 2) * B.sv + of];
    const bool first_cell = P.kind == CFD_BC_KIND_FARFIELD || P.kind == CFD_BC_KIND_EXTRAP;
    const int c = first_cell ? 1 : m;         // interior layer the ghost depends on
    const int64_t os = B.qoff + pos3(d, side ? n - c : c - 1, p1, p2, B.sj, B.sk);
    double w[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) w[v] = q[v * B.sv + os];
    const double nrm = sqrt(sx * sx + sy * sy + sz * sz);
    const double nx = sx / nrm, ny = sy / nrm, nz = sz / nrm;
    if (P.kind == CFD_BC_KIND_FARFIELD) {
      const double s = side ? 1.0 : -1.0;
      const FarState far = farfield_call(w[0], w[1], w[2], w[3], w[4], s * nx, s * ny, s * nz, gamma, P.uinf[0],
                                         P.uinf[1], P.uinf[2]);
#pragma unroll
      for (int v = 0; v < NV; ++v) g[v] = far.q[v];
    } else {
      // by selection: as branches on the kind, the compiler formed the no-slip
      // wall's negated momentum only in lanes that another branch excludes, and
      // such ghosts held what the registers held
      double wall[NV];
      wall_state(CFD_BC_KIND_SLIPWALL, w, nx, ny, nz, wall);
      const bool slip = P.kind == CFD_BC_KIND_SLIPWALL, same = P.kind == CFD_BC_KIND_EXTRAP;
#pragma unroll
      for (int v = 0; v < NV; ++v) g[v] = slip ? wall[v] : same || v == 0 || v == NV - 1 ? w[v] : -w[v];
    }
    return true;
  }
  return false;
}

}  // namespace cfd
