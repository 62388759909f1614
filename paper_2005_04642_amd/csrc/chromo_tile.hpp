// Tile form of the time step, for lattices too small for the march of
// chromo_kernels.hpp to amortise its pipeline fill.
//
// A workgroup owns a tile of lattice sites and works on the tile's region: the
// tile with H = r_g + r_K + r_u more columns and rows on every side.  The
// region is 64 columns wide, one wavefront per row, and wave w takes rows w,
// w + 16, ... of it (NSLOT of them), the same rows in every phase, so that all
// a site hands from one phase to the next stays in its thread's registers (FP64
// spills 4 of 128 VGPRs between walls and 2 with a mask, pass 1 there 4 of 256);
// only the six stencil operands go through LDS.  Four phases, three barriers:
//   gather of the whole region, colour densities, rho^N, Phi' (all rows' words
//     in flight at once in the step);
//   grad rho^N and the director, on the region less r_g;
//   curvature, force and velocity, on the tile and r_u more;
//   correction, collision, recolour and store of the tile.
// A site's arithmetic is the march's own functions on the same operands, so
// its results do not depend on which form ran.
//
// What bounds it: on lattices of a few thousand sites the chain of one launch,
// one gather and three barriers (64^2 FP32 16.0 us per step as a march, whose
// shortest chunk takes seven iterations of three barriers; 6.8 us as tiles);
// at one tile per CU the arithmetic, about half of it on halo sites (512^2
// FP32 22.1 -> 14.5 us, FP64 39.3 -> 29.4).  64 columns and 16 waves because
// every CU should get a tile on 512^2: wider regions leave too few tiles, and
// 8 waves with twice the rows each are slower (512^2 16.7 us).
#pragma once

#include "chromo_kernels.hpp"

namespace chromo {

namespace tile {

constexpr int COLS = 64;  // columns of a region row: one wavefront

enum { T_RHON, T_MX, T_MY, T_UX, T_UY, T_PHI, T_N };

template <typename T, int ROWS>
struct TileSmem {
  T lead[4];  // stencil taps of the first and last columns stay inside the arrays
  T d[T_N][ROWS][COLS];
  T tail[4];
};

template <bool MASK, int RS, typename T>
__device__ __forceinline__ void grad(int r, const T* s, int row, int tx, T& gx, T& gy) {
  if (r == 3) {
    ring_grad<3, 0, RS, 1, T, MASK>(s, row, tx, gx, gy);
  } else {
    ring_grad<1, 0, RS, 1, T, MASK>(s, row, tx, gx, gy);
  }
}

template <bool MASK, int RS, typename T>
__device__ __forceinline__ T div(int r, const T* sx, const T* sy, int row, int tx) {
  return r == 3 ? ring_div<3, 0, RS, 1, T, MASK>(sx, sy, row, tx) : ring_div<1, 0, RS, 1, T, MASK>(sx, sy, row, tx);
}

}  // namespace tile

// Tile `id` of one lattice.
template <typename ST, int NWV, int NSLOT, bool WALLS, int MODE, bool MASK>
__device__ __forceinline__ void tile_step(const StepArgs<typename ST::math>& a, const Radii& r, int id,
                                          tile::TileSmem<typename ST::math, NWV * NSLOT>& sm) {
  using T = typename ST::math;
  using namespace tile;
  const Geom& g = a.g;
  const Coef<T>& c = a.c;
  // fields need u at the tile's own sites only
  const int ru = MODE == MODE_FIELDS ? 0 : r.u;
  const int H = r.g + r.k + ru;
  Thread t;
  t.tx = threadIdx.x & (COLS - 1);
  t.ty = __builtin_amdgcn_readfirstlane(threadIdx.x / COLS);
  const int tx = t.tx;
  const int strip = id % g.nstrips, chunk = id / g.nstrips;
  const int x0 = strip * g.TX;
  const int txe = min(g.TX, g.nx - x0);
  const int col = tx - H;
  int xg = (x0 + col) % g.nx;
  if (xg < 0) xg += g.nx;
  t.xg = xg;
  const int E = (int)sizeof(typename ST::W);
  t.cols.o = xg * E;
  t.cols.m = (xg == 0 ? g.nx - 1 : xg - 1) * E;
  t.cols.p = (xg == g.nx - 1 ? 0 : xg + 1) * E;
  t.own = col >= 0 && col < txe;
  t.ya = chunk * g.TY;
  t.yb = min(g.F, t.ya + g.TY);
  const int RM = t.yb - t.ya + 2 * H;  // rows of the region

  const void* src = a.src;
  void* dst = MODE != MODE_STEP ? const_cast<void*>(a.src) : a.dst;

  // rows past the region repeat its last one (read, never used), so that every
  // load of the gather is unconditional and all of them are in flight at once
  T f[NSLOT][9], rR[NSLOT], rB[NSLOT], gnx[NSLOT], gny[NSLOT], fx[NSLOT], fy[NSLOT];
  int prow[NSLOT];
  bool refl[NSLOT];
#pragma unroll
  for (int k = 0; k < NSLOT; ++k) {
    RowTrack<WALLS> tr;
    tr.init(t.ya - H + min(t.ty + NWV * k, RM - 1), g);
    prow[k] = tr.phys(g);
    refl[k] = tr.refl(g);
  }
  // ---- gather: colour densities, rho^N, Phi' --------------------------------
  {
    unsigned bits[NSLOT];
    if constexpr (MASK) {
#pragma unroll
      for (int k = 0; k < NSLOT; ++k) bits[k] = bounce_bits_at(bounce_rsrc(a.bnc, g.plane), g, prow[k], xg);
    }
    if (a.force) {
#pragma unroll
      for (int k = 0; k < NSLOT; ++k) {
        const int site = prow[k] * g.nx + xg;
        fx[k] = a.force[site];
        fy[k] = a.force[g.plane + site];
      }
    }
    // rows whose words are in flight together: all of them, fewer where the
    // local backward needs the registers
    constexpr int GD = MODE == MODE_ADJ ? (NSLOT % 2 ? 1 : 2) : (NSLOT > 4 ? NSLOT / 2 : NSLOT);
#pragma unroll
    for (int k0 = 0; k0 < NSLOT; k0 += GD) {
      typename ST::W pw[GD][ST::NW];
#pragma unroll
      for (int j = 0; j < GD; ++j)
        gather_words<ST, WALLS, MASK>(src, g, prow[k0 + j], t.cols, pw[j], MASK ? bits[k0 + j] : 0u);
#pragma unroll
      for (int j = 0; j < GD; ++j) {
        const int k = k0 + j, q = t.ty + NWV * k;
        T pr[9], pb[9];
        decode<ST>(pw[j], c, pr, pb, f[k]);
        rR[k] = density(pr);
        rB[k] = density(pb);
        sm.d[T_RHON][q][tx] = colour_index(rR[k] * c.inv_rho0R, rB[k] * c.inv_rho0B);
        if (MODE != MODE_FIELDS) sm.d[T_PHI][q][tx] = phi_prime<MASK>(c, rR[k], rB[k]);
      }
    }
  }
  __syncthreads();

  // ---- grad rho^N and director ------------------------------------------------
#pragma unroll
  for (int k = 0; k < NSLOT; ++k) {
    const int q = t.ty + NWV * k;
    if (q >= r.g && q < RM - r.g && tx >= r.g && tx < COLS - r.g) {
      grad<MASK, COLS>(r.g, &sm.d[T_RHON][0][0], q, tx, gnx[k], gny[k]);
      T mx, my;
      director<MASK>(c, gnx[k], gny[k], MASK ? sm.d[T_RHON][q][tx] : T(0), mx, my);
      sm.d[T_MX][q][tx] = mx;
      sm.d[T_MY][q][tx] = my;
    }
  }
  __syncthreads();

  // ---- curvature, force, velocity ---------------------------------------------
  const int h2 = r.g + r.k;
  T Gx[NSLOT], Gy[NSLOT], ir[NSLOT], ux[NSLOT], uy[NSLOT];
#pragma unroll
  for (int k = 0; k < NSLOT; ++k) {
    const int q = t.ty + NWV * k;
    if (q >= h2 && q < RM - h2 && tx >= h2 && tx < COLS - h2) {
      T K;
      if (c.fixed_K) {
        K = c.K_fixed;
      } else {
        K = -div<MASK, COLS>(r.k, &sm.d[T_MX][0][0], &sm.d[T_MY][0][0], q, tx);
      }
      const bool ownrow = q >= H && q < RM - H;
      if (MODE == MODE_ADJ) {
        if (t.own && ownrow) adj::ws_row(a.out_save, g.nx, prow[k])[SV_K * g.nx + xg] = K;
      }
      const T rho = rR[k] + rB[k];
      force_velocity<MASK>(c, K, gnx[k], gny[k], a.force != nullptr, fx[k], fy[k], refl[k], f[k], rho, Gx[k], Gy[k],
                           ir[k], ux[k], uy[k]);
      if (MODE == MODE_FIELDS) {
        if (t.own && ownrow) {
          const int site = prow[k] * g.nx + xg;
          if (a.out_rho) a.out_rho[site] = rho;
          if (a.out_ux) a.out_ux[site] = ux[k];
          if (a.out_uy) a.out_uy[site] = uy[k];
          if (a.out_rhoN) a.out_rhoN[site] = sm.d[T_RHON][q][tx];
        }
      } else {
        sm.d[T_UX][q][tx] = ux[k];
        sm.d[T_UY][q][tx] = uy[k];
      }
    }
  }
  if constexpr (MODE == MODE_FIELDS) return;
  __syncthreads();

  // ---- correction, collision, recolour, store -----------------------------------
#pragma unroll
  for (int k = 0; k < NSLOT; ++k) {
    const int q = t.ty + NWV * k;
    if (q >= H && q < RM - H && t.own) {
      const int p = prow[k];
      T lam[18];
      if constexpr (MODE == MODE_ADJ) {
        const T* ln = a.lam_next + (size_t)p * 18 * g.nx + xg;
#pragma unroll
        for (int i = 0; i < 18; ++i) lam[i] = ln[i * g.nx];
      }
      T dPx, dPy;
      grad<MASK, COLS>(r.p, &sm.d[T_PHI][0][0], q, tx, dPx, dPy);
      const T theta = div<MASK, COLS>(r.u, &sm.d[T_UX][0][0], &sm.d[T_UY][0][0], q, tx);
      if (MODE == MODE_ADJ) {
        T* sv = adj::ws_row(a.out_save, g.nx, p) + xg;
        sv[SV_GNX * g.nx] = gnx[k];
        sv[SV_GNY * g.nx] = gny[k];
      }
      collide_store<ST, T, MODE, MASK>(a, dst, f[k], rR[k], rB[k], ux[k], uy[k], Gx[k], Gy[k], ir[k], dPx, dPy, theta,
                                       sm.d[T_RHON][q][tx], sm.d[T_MX][q][tx], sm.d[T_MY][q][tx], p, t, lam);
    }
  }
}

template <typename ST, int NWV, int NSLOT, bool WALLS, int MODE, bool MASK = false>
__global__ void __launch_bounds__(64 * NWV, 1) chromo_tile_kernel(StepArgs<typename ST::math> a, Radii r) {
  __shared__ tile::TileSmem<typename ST::math, NWV * NSLOT> sm;
  // contiguous runs of tiles per XCD, as in the march
  const int ntiles = a.g.nstrips * a.g.nchunks;
  const int per_xcd = (ntiles + 7) / 8;
  int block = blockIdx.x;
  if constexpr (MODE == MODE_ADJ) {
    if (adj::add_previous<64 * NWV>(a.prev, block)) return;
  }
  const int id = (block % 8) * per_xcd + block / 8;
  if (id >= ntiles) return;
  tile_step<ST, NWV, NSLOT, WALLS, MODE, MASK>(a, r, id, sm);
}

}  // namespace chromo
