// Passes 2-5 of the adjoint step (chromo_adjoint.hpp) in one kernel over tiles.
//
// A workgroup owns a tile of sites and works on its region: the tile with H =
// max(r_Phi, r_u) + r_K + r_g + 1 more columns and rows on every side (the
// chain of transposed stencils and the push).  As in the step's tile kernel
// (chromo_tile.hpp), the region is 64 columns wide, one wavefront per row, and
// wave w takes rows w, w + NWV, ... in every phase: what a site hands from one
// pass to the next stays in its thread's registers (FP64 in 16 waves spills 6 of
// 128 VGPRs between walls and 4 with a mask), the stencils' operands go through
// LDS, and every plane that passes 2-4 read is fetched up front, each
// only where it is used (lanes elsewhere hold an offset beyond the row's buffer
// resource, which fetches nothing).  The passes' intermediate planes (7 + 2 + 2
// per site, written once and read up to 24 times through the cache by the
// stencils) do not exist in memory.
//
// Same per-site functions and the same order of every stencil sum as the
// separate passes, so dL/d(pops) and dL/dG_ext are theirs bit for bit;
// dL/dsigma sums the same FP64 terms (Sum2): every tile leaves its part in the
// workspace, and the next kernel, the following step's pass 1 or sigma_kernel,
// adds the parts up.  (The last tile to finish doing so, found by an atomic
// count, cost 4 to 5 us per step.)
//
// What bounds it: on small lattices the chain of loads and five barriers (64^2
// FP32: four passes 14 us, this kernel 9); at one tile per CU the stencils'
// arithmetic and LDS reads, half of them on halo sites (512^2: 26.5 -> 20 us);
// on large lattices the planes' traffic, 28 of them read with the halo and 18
// written (4096^2: 1.18 -> 1.08 ms).  16 waves of 2 or 3 rows while one round
// of workgroups holds the lattice, 8 waves of 6 rows beyond: in FP32 two of those
// (74 KB of LDS each; FP64 148 KB) share a CU, one's loads under the other's
// arithmetic.
#pragma once

#include "chromo_adjoint.hpp"

namespace chromo {
namespace adj {

constexpr int TCOLS = 64;  // columns of a region row: one wavefront
constexpr int SIGMA_THREADS = 256;
static_assert(PART_PLANE == G_B, "the parts lie in planes the tail does not use");

// columns and rows by which a tile's region extends beyond the tile
__host__ __device__ inline int tail_halo(const Radii& r) { return (r.p > r.u ? r.p : r.u) + r.k + r.g + 1; }

// One row of the workspace as a buffer resource (all planes of the row).
template <typename T>
struct WsRow {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ WsRow(const T* ws, const Geom& g, int y) {
    const size_t rs = (size_t)WS_PLANES * (size_t)g.nx;
    r = __builtin_amdgcn_make_buffer_rsrc((void*)(ws + (size_t)y * rs), (short)0, (int)(rs * sizeof(T)), 0x00020000);
  }
  // element of plane k at byte offset voff within the plane's row (NOWHERE: 0, not fetched)
  __device__ __forceinline__ T at(int k, int voff, const Geom& g) const {
    return load_word<T>(r, voff, (int)((unsigned)k * (unsigned)g.nx * (unsigned)sizeof(T)));
  }
};
constexpr int NOWHERE = 0x7ffffff0;

// grad_at's sums over an LDS field; s points at the site.
template <int R, typename T>
__device__ __forceinline__ void lds_grad(const T* s, T& gx, T& gy) {
  const T wd = T(1.0 / 36.0), wa = T(1.0 / 9.0);
  gx = T(0);
  gy = T(0);
#pragma unroll
  for (int n = 1; n <= R; ++n) {
    const T b = stencil_b<R, T>(n);
    const T* rp = s + n * TCOLS;
    const T* rm = s - n * TCOLS;
    const T d1 = rp[n] - rm[-n];
    const T d3 = rp[-n] - rm[n];
    const T d8 = s[n] - s[-n];
    const T d2 = rp[0] - rm[0];
    gx += b * (wd * (d1 - d3) + wa * d8);
    gy += b * (wd * (d1 + d3) + wa * d2);
  }
}

// gradT_walls_at's sums over an LDS field at fluid row `row` of F (F >= 4):
// each link's source row directly, and through the mirror beside a wall.
template <int R, typename T>
__device__ __forceinline__ void lds_gradT(const T* s, int row, int F, bool odd, T& tx, T& ty) {
  const T wd = T(1.0 / 36.0), wa = T(1.0 / 9.0);
  const T sg = odd ? T(-1) : T(1);
  const bool inner = row >= R && row + R < F;
  tx = T(0);
  ty = T(0);
#pragma unroll
  for (int n = 1; n <= R; ++n) {
    const T b = stencil_b<R, T>(n);
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      const int cx = link_cx(i), cy = link_cy(i);
      const T bw = b * ((i & 1) ? wd : wa);
      T v = T(0);
      if (inner) {
        v += s[-n * cy * TCOLS - n * cx];
      } else {
        const int y1 = row - n * cy;
        if (y1 >= 0 && y1 < F) v += s[-n * cy * TCOLS - n * cx];
        if (cy == -1 && row <= n - 1) v += sg * s[(n - 1 - 2 * row) * TCOLS - n * cx];
        if (cy == 1 && row >= F - n) v += sg * s[(2 * F - 1 - n - 2 * row) * TCOLS - n * cx];
      }
      tx += bw * T(cx) * v;
      ty += bw * T(cy) * v;
    }
  }
}

// solid_tap_weights' sums from the rows' solid sites as bit masks (bit =
// region column); m points at the site's row.
template <int R, typename T>
__device__ __forceinline__ void lds_tap_weights(const unsigned long long* m, int tx, T& wx, T& wy) {
  const T wd = T(1.0 / 36.0), wa = T(1.0 / 9.0);
  wx = T(0);
  wy = T(0);
#pragma unroll
  for (int n = 1; n <= R; ++n) {
    const T b = stencil_b<R, T>(n);
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      const int cx = link_cx(i), cy = link_cy(i);
      if ((m[n * cy] >> (tx + n * cx)) & 1ull) {
        const T bw = b * ((i & 1) ? wd : wa);
        wx += bw * T(cx);
        wy += bw * T(cy);
      }
    }
  }
}

// Fields in LDS; the second group takes the place of fields read by then.
enum { L_TH, L_DPX, L_DPY, L_K, L_JX, L_JY, L_N };
enum { L_CX = L_TH, L_CY = L_DPX, L_RR = L_DPY, L_RB = L_K };

template <typename T, int NWV, int NSLOT, bool W, bool M>
__global__ void __launch_bounds__(64 * NWV, 1)
    tail_kernel(Geom g, Coef<T> c, T sigma, Radii r, T* ws, T* __restrict__ out, T* __restrict__ dforce,
                const unsigned char* __restrict__ solid) {
  constexpr int ROWS = NWV * NSLOT;
  struct Lds {
    T lead[4];
    T d[L_N][ROWS][TCOLS];
    T trail[4];
  };
  __shared__ Lds sm;
  __shared__ unsigned long long wall[M ? ROWS : 1];  // solid sites of every region row
  __shared__ Sum2 red[NWV];
  const int ntiles = g.nstrips * g.nchunks;
  const int per_xcd = (ntiles + 7) / 8;
  const int id = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (id >= ntiles) return;
  const int tx = threadIdx.x & (TCOLS - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / TCOLS);
  const int r0 = max(r.p, r.u), r1 = r0 + r.k, r2 = r1 + r.g, H = r2 + 1;
  const int strip = id % g.nstrips, chunk = id / g.nstrips;
  const int x0 = strip * g.TX;
  const int nx = g.nx, ny = g.ny;
  const int col = tx - H;
  int xg = (x0 + col) % nx;
  if (xg < 0) xg += nx;
  const bool owncol = col >= 0 && col < min(g.TX, nx - x0);
  const int ya = chunk * g.TY, yb = min(g.F, ya + g.TY);
  const int RM = yb - ya + 2 * H;
  constexpr int E = (int)sizeof(T);

  // lattice row of every region row (W: v counts fluid rows, those outside
  // the strip do not exist)
  int prow[NSLOT];
  bool here[NSLOT];
#pragma unroll
  for (int k = 0; k < NSLOT; ++k) {
    const int q = w + NWV * k;
    const int v = ya - H + q;
    if constexpr (W) {
      here[k] = q < RM && v >= 0 && v < g.F;
      prow[k] = here[k] ? v + 1 : 1;
    } else {
      here[k] = q < RM;
      const int m = v % ny;
      prow[k] = m < 0 ? m + ny : m;
    }
  }
  auto inside = [&](int k, int h) {
    const int q = w + NWV * k;
    return here[k] && q >= h && q < RM - h && tx >= h && tx < TCOLS - h;
  };
  auto own = [&](int k) {
    const int q = w + NWV * k;
    return here[k] && owncol && q >= H && q < RM - H;
  };

  // ---- every plane the first three phases read, each only where it is used -----
  T s[NSLOT][SV_N], a[NSLOT][A_N];
  bool sol[NSLOT];
  {
    T th[NSLOT], px[NSLOT], py[NSLOT];
#pragma unroll
    for (int k = 0; k < NSLOT; ++k) {
      const WsRow<T> row(ws, g, prow[k]);
      const int o = here[k] ? xg * E : NOWHERE;
      th[k] = row.at(G_A + A_TH, o, g);
      px[k] = row.at(G_A + A_DPX, o, g);
      py[k] = row.at(G_A + A_DPY, o, g);
      sol[k] = false;
      if constexpr (M) sol[k] = solid[(size_t)prow[k] * nx + xg] != 0;
    }
#pragma unroll
    for (int k = 0; k < NSLOT; ++k) {
      const WsRow<T> row(ws, g, prow[k]);
      const int o0 = inside(k, r0) ? xg * E : NOWHERE;
      const int o1 = inside(k, r1) ? xg * E : NOWHERE;
      const int o2 = inside(k, r2) ? xg * E : NOWHERE;
#pragma unroll
      for (int j = 0; j < SV_N; ++j) s[k][j] = row.at(G_SV + j, o0, g);
#pragma unroll
      for (int j = A_RR; j <= A_GY; ++j) a[k][j] = row.at(G_A + j, o0, g);
      a[k][A_MX] = row.at(G_A + A_MX, o1, g);
      a[k][A_MY] = row.at(G_A + A_MY, o1, g);
      a[k][A_RN] = row.at(G_A + A_RN, o2, g);
    }
#pragma unroll
    for (int k = 0; k < NSLOT; ++k) {
      const int q = w + NWV * k;
      sm.d[L_TH][q][tx] = th[k];
      sm.d[L_DPX][q][tx] = px[k];
      sm.d[L_DPY][q][tx] = py[k];
      if constexpr (M) {
        const unsigned long long b = __ballot(sol[k]);
        if (tx == 0) wall[q] = b;
      }
    }
  }
  __syncthreads();

  // transposed stencils of one LDS field at the site (k, tx)
  auto minus_grad = [&](int radius, int field, int k, T& gx, T& gy) {  // periodic: the transpose is -grad
    const T* p = &sm.d[field][w + NWV * k][tx];
    if (radius == 3) {
      lds_grad<3>(p, gx, gy);
    } else {
      lds_grad<1>(p, gx, gy);
    }
  };
  auto walls_gradT = [&](int radius, int field, int k, bool odd, T& gx, T& gy) {
    const T* p = &sm.d[field][w + NWV * k][tx];
    if (radius == 3) {
      lds_gradT<3>(p, prow[k] - 1, g.F, odd, gx, gy);
    } else {
      lds_gradT<1>(p, prow[k] - 1, g.F, odd, gx, gy);
    }
  };
  auto tap_weights = [&](int radius, int k, T& wx, T& wy) {
    const unsigned long long* m = &wall[M ? w + NWV * k : 0];
    if (radius == 3) {
      lds_tap_weights<3>(m, tx, wx, wy);
    } else {
      lds_tap_weights<1>(m, tx, wx, wy);
    }
  };

  // the push's adjoints of f_i, fetched over pass 4, or, where the lattice has
  // walls, from here: there the stencils of passes 2 and 3 take long enough to
  // hide them (FP32 walled adjoint step 512^2 66.3 -> 62.4 us, 2048^2 947 -> 867;
  // earlier on periodic lattices 45.6 -> 46.9, masks spill, FP64 5 % slower)
  constexpr bool EARLY = W && sizeof(T) == 4;
  T lf[NSLOT][9];
  unsigned bounce[NSLOT];  // bit i: the word of link i is bounced back at its own site
  auto load_f = [&] {
#pragma unroll
    for (int k = 0; k < NSLOT; ++k) {
      const bool mine = own(k);
      const int y = prow[k];
      const int yp = y + 1 >= ny ? y + 1 - ny : y + 1, ym = y < 1 ? y - 1 + ny : y - 1;
      const WsRow<T> row0(ws, g, y), rowP(ws, g, yp), rowM(ws, g, ym);
      const int xp = xg + 1 >= nx ? xg + 1 - nx : xg + 1, xm = xg < 1 ? xg - 1 + nx : xg - 1;
      bounce[k] = 0u;
#pragma unroll
      for (int i = 0; i < 9; ++i) {
        const int cx = link_cx(i), cy = link_cy(i);
        const int o = cx == 1 ? xp : (cx == -1 ? xm : xg);
        bool b = false;
        if constexpr (W) b = (cy == -1 && y == 1) || (cy == 1 && y == ny - 2);
        if constexpr (M) b = mine && (i != 0) && ((wall[min(max(w + NWV * k + cy, 0), ROWS - 1)] >> (tx + cx)) & 1ull);
        if (b) bounce[k] |= 1u << i;
        if constexpr (W) {
          lf[k][i] = (b ? row0 : (cy == 1 ? rowP : (cy == -1 ? rowM : row0)))
                         .at(G_A + A_F + (b ? link_opp(i) : i), mine ? (b ? xg : o) * E : NOWHERE, g);
        } else {
          lf[k][i] = (cy == 1 ? rowP : (cy == -1 ? rowM : row0)).at(G_A + A_F + i, mine && !b ? o * E : NOWHERE, g);
          if constexpr (M) {
            const T own_word = row0.at(G_A + A_F + link_opp(i), b ? xg * E : NOWHERE, g);
            lf[k][i] = b ? own_word : lf[k][i];
          }
        }
      }
    }
  };
  if constexpr (EARLY) load_f();

  // ---- pass 2 ---------------------------------------------------------------------
  T bgx[NSLOT], bgy[NSLOT], brr[NSLOT], brb[NSLOT];
  Sum2 acc = {0.0, 0.0};
#pragma unroll
  for (int k = 0; k < NSLOT; ++k) {
    const int q = w + NWV * k;
    if (!inside(k, r0)) continue;
    if (M && sol[k]) {
      sm.d[L_K][q][tx] = sm.d[L_JX][q][tx] = sm.d[L_JY][q][tx] = T(0);
      continue;
    }
    T lux, luy, lphi, ax, ay, bx, by;
    if constexpr (W) {
      walls_gradT(r.u, L_TH, k, false, ax, ay);
      walls_gradT(r.u, L_TH, k, true, bx, by);
      lux = a[k][A_UX] + ax;
      luy = a[k][A_UY] + by;
      walls_gradT(r.p, L_DPX, k, false, ax, ay);
      walls_gradT(r.p, L_DPY, k, false, bx, by);
      lphi = ax + by;
    } else {
      minus_grad(r.u, L_TH, k, ax, by);
      if constexpr (M) {
        T wx, wy;
        tap_weights(r.u, k, wx, wy);
        const T lth = sm.d[L_TH][q][tx];
        lux = a[k][A_UX] - ax + lth * wx;
        luy = a[k][A_UY] - by + lth * wy;
        tap_weights(r.p, k, wx, wy);
        minus_grad(r.p, L_DPX, k, ax, ay);
        minus_grad(r.p, L_DPY, k, bx, by);
        const T dv = ax + by;
        lphi = -dv + sm.d[L_DPX][q][tx] * wx + sm.d[L_DPY][q][tx] * wy;
      } else {
        lux = a[k][A_UX] - ax;
        luy = a[k][A_UY] - by;
        minus_grad(r.p, L_DPX, k, ax, ay);
        minus_grad(r.p, L_DPY, k, bx, by);
        lphi = -(ax + by);
      }
    }
    const Pass2<T> p = pass2_site(c, sigma, a[k], s[k], 1, lux, luy, lphi);
    bgx[k] = p.b[B_GX];
    bgy[k] = p.b[B_GY];
    brr[k] = p.b[B_RR];
    brb[k] = p.b[B_RB];
    sm.d[L_K][q][tx] = p.b[B_K];
    sm.d[L_JX][q][tx] = p.b[B_JX];
    sm.d[L_JY][q][tx] = p.b[B_JY];
    if (own(k)) {
      if (dforce) {
        const int site = prow[k] * nx + xg;
        dforce[site] += p.lGx;
        dforce[g.plane + site] += p.lGy;
      }
      const Sum2 t = two_sum(acc.hi, p.dsig);
      acc = {t.hi, acc.lo + t.lo};
    }
  }
  acc = wave_sum2(acc, acc.hi);
  if (tx == 0) red[w] = acc;
  __syncthreads();
  if (w == NWV - 1) {
    const Sum2 part = tx < NWV ? red[tx] : Sum2{0.0, 0.0};
    const Sum2 tot = wave_sum2(part, part.hi);
    if (tx == 0) *sigma_part(ws, g, strip, chunk) = tot;
  }

  // ---- pass 3 ---------------------------------------------------------------------
#pragma unroll
  for (int k = 0; k < NSLOT; ++k) {
    const int q = w + NWV * k;
    if (!inside(k, r1)) continue;
    T cx = T(0), cy = T(0);
    if (!(M && sol[k])) {
      T kx, ky;
      if constexpr (W) {
        T ax, ay, bx, by;
        walls_gradT(r.k, L_K, k, false, ax, ay);
        walls_gradT(r.k, L_K, k, true, bx, by);
        kx = -ax;
        ky = -by;
      } else {
        minus_grad(r.k, L_K, k, kx, ky);
        if constexpr (M) {
          T wx, wy;
          tap_weights(r.k, k, wx, wy);
          const T lk = sm.d[L_K][q][tx];
          kx -= lk * wx;
          ky -= lk * wy;
        }
      }
      pass3_site(c, a[k], s[k], 1, bgx[k], bgy[k], kx, ky, cx, cy);
    }
    sm.d[L_CX][q][tx] = cx;
    sm.d[L_CY][q][tx] = cy;
  }
  if constexpr (!EARLY) load_f();
  __syncthreads();

  // ---- pass 4 ---------------------------------------------------------------------
#pragma unroll
  for (int k = 0; k < NSLOT; ++k) {
    const int q = w + NWV * k;
    if (!inside(k, r2)) continue;
    T drr = T(0), drb = T(0);
    if (!(M && sol[k])) {
      T ax, ay, bx, by, dv;
      if constexpr (W) {
        walls_gradT(r.g, L_CX, k, false, ax, ay);
        walls_gradT(r.g, L_CY, k, false, bx, by);
        dv = -(ax + by);
      } else {
        minus_grad(r.g, L_CX, k, ax, ay);
        minus_grad(r.g, L_CY, k, bx, by);
        dv = ax + by;
        if constexpr (M) {
          T wx, wy;
          tap_weights(r.g, k, wx, wy);
          dv = dv - sm.d[L_CX][q][tx] * wx - sm.d[L_CY][q][tx] * wy;
        }
      }
      pass4_site(c, a[k], s[k], 1, brr[k], brb[k], dv, drr, drb);
    }
    sm.d[L_RR][q][tx] = drr;
    sm.d[L_RB][q][tx] = drb;
  }
  __syncthreads();

  // ---- pass 5 ---------------------------------------------------------------------
#pragma unroll
  for (int k = 0; k < NSLOT; ++k) {
    if (!own(k)) continue;
    const int q = w + NWV * k;
    T* o = out + (size_t)prow[k] * 18 * nx + xg;
    if (M && sol[k]) {
#pragma unroll
      for (int i = 0; i < 18; ++i) o[i * nx] = T(0);
      continue;
    }
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const bool b = (W || M) && ((bounce[k] >> i) & 1u);
      const int cx = link_cx(i), cy = link_cy(i);
      const int at = b ? 0 : cy * TCOLS + cx;
      const T fx = b ? T(-cx) : T(cx), fy = b ? T(-cy) : T(cy);  // the pulling link's velocity
      const T common = lf[k][i] + fx * (&sm.d[L_JX][q][tx])[at] + fy * (&sm.d[L_JY][q][tx])[at];
      o[i * nx] = common + (&sm.d[L_RR][q][tx])[at];
      o[(9 + i) * nx] = common + (&sm.d[L_RB][q][tx])[at];
    }
  }
  if constexpr (W) {  // the wall rows' words are read by no fluid site
    if (owncol && ((ya == 0 && w == 0) || (yb == g.F && w == 1))) {
      T* o = out + (size_t)(w == 0 ? 0 : ny - 1) * 18 * nx + xg;
#pragma unroll
      for (int i = 0; i < 18; ++i) o[i * nx] = T(0);
    }
  }
}

// the parts of one adjoint step, added to *dsigma
template <typename T>
__global__ void __launch_bounds__(SIGMA_THREADS) sigma_kernel(SigmaParts<T> p) {
  add_sigma_parts<SIGMA_THREADS>(p);
}

}  // namespace adj
}  // namespace chromo
