// Batched step: marches and tiles of many lattices in one launch.
#pragma once

#include "chromo_tile.hpp"

namespace chromo {

// ---------------------------------------------------------------------------
// Batched step: many independent lattices in one launch.  Each
// workgroup owns a bin of work items (lattice, tile), planned on the host so
// that the bins' costs are balanced, and runs them one after the other.
// ---------------------------------------------------------------------------
template <typename T>
struct SimDesc {
  Geom g;                 // per-lattice geometry and tile plan
  Coef<T> c;              // per-lattice constants
  unsigned long long off; // byte offset of the lattice's populations in both packed buffers
  const T* force;         // per-site force density [2][ny][nx] of the lattice, or null
  const unsigned char* bnc;  // bounce bits of the lattice's solid-site mask, or null
};

template <typename T>
struct BatchArgs {
  const char* src;              // packed population buffers
  char* dst;
  const SimDesc<T>* sims;
  const int* bin_start;         // [nbins + 1] offsets into items
  const int* items;             // pairs (lattice, tile)
};

// Region rows of a tile item of a batch: those of the tile kernel's taller
// shape, shared by the waves of the workgroup (12 with 4 rows each, or 8 with 6).
constexpr int BATCH_TILE_ROWS = 48;

// TILES: some of the plan's items are tiles (FP32 arithmetic; double has no
// registers for tiles of this height).  A plan of marches only takes the kernel
// without them: beside the tile's code the march itself runs 3 to 5 % slower
// (FP32, 1000 lattices of 64^2 at 128 columns 268 -> 257 us per step; 256 of
// them at stencil 1111 57.8 -> 56.3).
template <typename ST, int NTX, int NR, int RG, int RK, int RP, int RU, bool WALLS, bool MASK, bool TILES>
__global__ void __launch_bounds__(NTX * NR, 1) chromo_batch_kernel(BatchArgs<typename ST::math> b) {
  using T = typename ST::math;
  using PP = Pipe<NR>;
  static_assert(NTX > 2 * (RG + RK + RU), "strip must be wider than its halo");
  static_assert(!TILES || sizeof(T) == 4, "tile items need FP32 arithmetic");
  constexpr int NWV = NTX * NR / 64, NSLOT = BATCH_TILE_ROWS / NWV;
  constexpr Radii radii = {RG, RK, RP, RU};
  union Lds {
    Smem<T, NTX, PP::RING> march;
    tile::TileSmem<T, TILES ? NWV * NSLOT : 1> tile;
  };
  __shared__ Lds lds;
  Smem<T, NTX, PP::RING>& sm = lds.march;
  // The tables are never written while the kernel runs.  Kernels with FP32
  // arithmetic read them through the constant address space, by scalar loads
  // into scalar registers, as kernel arguments are (us per step, copied into
  // registers / that way: 48 periodic FP32 lattices of 64^2 to 512^2 138 / 120,
  // 24 masked ones at stencil 1111 68.7 / 61.8, 1000 FP16 ones of 64^2 240 /
  // 230), but for those that run slower so: walls (48 FP32 lattices 126 / 143),
  // and FP32 words without tiles or masks (1000 of 64^2 257 / 266).  FP64 (397 /
  // 416) copies them too.
  typedef const __attribute__((address_space(4))) int* ConstInts;
  typedef const __attribute__((address_space(4))) SimDesc<T>* ConstSims;
  constexpr bool SCALAR = sizeof(T) == 4 && !WALLS && (TILES || MASK || is_ofs16<ST>::value);
  const int k0 = b.bin_start[blockIdx.x], k1 = b.bin_start[blockIdx.x + 1];
  for (int k = k0; k < k1; ++k) {
    int sim, tile;
    SimDesc<T> d;
    if constexpr (SCALAR) {
      const ConstInts items = (ConstInts)(uintptr_t)b.items;
      sim = items[2 * k];
      tile = items[2 * k + 1];
      __builtin_memcpy(&d, (ConstSims)(uintptr_t)b.sims + sim, sizeof(d));
    } else {
      sim = b.items[2 * k];
      tile = b.items[2 * k + 1];
      d = b.sims[sim];
    }
    StepArgs<T> a;
    a.src = b.src + d.off;
    a.dst = b.dst + d.off;
    a.force = d.force;
    a.out_rho = a.out_ux = a.out_uy = a.out_rhoN = a.out_save = a.out_adj = nullptr;
    a.lam_next = nullptr;
    a.prev.ws = nullptr;
    a.bnc = d.bnc;
    a.g = d.g;
    a.c = d.c;
    // in a batch with masks, lattices without one take the plain march or tile
    const bool masked = MASK && a.bnc;
    if (TILES && a.g.tile) {
      if constexpr (TILES) {
        if (masked) {
          tile_step<ST, NWV, NSLOT, WALLS, MODE_STEP, MASK>(a, radii, tile, lds.tile);
        } else {
          tile_step<ST, NWV, NSLOT, WALLS, MODE_STEP, false>(a, radii, tile, lds.tile);
        }
      }
    } else if (masked) {
      march_tile<ST, NTX, NR, RG, RK, RP, RU, WALLS, MODE_STEP, MASK>(a, tile, sm);
    } else {
      march_tile<ST, NTX, NR, RG, RK, RP, RU, WALLS, MODE_STEP, false>(a, tile, sm);
    }
    __syncthreads();  // the next tile reuses the LDS rings
  }
}

}  // namespace chromo
