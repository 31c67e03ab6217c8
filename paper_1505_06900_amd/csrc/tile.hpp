// Tiles of the 3D kernels that march along z: a block updates 64 columns (a row
// segment starting at a multiple of 64) by TY rows through a chunk of a.lz planes,
// and brings the populations of the tile and of its one-node rim into LDS plane by
// plane.  TY + 2 waves hold the tile's columns of rows y0 - 1 .. y0 + TY (a wave per
// row) and one more wave the two columns beside the tile.  TY = kNarrowRows is the
// narrow tile: 32 columns, two rows a wave.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "kernels.hpp"

namespace lbrr {

template <int TY>
struct Tile {
  static constexpr int kWidth = TY == kNarrowRows ? 32 : 64;  // columns of the tile
  static constexpr int kPerWave = 64 / kWidth;                // rows a wave holds
  static constexpr int kRows = TY + 2, kCols = kWidth + 2;    // patch in LDS: the tile and its rim
  static constexpr int kRowWaves = kRows / kPerWave;
  static_assert(kRows % kPerWave == 0, "whole waves of rows");
  static_assert(2 * kRows <= 64, "one wave holds both rim columns of every patch row");
  bool empty;       // block past the last tile row
  int lane;         // column of the tile this thread holds
  int r, col;       // the node this thread brings: patch row, LDS column,
  int px, py;       //   lattice node
  bool writes;      //   inside the patch
  bool inner;       // this thread updates a node of the tile: (x, y), LDS (lane + 1, r)
  int x, y;
  int z0, z1;       // planes of the chunk

  // Blocks reach the eight XCDs round-robin by id, and each XCD has its own
  // L2: blocks b and b + 8 take x-neighbouring tiles of one tile row, so the rim
  // columns a block reads are lines its XCD's L2 holds for the neighbour.  Tile
  // rows past the last of a group of eight are empty.
  __device__ __forceinline__ explicit Tile(const StepArgs& a) {
    const int thread = int(threadIdx.x) & 63;  // of its wave
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    lane = thread & (kWidth - 1);
    const int gx = (a.nx + kWidth - 1) / kWidth, gy = (a.ny + TY - 1) / TY, gz = (a.nz + a.lz - 1) / a.lz;
    const int b = int(blockIdx.x);
    const int bxi = (b / 8) % gx, g = (b / (8 * gx)) * 8 + b % 8;
    empty = g >= gy * gz;
    const int byi = g % gy, bz = g / gy;
    const int x0 = bxi * kWidth, y0 = byi * TY;
    const int width = (a.nx - x0 < kWidth) ? a.nx - x0 : kWidth;
    if (wave < kRowWaves) {
      r = kPerWave == 1 ? wave : wave * kPerWave + thread / kWidth;
      writes = lane < width;
      col = lane + 1;
      px = x0 + (writes ? lane : 0);
    } else {
      const bool left = thread < kRows;
      writes = thread < 2 * kRows;
      r = left ? thread : (writes ? thread - kRows : 0);
      col = left ? 0 : width + 1;
      px = wrap_axis(left ? x0 - 1 : x0 + width, a.nx);
    }
    py = wrap_axis(y0 - 1 + r, a.ny);
    x = x0 + lane;
    y = y0 + r - 1;
    inner = wave < kRowWaves && r >= 1 && r <= TY && lane < width && y < a.ny;
    z0 = bz * a.lz;
    z1 = (z0 + a.lz < a.nz) ? z0 + a.lz : a.nz;
  }
  // blocks of a launch, all tiles dealt to the XCDs in groups of eight tile rows
  static int64_t blocks(const StepArgs& a) {
    const int64_t rows = int64_t((a.ny + TY - 1) / TY) * ((a.nz + a.lz - 1) / a.lz);
    return int64_t((a.nx + kWidth - 1) / kWidth) * 8 * ((rows + 7) / 8);
  }
  static constexpr int threads() { return 64 * (kRowWaves + 1); }
};

// What an inner thread keeps of the layer c_z = CZ that arrived at its node: the
// sums the moments need, or, where a node may lie on a wall and is completed from
// its populations one by one, the arrivals themselves.
template <class L, int CZ, class R>
struct LayerTotals : LayerSums<R> {
  template <class G>
  __device__ __forceinline__ void read(G&& get) {
    static_cast<LayerSums<R>&>(*this) = layer_sums<L, CZ, R>(get);
  }
};
template <class L, int CZ, class R>
struct LayerValues {
  R v[9];  // [c_x + 1 + 3 (c_y + 1)], the velocities the lattice has
  template <class G>
  __device__ __forceinline__ void read(G&& get) {
    sfor<0, 9>([&](auto K) {
      constexpr int i = velocity_index<L>(int(K) % 3 - 1, int(K) / 3 - 1, CZ);
      if constexpr (i >= 0) v[K] = get(std::integral_constant<int, i>{});
    });
  }
  __device__ __forceinline__ void put(R (&f)[L::Q]) const {
    sfor<0, 9>([&](auto K) {
      constexpr int i = velocity_index<L>(int(K) % 3 - 1, int(K) / 3 - 1, CZ);
      if constexpr (i >= 0) f[i] = v[K];
    });
  }
};
template <class L, int CZ, class R, bool W>
using Layer = std::conditional_t<W, LayerValues<L, CZ, R>, LayerTotals<L, CZ, R>>;

// Moments of a node from its three layers (W: on sides sx, sy, sz of the box).
template <class L, class R, bool W>
__device__ __forceinline__ Moments<R> layer_moments(const Layer<L, -1, R, W>& lo, const Layer<L, 0, R, W>& mid,
                                                    const Layer<L, 1, R, W>& up, int sx, int sy, int sz) {
  if constexpr (W) {
    R g[L::Q];
    lo.put(g);
    mid.put(g);
    up.put(g);
    const R drho = complete_walls<L, R>(g, sx, sy, sz);
    return moments_walls<L, R>(g, drho, sx, sy, sz);
  } else {
    return join_layers<L, R>(lo, mid, up);
  }
}

}  // namespace lbrr
