// Two steps of the population update in one launch (FP32 and FP64 storage,
// with or without walls; no walls for D3Q27 FP64).
//
// k_step moves the state through HBM once per step and is held by that
// traffic.  Here a block pulls and collides the nodes of a tile and of its
// one-node rim (first step) into LDS, and the tile's own nodes pull those
// populations and collide again (second step), so the state is read and
// written once for two steps.  Both collisions are the ones k_step runs, in
// the same operations and order, on values of the storage type: two steps here
// give the bits of two launches of k_step.
//
// D3Q27 order 4 FP32 at 256^3: 0.749 ms for two steps (44.8 GLUPS) against
// 2 x 0.614 ms (27.3).  rocprofv3 at 8 rows a block: reads 1.27x the state (rim rows and
// chunk edges), writes 1.00x, 4.11 GB at 5.5 TB/s; VALU busy 51%.  FP64: 1.54 ms against
// 2 x 1.34 ms, reads 1.55x, 6.0 TB/s.  So it is held by its traffic again, at 0.57 of
// the traffic of two single steps.
//
// FP16 storage keeps single steps: they are near their VALU bound (D3Q19 order 4: VALU
// issuing 86% of the launch), and a pair's rim adds a tenth to the collisions.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "tile.hpp"

namespace lbrr {

// Two steps in 3D on the tiles of tile.hpp.  The first step runs on the tile and
// its rim; its populations on plane p with c_z = +1, 0, -1 arrive on planes p + 1,
// p, p - 1: an inner thread keeps the layers of the planes it is waiting for and
// collides plane p - 1 when the c_z = -1 layer of plane p is there.  The pull of the
// next plane is issued as soon as the moments of the present one are formed, and
// is in flight through both collisions; the second collision follows the barrier
// that frees the LDS (before it: 44.1 -> 42.3 GLUPS, D3Q27 FP32 256^3).  W: resting
// walls on the axes of a.walls.
template <class L, int N, class S, int TY, bool W>
__global__ void __launch_bounds__(Tile<TY>::threads()) k_step_pair(const S* __restrict__ src, S* __restrict__ dst,
                                                             StepArgs a) {
  static_assert(L::D == 3, "3D lattices");
  using R = S;
  __shared__ R pop[L::Q][Tile<TY>::kRows][Tile<TY>::kCols];
  const Tile<TY> t(a);
  if (t.empty) return;
  // Byte offsets of the nodes populations come from, within a plane of one
  // population (pair_offsets_fit); plane and population
  // bases are block-uniform.
  const int px = t.px, py = t.py, r = t.r, lane = t.lane;
  const int xs[3] = {px == a.nx - 1 ? 0 : px + 1, px, px == 0 ? a.nx - 1 : px - 1};
  const int ys[3] = {py == a.ny - 1 ? 0 : py + 1, py, py == 0 ? a.ny - 1 : py - 1};
  uint32_t off[3][3];  // [c_y + 1][c_x + 1]
  sfor<0, 3>([&](auto Y) {
    sfor<0, 3>([&](auto X) { off[Y][X] = uint32_t((int64_t(ys[Y]) * a.sy + xs[X]) * int64_t(sizeof(S))); });
  });
  const uint32_t off_out = t.inner ? uint32_t((int64_t(t.y) * a.sy + t.x) * int64_t(sizeof(S))) : 0u;
  const R rho0 = R(a.rho0), om = R(a.omega1);
  // sides of the box of the first and the second node
  const int sx1 = W ? wall_side(a.walls, 0, px, a.nx) : 0, sy1 = W ? wall_side(a.walls, 1, py, a.ny) : 0;
  const int sx2 = W ? wall_side(a.walls, 0, t.x, a.nx) : 0, sy2 = W ? wall_side(a.walls, 1, t.y, a.ny) : 0;

  auto pull = [&](int z, R (&f)[L::Q]) __attribute__((always_inline)) {
    const int zs[3] = {z == a.nz - 1 ? 0 : z + 1, z, z == 0 ? a.nz - 1 : z - 1};
    // An empty asm hides that the offsets are the same in every plane, so that
    // each access keeps the form scalar base + 32-bit lane offset.
#pragma unroll
    for (int i = 0; i < 9; ++i) asm volatile("" : "+v"(off[i / 3][i % 3]));
    sfor<0, L::Q>([&](auto I) {
      constexpr int cx = L::cx(I), cy = L::cy(I), cz = L::cz(I);
      f[I] = at_offset(src + int64_t(I) * a.si + int64_t(zs[cz + 1]) * a.sz, off[cy + 1][cx + 1]);
    });
  };

  const int z0 = t.z0, z1 = t.z1, n = z1 - z0;
  // First-step planes z0 - 1 .. z1 (plane z0 - 1 + k, k = 0 .. n + 1), targets
  // z0 .. z1 - 1: plane k brings layer c_z = +1 to target k, 0 to target k - 1,
  // -1 to target k - 2, which is then complete.
  struct {  // a struct: a plain array carried around the loop ends in one 32-register tuple, copied whole
    R v[L::Q];
  } f;
  using Lo = Layer<L, -1, R, W>;
  using Mid = Layer<L, 0, R, W>;
  using Up = Layer<L, 1, R, W>;
  Up up1, up2;  // c_z = +1 layers of targets k - 1 and k - 2
  Mid mid2;     // c_z = 0 layer of target k - 2
  // Loads and stores complete in order under one counter: populations stored at
  // once are waited for with the pulled plane.  Stored late, they wait in registers
  // for the next iteration and go between the wait for its plane and the next pull.
  // Only where the registers hold them too: D3Q27 FP32 256^3 44.1 -> 44.6 GLUPS,
  // D3Q19 FP32 65 x 130 x 301 44.6 -> 45.8, walled 41.4 -> 43.6; FP64 D3Q19 +-1 %;
  // with spills (13 rows or walled D3Q27 FP32, D3Q27 FP64) 35 to 55 % are lost.
  constexpr bool kStoreLate = sizeof(S) == 4 && (L::Q == 27 ? !W : TY < 13);
  struct {
    R v[L::Q];
  } done;
  auto put = [&](int z, const R (&v)[L::Q]) __attribute__((always_inline)) {
    S* d = dst + int64_t(z) * a.sz;
    uint32_t o = off_out;
    asm volatile("" : "+v"(o));
    sfor<0, L::Q>([&](auto I) { __builtin_nontemporal_store(v[I], ptr_at_offset(d + int64_t(I) * a.si, o)); });
  };
  // First step of plane k into LDS; ZS selects all populations (2) or those
  // with c_z = ZS.  Next: pull plane k + 1 once the moments of plane k are formed.
  auto first = [&](int k, auto ZS, auto Next) __attribute__((always_inline)) {
    constexpr int Z = decltype(ZS)::value;
    Moments<R> m;
    if constexpr (W) {
      const int sz = wall_side(a.walls, 2, wrap_axis(z0 - 1 + k, a.nz), a.nz);
      const R drho = complete_walls<L, R>(f.v, sx1, sy1, sz);
      m = moments_walls<L, R>(f.v, drho, sx1, sy1, sz);
    } else {
      m = raw_moments<L, R>(f.v);
    }
    // the moments are pinned here, so that the pull can take the registers of f
    asm volatile("" : "+v"(m.d0), "+v"(m.jx), "+v"(m.jy), "+v"(m.jz), "+v"(m.pxx), "+v"(m.pyy), "+v"(m.pzz),
                 "+v"(m.pxy), "+v"(m.pxz), "+v"(m.pyz));
    if constexpr (kStoreLate)
      if (t.inner && k >= 3) put(z0 + k - 3, done.v);
    if constexpr (decltype(Next)::value) pull(wrap_axis(z0 + k, a.nz), f.v);
    const Hydro<R> h = hydro<L, R>(m, rho0);
    R C[3][3][3], out[L::Q];
    coefficients<L, N, R>(h, om, C);
    reconstruct<L, N, R, Z>(C, out);
    if (t.writes) {
      sfor<0, L::Q>([&](auto I) {
        if constexpr (Z == 2 || L::cz(I) == Z) pop[I][r][t.col] = out[I];
      });
    }
  };
  // population I arriving at the inner node
  auto arrived = [&](auto I) { return pop[I][r - L::cy(I)][lane + 1 - L::cx(I)]; };
  // second step of plane z from its layers
  auto second = [&](int z, const Lo& lo, const Mid& mid, const Up& up, R (&out)[L::Q]) __attribute__((always_inline)) {
    const int sz2 = W ? wall_side(a.walls, 2, z, a.nz) : 0;
    const Moments<R> m = layer_moments<L, R, W>(lo, mid, up, sx2, sy2, sz2);
    const Hydro<R> h = hydro<L, R>(m, rho0);
    R C[3][3][3];
    coefficients<L, N, R>(h, om, C);
    reconstruct<L, N, R>(C, out);
  };
  using all = std::integral_constant<int, 2>;
  using layer_m = std::integral_constant<int, -1>;
  using layer_p = std::integral_constant<int, 1>;
  pull(wrap_axis(z0 - 1, a.nz), f.v);
  first(0, layer_p{}, std::true_type{});
  lds_barrier();
  if (t.inner) up1.read(arrived);
  lds_barrier();
  for (int k = 1; k <= n; ++k) {
    first(k, all{}, std::true_type{});
    lds_barrier();
    Lo lo;
    Mid mid;
    Up up;
    if (t.inner) {
      lo.read(arrived);
      mid.read(arrived);
      up.read(arrived);
    }
    lds_barrier();
    if (t.inner) {
      if (k >= 2) {
        second(z0 + k - 2, lo, mid2, up2, done.v);
        if constexpr (!kStoreLate) put(z0 + k - 2, done.v);
      }
      up2 = up1;
      mid2 = mid;
      up1 = up;
    }
  }
  first(n + 1, layer_m{}, std::false_type{});
  lds_barrier();
  if (t.inner) {
    Lo lo;
    lo.read(arrived);
    R out[L::Q];
    second(z1 - 1, lo, mid2, up2, out);
    put(z1 - 1, out);
  }
}

// Two steps in 2D.  A block of kPairRowX threads runs the first step on a row of
// kPairRowX nodes (x0 - 1 .. x0 + kPairRowX - 2) and marches along y through a chunk
// of a.lz rows: the first step's populations on row p with c_y = +1, 0, -1
// arrive on rows p + 1, p, p - 1, so an inner thread keeps the three arrivals of
// each layer it is waiting for, and collides row p - 1 when row p is there.  The
// populations moving along y stay in their thread; the six others pass through
// LDS, in two buffers taken in turn (one barrier a row).  W: resting walls on the
// axes of a.walls.  The next row is pulled into the registers of the present one
// once its moments are formed (copied from a second set at the end of the loop, it
// was waited for there: 33.8 us); storing late as in k_step_pair loses 2 to 6 % on
// large grids.  Measured (pair_plan, api.hip): 2048^2 FP32 49.9 -> 32.5 us a step
// (129 GLUPS; 5.8 TB/s with the rows read twice), FP64 101 -> 61; small grids save
// a launch: 64^2 FP32 2.66 -> 1.92.
constexpr int kPairRowX = 256;

template <class L, int N, class S, bool W>
__global__ void __launch_bounds__(kPairRowX) k_step_pair2(const S* __restrict__ src, S* __restrict__ dst, StepArgs a) {
  static_assert(L::D == 2, "2D lattices");
  using R = S;
  constexpr int BX = kPairRowX;
  __shared__ R pop[2][6][BX];  // [c_y + 1 + (c_x > 0 ? 3 : 0)]
  const int tx = int(threadIdx.x);
  const int gx = (a.nx + BX - 3) / (BX - 2);
  const int bx = int(blockIdx.x) % gx, by = int(blockIdx.x) / gx;
  const int x0 = bx * (BX - 2);
  const int px = wrap_axis(x0 - 1 + tx, a.nx);
  const int xo = x0 + tx - 1;
  const bool inner = tx >= 1 && tx <= BX - 2 && xo < a.nx;
  uint32_t xs[3] = {uint32_t(px == a.nx - 1 ? 0 : px + 1) * uint32_t(sizeof(S)), uint32_t(px) * uint32_t(sizeof(S)),
                    uint32_t(px == 0 ? a.nx - 1 : px - 1) * uint32_t(sizeof(S))};
  const uint32_t off_out = uint32_t(xo) * uint32_t(sizeof(S));
  const R rho0 = R(a.rho0), om = R(a.omega1);
  const int sx1 = W ? wall_side(a.walls, 0, px, a.nx) : 0, sx2 = W ? wall_side(a.walls, 0, xo, a.nx) : 0;
  auto pull = [&](int y, R (&f)[L::Q]) __attribute__((always_inline)) {
    const int ys[3] = {y == a.ny - 1 ? 0 : y + 1, y, y == 0 ? a.ny - 1 : y - 1};
#pragma unroll
    for (int i = 0; i < 3; ++i) asm volatile("" : "+v"(xs[i]));  // keeps the scalar-base form (see k_step_pair)
    sfor<0, L::Q>([&](auto I) {
      constexpr int cx = L::cx(I), cy = L::cy(I);
      f[I] = at_offset(src + int64_t(I) * a.si + int64_t(ys[cy + 1]) * a.sy, xs[cx + 1]);
    });
  };
  // rows y0 .. y1 - 1; first-step rows y0 - 1 .. y1, row y0 - 1 + k of the march
  const int y0 = by * a.lz;
  const int y1 = (y0 + a.lz < a.ny) ? y0 + a.lz : a.ny;
  const int n = y1 - y0;
  struct {  // structs, as in k_step_pair
    R v[L::Q];
  } f;  // the pulled row
  struct {
    R v[3];  // arrivals with c_x = -1, 0, 1
  } up1, up2, mid2;
  // Moments of populations v of a node on row y, side sx of the box.
  auto moments = [&](R (&v)[L::Q], int sx, int y) __attribute__((always_inline)) {
    if constexpr (W) {
      const int sy = wall_side(a.walls, 1, y, a.ny);
      const R drho = complete_walls<L, R>(v, sx, sy, 0);
      return moments_walls<L, R>(v, drho, sx, sy, 0);
    } else {
      return raw_moments<L, R>(v);
    }
  };
  auto row = [&](int k, auto Next) __attribute__((always_inline)) {
    Moments<R> m = moments(f.v, sx1, wrap_axis(y0 - 1 + k, a.ny));
    asm volatile("" : "+v"(m.d0), "+v"(m.jx), "+v"(m.jy), "+v"(m.pxx), "+v"(m.pyy), "+v"(m.pxy));
    if constexpr (decltype(Next)::value) pull(wrap_axis(y0 + k, a.ny), f.v);
    R C[3][3][3], out[L::Q];
    coefficients<L, N, R>(hydro<L, R>(m, rho0), om, C);
    reconstruct<L, N, R>(C, out);
    const int b = k & 1;
    sfor<0, L::Q>([&](auto I) {
      constexpr int cx = L::cx(I), cy = L::cy(I);
      if constexpr (cx != 0) pop[b][cy + 1 + (cx > 0 ? 3 : 0)][tx] = out[I];
    });
    lds_barrier();
    if (inner) {
      // arrival from this row with velocity (c_x, c_y)
      auto arrived = [&](auto X, auto Y) {
        constexpr int cx = int(X) - 1, cy = int(Y) - 1;
        if constexpr (cx == 0) return out[velocity_index<L>(0, cy, 0)];
        else return pop[b][cy + 1 + (cx > 0 ? 3 : 0)][tx - cx];
      };
      using row_m = std::integral_constant<int, 0>;
      using row_0 = std::integral_constant<int, 1>;
      using row_p = std::integral_constant<int, 2>;
      if (k >= 2) {
        R g[L::Q];
        sfor<0, 3>([&](auto X) {
          constexpr int cx = int(X) - 1;
          g[velocity_index<L>(cx, 1, 0)] = up2.v[X];
          g[velocity_index<L>(cx, 0, 0)] = mid2.v[X];
          g[velocity_index<L>(cx, -1, 0)] = arrived(X, row_m{});
        });
        R D[3][3][3];
        coefficients<L, N, R>(hydro<L, R>(moments(g, sx2, y0 + k - 2), rho0), om, D);
        reconstruct<L, N, R>(D, g);
        S* d = dst + int64_t(y0 + k - 2) * a.sy;
        uint32_t o = off_out;
        asm volatile("" : "+v"(o));
        sfor<0, L::Q>([&](auto I) { __builtin_nontemporal_store(g[I], ptr_at_offset(d + int64_t(I) * a.si, o)); });
      }
      up2 = up1;
      sfor<0, 3>([&](auto X) {
        mid2.v[X] = arrived(X, row_0{});
        up1.v[X] = arrived(X, row_p{});
      });
    }
  };
  pull(wrap_axis(y0 - 1, a.ny), f.v);
  for (int k = 0; k <= n; ++k) row(k, std::true_type{});
  row(n + 1, std::false_type{});
}

// Walled boxes: D3Q27 FP64 would spill 25-69 registers and ran slower than single
// steps (256^3, walls along z: 12.7 -> 11.7 GLUPS), so it has no such form.
template <class L, class S>
constexpr bool pair_has_walls() {
  return !(L::Q == 27 && sizeof(S) == 8);
}

// Tile heights the host chooses from (pair_plan in api.hip).  GLUPS at 256^3,
// order 4, by rows: D3Q27 FP32 5 / 7 / 8 / 9 / 10 rows 40.4 / 38.7 / 43.6 / 40.6 / 31.9 (10 and
// more rows spill: 128 VGPRs), D3Q19 FP32 5 / 8 / 9 / 11 / 13 rows 57.1 / 56.7 / 56.5 /
// 59.4 / 60.6, D3Q27 FP64 3 / 4 / 5 rows 19.8 / 21.5 / 20.4, D3Q19 FP64 29.1 / 32.5 / 29.2 (6
// rows spill).  The second height serves boxes whose rows the first divides badly.
template <class L, class S>
constexpr int pair_rows_option(int i) {
  if (L::D == 2) return i == 0 ? 1 : 0;
  if (sizeof(S) == 8) return i == 0 ? 4 : (i == 1 ? 3 : 0);
  if (L::Q == 19) return i == 0 ? 13 : (i == 1 ? 9 : 0);
  return i == 0 ? 8 : (i == 1 ? 9 : 0);
}

template <class L, int N, class S, int TY>
hipError_t launch_step_pair(const void* src, void* dst, const StepArgs& a, hipStream_t s) {
  if (a.lz < 1) return hipErrorInvalidValue;
  if (!pair_offsets_fit(L::D, a, int(sizeof(S)))) return hipErrorInvalidValue;
  if constexpr (L::D == 2) {
    const int64_t nb = int64_t((a.nx + kPairRowX - 3) / (kPairRowX - 2)) * ((a.ny + a.lz - 1) / a.lz);
    if (nb >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    if (a.walls)
      hipLaunchKernelGGL((k_step_pair2<L, N, S, true>), dim3(unsigned(nb)), dim3(kPairRowX), 0, s,
                         static_cast<const S*>(src), static_cast<S*>(dst), a);
    else
      hipLaunchKernelGGL((k_step_pair2<L, N, S, false>), dim3(unsigned(nb)), dim3(kPairRowX), 0, s,
                         static_cast<const S*>(src), static_cast<S*>(dst), a);
    return hipGetLastError();
  } else {
    const int64_t blocks = Tile<TY>::blocks(a);
    if (blocks >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    if (a.walls) {
      if constexpr (pair_has_walls<L, S>()) {
        hipLaunchKernelGGL((k_step_pair<L, N, S, TY, true>), dim3(unsigned(blocks)), dim3(Tile<TY>::threads()), 0, s,
                           static_cast<const S*>(src), static_cast<S*>(dst), a);
        return hipGetLastError();
      }
      return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL((k_step_pair<L, N, S, TY, false>), dim3(unsigned(blocks)), dim3(Tile<TY>::threads()), 0, s,
                       static_cast<const S*>(src), static_cast<S*>(dst), a);
    return hipGetLastError();
  }
}

template <class L, int N, class S>
hipError_t step_pair_by_rows(const void* src, void* dst, const StepArgs& a, hipStream_t s) {
  if (a.rows == pair_rows_option<L, S>(0)) return launch_step_pair<L, N, S, pair_rows_option<L, S>(0)>(src, dst, a, s);
  if constexpr (L::D == 3) {
    if (a.rows == pair_rows_option<L, S>(1))
      return launch_step_pair<L, N, S, pair_rows_option<L, S>(1)>(src, dst, a, s);
  }
  return hipErrorInvalidValue;
}

template <class L, class S>
hipError_t step_pair_by_order(int order, const void* src, void* dst, const StepArgs& a, hipStream_t s) {
  switch (order) {
    case 2: return step_pair_by_rows<L, 2, S>(src, dst, a, s);
    case 3: return step_pair_by_rows<L, 3, S>(src, dst, a, s);
    case 4: return step_pair_by_rows<L, 4, S>(src, dst, a, s);
    case 5: if constexpr (L::NMAX >= 5) return step_pair_by_rows<L, 5, S>(src, dst, a, s); break;
    case 6: if constexpr (L::NMAX >= 6) return step_pair_by_rows<L, 6, S>(src, dst, a, s); break;
  }
  return hipErrorInvalidValue;
}

template <class L>
int pair_rows_of(int storage, int i, bool walls) {
  if (walls && !(storage == 0 ? pair_has_walls<L, double>() : pair_has_walls<L, float>())) return 0;
  return storage == 0 ? pair_rows_option<L, double>(i) : (storage == 1 ? pair_rows_option<L, float>(i) : 0);
}

}  // namespace lbrr
