// Moment-state form of the regularised update.
//
// After the collision of Eq. discr_bgk_reg every population of a node is a
// function of that node's rho, u and a1^(2) alone: f0 from a0_k = rho u^k and
// f1 from a1^(2) through the recursion of Sec. 3.1 (Eq. rel_a1), both
// reconstructed as in Sec. 3.2.  The state of a lattice node can therefore be
// stored as its pre-collision moments
//     m = (rho - rho0, j = rho u, a1^(2))       10 values in 3D, 6 in 2D,
// instead of q populations, and one step of the scheme becomes: rebuild the
// post-collision populations of every node from m, stream them (pull), and
// take the moments of the populations that arrive.  This is the same update
// in exact arithmetic, with 2 x 10 instead of 2 x 27 stored values moved per
// D3Q27 node update.
//
// Storage: field c of node (x, y, z) at element c*si + z*sz + y*sy + x.
// 3D fields: drho, jx, jy, jz, axx, ayy, azz, axy, axz, ayz; 2D: drho, jx,
// jy, axx, ayy, axy.  FP64 or FP32; the collision runs in the same precision.
//
// Step kernel (3D, k_mstep_t): a block rebuilds the populations of a tile and its
// rim (tile.hpp) plane by plane into LDS and marches along z; the populations
// rebuilt on plane p with c_z = -1, 0, +1 arrive on planes p-1, p, p+1, and plane p-1 is
// complete once plane p has been rebuilt.  A chunk of lz target planes rebuilds
// lz + 2 planes.  The rim and chunk overlaps are the price of the 2.7x smaller state.
// Bound: the rebuild's arithmetic (VALU about 60% busy) and the latency of the
// march behind one block per compute unit.  GLUPS, order 4, before (9 x 64 tiles of 12
// waves in FP32, 32 x 8 patches in FP64, fixed chunk lengths) and now:
//             n = 256          320          200          128           64
//   D3Q27 FP32  54.7 -> 59.0  54.9 -> 59.1  41.6 -> 48.9  38.0 -> 46.4  19.0 -> 25.1
//   D3Q19 FP32  56.6 -> 60.5  57.0 -> 61.3  43.7 -> 50.7  39.0 -> 48.5  19.7 -> 27.4
//   D3Q27 FP64  21.8 -> 27.6  20.4 -> 28.4  21.0 -> 23.5  18.7 -> 23.5  10.3 -> 16.3
//   D3Q19 FP64  22.4 -> 30.0  21.8 -> 30.9  22.4 -> 25.2  19.0 -> 26.6  10.4 -> 17.7
// What gave it: layer sums in place of running sums of three planes and two
// planes in flight in place of three buffers leave room for 16 waves (114 VGPRs);
// tile height and chunk length chosen together (tile_plan, api.hip).
// The 2D step (k_mstep2) does the same one dimension lower: a row of kRowX nodes
// marching along y.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "tile.hpp"

namespace lbrr {

template <class L>
constexpr int kNM = (L::D == 3) ? 10 : 6;

constexpr int kPrefetch = 2;  // 2D: rows of moments in flight ahead of the rebuild

// 2D: nodes per rebuilt row of a block.  Measured, D2Q9 order 4 FP32, GLUPS at
// 2 / 4 / 8 / 16 rows per chunk: 2048^2 rows of 128: 81 / 86 / 82 / 79, of 256:
// 86 / 93 / 89 / 81, of 512: 76 / 81 / 85 / 76; 4096^2 rows of 256: 93 / 100 /
// 94 / 85, of 512: 92 / 102 / 98 / 90 (population storage: 84 and 87).  The
// host picks 4 rows per chunk.
constexpr int kRowX = 256;

// Hydrodynamic state of a node from its stored moments m.
template <class L, class R>
__device__ __forceinline__ Hydro<R> state_hydro(const R (&m)[kNM<L>], R rho0) {
  Hydro<R> h;
  h.drho = m[0];
  h.rho = rho0 + m[0];
  const R inv = inv_density<L>(rho0, m[0], h.rho);
  h.jx = m[1];
  h.jy = m[2];
  h.ux = m[1] * inv;
  h.uy = m[2] * inv;
  if constexpr (L::D == 3) {
    h.jz = m[3];
    h.uz = m[3] * inv;
    h.axx = m[4];
    h.ayy = m[5];
    h.azz = m[6];
    h.axy = m[7];
    h.axz = m[8];
    h.ayz = m[9];
  } else {
    h.jz = h.uz = R(0);
    h.axx = m[3];
    h.ayy = m[4];
    h.axy = m[5];
    h.azz = h.axz = h.ayz = R(0);
  }
  return h;
}

// Stored moments of a node from the moment sums of its arrived populations.
template <class L, class R>
__device__ __forceinline__ void finalize_state(const Moments<R>& s, R rho0, R (&m)[kNM<L>]) {
  const Hydro<R> h = hydro<L, R>(s, rho0);
  m[0] = s.d0;
  m[1] = s.jx;
  m[2] = s.jy;
  if constexpr (L::D == 3) {
    m[3] = s.jz;
    m[4] = h.axx;
    m[5] = h.ayy;
    m[6] = h.azz;
    m[7] = h.axy;
    m[8] = h.axz;
    m[9] = h.ayz;
  } else {
    m[3] = h.axx;
    m[4] = h.ayy;
    m[5] = h.axy;
  }
}

template <class R>
__device__ __forceinline__ void clear(Moments<R>& s) {
  s.d0 = s.jx = s.jy = s.jz = s.pxx = s.pyy = s.pzz = s.pxy = s.pxz = s.pyz = R(0);
}

// 2D: add the populations with c_y = CY rebuilt on one row that arrive at
// inner node tx to its moment sums s: population (cx, CY) comes from row node
// tx - cx.
template <class L, int CY, int BX, class R, bool Assign = false>
__device__ __forceinline__ void add_row(Moments<R>& s, const R (*pop)[BX], int tx) {
  R v[3];
  sfor<0, 3>([&](auto X) {
    constexpr int cx = int(X) - 1;
    v[X] = pop[velocity_index<L>(cx, CY, 0)][tx - cx];
  });
  const R e = v[2] + v[0];
  const R s0 = e + v[1], s1 = v[2] - v[0];
  if constexpr (Assign) {  // the first row a target receives (c_y = +1) sets every sum
    static_assert(CY > 0, "assign with the c_y = +1 row");
    s.d0 = s0;
    s.jx = s1;
    s.pxx = e;
    s.pyy = s0;
    s.jy = s0;
    s.pxy = s1;
    s.jz = s.pzz = s.pxz = s.pyz = R(0);
    return;
  }
  s.d0 = s.d0 + s0;
  s.jx = s.jx + s1;
  s.pxx = s.pxx + e;
  if constexpr (CY != 0) {
    s.pyy = s.pyy + s0;
    if constexpr (CY > 0) {
      s.jy = s.jy + s0;
      s.pxy = s.pxy + s1;
    } else {
      s.jy = s.jy - s0;
      s.pxy = s.pxy - s1;
    }
  }
}

// ---- resting walls -----------------------------------------------------------
// Resting no-slip walls on the first and last node of the axes in a.walls: the
// regularised Dirichlet boundary of Sec. 3.7 with u = 0, as the population step
// applies it.  At a wall node a population whose source lies outside the box is
// unknown; it takes the value of its opposite if that one is known (the
// off-equilibrium bounce-back at u = 0, where w_i = w_opp), else w_i (rho - rho0);
// rho - rho0 follows from the zeroth moment of the completed set, the node keeps
// j = 0, and a1^(2) is the second moment of the completed set minus
// (rho - rho0) c_s^2 I.  The 3D step keeps the arrivals of a node and completes them as
// the population step does (LayerValues, tile.hpp).  The 2D step keeps sums: every step
// is linear in the arriving populations, so their contributions are added row by row as
// they arrive, a known population whose opposite is unknown counts twice (at xi and at
// -xi: the momentum cancels), and the buried ones enter when the node is finalised.

// Does a population moving along (cx, cy) arrive from outside the box?
__device__ __forceinline__ bool from_outside(int sx, int sy, int cx, int cy) {
  return (sx != 0 && cx == -sx) || (sy != 0 && cy == -sy);
}

// Contribution of the known population v moving along (cx, cy) to the moment sums of a
// wall node (sides sx, sy).
template <class R>
__device__ __forceinline__ void add_known(Moments<R>& s, R v, int cx, int cy, int sx, int sy) {
  const bool twice = from_outside(sx, sy, -cx, -cy);
  const R k = twice ? R(2) * v : v;
  s.d0 = s.d0 + k;
  if (!twice) {
    s.jx = s.jx + R(cx) * v;
    s.jy = s.jy + R(cy) * v;
  }
  s.pxx = s.pxx + R(cx * cx) * k;
  s.pyy = s.pyy + R(cy * cy) * k;
  s.pxy = s.pxy + R(cx * cy) * k;
}

// Wall node: the populations with c_y = CY rebuilt on one row arriving at inner node tx.
template <class L, int CY, int BX, class R>
__device__ __forceinline__ void add_row_walls(Moments<R>& s, const R (*pop)[BX], int tx, int sx, int sy) {
  sfor<0, 3>([&](auto X) {
    constexpr int cx = int(X) - 1;
    if (!from_outside(sx, sy, cx, CY)) add_known(s, pop[velocity_index<L>(cx, CY, 0)][tx - cx], cx, CY, sx, sy);
  });
}

// Stored moments of a wall node from its sums (known and bounced populations).
template <class L, class R>
__device__ __forceinline__ void finalize_walls(const Moments<R>& s, int sx, int sy, R (&m)[kNM<L>]) {
  static_assert(L::D == 2, "2D");
  R wb = R(0), bxx = R(0), byy = R(0), bxy = R(0);  // buried: sum w, w xi xi
  sfor<0, L::Q>([&](auto I) {
    constexpr int cx = L::cx(I), cy = L::cy(I);
    if (from_outside(sx, sy, cx, cy) && from_outside(sx, sy, -cx, -cy)) {
      const R w = R(L::w(I));
      wb = wb + w;
      bxx = bxx + R(cx * cx) * w;
      byy = byy + R(cy * cy) * w;
      bxy = bxy + R(cx * cy) * w;
    }
  });
  const R drho = s.d0 / (R(1) - wb);
  constexpr R cs2 = R(kCs2);
  m[0] = drho;
  m[1] = R(0);
  m[2] = R(0);
  m[3] = s.pxx + drho * bxx - drho * cs2;
  m[4] = s.pyy + drho * byy - drho * cs2;
  m[5] = s.pxy + drho * bxy;
}

// v in a register of its own.
__device__ __forceinline__ float copy_of(float v) {
  float c;
  asm volatile("v_mov_b32 %0, %1" : "=v"(c) : "v"(v));
  return c;
}
__device__ __forceinline__ double copy_of(double v) {
  double c;
  asm volatile("v_mov_b64 %0, %1" : "=v"(c) : "v"(v));
  return c;
}

// One step of the moment-state update in 3D on the tiles of tile.hpp: the tile's and
// the rim's populations are rebuilt from their moments plane by plane, and an
// inner thread that has the three layers of its plane forms and stores the new
// moments.  The moments of the next plane are loaded as soon as the present
// ones are in the collision's registers.  W: resting walls on the axes of a.walls.
template <class L, int N, class S, int TY, bool W>
__global__ void __launch_bounds__(Tile<TY>::threads()) k_mstep_t(const S* __restrict__ src, S* __restrict__ dst,
                                                                 StepArgs a) {
  static_assert(L::D == 3, "3D lattices; 2D runs k_mstep2");
  using R = S;
  constexpr int NM = kNM<L>;
  __shared__ R pop[L::Q][Tile<TY>::kRows][Tile<TY>::kCols];
  const Tile<TY> t(a);
  if (t.empty) return;
  // Byte offsets of the nodes within a plane of one field (the host checks that
  // they fit 32 bits); plane and field bases are block-uniform.
  const uint32_t off_in = uint32_t((int64_t(t.py) * a.sy + t.px) * int64_t(sizeof(S)));
  const uint32_t off_out = t.inner ? uint32_t((int64_t(t.y) * a.sy + t.x) * int64_t(sizeof(S))) : 0u;
  const R rho0 = R(a.rho0), om = R(a.omega1);
  const int sx = W ? wall_side(a.walls, 0, t.x, a.nx) : 0, sy = W ? wall_side(a.walls, 1, t.y, a.ny) : 0;
  struct Plane {  // a struct, as in k_step_pair
    R v[NM];
  };
  const int z0 = t.z0, z1 = t.z1, n = z1 - z0;
  // moments of plane k of the march, z0 - 1 + k (past the last plane: the last again)
  auto load = [&](int k, Plane& m) __attribute__((always_inline)) {
    const S* s = src + int64_t(wrap_axis(z0 - 1 + (k < n + 1 ? k : n + 1), a.nz)) * a.sz;
    // The empty asm hides that the lane offset is the same in every plane of
    // the march.  Without it the compiler hoists a 64-bit copy of the offset
    // out of the loop and adds it to every field's base with a 64-bit lane
    // add; with it each access takes the scalar-base form (scalar field base +
    // 32-bit lane offset) and the adds go away.
    uint32_t o = off_in;
    asm volatile("" : "+v"(o));
    sfor<0, NM>([&](auto C) { m.v[C] = at_offset(s + int64_t(C) * a.si, o); });
  };
  // Planes z0 - 1 .. z1 are rebuilt (plane z0 - 1 + k, k = 0 .. n + 1), targets z0 ..
  // z1 - 1: plane k brings layer c_z = +1 to target k, 0 to target k - 1, -1 to target
  // k - 2, which is then complete.  The first and the last plane rebuild the one
  // layer that reaches the chunk.
  using Lo = Layer<L, -1, R, W>;
  using Mid = Layer<L, 0, R, W>;
  using Up = Layer<L, 1, R, W>;
  Up up1, up2;  // c_z = +1 layers of targets k - 1 and k - 2
  Mid mid2;     // c_z = 0 layer of target k - 2
  // Populations of plane k from its moments m into LDS; m then takes plane k + 2.
  auto rebuild = [&](int k, Plane& m, auto ZS) __attribute__((always_inline)) {
    constexpr int Z = decltype(ZS)::value;
    // The moments move to registers of their own before the load takes theirs.
    // Left to itself the compiler loads into other registers and copies them back
    // at the end of the loop, which waits for the load there.
    R own[NM];
    sfor<0, NM>([&](auto C) { own[C] = copy_of(m.v[C]); });
    if constexpr (Z != -1) load(k + 2, m);
    const Hydro<R> h = state_hydro<L, R>(own, rho0);
    R C[3][3][3], out[L::Q];
    coefficients<L, N, R>(h, om, C);
    reconstruct<L, N, R, Z>(C, out);
    if (t.writes) {
      sfor<0, L::Q>([&](auto I) {
        if constexpr (Z == 2 || L::cz(I) == Z) pop[I][t.r][t.col] = out[I];
      });
    }
  };
  auto arrived = [&](auto I) { return pop[I][t.r - L::cy(I)][t.lane + 1 - L::cx(I)]; };
  auto finish = [&](int z, const Lo& lo, const Mid& mid, const Up& up) __attribute__((always_inline)) {
    R m[NM];
    finalize_state<L, R>(layer_moments<L, R, W>(lo, mid, up, sx, sy, W ? wall_side(a.walls, 2, z, a.nz) : 0), rho0, m);
    S* d = dst + int64_t(z) * a.sz;
    uint32_t o = off_out;
    asm volatile("" : "+v"(o));
    sfor<0, NM>([&](auto C) { __builtin_nontemporal_store(m[C], ptr_at_offset(d + int64_t(C) * a.si, o)); });
  };
  using all = std::integral_constant<int, 2>;
  using layer_m = std::integral_constant<int, -1>;
  using layer_p = std::integral_constant<int, 1>;
  // A completed plane is stored before the barrier that frees the LDS (after it,
  // as in k_step_pair: 53 -> 46 GLUPS with 9 rows, D3Q27 FP32 256^3).
  auto inside = [&](int k, Plane& m) __attribute__((always_inline)) {
    rebuild(k, m, all{});
    lds_barrier();
    if (t.inner) {
      Lo lo;
      Mid mid;
      Up up;
      lo.read(arrived);
      mid.read(arrived);
      up.read(arrived);
      if (k >= 2) finish(z0 + k - 2, lo, mid2, up2);
      up2 = up1;
      mid2 = mid;
      up1 = up;
    }
    lds_barrier();
  };
  Plane even, odd;  // the planes in flight: two ahead of the rebuild
  load(0, even);
  load(1, odd);
  rebuild(0, even, layer_p{});
  lds_barrier();
  if (t.inner) up1.read(arrived);
  lds_barrier();
  int k = 1;
  for (; k + 1 <= n; k += 2) {
    inside(k, odd);
    inside(k + 1, even);
  }
  if (k <= n) {
    inside(k, odd);
    rebuild(n + 1, even, layer_m{});
  } else {
    rebuild(n + 1, odd, layer_m{});
  }
  lds_barrier();
  if (t.inner) {
    Lo lo;
    lo.read(arrived);
    finish(z1 - 1, lo, mid2, up2);
  }
}

// One step of the 2D moment-state update.  A block of BX threads rebuilds a
// row of BX nodes (x0 - 1 ... x0 + BX - 2) and marches along y through a
// chunk of a.lz target rows: the populations rebuilt on row p with c_y = -1,
// 0, +1 arrive on rows p - 1, p, p + 1, so each inner thread keeps running
// moment sums for three target rows, and row p - 1 is complete once row p has
// been rebuilt.  Rows of BX nodes keep the loads and stores of a field nearly
// line-aligned (one partial 128-byte line per row and field); the moments of two
// rows are in flight ahead of the rebuild.
template <class L, int N, class S, int BX, bool W>
__global__ void __launch_bounds__(BX) k_mstep2(const S* __restrict__ src, S* __restrict__ dst, StepArgs a) {
  using R = S;
  constexpr int NM = kNM<L>;
  static_assert(L::D == 2, "2D lattices only");
  __shared__ R pop[L::Q][BX];
  const int tx = threadIdx.x;
  const int x0 = blockIdx.x * (BX - 2);
  const int px = wrap_axis(x0 - 1 + tx, a.nx);
  const bool inner = tx >= 1 && tx <= BX - 2 && x0 + tx - 1 < a.nx;
  const int xo = x0 + tx - 1;
  const R rho0 = R(a.rho0), om = R(a.omega1);
  // byte offsets within a row of one field; row and field bases are block-uniform
  const uint32_t off_in = uint32_t(px) * uint32_t(sizeof(S)), off_out = uint32_t(xo) * uint32_t(sizeof(S));
  auto load = [&](int y, R (&m)[NM]) {
    const S* s = src + int64_t(y) * a.sy;
    sfor<0, NM>([&](auto C) { m[C] = at_offset(s + int64_t(C) * a.si, off_in); });
  };
  auto put = [&](int y, const R (&m)[NM]) {
    S* d = dst + int64_t(y) * a.sy;
    sfor<0, NM>([&](auto C) { __builtin_nontemporal_store(m[C], ptr_at_offset(d + int64_t(C) * a.si, off_out)); });
  };
  // Target rows y0 .. y1-1; rows y0-1 .. y1 are rebuilt, row k of the march
  // being y0 - 1 + k (k = 0 .. n + 1, n = y1 - y0).  Row k adds its c_y = +1
  // populations to target k (first contribution), c_y = 0 to target k - 1 and
  // c_y = -1 to target k - 2, which is then complete.  Register roles rotate
  // with period 3: moments of row k in buffer k mod 3, sums
  // of target j in slot j mod 3, the march unrolled by 3 with no copies.
  const int y0 = blockIdx.y * a.lz;
  const int y1 = (y0 + a.lz < a.ny) ? y0 + a.lz : a.ny;
  const int n = y1 - y0;
  Moments<R> T[3];
  R B[3][NM];
  load(wrap_axis(y0 - 1, a.ny), B[0]);
  load(wrap_axis(y0, a.ny), B[1]);
  R out[NM];  // moments of target k - 3, stored during row k
  auto iteration = [&](int k, auto PHS) __attribute__((always_inline)) {
    constexpr int PH = decltype(PHS)::value;
    constexpr int P1 = (PH + 2) % 3, P2 = (PH + 1) % 3;  // (k - 1) mod 3, (k - 2) mod 3
    const int py = y0 - 1 + k;
    if (k + kPrefetch <= n + 1) load(wrap_axis(py + kPrefetch, a.ny), B[P1]);  // buffer (k + 2) mod 3
    if (inner && k >= 3) put(y0 + k - 3, out);
    {
      const Hydro<R> h = state_hydro<L, R>(B[PH], rho0);
      R C[3][3][3];
      coefficients<L, N, R>(h, om, C);
      R f[L::Q];
      reconstruct<L, N, R>(C, f);
      sfor<0, L::Q>([&](auto I) { pop[I][tx] = f[I]; });
    }
    lds_barrier();
    if (inner) {
      if constexpr (W) {
        // walls: sides of the target column and of the target rows py + 1, py, py - 1
        // (with no side the wall sums are the plain sums)
        const int sx = wall_side(a.walls, 0, xo, a.nx);
        if (k < n) {
          clear(T[PH]);
          add_row_walls<L, 1, BX, R>(T[PH], pop, tx, sx, wall_side(a.walls, 1, py + 1, a.ny));
        }
        if (k >= 1 && k <= n) add_row_walls<L, 0, BX, R>(T[P1], pop, tx, sx, wall_side(a.walls, 1, py, a.ny));
        if (k >= 2) {  // target row py - 1 is complete
          const int sm = wall_side(a.walls, 1, py - 1, a.ny);
          add_row_walls<L, -1, BX, R>(T[P2], pop, tx, sx, sm);
          if (sx != 0 || sm != 0) finalize_walls<L, R>(T[P2], sx, sm, out);
          else finalize_state<L, R>(T[P2], rho0, out);
        }
      } else {
        if (k < n) add_row<L, 1, BX, R, true>(T[PH], pop, tx);
        if (k >= 1 && k <= n) add_row<L, 0, BX, R>(T[P1], pop, tx);
        if (k >= 2) {
          add_row<L, -1, BX, R>(T[P2], pop, tx);
          finalize_state<L, R>(T[P2], rho0, out);  // target row py - 1 is complete
        }
      }
    }
    lds_barrier();
  };
  using ph0 = std::integral_constant<int, 0>;
  using ph1 = std::integral_constant<int, 1>;
  using ph2 = std::integral_constant<int, 2>;
  iteration(0, ph0{});
  int k = 1;
  for (; k + 2 <= n + 1; k += 3) {
    iteration(k, ph1{});
    iteration(k + 1, ph2{});
    iteration(k + 2, ph0{});
  }
  if (k <= n + 1) iteration(k++, ph1{});  // k = 1 mod 3 here
  if (k <= n + 1) iteration(k++, ph2{});
  if (inner) put(y1 - 1, out);
}

// Moment state at t = 0 from (rho, u[, pi1]): the pre-collision moments of
// f0(rho, u) + f1(u, pi1), i.e. rho - rho0, rho u and pi1 (Sec. 3.2).
template <class L, class S, class T>
__global__ void __launch_bounds__(256) k_minit(const T* __restrict__ rho, const T* __restrict__ u,
                                               const T* __restrict__ pi1, S* __restrict__ dst, StepArgs a) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  const int64_t n = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (n >= nodes) return;
  const int64_t off = node_offset(a, uint32_t(n));
  const double r = double(rho[n]);
  S m[kNM<L>];
  m[0] = S(r - a.rho0);
  m[1] = S(r * double(u[n]));
  m[2] = S(r * double(u[nodes + n]));
  if constexpr (L::D == 3) {
    m[3] = S(r * double(u[2 * nodes + n]));
    // pi1 order xx, xy, xz, yy, yz, zz -> state order axx, ayy, azz, axy, axz, ayz
    const int perm[6] = {0, 3, 5, 1, 2, 4};
    for (int c = 0; c < 6; ++c) m[4 + c] = pi1 ? S(pi1[perm[c] * nodes + n]) : S(0);
  } else {
    const int perm[3] = {0, 2, 1};  // xx, xy, yy -> axx, ayy, axy
    for (int c = 0; c < 3; ++c) m[3 + c] = pi1 ? S(pi1[perm[c] * nodes + n]) : S(0);
  }
  sfor<0, kNM<L>>([&](auto C) { dst[int64_t(C) * a.si + off] = m[C]; });
}

// rho, u, pi1 (= the stored pre-collision a1^(2)) of the moment state.
template <class L, class S, class T>
__global__ void __launch_bounds__(256) k_mmoments(const S* __restrict__ src, T* __restrict__ rho, T* __restrict__ u,
                                                  T* __restrict__ pi1, StepArgs a) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  const int64_t n = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (n >= nodes) return;
  const int64_t off = node_offset(a, uint32_t(n));
  double m[kNM<L>];  // a1^(2) is read only if asked for: 158 -> 89 us without it, 256^3 FP32 (268 of 671 MB)
  sfor<0, 1 + L::D>([&](auto C) { m[C] = double(src[int64_t(C) * a.si + off]); });
  if (pi1) sfor<1 + L::D, kNM<L>>([&](auto C) { m[C] = double(src[int64_t(C) * a.si + off]); });
  const double r = a.rho0 + m[0];
  if (rho) rho[n] = T(r);
  if (u) {
    u[n] = T(m[1] / r);
    u[nodes + n] = T(m[2] / r);
    if constexpr (L::D == 3) u[2 * nodes + n] = T(m[3] / r);
  }
  if (pi1) {
    if constexpr (L::D == 3) {
      const int from[6] = {4, 7, 8, 5, 9, 6};  // xx, xy, xz, yy, yz, zz
      for (int c = 0; c < 6; ++c) pi1[c * nodes + n] = T(m[from[c]]);
    } else {
      const int from[3] = {3, 5, 4};  // xx, xy, yy
      for (int c = 0; c < 3; ++c) pi1[c * nodes + n] = T(m[from[c]]);
    }
  }
}

// Per-block partial totals {rho, j_x, j_y, j_z, |j|^2 / (2 rho)} of the moment state.
template <class L, class S>
__global__ void __launch_bounds__(kReduceBlock) k_mtotals(const S* __restrict__ src, double* __restrict__ partials,
                                                          unsigned* __restrict__ ticket, StepArgs a,
                                                          int64_t per_block, double* __restrict__ out) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  const int64_t begin = int64_t(blockIdx.x) * per_block;
  const int64_t end = begin + per_block < nodes ? begin + per_block : nodes;
  double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int64_t n = begin + threadIdx.x; n < end; n += kReduceBlock) {
    const int64_t off = node_offset(a, uint32_t(n));
    const double r = a.rho0 + double(src[off]);
    const double jx = double(src[a.si + off]), jy = double(src[2 * a.si + off]);
    const double jz = (L::D == 3) ? double(src[3 * a.si + off]) : 0.0;
    acc[0] += r;
    acc[1] += jx;
    acc[2] += jy;
    acc[3] += jz;
    acc[4] += 0.5 * (jx * jx + jy * jy + jz * jz) / r;
  }
  reduce_blocks<5>(acc, partials, ticket, out);
}

// Velocity field (FP64) of the moment state.
template <class L, class S>
__global__ void __launch_bounds__(256) k_mvelocity(const S* __restrict__ src, double* __restrict__ u, StepArgs a) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  const int64_t n = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (n >= nodes) return;
  const int64_t off = node_offset(a, uint32_t(n));
  const double inv = 1.0 / (a.rho0 + double(src[off]));
  u[n] = double(src[a.si + off]) * inv;
  u[nodes + n] = double(src[2 * a.si + off]) * inv;
  if constexpr (L::D == 3) u[2 * nodes + n] = double(src[3 * a.si + off]) * inv;
}

// Post-collision deviations of the moment state (what the population form
// stores), compact SoA [q][node] in the state's precision.
template <class L, int N, class S>
__global__ void __launch_bounds__(256) k_mpopulations(const S* __restrict__ src, S* __restrict__ dst, StepArgs a) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  const int64_t n = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (n >= nodes) return;
  const int64_t off = node_offset(a, uint32_t(n));
  S m[kNM<L>];
  sfor<0, kNM<L>>([&](auto C) { m[C] = src[int64_t(C) * a.si + off]; });
  const Hydro<S> h = state_hydro<L, S>(m, S(a.rho0));
  S C[3][3][3];
  coefficients<L, N, S>(h, S(a.omega1), C);
  S f[L::Q];
  reconstruct<L, N, S>(C, f);
  sfor<0, L::Q>([&](auto I) { dst[int64_t(I) * nodes + n] = f[I]; });
}

// ---------------------------------------------------------------------------
// Launchers.  a.lz = z-planes per block of the 3D step (each chunk rebuilds
// lz + 2 planes) and a.rows = its tile height; the host picks both.
// Tile heights of the 3D step the host chooses from (tile_plan in api.hip).  GLUPS
// at 256^3, order 4, by rows: D3Q27 FP32 5 / 8 / 9 / 11 / 13 rows 52.6 / 56.6 / 54.1 / 56.3 /
// 58.8, D3Q19 FP32 51.9 / 58.8 / 56.1 / 61.6 / 59.7, D3Q27 FP64 3 / 4 / 5 rows 23.5 / 27.0 /
// 27.5 (6 rows spill: 12.7), D3Q19 FP64 26.0 / 30.0 / 30.1.  The lower tiles serve boxes whose rows
// the first divides badly, and small ones (64^3 FP32 13 rows 19.3, 8 rows 25.1).  Walled on all
// axes the 13- and 11-row D3Q27 FP32 forms spill 7 and 5 registers and stay level (us a step, 13 / 11 / 8
// rows: 256^3 360 / 365 / 367, 200^3 211 / 234 / 236, 128^3 56 / 56 / 53, D3Q19 301 / 304 / 328, 168 / 185 / 196,
// 48 / 46 / 46).  FP64 boxes
// whose last 64-column tile would stay half idle take 32 columns by 12 rows in
// the same eight waves (us a step, D3Q19 273 x 67 x 25 41.8 -> 30.9, 200 x 200 x 32 79.8 -> 52.9;
// tile_plan weighs the two).
template <class S>
constexpr int mom_rows_option(int i) {
  constexpr int f32[] = {13, 11, 8}, f64[] = {5, 4, kNarrowRows};
  return i > 2 ? 0 : (sizeof(S) == 8 ? f64[i] : f32[i]);
}

template <class L, int N, class S, int TY>
hipError_t launch_mstep_t(const void* src, void* dst, const StepArgs& a, hipStream_t s) {
  const int64_t blocks = Tile<TY>::blocks(a);
  if (blocks >= (int64_t(1) << 31)) return hipErrorInvalidValue;
  if (a.walls)
    hipLaunchKernelGGL((k_mstep_t<L, N, S, TY, true>), dim3(unsigned(blocks)), dim3(Tile<TY>::threads()), 0, s,
                       static_cast<const S*>(src), static_cast<S*>(dst), a);
  else
    hipLaunchKernelGGL((k_mstep_t<L, N, S, TY, false>), dim3(unsigned(blocks)), dim3(Tile<TY>::threads()), 0, s,
                       static_cast<const S*>(src), static_cast<S*>(dst), a);
  return hipGetLastError();
}

template <class L, int N, class S>
hipError_t launch_mstep(const void* src, void* dst, const StepArgs& a, hipStream_t s) {
  if (a.lz < 1) return hipErrorInvalidValue;
  if constexpr (L::D == 2) {
    dim3 grid2(unsigned((a.nx + kRowX - 3) / (kRowX - 2)), unsigned((a.ny + a.lz - 1) / a.lz));
    if (grid2.y > 65535u) return hipErrorInvalidValue;
    if (a.walls)
      hipLaunchKernelGGL((k_mstep2<L, N, S, kRowX, true>), grid2, dim3(kRowX), 0, s, static_cast<const S*>(src),
                         static_cast<S*>(dst), a);
    else
      hipLaunchKernelGGL((k_mstep2<L, N, S, kRowX, false>), grid2, dim3(kRowX), 0, s, static_cast<const S*>(src),
                         static_cast<S*>(dst), a);
    return hipGetLastError();
  } else {
    if (int64_t(a.ny) * a.sy * int64_t(sizeof(S)) >= (int64_t(1) << 32)) return hipErrorInvalidValue;
    if (a.rows == mom_rows_option<S>(0)) return launch_mstep_t<L, N, S, mom_rows_option<S>(0)>(src, dst, a, s);
    if (a.rows == mom_rows_option<S>(1)) return launch_mstep_t<L, N, S, mom_rows_option<S>(1)>(src, dst, a, s);
    if (a.rows == mom_rows_option<S>(2)) return launch_mstep_t<L, N, S, mom_rows_option<S>(2)>(src, dst, a, s);
    return hipErrorInvalidValue;
  }
}

template <class L, int N, class S>
hipError_t launch_mpopulations(const void* src, void* dst, const StepArgs& a, hipStream_t s) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  hipLaunchKernelGGL((k_mpopulations<L, N, S>), dim3(unsigned((nodes + 255) / 256)), dim3(256), 0, s,
                     static_cast<const S*>(src), static_cast<S*>(dst), a);
  return hipGetLastError();
}

template <class L, class S>
hipError_t launch_minit(int dtype, const void* rho, const void* u, const void* pi1, void* dst, const StepArgs& a,
                        hipStream_t s) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  dim3 grid(unsigned((nodes + 255) / 256));
  if (dtype == 0)
    hipLaunchKernelGGL((k_minit<L, S, double>), grid, dim3(256), 0, s, static_cast<const double*>(rho),
                       static_cast<const double*>(u), static_cast<const double*>(pi1), static_cast<S*>(dst), a);
  else
    hipLaunchKernelGGL((k_minit<L, S, float>), grid, dim3(256), 0, s, static_cast<const float*>(rho),
                       static_cast<const float*>(u), static_cast<const float*>(pi1), static_cast<S*>(dst), a);
  return hipGetLastError();
}

template <class L, class S>
hipError_t launch_mmoments(int dtype, const void* src, void* rho, void* u, void* pi1, const StepArgs& a,
                           hipStream_t s) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  dim3 grid(unsigned((nodes + 255) / 256));
  if (dtype == 0)
    hipLaunchKernelGGL((k_mmoments<L, S, double>), grid, dim3(256), 0, s, static_cast<const S*>(src),
                       static_cast<double*>(rho), static_cast<double*>(u), static_cast<double*>(pi1), a);
  else
    hipLaunchKernelGGL((k_mmoments<L, S, float>), grid, dim3(256), 0, s, static_cast<const S*>(src),
                       static_cast<float*>(rho), static_cast<float*>(u), static_cast<float*>(pi1), a);
  return hipGetLastError();
}

template <class L, class S>
hipError_t launch_mtotals(const void* src, double* partials, unsigned* ticket, int nblocks, double* out,
                          const StepArgs& a, hipStream_t s) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  const int64_t per_block = (nodes + nblocks - 1) / nblocks;
  hipLaunchKernelGGL((k_mtotals<L, S>), dim3(nblocks), dim3(kReduceBlock), 0, s, static_cast<const S*>(src),
                     partials, ticket, a, per_block, out);
  if (!ticket) hipLaunchKernelGGL((k_final<5>), dim3(1), dim3(kReduceBlock), 0, s, partials, nblocks, out);
  return hipGetLastError();
}

template <class L, class S>
hipError_t launch_mvelocity(const void* src, double* u, const StepArgs& a, hipStream_t s) {
  const int64_t nodes = int64_t(a.nx) * a.ny * a.nz;
  hipLaunchKernelGGL((k_mvelocity<L, S>), dim3(unsigned((nodes + 255) / 256)), dim3(256), 0, s,
                     static_cast<const S*>(src), u, a);
  return hipGetLastError();
}

}  // namespace lbrr
