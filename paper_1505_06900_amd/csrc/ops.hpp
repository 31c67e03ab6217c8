// Host-side interface between the C ABI (api.hip) and the per-lattice kernel
// translation units.  Plain function pointers; no torch types.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace lbrr {

constexpr int kNarrowRows = 12;  // tile height that stands for tiles of 32 columns (tile.hpp)

constexpr int kReduceBlock = 256;
// Launch parameters shared by the kernels.  Population (or moment field) i of node (x, y, z)
// lives at element i*si + z*sz + y*sy + x of a buffer; the host picks the
// strides (layout) and checks that every index stays inside the allocation.
struct StepArgs {
  int nx, ny, nz;
  int64_t si, sy, sz;  // element strides of population, row and plane
  double rho0;         // reference density of the deviation storage
  double omega1;       // 1 - 1/tau
  int lz;              // z-planes (2D: rows) per block of the moment-state step and of the step pair
  int rows;            // rows of a tile of the 3D moment step and of the step pair
  int walls;           // moment-state step and step pair: resting walls on the axes of this mask (bit 0 x, 1 y, 2 z)
};

// A step pair's lanes address a plane of one population (2D: a row) by 32-bit byte
// offsets.  With the rows of all populations together (layout 1) a D3Q27 FP32 plane
// passes that at 39.8 million nodes; larger boxes keep single steps, whose addresses are
// 64-bit in 3D.
inline bool pair_offsets_fit(int d, const StepArgs& a, int elem_bytes) {
  const int64_t span = (d == 2 ? int64_t(a.nx) : int64_t(a.ny - 1) * a.sy + a.nx) * elem_bytes;
  return span < (int64_t(1) << 32);
}

struct LatticeOps {
  int q, d, nmax;
  hipError_t (*step)(int order, int storage, const void* src, void* dst, const StepArgs& a, hipStream_t s);
  // two steps in one launch (population storage FP64 and FP32)
  hipError_t (*step_pair)(int order, int storage, const void* src, void* dst, const StepArgs& a, hipStream_t s);
  // the i-th tile height the step pair (moment storage: the 3D step) is built for, 0 past the last and where there
  // is no such kernel
  int (*tile_rows)(int storage, int i, bool walls);
  hipError_t (*init)(int order, int storage, int dtype, const void* rho, const void* u, const void* pi1, void* dst,
                     const StepArgs& a, hipStream_t s);
  hipError_t (*moments)(int storage, int dtype, const void* src, void* rho, void* u, void* pi1, const StepArgs& a,
                        double inv_omega1, hipStream_t s);
  // ticket: 0 before the launch and after it, or NULL: the partials are added in a launch of their own (reduce.hpp)
  hipError_t (*totals)(int storage, const void* src, double* partials, unsigned* ticket, int nblocks, double* out,
                       const StepArgs& a, hipStream_t s);
  hipError_t (*velocity)(int storage, const void* src, double* u, const StepArgs& a, hipStream_t s);
  // copy between the internal layout and compact SoA [q][nz][ny][nx] (to_compact: internal -> compact)
  hipError_t (*repack)(int storage, const void* src, void* dst, bool to_compact, const StepArgs& a, hipStream_t s);
  // moment storage: post-collision deviations of the state, compact SoA [q][nz][ny][nx]
  hipError_t (*mpopulations)(int order, int storage, const void* src, void* dst, const StepArgs& a, hipStream_t s);
  // population storage with resting walls on the axes of `walls` (bit 0 x, 1 y, 2 z)
  hipError_t (*step_walls)(int order, int storage, const void* src, void* dst, const StepArgs& a, int walls,
                           hipStream_t s);
};

// Storage kinds (values of lb_storage): populations 0 FP64, 1 FP32, 2 FP16;
// moments 3 FP64, 4 FP32.
constexpr bool is_moment_storage(int storage) { return storage == 3 || storage == 4; }

const LatticeOps& ops_d2q9();
const LatticeOps& ops_d3q19();
const LatticeOps& ops_d3q27();

// diagnostics kernels (diag.hip)
hipError_t launch_probe(int kind, int vec_bytes, int blocks_per_cu, int nontemporal, int streams, const void* src,
                        void* dst, size_t nbytes, int cus, hipStream_t s);
hipError_t launch_enstrophy(const double* u, int d, int nx, int ny, int nz, int walls, double* partials,
                            unsigned* ticket, int nblocks, double* out, hipStream_t s);
hipError_t launch_zero(unsigned* p, int n, hipStream_t s);
hipError_t launch_copy(const void* src, void* dst, size_t n, hipStream_t s);

}  // namespace lbrr
