// C ABI of the library (declarations and contracts in include/lbrr.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <type_traits>

#include "closure.hpp"
#include "lbrr.h"
#include "ops.hpp"
#include "reduce.hpp"

using lbrr::LatticeOps;
using lbrr::StepArgs;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  std::vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

int hip_fail(hipError_t e, const char* what) {
  return fail(LB_ERR_HIP, "%s: %s (%d)", what, hipGetErrorString(e), int(e));
}

#define HIP_TRY(expr, what)            \
  do {                                 \
    hipError_t e_ = (expr);            \
    if (e_ != hipSuccess) return hip_fail(e_, what); \
  } while (0)

size_t elem_size(int storage) {
  switch (storage) {
    case LB_STORE_FP64:
    case LB_STORE_MOM_FP64: return 8;
    case LB_STORE_FP32:
    case LB_STORE_MOM_FP32: return 4;
  }
  return 2;
}

// Row pitch in bytes: whole 128-byte lines, so that every row starts on a line and a
// wave's 64 consecutive x stay within the fewest lines (with nx = 300 unpadded, D3Q27
// FP32 ran at 13.9 GLUPS against 27 for 256 or 320).
size_t row_bytes(int64_t nx, size_t es) { return (size_t(nx) * es + 127) / 128 * 128; }

int compute_units() {
  int cus = 256;
  int dev = 0;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  return cus;
}

int env_int(const char* name, int none) {
  const char* e = std::getenv(name);
  return e ? std::atoi(e) : none;
}

// Tile height and chunk length of a launch that marches in chunks (rows of a 2D
// lattice, tiles of planes of a 3D one).
struct TilePlan {
  int rows = 0, lz = 0;
  double fill = 0.0;   // 3D: nodes updated, of those the chip's compute units take through the launch
  bool whole = false;  // step pairs: not for a call of five, six or seven steps
};

// 3D (tile.hpp): a compute unit holds one block, a block's time grows with the
// planes it rebuilds (lz + 2) and with its waves (rows + 3), and the tile rows are
// dealt to the eight XCDs in turn, so the plan taken is the one with the smallest
//   rounds * (lz + 2) * (rows + 3),  rounds = blocks per XCD / compute units per XCD, rounded up.
// A narrow tile (32 columns by 12 rows in eight waves) costs 9.5 rows' waves, 8.5 with
// walls: so it comes out of the best times of both widths (D3Q27 and D3Q19, 150 planes of 131
// rows by 65, 100, 130 and 200 columns: 9.5 to 10.5, walled 8.0 to 9.1).  It is the better one
// where 64-column tiles would stay half empty (us a step, 5 rows x 64 -> 12 x 32: D3Q27
// 65 x 131 x 150 99.8 -> 73.7, 130 x 131 x 150 135 -> 120, 100 x 131 x 150 101 -> 97).
// Chunk counts that give the same lz are tried once, and none past the one where even
// full rounds, columns * (planes + 2 chunks) of work for the whole chip, cost more than the
// best so far: every lb_step call makes its plan, on the host (24 x 24 x 65535, trying
// every count: 2.7 ms a call, so 3.3 us; 24 x 24 x 330 13.7 us and 2.5).
// forced_lz, forced_rows: > 0 overrides the choice (forced_rows if built).
TilePlan tile_plan(const LatticeOps& ops, int storage, int nx, int ny, int nz, bool walls, int forced_lz,
                   int forced_rows) {
  TilePlan p;
  const int64_t slots = compute_units() / 8 > 0 ? compute_units() / 8 : 1;
  int64_t cost = 0;
  bool built = false;
  for (int i = 0; const int rows = ops.tile_rows(storage, i, walls); ++i) built = built || rows == forced_rows;
  for (int i = 0; const int rows = ops.tile_rows(storage, i, walls); ++i) {
    if (built && rows != forced_rows) continue;
    const bool narrow = rows == lbrr::kNarrowRows;
    const int64_t gx = narrow ? (nx + 31) / 32 : (nx + 63) / 64, gy = (ny + rows - 1) / rows;
    const int64_t weight = narrow ? (walls ? 17 : 19) : 2 * (rows + 3);
    for (int chunks = 1;;) {
      const int lz = forced_lz > 0 ? forced_lz : (nz + chunks - 1) / chunks;
      const int64_t g = gy * ((nz + lz - 1) / lz);
      const int64_t rounds = (gx * ((g + 7) / 8) + slots - 1) / slots;
      const int64_t c = rounds * (lz + 2) * weight;
      if (p.lz == 0 || c < cost) {
        p.rows = rows;
        p.lz = lz;
        p.fill = double(nx) * ny * nz / (double(narrow ? 32 : 64) * rows * double(rounds * (lz + 2)) * double(8 * slots));
        cost = c;
      }
      if (forced_lz > 0 || lz == 1) break;
      chunks = (nz + lz - 2) / (lz - 1);  // the fewest with a smaller lz
      if (gx * gy * (nz + 2 * int64_t(chunks)) * weight >= cost * 8 * slots) break;
    }
  }
  return p;
}

// The step pair (k_step_pair, k_step_pair2); lz = 0 where lb_step takes single steps.
//
// 2D: pairs at every size; short chunks while there are few blocks (a chunk is a
// serial march), longer ones where their edge rows cost traffic.  us a step, order
// 4, single / lz = 1 / 2 / 4 / 6 / 12:
//   FP32   64^2  2.66 / 1.92 / 2.29 / 3.11 / 3.85 / 6.17    501^2  5.42 / 4.02 / 3.55 / 3.76 / 4.41 / 6.72
//        1024^2 14.5 / 14.3 / 11.9 / 10.1 / 10.8 / 10.4    2048^2 49.9 / 43.8 / 35.9 / 32.8 / 32.5 / 33.2
//   FP64  256^2  4.49 / 3.75 / 3.76 / 4.46 / 5.69 / 9.22    501^2  8.30 / 6.89 / 5.06 / 6.07 / 6.52 / 9.32
//        1024^2 27.0 / 26.3 / 21.6 / 18.3 / 19.9 / 18.9    2048^2 101 / 85.0 / 69.4 / 62.1 / 61.0 / 61.3
// (walled boxes within a few per cent of these: 501^2 FP64 8.51 / 7.16 / 5.22 / 5.86).
// lz = 1 only while two blocks a compute unit do: four steps of 288^2 FP64 in single
// steps 15.8 us, pairs at lz = 1 18.3 (576 blocks), at 2 16.2; 384^2 20.9 / 20.0 / 17.6.
// Narrow rows leave most of a block's 254 columns idle where k_step's blocks are 64 wide:
// below 0.3 of them used, pairs are for as many rows as the chip takes at once (four
// steps, single -> pairs: 20 columns FP32 1000 rows 13.8 -> 11.3, 3000 13.8 -> 17.4, 20000
// 39.7 -> 66.7; FP64 1000 13.9 -> 13.8, 64 columns 13.0 -> 15.4), and for rows used to 0.15 of a
// state that caches no longer hold (64 columns, 20000 rows FP32 67.5 -> 60.8).
// A state of 2.5 to 8 MB stays in the XCDs' L2 caches, where each finds the rows it wrote.
// Pairs and single steps share the rows out differently, so single steps after one pair of
// pairs cost more there than it gains: calls of five to seven steps stay single (us a call
// waited for, six steps, single / pairs: 320^2 FP32 31.3 / 34.1, 384^2 33.2 / 36.5, 256^2 FP64
// 34.3 / 36.4).  Longer calls, and runs between checks, gain by fewer launches (ten steps:
// 64.5 / 48.4, 65.0 / 51.4, 69.7 / 50.9; 27 steps checked every seven 293 / 178, 301 / 189, 309 / 195).
//
// 3D (GLUPS, order 4, single steps -> pairs), cubes of side n:
//            n = 256         320         200         128          64
//   D3Q27 FP32 27.3 -> 44.6  27.0 -> 41.7  22.9 -> 33.1  26.4 -> 37.5  22.3 -> 30.9
//   D3Q19 FP32 40.0 -> 61.5  39.1 -> 61.2  33.1 -> 49.3  38.0 -> 49.2  30.8 -> 35.3
//   D3Q27 FP64 12.5 -> 21.6  11.7 -> 21.0  12.9 -> 17.9  13.0 -> 20.5  12.2 -> 16.5
//   D3Q19 FP64 18.3 -> 33.0  17.2 -> 31.6  18.9 -> 25.7  18.6 -> 29.5  16.5 -> 23.7
// Smaller boxes leave most compute units without a block, and the pair's march
// along z is then longer than two single steps (D3Q27 FP32 48^3 13.7 -> 15.0, 36^3
// 8.6 -> 8.0, 32^3 7.3 -> 5.9; D3Q19 FP32 48^3 18.2 -> 17.6, 24 x 24 x 330 20.3 -> 19.5):
// pairs are taken where the state, weighted by the used share of a tile's 64
// columns, has at least 6.5 MB, 20 MB with walls (single -> pairs, walls along z / on
// all axes: D3Q19 FP32 256^3 39.3 -> 56.2 / 51.3, 128^3 37.7 -> 46.5 / 42.8, 64^3 28.7 -> 30.0
// / 26.9; D3Q27 FP32 256^3 26.9 -> 41.1 / 37.8; D3Q19 FP64 256^3 18.1 -> 31.1 / 27.3).
// The pair pays for tiles, chunk edges and compute units left empty, single steps for
// nothing of the kind, so pairs also need a plan whose launch is filled to 0.30 (single -> pairs, us
// for four steps: D3Q27 FP32 500 x 2 x 1000 fill 0.22 157 -> 185, 163 x 5 x 235 0.29 51 -> 38, 500 x 3 x 1000
// 0.34 230 -> 221; D3Q27 FP64 16 x 400 x 400 0.24 1189 -> 1232, 22 x 240 x 240 0.31 595 -> 505; one plane
// of 500 x 1000 0.32 177 -> 196, so two at least, six between walls: D3Q19 FP32 500 x 1000 x 3 0.47
// 169 -> 188), with walls to 0.42 (walls on y and z: D3Q27 FP32 400 x 5 x 400
// 0.41 142 -> 159, 163 x 10 x 235 even, 500 x 6 x 1000 0.66 456 -> 375; D3Q19 FP64 28 x 240 x 240 0.40 473 -> 519), with
// walls on x, which every tile row's first and last tile hold, to 0.50 (D3Q27 FP32 75 x 131 x 150 0.48 270 ->
// 293, D3Q19 FP64 65 x 130 x 301 0.43 675 -> 721, 100 x 131 x 150 0.62 475 -> 417).
// FP32 rows that end inside a 64-byte half line are written twice where the caches do not hold the state, by a
// pair half as often: from 280 MB of padded rows 0.10, 0.15 and 0.42 suffice (D3Q27 7 x 400 x 400 fill 0.10
// 1037 -> 586, walls on y and z 11 x 400 x 400 0.16 1030 -> 805, on x 65 x 130 x 301 0.43 627 -> 563).
// LBRR_PAIR_LZ (0: no pairs) and LBRR_PAIR_ROWS override the choice.
TilePlan pair_plan(const LatticeOps& ops, int storage, const StepArgs& a, int walls) {
  TilePlan p;
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int forced_lz = env_int("LBRR_PAIR_LZ", -1);
  if (forced_lz == 0 || !lbrr::pair_offsets_fit(ops.d, a, int(elem_size(storage)))) return p;
  if (ops.d == 2) {
    p.rows = ops.tile_rows(storage, 0, walls != 0);
    if (p.rows == 0) return p;
    const int64_t gx = (nx + 253) / 254, cus = compute_units();  // k_step_pair2: 254 columns a block
    p.lz = forced_lz > 0 ? forced_lz : 0;
    const double used = nx / (254.0 * double(gx)), state = double(nx) * ny * ops.q * double(elem_size(storage));
    const bool narrow = used < 0.3 && gx * ny > (storage == LB_STORE_FP64 ? 2 : 4) * cus;
    if (forced_lz < 0 && narrow && (used < 0.15 || state < 32e6)) return TilePlan();
    if (p.lz == 0 && gx * ny <= 2 * cus) p.lz = 1;
    if (p.lz == 0 && gx * ((ny + 1) / 2) <= 3 * cus) p.lz = 2;
    if (p.lz == 0) p.lz = gx * ((ny + 3) / 4) <= 12 * cus ? 4 : 6;
    p.whole = forced_lz < 0 && state >= 2.5e6 && state <= 8e6;
    return p;
  }
  const int64_t gx = (nx + 63) / 64;
  const size_t es = elem_size(storage);
  const double state = double(nx) * ny * nz * ops.q * double(es), used = nx / (64.0 * double(gx));
  if (forced_lz < 0 && state * used < (walls ? 2e7 : 6.5e6)) return p;
  p = tile_plan(ops, storage, nx, ny, nz, walls != 0, forced_lz, env_int("LBRR_PAIR_ROWS", 0));
  if (forced_lz > 0) return p;
  const bool torn = es == 4 && nx * es % 64 != 0 && double(row_bytes(nx, es)) * ny * nz * ops.q >= 2.8e8;
  const double least = walls & 1 ? (torn ? 0.42 : 0.50) : (walls ? (torn ? 0.15 : 0.42) : (torn ? 0.10 : 0.30));
  return p.fill < least || nz < (walls & 4 ? 6 : 2) ? TilePlan() : p;
}

// The moment-state step: four rows per block in 2D (see kRowX in mkernels.hpp), the
// tile plan in 3D.  LBRR_MOM_LZ and LBRR_MOM_ROWS override the choice.
TilePlan moment_plan(const LatticeOps& ops, int storage, int nx, int ny, int nz, bool walls) {
  const int forced_lz = env_int("LBRR_MOM_LZ", 0);
  if (ops.d == 2) {
    TilePlan p;
    p.lz = forced_lz > 0 ? forced_lz : 4;
    return p;
  }
  return tile_plan(ops, storage, nx, ny, nz, walls, forced_lz, env_int("LBRR_MOM_ROWS", 0));
}

// Extra bytes after each population plane (layouts 0 and 2).  Planes whose
// size is a large power of two would otherwise start at addresses that map to
// the same HBM channels; the default adds 4 KiB + 256 B when the plane is a
// multiple of 64 KiB.  LBRR_PLANE_PAD_BYTES overrides it (rounded up to 256 B).
size_t plane_pad_bytes(size_t plane_bytes) {
  if (const char* e = std::getenv("LBRR_PLANE_PAD_BYTES")) {
    const long long v = std::atoll(e);
    if (v >= 0) return size_t((v + 255) / 256 * 256);
  }
  return (plane_bytes % 65536 == 0) ? 4352 : 0;
}

// Scratch of lb_reduce_static: the per-block partial totals (5 doubles per
// block, at most LB_REDUCE_STATIC_MAX_BLOCKS blocks) and nothing else (no ticket:
// calls that overlap would leave it wrong for good).  A file-scope device array: every GPU the library runs on holds its own copy
// (82 KB) until the process ends.  Host code never uses the name `scratch`
// as an address; it uses the per-device address that hipGetSymbolAddress
// returns (static_scratch below).
static __device__ __align__(256) double scratch[5 * LB_REDUCE_STATIC_MAX_BLOCKS];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch[kMaxDevices] = {};

// Address of `scratch` on the current device, looked up once per device.
int static_scratch(double** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) return fail(LB_ERR_UNSUPPORTED, "device index %d beyond %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    g_scratch[dev] = static_cast<double*>(p);
  }
  *out = g_scratch[dev];
  return LB_OK;
}

// Per-block partial count of the totals: one block per 256 nodes (a node per
// thread), at most LB_REDUCE_STATIC_MAX_BLOCKS (the handle path and
// lb_reduce_static use the same partition, so their sums are the same bits).
// With 2048 nodes a block a 64^2 grid ran on two blocks, eight nodes in turn.
int totals_blocks(int64_t nodes) {
  const int64_t nb = (nodes + 255) / 256;
  return int(nb < 1 ? 1 : (nb > LB_REDUCE_STATIC_MAX_BLOCKS ? LB_REDUCE_STATIC_MAX_BLOCKS : nb));
}

// Where a handle's reductions leave their few results.  The kernels write them to
// pinned host memory, so the host reads them as soon as the stream is done; a
// copy from device memory took 10 us and more of each lb_reduce and
// lb_enstrophy.  One pinned page per process holds 64-byte slots; a handle that
// finds none free (or no pinned memory) keeps its results in device memory and
// copies them.
struct ResultSlot {
  static constexpr int kSlots = 256, kDoubles = 8;
  double* device = nullptr;  // the kernels' address
  volatile double* host = nullptr;

  hipError_t acquire() {
    if (device) return hipSuccess;
    std::lock_guard<std::mutex> lock(mu());
    Page& p = page();
    if (!p.tried) {
      p.tried = true;
      void* m = nullptr;
      if (hipHostMalloc(&m, sizeof(double) * kDoubles * kSlots, hipHostMallocPortable | hipHostMallocMapped) ==
          hipSuccess)
        p.host = static_cast<double*>(m);
      else
        (void)hipGetLastError();
    }
    for (int i = 0; p.host && i < kSlots; ++i) {
      if (p.used[i]) continue;
      void* d = nullptr;
      if (hipHostGetDevicePointer(&d, p.host + i * kDoubles, 0) != hipSuccess) {
        (void)hipGetLastError();
        break;
      }
      p.used[i] = true;
      host = p.host + i * kDoubles;
      device = static_cast<double*>(d);
      return hipSuccess;
    }
    return hipMalloc(&device, sizeof(double) * kDoubles);
  }
  hipError_t read(double* out, int n, hipStream_t s) {
    hipError_t e = hipSuccess;
    if (!host) e = hipMemcpyAsync(out, device, sizeof(double) * n, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    for (int c = 0; host && c < n; ++c) out[c] = host[c];
    return e;
  }
  void release() {
    if (host) {
      std::lock_guard<std::mutex> lock(mu());
      page().used[(const_cast<double*>(host) - page().host) / kDoubles] = false;
    } else if (device) {
      (void)hipFree(device);
    }
    device = nullptr;
    host = nullptr;
  }

 private:
  struct Page {
    bool tried = false;
    double* host = nullptr;
    bool used[kSlots] = {};
  };
  static std::mutex& mu() {
    static std::mutex m;
    return m;
  }
  static Page& page() {
    static Page p;
    return p;
  }
};

}  // namespace

struct lb_ctx {
  int lattice = 0;
  const LatticeOps* ops = nullptr;
  int nx = 0, ny = 0, nz = 0;
  double tau = 0.0;
  int order = 0;
  int storage = LB_STORE_FP32;
  double rho0 = 1.0;
  int device = 0;
  hipStream_t stream = nullptr;
  void* buf[2] = {nullptr, nullptr};
  int cur = 0;
  int layout = 0;                  // 0 [q][z][y][x], 1 [z][y][q][x], 2 [z][q][y][x]
  int64_t si = 0, sy = 0, sz = 0;  // element strides of population, row, plane
  size_t buf_elems = 0;
  bool ready = false;
  long long steps = 0;
  long long check_every = 0;
  int walls = 0;  // bit 0 x, bit 1 y, bit 2 z: resting no-slip walls on the first and last node
  double* partials = nullptr;
  int nblocks = 0;
  unsigned* ticket = nullptr;  // of the reductions' blocks, behind the partials; NULL for large grids (reduce.hpp)
  ResultSlot slot;             // where they write their results
  double* vel = nullptr;
  // learned closure (D2Q9)
  bool closure_on = false;
  float* cl_params = nullptr;   // kMlpNParam
  float* cl_norm = nullptr;     // kMlpNNorm
  uint16_t* cl_packed = nullptr;

  int64_t nodes() const { return int64_t(nx) * ny * nz; }
  int q() const { return ops->q; }
  int d() const { return ops->d; }
  bool moment() const { return lbrr::is_moment_storage(storage); }
  // stored values per node: q populations, or rho - rho0, j and a1^(2)
  int nvalues() const { return moment() ? 1 + d() + d() * (d() + 1) / 2 : q(); }
  StepArgs args() const {
    StepArgs a;
    a.nx = nx;
    a.ny = ny;
    a.nz = nz;
    a.si = si;
    a.sy = sy;
    a.sz = sz;
    a.rho0 = rho0;
    a.omega1 = 1.0 - 1.0 / tau;
    a.lz = 1;
    a.rows = 0;
    a.walls = moment() ? walls : 0;
    return a;
  }
  void release() {
    for (void*& b : buf) {
      if (b) (void)hipFree(b);
      b = nullptr;
    }
    if (partials) (void)hipFree(partials);
    if (vel) (void)hipFree(vel);
    partials = nullptr;
    ticket = nullptr;
    slot.release();
    vel = nullptr;
    ready = false;
  }
  void release_closure() {
    for (void* p : {static_cast<void*>(cl_params), static_cast<void*>(cl_norm), static_cast<void*>(cl_packed)})
      if (p) (void)hipFree(p);
    cl_params = nullptr;
    cl_norm = nullptr;
    cl_packed = nullptr;
    closure_on = false;
  }
};

namespace {

// Population layout.  Measured on MI355X for the step kernel (GLUPS, each
// layout three times in one run, interleaved; runs agree to 1%):
//   * planes of at most 256 KiB (256^2 FP32, 256^2 / 320^2 FP16): keeping the
//     q planes of a z-slab together ([z][q][y][x], layout 2) is best
//     (D3Q27 256^3 FP32 27.5 against 26.7 for layout 1);
//   * larger planes: the q rows of a (y, z) row together ([z][y][q][x],
//     layout 1) for FP32 at every size and for the rest up to 448^2 planes
//     (D3Q27 384^3 FP16 55.3 against 53.1 / 53.0);
//   * planes of 512^2 nodes and more: FP16 keeps layout 2 (D3Q27 512^3 50.3
//     against 46.4 for layout 1, D3Q19 78.5 against 70.4) and FP64 one volume
//     per population ([q][z][y][x], layout 0; D3Q27 12.7 against 11.1,
//     D3Q19 18.2 against 16.4).
// LBRR_LAYOUT=0|1|2 overrides the choice.
int layout_choice(int d, int64_t nx, int64_t ny, size_t es) {
  if (const char* e = std::getenv("LBRR_LAYOUT")) {
    const int v = std::atoi(e);
    if (v >= 0 && v <= 2) return v;
  }
  if (d != 3) return 1;
  const int64_t plane_nodes = nx * ny;
  if (size_t(plane_nodes) * es <= 262144) return 2;
  if (plane_nodes >= 512 * 512) {
    if (es == 2) return 2;
    if (es == 8) return 0;
  }
  return 1;
}

// Moment-state layout: the fields of a (y, z) row together ([z][y][c][x],
// layout 1), so the patch of a step block reads one contiguous run per row.
// LBRR_LAYOUT=0|1|2 overrides the choice.
int moment_layout_choice() {
  if (const char* e = std::getenv("LBRR_LAYOUT")) {
    const int v = std::atoi(e);
    if (v >= 0 && v <= 2) return v;
  }
  return 1;
}

int ensure_buffers(lb_ctx* h) {
  if (h->buf[0]) return LB_OK;
  const size_t es = elem_size(h->storage);
  const int64_t nx = h->nx, ny = h->ny, nz = h->nz, q = h->nvalues();
  h->layout = h->moment() ? moment_layout_choice() : layout_choice(h->d(), nx, ny, es);
  const int64_t px = int64_t(row_bytes(nx, es) / es);
  size_t elems = 0;
  if (h->layout == 1) {  // rows of all populations together
    h->si = px;
    h->sy = q * px;
    h->sz = ny * q * px;
    elems = size_t(nz * ny * q * px);
  } else {
    const size_t plane = size_t(h->layout == 0 ? px * ny * nz : px * ny) * es;
    const size_t plane_al = (plane + 255) / 256 * 256;
    const size_t plane_bytes = plane_al + plane_pad_bytes(plane_al);
    const int64_t p = int64_t(plane_bytes / es);
    if (h->layout == 0) {
      h->si = p;
      h->sy = px;
      h->sz = px * ny;
      elems = size_t(q * p);
    } else {
      h->si = p;
      h->sy = px;
      h->sz = q * p;
      elems = size_t(nz * q * p);
    }
  }
  // every kernel index i*si + z*sz + y*sy + x must stay inside the allocation
  const int64_t max_index = (q - 1) * h->si + (nz - 1) * h->sz + (ny - 1) * h->sy + (nx - 1);
  if (max_index < 0 || size_t(max_index) >= elems)
    return fail(LB_ERR_INVALID_ARG, "internal layout error: max index %lld >= %zu", (long long)max_index, elems);
  h->buf_elems = elems;
  const size_t total = elems * es;
  for (int k = 0; k < 2; ++k) {
    hipError_t e = hipMalloc(&h->buf[k], total);
    if (e != hipSuccess) {
      h->release();
      (void)hipGetLastError();
      return fail(LB_ERR_OOM, "hipMalloc of %zu bytes for populations failed: %s", total, hipGetErrorString(e));
    }
  }
  h->nblocks = totals_blocks(h->nodes());
  // a failure here frees the population buffers too: buf[0] marks a complete set
  hipError_t e = hipMalloc(&h->partials, sizeof(double) * (5 * size_t(h->nblocks) + 1));
  if (e == hipSuccess && h->nblocks <= lbrr::kTicketBlocks) {
    h->ticket = reinterpret_cast<unsigned*>(h->partials + 5 * size_t(h->nblocks));
    e = lbrr::launch_zero(h->ticket, 1, h->stream);
  }
  if (e == hipSuccess) e = h->slot.acquire();
  if (e != hipSuccess) {
    h->release();
    (void)hipGetLastError();
    return fail(LB_ERR_OOM, "hipMalloc of the reduction buffers failed: %s", hipGetErrorString(e));
  }
  return LB_OK;
}

int check_handle(lb_ctx* h) {
  if (!h) return fail(LB_ERR_INVALID_ARG, "NULL handle");
  HIP_TRY(hipSetDevice(h->device), "hipSetDevice");
  return LB_OK;
}

int totals(lb_ctx* h, double out[5]) {
  hipError_t e = h->ops->totals(h->storage, h->buf[h->cur], h->partials, h->ticket, h->nblocks, h->slot.device,
                                h->args(), h->stream);
  if (e != hipSuccess) return hip_fail(e, "totals kernel launch");
  HIP_TRY(h->slot.read(out, 5, h->stream), "read totals");
  for (int c = 0; c < 5; ++c)
    if (!std::isfinite(out[c])) return fail(LB_ERR_UNSTABLE, "non-finite total after step %lld", h->steps);
  return LB_OK;
}

}  // namespace

extern "C" {

const char* lb_last_error(void) { return g_err.c_str(); }

lb_handle lb_create(int lattice, int nx, int ny, int nz, double tau, int order) {
  const LatticeOps* ops = nullptr;
  switch (lattice) {
    case LB_D2Q9: ops = &lbrr::ops_d2q9(); break;
    case LB_D3Q19: ops = &lbrr::ops_d3q19(); break;
    case LB_D3Q27: ops = &lbrr::ops_d3q27(); break;
    default: fail(LB_ERR_INVALID_ARG, "unknown lattice %d", lattice); return nullptr;
  }
  if (nx < 1 || ny < 1 || nz < 1 || ny > 65535 || nz > 65535) {
    fail(LB_ERR_INVALID_ARG, "dims must be >= 1 (ny, nz <= 65535), got %d x %d x %d", nx, ny, nz);
    return nullptr;
  }
  if (int64_t(nx) * ny * nz >= (int64_t(1) << 31)) {
    fail(LB_ERR_INVALID_ARG, "nx*ny*nz must be < 2^31");
    return nullptr;
  }
  if (ops->d == 2 && nz != 1) {
    fail(LB_ERR_INVALID_ARG, "D2Q9 requires nz == 1, got %d", nz);
    return nullptr;
  }
  if (!std::isfinite(tau) || !(tau > 0.5)) {
    fail(LB_ERR_INVALID_ARG, "tau must be finite and > 0.5, got %g", tau);
    return nullptr;
  }
  if (order < 2 || order > ops->nmax) {
    fail(LB_ERR_INVALID_ARG, "order must be in [2, %d] for this lattice, got %d", ops->nmax, order);
    return nullptr;
  }
  lb_ctx* h = new (std::nothrow) lb_ctx();
  if (!h) {
    fail(LB_ERR_OOM, "host allocation failed");
    return nullptr;
  }
  h->lattice = lattice;
  h->ops = ops;
  h->nx = nx;
  h->ny = ny;
  h->nz = nz;
  h->tau = tau;
  h->order = order;
  const hipError_t e = hipGetDevice(&h->device);
  if (e != hipSuccess) {
    delete h;
    fail(LB_ERR_HIP, "hipGetDevice failed: %s (%d)", hipGetErrorString(e), int(e));
    return nullptr;
  }
  g_err.clear();
  return h;
}

int lb_config(lb_handle h, int storage, double rho0) {
  if (int r = check_handle(h)) return r;
  if (storage < LB_STORE_FP64 || storage > LB_STORE_MOM_FP32) return fail(LB_ERR_INVALID_ARG, "bad storage %d", storage);
  if (!std::isfinite(rho0) || !(rho0 > 0)) return fail(LB_ERR_INVALID_ARG, "rho0 must be finite and > 0");
  if (h->buf[0]) HIP_TRY(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
  h->release();
  h->storage = storage;
  h->rho0 = rho0;
  h->steps = 0;
  return LB_OK;
}

int lb_set_stream(lb_handle h, void* hip_stream) {
  if (int r = check_handle(h)) return r;
  hipStream_t next = static_cast<hipStream_t>(hip_stream);
  if (next != h->stream && h->buf[0]) {
    // work already enqueued on the old stream comes first: the new stream
    // waits for an event recorded behind it (nothing blocks the host)
    hipEvent_t ev;
    HIP_TRY(hipEventCreateWithFlags(&ev, hipEventDisableTiming), "hipEventCreate");
    hipError_t e = hipEventRecord(ev, h->stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(next, ev, 0);
    (void)hipEventDestroy(ev);
    if (e != hipSuccess) return hip_fail(e, "ordering the new stream after the old one");
  }
  h->stream = next;
  return LB_OK;
}

int lb_set_walls(lb_handle h, int walls) {
  if (int r = check_handle(h)) return r;
  if (walls < 0 || walls > 7) return fail(LB_ERR_INVALID_ARG, "walls must be a mask of bits 0 (x), 1 (y), 2 (z)");
  if ((walls & 4) && h->d() == 2) return fail(LB_ERR_INVALID_ARG, "a 2D lattice has no z walls");
  const int dims[3] = {h->nx, h->ny, h->nz};
  for (int k = 0; k < 3; ++k)
    if ((walls >> k & 1) && dims[k] < 3) return fail(LB_ERR_INVALID_ARG, "a walled axis needs at least 3 nodes");
  h->walls = walls;
  return LB_OK;
}

int lb_set_check_interval(lb_handle h, long long k) {
  if (int r = check_handle(h)) return r;
  if (k < 0) return fail(LB_ERR_INVALID_ARG, "check interval must be >= 0");
  h->check_every = k;
  return LB_OK;
}

int lb_init_fields(lb_handle h, const void* rho, const void* u, const void* pi1, int dtype, int on_device) {
  if (int r = check_handle(h)) return r;
  if (!rho || !u) return fail(LB_ERR_INVALID_ARG, "rho and u must not be NULL");
  if (dtype != LB_F64 && dtype != LB_F32) return fail(LB_ERR_INVALID_ARG, "bad dtype %d", dtype);
  if (int r = ensure_buffers(h)) return r;
  const size_t es = dtype == LB_F64 ? 8 : 4;
  const size_t nodes = size_t(h->nodes());
  const int d = h->d(), nc = d * (d + 1) / 2;
  const void *drho = rho, *du = u, *dpi = pi1;
  void* tmp = nullptr;
  if (!on_device) {
    const size_t n = nodes * (1 + d + (pi1 ? nc : 0));
    HIP_TRY(hipMalloc(&tmp, n * es), "hipMalloc staging");
    char* t = static_cast<char*>(tmp);
    hipError_t e = hipMemcpyAsync(t, rho, nodes * es, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(t + nodes * es, u, nodes * d * es, hipMemcpyHostToDevice, h->stream);
    if (e == hipSuccess && pi1)
      e = hipMemcpyAsync(t + nodes * (1 + d) * es, pi1, nodes * nc * es, hipMemcpyHostToDevice, h->stream);
    if (e != hipSuccess) {
      (void)hipFree(tmp);
      return hip_fail(e, "staging copy");
    }
    drho = t;
    du = t + nodes * es;
    dpi = pi1 ? t + nodes * (1 + d) * es : nullptr;
  }
  hipError_t e = h->ops->init(h->order, h->storage, dtype, drho, du, dpi, h->buf[0], h->args(), h->stream);
  if (tmp) {
    hipError_t s = hipStreamSynchronize(h->stream);
    (void)hipFree(tmp);
    if (e == hipSuccess) e = s;
  }
  if (e != hipSuccess) return hip_fail(e, "init kernel");
  h->cur = 0;
  h->steps = 0;
  h->ready = true;
  return LB_OK;
}

int lb_step(lb_handle h, long long n) {
  if (int r = check_handle(h)) return r;
  if (n < 0) return fail(LB_ERR_INVALID_ARG, "n must be >= 0");
  if (!h->ready) return fail(LB_ERR_STATE, "lb_step before lb_init_fields / lb_set_populations");
  if (h->closure_on && h->moment()) return fail(LB_ERR_UNSUPPORTED, "the learned closure needs population storage");
  if (h->walls && h->closure_on) return fail(LB_ERR_UNSUPPORTED, "walls and the learned closure exclude each other");
  StepArgs a = h->args();
  if (h->moment()) {
    const TilePlan p = moment_plan(*h->ops, h->storage, h->nx, h->ny, h->nz, h->walls != 0);
    a.rows = p.rows;
    a.lz = p.lz;
  }
  // Two steps in one launch where the population step has that form, always two
  // such launches at a time: every call then swaps the state buffers as often,
  // modulo 2, as single steps would (an even number of steps ends in the buffer
  // it started from, which replays of a captured run rely on).
  StepArgs ap = a;
  TilePlan pairs;
  if (n >= 4 && !h->moment() && !h->closure_on) pairs = pair_plan(*h->ops, h->storage, a, h->walls);
  if (pairs.whole && n > 4 && n < 8 && h->check_every == 0) pairs = TilePlan();
  ap.rows = pairs.rows;
  ap.lz = pairs.lz;
  ap.walls = h->walls;
  while (n > 0) {
    long long run = n;  // steps up to the end of the call or the next check
    if (h->check_every > 0) run = std::min(run, h->check_every - h->steps % h->check_every);
    n -= run;
    long long paired = pairs.lz > 0 ? run / 4 * 2 : 0;  // launches of two steps
    for (run -= 2 * paired; paired > 0 || run > 0;) {
      const int steps = paired > 0 ? 2 : 1;
      const void* src = h->buf[h->cur];
      void* dst = h->buf[1 - h->cur];
      hipError_t e;
      if (paired > 0)
        e = h->ops->step_pair(h->order, h->storage, src, dst, ap, h->stream);
      else if (h->closure_on)
        e = lbrr::closure_step(h->order, h->storage, src, dst, a, h->cl_packed, h->cl_params, h->cl_norm, h->stream);
      else if (h->walls && !h->moment())
        e = h->ops->step_walls(h->order, h->storage, src, dst, a, h->walls, h->stream);
      else
        e = h->ops->step(h->order, h->storage, src, dst, a, h->stream);
      if (e != hipSuccess) return hip_fail(e, "step kernel launch");
      h->cur ^= 1;
      h->steps += steps;
      --(steps == 2 ? paired : run);
    }
    if (h->check_every > 0 && h->steps % h->check_every == 0) {
      double t[5];
      if (int r = totals(h, t)) return r;
    }
  }
  return LB_OK;
}

int lb_moments(lb_handle h, void* rho, void* u, void* pi1, int dtype, int on_device) {
  if (int r = check_handle(h)) return r;
  if (!h->ready) return fail(LB_ERR_STATE, "no state: call lb_init_fields or lb_set_populations first");
  if (dtype != LB_F64 && dtype != LB_F32) return fail(LB_ERR_INVALID_ARG, "bad dtype %d", dtype);
  const double om = 1.0 - 1.0 / h->tau;
  if (pi1 && om == 0.0 && !h->moment())
    return fail(LB_ERR_UNSUPPORTED, "pi1 is not recoverable from the stored state when tau == 1");
  const double inv_om = (pi1 && !h->moment()) ? 1.0 / om : 0.0;
  const size_t es = dtype == LB_F64 ? 8 : 4;
  const size_t nodes = size_t(h->nodes());
  const int d = h->d(), nc = d * (d + 1) / 2;
  if (on_device) {
    hipError_t e = h->ops->moments(h->storage, dtype, h->buf[h->cur], rho, u, pi1, h->args(), inv_om, h->stream);
    if (e != hipSuccess) return hip_fail(e, "moments kernel");
    HIP_TRY(hipStreamSynchronize(h->stream), "hipStreamSynchronize");
    return LB_OK;
  }
  void* tmp = nullptr;
  HIP_TRY(hipMalloc(&tmp, nodes * (1 + d + nc) * es), "hipMalloc staging");
  char* t = static_cast<char*>(tmp);
  void* drho = rho ? t : nullptr;
  void* du = u ? t + nodes * es : nullptr;
  void* dpi = pi1 ? t + nodes * (1 + d) * es : nullptr;
  hipError_t e = h->ops->moments(h->storage, dtype, h->buf[h->cur], drho, du, dpi, h->args(), inv_om, h->stream);
  if (e == hipSuccess && rho) e = hipMemcpyAsync(rho, drho, nodes * es, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess && u) e = hipMemcpyAsync(u, du, nodes * d * es, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess && pi1) e = hipMemcpyAsync(pi1, dpi, nodes * nc * es, hipMemcpyDeviceToHost, h->stream);
  hipError_t s = hipStreamSynchronize(h->stream);
  (void)hipFree(tmp);
  if (e == hipSuccess) e = s;
  if (e != hipSuccess) return hip_fail(e, "moments");
  return LB_OK;
}

int lb_reduce(lb_handle h, double out[5]) {
  if (int r = check_handle(h)) return r;
  if (!out) return fail(LB_ERR_INVALID_ARG, "out must not be NULL");
  if (!h->ready) return fail(LB_ERR_STATE, "no state");
  return totals(h, out);
}

int lb_reduce_static(int lattice, int storage, int nx, int ny, int nz, double rho0, const void* populations,
                     double* out, void* hip_stream) {
  const LatticeOps* ops = nullptr;
  switch (lattice) {
    case LB_D2Q9: ops = &lbrr::ops_d2q9(); break;
    case LB_D3Q19: ops = &lbrr::ops_d3q19(); break;
    case LB_D3Q27: ops = &lbrr::ops_d3q27(); break;
    default: return fail(LB_ERR_INVALID_ARG, "unknown lattice %d", lattice);
  }
  if (storage != LB_STORE_FP64 && storage != LB_STORE_FP32 && storage != LB_STORE_FP16)
    return fail(LB_ERR_UNSUPPORTED, "lb_reduce_static takes population storage (FP64, FP32, FP16), got %d", storage);
  if (nx < 1 || ny < 1 || nz < 1 || (ops->d == 2 && nz != 1))
    return fail(LB_ERR_INVALID_ARG, "bad dims %d x %d x %d for this lattice", nx, ny, nz);
  const int64_t nodes = int64_t(nx) * ny * nz;
  if (nodes >= (int64_t(1) << 31)) return fail(LB_ERR_INVALID_ARG, "nx*ny*nz must be < 2^31");
  if (!std::isfinite(rho0) || !(rho0 > 0)) return fail(LB_ERR_INVALID_ARG, "rho0 must be finite and > 0");
  if (!populations || !out) return fail(LB_ERR_INVALID_ARG, "populations and out must not be NULL");
  const int nblocks = totals_blocks(nodes);
  if (nblocks > LB_REDUCE_STATIC_MAX_BLOCKS)
    return fail(LB_ERR_INVALID_ARG, "%d partial blocks exceed the static scratch (%d)", nblocks,
                LB_REDUCE_STATIC_MAX_BLOCKS);
  double* partials = nullptr;
  if (int r = static_scratch(&partials)) return r;
  StepArgs a{};
  a.nx = nx;
  a.ny = ny;
  a.nz = nz;
  a.si = nodes;  // compact [q][nz][ny][nx]
  a.sy = nx;
  a.sz = int64_t(nx) * ny;
  a.rho0 = rho0;
  a.omega1 = 0.0;
  a.lz = 1;
  a.walls = 0;
  const hipError_t e =
      ops->totals(storage, populations, partials, nullptr, nblocks, out, a, static_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return hip_fail(e, "totals kernel launch");
  return LB_OK;
}

int lb_enstrophy(lb_handle h, double* out) {
  if (int r = check_handle(h)) return r;
  if (!out) return fail(LB_ERR_INVALID_ARG, "out must not be NULL");
  if (!h->ready) return fail(LB_ERR_STATE, "no state");
  if (!h->vel) HIP_TRY(hipMalloc(&h->vel, sizeof(double) * size_t(h->nodes()) * h->d()), "hipMalloc velocity");
  hipError_t e = h->ops->velocity(h->storage, h->buf[h->cur], h->vel, h->args(), h->stream);
  if (e == hipSuccess)
    e = lbrr::launch_enstrophy(h->vel, h->d(), h->nx, h->ny, h->nz, h->walls, h->partials, h->ticket, h->nblocks,
                               h->slot.device, h->stream);
  if (e != hipSuccess) return hip_fail(e, "enstrophy kernels");
  double s = 0.0;
  HIP_TRY(h->slot.read(&s, 1, h->stream), "read enstrophy");
  // trapezoid volume: a walled axis of n nodes spans n - 1 cells, a periodic one n
  double vol = 1.0;
  const int dims[3] = {h->nx, h->ny, h->nz};
  for (int k = 0; k < h->d(); ++k) vol *= double((h->walls >> k & 1) ? dims[k] - 1 : dims[k]);
  *out = s / vol;
  if (!std::isfinite(*out)) return fail(LB_ERR_UNSTABLE, "non-finite enstrophy");
  return LB_OK;
}

int lb_get_populations(lb_handle h, void* dst, int on_device) {
  if (int r = check_handle(h)) return r;
  if (!dst) return fail(LB_ERR_INVALID_ARG, "dst must not be NULL");
  if (!h->ready) return fail(LB_ERR_STATE, "no state");
  const size_t bytes = size_t(h->nodes()) * h->q() * elem_size(h->storage);
  void* d = dst;
  if (!on_device) HIP_TRY(hipMalloc(&d, bytes), "hipMalloc staging");
  hipError_t e = h->moment() ? h->ops->mpopulations(h->order, h->storage, h->buf[h->cur], d, h->args(), h->stream)
                             : h->ops->repack(h->storage, h->buf[h->cur], d, true, h->args(), h->stream);
  if (e == hipSuccess && !on_device) e = hipMemcpyAsync(dst, d, bytes, hipMemcpyDeviceToHost, h->stream);
  hipError_t s = hipStreamSynchronize(h->stream);
  if (!on_device) (void)hipFree(d);
  if (e == hipSuccess) e = s;
  if (e != hipSuccess) return hip_fail(e, "copy populations out");
  return LB_OK;
}

int lb_set_populations(lb_handle h, const void* src, int on_device) {
  if (int r = check_handle(h)) return r;
  if (!src) return fail(LB_ERR_INVALID_ARG, "src must not be NULL");
  if (h->moment())
    return fail(LB_ERR_UNSUPPORTED, "moment storage holds only states reachable by the collision; use lb_init_fields");
  if (int r = ensure_buffers(h)) return r;
  const size_t bytes = size_t(h->nodes()) * h->q() * elem_size(h->storage);
  const void* d = src;
  void* tmp = nullptr;
  if (!on_device) {
    HIP_TRY(hipMalloc(&tmp, bytes), "hipMalloc staging");
    hipError_t e = hipMemcpyAsync(tmp, src, bytes, hipMemcpyHostToDevice, h->stream);
    if (e != hipSuccess) {
      (void)hipFree(tmp);
      return hip_fail(e, "copy populations in");
    }
    d = tmp;
  }
  hipError_t e = h->ops->repack(h->storage, d, h->buf[h->cur], false, h->args(), h->stream);
  hipError_t s = hipStreamSynchronize(h->stream);
  if (tmp) (void)hipFree(tmp);
  if (e == hipSuccess) e = s;
  if (e != hipSuccess) return hip_fail(e, "copy populations in");
  h->ready = true;
  return LB_OK;
}

long long lb_step_count(lb_handle h) { return h ? h->steps : -1; }

double lb_bytes_per_update(lb_handle h) {
  if (!h) return 0.0;
  return 2.0 * h->nvalues() * double(elem_size(h->storage));
}

void lb_destroy(lb_handle h) {
  if (!h) return;
  (void)hipSetDevice(h->device);
  if (h->buf[0]) (void)hipStreamSynchronize(h->stream);
  h->release();
  h->release_closure();
  delete h;
}

// ---------------------------------------------------------------------------
// Learned closure (D2Q9).

namespace {

// Reusable device workspace of the MLP entry points (grown on demand; calls
// that overlap on one device must not share it).
struct Workspace {
  void* ptr = nullptr;
  size_t size = 0;
  int device = -1;
};
Workspace g_ws;

int workspace(size_t bytes, void** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
  if (g_ws.ptr && (g_ws.size < bytes || g_ws.device != dev)) {
    int cur = dev;
    (void)hipSetDevice(g_ws.device);
    (void)hipDeviceSynchronize();
    (void)hipFree(g_ws.ptr);
    (void)hipSetDevice(cur);
    g_ws.ptr = nullptr;
  }
  if (!g_ws.ptr) {
    const size_t sz = bytes < (size_t(1) << 20) ? (size_t(1) << 20) : bytes;
    HIP_TRY(hipMalloc(&g_ws.ptr, sz), "hipMalloc MLP workspace");
    g_ws.size = sz;
    g_ws.device = dev;
  }
  *out = g_ws.ptr;
  return LB_OK;
}

// Scratch of one call, allocated and freed in stream order from a pool of the
// device's own, so calls on any streams and threads have their own.  The pool
// keeps at most kScratchKeep bytes between calls.  ptr stays NULL where there is none to be
// had: under stream capture (an allocation has no place in the graph), on a device
// without memory pools, and when the allocation fails; callers then take a form without it.
constexpr uint64_t kScratchKeep = uint64_t(8) << 20;
std::mutex g_pool_mu;
hipMemPool_t g_pool[kMaxDevices] = {};

struct Scratch {
  void* ptr = nullptr;
  hipStream_t stream = nullptr;
  Scratch() = default;
  Scratch(const Scratch&) = delete;
  Scratch& operator=(const Scratch&) = delete;
  ~Scratch() {
    if (ptr) (void)hipFreeAsync(ptr, stream);
  }
  void allocate(size_t bytes, hipStream_t s) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(s, &cap);
    if (e == hipSuccess && cap != hipStreamCaptureStatusNone) return;
    hipMemPool_t pool = nullptr;
    if (e == hipSuccess) e = device_pool(&pool);
    if (e == hipSuccess) e = hipMallocFromPoolAsync(&ptr, bytes, pool, s);
    if (e != hipSuccess) {
      ptr = nullptr;
      (void)hipGetLastError();
    }
    stream = s;
  }

 private:
  static hipError_t device_pool(hipMemPool_t* pool) {
    int dev = 0, has = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorNotSupported;
    std::lock_guard<std::mutex> lock(g_pool_mu);
    if (!g_pool[dev]) {
      e = hipDeviceGetAttribute(&has, hipDeviceAttributeMemoryPoolsSupported, dev);
      if (e != hipSuccess || !has) return hipErrorNotSupported;
      hipMemPoolProps props{};
      props.allocType = hipMemAllocationTypePinned;
      props.location.type = hipMemLocationTypeDevice;
      props.location.id = dev;
      e = hipMemPoolCreate(pool, &props);
      if (e != hipSuccess) return e;
      uint64_t keep = kScratchKeep;
      if (hipMemPoolSetAttribute(*pool, hipMemPoolAttrReleaseThreshold, &keep) != hipSuccess)
        (void)hipGetLastError();  // it then keeps nothing between calls
      g_pool[dev] = *pool;
    }
    *pool = g_pool[dev];
    return hipSuccess;
  }
};

}  // namespace

int lb_set_closure(lb_handle h, const float* params, const float* norm, int enable) {
  if (int r = check_handle(h)) return r;
  if (h->lattice != LB_D2Q9) return fail(LB_ERR_UNSUPPORTED, "the learned closure is implemented for D2Q9 only");
  if (enable && h->moment()) return fail(LB_ERR_UNSUPPORTED, "the learned closure needs population storage");
  if (!enable) {
    h->closure_on = false;
    return LB_OK;
  }
  if (!params || !norm) return fail(LB_ERR_INVALID_ARG, "params and norm must not be NULL");
  // each buffer on its own, through a temporary: after a failed allocation the
  // handle holds only complete buffers, and the next call allocates the rest
  auto alloc = [](auto*& dst, size_t bytes) {
    void* p = nullptr;
    const hipError_t e = dst ? hipSuccess : hipMalloc(&p, bytes);
    if (e == hipSuccess && !dst) dst = static_cast<std::remove_reference_t<decltype(dst)>>(p);
    return e;
  };
  HIP_TRY(alloc(h->cl_params, sizeof(float) * lbrr::kMlpNParam), "hipMalloc closure params");
  HIP_TRY(alloc(h->cl_norm, sizeof(float) * lbrr::kMlpNNorm), "hipMalloc closure norm");
  HIP_TRY(alloc(h->cl_packed, sizeof(uint16_t) * (lbrr::kMlpNPacked + lbrr::kMlpNRegImage)),
          "hipMalloc closure weights");
  HIP_TRY(hipMemcpyAsync(h->cl_params, params, sizeof(float) * lbrr::kMlpNParam, hipMemcpyDeviceToDevice, h->stream),
          "copy closure params");
  HIP_TRY(hipMemcpyAsync(h->cl_norm, norm, sizeof(float) * lbrr::kMlpNNorm, hipMemcpyDeviceToDevice, h->stream),
          "copy closure norm");
  hipError_t e = lbrr::mlp_pack_step(h->cl_params, h->cl_packed, h->stream);
  if (e != hipSuccess) return hip_fail(e, "pack closure weights");
  h->closure_on = true;
  return LB_OK;
}

int lb_closure_features(lb_handle h, const double* a_target, double plain_weight, float* features, float* labels) {
  if (int r = check_handle(h)) return r;
  if (h->lattice != LB_D2Q9) return fail(LB_ERR_UNSUPPORTED, "the learned closure is implemented for D2Q9 only");
  if (!features || !labels) return fail(LB_ERR_INVALID_ARG, "features and labels must not be NULL");
  if (h->moment()) return fail(LB_ERR_UNSUPPORTED, "closure features need population storage");
  if (!h->ready) return fail(LB_ERR_STATE, "no state");
  hipError_t e = lbrr::closure_features(h->storage, h->buf[h->cur], h->args(), a_target, plain_weight, features, labels,
                                        h->stream);
  if (e != hipSuccess) return hip_fail(e, "closure features");
  return LB_OK;
}

int lb_closure_coarsen(const void* rho, const void* u, const void* pi1, int dtype, int nfx, int nfy, int factor,
                       double alpha, double beta, double* rho_c, double* u_c, double* pi1_c, void* hip_stream) {
  if (!rho || !u || !pi1 || !rho_c || !u_c || !pi1_c) return fail(LB_ERR_INVALID_ARG, "NULL pointer");
  if (dtype != LB_F64 && dtype != LB_F32) return fail(LB_ERR_INVALID_ARG, "bad dtype %d", dtype);
  if (factor < 1 || nfx < factor || nfy < factor || nfx % factor || nfy % factor)
    return fail(LB_ERR_INVALID_ARG, "fine dims must be positive multiples of the factor");
  if (!std::isfinite(alpha) || !std::isfinite(beta)) return fail(LB_ERR_INVALID_ARG, "alpha, beta must be finite");
  hipError_t e = lbrr::closure_coarsen(dtype, rho, u, pi1, nfx, nfy, factor, alpha, beta, rho_c, u_c, pi1_c,
                                       static_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return hip_fail(e, "coarsen kernel");
  return LB_OK;
}

int lb_mlp_forward(const float* params, const float* norm, const float* x, long long n, float* y, void* hip_stream) {
  if (!params || !norm || (n > 0 && (!x || !y))) return fail(LB_ERR_INVALID_ARG, "NULL pointer");
  if (n < 0) return fail(LB_ERR_INVALID_ARG, "n must be >= 0");
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const hipError_t e = lbrr::mlp_infer(x, n, params, norm, y, s);
  if (e != hipSuccess) return hip_fail(e, "MLP forward");
  return LB_OK;
}

int lb_mlp_gradient(const float* params, const float* norm, const float* x, const float* t, long long n,
                    const int* idx, int batch, float* grad, float* loss, void* hip_stream) {
  if (!params || !norm || !x || !t || !idx || !grad) return fail(LB_ERR_INVALID_ARG, "NULL pointer");
  if (batch < 1 || n < 1) return fail(LB_ERR_INVALID_ARG, "batch and n must be >= 1");
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int nb = lbrr::mlp_train_blocks(batch);
  const size_t part_bytes = sizeof(float) * size_t(nb) * lbrr::kMlpNParam;
  void* ws = nullptr;
  if (int r = workspace(part_bytes + sizeof(float) * size_t(nb), &ws)) return r;
  float* gpart = static_cast<float*>(ws);
  float* lpart = gpart + size_t(nb) * lbrr::kMlpNParam;
  const hipError_t e = lbrr::mlp_gradient(x, t, n, idx, batch, params, norm, gpart, lpart, grad, loss, s);
  if (e != hipSuccess) return hip_fail(e, "MLP gradient");
  return LB_OK;
}

int lb_column_stats(const float* x, long long n, int dim, float* mean, float* std, void* hip_stream) {
  if (!x || !mean || !std) return fail(LB_ERR_INVALID_ARG, "NULL pointer");
  if (n < 1 || dim < 1) return fail(LB_ERR_INVALID_ARG, "n and dim must be >= 1");
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  Scratch part;
  if (!lbrr::column_stats_direct(n, dim)) {
    const size_t bytes = sizeof(double) * 2 * size_t(dim) * size_t(lbrr::column_stats_runs(n, dim));
    part.allocate(bytes, s);
  }
  const hipError_t e = lbrr::column_stats(x, n, dim, static_cast<double*>(part.ptr), mean, std, s);
  if (e != hipSuccess) return hip_fail(e, "column stats kernel");
  return LB_OK;
}

int lb_mlp_adam(float* params, float* m, float* v, const float* grad, long long step, float lr, float beta1,
                float beta2, float eps, void* hip_stream) {
  if (!params || !m || !v || !grad) return fail(LB_ERR_INVALID_ARG, "NULL pointer");
  if (step < 1) return fail(LB_ERR_INVALID_ARG, "step counts from 1");
  hipError_t e = lbrr::mlp_adam(params, m, v, grad, step, lr, beta1, beta2, eps, static_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return hip_fail(e, "Adam kernel");
  return LB_OK;
}

int lb_probe_copy(const void* src, void* dst, size_t n, void* hip_stream) {
  if (!src || !dst) return fail(LB_ERR_INVALID_ARG, "NULL pointer");
  if (n % 16 || (reinterpret_cast<uintptr_t>(src) % 16) || (reinterpret_cast<uintptr_t>(dst) % 16))
    return fail(LB_ERR_INVALID_ARG, "copy needs 16-byte aligned pointers and a size multiple of 16");
  hipError_t e = lbrr::launch_copy(src, dst, n, static_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return hip_fail(e, "copy kernel");
  return LB_OK;
}

int lb_probe_bandwidth(int kind, int vec_bytes, int blocks_per_cu, int nontemporal, int streams, const void* src,
                       void* dst, size_t n, void* hip_stream) {
  if (kind < 0 || kind > 3) return fail(LB_ERR_INVALID_ARG, "kind must be 0 (copy), 1 (read), 2 (write) or 3 (streams)");
  if (vec_bytes != 4 && vec_bytes != 8 && vec_bytes != 16) return fail(LB_ERR_INVALID_ARG, "vec_bytes must be 4, 8 or 16");
  if (blocks_per_cu < 0 || blocks_per_cu > 64) return fail(LB_ERR_INVALID_ARG, "blocks_per_cu must be in [0, 64]");
  if (kind == 3 && (streams < 1 || streams > 32)) return fail(LB_ERR_INVALID_ARG, "streams must be in [1, 32]");
  if (kind == 3 && blocks_per_cu != 0) return fail(LB_ERR_INVALID_ARG, "the stream copy launches one thread per element");
  if (!src || !dst) return fail(LB_ERR_INVALID_ARG, "NULL pointer");
  if (n % 16 || (reinterpret_cast<uintptr_t>(src) % 16) || (reinterpret_cast<uintptr_t>(dst) % 16))
    return fail(LB_ERR_INVALID_ARG, "probes need 16-byte aligned pointers and a size multiple of 16");
  if (kind == 3 && (n / size_t(vec_bytes)) % size_t(streams))
    return fail(LB_ERR_INVALID_ARG, "the stream copy needs a whole number of elements per stream");
  int dev = 0, cus = 0;
  HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
  HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), "hipDeviceGetAttribute");
  const hipError_t e = lbrr::launch_probe(kind, vec_bytes, blocks_per_cu, nontemporal, streams, src, dst, n, cus,
                                          static_cast<hipStream_t>(hip_stream));
  if (e != hipSuccess) return hip_fail(e, "probe kernel");
  return LB_OK;
}

}  // extern "C"
