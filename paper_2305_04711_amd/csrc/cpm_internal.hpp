// Internal declarations of libcpm (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdio>
#include <string>
#include <vector>

#include "../../include/cpm.h"

namespace cpm {

// ------------------------------------------------------------------ errors
void set_error(const char* fmt, ...);

struct Error {
  cpm_status code;
};

#define CPM_HIP(call)                                                        \
  do {                                                                       \
    hipError_t e_ = (call);                                                  \
    if (e_ != hipSuccess) {                                                  \
      ::cpm::set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), \
                       __FILE__, __LINE__);                                  \
      throw ::cpm::Error{e_ == hipErrorOutOfMemory ? CPM_E_OOM : CPM_E_HIP}; \
    }                                                                        \
  } while (0)

#define CPM_FAIL(code, ...)          \
  do {                               \
    ::cpm::set_error(__VA_ARGS__);   \
    throw ::cpm::Error{code};        \
  } while (0)

#define CPM_LAUNCH_CHECK() CPM_HIP(hipGetLastError())

// Runs f and converts exceptions into a status (no exception crosses the ABI).
template <class F>
cpm_status guard(F&& f) {
  try {
    f();
    return CPM_OK;
  } catch (const Error& e) {
    return e.code;
  } catch (const std::exception& e) {
    set_error("internal error: %s", e.what());
    return CPM_E_INVALID;
  } catch (...) {
    set_error("internal error");
    return CPM_E_INVALID;
  }
}

// --------------------------------------------------------------- geometry
// Block layout: 3-D blocks are 4x4x4 nodes, 2-D blocks 8x8 nodes; both hold
// 64 nodes, one wavefront, one 64-bit occupancy mask.  Slot s of a block:
// 3-D s = lx + 4 ly + 16 lz, 2-D s = lx + 8 ly.
template <int DIM> struct Geo;
template <> struct Geo<3> {
  static constexpr int BX = 4, SH = 2, NNBR = 27;
  __host__ __device__ static int slot(int lx, int ly, int lz) { return lx + 4 * ly + 16 * lz; }
  __host__ __device__ static int lx(int s) { return s & 3; }
  __host__ __device__ static int ly(int s) { return (s >> 2) & 3; }
  __host__ __device__ static int lz(int s) { return s >> 4; }
  __host__ __device__ static int code(int dx, int dy, int dz) { return (dz + 1) * 9 + (dy + 1) * 3 + (dx + 1); }
};
template <> struct Geo<2> {
  static constexpr int BX = 8, SH = 3, NNBR = 9;
  __host__ __device__ static int slot(int lx, int ly, int) { return lx + 8 * ly; }
  __host__ __device__ static int lx(int s) { return s & 7; }
  __host__ __device__ static int ly(int s) { return s >> 3; }
  __host__ __device__ static int lz(int) { return 0; }
  __host__ __device__ static int code(int dx, int dy, int) { return (dy + 1) * 3 + (dx + 1); }
};

struct Workspace;

// Device memory of a band or batch: through the caller's cpm_allocator (with
// the stream given at creation), or hipMalloc / hipFree when none was given.
// get() throws CPM_E_OOM when the allocator fails; after a caller's
// allocation it synchronises that stream, so that no work the allocator's
// stream still had queued on the block overlaps the library's use of it on
// other streams.
struct DevAlloc {
  cpm_allocator a{};
  hipStream_t st = nullptr;
  bool custom() const { return a.alloc != nullptr; }
  void* get(size_t bytes) const;
  void put(void* p, size_t bytes) const noexcept;
};

// Occupancy mask and first DOF of one block (mask 0 when the block is absent).
struct QMeta {
  unsigned long long mask;
  int off;
  int pad;
};

// Explicit E rows as a wavefront takes them: kRows rows, four to a lane (M
// lanes to a row, lane = member).  Row j of lane l is
// row(wavefront, j, l); its column is component j of the lane's int4.
template <int DIM> struct ERowPack {
  static constexpr int M = DIM == 3 ? 64 : 16, kRows = 4 * (64 / M);
  __host__ __device__ static int64_t row(int64_t wave, int j, int lane) {
    return (wave * 4 + j) * (64 / M) + lane / M;
  }
  static int padded(int n) { return (n + kRows - 1) / kRows * kRows; }
};
inline int erow_padded(int dim, int n) {
  return dim == 3 ? ERowPack<3>::padded(n) : ERowPack<2>::padded(n);
}


// The slots of a block (mask) that have an entry in some buffer, one after
// the other from off.
struct Pull {
  unsigned long long mask;
  long long off;
};

// Supertiles stage the blocks from their corner on, 3 x 3 x 2 (2-D: 3 x 3);
// the last node along each axis is beyond every stencil.  Slots of staged
// block q that are inside, and the nodes inside altogether (at most).
template <int DIM> struct Super {
  static constexpr int EX = 3 * Geo<DIM>::BX - 1;              // staged edge, x and y
  static constexpr int EZ = DIM == 3 ? 2 * Geo<3>::BX - 1 : 1; // staged edge, z
  static constexpr int NB = DIM == 3 ? 18 : 9;                 // staged blocks
  static constexpr int CELLS = EX * EX * EZ;
  __host__ __device__ static constexpr unsigned long long inside(int q) {
    unsigned long long in = 0ull;
    constexpr int BX = DIM == 3 ? 4 : 8;
    for (int s = 0; s < 64; ++s) {
      const int x = DIM == 3 ? s & 3 : s & 7, y = DIM == 3 ? (s >> 2) & 3 : s >> 3,
                z = DIM == 3 ? s >> 4 : 0;
      const bool out = (q % 3 == 2 && x == BX - 1) || ((q / 3) % 3 == 2 && y == BX - 1) ||
                       (DIM == 3 && q / 9 == 1 && z == BX - 1);
      if (!out) in |= 1ull << s;
    }
    return in;
  }
};

// the same for every block, evaluated at compile time
template <int DIM> struct InsideMasks {
  unsigned long long m[18];
};
template <int DIM> constexpr InsideMasks<DIM> inside_masks() {
  InsideMasks<DIM> t{};
  for (int q = 0; q < Super<DIM>::NB; ++q) t.m[q] = Super<DIM>::inside(q);
  return t;
}

// Launch variants of the apply kernels (chosen by the autotuner).
struct Tune {
  int pad = 1;     // LDS x-line padding of the staged cube (elements)
  int xcd = 1;     // map consecutive supertiles / blocks to one XCD
  int tuned = 0;
};
// variant k: pad = k & 1, order = (k >> 1) & 3 (0 block order, else one
// contiguous range per XCD); the higher bits select nothing any more
constexpr int kTuneVariants = 32;
inline Tune tune_variant(int k) {
  Tune t;
  t.pad = k & 1;
  t.xcd = ((k >> 1) & 3) != 0;
  t.tuned = 1;
  return t;
}

}  // namespace cpm

// The band: everything a call needs, all arrays on the device.
struct cpm_band {
  int dim = 0, N = 0, order = 2, n_ibc = 0, p = 3;
  int band_kind = CPM_BAND_TUBE;
  cpm_surface surf{};
  std::vector<cpm_ibc> ibcs;
  double h = 0, r = 0, tau = 0, check_factor = 2;
  int64_t n_s = 0, n_c = 0, n = 0;
  int device = 0;

  // occupied blocks (block order = Morton order of the block coordinates)
  int nb = 0;
  int4* blk_coord = nullptr;          // [nb] block coordinates
  unsigned long long* blk_mask = nullptr;  // [nb] occupied slots
  int* blk_off = nullptr;             // [nb + 1] first PDE DOF of the block
  int* blk_nbr = nullptr;             // [nb][NNBR] neighbour block ids or -1
  unsigned long long* lrow_mask = nullptr; // [nb] slots whose L row is explicit
  // [nb][8] per-block Laplacian metadata: entry 0 the block itself, 1..2d its
  // face neighbours (-x,+x,-y,+y,-z,+z), 7 the explicit-row mask in .mask
  cpm::QMeta* blk_face = nullptr;

  // hash table block key -> block id (open addressing)
  unsigned long long* hkeys = nullptr;
  int* hvals = nullptr;
  unsigned int hcap = 0;

  // PDE rows
  double* cp = nullptr;               // [dim][n_s] stored cp_S (SoA)

  // tiles: the blocks that hold the stencil base of some PDE row without
  // swapped interpolation members (a tile row)
  int ntiles = 0, n_tile_rows = 0;

  // supertiles: the tile rows whose stencil bases lie in 2 x 2 neighbouring
  // blocks (x and y), two rows of one stencil base to a slot.  Slots are grouped by
  // supertile, in it by tile and base; the rows of a base ascend by DOF, an
  // odd last one is alone in its slot (second DOF -1, fraction repeated)
  int nst = 0;
  int64_t n_slots = 0;
  cpm::QMeta* st_meta = nullptr;      // [nst][18, 2-D: 9] staged blocks
  int4* st_rng = nullptr;             // [nst] first slot, slots, instance, 0
  int2* slot_dof = nullptr;           // [n_slots]
  unsigned short* slot_base = nullptr;   // [n_slots] stencil base from the supertile's
                                      // corner, 4 bits per axis
  double2* slot_frac64 = nullptr;     // [dim][n_slots]
  float2* slot_frac32 = nullptr;      // [dim][n_slots]
  // The transposed gather adds each supertile's rows up in its staged cube
  // and stores the sums of the blocks' nodes one after the other in its part
  // of a buffer.  st_pull: per block of PDE DOFs what it takes from there,
  // [nb][9] {mask, first entry}: up to 2^d supertiles (of the blocks' nodes
  // inside their cubes), then its targets among the explicit rows' (et_tgt).
  cpm::Pull* st_pull = nullptr;
  int* bc_et = nullptr;               // [n_c] explicit E target of a BC DOF, or -1
  cpm::Pull* lt_pull = nullptr;       // [nb] the block's explicit FD targets (lt_tgt)
  int* bc_lt = nullptr;               // [n_c] explicit FD target of a BC DOF, or -1

  // rows with explicit interpolation stencils (swapped PDE rows, BC rows)
  int n_erows = 0;
  int* erow_id = nullptr;             // [padded n_erows], -1 past the last
  int* ecol = nullptr;                // [n_erows][4^dim]
  int* ecol4 = nullptr;               // [padded n_erows][4^dim]: ecol as the apply loads it (ERowPack)
  double* ew1 = nullptr;              // [padded n_erows][dim][4]: 1-D weights, the row's sign with
                                      // the last axis
  int* ebase = nullptr;               // [n_erows][dim]

  // rows with explicit FD stencils (swapped PDE rows, BC rows)
  int n_lrows = 0;
  int* lrow_id = nullptr;             // [n_lrows]
  int* lcol = nullptr;                // [n_lrows][2 dim] after swaps, -1 none
  int* lcol0 = nullptr;               // [n_lrows][2 dim] before swaps (PDE rows)

  // pull lists of the transposed explicit rows (single bands; a batch's
  // composite has none: batches apply only the forward operator): target DOFs, segment
  // starts and sources in ascending order per target.  E: per entry the DOF
  // of its row and its weight (et_src, et_w; sources i * 4^d + o,
  // entry o of explicit E row i, in ascending order).  L: source 2 i + s,
  // explicit FD row i, s = 1 for the subtracted unswapped column of a
  // swapped PDE entry.
  int n_et = 0, n_lt = 0, n_et_entries = 0;
  int *et_tgt = nullptr, *et_start = nullptr, *et_src = nullptr;
  double* et_w = nullptr;
  int *lt_tgt = nullptr, *lt_start = nullptr, *lt_src = nullptr;

  // BC DOFs
  int* bc_node = nullptr;             // [n_c]
  double* bc_cpc = nullptr;           // [n_c][dim]
  int* bc_side = nullptr;             // [n_c]
  int* bc_curve = nullptr;            // [n_c]
  double* bc_ecoef = nullptr;         // [n_c] multiplier of g in the row constant

  // composite of several bands (batched solves): per-instance FD
  // coefficients (cd, co) of A, instance of each explicit FD row
  double* inst_coef = nullptr;
  int* lrow_inst = nullptr;
  int* erow_inst = nullptr;           // instance of each explicit E row
  bool composite = false;

  int64_t on_c_nodes = 0, no_bc_dof_swaps = 0;
  size_t bytes = 0;
  cpm::DevAlloc da;                   // provider of every device allocation
  std::vector<std::pair<void*, size_t>> allocs;
  cpm::Workspace* ws = nullptr;
  cpm::Tune tune[2];                  // per dtype (0 = FP64, 1 = FP32)

  template <class T>
  T* alloc(size_t count) {
    size_t b = count * sizeof(T);
    if (b == 0) b = 16;
    void* p = da.get(b);
    allocs.push_back({p, b});
    bytes += b;
    return static_cast<T*>(p);
  }
  ~cpm_band();
};

namespace cpm {

// Scratch vectors owned by a band, grown on demand through the band's
// allocator (calls on one band from several threads at once race on them).
// A slot that grows is released after the device has finished its work.
struct Workspace {
  const DevAlloc* da = nullptr;
  size_t total = 0;
  std::vector<std::pair<void*, size_t>> slots;
  void* get(int i, size_t bytes);
  ~Workspace();
};
void* band_scratch(const cpm_band* b, int slot, size_t bytes);
size_t band_scratch_bytes(const cpm_band* b);

// Device-wide exclusive scan; returns the total (synchronises the stream).
// Its temporaries come from da.
int64_t scan_exclusive_i32(const int* in, int* out, int64_t n, hipStream_t s, const DevAlloc& da);

// Device flags of systems (right-hand side r, instance i) that a launch leaves
// out: f[(r * stride + i) * elem] != 0; f null leaves none out.
struct Skip {
  const int* f = nullptr;
  int stride = 1, elem = 1;
};

// The Laplacian pass takes kLapBlocksPerWave blocks to a wavefront (one 0.308,
// two 0.270, four 0.296 ms at 34.1M rows), and an explicit FD row to a thread.
// A batch pads an instance's blocks and rows to whole workgroups, so that each
// workgroup has one instance.
constexpr int kLapThreads = 256;
constexpr int kLapBlocksPerWave = 2;
constexpr int kLapBlocksPerGroup = kLapThreads / 64 * kLapBlocksPerWave;

// apply entry points used by the solvers (optional gauge).  With dy set, the
// kernel that writes v also writes the partials of (dy, v) and (v, v) of
// right-hand side r to dpart + 2 r np and np entries further, np =
// apply_dot_parts; those of a system that is skipped are not written.
template <class T>
void apply_impl(const cpm_band* b, double m, double n, int nrhs, const T* u,
                T* v, hipStream_t s, const double* gauge_sum = nullptr,
                double gamma = 0.0, const T* dy = nullptr, double* dpart = nullptr,
                Skip skip = {});
template <class T>
void apply_transpose_impl(const cpm_band* b, double m, double n, int nrhs,
                          const T* w, T* z, hipStream_t s,
                          const double* gauge_sum = nullptr, double gamma = 0.0,
                          const T* dy = nullptr, double* dpart = nullptr, Skip skip = {});
// makes the scratch of apply_transpose_impl (before a graph capture)
void apply_transpose_scratch(const cpm_band* b, int nrhs);
int apply_dot_parts(const cpm_band* b, bool transpose);
// bytes of the forward apply's scratch vector (the FP64 intermediate a = E u)
size_t apply_scratch_bytes(const cpm_band* b, int nrhs);
// out -= n (L - diag L) e(g): the Dirichlet part of a right-hand side
void add_dirichlet_term(const cpm_band* b, double n, const double* g, int nrhs, double* out,
                        hipStream_t st);

// Workgroups that hold n items, one to a thread (at least one workgroup).  A
// launch holds fewer than 2^32 threads.
inline int grid_for(int64_t n, int threads) {
  const int64_t g = n > 0 ? (n + threads - 1) / threads : 1;
  if (g * threads >= (1ll << 32))
    CPM_FAIL(CPM_E_INVALID, "%lld items are too many for a launch", (long long)n);
  return static_cast<int>(g);
}
// The same, at most cap of them, for kernels that go through their items in
// strides of the grid.
inline int grid_for(int64_t n, int threads, int cap) {
  const int64_t g = n > 0 ? (n + threads - 1) / threads : 1;
  return static_cast<int>(g < cap ? g : cap);
}

}  // namespace cpm
