// The CPM operator A = m I + n [diag L + (L - diag L) E] (Sec. 5.4) and its
// transpose, matrix-free, in two passes (the paper's four steps with steps 3
// and 4 folded into the second pass):
//   pass 1  a = E u                                 k_gather (eq. interp-stencil)
//   pass 2  v = (m + n D) u + n N^2 sum_nbr a       k_lap
// Pass 1 interpolates supertile by supertile: the rows whose stencil bases
// lie in 2 x 2 neighbouring blocks read their members from the blocks around
// them, staged in LDS.  Rows whose stencils were changed by an interior
// boundary (and every BC row) are explicit rows with stored columns and
// weights, in the same launch.  Pass 2 maps one wavefront to two blocks of 64
// nodes and finds face neighbours through the block metadata; rows with
// swapped FD neighbours (and BC rows) are explicit, in the same launch.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "cpm_internal.hpp"
#include "lagrange.hpp"

namespace cpm {

struct BlockView {
  const unsigned long long* mask;
  const int* off;
  const int* nbr;
  const unsigned long long* lrow_mask;
  const QMeta* face;
  int nb;
};

static BlockView bview(const cpm_band* b) {
  return BlockView{b->blk_mask, b->blk_off, b->blk_nbr, b->lrow_mask, b->blk_face, b->nb};
}

// Wave-uniform broadcast of lane k (k must be the same in every lane).
__device__ __forceinline__ int lane_i32(int v, int k) { return __builtin_amdgcn_readlane(v, k); }
__device__ __forceinline__ unsigned long long lane_u64(unsigned long long v, int k) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, k);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), k);
  return ((unsigned long long)hi << 32) | lo;
}

// With a wave-uniform mask m (in scalar registers): base + the number of
// bits of m below the lane (masked bit counts, two vector instructions), and
// whether the lane's own bit is set (the mask used as an execution mask).
__device__ __forceinline__ int lane_count_below(unsigned long long m, int base) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((unsigned)m, (unsigned)base));
}
__device__ __forceinline__ bool lane_in(unsigned long long m) {
  return __builtin_amdgcn_inverse_ballot_w64(m);
}
// the lane's DOF in a block of mask m, relative to the block's first; 0 where
// the lane's node is absent (an entry every lane may load)
__device__ __forceinline__ unsigned lane_rank(unsigned long long m) {
  const unsigned d = (unsigned)lane_count_below(m, 0);
  return lane_in(m) ? d : 0u;
}

// Workgroups are dispatched to the 8 XCDs round robin; this bijection on
// [0, g) gives each XCD a contiguous range of work items so that neighbouring
// tiles, which stage the same blocks, share one L2.
__device__ __forceinline__ int xcd_remap(int b, int g) {
  const int q = g >> 3, r = g & 7, x = b & 7, k = b >> 3;
  return x * q + (x < r ? x : r) + k;
}

struct TileView {
  const QMeta* meta;
  const int* tile_blk;
  const int* tile_start;
  const int* perm;
  const double* frac64;
  const float* frac32;
  const unsigned* lbase;
  int ntr;
  int p;                  // interpolation degree: 3, or 2 (fourth weight 0)
};

static TileView tview(const cpm_band* b) {
  return TileView{b->tile_meta, b->tile_blk, b->tile_start, b->perm, b->frac64, b->frac32,
                  b->lbase, b->n_tile_rows, b->p};
}

template <int DIM> struct Cube {
  static constexpr int E = 2 * Geo<DIM>::BX;              // cube edge
  static constexpr int SIZE = DIM == 3 ? E * E * E : E * E;
};

// Per-row stencil base (local to the tile block) and fraction.  The fraction
// is stored in the vector precision TS (FP64 or FP32) and returned in FP64:
// the weights are always evaluated in FP64, so they sum to one to FP64
// rounding whatever precision the fraction was stored in.
template <class TS>
__device__ __forceinline__ const TS* frac_of(const TileView& tv);
template <>
__device__ __forceinline__ const double* frac_of<double>(const TileView& tv) { return tv.frac64; }
template <>
__device__ __forceinline__ const float* frac_of<float>(const TileView& tv) { return tv.frac32; }

template <class TS, int DIM>
__device__ __forceinline__ void row_stencil(const TileView& tv, int pos, int lb[3], double t[3]) {
  const unsigned p = tv.lbase[pos];
  const TS* fr = frac_of<TS>(tv);
  lb[0] = p & 0xff;
  lb[1] = (p >> 8) & 0xff;
  lb[2] = DIM == 3 ? (p >> 16) & 0xff : 0;
#pragma unroll
  for (int a = 0; a < DIM; ++a) t[a] = (double)fr[(int64_t)a * tv.ntr + pos];
  if (DIM == 2) t[2] = 0.0;
}

// ---------------------------------------------------------------- pass 1
__device__ __forceinline__ bool skipped(const Skip& s, int r, int inst) {
  return s.f && s.f[(r * s.stride + inst) * s.elem];
}

// Sum over each aligned group of W lanes (16 or 64) by data-parallel
// primitive moves, in a fixed order: quads, halves of a 16-lane row, rows,
// then the four rows.  The sum is valid in every lane for W = 16 and in lane
// 63 for W = 64.
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp_add(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b & 0xffffffffll), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
  return v + __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <int W>
__device__ __forceinline__ double lanes_sum(double v) {
  v = dpp_add<0xb1>(v);            // quad_perm 1 0 3 2
  v = dpp_add<0x4e>(v);            // quad_perm 2 3 0 1
  v = dpp_add<0x141>(v);           // row_half_mirror
  v = dpp_add<0x140>(v);           // row_mirror
  if (W == 64) {
    v = dpp_add<0x142, 0xa>(v);    // row_bcast 15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);    // row_bcast 31 into rows 2 and 3
  }
  return v;
}

// Explicit interpolation rows: a[id] = sum_o w_o u[col_o], 4^d lanes per row
// (a wavefront in 3-D, a quarter of one in 2-D), lane = member; FP64 weights
// and sums for both storage precisions.
struct ERows {
  int n, groups;          // rows; workgroups that hold them (a multiple of 8)
  const int* id;
  const int* col;
  const double* w;
  const int* inst;        // composite: instance of each row
};
constexpr int kERowPasses = 4;   // row groups per wavefront whose loads go out together
template <int DIM> constexpr int erows_per_group() {
  return kERowPasses * (DIM == 3 ? 1 : 4);
}

template <class TS, int DIM>
__device__ __forceinline__ void explicit_rows(const ERows& er, int wave, int lane,
                                              const TS* __restrict__ u, double* __restrict__ a,
                                              int64_t ld, int nrhs, const Skip& skip) {
  constexpr int M = DIM == 3 ? 64 : 16, RPW = 64 / M;
  if (!er.inst && nrhs == 1 && skipped(skip, 0, 0)) return;
  const int o = lane & (M - 1);
  int row[kERowPasses], c[kERowPasses];
  double w[kERowPasses];
#pragma unroll
  for (int j = 0; j < kERowPasses; ++j) {
    const int i = (wave * kERowPasses + j) * RPW + lane / M;
    row[j] = i < er.n ? i : -1;
    const int64_t e = (int64_t)min(i, er.n - 1) * M + o;
    c[j] = er.col[e];
    w[j] = er.w[e];
  }
  for (int r = 0; r < nrhs; ++r) {
    // every lane loads (an absent member's lane entry 0, which it drops), so
    // that no load waits behind a branch for the one before it
    double v[kERowPasses];
#pragma unroll
    for (int j = 0; j < kERowPasses; ++j) v[j] = (double)u[r * ld + max(c[j], 0)];
#pragma unroll
    for (int j = 0; j < kERowPasses; ++j) v[j] = c[j] >= 0 ? w[j] * v[j] : 0.0;
#pragma unroll
    for (int j = 0; j < kERowPasses; ++j) {
      const double s = lanes_sum<M>(v[j]);
      if (row[j] < 0 || o != M - 1) continue;
      if (skipped(skip, r, er.inst ? er.inst[row[j]] : 0)) continue;
      a[r * ld + er.id[row[j]]] = s;
    }
  }
}

// The tile rows of 2 x 2 neighbouring tiles (x and y) are interpolated
// together.  Their stencils lie in the 3 x 3 x 2 (2-D: 3 x 3) blocks from the
// corner, of which the last node along each axis is beyond every stencil.
template <int DIM> struct Super {
  static constexpr int EX = 3 * Geo<DIM>::BX - 1;              // staged edge, x and y
  static constexpr int EZ = DIM == 3 ? 2 * Geo<3>::BX - 1 : 1; // staged edge, z
  static constexpr int NB = DIM == 3 ? 18 : 9;                 // staged blocks
};
struct SuperView {
  const int2* dof;                // [slots] DOFs of a slot's two rows (second -1: one row)
  const unsigned short* base;     // [slots] their stencil base, 4 bits per axis from the corner
  const double2* frac64;          // [d][slots]
  const float2* frac32;           // [d][slots]
  int64_t ns;
  int n, p;
};

static SuperView sview(const cpm_band* b) {
  return SuperView{b->slot_dof, b->slot_base, b->slot_frac64,
                   b->slot_frac32, b->n_slots, b->nst, b->p};
}

template <class TS> __device__ __forceinline__ double2 frac2_of(const SuperView& sv, int64_t i);
template <> __device__ __forceinline__ double2 frac2_of<double>(const SuperView& sv, int64_t i) {
  return sv.frac64[i];
}
template <> __device__ __forceinline__ double2 frac2_of<float>(const SuperView& sv, int64_t i) {
  const float2 f = sv.frac32[i];
  return make_double2((double)f.x, (double)f.y);
}

// Interpolation of the two rows of a slot from the staged cube (sum-factorised
// tensor product): x lines first, then y, then z; FP64 arithmetic.  NP = p + 1
// stencil nodes per axis.  Both rows read the same members, each once.
template <int DIM, int NP, int E, int EP, class NEXT>
__device__ __forceinline__ void interp_pair(const double* __restrict__ s, const double2 t[DIM],
                                            double out[2], NEXT next) {
  double wx[2][4], wy[2][4], wz[2][4];
  constexpr int P = NP - 1;
  lagrange_p<double>(P, t[0].x, wx[0]);
  lagrange_p<double>(P, t[0].y, wx[1]);
  lagrange_p<double>(P, t[1].x, wy[0]);
  lagrange_p<double>(P, t[1].y, wy[1]);
  const double2 tz = DIM == 3 ? t[DIM - 1] : make_double2(0.0, 0.0);
  // t is free from here on: the caller requests the next slot's data
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int o = 0; o < NP; ++o) asm volatile("" : "+v"(wx[k][o]), "+v"(wy[k][o]));
  next();
  if constexpr (DIM == 3) {
    lagrange_p<double>(P, tz.x, wz[0]);
    lagrange_p<double>(P, tz.y, wz[1]);
  }
  out[0] = out[1] = 0.0;
#pragma unroll
  for (int c = 0; c < (DIM == 3 ? NP : 1); ++c) {
    double acc[2] = {0.0, 0.0};
#pragma unroll
    for (int b = 0; b < NP; ++b) {
      const double* row = s + (c * E + b) * EP;
      const double r0 = row[0], r1 = row[1], r2 = row[2], r3 = NP == 4 ? row[3] : 0.0;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        double x = wx[k][0] * r0 + wx[k][1] * r1 + wx[k][2] * r2;
        if (NP == 4) x += wx[k][3] * r3;
        acc[k] += wy[k][b] * x;
      }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) out[k] = DIM == 3 ? out[k] + wz[k][c] * acc[k] : acc[k];
  }
}

// lanes on the low and high face of the block along each axis (slots with
// local coordinate 0, or BX - 1, along it), evaluated at compile time
template <int DIM>
struct FaceLanes {
  unsigned long long lo[3], hi[3];
};
template <int DIM>
constexpr FaceLanes<DIM> face_lanes() {
  FaceLanes<DIM> f{{0ull, 0ull, 0ull}, {0ull, 0ull, 0ull}};
  constexpr int BX = DIM == 3 ? 4 : 8;
  for (int d = 0; d < DIM; ++d)
    for (int s = 0; s < 64; ++s) {
      const int l = DIM == 3 ? (d == 0 ? s & 3 : d == 1 ? (s >> 2) & 3 : s >> 4)
                             : (d == 0 ? s & 7 : s >> 3);
      if (l == 0) f.lo[d] |= 1ull << s;
      if (l == BX - 1) f.hi[d] |= 1ull << s;
    }
  return f;
}

// Pass 1 in one launch of single wavefronts: the first er.groups take
// explicit rows, the others a supertile each (er.groups is a multiple of 8,
// so both parts keep the XCD of a workgroup id).
//
// What bounds it: with one tile per wavefront and one row per lane every row
// read its 4^d members from LDS by itself, at 128 B a clock and CU, with 71%
// of the lanes filled, and the LDS was busy in 84% of the cycles (0.49 ms for
// the 34.0M tile rows of the torus at h = 1/512, FP64).  A lane that
// interpolates two rows of one stencil base reads the members once for both,
// and the pooled slots of 2 x 2 tiles fill 77% of the lanes: LDS busy 52%.
// The staged blocks' loads, each under a branch of its own, also waited for
// one another; all 18 are now in flight at once.  The kernel then moves
// 2.2 GB at 5.0 TB/s (explicit rows included, 0.48 ms against 0.55 ms), the
// rate of a large copy.  Four such tiles by four wavefronts with a barrier
// (27 blocks) took 0.63 ms and a persistent pipeline over them 0.55 ms:
// wavefronts that wait for one another hold their slots idle.
// Registers, not LDS, set the occupancy (4 or 5 wavefronts per SIMD, which
// time the same); forcing a sixth spills and loses.
template <class TS, int DIM, int PAD, int NP>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) void k_gather(
    ERows er, SuperView sv, const QMeta* __restrict__ meta, const int4* __restrict__ rng,
    const TS* __restrict__ u, double* __restrict__ a, int64_t ld, int nrhs, int xcd, Skip skip) {
  using G = Geo<DIM>;
  using SP = Super<DIM>;
  constexpr int EX = SP::EX, EP = EX + PAD, BX = G::BX, NB = SP::NB;
  constexpr FaceLanes<DIM> FL = face_lanes<DIM>();
  constexpr int CS = SP::EZ * EX * EP;
  __shared__ double s_u[CS + 1];
  const int lane = threadIdx.x;
  int g = blockIdx.x;
  if (g < er.groups) {
    if (xcd) g = xcd_remap(g, er.groups);
    explicit_rows<TS, DIM>(er, g, lane, u, a, ld, nrhs, skip);
    return;
  }
  g -= er.groups;
  if (xcd) g = xcd_remap(g, sv.n);
  const int4 rg = rng[g];
  // the staged blocks' masks and first DOFs: block q's in lane q
  const int4 qm = reinterpret_cast<const int4*>(meta)[(int64_t)g * NB + min(lane, NB - 1)];
  auto qmask = [&](int q) {
    return ((unsigned long long)(unsigned)lane_i32(qm.y, q) << 32) | (unsigned)lane_i32(qm.x, q);
  };
  // row data of slot k (the last slot's past the end: loads under no branch)
  int2 dof;
  int code;
  double2 t[DIM];
  auto rows = [&](int k) {
    const int64_t i = (int64_t)rg.x + min(k, rg.y - 1);
    dof = sv.dof[i];
    code = sv.base[i];
#pragma unroll
    for (int d = 0; d < DIM; ++d) t[d] = frac2_of<TS>(sv, d * sv.ns + i);
  };
  int cell0 = DIM == 3 ? (G::lz(lane) * EX + G::ly(lane)) * EP + G::lx(lane)
                       : G::ly(lane) * EP + G::lx(lane);
  for (int r = 0; r < nrhs; ++r) {
    // keeps the cells of all staged blocks from living in registers throughout
    asm volatile("" : "+v"(cell0));
    if (skipped(skip, r, rg.z)) continue;
    // the first pass's row data is requested before the staging loads
    rows(lane);
    __syncthreads();   // the previous right-hand side's rows are done
    // Every lane loads (an absent node's lane the block's first value, which
    // it drops): under a condition each load would be a basic block of its
    // own and wait for the one before it.
    // Cells of absent nodes hold that value: no tile row's stencil has one.
    const TS* ur = u + r * ld;
    TS x[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) x[q] = ur[lane_i32(qm.z, q) + (int64_t)lane_rank(qmask(q))];
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const int qx = q % 3, qy = (q / 3) % 3, qz = q / 9;
      unsigned long long in = ~0ull;
      if (qx == 2) in &= ~FL.hi[0];
      if (qy == 2) in &= ~FL.hi[1];
      if (DIM == 3 && qz == 1) in &= ~FL.hi[DIM - 1];
      const int off = (DIM == 3 ? (qz * BX * EX + qy * BX) * EP : qy * BX * EP) + qx * BX;
      s_u[in == ~0ull || lane_in(in) ? cell0 + off : CS] = (double)x[q];
    }
    __syncthreads();
    for (int k = lane; k - lane < rg.y; k += 64) {
      const int2 dc = dof;
      const int bc = ((DIM == 3 ? (code >> 8) * EX : 0) + ((code >> 4) & 15)) * EP + (code & 15);
      double v[2];
      interp_pair<DIM, NP, EX, EP>(s_u + bc, t, v, [&] { rows(k + 64); });
      // keeps the sums out of the branches below (the compiler would sink
      // them there and hold every member in a register for them)
      asm volatile("" : "+v"(v[0]), "+v"(v[1]));
      if (k < rg.y) {
        a[r * ld + dc.x] = v[0];
        if (dc.y >= 0) a[r * ld + dc.y] = v[1];
      }
    }
  }
}

template <class T>
__device__ __forceinline__ T wave_sum(T v, int width) {
  for (int o = width >> 1; o > 0; o >>= 1) v += __shfl_xor(v, o, width);
  return v;
}

// Workgroup sums of d0 and d1 (256 threads, every one must call it), written
// to part[idx] and part[np + idx]: the partials of a fused dot product, one
// per workgroup, finished in a fixed order by the solver.
__device__ __forceinline__ void group_dot2(double d0, double d1, double* part, int np, int idx) {
  __shared__ double sh[4][2];
  d0 = lanes_sum<64>(d0);
  d1 = lanes_sum<64>(d1);
  if ((threadIdx.x & 63) == 63) {
    sh[threadIdx.x >> 6][0] = d0;
    sh[threadIdx.x >> 6][1] = d1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    part[idx] = ((sh[0][0] + sh[1][0]) + sh[2][0]) + sh[3][0];
    part[np + idx] = ((sh[0][1] + sh[1][1]) + sh[2][1]) + sh[3][1];
  }
}

// ---------------------------------------------------------------- pass 2
// cd u + co s with one explicit rounding order, whatever the compiler
// contracts.
__device__ __forceinline__ double lap_out(double cd, double u, double co, double s) {
  return __fma_rn(co, s, cd * u);
}

// v = cd u + co sum_nbr a (+ gauge); lane = slot of a block, two blocks per
// wavefront.  A form with per-lane mask arithmetic is bound by vector issue
// (about 250 vector instructions per block, almost all of them integer work
// on 64-bit masks), so the index arithmetic is kept off the vector unit:
//   * the block's metadata (its own and its face neighbours' masks and first
//     DOFs, the explicit-row mask) is read with scalar loads: every mask is
//     wave-uniform and stays in scalar registers;
//   * lane sets (present slots, output rows, the lanes on a face whose
//     neighbour across it is present) are built with scalar mask arithmetic
//     and applied as execution masks (inverse ballot);
//   * a DOF is first DOF + the count of mask bits below the lane (two
//     masked-bit-count instructions), for the neighbour across a face on the
//     mask shifted by the face's slot offset;
//   * in-block neighbours' values come from other lanes: data-parallel
//     primitive moves inside 16-lane rows (x, and y in 3-D), lane permutes
//     across rows (z in 3-D, y in 2-D).
// ALL = false skips rows with explicit FD stencils and reads u for the
// diagonal term; ALL = true (transpose) visits every PDE row and writes
// co sum_nbr a only.  TU, TA, TV are the storage types of u, a and v; the
// arithmetic is FP64.
template <class T>
__device__ __forceinline__ T lane_perm(T v, int addr) {
  if constexpr (sizeof(T) == 8) {
    const long long b = __double_as_longlong((double)v);
    const int lo = __builtin_amdgcn_ds_bpermute(addr, (int)(unsigned)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_ds_bpermute(addr, (int)(b >> 32));
    return (T)__longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  } else {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(addr, __float_as_int((float)v)));
  }
}
// value of lane (lane - k) (SHR) or (lane + k) (SHL) within a 16-lane row;
// lanes whose source lies outside their row get an unspecified value
template <class T, int CTRL>
__device__ __forceinline__ T lane_dpp(T v) {
  if constexpr (sizeof(T) == 8) {
    const long long b = __double_as_longlong((double)v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)(b & 0xffffffffll), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, false);
    return (T)__longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  } else {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int((float)v), CTRL, 0xf, 0xf, false));
  }
}
template <int K> constexpr int dpp_shr() { return 0x110 + K; }   // from lane - K
template <int K> constexpr int dpp_shl() { return 0x100 + K; }   // from lane + K


// Explicit FD rows (swapped PDE rows and BC rows), one thread each.
struct LRows {
  int n, groups;          // rows; workgroups that hold them
  int nf;
  const int* id;          // row DOF (-1: padding of a composite)
  const int* col;
  const int* inst;        // composite: instance of each row
};

// Fused dot products of the pass: with y set, the partials of (y, v) and
// (v, v) of right-hand side r go to part + 2 r np, one per workgroup.
template <class TV>
struct DotOut {
  const TV* y;
  double* part;
  int np;
};

// two blocks per wavefront: one 0.308, two 0.270, four 0.296 ms at 34.1M rows
constexpr int kLapBlocksPerWave = 2;
constexpr int kLapBlocksPerGroup = 4 * kLapBlocksPerWave;

// The first lr.groups workgroups take explicit rows, the others blocks.
template <class TU, class TA, class TV, int DIM, bool ALL, bool DOT = false>
__global__ __launch_bounds__(256) void k_lap(
    LRows lr, const QMeta* __restrict__ face, int nb, const TU* __restrict__ u,
    const TA* __restrict__ a, TV* __restrict__ v, int64_t ld, int nrhs, double cd, double co,
    const double* __restrict__ gsum, double gscale, int xcd, const double* __restrict__ coef,
    Skip skip, DotOut<TV> dot) {
  using G = Geo<DIM>;
  constexpr int BX = G::BX, KB = kLapBlocksPerWave;
  constexpr int step[3] = {1, BX, BX * BX};
  constexpr FaceLanes<DIM> FL = face_lanes<DIM>();
  if (!ALL && (int)blockIdx.x < lr.groups) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int id = i < lr.n ? lr.id[i] : -1;
    const int inst = coef && id >= 0 ? lr.inst[i] : 0;
    if (coef && id >= 0) {
      cd = coef[2 * inst];
      co = coef[2 * inst + 1];
    }
    int c[2 * DIM];
#pragma unroll
    for (int f = 0; f < 2 * DIM; ++f) c[f] = id >= 0 ? lr.col[(int64_t)i * lr.nf + f] : -1;
    for (int r = 0; r < nrhs; ++r) {
      double d0 = 0.0, d1 = 0.0;
      if (id >= 0 && !skipped(skip, r, inst)) {
        double s = 0.0;
#pragma unroll
        for (int f = 0; f < 2 * DIM; ++f)
          if (c[f] >= 0) s += (double)a[r * ld + c[f]];
        double out = lap_out(cd, (double)u[r * ld + id], co, s);
        if (gsum) out += gscale * gsum[r];
        const TV ov = (TV)out;
        v[r * ld + id] = ov;
        if (DOT) {
          d0 = (double)dot.y[r * ld + id] * (double)ov;
          d1 = (double)ov * (double)ov;
        }
      }
      if constexpr (DOT) {
        if (r > 0) __syncthreads();
        group_dot2(d0, d1, dot.part + (int64_t)2 * r * dot.np, dot.np, blockIdx.x);
      }
    }
    return;
  }
  const int ng = gridDim.x - lr.groups, gb = blockIdx.x - lr.groups;
  const int wg = xcd ? xcd_remap(gb, ng) : gb;
  const int blk0 = (wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * KB;
  const int lane = threadIdx.x & 63;
  if (!DOT && blk0 >= nb) return;
  // per block j of the wave: coefficients, lane sets, DOFs (all but the DOFs
  // wave-uniform).  A wave past the last block repeats it without output.
  double cdi[KB], coi[KB];
  unsigned long long present[KB], outm[KB], xload[KB][DIM];
  int own[KB], xdof[KB][DIM], inst = 0;
  // entry e of block j's metadata in lane 8 j + e: one load, no chain of
  // scalar ones
  const int4 fm = reinterpret_cast<const int4*>(
      face)[(int64_t)min(blk0 + min(lane >> 3, KB - 1), nb - 1) * 8 + (lane & 7)];
  auto fmask = [&](int j, int e) {
    return ((unsigned long long)(unsigned)lane_i32(fm.y, 8 * j + e) << 32) |
           (unsigned)lane_i32(fm.x, 8 * j + e);
  };
  auto foff = [&](int j, int e) { return lane_i32(fm.z, 8 * j + e); };
#pragma unroll
  for (int j = 0; j < KB; ++j) {
    const bool live = blk0 + j < nb;
    cdi[j] = cd;
    coi[j] = co;
    const unsigned long long m = fmask(j, 0);
    if (coef) {
      // blocks of one workgroup belong to one instance (build_composite)
      inst = max(lane_i32(fm.w, 8 * j + 7), 0);
      cdi[j] = coef[2 * inst];
      coi[j] = coef[2 * inst + 1];
    }
    present[j] = m;
    outm[j] = live ? (ALL ? m : (m & ~fmask(j, 7))) : 0ull;
    own[j] = foff(j, 0) + (int)lane_rank(m);
    // per axis: the DOF of the neighbour across the face the lane lies on,
    // and the lanes that have one (on that face, neighbour present, output row)
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const int K = (BX - 1) * step[d];
      const unsigned long long mlo = fmask(j, 2 * d + 1), mhi = fmask(j, 2 * d + 2);
      // low face: neighbour slot lane + K; high face: lane - K
      const unsigned long long slo = mlo >> K, shi = mhi << K;
      const int blo = foff(j, 2 * d + 1) + __popcll(mlo & ((1ull << K) - 1ull));
      const int dlo = lane_count_below(slo, blo), dhi = lane_count_below(shi, foff(j, 2 * d + 2));
      xload[j][d] = ((FL.lo[d] & slo) | (FL.hi[d] & shi)) & outm[j];
      const int dx = lane_in(FL.lo[d]) ? dlo : dhi;
      xdof[j][d] = lane_in(xload[j][d]) ? dx : own[j];
    }
  }
  const int zl = ((lane + step[DIM - 1]) & 63) << 2, zh = ((lane - step[DIM - 1]) & 63) << 2;
  for (int r = 0; r < nrhs; ++r) {
    if (skipped(skip, r, inst)) continue;
    // Every load of the wave's blocks first, then the exchanges and sums.
    // Every lane loads (its own or, absent, its block's first value where it
    // has no neighbour across a face) and drops what it has no use for: under
    // a condition each load would be a basic block of its own and wait for
    // the one before it.
    const TA* ar = a + r * ld;
    TA al[KB], xl[KB][DIM];
    TU ul[KB];
    TV yl[KB];
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      al[j] = ar[own[j]];
      if (!ALL) ul[j] = u[r * ld + own[j]];
      if (DOT) yl[j] = dot.y[r * ld + own[j]];
#pragma unroll
      for (int d = 0; d < DIM; ++d) xl[j][d] = ar[xdof[j][d]];
    }
    TA aown[KB];
    double uv[KB], yv[KB], across[KB][DIM];
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      asm volatile("" : "+v"(al[j]));   // the loads stay above, whoever uses them
      aown[j] = lane_in(present[j]) ? al[j] : TA(0);
      uv[j] = ALL ? 0.0 : (double)ul[j];
      yv[j] = DOT ? (double)yl[j] : 0.0;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        asm volatile("" : "+v"(xl[j][d]));
        across[j][d] = lane_in(xload[j][d]) ? (double)xl[j][d] : 0.0;
      }
      if (!ALL) asm volatile("" : "+v"(uv[j]));
      if (DOT) asm volatile("" : "+v"(yv[j]));
    }
    double d0 = 0.0, d1 = 0.0;
#pragma unroll
    for (int j = 0; j < KB; ++j) {
      // in-block neighbours: low (-) and high (+) along each axis
      double lo[DIM], hi[DIM];
      lo[0] = (double)lane_dpp<TA, dpp_shr<1>()>(aown[j]);
      hi[0] = (double)lane_dpp<TA, dpp_shl<1>()>(aown[j]);
      if constexpr (DIM == 3) {
        lo[1] = (double)lane_dpp<TA, dpp_shr<4>()>(aown[j]);
        hi[1] = (double)lane_dpp<TA, dpp_shl<4>()>(aown[j]);
      }
      lo[DIM - 1] = (double)lane_perm<TA>(aown[j], zh);
      hi[DIM - 1] = (double)lane_perm<TA>(aown[j], zl);
      double sum = 0.0;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        sum += lane_in(FL.lo[d]) ? across[j][d] : lo[d];
        sum += lane_in(FL.hi[d]) ? across[j][d] : hi[d];
      }
      if (lane_in(outm[j])) {
        double o = ALL ? coi[j] * sum : lap_out(cdi[j], uv[j], coi[j], sum);
        if (gsum) o += gscale * gsum[r];
        const TV ov = (TV)o;
        v[r * ld + own[j]] = ov;
        if (DOT) {
          d0 += yv[j] * (double)ov;
          d1 += (double)ov * (double)ov;
        }
      }
    }
    if constexpr (DOT) {
      if (r > 0) __syncthreads();
      group_dot2(d0, d1, dot.part + (int64_t)2 * r * dot.np, dot.np, lr.groups + wg);
    }
  }
}

// ---------------------------------------------------------------- gauge
// gsum[r] = sum_{i < n_s} u[r][i] (deterministic two-stage sum)
template <class T>
__global__ __launch_bounds__(256) void k_sum_part(const T* __restrict__ u, int64_t n_s, int64_t ld,
                                                  double* part) {
  __shared__ double s[256];
  const int r = blockIdx.y;
  double acc = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n_s; i += (int64_t)gridDim.x * 256)
    acc += (double)u[r * ld + i];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[r * gridDim.x + blockIdx.x] = s[0];
}

__global__ void k_sum_final(const double* part, int np, double* out) {
  __shared__ double s[256];
  const int r = blockIdx.x;
  double acc = 0.0;
  for (int i = threadIdx.x; i < np; i += 256) acc += part[r * np + i];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[r] = s[0];
}

// ---------------------------------------------------------------- transpose
// E^T c for the tile rows of one parity class, one wavefront per tile.  The
// wave takes its tile and row range from one entry of the class table, so the
// tile's metadata and first row data are requested together, one load after
// it.  Rows go in chunks of kTRows: each lane of a chunk puts the stencil
// base of one row into LDS with the row's 1-D weights (the forward gather's
// FP64 weights), c_i folded into the last factor; then the wave walks the
// chunk's rows with one lane per stencil member (4 rows at a time in 2-D,
// where a stencil has 16 members), adding w c_i into the tile's (2 BX)^d cube
// in LDS.  A 3-D member's weight is the product of three 1-D weights read
// from LDS, and each lane sums over runs of rows with the same stencil base;
// 2-D uses LDS atomic adds (rows past the last one carry zero weights).  The
// cube is accumulated in FP64 for both precisions.  It is then added into z
// with plain loads and stores: tiles of one parity class stage disjoint
// blocks and the classes run as successive launches, so no two waves of a
// launch touch the same entry of z.  Chunks of 32 rows keep the LDS of a wave
// at 7.9 KB (20 waves per CU) where whole 64-row passes took 11.1 KB (14).
constexpr int kTRows = 32;
constexpr int kTGroup = 4;
template <class TS, int DIM>
__global__ __launch_bounds__(64) void k_gather_T(BlockView B, TileView tv, const int4* __restrict__ tbl,
                                                 int N, const double* __restrict__ c,
                                                 double* __restrict__ z, int64_t ld, int r,
                                                 int xcd) {
  using G = Geo<DIM>;
  constexpr int E = Cube<DIM>::E, EP = E + 1, NQ = 1 << DIM;
  constexpr int CS = DIM == 3 ? E * E * EP : E * EP;
  constexpr int M = DIM == 3 ? 64 : 16;       // stencil members
  constexpr int RPI = 64 / M;                 // rows per wave instruction
  constexpr int NW = DIM == 3 ? 12 : 8;       // 1-D weights per row
  constexpr int RC = kTRows;
  constexpr int RG = kTGroup;                 // rows whose LDS reads go out together
  static_assert(RC % 16 == 0 && RC <= 64 && RC % RG == 0, "chunk rows: a multiple of 16 and RG");
  __shared__ double s_z[CS];
  // per-row 1-D weights, component major; rows padded to RC + 1 entries so
  // that the four values of one component a wave reads for a row lie in
  // distinct LDS banks
  __shared__ double s_w[NW][RC + 1];
  __shared__ int s_b[RC];                     // per-row cube offset of member 0
  const int4 te = tbl[xcd ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x];
  const int t = te.x, beg = te.y, end = te.z;
  if (beg == end) return;
  const int lane = threadIdx.x;
  unsigned long long qm = 0ull;
  int qoff = 0;
  if (lane < NQ) {
    const QMeta q = tv.meta[(int64_t)t * 8 + lane];
    qm = q.mask;
    qoff = q.off;
  }
  // entry of z (or -1) of this lane's node in staged block q, and its cube cell
  const int cx0 = G::lx(lane), cy0 = G::ly(lane), cz0 = G::lz(lane);
  auto zidx = [&](int q) {
    const unsigned long long m = lane_u64(qm, q);
    const int off = lane_i32(qoff, q);
    return ((m >> lane) & 1ull) ? off + __popcll(m & ((1ull << lane) - 1ull)) : -1;
  };
  auto cell = [&](int q) {
    const int qx = q & 1, qy = (q >> 1) & 1, qz = DIM == 3 ? (q >> 2) : 0;
    const int cx = qx * G::BX + cx0, cy = qy * G::BX + cy0, cz = qz * G::BX + cz0;
    return DIM == 3 ? (cz * E + cy) * EP + cx : cy * EP + cx;
  };
  // the old entries of z under the staged blocks, requested now so that the
  // loads overlap the row work (no other wave of this launch touches them);
  // the cube starts at zero and is added to them at the end
  double old[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int zi = zidx(q);
    old[q] = zi >= 0 ? z[r * ld + zi] : 0.0;
  }
  for (int idx = lane; idx < CS; idx += 64) s_z[idx] = 0.0;
  // this lane's stencil member and row slot within an instruction
  const int mo = lane & (M - 1), sub = lane / M;
  const int ma = mo & 3, mb = (mo >> 2) & 3, mc = DIM == 3 ? (mo >> 4) : 0;
  const int moff = DIM == 3 ? (mc * E + mb) * EP + ma : mb * EP + ma;
  // Row data of a chunk (lane < RC: row p0 + lane): local base, fraction
  // and c.  The next chunk's is requested before the current chunk's rows
  // are walked, and the DOFs (which c is read through) one chunk further
  // ahead, so only the first chunk waits for its loads.
  int lbn[3] = {0, 0, 0}, pmn = 0;
  double ttn[3] = {0.0, 0.0, 0.0}, cn = 0.0;
  if (lane < RC && beg + lane < end) {
    row_stencil<TS, DIM>(tv, beg + lane, lbn, ttn);
    cn = c[r * ld + tv.perm[beg + lane]];
  }
  if (lane < RC && beg + RC + lane < end) pmn = tv.perm[beg + RC + lane];
  for (int p0 = beg; p0 < end; p0 += RC) {
    const int nrow = min(RC, end - p0);
    const int lb[3] = {lbn[0], lbn[1], lbn[2]};
    const double tt[3] = {ttn[0], ttn[1], ttn[2]}, ci = cn;
    const int p1 = p0 + RC;
    if (lane < RC && p1 + lane < end) {
      row_stencil<TS, DIM>(tv, p1 + lane, lbn, ttn);
      cn = c[r * ld + pmn];
    }
    if (lane < RC && p1 + RC + lane < end) pmn = tv.perm[p1 + RC + lane];
    double wx[4] = {0.0, 0.0, 0.0, 0.0}, wy[4] = {0.0, 0.0, 0.0, 0.0};
    double wz[4] = {0.0, 0.0, 0.0, 0.0};
    int bs = 0;
    if (lane < nrow) {
      lagrange_p<double>(tv.p, tt[0], wx);
      lagrange_p<double>(tv.p, tt[1], wy);
      if (DIM == 3) {
        lagrange_p<double>(tv.p, tt[2], wz);
#pragma unroll
        for (int k = 0; k < 4; ++k) wz[k] *= ci;
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) wy[k] *= ci;
      }
      bs = DIM == 3 ? (lb[2] * E + lb[1]) * EP + lb[0] : lb[1] * EP + lb[0];
    }
    if (lane < RC) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        s_w[k][lane] = wx[k];
        s_w[4 + k][lane] = wy[k];
        if constexpr (DIM == 3) s_w[8 + k][lane] = wz[k];
      }
      s_b[lane] = bs;
    }
    __syncthreads();
    if constexpr (DIM == 3) {
      // Rows are sorted by stencil base, and runs of rows share one: each
      // lane sums its member's contributions in a register while the base
      // stays the same and adds the sum into the cube when it changes.  A
      // row's 64 members are distinct cells, and a wave's LDS operations
      // complete in order, so these read-add-writes need no atomics.
      double acc = 0.0;
      int cur = __builtin_amdgcn_readfirstlane(s_b[0]);
      for (int j = 0; j < nrow; j += RG) {
        // RG rows' bases and weights read at once (indices stay below RC)
        int bq[RG];
        double wq[RG];
#pragma unroll
        for (int u = 0; u < RG; ++u) {
          bq[u] = __builtin_amdgcn_readfirstlane(s_b[j + u]);
          wq[u] = (s_w[ma][j + u] * s_w[4 + mb][j + u]) * s_w[8 + mc][j + u];
        }
#pragma unroll
        for (int u = 0; u < RG; ++u) {
          if (j + u >= nrow) break;
          if (bq[u] != cur) {
            s_z[cur + moff] += acc;
            acc = 0.0;
            cur = bq[u];
          }
          acc += wq[u];
        }
      }
      s_z[cur + moff] += acc;
    } else {
      constexpr int UR = 4;                   // rows per lane per step
      const int nr = (nrow + UR * RPI - 1) / (UR * RPI) * (UR * RPI);
      for (int j0 = 0; j0 < nr; j0 += UR * RPI) {
        double v[UR];
        int o[UR];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
          const int j = j0 + u * RPI + sub;
          v[u] = s_w[ma][j] * s_w[4 + mb][j];
          o[u] = s_b[j] + moff;
        }
#pragma unroll
        for (int u = 0; u < UR; ++u) atomicAdd(&s_z[o[u]], v[u]);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int zi = zidx(q);
    if (zi >= 0) z[r * ld + zi] = old[q] + s_z[cell(q)];
  }
}

// E^T c over the explicit rows by pull lists: one wavefront per target DOF
// (four per workgroup).  The lanes take the target's contiguous segment of
// entries 64 at a time (entry e: weight w[e] of source row src[e], FP64 for
// both precisions), sum the products w c_src in their own order and the wave
// adds the tree sum of its lanes into z once: the same value on every run,
// with no atomics.
__global__ __launch_bounds__(256) void k_et_pull(int n_tgt, const int* __restrict__ tgt,
                                                 const int* __restrict__ start,
                                                 const int* __restrict__ src,
                                                 const double* __restrict__ w,
                                                 const double* __restrict__ c,
                                                 double* __restrict__ z) {
  const int k = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (k >= n_tgt) return;                     // whole waves leave together
  const int lane = threadIdx.x & 63;
  const int b0 = start[k], b1 = start[k + 1];
  double acc = 0.0;
  for (int e = b0 + lane; e < b1; e += 64) acc += w[e] * c[src[e]];
  acc = wave_sum(acc, 64);
  if (lane == 0) z[tgt[k]] += acc;
}

// The corrections of (L - diag L)^T w for explicit FD rows by pull lists:
// c[t] += co (sum of +w_i over rows adding to t, -w_i over swapped rows
// moving their entry away from t), in ascending source order.
template <class TS>
__global__ void k_lt_pull(int n_tgt, const int* __restrict__ tgt, const int* __restrict__ start,
                          const int* __restrict__ src, const int* __restrict__ row_id,
                          const TS* __restrict__ w, double* __restrict__ c, int64_t ld, int nrhs,
                          double co) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_tgt) return;
  const int t = tgt[k], b0 = start[k], b1 = start[k + 1];
  for (int r = 0; r < nrhs; ++r) {
    double acc = 0.0;
    for (int e = b0; e < b1; ++e) {
      const int v = src[e];
      const double wi = co * (double)w[r * ld + row_id[v >> 1]];
      acc += (v & 1) ? -wi : wi;
    }
    c[r * ld + t] += acc;
  }
}

template <class T>
__global__ void k_fill(T* __restrict__ p, int64_t n, T val) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = val;
}

// out = cd w + nn e (FP64 arithmetic, stored in the vector precision TS);
// with DOT also the partials of (dy, out) and (out, out)
template <class TS, bool DOT = false>
__global__ void k_combine(const TS* __restrict__ w, const double* __restrict__ z,
                          TS* __restrict__ out, double cd, double nn, int64_t total,
                          const TS* __restrict__ dy = nullptr, double* __restrict__ dpart = nullptr,
                          int dnp = 0) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double d0 = 0.0, d1 = 0.0;
  if (i < total) {
    const TS o = (TS)(cd * (double)w[i] + nn * z[i]);
    out[i] = o;
    if (DOT) {
      d0 = (double)dy[i] * (double)o;
      d1 = (double)o * (double)o;
    }
  }
  if constexpr (DOT) group_dot2(d0, d1, dpart, dnp, blockIdx.x);
}

// ---------------------------------------------------------------- rhs
__global__ void k_rhs_init(int64_t n_s, int64_t n_c, int nrhs, const double* __restrict__ f,
                           const int* __restrict__ bc_node, double* __restrict__ b) {
  const int64_t n = n_s + n_c;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n * nrhs) return;
  const int64_t r = t / n, i = t % n;
  b[t] = i < n_s ? f[r * n_s + i] : f[r * n_s + bc_node[i - n_s]];
}

__global__ void k_rhs_rows(int nrows, int nf, int64_t n_s, int64_t n_c, int nrhs,
                           const int* __restrict__ row_id, const int* __restrict__ col,
                           const double* __restrict__ g, const double* __restrict__ ecoef,
                           double scale, double* __restrict__ b) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nrows) return;
  const int id = row_id[i];
  const int64_t n = n_s + n_c;
  for (int r = 0; r < nrhs; ++r) {
    double s = 0.0;
    for (int f = 0; f < nf; ++f) {
      const int c = col[i * nf + f];
      if (c >= n_s) s += ecoef[c - n_s] * g[r * n_c + (c - n_s)];
    }
    b[r * n + id] -= scale * s;
  }
}

__global__ void k_gradf(int64_t n_s, int64_t n_c, int nrhs, const double* __restrict__ lam,
                        double* __restrict__ gf) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_s * nrhs) return;
  const int64_t r = t / n_s, i = t % n_s;
  gf[t] = lam[r * (n_s + n_c) + i];
}

__global__ void k_gradf_bc(int64_t n_s, int64_t n_c, int nrhs, const int* __restrict__ bc_node,
                           const double* __restrict__ lam, double* __restrict__ gf) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_c * nrhs) return;
  const int64_t r = t / n_c, k = t % n_c;
  gf[r * n_s + bc_node[k]] += lam[r * (n_s + n_c) + n_s + k];
}

__global__ void k_gradg(int nrows, int nf, int64_t n_s, int64_t n_c, int nrhs,
                        const int* __restrict__ row_id, const int* __restrict__ col,
                        const double* __restrict__ lam, const double* __restrict__ ecoef,
                        double scale, double* __restrict__ gg) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nrows) return;
  const int id = row_id[i];
  const int64_t n = n_s + n_c;
  for (int r = 0; r < nrhs; ++r) {
    const double li = lam[r * n + id];
    for (int f = 0; f < nf; ++f) {
      const int c = col[i * nf + f];
      if (c >= n_s && ecoef[c - n_s] != 0.0)
        atomicAdd(&gg[r * n_c + (c - n_s)], scale * ecoef[c - n_s] * li);
    }
  }
}

// ================================================================ host
template <class T>
static const Tune& tune_of(const cpm_band* b) {
  return b->tune[sizeof(T) == 8 ? 0 : 1];
}

// What of a pass a launch does: all of it, or (measurement only) one part.
enum { PART_ALL = 0, PART_MAIN = 1, PART_EXPLICIT = 2 };

// a = E u for nrhs right-hand sides, in one launch.
template <class T, int DIM>
static void launch_gather(const cpm_band* b, int nrhs, const T* u, double* a, hipStream_t st,
                          int part, const Skip& skip) {
  const Tune& tn = tune_of<T>(b);
  constexpr int RG = erows_per_group<DIM>();
  ERows er{b->n_erows, (int)(((int64_t)b->n_erows + 8 * RG - 1) / (8 * RG)) * 8, b->erow_id,
           b->ecol, b->ew, b->erow_inst};
  SuperView sv = sview(b);
  if (part == PART_MAIN) er.groups = 0;
  if (part == PART_EXPLICIT) sv.n = 0;
  const int64_t g = (int64_t)er.groups + sv.n;
  if (!g) return;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)g), dim3(64), 0, st, er, sv, b->st_meta, b->st_rng, u, a, b->n, nrhs, tn.xcd,
                       skip);
  };
  auto multi = [&](auto pad, auto np) { go(k_gather<T, DIM, pad(), np()>); };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using N3 = std::integral_constant<int, 3>;
  using N4 = std::integral_constant<int, 4>;
  if (b->p == 2) {
      if (tn.pad) multi(I1{}, N3{});
    else multi(I0{}, N3{});
  } else {
    if (tn.pad) multi(I1{}, N4{});
    else multi(I0{}, N4{});
  }
  CPM_LAUNCH_CHECK();
}

// Workgroups of the Laplacian pass over the blocks and over explicit rows.
static int lap_groups(const cpm_band* b) {
  return (b->nb + kLapBlocksPerGroup - 1) / kLapBlocksPerGroup;
}
static int lap_row_groups(const cpm_band* b) { return (b->n_lrows + 255) / 256; }

// Number of partials a fused dot product of an apply writes (per value): one
// per workgroup of the kernel that writes the result.
int apply_dot_parts(const cpm_band* b, bool transpose) {
  if (transpose) return grid_for(b->n, 256);
  return lap_row_groups(b) + lap_groups(b);
}

template <class TU, class TA, class TV, int DIM, bool ALL, bool DOT>
static void launch_lap(const cpm_band* b, const Tune& tn, hipStream_t st, const TU* u,
                       const TA* a, TV* v, int64_t ld, int nrhs, double cd, double co,
                       const double* gsum, double gscale, const double* coef, DotOut<TV> dot,
                       int part, const Skip& skip) {
  LRows lr{b->n_lrows, ALL || part == PART_MAIN ? 0 : lap_row_groups(b), 2 * DIM, b->lrow_id,
           b->lcol, b->lrow_inst};
  const int64_t g = (int64_t)lr.groups + (part == PART_EXPLICIT ? 0 : lap_groups(b));
  if (!g) return;
  hipLaunchKernelGGL((k_lap<TU, TA, TV, DIM, ALL, DOT>), dim3((unsigned)g), dim3(256), 0, st, lr,
                     b->blk_face, b->nb, u, a, v, ld, nrhs, cd, co, gsum, gscale, tn.xcd, coef,
                     skip, dot);
  CPM_LAUNCH_CHECK();
}

// Bytes of scratch one forward apply of nrhs right-hand sides needs: the
// intermediate a = E u, FP64 for both vector precisions.
size_t apply_scratch_bytes(const cpm_band* b, int nrhs) {
  return sizeof(double) * (size_t)b->n * (size_t)nrhs;
}

// The two passes of the forward apply with a given scratch vector a (at
// least apply_scratch_bytes).  ev (measurement, optional): five events; each
// pass's explicit rows then run in a launch of their own, with the events
// between the four phases.
template <class T, int DIM>
static void apply_dim(const cpm_band* b, double m, double n, int nrhs, const T* u, T* v,
                      hipStream_t st, const double* gsum, double gamma, double* a,
                      hipEvent_t* ev = nullptr, const T* dy = nullptr, double* dpart = nullptr,
                      const Skip& skip = {}) {
  const int64_t ld = b->n;
  const double N2 = (double)b->N * (double)b->N;
  const double cd = m + n * (-2.0 * DIM * N2);
  const double co = n * N2;
  const double gscale = gsum ? gamma / (double)b->n_s : 0.0;
  const Tune& tn = tune_of<T>(b);
  auto gather = [&](int part) { launch_gather<T, DIM>(b, nrhs, u, a, st, part, skip); };
  auto lap = [&](int part) {
    if (dy)
      launch_lap<T, double, T, DIM, false, true>(
          b, tn, st, u, a, v, ld, nrhs, cd, co, gsum, gscale, b->inst_coef,
          DotOut<T>{dy, dpart, apply_dot_parts(b, false)}, part, skip);
    else
      launch_lap<T, double, T, DIM, false, false>(b, tn, st, u, a, v, ld, nrhs, cd, co, gsum,
                                                  gscale, b->inst_coef,
                                                  DotOut<T>{nullptr, nullptr, 0}, part, skip);
  };
  if (!ev) {
    gather(PART_ALL);
    lap(PART_ALL);
    return;
  }
  CPM_HIP(hipEventRecord(ev[0], st));
  gather(PART_MAIN);
  CPM_HIP(hipEventRecord(ev[1], st));
  gather(PART_EXPLICIT);
  CPM_HIP(hipEventRecord(ev[2], st));
  lap(PART_MAIN);
  CPM_HIP(hipEventRecord(ev[3], st));
  lap(PART_EXPLICIT);
  CPM_HIP(hipEventRecord(ev[4], st));
}

template <class T>
void apply_with_scratch(const cpm_band* b, double m, double n, int nrhs, const T* u, T* v,
                        hipStream_t st, double* a, hipEvent_t* ev) {
  if (b->dim == 3) apply_dim<T, 3>(b, m, n, nrhs, u, v, st, nullptr, 0.0, a, ev);
  else apply_dim<T, 2>(b, m, n, nrhs, u, v, st, nullptr, 0.0, a, ev);
}

template <class T>
void apply_impl(const cpm_band* b, double m, double n, int nrhs, const T* u, T* v, hipStream_t st,
                const double* gauge_sum, double gamma, const T* dy, double* dpart,
                Skip skip) {
  double* gs = nullptr;
  if (gamma != 0.0) {
    // gauge: gamma * (sum of the PDE entries of u) / n_s on every row
    const int np = 256;
    double* part = static_cast<double*>(band_scratch(b, 3, sizeof(double) * np * nrhs + 64));
    gs = gauge_sum ? const_cast<double*>(gauge_sum)
                   : static_cast<double*>(band_scratch(b, 4, sizeof(double) * nrhs + 64));
    hipLaunchKernelGGL(k_sum_part<T>, dim3(np, nrhs), dim3(256), 0, st, u, b->n_s, b->n, part);
    CPM_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_sum_final, dim3(nrhs), dim3(256), 0, st, part, np, gs);
    CPM_LAUNCH_CHECK();
  }
  double* a = static_cast<double*>(band_scratch(b, 0, apply_scratch_bytes(b, nrhs)));
  if (b->dim == 3) apply_dim<T, 3>(b, m, n, nrhs, u, v, st, gs, gamma, a, nullptr, dy, dpart, skip);
  else apply_dim<T, 2>(b, m, n, nrhs, u, v, st, gs, gamma, a, nullptr, dy, dpart, skip);
}

// The transposed apply.  c = (L - diag L)^T w and e = E^T c are FP64 scratch
// vectors for both storage precisions (the combine step cancels the two
// terms of size N^2, as the forward Laplacian pass does).
template <class T, int DIM>
static void apply_T_dim(const cpm_band* b, double m, double n, int nrhs, const T* w, T* z,
                        hipStream_t st, const T* dy = nullptr, double* dpart = nullptr) {
  const int64_t ld = b->n;
  double* c = static_cast<double*>(band_scratch(b, 1, sizeof(double) * (size_t)ld * nrhs));
  double* e = static_cast<double*>(band_scratch(b, 2, sizeof(double) * (size_t)ld * nrhs));
  const double N2 = (double)b->N * (double)b->N;
  const double co = N2;
  // c = (L - diag L)^T w: symmetric bulk over every PDE row, then corrections
  // (fill kernels, not memsets: this sequence may be captured into a graph);
  // k_lap<ALL> writes every PDE entry, so only the BC entries need clearing
  if (b->n_c)
    for (int r = 0; r < nrhs; ++r)
      hipLaunchKernelGGL(k_fill<double>, dim3(grid_for(b->n_c, 256, 4096)), dim3(256), 0, st,
                         c + r * ld + b->n_s, (int64_t)b->n_c, 0.0);
  launch_lap<T, T, double, DIM, true, false>(b, tune_of<T>(b), st, w, w, c, ld, nrhs, 0.0, co,
                                             nullptr, 0.0, nullptr,
                                             DotOut<double>{nullptr, nullptr, 0}, PART_ALL, Skip{});
  if (b->lt_tgt) {
    if (b->n_lt) {
      hipLaunchKernelGGL(k_lt_pull<T>, dim3(grid_for(b->n_lt, 256)), dim3(256), 0, st, b->n_lt,
                         b->lt_tgt, b->lt_start, b->lt_src, b->lrow_id, w, c, ld, nrhs, co);
      CPM_LAUNCH_CHECK();
    }
  } else if (b->n_lrows) {
    CPM_FAIL(CPM_E_INVALID, "this band has no transposed FD pull lists");
  }
  // e = E^T c
  hipLaunchKernelGGL(k_fill<double>, dim3(grid_for(ld * nrhs, 256, 4096)), dim3(256), 0, st, e,
                     ld * nrhs, 0.0);
  if (b->ntiles) {
    if (!b->tile_col) CPM_FAIL(CPM_E_INVALID, "this band has no transpose schedule");
    for (int r = 0; r < nrhs; ++r)
      for (int k = 0; k < 8; ++k) {
        const int cnt = b->col_start[k + 1] - b->col_start[k];
        if (!cnt) continue;
        hipLaunchKernelGGL((k_gather_T<T, DIM>), dim3(cnt), dim3(64), 0, st, bview(b), tview(b),
                           b->tile_col + b->col_start[k], b->N, c, e, ld, r, tune_of<T>(b).xcd);
        CPM_LAUNCH_CHECK();
      }
  }
  if (b->et_tgt) {
    if (b->n_et) {
      for (int r = 0; r < nrhs; ++r)
        hipLaunchKernelGGL(k_et_pull, dim3((b->n_et + 3) / 4), dim3(256), 0, st, b->n_et,
                           b->et_tgt, b->et_start, b->et_src, b->et_w, c + r * ld, e + r * ld);
      CPM_LAUNCH_CHECK();
    }
  } else if (b->n_erows) {
    CPM_FAIL(CPM_E_INVALID, "this band has no transposed interpolation pull lists");
  }
  const double cd = m + n * (-2.0 * DIM * N2);
  const int64_t total = ld * nrhs;
  const int gc = grid_for(total, 256);
  if (dy) {
    if ((int64_t)gc * 256 < total) CPM_FAIL(CPM_E_INVALID, "internal: fused dot grid too small");
    hipLaunchKernelGGL((k_combine<T, true>), dim3(gc), dim3(256), 0, st, w, e, z, cd, n, total,
                       dy, dpart, gc);
  } else {
    hipLaunchKernelGGL((k_combine<T>), dim3(gc), dim3(256), 0, st, w, e, z, cd, n, total,
                       nullptr, nullptr, 0);
  }
  CPM_LAUNCH_CHECK();
}

template <class T>
void apply_transpose_impl(const cpm_band* b, double m, double n, int nrhs, const T* w, T* z,
                          hipStream_t st, const double*, double gamma, const T* dy,
                          double* dpart) {
  if (gamma != 0.0) CPM_FAIL(CPM_E_INVALID, "the gauge is not supported for the transpose");
  if (b->dim == 3) apply_T_dim<T, 3>(b, m, n, nrhs, w, z, st, dy, dpart);
  else apply_T_dim<T, 2>(b, m, n, nrhs, w, z, st, dy, dpart);
}

template void apply_impl<double>(const cpm_band*, double, double, int, const double*, double*,
                                 hipStream_t, const double*, double, const double*, double*, Skip);
template void apply_impl<float>(const cpm_band*, double, double, int, const float*, float*,
                                hipStream_t, const double*, double, const float*, double*, Skip);
template void apply_transpose_impl<double>(const cpm_band*, double, double, int, const double*,
                                           double*, hipStream_t, const double*, double,
                                           const double*, double*);
template void apply_transpose_impl<float>(const cpm_band*, double, double, int, const float*,
                                          float*, hipStream_t, const double*, double,
                                          const float*, double*);

}  // namespace cpm

using namespace cpm;

static void check_vec_args(const cpm_band* b, int dtype, int nrhs, const void* x, const void* y) {
  if (!b) CPM_FAIL(CPM_E_INVALID, "null band");
  if (dtype != CPM_F64 && dtype != CPM_F32) CPM_FAIL(CPM_E_INVALID, "unknown dtype %d", dtype);
  if (nrhs < 1) CPM_FAIL(CPM_E_INVALID, "nrhs must be >= 1 (got %d)", nrhs);
  if ((int64_t)nrhs * b->n >= (1ll << 31))
    CPM_FAIL(CPM_E_INVALID, "nrhs * n exceeds the 32-bit index range");
  if (!x || !y) CPM_FAIL(CPM_E_INVALID, "null vector");
  if (x == y) CPM_FAIL(CPM_E_INVALID, "input and output must not alias");
}

extern "C" cpm_status cpm_apply(const cpm_band* b, double m, double n, int dtype, int nrhs,
                                const void* u, void* v, void* hip_stream) {
  return guard([&] {
    check_vec_args(b, dtype, nrhs, u, v);
    hipStream_t st = (hipStream_t)hip_stream;
    if (dtype == CPM_F64)
      apply_impl<double>(b, m, n, nrhs, (const double*)u, (double*)v, st);
    else
      apply_impl<float>(b, m, n, nrhs, (const float*)u, (float*)v, st);
  });
}

// ---------------------------------------------------------------- no-alloc
// cpm_apply for callers that cannot allocate device memory.  The scratch the
// apply needs (the FP64 intermediate a = E u) lives in a file-scope device
// array of kNoAllocScratchBytes, one copy per GPU the library runs on, held
// until the process ends.  Host code never passes the array's name to a
// kernel (on the host it only stands in for the symbol): its device address
// is looked up once per device with hipGetSymbolAddress and kept in
// g_noalloc_ptr.  Calls on one GPU share the array, so calls that overlap on
// one GPU (different streams, or threads) race on it.  Every entry of a the
// apply reads is written by the same apply first, so nothing needs clearing.
constexpr size_t kNoAllocScratchBytes = size_t(32) << 20;   // 32 MiB
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[kMaxDevices] = {};

void* noalloc_scratch() {
  int dev = 0;
  CPM_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) CPM_FAIL(CPM_E_INVALID, "device ordinal %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_noalloc_mu);
  if (!g_noalloc_ptr[dev]) {
    void* ptr = nullptr;
    CPM_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) CPM_FAIL(CPM_E_HIP, "hipGetSymbolAddress returned a null scratch address");
    g_noalloc_ptr[dev] = ptr;
  }
  return g_noalloc_ptr[dev];
}
}  // namespace

extern "C" cpm_status cpm_apply_noalloc(const cpm_band* b, double m, double n, int dtype,
                                        int nrhs, const void* u, void* v, void* hip_stream) {
  return guard([&] {
    check_vec_args(b, dtype, nrhs, u, v);
    const size_t need = apply_scratch_bytes(b, nrhs);
    if (need > kNoAllocScratchBytes)
      CPM_FAIL(CPM_E_INVALID,
               "cpm_apply_noalloc: n * nrhs = %lld needs %zu bytes of scratch, above the "
               "%zu-byte static limit (n * nrhs <= %zu); use cpm_apply",
               (long long)(b->n * nrhs), need, kNoAllocScratchBytes,
               kNoAllocScratchBytes / sizeof(double));
    double* a = static_cast<double*>(noalloc_scratch());
    hipStream_t st = (hipStream_t)hip_stream;
    if (dtype == CPM_F64)
      apply_with_scratch<double>(b, m, n, nrhs, (const double*)u, (double*)v, st, a, nullptr);
    else
      apply_with_scratch<float>(b, m, n, nrhs, (const float*)u, (float*)v, st, a, nullptr);
  });
}

extern "C" cpm_status cpm_apply_profile(const cpm_band* b, double m, double n, int dtype,
                                        int nrhs, const void* u, void* v, int reps,
                                        void* hip_stream, double* ms) {
  return guard([&] {
    check_vec_args(b, dtype, nrhs, u, v);
    if (reps < 1 || !ms) CPM_FAIL(CPM_E_INVALID, "reps must be >= 1 and ms non-null");
    hipStream_t st = (hipStream_t)hip_stream;
    hipEvent_t ev[5];
    for (auto& e : ev) CPM_HIP(hipEventCreate(&e));
    double acc[4] = {0, 0, 0, 0};
    try {
      for (int k = 0; k < reps; ++k) {
        double* a = static_cast<double*>(band_scratch(b, 0, apply_scratch_bytes(b, nrhs)));
        if (dtype == CPM_F64)
          apply_with_scratch<double>(b, m, n, nrhs, (const double*)u, (double*)v, st, a, ev);
        else
          apply_with_scratch<float>(b, m, n, nrhs, (const float*)u, (float*)v, st, a, ev);
        CPM_HIP(hipEventSynchronize(ev[4]));
        for (int p = 0; p < 4; ++p) {
          float t = 0.f;
          CPM_HIP(hipEventElapsedTime(&t, ev[p], ev[p + 1]));
          acc[p] += t;
        }
      }
    } catch (...) {
      for (auto& e : ev) (void)hipEventDestroy(e);
      throw;
    }
    for (auto& e : ev) (void)hipEventDestroy(e);
    for (int p = 0; p < 4; ++p) ms[p] = acc[p] / reps;
  });
}

extern "C" cpm_status cpm_autotune(cpm_band* b, int dtype, int nrhs, const void* u, void* v,
                                   int reps, void* hip_stream, double* ms, int* best) {
  return guard([&] {
    check_vec_args(b, dtype, nrhs, u, v);
    if (reps < 1) CPM_FAIL(CPM_E_INVALID, "reps must be >= 1");
    hipStream_t st = (hipStream_t)hip_stream;
    Tune& tn = b->tune[dtype == CPM_F64 ? 0 : 1];
    const Tune saved = tn;
    hipEvent_t e0, e1;
    CPM_HIP(hipEventCreate(&e0));
    CPM_HIP(hipEventCreate(&e1));
    double t[kTuneVariants], seen[4] = {-1.0, -1.0, -1.0, -1.0};
    int arg = 0;
    try {
      for (int k = 0; k < kTuneVariants; ++k) {
        tn = tune_variant(k);
        if (((k >> 1) & 3) >= 2 && b->composite) {   // single bands only
          t[k] = HUGE_VAL;
          continue;
        }
        double& known = seen[2 * tn.xcd + tn.pad];
        if (known < 0.0) {
          auto run = [&] {
            if (dtype == CPM_F64) apply_impl<double>(b, 0.0, -1.0, nrhs, (const double*)u, (double*)v, st);
            else apply_impl<float>(b, 0.0, -1.0, nrhs, (const float*)u, (float*)v, st);
          };
          run();   // warm up
          CPM_HIP(hipEventRecord(e0, st));
          for (int r = 0; r < reps; ++r) run();
          CPM_HIP(hipEventRecord(e1, st));
          CPM_HIP(hipEventSynchronize(e1));
          float f = 0.f;
          CPM_HIP(hipEventElapsedTime(&f, e0, e1));
          known = f / reps;
        }
        t[k] = known;
        if (t[k] < t[arg]) arg = k;
      }
    } catch (...) {
      tn = saved;
      (void)hipEventDestroy(e0);
      (void)hipEventDestroy(e1);
      throw;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    tn = tune_variant(arg);
    if (ms)
      for (int k = 0; k < kTuneVariants; ++k) ms[k] = t[k];
    if (best) *best = arg;
  });
}

extern "C" cpm_status cpm_tune_set(cpm_band* b, int dtype, int variant) {
  return guard([&] {
    if (!b) CPM_FAIL(CPM_E_INVALID, "null band");
    if (dtype != CPM_F64 && dtype != CPM_F32) CPM_FAIL(CPM_E_INVALID, "unknown dtype %d", dtype);
    if (variant < 0 || variant >= kTuneVariants)
      CPM_FAIL(CPM_E_INVALID, "launch variant %d out of range [0, %d)", variant, kTuneVariants);
    b->tune[dtype == CPM_F64 ? 0 : 1] = tune_variant(variant);
  });
}

extern "C" cpm_status cpm_apply_transpose(const cpm_band* b, double m, double n, int dtype,
                                          int nrhs, const void* w, void* z, void* hip_stream) {
  return guard([&] {
    check_vec_args(b, dtype, nrhs, w, z);
    hipStream_t st = (hipStream_t)hip_stream;
    if (dtype == CPM_F64)
      apply_transpose_impl<double>(b, m, n, nrhs, (const double*)w, (double*)z, st);
    else
      apply_transpose_impl<float>(b, m, n, nrhs, (const float*)w, (float*)z, st);
  });
}

extern "C" cpm_status cpm_rhs(const cpm_band* b, double n, int nrhs, const double* f,
                              const double* g, double* out, void* hip_stream) {
  return guard([&] {
    if (!b || !f || !out || nrhs < 1) CPM_FAIL(CPM_E_INVALID, "bad argument");
    if (b->n_c && !g) CPM_FAIL(CPM_E_INVALID, "g is required when the band has BC DOFs");
    hipStream_t st = (hipStream_t)hip_stream;
    const int64_t total = b->n * nrhs;
    hipLaunchKernelGGL(k_rhs_init, dim3(grid_for(total, 256)), dim3(256), 0, st, b->n_s, b->n_c,
                       nrhs, f, b->bc_node, out);
    CPM_LAUNCH_CHECK();
    if (g) add_dirichlet_term(b, n, g, nrhs, out, st);
  });
}

namespace cpm {
// out -= n (L - diag L) e(g) over the rows that reference BC DOFs: the
// Dirichlet part of the right-hand side (Sec. 4.3), nrhs vectors.
void add_dirichlet_term(const cpm_band* b, double n, const double* g, int nrhs, double* out,
                        hipStream_t st) {
  if (!b->n_c || !b->n_lrows) return;
  const double N2 = (double)b->N * (double)b->N;
  hipLaunchKernelGGL(k_rhs_rows, dim3(grid_for(b->n_lrows, 128)), dim3(128), 0, st, b->n_lrows,
                     2 * b->dim, b->n_s, b->n_c, nrhs, b->lrow_id, b->lcol, g, b->bc_ecoef,
                     n * N2, out);
  CPM_LAUNCH_CHECK();
}
}  // namespace cpm

extern "C" cpm_status cpm_rhs_adjoint(const cpm_band* b, double n, int nrhs, const double* lam,
                                      double* grad_f, double* grad_g, void* hip_stream) {
  return guard([&] {
    if (!b || !lam || !grad_f || nrhs < 1) CPM_FAIL(CPM_E_INVALID, "bad argument");
    hipStream_t st = (hipStream_t)hip_stream;
    hipLaunchKernelGGL(k_gradf, dim3(grid_for(b->n_s * nrhs, 256)), dim3(256), 0, st, b->n_s,
                       b->n_c, nrhs, lam, grad_f);
    CPM_LAUNCH_CHECK();
    if (b->n_c) {
      hipLaunchKernelGGL(k_gradf_bc, dim3(grid_for(b->n_c * nrhs, 256)), dim3(256), 0, st,
                         b->n_s, b->n_c, nrhs, b->bc_node, lam, grad_f);
      CPM_LAUNCH_CHECK();
    }
    if (grad_g && b->n_c) {
      CPM_HIP(hipMemsetAsync(grad_g, 0, sizeof(double) * b->n_c * nrhs, st));
      const double N2 = (double)b->N * (double)b->N;
      hipLaunchKernelGGL(k_gradg, dim3(grid_for(b->n_lrows, 128)), dim3(128), 0, st, b->n_lrows,
                         2 * b->dim, b->n_s, b->n_c, nrhs, b->lrow_id, b->lcol, lam,
                         b->bc_ecoef, -n * N2, grad_g);
      CPM_LAUNCH_CHECK();
    }
  });
}
