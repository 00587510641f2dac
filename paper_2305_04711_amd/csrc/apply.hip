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

// Wave-uniform broadcast of lane k (k must be the same in every lane).
__device__ __forceinline__ int lane_i32(int v, int k) { return __builtin_amdgcn_readlane(v, k); }

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

// Orders a wavefront's LDS accesses among its lanes: the hardware takes them in
// program order, so only the compiler is held back.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Explicit interpolation rows: a[id] = sum_o w_o u[col_o], 4^d lanes per row
// (a wavefront in 3-D, a quarter of one in 2-D), lane = member; FP64 weights
// and sums for both storage precisions.
constexpr int kERowLds = 128;   // doubles of a wavefront
struct ERows {
  int waves, groups;      // wavefronts of rows (ERowPack); those of the grid (a multiple of 8)
  const int* id;
  const int* col;
  const double* w1;       // 1-D weights, 4 per axis
  int p;
  const int* inst;        // composite: instance of each row
};

// The wavefront's rows are bound by its vector-memory instructions, not by
// bytes: with a load for each row's columns, member weights and number and a
// store each, 1-D weights alone (96 bytes a row for 512) made them slower.
// Four rows' columns now come in one load, their 1-D weights in another (s:
// ERowPack::kRows * 4 * DIM doubles of the wavefront's own, the products formed
// in registers) and the sums leave in one store.  Whole apply before and now:
// sphere at h = 1/64 18.1, 17.4 us, 1/256, FP32, 142.7, 134.3 us; torus at
// 1/512, FP64, 743, 731 us (the rows alone 39 and 25 us).
template <class TS, int DIM>
__device__ __forceinline__ void explicit_rows(const ERows& er, int wave, int lane,
                                              const TS* __restrict__ u, double* __restrict__ a,
                                              int64_t ld, int r0, int r1, const Skip& skip,
                                              double* s) {
  using EP = ERowPack<DIM>;
  constexpr int M = EP::M, NW = EP::kRows * 4 * DIM;
  if (wave >= er.waves) return;
  if (!er.inst && r1 == r0 + 1 && skipped(skip, r0, 0)) return;
  const int4 c4 = reinterpret_cast<const int4*>(er.col)[(int64_t)wave * 64 + lane];
  const int c[4] = {c4.x, c4.y, c4.z, c4.w};
  // lane j (2-D: of each 16) stores row j
  const int j0 = lane & (M - 1);
  const int64_t row = EP::row(wave, min(j0, 3), lane);
  const int id = er.id[row], inst = er.inst ? er.inst[row] : 0;
  double wl[(NW + 63) / 64];
#pragma unroll
  for (int k = 0; k < (NW + 63) / 64; ++k)
    wl[k] = er.w1[(int64_t)wave * NW + min(64 * k + lane, NW - 1)];
#pragma unroll
  for (int k = 0; k < (NW + 63) / 64; ++k) s[min(64 * k + lane, NW - 1)] = wl[k];
  wave_sync();
  const int mo = erow_member<DIM>(er.p, j0);
  double w[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) w[j] = erow_weight<DIM>(s + EP::row(0, j, lane) * 4 * DIM, mo);
  for (int r = r0; r < r1; ++r) {
    // every lane loads (an absent member's lane entry 0, which it drops), so
    // that no load waits behind a branch for the one before it
    double v[4], out = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (double)u[r * ld + max(c[j], 0)];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = lanes_sum<M>(c[j] >= 0 ? w[j] * v[j] : 0.0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (DIM == 3) {
        const long long b = __double_as_longlong(v[j]);
        v[j] = __longlong_as_double(((long long)lane_i32((int)(b >> 32), 63) << 32) |
                                    (unsigned)lane_i32((int)(unsigned)(b & 0xffffffffll), 63));
      }
      out = j0 == j ? v[j] : out;
    }
    if (j0 < 4 && id >= 0 && !skipped(skip, r, inst)) a[r * ld + id] = out;
  }
}

// The tile rows of 2 x 2 neighbouring tiles (x and y) are interpolated
// together: a supertile (Super), its rows two of a stencil base to a slot.
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

// fraction of row i (two to a slot) along the axis whose slots begin at s0
template <class TS> __device__ __forceinline__ double frac_row(const SuperView& sv, int64_t s0, int64_t i);
template <> __device__ __forceinline__ double frac_row<double>(const SuperView& sv, int64_t s0, int64_t i) {
  return reinterpret_cast<const double*>(sv.frac64 + s0)[i];
}
template <> __device__ __forceinline__ double frac_row<float>(const SuperView& sv, int64_t s0, int64_t i) {
  return (double)reinterpret_cast<const float*>(sv.frac32 + s0)[i];
}

// Interpolation of the two rows of a slot from the staged cubes, one of each
// right-hand side that is on (sum-factorised tensor product): x lines first,
// then y, then z; FP64 arithmetic.  NP = p + 1 stencil nodes per axis.  Both
// rows read the same members, each once.
template <int DIM, int NP, int E, int EP, int NR, class NEXT, class PUT>
__device__ __forceinline__ void interp_pair(const double* __restrict__ s0, int cube,
                                            const bool on[NR], const double2 t[DIM], NEXT next,
                                            PUT put) {
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
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    if (!on[i]) continue;
    const double* s = s0 + i * cube;
    double out[2] = {0.0, 0.0};
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
    // keeps the sums out of the branches that store them (the compiler would
    // sink them there and hold every member in a register for them)
    asm volatile("" : "+v"(out[0]), "+v"(out[1]));
    put(i, out);
  }
}

// Pass 1 in one launch, W wavefronts to a workgroup: the first sv.n take a
// supertile each, the last ones explicit rows.  Those are short and fill the
// chip while the last supertiles end: first in the grid they cost the whole
// apply 22.6, 149 and 756 us against 18.2, 143 and 745 us (sphere at h = 1/64,
// FP64, and 1/256, FP32; torus at 1/512, FP64).
//
// What bounds it: with one tile per wavefront and one row per lane every row
// read its 4^d members from LDS by itself, at 128 B a clock and CU, with 71%
// of the lanes filled, and the LDS was busy in 84% of the cycles (0.49 ms for
// the 34.0M tile rows of the torus at h = 1/512, FP64).  A lane that
// interpolates two rows of one stencil base reads the members once for both,
// and the pooled slots of 2 x 2 tiles fill 77% of the lanes: LDS busy 52%.
// The staged blocks' loads, each under a branch of its own, also waited for
// one another; all 18 are now in flight at once.  The kernel moves 2.06
// GB at 4.4 TB/s (explicit rows included, 0.47 ms against 0.55 ms), with the
// vector unit busy 60% and the LDS 56% of the time.  Four such tiles by four
// wavefronts with a barrier (27 blocks) took 0.63 ms and a persistent pipeline
// over them 0.55 ms: wavefronts that wait for one another hold their slots
// idle.  Registers, not LDS, set the occupancy (4 or 5 wavefronts per SIMD);
// forcing a sixth spills and loses.

// Two wavefronts share a supertile where supertiles are few or take several
// right-hand sides in turn: half the chain of each, next to a barrier.
// Transpose of one column, one wavefront, two: 28.6, 21.8 us at 600
// supertiles; 45.6, 41.7 at 2300; 60.6, 60.6 at 4500; 100, 109 at 9100 (two
// fill and clear two cubes).  Forward apply: 18.3, 17.9 us at 2000; 20.6, 19.3
// at 2300; 29.9, 29.9 at 4500; 47.0, 47.8 at 9100; of three columns 34.4, 31.4
// at 1100; 63.4, 61.6 at 4500; 323, 306 at 20000 (FP64 spheres and tori).
constexpr int kSplitBelow = 4096;
// Right-hand sides go to workgroups of their own while there are fewer
// supertiles than this in flight (eight columns, in turn and apart: 58 and 39
// us at 600 supertiles, 21 and 14 us in 2-D at 40; five: 54 and 56 us at
// 2000), and in pass 1 of a solver, whose systems end at different times
// (batched solve of 18 systems: 220 and 195 ms).
constexpr int kFillSupertiles = 2048, kMaxRhsGroups = 4096;
// A workgroup with several right-hand sides takes two at a time (NR), a cube
// each, so that a slot's data and weights are read and formed once for both:
// two, three and eight columns 203, 302, 795 us with one at a time, 178, 282,
// 728 now (torus at h = 1/192, FP64).
// Wavefronts per SIMD to fit the registers to: five where that spills nothing
// (FP64 pairs at five spill 6 registers: 198, 306, 766 us).
constexpr int gather_waves(int size, int w, int nr) {
  return nr == 2 ? (size == 8 ? 4 : 5) : w == 2 ? 5 : 4;
}
template <class TS, int DIM, int PAD, int NP, int W, int NR>
__global__ __launch_bounds__(64 * W) __attribute__((
    amdgpu_waves_per_eu(gather_waves(sizeof(TS), W, NR)))) void k_gather(
    ERows er, SuperView sv, const QMeta* __restrict__ meta, const int4* __restrict__ rng,
    const TS* __restrict__ u, double* __restrict__ a, int64_t ld, int nrhs, int per, int xcd,
    Skip skip) {
  using G = Geo<DIM>;
  using SP = Super<DIM>;
  constexpr int EX = SP::EX, EP = EX + PAD, BX = G::BX, NB = SP::NB;
  constexpr InsideMasks<DIM> IN = inside_masks<DIM>();
  constexpr int CS = SP::EZ * EX * EP;
  static_assert(CS >= W * kERowLds, "explicit rows' weights");
  __shared__ double s_u[NR][CS + 1];
  constexpr int NQ = (NB + W - 1) / W;   // blocks staged by a wave
  const int lane = threadIdx.x & 63;
  const int wv = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = blockIdx.y * per, r1 = min(nrhs, r0 + per);
  int g = blockIdx.x;
  if (g >= sv.n) {
    g -= sv.n;
    if (xcd) g = xcd_remap(g, er.groups / W);
    explicit_rows<TS, DIM>(er, g * W + wv, lane, u, a, ld, r0, r1, skip, s_u[0] + wv * kERowLds);
    return;
  }
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
  for (int r = r0; r < r1; r += NR) {
    // keeps the cells of all staged blocks from living in registers throughout
    asm volatile("" : "+v"(cell0));
    bool on[NR];
    if constexpr (NR == 1) {
      if (skipped(skip, r, rg.z)) continue;
      on[0] = true;
    } else {
      bool any = false;
#pragma unroll
      for (int i = 0; i < NR; ++i) {
        on[i] = r + i < r1 && !skipped(skip, r + i, rg.z);
        any |= on[i];
      }
      if (!any) continue;
    }
    // the first pass's row data is requested before the staging loads
    rows(64 * wv + lane);
    __syncthreads();   // the previous right-hand sides' rows are done
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      if (!on[i]) continue;
      // Every lane loads (an absent node's lane the block's first value, which
      // it drops): under a condition each load would be a basic block of its
      // own and wait for the one before it.
      // Cells of absent nodes hold that value: no tile row's stencil has one.
      const TS* ur = u + (r + i) * ld;
      TS x[NQ];
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        const int q = min(j * W + wv, NB - 1);
        x[j] = ur[lane_i32(qm.z, q) + (int64_t)lane_rank(qmask(q))];
      }
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        const int q = min(j * W + wv, NB - 1);
        const int qx = q % 3, qy = (q / 3) % 3, qz = q / 9;
        const int off = (DIM == 3 ? (qz * BX * EX + qy * BX) * EP : qy * BX * EP) + qx * BX;
        bool in;
        if constexpr (W == 1) in = IN.m[q] == ~0ull || lane_in(IN.m[q]);
        else
          in = qx * BX + G::lx(lane) < EX && qy * BX + G::ly(lane) < EX &&
               (DIM == 2 || qz * BX + G::lz(lane) < SP::EZ);
        s_u[i][in ? cell0 + off : CS] = (double)x[j];
      }
    }
    __syncthreads();
    for (int k = 64 * wv + lane; k - lane < rg.y; k += 64 * W) {
      const int2 dc = dof;
      const int bc = ((DIM == 3 ? (code >> 8) * EX : 0) + ((code >> 4) & 15)) * EP + (code & 15);
      interp_pair<DIM, NP, EX, EP, NR>(
          &s_u[0][bc], CS + 1, on, t, [&] { rows(k + 64 * W); },
          [&](int i, const double v[2]) {
            if (k < rg.y) {
              a[(r + i) * ld + dc.x] = v[0];
              if (dc.y >= 0) a[(r + i) * ld + dc.y] = v[1];
            }
          });
    }
  }
}

// Workgroup sums of d0 and d1 (256 threads, every one must call it), written
// to part[idx] and part[np + idx]: the partials of a fused dot product, one
// per workgroup, finished in a fixed order by the solver.
static_assert(kLapThreads == 256, "four wavefronts");
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
//   * the blocks' metadata (their own and their face neighbours' masks and
//     first DOFs, the explicit-row masks) comes in one vector load, an entry to
//     a lane, and is broadcast from there: every mask is wave-uniform and stays
//     in scalar registers (a chain of scalar loads: 315 us for 290 at 34.1M
//     rows);
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

// Explicit FD rows (swapped PDE rows and BC rows), one thread each.
struct LRows {
  int n, groups;          // rows; workgroups that hold them
  int nf;
  const int* id;          // row DOF (-1: padding of a composite)
  const int* col;
  const int* inst;        // composite: instance of each row
};

// The transpose's explicit FD rows by pull lists: target k of the ascending
// list takes +-co w of the rows src[start[k] .. start[k + 1]) (an entry is
// 2 row + (1: subtracted)), in that order.  blk and bc find the targets of a
// block and of a BC DOF.
struct LPull {
  const Pull* blk;
  const int* bc;
  const int* start;
  const int* src;
  const int* row_id;
  int n_s, n_c;
};
template <class TU>
__device__ __forceinline__ double pull_rows(const LPull& lp, int64_t k, const TU* __restrict__ w,
                                            double co) {
  double acc = 0.0;
  for (int e = lp.start[k], e1 = lp.start[k + 1]; e < e1; ++e) {
    const int v = lp.src[e];
    const double wi = co * (double)w[lp.row_id[v >> 1]];
    acc += (v & 1) ? -wi : wi;
  }
  return acc;
}

// Fused dot products of the pass: with y set, the partials of (y, v) and
// (v, v) of right-hand side r go to part + 2 r np, one per workgroup.
template <class TV>
struct DotOut {
  const TV* y;
  double* part;
  int np;
};

// The first lr.groups workgroups take explicit rows (ALL: the BC entries), the
// others blocks.
template <class TU, class TA, class TV, int DIM, bool ALL, bool DOT = false>
__global__ __launch_bounds__(kLapThreads) void k_lap(
    LRows lr, LPull lp, const QMeta* __restrict__ face, int nb, const TU* __restrict__ u,
    const TA* __restrict__ a, TV* __restrict__ v, int64_t ld, int nrhs, int per, double cd, double co,
    const double* __restrict__ gsum, double gscale, int xcd, const double* __restrict__ coef,
    Skip skip, DotOut<TV> dot) {
  using G = Geo<DIM>;
  constexpr int BX = G::BX, KB = kLapBlocksPerWave;
  constexpr int step[3] = {1, BX, BX * BX};
  constexpr FaceLanes<DIM> FL = face_lanes<DIM>();
  const int r0 = blockIdx.y * per, r1 = min(nrhs, r0 + per);
  if (ALL && (int)blockIdx.x < lr.groups) {   // BC entries: explicit rows only
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= lp.n_c) return;
    const int k = lp.bc[i];
    for (int r = r0; r < r1; ++r)
      if (!skipped(skip, r, 0))
        v[r * ld + lp.n_s + i] = (TV)(k >= 0 ? pull_rows(lp, k, u + r * ld, co) : 0.0);
    return;
  }
  if (!ALL && (int)blockIdx.x < lr.groups) {
    const int i = blockIdx.x * kLapThreads + threadIdx.x;
    const int id = i < lr.n ? lr.id[i] : -1;
    const int inst = coef && id >= 0 ? lr.inst[i] : 0;
    if (coef && id >= 0) {
      cd = coef[2 * inst];
      co = coef[2 * inst + 1];
    }
    int c[2 * DIM];
#pragma unroll
    for (int f = 0; f < 2 * DIM; ++f) c[f] = id >= 0 ? lr.col[(int64_t)i * lr.nf + f] : -1;
    for (int r = r0; r < r1; ++r) {
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
  // (ALL: and its explicit targets in lane 8 KB + j)
  const int4* fp = reinterpret_cast<const int4*>(face) +
                   ((int64_t)min(blk0 + min(lane >> 3, KB - 1), nb - 1) * 8 + (lane & 7));
  if (ALL && lane >= 8 * KB)
    fp = reinterpret_cast<const int4*>(lp.blk) + min(blk0 + min(lane - 8 * KB, KB - 1), nb - 1);
  const int4 fm = *fp;
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
  for (int r = r0; r < r1; ++r) {
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
        if constexpr (ALL) {
          const unsigned long long t =
              ((unsigned long long)(unsigned)lane_i32(fm.y, 8 * KB + j) << 32) |
              (unsigned)lane_i32(fm.x, 8 * KB + j);
          if (lane_in(t))
            o += pull_rows(lp, lane_i32(fm.z, 8 * KB + j) + (int64_t)lane_rank(t), u + r * ld,
                           coi[j]);
        }
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
// E^T c over the explicit rows by pull lists: entry e of the list has weight
// w[e] and source row src[e]; target k's entries are start[k] .. start[k + 1).
struct EPull {
  int n, groups;          // targets; wavefronts that hold them (a multiple of 8)
  const int* start;
  const int* src;
  const double* w;
};
constexpr int kEPullTargets = 4;   // targets per wavefront whose loads go out together

// x[k] = sum of target k's products w c_src: the lanes take the entries 64 at
// a time and sum their own in order, then the lanes' sums in a fixed order.
__device__ __forceinline__ void explicit_targets(const EPull& ep, int wave, int lane,
                                                 const double* __restrict__ c,
                                                 double* __restrict__ x) {
  int b0[kEPullTargets], b1[kEPullTargets], longest = 0;
#pragma unroll
  for (int j = 0; j < kEPullTargets; ++j) {
    const int k = min(wave * kEPullTargets + j, ep.n - 1);
    b0[j] = ep.start[k];
    b1[j] = ep.start[k + 1];
    longest = max(longest, b1[j] - b0[j]);
  }
  double acc[kEPullTargets] = {0.0, 0.0, 0.0, 0.0};
  for (int o = lane; o - lane < longest; o += 64) {
    int src[kEPullTargets];
    double w[kEPullTargets], v[kEPullTargets];
#pragma unroll
    for (int j = 0; j < kEPullTargets; ++j) {
      const int e = min(b0[j] + o, b1[j] - 1);   // every target has an entry
      src[j] = ep.src[e];
      w[j] = ep.w[e];
    }
#pragma unroll
    for (int j = 0; j < kEPullTargets; ++j) v[j] = c[src[j]];
#pragma unroll
    for (int j = 0; j < kEPullTargets; ++j)
      acc[j] += b0[j] + o < b1[j] ? w[j] * v[j] : 0.0;
  }
#pragma unroll
  for (int j = 0; j < kEPullTargets; ++j) {
    const double s = lanes_sum<64>(acc[j]);
    if (lane == 63 && wave * kEPullTargets + j < ep.n) x[wave * kEPullTargets + j] = s;
  }
}

// E^T c of the tile rows, a workgroup of W wavefronts per supertile.  The rows
// of one stencil base add w c into the same 4^d members, a small matrix
// product summed over the rows: in 3-D G[z][y][x] += sum_i (c_i wz_i[z]
// wy_i[y]) wx_i[x], four 4 x 4 blocks (z) with four rows to an instruction of
// the FP64 matrix unit, whose accumulator is one register (a member) per lane;
// in 2-D one 4 x 4 block, with sixteen rows in the four places, added up at
// the end.  Slots go in chunks of kTSlots: each lane puts a row's 1-D weights
// into LDS (c_i folded into the last), then the wave walks the chunk in steps
// of up to four (2-D: sixteen) rows of one base, kTSteps steps' reads at once,
// and adds each step's members into its cube in LDS without reading it back
// (a step's members are distinct cells and a wave's LDS operations complete in
// order, so the sum's order is fixed).  The cube's entries of the blocks'
// nodes, summed over the waves in order, then go to the supertile's part of
// buf, one after the other, where k_combine finds them (Pull): no order
// between supertiles, no clearing, one launch.  The explicit targets come last
// and fill the chip while the last supertiles end (torus at h = 1/256: 414 to
// 403 us for the whole transpose).
//
// What bounds it: LDS (55% of the cycles: three reads and one add a step) and
// the vector unit (41%) at 11 waves per CU at large sizes, a wave's chain of
// steps at small ones.  Whole transposes, FP64: torus at h = 1/256 (8.6M DOFs)
// 647 us with lane = member, one row at a time and a launch per parity class,
// 453 with one step at a time whose sums are read, added and written back,
// 403 now; sphere at h = 1/48, FP32, two right-hand sides: 319, 76 and 53.
// Chunks of 16, 32 slots: 432, 414 us; 4, 8 steps at once: 414, 434.
constexpr int kTSlots = 32, kTSteps = 4;
// Wavefronts of a supertile: kSplitBelow.
template <class TS, int DIM, int W>
__global__ __launch_bounds__(64 * W) void k_gather_T(EPull ep, SuperView sv,
                                                     const QMeta* __restrict__ meta,
                                                     const int4* __restrict__ rng,
                                                     const double* __restrict__ c,
                                                     double* __restrict__ x,
                                                     double* __restrict__ buf, int64_t ld,
                                                     int64_t bufld, int r0, int xcd, Skip skip) {
  using G = Geo<DIM>;
  using SP = Super<DIM>;
  constexpr int EX = SP::EX, EP = EX + 1, BX = G::BX, NB = SP::NB;
  constexpr int NW = DIM == 3 ? 12 : 8;       // 1-D weights per row
  constexpr int RC = 2 * kTSlots;             // rows of a chunk
  constexpr int RS = DIM == 3 ? 4 : 16;       // rows of a matrix instruction
  // Strides at which a half-wave's cells, and a step's weights, lie in
  // distinct banks.
  constexpr int PL = DIM == 3 ? 136 : EX * EP, CS = SP::EZ * PL;
  constexpr int WS = RC + RS;
  constexpr int U = kTSteps;
  constexpr InsideMasks<DIM> IN = inside_masks<DIM>();
  static_assert(RC <= 64, "a row per lane");
  static_assert(PL >= EX * EP, "planes apart");
  __shared__ double s_z[W][CS + 1];
  __shared__ double s_w[W][NW * WS];
  const int lane = threadIdx.x & 63;
  const int wv = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = blockIdx.y;
  if (skipped(skip, r0 + r, 0)) return;
  c += (r0 + r) * ld;
  int g = blockIdx.x;
  if (g >= sv.n) {
    g -= sv.n;
    if (xcd) g = xcd_remap(g, ep.groups / W);
    g = g * W + wv;
    if (g * kEPullTargets < ep.n) explicit_targets(ep, g, lane, c, x + (int64_t)r * ep.n);
    return;
  }
  if (xcd) g = xcd_remap(g, sv.n);
  const int4 rg = rng[g];
  const int4 qm = reinterpret_cast<const int4*>(meta)[(int64_t)g * NB + min(lane, NB - 1)];
  const int* dofs = reinterpret_cast<const int*>(sv.dof);
  // row data of the lane's row of a chunk (its last row's past the end: loads
  // under no branch); the wave's next chunk's is requested before a chunk is
  // walked, the DOFs (which c is read through) one chunk further ahead
  const int rows = 2 * rg.y;
  const int64_t first = 2 * (int64_t)rg.x;
  auto at = [&](int k) { return first + min(k + (lane & (RC - 1)), rows - 1); };
  auto frac = [&](int k, double t[DIM]) {
    const int64_t i = at(k);
#pragma unroll
    for (int d = 0; d < DIM; ++d) t[d] = frac_row<TS>(sv, d * sv.ns, i);
  };
  double t[DIM], ci;
  const int kw = wv * RC;
  int code, dof = dofs[at(kw)], dofn = dofs[at(kw + W * RC)];
  frac(kw, t);
  code = sv.base[at(kw) >> 1];
  ci = c[max(dof, 0)];
  double* z = s_z[wv];
  double* ws = s_w[wv];
  for (int k = lane; k < CS + 1; k += 64) z[k] = 0.0;
  for (int k = lane; k < NW * RS; k += 64) ws[(k / RS) * WS + RC + k % RS] = 0.0;
  // the lane's operands: rows rk of a step, entries ia (A) and ja (B), and its
  // member's cell
  const int rk = DIM == 3 ? lane >> 4 : (lane >> 4) + 4 * ((lane >> 2) & 3);
  const int ia = lane & 3, iz = (lane >> 2) & 3;
  double* cell = z + (DIM == 3 ? iz * PL : 0) + (lane >> 4) * EP + (lane & 3);
  const double* wb = ws + ia * WS + rk;
  const double* wz = ws + (8 + iz) * WS + rk;
  for (int k0 = kw; k0 < rows; k0 += W * RC) {
    const int nr = min(RC, rows - k0);                // rows of this chunk
    double w[DIM][4];
#pragma unroll
    for (int d = 0; d < DIM; ++d) lagrange_p<double>(sv.p, t[d], w[d]);
    const double cw = dof >= 0 ? ci : 0.0;            // a lone row's partner adds nothing
#pragma unroll
    for (int o = 0; o < 4; ++o) w[DIM - 1][o] *= cw;
    const int codes = code;
    // requested ahead
    frac(k0 + W * RC, t);
    code = sv.base[at(k0 + W * RC) >> 1];
    dof = dofn;
    ci = c[max(dofn, 0)];
    dofn = dofs[at(k0 + 2 * W * RC)];
    wave_sync();   // the previous chunk is walked
    if (lane < RC) {
#pragma unroll
      for (int d = 0; d < DIM; ++d)
#pragma unroll
        for (int o = 0; o < 4; ++o) ws[(4 * d + o) * WS + lane] = w[d][o];
    }
    wave_sync();
    // A step is up to RS rows of one base: the rows at which a base begins,
    // the row's place in its base's, and the rows at which a step begins.
    const unsigned long long starts =
        __ballot(codes != __builtin_amdgcn_update_dpp(-1, codes, 0x138, 0xf, 0xf, false));
    const int place = lane - (63 - __clzll((long long)(starts & (~0ull >> (63 - lane)))));
    unsigned long long steps = __ballot(place % RS == 0 && lane < nr);
    const int off = ((DIM == 3 ? (codes >> 8) * PL : 0) + ((codes >> 4) & 15) * EP + (codes & 15)) * 8;
    while (steps) {
      // U steps at a time, the reads of all first; past the last: no rows
      int k[U], m[U], o[U];
#pragma unroll
      for (int j = 0; j < U; ++j) {
        k[j] = steps ? __ffsll((long long)steps) - 1 : 0;
        const unsigned long long rest = steps & (steps - 1);
        m[j] = steps ? (rest ? __ffsll((long long)rest) - 1 : nr) - k[j] : 0;
        o[j] = lane_i32(off, k[j]);
        steps = steps ? rest : 0;
      }
      double A0[U], A1[U], B[U], acc[U];
#pragma unroll
      for (int j = 0; j < U; ++j) {
        A0[j] = (wb + 4 * WS)[k[j]];
        if (DIM == 3) A1[j] = wz[k[j]];
        B[j] = wb[k[j]];
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        double A = DIM == 3 ? A0[j] * A1[j] : A0[j];
        A = rk < m[j] ? A : 0.0;
        acc[j] = __builtin_amdgcn_mfma_f64_4x4x4f64(A, B[j], 0.0, 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        if constexpr (DIM == 2) {
          // the four places' sums of the lanes 4 and 8 apart
          acc[j] = dpp_add<0x124>(acc[j]);
          acc[j] = dpp_add<0x128>(acc[j]);
        }
        double* to = reinterpret_cast<double*>(reinterpret_cast<char*>(cell) + o[j]);
        if (DIM == 3 || iz == 0)
          (void)__hip_atomic_fetch_add(to, acc[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    }
  }
  if (W > 1) __syncthreads();
  else wave_sync();
  // the cube's entries of the staged blocks' nodes, summed over the waves
  double* out = buf + (int64_t)r * bufld + (int64_t)g * SP::CELLS;
  const int cell0 = DIM == 3 ? G::lz(lane) * PL + G::ly(lane) * EP + G::lx(lane)
                             : G::ly(lane) * EP + G::lx(lane);
  double v[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const int qx = q % 3, qy = (q / 3) % 3, qz = q / 9;
    const unsigned long long in = IN.m[q];
    const int off = (DIM == 3 ? qz * BX * PL : 0) + qy * BX * EP + qx * BX;
    const int at_q = in == ~0ull || lane_in(in) ? cell0 + off : CS;
    if (W > 1 && q % W != wv) continue;
    v[q] = s_z[0][at_q];
#pragma unroll
    for (int j = 1; j < W; ++j) v[q] += s_z[j][at_q];
  }
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    const unsigned long long m = IN.m[q] & (((unsigned long long)(unsigned)lane_i32(qm.y, q) << 32) |
                                            (unsigned)lane_i32(qm.x, q));
    if ((W == 1 || q % W == wv) && lane_in(m)) out[lane_count_below(m, 0)] = v[q];
    out += __popcll(m);
  }
}

// z = cd w + nn E^T c, with E^T c of a node the sum of what its block's
// supertiles and its explicit rows stored (Pull, in the entries' order); lane
// = slot of a block, two blocks per wavefront.  The first bc.groups workgroups
// take the BC entries, which only explicit rows reach.  With DOT also the
// partials of (dy, z) and (z, z), one per workgroup.
struct BcPull {
  const int* et;          // [n_c] explicit target of a BC DOF, or -1
  int groups, n_s, n_c;
};
template <class TS, int DIM, bool DOT>
__global__ __launch_bounds__(256) void k_combine(BcPull bc, const QMeta* __restrict__ face,
                                                 const Pull* __restrict__ pull, int nb,
                                                 const double* __restrict__ buf,
                                                 const double* __restrict__ x, int64_t bufld,
                                                 int n_et, const TS* __restrict__ w,
                                                 TS* __restrict__ z, int64_t ld, int r0, double cd,
                                                 double nn, int xcd, DotOut<TS> dot, Skip skip) {
  constexpr int KB = kLapBlocksPerWave, NP = 1 << DIM;
  const int r = blockIdx.y;
  if (skipped(skip, r0 + r, 0)) return;
  w += (r0 + r) * ld;
  z += (r0 + r) * ld;
  buf += (int64_t)r * bufld;
  x += (int64_t)r * n_et;
  double d0 = 0.0, d1 = 0.0;
  int part = blockIdx.x;
  auto put = [&](int i, double wv, double e, double y) {
    const TS o = (TS)(cd * wv + nn * e);
    z[i] = o;
    if (DOT) {
      d0 += y * (double)o;
      d1 += (double)o * (double)o;
    }
  };
  if ((int)blockIdx.x < bc.groups) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < bc.n_c) {
      const int k = bc.et[i];
      put(bc.n_s + i, (double)w[bc.n_s + i], k >= 0 ? x[k] : 0.0,
          DOT ? (double)dot.y[bc.n_s + i] : 0.0);
    }
  } else {
    const int ng = gridDim.x - bc.groups, gb = blockIdx.x - bc.groups;
    const int wg = xcd ? xcd_remap(gb, ng) : gb;
    part = bc.groups + wg;
    const int blk0 = (wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * KB;
    const int lane = threadIdx.x & 63;
    // entry e of block j in lane 16 j + e: its supertiles' and explicit
    // targets' (0 .. NP - 1, 8), and the block's own mask and first DOF (15)
    const int jb = min(blk0 + min(lane >> 4, KB - 1), nb - 1), e = lane & 15;
    const int4 pm = e == 15 ? reinterpret_cast<const int4*>(face)[(int64_t)jb * 8]
                            : reinterpret_cast<const int4*>(pull)[(int64_t)jb * 9 + min(e, 8)];
    auto mask = [&](int j, int q) {
      return ((unsigned long long)(unsigned)lane_i32(pm.y, 16 * j + q) << 32) |
             (unsigned)lane_i32(pm.x, 16 * j + q);
    };
    auto from = [&](int j, int q) {
      return ((long long)lane_i32(pm.w, 16 * j + q) << 32) | (unsigned)lane_i32(pm.z, 16 * j + q);
    };
    // Loads for the longer of the blocks' lists of supertiles, two, four or
    // all 2^d long (the rest are empty): a wave is bound by its accesses to
    // memory.  Whole transpose, torus at h = 1/256: 398 us with 2^d always, 380.
    const unsigned long long some = __ballot(e < NP && (pm.x | pm.y) != 0);
    int longest = 0;
#pragma unroll
    for (int j = 0; j < KB; ++j) longest = max(longest, __popcll((some >> (16 * j)) & 0xffffull));
    auto take = [&](auto nq) {
      constexpr int NQ = nq();
      double s[KB][NQ + 1];
      TS wl[KB], yl[KB];
      int own[KB];
      // every load first (a lane without an entry loads its block's first)
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        own[j] = lane_i32(pm.z, 16 * j + 15) + (int)lane_rank(mask(j, 15));
        wl[j] = w[own[j]];
        if (DOT) yl[j] = dot.y[own[j]];
#pragma unroll
        for (int q = 0; q < NQ; ++q) s[j][q] = (buf + from(j, q))[lane_rank(mask(j, q))];
        s[j][NQ] = mask(j, 8) ? (x + from(j, 8))[lane_rank(mask(j, 8))] : 0.0;
      }
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        double ev = 0.0;
#pragma unroll
        for (int q = 0; q <= NQ; ++q) {
          asm volatile("" : "+v"(s[j][q]));   // the loads stay above
          ev += lane_in(mask(j, q < NQ ? q : 8)) ? s[j][q] : 0.0;
        }
        if (blk0 + j < nb && lane_in(mask(j, 15)))
          put(own[j], (double)wl[j], ev, DOT ? (double)yl[j] : 0.0);
      }
    };
    if (longest <= 2) take(std::integral_constant<int, 2>{});
    else if (DIM == 2 || longest <= 4) take(std::integral_constant<int, 4>{});
    else take(std::integral_constant<int, NP>{});
  }
  if constexpr (DOT) group_dot2(d0, d1, dot.part, dot.np, part);
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

// Right-hand sides that a workgroup of the forward apply takes in turn.
static int rhs_per_group(const cpm_band* b, int nrhs, const Skip& skip) {
  const int fill = skip.f ? kMaxRhsGroups : kFillSupertiles / std::max(1, b->nst);
  const int groups = std::max(1, std::min(nrhs, fill));
  return (nrhs + groups - 1) / groups;
}

template <class T, int DIM>
static void launch_gather(const cpm_band* b, int nrhs, const T* u, double* a, hipStream_t st,
                          int part, const Skip& skip) {
  const Tune& tn = tune_of<T>(b);
  const int ew = ERowPack<DIM>::padded(b->n_erows) / ERowPack<DIM>::kRows;
  ERows er{ew, (ew + 7) / 8 * 8, b->erow_id, b->ecol4, b->ew1, b->p, b->erow_inst};
  SuperView sv = sview(b);
  if (part == PART_MAIN) er.groups = 0;
  if (part == PART_EXPLICIT) sv.n = 0;
  const int per = rhs_per_group(b, nrhs, skip);
  const int waves = per > 1 || sv.n <= kSplitBelow ? 2 : 1;
  const int64_t g = (int64_t)er.groups / waves + sv.n;
  if (!g) return;
  auto multi = [&](auto pad, auto np) {
    auto kern = per > 1      ? k_gather<T, DIM, pad(), np(), 2, 2>
                : waves == 2 ? k_gather<T, DIM, pad(), np(), 2, 1>
                             : k_gather<T, DIM, pad(), np(), 1, 1>;
    hipLaunchKernelGGL(kern, dim3((unsigned)g, (nrhs + per - 1) / per), dim3(64 * waves), 0, st,
                       er, sv, b->st_meta, b->st_rng, u, a, b->n, nrhs, per, tn.xcd, skip);
  };
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
static int lap_row_groups(const cpm_band* b) {
  return (b->n_lrows + kLapThreads - 1) / kLapThreads;
}
static int bc_groups(const cpm_band* b) { return (int)((b->n_c + 255) / 256); }

// Number of partials a fused dot product of an apply writes (per value): one
// per workgroup of the kernel that writes the result.
int apply_dot_parts(const cpm_band* b, bool transpose) {
  if (transpose) return bc_groups(b) + lap_groups(b);
  return lap_row_groups(b) + lap_groups(b);
}

template <class TU, class TA, class TV, int DIM, bool ALL, bool DOT>
static void launch_lap(const cpm_band* b, const Tune& tn, hipStream_t st, const TU* u,
                       const TA* a, TV* v, int64_t ld, int nrhs, double cd, double co,
                       const double* gsum, double gscale, const double* coef, DotOut<TV> dot,
                       int part, const Skip& skip) {
  LRows lr{b->n_lrows, part == PART_MAIN ? 0 : ALL ? bc_groups(b) : lap_row_groups(b), 2 * DIM,
           b->lrow_id, b->lcol, b->lrow_inst};
  LPull lp{b->lt_pull, b->bc_lt, b->lt_start, b->lt_src, b->lrow_id, (int)b->n_s, (int)b->n_c};
  const int64_t g = (int64_t)lr.groups + (part == PART_EXPLICIT ? 0 : lap_groups(b));
  if (!g) return;
  // in a solver too: apart they read the blocks' masks each (203 against 196 ms)
  const int per = rhs_per_group(b, nrhs, Skip{});
  hipLaunchKernelGGL((k_lap<TU, TA, TV, DIM, ALL, DOT>), dim3((unsigned)g, (nrhs + per - 1) / per),
                     dim3(kLapThreads), 0, st, lr, lp, b->blk_face, b->nb, u, a, v, ld, nrhs, per, cd, co,
                     gsum, gscale, tn.xcd, coef, skip, dot);
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

// Right-hand sides of one transposed gather: its buffer takes CELLS entries a
// supertile each, so several share it only while it stays small (and their
// number is a grid dimension).
constexpr size_t kTransposeBufBytes = size_t(256) << 20;
constexpr size_t kMaxTransposeRhs = 32768;
static int transpose_rhs(const cpm_band* b, int nrhs) {
  const size_t one = sizeof(double) * (size_t)b->nst *
                     (b->dim == 3 ? Super<3>::CELLS : Super<2>::CELLS);
  const size_t k = one ? std::min(kTransposeBufBytes / one, kMaxTransposeRhs) : kMaxTransposeRhs;
  return (int)std::max<size_t>(1, std::min<size_t>(k, (size_t)nrhs));
}

// scratch: c = (L - diag L)^T w, the supertiles' sums, the explicit targets'
struct TransposeScratch {
  double *c, *buf, *x;
  int64_t bufld;
  int nr;                 // right-hand sides buf and x hold
};
static TransposeScratch transpose_scratch(const cpm_band* b, int nrhs) {
  TransposeScratch t;
  t.nr = transpose_rhs(b, nrhs);
  t.bufld = (int64_t)b->nst * (b->dim == 3 ? Super<3>::CELLS : Super<2>::CELLS);
  t.c = static_cast<double*>(band_scratch(b, 1, sizeof(double) * (size_t)b->n * nrhs));
  // at least one entry each: lanes without one load the first
  t.buf = static_cast<double*>(
      band_scratch(b, 2, sizeof(double) * ((size_t)t.bufld * t.nr + 1)));
  t.x = static_cast<double*>(
      band_scratch(b, 5, sizeof(double) * ((size_t)b->n_et * t.nr + 1)));
  return t;
}
void apply_transpose_scratch(const cpm_band* b, int nrhs) { transpose_scratch(b, nrhs); }

// The transposed apply in three launches (the last two once for every few
// right-hand sides).  c = (L - diag L)^T w and E^T c are FP64 for both storage
// precisions (the combine step cancels the two terms of size N^2, as the
// forward Laplacian pass does).
template <class T, int DIM>
static void apply_T_dim(const cpm_band* b, double m, double n, int nrhs, const T* w, T* z,
                        hipStream_t st, const T* dy, double* dpart, const Skip& skip) {
  if (!b->st_pull) CPM_FAIL(CPM_E_INVALID, "this band has no transpose schedule");
  const int64_t ld = b->n;
  const TransposeScratch t = transpose_scratch(b, nrhs);
  const double N2 = (double)b->N * (double)b->N;
  const double cd = m + n * (-2.0 * DIM * N2);
  const Tune& tn = tune_of<T>(b);
  launch_lap<T, T, double, DIM, true, false>(b, tn, st, w, w, t.c, ld, nrhs, 0.0, N2, nullptr, 0.0,
                                             nullptr, DotOut<double>{nullptr, nullptr, 0},
                                             PART_ALL, skip);
  constexpr int64_t EG = 8 * kEPullTargets;
  const EPull ep{b->n_et, (int)((b->n_et + EG - 1) / EG * 8), b->et_start, b->et_src, b->et_w};
  const BcPull bc{b->bc_et, bc_groups(b), (int)b->n_s, (int)b->n_c};
  for (int r = 0; r < nrhs; r += t.nr) {
    const int k = std::min(t.nr, nrhs - r);
    const int waves = (int64_t)b->nst * k <= kSplitBelow ? 2 : 1;
    const int64_t g = (int64_t)ep.groups / waves + b->nst;
    auto kern = waves == 2 ? k_gather_T<T, DIM, 2> : k_gather_T<T, DIM, 1>;
    if (g)
      hipLaunchKernelGGL(kern, dim3((unsigned)g, k), dim3(64 * waves), 0, st, ep, sview(b),
                         b->st_meta, b->st_rng, t.c, t.x, t.buf, ld, t.bufld, r, tn.xcd, skip);
    CPM_LAUNCH_CHECK();
    const dim3 gc((unsigned)(bc.groups + lap_groups(b)), k);
    if (dy)
      hipLaunchKernelGGL((k_combine<T, DIM, true>), gc, dim3(256), 0, st, bc, b->blk_face,
                         b->st_pull, b->nb, t.buf, t.x, t.bufld, b->n_et, w, z, ld, r, cd, n,
                         tn.xcd, DotOut<T>{dy, dpart, (int)gc.x}, skip);
    else
      hipLaunchKernelGGL((k_combine<T, DIM, false>), gc, dim3(256), 0, st, bc, b->blk_face,
                         b->st_pull, b->nb, t.buf, t.x, t.bufld, b->n_et, w, z, ld, r, cd, n,
                         tn.xcd, DotOut<T>{nullptr, nullptr, 0}, skip);
    CPM_LAUNCH_CHECK();
  }
}

template <class T>
void apply_transpose_impl(const cpm_band* b, double m, double n, int nrhs, const T* w, T* z,
                          hipStream_t st, const double*, double gamma, const T* dy,
                          double* dpart, Skip skip) {
  if (gamma != 0.0) CPM_FAIL(CPM_E_INVALID, "the gauge is not supported for the transpose");
  if (dy && nrhs != 1) CPM_FAIL(CPM_E_INVALID, "internal: fused dots take one right-hand side");
  if (b->dim == 3) apply_T_dim<T, 3>(b, m, n, nrhs, w, z, st, dy, dpart, skip);
  else apply_T_dim<T, 2>(b, m, n, nrhs, w, z, st, dy, dpart, skip);
}

template void apply_impl<double>(const cpm_band*, double, double, int, const double*, double*,
                                 hipStream_t, const double*, double, const double*, double*, Skip);
template void apply_impl<float>(const cpm_band*, double, double, int, const float*, float*,
                                hipStream_t, const double*, double, const float*, double*, Skip);
template void apply_transpose_impl<double>(const cpm_band*, double, double, int, const double*,
                                           double*, hipStream_t, const double*, double,
                                           const double*, double*, Skip);
template void apply_transpose_impl<float>(const cpm_band*, double, double, int, const float*,
                                          float*, hipStream_t, const double*, double,
                                          const float*, double*, Skip);

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
        if (((k >> 1) & 3) >= 2 && b->composite) {   // a batch reports mode 1 only
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
