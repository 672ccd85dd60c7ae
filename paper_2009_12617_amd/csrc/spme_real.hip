// Real-space part of the Ewald electrostatics on gfx950: the erfc-screened
// pair sum within a cutoff, the self term and the exclusion correction --
// the short-range work that the paper's system runs beside the long-range
// pipeline (§II, §V.A), so that reciprocal + real + self + exclusions give
// the full Ewald energy and forces.
//
// One evaluation is three launches on one stream for small systems, five for
// larger ones (six past kRsTable sub-cells), over a cell grid of at least
// three cells of edge >= rcut per axis:
//   k_rs_sort    (small) atoms into (cell, slab in x) order through the LDS of
//                one workgroup; the self and exclusion terms in the others
//   k_rs_zero    (larger) clear the sub-cell counts
//   k_rs_count   atoms per sub-cell, each atom's rank, self and exclusion terms
//   k_rs_scan    prefix sum of the counts, where k_rs_fill does not do it
//   k_rs_fill    atoms into (cell, slab) order
//                (whichever of the three has the sums also lists the groups of
//                home atoms of the pair workgroups)
//   k_rs_pairs   the pair sum, forces to the caller's order
//   k_rs_reduce  energies from the per-workgroup rows, in a fixed order
// Arithmetic is FP64 throughout, but for tests that may only let too many
// candidates through.  The order of atoms inside a cell and of the force
// additions depends on atomic ordering, so forces are reproducible to FP64
// rounding, not bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "spme_device.h"
#include "spme_internal.h"
#include "../../include/spme.h"

namespace spme {
namespace {

constexpr int kRsGroup = 16;     // home atoms of a wavefront (the columns of a 16x16 tile)
constexpr int kRsWaves = 4;      // wavefronts of a pair workgroup
constexpr int kRsThreads = 64 * kRsWaves;
constexpr int kRsHome = kRsGroup * kRsWaves;  // most home atoms of a workgroup
constexpr int kRsList = 2048;    // candidates listed at a time
constexpr int kRsPer = 4;        // ... that each thread looks at in one go
constexpr int kRsIdxBits = 27;   // record of a listed candidate; its segment above it
constexpr int kRsSegs = 27;      // runs of neighbour atoms: 9 rows of cells, 3 periodic images in x
static_assert(kRsSegs <= (1 << (32 - kRsIdxBits)), "a segment fits above the record index");
constexpr int kRsCountThreads = 512;
constexpr int kRsCheb = 32;         // Chebyshev terms of exp(x^2) erfc(x)
constexpr int kRsChebShort = 24;    // terms enough for beta rcut <= kRsShortRange
constexpr double kRsShortRange = 3.2;  // 24 terms: <= 1.3e-14 relative up to here
constexpr double kRsMaxBetaRcut = 6.0;  // series error <= 2e-14 relative up to here
constexpr int kRsScanThreads = 1024, kRsSortThreads = 1024;
constexpr int kRsTable = 8192;      // sub-cell counts one workgroup scans in LDS
constexpr int kRsSortTable = 2048, kRsSmall = 8 * kRsSortThreads;  // sub-cells and atoms one workgroup sorts
// Atoms are ordered by cell (x fastest) and, inside a cell, by slab in x, so
// that consecutive atoms of a row of cells lie close together (the box of a
// workgroup's home atoms, which bounds their candidates, is then small).
constexpr int kRsSlabs = 8;
constexpr float kRsFar = 1e30f;  // (of lengths in units of the box: RsArgs::unit_len)

struct RsArgs {
  int N, nc[3], ncell, n_count_blocks;
  int nrow;             // pair workgroups launched: at least as many as there are groups
  double L[3], invL[3], cell_inv[3];
  double beta, rc2, rcut, coulomb;
  double poly[kRsCheb];  // exp(x^2) erfc(x), x = beta r, as a polynomial in t = 2 r / rcut - 1
  int ncheb;             // terms the pair kernel uses: kRsChebShort or kRsCheb
  double two_over_rcut, exp_scale;  // 2 / rcut, -32 beta^2 / ln 2
  int split;             // wavefronts of a pair workgroup
  int unit, nunit;       // cells of a home unit, units
  int max_span;          // most cells a group may reach past its first one
  // The FP32 tests take lengths times unit_len, the power of two that brings
  // half the box diagonal + rcut into [1, 2): their squares neither overflow
  // nor vanish whatever the unit of length, and no rounding is added.
  double unit_len, len_unit;  // ... and its inverse
  float list_lim;        // listing: rcut^2 and the margin of the whole box
  double slack;          // most that FP32 moves a coordinate relative to the box centre
  const double* pos;
  const double* q;
  const int* excl_off;  // may be null
  const int* excl_idx;
  double* forces;
  int accumulate;
  double* energies;
  // workspace
  unsigned* count;      // [ncell * kRsSlabs]: per (cell, slab)
  unsigned* start;      // [ncell * kRsSlabs + 1]
  unsigned* rank;       // [N] place of each atom within its sub-cell
  double4* rec;         // [N] wrapped position and charge, in cell order
  float4* rec32;        // [N] position relative to the box centre (times unit_len) in FP32 and its square
  int* ridx;            // [N] original index, in cell order
  int4* groups;         // [nrow] first and last + 1 home atom, unit, of each pair workgroup
  int* ngroup;          // groups, rounded up to a multiple of kXcds
  double* rows;         // [nrow] pair energies; [n_count_blocks] q^2 sums; [n_count_blocks] exclusions
};

__device__ __forceinline__ double wrap(double x, double L, double invL) {
  double s = x - L * floor(x * invL);
  if (s >= L) s -= L;  // rounding at the upper edge
  if (s < 0.0) s = 0.0;
  return s;
}

__device__ __forceinline__ int cell_of(const RsArgs& a, double x, double y, double z) {
  // (cell, slab): cell index times kRsSlabs plus the slab in x
  int c[3];
  const double w[3] = {x, y, z};
  int o = 0;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double u = w[d] * a.cell_inv[d];
    c[d] = (int)u;
    if (c[d] >= a.nc[d]) c[d] = a.nc[d] - 1;
    if (c[d] < 0) c[d] = 0;
    if (d == 0) o = min(max((int)((u - c[0]) * kRsSlabs), 0), kRsSlabs - 1);
  }
  return ((c[2] * a.nc[1] + c[1]) * a.nc[0] + c[0]) * kRsSlabs + o;
}

// Adds n to counter[c] once per distinct c among the lanes of the
// wavefront (lanes with c < 0 take no part) and returns each lane's slot:
// the counter's old value plus the number of lanes of the same c below it.
// Neighbouring atoms (the atoms of a molecule) usually share a cell, so this
// issues a fraction of the per-atom atomics on the contended counters.  The
// groups of equal c are found first (ballots only); then every group's
// first lane issues its atomic at once, so the wavefront waits for one
// atomic round trip, not one per group.
__device__ __forceinline__ unsigned wave_add(unsigned* counter, int c) {
  const int lane = threadIdx.x & 63;
  unsigned long long todo = __ballot(c >= 0);
  int leader = lane;  // first lane of this lane's group
  unsigned n = 0u, below = 0u;
  while (todo != 0ull) {  // uniform over the wavefront
    const int first = __ffsll((long long)todo) - 1;
    const int cl = __builtin_amdgcn_readlane(c, first);  // first is uniform
    const unsigned long long same = __ballot(c == cl) & todo;
    if (c == cl) {
      leader = first;
      below = __builtin_amdgcn_mbcnt_hi((unsigned)(same >> 32),
                                        __builtin_amdgcn_mbcnt_lo((unsigned)same, 0u));
    }
    if (lane == first) n = (unsigned)__popcll(same);
    todo &= ~same;
  }
  unsigned base = 0u;
  if (c >= 0 && lane == leader) base = atomicAdd(&counter[c], n);
  return __shfl(base, leader, 64) + below;
}

// Exclusive prefix sums, in place, of a table of M counts in LDS by a
// workgroup of NT threads; the sum goes to entry M.
template <int NT, int M>
__device__ __forceinline__ void table_scan(unsigned* table, unsigned* wsum) {
  constexpr int PER = M / NT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  unsigned v[PER], sum = 0u;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const unsigned c = table[tid * PER + i];
    v[i] = sum;
    sum += c;
  }
  unsigned inc = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned o = __shfl_up(inc, d, 64);
    if (lane >= d) inc += o;
  }
  if (lane == 63) wsum[wave] = inc;
  __syncthreads();
  unsigned before = inc - sum;
  for (int w = 0; w < wave; ++w) before += wsum[w];
#pragma unroll
  for (int i = 0; i < PER; ++i) table[tid * PER + i] = before + v[i];
  if (tid == NT - 1) table[M] = before + sum;
  __syncthreads();
}

// One atom into its place in cell order.
__device__ __forceinline__ void place(const RsArgs& a, int i, unsigned slot, const double* w, double qi) {
  a.rec[slot] = make_double4(w[0], w[1], w[2], qi);
  const float x = (float)((w[0] - 0.5 * a.L[0]) * a.unit_len), y = (float)((w[1] - 0.5 * a.L[1]) * a.unit_len),
              z = (float)((w[2] - 0.5 * a.L[2]) * a.unit_len);
  const float sq = x * x + y * y + z * z;
  // (a non-finite position is never within the cutoff of anything)
  a.rec32[slot] = sq < kRsFar ? make_float4(x, y, z, sq) : make_float4(0.f, 0.f, 0.f, kRsFar);
  a.ridx[slot] = i;
}

// Wraps a position into the box and returns its (cell, slab).
__device__ __forceinline__ int wrapped_cell(const RsArgs& a, double* w) {
#pragma unroll
  for (int d = 0; d < 3; ++d) w[d] = wrap(w[d], a.L[d], a.invL[d]);
  return cell_of(a, w[0], w[1], w[2]);
}

// Self and exclusion terms of the atoms of workgroup `blk` of
// ceil(N / blockDim.x): sum q^2 and, with exclusion lists, each atom's
// excluded partners -- the force of removing them goes to the caller's array
// (which the pair kernel then adds to), the energy to the workgroup's row.
__device__ __forceinline__ void self_and_excluded(const RsArgs& a, int blk, double* wred) {
  const int i = blk * blockDim.x + threadIdx.x;
  double v[2] = {0.0, 0.0};
  if (i < a.N) {
    const double qi = a.q[i];
    v[0] = qi * qi;
    if (a.excl_off != nullptr) {
      // removed: the erfc/r the pair sum takes (inside the cutoff) and the
      // erf/r the reciprocal sum carries
      const double two_over_sqrtpi = 1.12837916709551257390;
      double p[3], f[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int d = 0; d < 3; ++d) p[d] = a.pos[3 * (size_t)i + d];
      const int k1 = a.excl_off[i + 1];
      for (int k = a.excl_off[i]; k < k1; ++k) {
        const int j = a.excl_idx[k];
        double d[3];
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          d[t] = p[t] - a.pos[3 * (size_t)j + t];
          d[t] -= a.L[t] * rint(d[t] * a.invL[t]);
        }
        const double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
        const double r = sqrt(r2);
        const double qq = a.coulomb * qi * a.q[j];
        double u, du;
        if (r2 <= a.rc2) {
          u = 1.0 / r;
          du = -1.0 / r2;
        } else {
          const double ef = erf(a.beta * r);
          u = ef / r;
          du = (two_over_sqrtpi * a.beta * exp(-a.beta * a.beta * r2) - ef / r) / r;
        }
        v[1] -= 0.5 * qq * u;
        const double g = qq * du / r;
#pragma unroll
        for (int t = 0; t < 3; ++t) f[t] = fma(g, d[t], f[t]);
      }
      double* out = a.forces + 3 * (size_t)i;
#pragma unroll
      for (int t = 0; t < 3; ++t) out[t] = a.accumulate ? out[t] + f[t] : f[t];
    }
  }
  block_sums<2>(v, wred);
  if (threadIdx.x == 15) {
    a.rows[(size_t)a.nrow + blk] = v[0];
    a.rows[(size_t)a.nrow + a.n_count_blocks + blk] = v[1];
  }
}

// Workgroups are dispatched round-robin over the XCDs, each with its own L2.
constexpr int kXcds = 8;

// The home atoms of the pair workgroups, listed by a workgroup of NT threads:
// each unit's atoms in groups of equal size, at most kRsHome / split.  From
// the counts themselves, so that a box with dense and empty parts fills the
// chip as a uniform one does (a fixed number of workgroups per unit, from the
// mean density, took the groups of dense units one after the other: 65,535
// atoms in a slab across a tenth of its box 646 us, now 180; a uniform box 146,
// now 143).  XCD x takes a contiguous eighth of the groups.  start(u): first
// atom of unit u.
template <int NT, class Start>
__device__ __forceinline__ void list_groups(const RsArgs& a, Start&& start, unsigned* wsum) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int most = kRsHome / a.split;
  auto groups_of = [&](int u) { return u < a.nunit ? ((int)(start(u + 1) - start(u)) + most - 1) / most : 0; };
  auto put = [&](int i, int per, int4 g) { a.groups[i % per * kXcds + i / per] = g; };
  // the n groups of unit u, from the i-th on
  auto put_unit = [&](int u, int n, int i, int per) {
    if (n == 0) return;
    const int u0 = (int)start(u), u1 = (int)start(u + 1), gs = (u1 - u0 + n - 1) / n;
    for (int k = 0; k < n; ++k) put(i + k, per, make_int4(u0 + k * gs, min(u0 + (k + 1) * gs, u1), u, 0));
  };
  auto put_rest = [&](int total, int per, int first, int step) {
    for (int i = total + first; i < per * kXcds; i += step) put(i, per, make_int4(0, 0, 0, 0));
    if (first == 0) *a.ngroup = per * kXcds;
  };
  if (a.nunit <= 64) {  // one wavefront, without a barrier (small systems: a microsecond of the sort)
    if (wave != NT / 64 - 1) return;
    const int n = groups_of(lane), inc = wave_scan_add(n);
    const int total = __builtin_amdgcn_readlane(inc, 63), per = (total + kXcds - 1) / kXcds;
    put_unit(lane, n, inc - n, per);
    put_rest(total, per, lane, 64);
    return;
  }
  int mine = 0;
  for (int u = tid; u < a.nunit; u += NT) mine += groups_of(u);
  mine = wave_scan_add(mine);
  if (lane == 63) wsum[wave] = (unsigned)mine;
  __syncthreads();
  int total = 0;
  for (int w = 0; w < NT / 64; ++w) total += (int)wsum[w];
  const int per = (total + kXcds - 1) / kXcds;
  int carry = 0;
  for (int b = 0; b < a.nunit; b += NT) {
    const int u = b + tid, n = groups_of(u), inc = wave_scan_add(n);
    __syncthreads();  // the previous sums are read
    if (lane == 63) wsum[wave] = (unsigned)inc;
    __syncthreads();
    int i = carry + inc - n;
    for (int w = 0; w < NT / 64; ++w) {
      if (w < wave) i += (int)wsum[w];
      carry += (int)wsum[w];
    }
    put_unit(u, n, i, per);
  }
  put_rest(total, per, tid, NT);
}

// Small systems (at most PER atoms per thread and kRsSortTable sub-cells): workgroup 0
// counts, scans and places every atom through LDS; the others do the self and
// exclusion terms.  One launch in place of four.
template <int PER>
__global__ __launch_bounds__(kRsSortThreads) void k_rs_sort(RsArgs a) {
  __shared__ unsigned table[kRsSortTable + 1];
  __shared__ unsigned wsum[kRsSortThreads / 64];
  __shared__ double wred[16 * 8];
  if (blockIdx.x > 0) {
    self_and_excluded(a, blockIdx.x - 1, wred);
    return;
  }
  const int tid = threadIdx.x;
  for (int c = tid; c < kRsSortTable; c += kRsSortThreads) table[c] = 0u;
  __syncthreads();
  // (loads of absent atoms repeat the last one, so that none waits for a branch)
  double w[PER][3], qi[PER];
  int cell[PER];
  unsigned rank[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = min(k * kRsSortThreads + tid, a.N - 1);
#pragma unroll
    for (int d = 0; d < 3; ++d) w[k][d] = a.pos[3 * (size_t)i + d];
    qi[k] = a.q[i];
  }
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    cell[k] = wrapped_cell(a, w[k]);
    if (k * kRsSortThreads + tid < a.N) rank[k] = atomicAdd(&table[cell[k]], 1u);
  }
  __syncthreads();
  table_scan<kRsSortThreads, kRsSortTable>(table, wsum);
  const int nsub = a.ncell * kRsSlabs;
  for (int c = tid; c <= nsub; c += kRsSortThreads) a.start[c] = table[c];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int i = k * kRsSortThreads + tid;
    if (i < a.N) place(a, i, table[cell[k]] + rank[k], w[k], qi[k]);
  }
  list_groups<kRsSortThreads>(a, [&](int u) { return table[u * a.unit * kRsSlabs]; }, wsum);
}

__global__ __launch_bounds__(256) void k_rs_zero(RsArgs a) {
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < a.ncell * kRsSlabs; c += gridDim.x * blockDim.x)
    a.count[c] = 0u;
}

// Counts the atoms of each sub-cell, keeps each atom's rank in its own (so
// that k_rs_fill needs no atomics), and the self and exclusion terms.
__global__ __launch_bounds__(kRsCountThreads) void k_rs_count(RsArgs a) {
  __shared__ double wred[16 * 8];
  const int i = blockIdx.x * kRsCountThreads + threadIdx.x;
  int c = -1;
  if (i < a.N) {
    double w[3] = {a.pos[3 * (size_t)i], a.pos[3 * (size_t)i + 1], a.pos[3 * (size_t)i + 2]};
    c = wrapped_cell(a, w);
  }
  const unsigned r = wave_add(a.count, c);
  if (c >= 0) a.rank[i] = r;
  self_and_excluded(a, blockIdx.x, wred);
}

// Exclusive prefix sum of more than kRsTable counts by one workgroup, and the
// groups of the pair kernel.
__global__ __launch_bounds__(kRsScanThreads) void k_rs_scan(RsArgs a) {
  __shared__ unsigned table[kRsTable + 1];
  __shared__ unsigned wsum[kRsScanThreads / 64];
  const int tid = threadIdx.x;
  const int nsub = a.ncell * kRsSlabs;
  unsigned carry = 0u;
  for (int s0 = 0; s0 < nsub; s0 += kRsTable) {
    for (int c = tid; c < kRsTable; c += kRsScanThreads) table[c] = s0 + c < nsub ? a.count[s0 + c] : 0u;
    __syncthreads();
    table_scan<kRsScanThreads, kRsTable>(table, wsum);
    for (int c = tid; c < kRsTable && s0 + c < nsub; c += kRsScanThreads) a.start[s0 + c] = carry + table[c];
    carry += table[kRsTable];
    __syncthreads();
  }
  if (tid == 0) a.start[nsub] = carry;
  __syncthreads();  // (the starts this workgroup wrote)
  list_groups<kRsScanThreads>(a, [&](int u) { return a.start[(size_t)u * a.unit * kRsSlabs]; }, wsum);
}

// Atoms into cell order.  SCAN: at most kRsTable sub-cells, whose counts each
// workgroup scans itself (a few microseconds less than a launch of its own);
// one more, the first, writes the starts and the groups for the pair kernel.
template <bool SCAN>
__global__ __launch_bounds__(kRsCountThreads) void k_rs_fill(RsArgs a) {
  const int tid = threadIdx.x, blk = SCAN ? (int)blockIdx.x - 1 : (int)blockIdx.x;
  const int i = blk < 0 ? a.N : blk * kRsCountThreads + tid;
  double w[3] = {0.0, 0.0, 0.0}, qi = 0.0;
  int c = 0;
  unsigned r = 0u;
  if (i < a.N) {
#pragma unroll
    for (int d = 0; d < 3; ++d) w[d] = a.pos[3 * (size_t)i + d];
    qi = a.q[i];
    r = a.rank[i];
    c = wrapped_cell(a, w);
  }
  if constexpr (SCAN) {
    __shared__ unsigned table[kRsTable + 1];
    __shared__ unsigned wsum[kRsCountThreads / 64];
    const int nsub = a.ncell * kRsSlabs;
    for (int k = tid; k < kRsTable; k += kRsCountThreads) table[k] = k < nsub ? a.count[k] : 0u;
    __syncthreads();
    table_scan<kRsCountThreads, kRsTable>(table, wsum);
    if (blk < 0) {
      for (int k = tid; k <= nsub; k += kRsCountThreads) a.start[k] = table[k];
      list_groups<kRsCountThreads>(a, [&](int u) { return table[u * a.unit * kRsSlabs]; }, wsum);
      return;
    }
    if (i < a.N) place(a, i, table[c] + r, w, qi);
  } else {
    if (i < a.N) place(a, i, a.start[c] + r, w, qi);
  }
}

// 2^(y/32) for y in [-2000, 0]: y = 32 n + j + r with |r| <= 1/2, 2^(r/32) by
// its Taylor series to r^6 (remainder below 4e-18), 2^(j/32) from the
// workgroup's table.
constexpr int kRsExp = 32;
__device__ __forceinline__ double rs_exp2(double y, const double* two_to) {
  constexpr double c = 0.69314718055994530942 / kRsExp;
  const double n = rint(y), r = y - n;
  const int i = (int)n;
  const double scale = two_to[i & (kRsExp - 1)];
  double p = fma(r, c * c * c * c * c * c / 720.0, c * c * c * c * c / 120.0);
  p = fma(p, r, c * c * c * c / 24.0);
  p = fma(p, r, c * c * c / 6.0);
  p = fma(p, r, c * c / 2.0);
  p = fma(p, r, c);
  return ldexp(fma(p * r, scale, scale), i >> 5);
}

// Constants of rs_pair kept in vector registers (the polynomial takes most
// of the scalar ones).
struct RsConst {
  double exp_scale, two_over_rcut, dbeta;  // -32 beta^2 / ln 2, 2 / rcut, 2 beta / sqrt(pi)
};

// One ordered pair: adds the energy of home atom ri with candidate rj (twice
// its share) to e and the force on the home atom to f, if the pair lies
// inside the cutoff in FP64 (ok: the lane has a candidate).  erfc(x) =
// exp(-x^2) erfcx(x) with erfcx = exp(x^2) erfc(x) a polynomial of NC terms
// in t = 2 r / rcut - 1 (Horner's rule; the coefficients, uniform over the
// launch, sum to about 1 in absolute value, so that it is as accurate as
// Clenshaw's recurrence on the Chebyshev form with half its operations),
// 1/r from the hardware reciprocal square root and one third-order step.
template <int NC>
__device__ __forceinline__ void rs_pair(const RsArgs& a, const RsConst& k, const double4& ri, const double4& rj,
                                        const double* two_to, bool ok, double& e, double* f) {
  const double d[3] = {ri.x - rj.x, ri.y - rj.y, ri.z - rj.z};
  double r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2];
  // (the home atom's own record, and an atom on the same position, lie at
  // distance exactly 0 and add nothing)
  const bool in = ok && r2 <= a.rc2 && r2 > 0.0;
  const double qq = in ? ri.w * rj.w : 0.0;
  r2 = in ? r2 : a.rc2;  // (keeps every factor of qq = 0 finite)
  double rinv = __builtin_amdgcn_rsq(r2);
  const double u = fma(-(r2 * rinv), rinv, 1.0);
  rinv = fma(fma(u, 0.375, 0.5), u * rinv, rinv);
  const double ex = rs_exp2(k.exp_scale * r2, two_to);
  const double t = fma(r2 * rinv, k.two_over_rcut, -1.0);
  double p = a.poly[NC - 1];
#pragma unroll
  for (int k = NC - 2; k >= 0; --k) p = fma(p, t, a.poly[k]);
  const double ec = ex * p * rinv;  // erfc(beta r) / r
  e = fma(qq, ec, e);
  const double g = qq * fma(k.dbeta, ex, ec) * (rinv * rinv);
#pragma unroll
  for (int c = 0; c < 3; ++c) f[c] = fma(g, d[c], f[c]);
}

using f32x4 = __attribute__((__vector_size__(4 * sizeof(float)))) float;

// At most 64 / S home atoms, consecutive records of a row of cells (or of a
// cell), by four wavefronts; S wavefronts share a group of 16 (NC: terms of
// the polynomial).  Lane (g, col) of a wavefront works for home atom col of
// its group.
//
// Candidates: the atoms of the 9 rows of cells around the home atoms', from
// one cell before to one cell after them in x, are at most 27 runs of
// consecutive records (segments), each with its periodic shift.  Those within
// the cutoff of the home atoms' box are listed, then staged in LDS pass by
// pass: each is read about 80 times at random, which the vector cache serves
// one line a cycle (128 cycles for the two halves of 64 records).
//
// Distance tests: a tile of 16 candidates by the 16 home atoms in one FP32
// matrix instruction,
//   |j|^2 - 2 i.j + (|i|^2 - rcut^2 - margin),
// relative to the centre of the home atoms' box.  A negative value may be a
// pair, which the pair evaluation decides in FP64.  Every candidate that may
// be one lies within ext of the centre (ext: half the box's diagonal + rcut,
// and slack for the rounding of the box itself) and every home atom closer, so
// rounding moves the sum by less than 44 2^-24 ext^2 = 2.7e-6 ext^2; the margin
// is 4e-6 ext^2, so no pair is missed.  Lane (g, col) receives rows 4g .. 4g+3 of a tile and
// shifts their sign bits into a mask word; a word covers 8 tiles.
//
// Pair evaluation: each lane walks its own hits, the next candidate being
// loaded while one is evaluated; forces stay in registers.  The fullest of
// the 64 lanes sets the time, so the candidates of a pass, of a wavefront and
// of a mask word are every n-th of the (spatially ordered) list, which keeps
// the lanes' counts close: 97 evaluations for 76 on average in liquid water
// at a 9 A cutoff.  (Dealing an atom's hits out evenly to its four lanes takes
// 84, and as much again to find each lane's share.)
//
// What bounds it: FP64 issue, about 65 of the 80 instructions of an evaluation;
// 65,535 atoms at 9 A: 223 -> 141 us by the profiler, of which the instructions
// take 75 at full rate and the listing and staging of candidates most of the
// rest.  Measured and not taken, us per evaluation of the whole term where this
// form took 149 (143 now, with the groups listed from the counts): records read
// from the vector cache, 165; one wavefront per workgroup and group, 208; each
// pair once with the candidates' forces summed in LDS, 175 (64-bit LDS atomics,
// and half-neighbourhoods differ too much between lanes).
//
// Stage slot 32 w + p of column c (p = 4b + r) holds the candidate of word
// w's tile b, row 4c + r: bit p (from the top) of lane (c, col)'s word w.

// Candidates in LDS at a time: three workgroups share a CU's LDS where there
// are many (S = 1); fewer and fuller passes where a workgroup has few atoms.
constexpr int rs_stage(int S) { return S == 1 ? 768 : 1024; }

template <int NC, int S>
__global__ __launch_bounds__(kRsThreads, S == 1 ? 3 : 2) void k_rs_pairs(RsArgs a) {
  constexpr int kStage = rs_stage(S), kWords = kStage / (128 * S);
  // x, y, z (with the periodic shift), |position - centre|^2 and charge, in
  // arrays of their own: a record's 32 bytes would meet 8 bank groups, these
  // 8-byte reads meet 32 (43 conflict cycles a read against 3, by the counters)
  constexpr int kPlane = (kStage + 16 * S + 31) / 32 * 32 + 16;  // (consecutive planes start half the banks apart)
  __shared__ double stage[5][kPlane];
  __shared__ unsigned list[kRsList];    // record | segment << kRsIdxBits
  __shared__ unsigned masks_all[kRsWaves][kWords + 2][64];  // two words of zeros at the end
  __shared__ double seg_shift[kRsSegs][3];
  __shared__ float seg_unit[kRsSegs][3];  // the same times unit_len
  __shared__ int seg_start[kRsSegs], seg_pre[32];  // (seg_pre: the segments' first items, then INT_MAX)
  __shared__ double two_to[kRsExp];
  __shared__ double home_f[S > 1 ? kRsHome / S : 1][3];
  __shared__ double home_e[kRsWaves];
  __shared__ float hbox[6];  // home atoms' box, relative to the box centre: low x y z, high x y z
  __shared__ int listed, nitem;
  const int id = blockIdx.x;
  const int4 group = a.groups[id];  // (of a workgroup past the last group: not written)
  if (id >= *a.ngroup || group.x >= group.y) {
    if (threadIdx.x == 0) a.rows[id] = 0.0;
    return;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int spl = wave % S;
  unsigned(*masks)[64] = masks_all[wave];
  const int cell0 = __builtin_amdgcn_readfirstlane(group.z) * a.unit;  // the unit's first cell
  const int gend = __builtin_amdgcn_readfirstlane(group.y);
  const int cx0 = cell0 % a.nc[0], cy = (cell0 / a.nc[0]) % a.nc[1], cz = cell0 / (a.nc[0] * a.nc[1]);
  const int col = lane & 15, g4 = lane >> 4;
  if (tid >= 64 && tid < 64 + kRsExp) two_to[tid - 64] = exp2((tid - 64) * (1.0 / kRsExp));
  RsConst kc = {a.exp_scale, a.two_over_rcut, 1.12837916709551257390 * a.beta};
  __asm__ __volatile__("" : "+v"(kc.exp_scale), "+v"(kc.two_over_rcut), "+v"(kc.dbeta));
  double e_pair = 0.0;

  // (a group whose atoms span more cells than may share their neighbours is
  // taken in several parts, `first` to `last`)
  for (int first = __builtin_amdgcn_readfirstlane(group.x); first < gend;) {
    // cells (within the unit) of the first atom and of the last one allowed
    int ca = 0, cb = 0;
    for (int i0 = 0; i0 < a.unit; i0 += 64) {
      const int i = i0 + lane;
      const int st = i < a.unit ? (int)a.start[(cell0 + i) * kRsSlabs] : 0x7fffffff;
      ca += __popcll(__ballot(st <= first));
      cb += __popcll(__ballot(st < gend));
    }
    --ca;
    --cb;
    int last = gend;
    if (cb - ca > a.max_span) {
      cb = ca + a.max_span;
      last = __builtin_amdgcn_readfirstlane((int)a.start[(cell0 + cb + 1) * kRsSlabs]);
    }
    const int ng = last - first;
    __syncthreads();  // the previous part is done with the tables
    if (wave == 0) {
      // lane j < 27: image x = j mod 3 of row j / 3
      int n = 0;
      if (lane < kRsSegs) {
        const int rw = lane / 3, im = lane - 3 * rw - 1;
        int y = cy + rw % 3 - 1, z = cz + rw / 3 - 1;
        double sy = 0.0, sz = 0.0;
        if (y < 0) y += a.nc[1], sy = -a.L[1];
        if (y >= a.nc[1]) y -= a.nc[1], sy = a.L[1];
        if (z < 0) z += a.nc[2], sz = -a.L[2];
        if (z >= a.nc[2]) z -= a.nc[2], sz = a.L[2];
        // cells xa .. xb of image im (at least three cells per axis and at
        // most nc[0] cells in all: each neighbour appears once)
        const int xa = max(cx0 + ca - 1, im * a.nc[0]) - im * a.nc[0];
        const int xb = min(cx0 + cb + 1, (im + 1) * a.nc[0] - 1) - im * a.nc[0];
        int r0 = 0;
        if (xa <= xb) {
          const int row = (z * a.nc[1] + y) * a.nc[0];
          r0 = (int)a.start[(row + xa) * kRsSlabs];
          n = (int)a.start[(row + xb + 1) * kRsSlabs] - r0;
        }
        seg_start[lane] = r0;
        seg_shift[lane][0] = im * a.L[0];
        seg_shift[lane][1] = sy;
        seg_shift[lane][2] = sz;
        seg_unit[lane][0] = (float)(im * a.L[0] * a.unit_len);
        seg_unit[lane][1] = (float)(sy * a.unit_len);
        seg_unit[lane][2] = (float)(sz * a.unit_len);
      }
      int inc = n;
#pragma unroll
      for (int d = 1; d < 32; d <<= 1) {
        const int o = __shfl_up(inc, d);
        if (lane >= d) inc += o;
      }
      if (lane < 32) seg_pre[lane] = lane < kRsSegs ? inc - n : 0x7fffffff;
      if (lane == kRsSegs - 1) nitem = inc;
    } else if (wave == 1) {
      // the home atoms' box (ng <= 64)
      const float4 h = a.rec32[first + min(lane, ng - 1)];
      const bool in = h.w < kRsFar;
      float bx[6] = {in ? h.x : kRsFar, in ? h.y : kRsFar, in ? h.z : kRsFar,
                     in ? h.x : -kRsFar, in ? h.y : -kRsFar, in ? h.z : -kRsFar};
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          bx[c] = fminf(bx[c], __shfl_xor(bx[c], d));
          bx[3 + c] = fmaxf(bx[3 + c], __shfl_xor(bx[3 + c], d));
        }
      }
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < 6; ++c) hbox[c] = bx[c];
      }
    } else if (S > 1 && tid >= 128 && tid < 128 + kRsHome / S) {
      home_f[tid - 128][0] = home_f[tid - 128][1] = home_f[tid - 128][2] = 0.0;
    }
    // this wavefront's home atoms (ng shared evenly by the wavefronts it needs)
    const int nwave = (ng + kRsGroup - 1) / kRsGroup, per = (ng + nwave - 1) / nwave;
    const int h0 = wave / S * per, nh = min(per, ng - h0);  // nh <= 0: none
    const int own = first + min(h0 + min(col, max(nh, 1) - 1), ng - 1);
    double4 ri = a.rec[own];
    ri.w *= a.coulomb;
    const bool active = col < nh && a.rec32[own].w < kRsFar;
    __syncthreads();
    const int total = nitem;
    auto centre = [&](int d) { return 0.5 * a.L[d] + 0.5 * (hbox[d] + hbox[3 + d]) * a.len_unit; };
    // the matrix instruction's column (-2 i, 1) and |i|^2 - rcut^2 - margin,
    // lengths times unit_len
    float bcol, q;
    {
      const float x = (float)((ri.x - centre(0)) * a.unit_len), y = (float)((ri.y - centre(1)) * a.unit_len),
                  z = (float)((ri.z - centre(2)) * a.unit_len);
      const float v = g4 == 0 ? x : g4 == 1 ? y : z;
      const double w[3] = {(double)hbox[3] - hbox[0], (double)hbox[4] - hbox[1], (double)hbox[5] - hbox[2]};
      const double rc = a.rcut * a.unit_len;
      const double ext = 0.5 * sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]) + rc + a.slack;
      bcol = g4 == 3 ? 1.f : active ? -2.f * v : 0.f;
      q = active ? (float)((double)x * x + (double)y * y + (double)z * z - rc * rc - 4e-6 * ext * ext) : kRsFar;
    }
    double f[3] = {0.0, 0.0, 0.0};
    for (int s0 = 0; s0 < total;) {
      // --- list the candidates within the cutoff of the home atoms' box (a
      // lower bound of every distance; in FP32, with the margin of the whole
      // box for its rounding), as many as surely fit
      __syncthreads();
      if (tid == 0) listed = 0;
      __syncthreads();
      int cnt = 0;
      const float lim = a.list_lim;
      do {
        const int n = min(total - s0, kRsList - cnt);
        float4 ahead[kRsPer];
        unsigned ahead_item[kRsPer];
        auto look = [&](int t0) {
#pragma unroll
          for (int j = 0; j < kRsPer; ++j) {
            const int g = s0 + min(t0 + j * kRsThreads + tid, n - 1);
            int k = 0;  // the segment: last k with seg_pre[k] <= g
#pragma unroll
            for (int st = 16; st >= 1; st >>= 1) k += g >= seg_pre[k + st] ? st : 0;
            const int r = seg_start[k] + (g - seg_pre[k]);
            ahead_item[j] = (unsigned)r | ((unsigned)k << kRsIdxBits);
            ahead[j] = a.rec32[r];
          }
          lds_order();  // keeps the loads here, ahead of the tests of the previous ones
        };
        look(0);
        for (int t0 = 0; t0 < n; t0 += kRsPer * kRsThreads) {
          float4 cand[kRsPer];
          unsigned item[kRsPer];
#pragma unroll
          for (int j = 0; j < kRsPer; ++j) cand[j] = ahead[j], item[j] = ahead_item[j];
          if (t0 + kRsPer * kRsThreads < n) look(t0 + kRsPer * kRsThreads);
          unsigned long long kept[kRsPer];
          int nkept = 0;
#pragma unroll
          for (int j = 0; j < kRsPer; ++j) {
            const float* sh = seg_unit[item[j] >> kRsIdxBits];
            const float x = cand[j].x + sh[0], y = cand[j].y + sh[1], z = cand[j].z + sh[2];
            const float dx = fmaxf(fmaxf(hbox[0] - x, x - hbox[3]), 0.f);
            const float dy = fmaxf(fmaxf(hbox[1] - y, y - hbox[4]), 0.f);
            const float dz = fmaxf(fmaxf(hbox[2] - z, z - hbox[5]), 0.f);
            kept[j] = __ballot(t0 + j * kRsThreads + tid < n && cand[j].w < kRsFar &&
                               dx * dx + dy * dy + dz * dz <= lim);
            nkept += __popcll(kept[j]);
          }
          int base = 0;
          if (lane == 0) base = atomicAdd(&listed, nkept);
          base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
          for (int j = 0; j < kRsPer; ++j) {
            const int below = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(kept[j] >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((unsigned)kept[j], 0u));
            if (kept[j] >> lane & 1ull) list[base + below] = item[j];
            base += __popcll(kept[j]);
          }
        }
        s0 += n;
        __syncthreads();
        cnt = listed;
        __syncthreads();
      } while (s0 < total && kRsList - cnt >= min(total - s0, kRsThreads));

      // --- passes over the list, each taking every npass-th entry
      const int npass = (cnt + kStage - 1) / kStage;
      for (int ps = 0; ps < npass; ++ps) {
        const int n = (cnt - ps + npass - 1) / npass;
        const int nw = (n + 128 * S - 1) / (128 * S), nu = 4 * nw;  // words per lane, per home atom
        __syncthreads();  // the previous pass is done with the stage
        const double ctr[3] = {centre(0), centre(1), centre(2)};
        const int pitch = 32 * nw + 4;  // slots of a column (4 more, so that the columns' banks differ)
        for (int i = tid; i < 128 * S * nw; i += kRsThreads) {
          const int part = S == 1 ? 0 : i / (32 * nu), u = (i >> 5) - part * nu;
          const int t = ((i & 31) * nu + u) * S + part;
          const int c = (u >= nw) + (u >= 2 * nw) + (u >= 3 * nw);  // the column
          const int slot = part * 4 * pitch + 4 * c + 32 * u + (i & 31);
          double x = ctr[0], y = ctr[1], z = ctr[2], sq = kRsFar, qj = 0.0;  // (past the last one)
          if (t < n) {
            const unsigned it = list[t * npass + ps];
            const double* sh = seg_shift[it >> kRsIdxBits];
            const double4 r = a.rec[it & ((1u << kRsIdxBits) - 1)];
            x = r.x + sh[0];
            y = r.y + sh[1];
            z = r.z + sh[2];
            qj = r.w;
            const float fx = (float)((x - ctr[0]) * a.unit_len), fy = (float)((y - ctr[1]) * a.unit_len),
                        fz = (float)((z - ctr[2]) * a.unit_len);
            sq = fx * fx + fy * fy + fz * fz;
          }
          stage[0][slot] = x;
          stage[1][slot] = y;
          stage[2][slot] = z;
          stage[3][slot] = sq;
          stage[4][slot] = qj;
        }
        __syncthreads();
        if (nh <= 0) continue;
        // --- distance tests
        const double sc = g4 == 3 ? 1.0 : a.unit_len;
        const double cg = g4 == 3 ? 0.0 : (g4 == 0 ? ctr[0] : g4 == 1 ? ctr[1] : ctr[2]) * sc;
        const int slot0 = spl * 4 * pitch;
        {
          // this lane's component of row col: tile b of word w lies 32 w + 4 b slots on
          const double* src = &stage[g4][slot0 + (col >> 2) * pitch + (col & 3)];
          for (int w = 0; w < nw; ++w, src += 32) {
            float v[8];
#pragma unroll
            for (int b = 0; b < 8; ++b) v[b] = (float)fma(src[4 * b], sc, -cg);
            f32x4 dd[8];
#pragma unroll
            for (int b = 0; b < 8; ++b)
              dd[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[b], bcol, f32x4{q, q, q, q}, 0, 0, 0);
            unsigned mask = 0u;
#pragma unroll
            for (int b = 0; b < 8; ++b)
#pragma unroll
              for (int r = 0; r < 4; ++r)  // the sign bit shifted in from below
                mask = __builtin_amdgcn_alignbit(mask, __float_as_uint(dd[b][r]), 31);
            masks[w][lane] = mask;
          }
          masks[nw][lane] = masks[nw + 1][lane] = 0u;
        }
        lds_order();
        // --- pair evaluation
        unsigned up = lane * (unsigned)sizeof(unsigned);  // byte offset of the word being walked
        const unsigned end = up + (unsigned)nw * (unsigned)sizeof(masks[0]);
        // (32 slots a word: byte offset up + slots0 in a plane of the stage)
        const unsigned slots0 = (unsigned)(slot0 + g4 * pitch) * (unsigned)sizeof(double) - up;
        const unsigned last_slot = (4u * S * (unsigned)pitch - 5u) * (unsigned)sizeof(double);  // (walk over)
        static_assert(sizeof(masks[0]) == 32 * sizeof(double), "offsets of a word");
        auto word = [&](unsigned o) {
          return *reinterpret_cast<const unsigned*>(reinterpret_cast<const char*>(masks) + o);
        };
        unsigned m = word(up), mn = word(up + (unsigned)sizeof(masks[0]));
        struct Cand {
          double4 r;
          bool ok;
        };
        auto next = [&](Cand& cd) {
          cd.ok = m != 0u;
          const unsigned p = (unsigned)__clz((int)(m | 1u));
          const double* r = reinterpret_cast<const double*>(
              reinterpret_cast<const char*>(stage[0]) + min(slots0 + up + (p << 3), last_slot));
          cd.r = make_double4(r[0], r[kPlane], r[2 * kPlane], r[4 * kPlane]);
          lds_order();  // keeps the load here, ahead of the other candidate's evaluation
          m &= ~(0x80000000u >> p);
          up = min(up + (m == 0u ? (unsigned)sizeof(masks[0]) : 0u), end);
          m = m == 0u ? mn : m;
          mn = word(up + (unsigned)sizeof(masks[0]));
        };
        Cand x, y;
        do {
          next(x);
          next(y);
          rs_pair<NC>(a, kc, ri, x.r, two_to, x.ok, e_pair, f);
          rs_pair<NC>(a, kc, ri, y.r, two_to, y.ok, e_pair, f);
        } while (__any(m != 0u || up < end));
      }
    }
    // the four lanes of a home atom, then the wavefronts sharing it
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      f[d] = active ? f[d] : 0.0;  // (a non-finite home atom takes no part)
      f[d] += __shfl_xor(f[d], 16);
      f[d] += __shfl_xor(f[d], 32);
    }
    if constexpr (S > 1) {
      if (g4 == 0 && col < nh) {
#pragma unroll
        for (int d = 0; d < 3; ++d) atomicAdd(&home_f[h0 + col][d], f[d]);
      }
      __syncthreads();
      if (g4 == 0 && col < nh) {
#pragma unroll
        for (int d = 0; d < 3; ++d) f[d] = home_f[h0 + col][d];
      }
    }
    if (g4 == 0 && col < nh && spl == 0) {
      const bool add = a.accumulate || a.excl_off != nullptr;  // (k_rs_sort or k_rs_count wrote the exclusions)
      double* out = a.forces + 3 * (size_t)a.ridx[own];
#pragma unroll
      for (int d = 0; d < 3; ++d) out[d] = add ? out[d] + f[d] : f[d];
    }
    first = last;
  }
  double v[1] = {0.5 * e_pair};
  wave_sums<1>(v);
  if (lane == 63) home_e[wave] = v[0];
  __syncthreads();
  if (tid == 0) a.rows[id] = (home_e[0] + home_e[1]) + (home_e[2] + home_e[3]);
}

// Energies in a fixed order by one workgroup: E_real, E_self, E_excl.
__global__ __launch_bounds__(kRsCountThreads) void k_rs_reduce(RsArgs a) {
  __shared__ double wred[16 * 8];
  double v[3] = {0.0, 0.0, 0.0};
#pragma unroll 4
  for (int r = threadIdx.x; r < a.nrow; r += kRsCountThreads) v[0] += a.rows[r];
  for (int r = threadIdx.x; r < a.n_count_blocks; r += kRsCountThreads) {
    v[1] += a.rows[(size_t)a.nrow + r];
    v[2] += a.rows[(size_t)a.nrow + a.n_count_blocks + r];
  }
  block_sums<3>(v, wred);
  if (threadIdx.x == 15) {
    a.energies[0] = v[0];
    a.energies[1] = -a.coulomb * a.beta * 0.56418958354775628695 * v[1];  // -c beta/sqrt(pi) sum q^2
    a.energies[2] = v[2];
  }
}

template <int NC>
void launch_pairs(const RsArgs& a, hipStream_t s) {
  const dim3 grid(a.nrow), block(kRsThreads);
  switch (a.split) {
    case 1: k_rs_pairs<NC, 1><<<grid, block, 0, s>>>(a); break;
    case 2: k_rs_pairs<NC, 2><<<grid, block, 0, s>>>(a); break;
    default: k_rs_pairs<NC, 4><<<grid, block, 0, s>>>(a); break;
  }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Wavefronts sharing a group of 16 home atoms: enough workgroups to occupy the
// chip, no more (each repeats the listing of candidates).  Measured at rcut 9 A,
// us per evaluation for 1 / 2 / 4: 50 / 40 / 35 at 2,100 atoms, 62 / 47 / 48 at
// 4,095, 66 / 60 / 68 at 11,100, 68 / 62 / 81 at 15,000, 78 / 75 / 80 at 16,400,
// 83 / 81 / 97 at 21,000, 81 / 90 / 104 at 26,000, 150 / 176 / 223 at 65,535
// (between 16,000 and 21,000 one and two are within 4%).
int rs_split(int N) { return N <= 5120 ? 4 : N <= 16384 ? 2 : 1; }

// Pair workgroups launched: no fewer than the groups that list_groups makes of
// N atoms in nunit units (each unit's last may be part full, none is empty).
int rs_rows(int N, int nunit, int split) {
  const long long n = std::min<long long>(N, (long long)N * split / kRsHome + nunit);
  return (int)((n + kXcds - 1) / kXcds * kXcds);
}
// Upper bound of it.
size_t rs_max_rows(int max_atoms, int max_cells) {
  return (size_t)max_atoms * 4 / kRsHome + (size_t)max_cells + kXcds;
}

struct RsLayout {
  size_t count, start, rank, rec, rec32, ridx, groups, ngroup, rows, total;
};

RsLayout rs_layout(int max_atoms, int max_cells) {
  const int nblk = (max_atoms + kRsCountThreads - 1) / kRsCountThreads;
  RsLayout L{};
  size_t o = 0;
  const size_t nsub = (size_t)max_cells * kRsSlabs;
  L.count = o;   o = align256(o + nsub * sizeof(unsigned));
  L.start = o;   o = align256(o + (nsub + 1) * sizeof(unsigned));
  L.rank = o;    o = align256(o + (size_t)max_atoms * sizeof(unsigned));
  L.rec = o;     o = align256(o + (size_t)max_atoms * sizeof(double4));
  L.rec32 = o;   o = align256(o + (size_t)max_atoms * sizeof(float4));
  L.ridx = o;    o = align256(o + (size_t)max_atoms * sizeof(int));
  L.groups = o;  o = align256(o + rs_max_rows(max_atoms, max_cells) * sizeof(int4));
  L.ngroup = o;  o = align256(o + sizeof(int));
  L.rows = o;    o = align256(o + (rs_max_rows(max_atoms, max_cells) + 2 * (size_t)nblk) * sizeof(double));
  L.total = o;
  return L;
}

// exp(x^2) erfc(x) on [0, X] as a polynomial of n terms in t = 2x/X - 1: its
// Chebyshev coefficients from its values at kNodes Chebyshev nodes (a
// discrete cosine transform, whose cosines all are multiples of pi/(2 kNodes)
// and come from one table), the first n kept, expanded into powers of t.
void erfcx_poly(double X, int n, double* poly) {
  constexpr int kNodes = 48;
  struct Cosines {
    double c[4 * kNodes];
    Cosines() {
      for (int i = 0; i < 4 * kNodes; ++i)
        c[i] = (double)std::cos(3.14159265358979323846264338328L * i / (2 * kNodes));
    }
  };
  static const Cosines table;
  double f[kNodes];
  for (int j = 0; j < kNodes; ++j) {
    const double x = 0.5 * X * (table.c[2 * j + 1] + 1.0);
    // (x^2 exact in extended precision: its rounding would be magnified by x^2)
    f[j] = (double)(std::erfc(x) * std::exp((long double)x * x));
  }
  // power coefficients of T_{k-1}, T_k and of the sum so far
  long double lo[kRsCheb] = {1.0L}, hi[kRsCheb] = {0.0L, 1.0L}, sum[kRsCheb] = {};
  for (int k = 0; k < n; ++k) {
    long double c = 0.0L;
    for (int j = 0; j < kNodes; ++j) c += (long double)f[j] * table.c[k * (2 * j + 1) % (4 * kNodes)];
    c *= (k == 0 ? 1.0L : 2.0L) / kNodes;
    for (int i = 0; i <= k; ++i) sum[i] += c * lo[i];
    // (lo, hi) = (T_k, T_{k+1}) -> (T_{k+1}, T_{k+2})
    for (int i = n - 1; i >= 0; --i) {
      const long double next = (i > 0 ? 2.0L * hi[i - 1] : 0.0L) - lo[i];
      lo[i] = next;
    }
    for (int i = 0; i < n; ++i) std::swap(lo[i], hi[i]);
  }
  for (int i = 0; i < n; ++i) poly[i] = (double)sum[i];
}

constexpr int kRsMaxAtoms = 1 << 26;
constexpr int kRsMaxCells = 1 << 20;

}  // namespace
}  // namespace spme

extern "C" {

size_t pme_real_workspace_bytes(int max_atoms, int max_cells) {
  if (max_atoms < 0 || max_atoms > spme::kRsMaxAtoms || max_cells < 27 ||
      max_cells > spme::kRsMaxCells)
    return 0;
  return spme::rs_layout(max_atoms, max_cells).total;
}

int pme_real(const double* pos, const double* q, int N, const double box[9], double beta,
             double rcut, double coulomb, const int* excl_off, const int* excl_idx, double* forces,
             int accumulate, double* energies, void* workspace, size_t workspace_bytes,
             int max_atoms, int max_cells, void* stream) {
  using namespace spme;
  if (box == nullptr || energies == nullptr || workspace == nullptr) return PME_EINVAL;
  if (N < 0 || N > max_atoms || (N > 0 && (pos == nullptr || q == nullptr || forces == nullptr)))
    return PME_EINVAL;
  if ((excl_off == nullptr) != (excl_idx == nullptr)) return PME_EINVAL;
  if (!(beta > 0.0) || !(rcut > 0.0) || !std::isfinite(beta) || !std::isfinite(rcut))
    return PME_EINVAL;
  if (beta * rcut > kRsMaxBetaRcut) return PME_EUNSUPPORTED;  // erfc(6) < 3e-17
  if (coulomb == 0.0) coulomb = 1.0;
  for (int i = 0; i < 9; ++i)
    if (!std::isfinite(box[i])) return PME_EINVAL;
  if (box[1] != 0.0 || box[2] != 0.0 || box[3] != 0.0 || box[5] != 0.0 || box[6] != 0.0 ||
      box[7] != 0.0)
    return PME_EUNSUPPORTED;  // the cell search assumes a diagonal box
  const double L[3] = {box[0], box[4], box[8]};
  if (!(L[0] > 0.0 && L[1] > 0.0 && L[2] > 0.0)) return PME_EINVAL;
  const size_t need = pme_real_workspace_bytes(max_atoms, max_cells);
  if (need == 0) return PME_EINVAL;
  if (workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0)
    return PME_EWORKSPACE;
  RsArgs a{};
  long long ncell = 1;
  for (int d = 0; d < 3; ++d) {
    // (no axis ends with more than max_cells; the product of three fits)
    a.nc[d] = (int)std::min(std::floor(L[d] / rcut), (double)max_cells);
    if (a.nc[d] < 3) return PME_EUNSUPPORTED;  // rcut must be <= L/3 along every axis
    ncell *= a.nc[d];
  }
  while (ncell > max_cells) {  // coarser cells (edge still >= rcut)
    int big = 0;
    for (int d = 1; d < 3; ++d)
      if (a.nc[d] > a.nc[big]) big = d;
    if (a.nc[big] <= 3) return PME_EWORKSPACE;
    ncell = ncell / a.nc[big] * (a.nc[big] - 1);
    a.nc[big] -= 1;
  }
  a.ncell = (int)ncell;
  // home atoms are taken from whole rows of cells along x where a group may
  // span two cells without meeting its own image (at least four cells), so
  // that all groups but a row's last are full
  a.unit = a.nc[0] >= 4 ? a.nc[0] : 1;
  a.nunit = a.ncell / a.unit;
  a.max_span = a.unit > 1 ? std::min(a.nc[0] - 3, 2) : 0;
  const double ext = 0.5 * std::sqrt(L[0] * L[0] + L[1] * L[1] + L[2] * L[2]) + rcut;
  int e2 = 0;
  (void)std::frexp(ext, &e2);
  a.unit_len = std::ldexp(1.0, 1 - e2);
  a.len_unit = std::ldexp(1.0, e2 - 1);
  const double eu = ext * a.unit_len, ru = rcut * a.unit_len;
  a.list_lim = (float)(ru * ru + 4e-6 * eu * eu);
  a.slack = 0x1p-22 * eu;
  a.split = rs_split(N);
  a.nrow = rs_rows(N, a.nunit, a.split);
  a.N = N;
  a.n_count_blocks = (N + kRsCountThreads - 1) / kRsCountThreads;
  for (int d = 0; d < 3; ++d) {
    a.L[d] = L[d];
    a.invL[d] = 1.0 / L[d];
    a.cell_inv[d] = a.nc[d] / L[d];
  }
  a.beta = beta;
  a.rcut = rcut;
  a.rc2 = rcut * rcut;
  // a shorter range needs fewer terms (the coefficients of this entire
  // function fall off faster on a shorter interval)
  a.ncheb = beta * rcut <= kRsShortRange ? kRsChebShort : kRsCheb;
  erfcx_poly(beta * rcut, a.ncheb, a.poly);
  a.two_over_rcut = 2.0 / rcut;
  a.exp_scale = -kRsExp * beta * beta / 0.69314718055994530942;
  a.coulomb = coulomb;
  a.pos = pos;
  a.q = q;
  a.excl_off = excl_off;
  a.excl_idx = excl_idx;
  a.forces = forces;
  a.accumulate = accumulate ? 1 : 0;
  a.energies = energies;
  const RsLayout W = rs_layout(max_atoms, max_cells);
  char* ws = static_cast<char*>(workspace);
  a.count = reinterpret_cast<unsigned*>(ws + W.count);
  a.start = reinterpret_cast<unsigned*>(ws + W.start);
  a.rank = reinterpret_cast<unsigned*>(ws + W.rank);
  a.rec = reinterpret_cast<double4*>(ws + W.rec);
  a.rec32 = reinterpret_cast<float4*>(ws + W.rec32);
  a.ridx = reinterpret_cast<int*>(ws + W.ridx);
  a.groups = reinterpret_cast<int4*>(ws + W.groups);
  a.ngroup = reinterpret_cast<int*>(ws + W.ngroup);
  a.rows = reinterpret_cast<double*>(ws + W.rows);
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int nsub = a.ncell * kRsSlabs;
  const dim3 atoms(a.n_count_blocks), block(kRsCountThreads);
  if (N > 0 && N <= kRsSmall && nsub <= kRsSortTable) {
    a.n_count_blocks = (N + kRsSortThreads - 1) / kRsSortThreads;
    const dim3 grid(a.n_count_blocks + 1), threads(kRsSortThreads);
    if (a.n_count_blocks <= 2)
      k_rs_sort<2><<<grid, threads, 0, s>>>(a);
    else if (a.n_count_blocks <= 4)
      k_rs_sort<4><<<grid, threads, 0, s>>>(a);
    else
      k_rs_sort<8><<<grid, threads, 0, s>>>(a);
  } else {
    k_rs_zero<<<dim3((nsub + 255) / 256), dim3(256), 0, s>>>(a);
    if (N > 0) k_rs_count<<<atoms, block, 0, s>>>(a);
    if (nsub > kRsTable || N == 0) k_rs_scan<<<dim3(1), dim3(kRsScanThreads), 0, s>>>(a);
    if (N > 0) {
      if (nsub > kRsTable)
        k_rs_fill<false><<<atoms, block, 0, s>>>(a);
      else
        k_rs_fill<true><<<dim3(a.n_count_blocks + 1), block, 0, s>>>(a);
    }
  }
  if (N > 0) {
    if (a.ncheb == kRsChebShort)
      launch_pairs<kRsChebShort>(a, s);
    else
      launch_pairs<kRsCheb>(a, s);
  }
  k_rs_reduce<<<dim3(1), block, 0, s>>>(a);
  return hipGetLastError() == hipSuccess ? PME_OK : PME_EDEVICE;
}

}  // extern "C"
