// Neighbour list of a periodic cubic box (DP Compress, Sec. II: the rows of
// the environment matrix are the neighbours within r_c, grouped by type into
// sel_beta rows each, sorted by distance inside a group, unused rows empty).
//
// Definition (the same as the plain oracle's): minimum image per component,
// d = x_j - x_i - box rint((x_j - x_i) / box); r2 = dx dx + dy dy + dz dz,
// every operation rounded on its own; j != i is a neighbour when
// r2 < rc * rc; neighbours are ordered by (type, r2, j) and the first
// sel[beta] of type beta fill block beta; empty slots hold -1.
//
// Cell list: cells of edge box / nc >= r_c (slightly more, so that rounding
// at a cell face cannot put two atoms closer than r_c two cells apart).
//   1. zero the counters;  2. cell of each atom, counted with atomics;
//   3. exclusive scan (one workgroup);  4. scatter the atoms into cell order
//   with their coordinates, index and type packed in 32 bytes (1 to 4 in one
//   workgroup for small systems);
//   5. one wavefront per atom walks the (up to) 27 cells around its own as
//   column spans of the cell-ordered array, 64 candidates at a time with
//   the next batch in flight, keeps those within r_c in LDS, ranks each of
//   them among the neighbours of its type and writes its slot.
// The order inside a cell depends on the atomics, but the ranking is a total
// order, so the list does not.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>

#include "dpc.h"
#include "dpc_internal.h"

namespace {

constexpr int kNlWaves = 4;      // wavefronts (atoms) per workgroup of the list kernel
constexpr int kNlCap = 1024;     // neighbours within rc an atom may have
constexpr int kNlKeep = 512;     // of these, what a wavefront's LDS holds in systems with fewer
constexpr int kScanThreads = 1024;

struct alignas(16) NlAtom {      // an atom in cell order
  double x, y, z;                // x is NaN for an atom of an invalid type: never a neighbour
  int j;                         // index | kOutside when the position is outside [0, box)
  int type;
};
constexpr int kOutside = 1 << 30;

// A neighbour within r_c as kept in LDS: the bits of r2 (>= 0: ordered like
// the value) in one array, type and index packed as type << 28 | j in another
// (12 bytes per neighbour, so that three workgroups share a CU).
constexpr int kJBits = 28;
constexpr uint32_t kJMask = (1u << kJBits) - 1;

struct NlGeo {
  int nloc, ntypes, nnei, nc, ncell;
  int lo_off, n_off;             // stencil offsets per axis: lo_off .. lo_off + n_off - 1
  int type_buckets;              // r2 buckets per type in the ranking
  double box, rc2, inv_cs, inv_box;
  double bucket_scale;           // buckets per unit of r2
  int sel[DPC_MAX_TYPES];
  int blk[DPC_MAX_TYPES + 1];    // first slot of each type block
};

// d - box rint(d / box) with the quotient correctly rounded, as defined.
// rint(d / box) is taken from d (1 / box) instead of a division whenever that
// product lies more than 1e-6 away from a half-integer (and |q| < 2^20): the
// two quotients differ by a few units in the last place (< 1e-9 there), so
// both round to the same integer.  Otherwise (rare; NaN and infinities too)
// the division decides.
__device__ __forceinline__ double min_image(double d, const NlGeo& g) {
#pragma clang fp contract(off)
  const double q = d * g.inv_box;
  double n = rint(q);
  if (!(fabs(q - n) < 0.499999 && fabs(q) < 1048576.0)) n = rint(d / g.box);
  return d - g.box * n;
}

// all three coordinates in [0, box): cell_axis wraps nothing
__device__ __forceinline__ bool in_box(const double* p, const NlGeo& g) {
#pragma clang fp contract(off)
  return p[0] >= 0.0 && p[0] < g.box && p[1] >= 0.0 && p[1] < g.box && p[2] >= 0.0 && p[2] < g.box &&
         p[0] / g.box < 1.0 && p[1] / g.box < 1.0 && p[2] / g.box < 1.0;
}

__device__ __forceinline__ int cell_axis(double x, const NlGeo& g) {
#pragma clang fp contract(off)
  const double w = x - g.box * floor(x / g.box);       // into [0, box]
  // clamped as a double first: NaN and infinite positions land in cell 0
  return (int)fmin(fmax(w * g.inv_cs, 0.0), (double)(g.nc - 1));
}

__device__ __forceinline__ int cell_index(const double* p, const NlGeo& g) {
  return (cell_axis(p[0], g) * g.nc + cell_axis(p[1], g)) * g.nc + cell_axis(p[2], g);
}

// atom i at place p of the cell order
__device__ __forceinline__ void put_atom(const NlGeo& g, const double* __restrict__ coord,
                                         const int* __restrict__ atype, int i, int p,
                                         NlAtom* __restrict__ sorted) {
  const double* c = coord + 3 * (size_t)i;
  NlAtom a;
  a.x = c[0];
  a.y = c[1];
  a.z = c[2];
  a.j = i | (in_box(c, g) ? 0 : kOutside);
  a.type = atype[i];
  if (a.type < 0 || a.type >= g.ntypes) a.x = (double)NAN;
  sorted[p] = a;
}

// Inclusive sum over the lanes of a wavefront.
__device__ __forceinline__ int wave_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

// the counters and the two status words
__global__ void nl_zero_kernel(int n, int* __restrict__ p, int* __restrict__ status) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
  if (i < 2) status[i] = 0;
}

// Small systems: counters, cells, scan and scatter in one workgroup, with the
// counters in LDS.  Four launches of a few microseconds each become one, until
// one workgroup's passes over the atoms cost more.  Whole build, us, four
// launches and one: 256 atoms 24.9 / 14.4, 2,048: 36 / 20, 6,912: 73 / 55,
// 8,232: 53 / 49, 12,288: 63 / 67, 16,384: 66 / 75.
constexpr int kOneMaxCells = 4096, kOneMaxAtoms = 8192;
__global__ __launch_bounds__(kScanThreads) void nl_cells_one_kernel(const NlGeo g, const double* __restrict__ coord,
                                                                    const int* __restrict__ atype,
                                                                    int* __restrict__ start,
                                                                    int* __restrict__ cell_of,
                                                                    NlAtom* __restrict__ sorted,
                                                                    int* __restrict__ status) {
  __shared__ int cursor[kOneMaxCells];
  __shared__ int part[kScanThreads / 64];
  const int t = threadIdx.x;
  if (t < 2) status[t] = 0;
  for (int c = t; c < g.ncell; c += kScanThreads) cursor[c] = 0;
  __syncthreads();
  for (int i = t; i < g.nloc; i += kScanThreads) {
    const int c = cell_index(coord + 3 * (size_t)i, g);
    cell_of[i] = c;
    atomicAdd(cursor + c, 1);
  }
  __syncthreads();
  // exclusive scan: kPer consecutive cells per thread, wavefronts' sums through LDS
  constexpr int kPer = kOneMaxCells / kScanThreads;
  int v[kPer], sum = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    v[k] = kPer * t + k < g.ncell ? cursor[kPer * t + k] : 0;
    sum += v[k];
  }
  const int upto = wave_scan(sum);
  if ((t & 63) == 63) part[t >> 6] = upto;
  __syncthreads();
  int run = upto - sum;
  for (int w = 0; w < (t >> 6); ++w) run += part[w];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (kPer * t + k < g.ncell) {
      start[kPer * t + k] = run;
      cursor[kPer * t + k] = run;
    }
    run += v[k];
  }
  if (t == 0) start[g.ncell] = g.nloc;
  __syncthreads();
  for (int i = t; i < g.nloc; i += kScanThreads)
    put_atom(g, coord, atype, i, atomicAdd(cursor + cell_of[i], 1), sorted);
}

__global__ void nl_cell_kernel(const NlGeo g, const double* __restrict__ coord,
                               int* __restrict__ count, int* __restrict__ cell_of) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.nloc) return;
  const int c = cell_index(coord + 3 * (size_t)i, g);
  cell_of[i] = c;
  atomicAdd(count + c, 1);
}

// exclusive scan of count[0..ncell) into start[0..ncell] and cursor[0..ncell)
__global__ __launch_bounds__(kScanThreads) void nl_scan_kernel(int ncell,
                                                               const int* __restrict__ count,
                                                               int* __restrict__ start,
                                                               int* __restrict__ cursor) {
  __shared__ int part[kScanThreads];
  const int t = threadIdx.x;
  const int per = (ncell + kScanThreads - 1) / kScanThreads;
  const int c0 = min(ncell, t * per), c1 = min(ncell, c0 + per);
  int sum = 0;
  for (int c = c0; c < c1; ++c) sum += count[c];
  part[t] = sum;
  __syncthreads();
  for (int off = 1; off < kScanThreads; off <<= 1) {   // inclusive scan of the parts
    const int v = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int run = part[t] - sum;
  for (int c = c0; c < c1; ++c) {
    start[c] = run;
    cursor[c] = run;
    run += count[c];
  }
  if (t == kScanThreads - 1) start[ncell] = part[t];
}

__global__ void nl_scatter_kernel(const NlGeo g, const double* __restrict__ coord,
                                  const int* __restrict__ atype,
                                  const int* __restrict__ cell_of, int* __restrict__ cursor,
                                  NlAtom* __restrict__ sorted) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= g.nloc) return;
  put_atom(g, coord, atype, i, atomicAdd(cursor + cell_of[i], 1), sorted);
}

__device__ __forceinline__ uint64_t ballot(bool b) { return __ballot(b); }

// rank + 1 if (type, r2, j) of the packed neighbour (or2, ojt) is below
// (t, r2, j) as unsigned words (the borrow
// of the four-word subtraction), else rank.  r2 >= 0, so its bits order like
// its value.  A subtraction chain keeps the whole comparison in the vector
// unit; compares combined with mask logic would go through scalar registers.
__device__ __forceinline__ unsigned count_before(uint64_t or2, uint32_t ojt, uint32_t j, uint32_t r2lo,
                                                 uint32_t r2hi, uint32_t t, unsigned rank) {
  uint32_t d;
  asm("v_sub_co_u32 %0, vcc, %2, %3\n\t"
      "v_subb_co_u32 %0, vcc, %4, %5, vcc\n\t"
      "v_subb_co_u32 %0, vcc, %6, %7, vcc\n\t"
      "v_subb_co_u32 %0, vcc, %8, %9, vcc\n\t"
      "v_addc_co_u32 %1, vcc, 0, %1, vcc"
      : "=&v"(d), "+v"(rank)
      : "v"(ojt & kJMask), "v"(j), "v"((uint32_t)or2), "v"(r2lo), "v"((uint32_t)(or2 >> 32)),
        "v"(r2hi), "v"(ojt >> kJBits), "v"(t)
      : "vcc");
  return rank;
}

__device__ __forceinline__ int lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int kNlBuckets = 256;

// One wavefront per atom.  Both halves are bound by vector issue.
//   Candidates: the atoms of the 27 cells, 64 at a time.  Their periodic
// image follows from the cells (no rounding of d / box per component), and
// most batches need none.  1,048,576 atoms, 1,160 candidates and 180
// neighbours each: 27 batches of one column's atoms with a rounded quotient
// each, and every neighbour compared with every other for its rank, took
// 10.8 ms; 19 full batches and the buckets take 3.7 ms (VALU 80% busy).
//   Ranks: neighbours are counted into buckets of equal width in r2 (per
// type), the buckets' starts are summed over the lanes, each neighbour moves
// to its bucket, and its rank inside the bucket (one or two neighbours; a
// whole shell in a perfect crystal) comes from comparing with the bucket only.
//   kKeep neighbours per atom fit the wavefront's own LDS: 512, so that 20
// wavefronts share a CU and not 12, or all 1,024 where more than 512 are
// expected (long_lists).  An atom with more than kKeep is done after the others
// of its workgroup, with all of the workgroup's LDS.
template <bool kOne, int kKeep>
__global__ __launch_bounds__(64 * kNlWaves) __attribute__((amdgpu_waves_per_eu(kKeep > kNlKeep ? 3 : 5))) void nl_list_kernel(
    const NlGeo g, const double* __restrict__ coord, const int* __restrict__ cell_of,
    const int* __restrict__ start, const NlAtom* __restrict__ sorted, int* __restrict__ nlist,
    int* __restrict__ status) {
#pragma clang fp contract(off)
  static_assert(kNlWaves * kKeep >= kNlCap + 4, "the workgroup's LDS holds one long list");
  constexpr int kNlPer = kKeep / 64;
  __shared__ uint64_t cand_r2[kNlWaves * kKeep];
  __shared__ uint32_t cand_jt[kNlWaves * kKeep];
  __shared__ __align__(16) uint32_t buckets[kNlWaves][kNlBuckets];   // read and written 16 bytes at a time
  __shared__ int longer[kNlWaves];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ntypes = kOne ? 1 : g.ntypes;
  const bool active = (int)(blockIdx.x * kNlWaves) + wave < g.nloc;
  // past the last atom: the last one again, for the barriers' sake; nothing is written
  const int i = active ? (int)(blockIdx.x * kNlWaves) + wave : g.nloc - 1;
  uint64_t* my_r2 = cand_r2 + wave * kKeep;
  uint32_t* my_jt = cand_jt + wave * kKeep;
  const double xi = coord[3 * (size_t)i], yi = coord[3 * (size_t)i + 1], zi = coord[3 * (size_t)i + 2];
  const int ci = __builtin_amdgcn_readfirstlane(cell_of[i]);
  const int cx = ci / (g.nc * g.nc), cy = (ci / g.nc) % g.nc, cz = ci % g.nc;
  // the periodic images follow from the cells only with three or more cells
  // per axis and positions inside the box
  const double pi[3] = {xi, yi, zi};
  const bool by_cell = g.nc >= 3 && in_box(pi, g);

  // candidates within rc, in the order they are met (n may pass kNlCap:
  // the extra ones are counted, not kept).  The stencil's cells are read as
  // spans of `sorted`: the cells of one (x, y) column that are consecutive
  // in z are consecutive there too, so a column is one span, or two where
  // it wraps around the box.  Lane k < 2 n_off^2 holds span k (column k / 2,
  // part k % 2, possibly empty) with its periodic image: two bits per axis,
  // n + 1 with d = x_j - x_i - n box.  An atom within rc of i in the image n
  // lies in the cell that is met with that n: i is then within rc of the same
  // face, so in the cell beside it.
  const int nsp = 2 * g.n_off * g.n_off;
  int sp0 = 0, sp1 = 0, img = 1 | 1 << 2 | 1 << 4;
  if (lane < nsp) {
    const int col = lane >> 1, part = lane & 1;
    const int rx = cx + g.lo_off + col / g.n_off, ry = cy + g.lo_off + col % g.n_off;
    const int ax = (rx + g.nc) % g.nc, ay = (ry + g.nc) % g.nc;
    const int base = (ax * g.nc + ay) * g.nc;
    int c0 = 0, c1 = 0, nz = 0;         // cells [c0, c1) of this column
    if (g.nc < 3) {
      if (part == 0) c1 = g.nc;
    } else if (cz > 0 && cz < g.nc - 1) {
      if (part == 0) { c0 = cz - 1; c1 = cz + 2; }
    } else if (cz == 0) {
      if (part == 0) { c0 = g.nc - 1; c1 = g.nc; nz = 1; } else { c0 = 0; c1 = 2; }
    } else {
      if (part == 0) { c0 = g.nc - 2; c1 = g.nc; } else { c0 = 0; c1 = 1; nz = -1; }
    }
    sp0 = start[base + c0];
    sp1 = start[base + c1];
    const int nx = rx < 0 ? 1 : (rx >= g.nc ? -1 : 0), ny = ry < 0 ? 1 : (ry >= g.nc ? -1 : 0);
    img = (nx + 1) | (ny + 1) << 2 | (nz + 1) << 4;
  }
  // candidate c of the spans' concatenation is atom c - before + sp0 of the
  // span that holds it; lane k: first candidate after span k, and sp0 - before
  const int upto = wave_scan(sp1 - sp0), shift = sp1 - upto;
  const int total = __builtin_amdgcn_readlane(upto, 63);
  int sp = 0;                              // span that holds the batch's first candidate
  // this lane's atom of the batch from candidate c0 on, and its image
  auto locate = [&](int c0, int& at, int& im) __attribute__((always_inline)) {
    const int c = c0 + lane;
    while (__builtin_amdgcn_readlane(upto, sp) <= c0) ++sp;    // c0 < total
    at = c + __builtin_amdgcn_readlane(shift, sp);
    im = __builtin_amdgcn_readlane(img, sp);
    int end = __builtin_amdgcn_readlane(upto, sp);
    for (int k = sp + 1; end <= c0 + 63 && k < nsp; ++k) {
      const int sh = __builtin_amdgcn_readlane(shift, k), m = __builtin_amdgcn_readlane(img, k);
      at = c >= end ? c + sh : at;
      im = c >= end ? m : im;
      end = __builtin_amdgcn_readlane(upto, k);
    }
    at = c < total ? at : 0;               // every lane loads an atom of the array
  };
  // the first `cap` neighbours go to my_r2, my_jt; all are counted
  auto collect = [&](int cap) __attribute__((always_inline)) {
    int n = 0, im = 0, at = 0;
    sp = 0;
    if (total > 0) locate(0, at, im);
    NlAtom cur = sorted[at];
    for (int c0 = 0; c0 < total; c0 += 64) {
      const int im0 = im;
      if (c0 + 64 < total) locate(c0 + 64, at, im);
      const NlAtom nxt = sorted[at];
      const bool in = c0 + lane < total;
      double dx = cur.x - xi, dy = cur.y - yi, dz = cur.z - zi;
      if (!by_cell || __ballot(in && (cur.j & kOutside))) {
        dx = min_image(dx, g);
        dy = min_image(dy, g);
        dz = min_image(dz, g);
      } else if (__ballot(in && im0 != (1 | 1 << 2 | 1 << 4))) {
        dx -= g.box * (double)((im0 & 3) - 1);
        dy -= g.box * (double)(((im0 >> 2) & 3) - 1);
        dz -= g.box * (double)((im0 >> 4) - 1);
      }
      const double r2 = dx * dx + dy * dy + dz * dz;
      const int j = cur.j & ~kOutside;
      const bool ok = in && r2 < g.rc2 && j != i;
      const uint64_t msk = ballot(ok);
      const int pos = n + lanes_below(msk);
      if (ok && pos < cap) {
        my_r2[pos] = __builtin_bit_cast(uint64_t, r2);
        my_jt[pos] = (uint32_t)cur.type << kJBits | (uint32_t)j;
      }
      n += __popcll(msk);
      cur = nxt;
    }
    return n;
  };
  const int n = active ? collect(kKeep) : 0;
  const int m = n < kNlCap ? n : kNlCap;
  int* row = nlist + (size_t)i * g.nnei;

  int cntv = 0;                   // lane t: neighbours of type t (all of them, before truncation)
  if (kKeep >= kNlCap || m <= kKeep) {
    uint32_t* hist = buckets[wave];
#pragma unroll
    for (int q = 0; q < kNlBuckets / 64; ++q) hist[64 * q + lane] = 0;
    uint64_t r2[kNlPer];
    uint32_t jt[kNlPer];
    int bk[kNlPer], ar[kNlPer];   // bucket, and order of arrival in it
    wave_sync();
    const int nu = (m + 63) >> 6;
    constexpr bool kReread = kKeep > kNlKeep;    // too many neighbours per lane to hold them all
    // equal r2 share a bucket, larger r2 never come in an earlier one
    auto bucket = [&](uint64_t v, uint32_t w) __attribute__((always_inline)) {
      int b = min((int)(__builtin_bit_cast(double, v) * g.bucket_scale), g.type_buckets - 1);
      if (!kOne) b += (int)(w >> kJBits) * g.type_buckets;
      return b;
    };
#pragma unroll
    for (int u = 0; u < kNlPer; ++u) {
      if (kReread ? false : u >= nu) break;      // (sixteen of them: the compiler unrolls no loop with a break)
      const int q = 64 * u + lane;
      r2[u] = my_r2[q];
      jt[u] = my_jt[q];
      bk[u] = ar[u] = 0;
      if (q < m) {
        bk[u] = bucket(r2[u], jt[u]);
        ar[u] = (int)atomicAdd(&hist[bk[u]], 1u);
      }
    }
    wave_sync();
    {
      uint4 h = *reinterpret_cast<const uint4*>(hist + 4 * lane);
      const int sum = (int)(h.x + h.y + h.z + h.w);
      const uint32_t before = (uint32_t)(wave_scan(sum) - sum);
      wave_sync();
      *reinterpret_cast<uint4*>(hist + 4 * lane) =
          make_uint4(before, before + h.x, before + h.x + h.y, before + h.x + h.y + h.z);
    }
    wave_sync();
    // lane t: first rank of type t among all neighbours (m past the last type)
    const int firstv = lane < ntypes ? (int)hist[lane * g.type_buckets] : m;
    cntv = __builtin_amdgcn_ds_bpermute((lane + 1) << 2, firstv) - firstv;
    auto ends = [&](int b, int& lo, int& hi) __attribute__((always_inline)) {
      lo = (int)hist[b];
      hi = b + 1 < kNlBuckets ? (int)hist[b + 1] : m;
    };
    // a neighbour's slot from its rank inside its bucket [lo, hi)
    auto place = [&](bool in, uint64_t v, uint32_t w, int lo, int hi) __attribute__((always_inline)) {
      int rank = lo;
      for (int e = lo; __ballot(e < hi); ++e) {
        if (e < hi) {
          const uint64_t o = my_r2[e];
          // one type per bucket: (r2, j) decides
          rank += o < v || (o == v && my_jt[e] < w) ? 1 : 0;
        }
      }
      int to = rank, end = g.sel[0];       // the slot, and the end of its block
      if constexpr (!kOne) {
        const int t = (int)(w >> kJBits);
        for (int u = 0; u < ntypes; ++u) {
          const int shift_u = g.blk[u] - __builtin_amdgcn_readlane(firstv, u);
          to = u == t ? rank + shift_u : to;
          end = u == t ? g.blk[u + 1] : end;
        }
      }
      if (in && to < end) row[to] = (int)(w & kJMask);
    };
    int lo[kNlPer], hi[kNlPer];
#pragma unroll
    for (int u = 0; u < kNlPer; ++u) {
      if (kReread ? false : u >= nu) break;
      lo[u] = hi[u] = 0;
      if (64 * u + lane < m) {
        ends(bk[u], lo[u], hi[u]);
        my_r2[lo[u] + ar[u]] = r2[u];
        my_jt[lo[u] + ar[u]] = jt[u];
      }
    }
    wave_sync();
    if constexpr (kReread) {
#pragma unroll 1
      for (int q = lane; q - lane < m; q += 64) {
        const uint64_t v = my_r2[q];
        const uint32_t w = my_jt[q];
        int l = 0, h = 0;
        if (q < m) ends(bucket(v, w), l, h);
        place(q < m, v, w, l, h);
      }
    } else {
#pragma unroll
      for (int u = 0; u < kNlPer; ++u) {
        if (u >= nu) break;
        place(64 * u + lane < m, r2[u], jt[u], lo[u], hi[u]);
      }
    }
  }
  // lists that did not fit: one wavefront after the other, in all of the LDS
  if constexpr (kKeep < kNlCap) {
    if (lane == 0) longer[wave] = m > kKeep;
    __syncthreads();
  }
  for (int w = 0; w < (kKeep < kNlCap ? kNlWaves : 0); ++w) {
    if (!longer[w]) continue;              // the same for every thread
    __syncthreads();
    if (w != wave) continue;
    my_r2 = cand_r2;
    my_jt = cand_jt;
    collect(kNlCap);
    int cnt[DPC_MAX_TYPES];
#pragma unroll
    for (int t = 0; t < DPC_MAX_TYPES; ++t) cnt[t] = 0;
    // four entries that rank after every neighbour (type field 15) after the
    // kept ones, so that the ranking below reads the list four at a time
    if (lane < 4) {
      my_r2[m + lane] = ~0ull;
      my_jt[m + lane] = ~0u;
    }
    wave_sync();
    for (int b = 0; b < m; b += 64) {
      const int q = b + lane;
      const int ty = q < m ? (int)(my_jt[q] >> kJBits) : -1;
#pragma unroll
      for (int t = 0; t < DPC_MAX_TYPES; ++t) cnt[t] += __popcll(ballot(ty == t));
    }
    // slot of each kept neighbour: its rank among the neighbours of its type
    // by (r2, j), i.e. its rank among all of them by (type, r2, j) less the
    // number of neighbours of smaller types; up to four candidates per lane
    // per pass over all m, four list entries per step
    for (int b = 0; b < m; b += 256) {
      uint64_t own_r2[4];
      uint32_t own_jt[4];
      unsigned rank[4];
      const int nu = min(4, (m - b + 63) / 64);   // candidate sets of this pass
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = b + 64 * u + lane;
        own_r2[u] = q < m ? my_r2[q] : ~0ull;
        own_jt[u] = q < m ? my_jt[q] : ~0u;
        rank[u] = 0;
#pragma unroll
        for (int t = 0; t < DPC_MAX_TYPES; ++t)
          rank[u] -= (uint32_t)t < (own_jt[u] >> kJBits) ? (unsigned)cnt[t] : 0u;
      }
      for (int e = 0; e < m; e += 4) {
        uint64_t o_r2[4];
        uint32_t o_jt[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          o_r2[v] = my_r2[e + v];
          o_jt[v] = my_jt[e + v];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (u >= nu) break;
#pragma unroll
          for (int v = 0; v < 4; ++v)
            rank[u] = count_before(o_r2[v], o_jt[v], own_jt[u] & kJMask, (uint32_t)own_r2[u],
                                   (uint32_t)(own_r2[u] >> 32), own_jt[u] >> kJBits, rank[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = b + 64 * u + lane;
        const int t = (int)(own_jt[u] >> kJBits);
        if (q < m && (int)rank[u] < g.sel[t]) row[g.blk[t] + (int)rank[u]] = (int)(own_jt[u] & kJMask);
      }
    }
#pragma unroll
    for (int t = 0; t < DPC_MAX_TYPES; ++t) cntv = lane == t ? cnt[t] : cntv;
  }
  if (!active) return;
  // empty slots of each block
  for (int t = 0; t < ntypes; ++t) {
    const int end = g.blk[t + 1];
    for (int s = g.blk[t] + __builtin_amdgcn_readlane(cntv, t) + lane; s < end; s += 64) row[s] = -1;
  }
  if (lane < DPC_MAX_TYPES) {
    const bool trunc = lane < ntypes && cntv > g.blk[lane + 1] - g.blk[lane];
    if (__ballot(trunc) && lane == 0) atomicAdd(status, 1);
    if (n > kNlCap && lane == 0) atomicAdd(status + 1, 1);
  }
}

// Whether atoms with more than kNlKeep neighbours are to be expected: by the
// neighbours of a mean atom, and well below that where more slots are asked for
// (a slab or a cluster is denser than its box).  us, 512 and 1,024 neighbours in
// a wavefront's LDS: 16,384 atoms with 531 neighbours 2,421 / 296, 131,072 with
// 603 20,300 / 2,310, with 464 1,270 / 1,704, with 180 547 / 751; ranking by
// comparison in a list of 1,024, one wavefront each, took 1,030 and 9,270 for
// the first two.
bool long_lists(const NlGeo& g) {
  const double r = std::sqrt(g.rc2), mean = 4.0 / 3.0 * 3.14159265358979 * g.rc2 * r / (g.box * g.box * g.box) * g.nloc;
  return mean > (g.nnei > kNlKeep ? kNlKeep / 2 : kNlKeep - 32);
}

constexpr size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// cells per axis: edge >= rc (1 + 1e-9); at most 1024 per axis and one cell per atom
int cells_per_axis(int nloc, double box, double rc) {
  double n = std::floor(box / (rc * (1.0 + 1e-9)));
  if (!(n >= 1.0)) n = 1.0;
  if (n > 1024.0) n = 1024.0;
  const double cap = std::max(64.0, (double)nloc);
  while (n > 1.0 && n * n * n > cap) n -= 1.0;
  return (int)n;
}

struct NlLayout {
  size_t status, count, start, cursor, cell_of, sorted, total;
};

constexpr NlLayout layout(int nloc, int ncell) {
  NlLayout L{};
  size_t o = 0;
  L.status = o; o += align256(2 * sizeof(int));
  L.count = o; o += align256((size_t)ncell * sizeof(int));
  L.start = o; o += align256(((size_t)ncell + 1) * sizeof(int));
  L.cursor = o; o += align256((size_t)ncell * sizeof(int));
  L.cell_of = o; o += align256((size_t)nloc * sizeof(int));
  L.sorted = o; o += align256((size_t)nloc * sizeof(NlAtom));
  L.total = o;
  return L;
}

int make_geo(int nloc, int ntypes, const int* sel, double box, double rc, NlGeo* g) {
#pragma clang fp contract(off)
  if (nloc < 0 || ntypes < 1 || !sel) return DPC_EINVAL;
  // neighbour indices are kept in kJBits bits
  if (ntypes > DPC_MAX_TYPES || nloc > (1 << kJBits)) return DPC_ENOTSUP;
  if (!(std::isfinite(box) && std::isfinite(rc) && rc > 0.0 && box > 2.0 * rc)) return DPC_ERANGE;
  int64_t nnei = 0;
  for (int t = 0; t < ntypes; ++t) {
    if (sel[t] < 0) return DPC_EINVAL;
    g->blk[t] = (int)nnei;
    g->sel[t] = sel[t];
    nnei += sel[t];
  }
  if (nnei < 1 || nnei > (1 << 20)) return DPC_EINVAL;
  for (int t = ntypes; t < DPC_MAX_TYPES; ++t) g->sel[t] = 0;
  for (int t = ntypes; t <= DPC_MAX_TYPES; ++t) g->blk[t] = (int)nnei;
  g->nloc = nloc;
  g->ntypes = ntypes;
  g->nnei = (int)nnei;
  g->nc = cells_per_axis(nloc, box, rc);
  g->ncell = g->nc * g->nc * g->nc;
  g->lo_off = g->nc >= 3 ? -1 : 0;
  g->n_off = g->nc >= 3 ? 3 : g->nc;
  g->box = box;
  g->rc2 = rc * rc;
  g->inv_cs = g->nc / box;
  g->inv_box = 1.0 / box;
  g->type_buckets = 256 / ntypes;      // kNlBuckets shared out
  g->bucket_scale = g->type_buckets / g->rc2;
  return DPC_OK;
}

}  // namespace

static size_t dpc_nlist_scratch_bytes(int nloc, double box, double rc) {
  if (nloc < 0 || !(std::isfinite(box) && std::isfinite(rc) && rc > 0.0 && box > 2.0 * rc)) return 0;
  const int nc = cells_per_axis(nloc, box, rc);
  return layout(nloc, nc * nc * nc).total;
}

// status_dev: device int[2] for the two counters (NULL: the first 8 bytes of
// the workspace); status_host: host int[2] to wait for and copy them to, or NULL
static int dpc_nlist_launch(void* stream, int nloc, int ntypes, const int* sel, double box, double rc,
                            const double* coord, const int* atype, void* workspace,
                            size_t workspace_bytes, int* nlist, int* status_dev,
                            int* status_host) {
  NlGeo g;
  const int st = make_geo(nloc, ntypes, sel, box, rc, &g);
  if (st != DPC_OK) return st;
  if (nloc == 0) {
    if (status_host) status_host[0] = status_host[1] = 0;
    return DPC_OK;
  }
  if (!coord || !atype || !workspace || !nlist) return DPC_EINVAL;
  const NlLayout L = layout(nloc, g.ncell);
  if (workspace_bytes < L.total || reinterpret_cast<uintptr_t>(workspace) % 256) return DPC_EINVAL;
  unsigned char* w = static_cast<unsigned char*>(workspace);
  int* status = status_dev ? status_dev : reinterpret_cast<int*>(w + L.status);
  int* count = reinterpret_cast<int*>(w + L.count);
  int* start = reinterpret_cast<int*>(w + L.start);
  int* cursor = reinterpret_cast<int*>(w + L.cursor);
  int* cell_of = reinterpret_cast<int*>(w + L.cell_of);
  NlAtom* sorted = reinterpret_cast<NlAtom*>(w + L.sorted);
  hipStream_t s = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();  // report only what these launches raise
  const dim3 ga((nloc + 255) / 256), b256(256);
  if (nloc <= kOneMaxAtoms && g.ncell <= kOneMaxCells) {
    hipLaunchKernelGGL(nl_cells_one_kernel, dim3(1), dim3(kScanThreads), 0, s, g, coord, atype, start, cell_of,
                       sorted, status);
  } else {
    // the counters and the status words start at zero (a fill kernel, not a memset)
    hipLaunchKernelGGL(nl_zero_kernel, dim3((g.ncell + 255) / 256), b256, 0, s, g.ncell, count, status);
    hipLaunchKernelGGL(nl_cell_kernel, ga, b256, 0, s, g, coord, count, cell_of);
    hipLaunchKernelGGL(nl_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, g.ncell, count, start, cursor);
    hipLaunchKernelGGL(nl_scatter_kernel, ga, b256, 0, s, g, coord, atype, cell_of, cursor, sorted);
  }
  auto list = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((nloc + kNlWaves - 1) / kNlWaves), dim3(64 * kNlWaves), 0, s, g, coord, cell_of,
                       start, sorted, nlist, status);
  };
  if (long_lists(g)) list(ntypes == 1 ? nl_list_kernel<true, kNlCap> : nl_list_kernel<false, kNlCap>);
  else list(ntypes == 1 ? nl_list_kernel<true, kNlKeep> : nl_list_kernel<false, kNlKeep>);
  const int ls = dpc_internal_launch_status();
  if (ls != DPC_OK || !status_host) return ls;
  int h[2] = {0, 0};
  if (hipMemcpyAsync(h, status, sizeof h, hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess) {
    const int e = dpc_internal_launch_status();   // keeps the HIP error for dpc_last_hip_error
    return e == DPC_OK ? DPC_EHIP : e;
  }
  status_host[0] = h[0];
  status_host[1] = h[1];
  if (h[1] > 0) return DPC_ENOTSUP;
  if (h[0] > 0) return DPC_EOVERFLOW;
  return DPC_OK;
}

// ---------------------------------------------------------------------------
// The same list with the cell list in a static device array of the library,
// for callers that cannot allocate device memory.  Each GPU that runs it
// holds one copy of the array until the process ends; host code reaches it
// only through the device address hipGetSymbolAddress gives for that GPU.
// ---------------------------------------------------------------------------
// the cell count is capped at max(64, nloc): the largest layout is that of
// DPC_NLIST_NOALLOC_MAX_ATOMS atoms and as many cells
static constexpr size_t kScratchBytes =
    layout(DPC_NLIST_NOALLOC_MAX_ATOMS, DPC_NLIST_NOALLOC_MAX_ATOMS).total;

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// device address of this GPU's copy of `scratch`, looked up once per device
// with that device current
int scratch_address(int dev, void** out) {
  if (dev < 0 || dev >= kMaxDevices) return DPC_ENOTSUP;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      const int e = dpc_internal_launch_status();
      return e == DPC_OK ? DPC_EHIP : e;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return DPC_OK;
}

}  // namespace

extern "C" int dpc_nlist_build_noalloc(void* stream, int nloc, int ntypes, const int* sel,
                                       double box, double rc, const double* coord,
                                       const int* atype, int* nlist, int* status) {
  NlGeo g;
  const int st = make_geo(nloc, ntypes, sel, box, rc, &g);
  if (st != DPC_OK) return st;
  if (nloc > DPC_NLIST_NOALLOC_MAX_ATOMS || layout(nloc, g.ncell).total > kScratchBytes)
    return DPC_ENOTSUP;
  if (nloc == 0) return DPC_OK;
  if (!coord || !atype || !nlist) return DPC_EINVAL;
  // the array of the GPU the stream runs on, which must be the current one
  int cur = -1;
  hipDevice_t sdev = -1;
  if (hipGetDevice(&cur) != hipSuccess ||
      hipStreamGetDevice(static_cast<hipStream_t>(stream), &sdev) != hipSuccess) {
    const int e = dpc_internal_launch_status();
    return e == DPC_OK ? DPC_EHIP : e;
  }
  if (sdev != cur) return DPC_EINVAL;
  void* ws = nullptr;
  const int sa = scratch_address(cur, &ws);
  if (sa != DPC_OK) return sa;
  return dpc_nlist_launch(stream, nloc, ntypes, sel, box, rc, coord, atype, ws, kScratchBytes,
                          nlist, status, nullptr);
}

extern "C" size_t dpc_nlist_workspace_bytes(int nloc, double box, double rc) {
  return dpc_nlist_scratch_bytes(nloc, box, rc);
}

extern "C" int dpc_nlist_build(void* stream, int nloc, int ntypes, const int* sel, double box,
                               double rc, const double* coord, const int* atype, void* workspace,
                               size_t workspace_bytes, int* nlist, int* status_host) {
  return dpc_nlist_launch(stream, nloc, ntypes, sel, box, rc, coord, atype, workspace,
                          workspace_bytes, nlist, nullptr, status_host);
}
