// Environment matrix R~ from positions, and forces / virials from dE/dR~
// (DP Compress, Sec. II: the weighting function of Eq. (1), the per-type
// normalisation after it, and F = -dE/dr).
//
// For neighbour slot s of atom i with j = nlist[i][s] >= 0, r_ij = r_j - r_i
// is the minimum image in a cubic periodic box of edge L (L > 2 r_c), r =
// |r_ij|, and the row of R~ is
//   ((s(r) - mean_t) / sigma_t, s(r) x / sigma_all_t, s(r) y / ..., s(r) z / ...)
// with t the type of atom i; padding rows are zero.
//
// Forces: g_is = dE/dr_ij = sum_c dE/dR~_is[c] dR~_is[c]/dr_ij, which is
//   g = (s'(r) / r) (lam_0 / sigma_t + <lam_xyz, r_ij> / sigma_all_t) r_ij
//       + (s(r) / sigma_all_t) lam_xyz          (lam = dE/dR~_is).
// F_i = sum_s g_is - sum over the rows (j, s') in which i is the neighbour of
// g_js'.  Those rows are found once per neighbour list (dpc_nlist_reverse),
// so that each atom gathers its force in a fixed order: no atomics, and the
// result is bitwise reproducible.  The derivative dR~/dr (12 numbers per
// slot) is recomputed from the positions, not stored.  The per-atom virial
// is V_i = -sum_s r_is (x) g_is.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "dpc.h"
#include "dpc_internal.h"

namespace {

struct EnvGeo {
  int nloc, nnei, ntypes;
  double box, rc, rcs;
  double inv_box, inv_w;            // 1 / box, 1 / (rc - rcs)
  double mean[DPC_MAX_TYPES], inv_sigma[DPC_MAX_TYPES], inv_sigma_all[DPC_MAX_TYPES];
  int blk[DPC_MAX_TYPES + 1];       // sel block boundaries (slot offsets)
};

// minimum image of b - a in the cubic box
__device__ __forceinline__ void min_image(const EnvGeo& g, const double* a, const double* b,
                                          double (&d)[3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double x = b[c] - a[c];
    d[c] = x - g.box * round(x * g.inv_box);
  }
}

// s(r) and ds/dr of Eq. (1)
__device__ __forceinline__ void weight(const EnvGeo& g, double r, double& s, double& ds) {
  const double ir = 1.0 / r;
  if (r < g.rcs) {
    s = ir;
    ds = -ir * ir;
  } else if (r < g.rc) {
    const double u = (r - g.rcs) * g.inv_w;
    const double u2 = u * u, u3 = u2 * u;
    const double sw = u3 * (-6.0 * u2 + 15.0 * u - 10.0) + 1.0;
    const double dsw = (-30.0 * u2 * (u - 1.0) * (u - 1.0)) * g.inv_w;
    s = sw * ir;
    ds = (dsw - sw * ir) * ir;
  } else {
    s = 0.0;
    ds = 0.0;
  }
}

// workgroup b covers slots 256 c .. 256 c + 255 of atom b / chunks (c = b mod
// chunks), so that the atom index is uniform; rows are written 16 bytes at a
// time when the output is 16-byte aligned (kPair), float64 rows of whole
// wavefronts in contiguous 1 KB stores
template <typename TO, bool kPair>
__global__ __launch_bounds__(256) void env_mat_kernel(const EnvGeo g, int chunks,
                                                      const double* __restrict__ coord,
                                                      const int* __restrict__ atype,
                                                      const int* __restrict__ nlist,
                                                      TO* __restrict__ em) {
  const int i = __builtin_amdgcn_readfirstlane((int)(blockIdx.x / (unsigned)chunks));
  const int s = (int)(blockIdx.x - (unsigned)i * chunks) * 256 + threadIdx.x;
  if (s >= g.nnei) return;
  const size_t e = (size_t)i * g.nnei + s;
  const int j = __builtin_nontemporal_load(nlist + e);
  double row[4] = {0.0, 0.0, 0.0, 0.0};
  const int t = atype[i];
  if (j >= 0 && j < g.nloc && t >= 0 && t < g.ntypes) {
    double d[3];
    min_image(g, coord + 3 * (size_t)i, coord + 3 * (size_t)j, d);
    const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    double sv, ds;
    weight(g, r, sv, ds);
    row[0] = (sv - g.mean[t]) * g.inv_sigma[t];
    const double f = sv * g.inv_sigma_all[t];
    row[1] = f * d[0];
    row[2] = f * d[1];
    row[3] = f * d[2];
  } else if (j >= 0) {   // neighbour or centre out of range: the row is NaN
    row[0] = row[1] = row[2] = row[3] = (double)NAN;
  }
  TO* o = em + 4 * e;
  if constexpr (kPair && sizeof(TO) == 8) {
    typedef double D2 __attribute__((ext_vector_type(2)));
    // a wavefront whose 64 slots are all in the list writes its 2 KB of rows
    // as two fully contiguous 1 KB stores, transposed through LDS (each lane
    // storing its own 32-byte row leaves every store instruction with gaps)
    __shared__ __align__(16) D2 stage[4][128];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const int sw = __builtin_amdgcn_readfirstlane(s - l);
    if (sw + 64 <= g.nnei) {
      stage[w][2 * l] = D2{row[0], row[1]};
      stage[w][2 * l + 1] = D2{row[2], row[3]};
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      D2* ow = reinterpret_cast<D2*>(em + 4 * ((size_t)i * g.nnei + sw));
      __builtin_nontemporal_store(stage[w][l], ow + l);
      __builtin_nontemporal_store(stage[w][l + 64], ow + l + 64);
      return;
    }
    __builtin_nontemporal_store(D2{row[0], row[1]}, reinterpret_cast<D2*>(o));
    __builtin_nontemporal_store(D2{row[2], row[3]}, reinterpret_cast<D2*>(o) + 1);
  } else if constexpr (kPair) {
    typedef float F4 __attribute__((ext_vector_type(4)));
    __builtin_nontemporal_store(F4{(float)row[0], (float)row[1], (float)row[2], (float)row[3]},
                                reinterpret_cast<F4*>(o));
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) __builtin_nontemporal_store((TO)row[c], o + c);
  }
}

// rev[i][s] = slot of i in the list of j = nlist[i][s], in the sel block of
// i's type, or -1 (also for padding, j out of range and j = i).
//
// One wavefront per atom i.  Its slots are read a window of 512 at a time;
// the neighbours are packed densely into LDS, and each lane then looks for i
// in the list of a neighbour of its own: 16 entries (four 16-byte loads)
// around the place where i is expected, j's rank in its block of i's list
// scaled by the counts of the two blocks in i's list (the same distance
// orders both lists).  98% of the pairs of the Cu and water systems are
// there, 90% of the alloy's, the rest mostly in the 16 entries on either side,
// which the lanes that missed read next.  What is still missing (lists in
// another order) is looked for by the whole wavefront in all of the block.
// Each lane reads a line of its own, about 34 GB of lines on 1,048,576 atoms
// with 180 neighbours (512 slots; 6.3 GB of them come from HBM): the kernel is
// bound by that traffic (address unit 87% busy; 8 or 12 entries first and the misses packed again
// gave 3.4 and 3.7 ms).  Both directions of a pair are searched, because a
// coalesced row of results is cheaper than writing the partner's entry.
// 13.6 ms with a search of one pair at a time by the whole wavefront, now 3.3.
constexpr int kRevWindow = 512;
constexpr int kRevLoads = 4;                 // 16-byte loads of one look
constexpr int kRevLook = 4 * kRevLoads;
constexpr int kXcds = 8;                     // workgroups go to the XCDs in turn

__device__ __forceinline__ int rev_lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// slot in [w, w + 16) and in [b0, b1) of `row` that holds i, else -1; all 16
// entries lie inside the row
__device__ __forceinline__ int rev_look(const int* __restrict__ row, int w, int b0, int b1, int i) {
  typedef int V4 __attribute__((ext_vector_type(4), aligned(4)));
  V4 v[kRevLoads];
#pragma unroll
  for (int q = 0; q < kRevLoads; ++q) v[q] = *reinterpret_cast<const V4*>(row + w + 4 * q);
  int at = -1;
#pragma unroll
  for (int q = kRevLook - 1; q >= 0; --q) at = v[q >> 2][q & 3] == i ? q : at;
  at += at >= 0 ? w : 0;
  return at >= b0 && at < b1 ? at : -1;
}

__global__ __launch_bounds__(256) void reverse_kernel(const EnvGeo g, int per_xcd,
                                                      const int* __restrict__ atype,
                                                      const int* __restrict__ nlist,
                                                      int* __restrict__ rev) {
  __shared__ int sh_j[4][kRevWindow], sh_s[4][kRevWindow];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // each XCD takes a contiguous range of atoms: neighbours' rows stay in its L2
  const int blk = (int)(blockIdx.x % kXcds) * per_xcd + (int)(blockIdx.x / kXcds);
  const int i = __builtin_amdgcn_readfirstlane(blk * 4 + wave);
  if (i >= g.nloc) return;
  const int nnei = g.nnei;
  const int* li = nlist + (size_t)i * nnei;
  int* ri = rev + (size_t)i * nnei;
  const int t = __builtin_amdgcn_readfirstlane(atype[i]);
  if (t < 0 || t >= g.ntypes) {
    for (int s = lane; s < nnei; s += 64) ri[s] = -1;
    return;
  }
  const int b0 = g.blk[t], b1 = g.blk[t + 1];
  int* my_j = sh_j[wave];
  int* my_s = sh_s[wave];
  for (int w0 = 0; w0 < nnei; w0 += kRevWindow) {
    int v[kRevWindow / 64];
#pragma unroll
    for (int q = 0; q < kRevWindow / 64; ++q) {
      const int s = w0 + 64 * q + lane;
      v[q] = s < nnei ? li[s] : -1;
    }
    int np = 0;
    float cnt[DPC_MAX_TYPES];
#pragma unroll
    for (int u = 0; u < DPC_MAX_TYPES; ++u) cnt[u] = 0.0f;
#pragma unroll
    for (int q = 0; q < kRevWindow / 64; ++q) {
      const int s = w0 + 64 * q + lane;
      const bool ok = v[q] >= 0 && v[q] < g.nloc && v[q] != i;
      const uint64_t m = __ballot(ok);
      if (ok) {
        const int p = np + rev_lanes_below(m);
        my_j[p] = v[q];
        my_s[p] = s;
      } else if (s < nnei) {
        ri[s] = -1;
      }
      np += __popcll(m);
      if (g.ntypes > 1 && m) {
#pragma unroll
        for (int u = 0; u < DPC_MAX_TYPES; ++u)
          if (u < g.ntypes) cnt[u] += (float)__popcll(__ballot(ok && s >= g.blk[u] && s < g.blk[u + 1]));
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    float own = 0.0f;
#pragma unroll
    for (int u = 0; u < DPC_MAX_TYPES; ++u) own = u == t ? cnt[u] : own;
    for (int p0 = 0; p0 < np; p0 += 64) {
      const bool live = p0 + lane < np;
      const int p = live ? p0 + lane : 0;
      const int j = my_j[p], s = my_s[p];
      int rank = s;                    // of j in its block, scaled to i's block in j's list
      if (g.ntypes > 1) {
        int bs = 0;
        float c = cnt[0];
#pragma unroll
        for (int u = 1; u < DPC_MAX_TYPES; ++u) {
          const bool in = u < g.ntypes && s >= g.blk[u];
          bs = in ? g.blk[u] : bs;
          c = in ? cnt[u] : c;
        }
        rank = (int)(((float)(s - bs) + 0.5f) * own * __builtin_amdgcn_rcpf(fmaxf(c, 1.0f)));
      }
      const int* row = nlist + (size_t)j * nnei;
      int found = -1;
      if (nnei >= kRevLook) {
        // the look's first entry: inside the block where that holds 16, and inside the row
        const int lo = min(b0, nnei - kRevLook), hi = max(lo, b1 - kRevLook);
        const int w = min(max(b0 + rank - kRevLook / 2, lo), hi);
        found = rev_look(row, w, b0, b1, i);
        if (__ballot(live && found < 0)) {
          if (live && found < 0) {
            const int wl = max(w - kRevLook, lo), wh = min(w + kRevLook, hi);
            const int f0 = rev_look(row, wl, b0, b1, i), f1 = rev_look(row, wh, b0, b1, i);
            found = f0 >= 0 ? f0 : f1;
          }
        }
      }
      uint64_t todo = __ballot(live && found < 0);
      while (todo) {                   // the whole block, 512 entries per round trip
        const int src = (int)__builtin_ctzll(todo);
        todo &= todo - 1;
        const int* r = nlist + (size_t)__builtin_amdgcn_readlane(j, src) * nnei;
        int kk = -1;
        for (int c0 = b0; kk < 0 && c0 < b1; c0 += kRevWindow) {
          int e[kRevWindow / 64];
#pragma unroll
          for (int q = 0; q < kRevWindow / 64; ++q) {
            const int k = c0 + 64 * q + lane;
            e[q] = k < b1 ? r[k] : -1;
          }
#pragma unroll
          for (int q = kRevWindow / 64 - 1; q >= 0; --q) {
            const uint64_t h = __ballot(e[q] == i);
            kk = h ? c0 + 64 * q + (int)__builtin_ctzll(h) : kk;
          }
        }
        if (lane == src) found = kk;
      }
      if (live) ri[s] = found;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// one wavefront per atom; lane l takes slots l, l + 64, ...
template <typename TI>
__global__ __launch_bounds__(256) void force_kernel(const EnvGeo g, const double* __restrict__ coord,
                                                    const int* __restrict__ atype,
                                                    const int* __restrict__ nlist,
                                                    const int* __restrict__ rev,
                                                    const TI* __restrict__ dem,
                                                    double* __restrict__ force,
                                                    double* __restrict__ virial) {
  const int lane = threadIdx.x & 63;
  const int i = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6));
  if (i >= g.nloc) return;
  const int ti = atype[i];
  const bool ok_i = ti >= 0 && ti < g.ntypes;
  double acc[12];                          // F (3), then V row-major (9)
#pragma unroll
  for (int c = 0; c < 12; ++c) acc[c] = 0.0;
  const double* ci = coord + 3 * (size_t)i;
  // g for a pair vector d of a row with dE/dR~ lam, centre type t
  auto pair_grad = [&](const double (&d)[3], const TI* lam_p, int t, double (&gv)[3]) {
    const double r = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    double s, ds;
    weight(g, r, s, ds);
    const double l0 = (double)lam_p[0], l1 = (double)lam_p[1], l2 = (double)lam_p[2],
                 l3 = (double)lam_p[3];
    const double c1 = (ds / r) * (l0 * g.inv_sigma[t] + (l1 * d[0] + l2 * d[1] + l3 * d[2]) * g.inv_sigma_all[t]);
    const double c2 = s * g.inv_sigma_all[t];
    gv[0] = c1 * d[0] + c2 * l1;
    gv[1] = c1 * d[1] + c2 * l2;
    gv[2] = c1 * d[2] + c2 * l3;
  };
  for (int s0 = 0; s0 < g.nnei; s0 += 64) {
    const int s = s0 + lane;
    if (s >= g.nnei || !ok_i) continue;
    const size_t e = (size_t)i * g.nnei + s;
    const int j = nlist[e];
    if (j < 0 || j >= g.nloc) continue;
    double d[3];
    min_image(g, ci, coord + 3 * (size_t)j, d);
    double go[3];
    pair_grad(d, dem + 4 * e, ti, go);
    acc[0] += go[0];
    acc[1] += go[1];
    acc[2] += go[2];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int b = 0; b < 3; ++b) acc[3 + 3 * a + b] -= d[a] * go[b];
    }
    const int rs = rev[e];
    const int tj = atype[j];
    if (rs >= 0 && rs < g.nnei && tj >= 0 && tj < g.ntypes) {
      // the row of j in which i is the neighbour: pair vector r_ji
      const double dr[3] = {-d[0], -d[1], -d[2]};
      double gr[3];
      pair_grad(dr, dem + 4 * ((size_t)j * g.nnei + rs), tj, gr);
      acc[0] -= gr[0];
      acc[1] -= gr[1];
      acc[2] -= gr[2];
    }
  }
  // sum over the wavefront in a fixed order
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    double v = acc[c];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      const int lo = __builtin_amdgcn_ds_bpermute(((lane ^ off) & 63) << 2,
                                                  (int)(uint32_t)__builtin_bit_cast(uint64_t, v));
      const int hi = __builtin_amdgcn_ds_bpermute(((lane ^ off) & 63) << 2,
                                                  (int)(uint32_t)(__builtin_bit_cast(uint64_t, v) >> 32));
      const double w = __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
      v = lane < (lane ^ off) ? v + w : w + v;
    }
    acc[c] = v;
  }
  if (lane == 0) {
    const double nan = ok_i ? 0.0 : (double)NAN;
    for (int c = 0; c < 3; ++c) force[3 * (size_t)i + c] = acc[c] + nan;
    if (virial)
      for (int c = 0; c < 9; ++c) virial[9 * (size_t)i + c] = acc[3 + c] + nan;
  }
}

int make_env_geo(int nloc, int ntypes, int nnei, double box, double rc, double rcs,
                 const double* mean, const double* sigma, const double* sigma_all, EnvGeo* g) {
  if (nloc < 0 || nnei < 1 || ntypes < 1) return DPC_EINVAL;
  if (ntypes > DPC_MAX_TYPES) return DPC_ENOTSUP;
  if (!(std::isfinite(box) && std::isfinite(rc) && std::isfinite(rcs) && rc > 0 && rcs >= 0 &&
        rcs < rc && box > 2 * rc))
    return DPC_ERANGE;
  if ((int64_t)nloc * nnei >= (int64_t(1) << 40)) return DPC_ENOTSUP;
  g->nloc = nloc;
  g->nnei = nnei;
  g->ntypes = ntypes;
  g->box = box;
  g->rc = rc;
  g->rcs = rcs;
  g->inv_box = 1.0 / box;
  g->inv_w = 1.0 / (rc - rcs);
  for (int t = 0; t < DPC_MAX_TYPES; ++t) {
    g->mean[t] = 0.0;
    g->inv_sigma[t] = g->inv_sigma_all[t] = 0.0;
    g->blk[t] = 0;
  }
  g->blk[DPC_MAX_TYPES] = 0;
  for (int t = 0; t < ntypes; ++t) {
    if (mean) {
      if (!std::isfinite(mean[t])) return DPC_ERANGE;
      g->mean[t] = mean[t];
    }
    if (sigma) {
      if (!(sigma[t] > 0 && std::isfinite(sigma[t]))) return DPC_ERANGE;
      g->inv_sigma[t] = 1.0 / sigma[t];
    }
    if (sigma_all) {
      if (!(sigma_all[t] > 0 && std::isfinite(sigma_all[t]))) return DPC_ERANGE;
      g->inv_sigma_all[t] = 1.0 / sigma_all[t];
    }
  }
  return DPC_OK;
}

}  // namespace

extern "C" int dpc_env_mat_a(void* stream, dpc_dtype dtype, int nloc, int ntypes, int nnei,
                             double box, double rc, double rcs, const double* mean,
                             const double* sigma, const double* sigma_all, const double* coord,
                             const int* atype, const int* nlist, void* em) {
  if (dtype != DPC_F64 && dtype != DPC_F32 && dtype != DPC_F32_ACC64) return DPC_EINVAL;
  if (!mean || !sigma || !sigma_all) return DPC_EINVAL;
  EnvGeo g;
  const int st = make_env_geo(nloc, ntypes, nnei, box, rc, rcs, mean, sigma, sigma_all, &g);
  if (st != DPC_OK) return st;
  if (nloc == 0) return DPC_OK;
  if (!coord || !atype || !nlist || !em) return DPC_EINVAL;
  const int chunks = (nnei + 255) / 256;
  if ((int64_t)nloc * chunks >= (int64_t(1) << 31)) return DPC_ENOTSUP;
  const dim3 grid((unsigned)(nloc * chunks));
  const bool pair = reinterpret_cast<uintptr_t>(em) % 16 == 0;
  hipStream_t s = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();  // report only what this launch raises
  auto go = [&](auto kern, auto* out) {
    hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, g, chunks, coord, atype, nlist, out);
  };
  if (dtype == DPC_F64) {
    if (pair) go(env_mat_kernel<double, true>, (double*)em);
    else go(env_mat_kernel<double, false>, (double*)em);
  } else {
    if (pair) go(env_mat_kernel<float, true>, (float*)em);
    else go(env_mat_kernel<float, false>, (float*)em);
  }
  return dpc_internal_launch_status();
}

extern "C" int dpc_nlist_reverse(void* stream, int nloc, int ntypes, const int* sel, double box,
                                 const double* coord, const int* atype, const int* nlist,
                                 int* rev) {
  if (!sel) return DPC_EINVAL;
  if (ntypes < 1) return DPC_EINVAL;
  if (ntypes > DPC_MAX_TYPES) return DPC_ENOTSUP;
  int64_t nnei = 0;
  for (int t = 0; t < ntypes; ++t) {
    if (sel[t] < 0) return DPC_EINVAL;
    nnei += sel[t];
  }
  if (nnei < 1 || nnei > (1 << 20)) return DPC_EINVAL;
  EnvGeo g;
  // rc only bounds the box check here: any cutoff below half the box
  const int st = make_env_geo(nloc, ntypes, (int)nnei, box, 0.5 * box * 0.999, 0.0, nullptr,
                              nullptr, nullptr, &g);
  if (st != DPC_OK) return st;
  int off = 0;
  for (int t = 0; t < ntypes; ++t) {
    g.blk[t] = off;
    off += sel[t];
  }
  for (int t = ntypes; t <= DPC_MAX_TYPES; ++t) g.blk[t] = off;
  if (nloc == 0) return DPC_OK;
  if (!coord || !atype || !nlist || !rev) return DPC_EINVAL;
  const int64_t nslot = (int64_t)nloc * nnei;
  if ((nslot + 255) / 256 >= (int64_t(1) << 31)) return DPC_ENOTSUP;
  hipStream_t s = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  const int blocks = (nloc + 3) / 4, per_xcd = (blocks + kXcds - 1) / kXcds;
  hipLaunchKernelGGL(reverse_kernel, dim3(per_xcd * kXcds), dim3(256), 0, s, g, per_xcd, atype, nlist, rev);
  return dpc_internal_launch_status();
}

extern "C" int dpc_force_a(void* stream, dpc_dtype dtype, int nloc, int ntypes, int nnei,
                           double box, double rc, double rcs, const double* sigma,
                           const double* sigma_all, const double* coord, const int* atype,
                           const int* nlist, const int* rev, const void* dE_dem, double* force,
                           double* virial) {
  if (dtype != DPC_F64 && dtype != DPC_F32 && dtype != DPC_F32_ACC64) return DPC_EINVAL;
  if (!sigma || !sigma_all) return DPC_EINVAL;
  EnvGeo g;
  const int st = make_env_geo(nloc, ntypes, nnei, box, rc, rcs, nullptr, sigma, sigma_all, &g);
  if (st != DPC_OK) return st;
  if (nloc == 0) return DPC_OK;
  if (!coord || !atype || !nlist || !rev || !dE_dem || !force) return DPC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const dim3 grid((nloc + 3) / 4), block(256);
  (void)hipGetLastError();
  if (dtype == DPC_F32)
    hipLaunchKernelGGL(force_kernel<float>, grid, block, 0, s, g, coord, atype, nlist, rev,
                       (const float*)dE_dem, force, virial);
  else
    hipLaunchKernelGGL(force_kernel<double>, grid, block, 0, s, g, coord, atype, nlist, rev,
                       (const double*)dE_dem, force, virial);
  return dpc_internal_launch_status();
}
