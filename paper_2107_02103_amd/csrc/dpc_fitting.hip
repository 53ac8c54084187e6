// Fitting net: descriptor D_i -> atomic energy E_i and dE/dD_i (DP Compress,
// Sec. II: a fully connected network maps the descriptor to E^i; Sec. III:
// widths (240, 240, 240)).  Read as
//   h_1 = tanh(x W_1 + b_1),  h_l = h_{l-1} + tanh(h_{l-1} W_l + b_l) (l = 2, 3),
//   E = h_3 . w_out + b_out,
// with x = D_i flattened row-major.  Backward (delta_l = dE/dh_l):
//   delta_3 = w_out,  delta_{l-1} = delta_l + W_l ((1 - t_l^2) delta_l),
//   dE/dx = W_1 ((1 - t_1^2) delta_1).
//
// Width 240 (the paper's) runs in three kernels on the float64 matrix cores:
// layer 1 (n_in x 240, bias and tanh as it finishes), the middle of the net
// (layers 2 and 3, the energy, and the backward of both; the activations of a
// workgroup's atoms stay in registers and LDS, but for 22 registers that the
// shape for large systems spills) and dE/dx.  Other widths, an n_in that is
// not a multiple of 4 and unaligned buffers go through plain GEMMs (rocBLAS,
// on the caller's handle) with atoms as the long dimension and four streaming
// kernels: bias + tanh (layer 1), bias + tanh + residual (layer 2), layer 3
// fused with the energy dot product and the first backward scaling (h_3 is
// never stored), and (1 - t^2) (w_out + e) for the two remaining layers, where
// e = delta - w_out accumulates in the backward GEMMs so that the constant
// delta_3 = w_out is never materialised.  There, row-major X [N][c] is
// column-major [c][N], so Z^T = W^T H^T is dgemm(N, N, out, N, in, W, ld out,
// H, ld in) and dH^T = W dZ^T is dgemm(T, N, in, N, out, W, ld out, dZ, ld out).
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "dpc.h"
#include "dpc_fit_tiles.h"
#include "dpc_internal.h"

namespace {

// tanh(x) = expm1(2x) / (expm1(2x) + 2): expm1 keeps its relative accuracy
// near 0, so the quotient does too, and it costs about two thirds of the
// library tanh here.  |x| is capped at 20, where tanh(x) rounds to +-1 in
// float64 and expm1(2x) is still finite; NaN passes through.
__device__ inline double tanh_e(double x) {
  const double c = x > 20.0 ? 20.0 : (x < -20.0 ? -20.0 : x);
  const double y = expm1(2.0 * c);
  return y / (y + 2.0);
}


// Grid-stride walk over the element pairs (e, e + 1), e = 0, 2, 4, ... of a
// row-major [n][w] array, tracking the column of e without a division per
// step.  nw = n * w may be odd: the last element then goes alone.
struct PairWalk {
  int64_t e, step, nw;
  int col, w, step_col;
  __device__ PairWalk(int64_t nw_, int w_) : nw(nw_), w(w_) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    step = 2 * (int64_t)gridDim.x * blockDim.x;
    e = 2 * t;
    col = (int)(e % w);
    step_col = (int)(step % w);
  }
  __device__ bool ok() const { return e < nw; }
  __device__ bool pair() const { return e + 1 < nw; }
  __device__ int col1() const { return col + 1 == w ? 0 : col + 1; }
  __device__ void next() {
    e += step;
    col += step_col;
    if (col >= w) col -= w;
  }
};

__device__ inline double2 ld2(const double* p) { return *reinterpret_cast<const double2*>(p); }
__device__ inline void st2(double* p, double a, double b) { *reinterpret_cast<double2*>(p) = make_double2(a, b); }

// layer 1: t1 = tanh(z + b1)
__global__ __launch_bounds__(256) void layer1_kernel(int64_t nw, int w, const double* __restrict__ z,
                                                     const double* __restrict__ b, double* __restrict__ t1) {
  for (PairWalk it(nw, w); it.ok(); it.next()) {
    if (it.pair()) {
      const double2 v = ld2(z + it.e);
      st2(t1 + it.e, tanh_e(v.x + b[it.col]), tanh_e(v.y + b[it.col1()]));
    } else {
      t1[it.e] = tanh_e(z[it.e] + b[it.col]);
    }
  }
}

// layer 2: t2 = tanh(z + b2), h2 = t1 + t2
__global__ __launch_bounds__(256) void layer2_kernel(int64_t nw, int w, const double* __restrict__ z,
                                                     const double* __restrict__ b,
                                                     const double* __restrict__ t1, double* __restrict__ t2,
                                                     double* __restrict__ h2) {
  for (PairWalk it(nw, w); it.ok(); it.next()) {
    if (it.pair()) {
      const double2 v = ld2(z + it.e), u = ld2(t1 + it.e);
      const double a = tanh_e(v.x + b[it.col]), c = tanh_e(v.y + b[it.col1()]);
      st2(t2 + it.e, a, c);
      st2(h2 + it.e, u.x + a, u.y + c);
    } else {
      const double a = tanh_e(z[it.e] + b[it.col]);
      t2[it.e] = a;
      h2[it.e] = t1[it.e] + a;
    }
  }
}

// layer 3 and the energy, one wavefront per atom:
//   t3 = tanh(z + b3), E = (h2 + t3) . w_out + b_out (fixed-order sum),
//   and, when dz is given, dz = (1 - t3^2) w_out (dz may alias z)
__global__ __launch_bounds__(256) void layer3_energy_kernel(int n, int w, const double* z,
                                                            const double* __restrict__ b,
                                                            const double* __restrict__ h2,
                                                            const double* __restrict__ wout, double bout,
                                                            double* __restrict__ E, double* dz) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (i >= n) return;
  const size_t row = (size_t)i * w;
  double acc = 0.0;
  for (int c = lane; c < w; c += 64) {
    const double t = tanh_e(z[row + c] + b[c]);
    acc = fma(h2[row + c] + t, wout[c], acc);
    if (dz) dz[row + c] = (1.0 - t * t) * wout[c];
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint64_t u = __builtin_bit_cast(uint64_t, acc);
    const int lo = __builtin_amdgcn_ds_bpermute(((lane ^ off) & 63) << 2, (int)(uint32_t)u);
    const int hi = __builtin_amdgcn_ds_bpermute(((lane ^ off) & 63) << 2, (int)(uint32_t)(u >> 32));
    acc += __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
  }
  if (lane == 0) E[i] = acc + bout;
}

// dz = (1 - t^2) (w_out + e), where e = delta - w_out
__global__ __launch_bounds__(256) void tanh_grad_kernel(int64_t nw, int w, const double* __restrict__ t,
                                                        const double* __restrict__ wout,
                                                        const double* __restrict__ e,
                                                        double* __restrict__ dz) {
  for (PairWalk it(nw, w); it.ok(); it.next()) {
    if (it.pair()) {
      const double2 tv = ld2(t + it.e), ev = ld2(e + it.e);
      st2(dz + it.e, (1.0 - tv.x * tv.x) * (wout[it.col] + ev.x),
          (1.0 - tv.y * tv.y) * (wout[it.col1()] + ev.y));
    } else {
      dz[it.e] = (1.0 - t[it.e] * t[it.e]) * (wout[it.col] + e[it.e]);
    }
  }
}

// ---------------------------------------------------------------------------
// Width 240 on the matrix cores
// ---------------------------------------------------------------------------
// All products are formed transposed, out^T = W^T X^T: v_mfma_f64_16x16x4f64
// takes 16 channels as its rows (A = weights, lane (i = l % 16, kk = l / 16)
// holds row i, K index kk) and 16 atoms as its columns (B = activations, lane
// (kk, j = l % 16)); lane (q = l / 16, j) then holds rows q + 4 r, r = 0..3, of
// column j (measured on gfx950).  Row i of a tile stands for channel
// 4 (i % 4) + i / 4, so that a lane's four results are the consecutive
// channels 4 q + r, and K step r of a chunk of 16 takes k = 4 kk + r: results
// are stored and activations loaded 32 bytes per lane, and one layer's results
// are laid out as the next one's operand.
//
// The kernels are bound by the float64 matrix rate (70 to 78 TFLOP/s in a
// loop of these instructions alone, the same with one chain per wavefront as
// with eight; matrix cores 75 to 82% busy on 131,072 atoms).  Through rocBLAS a
// 240-wide side wastes a sixteenth of the 128-wide tiles, 96 tiles for 12,288
// atoms leave most of the chip idle, and the products need ten passes over the
// activations between them.  Energy and dE/dD, n_in 1,600, us through rocBLAS
// and here: 256 atoms 147 / 49, 1,000: 114 / 104, 2,048: 146 / 146, 4,000:
// 214 / 193, 12,288: 580 / 456, 131,072: 5,190 / 4,440, 1,048,576: 39,700 / 35,100.
constexpr int kXcd = 8;                    // workgroups go to the XCDs in turn

typedef double D2 __attribute__((ext_vector_type(2)));
typedef double D4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ D4 mfma16(double a, double b, D4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ D4 ld4(const double* p) {      // 16-byte aligned
  const D2 a = *reinterpret_cast<const D2*>(p), b = *reinterpret_cast<const D2*>(p + 2);
  return D4{a.x, a.y, b.x, b.y};
}
__device__ __forceinline__ void st4(double* p, D4 v) {
  *reinterpret_cast<D2*>(p) = D2{v.x, v.y};
  *reinterpret_cast<D2*>(p + 2) = D2{v.z, v.w};
}

// Layer 1: t1 = tanh(X W + b).  A workgroup takes 64 atoms (16 per wavefront)
// and CT tiles of channels; KC rows of its weights at a time go through LDS,
// the next ones on their way in registers; each wavefront reads its atoms' X
// from memory itself.  Rows of the LDS copy are 4 doubles past a multiple of 8
// apart: two K indices' rows fall into different halves of the banks.
// Workgroups that share atoms run on one XCD (they read the same X).
// Four channel tiles (the last group has three) fill the CUs where five leave a
// quarter of them idle: 4,000 atoms, n_in 2,048, energy and gradient 245 / 228 us
// with 5 / 4 (224 through rocBLAS), 8,000: 406 / 392 with 3 / 4 (421).
template <int CT, int KC>
__global__ __launch_bounds__(256, 2) void fit_layer1_kernel(int n, int nin, int nag,
                                                            const double* __restrict__ X,
                                                            const double* __restrict__ W,
                                                            const double* __restrict__ bias,
                                                            double* __restrict__ t1) {
  constexpr int kGroups = (kFt + CT - 1) / CT, kLd = 16 * CT + 4, kSub = KC / 16;
  constexpr int kUnits = KC * CT * 8, kPer = (kUnits + 255) / 256;   // 16-byte pieces of a stage
  __shared__ __align__(16) double sW[2][KC * kLd];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int loc = (int)(blockIdx.x / kXcd), cg = loc % kGroups;
  const int ag = (int)(blockIdx.x % kXcd) + kXcd * (loc / kGroups);
  if (ag >= nag) return;
  const int i = lane & 15, kk = lane >> 4;
  const int ch = 4 * (i & 3) + (i >> 2);               // channel of the lane's A row
  const int atom = ag * 64 + wave * 16 + i;
  const double* Xa = X + (size_t)min(atom, n - 1) * nin;
  const double* Wc = W + cg * CT * 16;
  // the last column a 16-byte piece may start at (CT = 4: the last group's
  // fourth tile does not exist; existing columns are read in its place and its
  // results not stored)
  const int cmax = min(CT * 16, kFw - cg * CT * 16) - 2;
  D2 w[kPer];
  D4 x[kSub], xn[kSub];
  auto load = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = (int)threadIdx.x + 256 * u, row = e / (CT * 8), c = e % (CT * 8);
      const int col = 2 * (e < kUnits ? c : 0);
      w[u] = *reinterpret_cast<const D2*>(Wc + (size_t)min(k0 + row, nin - 1) * kFw +
                                          (kFt % CT == 0 ? col : min(col, cmax)));
    }
#pragma unroll
    for (int s = 0; s < kSub; ++s) xn[s] = ld4(Xa + min(k0 + 16 * s + 4 * kk, nin - 4));
  };
  // what was loaded from k0 on; the K indices past n_in become zero here and
  // not with the load, so that nothing waits for a load before the products
  auto stage = [&](int buf, int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = (int)threadIdx.x + 256 * u, row = e / (CT * 8), c = e % (CT * 8);
      if (e < kUnits) *reinterpret_cast<D2*>(&sW[buf][row * kLd + 2 * c]) = k0 + row < nin ? w[u] : D2{0.0, 0.0};
    }
#pragma unroll
    for (int s = 0; s < kSub; ++s) x[s] = k0 + 16 * s + 4 * kk < nin ? xn[s] : D4{0.0, 0.0, 0.0, 0.0};
  };
  D4 acc[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) acc[c] = D4{0.0, 0.0, 0.0, 0.0};
  load(0);
  stage(0, 0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < nin; k0 += KC) {
    const bool more = k0 + KC < nin;
    if (more) load(k0 + KC);
    const double* a = &sW[buf][4 * kk * kLd + ch];
#pragma unroll
    for (int s = 0; s < kSub; ++s) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[c] = mfma16(a[(16 * s + r) * kLd + 16 * c], x[s][r], acc[c]);
      }
    }
    buf ^= 1;
    if (more) stage(buf, k0 + KC);   // last read before the previous barrier
    __syncthreads();
  }
  if (atom >= n) return;
  double* out = t1 + (size_t)atom * kFw + cg * CT * 16 + 4 * kk;
  const double* bc = bias + cg * CT * 16 + 4 * kk;
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    if (kFt % CT != 0 && cg * CT + c >= kFt) continue;
    D4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = tanh_e(acc[c][r] + bc[16 * c + r]);
    st4(out + 16 * c, v);
  }
}

// One product of the net for few atoms: a workgroup takes 16 atoms and CT
// tiles of channels, its KW wavefronts take K chunks of 16 in turn, straight
// from the caches, and their sums meet in LDS, in wavefront order.  The step
// says what becomes of the sums z:
//   kStep1  t1 = tanh(z + b)                     kStep2  t2 = tanh(z + b), h2 = t1 + t2
//   kStep3  t3 = tanh(z + b): the tile's share of the energy, dz3 = (1 - t3^2) w_out
//   kBack3  delta2 = w_out + z, dz2 = (1 - t2^2) delta2 (over t2); the energy from its shares
//   kBack2  dz1 = (1 - t1^2) (delta2 + z)
// Many small workgroups: 256 atoms take 240 of them for a product (5 us; in
// one kernel for the middle of the net they would be 16, 55 us).
enum FitStep { kStep1, kStep2, kStep3, kBack3, kBack2 };
struct FitSmall {
  int n, kdim, groups;             // atoms, K, workgroups per 16 atoms
  const double *X, *W, *bias, *wout;
  double *t1, *t2, *h2, *dz, *share;   // h2: then delta2; share: [15][n]
  double bout, *E;
  bool back;                       // kStep3: dz3 is wanted
};

// sum over the four lanes of an atom (q = 0..3)
__device__ __forceinline__ double fit_lane_sum(double e, int lane) {
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const uint64_t v = __builtin_bit_cast(uint64_t, e);
    const int lo = __builtin_amdgcn_ds_bpermute((lane ^ off) << 2, (int)(uint32_t)v);
    const int hi = __builtin_amdgcn_ds_bpermute((lane ^ off) << 2, (int)(uint32_t)(v >> 32));
    e += __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
  }
  return e;
}

__device__ __forceinline__ double fit_energy(const FitSmall& f, int atom) {
  double e = f.share[atom];
#pragma unroll
  for (int t = 1; t < kFt; ++t) e += f.share[(size_t)t * f.n + atom];
  return e + f.bout;
}

template <int CT, int KW, FitStep kStep>
__global__ __launch_bounds__(64 * KW) void fit_small_kernel(const FitSmall f) {
  constexpr bool kBackW = kStep >= kBack3;
  constexpr int kAhead = 2;
  __shared__ __align__(16) double part[KW][CT][64][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cg = (int)(blockIdx.x % f.groups), a0 = (int)(blockIdx.x / f.groups) * 16;
  const int i = lane & 15, kk = lane >> 4, ch = 4 * (i & 3) + (i >> 2);
  const double* Xa = f.X + (size_t)min(a0 + i, f.n - 1) * f.kdim;
  static_assert(kFt % CT == 0, "whole groups of tiles");
  const int nch = (f.kdim + 15) / 16;
  const double* Wt[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int tc = 16 * (cg * CT + c) + ch;
    Wt[c] = kBackW ? f.W + (size_t)tc * kFw + 4 * kk : f.W + (size_t)(4 * kk) * kFw + tc;
  }
  D4 acc[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) acc[c] = D4{0.0, 0.0, 0.0, 0.0};
  for (int c0 = wave; c0 < nch; c0 += KW * kAhead) {
    D4 x[kAhead], w[kAhead][CT];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int k0 = 16 * (c0 + KW * u);
      const bool ok = k0 + 4 * kk < f.kdim;
      const int kc = ok ? k0 : -4 * kk;              // K past the end: row 0, times zero
      x[u] = ld4(Xa + kc + 4 * kk);
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        if constexpr (kBackW) {
          w[u][c] = ld4(Wt[c] + kc);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) w[u][c][r] = Wt[c][(ptrdiff_t)(kc + r) * kFw];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const bool ok = 16 * (c0 + KW * u) + 4 * kk < f.kdim;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int c = 0; c < CT; ++c)
          acc[c] = mfma16(ok ? w[u][c][r] : 0.0, ok ? x[u][r] : 0.0, acc[c]);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < CT; ++c) st4(part[wave][c][lane], acc[c]);
  __syncthreads();
  const int atom = a0 + i;
  for (int c = wave; c < CT; c += KW) {
    const int tile = cg * CT + c;
    D4 z = ld4(part[0][c][lane]);
#pragma unroll
    for (int v = 1; v < KW; ++v) z += ld4(part[v][c][lane]);
    const int col = 16 * tile + 4 * kk;
    const size_t at = (size_t)min(atom, f.n - 1) * kFw + col;
    const D4 one = D4{1.0, 1.0, 1.0, 1.0};
    if constexpr (kStep == kBack3) {
      const D4 g = ld4(f.wout + col) + z, t = ld4(f.t2 + at);
      if (atom < f.n) {
        st4(f.h2 + at, g);
        st4(f.t2 + at, (one - t * t) * g);
      }
    } else if constexpr (kStep == kBack2) {
      const D4 t = ld4(f.t1 + at);
      if (atom < f.n) st4(f.dz + at, (one - t * t) * (ld4(f.h2 + at) + z));
    } else {
      D4 t;
#pragma unroll
      for (int r = 0; r < 4; ++r) t[r] = tanh_e(z[r] + f.bias[col + r]);
      if constexpr (kStep == kStep1) {
        if (atom < f.n) st4(f.t1 + at, t);
      } else if constexpr (kStep == kStep2) {
        if (atom < f.n) {
          st4(f.t2 + at, t);
          st4(f.h2 + at, ld4(f.t1 + at) + t);
        }
      } else {
        const D4 wo = ld4(f.wout + col), h = ld4(f.h2 + at);
        if (f.back && atom < f.n) st4(f.dz + at, (one - t * t) * wo);
        double e = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) e = fma(h[r] + t[r], wo[r], e);
        e = fit_lane_sum(e, lane);
        if (kk == 0 && atom < f.n) f.share[(size_t)tile * f.n + atom] = e;
      }
    }
  }
  if constexpr (kStep == kBack3) {
    if (cg == 0 && wave == 0 && kk == 0 && atom < f.n) f.E[atom] = fit_energy(f, atom);
  }
}

// The energies alone, from their shares (no gradient is wanted).
__global__ __launch_bounds__(256) void fit_energy_kernel(const FitSmall f) {
  const int atom = (int)(blockIdx.x * 256 + threadIdx.x);
  if (atom < f.n) f.E[atom] = fit_energy(f, atom);
}

// The middle of the net for 16 MT atoms per workgroup of NW wavefronts: from
// t1 through layers 2 and 3 to the energy, and back to dz1 = (1 - t1^2) dE/dh_1.
// A wavefront owns the channel tiles wave, wave + NW, ...: their t1, t2 and
// gradients stay in its registers.  What a layer multiplies goes through LDS
// (row = channel, rows 4 doubles past a multiple of 8 apart); weights come
// straight from the caches (the other wavefronts of the SIMD cover the wait:
// more chunks in flight were no faster).  A weight load of 8 bytes
// feeds MT instructions of 64 cycles; two atom tiles leave the address unit
// half idle, one fills more of the chip when there are few atoms.
template <int MT, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(4))) void fit_middle_kernel(
    int n, const double* __restrict__ t1, const double* __restrict__ W2, const double* __restrict__ b2,
    const double* __restrict__ W3, const double* __restrict__ b3, const double* __restrict__ wout,
    double bout, double* __restrict__ E, double* __restrict__ dz1) {
  constexpr int kTp = (kFt + NW - 1) / NW;       // tiles per wavefront
  constexpr int kLa = 16 * MT + 4;
  extern __shared__ __align__(16) double smem[];
  double* act = smem;                            // [240][kLa]
  double* eb = smem + kFw * kLa;                 // [NW][16 MT]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int a0 = (int)blockIdx.x * 16 * MT;
  const int i = lane & 15, kk = lane >> 4, ch = 4 * (i & 3) + (i >> 2);
  static_assert(fit_tiles_ok(NW), "every tile a wavefront reads exists");
  int tile[kTp];
  bool own[kTp];
#pragma unroll
  for (int u = 0; u < kTp; ++u) {
    own[u] = fit_owns(wave, NW, u);
    tile[u] = fit_tile(wave, NW, u);
  }
  D4 T2[kTp][MT], G[kTp][MT], acc[kTp][MT];
  // t1 of the wavefront's tiles (read again at the end, not held meanwhile)
  auto first = [&](int u, int m) __attribute__((always_inline)) {
    return ld4(t1 + (size_t)min(a0 + 16 * m + i, n - 1) * kFw + 16 * tile[u] + 4 * kk);
  };
  auto publish = [&](const D4 (&v)[kTp][MT]) __attribute__((always_inline)) {
    __syncthreads();                             // the previous operand has been read
#pragma unroll
    for (int u = 0; u < kTp; ++u) {
      if (!own[u]) continue;
#pragma unroll
      for (int m = 0; m < MT; ++m) {
#pragma unroll
        for (int r = 0; r < 4; ++r) act[(16 * tile[u] + 4 * kk + r) * kLa + 16 * m + i] = v[u][m][r];
      }
    }
    __syncthreads();
  };
  // acc = (W^T act) (kBack: W act) of the wavefront's tiles
  auto gemm = [&](const double* __restrict__ W, auto back) __attribute__((always_inline)) {
    constexpr bool kBack = decltype(back)::value;
    auto weights = [&](int t, D4 (&w)[kTp]) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < kTp; ++u) {
        if constexpr (kBack) {
          w[u] = ld4(W + (size_t)(16 * tile[u] + ch) * kFw + 16 * t + 4 * kk);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) w[u][r] = W[(size_t)(16 * t + 4 * kk + r) * kFw + 16 * tile[u] + ch];
        }
      }
    };
#pragma unroll
    for (int u = 0; u < kTp; ++u) {
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[u][m] = D4{0.0, 0.0, 0.0, 0.0};
    }
    D4 w[kTp];
    weights(0, w);
#pragma unroll 1
    for (int t = 0; t < kFt; ++t) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double x[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) x[m] = act[(16 * t + 4 * kk + r) * kLa + 16 * m + i];
#pragma unroll
        for (int u = 0; u < kTp; ++u) {
#pragma unroll
          for (int m = 0; m < MT; ++m) acc[u][m] = mfma16(w[u][r], x[m], acc[u][m]);
        }
      }
      weights(min(t + 1, kFt - 1), w);
    }
  };
#pragma unroll
  for (int u = 0; u < kTp; ++u) {
#pragma unroll
    for (int m = 0; m < MT; ++m) G[u][m] = first(u, m);
  }
  publish(G);
  gemm(W2, std::false_type{});
#pragma unroll
  for (int u = 0; u < kTp; ++u) {
    const D4 b = ld4(b2 + 16 * tile[u] + 4 * kk);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
#pragma unroll
      for (int r = 0; r < 4; ++r) T2[u][m][r] = tanh_e(acc[u][m][r] + b[r]);
      G[u][m] += T2[u][m];                       // h_2
    }
  }
  publish(G);
  gemm(W3, std::false_type{});
  double e[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) e[m] = 0.0;
#pragma unroll
  for (int u = 0; u < kTp; ++u) {
    const D4 b = ld4(b3 + 16 * tile[u] + 4 * kk), wo = ld4(wout + 16 * tile[u] + 4 * kk);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double t = tanh_e(acc[u][m][r] + b[r]);
        if (own[u]) e[m] = fma(G[u][m][r] + t, wo[r], e[m]);
        G[u][m][r] = (1.0 - t * t) * wo[r];      // dz3
      }
    }
  }
  // the energy: over the lanes of an atom, then over the wavefronts, in order
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    e[m] = fit_lane_sum(e[m], lane);
    if (kk == 0) eb[wave * 16 * MT + 16 * m + i] = e[m];
  }
  publish(G);
  if (threadIdx.x < 16 * MT && a0 + (int)threadIdx.x < n) {
    double s = eb[threadIdx.x];
#pragma unroll
    for (int v = 1; v < NW; ++v) s += eb[v * 16 * MT + threadIdx.x];
    E[a0 + threadIdx.x] = s + bout;
  }
  if (!dz1) return;
  gemm(W3, std::true_type{});
#pragma unroll
  for (int u = 0; u < kTp; ++u) {
    const D4 wo = ld4(wout + 16 * tile[u] + 4 * kk);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      G[u][m] = wo + acc[u][m];                  // delta_2
      T2[u][m] = (D4{1.0, 1.0, 1.0, 1.0} - T2[u][m] * T2[u][m]) * G[u][m];
    }
  }
  publish(T2);                                   // dz2
  gemm(W2, std::true_type{});
#pragma unroll
  for (int u = 0; u < kTp; ++u) {
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int atom = a0 + 16 * m + i;
      const D4 f = first(u, m);
      const D4 v = (D4{1.0, 1.0, 1.0, 1.0} - f * f) * (G[u][m] + acc[u][m]);
      if (own[u] && atom < n) st4(dz1 + (size_t)atom * kFw + 16 * tile[u] + 4 * kk, v);
    }
  }
}

// dE/dx = dz1 W_1^T: a workgroup takes 64 atoms (16 per wavefront, their dz1
// in registers as all 60 K steps' operands) and `per` tiles of 16 inputs;
// each tile's weights go through LDS, the next tile's on their way in
// registers.  Rows of the LDS copy are 242 doubles apart: the 16 rows that one
// 16-byte read takes start in different bank groups.
__global__ __launch_bounds__(256, 2) void fit_input_grad_kernel(int n, int nin, int nag, int groups, int per,
                                                                const double* __restrict__ dz,
                                                                const double* __restrict__ W,
                                                                double* __restrict__ dX) {
  constexpr int kLd = kFw + 2, kUnits = 16 * kFw / 2, kPer = (kUnits + 255) / 256;
  __shared__ __align__(16) double sW[2][16 * kLd];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int loc = (int)(blockIdx.x / kXcd), cg = loc % groups;
  const int ag = (int)(blockIdx.x % kXcd) + kXcd * (loc / groups);
  if (ag >= nag) return;
  const int i = lane & 15, kk = lane >> 4, ch = 4 * (i & 3) + (i >> 2);
  const int atom = ag * 64 + wave * 16 + i;
  const int t0 = cg * per, tend = min(t0 + per, (nin + 15) / 16);
  if (t0 >= tend) return;
  D2 w[kPer];
  auto load = [&](int t) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = (int)threadIdx.x + 256 * u, row = e / (kFw / 2), c = e % (kFw / 2);
      const int in = min(16 * t + row, nin - 1);     // rows past n_in: not stored below
      if (e < kUnits) w[u] = *reinterpret_cast<const D2*>(W + (size_t)in * kFw + 2 * c);
    }
  };
  auto stage = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = (int)threadIdx.x + 256 * u, row = e / (kFw / 2), c = e % (kFw / 2);
      if (e < kUnits) *reinterpret_cast<D2*>(&sW[buf][row * kLd + 2 * c]) = w[u];
    }
  };
  load(t0);
  D4 x[kFt];
#pragma unroll
  for (int t = 0; t < kFt; ++t) x[t] = ld4(dz + (size_t)min(atom, n - 1) * kFw + 16 * t + 4 * kk);
  stage(0);
  __syncthreads();
  int buf = 0;
  double* out = dX + (size_t)min(atom, n - 1) * nin + 4 * kk;
  for (int t = t0; t < tend; ++t) {
    if (t + 1 < tend) load(t + 1);
    const double* a = &sW[buf][ch * kLd + 4 * kk];
    D4 acc = D4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < kFt; ++s) {
      const D4 v = ld4(a + 16 * s);
#pragma unroll
      for (int r = 0; r < 4; ++r) acc = mfma16(v[r], x[s][r], acc);
    }
    buf ^= 1;
    if (t + 1 < tend) stage(buf);
    if (atom < n && 16 * t + 4 * kk < nin) {
      __builtin_nontemporal_store(D2{acc.x, acc.y}, reinterpret_cast<D2*>(out + 16 * t));
      __builtin_nontemporal_store(D2{acc.z, acc.w}, reinterpret_cast<D2*>(out + 16 * t + 2));
    }
    __syncthreads();
  }
}

constexpr int kCus = 256;
template <int N>
using Int = std::integral_constant<int, N>;
int ceil_div(int a, int b) { return (a + b - 1) / b; }

// The number of workgroups that share an atom group's tiles: a CU's time is
// its number of workgroups times the tiles of one.
void launch_input_grad(hipStream_t s, int n, int nin, const double* dz, const double* W, double* dX) {
  const int nag = ceil_div(n, 64), tiles = ceil_div(nin, 16);
  int groups = 1, best = ceil_div(nag, kCus) * tiles;
  for (int g = 2; g <= 64 && g <= tiles; ++g) {
    // a workgroup's own start (its dz) counts as one more tile
    const int c = ceil_div(nag * g, kCus) * (ceil_div(tiles, g) + 1);
    if (c < best) {
      best = c;
      groups = g;
    }
  }
  hipLaunchKernelGGL(fit_input_grad_kernel, dim3(kXcd * ceil_div(nag, kXcd) * groups), dim3(256), 0, s, n, nin, nag,
                     groups, ceil_div(tiles, groups), dz, W, dX);
}

// Few atoms: one launch per product.
int fit_240_small(hipStream_t s, int n, const dpc_fitting_net* net, const double* D, double* ws, int64_t np,
                  double* E, double* dD) {
  const int nin = net->n_in, at = ceil_div(n, 16);
  FitSmall f{n, nin, 0, D, net->W[0], net->b[0], net->w_out, ws, ws + np, ws + 2 * np, ws + 3 * np,
             ws + 4 * np, net->b_out, E, dD != nullptr};
  auto go = [&](auto kern, int ct, int kw, int kdim, const double* X, const double* W, const double* b) {
    f.kdim = kdim;
    f.groups = kFt / ct;
    f.X = X;
    f.W = W;
    f.bias = b;
    hipLaunchKernelGGL(kern, dim3(at * f.groups), dim3(64 * kw), 0, s, f);
  };
  // one tile per workgroup spreads a few atoms best (256: 52 us, 69 with three),
  // three share the loads of X (2,048: 158, 216 with one)
  const bool few = n <= 512;
  if (few) go(fit_small_kernel<1, 8, kStep1>, 1, 8, nin, D, net->W[0], net->b[0]);
  else go(fit_small_kernel<3, 8, kStep1>, 3, 8, nin, D, net->W[0], net->b[0]);
  auto step = [&](auto one, auto three, const double* X, const double* W, const double* b) {
    if (few) go(one, 1, 4, kFw, X, W, b);
    else go(three, 3, 4, kFw, X, W, b);
  };
  step(fit_small_kernel<1, 4, kStep2>, fit_small_kernel<3, 4, kStep2>, f.t1, net->W[1], net->b[1]);
  step(fit_small_kernel<1, 4, kStep3>, fit_small_kernel<3, 4, kStep3>, f.h2, net->W[2], net->b[2]);
  if (!dD) {
    hipLaunchKernelGGL(fit_energy_kernel, dim3(ceil_div(n, 256)), dim3(256), 0, s, f);
    return dpc_internal_launch_status();
  }
  step(fit_small_kernel<1, 4, kBack3>, fit_small_kernel<3, 4, kBack3>, f.dz, net->W[2], nullptr);
  step(fit_small_kernel<1, 4, kBack2>, fit_small_kernel<3, 4, kBack2>, f.t2, net->W[1], nullptr);
  launch_input_grad(s, n, nin, f.dz, net->W[0], dD);
  return dpc_internal_launch_status();
}

// Width 240, n_in a multiple of 4, 16-byte aligned buffers.  Tile shapes are
// chosen by how evenly they fill the CUs: a CU's time is its number of
// workgroups times the tiles of one, and larger tiles win ties (they read the
// activations less often).
int fit_240(hipStream_t s, int n, const dpc_fitting_net* net, const double* D, double* ws, int64_t np,
            double* E, double* dD) {
  const int nin = net->n_in, nag = ceil_div(n, 64);
  (void)hipGetLastError();
  // 2,048 atoms: 158 us, about 200 below; 3,000: 230 and 182
  if (n <= 2048) return fit_240_small(s, n, net, D, ws, np, E, dD);
  double *t1 = ws, *dz1 = ws + np;
  {
    auto cost = [&](int ct) { return ceil_div(nag * ceil_div(kFt, ct), kCus) * ct; };
    auto go = [&](auto kern, int ct) {
      hipLaunchKernelGGL(kern, dim3(kXcd * ceil_div(nag, kXcd) * ceil_div(kFt, ct)), dim3(256), 0, s, n, nin, nag, D,
                         net->W[0], net->b[0], t1);
    };
    const int best = std::min(std::min(cost(15), cost(5)), std::min(cost(4), cost(3)));
    if (cost(15) == best) go(fit_layer1_kernel<15, 16>, 15);
    else if (cost(5) == best) go(fit_layer1_kernel<5, 32>, 5);
    else if (cost(4) == best) go(fit_layer1_kernel<4, 32>, 4);
    else go(fit_layer1_kernel<3, 32>, 3);
  }
  auto middle = [&](auto kern, auto mt_, auto nw_) {
    constexpr int mt = decltype(mt_)::value, nw = decltype(nw_)::value;
    constexpr size_t lds = (kFw * (16 * mt + 4) + nw * 16 * mt) * sizeof(double);
    static_assert(lds <= kMaxLds, "a workgroup's LDS");
    hipLaunchKernelGGL(kern, dim3(ceil_div(n, 16 * mt)), dim3(64 * nw), lds, s, n, t1, net->W[1], net->b[1],
                       net->W[2], net->b[2], net->w_out, net->b_out, E, dD ? dz1 : nullptr);
  };
  // at most one workgroup of 16 atoms per CU: a tile per wavefront (4,096 atoms: 62 us, 85 with 32 atoms)
  if (n <= 16 * kCus) middle(fit_middle_kernel<1, 16>, Int<1>{}, Int<16>{});
  // three atom tiles where they leave fewer of them per CU (12,288 atoms: 256
  // workgroups, 131 us; 384 with two tiles, 163)
  else if (3 * ceil_div(ceil_div(n, 48), kCus) < 2 * ceil_div(ceil_div(n, 32), kCus))
    middle(fit_middle_kernel<3, 16>, Int<3>{}, Int<16>{});
  else middle(fit_middle_kernel<2, 8>, Int<2>{}, Int<8>{});
  if (dD) launch_input_grad(s, n, nin, dz1, net->W[0], dD);
  return dpc_internal_launch_status();
}

dim3 stream_grid(int64_t nw) {
  const int64_t b = (nw / 2 + 255) / 256;
  return dim3((unsigned)(b < 8192 ? (b > 0 ? b : 1) : 8192));
}

}  // namespace

extern "C" size_t dpc_fitting_workspace_bytes(int nloc, int width) {
  if (nloc < 0 || width < 1) return 0;
  const size_t nw = (size_t)nloc * width;
  return 5 * (nw + (nw & 1)) * sizeof(double);   // each array 16-byte aligned
}

extern "C" int dpc_fitting_fwd_bwd(void* stream, void* blas, int nloc, const dpc_fitting_net* net,
                                   const double* D, void* workspace, size_t workspace_bytes,
                                   double* E, double* dE_dD) {
  if (!net || nloc < 0) return DPC_EINVAL;
  const int nin = net->n_in, w = net->width;
  if (nin < 1 || w < 1) return DPC_EINVAL;
  for (int l = 0; l < 3; ++l)
    if (!net->W[l] || !net->b[l]) return DPC_EINVAL;
  if (!net->w_out) return DPC_EINVAL;
  if (nloc == 0) return DPC_OK;
  if (!blas || !D || !workspace || !E) return DPC_EINVAL;
  if (workspace_bytes < dpc_fitting_workspace_bytes(nloc, w)) return DPC_EINVAL;
  if ((uintptr_t)workspace % 16) return DPC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  rocblas_handle hb = static_cast<rocblas_handle>(blas);
  if (rocblas_set_stream(hb, s) != rocblas_status_success) return DPC_EHIP;
  // alpha and beta live on the host: host pointer mode for this call, the
  // caller's mode restored on every return
  struct ModeGuard {
    rocblas_handle h;
    rocblas_pointer_mode old = rocblas_pointer_mode_host;
    bool set = false;
    ~ModeGuard() {
      if (set) rocblas_set_pointer_mode(h, old);
    }
  } mode{hb};
  if (rocblas_get_pointer_mode(hb, &mode.old) != rocblas_status_success ||
      rocblas_set_pointer_mode(hb, rocblas_pointer_mode_host) != rocblas_status_success)
    return DPC_EHIP;
  mode.set = true;
  const int64_t nw = (int64_t)nloc * w;
  const uintptr_t all = (uintptr_t)D | (uintptr_t)dE_dD | (uintptr_t)net->W[0] | (uintptr_t)net->W[1] |
                        (uintptr_t)net->W[2] | (uintptr_t)net->b[0] | (uintptr_t)net->b[1] |
                        (uintptr_t)net->b[2] | (uintptr_t)net->w_out;
  if (w == kFw && nin % 4 == 0 && all % 16 == 0 && (int64_t)nloc * ((nin + 15) / 16) < (int64_t(1) << 31))
    return fit_240(s, nloc, net, D, static_cast<double*>(workspace), nw, E, dE_dD);
  double* ws = static_cast<double*>(workspace);
  const int64_t np = nw + (nw & 1);   // array pitch: keeps every array 16-byte aligned
  double* t1 = ws;            // tanh outputs of layers 1 and 2
  double* t2 = ws + np;
  double* h2 = ws + 2 * np;   // h_2 = t_1 + t_2
  double* z = ws + 3 * np;    // pre-activations, then dz
  double* e = ws + 4 * np;    // delta_l - w_out in the backward pass
  const double one = 1.0, zero = 0.0;
  (void)hipGetLastError();
  auto gemm_fwd = [&](const double* W, int in, const double* H) {
    return rocblas_dgemm(hb, rocblas_operation_none, rocblas_operation_none, w, nloc, in, &one, W, w,
                         H, in, &zero, z, w) == rocblas_status_success;
  };
  // dH^T = W dZ^T (+ beta C): the data gradient of one layer
  auto gemm_bwd = [&](const double* W, int in, const double* beta, double* C) {
    return rocblas_dgemm(hb, rocblas_operation_transpose, rocblas_operation_none, in, nloc, w, &one, W,
                         w, z, w, beta, C, in) == rocblas_status_success;
  };
  if (!gemm_fwd(net->W[0], nin, D)) return DPC_EHIP;
  hipLaunchKernelGGL(layer1_kernel, stream_grid(nw), dim3(256), 0, s, nw, w, z, net->b[0], t1);
  if (!gemm_fwd(net->W[1], w, t1)) return DPC_EHIP;
  hipLaunchKernelGGL(layer2_kernel, stream_grid(nw), dim3(256), 0, s, nw, w, z, net->b[1], t1, t2, h2);
  if (!gemm_fwd(net->W[2], w, h2)) return DPC_EHIP;
  // h_3 is used only by the energy: it is never stored; dz_3 replaces z_3
  hipLaunchKernelGGL(layer3_energy_kernel, dim3((nloc + 3) / 4), dim3(256), 0, s, nloc, w, z, net->b[2],
                     h2, net->w_out, net->b_out, E, dE_dD ? z : nullptr);
  if (dE_dD) {
    // delta_2 = w_out + W_3 dz_3; e holds delta - w_out so that the constant
    // delta_3 = w_out is never stored
    if (!gemm_bwd(net->W[2], w, &zero, e)) return DPC_EHIP;
    hipLaunchKernelGGL(tanh_grad_kernel, stream_grid(nw), dim3(256), 0, s, nw, w, t2, net->w_out, e, z);
    if (!gemm_bwd(net->W[1], w, &one, e)) return DPC_EHIP;   // delta_1 - w_out
    hipLaunchKernelGGL(tanh_grad_kernel, stream_grid(nw), dim3(256), 0, s, nw, w, t1, net->w_out, e, z);
    if (!gemm_bwd(net->W[0], nin, &zero, dE_dD)) return DPC_EHIP;
  }
  return dpc_internal_launch_status();
}
