// Propagator series and Wick contractions (FP64).
//
//  * eq. Dseries: terms[0] = S^(0), terms[i] = S^(i) - S^(i-1) (in place, from
//    the last level down) with every S^(i) zero outside its domain.
//  * Section 3 (eqs. W0, rall0, rall): t = tr{g5 S^(i)(x,x)} from the 12
//    point-source columns; pieces f, r1, r2 and the full product.
//  * Section 5.2 (eq. baryfact), C = i g0 g2, P_- = (1 - g0)/2, S_u = S_d = S:
//      W_N1 = eps^{abc} eps^{feg} tr[S^{ag T} C g5 S^{bf} C g5] tr[S^{ce} P_-]
//      W_N2 = eps^{abc} eps^{feg} tr[S^{ag T} C g5 S^{be} P_- S^{cf} C g5]
//    per sink site, then summed over each sink time slice (eq. baryN) in a
//    fixed order.
//  * Connected pseudoscalar (eqs. pipi, W0pc): W(y) = tr{S(y,x) S(y,x)^dag},
//    the sum of |S|^2 over the 144 entries at the sink, summed per time slice
//    and scaled by -1/L^3; series differences (eq. seriespi) and the rest
//    against the full propagator (eq. W0pc2).
//  * Stochastic traces (Section 6, eq. HPEtr and the estimator after it):
//    gamma5 on the sources, and sum_i sum_c conj(eta_i(x)_c) phi_i(x)_c per
//    site (sources, then components, in order) before the slice sums.
// In the chiral basis C = diag(s_2, -s_2), so C g5 = diag(s_2, s_2), and
// P_- = [[1,1],[1,1]]/2 in 2x2 spin blocks; both are applied in closed form below.
#include <mutex>

#include "ddml_common.hpp"
#include "launchers.hpp"

namespace ddml {

// terms[l] <- terms[l] - terms[l-1] (l >= 1) and sum <- terms[last] on the
// elements [lo, lo + len) of each of ncol columns (column stride cstride) of
// fields n apart; the elements outside hold zeros in every level.
__global__ void k_series_diff(double2* __restrict__ terms, size_t n, int nlevels, double2* __restrict__ sum,
                              int ncol, size_t cstride, size_t lo, size_t len) {
  const size_t total = (size_t)ncol * len;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < total; t += (size_t)gridDim.x * blockDim.x) {
    const size_t k = (t / len) * cstride + lo + t % len;
    double2 prev = terms[k];
    for (int l = 1; l < nlevels; ++l) {
      const double2 cur = terms[(size_t)l * n + k];
      terms[(size_t)l * n + k] = make_double2(cur.x - prev.x, cur.y - prev.y);
      prev = cur;
    }
    if (sum) sum[k] = prev;
  }
}

hipError_t launch_series_diff(double2* terms, size_t n, int nlevels, double2* sum, hipStream_t st, int ncol,
                              size_t cstride, size_t lo, size_t len) {
  if (ncol <= 0) {   // the whole field
    ncol = 1;
    cstride = n;
    lo = 0;
    len = n;
  }
  size_t g = ((size_t)ncol * len + 255) / 256;
  if (g > 16384) g = 16384;
  if (g == 0) return hipSuccess;
  hipLaunchKernelGGL(k_series_diff, dim3((int)g), dim3(256), 0, st, terms, n, nlevels, sum, ncol, cstride, lo, len);
  return hipGetLastError();
}

// ---------------------------------------------------- disconnected pseudoscalar
// S^(i)(x,x)[alpha a][beta b] = sum_{j<=i} terms[j][3 beta + b][x][alpha][a]
__device__ double2 g5_trace(const double2* __restrict__ terms, size_t V, int level, size_t site) {
  double2 t = make_double2(0, 0);
  for (int j = 0; j <= level; ++j)
    for (int col = 0; col < 12; ++col) {
      const int beta = col / 3, b = col % 3;
      const double2 v = terms[(((size_t)j * 12 + col) * V + site) * 12 + beta * 3 + b];
      const double sg = beta < 2 ? 1.0 : -1.0;   // (g5)_{beta beta}
      t.x += sg * v.x;
      t.y += sg * v.y;
    }
  return t;
}

__global__ void k_pp(const double2* __restrict__ tx_terms, const double2* __restrict__ ty_terms, size_t V,
                     int nlevels, size_t xs, size_t ys, double invL3, double2* __restrict__ out) {
  const int i = threadIdx.x;
  if (i >= nlevels) return;
  const double2 tx = g5_trace(tx_terms, V, i, xs), ty = g5_trace(ty_terms, V, i, ys);
  const double2 fx = g5_trace(tx_terms, V, nlevels - 1, xs), fy = g5_trace(ty_terms, V, nlevels - 1, ys);
  const double2 dx = make_double2(fx.x - tx.x, fx.y - tx.y), dy = make_double2(fy.x - ty.x, fy.y - ty.y);
  auto mul = [](double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); };
  const double2 f = mul(tx, ty);
  const double2 r1a = mul(dx, ty), r1b = mul(tx, dy);
  const double2 r2 = mul(dx, dy);
  const double2 full = mul(fx, fy);
  out[4 * i + 0] = make_double2(f.x * invL3, f.y * invL3);
  out[4 * i + 1] = make_double2((r1a.x + r1b.x) * invL3, (r1a.y + r1b.y) * invL3);
  out[4 * i + 2] = make_double2(r2.x * invL3, r2.y * invL3);
  out[4 * i + 3] = make_double2(full.x * invL3, full.y * invL3);
}

__global__ void k_g5_traces(const double2* __restrict__ terms, size_t V, int nlevels, size_t xs,
                            double2* __restrict__ out) {
  const int i = threadIdx.x;
  if (i < nlevels) out[i] = g5_trace(terms, V, i, xs);
}

hipError_t launch_g5_traces(const double2* terms, size_t V, int nlevels, size_t xs, double2* out, hipStream_t st) {
  hipLaunchKernelGGL(k_g5_traces, dim3(1), dim3(64), 0, st, terms, V, nlevels, xs, out);
  return hipGetLastError();
}

hipError_t launch_pp(const double2* tx, const double2* ty, size_t V, int nlevels, size_t xs, size_t ys, double invL3,
                     double2* out, hipStream_t st) {
  hipLaunchKernelGGL(k_pp, dim3(1), dim3(64), 0, st, tx, ty, V, nlevels, xs, ys, invL3, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ nucleon
__device__ __forceinline__ double2 cadd2(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }

// Sixteen lanes per sink site, lane 4 r + k holding the spin component (k, r) of
// the nine colour pairs S^{ag}; a workgroup is two wavefronts, eight sites.
// The levels are walked in order and S^(i) = sum_{j<=i} terms[j] stays in
// registers, so each term is read once and nothing goes through LDS; every
// sum over spin is between lanes of one 16-lane row, where a value moves with
// one or two DPP moves.  A quad of lanes loads a column's 192 bytes of a site as
// three runs of 64 and sorts them into spins the same way.
//
// With C g5 = diag(s_2, s_2), (C g5 S C g5)_{kr} = St_{kr} = +-S_{k^1, r^1} (+ for
// k = r mod 2), and P_- of rank 2 (see y, z), both traces are the same sum:
//   W_N1 - W_N2 = sum_{ag} sum_{kr} St^{ag}_{kr} G^{ag}_{kr},
//   G^{ag}_{kr} = sum eps^{abc} eps^{feg} [ p^{ce} S^{bf}_{kr} - sum_j y^{be}_{kj} z^{cf}_{jr} ],
//   y_{kj} = (S_{kj} + S_{k,j+2}) / 2,  z_{jr} = S_{jr} + S_{j+2,r},  p = tr[S P_-] = sum_k y_{k, k mod 2}:
// 126 complex products per lane instead of 57 per site for each of the 36 colour
// terms, with no operand read twice.  Sites where S^(i) vanishes (outside the
// outermost domain of the series) skip the algebra, which is exact: every
// product there is zero.
//
// Bound by its FP64 work with two waves per SIMD, near the time of reading the
// terms (0.75 ms at 6.1 TB/s for 3 levels of 48 x 24^3): 1.10 ms for the call,
// 1.37 with a lane per (k, r) that loaded its own components from four columns at
// once (80% of the time in the texture addresser), 2.59 when the 36 colour terms
// read their operands from LDS, sites 2304 bytes apart (one bank).
constexpr int kNucSites = 8;

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ double2 dpp(double2 v) {
  return make_double2(dpp<CTRL>(v.x), dpp<CTRL>(v.y));
}
constexpr int kQuadXor2 = 0x4E, kQuadXor3 = 0x1B;   // quad_perm: lane ^ 2, lane ^ 3
constexpr int kQuad0 = 0x00, kQuad1 = 0x55;         // quad_perm: lane 0 or 1 of each quad
constexpr int kRor8 = 0x128, kHalfMirror = 0x141;   // lane ^ 8, lane ^ 7 of the row
// lane ^ 4 and lane ^ 5
__device__ __forceinline__ double2 xor4(double2 v) { return dpp<kHalfMirror>(dpp<kQuadXor3>(v)); }
__device__ __forceinline__ double2 xor5(double2 v) { return dpp<kHalfMirror>(dpp<kQuadXor2>(v)); }
__device__ __forceinline__ double2 sel(bool c, double2 a, double2 b) {
  return make_double2(c ? a.x : b.x, c ? a.y : b.y);
}
// acc +- a b
__device__ __forceinline__ void mac(double2& acc, double2 a, double2 b) {
  acc.x += a.x * b.x;
  acc.x -= a.y * b.y;
  acc.y += a.x * b.y;
  acc.y += a.y * b.x;
}
__device__ __forceinline__ void msc(double2& acc, double2 a, double2 b) {
  acc.x -= a.x * b.x;
  acc.x += a.y * b.y;
  acc.y -= a.x * b.y;
  acc.y -= a.y * b.x;
}

// This lane's part of W_N1 - W_N2 of its site.  The two are summed apart, W_N1 waiting
// in LDS at *w1: one chain through both rounds a tenth worse, and a second pair of
// registers spills.
__device__ __forceinline__ double2 nucleon_lane(const double2 (&S)[3][3], int lane, double2* w1) {
  const bool odd = (lane >> 2) & 1;                  // r mod 2
  const bool minus = ((lane >> 2) ^ lane) & 1;       // k != r mod 2
  double2 W = make_double2(0, 0);
  auto St = [&](int a, int g) {
    const double2 v = xor5(S[a][g]);
    return minus ? make_double2(-v.x, -v.y) : v;
  };
  double2 ym[3][3], p[3][3];                         // y_{k, r mod 2}
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      const double2 u = dpp<kRor8>(S[a][g]);
      ym[a][g] = make_double2(0.5 * (S[a][g].x + u.x), 0.5 * (S[a][g].y + u.y));
      // the quads of even r hold y_{k0} and give y_00 + y_20, those of odd r y_11 + y_31
      const double2 t = cadd2(ym[a][g], dpp<kQuadXor2>(ym[a][g]));
      const double2 q = sel(odd, dpp<kQuad1>(t), dpp<kQuad0>(t));
      p[a][g] = cadd2(q, xor4(q));
    }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      const int b = (a + 1) % 3, c = (a + 2) % 3, f = (g + 1) % 3, e = (g + 2) % 3;
      double2 G = make_double2(0, 0);
      mac(G, p[c][e], S[b][f]);
      msc(G, p[c][f], S[b][e]);
      msc(G, p[b][e], S[c][f]);
      mac(G, p[b][f], S[c][e]);
      mac(W, St(a, g), G);
    }
  __builtin_amdgcn_sched_barrier(0);   // (nothing of W_N2 is started ahead of this: it would spill)
  *w1 = W;
  W = make_double2(0, 0);
  double2 yo[3][3], zm[3][3], zo[3][3];              // y_{k, 1 - r mod 2}, z_{r mod 2, r}, z_{1 - r mod 2, r}
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      yo[a][g] = xor4(ym[a][g]);
      const double2 z = cadd2(S[a][g], dpp<kQuadXor2>(S[a][g]));   // z_{k mod 2, r}
      const double2 z0 = dpp<kQuad0>(z), z1 = dpp<kQuad1>(z);
      zm[a][g] = sel(odd, z1, z0);
      zo[a][g] = sel(odd, z0, z1);
    }
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int g = 0; g < 3; ++g) {
      const int b = (a + 1) % 3, c = (a + 2) % 3, f = (g + 1) % 3, e = (g + 2) % 3;
      double2 G = make_double2(0, 0);
      mac(G, ym[b][e], zm[c][f]);
      mac(G, yo[b][e], zo[c][f]);
      msc(G, ym[b][f], zm[c][e]);
      msc(G, yo[b][f], zo[c][e]);
      msc(G, ym[c][e], zm[b][f]);
      msc(G, yo[c][e], zo[b][f]);
      mac(G, ym[c][f], zm[b][e]);
      mac(G, yo[c][f], zo[b][e]);
      msc(W, St(a, g), G);
    }
  return cadd2(*w1, W);
}

// P[level][block]: the sum over the workgroup's kNucSites sites (they lie in one
// time slice: every extent is even, so L^3 is a multiple of 8).
__global__ void __launch_bounds__(128, 2) k_nucleon(const double2* __restrict__ terms, size_t V, int nlevels,
                                                    double2* __restrict__ P) {
  __shared__ double2 part[2][2], w1[128];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r = (lane >> 2) & 3, k = lane & 3;
  const size_t y = (size_t)blockIdx.x * kNucSites + 4 * w + (lane >> 4);
  // column 3 r + b holds S[k a][r b] at component 3 k + a; lane k of the quad
  // loads components k, k + 4 and k + 8
  const DDML_GLOBAL f64x2* src = (const DDML_GLOBAL f64x2*)(terms + ((size_t)3 * r * V + y) * 12 + k);
  double2 S[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) S[a][b] = make_double2(0, 0);
  f64x2 next[3][3];
  auto load = [&](int level) {
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        next[b][j] = __builtin_nontemporal_load(src + ((size_t)level * 12 + b) * V * 12 + 4 * j);
  };
  load(0);
  bool live = false;
  for (int level = 0; level < nlevels; ++level) {
    bool any = false;
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int j = 0; j < 3; ++j) any = any || next[b][j].x != 0 || next[b][j].y != 0;
    if (__ballot(any)) {   // (uniform over the wavefront; a term of zeros leaves S as it is)
      live = true;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        double2 raw[3], v[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) raw[j] = make_double2(next[b][j].x, next[b][j].y);
        quad_to_spin(k, raw, v);
#pragma unroll
        for (int a = 0; a < 3; ++a) S[a][b] = cadd2(S[a][b], v[a]);
      }
    }
    if (level + 1 < nlevels) load(level + 1);
    double2 s = make_double2(0, 0);
    if (live) {
      s = nucleon_lane(S, lane, &w1[threadIdx.x]);
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) {
        s.x += __shfl_xor(s.x, off, 64);
        s.y += __shfl_xor(s.y, off, 64);
      }
    }
    if (lane == 0) part[level & 1][w] = s;
    __syncthreads();
    if (threadIdx.x == 0) P[(size_t)level * (V / kNucSites) + blockIdx.x] = cadd2(part[level & 1][0], part[level & 1][1]);
  }
}

// Fixed-order sum over each time slice: one workgroup per (level, t).
__global__ void k_slice_sum(const double2* __restrict__ W, size_t V, int T, double2* __restrict__ out) {
  const int level = blockIdx.y, t = blockIdx.x;
  const size_t V3 = V / T;
  __shared__ double2 part[256];
  double2 s = make_double2(0, 0);
  for (size_t k = threadIdx.x; k < V3; k += blockDim.x) {
    const double2 w = W[(size_t)level * V + (size_t)t * V3 + k];
    s.x += w.x;
    s.y += w.y;
  }
  part[threadIdx.x] = s;
  __syncthreads();
  for (int off = blockDim.x / 2; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) part[threadIdx.x] = cadd2(part[threadIdx.x], part[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[(size_t)level * T + t] = part[0];
}

// ---------------------------------------------------- connected pseudoscalar
// W[prop][site] = sum over the 12 columns and 12 components of |S|^2 (column
// by column, components in order).  Real, kept as double2 (im = 0) for the slice sum.
__global__ void k_pion_site(const double2* __restrict__ props, size_t V, double2* __restrict__ W) {
  const int prop = blockIdx.y;
  for (size_t y = blockIdx.x * (size_t)blockDim.x + threadIdx.x; y < V; y += (size_t)gridDim.x * blockDim.x) {
    double w = 0;
    for (int col = 0; col < 12; ++col) {
      const double2* v = props + (((size_t)prop * 12 + col) * V + y) * 12;
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const double2 e = v[c];
        w += e.x * e.x + e.y * e.y;
      }
    }
    W[(size_t)prop * V + y] = make_double2(w, 0.0);
  }
}

// out rows: [0, n) levels C^(i) = -sums[i]/L^3; [n, 2n) differences; 2n: rest.
__global__ void k_pion_fin(const double2* __restrict__ sums, int nlevels, int T, int has_full, double invL3,
                           double* __restrict__ out) {
  for (int t = threadIdx.x; t < T; t += blockDim.x) {
    double prev = 0;
    for (int i = 0; i < nlevels; ++i) {
      const double c = -sums[(size_t)i * T + t].x * invL3;
      out[(size_t)i * T + t] = c;
      out[(size_t)(nlevels + i) * T + t] = i == 0 ? c : c - prev;
      prev = c;
    }
    out[(size_t)2 * nlevels * T + t] = has_full ? -sums[(size_t)nlevels * T + t].x * invL3 - prev : 0.0;
  }
}

hipError_t launch_pion(const double2* props, size_t V, int T, int nprops, double2* W, double2* sums,
                       hipStream_t st) {
  size_t g = (V + 255) / 256;
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_pion_site, dim3((unsigned)g, nprops), dim3(256), 0, st, props, V, W);
  hipLaunchKernelGGL(k_slice_sum, dim3(T, nprops), dim3(256), 0, st, W, V, T, sums);
  return hipGetLastError();
}

hipError_t launch_pion_fin(const double2* sums, int nlevels, int T, int has_full, double invL3, double* out,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_pion_fin, dim3(1), dim3(256), 0, st, sums, nlevels, T, has_full, invL3, out);
  return hipGetLastError();
}

// ------------------------------------------------------- stochastic traces
// out = gamma5 in for n sites of canonical spinors (gamma5 = diag(1, 1, -1, -1))
__global__ void k_gamma5(const double2* __restrict__ in, double2* __restrict__ out, size_t n) {
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n * 12; k += (size_t)gridDim.x * blockDim.x) {
    const double2 v = in[k];
    const int comp = (int)(k % 12);
    out[k] = comp < 6 ? v : make_double2(-v.x, -v.y);
  }
}

__global__ void k_noise_dot(const double2* __restrict__ eta, const double2* __restrict__ phi, int nsrc, size_t V,
                            double2* __restrict__ W) {
  for (size_t y = blockIdx.x * (size_t)blockDim.x + threadIdx.x; y < V; y += (size_t)gridDim.x * blockDim.x) {
    double2 w = make_double2(0, 0);
    for (int i = 0; i < nsrc; ++i) {
      const double2* e = eta + ((size_t)i * V + y) * 12;
      const double2* f = phi + ((size_t)i * V + y) * 12;
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const double2 a = e[c], b = f[c];
        w.x += a.x * b.x + a.y * b.y;
        w.y += a.x * b.y - a.y * b.x;
      }
    }
    W[y] = w;
  }
}

hipError_t launch_gamma5(const double2* in, double2* out, size_t nsites, hipStream_t st) {
  size_t g = (nsites * 12 + 255) / 256;
  if (g > 16384) g = 16384;
  hipLaunchKernelGGL(k_gamma5, dim3((unsigned)g), dim3(256), 0, st, in, out, nsites);
  return hipGetLastError();
}

hipError_t launch_noise_trace(const double2* eta, const double2* phi, int nsrc, size_t V, int T, double2* W,
                              double2* sums, hipStream_t st) {
  size_t g = (V + 255) / 256;
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_noise_dot, dim3((unsigned)g), dim3(256), 0, st, eta, phi, nsrc, V, W);
  hipLaunchKernelGGL(k_slice_sum, dim3(T, 1), dim3(256), 0, st, W, V, T, sums);
  return hipGetLastError();
}

hipError_t launch_nucleon(const double2* terms, size_t V, int T, int nlevels, double2* P, double2* out,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_nucleon, dim3((unsigned)(V / kNucSites)), dim3(128), 0, st, terms, V, nlevels, P);
  hipLaunchKernelGGL(k_slice_sum, dim3(T, nlevels), dim3(256), 0, st, P, V / kNucSites, T, out);
  return hipGetLastError();
}

// ------------------------------------------- nucleon without allocations
// Scratch of the allocation-free nucleon contraction: the per-workgroup
// partial sums [nlevels][V / 8] complex.  One copy per device, resolved once
// per device with hipGetSymbolAddress and used through that address only (in
// host code the array's name is not a device address).  Every call on a
// device shares it; calls that overlap on one device race.
static __device__ __align__(256) double2 scratch[kNucScratchBytes / sizeof(double2)];

namespace {
std::mutex g_scratch_mu;
double2* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

hipError_t nucleon_scratch_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  if (cur != device) return hipErrorInvalidDevice;   // the caller makes `device` current
  void* p = nullptr;
  e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch_ptr[device] = static_cast<double2*>(p);
  return hipSuccess;
}

// diffs[0] = levels[0], diffs[i] = levels[i] - levels[i-1] (eq. seriesN)
__global__ void k_level_diffs(const double2* __restrict__ levels, int nlevels, int T, double2* __restrict__ diffs) {
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < T; t += gridDim.x * blockDim.x) {
    double2 prev = make_double2(0, 0);
    for (int i = 0; i < nlevels; ++i) {
      const double2 c = levels[(size_t)i * T + t];
      diffs[(size_t)i * T + t] = make_double2(c.x - prev.x, c.y - prev.y);
      prev = c;
    }
  }
}

hipError_t launch_nucleon_noalloc(const double2* terms, size_t V, int T, int nlevels, double2* levels,
                                  double2* diffs, int device, hipStream_t st) {
  if (device < 0 || device >= kMaxDevices || nlevels < 1 || T < 1 || V % ((size_t)T * kNucSites))
    return hipErrorInvalidValue;
  double2* P;
  hipError_t e;
  {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    P = g_scratch_ptr[device];
  }
  if (!P) return hipErrorNotInitialized;
  if ((size_t)nlevels * (V / kNucSites) * sizeof(double2) > kNucScratchBytes) return hipErrorInvalidValue;
  e = launch_nucleon(terms, V, T, nlevels, P, levels, st);
  if (e != hipSuccess) return e;
  if (diffs) hipLaunchKernelGGL(k_level_diffs, dim3((T + 63) / 64), dim3(64), 0, st, levels, nlevels, T, diffs);
  return hipGetLastError();
}

}  // namespace ddml
