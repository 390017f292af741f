// Even-odd Wilson-clover stencil kernels on domain-local boxes (gfx950).
//
// The hopping term H = D_hop of Section 6 (from the covariant differences of
// Appendix A):
//   (H psi)(x) = sum_mu [ (1 - g_mu) U_mu(x) psi(x+mu) + (1 + g_mu) U_mu(x-mu)^dag psi(x-mu) ].
// In the chiral basis g_mu = [[0, e_mu], [e_mu^dag, 0]] (e_0 = -1, e_k = -i s_k),
// so (1 -+ g_mu) psi = [h ; -+ e_mu^dag h] with the half spinor h = psi_u -+ e_mu psi_l.
// Only h (2 spins x 3 colours) is multiplied by the link, then the lower two
// spins are rebuilt; that halves the SU(3) work.
//
// One thread owns one site of the output parity and R right-hand sides; a
// workgroup is one 64-site tile (one wavefront per group of R columns), so the
// waves of one workgroup read the same links and clover data and hit in L1/L2
// instead of HBM.  Domain restriction comes from zeroed face links, so the
// inner loop has no masking branch.  Tiles are visited either linearly or in
// XCD bands (see ddml_common.hpp) so that neighbour tiles share an L2.
#include <algorithm>
#include <type_traits>

// No implicit contraction of a multiply and an add into one FMA in this file:
// every FMA of the stencil is written out (cmac, cmas, fmadd), so each site is
// computed by the same operations whatever launch variant or tile order the
// compiler sees around it, and all variants agree bit for bit by construction.
#pragma clang fp contract(off)

#include "ddml_common.hpp"
#include "launchers.hpp"

namespace ddml {

// ---------------------------------------------------------------- spin maths
template <typename T2>
__device__ __forceinline__ void project(int mu, bool fwd, const T2 psi[12], T2 h[6]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T2 p0 = psi[c], p1 = psi[3 + c], p2 = psi[6 + c], p3 = psi[9 + c];
    T2 h0, h1;
    switch (mu) {
      case 0:
        h0 = fwd ? cadd(p0, p2) : csub(p0, p2);
        h1 = fwd ? cadd(p1, p3) : csub(p1, p3);
        break;
      case 1:
        h0 = fwd ? cadd(p0, ci(p3)) : csub(p0, ci(p3));
        h1 = fwd ? cadd(p1, ci(p2)) : csub(p1, ci(p2));
        break;
      case 2:
        h0 = fwd ? cadd(p0, p3) : csub(p0, p3);
        h1 = fwd ? csub(p1, p2) : cadd(p1, p2);
        break;
      default:
        h0 = fwd ? cadd(p0, ci(p2)) : csub(p0, ci(p2));
        h1 = fwd ? csub(p1, ci(p3)) : cadd(p1, ci(p3));
        break;
    }
    h[c] = h0;
    h[3 + c] = h1;
  }
}

template <typename T2>
__device__ __forceinline__ void reconstruct(int mu, bool fwd, const T2 g[6], T2 acc[12]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T2 g0 = g[c], g1 = g[3 + c];
    acc[c] = cadd(acc[c], g0);
    acc[3 + c] = cadd(acc[3 + c], g1);
    switch (mu) {
      case 0:
        acc[6 + c] = fwd ? cadd(acc[6 + c], g0) : csub(acc[6 + c], g0);
        acc[9 + c] = fwd ? cadd(acc[9 + c], g1) : csub(acc[9 + c], g1);
        break;
      case 1:
        acc[6 + c] = fwd ? cadd(acc[6 + c], cmi(g1)) : cadd(acc[6 + c], ci(g1));
        acc[9 + c] = fwd ? cadd(acc[9 + c], cmi(g0)) : cadd(acc[9 + c], ci(g0));
        break;
      case 2:
        acc[6 + c] = fwd ? csub(acc[6 + c], g1) : cadd(acc[6 + c], g1);
        acc[9 + c] = fwd ? cadd(acc[9 + c], g0) : csub(acc[9 + c], g0);
        break;
      default:
        acc[6 + c] = fwd ? cadd(acc[6 + c], cmi(g0)) : cadd(acc[6 + c], ci(g0));
        acc[9 + c] = fwd ? cadd(acc[9 + c], ci(g1)) : cadd(acc[9 + c], cmi(g1));
        break;
    }
  }
}

// reconstruct with a scale s folded in (acc += s times the rebuilt spinor):
// every add is a fused multiply-add by s, so a 16-bit input spinor's per-site
// scale is applied here once instead of to each of its loaded components
template <typename T2>
__device__ __forceinline__ void reconstruct_s(int mu, bool fwd, const T2 g[6], decltype(T2::x) s, T2 acc[12]) {
  const decltype(T2::x) m = -s;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const T2 g0 = g[c], g1 = g[3 + c];
    acc[c] = cmas(acc[c], g0, s);
    acc[3 + c] = cmas(acc[3 + c], g1, s);
    switch (mu) {
      case 0:
        acc[6 + c] = cmas(acc[6 + c], g0, fwd ? s : m);
        acc[9 + c] = cmas(acc[9 + c], g1, fwd ? s : m);
        break;
      case 1:
        acc[6 + c] = cmas(acc[6 + c], fwd ? cmi(g1) : ci(g1), s);
        acc[9 + c] = cmas(acc[9 + c], fwd ? cmi(g0) : ci(g0), s);
        break;
      case 2:
        acc[6 + c] = cmas(acc[6 + c], g1, fwd ? m : s);
        acc[9 + c] = cmas(acc[9 + c], g0, fwd ? s : m);
        break;
      default:
        acc[6 + c] = cmas(acc[6 + c], fwd ? cmi(g0) : ci(g0), s);
        acc[9 + c] = cmas(acc[9 + c], fwd ? ci(g1) : cmi(g1), s);
        break;
    }
  }
}

// g = U h (dag=false) or U^dag h (dag=true), per spin of the half spinor;
// every complex multiply-add is four fused multiply-adds
template <typename T2>
__device__ __forceinline__ void su3_mul(const T2 u[9], bool dag, const T2 h[6], T2 g[6]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      T2 acc = mk<T2>(0, 0);
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (!dag) acc = cmac(acc, u[3 * a + b], h[3 * s + b]);
        else acc = cmacc(acc, u[3 * b + a], h[3 * s + b]);
      }
      g[3 * s + a] = acc;
    }
}

// g = W h per spin of the half spinor, W a link staged in LDS as 5 pairs of
// its 9 row-major entries (pair k at ul + 128 k): each row is read when it is
// needed, so at most a row and a half of W is live.  Every g is the same
// sequence of fused multiply-adds as su3_mul (with W = U^dag for a backward
// hop, conj(u) * h in cmacc is the product w * h in cmac).
template <typename T2>
__device__ __forceinline__ void su3_rows(const T2* ul, const T2 h[6], T2 g[6]);

// Loads of one pair from the LDS staging area of a tile (same pair stride as
// the global layout: pair k of lane l at base + 128 k, base = area + 2 l).
__device__ __forceinline__ void lds2(const float2* p, float2& a, float2& b) {
  const f32x4 v = *(const __attribute__((address_space(3))) f32x4*)p;
  a = make_float2(v.x, v.y);
  b = make_float2(v.z, v.w);
}
__device__ __forceinline__ void lds2(const double2* p, double2& a, double2& b) {
  const __attribute__((address_space(3))) f64x2* q = (const __attribute__((address_space(3))) f64x2*)p;
  const f64x2 u = q[0], v = q[1];
  a = make_double2(u.x, u.y);
  b = make_double2(v.x, v.y);
}
__device__ __forceinline__ void sts2(float2* p, float2 a, float2 b) {
  f32x4 v;
  v.x = a.x; v.y = a.y; v.z = b.x; v.w = b.y;
  *(__attribute__((address_space(3))) f32x4*)p = v;
}
__device__ __forceinline__ void sts2(double2* p, double2 a, double2 b) {
  __attribute__((address_space(3))) f64x2* q = (__attribute__((address_space(3))) f64x2*)p;
  f64x2 u, v;
  u.x = a.x; u.y = a.y; v.x = b.x; v.y = b.y;
  q[0] = u;
  q[1] = v;
}

template <typename T2>
__device__ __forceinline__ void su3_row(const T2 w0, const T2 w1, const T2 w2, const T2 h[6], int a, T2 g[6]) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    T2 acc = mk<T2>(0, 0);
    acc = cmac(acc, w0, h[3 * s]);
    acc = cmac(acc, w1, h[3 * s + 1]);
    acc = cmac(acc, w2, h[3 * s + 2]);
    g[3 * s + a] = acc;
  }
}
template <typename T2>
__device__ __forceinline__ void su3_rows(const T2* ul, const T2 h[6], T2 g[6]) {
  T2 w0, w1, w2, w3, w4, w5, w6, w7, w8, wp;
  lds2(ul, w0, w1);
  lds2(ul + 128, w2, w3);
  su3_row(w0, w1, w2, h, 0, g);
  lds2(ul + 256, w4, w5);
  su3_row(w3, w4, w5, h, 1, g);
  lds2(ul + 384, w6, w7);
  lds2(ul + 512, w8, wp);
  su3_row(w6, w7, w8, h, 2, g);
}

// 18 slots of one Hermitian 6x6 block (9 pairs, pair k at base + 128 k)
template <typename T2>
__device__ __forceinline__ void herm6_load(const T2* __restrict__ base, T2 m[18]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) ld2nt(base + 128 * k, m[2 * k], m[2 * k + 1]);
}
template <typename T2>
__device__ __forceinline__ void herm6_load_lds(const T2* base, T2 m[18]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) lds2(base + 128 * k, m[2 * k], m[2 * k + 1]);
}
// the 12 components of a spinor (6 pairs) starting at base
template <typename T2>
__device__ __forceinline__ void spinor_load(const T2* __restrict__ base, T2 v[12]) {
#pragma unroll
  for (int k = 0; k < 6; ++k) ld2(base + 128 * k, v[2 * k], v[2 * k + 1]);
}
template <typename T2>
__device__ __forceinline__ void spinor_store(T2* __restrict__ base, const T2 v[12]) {
#pragma unroll
  for (int k = 0; k < 6; ++k) st2(base + 128 * k, v[2 * k], v[2 * k + 1]);
}
// streaming spinor access: fields read or written once per stencil launch
template <typename T2>
__device__ __forceinline__ void spinor_load_nt(const T2* __restrict__ base, T2 v[12]) {
#pragma unroll
  for (int k = 0; k < 6; ++k) ld2nt(base + 128 * k, v[2 * k], v[2 * k + 1]);
}
template <typename T2>
__device__ __forceinline__ void spinor_store_nt(T2* __restrict__ base, const T2 v[12]) {
#pragma unroll
  for (int k = 0; k < 6; ++k) st2nt(base + 128 * k, v[2 * k], v[2 * k + 1]);
}
template <typename T2>
__device__ __forceinline__ void herm6_apply(const T2 m[18], const T2 x[6], T2 y[6]) {
  using T = decltype(T2::x);
  T d[6] = {m[0].x, m[0].y, m[1].x, m[1].y, m[2].x, m[2].y};
#pragma unroll
  for (int i = 0; i < 6; ++i) y[i] = cscale(x[i], d[i]);
  int k = 3;
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int j = i + 1; j < 6; ++j) {
      const T2 h = m[k++];
      y[i] = cmac(y[i], h, x[j]);
      y[j] = cmacc(y[j], h, x[i]);
    }
}

// y = M x for one Hermitian 6x6 block staged in LDS (18 slots in 9 pairs:
// the diagonal packed in slots 0..2, then the 15 upper entries, row by row),
// reading each pair when it is needed: the same operations in the same order
// as herm6_apply on the whole block.
template <typename T2>
__device__ __forceinline__ void herm6_apply_lds(const T2* base, const T2 x[6], T2 y[6]) {
  T2 m0, m1;
  lds2(base, m0, m1);
  y[0] = cscale(x[0], m0.x);
  y[1] = cscale(x[1], m0.y);
  y[2] = cscale(x[2], m1.x);
  y[3] = cscale(x[3], m1.y);
  lds2(base + 128, m0, m1);
  y[4] = cscale(x[4], m0.x);
  y[5] = cscale(x[5], m0.y);
  // slot k (k >= 3) holds entry (i, j) of the upper triangle, row by row
  T2 h = m1;   // slot 3
  int k = 3;
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int j = i + 1; j < 6; ++j) {
      if (k > 3) {
        if (k & 1) {
          h = m1;
        } else {
          lds2(base + 128 * (k >> 1), m0, m1);
          h = m0;
        }
      }
      y[i] = cmac(y[i], h, x[j]);
      y[j] = cmacc(y[j], h, x[i]);
      ++k;
    }
}

// ------------------------------------------------------------ the stencil core
// LDS staging of the operator data of one tile (ST = true): the links of the
// 8 hops of every site ([hop = 2 mu + backward][5 pairs]) and the 18 clover
// pairs, as [58 pairs][64 lanes][2] complex (the pair stride of the global
// layout).  The workgroup reads them from HBM/L2 once instead of once per
// wavefront (12 wavefronts share a tile at R = 1).  FP64 links are read whole;
// the FP32 and 16-bit copies hold the first two rows of each link (3 pairs)
// and the third is rebuilt here, as conj(row 0 x row 1) for an SU(3) matrix,
// times -1 for the time links of the last slice of a box that spans the
// whole antiperiodic time extent (the sign folded into the stored rows
// cancels in the cross product); a zeroed face link rebuilds to zero.  One
// wavefront stages all of a link, so one barrier closes the staging.  A
// backward hop's link is staged as U^dag (conjugated transpose), so every hop
// multiplies by the rows of its staged matrix (su3_rows).
constexpr int kStageLinkPairs = 8 * 5;
constexpr int kStagePairs = kStageLinkPairs + 18;

template <typename E>
constexpr bool kIs16 = std::is_same<E, h16c>::value;
template <typename E>
constexpr bool kTwoRow = !std::is_same<E, double2>::value;

// one pair of a staged field (16-bit: dequantised with scale sc)
template <typename E, typename C>
__device__ __forceinline__ void stage_load(const E* src, float sc, C& a, C& b) {
  if constexpr (kIs16<E>) {
    ld2q_nt(src, a, b);
    a = make_float2(a.x * sc, a.y * sc);
    b = make_float2(b.x * sc, b.y * sc);
  } else {
    ld2nt(src, a, b);
  }
}

// E: element type of the fields (float2, double2 or 16-bit h16c); C: compute type.
template <typename E, typename C = typename CompOf<E>::type>
__device__ __forceinline__ void stage_tile(const BoxGeom& g, const E* __restrict__ U, const E* __restrict__ clov,
                                           const float* __restrict__ clov_n, int p, int tile, C* sm) {
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6, W = blockDim.x >> 6;
  const int i = tile * kTile + lane;
  const bool valid = i < g.Vh;
  const int nt = g.ntiles;
  const int q = 1 - p;
  int y[4] = {0, 0, 0, 0};
  if (valid) eo_coords(g, p, i, y);
  const C z = mk<C>(0, 0);
  // No load here stands behind a branch on valid: padding sites have their
  // places (and hold zeros), and a load per branch is a trip to memory each,
  // three of a link and two of the clover data (solves of 12 columns: 8^3 x 8
  // 9.69 -> 9.31 ms, 32^3 x 16 328.8 -> 324.0 ms).  Two clover pairs in flight
  // and not more: the even half then spills, and with the pairs loaded ahead of
  // the links, or by the four waves without a link, 8^3 x 8 takes 9.30 and
  // 9.20 ms but 32^3 x 16 332.5 and 327.9.
  // links: hop h = 2 mu + backward, forward from this site, backward from y - mu
  for (int h = w; h < 8; h += W) {
    const int mu = h >> 1;
    const bool bwd = h & 1;
    int par = p, site = i;
    if (valid && bwd) {
      int zz[4] = {y[0], y[1], y[2], y[3]};
      zz[mu] = (y[mu] == 0) ? g.L[mu] - 1 : y[mu] - 1;
      par = q;
      site = eo_index(g, zz);
    }
    C e[10];
    if constexpr (kTwoRow<E>) {
#pragma unroll
      for (int k = 0; k < 3; ++k) stage_load<E, C>(U + lidx2(nt, par, mu, 2 * k, site), 1.0f / kQ, e[2 * k], e[2 * k + 1]);
      // the time link of the box's last slice, if it carries the antiperiodic sign
      const bool flip = g.twrap && mu == 0 && valid && (bwd ? y[0] == 0 : y[0] == g.L[0] - 1);
#pragma unroll
      for (int c3 = 0; c3 < 3; ++c3) {
        const int a = (c3 + 1) % 3, b = (c3 + 2) % 3;
        C v = csub(cmul(e[a], e[3 + b]), cmul(e[b], e[3 + a]));
        e[6 + c3] = flip ? mk<C>(-v.x, v.y) : mk<C>(v.x, -v.y);
      }
      e[9] = z;
    } else {
#pragma unroll
      for (int k = 0; k < 5; ++k) ld2nt(U + lidx(nt, par, mu, 2 * k, site), e[2 * k], e[2 * k + 1]);
    }
    if (bwd) {   // the hop multiplies by U^dag: stage it as such (rows of U^dag = conj columns of U)
      C t[9];
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) t[3 * a + b] = mk<C>(e[3 * b + a].x, -e[3 * b + a].y);
#pragma unroll
      for (int k = 0; k < 9; ++k) e[k] = t[k];
    }
#pragma unroll
    for (int k = 0; k < 5; ++k) sts2(sm + (h * 5 + k) * 128 + lane * 2, e[2 * k], e[2 * k + 1]);
  }
  // clover data of the output parity, kClov pairs in flight
  constexpr int kClov = 2;
  float sc = 1.0f / kQ;
  if constexpr (kIs16<E>) sc = ldgf(clov_n + (size_t)p * nt * kTile + i) / kQ;
  for (int j0 = w; j0 < 18; j0 += kClov * W) {
    C a[kClov], b[kClov];
#pragma unroll
    for (int k = 0; k < kClov; ++k)   // (past the end: the last pair again, not kept)
      stage_load<E, C>(clov + cidx(nt, p, 2 * min(j0 + k * W, 17), i), sc, a[k], b[k]);
#pragma unroll
    for (int k = 0; k < kClov; ++k)
      if (j0 + k * W < 18) sts2(sm + (kStageLinkPairs + j0 + k * W) * 128 + lane * 2, a[k], b[k]);
  }
  __syncthreads();
}

// on: bit r set if column r0 + r is active (read once per tile by the caller,
// so the direction loop has no load-dependent branch and its loads can overlap)
template <typename E, int R, bool ST, typename C = typename CompOf<E>::type>
__device__ __forceinline__ void hop_sum(const BoxGeom& g, int p, int i, const E* __restrict__ U, const C* sm,
                                        const E* __restrict__ in, const float* __restrict__ in_n, int r0, int nr,
                                        unsigned on, C acc[R][12]) {
  int y[4];
  eo_coords(g, p, i, y);
  const int q = 1 - p;
  const int nt = g.ntiles;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[r][c] = mk<C>(0, 0);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
      const bool fwd = dir == 0;
      int z[4] = {y[0], y[1], y[2], y[3]};
      if (fwd) z[mu] = (y[mu] + 1 == g.L[mu]) ? 0 : y[mu] + 1;
      else z[mu] = (y[mu] == 0) ? g.L[mu] - 1 : y[mu] - 1;
      const int n = eo_index(g, z);
      C u[10];
      const C* ul = nullptr;
      if constexpr (ST) {
        ul = sm + (2 * mu + dir) * 5 * 128 + (i & 63) * 2;
      } else {
        static_assert(!kTwoRow<E>, "two-row links (FP32, 16-bit) are read through the LDS staging only");
        const E* __restrict__ ug = fwd ? U + lidx(nt, p, mu, 0, i) : U + lidx(nt, q, mu, 0, n);
#pragma unroll
        for (int k = 0; k < 5; ++k) ld2nt(ug + 128 * k, u[2 * k], u[2 * k + 1]);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r < nr && ((on >> r) & 1u)) {
          C psi[12], h[6], gg[6];
          if constexpr (kIs16<E>) {
            // the stored integers are projected and multiplied as they are
            // (a sum of two of them is exact in 32 bits and in FP32) and the
            // spinor's scale enters once, in the fused rebuild.  Summed before
            // they are converted: 12 conversions per hop instead of 24, 1944
            // instead of 2040 vector instructions in the odd half (16-bit
            // solves of 16^3 x 8, 32^3 x 16: 15.50 -> 15.27, 245 -> 241.6 ms)
            const h16c* b = in + qidx(nt, r0 + r, n);
            const float sc = ldgf(in_n + (size_t)(r0 + r) * nt * kTile + n) * (1.0f / kQ);
            s16x8 w[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) w[k] = *(const DDML_GLOBAL s16x8*)(b + 256 * k);
            __builtin_amdgcn_sched_barrier(0);
            int2 pq[12], hq[6];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
              for (int j = 0; j < 4; ++j) pq[4 * k + j] = make_int2(w[k][2 * j], w[k][2 * j + 1]);
            project(mu, fwd, pq, hq);
#pragma unroll
            for (int c = 0; c < 6; ++c) h[c] = make_float2((float)hq[c].x, (float)hq[c].y);
            su3_rows(ul, h, gg);
            reconstruct_s(mu, fwd, gg, sc, acc[r]);
          } else {
            spinor_load(in + fidx(nt, r0 + r, 0, n), psi);
            project(mu, fwd, psi, h);
            if constexpr (ST) su3_rows(ul, h, gg);
            else su3_mul(u, !fwd, h, gg);
            reconstruct(mu, fwd, gg, acc[r]);
          }
        }
      }
    }
  }
}

__device__ __forceinline__ double2 wave_sum(double2 v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    v.x += __shfl_xor(v.x, off, 64);
    v.y += __shfl_xor(v.y, off, 64);
  }
  return v;
}

// Epilogue on one column.  acc = (H in)(x); cl points at slot 0 of this site.
template <typename T2, int MODE, bool ST>
__device__ __forceinline__ void epilogue_block(const T2* cl, int b, const T2 acc[6], const T2 aux[6], const T2 ra[6],
                                               double c1, T2 out[6]) {
  using T = decltype(T2::x);
  const T k1 = (T)c1;
  T2 m[18];
  const T2* cb = cl + 128 * 9 * b;
  if (!ST) herm6_load(cb, m);
  auto apply = [&](const T2 x[6], T2 y[6]) {
    if (ST) herm6_apply_lds(cb, x, y);
    else herm6_apply(m, x, y);
  };
  if (MODE == MODE_CINV_HOP) {
    apply(acc, out);
  } else if (MODE == MODE_SCHUR) {
    T2 y[6];
    apply(acc, y);
#pragma unroll
    for (int c = 0; c < 6; ++c) out[c] = cmas(aux[c], y[c], -k1);
  } else if (MODE == MODE_RES) {
    T2 y[6];
    apply(aux, y);
#pragma unroll
    for (int c = 0; c < 6; ++c) out[c] = csub(ra[c], cmas(y[c], acc[c], -k1));
  } else {  // MODE_PREP: out = C (aux + c1 acc)
    T2 v[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) v[c] = cmas(aux[c], acc[c], k1);
    apply(v, out);
  }
}

// The epilogue on the two chiral blocks of one column (acc = (H in)(x); cl
// points at slot 0 of this site's clover data).
template <typename T2, int MODE, bool ST>
__device__ __forceinline__ void epilogue(const T2* cl, const T2 acc[12], const T2 aux[12],
                                         const T2 ra[12], double c1, T2 out[12]) {
#pragma unroll
  for (int b = 0; b < 2; ++b)
    epilogue_block<T2, MODE, ST>(cl, b, acc + 6 * b, aux + 6 * b, ra + 6 * b, c1, out + 6 * b);
}

// The fused reductions of one output column over its components [c0, c0 + N)
// (o the output, av the aux field), each accumulated in component order.
template <int RED, int N, typename C>
__device__ __forceinline__ void fused_reductions(unsigned hb, int c0, const C o[N], const C av[N], double2& s0,
                                                 double2& s1, double2& s2) {
  if (RED == RED_DOT) {
    shadow_dot_part<C, N>(hb, c0, o, s0);
  } else if (RED == RED_TS) {
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const double ox = o[c].x, oy = o[c].y, ax = av[c].x, ay = av[c].y;
      s0.x = fmadd(ox, ax, fmadd(oy, ay, s0.x));
      s0.y = fmadd(ox, ay, fmadd(-oy, ax, s0.y));
      s1.x = fmadd(ox, ox, fmadd(oy, oy, s1.x));
    }
    shadow_dot_part<C, N>(hb, c0, o, s2);
  } else if (RED == RED_NORM) {
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const double ox = o[c].x, oy = o[c].y;
      s0.x = fmadd(ox, ox, fmadd(oy, oy, s0.x));
    }
  }
}

// Field arguments of one tile launch: element pointers and, for 16-bit
// fields, their per-(site, column) scales.
template <typename E> struct TileArgs {
  const E* U;
  const E* clov;
  const float* clov_n;
  const E* in;
  const float* in_n;
  const E* aux;
  const float* aux_n;
  const E* red_a;
  const float* red_n;
  E* out;
  float* out_n;
};

// The columns that are active as a mask: lane c loads the flag of column c, so
// that one load serves the workgroup's test and every wave's own (a load of its
// own for each was two more trips to memory per tile).
__device__ __forceinline__ int active_flag(const int* active, int nrhs) {
  const int lane = threadIdx.x & 63;
  return ldg(active + min(lane, nrhs - 1));
}
__device__ __forceinline__ unsigned active_of(int flag) { return (unsigned)__ballot(flag != 0); }

// One tile on the output parity p.  ST: the tile's links and clover data are
// staged in LDS at sm (stage_tile) and taken from there.  16-bit outputs are
// quantised before the fused reductions, so the dot products are those of the
// stored vectors.
template <typename E, int R, int MODE, int RED, bool ST = false, typename C = typename CompOf<E>::type>
__device__ __forceinline__ void hop_tile(const BoxGeom g, const TileArgs<E>& a, double2* __restrict__ partial,
                                         unsigned act, int p, int nrhs, double c1, int tile,
                                         int wave0 = 0, const C* sm = nullptr) {
  const int lane = threadIdx.x & 63;
  const int grp = wave0 + (threadIdx.x >> 6);
  const int r0 = grp * R;
  if (r0 >= nrhs) return;  // whole wave idle (uniform)
  const int nr = min(R, nrhs - r0);
  const int i = tile * kTile + lane;
  const bool valid = i < g.Vh;
  const int nt = g.ntiles;
  unsigned on = 0;  // active columns of this wavefront
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (r < nr && ((act >> (r0 + r)) & 1u)) on |= 1u << r;
  if (on == 0) return;  // uniform across the wave
  C acc[R][12];
  if (valid) hop_sum<E, R, ST>(g, p, i, a.U, sm, a.in, a.in_n, r0, nr, on, acc);
  // keep the epilogue's loads after the hop sum: hoisted above it they would
  // stay live through the hop loop and cost occupancy
  __builtin_amdgcn_sched_barrier(0);
  const C* cl;
  if constexpr (ST) cl = sm + kStageLinkPairs * 128 + lane * 2;
  else cl = a.clov + cidx(nt, p, 0, i);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r >= nr) break;
    const int col = r0 + r;
    if (!((on >> r) & 1u)) continue;  // uniform across the wave
    double2 s0 = make_double2(0, 0), s1 = make_double2(0, 0), s2 = make_double2(0, 0);
    const size_t base = fidx(nt, col, 0, i);
    const size_t ns = (size_t)col * nt * kTile + i;  // scale index of 16-bit fields
    if (valid) {
      const unsigned hb = shadow_bits(col, i);
      if constexpr (kIs16<E>) {
        // one scale over the 12 output components, so the epilogue runs on all
        // of them before the store.  To stay within the register budget it
        // works in place: the aux components become the output, the store
        // returns the stored values in the same registers, and the (t, s)
        // sums read aux again (the first load leaves it in cache for that)
        C w[12], ra[12];
        const size_t qb = qidx(nt, col, i);
        if (MODE != MODE_CINV_HOP) spinor_load_q(a.aux + qb, ldgf(a.aux_n + ns), w, RED != RED_TS);
        if (MODE == MODE_RES) spinor_load_q(a.red_a + qb, ldgf(a.red_n + ns), ra, true);
        epilogue<C, MODE, ST>(cl, acc[r], w, ra, c1, w);
        spinor_store_q(a.out + qb, a.out_n + ns, w, w, true);
        if constexpr (RED == RED_TS) {
          C av[12];
          spinor_load_q(a.aux + qb, ldgf(a.aux_n + ns), av, true);
          fused_reductions<RED, 12>(hb, 0, w, av, s0, s1, s2);
        } else {
          fused_reductions<RED, 12>(hb, 0, w, w, s0, s1, s2);
        }
      } else {
        // chiral block by block: aux in, 6x6 clover block, out, reductions
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          C av[6], ra[6], o[6];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            if (MODE != MODE_CINV_HOP) ld2nt(a.aux + base + 128 * (3 * b + k), av[2 * k], av[2 * k + 1]);
            if (MODE == MODE_RES) ld2nt(a.red_a + base + 128 * (3 * b + k), ra[2 * k], ra[2 * k + 1]);
          }
          epilogue_block<C, MODE, ST>(cl, b, acc[r] + 6 * b, av, ra, c1, o);
#pragma unroll
          for (int k = 0; k < 3; ++k) st2nt(a.out + base + 128 * (3 * b + k), o[2 * k], o[2 * k + 1]);
          fused_reductions<RED, 6>(hb, 6 * b, o, av, s0, s1, s2);
        }
      }
    } else {
      // padding sites of the last tile stay zero
      C z[12], zq[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) z[c] = mk<C>(0, 0);
      if constexpr (kIs16<E>) spinor_store_q(a.out + qidx(nt, col, i), a.out_n + ns, z, zq, false);
      else spinor_store(a.out + base, z);
    }
    if (RED != RED_NONE) {
      s0 = wave_sum(s0);
      if (RED == RED_TS) {
        s1 = wave_sum(s1);
        s2 = wave_sum(s2);
      }
      if (lane == 0) {
        stg2(partial + (size_t)col * nt + tile, s0);
        if (RED == RED_TS) {
          stg2(partial + ((size_t)nrhs + col) * nt + tile, s1);
          stg2(partial + ((size_t)2 * nrhs + col) * nt + tile, s2);
        }
      }
    }
  }
}

// Banded tile order of one box for XCD x: the box is nslice slices of S
// tiles (S = tps, or the whole box if a slice is not a whole number of tiles);
// XCD x owns tiles [x S / 8, (x+1) S / 8) of every slice, slice after slice.
__device__ __forceinline__ void band_of(int ntiles, int tps, int x, int& S, int& lo, int& bs) {
  S = tps > 0 ? tps : ntiles;
  lo = (int)((long)x * S / kXcd);
  bs = (int)((long)(x + 1) * S / kXcd) - lo;
}
__device__ __forceinline__ int band_tile(int S, int lo, int bs, int local) {
  return (local / bs) * S + lo + local % bs;
}

// Single-item launch (apply_eo in FP64, outer FP64 steps).  Every column is
// active, by a mask that the compiler does not see and that is set anew for each
// tile: from a constant, or a mask made before the loop over tiles, it moves loads
// of the epilogue above the hops and spills (47 to 1517 registers with a constant,
// 59, 62 and 63 at R = 1 with a mask per launch; 0, 10 and 10 this way).  Bound
// by links and clover data that every wave reads itself, it takes the same time with
// those 60 registers spilled (24^3 x 16: 0.212 ms with 1 column, 1.51 with 12).
__device__ __forceinline__ unsigned all_columns() {
  unsigned m;
  asm volatile("s_mov_b32 %0, -1" : "=s"(m));
  return m;
}
template <typename T2, int R, int MODE, int RED>
__global__ void __launch_bounds__(64 * ((kMaxRhs + R - 1) / R)) k_hop_item(HopItem<T2> it, int order) {
  const TileArgs<T2> ta{it.U, it.clov, nullptr, it.in, nullptr, it.aux, nullptr, it.red_a, nullptr, it.out, nullptr};
  if (order != TILE_ORDER_LINEAR) {
    const int x = blockIdx.x % kXcd, j = blockIdx.x / kXcd, nb = gridDim.x / kXcd;
    int S = 0, lo = 0, bs = 1, total;
    if (order == TILE_ORDER_BANDED) {
      band_of(it.ntiles, it.tps, x, S, lo, bs);
      total = bs * (it.ntiles / S);
    } else {
      total = it.xoff[x + 1] - it.xoff[x];
    }
    for (int v = j; v < total; v += nb) {
      const int tile = order == TILE_ORDER_BANDED ? band_tile(S, lo, bs, v) : ldg(it.walk + it.xoff[x] + v);
      hop_tile<T2, R, MODE, RED>(it.g, ta, it.partial, all_columns(), it.par_out, it.nrhs, it.c1, tile);
    }
  } else {
    for (int tile = blockIdx.x; tile < it.ntiles; tile += gridDim.x)
      hop_tile<T2, R, MODE, RED>(it.g, ta, it.partial, all_columns(), it.par_out, it.nrhs, it.c1, tile);
  }
}

// ------------------------------------------------ D on canonical fields
// out = D_Gamma in, both fields in the canonical layout of the host lattice,
// out zero outside Gamma: one kernel from the caller's field to the caller's
// field.  Four lanes per site, one per spin.  A quad of lanes loads and stores a
// site's 192 contiguous bytes as three runs of 64 and sorts them into spins with
// DPP moves.  The spin structure stays inside the quad as well:
// ((1 -+ g_mu) psi)_s = psi_s -+ ph psi_{s'} with s' = s ^ 2 or 3 - s, and every lane
// multiplies its own colour vector by the link, which is twice the SU(3) products
// of the half-spinor form and no reconstruction.  A lane keeps R columns, so
// that a link is read once for all of them.  The rows outside Gamma are cleared by
// the same workgroups or by others of the launch (kShareTiles).
//
// Bound by what the L2s fetch again: neighbour spinors and, once per group of
// columns, links (32^3 x 16 of a 32^3 x 32 field, 12 columns: 8.7 GB read and 2.5 GB
// written past the L2s, 7.1 TB/s; 4.4 GB is what each input and output takes once).  So
// more columns per lane are faster and more waves are not: 2.7 ms at R = 1 with
// four waves per SIMD, 1.8 at R = 3, 1.65 at R = 4, 1.58 at R = 6, both with two.
// The quadrant walk gives 1.72 against 2.03 ms for bands of time slices (R = 4),
// streaming stores of rows that nothing reads again 1.53 against 1.59.  Measured
// in all: 1.56 ms; 1.53 with one chain of FMAs through the eight hops, whose sum
// rounds 40% worse; 4.43 when the field was reordered to even-odd tiles and back
// around two stencil launches (two gathers, two scatters and three fills, 1.75 ms
// of it).  On 8 x 4^3 with one column 8 us instead of nine launches of 37.
struct LexSite {
  int y[4];
  int s;   // lexicographic index in the box
};
__device__ __forceinline__ LexSite lex_site(const BoxGeom& g, int s) {
  LexSite l;
  l.s = s;
  int r = s;
  l.y[3] = r % g.L[3]; r /= g.L[3];
  l.y[2] = r % g.L[2]; r /= g.L[2];
  l.y[1] = r % g.L[1];
  l.y[0] = r / g.L[1];
  return l;
}
// Where the box lies in a field: lattice and origin.
struct FieldBox {
  int L[4], lo[4];
};
__host__ __device__ __forceinline__ FieldBox field_box(const BlockSpec& bs) {
  return {{bs.L[0], bs.L[1], bs.L[2], bs.L[3]}, {bs.lo[0], bs.lo[1], bs.lo[2], bs.lo[3]}};
}
__host__ __device__ __forceinline__ size_t field_col(const FieldBox& f) {   // numbers of one column
  return (size_t)f.L[0] * f.L[1] * f.L[2] * f.L[3] * 12;
}
__device__ __forceinline__ size_t field_site(const FieldBox& f, const LexSite& l) {
  return (((size_t)(f.lo[0] + l.y[0]) * f.L[1] + f.lo[1] + l.y[1]) * f.L[2] + f.lo[2] + l.y[2]) * f.L[3] + f.lo[3] +
         l.y[3];
}
__device__ __forceinline__ int box_stride(const BoxGeom& g, int mu) {
  return (mu < 3 ? g.L[3] : 1) * (mu < 2 ? g.L[2] : 1) * (mu < 1 ? g.L[1] : 1);
}
__device__ __forceinline__ long field_stride(const FieldBox& f, int mu) {
  return (long)(mu < 3 ? f.L[3] : 1) * (mu < 2 ? f.L[2] : 1) * (mu < 1 ? f.L[1] : 1);
}

__device__ __forceinline__ double2 ldg2(const double2* p) {
  const f64x2 u = *(const DDML_GLOBAL f64x2*)p;
  return make_double2(u.x, u.y);
}
__device__ __forceinline__ void stg2nt(double2* p, double2 v) {
  f64x2 u;
  u.x = v.x; u.y = v.y;
  __builtin_nontemporal_store(u, (DDML_GLOBAL f64x2*)p);
}
// the value of lane ^ 1, lane ^ 2 or lane ^ 3 of the quad
template <int X>
__device__ __forceinline__ double quad_xor(double v) {
  constexpr int ctrl = X == 1 ? 0xB1 : (X == 2 ? 0x4E : 0x1B);
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <int X>
__device__ __forceinline__ double2 quad_xor(double2 v) {
  return make_double2(quad_xor<X>(v.x), quad_xor<X>(v.y));
}

// ((1 - d g_mu) psi)_s of this lane's spin: psi - d g_mu psi with
//   (g_0 psi)_s = -psi_{s^2},              (g_2 psi)_s = -sg2 psi_{3-s}, sg2 = +, -, -, +
//   (g_1 psi)_s = -i sg1 psi_{3-s}, sg1 = +, +, -, -,   (g_3 psi)_s = -i sg2 psi_{s^2}
__device__ __forceinline__ double2 spin_term(int mu, bool fwd, double2 psi, double sg1, double sg2) {
  const double2 o = (mu == 0 || mu == 3) ? quad_xor<2>(psi) : quad_xor<3>(psi);
  const double d = fwd ? 1.0 : -1.0;
  switch (mu) {
    case 0: return fwd ? cadd(psi, o) : csub(psi, o);
    case 1: return make_double2(fmadd(-d * sg1, o.y, psi.x), fmadd(d * sg1, o.x, psi.y));
    case 2: return cmas(psi, o, d * sg2);
    default: return make_double2(fmadd(-d * sg2, o.y, psi.x), fmadd(d * sg2, o.x, psi.y));
  }
}

// R columns of one site (nr of them in use), this lane's spin
template <int R>
__device__ __forceinline__ void dw_site(const BoxGeom& g, const BlockSpec& bs, const FieldBox& fin, const LexSite& l,
                                        int spin, const double2* __restrict__ U, const double2* __restrict__ A,
                                        const double2* __restrict__ in, size_t icol, double2* __restrict__ out,
                                        size_t col, int nr) {
  const int nt = g.ntiles, i = l.s >> 1;
  const int par = (l.y[0] + l.y[1] + l.y[2] + l.y[3]) & 1;
  const double sg1 = spin < 2 ? 1.0 : -1.0, sg2 = (spin == 0 || spin == 3) ? 1.0 : -1.0;
  const double2* const mine = in + field_site(fin, l) * 12 + spin;   // lane q loads numbers q, q + 4, q + 8
  // all eight hops, by a number that the compiler does not see: in one basic
  // block it moves the loads of later hops up until registers spill
  int hops;
  asm volatile("s_movk_i32 %0, 0xff" : "=s"(hops));
  double2 acc[R][3];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int a = 0; a < 3; ++a) acc[r][a] = make_double2(0, 0);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu)
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
      if (!((hops >> (2 * mu + dir)) & 1)) continue;
      const bool fwd = dir == 0;
      const int y = l.y[mu];
      const int step = fwd ? (y + 1 == g.L[mu] ? 1 - g.L[mu] : 1) : (y == 0 ? g.L[mu] - 1 : -1);
      const double2* src = mine + step * field_stride(fin, mu) * 12;
      double2 raw[R][3], w[3], u[9];
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < 3; ++j) raw[r][j] = ldg2(src + (r < nr ? r : 0) * icol + 4 * j);
      // the link the same way: lane q loads entries q, q + 4 and 8
      const double2* ug = U + (fwd ? lidx(nt, par, mu, 0, i) : lidx(nt, 1 - par, mu, 0, (l.s + step * box_stride(g, mu)) >> 1));
      const double2* uq = ug + 128 * (spin >> 1) + (spin & 1);
      w[0] = ldg2(uq);
      w[1] = ldg2(uq + 256);
      w[2] = ldg2(ug + 512);
#pragma unroll
      for (int k = 0; k < 9; ++k)
        u[k] = k == 8 ? w[2] : ((k & 3) == 0 ? quad_move<0x00>(w[k >> 2]) : ((k & 3) == 1 ? quad_move<0x55>(w[k >> 2]) :
               ((k & 3) == 2 ? quad_move<0xAA>(w[k >> 2]) : quad_move<0xFF>(w[k >> 2]))));
#pragma unroll
      for (int r = 0; r < R; ++r) {
        double2 psi[3], h[3];
        quad_to_spin(spin, raw[r], psi);
#pragma unroll
        for (int a = 0; a < 3; ++a) h[a] = spin_term(mu, fwd, psi[a], sg1, sg2);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          double2 t = make_double2(0, 0);
#pragma unroll
          for (int b = 0; b < 3; ++b) t = fwd ? cmac(t, u[3 * a + b], h[b]) : cmacc(t, u[3 * b + a], h[b]);
          acc[r][a] = cadd(acc[r][a], t);
        }
      }
    }
  // (A psi)_s: this spin's three rows of its chiral 6x6 block.  Spin 0 of the
  // block (rows 0..2) takes the cross entries as they are stored, spin 1 their
  // adjoint.
  const int blk = spin >> 1;
  const bool low = spin & 1;
  const double2* cl = A + cidx(nt, par, 18 * blk, i);
  auto slot = [&](int k) { return ldg2(cl + 128 * (k >> 1) + (k & 1)); };
  auto up = [](int r, int c) { return 3 + r * (11 - r) / 2 + (c - r - 1); };
  const double2 d0 = slot(0), d1 = slot(1), d2 = slot(2);
  const double dg[3] = {low ? d1.y : d0.x, low ? d2.x : d0.y, low ? d2.y : d1.x};
  const double2 o01 = slot(low ? up(3, 4) : up(0, 1)), o02 = slot(low ? up(3, 5) : up(0, 2)),
                o12 = slot(low ? up(4, 5) : up(1, 2));
  double2 x[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) x[a][b] = slot(up(a, 3 + b));
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a; b < 3; ++b) {
      const double2 p = x[a][b], q = x[b][a];
      x[a][b] = make_double2(low ? q.x : p.x, low ? -q.y : p.y);
      if (b > a) x[b][a] = make_double2(low ? p.x : q.x, low ? -p.y : q.y);
    }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    double2 raw[3], v[3], w[3], q[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) raw[j] = ldg2(mine + (r < nr ? r : 0) * icol + 4 * j);
    quad_to_spin(spin, raw, v);
#pragma unroll
    for (int a = 0; a < 3; ++a) w[a] = quad_xor<1>(v[a]);
#pragma unroll
    for (int a = 0; a < 3; ++a) q[a] = cscale(v[a], dg[a]);
    q[0] = cmac(cmac(q[0], o01, v[1]), o02, v[2]);
    q[1] = cmac(cmacc(q[1], o01, v[0]), o12, v[2]);
    q[2] = cmacc(cmacc(q[2], o02, v[0]), o12, v[1]);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
      for (int b = 0; b < 3; ++b) q[a] = cmac(q[a], x[a][b], w[b]);
      q[a] = cscale(cmas(q[a], acc[r][a], -bs.kappa), 1.0 / (2.0 * bs.kappa));
    }
    if (r < nr) {
      double2* o = out + field_site(field_box(bs), l) * 12 + spin + r * col;
      double2 t[3];
      spin_to_quad(spin, q, t);
#pragma unroll
      for (int j = 0; j < 3; ++j) stg2nt(o + 4 * j, t[j]);
    }
  }
}

// Clears the part outside Gamma of rows [r0, r1) of the field's nrhs L0 L1 L2
// rows of L3 sites (fewer than 2^31 in 288 GB), one wave per row.
__device__ __forceinline__ void clear_rows(const BoxGeom& g, const BlockSpec& bs, double2* __restrict__ out,
                                           unsigned r0, unsigned r1) {
  const int lane = threadIdx.x & 63;
  for (unsigned r = r0 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); r < r1; r += blockDim.x >> 6) {
    const unsigned q = r / (unsigned)bs.L[2];
    const int x2 = (int)(r - q * bs.L[2]) - bs.lo[2];
    const unsigned p = q / (unsigned)bs.L[1];
    const int x1 = (int)(q - p * bs.L[1]) - bs.lo[1], x0 = (int)(p % (unsigned)bs.L[0]) - bs.lo[0];
    const bool crosses = (unsigned)x0 < (unsigned)g.L[0] && (unsigned)x1 < (unsigned)g.L[1] &&
                         (unsigned)x2 < (unsigned)g.L[2];
    if (crosses && g.L[3] == bs.L[3]) continue;
    const int a = crosses ? 12 * bs.lo[3] : 0, skip = crosses ? 12 * g.L[3] : 0;   // the row's part inside Gamma
    double2* row = out + (size_t)r * bs.L[3] * 12;
    for (int k = lane; k < 12 * bs.L[3] - skip; k += 64) stg2nt(row + (k < a ? k : k + skip), make_double2(0, 0));
  }
}

// A workgroup is R columns of 64 sites of the box in lexicographic order (one
// tile, 16 sites per wavefront); the groups of columns of a tile follow each
// other on its XCD.
struct DwWalk {
  const int* tile;       // XCD x works through tile[xoff[x] .. xoff[x+1])
  int xoff[kXcd + 1];
};
template <int R>
__global__ void __launch_bounds__(256, 2)
    k_apply_d(BoxGeom g, BlockSpec bs, FieldBox fin, DwWalk walk, const double2* __restrict__ U,
              const double2* __restrict__ A, const double2* __restrict__ in, double2* __restrict__ out, int nrhs,
              int ntl, long rows, int nclear) {
  // the last nclear workgroups only clear
  const int nwork = gridDim.x - nclear, c0 = (int)blockIdx.x - nwork;
  if (c0 >= 0) {
    clear_rows(g, bs, out, c0 * rows / nclear, (c0 + 1) * rows / nclear);
    return;
  }
  const size_t col = field_col(field_box(bs)), icol = field_col(fin);
  const int x = blockIdx.x % kXcd, nb = nwork / kXcd;
  const int* tiles = walk.tile + walk.xoff[x];
  const int ng = (nrhs + R - 1) / R, n = (walk.xoff[x + 1] - walk.xoff[x]) * ng;
  const bool share = rows && nclear == 0;
  for (int v = blockIdx.x / kXcd; v < n; v += nb) {
    const int tile = ldg(tiles + v / ng), c = (v % ng) * R;
    if (share && c == 0) clear_rows(g, bs, out, tile * rows / ntl, (tile + 1) * rows / ntl);
    const int s = tile * kTile + (threadIdx.x >> 2);
    if (s >= 2 * g.Vh) continue;   // (the four lanes of a site together)
    dw_site<R>(g, bs, fin, lex_site(g, s), threadIdx.x & 3, U, A, in + c * icol, icol, out + c * col, col,
               min(R, nrhs - c));
  }
}

// Gamma's sites of every column of a canonical field, one after the other.
__global__ void __launch_bounds__(256) k_box_sites(BoxGeom g, FieldBox f, const double2* __restrict__ in,
                                                   double2* __restrict__ box) {
  const int n = 2 * g.Vh, s0 = blockIdx.x * 64;
  in += blockIdx.y * field_col(f);
  box += ((size_t)blockIdx.y * n + s0) * 12;
  for (int k = threadIdx.x; k < 64 * 12 && s0 + k / 12 < n; k += 256)
    box[k] = ldg2(in + field_site(f, lex_site(g, s0 + k / 12)) * 12 + k % 12);
}

// Tiles from which on their workgroups clear the rows outside Gamma on the way:
// four per CU, enough to keep the stores of the whole chip busy, and the stores
// then wait for nothing (12 columns, 16 of 32^4's slices, 8192 tiles: 1.49 ms and
// 1.54 with workgroups of their own; 4 of 64 x 32^3, 2048 tiles: 1.11 and 1.19; 2 of
// them, 1024 tiles: 1.06 and 1.06).  Fewer cannot clear a large lattice, so that is
// done beside them (14 x 10 x 8 x 12 of 20 x 12 x 10 x 14, 210 tiles: 70 and 61 us;
// two slices of 32 x 16^3, 128 tiles: 94 and 78; 4^4 of it, 4 tiles: 1620 and 75).
constexpr int kShareTiles = 1024;
constexpr int kClearRows = 4;   // per wave of a workgroup that only clears (1 and 16 rows: the same within 5%)
hipError_t launch_apply_d(const BoxGeom& g, const BlockSpec& bs, const int* walk, const int* xoff, const double2* U,
                          const double2* A, const double2* in, double2* out, int nrhs, double2* copy, hipStream_t st) {
  if (nrhs < 1 || nrhs > kMaxRhs) return hipErrorInvalidValue;
  FieldBox fin = field_box(bs);
  if (copy) {   // the input first moves there, Gamma's sites side by side
    hipLaunchKernelGGL(k_box_sites, dim3((2 * g.Vh + 63) / 64, nrhs), dim3(256), 0, st, g, fin, in, copy);
    for (int m = 0; m < 4; ++m) fin.L[m] = g.L[m], fin.lo[m] = 0;
    in = copy;
  }
  DwWalk w{walk, {}};
  for (int x = 0; x <= kXcd; ++x) w.xoff[x] = xoff[x];
  const int ntl = xoff[kXcd];
  bool all = true;
  for (int m = 0; m < 4; ++m) all = all && g.L[m] == bs.L[m];
  const long rows = all ? 0 : (long)nrhs * bs.L[0] * bs.L[1] * bs.L[2];
  // groups of six columns at most (what two waves per SIMD have registers for),
  // as even as they come
  const int groups = (nrhs + 5) / 6;
  // (a small box may lie on few XCDs: a workgroup for each of the longest list)
  int longest = 0;
  for (int x = 0; x < kXcd; ++x) longest = xoff[x + 1] - xoff[x] > longest ? xoff[x + 1] - xoff[x] : longest;
  const int work = kXcd * (longest * groups < 2048 ? longest * groups : 2048);
  const int nclear =
      rows && ntl < kShareTiles ? (int)std::min((rows + 4 * kClearRows - 1) / (4 * kClearRows), 65536L) : 0;
#define DDML_DW(Rv)                                                                                                 \
  case Rv:                                                                                                          \
    hipLaunchKernelGGL(k_apply_d<Rv>, dim3(work + nclear), dim3(256), 0, st, g, bs, fin, w, U, A, in, out, nrhs, ntl,  \
                       rows, nclear);                                                                               \
    break;
  switch ((nrhs + groups - 1) / groups) {
    DDML_DW(1)
    DDML_DW(2)
    DDML_DW(3)
    DDML_DW(4)
    DDML_DW(5)
    DDML_DW(6)
    default: return hipErrorInvalidValue;
  }
#undef DDML_DW
  return hipGetLastError();
}

// ------------------------------------------------- boundary block D_{dGamma}
// The entries of D that join a site x of the domain Gamma to a neighbour y
// outside it (eq. blkdec; the off-diagonal block of eq. Scmpt2):
//   y = x + mu:  -1/2 (1 - gamma_mu) U_mu(x) psi(y)
//   y = x - mu:  -1/2 (1 + gamma_mu) U_mu(y)^dag psi(y)
// with the time-boundary phase (antiperiodic -1, open: no such hop), on
// canonical fields and links.  Nearly all of the output is zero: a wavefront takes
// a run of 16 sites of the field, and one that no coupling reaches is only cleared,
// in contiguous streaming stores.  The rest go through the quads of lanes of
// k_apply_d, a lane's site taking the hops that leave Gamma.
// Bound by the stores: 12 columns of a 32^3 x 32 field, one face of 32^3, 473 us of
// calls in a row for 2.4 GB, 735 with a thread per site, 485 by rows of L3 sites.
// (A fill in 4 KB workgroups takes 345 us, but the faces in a launch of their own
// 100 more, and a launch more is 4 us on a small field.)
__device__ __forceinline__ const double2* canon_link(const GaugeView& gv, const BlockSpec& bs, size_t site, int t,
                                                     int mu) {
  if (gv.region && t >= gv.r_t0 && t < gv.r_t1)
    return gv.region + ((site - (size_t)gv.r_t0 * bs.L[1] * bs.L[2] * bs.L[3]) * 4 + mu) * 9;
  return gv.base + (site * 4 + mu) * 9;
}

__device__ __forceinline__ void boundary_site(const GaugeView& gv, const BlockSpec& bs, const int x[4], int spin,
                                              const double2* __restrict__ in, double scale, double2 out[3]) {
  const double sg1 = spin < 2 ? 1.0 : -1.0, sg2 = (spin == 0 || spin == 3) ? 1.0 : -1.0;
  double2 acc[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) acc[a] = make_double2(0, 0);
#pragma unroll
  for (int mu = 0; mu < 4; ++mu)
#pragma unroll
    for (int dir = 0; dir < 2; ++dir) {
      const bool fwd = dir == 0;
      // a hop leaves Gamma at the last (first) site of a cut direction only
      const int edge = fwd ? bs.lo[mu] + bs.Lb[mu] - 1 : bs.lo[mu];
      if (bs.Lb[mu] == bs.L[mu] || x[mu] != edge) continue;   // (the four lanes of a site together)
      int y[4] = {x[0], x[1], x[2], x[3]};
      y[mu] += fwd ? 1 : -1;
      double ph = -0.5 * scale;
      if (y[mu] < 0 || y[mu] >= bs.L[mu]) {
        y[mu] = fwd ? 0 : bs.L[mu] - 1;
        if (mu == 0 && bs.tbc == 2) continue;
        if (mu == 0 && bs.tbc == 1) ph = -ph;
      }
      const size_t sy = (((size_t)y[0] * bs.L[1] + y[1]) * bs.L[2] + y[2]) * bs.L[3] + y[3];
      const size_t sx = (((size_t)x[0] * bs.L[1] + x[1]) * bs.L[2] + x[2]) * bs.L[3] + x[3];
      const double2* ug = canon_link(gv, bs, fwd ? sx : sy, fwd ? x[0] : y[0], mu);
      double2 raw[3], psi[3], h[3], u[9];
#pragma unroll
      for (int j = 0; j < 3; ++j) raw[j] = ldg2(in + sy * 12 + 4 * j + spin);
#pragma unroll
      for (int k = 0; k < 9; ++k) u[k] = ldg2(ug + k);
      quad_to_spin(spin, raw, psi);
#pragma unroll
      for (int a = 0; a < 3; ++a) h[a] = spin_term(mu, fwd, psi[a], sg1, sg2);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        double2 t = make_double2(0, 0);
#pragma unroll
        for (int b = 0; b < 3; ++b) t = fwd ? cmac(t, u[3 * a + b], h[b]) : cmacc(t, u[3 * b + a], h[b]);
        acc[a] = cmas(acc[a], t, ph);
      }
    }
  spin_to_quad(spin, acc, out);
}

__global__ void __launch_bounds__(256) k_boundary(GaugeView gv, BlockSpec bs, const double2* __restrict__ in,
                                                       double2* __restrict__ out, unsigned runs, double scale) {
  const int lane = threadIdx.x & 63;
  const size_t vol = (size_t)bs.L[0] * bs.L[1] * bs.L[2] * bs.L[3] * 12;
  for (unsigned run = blockIdx.x * 4 + (threadIdx.x >> 6); run < runs; run += gridDim.x * 4) {
    int x[4];
    unsigned q = run * 16 + (lane >> 2);
    double2* const o = out + (size_t)run * 16 * 12;
#pragma unroll
    for (int m = 3; m >= 0; --m) {
      const unsigned r = q / (unsigned)bs.L[m];
      x[m] = (int)(q - r * bs.L[m]);
      q = r;
    }
    bool inside = true, face = false;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      inside = inside && x[m] >= bs.lo[m] && x[m] < bs.lo[m] + bs.Lb[m];
      face = face || (bs.Lb[m] != bs.L[m] && (x[m] == bs.lo[m] || x[m] == bs.lo[m] + bs.Lb[m] - 1));
    }
    if (!__ballot(inside && face)) {
#pragma unroll
      for (int j = 0; j < 3; ++j) stg2nt(o + 64 * j + lane, make_double2(0, 0));
      continue;
    }
    double2 v[3] = {make_double2(0, 0), make_double2(0, 0), make_double2(0, 0)};
    if (inside && face) boundary_site(gv, bs, x, lane & 3, in + q * vol, scale, v);
#pragma unroll
    for (int j = 0; j < 3; ++j) stg2nt(o + (lane >> 2) * 12 + 4 * j + (lane & 3), v[j]);
  }
}

// The same by rows of L3 sites, 16 at a time: only x3 differs within a wave, which
// makes the hops of the other directions uniform branches.  Faster where every row
// of Gamma has couplings at its ends and fills a wave (16^3 x L3 with all faces cut, 12
// columns: 88 and 93 us for L3 = 24 and 32, 91 and 99 by runs).  With L3 = 18 it is 87
// against 80 and with 4 it is 75 against 50.  Without cut ends most rows are only
// cleared: 96 against 81 with 32, and 128 against 49 on 16 x 32^2 x 2, where a row fills
// 24 lanes.
__global__ void __launch_bounds__(256) k_boundary_rows(GaugeView gv, BlockSpec bs, const double2* __restrict__ in,
                                                       double2* __restrict__ out, unsigned rows, double scale) {
  const int lane = threadIdx.x & 63, L3 = bs.L[3];
  const size_t vol = (size_t)bs.L[0] * bs.L[1] * bs.L[2] * L3 * 12;
  for (unsigned row = blockIdx.x * 4 + (threadIdx.x >> 6); row < rows; row += gridDim.x * 4) {
    int x[4] = {0, 0, 0, 0};
    unsigned q = __builtin_amdgcn_readfirstlane(row);
    x[2] = (int)(q % (unsigned)bs.L[2]); q /= (unsigned)bs.L[2];
    x[1] = (int)(q % (unsigned)bs.L[1]); q /= (unsigned)bs.L[1];
    x[0] = (int)(q % (unsigned)bs.L[0]);
    const size_t col = q / (unsigned)bs.L[0];
    bool in_row = true, face = bs.Lb[3] != bs.L[3];
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      in_row = in_row && x[m] >= bs.lo[m] && x[m] < bs.lo[m] + bs.Lb[m];
      face = face || (bs.Lb[m] != bs.L[m] && (x[m] == bs.lo[m] || x[m] == bs.lo[m] + bs.Lb[m] - 1));
    }
    double2* const o = out + (size_t)row * L3 * 12;
    if (!(in_row && face)) {   // (uniform over the wavefront)
      for (int k = lane; k < 12 * L3; k += 64) stg2nt(o + k, make_double2(0, 0));
      continue;
    }
    for (int s = lane >> 2; s < L3; s += 16) {
      x[3] = s;
      double2 v[3] = {make_double2(0, 0), make_double2(0, 0), make_double2(0, 0)};
      if (s >= bs.lo[3] && s < bs.lo[3] + bs.Lb[3]) boundary_site(gv, bs, x, lane & 3, in + col * vol, scale, v);
#pragma unroll
      for (int j = 0; j < 3; ++j) stg2nt(o + s * 12 + 4 * j + (lane & 3), v[j]);
    }
  }
}

constexpr int kLongRow = 24;
hipError_t launch_boundary(const GaugeView& gv, const BlockSpec& bs, const double2* in, double2* out, int nrhs,
                           double scale, hipStream_t st) {
  const unsigned rows = (unsigned)nrhs * bs.L[0] * bs.L[1] * bs.L[2];   // (fewer than 2^31 in 288 GB)
  if (bs.L[3] >= kLongRow && bs.Lb[3] != bs.L[3]) {
    const unsigned grid = std::min((rows + 3) / 4, 65536u);
    hipLaunchKernelGGL(k_boundary_rows, dim3(grid), dim3(256), 0, st, gv, bs, in, out, rows, scale);
  } else {
    const unsigned runs = (unsigned)((size_t)rows * bs.L[3] / 16);   // (every extent is even)
    const unsigned grid = std::min((runs + 3) / 4, 65536u);
    hipLaunchKernelGGL(k_boundary, dim3(grid), dim3(256), 0, st, gv, bs, in, out, runs, scale);
  }
  return hipGetLastError();
}

// Batched launch over solver slots.  Linear order: virtual tile vt of the
// batch maps to (slot, tile) through tile_start[nslots+1].  Other orders:
// XCD x walks xstart[x][*], the prefix over slots of its share of the tiles.
__device__ __forceinline__ int find_slot(const int* __restrict__ start, int n, int vt) {
  int lo = 0, hi = n;  // start[lo] <= vt < start[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (start[mid] <= vt) lo = mid; else hi = mid;
  }
  return lo;
}

// The columns of a tile are split into ng groups of W = blockDim.x / 64
// waves (W * R columns each); virtual item v is (tile v / ng, group v % ng),
// so the groups of one tile run back to back on the same XCD.  ST: the
// workgroup stages each tile's links and clover data in LDS first (the trip
// count of the tile loop is uniform over the workgroup, so every wavefront
// reaches both barriers).
// The FP32 and 16-bit stencil at R = 1 is held to 6 waves per SIMD (80
// VGPRs), so that two 12-wave workgroups (one tile each) share a CU: the odd
// half fits without spills, the even half spills 3-5 registers and still
// runs 4-6% faster than at one workgroup per CU.
template <typename T2, int R, int MODE>
constexpr int kHopWaves = (!std::is_same<T2, double2>::value && R == 1) ? 6 : 1;

template <typename T2, int R, int MODE, int RED, bool ST>
__global__ void __launch_bounds__(64 * ((kMaxRhs + R - 1) / R))
    __attribute__((amdgpu_waves_per_eu(kHopWaves<T2, R, MODE>))) k_hop_batch(const SlotDesc<T2>* __restrict__ slots, const int* __restrict__ tile_start,
                const int* __restrict__ xstart, int xstride, const int* __restrict__ nslots_p, int fin, int faux,
                int fout, int fred, int par_out, int order, int ng) {
  using C = typename CompOf<T2>::type;
  __shared__ C sm[ST ? kStagePairs * 128 : 1];
  const int ns = *nslots_p;
  const int W = blockDim.x >> 6;
  const bool banded = order != TILE_ORDER_LINEAR;
  const int x = blockIdx.x % kXcd;
  const int* P = banded ? xstart + (size_t)x * xstride : tile_start;
  const int first = banded ? blockIdx.x / kXcd : blockIdx.x;
  const int step = banded ? gridDim.x / kXcd : gridDim.x;
  const int total = P[ns] * ng;
  for (int v = first; v < total; v += step) {
    const int tv = v / ng, grp = v - tv * ng;
    const int s = find_slot(P, ns, tv);
    const SlotDesc<T2>& d = slots[s];
    const int flag = active_flag(d.active, d.nrhs);   // on its way with the walk's entry
    int tile = tv - P[s];
    if (order == TILE_ORDER_BANDED) {
      int S, lo, bs;
      band_of(d.ntiles, d.tps, x, S, lo, bs);
      tile = band_tile(S, lo, bs, tile);
    } else if (order != TILE_ORDER_LINEAR) {
      tile = ldg(d.walk + d.xoff[x] + tile);
    }
    // a workgroup whose columns are all inactive skips the tile before the staging
    // (uniform: every wave reads the same flags)
    const unsigned act = active_of(flag);
    const int c0 = grp * W * R, c1 = min(d.nrhs, c0 + W * R);
    if (c0 >= c1 || !((act >> c0) & ((1u << (c1 - c0)) - 1u))) continue;
    const bool h16 = kIs16<T2>;
    const T2* clov = MODE == MODE_RES ? d.A : d.Ainv;   // M = A - kappa H needs A itself
    const TileArgs<T2> ta{d.U, clov, h16 ? d.Ainv_nrm : nullptr,
                          d.f[fin], h16 ? d.nrm[fin] : nullptr,
                          faux >= 0 ? d.f[faux] : nullptr, h16 && faux >= 0 ? d.nrm[faux] : nullptr,
                          fred >= 0 ? d.f[fred] : nullptr, h16 && fred >= 0 ? d.nrm[fred] : nullptr,
                          d.f[fout], h16 ? d.nrm[fout] : nullptr};
    if constexpr (ST) stage_tile<T2>(d.g, d.U, clov, ta.clov_n, par_out, tile, sm);
    // kappa^2 in the Schur operator, kappa in the FP64 residual and preparation
    const double kap = (MODE == MODE_PREP || MODE == MODE_RES) ? d.kappa : d.kappa * d.kappa;
    hop_tile<T2, R, MODE, RED, ST>(d.g, ta, d.partial, act, par_out, d.nrhs, kap, tile, grp * W, sm);
    if constexpr (ST) __syncthreads();
  }
}

// Site-local clover application out = C in on parity p.
template <typename T2>
__global__ void k_clover_apply(BoxGeom g, const T2* __restrict__ clov, int p, const T2* __restrict__ in,
                               T2* __restrict__ out, int nrhs) {
  const size_t per = (size_t)g.ntiles * 64;
  const size_t n = per * nrhs;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(t % per);  // a thread per (site, column)
    const int col = (int)(t / per);
    const size_t base = fidx(g.ntiles, col, 0, i);
    const T2* cl = clov + cidx(g.ntiles, p, 0, i);
    T2 x[12], y[12];
    spinor_load(in + base, x);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      T2 m[18];
      herm6_load(cl + 128 * 9 * b, m);
      herm6_apply(m, x + 6 * b, y + 6 * b);
    }
    if (i >= g.Vh)
#pragma unroll
      for (int c = 0; c < 12; ++c) y[c] = mk<T2>(0, 0);
    spinor_store(out + base, y);
  }
}

// --------------------------------------------------------------- launchers
#define DDML_HOP_DISPATCH(T2, Rv, MODEv, REDv)                                                        \
  if (R == Rv && mode == MODEv && red == REDv) {                                                      \
    hipLaunchKernelGGL((k_hop_item<T2, Rv, MODEv, REDv>), dim3(grid), dim3(block), 0, st, it, order); \
    return hipGetLastError();                                                                         \
  }

template <typename T2>
static hipError_t hop_item_impl(const HopItem<T2>& it, int mode, int red, int R, int order, hipStream_t st) {
  const int block = 64 * ((it.nrhs + R - 1) / R);
  int grid = it.ntiles < 65535 ? it.ntiles : 65535;
  if (order < 0 || order >= TILE_ORDER_NUM || (order >= TILE_ORDER_SUB2 && it.walk == nullptr))
    return hipErrorInvalidValue;
  if (order != TILE_ORDER_LINEAR) grid = ((grid + kXcd - 1) / kXcd) * kXcd;
  DDML_HOP_DISPATCH(T2, 1, MODE_CINV_HOP, RED_NONE)
  DDML_HOP_DISPATCH(T2, 1, MODE_SCHUR, RED_NONE)
  DDML_HOP_DISPATCH(T2, 1, MODE_PREP, RED_NONE)
  DDML_HOP_DISPATCH(T2, 1, MODE_RES, RED_NORM)
  DDML_HOP_DISPATCH(T2, 2, MODE_CINV_HOP, RED_NONE)
  DDML_HOP_DISPATCH(T2, 2, MODE_SCHUR, RED_NONE)
  DDML_HOP_DISPATCH(T2, 3, MODE_CINV_HOP, RED_NONE)
  DDML_HOP_DISPATCH(T2, 3, MODE_SCHUR, RED_NONE)
  (void)block;
  return hipErrorInvalidValue;
}

hipError_t launch_hop_item(const HopItem<double2>& it, int mode, int red, int R, int order, hipStream_t st) {
  return hop_item_impl(it, mode, red, R, order, st);
}

#define DDML_HOPB_DISPATCH1(T2, Rv, MODEv, REDv, STv)                                                    \
  if (R == Rv && mode == MODEv && red == REDv) {                                                         \
    hipLaunchKernelGGL((k_hop_batch<T2, Rv, MODEv, REDv, STv>), dim3(grid), dim3(block), 0, st, slots,   \
                       tile_start, xstart, xstride, nslots_p, fin, faux, fout, fred, par_out, order, ng); \
    return hipGetLastError();                                                                            \
  }
#define DDML_HOPB_DISPATCH_R(T2, Rv, STv)                        \
  DDML_HOPB_DISPATCH1(T2, Rv, MODE_CINV_HOP, RED_NONE, STv)      \
  DDML_HOPB_DISPATCH1(T2, Rv, MODE_SCHUR, RED_DOT, STv)          \
  DDML_HOPB_DISPATCH1(T2, Rv, MODE_SCHUR, RED_TS, STv)           \
  if constexpr (!kIs16<T2>) {                                    \
    DDML_HOPB_DISPATCH1(T2, Rv, MODE_SCHUR, RED_NONE, STv)       \
  }                                                              \
  if constexpr (std::is_same<T2, double2>::value && Rv == 1) {   \
    DDML_HOPB_DISPATCH1(T2, Rv, MODE_PREP, RED_NONE, STv)        \
    DDML_HOPB_DISPATCH1(T2, Rv, MODE_RES, RED_NORM, STv)         \
  }
#define DDML_HOPB_DISPATCH_ST(T2, STv) \
  DDML_HOPB_DISPATCH_R(T2, 1, STv)     \
  DDML_HOPB_DISPATCH_R(T2, 2, STv)     \
  DDML_HOPB_DISPATCH_R(T2, 3, STv)

template <typename T2>
static hipError_t hop_batch_impl(const SlotDesc<T2>* slots, const int* tile_start, const int* xstart, int xstride,
                                 const int* nslots_p, int nrhs, int R, int mode, int red, int fin, int faux, int fout,
                                 int fred, int par_out, int grid, int order, int splits, int stage,
                                 hipStream_t st) {
  // nw waves cover the columns of a tile; they are split into ng blocks of W
  // waves.  A staged, unsplit workgroup always has the most waves its kernel
  // is built for: those beyond the columns only copy links and clover data,
  // which one wave does 58 pairs of in turn.  M-hat pair without and with them, us:
  //            FP32, 1, 3, 8 columns        FP64, 1, 3, 8 columns
  //   4^4      35 22, 27 22, 25 24          38 23, 29 25, 32 30
  //   16^3 x 8 49 25, 39 28, 38 35          69 33, 49 40, 65 64
  //   24^3 x 16 222 85, 140 99, 162 152     454 182, 278 212, 382 379
  const int nw = (nrhs + R - 1) / R;
  if (splits < 1 || splits > nw) return hipErrorInvalidValue;
  const int W = stage && splits == 1 ? (kMaxRhs + R - 1) / R : (nw + splits - 1) / splits;
  const int ng = (nw + W - 1) / W;
  const int block = 64 * W;
  if (order < 0 || order >= TILE_ORDER_NUM || (order != TILE_ORDER_LINEAR && grid % kXcd)) return hipErrorInvalidValue;
  if (stage) {
    DDML_HOPB_DISPATCH_ST(T2, true)
  } else {
    if constexpr (!kTwoRow<T2>) {
      DDML_HOPB_DISPATCH_ST(T2, false)
    }
  }
  return hipErrorInvalidValue;  // unknown variant; FP32 and 16-bit fields need stage = 1
}

hipError_t launch_hop_batch(const SlotDesc<float2>* slots, const int* tile_start, const int* xstart, int xstride,
                            const int* nslots_p, int nrhs, int R, int mode, int red, int fin, int faux, int fout,
                            int fred, int par_out, int grid, int order, int splits, int stage, hipStream_t st) {
  return hop_batch_impl(slots, tile_start, xstart, xstride, nslots_p, nrhs, R, mode, red, fin, faux, fout, fred,
                        par_out, grid, order, splits, stage, st);
}
hipError_t launch_hop_batch(const SlotDesc<double2>* slots, const int* tile_start, const int* xstart, int xstride,
                            const int* nslots_p, int nrhs, int R, int mode, int red, int fin, int faux, int fout,
                            int fred, int par_out, int grid, int order, int splits, int stage, hipStream_t st) {
  return hop_batch_impl(slots, tile_start, xstart, xstride, nslots_p, nrhs, R, mode, red, fin, faux, fout, fred,
                        par_out, grid, order, splits, stage, st);
}
hipError_t launch_hop_batch(const SlotDesc<h16c>* slots, const int* tile_start, const int* xstart, int xstride,
                            const int* nslots_p, int nrhs, int R, int mode, int red, int fin, int faux, int fout,
                            int fred, int par_out, int grid, int order, int splits, int stage, hipStream_t st) {
  return hop_batch_impl(slots, tile_start, xstart, xstride, nslots_p, nrhs, R, mode, red, fin, faux, fout, fred,
                        par_out, grid, order, splits, stage, st);
}

template <typename T2>
static hipError_t clover_apply_impl(const BoxGeom& g, const T2* clov, int p, const T2* in, T2* out, int nrhs,
                                    hipStream_t st) {
  size_t n = (size_t)g.ntiles * 64 * nrhs;
  int grid = (int)((n + 255) / 256);
  if (grid > 65535) grid = 65535;
  hipLaunchKernelGGL((k_clover_apply<T2>), dim3(grid), dim3(256), 0, st, g, clov, p, in, out, nrhs);
  return hipGetLastError();
}
hipError_t launch_clover_apply(const BoxGeom& g, const double2* clov, int p, const double2* in, double2* out,
                               int nrhs, hipStream_t st) {
  return clover_apply_impl(g, clov, p, in, out, nrhs, st);
}

}  // namespace ddml
