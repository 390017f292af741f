// Operator blocks: links, clover term and its inverse for one domain box.
//
// Clover term (the O(a) improvement the paper refers to in the footnotes of
// Sections 4 and 6; it gives no formula): Sheikholeslami-Wohlert form
//   c_sw (i/4) sum_{mu,nu} sigma_{mu nu} Fhat_{mu nu}(x),   Fhat = (Q_{mu nu} - Q_{nu mu}) / 8,
// Q_{mu nu}(x) the four plaquettes of the (mu,nu) plane at x.  In hopping units
// (M = 2 kappa D) A = 1 + (i kappa c_sw/2) sum_{mu,nu} sigma Fhat = 1 + i kappa c_sw
// sum_{mu<nu} sigma_{mu nu} Fhat_{mu nu}.  In the chiral basis sigma_{0k} = diag(s_k, -s_k)
// and sigma_{jk} = -eps_{jkl} diag(s_l, s_l), so
//   A = diag(1 + sum_l s_l (x) X_l^+,  1 + sum_l s_l (x) X_l^-),
//   X_l^{+-} = i kappa c_sw (+-Fhat_{0l} - B_l),  B_1 = Fhat_23, B_2 = Fhat_31, B_3 = Fhat_12.
// Each 6x6 block is Hermitian; it is inverted in FP64 by a Cholesky
// factorisation (a non-positive pivot is reported).  The clover term of every
// site of the domain is built from the full gauge field, so D_Gamma is exactly
// the diagonal block of D (eq. blkdec).
#include <type_traits>

#include "ddml_common.hpp"
#include "launchers.hpp"

namespace ddml {

__device__ __forceinline__ size_t gidx(const int L[4], const int x[4]) {
  return (((size_t)x[0] * L[1] + x[1]) * L[2] + x[2]) * L[3] + x[3];
}

__device__ __forceinline__ const double2* link_ptr(const GaugeView& gv, const int L[4], const int x[4], int mu) {
  const size_t s = gidx(L, x);
  if (gv.region && x[0] >= gv.r_t0 && x[0] < gv.r_t1) {
    const size_t V3 = (size_t)L[1] * L[2] * L[3];
    return gv.region + ((s - (size_t)gv.r_t0 * V3) * 4 + mu) * 9;
  }
  return gv.base + (s * 4 + mu) * 9;
}

// local lexicographic index -> local coords
__device__ __forceinline__ void lex_coords(const int Lb[4], int s, int y[4]) {
  y[3] = s % Lb[3]; s /= Lb[3];
  y[2] = s % Lb[2]; s /= Lb[2];
  y[1] = s % Lb[1];
  y[0] = s / Lb[1];
}

__host__ __device__ __forceinline__ int ntiles_of(const BlockSpec& bs) {
  const int Vh = bs.Lb[0] * bs.Lb[1] * bs.Lb[2] * bs.Lb[3] / 2;
  return (Vh + kTile - 1) / kTile;
}

// Where a kernel finds the links around the sites it works on.  In a working
// copy (launch_box_links) entry e of a link lies 64 e complex numbers from its
// first, the 64 sites of a parity's tile side by side, so that a wavefront reads
// an entry as one contiguous run; in the canonical links, read when the copy
// does not fit, every lane reads cache lines of its own.
__device__ __forceinline__ double2* BoxLinks::at(const int L[4], const int x[4], int mu) const {
  int y[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    y[m] = x[m] - o[m];
    y[m] = y[m] < 0 ? y[m] + L[m] : y[m];
  }
  const int lex = ((y[0] * E[1] + y[1]) * E[2] + y[2]) * E[3] + y[3];
  const int par = (y[0] + y[1] + y[2] + y[3]) & 1, i = lex >> 1;
  return W + (((size_t)(mu * 2 + par) * nt + (i >> 6)) * 9) * 64 + (i & 63);
}
// Block b of n in the order in which XCD b mod 8 works through one contiguous
// eighth: neighbours in the lattice then share an L2.
__device__ __forceinline__ int xcd_chunk(int b, int n) {
  const int x = b % kXcd, q = n / kXcd, r = n % kXcd;   // the first r XCDs have one block more
  return x * q + (x < r ? x : r) + b / kXcd;
}
struct CanonLinks {
  GaugeView gv;
  static constexpr int kStep = 1;
  __device__ __forceinline__ double2* at(const int L[4], const int x[4], int mu) const {
    return const_cast<double2*>(link_ptr(gv, L, x, mu));
  }
};

// Canonical links of a box (lattice-periodic) <-> its working copy: 64 sites per
// workgroup through LDS, both sides in contiguous runs.  Writing back (IN =
// false) goes to the slices of a region that starts with the box.
constexpr int kCopyPitch = 37;   // 36 complex per site and one pad (bank conflicts)
template <bool IN>
__global__ void __launch_bounds__(256) k_box_copy(GaugeView gv, double2* __restrict__ region, BlockSpec bs,
                                                   BoxLinks bl, int nsites) {
  __shared__ double2 sm[64 * kCopyPitch];
  const int s0 = blockIdx.x * 64, ns = min(64, nsites - s0);
  auto coords = [&](int lex, int y[4]) {
    y[3] = lex % bl.E[3]; lex /= bl.E[3];
    y[2] = lex % bl.E[2]; lex /= bl.E[2];
    y[1] = lex % bl.E[1];
    y[0] = lex / bl.E[1];
  };
  auto pack = [&](int q, int& lds, double2*& w) {   // q: entry of the tile, sites of a parity fastest
    const int e = q >> 6, p = (q >> 5) & 1, j = q & 31;
    if (2 * j >= ns) return false;
    int y[4];
    coords(s0 + 2 * j, y);
    const int odd = (p + y[0] + y[1] + y[2]) & 1;   // the pair's site of parity p
    lds = (2 * j + odd) * kCopyPitch + e;
    const int mu = e / 9, i = (s0 >> 1) + j;
    w = bl.W + (((size_t)(mu * 2 + p) * bl.nt + (i >> 6)) * 9 + (e - 9 * mu)) * 64 + (i & 63);
    return true;
  };
  auto canon = [&](int q, int& lds) {   // q: entry of the tile, entries of a site fastest
    const int site = q / 36, e = q - 36 * site;
    lds = site * kCopyPitch + e;
    if (!IN) return region + ((size_t)(s0 + site) * 36 + e);
    int x[4];
    coords(s0 + site, x);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      x[m] += bl.o[m];
      x[m] = x[m] >= bs.L[m] ? x[m] - bs.L[m] : x[m];
    }
    return const_cast<double2*>(link_ptr(gv, bs.L, x, 0) + e);
  };
  if (IN) {
    for (int q = threadIdx.x; q < 36 * ns; q += 256) {
      int lds;
      const double2* src = canon(q, lds);
      sm[lds] = *src;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < 36 * 64; q += 256) {
      int lds;
      double2* w;
      if (pack(q, lds, w)) *w = sm[lds];
    }
  } else {
    for (int q = threadIdx.x; q < 36 * 64; q += 256) {
      int lds;
      double2* w;
      if (pack(q, lds, w)) sm[lds] = *w;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < 36 * ns; q += 256) {
      int lds;
      double2* dst = canon(q, lds);
      *dst = sm[lds];
    }
  }
}

static int sites_of(const BoxLinks& bl) { return bl.E[0] * bl.E[1] * bl.E[2] * bl.E[3]; }

size_t box_links_bytes(const BoxLinks& bl) { return (size_t)8 * bl.nt * 9 * 64 * sizeof(double2); }

static void set_box(BoxLinks& bl) { bl.nt = (sites_of(bl) / 2 + 63) / 64; }

BoxLinks clover_box(const BlockSpec& bs) {
  BoxLinks bl{};
  for (int m = 0; m < 4; ++m) {
    const bool cut = bs.Lb[m] != bs.L[m];
    bl.o[m] = cut ? (bs.lo[m] + bs.L[m] - 1) % bs.L[m] : 0;
    bl.E[m] = cut ? bs.Lb[m] + 2 : bs.L[m];
  }
  set_box(bl);
  return bl;
}

BoxLinks level1_box(const BlockSpec& bs, int t0, int t1) {
  BoxLinks bl{};
  for (int m = 0; m < 4; ++m) bl.E[m] = bs.L[m];
  if (t1 - t0 < bs.L[0]) {
    bl.o[0] = t0;
    bl.E[0] = t1 - t0 + 1;
  }
  set_box(bl);
  return bl;
}

static hipError_t launch_box_links(const GaugeView& gv, const BoxLinks& bl, const BlockSpec& bs, hipStream_t st) {
  const int n = sites_of(bl);
  hipLaunchKernelGGL(k_box_copy<true>, dim3((n + 63) / 64), dim3(256), 0, st, gv, nullptr, bs, bl, n);
  return hipGetLastError();
}

// FP64 links in the 5-pair layout; the FP32 copy keeps the first two rows
// (two-row layout, lidx2) and the stencil rebuilds the third as the complex
// conjugate of the cross product of the first two, times the face factor
// (+-1; 0 zeroes all rows).  That holds for SU(3) matrices only: a link whose
// third row differs from the rebuilt one by more than 1e-5 sets bit 2 of *bad.
// One wavefront per (parity, 64-site tile, direction); padding sites are zeroed.
template <typename Links>
__global__ void __launch_bounds__(256) k_build_links(Links links, BlockSpec bs, BoxGeom g, double2* __restrict__ U64,
                                                     float2* __restrict__ U32, int* __restrict__ bad) {
  const int nt = g.ntiles;
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (item >= 8 * nt) return;
  const int mu = item & 3, tile = (item >> 2) % nt, p = (item >> 2) / nt;
  const int i = tile * kTile + lane;
  double2 u[10];
#pragma unroll
  for (int k = 0; k < 10; ++k) u[k] = make_double2(0, 0);   // entry 9 is the zero pad of the last pair
  if (i < g.Vh) {
    int y[4], x[4];
    eo_coords(g, p, i, y);
#pragma unroll
    for (int m = 0; m < 4; ++m) x[m] = bs.lo[m] + y[m];
    const double2* src = links.at(bs.L, x, mu);
#pragma unroll
    for (int k = 0; k < 9; ++k) u[k] = src[Links::kStep * k];
    // third row against conj(row 0 x row 1)
    double dev = 0;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int a = (q + 1) % 3, b = (q + 2) % 3;
      const double2 x1 = u[a], y1 = u[3 + b], x2 = u[b], y2 = u[3 + a];
      const double cr = (x1.x * y1.x - x1.y * y1.y) - (x2.x * y2.x - x2.y * y2.y);
      const double ci = (x1.x * y1.y + x1.y * y1.x) - (x2.x * y2.y + x2.y * y2.x);
      dev = fmax(dev, fabs(u[6 + q].x - cr) + fabs(u[6 + q].y + ci));
    }
    if (!(dev <= 1e-5)) atomicOr(bad, 2);
    const int ym = mu == 0 ? y[0] : (mu == 1 ? y[1] : (mu == 2 ? y[2] : y[3]));
    const int Lb = mu == 0 ? g.L[0] : (mu == 1 ? g.L[1] : (mu == 2 ? g.L[2] : g.L[3]));
    const int Ll = mu == 0 ? bs.L[0] : (mu == 1 ? bs.L[1] : (mu == 2 ? bs.L[2] : bs.L[3]));
    double f = 1.0;
    if (ym == Lb - 1) {
      if (Lb != Ll) f = 0.0;                          // Dirichlet face of the domain
      else if (mu == 0 && bs.tbc == 1) f = -1.0;      // antiperiodic wrap in time
      else if (mu == 0 && bs.tbc == 2) f = 0.0;       // open: no hop across the time boundary
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) u[k] = make_double2(f * u[k].x, f * u[k].y);
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) st2nt(U64 + lidx(nt, p, mu, 2 * k, i), u[2 * k], u[2 * k + 1]);
#pragma unroll
  for (int k = 0; k < 3; ++k)
    st2nt(U32 + lidx2(nt, p, mu, 2 * k, i), make_float2((float)u[2 * k].x, (float)u[2 * k].y),
          make_float2((float)u[2 * k + 1].x, (float)u[2 * k + 1].y));
}

// --------------------------------------------------------------- SU(3) FP64
__device__ __forceinline__ double2 dmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 dmulc(double2 a, double2 b) {  // conj(a) b
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}
// y = x + dmu mu + dnu nu (periodic gauge field), without indexing x by mu
__device__ __forceinline__ void nbr(const int L[4], const int x[4], int mu, int dmu, int nu, int dnu, int y[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int v = x[m] + (m == mu ? dmu : 0) + (m == nu ? dnu : 0);
    y[m] = v < 0 ? v + L[m] : (v >= L[m] ? v - L[m] : v);
  }
}

// A += sign times one staple of U_mu(x) in the (mu, nu) plane:
//   up    U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
//   down  U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
// row by row, so that two of its three links and A are live.
template <typename Links>
__device__ __forceinline__ void add_staple(const Links& links, const int L[4], const int x[4], int mu, int nu,
                                           bool down, double sign, double2 A[9]) {
  constexpr int S = Links::kStep;
  int y[4];
  nbr(L, x, mu, 1, nu, down ? -1 : 0, y);
  const double2* pa = links.at(L, y, nu);
  nbr(L, x, mu, 0, nu, down ? -1 : 1, y);
  const double2* pb = links.at(L, y, mu);
  nbr(L, x, mu, 0, nu, down ? -1 : 0, y);
  const double2* pc = links.at(L, y, nu);
  double2 b[9], c[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) b[k] = pb[S * k];
  // c^dag (up) or c (down), as the right factor
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      const double2 v = pc[S * (down ? 3 * i + j : 3 * j + i)];
      c[3 * i + j] = make_double2(v.x, down ? v.y : -v.y);
    }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    double2 a[3], t[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {   // row i of a (up) or a^dag (down)
      const double2 v = pa[S * (down ? 3 * k + i : 3 * i + k)];
      a[k] = make_double2(sign * v.x, sign * (down ? -v.y : v.y));
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      t[j] = make_double2(0, 0);
#pragma unroll
      for (int k = 0; k < 3; ++k) {   // a_k conj(b_jk)
        t[j].x += a[k].x * b[3 * j + k].x + a[k].y * b[3 * j + k].y;
        t[j].y += a[k].y * b[3 * j + k].x - a[k].x * b[3 * j + k].y;
      }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double2 w = dmul(t[k], c[3 * k + j]);
        A[3 * i + j].x += w.x;
        A[3 * i + j].y += w.y;
      }
  }
}

// Fhat_{mu nu}(x) = (Q - Q^dag)/8, Q the sum of the four counter-clockwise
// leaves at x.  With D(x) the up staple of U_mu(x) minus the down one, two of
// the leaves and the adjoints of the others make Q - Q^dag = Z - Z^dag with
//   Z = U_mu(x) D(x) + D(x-mu) U_mu(x-mu):
// ten 3x3 products instead of the twelve of four leaves.  Z - Z^dag is
// anti-Hermitian and kept as nine numbers: F[0..2] the imaginary diagonal, then
// entries (0,1), (0,2), (1,2).
template <typename Links>
__device__ __forceinline__ void field_strength(const Links& links, const int L[4], const int x[4], int mu, int nu,
                                               double F[9]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) F[k] = 0;
#pragma unroll 1
  for (int back = 0; back < 2; ++back) {
    int y[4];
    nbr(L, x, mu, -back, nu, 0, y);
    double2 D[9], u[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) D[k] = make_double2(0, 0);
#pragma unroll 1
    for (int down = 0; down < 2; ++down) add_staple(links, L, y, mu, nu, down, down ? -0.125 : 0.125, D);
    const double2* pu = links.at(L, y, mu);
#pragma unroll
    for (int k = 0; k < 9; ++k) u[k] = pu[Links::kStep * k];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        double2 z = make_double2(0, 0);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double2 l = back ? D[3 * i + k] : u[3 * i + k], r = back ? u[3 * k + j] : D[3 * k + j];
          const double2 w = dmul(l, r);
          z.x += w.x;
          z.y += w.y;
        }
        if (i == j) {
          F[i] += 2 * z.y;
        } else {
          const int e = 3 + 2 * (i + j - 1);   // pair (0,1), (0,2) or (1,2)
          F[e] += i < j ? z.x : -z.x;
          F[e + 1] += z.y;
        }
      }
  }
}

// A Hermitian 6x6 block is kept packed: the real diagonal d[6] and the 15
// upper elements u[] row-major (row r holds columns r+1..5).
__device__ __forceinline__ constexpr int up_idx(int r, int c) { return r * (11 - r) / 2 + (c - r - 1); }
// strictly lower (i > j) packed row-major
__device__ __forceinline__ constexpr int lo_idx(int i, int j) { return i * (i - 1) / 2 + j; }

// Clover term of every site of the box, as the two chiral 6x6 blocks of
//   A = 1 + sum_l s_l (x) X_l^{+-},  X_l^{+-} = i kappa c_sw (+-Fhat_{0l} - B_l).
// A workgroup is one 64-site tile of a parity and six wavefronts, one per plane
// (0,1) (0,2) (0,3) (2,3) (1,3) (1,2): each leaves its Fhat in LDS, then wavefront
// b packs block b.  s_3 puts X_3 on the diagonal spin blocks with + and -, s_1
// and s_2 put X_1 - i X_2 on the upper off-diagonal spin block.
// Bound by its chain of link loads (three waves per SIMD): 24^3 x 16 takes 0.30 ms
// with the working copy (0.07 ms to make); 0.52 ms with the nine complex numbers
// of Fhat, which spill, and parity by parity over the box; 0.81 ms when a thread
// built both blocks of a site from canonical links, every plane twice.
template <typename Links>
__global__ void __launch_bounds__(384) __attribute__((amdgpu_waves_per_eu(3)))
    k_build_clover(Links links, BlockSpec bs, BoxGeom g, double2* __restrict__ A64) {
  __shared__ double Fs[6][9][kTile];
  const int nt = g.ntiles, w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int id = xcd_chunk(blockIdx.x, 2 * nt);
  const int p = id & 1, tile = id >> 1;
  const int i = tile * kTile + lane;
  const double c = bs.kappa * bs.csw;
  double F[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) F[k] = 0;
  if (i < g.Vh && c != 0.0) {
    int y[4], x[4];
    eo_coords(g, p, i, y);
#pragma unroll
    for (int m = 0; m < 4; ++m) x[m] = bs.lo[m] + y[m];
    const int mu = w < 3 ? 0 : (w == 3 ? 2 : 1);
    const int nu = w < 3 ? w + 1 : (w == 5 ? 2 : 3);
    field_strength(links, bs.L, x, mu, nu, F);
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) Fs[w][k][lane] = F[k];
  __syncthreads();
  if (w >= 2) return;
  const double sg = w == 0 ? 1.0 : -1.0, one = i < g.Vh ? 1.0 : 0.0;   // padding sites hold zeros
  // number k of +-Fhat_{0l} - B_l: B_1 = Fhat_23, B_2 = -Fhat_13, B_3 = Fhat_12
  auto f = [&](int l, int k) { return sg * Fs[l][k][lane] + (l == 1 ? 1.0 : -1.0) * Fs[3 + l][k][lane]; };
  // entry (a, b) of X_{l+1} = i c (...)
  auto X = [&](int l, int a, int b) {
    if (a == b) return make_double2(-c * f(l, a), 0.0);
    const int e = 3 + 2 * (a + b - 1);
    const double x = f(l, e), y = f(l, e + 1);
    return make_double2(-c * y, a < b ? c * x : -c * x);
  };
  double dg[6];
  double2 up[15];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double d = X(2, a, a).x;
    dg[a] = one + d;
    dg[3 + a] = one - d;
#pragma unroll
    for (int b = a + 1; b < 3; ++b) {
      const double2 z = X(2, a, b);
      up[up_idx(a, b)] = z;
      up[up_idx(3 + a, 3 + b)] = make_double2(-z.x, -z.y);
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const double2 z1 = X(0, a, b), z2 = X(1, a, b);
      up[up_idx(a, 3 + b)] = make_double2(z1.x + z2.y, z1.y - z2.x);
    }
  }
  double2* A = A64 + cidx(nt, p, 18 * w, i);
  st2(A, make_double2(dg[0], dg[1]), make_double2(dg[2], dg[3]));
  st2(A + 128, make_double2(dg[4], dg[5]), up[0]);
#pragma unroll
  for (int k = 0; k < 7; ++k) st2(A + 128 * (2 + k), up[1 + 2 * k], up[2 + 2 * k]);
}

// Inverse of each packed block by Cholesky A = L L^dag in FP64:
//   L_jj = sqrt(A_jj - sum_{k<j} |L_jk|^2),  L_ij = (A_ij - sum_{k<j} L_ik conj(L_jk)) / L_jj,
//   W = L^{-1} (lower),  A^{-1} = W^dag W.
// One thread per (parity, block, site); a non-positive pivot sets *bad.
// Padding sites are zeroed.
__global__ void __launch_bounds__(128) k_invert_clover(const double2* __restrict__ A64, int nt, int Vh,
                                                       double2* __restrict__ Ainv64, float2* __restrict__ Ainv32,
                                                       int* __restrict__ bad) {
  const size_t per = (size_t)nt * kTile, n = 4 * per;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(t % per);
    const int pb = (int)(t / per);
    const int p = pb >> 1, blk = pb & 1;
    if (i >= Vh) {
      for (int k = 0; k < 18; ++k) {
        Ainv64[cidx(nt, p, 18 * blk + k, i)] = make_double2(0, 0);
        Ainv32[cidx(nt, p, 18 * blk + k, i)] = make_float2(0, 0);
      }
      continue;
    }
    double ad[6];
    double2 au[15];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double2 v = A64[cidx(nt, p, 18 * blk + k, i)];
      ad[2 * k] = v.x;
      ad[2 * k + 1] = v.y;
    }
#pragma unroll
    for (int k = 0; k < 15; ++k) au[k] = A64[cidx(nt, p, 18 * blk + 3 + k, i)];
    double ld[6], dinv[6];
    double2 lo[15];
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      double dj = ad[j];
#pragma unroll
      for (int k = 0; k < j; ++k) dj -= lo[lo_idx(j, k)].x * lo[lo_idx(j, k)].x + lo[lo_idx(j, k)].y * lo[lo_idx(j, k)].y;
      if (!(dj > 0)) {
        ok = false;
        dj = 1.0;
      }
      ld[j] = sqrt(dj);
      dinv[j] = 1.0 / ld[j];
#pragma unroll
      for (int r = j + 1; r < 6; ++r) {
        // A_rj = conj(A_jr) for r > j
        double2 s2 = make_double2(au[up_idx(j, r)].x, -au[up_idx(j, r)].y);
#pragma unroll
        for (int k = 0; k < j; ++k) {
          const double2 q = dmulc(lo[lo_idx(j, k)], lo[lo_idx(r, k)]);  // L_rk conj(L_jk)
          s2.x -= q.x;
          s2.y -= q.y;
        }
        lo[lo_idx(r, j)] = make_double2(s2.x * dinv[j], s2.y * dinv[j]);
      }
    }
    if (!ok) atomicOr(bad, 1);
    // W = L^{-1}: diagonal dinv, strictly lower wo
    double2 wo[15];
#pragma unroll
    for (int j = 0; j < 6; ++j)
#pragma unroll
      for (int r = j + 1; r < 6; ++r) {
        double2 s2 = dmul(lo[lo_idx(r, j)], make_double2(dinv[j], 0.0));
#pragma unroll
        for (int k = j + 1; k < r; ++k) {
          const double2 q = dmul(lo[lo_idx(r, k)], wo[lo_idx(k, j)]);
          s2.x += q.x;
          s2.y += q.y;
        }
        wo[lo_idx(r, j)] = make_double2(-s2.x * dinv[r], -s2.y * dinv[r]);
      }
    // (A^{-1})_rc = sum_{k >= max(r,c)} conj(W_kr) W_kc; diagonal real
    auto w = [&](int k, int j) { return k == j ? make_double2(dinv[j], 0.0) : wo[lo_idx(k, j)]; };
    double idg[6];
#pragma unroll
    for (int r = 0; r < 6; ++r) {
      double acc = 0;
#pragma unroll
      for (int k = r; k < 6; ++k) {
        const double2 v = w(k, r);
        acc += v.x * v.x + v.y * v.y;
      }
      idg[r] = acc;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double2 v = make_double2(idg[2 * k], idg[2 * k + 1]);
      Ainv64[cidx(nt, p, 18 * blk + k, i)] = v;
      Ainv32[cidx(nt, p, 18 * blk + k, i)] = make_float2((float)v.x, (float)v.y);
    }
#pragma unroll
    for (int r = 0; r < 6; ++r)
#pragma unroll
      for (int cc = r + 1; cc < 6; ++cc) {
        double2 acc = make_double2(0, 0);
#pragma unroll
        for (int k = cc; k < 6; ++k) {
          const double2 q = dmulc(w(k, r), w(k, cc));
          acc.x += q.x;
          acc.y += q.y;
        }
        Ainv64[cidx(nt, p, 18 * blk + 3 + up_idx(r, cc), i)] = acc;
        Ainv32[cidx(nt, p, 18 * blk + 3 + up_idx(r, cc), i)] = make_float2((float)acc.x, (float)acc.y);
      }
  }
}

template <typename Links>
static hipError_t build_block(const Links& links, const BlockSpec& bs, const BoxGeom& g, double2* U64, float2* U32,
                              double2* A64, int* bad, hipStream_t st) {
  hipLaunchKernelGGL(k_build_links<Links>, dim3(2 * g.ntiles), dim3(256), 0, st, links, bs, g, U64, U32, bad);
  hipLaunchKernelGGL(k_build_clover<Links>, dim3(2 * g.ntiles), dim3(384), 0, st, links, bs, g, A64);
  return hipGetLastError();
}

hipError_t launch_build_block(const GaugeView& gv, const BoxLinks* copy, const BlockSpec& bs, const BoxGeom& g,
                              double2* U64, float2* U32, double2* A64, double2* Ainv64, float2* Ainv32, int* bad,
                              hipStream_t st) {
  hipError_t e = hipSuccess;
  if (copy) {
    e = launch_box_links(gv, *copy, bs, st);
    if (e == hipSuccess) e = build_block(*copy, bs, g, U64, U32, A64, bad, st);
  } else {
    e = build_block(CanonLinks{gv}, bs, g, U64, U32, A64, bad, st);
  }
  if (e != hipSuccess) return e;
  size_t grid = ((size_t)4 * g.ntiles * kTile + 127) / 128;
  if (grid > 16384) grid = 16384;
  hipLaunchKernelGGL(k_invert_clover, dim3((unsigned)grid), dim3(128), 0, st, A64, g.ntiles, g.Vh, Ainv64, Ainv32,
                     bad);
  return hipGetLastError();
}

// ------------------------------------------------------------ reordering
__global__ void k_gather(const double2* __restrict__ canon, BlockSpec bs, int p, int nrhs, double scale,
                         double2* __restrict__ eo) {
  const int Vb = bs.Lb[0] * bs.Lb[1] * bs.Lb[2] * bs.Lb[3];
  const int nt = ntiles_of(bs);
  const size_t V = (size_t)bs.L[0] * bs.L[1] * bs.L[2] * bs.L[3];
  const size_t n = (size_t)Vb * nrhs;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
    const int s = (int)(t % Vb);
    const int col = (int)(t / Vb);
    int y[4], x[4];
    lex_coords(bs.Lb, s, y);
    if (((y[0] + y[1] + y[2] + y[3]) & 1) != p) continue;
    for (int m = 0; m < 4; ++m) x[m] = bs.lo[m] + y[m];
    const double2* src = canon + ((size_t)col * V + gidx(bs.L, x)) * 12;
    const int i = s >> 1;
#pragma unroll
    for (int c = 0; c < 12; ++c)
      eo[fidx(nt, col, c, i)] = make_double2(scale * src[c].x, scale * src[c].y);
  }
}
__global__ void k_scatter(const double2* __restrict__ eo, BlockSpec bs, int p, int nrhs, double scale,
                          double2* __restrict__ canon) {
  const int Vb = bs.Lb[0] * bs.Lb[1] * bs.Lb[2] * bs.Lb[3];
  const int nt = ntiles_of(bs);
  const size_t V = (size_t)bs.L[0] * bs.L[1] * bs.L[2] * bs.L[3];
  const size_t n = (size_t)Vb * nrhs;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
    const int s = (int)(t % Vb);
    const int col = (int)(t / Vb);
    int y[4], x[4];
    lex_coords(bs.Lb, s, y);
    if (((y[0] + y[1] + y[2] + y[3]) & 1) != p) continue;
    for (int m = 0; m < 4; ++m) x[m] = bs.lo[m] + y[m];
    double2* dst = canon + ((size_t)col * V + gidx(bs.L, x)) * 12;
    const int i = s >> 1;
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      const double2 v = eo[fidx(nt, col, c, i)];
      dst[c] = make_double2(scale * v.x, scale * v.y);
    }
  }
}
// ----------------------------------------------------------- level-1 updates
// Quenched updates of the links of the slab [t0, t1) of a gauge version with
// the spatial links of slice t0 fixed (the level-1 updates of the two-level
// integration): Wilson plaquette action; per link a Cabibbo-Marinari
// heatbath over the SU(2) subgroups (0,1), (0,2), (1,2) with the
// Kennedy-Pendleton sampler, n_or SU(2) over-relaxation passes, projection
// onto SU(3).  One launch updates one (direction, parity) class, whose links
// do not enter each other's staples.  Random numbers: Philox4x32-10 (Salmon
// et al., SC'11), key (seed low word, seed high word ^ stream * 0x85EBCA6B),
// counter (site, mu | sweep << 2, 0x5EED, n), uniform (w + 1) / 2^32.
__device__ __forceinline__ void philox4x32_10(uint32_t x[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * x[0], p1 = (uint64_t)0xCD9E8D57u * x[2];
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0, hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    const uint32_t y0 = hi1 ^ x[1] ^ k0, y2 = hi0 ^ x[3] ^ k1;
    x[0] = y0;
    x[1] = lo1;
    x[2] = y2;
    x[3] = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

struct LinkDraws {
  uint32_t k0, k1, c0, c1, n;
  uint32_t w0, w1, w2, w3;
  int left;
  __device__ double next() {
    if (left == 0) {
      uint32_t x[4] = {c0, c1, 0x5EEDu, n};
      philox4x32_10(x, k0, k1);
      w0 = x[0];
      w1 = x[1];
      w2 = x[2];
      w3 = x[3];
      ++n;
      left = 4;
    }
    const uint32_t w = left == 4 ? w0 : (left == 3 ? w1 : (left == 2 ? w2 : w3));
    --left;
    return ((double)w + 1.0) * (1.0 / 4294967296.0);
  }
};

__device__ __forceinline__ void quat_times(const double a[4], const double b[4], double c[4]) {
  c[0] = a[0] * b[0] - a[1] * b[1] - a[2] * b[2] - a[3] * b[3];
  c[1] = a[0] * b[1] + b[0] * a[1] - (a[2] * b[3] - a[3] * b[2]);
  c[2] = a[0] * b[2] + b[0] * a[2] - (a[3] * b[1] - a[1] * b[3]);
  c[3] = a[0] * b[3] + b[0] * a[3] - (a[1] * b[2] - a[2] * b[1]);
}

// Angles are 2 pi r rounded to FP64, as the documented formula evaluates: sincospi(2 r)
// skips that rounding and takes 1% less, but then the angles are not those of any
// other FP64 evaluation of the same random numbers.
constexpr double kTwoPi = 2.0 * 3.14159265358979323846;

// Kennedy-Pendleton: x0 with density ~ sqrt(1 - x0^2) exp(alpha x0)
__device__ double kp_sample(double alpha, LinkDraws& d) {
  for (int tries = 0; tries <= 10000; ++tries) {
    const double r1 = d.next(), r2 = d.next(), r3 = d.next(), r4 = d.next();
    const double c = cos(kTwoPi * r2);
    const double lam2 = -(log(r1) + c * c * log(r3)) / (2.0 * alpha);
    if (r4 * r4 <= 1.0 - lam2) return 1.0 - 2.0 * lam2;
  }
  return 1.0;
}

__device__ void level1_link(double2 U[9], const double2 A[9], double beta, int n_or, LinkDraws& d) {
  for (int pass = 0; pass <= n_or; ++pass)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int i = k == 2 ? 1 : 0, j = k == 0 ? 1 : 2;
      // the 2x2 block (rows and columns i, j) of W = U A
      double2 wii = make_double2(0, 0), wij = wii, wji = wii, wjj = wii;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double2 ui = U[3 * i + c], uj = U[3 * j + c], ai = A[3 * c + i], aj = A[3 * c + j];
        wii = make_double2(wii.x + ui.x * ai.x - ui.y * ai.y, wii.y + ui.x * ai.y + ui.y * ai.x);
        wij = make_double2(wij.x + ui.x * aj.x - ui.y * aj.y, wij.y + ui.x * aj.y + ui.y * aj.x);
        wji = make_double2(wji.x + uj.x * ai.x - uj.y * ai.y, wji.y + uj.x * ai.y + uj.y * ai.x);
        wjj = make_double2(wjj.x + uj.x * aj.x - uj.y * aj.y, wjj.y + uj.x * aj.y + uj.y * aj.x);
      }
      const double q[4] = {0.5 * (wii.x + wjj.x), 0.5 * (wij.y + wji.y), 0.5 * (wij.x - wji.x),
                           0.5 * (wii.y - wjj.y)};
      const double norm = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
      if (norm < 1e-14) continue;
      const double vd[4] = {q[0] / norm, -q[1] / norm, -q[2] / norm, -q[3] / norm};
      double R[4];
      if (pass == 0) {
        const double x0 = kp_sample(2.0 * beta * norm / 3.0, d);
        const double rad = sqrt(fmax(0.0, 1.0 - x0 * x0));
        const double ct = 2.0 * d.next() - 1.0, ph = kTwoPi * d.next();
        const double st = sqrt(fmax(0.0, 1.0 - ct * ct));
        double sn, cs;
        sincos(ph, &sn, &cs);
        const double X[4] = {x0, rad * st * cs, rad * st * sn, rad * ct};
        quat_times(X, vd, R);
      } else {
        quat_times(vd, vd, R);  // over-relaxation keeps Re tr(R W)
      }
      // rows i, j of U <- [[r0 + i r3, r2 + i r1], [-r2 + i r1, r0 - i r3]] (rows i, j)
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const double2 ui = U[3 * i + c], uj = U[3 * j + c];
        U[3 * i + c] = make_double2(R[0] * ui.x - R[3] * ui.y + R[2] * uj.x - R[1] * uj.y,
                                    R[0] * ui.y + R[3] * ui.x + R[2] * uj.y + R[1] * uj.x);
        U[3 * j + c] = make_double2(-R[2] * ui.x - R[1] * ui.y + R[0] * uj.x + R[3] * uj.y,
                                    -R[2] * ui.y + R[1] * ui.x + R[0] * uj.y - R[3] * uj.x);
      }
    }
  // back onto SU(3): Gram-Schmidt on rows 0 and 1, row 2 = conj(row 0 x row 1)
  double n = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) n += U[c].x * U[c].x + U[c].y * U[c].y;
  n = 1.0 / sqrt(n);
#pragma unroll
  for (int c = 0; c < 3; ++c) U[c] = make_double2(U[c].x * n, U[c].y * n);
  double2 p = make_double2(0, 0);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double2 t = dmulc(U[c], U[3 + c]);
    p.x += t.x;
    p.y += t.y;
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double2 t = dmul(p, U[c]);
    U[3 + c] = make_double2(U[3 + c].x - t.x, U[3 + c].y - t.y);
  }
  n = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) n += U[3 + c].x * U[3 + c].x + U[3 + c].y * U[3 + c].y;
  n = 1.0 / sqrt(n);
#pragma unroll
  for (int c = 0; c < 3; ++c) U[3 + c] = make_double2(U[3 + c].x * n, U[3 + c].y * n);
  auto cross = [&](int a, int b, int e, int f) {  // conj(U[a] U[b] - U[e] U[f])
    const double2 t1 = dmul(U[a], U[b]), t2 = dmul(U[e], U[f]);
    return make_double2(t1.x - t2.x, -(t1.y - t2.y));
  };
  U[6] = cross(1, 5, 2, 4);
  U[7] = cross(2, 3, 0, 5);
  U[8] = cross(0, 4, 1, 3);
}

// One (direction, parity) class of a sweep: its links are those of the sites of
// parity `par` in slices [t0, t1) (spatial directions: [t0 + 1, t1)), enumerated
// as pairs along x3, 64 to a tile.  None of them enters another's staples.
struct LinkClass {
  int t0, t1, mu, par;
  __host__ __device__ size_t size(const int L[4]) const {   // frozen spatial links of the first slice
    return (size_t)(t1 - t0 - (mu != 0)) * L[1] * L[2] * (L[3] / 2);
  }
  __device__ __forceinline__ void site(const int L[4], size_t k, int x[4]) const {
    const int h3 = L[3] / 2;
    size_t r = k / h3;
    const int j = (int)(k - r * h3);
    x[2] = (int)(r % L[2]); r /= L[2];
    x[1] = (int)(r % L[1]);
    x[0] = t0 + (mu != 0) + (int)(r / L[1]);
    x[3] = 2 * j + ((par + x[0] + x[1] + x[2]) & 1);
  }
};

// Staple sums of a class, A[tile][9][64].  One workgroup per tile and one
// wavefront per staple: a wavefront that adds up all six waits for one set of
// loads after the other, and with a tile per wavefront the tiles in flight read
// the links around them from beyond the L2 about twice.
template <typename Links>
__global__ void __launch_bounds__(384) __attribute__((amdgpu_waves_per_eu(4)))
    k_level1_staples(Links links, BlockSpec bs, LinkClass cl, double2* __restrict__ out) {
  __shared__ double2 sm[3][9][64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int tile = xcd_chunk(blockIdx.x, gridDim.x);
  const size_t k = (size_t)tile * 64 + lane;
  double2 A[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) A[c] = make_double2(0, 0);
  if (k < cl.size(bs.L)) {
    int x[4];
    cl.site(bs.L, k, x);
    const int nu = w >> 1;
    add_staple(links, bs.L, x, cl.mu, nu < cl.mu ? nu : nu + 1, w & 1, 1.0, A);
  }
  // (0 + 3) + (1 + 4) + (2 + 5), in this order
  if (w >= 3)
#pragma unroll
    for (int c = 0; c < 9; ++c) sm[w - 3][c][lane] = A[c];
  __syncthreads();
  if (w < 3)
#pragma unroll
    for (int c = 0; c < 9; ++c) {
      const double2 v = sm[w][c][lane];
      sm[w][c][lane] = make_double2(A[c].x + v.x, A[c].y + v.y);
    }
  __syncthreads();
  for (int q = threadIdx.x; q < 9 * 64; q += 384) {
    const double2 u = (&sm[0][0][0])[q], v = (&sm[1][0][0])[q], z = (&sm[2][0][0])[q];
    out[(size_t)tile * 9 * 64 + q] = make_double2(u.x + v.x + z.x, u.y + v.y + z.y);
  }
}

// The update of the links of a class, one per thread, from their staple sums;
// without a place for those (staples null, canonical links) a thread adds up its
// own.
// On a 16 x 32^3 slab the staples of a class (262144 links) take 80 us, bound by
// the links they read (0.3 GB at least), and the updates 41 us, bound by the
// sampler's dependent FP64 operations (three waves per SIMD; four spill: 56 us).
// In one kernel a class took 193 us from canonical links and 123 us from the
// working copy, a wavefront for all six staples of its links, or 120 us with the
// first of six wavefronts updating; working copy in and out 0.23 ms per call.
template <typename Links>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3)))
    k_level1_update(Links links, BlockSpec bs, LinkClass cl, const double2* __restrict__ staples, double beta,
                    uint32_t k0, uint32_t k1, int sweep, int n_or) {
  const int tile = xcd_chunk(blockIdx.x, gridDim.x);
  const size_t k = (size_t)tile * 64 + threadIdx.x;
  if (k >= cl.size(bs.L)) return;
  int x[4];
  cl.site(bs.L, k, x);
  double2* own = links.at(bs.L, x, cl.mu);
  double2 A[9], U[9];
  if constexpr (std::is_same<Links, CanonLinks>::value) {
#pragma unroll
    for (int c = 0; c < 9; ++c) A[c] = make_double2(0, 0);
#pragma unroll 1
    for (int s = 0; s < 6; ++s)
      add_staple(links, bs.L, x, cl.mu, (s >> 1) < cl.mu ? s >> 1 : (s >> 1) + 1, s & 1, 1.0, A);
  } else {
    const double2* st = staples + (size_t)tile * 9 * 64 + threadIdx.x;
#pragma unroll
    for (int c = 0; c < 9; ++c) A[c] = st[64 * c];
  }
#pragma unroll
  for (int c = 0; c < 9; ++c) U[c] = own[Links::kStep * c];
  LinkDraws d{k0, k1, (uint32_t)gidx(bs.L, x), (uint32_t)(cl.mu | (sweep << 2)), 0u, 0u, 0u, 0u, 0u, 0};
  level1_link(U, A, beta, n_or, d);
#pragma unroll
  for (int c = 0; c < 9; ++c) own[Links::kStep * c] = U[c];
}

size_t level1_staple_bytes(const BlockSpec& bs, int t0, int t1) {
  return (LinkClass{t0, t1, 0, 0}.size(bs.L) + 63) / 64 * 9 * 64 * sizeof(double2);
}

template <typename Links>
static hipError_t level1_classes(const Links& links, double2* staples, const BlockSpec& bs, int t0, int t1,
                                 double beta, uint64_t seed, uint32_t stream, int nsweeps, int n_or, hipStream_t st) {
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32) ^ (stream * 0x85EBCA6Bu);
  for (int sweep = 0; sweep < nsweeps; ++sweep)
    for (int mu = 0; mu < 4; ++mu)
      for (int par = 0; par < 2; ++par) {
        const LinkClass cl{t0, t1, mu, par};
        const unsigned grid = (unsigned)((cl.size(bs.L) + 63) / 64);   // V <= 2^30: at most 2^23
        if (grid == 0) continue;   // a slab of one slice has no free spatial links
        if constexpr (!std::is_same<Links, CanonLinks>::value)
          hipLaunchKernelGGL(k_level1_staples<Links>, dim3(grid), dim3(384), 0, st, links, bs, cl, staples);
        hipLaunchKernelGGL(k_level1_update<Links>, dim3(grid), dim3(64), 0, st, links, bs, cl, staples, beta, k0, k1,
                           sweep, n_or);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
      }
  return hipSuccess;
}

// The slab's links and, when it is not the whole time extent, those of the
// slice above it (the only ones outside that staples of its free links read)
// are copied to `copy`, swept there and written back to the region.
hipError_t launch_level1_slab(const GaugeView& parent, double2* region, const BoxLinks& copy, double2* staples,
                              const BlockSpec& bs, int t0, int t1, double beta, uint64_t seed, uint32_t stream, int nsweeps, int n_or,
                              hipStream_t st) {
  hipError_t e = launch_box_links(parent, copy, bs, st);
  if (e == hipSuccess) e = level1_classes(copy, staples, bs, t0, t1, beta, seed, stream, nsweeps, n_or, st);
  if (e != hipSuccess) return e;
  const int n = (t1 - t0) * bs.L[1] * bs.L[2] * bs.L[3];
  hipLaunchKernelGGL(k_box_copy<false>, dim3((n + 63) / 64), dim3(256), 0, st, parent, region, bs, copy, n);
  return hipGetLastError();
}

hipError_t launch_level1_sweeps(const GaugeView& gv, const BlockSpec& bs, double beta, uint64_t seed, uint32_t stream,
                                int nsweeps, int n_or, hipStream_t st) {
  return level1_classes(CanonLinks{gv}, nullptr, bs, gv.r_t0, gv.r_t1, beta, seed, stream, nsweeps, n_or, st);
}

// 16-bit copies for the FP16-storage inner solver: links with scale 1 (their
// entries are bounded by 1 in magnitude), A^{-1} with one scale per site.
__global__ void k_quant_links(const float2* __restrict__ U32, h16c* __restrict__ U16, size_t n) {
  for (size_t k = blockIdx.x * (size_t)blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x) {
    const float2 u = U32[k];
    U16[k] = h16c{q16(u.x * kQ), q16(u.y * kQ)};
  }
}
__global__ void k_quant_clover(const double2* __restrict__ A, h16c* __restrict__ A16, float* __restrict__ nrm,
                               int nt) {
  const size_t nsite = (size_t)2 * nt * kTile;
  for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < nsite; t += (size_t)gridDim.x * blockDim.x) {
    const int p = (int)(t / ((size_t)nt * kTile)), i = (int)(t % ((size_t)nt * kTile));
    double m = 0;
    for (int k = 0; k < kCloverSlots; ++k) {
      const double2 a = A[cidx(nt, p, k, i)];
      m = fmax(m, fmax(fabs(a.x), fabs(a.y)));
    }
    const float mf = (float)m;
    const float inv = mf > 0.f ? kQ / mf : 0.f;
    for (int k = 0; k < kCloverSlots; ++k) {
      const double2 a = A[cidx(nt, p, k, i)];
      A16[cidx(nt, p, k, i)] = h16c{q16((float)a.x * inv), q16((float)a.y * inv)};
    }
    nrm[t] = mf;
  }
}
hipError_t launch_quant_links(const float2* U32, h16c* U16, size_t n, hipStream_t st) {
  size_t g = (n + 255) / 256;
  hipLaunchKernelGGL(k_quant_links, dim3((int)(g > 16384 ? 16384 : (g ? g : 1))), dim3(256), 0, st, U32, U16, n);
  return hipGetLastError();
}
hipError_t launch_quant_clover(const double2* Ainv64, h16c* Ainv16, float* nrm, int ntiles, hipStream_t st) {
  size_t g = ((size_t)2 * ntiles * kTile + 255) / 256;
  hipLaunchKernelGGL(k_quant_clover, dim3((int)(g > 16384 ? 16384 : (g ? g : 1))), dim3(256), 0, st, Ainv64, Ainv16,
                     nrm, ntiles);
  return hipGetLastError();
}

static int grid_of(size_t n) {
  size_t g = (n + 255) / 256;
  return (int)(g > 16384 ? 16384 : (g == 0 ? 1 : g));
}
hipError_t launch_gather(const double2* canon, const BlockSpec& bs, int p, int nrhs, double scale, double2* eo,
                         hipStream_t st) {
  const size_t n = (size_t)bs.Lb[0] * bs.Lb[1] * bs.Lb[2] * bs.Lb[3] * nrhs;
  hipLaunchKernelGGL(k_gather, dim3(grid_of(n)), dim3(256), 0, st, canon, bs, p, nrhs, scale, eo);
  return hipGetLastError();
}
hipError_t launch_scatter(const double2* eo, const BlockSpec& bs, int p, int nrhs, double scale, double2* canon,
                          hipStream_t st) {
  const size_t n = (size_t)bs.Lb[0] * bs.Lb[1] * bs.Lb[2] * bs.Lb[3] * nrhs;
  hipLaunchKernelGGL(k_scatter, dim3(grid_of(n)), dim3(256), 0, st, eo, bs, p, nrhs, scale, canon);
  return hipGetLastError();
}

}  // namespace ddml
