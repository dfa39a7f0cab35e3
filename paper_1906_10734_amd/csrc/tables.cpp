// Constant tables, in double precision and rounded once to the plan's dtype (the paper precomputes
// the Green function and the matrices A, B, T before timing, Sec. 4). The host computes what is one
// dimensional (cosines, the 1-D fit and interpolation matrices, at most 4 KB) and passes it to the
// kernels below by value; they form the tables in place. A plan's creation pays for them: on the
// host they took 2.3 of the 3.5 ms of a one-shot solve of 3000 particles at N_g = 4, and 0.1 s of a
// plan with cell spectra at N_g = 6; here they are four launches with no copy and no wait. Sums run
// in index order without contraction, as they did there, so the values are the same; those of the
// screened kernel up to the last bit of the device's exp.
//
//   fit matrix   Effective masses from moments (Sec. 2.2, Eq. 4-5). The moments here are taken
//                in the tensor Legendre basis phi_n(x) = P_nx(2x) P_ny(2y) P_nz(2z), which spans
//                the same polynomials as the Cartesian monomials x^n of Eq. (2), so the matched
//                effective masses are identical; the fit matrix is B^phi = (Pmat)^{-1} with
//                Pmat[n][p] = phi_n(x_p), a Kronecker product of the 1-D inverse. Stored as the
//                GEMM operand W[n][p] = B^phi[p][n], zero padded.
//   child-to-parent  1-D factors of T^C (Sec. 2.3): T1^a[p][q] = l_p((a + x_q)/2) with
//                a = -1/2 or +1/2, the Lagrange basis l_p on the gridlet nodes (the matrix of
//                the paper's double sum, in closed form). Parent-to-child uses the transpose,
//                on the target gridlet's nodes (N_g + 2 of them when extended, Sec. 2.5).
//   Green transform  per level l >= 2: the exact lattice Green function G(d) = g(h_l |d|_p) of
//                Eq. (1) on the (8 N_g)^3 grid, h_l = size / (2^l N_g), with the problem's
//                kernel g (softened Newtonian -G (r^2+eps^2)^{-1/2}, or the screened one;
//                any kernel works, Sec. 4); for eps = 0 the origin takes the value at unit
//                offset. G is real and even along each axis, so its DFT is real, even and a
//                product of cosine sums; only the octant k in [0, n/2]^3 is stored, divided by
//                n^3 (the normalisation of the unnormalised inverse FFT). The same function
//                transformed along x and y only, at the z offsets 0 .. 4 N_g that separate a
//                target node from a source node (4 N_g = n/2 only with extended target gridlets),
//                and divided by n^2, serves the variant of the source-to-target step that
//                convolves along z in real space.
//   cell-by-cell Green transforms  (only for the cell-by-cell route, Sec. 2.5) per level and
//                source cube offset d in [-3, 3]^3: the C^3 cyclic array, C = 2 N_g + 2 ext,
//                whose entry u holds g(h_l |d N_g - u_c|), u_c = u for u < N_g + ext and u - C
//                otherwise, so that each node offset between a target node (N_g + 2 ext per
//                axis) and a source node sits on its own entry; its half spectrum
//                [kz][ky][kx <= C/2] by separable direct sums, divided by C^3, each offset's
//                row padded with zeros to a multiple of 16 modes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "hpm_internal.h"

namespace hpm {

// node i of a gridlet of N_g points per axis widened by ext nodes on each side
static double node(int ng, int i, int ext = 0) { return (2.0 * (i - ext) + 1.0 - ng) / (2.0 * ng); }

static double lagrange(int ng, int p, double u, int ext = 0) {
  double v = 1.0;
  for (int m = 0; m < ng + 2 * ext; ++m)
    if (m != p) v *= (u - node(ng, m, ext)) / (node(ng, p, ext) - node(ng, m, ext));
  return v;
}

static double legendre(int k, double t) {
  double p0 = 1.0, p1 = t;
  if (k == 0) return p0;
  for (int j = 1; j < k; ++j) {
    const double p2 = ((2.0 * j + 1.0) * t * p1 - j * p0) / (j + 1.0);
    p0 = p1;
    p1 = p2;
  }
  return p1;
}

// Gauss-Jordan inverse with partial pivoting of a small dense matrix (row-major, n x n).
static std::vector<double> invert(std::vector<double> a, int n) {
  std::vector<double> inv(size_t(n) * n, 0.0);
  for (int i = 0; i < n; ++i) inv[size_t(i) * n + i] = 1.0;
  for (int c = 0; c < n; ++c) {
    int piv = c;
    for (int r = c + 1; r < n; ++r)
      if (std::fabs(a[size_t(r) * n + c]) > std::fabs(a[size_t(piv) * n + c])) piv = r;
    for (int k = 0; k < n; ++k) {
      std::swap(a[size_t(c) * n + k], a[size_t(piv) * n + k]);
      std::swap(inv[size_t(c) * n + k], inv[size_t(piv) * n + k]);
    }
    const double d = a[size_t(c) * n + c];
    for (int k = 0; k < n; ++k) {
      a[size_t(c) * n + k] /= d;
      inv[size_t(c) * n + k] /= d;
    }
    for (int r = 0; r < n; ++r) {
      if (r == c) continue;
      const double f = a[size_t(r) * n + c];
      if (f == 0.0) continue;
      for (int k = 0; k < n; ++k) {
        a[size_t(r) * n + k] -= f * a[size_t(c) * n + k];
        inv[size_t(r) * n + k] -= f * inv[size_t(c) * n + k];
      }
    }
  }
  return inv;
}

// ---- kernels ------------------------------------------------------------------------------------
struct GreenKernel {
  double gconst, eps, screening, box;
  int yukawa;
  // the kernel at lattice distance h sqrt(q)
  __device__ double at(double h, double q) const {
#pragma clang fp contract(off)
    const double sd = sqrt(q * h * h + eps * eps);
    return yukawa ? -gconst * exp(-sd / screening) / sd : -gconst / sd;
  }
};

struct Cosines {  // cos and sin of 2 pi m / n, m < n
  double c[64];
};
struct CellTrig {  // cos and sin of 2 pi m / C
  double c[16], s[16];
};

constexpr int kTableThreads = 256;

// one plane z of the x-y transformed Green function of one level (grid: planes, levels), z, ky and
// kx <= n/2: LDS holds the plane's kernel values, then its x transform
__device__ __forceinline__ void green_plane(const GreenKernel& g, const double* s_cos, double* s_g,
                                            double* s_a, int ng, int ext, int li, int z) {
#pragma clang fp contract(off)
  const int n = 8 * ng, H = n / 2 + 1;
  const double h = g.box / (double(1 << (li + 2)) * ng);
  for (int e = threadIdx.x; e < H * H; e += kTableThreads) {
    const int x = e % H, y = e / H;
    // Offsets with max-norm <= N_g join a target node only to nodes of the 27 cubes around the
    // target, which are not sources; every interaction-zone pair is at least N_g + 1 apart along
    // some axis (N_g with the extended target gridlet, whose outer nodes lie one spacing closer to
    // the sources). Their values never reach a target potential, and zero keeps the largest
    // (near-origin) kernel values out of the transform, where they would only add rounding error.
    const bool unreachable = max(x, max(y, z)) <= ng - ext;
    double v = 0.0;
    if (!unreachable) {
      const double r2 = h * h * double(x * x + y * y + z * z);
      const double sd = sqrt(r2 + g.eps * g.eps);
      v = g.yukawa ? -g.gconst * exp(-sd / g.screening) / sd : -g.gconst / sd;
    }
    s_g[e] = v;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < H * H; e += kTableThreads) {  // [y][kx]
    const int kx = e % H, y = e / H;
    double acc = 0.0;
    for (int x = 0, m = 0; x < n; ++x) {
      acc += s_g[y * H + (x <= n / 2 ? x : n - x)] * s_cos[m];
      m += kx;
      if (m >= n) m -= n;
    }
    s_a[e] = acc;
  }
  __syncthreads();
}

// sum over y of the x transform: entry (ky, kx) of the plane
__device__ __forceinline__ double green_entry(const double* s_cos, const double* s_a, int n, int ky,
                                              int kx) {
#pragma clang fp contract(off)
  const int H = n / 2 + 1;
  double acc = 0.0;
  for (int y = 0, m = 0; y < n; ++y) {
    acc += s_a[(y <= n / 2 ? y : n - y) * H + kx] * s_cos[m];
    m += ky;
    if (m >= n) m -= n;
  }
  return acc;
}

constexpr int kMaxH = 33;  // N_g = 8

template <typename T>
__global__ __launch_bounds__(kTableThreads) void k_green_xy(GreenKernel g, Cosines cs, int ng, int ext,
                                                            T* gxy) {
#pragma clang fp contract(off)
  __shared__ double s_cos[64], s_g[kMaxH * kMaxH], s_a[kMaxH * kMaxH];
  const int n = 8 * ng, H = n / 2 + 1, z = blockIdx.x, li = blockIdx.y;
  if (threadIdx.x < 64) s_cos[threadIdx.x] = cs.c[threadIdx.x];
  green_plane(g, s_cos, s_g, s_a, ng, ext, li, z);
  const double inv_n2 = 1.0 / (double(n) * n);
  T* out = gxy + (size_t(li) * H + z) * H * H;  // planes d = z <= 4 N_g = n/2
  for (int e = threadIdx.x; e < H * H; e += kTableThreads)
    out[e] = T(green_entry(s_cos, s_a, n, e / H, e % H) * inv_n2);
}

// the full transform (N_g <= 3, the whole-grid kernel's table), one workgroup per level
constexpr int kMaxSmallH = 13;
template <typename T>
__global__ __launch_bounds__(kTableThreads) void k_green_xyz(GreenKernel g, Cosines cs, int ng, int ext,
                                                             T* ghat) {
#pragma clang fp contract(off)
  __shared__ double s_cos[64], s_g[kMaxSmallH * kMaxSmallH], s_a[kMaxSmallH * kMaxSmallH];
  __shared__ double s_p[kMaxSmallH * kMaxSmallH * kMaxSmallH];
  const int n = 8 * ng, H = n / 2 + 1, li = blockIdx.x;
  if (threadIdx.x < 64) s_cos[threadIdx.x] = cs.c[threadIdx.x];
  for (int z = 0; z < H; ++z) {
    green_plane(g, s_cos, s_g, s_a, ng, ext, li, z);
    for (int e = threadIdx.x; e < H * H; e += kTableThreads)
      s_p[z * H * H + e] = green_entry(s_cos, s_a, n, e / H, e % H);
    __syncthreads();
  }
  const double inv_n3 = 1.0 / (double(n) * n * n);
  for (int e = threadIdx.x; e < H * H * H; e += kTableThreads) {
    const int kz = e / (H * H), col = e % (H * H);
    double acc = 0.0;
    for (int z = 0, m = 0; z < n; ++z) {
      acc += s_p[(z <= n / 2 ? z : n - z) * H * H + col] * s_cos[m];
      m += kz;
      if (m >= n) m -= n;
    }
    ghat[size_t(li) * H * H * H + e] = T(acc * inv_n3);
  }
}

// Transform of the cyclic Green array of one source cube offset and level (grid: offsets, levels),
// C <= kMaxCellC: the kernel values and the y pass share one part of LDS, the x pass has the other.
template <typename T>
__global__ __launch_bounds__(kTableThreads) void k_green_cell(GreenKernel g, CellTrig tg, int ng, int ext,
                                                              int KP, T* gcell) {
#pragma clang fp contract(off)
  __shared__ double s_c[16], s_s[16];
  constexpr int kMaxModes = kMaxCellC * kMaxCellC * (kMaxCellC / 2 + 1);
  __shared__ double s_gv[2 * kMaxModes], s_a[2 * kMaxModes];
  const int C = 2 * ng + 2 * ext, HC = C / 2 + 1, tid = threadIdx.x;
  const int od = blockIdx.x, li = blockIdx.y;
  const int d0 = od % 7 - 3, d1 = (od / 7) % 7 - 3, d2 = od / 49 - 3;
  T* out = gcell + (size_t(li) * 343 + od) * KP * 2;
  const bool near = abs(d0) <= 1 && abs(d1) <= 1 && abs(d2) <= 1;  // never used: zero
  const int K = C * C * HC;
  for (int e = near ? tid : 2 * K + tid; e < 2 * KP; e += kTableThreads) out[e] = T(0);
  if (near) return;
  if (tid < 16) {
    s_c[tid] = tg.c[tid];
    s_s[tid] = tg.s[tid];
  }
  const double h = g.box / (double(1 << (li + 2)) * ng);
  for (int e = tid; e < C * C * C; e += kTableThreads) {
    const int x = e % C, y = (e / C) % C, z = e / (C * C);
    const double o0 = double(d0 * ng - (x < ng + ext ? x : x - C));
    const double o1 = double(d1 * ng - (y < ng + ext ? y : y - C));
    const double o2 = double(d2 * ng - (z < ng + ext ? z : z - C));
    s_gv[e] = g.at(h, o0 * o0 + o1 * o1 + o2 * o2);
  }
  __syncthreads();
  // x (real input): [z][y][kx]
  for (int e = tid; e < K; e += kTableThreads) {
    const int kx = e % HC, zy = e / HC;
    double re = 0.0, im = 0.0;
    for (int x = 0, m = 0; x < C; ++x) {
      const double v = s_gv[zy * C + x];
      re += v * s_c[m];
      im += v * -s_s[m];
      m += kx;
      if (m >= C) m -= C;
    }
    s_a[2 * e] = re;
    s_a[2 * e + 1] = im;
  }
  __syncthreads();
  // y: [z][ky][kx]
  for (int e = tid; e < K; e += kTableThreads) {
    const int kx = e % HC, ky = (e / HC) % C, z = e / (HC * C);
    double re = 0.0, im = 0.0;
    for (int y = 0, m = 0; y < C; ++y) {
      const int i = (z * C + y) * HC + kx;
      const double ar = s_a[2 * i], ai = s_a[2 * i + 1], c = s_c[m], sv = -s_s[m];
      re += ar * c - ai * sv;
      im += ar * sv + ai * c;
      m += ky;
      if (m >= C) m -= C;
    }
    s_gv[2 * e] = re;
    s_gv[2 * e + 1] = im;
  }
  __syncthreads();
  // z, / C^3, into the stored order: kz fastest; (re, im) interleaved, or in FP64 two real parts,
  // then two imaginary ones
  const double inv = 1.0 / (double(C) * C * C);
  constexpr int gm = sizeof(T) == 4 ? 1 : 2;
  for (int e = tid; e < K; e += kTableThreads) {
    const int kz = e % C, col = e / C;
    double re = 0.0, im = 0.0;
    for (int z = 0, m = 0; z < C; ++z) {
      const int i = z * C * HC + col;
      const double ar = s_gv[2 * i], ai = s_gv[2 * i + 1], c = s_c[m], sv = -s_s[m];
      re += ar * c - ai * sv;
      im += ar * sv + ai * c;
      m += kz;
      if (m >= C) m -= C;
    }
    const int at = (e / gm) * 2 * gm + e % gm;
    out[at] = T(re * inv);
    out[at + gm] = T(im * inv);
  }
}

// the 1-D matrices, and what is formed from them
struct Small {
  double b1[64];    // 1-D fit matrix [p][k]
  double t1[128];   // child-to-parent factors [2][N_g][N_g]
  double t1l[128];  // the same on the target gridlet's nodes [2][NL][NL]
  float tw[256];    // [8 N_g] {cos hi, sin hi, cos lo, sin lo}
};

template <typename T>
__global__ __launch_bounds__(kTableThreads) void k_small_tables(Small s, int ng, int nl, int kpad,
                                                                int mpad, T* fitw, T* m2m, T* l2l,
                                                                float* twff) {
#pragma clang fp contract(off)
  const int M = ng * ng * ng;
  const int e = blockIdx.x * kTableThreads + threadIdx.x;
  if (e < kpad * mpad) {
    const int n = e / mpad, q = e % mpad;
    double w = 0.0;
    if (n < M && q < M) {
      const int nx = n % ng, ny = (n / ng) % ng, nz = n / (ng * ng);
      const int px = q % ng, py = (q / ng) % ng, pz = q / (ng * ng);
      w = s.b1[px * ng + nx] * s.b1[py * ng + ny] * s.b1[pz * ng + nz];
    }
    fitw[e] = T(w);
  }
  if (e < 2 * ng * ng) m2m[e] = T(s.t1[e]);
  if (e < 2 * nl * nl) l2l[e] = T(s.t1l[e]);
  if (twff && e < 32 * ng) twff[e] = s.tw[e];
}

template <typename T>
static void tables_t(Plan& p, int nlev, const Small& small, const Cosines& cs, const CellTrig& tg,
                     hipStream_t s) {
  const int ng = p.ng, n = 8 * ng, H = n / 2 + 1, kpad = p.tab.kpad, mpad = p.tab.mpad;
  const GreenKernel g{p.prob.gconst, p.prob.softening, p.prob.screening, p.prob.box_size,
                      p.prob.kernel == HPM_KERNEL_YUKAWA ? 1 : 0};
  Tables& t = p.tab;
  t.fitw.reserve(size_t(kpad) * mpad * sizeof(T));
  t.m2m.reserve(size_t(2) * ng * ng * sizeof(T));
  t.l2l.reserve(size_t(2) * p.NL * p.NL * sizeof(T));
  if (sizeof(T) == 4) t.twff.reserve(size_t(n) * 16);
  k_small_tables<T><<<(kpad * mpad + kTableThreads - 1) / kTableThreads, kTableThreads, 0, s>>>(
      small, ng, p.NL, kpad, mpad, t.fitw.as<T>(), t.m2m.as<T>(), t.l2l.as<T>(),
      sizeof(T) == 4 ? t.twff.as<float>() : nullptr);
  HPM_LAUNCH_CHECK();
  t.gxy.reserve(size_t(std::max(nlev, 1)) * H * H * H * sizeof(T));
  if (nlev > 0) {
    k_green_xy<T><<<dim3(H, nlev), kTableThreads, 0, s>>>(g, cs, ng, p.ext, t.gxy.as<T>());
    HPM_LAUNCH_CHECK();
  }
  if (ng < 4) {
    t.ghat.reserve(size_t(std::max(nlev, 1)) * H * H * H * sizeof(T));
    if (nlev > 0) {
      k_green_xyz<T><<<nlev, kTableThreads, 0, s>>>(g, cs, ng, p.ext, t.ghat.as<T>());
      HPM_LAUNCH_CHECK();
    }
  }
  if (p.prob.m2l_mode != HPM_M2L_GRID) {
    if (2 * ng + 2 * p.ext > kMaxCellC) fail(HPM_ERR_UNSUPPORTED, "no cell spectra for this gridlet");
    const int KP = int(cell_modes(ng, p.ext));
    t.gcell.reserve(size_t(std::max(nlev, 1)) * 343 * KP * 2 * sizeof(T));
    if (nlev > 0) {
      k_green_cell<T><<<dim3(343, nlev), kTableThreads, 0, s>>>(g, tg, ng, p.ext, KP, t.gcell.as<T>());
      HPM_LAUNCH_CHECK();
    }
    t.gcell_levels = nlev;
  }
}

void build_tables(Plan& p, int max_levels, hipStream_t s) {
  const int ng = p.ng, M = ng * ng * ng, nl = p.NL, n = 8 * ng;
  p.tab.kpad = (M + 3) / 4 * 4;
  p.tab.mpad = (M + 15) / 16 * 16;
  Small small{};
  // 1-D Legendre-at-nodes matrix and its inverse
  std::vector<double> pm(size_t(ng) * ng);
  for (int k = 0; k < ng; ++k)
    for (int q = 0; q < ng; ++q) pm[size_t(k) * ng + q] = legendre(k, 2.0 * node(ng, q));
  const std::vector<double> b1 = invert(pm, ng);  // b1[p][k]
  std::copy(b1.begin(), b1.end(), small.b1);
  for (int a = 0; a < 2; ++a)
    for (int pp = 0; pp < ng; ++pp)
      for (int q = 0; q < ng; ++q)
        small.t1[(a * ng + pp) * ng + q] = lagrange(ng, pp, ((a ? 0.5 : -0.5) + node(ng, q)) / 2.0);
  for (int a = 0; a < 2; ++a)
    for (int pp = 0; pp < nl; ++pp)
      for (int q = 0; q < nl; ++q)
        small.t1l[(a * nl + pp) * nl + q] =
            lagrange(ng, pp, ((a ? 0.5 : -0.5) + node(ng, q, p.ext)) / 2.0, p.ext);
  // e^{+2 pi i m / n} as float pairs (hi, lo) per component, for the all-FP32 inverse transform
  Cosines cs{};
  for (int m = 0; m < n; ++m) {
    const double c = std::cos(2.0 * M_PI * m / n), sn = std::sin(2.0 * M_PI * m / n);
    const float ch = float(c), sh = float(sn);
    small.tw[4 * m] = ch;
    small.tw[4 * m + 1] = sh;
    small.tw[4 * m + 2] = float(c - double(ch));
    small.tw[4 * m + 3] = float(sn - double(sh));
    cs.c[m] = c;
  }
  const int C = 2 * ng + 2 * p.ext;
  CellTrig tg{};
  for (int m = 0; m < C && m < 16; ++m) {
    tg.c[m] = std::cos(2.0 * M_PI * double(m) / double(C));
    tg.s[m] = std::sin(2.0 * M_PI * double(m) / double(C));
  }
  // Green transforms of levels 2 .. nlevels-1
  const int nlev = std::max(0, max_levels - 2);
  if (p.prec == HPM_F32) tables_t<float>(p, nlev, small, cs, tg, s);
  else tables_t<double>(p, nlev, small, cs, tg, s);
}

}  // namespace hpm
