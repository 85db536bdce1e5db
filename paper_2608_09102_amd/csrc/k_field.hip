// k_field.hip -- the explicit field of the full model (Sec. 2): uniaxial
// anisotropy, a uniform external field and the stray field of the
// magnetization, entering the right-hand side of the scheme.
//
// The stray field is h = -N * m, the discrete convolution of m with the
// cell-averaged demagnetizing tensor of the grid's cubic cells (Newell,
// Williams and Dunlop 1993; the point-dipole tensor beyond 16 cells), taken as
// a cyclic convolution on the grid zero-padded to powers of two P >= 2n - 1
// per axis.  The three real components travel as two complex planes
// (m1 + i m2, and the half of m3's that its conjugate symmetry leaves); the
// forward transform reads the field itself and skips the lines that are zero,
// the product with the (real) transformed tensor separates the packed pair by
// conjugate symmetry, and the inverse transform writes h on the n-box.  The
// last axis is taken there and back in one kernel with the product between.
// Line transforms are mixed-radix Stockham passes in registers and LDS,
// several lines per workgroup.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "llg.h"
#include "llg_internal.h"

namespace llg {

namespace {

constexpr int TPB = 256;
inline unsigned nblk(int64_t n, int t = TPB) { return (unsigned)ceil_div(n > 0 ? n : 1, t); }

// ------------------------------------------------------------ demag tensor
// With m constant on the cubic cells of side h and the field averaged over
// each cell, the stray field of eq. stray_field is h_i = -sum_j N(k_i - k_j) m_j,
// where for the cell offset k (in cells, r = k h)
//   N_ab(k) = -(1/4pi) int_{[-1,1]^3} prod_d (1 - |s_d|) K_ab(k + s) ds,
//   K_ab(y) = d_a d_b (1/|y|) = (3 y_a y_b - delta_ab |y|^2) / |y|^5:
// averaging the field of one uniformly magnetized cube over another is the
// convolution of the point kernel with the autocorrelation of the cube, a tent
// of half-width one cell along each axis.  N does not depend on h.  The offset
// is handled by range (max norm of k):
//  - |k| <= 1, cells that touch or coincide (the integrand is singular):
//    closed form.  Along an axis where the kernel is differentiated twice the
//    tent average is the second difference of the kernel; along an axis where
//    it is not, the second difference of a second antiderivative.  So N is the
//    27-point second difference (weights 2 at 0, -1 at +-1 per axis), over
//    4 pi, of a generating function whose mixed derivatives give 1/|y| (Newell,
//    Williams and Dunlop 1993); the six generating functions are evaluated
//    together at each lattice point from the three logarithms and three
//    arctangents they share (gen6).
//  - 2 <= |k| <= 16: the integral above by Gauss-Legendre quadrature.  The
//    nearest point of the other cell is a cell away, so the integrand is
//    analytic on the domain; each axis is folded onto [0, 1], which leaves
//    the tent as the weight (1 - s).  Twelve nodes per folded axis reproduce
//    the closed form evaluated at 40 digits to about 1e-18 at |k| = 2, and
//    better beyond.
//  - |k| > 16: the point dipole -(1/4pi) K(k).
// Entries: 0 xx, 1 yy, 2 zz, 3 xy, 4 xz, 5 yz.  The diagonal entries are even
// in every coordinate of k; the xy entry is odd in k_x and k_y and even in
// k_z, and so on, so the positive octant determines the tensor.

constexpr int DEMAG_NEAR = 1, DEMAG_FAR = 16, GL_NODES = 12, GL_AXIS = 2 * GL_NODES;

// Nodes and weights of the folded rule on [0, 1] for the weight (1 - s).
struct GlRule {
  double t[GL_NODES], w[GL_NODES];
};

// The six generating values at a lattice point (coordinates taken by
// absolute value; the off-diagonal ones are odd in their first two
// arguments, applied by the caller).  With R = |y|, l_a = log((y_a + R) / rho_a)
// (rho_a the distance to the a axis; set to 0 where rho_a = 0, where each of
// its coefficients vanishes) and t_a = atan2(y_b y_c, y_a R):
//   F_aa = y_b (y_c^2 - y_a^2) l_b / 2 + y_c (y_b^2 - y_a^2) l_c / 2
//          - y_a y_b y_c t_a + (2 y_a^2 - y_b^2 - y_c^2) R / 6,
//   F_ab = y_a y_b y_c l_c + y_b (3 y_c^2 - y_b^2) l_a / 6 + y_a (3 y_c^2 - y_a^2) l_b / 6
//          - y_c^3 t_c / 6 - y_c y_b^2 t_b / 2 - y_c y_a^2 t_a / 2 - y_a y_b R / 3
// for (a, b, c) a cyclic or the matching order of (x, y, z).
__device__ void gen6(double x, double y, double z, double F[6]) {
  x = fabs(x);
  y = fabs(y);
  z = fabs(z);
  const double xx = x * x, yy = y * y, zz = z * z;
  const double R = sqrt(xx + yy + zz);
  if (R == 0.0) {
    for (int c = 0; c < 6; ++c) F[c] = 0.0;
    return;
  }
  const double ryz = sqrt(yy + zz), rxz = sqrt(xx + zz), rxy = sqrt(xx + yy);
  const double lx = ryz > 0.0 ? log((x + R) / ryz) : 0.0;
  const double ly = rxz > 0.0 ? log((y + R) / rxz) : 0.0;
  const double lz = rxy > 0.0 ? log((z + R) / rxy) : 0.0;
  const double tx = atan2(y * z, x * R), ty = atan2(x * z, y * R), tz = atan2(x * y, z * R);
  const double xyz = x * y * z, R6 = R / 6.0;
  F[0] = 0.5 * y * (zz - xx) * ly + 0.5 * z * (yy - xx) * lz - xyz * tx + (2.0 * xx - yy - zz) * R6;
  F[1] = 0.5 * x * (zz - yy) * lx + 0.5 * z * (xx - yy) * lz - xyz * ty + (2.0 * yy - xx - zz) * R6;
  F[2] = 0.5 * y * (xx - zz) * ly + 0.5 * x * (yy - zz) * lx - xyz * tz + (2.0 * zz - xx - yy) * R6;
  F[3] = xyz * lz + y * (3.0 * zz - yy) * lx / 6.0 + x * (3.0 * zz - xx) * ly / 6.0 - z * zz * tz / 6.0 -
         0.5 * z * yy * ty - 0.5 * z * xx * tx - x * y * R / 3.0;
  F[4] = xyz * ly + z * (3.0 * yy - zz) * lx / 6.0 + x * (3.0 * yy - xx) * lz / 6.0 - y * yy * ty / 6.0 -
         0.5 * y * zz * tz - 0.5 * y * xx * tx - x * z * R / 3.0;
  F[5] = xyz * lx + z * (3.0 * xx - zz) * ly / 6.0 + y * (3.0 * xx - yy) * lz / 6.0 - x * xx * tx / 6.0 -
         0.5 * x * zz * tz - 0.5 * x * yy * ty - y * z * R / 3.0;
}

__device__ inline double sgn(int64_t v) { return v > 0 ? 1.0 : (v < 0 ? -1.0 : 0.0); }

// closed form for |k| <= 1
__device__ void demag_near(int64_t X, int64_t Y, int64_t Z, double t[6]) {
  for (int c = 0; c < 6; ++c) t[c] = 0.0;
  for (int k = -1; k <= 1; ++k)
    for (int j = -1; j <= 1; ++j)
      for (int i = -1; i <= 1; ++i) {
        const double W = (i ? -1.0 : 2.0) * (j ? -1.0 : 2.0) * (k ? -1.0 : 2.0);
        const int64_t a = X + i, b = Y + j, c = Z + k;
        double F[6];
        gen6((double)a, (double)b, (double)c, F);
        const double sab = sgn(a) * sgn(b), sac = sgn(a) * sgn(c), sbc = sgn(b) * sgn(c);
        t[0] += W * F[0];
        t[1] += W * F[1];
        t[2] += W * F[2];
        t[3] += W * sab * F[3];
        t[4] += W * sac * F[4];
        t[5] += W * sbc * F[5];
      }
  for (int c = 0; c < 6; ++c) t[c] = t[c] / (4.0 * M_PI);
}

// -(1/4pi) K(y) (the point dipole; also the quadrature's integrand)
__device__ inline void dipole(double x, double y, double z, double t[6]) {
  const double r2 = x * x + y * y + z * z;
  const double s = -1.0 / (4.0 * M_PI * r2 * r2 * sqrt(r2));
  t[0] = s * (3.0 * x * x - r2);
  t[1] = s * (3.0 * y * y - r2);
  t[2] = s * (3.0 * z * z - r2);
  t[3] = s * 3.0 * x * y;
  t[4] = s * 3.0 * x * z;
  t[5] = s * 3.0 * y * z;
}

// The positive octant of offsets, T[c][node] on the n-box: the near and far
// ranges, one thread per offset (the quadrature range is k_demag_mid's).
__global__ void k_demag_octant(FieldDims f, double* __restrict__ T) {
  const int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t N = f.nx * f.ny * f.nz;
  if (node >= N) return;
  const int64_t X = node % f.nx, Y = (node / f.nx) % f.ny, Z = node / (f.nx * f.ny);
  const int64_t far = X > Y ? (X > Z ? X : Z) : (Y > Z ? Y : Z);
  double t[6];
  if (far <= DEMAG_NEAR)
    demag_near(X, Y, Z, t);
  else if (far > DEMAG_FAR)
    dipole((double)X, (double)Y, (double)Z, t);
  else
    return;
  for (int c = 0; c < 6; ++c) T[c * N + node] = t[c];
}

// The quadrature range, one workgroup per offset of the box
// [0, min(n, 17))^3; GL_AXIS^3 points (both halves of every folded axis).
constexpr int MID_TPB = 256;
__global__ __launch_bounds__(MID_TPB) void k_demag_mid(FieldDims f, GlRule q, double* __restrict__ T) {
  const int64_t mx = f.nx < DEMAG_FAR + 1 ? f.nx : DEMAG_FAR + 1;
  const int64_t my = f.ny < DEMAG_FAR + 1 ? f.ny : DEMAG_FAR + 1;
  const int64_t X = blockIdx.x % mx, Y = (blockIdx.x / mx) % my, Z = blockIdx.x / (mx * my);
  const int64_t far = X > Y ? (X > Z ? X : Z) : (Y > Z ? Y : Z);
  if (far <= DEMAG_NEAR) return;
  double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int p = threadIdx.x; p < GL_AXIS * GL_AXIS * GL_AXIS; p += MID_TPB) {
    const int a = p % GL_AXIS, b = (p / GL_AXIS) % GL_AXIS, c = p / (GL_AXIS * GL_AXIS);
    const double sa = a < GL_NODES ? q.t[a] : -q.t[a - GL_NODES];
    const double sb = b < GL_NODES ? q.t[b] : -q.t[b - GL_NODES];
    const double sc = c < GL_NODES ? q.t[c] : -q.t[c - GL_NODES];
    const double W = q.w[a % GL_NODES] * q.w[b % GL_NODES] * q.w[c % GL_NODES];
    double t[6];
    dipole((double)X + sa, (double)Y + sb, (double)Z + sc, t);
    for (int k = 0; k < 6; ++k) acc[k] += W * t[k];
  }
  __shared__ double red[6][MID_TPB];
  for (int k = 0; k < 6; ++k) red[k][threadIdx.x] = acc[k];
  __syncthreads();
  for (int s = MID_TPB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s)
      for (int k = 0; k < 6; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const int64_t N = f.nx * f.ny * f.nz, node = X + f.nx * (Y + f.ny * Z);
    for (int k = 0; k < 6; ++k) T[k * N + node] = red[k][0];
  }
}

// offset of padded index a along an axis of n cells padded to P (cyclic):
// a < n: +a; a > P - n: a - P; otherwise outside every cell pair (flag)
__device__ inline bool wrap(int64_t a, int64_t n, int64_t P, int64_t& off) {
  if (a < n) {
    off = a;
    return true;
  }
  if (a > P - n) {
    off = a - P;
    return true;
  }
  return false;
}

// ------------------------------------------------------------ FFT
// Line transforms by a mixed-radix Stockham scheme: a line of L = 2^BITS
// complex values is held by T = L / 8 threads, eight values each.  The first
// pass (radix 2, 4 or 8, no twiddles) works on the values as loaded from HBM,
// the radix-8 passes after it exchange through LDS, and the last one stores
// straight to HBM in natural order.  C lines share a workgroup (512 threads);
// for strided lines the C lines are adjacent in memory and lanes run across
// them first, so that a row of C values is read together.
struct FftPass {
  int64_t n_inner, n_inner1, inner_stride, outer_stride, s, plane_stride;  // n_inner1: of plane 1
  int n_load, n_store, dir;
  double scale;
};

__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ inline double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// times dir * i
__device__ inline double2 cmul_i(double2 a, double dir) { return make_double2(-dir * a.y, dir * a.x); }

// DFT of 2, 4 or 8 values with kernel exp(dir 2 pi i n k / R), in place
__device__ inline void dft4(double2& a0, double2& a1, double2& a2, double2& a3, double dir) {
  const double2 t0 = cadd(a0, a2), t1 = csub(a0, a2), t2 = cadd(a1, a3), t3 = cmul_i(csub(a1, a3), dir);
  a0 = cadd(t0, t2);
  a2 = csub(t0, t2);
  a1 = cadd(t1, t3);
  a3 = csub(t1, t3);
}
template <int R>
__device__ inline void dft(double2* v, double dir) {
  if constexpr (R == 2) {
    const double2 t = v[0];
    v[0] = cadd(t, v[1]);
    v[1] = csub(t, v[1]);
  } else if constexpr (R == 4) {
    dft4(v[0], v[1], v[2], v[3], dir);
  } else {
    double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1], o1 = v[3], o2 = v[5], o3 = v[7];
    dft4(e0, e1, e2, e3, dir);
    dft4(o0, o1, o2, o3, dir);
    const double r2 = 0.70710678118654752440;
    o1 = make_double2(r2 * (o1.x - dir * o1.y), r2 * (o1.y + dir * o1.x));     // (1 + dir i) / sqrt 2
    o2 = cmul_i(o2, dir);                                                       // dir i
    o3 = make_double2(r2 * (-o3.x - dir * o3.y), r2 * (-o3.y + dir * o3.x));   // (-1 + dir i) / sqrt 2
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1);
    v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2);
    v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3);
    v[7] = csub(e3, o3);
  }
}

// exp(2 pi i k / 4096), filled with every tensor (the same values each time,
// so streams may overlap).  Three loads replace three sincospi a pass, most of
// its arithmetic: the last axis of 120 x 90 x 50 88 -> 80 us, 500^2's 45 -> 33.
constexpr int FFT_MAX_BITS = 12;
__device__ double2 fft_unit[1 << FFT_MAX_BITS];
__global__ void k_fft_unit() {
  const int k = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (k >= 1 << FFT_MAX_BITS) return;
  double s, c;
  sincospi(2.0 * (double)k / (double)(1 << FFT_MAX_BITS), &s, &c);
  fft_unit[k] = make_double2(c, s);
}

// w[r - 1] = exp(dir 2 pi i k r / 2^bits) for r = 1..7, k < 2^bits / 8
__device__ inline void twiddles8(double2* w, double dir, int k, int bits) {
  k <<= FFT_MAX_BITS - bits;
  w[0] = fft_unit[k];
  w[1] = fft_unit[2 * k];
  w[3] = fft_unit[4 * k];
  w[0].y *= dir;
  w[1].y *= dir;
  w[3].y *= dir;
  w[2] = cmul(w[0], w[1]);
  w[4] = cmul(w[0], w[3]);
  w[5] = cmul(w[1], w[3]);
  w[6] = cmul(w[2], w[3]);
}

// The product H = Nhat M on the packed transforms.  Plane 0 holds
// Z = M1 + i M2, so M1(k) = (Z(k) + conj Z(-k)) / 2 and
// M2(k) = (Z(k) - conj Z(-k)) / 2i; plane 1 holds M3.  The result is packed
// the same way (H1 + i H2, H3).  e: the tensor at k; z, zm: Z at k and -k.
__device__ inline void demag_apply(const double* e, double2 z, double2 zm, double2 m3, double2& o0, double2& o1) {
  const double2 m1 = make_double2(0.5 * (z.x + zm.x), 0.5 * (z.y - zm.y));
  const double2 m2 = make_double2(0.5 * (z.y + zm.y), -0.5 * (z.x - zm.x));
  const double xx = e[0], yy = e[1], zz = e[2], xy = e[3], xz = e[4], yz = e[5];
  const double2 h1 = make_double2(xx * m1.x + xy * m2.x + xz * m3.x, xx * m1.y + xy * m2.y + xz * m3.y);
  const double2 h2 = make_double2(xy * m1.x + yy * m2.x + yz * m3.x, xy * m1.y + yy * m2.y + yz * m3.y);
  o1 = make_double2(xz * m1.x + yz * m2.x + zz * m3.x, xz * m1.y + yz * m2.y + zz * m3.y);
  o0 = make_double2(h1.x - h2.y, h1.y + h2.x);
}

// The shape of a line transform: threads per line, values per thread, lines
// per workgroup of NT threads.
template <int BITS, int NT>
struct FftShape {
  static constexpr int L = 1 << BITS;
  static constexpr int T = L >= 8 ? L / 8 : 1;
  static constexpr int NR = L >= 8 ? 8 : L;
  static constexpr int C = NT / T;
  static constexpr int LP = L + (L >> 3);  // padded line in LDS
  static constexpr int LDS = L >= 16 ? C * LP : 1;
};

constexpr int ilog2c(int v) { return v <= 1 ? 0 : 1 + ilog2c(v >> 1); }

// The transform of M lines in registers: v[m][r] holds entry j + r T of line m
// before and after.  Every thread of the workgroup calls it; LDS is free
// again after the next barrier.  The M lines share a pass's twiddle factors.
template <int BITS, int NT, bool CF, int M, typename V>
__device__ inline void fft_regs(V& v, double dir, double2* sm, int c, int j) {
  using S = FftShape<BITS, NT>;
  constexpr int L = S::L, T = S::T, C = S::C, LP = S::LP;
  if constexpr (L <= 8) {
#pragma unroll
    for (int m = 0; m < M; ++m) dft<L>(v[m], dir);
  } else {
    constexpr int R0 = (BITS % 3 == 0) ? 8 : (1 << (BITS % 3));
    constexpr int NMID = (BITS - (R0 == 8 ? 3 : BITS % 3)) / 3 - 1;  // radix-8 passes between
    auto lds = [&](int i) -> double2& { return CF ? sm[(i + (i >> 3)) * C + c] : sm[c * LP + i + (i >> 3)]; };
    // first pass: butterflies u of radix R0 on registers u + r (8 / R0)
    constexpr int U = 8 / R0;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      if (m > 0) __syncthreads();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        double2 w[R0];
#pragma unroll
        for (int r = 0; r < R0; ++r) w[r] = v[m][u + r * U];
        dft<R0>(w, dir);
        const int jj = j + u * T;
#pragma unroll
        for (int r = 0; r < R0; ++r) lds(jj * R0 + r) = w[r];
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 8; ++r) v[m][r] = lds(j + r * T);
    }
    double2 w[7];
#pragma unroll
    for (int mid = 0; mid < NMID; ++mid) {
      const int ns = R0 << (3 * mid), k = j & (ns - 1);
      twiddles8(w, dir, k, ilog2c(8 * ns));
      const int d = (j - k) * 8 + k;
#pragma unroll
      for (int m = 0; m < M; ++m) {
#pragma unroll
        for (int r = 1; r < 8; ++r) v[m][r] = cmul(v[m][r], w[r - 1]);
        dft<8>(v[m], dir);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 8; ++r) lds(d + r * ns) = v[m][r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 8; ++r) v[m][r] = lds(j + r * T);
      }
    }
    twiddles8(w, dir, j, BITS);  // ns = L / 8 = T, so k = j
#pragma unroll
    for (int m = 0; m < M; ++m) {
#pragma unroll
      for (int r = 1; r < 8; ++r) v[m][r] = cmul(v[m][r], w[r - 1]);
      dft<8>(v[m], dir);
    }
  }
}

template <int BITS, int NT, bool CF>
__global__ __launch_bounds__(NT) void k_fft(double2* __restrict__ data, FftPass p) {
  using S = FftShape<BITS, NT>;
  constexpr int T = S::T, NR = S::NR, C = S::C;
  __shared__ double2 sm[S::LDS];
  const int t = threadIdx.x;
  const int c = CF ? t % C : t / T;
  const int j = CF ? t / C : t % T;
  int64_t g = blockIdx.x;
  if (CF && (gridDim.x & 31) == 0) g = (g & ~(int64_t)31) | ((g & 7) << 2) | ((g >> 3) & 3);
  const int64_t gpo = (p.n_inner + C - 1) / C;
  const int64_t outer = (uint32_t)g / (uint32_t)gpo, first = (g - outer * gpo) * C;
  const int64_t n_inner = blockIdx.y == 0 ? p.n_inner : p.n_inner1;
  if (first >= n_inner) return;
  const int64_t inner = first + c;
  const bool live = inner < n_inner;
  double2* line = data + (int64_t)blockIdx.y * p.plane_stride + (live ? inner : 0) * p.inner_stride +
                  outer * p.outer_stride;
  const double dir = (double)p.dir;
  double2 v[1][NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int i = j + q * T;
    v[0][q] = (live && i < p.n_load) ? line[(int64_t)i * p.s] : make_double2(0.0, 0.0);
  }
  fft_regs<BITS, NT, CF, 1>(v, dir, sm, c, j);
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int i = j + q * T;
    if (live && i < p.n_store) line[(int64_t)i * p.s] = make_double2(v[0][q].x * p.scale, v[0][q].y * p.scale);
  }
}

// ---------------------------------------------- fused ends of the convolution
// The x transforms read the field itself (m~1 + i m~2 into plane 0, m~3 into
// plane 1) and, at the end, write h itself: the padded copy of the field and
// the copy back take no pass of their own.  m~3 is real, so plane 1 holds the
// columns kx <= px / 2 only, on the way there and back.  A row's two planes
// share a workgroup where a line leaves room for it, so that the 24 bytes of
// a node are read and written from one CU.  Bound by HBM and by the latency
// of one round of workgroups: 1024^2 23 us each (25 + 14 us for the transform
// and the padded copy, 25 + 10 at the end), 120 x 90 x 50 15 us (16 + 9, 16 + 7).
struct FieldRows {
  int64_t nx, rows, px, py, ny;  // cells of a row, rows of the box, padded lengths
  int64_t plane;
};
template <int C>
struct RowLine {
  int64_t row;
  int plane;
  bool live;
  __device__ RowLine(const FieldRows& f, int c) {
    if (C > 1) {
      row = (int64_t)blockIdx.x * (C / 2) + c / 2;
      plane = c & 1;
    } else {
      row = blockIdx.x;
      plane = (int)blockIdx.y;
    }
    live = row < f.rows;
    if (!live) row = 0;
  }
  __device__ int64_t line(const FieldRows& f) const {
    const int64_t b = (uint32_t)row / (uint32_t)f.ny;  // rows < 2^31
    return plane * f.plane + f.px * (row - b * f.ny + f.py * b);
  }
};

template <int BITS, int NT>
__global__ __launch_bounds__(NT) void k_fft_field_in(FieldRows f, const double* __restrict__ m,
                                                     const double* __restrict__ mprev, double2* __restrict__ w) {
  using S = FftShape<BITS, NT>;
  __shared__ double2 sm[S::LDS];
  const int c = (int)threadIdx.x / S::T, j = (int)threadIdx.x % S::T;
  const RowLine<S::C> r(f, c);
  double2 v[1][S::NR];
#pragma unroll
  for (int q = 0; q < S::NR; ++q) {
    const int64_t i = j + q * S::T;
    v[0][q] = make_double2(0.0, 0.0);
    if (r.live && i < f.nx) {
      const int64_t o = 3 * (r.row * f.nx + i) + (r.plane ? 2 : 0);
      v[0][q].x = mprev ? 2.0 * m[o] - mprev[o] : m[o];
      if (!r.plane) v[0][q].y = mprev ? 2.0 * m[o + 1] - mprev[o + 1] : m[o + 1];
    }
  }
  fft_regs<BITS, NT, false, 1>(v, -1.0, sm, c, j);
  if (!r.live) return;
  double2* line = w + r.line(f);
  const int last = r.plane ? S::L / 2 : S::L - 1;
#pragma unroll
  for (int q = 0; q < S::NR; ++q) {
    const int i = j + q * S::T;
    if (i <= last) line[i] = v[0][q];
  }
}

// h = -N * m: plane 0 gives h1 + i h2, plane 1 h3
template <int BITS, int NT>
__global__ __launch_bounds__(NT) void k_fft_field_out(FieldRows f, const double2* __restrict__ w, double scale,
                                                      double* __restrict__ h) {
  using S = FftShape<BITS, NT>;
  __shared__ double2 sm[S::LDS];
  const int c = (int)threadIdx.x / S::T, j = (int)threadIdx.x % S::T;
  const RowLine<S::C> r(f, c);
  const double2* line = w + r.line(f);
  double2 v[1][S::NR];
#pragma unroll
  for (int q = 0; q < S::NR; ++q) {
    const int i = j + q * S::T;
    const bool conj = r.plane && i > S::L / 2;
    v[0][q] = r.live ? line[conj ? S::L - i : i] : make_double2(0.0, 0.0);
    if (conj) v[0][q].y = -v[0][q].y;
  }
  fft_regs<BITS, NT, false, 1>(v, 1.0, sm, c, j);
  if (!r.live) return;
#pragma unroll
  for (int q = 0; q < S::NR; ++q) {
    const int64_t i = j + q * S::T;
    if (i >= f.nx) continue;
    const int64_t o = 3 * (r.row * f.nx + i) + (r.plane ? 2 : 0);
    h[o] = -(v[0][q].x * scale);
    if (!r.plane) h[o + 1] = -(v[0][q].y * scale);
  }
}

// The lines of the last axis, in pairs a = (kx, ky), b = (-kx, -ky): the
// product at k needs the transform at -k.  Pairs run over kx < px / 2 and all
// ky.  The columns kx = 0 and kx = px / 2, which mirror into themselves, share
// the turns of kx = 0: (0, ky) with (0, -ky) for ky < py / 2, (px / 2, ky)
// with (px / 2, -ky) above; where a line is its own mirror ("self": ky = 0,
// py / 2) the turn has a = (0, ky) and b = (px / 2, ky).
struct FusedPass {
  int64_t px, py;  // lines: kx < px, ky < py (1 where the last axis is y)
  int64_t s;       // stride of the last axis
  int64_t plane;   // values of a plane
  int n;           // cells along the last axis
  int hb;          // px / 2 = 2^hb
};
struct LinePair {
  int64_t ax, ky, bx, my;
  bool live, self;
  __device__ LinePair(const FusedPass& p, int64_t at) {
    const int64_t half = (int64_t)1 << p.hb;
    live = at < half * p.py;
    ky = live ? at >> p.hb : 0;
    my = (p.py - ky) & (p.py - 1);
    ax = at & (half - 1);
    bx = (p.px - ax) & (p.px - 1);
    self = live && ax == 0 && ky == my;
    if (self) bx = half;
    if (ax == 0 && ky > my) ax = bx = half;
  }
};

// The tensor's transform at entry k of line (kx, ky), kx <= px / 2.  It is
// real, even or odd along each axis, and only its octant is read: xy is odd
// along y, xz along z, yz along both; in 2D (FLAT) the last axis is y and xz
// and yz are zero.
template <bool FLAT>
__device__ inline void demag_entry(const FusedPass& p, const double* __restrict__ nhat, int64_t kx, int64_t ky,
                                   int k, int L, double* e) {
  const int64_t my = (p.py - ky) & (p.py - 1);
  const bool far = k > L / 2;
  const double* t = nhat + kx + p.px * (ky <= my ? ky : my) + (int64_t)(far ? L - k : k) * p.s;
  const double sy = ky <= my ? 1.0 : -1.0, sl = far ? -1.0 : 1.0;
  e[0] = t[0];
  e[1] = t[p.plane];
  e[2] = t[2 * p.plane];
  e[3] = t[3 * p.plane] * (FLAT ? sl : sy);
  e[4] = FLAT ? 0.0 : t[4 * p.plane] * sl;
  e[5] = FLAT ? 0.0 : t[5 * p.plane] * (sy * sl);
}

// The last axis in one kernel: forward transform, product with the tensor and
// inverse transform of a pair of lines without leaving the registers.  b is
// read backwards, so that a thread holds k of the one and -k of the other.
// Plane 1 is real in space: its line b is the conjugate of its line a and is
// neither read nor transformed.  Self lines are read forwards and their
// values at -k come through LDS; plane 1 is real along them, so its two lines
// are packed as a + i b.
// Bound by the requests of the strided loads (a wavefront's load takes a clock
// for each 128-byte line that it touches, C lines of 16 bytes abreast), then
// by latency at two wavefronts per SIMD: the three arrays take 96 registers
// of a thread.  120 x 90 x 50 (128 entries): 77 us, against 304 us for a
// pass each way and the product on all of the tensor between; 1024^2: 92 us
// against 198 us.  Workgroups of 128 threads where a line leaves the choice
// (120 x 90 x 50: 80 us with 256, 103 with 512), of 512 for 2048 entries and
// more (1024^2: 118 us with 256, which leaves one line abreast).
template <int BITS, int NT, bool FLAT>
__global__ __launch_bounds__(NT, 2) void k_fft_demag(double2* __restrict__ w, const double* __restrict__ nhat,
                                                  FusedPass p) {
  using S = FftShape<BITS, NT>;
  constexpr int L = S::L, T = S::T, C = S::C, NR = S::NR;
  __shared__ double2 sm[S::LDS];
  const int c = (int)threadIdx.x % C;
  int j = (int)threadIdx.x / C;
  int64_t g = blockIdx.x;
  if ((gridDim.x & 31) == 0) g = (g & ~(int64_t)31) | ((g & 7) << 2) | ((g >> 3) & 3);
  const LinePair l(p, g * C + c);
  const bool live = l.live, self = l.self;
  const int n = p.n;
  double2* la = w + l.ax + p.px * l.ky;
  double2* lb = w + l.bx + p.px * l.my;
  double2 v[3][NR];  // planes 0 and 1 of line a, plane 0 of line b
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const double2 zero = make_double2(0.0, 0.0);
    const int i = j + q * T, r = self ? i : (L - i) & (L - 1);
    v[0][q] = live && i < n ? la[(int64_t)i * p.s] : zero;
    v[1][q] = live && i < n ? la[p.plane + (int64_t)i * p.s] : zero;
    v[2][q] = live && r < n ? lb[(int64_t)r * p.s] : zero;
    if (self && i < n) v[1][q].y = lb[p.plane + (int64_t)i * p.s].x;
  }
  // no addresses or twiddle factors kept across the transforms, for the registers
  asm volatile("" : "+v"(j));
  fft_regs<BITS, NT, true, 3>(v, -1.0, sm, c, j);
  __syncthreads();
  // the turns 0 and py / 2 of kx = 0 (the same on the whole workgroup)
  const int64_t mid = p.py > 1 ? p.py / 2 << p.hb : 0;
  const bool any_self = g == 0 || g == mid / C;
  double2 m3b[NR];
  if (any_self) {
    auto mirrored = [&](const double2* x, double2* o) {  // x at -k
      if constexpr (T == 1) {
#pragma unroll
        for (int q = 0; q < NR; ++q) o[q] = x[(L - q) & (L - 1)];
      } else {
        auto lds = [&](int i) -> double2& { return sm[(i + (i >> 3)) * C + c]; };
#pragma unroll
        for (int q = 0; q < NR; ++q) lds(j + q * T) = x[q];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NR; ++q) o[q] = lds((L - (j + q * T)) & (L - 1));
        __syncthreads();
      }
    };
    double2 o[NR];
    double e[6];
    mirrored(v[1], o);
    if (self) {
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        const double2 z = v[1][q], zm = o[q];
        v[1][q] = make_double2(0.5 * (z.x + zm.x), 0.5 * (z.y - zm.y));
        m3b[q] = make_double2(0.5 * (z.y + zm.y), -0.5 * (z.x - zm.x));
      }
    }
    mirrored(v[0], o);
    if (self) {
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        demag_entry<FLAT>(p, nhat, l.ax, l.ky, j + q * T, L, e);
        demag_apply(e, v[0][q], o[q], v[1][q], v[0][q], v[1][q]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    mirrored(v[2], o);
    if (self) {
#pragma unroll
      for (int q = 0; q < NR; ++q) {
        double2 h3;
        demag_entry<FLAT>(p, nhat, l.bx, l.ky, j + q * T, L, e);
        demag_apply(e, v[2][q], o[q], m3b[q], v[2][q], h3);
        v[1][q] = make_double2(v[1][q].x - h3.y, v[1][q].y + h3.x);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (!self) {
#pragma unroll
    for (int q = 0; q < NR; ++q) {
      const double2 za = v[0][q], zb = v[2][q], m3 = v[1][q];
      double e[6];
      double2 none;
      demag_entry<FLAT>(p, nhat, l.ax, l.ky, j + q * T, L, e);
      demag_apply(e, za, zb, m3, v[0][q], v[1][q]);
      demag_apply(e, zb, za, make_double2(m3.x, -m3.y), v[2][q], none);
      if (q & 1) __builtin_amdgcn_sched_barrier(0);  // two entries' loads at a time
    }
  }
  asm volatile("" : "+v"(j));
  fft_regs<BITS, NT, true, 3>(v, 1.0, sm, c, j);
  asm volatile("" : "+v"(j));
  if (!live) return;
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int i = j + q * T, r = self ? i : (L - i) & (L - 1);
    if (r < n) lb[(int64_t)r * p.s] = v[2][q];
    if (i >= n) continue;
    la[(int64_t)i * p.s] = v[0][q];
    la[p.plane + (int64_t)i * p.s] = self ? make_double2(v[1][q].x, 0.0) : v[1][q];
    if (self) lb[p.plane + (int64_t)i * p.s] = make_double2(v[1][q].y, 0.0);
    if (!self && l.ax == l.bx) lb[p.plane + (int64_t)i * p.s] = make_double2(v[1][q].x, -v[1][q].y);
  }
}

// The same with a pair's three arrays (planes 0 and 1 of line a, plane 0 of
// line b) in the hands of S threads each, for grids that leave most of the
// chip idle: a third of the chain of transforms (200^2: 13 us against 18),
// but three times the twiddle factors and reads of the tensor (120 x 90 x 50:
// 113 us against 77).  The product reads the other arrays through LDS.
template <int BITS, int S, bool FLAT>
__global__ __launch_bounds__(3 * S, 3) void k_fft_demag3(double2* __restrict__ w, const double* __restrict__ nhat,
                                                         FusedPass p) {
  using F = FftShape<BITS, S>;
  constexpr int L = F::L, T = F::T, C = F::C, NR = F::NR, ARR = C * F::LP;
  __shared__ double2 sm[3 * ARR];
  const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x / S), tid = (int)threadIdx.x % S;
  const int c = tid % C;
  int j = tid / C;
  int64_t g = blockIdx.x;
  if ((gridDim.x & 31) == 0) g = (g & ~(int64_t)31) | ((g & 7) << 2) | ((g >> 3) & 3);
  const LinePair l(p, g * C + c);
  const bool live = l.live, self = l.self;
  const int n = p.n;
  double2* la = w + l.ax + p.px * l.ky;
  double2* lb = w + l.bx + p.px * l.my;
  double2* line = grp == 0 ? la : grp == 1 ? la + p.plane : lb;
  const bool back = grp == 2 && !self;  // line b is read backwards
  double2 v[1][NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int i = j + q * T, r = back ? (L - i) & (L - 1) : i;
    v[0][q] = live && r < n ? line[(int64_t)r * p.s] : make_double2(0.0, 0.0);
    if (grp == 1 && self && r < n) v[0][q].y = lb[p.plane + (int64_t)r * p.s].x;
  }
  asm volatile("" : "+v"(j));  // addresses and twiddle factors are not kept across the transforms
  double2* own = sm + grp * ARR;
  fft_regs<BITS, S, true, 1>(v, -1.0, own, c, j);
  __syncthreads();
  auto idx = [&](int i) { return (i + (i >> 3)) * C + c; };
#pragma unroll
  for (int q = 0; q < NR; ++q) own[idx(j + q * T)] = v[0][q];
  __syncthreads();
  const int64_t nx = self ? l.bx : l.ax;  // line b's column of the tensor
  const double2 *a0 = sm, *a1 = sm + ARR, *b0 = sm + 2 * ARR;
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int k = j + q * T, ik = idx(k), im = idx((L - k) & (L - 1));
    double e[6];
    double2 none, m3 = a1[ik], m3b = make_double2(m3.x, -m3.y);
    if (self) {
      const double2 z = m3, zm = a1[im];
      m3 = make_double2(0.5 * (z.x + zm.x), 0.5 * (z.y - zm.y));
      m3b = make_double2(0.5 * (z.y + zm.y), -0.5 * (z.x - zm.x));
    }
    if (grp == 0) {
      demag_entry<FLAT>(p, nhat, l.ax, l.ky, k, L, e);
      demag_apply(e, v[0][q], self ? a0[im] : b0[ik], m3, v[0][q], none);
    } else if (grp == 1) {
      demag_entry<FLAT>(p, nhat, l.ax, l.ky, k, L, e);
      demag_apply(e, a0[ik], self ? a0[im] : b0[ik], m3, none, v[0][q]);
      if (self) {
        double2 h;
        demag_entry<FLAT>(p, nhat, nx, l.ky, k, L, e);
        demag_apply(e, b0[ik], b0[im], m3b, none, h);
        v[0][q] = make_double2(v[0][q].x - h.y, v[0][q].y + h.x);
      }
    } else {
      demag_entry<FLAT>(p, nhat, nx, l.ky, k, L, e);
      demag_apply(e, v[0][q], self ? b0[im] : a0[ik], m3b, v[0][q], none);
    }
  }
  __syncthreads();
  asm volatile("" : "+v"(j));
  fft_regs<BITS, S, true, 1>(v, 1.0, own, c, j);
  asm volatile("" : "+v"(j));
  if (!live) return;
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    const int i = j + q * T, r = back ? (L - i) & (L - 1) : i;
    if (r >= n) continue;
    line[(int64_t)r * p.s] = grp == 1 && self ? make_double2(v[0][q].x, 0.0) : v[0][q];
    if (grp == 1 && self) lb[p.plane + (int64_t)r * p.s] = make_double2(v[0][q].y, 0.0);
    if (grp == 1 && !self && l.ax == l.bx) lb[p.plane + (int64_t)r * p.s] = make_double2(v[0][q].x, -v[0][q].y);
  }
}

// The product by itself, for long lines that are too few to fill the chip:
// there the transforms run plane by plane and line by line in passes of their
// own (5 x 2048: 52 us for the last axis in one kernel).
template <bool FLAT>
__global__ void k_demag_pairs(double2* __restrict__ w, const double* __restrict__ nhat, FusedPass p, int L) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, lines = p.py << p.hb;
  if (x >= lines * L) return;
  const int k = (int)(x / lines), m = (L - k) & (L - 1);
  const LinePair l(p, x % lines);
  if (l.self && k > m) return;  // done with -k
  for (int u = 0; u < (l.self ? 2 : 1); ++u) {
    const int64_t ax = u ? l.bx : l.ax, bx = l.self ? ax : l.bx;
    double2* a = w + ax + p.px * l.ky + k * p.s;
    double2* b = w + bx + p.px * l.my + m * p.s;
    const double2 z = a[0], zm = b[0], m3 = a[p.plane];
    double e[6];
    double2 o0, o1, r0, r1;
    demag_entry<FLAT>(p, nhat, ax, l.ky, k, L, e);
    demag_apply(e, z, zm, m3, o0, o1);
    demag_apply(e, zm, z, make_double2(m3.x, -m3.y), r0, r1);
    a[0] = o0;
    a[p.plane] = o1;
    if (a == b) continue;
    b[0] = r0;
    if (ax == bx) b[p.plane] = r1;
  }
}

// Workgroups of 512 threads; of 128 where the larger leave CUs without one
// (and a line fits): 200^2, 50 workgroups of an x pass, 6.5 -> 4.9 us.
constexpr int64_t FFT_FEW = 256;
// Workgroups of the kernel with an array per S threads up to which it is
// taken: four to a CU run at once (100 x 100 x 4: 10 us against 12; 50 x 60 x
// 33, 4096 of them: 32 us against 26).
constexpr int64_t DEMAG_FEW = 1024;
template <int BITS>
constexpr bool fft_narrow() {
  return FftShape<BITS, 512>::T <= 128;
}

template <int BITS, bool CF>
void launch_fft_t(hipStream_t st, double2* data, const FftPass& p, int64_t n_outer, int planes) {
  auto go = [&](auto nt) {
    constexpr int NT = decltype(nt)::value;
    const int64_t groups = ceil_div(p.n_inner, FftShape<BITS, NT>::C) * n_outer;
    if (NT > 128 && fft_narrow<BITS>() && groups * planes < FFT_FEW) return false;
    hipLaunchKernelGGL((k_fft<BITS, NT, CF>), dim3((unsigned)groups, (unsigned)planes), dim3(NT), 0, st, data, p);
    return true;
  };
  if (go(std::integral_constant<int, 512>{})) return;
  if constexpr (fft_narrow<BITS>()) go(std::integral_constant<int, 128>{});
}

template <bool CF>
void launch_fft_cf(hipStream_t st, int bits, double2* data, const FftPass& p, int64_t n_outer, int planes) {
  switch (bits) {
    case 1: return launch_fft_t<1, CF>(st, data, p, n_outer, planes);
    case 2: return launch_fft_t<2, CF>(st, data, p, n_outer, planes);
    case 3: return launch_fft_t<3, CF>(st, data, p, n_outer, planes);
    case 4: return launch_fft_t<4, CF>(st, data, p, n_outer, planes);
    case 5: return launch_fft_t<5, CF>(st, data, p, n_outer, planes);
    case 6: return launch_fft_t<6, CF>(st, data, p, n_outer, planes);
    case 7: return launch_fft_t<7, CF>(st, data, p, n_outer, planes);
    case 8: return launch_fft_t<8, CF>(st, data, p, n_outer, planes);
    case 9: return launch_fft_t<9, CF>(st, data, p, n_outer, planes);
    case 10: return launch_fft_t<10, CF>(st, data, p, n_outer, planes);
    case 11: return launch_fft_t<11, CF>(st, data, p, n_outer, planes);
    case 12: return launch_fft_t<12, CF>(st, data, p, n_outer, planes);
    default: throw LLG_ERR_UNSUPPORTED;  // lengths are checked when the context is created
  }
}

int ilog2(int64_t v) {
  int b = 0;
  while (((int64_t)1 << b) < v) ++b;
  return b;
}

// One transform along one axis, lines (inner, outer; of plane 1 only inner < n_inner1) of `planes` planes of P
// values: elements i < n_load are read (the rest taken as zero), i < n_store
// written; the inverse pass that ends a transform is scaled by 1 / P.
void fft_axis(hipStream_t st, double2* data, int64_t P, int planes, int64_t L, int64_t s, int64_t n_inner,
              int64_t n_inner1, int64_t inner_stride, int64_t n_outer, int64_t outer_stride, int64_t n_load, int64_t n_store, int dir,
              double scale) {
  if (L <= 1) return;
  FftPass p;
  p.n_inner = n_inner;
  p.n_inner1 = n_inner1;
  p.inner_stride = inner_stride;
  p.outer_stride = outer_stride;
  p.s = s;
  p.plane_stride = P;
  p.n_load = (int)n_load;
  p.n_store = (int)n_store;
  p.dir = dir;
  p.scale = scale;
  if (s == 1)
    launch_fft_cf<false>(st, ilog2(L), data, p, n_outer, planes);
  else
    launch_fft_cf<true>(st, ilog2(L), data, p, n_outer, planes);
}

// Forward transform of `planes` full padded planes.
void fft_forward_full(hipStream_t st, FieldDims f, double2* w, int planes) {
  const int64_t P = f.px * f.py * f.pz, pxy = f.px * f.py;
  fft_axis(st, w, P, planes, f.px, 1, f.py, f.py, f.px, f.pz, pxy, f.px, f.px, -1, 1.0);
  fft_axis(st, w, P, planes, f.py, f.px, f.px, f.px, 1, f.pz, pxy, f.py, f.py, -1, 1.0);
  fft_axis(st, w, P, planes, f.pz, pxy, pxy, pxy, 1, 1, 0, f.pz, f.pz, -1, 1.0);
}

// Two tensor components packed as one complex plane, a + i b, on the padded
// grid (cyclic offsets), from the octant table by the parities of the
// entries: both are real and even up to sign flips that the transform sees
// as real, so the packed transform's real and imaginary parts are the two
// transforms.
__global__ void k_demag_pair(FieldDims f, int c0, int c1, const double* __restrict__ T, double2* out) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t P = f.px * f.py * f.pz;
  if (p >= P) return;
  const int64_t a = p % f.px, b = (p / f.px) % f.py, c = p / (f.px * f.py);
  int64_t X, Y, Z;
  double v[2] = {0.0, 0.0};
  if (wrap(a, f.nx, f.px, X) && wrap(b, f.ny, f.py, Y) && wrap(c, f.nz, f.pz, Z)) {
    const int64_t N = f.nx * f.ny * f.nz;
    const int64_t node = (X < 0 ? -X : X) + f.nx * ((Y < 0 ? -Y : Y) + f.ny * (Z < 0 ? -Z : Z));
    const int cc[2] = {c0, c1};
    for (int r = 0; r < 2; ++r) {
      const int comp = cc[r];
      double s = 1.0;
      if (comp == 3) s = (X < 0 ? -1.0 : 1.0) * (Y < 0 ? -1.0 : 1.0);
      if (comp == 4) s = (X < 0 ? -1.0 : 1.0) * (Z < 0 ? -1.0 : 1.0);
      if (comp == 5) s = (Y < 0 ? -1.0 : 1.0) * (Z < 0 ? -1.0 : 1.0);
      v[r] = s * T[comp * N + node];
    }
  }
  out[p] = make_double2(v[0], v[1]);
}

__global__ void k_take_pair(int64_t P, int c0, int c1, const double2* in, double* nhat) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P) return;
  const double2 v = in[p];
  nhat[c0 * P + p] = v.x;
  nhat[c1 * P + p] = v.y;
}

// ------------------------------------------------------------ field terms
// b -= dt' (m~ x f + alpha m~ x (m~ x f)), f = (h_s + h_e) - q (0, m~2, m~3);
// prm: [0] alpha, [2] dt', [3] q, [4..6] h_e
__global__ void k_field_rhs(int64_t N, const double* prm, const double* m, const double* mprev, const double* h,
                            double* b) {
  const int64_t node = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= N) return;
  const double alpha = prm[0], dtp = prm[2], q = prm[3];
  double x[3], hs[3] = {0.0, 0.0, 0.0};
  for (int k = 0; k < 3; ++k) x[k] = mprev ? 2.0 * m[3 * node + k] - mprev[3 * node + k] : m[3 * node + k];
  if (h)
    for (int k = 0; k < 3; ++k) hs[k] = h[3 * node + k];
  const double fp[3] = {hs[0] + prm[4], (hs[1] + prm[5]) - q * x[1], (hs[2] + prm[6]) - q * x[2]};
  const double c1[3] = {x[1] * fp[2] - x[2] * fp[1], x[2] * fp[0] - x[0] * fp[2], x[0] * fp[1] - x[1] * fp[0]};
  const double c2[3] = {x[1] * c1[2] - x[2] * c1[1], x[2] * c1[0] - x[0] * c1[2], x[0] * c1[1] - x[1] * c1[0]};
  for (int k = 0; k < 3; ++k) b[3 * node + k] = b[3 * node + k] - dtp * (c1[k] + alpha * c2[k]);
}

}  // namespace

int64_t next_pow2(int64_t v) {
  int64_t p = 1;
  while (p < v) p <<= 1;
  return p;
}

FieldDims field_dims(int nx, int ny, int nz) {
  FieldDims f;
  f.nx = nx;
  f.ny = ny;
  f.nz = nz;
  f.px = next_pow2(2 * (int64_t)nx - 1);
  f.py = next_pow2(2 * (int64_t)ny - 1);
  f.pz = nz > 1 ? next_pow2(2 * (int64_t)nz - 1) : 1;
  return f;
}

void init_field_attributes() {}

// Gauss-Legendre nodes x_i and weights on [-1, 1] by Newton's method on the
// Legendre polynomial (three-term recurrence), mapped to [0, 1] with the
// weight (1 - s) folded into the weights.
GlRule folded_rule() {
  GlRule q;
  const int n = GL_NODES;
  for (int i = 0; i < n; ++i) {
    double x = cos(M_PI * (i + 0.75) / (n + 0.5)), dp = 1.0;
    for (int it = 0; it < 100; ++it) {
      double p0 = 1.0, p1 = x;
      for (int k = 2; k <= n; ++k) {
        const double p2 = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      dp = n * (x * p1 - p0) / (x * x - 1.0);
      const double dx = p1 / dp;
      x -= dx;
      if (fabs(dx) < 1e-17) break;
    }
    double p0 = 1.0, p1 = x;
    for (int k = 2; k <= n; ++k) {
      const double p2 = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k;
      p0 = p1;
      p1 = p2;
    }
    dp = n * (x * p1 - p0) / (x * x - 1.0);
    const double w = 2.0 / ((1.0 - x * x) * dp * dp);
    const double t = 0.5 * (x + 1.0);
    q.t[i] = t;
    q.w[i] = 0.5 * w * (1.0 - t);
  }
  return q;
}

// The octant table T[6][N] (N = nx ny nz doubles each) of the tensor.
void launch_demag_table(hipStream_t st, FieldDims f, double* T) {
  const int64_t N = f.nx * f.ny * f.nz;
  hipLaunchKernelGGL(k_demag_octant, dim3(nblk(N)), dim3(TPB), 0, st, f, T);
  const int64_t mx = std::min<int64_t>(f.nx, DEMAG_FAR + 1), my = std::min<int64_t>(f.ny, DEMAG_FAR + 1),
                mz = std::min<int64_t>(f.nz, DEMAG_FAR + 1);
  hipLaunchKernelGGL(k_demag_mid, dim3((unsigned)(mx * my * mz)), dim3(MID_TPB), 0, st, f, folded_rule(), T);
}

// Components c0 (real part) and c1 (imaginary part) on the padded grid.
void launch_demag_pair(hipStream_t st, FieldDims f, int c0, int c1, const double* T, double2* out) {
  const int64_t P = f.px * f.py * f.pz;
  hipLaunchKernelGGL(k_demag_pair, dim3(nblk(P)), dim3(TPB), 0, st, f, c0, c1, T, out);
}

// The octant table goes to the second work plane (16 P bytes >= 48 N: every
// padded length is at least twice the grid's), the packed pairs to the first.
void launch_demag_setup(hipStream_t st, FieldDims f, double2* work, double* nhat) {
  const int64_t P = f.px * f.py * f.pz;
  double* T = (double*)(work + P);
  hipLaunchKernelGGL(k_fft_unit, dim3((1 << FFT_MAX_BITS) / TPB), dim3(TPB), 0, st);
  launch_demag_table(st, f, T);
  const int pairs[3][2] = {{0, 1}, {2, 3}, {4, 5}};
  for (int r = 0; r < 3; ++r) {
    launch_demag_pair(st, f, pairs[r][0], pairs[r][1], T, work);
    fft_forward_full(st, f, work, 1);
    hipLaunchKernelGGL(k_take_pair, dim3(nblk(P)), dim3(TPB), 0, st, P, pairs[r][0], pairs[r][1], work, nhat);
  }
}

// ------------------------------------------------------------ no-allocation stray field
// The stray field of a device field without a context: the transformed tensor
// (6 P doubles) and the two work planes (4 P doubles) live in one static
// device array, so the call allocates nothing.  Each device holds its own
// copy of the array; its address is looked up once per device.  The array
// keeps the last call's contents: the transformed tensor is reused when the
// grid dimensions repeat.  Calls that overlap on one device race.
constexpr size_t NOALLOC_BYTES = LLG_STRAY_NOALLOC_MAX_BYTES;
static __device__ __align__(256) char scratch[NOALLOC_BYTES];

namespace {
constexpr int NOALLOC_MAX_DEV = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[NOALLOC_MAX_DEV] = {};
int64_t g_noalloc_dims[NOALLOC_MAX_DEV][3] = {};
}  // namespace

size_t stray_noalloc_bytes(FieldDims f) { return (size_t)(f.px * f.py * f.pz) * 10 * sizeof(double); }

hipError_t stray_noalloc(FieldDims f, const double* m, double* h, hipStream_t st) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= NOALLOC_MAX_DEV) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_noalloc_mu);
  if (!g_noalloc_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_noalloc_ptr[dev] = p;
  }
  const int64_t P = f.px * f.py * f.pz;
  double* nhat = (double*)g_noalloc_ptr[dev];
  double2* work = (double2*)(nhat + 6 * P);
  const bool same = g_noalloc_dims[dev][0] == f.nx && g_noalloc_dims[dev][1] == f.ny && g_noalloc_dims[dev][2] == f.nz;
  if (!same) {
    g_noalloc_dims[dev][0] = 0;  // invalid until the new tensor is in place
    launch_demag_setup(st, f, work, nhat);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  launch_stray(st, f, m, nullptr, nhat, work, h);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(st);
  if (e != hipSuccess) return e;
  g_noalloc_dims[dev][0] = f.nx;
  g_noalloc_dims[dev][1] = f.ny;
  g_noalloc_dims[dev][2] = f.nz;
  return hipSuccess;
}

namespace {
template <int BITS>
void launch_field_rows(hipStream_t st, const FieldRows& f, const double* m, const double* mprev, double2* w,
                       double scale, double* h) {
  auto go = [&](auto nt) {
    constexpr int NT = decltype(nt)::value, C = FftShape<BITS, NT>::C;
    const dim3 g((unsigned)(C > 1 ? ceil_div(f.rows, C / 2) : f.rows), C > 1 ? 1 : 2);
    if (NT > 128 && fft_narrow<BITS>() && g.x * g.y < FFT_FEW) return false;
    if (h)
      hipLaunchKernelGGL((k_fft_field_out<BITS, NT>), g, dim3(NT), 0, st, f, w, scale, h);
    else
      hipLaunchKernelGGL((k_fft_field_in<BITS, NT>), g, dim3(NT), 0, st, f, m, mprev, w);
    return true;
  };
  if (go(std::integral_constant<int, 512>{})) return;
  if constexpr (fft_narrow<BITS>()) go(std::integral_constant<int, 128>{});
}
template <int BITS, bool FLAT>
void launch_fft_demag(hipStream_t st, const FusedPass& p, double2* w, const double* nhat) {
  constexpr int L = 1 << BITS, T = FftShape<BITS, 512>::T, NT = T <= 128 ? 128 : 512;
  const int64_t lines = p.px / 2 * p.py, groups = ceil_div(lines, FftShape<BITS, NT>::C);
  if constexpr (T <= 64) {
    const int64_t few = ceil_div(lines, FftShape<BITS, 64>::C);
    if (few < DEMAG_FEW) {
      hipLaunchKernelGGL((k_fft_demag3<BITS, 64, FLAT>), dim3((unsigned)few), dim3(192), 0, st, w, nhat, p);
      return;
    }
  }
  if (T > 128 && groups < FFT_FEW) {
    const int64_t all = p.px * p.py, real = FLAT ? p.px / 2 + 1 : all;
    fft_axis(st, w, p.plane, 2, L, p.s, all, real, 1, 1, 0, p.n, L, -1, 1.0);
    hipLaunchKernelGGL((k_demag_pairs<FLAT>), dim3(nblk(lines * L)), dim3(TPB), 0, st, w, nhat, p, L);
    fft_axis(st, w, p.plane, 2, L, p.s, all, real, 1, 1, 0, L, p.n, +1, 1.0);
    return;
  }
  hipLaunchKernelGGL((k_fft_demag<BITS, NT, FLAT>), dim3((unsigned)groups), dim3(NT), 0, st, w, nhat, p);
}

// f(integral_constant<ilog2 L>): every axis of a padded grid has 4 cells or more
template <typename F>
void for_bits(int64_t L, F f) {
  switch (ilog2(L)) {
#define X(B) \
  case B: return f(std::integral_constant<int, B>{});
    X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12)
#undef X
    default: throw LLG_ERR_UNSUPPORTED;  // lengths are checked when the context is created
  }
}
}  // namespace

// h = -N * m~ (m, or 2 m - mprev), [N][3]: the transforms along x read the
// field and write h, the last axis is taken there and back in one kernel, and
// in 3D the y passes stand between.
void launch_stray(hipStream_t st, FieldDims f, const double* m, const double* mprev, const double* nhat,
                  double2* work, double* h) {
  const int64_t P = f.px * f.py * f.pz, pxy = f.px * f.py;
  const bool flat = f.pz == 1;
  const FieldRows rows{f.nx, f.ny * f.nz, f.px, f.py, f.ny, P};
  const FusedPass fused{f.px, flat ? 1 : f.py, flat ? f.px : pxy, P, (int)(flat ? f.ny : f.nz), ilog2(f.px) - 1};
  auto x_pass = [&](double* out) {
    for_bits(f.px, [&](auto b) { launch_field_rows<b.value>(st, rows, m, mprev, work, 1.0 / (double)P, out); });
  };
  x_pass(nullptr);
  if (!flat) fft_axis(st, work, P, 2, f.py, f.px, f.px, f.px / 2 + 1, 1, f.nz, pxy, f.ny, f.py, -1, 1.0);
  if (flat)
    for_bits(f.py, [&](auto b) { launch_fft_demag<b.value, true>(st, fused, work, nhat); });
  else
    for_bits(f.pz, [&](auto b) { launch_fft_demag<b.value, false>(st, fused, work, nhat); });
  if (!flat) fft_axis(st, work, P, 2, f.py, f.px, f.px, f.px / 2 + 1, 1, f.nz, pxy, f.py, f.ny, +1, 1.0);
  x_pass(h);
}

// Room for h in the work planes: past the box in the second plane, which
// the last x pass does not read (half a plane and more, 8 P >= 32 N bytes).
double* stray_room(FieldDims f, double2* work) {
  const int64_t P = f.px * f.py * f.pz;
  return (double*)(work + P + (f.pz > 1 ? f.px * f.py * f.nz : f.px * f.ny));
}

void launch_field_rhs(hipStream_t st, int64_t N, const double* prm, const double* m, const double* mprev,
                      const double* h, double* b) {
  hipLaunchKernelGGL(k_field_rhs, dim3(nblk(N)), dim3(TPB), 0, st, N, prm, m, mprev, h, b);
}

}  // namespace llg
