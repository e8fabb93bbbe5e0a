// Initial conditions of the orbit library (Sec. 2.2.1): velocities from the
// anisotropic Jeans equations, dithered realisations, and the bundle means of
// the orbit matrix.
//
// jeans_ics: at each starting position, the velocity dispersions and the
// mean rotation of a tracer with the fiducial density
// nu(R, z) ~ exp(-R/h_R - |z|/h_z) in the azimuth-averaged potential, then one
// Gaussian draw per velocity component.
//
// With the velocity ellipsoid aligned with (R, phi, z), sigma_R^2 = b sigma_z^2,
// sigma_phi = sigma_R and F the azimuth-averaged force:
//   sigma_z^2(R, z) = h_z int_0^inf e^-s (-F_z(R, |z| + h_z s)) ds   (vertical equation)
//   <v_phi^2> = b [sigma_z^2 (1 - R/h_R) + R d sigma_z^2/dR] - R F_R(R, z)   (radial equation)
//   mean v_phi = sqrt(max(<v_phi^2> - sigma_phi^2, 0)).
// The ln-nu gradients of the exponential tracer are constants, so only the
// force enters the integrals.  d/dR is the Richardson combination of central
// differences with steps h and h/2, h = 2e-3 max(R, h_z).
//
// One workgroup per position.  The s-integral uses 13 panels with edges 0 and
// 2^-6 .. 2^6 (fine near s = 0, where a thin disc's force turns over), each with
// an 8-point Gauss-Legendre rule; the azimuth average is the 128-point
// trapezoid rule (periodic integrand).  Every component is symmetric under
// x -> -x and y -> -y, so the 128 azimuths hold 33 distinct ones (weight 2 on
// the axes, 4 between them), and the axisymmetric components take one
// evaluation per (s, radius).  The lanes own (s, phi) node pairs of the bars
// and evaluate them at the five radii; the workgroup adds the partial sums by
// a fixed tree.
//
// Bound by FP64 vector issue in the bar's 32 quadrature nodes.  Each node takes
// one reciprocal square root refined to FP64 (its three divisions follow from
// the square of it) instead of an IEEE square root and seven divisions, and
// the confocal coordinate lam of a radius starts from its neighbour's.
// 7,500 positions of the barred model: 60.1 ms with 128 azimuths of the whole
// potential and IEEE divisions, 4.0 ms now.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "common.h"
#include "potential.h"

namespace sw {
namespace {

constexpr int kJnThreads = 256;
// Up to this many positions (one workgroup per CU at most) a position takes
// 1,024 threads: with 256 each SIMD would hold one wave and wait out its latencies
// (250 positions of the barred model: 210 us with 256 threads, 173 with 1,024; 400:
// 329 and 311; 700: 456 and 459; 7,500: 4.00 ms and 4.43).
constexpr int kJnWide = 256;
constexpr int kJnQ = 8;
constexpr int kJnPanels = 13;
constexpr int kJnS = kJnQ * kJnPanels;
constexpr int kJnPhi = 128;
constexpr int kJnQuad = kJnPhi / 4 + 1;  // distinct azimuths, 0 .. pi/2
constexpr int kJnSums = 6;  // sigma_z^2 integrals at R - h, R - h/2, R, R + h/2, R + h; F_R at (R, z)

struct JeansK {
  double hR, hz, b;
  double gt[kJnQ], gw[kJnQ];  // Gauss-Legendre rule on [-1, 1]
  int32_t n_all;              // components; the axisymmetric ones come first (P.n_comp of them)
};

__device__ __forceinline__ double panel_edge(int k) { return k == 0 ? 0.0 : ldexp(1.0, k - 7); }

// node j of the s-integral and its weight (e^-s included)
__device__ __forceinline__ double s_node(const JeansK& K, int j, double& ws) {
  const int pj = j / kJnQ, q = j % kJnQ;
  const double e0 = panel_edge(pj), e1 = panel_edge(pj + 1);
  const double half = 0.5 * (e1 - e0), s = 0.5 * (e0 + e1) + half * K.gt[q];
  ws = half * K.gw[q] * exp(-s);
  return s;
}

// reciprocal and reciprocal square root in FP64: the hardware estimate (about
// 2^-23) and one third-order step, which leaves about 2^-65
__device__ __forceinline__ double rcp3(double v) {
  const double r = __builtin_amdgcn_rcp(v), e = fma(-v, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ double rsq3(double v) {
  const double r = __builtin_amdgcn_rsq(v), e = fma(-v * r, r, 1.0);
  return fma(r * e, fma(0.375, e, 0.5), r);
}

// Force of a Ferrers bar (ALL: g[0..2], else g[2] alone is formed) by the
// 32-node rule of ferrers_f64.  lam < 0: Newton from the left bracket; else from
// that value: m^2(lam) is convex and decreasing, so a step from the right of the
// root lands left of it and the next ones rise.  A step below 1e-9 of
// A_min + lam is the last (the error after it is of the order of its square).
template <bool ALL>
__device__ __forceinline__ void ferrers_bar(const CompK& C, const double* gq, const double* gw, double x, double y,
                                            double z, double& lam, double* g) {
  const double A0 = C.c[0], A1 = C.c[1], A2 = C.c[2];
  const double x2 = x * x, y2 = y * y, z2 = z * z;
  bool right = lam > 0.0;  // the start may lie right of the root
  if (!(lam >= 0.0)) lam = fmax(0.0, x2 + y2 + z2 - C.c[6]);
  for (int it = 0; it < 60; ++it) {
    const double i0 = rcp3(A0 + lam), i1 = rcp3(A1 + lam), i2 = rcp3(A2 + lam);
    const double t0 = x2 * i0, t1 = y2 * i1, t2 = z2 * i2;
    const double f = t0 + t1 + t2 - 1.0;
    if (!(f > 0.0) && !right) break;
    const double d = f * rcp3(t0 * i0 + t1 * i1 + t2 * i2), nl = fmax(0.0, lam + d);
    const bool last = !(fabs(nl - lam) > 1e-9 * (C.c[3] + lam));
    right = false;
    lam = nl;
    if (last) break;
  }
  const double K = C.c[3] + lam, iK = rcp3(K);
  const double D0 = (A0 + lam) * iK, D1 = (A1 + lam) * iK, D2 = (A2 + lam) * iK;
  const double xs = x2 * iK, ys = y2 * iK, zs = z2 * iK;
  double F0 = 0.0, F1 = 0.0, F2 = 0.0;
#pragma unroll 4
  for (int n = 0; n < kGL64; ++n) {
    const double q = gq[n], W = gw[n];
    const double e0 = D0 + q, e1 = D1 + q, e2 = D2 + q;
    const double e12 = e1 * e2, e02 = e0 * e2, e01 = e0 * e1;
    const double s = rsq3(e0 * e12), iP = s * s;
    const double w = fmax(fma(-iP, xs * e12 + ys * e02 + zs * e01, 1.0), 0.0);
    const double c = (W * s) * (w * w) * iP;
    if (ALL) {
      F0 = fma(c, e12, F0);
      F1 = fma(c, e02, F1);
    }
    F2 = fma(c, e01, F2);
  }
  const double sc = C.c[4] * iK * rsq3(K);
  if (ALL) {
    g[0] -= sc * x * F0;
    g[1] -= sc * y * F1;
  }
  g[2] -= sc * z * F2;
}

// force of the components that are not axisymmetric, added into g
template <bool NB, bool ALL>
__device__ __forceinline__ void bars_accel(const PotK& P, int n_all, double x, double y, double z, double& lam,
                                           double* g) {
  for (int i = P.n_comp; i < n_all; ++i) {
    const CompK& C = P.comp[i];
    if (C.kind == SW_FERRERS2) {
      double l = i == P.n_comp ? lam : -1.0;  // the first bar's lam carries over from radius to radius
      ferrers_bar<ALL>(C, P.gq64, P.gw64, x, y, z, l, g);
      if (i == P.n_comp) lam = l;
    } else if constexpr (NB) {
      if (C.kind == SW_DA_T3) needle_bar<double, 3, kGL64>(C.c, P.gq64, P.gw64, x, y, z, nullptr, g);
      else needle_bar<double, 5, kGL64>(C.c, P.gq64, P.gw64, x, y, z, nullptr, g);
    }
  }
}

template <bool NB, int THREADS>
__global__ __launch_bounds__(THREADS) void k_jeans(PotK P, JeansK K, const double* __restrict__ pos,
                                                       const double* __restrict__ eps, int64_t n,
                                                       double* __restrict__ mom, double* __restrict__ ics) {
  __shared__ double red[kJnSums][THREADS];
  const int64_t i = blockIdx.x;
  const int tid = threadIdx.x;
  const double x = pos[i], y = pos[n + i], z = pos[2 * n + i];
  const double R = sqrt(x * x + y * y), az = fabs(z);
  const double h = 2e-3 * fmax(R, K.hz);
  const double radii[5] = {R - h, R - 0.5 * h, R, R + 0.5 * h, R + h};
  double acc[kJnSums];
#pragma unroll
  for (int r = 0; r < kJnSums; ++r) acc[r] = 0.0;
  // the axisymmetric components: one evaluation stands for the 128 azimuths
  if (P.n_comp > 0) {
    for (int p = tid; p < 5 * kJnS; p += THREADS) {
      const int r = p / kJnS;
      double ws, g[3];
      const double s = s_node(K, p - r * kJnS, ws);
      const double rad = r == 0 ? radii[0] : r == 1 ? radii[1] : r == 2 ? radii[2] : r == 3 ? radii[3] : radii[4];
      const double xv[3] = {rad, 0.0, az + K.hz * s};
      accel_f64<false>(P, xv, g);
#pragma unroll
      for (int q = 0; q < 5; ++q) acc[q] += q == r ? kJnPhi * (ws * -g[2]) : 0.0;
    }
    if (tid == THREADS - 1) {
      double g[3];
      const double xv[3] = {R, 0.0, z};
      accel_f64<false>(P, xv, g);
      acc[5] += kJnPhi * g[0];
    }
  }
  // the bars: (s, azimuth) pairs, then the azimuths of F_R at the position itself
  for (int p = tid; K.n_all > P.n_comp && p < (kJnS + 1) * kJnQuad; p += THREADS) {
    const int j = p / kJnQuad, k = p - j * kJnQuad;
    double sp, cp;
    sincospi((double)k * (2.0 / kJnPhi), &sp, &cp);
    const double wk = k == 0 || k == kJnQuad - 1 ? 2.0 : 4.0;
    double lam = -1.0;
    if (j < kJnS) {
      double ws;
      const double s = s_node(K, j, ws);
      const double zz = az + K.hz * s;
      ws *= wk;
#pragma unroll
      for (int r = 0; r < 5; ++r) {
        double g[3] = {0.0, 0.0, 0.0};
        bars_accel<NB, false>(P, K.n_all, radii[r] * cp, radii[r] * sp, zz, lam, g);
        acc[r] += ws * -g[2];
      }
    } else {
      double g[3] = {0.0, 0.0, 0.0};
      bars_accel<NB, true>(P, K.n_all, R * cp, R * sp, z, lam, g);
      acc[5] += wk * (g[0] * cp + g[1] * sp);
    }
  }
#pragma unroll
  for (int r = 0; r < kJnSums; ++r) red[r][tid] = acc[r];
  __syncthreads();
  for (int st = THREADS / 2; st > 0; st >>= 1) {
    if (tid < st) {
#pragma unroll
      for (int r = 0; r < kJnSums; ++r) red[r][tid] += red[r][tid + st];
    }
    __syncthreads();
  }
  if (tid == 0) {
    double sig[5];
#pragma unroll
    for (int r = 0; r < 5; ++r) sig[r] = K.hz * red[r][0] / kJnPhi;
    const double FR = red[5][0] / kJnPhi;
    const double d1 = (sig[4] - sig[0]) / (2.0 * h), d2 = (sig[3] - sig[1]) / h;
    const double dsig = (4.0 * d2 - d1) / 3.0;
    const double s0 = sig[2], b = K.b;
    const double vphi2 = b * (s0 * (1.0 - R / K.hR) + R * dsig) - R * FR;
    const double sz = sqrt(fmax(s0, 0.0)), sR = sqrt(b) * sz;
    const double mean = sqrt(fmax(vphi2 - b * s0, 0.0));
    mom[i] = sR;
    mom[n + i] = sR;
    mom[2 * n + i] = sz;
    mom[3 * n + i] = mean;
    mom[4 * n + i] = sqrt(fmax(-R * FR, 0.0));
    const double ph = atan2(y, x), c = cos(ph), sn = sin(ph);
    const double vR = sR * eps[i], vp = mean + sR * eps[n + i], vz = sz * eps[2 * n + i];
    ics[i] = x;
    ics[n + i] = y;
    ics[2 * n + i] = z;
    ics[3 * n + i] = vR * c - vp * sn;
    ics[4 * n + i] = vR * sn + vp * c;
    ics[5 * n + i] = vz;
  }
}

// realisation k of initial condition i -> column i nd + k: each coordinate
// moved by its deviate times dx (positions) or fv v_c (velocities); products
// and sums rounded separately
__global__ void k_dither(const double* __restrict__ ics, const double* __restrict__ vc, const double* __restrict__ u,
                         int64_t n, int32_t nd, double dx, double fv, double* __restrict__ out) {
#pragma clang fp contract(off)
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, m = n * nd;
  if (j >= m) return;
  const int64_t i = j / nd, k = j % nd;
  for (int c = 0; c < 6; ++c) {
    const double scale = c < 3 ? dx : fv * vc[i];
    out[c * m + j] = ics[c * n + i] + u[(k * 6 + c) * n + i] * scale;
  }
}

// bundle row b = mean of rows b nd .. b nd + nd - 1, summed in row order in FP64
template <typename T>
__global__ void k_bundle(const T* __restrict__ A, int64_t nb, int64_t C, int32_t nd, T* __restrict__ out) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= nb * C) return;
  const int64_t b = idx / C, c = idx % C;
  const T* a = A + (b * nd) * C + c;
  double s = (double)a[0];
  for (int k = 1; k < nd; ++k) s = s + (double)a[(int64_t)k * C];
  out[idx] = (T)(s / nd);
}

// n-point Gauss-Legendre rule on [-1, 1] by Newton's iteration on P_n
void gl_rule(int n, double* t, double* w) {
  for (int i = 0; i < n; ++i) {
    double x = std::cos(M_PI * (i + 0.75) / (n + 0.5)), dp = 0.0;
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
      if (std::fabs(dx) < 1e-16) break;
    }
    t[i] = -x;
    w[i] = 2.0 / ((1.0 - x * x) * dp * dp);
  }
}

}  // namespace
}  // namespace sw

using namespace sw;

extern "C" int jeans_ics(const sw_potential* pot, const double* pos, const double* eps, int64_t n, double h_R,
                         double h_z, double b, double* moments, double* ics, void* stream) {
  SW_CHECK(pot, "jeans_ics: null potential");
  SW_CHECK(n >= 0 && n <= 0x7fffffff, "jeans_ics: n must be in [0, 2^31)");
  SW_CHECK(std::isfinite(h_R) && h_R > 0.0 && std::isfinite(h_z) && h_z > 0.0,
           "jeans_ics: tracer scale lengths must be finite and > 0");
  SW_CHECK(std::isfinite(b) && b > 0.0, "jeans_ics: b = sigma_R^2 / sigma_z^2 must be finite and > 0");
  if (n == 0) return SW_OK;
  SW_CHECK(pos && eps && moments && ics, "jeans_ics: null device buffer");
  PotK P;
  std::memcpy(&P, pot, sizeof P);
  SW_CHECK(P.n_comp >= 1 && P.n_comp <= SW_MAX_COMP, "jeans_ics: potential not built");
  bool nb = false;
  for (int c = 0; c < P.n_comp; ++c) nb = nb || P.comp[c].kind == SW_DA_T3 || P.comp[c].kind == SW_DA_V4;
  JeansK K;
  std::memset(&K, 0, sizeof K);
  K.hR = h_R;
  K.hz = h_z;
  K.b = b;
  K.n_all = P.n_comp;
  // axisymmetric components first
  const auto axisym = [](const CompK& c) {
    return c.kind != SW_FERRERS2 && c.kind != SW_DA_T3 && c.kind != SW_DA_V4;
  };
  P.n_comp = (int32_t)(std::stable_partition(P.comp, P.comp + K.n_all, axisym) - P.comp);
  gl_rule(kJnQ, K.gt, K.gw);
  hipStream_t st = (hipStream_t)stream;
  if (nb)
    hipLaunchKernelGGL((k_jeans<true, kJnThreads>), dim3((unsigned)n), dim3(kJnThreads), 0, st, P, K, pos, eps, n,
                       moments, ics);
  else if (n <= kJnWide)
    hipLaunchKernelGGL((k_jeans<false, 1024>), dim3((unsigned)n), dim3(1024), 0, st, P, K, pos, eps, n, moments, ics);
  else
    hipLaunchKernelGGL((k_jeans<false, kJnThreads>), dim3((unsigned)n), dim3(kJnThreads), 0, st, P, K, pos, eps, n,
                       moments, ics);
  SW_HIP(hipGetLastError());
  return SW_OK;
}

extern "C" int dither_ics(const double* ics, const double* vc, const double* u, int64_t n, int32_t n_dither, double dx,
                          double fv, double* out, void* stream) {
  SW_CHECK(n >= 0 && n_dither >= 1 && n_dither <= 64, "dither_ics: need n >= 0 and 1 <= n_dither <= 64");
  SW_CHECK(std::isfinite(dx) && dx >= 0.0 && std::isfinite(fv) && fv >= 0.0, "dither_ics: box sizes must be >= 0");
  if (n == 0) return SW_OK;
  SW_CHECK(ics && vc && u && out, "dither_ics: null device buffer");
  const int64_t m = n * n_dither;
  SW_CHECK((m + 255) / 256 <= 0x7fffffff, "dither_ics: too many realisations for one launch");
  hipLaunchKernelGGL(k_dither, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, (hipStream_t)stream, ics, vc, u, n,
                     n_dither, dx, fv, out);
  SW_HIP(hipGetLastError());
  return SW_OK;
}

extern "C" int bundle_rows(const void* A, int32_t dtype, int64_t n_bundle, int64_t n_con, int32_t n_dither, void* out,
                           void* stream) {
  SW_CHECK(dtype == SW_F32 || dtype == SW_F64, "bundle_rows: dtype must be SW_F32 or SW_F64");
  SW_CHECK(n_bundle >= 0 && n_con >= 0 && n_dither >= 1, "bundle_rows: need n_bundle, n_con >= 0, n_dither >= 1");
  const int64_t m = n_bundle * n_con;
  if (m == 0) return SW_OK;
  SW_CHECK(A && out && A != out, "bundle_rows: null or aliased device buffer");
  SW_CHECK((m + 255) / 256 <= 0x7fffffff, "bundle_rows: too many entries for one launch");
  const dim3 grid((unsigned)((m + 255) / 256));
  hipStream_t st = (hipStream_t)stream;
  if (dtype == SW_F32)
    hipLaunchKernelGGL(k_bundle<float>, grid, dim3(256), 0, st, (const float*)A, n_bundle, n_con, n_dither,
                       (float*)out);
  else
    hipLaunchKernelGGL(k_bundle<double>, grid, dim3(256), 0, st, (const double*)A, n_bundle, n_con, n_dither,
                       (double*)out);
  SW_HIP(hipGetLastError());
  return SW_OK;
}
