// Adaptive orbit integration (Sec. 2.2.2: Bogacki-Shampine 3(2) with a fixed
// number of accepted steps) and time-weighted binning (Sec. 2.2.4: the sample
// after accepted step k weighs dt_k / t_total), in FP64.
//
// Two kernels:
//  1. k_bs23: one orbit per lane of an integrating wave, in double or in single precision (the
//     single-precision force is the leapfrog integrator's: the bar's 16-node
//     rule, hardware reciprocals); the total time is summed and the Jacobi
//     drift evaluated in double either way.  Equations of motion in the bar frame for
//     (x, p), p the inertial velocity on the rotating axes:
//       dx/dt = p + Omega (y, -x, 0),  dp/dt = -grad Phi + Omega (p_y, -p_x, 0).
//     Per attempt: stages k2 = f(y + h/2 k1), k3 = f(y + 3h/4 k2), the third-order
//     solution y3 = y + h (2/9 k1 + 1/3 k2 + 4/9 k3), k4 = f(y3) (reused as the
//     next k1), the embedded second-order y2 = y + h (7/24 k1 + 1/4 k2 + 1/3 k3
//     + 1/8 k4); err = max_i |y3_i - y2_i| / (atol + rtol max(|y_i|, |y3_i|)),
//     accepted when err <= 1, next step h min(5, max(0.2, 0.9 err^(-1/3))); 100
//     rejections in a row end the step (length 0) with the non-finite flag.
//     Every accepted step appends its mirror copies' packed cells (as the
//     leapfrog path does) and its step to the orbit's streams.
//     Bound by the serial chain of an attempt (three forces, the error norm, a
//     power): 30,000 orbits are 469 waves for 1,024 SIMDs.  So (a) every lane
//     takes its own attempts, whether or not its neighbours' were accepted (a
//     wave that repeats a step until all 64 lanes accept takes more attempts than
//     any of them), and (b) what does not feed the next
//     attempt is done by three other waves of the workgroup, one binning and two
//     evaluating the Jacobi drift (half of the orbits each, two steps of an orbit
//     at a time), from states handed over in LDS, kRound attempts at a time.  Each lane's arithmetic is the same as in one wave.
//     30,000 x 5,000 steps of the barred model in FP32: 107.5 ms in one wave with
//     common steps, 44.9 now (54.9 with one drift wave, 46.7 without a raised
//     priority for the integrating waves).
//     Launches of many more tiles than the CUs hold of these workgroups take one
//     wave per tile (k_bs23_one; shares_tile has the rule and its figures).
//  2. k_hist_w: one workgroup per orbit (and window of columns when a row does
//     not fit LDS): each event's weight dt_k / t_total is rounded to a 64-bit
//     fixed-point integer in units of 2^-52 and added into an LDS histogram of
//     integers, written as sum / (copies 2^52) (divided by Upsilon for the
//     surface block).  Integer adds are exact, so the result does not depend on
//     the order in which the lanes add (repeated runs are identical to the bit);
//     the rounding moves each weight by at most 2^-53, under 1e-12 of an entry
//     over 5,000 steps.  The three blocks of a row are one histogram, so a row of
//     up to 20,000 columns (10,000 of few steps) reads its events once: 30,000 rows of 19,541 columns
//     took 6.2 ms in five passes, 4.0 now.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "common.h"
#include "potential.h"

namespace sw {
extern int g_num_cus;

namespace {

constexpr int kBsWindow = 20000;  // histogram columns per pass (160,000 bytes of LDS)
constexpr int kBsFewSteps = 64, kBsFewWindow = 10000;  // and for orbits of few steps, whose events cost little to read again
constexpr int kRound = 8;          // attempts between two hand-overs
constexpr int kBsThreads = 256;    // the integrating, the binning and two drift waves

template <bool NB>
__device__ __forceinline__ void bs_rhs(const PotK& P, const double* y, double* f) {
#pragma clang fp contract(off)
  double g[3];
  accel_f64<NB>(P, y, g);
  const double W = P.omega;
  f[0] = y[3] + W * y[1];
  f[1] = y[4] - W * y[0];
  f[2] = y[5];
  f[3] = g[0] + W * y[4];
  f[4] = g[1] - W * y[3];
  f[5] = g[2];
}

// single precision: the bar's 16-node rule with hardware reciprocals, lam warm
// started from the previous evaluation (as the leapfrog integrator does)
template <bool NB>
__device__ __forceinline__ void bs_rhs(const PotK& P, const float* y, float* f, float& lamw) {
  float g[3], gb[3];
  accel_f32<1, NB, false>(P, y[0], y[1], y[2], g[0], g[1], g[2], gb, lamw, 0);
  const float W = (float)P.omega;
  f[0] = y[3] + W * y[1];
  f[1] = y[4] - W * y[0];
  f[2] = y[5];
  f[3] = (g[0] + gb[0]) + W * y[4];
  f[4] = (g[1] + gb[1]) - W * y[3];
  f[5] = g[2] + gb[2];
}

template <bool NB>
__device__ __forceinline__ void bs_rhs(const PotK& P, const double* y, double* f, float&) {
  bs_rhs<NB>(P, y, f);
}

template <bool NB>
__device__ __forceinline__ double bs_jacobi(const PotK& P, const double* y, float) {
  return jacobi_f64<NB>(P, y);
}

template <bool NB>
__device__ __forceinline__ double bs_jacobi(const PotK& P, const float* y, float lamw) {
  double yd[6];
  for (int i = 0; i < 6; ++i) yd[i] = (double)y[i];
  return jacobi_f64_drift<NB, false>(P, yd, lamw);
}

__device__ __forceinline__ double bs_pow(double e) { return pow(e, -1.0 / 3.0); }
__device__ __forceinline__ float bs_pow(float e) { return powf(e, -1.0f / 3.0f); }

// One attempt at a step of length h: true when it is accepted (y and k1 then
// are the new state's); hh is the length it tried, h that of the next one.
template <bool NB, typename T>
__device__ __forceinline__ bool bs_attempt(const PotK& P, T* y, T* k1, T& h, float& lamw, T rt, T at, T& hh) {
#pragma clang fp contract(off)
  hh = h;
  T t[6], k2[6], k3[6], y3[6], k4[6];
  for (int i = 0; i < 6; ++i) t[i] = y[i] + (T)0.5 * hh * k1[i];
  bs_rhs<NB>(P, t, k2, lamw);
  for (int i = 0; i < 6; ++i) t[i] = y[i] + (T)0.75 * hh * k2[i];
  bs_rhs<NB>(P, t, k3, lamw);
  for (int i = 0; i < 6; ++i)
    y3[i] = y[i] + hh * ((T)(2.0 / 9.0) * k1[i] + (T)(1.0 / 3.0) * k2[i] + (T)(4.0 / 9.0) * k3[i]);
  bs_rhs<NB>(P, y3, k4, lamw);
  T err = (T)0;
  for (int i = 0; i < 6; ++i) {
    const T y2 = y[i] + hh * ((T)(7.0 / 24.0) * k1[i] + (T)0.25 * k2[i] + (T)(1.0 / 3.0) * k3[i] + (T)0.125 * k4[i]);
    const T sc = at + rt * fmax(fabs(y[i]), fabs(y3[i]));
    err = fmax(err, fabs(y3[i] - y2) / sc);
  }
  T fac = err > (T)0 ? (T)0.9 * bs_pow(err) : (T)5;
  fac = fmin((T)5, fmax((T)0.2, fac));
  h = hh * fac;
  const bool ok = err <= (T)1;
  if (ok) {
    for (int i = 0; i < 6; ++i) {
      y[i] = y3[i];
      k1[i] = k4[i];
    }
  }
  return ok;
}

// accepted steps handed from the integrating wave to the others
template <typename T>
struct BsRound {
  T y[kRound][6][64];
  T dt[kRound][64];
  float lamw[kRound][64];
  int32_t n[64];  // accepted steps of each lane in the round
};

// T: the arithmetic of the state, the stages and the step control (the total
// time is summed in double, the Jacobi drift evaluated in double)
template <typename T, bool NB, bool CYL>
__global__ __launch_bounds__(kBsThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 && CYL ? 2 : 1))) void k_bs23(PotK P, ObsK O, const double* __restrict__ ics,
                                                      const double* __restrict__ h0, int64_t n, int32_t S,
                                                      double rtol, double atol, uint64_t* __restrict__ ev_m,
                                                      uint64_t* __restrict__ ev_k, double* __restrict__ wts,
                                                      double* __restrict__ ttot, double* __restrict__ drift,
                                                      uint8_t* __restrict__ flags) {
#pragma clang fp contract(off)
  __shared__ BsRound<T> rounds[2];
  __shared__ float lam0[64];
  __shared__ int32_t badl[64];
  __shared__ int32_t last;  // the round after which every lane has its S steps (-1: not yet)
  const int lane = threadIdx.x & 63, role = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // this lane's orbit; a drift wave's lanes l and l + 32 share one
  const int ol = role < 2 ? lane : 32 * (role - 2) + (lane & 31);
  const int64_t o = (int64_t)blockIdx.x * 64 + ol;
  const bool mine = o < n;
  const int64_t oi = mine ? o : n - 1;  // lanes past the end repeat the last orbit and write nothing
  T y[6], k1[6];
  for (int i = 0; i < 6; ++i) y[i] = (T)ics[(int64_t)i * n + oi];
  const T rt = (T)rtol, at = (T)atol;
  T h = (T)h0[oi];
  float lamw = -1.0f;
  int s = 0, tries = 0;  // steps taken (each role counts its own), rejections in a row
  double tt = 0.0, dmax = 0.0, E0 = 0.0;
  bool bad = false;
  if (role == 0) {
    __builtin_amdgcn_s_setprio(3);  // ahead of the other roles' waves on its SIMD
    bs_rhs<NB>(P, y, k1, lamw);
    lam0[lane] = lamw;
    if (lane == 0) last = -1;
  }
  __syncthreads();
  if (role >= 2) E0 = bs_jacobi<NB>(P, y, lam0[ol]);
  for (int round = 0;; ++round) {
    if (role == 0) {
      BsRound<T>& R = rounds[round & 1];
      int got = 0;
      if (last < 0) {
        for (int a = 0; a < kRound; ++a) {
          if (s >= S) continue;
          T hh;
          const bool ok = bs_attempt<NB>(P, y, k1, h, lamw, rt, at, hh);
          ++tries;
          if (ok || tries == 100) {  // a step: accepted, or of length 0 after 100 rejections
            for (int i = 0; i < 6; ++i) R.y[got][i][lane] = y[i];
            R.dt[got][lane] = ok ? hh : (T)0;
            R.lamw[got][lane] = lamw;
            ++got;
            ++s;
            tries = 0;
          }
        }
        if (__ballot(s < S) == 0 && lane == 0) last = round;
      }
      R.n[lane] = got;
    } else if (round > 0 && role == 1) {
      const BsRound<T>& R = rounds[(round - 1) & 1];
      const int got = R.n[lane];
      for (int a = 0; a < kRound; ++a) {
        if (a >= got) continue;
        for (int i = 0; i < 6; ++i) y[i] = R.y[a][i][lane];
        const T dt = R.dt[a][lane];
        if (dt == (T)0) bad = true;
        for (int i = 0; i < 6; ++i)
          if (!isfinite(y[i])) bad = true;
        tt += (double)dt;
        uint32_t mc[4], kc[4];
        cells4<T, CYL>(P, O, y, mc, kc);
        if (mine) {
          const int64_t e = o * S + s;
          ev_m[e] = pack4(mc);
          ev_k[e] = pack4(kc);
          wts[e] = (double)dt;
        }
        ++s;
      }
    } else if (round > 0 && O.drift_every > 0) {
      const BsRound<T>& R = rounds[(round - 1) & 1];
      const int got = R.n[ol];
      for (int a0 = 0; a0 < kRound; a0 += 2) {
        const int a = a0 + (lane >> 5);  // lanes below 32 take the earlier step of the two
        double d = 0.0;
        const bool on = a < got && (s + a + 1) % O.drift_every == 0;
        if (on) {
          for (int i = 0; i < 6; ++i) y[i] = R.y[a][i][ol];
          d = fabs(bs_jacobi<NB>(P, y, R.lamw[a][ol]) / E0 - 1.0);
        }
        // both lanes keep the maximum, in the order of the steps (a NaN ends a
        // maximum, so the order counts)
        const double de = __shfl(d, lane & 31, 64), dl = __shfl(d, (lane & 31) + 32, 64);
        const bool oe = __shfl((int)on, lane & 31, 64) != 0, ol2 = __shfl((int)on, (lane & 31) + 32, 64) != 0;
        if (oe && !(de <= dmax)) dmax = de;
        if (ol2 && !(dl <= dmax)) dmax = dl;
      }
      s += got;
    }
    __syncthreads();
    // the rounds end with the one in which the last steps were binned.  `last` is set
    // once, before a barrier; a wave that reads it late, in the next round, may see
    // that round's number, which is not below its own
    const int l = last;
    if (l >= 0 && round > l) break;
  }
  if (role == 1) badl[lane] = bad ? 1 : 0;
  __syncthreads();
  if (!mine) return;
  if (role == 1) ttot[o] = tt;
  if (role >= 2 && lane < 32) {
    drift[o] = dmax;
    flags[o] = (uint8_t)((!(dmax <= 0.1) ? SW_FLAG_DRIFT : 0) | (badl[ol] ? SW_FLAG_NONFINITE : 0));
  }
}

// The same in one wave per 64 orbits, without LDS, for the launches whose
// four-wave workgroups would queue (shares_tile): the orbits of a wave take their
// steps together, an attempt being repeated until every lane has accepted.  Bound
// by the issue of the attempts, two waves per SIMD (about 250 registers in FP64).
template <typename T, bool NB, bool CYL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 1))) void k_bs23_one(PotK P, ObsK O, const double* __restrict__ ics,
                                                 const double* __restrict__ h0, int64_t n, int32_t S, double rtol,
                                                 double atol, uint64_t* __restrict__ ev_m, uint64_t* __restrict__ ev_k,
                                                 double* __restrict__ wts, double* __restrict__ ttot,
                                                 double* __restrict__ drift, uint8_t* __restrict__ flags) {
#pragma clang fp contract(off)
  const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= n) return;
  T y[6], k1[6];
  for (int i = 0; i < 6; ++i) y[i] = (T)ics[(int64_t)i * n + o];
  const T rt = (T)rtol, at = (T)atol;
  T h = (T)h0[o];
  double tt = 0.0, dmax = 0.0;
  float lamw = -1.0f;
  bool bad = false;
  bs_rhs<NB>(P, y, k1, lamw);
  const double E0 = bs_jacobi<NB>(P, y, lamw);
  for (int s = 0; s < S; ++s) {
    T dt = (T)0;
    for (int tries = 0; tries < 100; ++tries) {
      T hh;
      if (bs_attempt<NB>(P, y, k1, h, lamw, rt, at, hh)) {
        dt = hh;
        break;
      }
    }
    if (dt == (T)0) bad = true;
    for (int i = 0; i < 6; ++i)
      if (!isfinite(y[i])) bad = true;
    tt += (double)dt;
    uint32_t mc[4], kc[4];
    cells4<T, CYL>(P, O, y, mc, kc);
    const int64_t e = o * S + s;
    ev_m[e] = pack4(mc);
    ev_k[e] = pack4(kc);
    wts[e] = (double)dt;
    if (O.drift_every > 0 && (s + 1) % O.drift_every == 0) {
      const double d = fabs(bs_jacobi<NB>(P, y, lamw) / E0 - 1.0);
      if (!(d <= dmax)) dmax = d;
    }
  }
  ttot[o] = tt;
  drift[o] = dmax;
  flags[o] = (uint8_t)((!(dmax <= 0.1) ? SW_FLAG_DRIFT : 0) | (bad ? SW_FLAG_NONFINITE : 0));
}

// Columns [win0, win0 + wn) of a row; the blocks' first columns are 0, n_mass and
// n_mass + n_kin (nv > 0: surface block, kinematic codes ap nv + v_bin and
// n_kin + ap count in its column ap).  The window 0 also writes the overflow.
template <int NT>
__global__ __launch_bounds__(NT) void k_hist_w(const uint64_t* __restrict__ ev_m, const uint64_t* __restrict__ ev_k,
                                               const double* __restrict__ wts, const double* __restrict__ ttot,
                                               int32_t S, int32_t ncopy, int32_t n_mass, int32_t n_kin, int32_t nv,
                                               int32_t win0, int32_t wn, int64_t n_con, double* __restrict__ A,
                                               double* __restrict__ overflow, double div) {
  extern __shared__ unsigned long long hq[];
  __shared__ unsigned long long ovq[2];
  const int64_t o = blockIdx.x;
  const int tid = threadIdx.x;
  for (int c = tid; c < wn; c += NT) hq[c] = 0ull;
  if (tid < 2) ovq[tid] = 0ull;
  __syncthreads();
  const double inv_t = 1.0 / ttot[o];
  const uint32_t nm = (uint32_t)n_mass, nk = (uint32_t)n_kin, w0 = (uint32_t)win0, w1 = (uint32_t)(win0 + wn);
  const auto add = [&](uint32_t col, unsigned long long q) {
    if (col >= w0 && col < w1) atomicAdd(&hq[col - w0], q);
  };
  constexpr int U = 4;  // steps in flight
  for (int s0 = tid; s0 < S; s0 += U * NT) {
    uint64_t vm[U], vk[U];
    double wt[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t e = o * S + (s0 + u * NT < S ? s0 + u * NT : s0);
      vm[u] = ev_m[e];
      vk[u] = ev_k[e];
      wt[u] = wts[e];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u * NT >= S) break;
      const unsigned long long q = (unsigned long long)llrint(wt[u] * inv_t * 0x1p52);
      for (int c = 0; c < ncopy; ++c) {
        const uint32_t im = (uint32_t)(vm[u] >> (16 * c)) & 0xFFFFu, ik = (uint32_t)(vk[u] >> (16 * c)) & 0xFFFFu;
        if (im < nm) add(im, q);
        else if (win0 == 0) atomicAdd(&ovq[0], q);
        if (ik < nk) add(nm + ik, q);
        else if (win0 == 0) atomicAdd(&ovq[1], q);
        if (nv > 0 && ik != 0xFFFFu) add(nm + nk + (ik < nk ? ik / (uint32_t)nv : ik - nk), q);
      }
    }
  }
  __syncthreads();
  const double scale = 0x1p-52 / (double)ncopy;
  double* row = A + o * n_con + win0;
  for (int c = tid; c < wn; c += NT) {
    const double v = (double)hq[c] * scale;
    row[c] = (uint32_t)(win0 + c) >= nm + nk ? v / div : v;
  }
  if (tid < 2 && win0 == 0) overflow[o * 2 + tid] = (double)ovq[tid] * scale;
}

// Whether four waves share a tile.  Where the CUs hold all of these workgroups
// (three a CU in single precision, two in double and with needle bars) they do.
// Of more, some wait, while one wave per tile leaves a wave its SIMD up to four
// tiles per CU and two waves share one up to eight; the tiles of a workgroup are
// spread over the SIMDs.  40 steps of the barred model in FP64, four waves and one:
// 32,700 orbits 2.7 and 5.0 ms, 65,500 5.2 and 5.1, 131,000 10.2 and 8.5; 70,000 x
// 32 steps of three discs 0.71 and 0.61.  In single precision a second round of
// workgroups pays from some 32 steps on, and a third where the drift is evaluated
// at each step (the wave that the drift is taken from has the more to do): the
// barred model, 70,000 orbits x 300 steps 5.6 and 7.9 ms, 140,000 with each step's
// drift 9.8 and 12.5; three discs, 200,000 x 68 1.66 and 1.25.  With needle bars a
// second and a third round pay with each step's drift only: 44,000 orbits x 32
// steps 4.1 and 4.8 ms, with that of every tenth step 3.6 and 3.0.
bool shares_tile(int64_t tiles, int32_t n_steps, bool f64, bool needle, int32_t drift_every) {
  const int64_t cus = g_num_cus;
  const bool each = drift_every == 1;
  if (f64) return tiles <= 2 * cus;
  if (needle) return tiles <= 2 * cus || (each && ((tiles <= 4 * cus && n_steps >= 16) || (tiles <= 6 * cus && n_steps >= 32)));
  return tiles <= 3 * cus || (tiles <= (each ? 9 : 6) * cus && n_steps >= 32);
}

size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

// Threads by the workgroups that a row's LDS leaves per CU: one or two take 1,024,
// two to five 512, more 256 (fewer where a launch would reach 2^32 threads).
// Calls of 100,000 orbits x 8 steps: rows of 5,198 columns 0.97 to 1.09 ms with 256
// threads, 0.93 with 512; rows of 13,964 columns leave one workgroup per CU, in two
// windows two: 2.70 and 2.42 ms.
int hist_w(const uint64_t* ev_m, const uint64_t* ev_k, const double* wts, const double* ttot, int64_t n, int32_t S,
           const ObsK& O, int64_t n_con, double* A, double* overflow, double upsilon, hipStream_t st) {
  const int32_t nv = O.surface ? O.nv : 0;
  const int64_t win = S <= kBsFewSteps ? kBsFewWindow : kBsWindow;
  for (int64_t w0 = 0; w0 < n_con; w0 += win) {
    const int32_t wn = (int32_t)(n_con - w0 < win ? n_con - w0 : win);
    const size_t lds = (size_t)wn * 8;
    const auto go = [&](auto kernel, int nt) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(nt), lds, st, ev_m, ev_k, wts, ttot, S, O.ncopy, O.n_mass,
                         O.n_kin, nv, (int32_t)w0, wn, n_con, A, overflow, upsilon);
    };
    if (lds > 64 * 1024 && n < (int64_t)1 << 22) go(k_hist_w<1024>, 1024);
    else if (lds > 32 * 1024 && n < (int64_t)1 << 23) go(k_hist_w<512>, 512);
    else go(k_hist_w<256>, 256);
    SW_HIP(hipGetLastError());
  }
  return SW_OK;
}

}  // namespace
}  // namespace sw

using namespace sw;

extern "C" size_t integrate_bs23_workspace_bytes(int64_t n_orb, int32_t n_steps) {
  if (n_orb < 0 || n_steps < 1) return 0;
  const size_t per = (size_t)n_orb * (size_t)n_steps * 8;
  return 3 * al256(per) + al256((size_t)n_orb * 8);
}

extern "C" int integrate_bs23_and_bin(const sw_potential* pot, const double* ics, const double* h0, int64_t n_orb,
                                      int32_t n_steps, double rtol, double atol, int32_t precision,
                                      const sw_obs_spec* obs, double* A, double* overflow, double* drift,
                                      uint8_t* flags, void* workspace, size_t ws_bytes, void* stream) {
  SW_CHECK(pot && obs, "integrate_bs23_and_bin: null argument");
  SW_CHECK(precision == SW_F32 || precision == SW_F64, "integrate_bs23_and_bin: precision must be SW_F32 or SW_F64");
  SW_CHECK(n_orb >= 0 && n_orb <= 0x7fffffffLL && n_steps >= 1,
           "integrate_bs23_and_bin: need n_orb >= 0 and n_steps >= 1");
  SW_CHECK(std::isfinite(rtol) && rtol > 0.0 && std::isfinite(atol) && atol > 0.0,
           "integrate_bs23_and_bin: tolerances must be finite and > 0");
  ObsK O;
  SW_CHECK(obs_to_k(obs, &O), "integrate_bs23_and_bin: invalid observable specification");
  if (n_orb == 0) return SW_OK;
  SW_CHECK(ics && h0 && A && overflow && drift && flags && workspace, "integrate_bs23_and_bin: null device buffer");
  SW_CHECK(ws_bytes >= integrate_bs23_workspace_bytes(n_orb, n_steps), "integrate_bs23_and_bin: workspace too small");
  PotK P;
  std::memcpy(&P, pot, sizeof P);
  bool nb = false;
  for (int c = 0; c < P.n_comp; ++c) nb = nb || P.comp[c].kind == SW_DA_T3 || P.comp[c].kind == SW_DA_V4;
  const size_t per = al256((size_t)n_orb * (size_t)n_steps * 8);
  char* ws = (char*)workspace;
  uint64_t* ev_m = (uint64_t*)ws;
  uint64_t* ev_k = (uint64_t*)(ws + per);
  double* wts = (double*)(ws + 2 * per);
  double* ttot = (double*)(ws + 3 * per);
  hipStream_t st = (hipStream_t)stream;
  const auto launch = [&](auto t, auto needle, auto cyl) {
    typedef decltype(t) T;
    constexpr bool NB = decltype(needle)::value, CYL = decltype(cyl)::value;
    const int64_t tiles = (n_orb + 63) / 64;
    const auto go = [&](auto kernel, int64_t groups, int nt) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(nt), 0, st, P, O, ics, h0, n_orb, n_steps, rtol, atol,
                         ev_m, ev_k, wts, ttot, drift, flags);
    };
    if (shares_tile(tiles, n_steps, sizeof(T) == 8, NB, O.drift_every)) {
      go(k_bs23<T, NB, CYL>, tiles, kBsThreads);
    } else {
      const int64_t nw = std::min<int64_t>(4, (tiles + g_num_cus - 1) / g_num_cus);
      go(k_bs23_one<T, NB, CYL>, (tiles + nw - 1) / nw, (int)nw * 64);
    }
  };
  const auto with_bars = [&](auto t, auto cyl) {
    if (nb) launch(t, std::true_type{}, cyl);
    else launch(t, std::false_type{}, cyl);
  };
  const auto with_grid = [&](auto t) {
    if (O.cyl) with_bars(t, std::true_type{});
    else with_bars(t, std::false_type{});
  };
  if (precision == SW_F32) with_grid(float{});
  else with_grid(double{});
  SW_HIP(hipGetLastError());
  const int64_t n_con = (int64_t)O.n_mass + O.n_kin + (O.surface ? O.n_ap : 0);
  return hist_w(ev_m, ev_k, wts, ttot, n_orb, n_steps, O, n_con, A, overflow, obs->upsilon, st);
}
