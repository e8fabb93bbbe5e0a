// Orbit integration kernel (Sec. 2.2.2-2.2.4), templated on the working
// precision.  One orbit per lane.  Each lane integrates its orbit with a
// kick-drift-kick leapfrog in the corotating bar frame, keeps the force of the
// last kick for the next step's first kick, bins the four mirror copies of
// every synchronised state and stages the packed cell indices of
// up to kStage steps in LDS.  The wave then writes each orbit's staged steps as
// one contiguous segment of that orbit's event stream (128 bytes where three
// waves share a tile, else 64), so that lanes that own different orbits store
// whole runs of bytes.  Bound by the serial chain of a step: up to
// one wave per SIMD, its latency; above, the issue of its ~1,300 instructions.
//
// Event word (uint64, one per orbit per step per block): four 16-bit cell
// indices, copy c in bits [16c, 16c+16), 0xFFFF = outside the block.
#pragma once
#include <algorithm>
#include <type_traits>

#include "potential.h"

namespace sw {

constexpr int kStage = 16;  // staged steps of a tile (half where the LDS of several tiles shares a workgroup)
constexpr int kWave = 64;
constexpr int kTileWaves = 4;  // tiles per workgroup of k_integrate, at most

// lamw: the single-precision path's warm-start state of the bar's lam (unused in double)
template <typename T>
struct Prec;
template <>
struct Prec<float> {
  // LPO lanes per orbit: each lane's share, then the sum over the lane group
  // (the same sum in every lane of the group, so their states stay identical)
  template <int LPO = 1, int NB = 0>
  __device__ static void accel(const PotK& P, const float* s, float* g, float& lamw, int part = 0) {
    float gb[3];
    accel_f32<LPO, NB != 0, true>(P, s[0], s[1], s[2], g[0], g[1], g[2], gb, lamw, part);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if constexpr (LPO == 2) gb[k] += __shfl_xor(gb[k], 1, 64);
      g[k] += gb[k];
    }
  }
  template <int NB = 0>
  __device__ static double jacobi(const PotK& P, const double* sd, float lamw) {
    return jacobi_f64_drift<NB != 0>(P, sd, lamw);
  }
};
template <>
struct Prec<double> {
  template <int LPO = 1, int NB = 0>
  __device__ static void accel(const PotK& P, const double* s, double* g, float&, int = 0) {
    static_assert(LPO == 1, "the double-precision path runs one lane per orbit");
    accel_f64<NB>(P, s, g);
  }
  template <int NB = 0>
  __device__ static double jacobi(const PotK& P, const double* sd, float) { return jacobi_f64<NB>(P, sd); }
};

// Where a kernel finds its potential: the launch's one potential (by value);
// one per tile (kPotTile: tiles do not straddle potentials, so that a tile's
// constants come by scalar loads); or one per orbit (kPotOrbit).
enum PotMode { kPotOne, kPotTile, kPotOrbit };

// Potential index of orbit o: the last k with offsets[k] <= o.
__device__ __forceinline__ int pot_index(const int64_t* offsets, int n_pot, int64_t o) {
  int lo = 0, hi = n_pot - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (offsets[mid] <= o) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Tiles of OPW orbits of the chunk [orb0, orb0 + n_chunk).  kPotTile: with a_k
// the chunk-local first orbit of potential k, potential k owns the tile numbers
// a_k / OPW + k .. a_(k+1) / OPW + k (rounded down), at least as many as its
// orbits fill; the n_chunk / OPW + n_pot tiles hold a few empty ones.
struct Tile {
  int kpot;
  int64_t j0;  // chunk-local index of the first orbit
  int cnt;     // orbits, 0 for an empty tile
};
template <int MODE, int OPW>
__device__ __forceinline__ Tile tile_at(int64_t t, const int64_t* offsets, int n_pot, int64_t orb0, int64_t n_chunk) {
  Tile r;
  int64_t end = n_chunk;
  if constexpr (MODE == kPotTile) {
    const auto first = [&](int k) {
      const int64_t a = offsets[k] - orb0;
      return a < 0 ? (int64_t)0 : (a > n_chunk ? n_chunk : a);
    };
    int lo = 0, hi = n_pot - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (first(mid) / OPW + mid <= t) lo = mid; else hi = mid - 1;
    }
    r.kpot = lo;
    end = first(lo + 1);
    r.j0 = first(lo) + (t - lo - first(lo) / OPW) * OPW;
  } else {
    r.kpot = 0;
    r.j0 = t * OPW;
  }
  const int64_t left = end - r.j0;
  r.cnt = left < 0 ? 0 : (left > OPW ? OPW : (int)left);
  return r;
}
template <int OPW>
__host__ __device__ inline int64_t tile_count(int mode, int n_pot, int64_t n_chunk) {
  return mode == kPotTile ? n_chunk / OPW + n_pot : (n_chunk + OPW - 1) / OPW;
}

// The potential of a tile, read as constant memory (scalar loads).
__device__ __forceinline__ const PotK& tile_pot(const sw_potential* pots, int k) {
  typedef const __attribute__((address_space(4))) PotK* cptr;
  return *(const PotK*)(cptr)(reinterpret_cast<const PotK*>(pots + __builtin_amdgcn_readfirstlane(k)));
}

// One orbit's leapfrog state.
template <typename T, int LPO, int NB>
struct Leap {
  T s[6], g[3], dt, h, c, sn, cm1;
  float lamw;
  int part;
  __device__ __forceinline__ void start(const PotK& P, const T* ics, T dt_, int64_t n_orb, int64_t o, int part_) {
#pragma unroll
    for (int i = 0; i < 6; ++i) s[i] = ics[(int64_t)i * n_orb + o];
    part = part_;
    dt = dt_;
    h = T(0.5) * dt;
    const double th = P.omega * (double)dt;
    // FP64 rotates with (cos, sin) exactly as the oracle does.  FP32 rotates with
    // (cos - 1, sin): cos rounded to binary32 would scale the radius by up to one
    // ulp of 1 per step, a systematic drift over 10^4 steps, whereas cos - 1 =
    // -2 sin^2(th/2) keeps its full relative precision.
    c = (T)cos(th);
    sn = (T)sin(th);
    cm1 = (T)(-2.0 * sin(0.5 * th) * sin(0.5 * th));
    lamw = -1.0f;
    Prec<T>::template accel<LPO, NB>(P, s, g, lamw, part);
  }
  __device__ __forceinline__ void step(const PotK& P) {
#pragma clang fp contract(off)
    constexpr bool F = sizeof(T) == 4;
    s[3] = mad_<F>(h, g[0], s[3]);
    s[4] = mad_<F>(h, g[1], s[4]);
    s[5] = mad_<F>(h, g[2], s[5]);
    s[0] = mad_<F>(dt, s[3], s[0]);
    s[1] = mad_<F>(dt, s[4], s[1]);
    s[2] = mad_<F>(dt, s[5], s[2]);
    if constexpr (sizeof(T) == 8) {
      T x = c * s[0] + sn * s[1];
      T y = c * s[1] - sn * s[0];
      T px = c * s[3] + sn * s[4];
      T py = c * s[4] - sn * s[3];
      s[0] = x; s[1] = y; s[3] = px; s[4] = py;
    } else {
      T x = s[0] + mad_<F>(cm1, s[0], sn * s[1]);
      T y = s[1] + mad_<F>(cm1, s[1], -(sn * s[0]));
      T px = s[3] + mad_<F>(cm1, s[3], sn * s[4]);
      T py = s[4] + mad_<F>(cm1, s[4], -(sn * s[3]));
      s[0] = x; s[1] = y; s[3] = px; s[4] = py;
    }
    Prec<T>::template accel<LPO, NB>(P, s, g, lamw, part);
    s[3] = mad_<F>(h, g[0], s[3]);
    s[4] = mad_<F>(h, g[1], s[4]);
    s[5] = mad_<F>(h, g[2], s[5]);
  }
};

template <typename T, int NB>
__device__ __forceinline__ double energy(const PotK& P, const T* s, float lamw) {
  double sd[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) sd[i] = (double)s[i];
  return Prec<T>::template jacobi<NB>(P, sd, lamw);
}

template <typename T>
__device__ __forceinline__ void write_checks(const T* s, double dmax, int64_t o, double* drift, uint8_t* flags) {
  bool nonfinite = false;
#pragma unroll
  for (int i = 0; i < 6; ++i) nonfinite |= !isfinite(s[i]);
  if (drift) drift[o] = dmax;
  if (flags) flags[o] = (uint8_t)((!(dmax <= 0.1) ? SW_FLAG_DRIFT : 0) | (nonfinite ? SW_FLAG_NONFINITE : 0));
}

// A wave writes the n staged steps (at most ST) from step0 on of its tile's orbits.
template <int ST, int OPW>
__device__ __forceinline__ void write_stage(const uint64_t (*stm)[OPW + 1], const uint64_t (*stk)[OPW + 1], int n,
                                            const Tile& tl, int64_t n_steps, int64_t step0, int lane, uint64_t* ev_m,
                                            uint64_t* ev_k) {
  if (n == ST) {
    const int ss = lane % ST;
    int64_t at = (tl.j0 + lane / ST) * n_steps + step0 + ss;
#pragma unroll 4
    for (int jj = lane / ST; jj < OPW; jj += kWave / ST, at += kWave / ST * n_steps) {
      if (jj < tl.cnt) {
        ev_m[at] = stm[ss][jj];
        ev_k[at] = stk[ss][jj];
      }
    }
  } else {
    for (int idx = lane; idx < n * tl.cnt; idx += kWave) {
      const int jj = idx / n, ss = idx - jj * n;
      const int64_t at = (tl.j0 + jj) * n_steps + step0 + ss;
      ev_m[at] = stm[ss][jj];
      ev_k[at] = stk[ss][jj];
    }
  }
}

// One wave does all of a tile's work; a workgroup carries up to kTileWaves tiles,
// which share nothing: the waves of a workgroup are spread over the SIMDs of its
// CU, while workgroups of one wave may meet on one SIMD with others idle (the
// barred model in FP64, 300 steps, 1,024 tiles: 8.3 ms in workgroups of one
// tile, 5.1 of four).  At most 168 registers, so that three waves share a SIMD (the default
// allocation lands one register above that, at two waves); with needle bars, where
// more are live, 14 to 41 of them go to scratch, most of them constants that a step
// reloads once.  In FP64 the cylindrical grid's binning and constants held per lane
// would spill up to 86: those forms take 184 to 256 registers and two waves a SIMD
// (FP64, 300 orbits of 100 potentials of the barred model x 400 steps on a
// cylindrical grid 7.7 ms with 168, 6.9 now, 7.5 before the branch-free binning;
// 400,000 orbits x 500 of a point mass there 8.4 and 7.4).  On that grid the form
// of three waves (THREE, 42 spilled) is left for the launches whose tiles all reside with it
// and not with two (133,000 such orbits 3.1 ms with three, 3.5 with two; with
// needle bars both take the same time).
//
// LPO lanes per orbit (1, or 2 in single precision): a wave carries 64 / LPO
// orbits; the lanes of a pair hold the same state, each evaluates its share of
// the force and the pair adds the shares, so both advance identically; the
// first lane of the pair writes the orbit's events and results.
template <typename T, int MODE, bool BIN, int LPO = 1, bool NB = false, bool CYL = false, bool THREE = false>
__global__ __launch_bounds__(kTileWaves* kWave)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 && BIN && ((CYL && !THREE) || MODE == kPotOrbit) ? 2 : 3)))
void k_integrate(const PotK p0, const sw_potential* __restrict__ pots, const int64_t* __restrict__ offsets,
                 int32_t n_pot, ObsK O, const T* __restrict__ ics, const T* __restrict__ dts, int64_t n_orb,
                 int64_t orb0, int64_t n_chunk, int32_t n_steps, uint64_t* __restrict__ ev_m,
                 uint64_t* __restrict__ ev_k, double* __restrict__ drift, uint8_t* __restrict__ flags,
                 T* __restrict__ final_state) {
  constexpr int OPW = kWave / LPO;  // orbits per wave
  constexpr int KB = NB && MODE == kPotOrbit ? 2 : NB;
  constexpr int ST = kStage / 2;
  __shared__ uint64_t staged[kTileWaves][2][ST][OPW + 1];
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int nw = blockDim.x / kWave;
  auto& stm = staged[wave][0];
  auto& stk = staged[wave][1];
  const int part = lane % LPO, lo = lane / LPO;  // share and orbit of this lane
  const int64_t n_tiles = tile_count<OPW>(MODE, n_pot, n_chunk);
  // persistent launch: each wave walks the orbit tiles at the stride of the grid's waves
  for (int64_t tile = (int64_t)blockIdx.x * nw + wave; tile < n_tiles; tile += (int64_t)gridDim.x * nw) {
    const Tile tl = tile_at<MODE, OPW>(tile, offsets, n_pot, orb0, n_chunk);
    if (tl.cnt == 0) continue;
    const bool valid = lo < tl.cnt;
    const int64_t o = orb0 + tl.j0 + (valid ? lo : tl.cnt - 1);
    const PotK& P = MODE == kPotOne    ? p0
                    : MODE == kPotTile ? tile_pot(pots, tl.kpot)
                                       : *reinterpret_cast<const PotK*>(pots + pot_index(offsets, n_pot, o));
    Leap<T, LPO, KB> L;
    L.start(P, ics, dts[o], n_orb, o, part);
    double E0 = 0.0, dmax = 0.0;
    if constexpr (BIN) E0 = energy<T, KB>(P, L.s, L.lamw);
    const int de = O.drift_every;
    int slot = 0;
    for (int k = 1; k <= n_steps; ++k) {
      L.step(P);
      if constexpr (BIN) {
        if (de > 0 && k % de == 0) {
          const double e = fabs(energy<T, KB>(P, L.s, L.lamw) / E0 - 1.0);
          if (!(e <= dmax)) dmax = e;
        }
        uint32_t mc[4], kc[4];
        cells4<T, CYL>(P, O, L.s, mc, kc);
        if (part == 0) {
          stm[slot][lo] = pack4(mc);
          stk[slot][lo] = pack4(kc);
        }
        ++slot;
        if (slot == ST || k == n_steps) {
          wave_fence();
          write_stage<ST, OPW>(stm, stk, slot, tl, n_steps, k - slot, lane, ev_m, ev_k);
          wave_fence();
          slot = 0;
        }
      }
    }
    if (valid && part == 0) {
      if constexpr (BIN) {
        write_checks<T>(L.s, dmax, o, drift, flags);
      } else {
#pragma unroll
        for (int i = 0; i < 6; ++i) final_state[(int64_t)i * n_orb + o] = L.s[i];
      }
    }
  }
}

// ROLES waves share a tile: the first one integrates, handing its states over
// in LDS kHand steps at a time; the second bins them and writes the events; the
// last (the second as well when there are two) evaluates the drift, in the order
// of the steps, since a NaN ends a maximum.  A step is a serial chain, and what
// does not feed the next force leaves it.
constexpr int kHand = 4;
template <typename T>
struct Handed {
  T s[kHand][6][kWave];
  float lamw[kHand][kWave];
};
template <typename T, int MODE, int ROLES, bool NB, bool CYL>
__global__ __launch_bounds__(ROLES* kWave) __attribute__((amdgpu_waves_per_eu(ROLES == 2 ? 4 : 2)))
void k_integrate_split(const PotK p0, const sw_potential* __restrict__ pots, const int64_t* __restrict__ offsets,
                       int32_t n_pot, ObsK O, const T* __restrict__ ics, const T* __restrict__ dts, int64_t n_orb,
                       int64_t orb0, int64_t n_chunk, int32_t n_steps, uint64_t* __restrict__ ev_m,
                       uint64_t* __restrict__ ev_k, double* __restrict__ drift, uint8_t* __restrict__ flags) {
  constexpr int ST = ROLES == 2 ? kStage / 2 : kStage;  // staged steps
  static_assert(ST % kHand == 0, "a stage is a number of whole hand-overs");
  __shared__ Handed<T> hand[2];
  __shared__ float lam0[kWave];
  __shared__ uint64_t stm[ST][kWave + 1];
  __shared__ uint64_t stk[ST][kWave + 1];
  const int lane = threadIdx.x % kWave, role = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const bool bins = role == 1, checks = role == ROLES - 1;
  const int64_t n_tiles = tile_count<kWave>(MODE, n_pot, n_chunk);
  const int n_rounds = (n_steps + kHand - 1) / kHand;
  const int de = O.drift_every;
  const int64_t tile = blockIdx.x;
  if (tile >= n_tiles) return;
  const Tile tl = tile_at<MODE, kWave>(tile, offsets, n_pot, orb0, n_chunk);
  if (tl.cnt == 0) return;  // the same for all waves
  const bool valid = lane < tl.cnt;
  const int64_t o = orb0 + tl.j0 + (valid ? lane : tl.cnt - 1);
  const PotK& P = MODE == kPotOne ? p0 : tile_pot(pots, tl.kpot);
  if (role == 0) {
    __builtin_amdgcn_s_setprio(3);  // ahead of the other roles' waves on its SIMD
    Leap<T, 1, NB> L;
    L.start(P, ics, dts[o], n_orb, o, 0);
    lam0[lane] = L.lamw;
    __syncthreads();
    for (int r = 0; r < n_rounds; ++r) {
      Handed<T>& H = hand[r & 1];
      const int n = n_steps - r * kHand < kHand ? n_steps - r * kHand : kHand;
      for (int a = 0; a < n; ++a) {
        L.step(P);
#pragma unroll
        for (int i = 0; i < 6; ++i) H.s[a][i][lane] = L.s[i];
        H.lamw[a][lane] = L.lamw;
      }
      __syncthreads();
    }
  } else {
    T s[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) s[i] = ics[(int64_t)i * n_orb + o];
    __syncthreads();
    const double E0 = checks ? energy<T, NB>(P, s, lam0[lane]) : 0.0;
    double dmax = 0.0;
    int slot = 0;
    for (int r = 0; r < n_rounds; ++r) {
      __syncthreads();  // round r is handed over; round r + 1 goes to the other buffer
      const Handed<T>& H = hand[r & 1];
      const int n = n_steps - r * kHand < kHand ? n_steps - r * kHand : kHand;
      for (int a = 0; a < n; ++a) {
        const int k = r * kHand + a + 1;
#pragma unroll
        for (int i = 0; i < 6; ++i) s[i] = H.s[a][i][lane];
        if (checks && de > 0 && k % de == 0) {
          const double e = fabs(energy<T, NB>(P, s, H.lamw[a][lane]) / E0 - 1.0);
          if (!(e <= dmax)) dmax = e;
        }
        if (bins) {
          uint32_t mc[4], kc[4];
          cells4<T, CYL>(P, O, s, mc, kc);
          stm[slot][lane] = pack4(mc);
          stk[slot][lane] = pack4(kc);
          ++slot;
        }
      }
      if (slot == ST || (bins && r == n_rounds - 1)) {
        wave_fence();  // this wave alone stages and reads back
        write_stage<ST, kWave>(stm, stk, slot, tl, n_steps, r * kHand + n - slot, lane, ev_m, ev_k);
        wave_fence();
        slot = 0;
      }
    }
    if (checks && valid) write_checks<T>(s, dmax, o, drift, flags);
  }
}

// the integration kernels take the potential and the observables by value
static_assert(sizeof(PotK) + sizeof(ObsK) + 256 <= 4096, "kernel arguments exceed 4 KiB");

struct IntegrateLaunch {
  PotK p0;                     // the potential when n_pot == 1
  const sw_potential* pots_dev;  // device copies when n_pot > 1
  const int64_t* offsets_dev;
  int32_t n_pot;
  ObsK obs;
  const void* ics;
  const void* dt;
  int64_t n_orb, orb0, n_chunk;
  int32_t n_steps;
  uint64_t* ev_m;
  uint64_t* ev_k;
  double* drift;
  uint8_t* flags;
  void* final_state;
  bool bin;
  bool needle;  // some potential holds a needle bar: the kernels built with its code
};

// Process-wide launch knobs (set through sw_set_tuning):
//  g_waves_per_cu  0: a tile of 64 orbits to one wave (one to four such tiles per workgroup) or to a workgroup of
//                  two or three waves (below); k > 0: persistent grid of k waves per CU, one wave per tile
//  g_hist_lds_kb   LDS budget of one histogram workgroup (orbits per workgroup follow)
extern int g_waves_per_cu;
extern int g_hist_lds_kb;
extern int g_lanes_per_orbit;  // 1 or 2 lanes per orbit (single precision with binning)
extern int g_num_cus;

// Waves per tile.  Three up to two tiles per CU: 2,000 FP64 orbits x 1,000 steps
// with the drift checked at each took 2.0 ms with one wave, 1.4 with two, 0.84
// with three; 8,000 FP32 orbits of the barred model x 2,000 steps 5.3, 3.6, 3.6.
// Above, two in single precision: 65,536 such orbits 10.0 -> 8.2 ms, 100,000 11.8
// -> 10.8 (three: 8.3, 13.7), up to the seven tiles that a CU's LDS takes at once;
// of more, some wait for a whole tile's steps (119,637 FP32 orbits x 300 steps:
// 1.82 ms with two waves and 1.37 with one of two Plummer spheres on a cylindrical
// grid, 1.61 and 1.35 of the barred model).  In double precision a
// wave fills its SIMD, and integrating waves that share one lose more than the
// others give (the barred model, 768 tiles x 300 steps: 5.2 ms with one wave, 7.1
// with two); needle bars need more registers than two waves per tile leave.
constexpr int kSplit3TilesPerCu = 2, kSplit2TilesPerCu = 7;

template <typename T, bool NB, bool CYL>
void launch_integrate_v(const IntegrateLaunch& L, hipStream_t st) {
  // potentials with needle bars, and cylindrical grids, run one lane per orbit
  const bool pair = sizeof(T) == 4 && L.bin && g_lanes_per_orbit == 2 && !NB && !CYL;
  const int64_t full = (L.n_chunk + (pair ? 32 : 64) - 1) / (pair ? 32 : 64);
  // Tiles cut at the potentials' bounds pay when they stay few: n_pot <= full / 4
  // adds at most a quarter to their number, and scalar constants leave their
  // waves free to share tiles (64 potentials of 2,000 FP32 orbits x 1,000 steps:
  // 10.9 ms lane by lane, 10.6 with scalar constants in one wave, 8.7 in two).
  int mode = L.n_pot == 1 ? kPotOne : (4 * (int64_t)L.n_pot <= full ? kPotTile : kPotOrbit);
  int64_t tiles = pair ? tile_count<32>(mode, L.n_pot, L.n_chunk) : tile_count<64>(mode, L.n_pot, L.n_chunk);
  int roles = 1;
  if (L.bin && !pair && mode != kPotOrbit && g_waves_per_cu == 0) {
    if (tiles <= (int64_t)kSplit3TilesPerCu * g_num_cus) roles = 3;
    else if (sizeof(T) == 4 && !NB && tiles <= (int64_t)kSplit2TilesPerCu * g_num_cus) roles = 2;
  }
  // One wave per tile: not where the cut tiles take one wave more per SIMD than
  // the uncut ones (60 steps of the barred model in FP64, 65,000 orbits of 30
  // potentials, 1,016 tiles or 1,046: 1.61 ms cut, 1.18 lane by lane; 120,000 of
  // 100, 1,875 or 1,975 of 2,048: 1.79 and 1.85).  Pairs of lanes stay cut (32,000
  // FP32 orbits of 30 potentials: 0.25 ms, 0.27 lane by lane).
  const int64_t simds = (int64_t)kTileWaves * g_num_cus;
  if (mode == kPotTile && roles == 1 && !pair && (tiles + simds - 1) / simds != (full + simds - 1) / simds) {
    mode = kPotOrbit;
    tiles = full;
  }
  if (g_waves_per_cu > 0) {
    const int64_t cap = (int64_t)g_waves_per_cu * g_num_cus;
    if (tiles > cap) tiles = cap;
  }
  // one-wave tiles per workgroup: as few as leave one workgroup per CU
  const int nw = (int)std::min<int64_t>(kTileWaves, (tiles + g_num_cus - 1) / g_num_cus);
  const dim3 grid((unsigned)tiles), grid1((unsigned)((tiles + nw - 1) / nw));
  const T* ics = (const T*)L.ics;
  const T* dt = (const T*)L.dt;
  const auto one = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid1, dim3(nw * kWave), 0, st, L.p0, L.pots_dev, L.offsets_dev, L.n_pot, L.obs, ics, dt,
                       L.n_orb, L.orb0, L.n_chunk, L.n_steps, L.ev_m, L.ev_k, L.drift, L.flags, (T*)L.final_state);
  };
  const auto split = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(roles * kWave), 0, st, L.p0, L.pots_dev, L.offsets_dev, L.n_pot, L.obs, ics, dt,
                       L.n_orb, L.orb0, L.n_chunk, L.n_steps, L.ev_m, L.ev_k, L.drift, L.flags);
  };
  if (!L.bin) {
    if constexpr (!CYL) one(k_integrate<T, kPotOne, false, 1, NB>);
    return;
  }
  if constexpr (sizeof(T) == 4 && !NB && !CYL) {
    if (pair) {
      if (mode == kPotOne) one(k_integrate<T, kPotOne, true, 2>);
      else if (mode == kPotTile) one(k_integrate<T, kPotTile, true, 2>);
      else one(k_integrate<T, kPotOrbit, true, 2>);
      return;
    }
  }
  const auto split_or_one = [&](auto m) {
    constexpr int M = decltype(m)::value;
    if (roles == 3) {
      split(k_integrate_split<T, M, 3, NB, CYL>);
      return;
    }
    if constexpr (sizeof(T) == 4 && !NB) {
      if (roles == 2) {
        split(k_integrate_split<T, M, 2, NB, CYL>);
        return;
      }
    }
    if constexpr (sizeof(T) == 8 && CYL && !NB) {
      if (tiles > 2 * simds && tiles <= 3 * simds) {
        one(k_integrate<T, M, true, 1, NB, CYL, true>);
        return;
      }
    }
    one(k_integrate<T, M, true, 1, NB, CYL>);
  };
  if (mode == kPotOne) {
    split_or_one(std::integral_constant<int, kPotOne>{});
  } else if (mode == kPotTile) {
    split_or_one(std::integral_constant<int, kPotTile>{});
  } else {
    one(k_integrate<T, kPotOrbit, true, 1, NB, CYL>);
  }
}

template <typename T>
hipError_t launch_integrate_t(const IntegrateLaunch& L, hipStream_t st) {
  // needle bars and the cylindrical grid are compiled in only where they occur
  if (L.bin && L.obs.cyl) {
    if (L.needle) launch_integrate_v<T, true, true>(L, st);
    else launch_integrate_v<T, false, true>(L, st);
  } else {
    if (L.needle) launch_integrate_v<T, true, false>(L, st);
    else launch_integrate_v<T, false, false>(L, st);
  }
  return hipGetLastError();
}

hipError_t launch_integrate_f32(const IntegrateLaunch& L, hipStream_t st);
hipError_t launch_integrate_f64(const IntegrateLaunch& L, hipStream_t st);

}  // namespace sw
