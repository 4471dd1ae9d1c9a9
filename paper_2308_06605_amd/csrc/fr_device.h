// fr_device.h -- device-side building blocks shared by the FP64 and FP32 kernels of libfr:
// the physical and numerical fluxes of the compressible Navier-Stokes equations (the paper's
// section "FR Algorithm", Eq. (1) and the interface Riemann solver), the launch configuration
// per polynomial degree and the 1-D operator tables passed to the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "fr_internal.h"

using namespace frk;

// ------------------------------------------------------------------------------------------
// Device physics (Eq. (1)): inviscid flux, viscous flux with constant mu, Riemann solvers.
// ------------------------------------------------------------------------------------------
template <typename real>
struct Phys {
  real gamma, gm1, mu, kappa;
};

// a.b in one order of rounding. Written as a sum of products, which product is fused with the
// additions depends on the code around it, and kernels that share an expression (the volume
// kernel with and without the next stage's pre-pass) could then differ in the last place.
template <typename real>
__device__ __forceinline__ real dot3(real a0, real b0, real a1, real b1, real a2, real b2) {
  return fma(a2, b2, fma(a0, b0, a1 * b1));
}

// Inviscid flux along a unit or scaled direction n: F(U).n, plus u.n and c.
template <typename real>
__device__ __forceinline__ void flux_n(const real U[5], const real n[3], const Phys<real> &ph, real F[5],
                                       real &un, real &c) {
  const real ir = real(1) / U[0];
  const real u = U[1] * ir, v = U[2] * ir, w = U[3] * ir;
  const real p = ph.gm1 * (U[4] - real(0.5) * U[0] * dot3(u, u, v, v, w, w));
  un = dot3(u, n[0], v, n[1], w, n[2]);
  F[0] = U[0] * un;
  F[1] = U[1] * un + p * n[0];
  F[2] = U[2] * un + p * n[1];
  F[3] = U[3] * un + p * n[2];
  F[4] = (U[4] + p) * un;
  c = sqrt(ph.gamma * p * ir);
}

template <typename real>
__device__ __forceinline__ void rusanov(const real UL[5], const real UR[5], const real n[3], const Phys<real> &ph,
                                        real F[5]) {
  real FL[5], FR[5], unL, unR, cL, cR;
  flux_n(UL, n, ph, FL, unL, cL);
  flux_n(UR, n, ph, FR, unR, cR);
  const real lam = fmax(fabs(unL) + cL, fabs(unR) + cR);
#pragma unroll
  for (int v = 0; v < 5; ++v) F[v] = real(0.5) * (FL[v] + FR[v]) - real(0.5) * lam * (UR[v] - UL[v]);
}

// Roe: mean flux minus half of sum |lambda_k| alpha_k r_k; sqrt(rho) averages; no entropy fix.
template <typename real>
__device__ __forceinline__ void roe(const real UL[5], const real UR[5], const real n[3], const Phys<real> &ph,
                                    real F[5]) {
  real FL[5], FR[5], t0, t1;
  flux_n(UL, n, ph, FL, t0, t1);
  flux_n(UR, n, ph, FR, t0, t1);
  const real rL = UL[0], rR = UR[0];
  const real iL = real(1) / rL, iR = real(1) / rR;
  const real uL[3] = {UL[1] * iL, UL[2] * iL, UL[3] * iL};
  const real uR[3] = {UR[1] * iR, UR[2] * iR, UR[3] * iR};
  const real pL = ph.gm1 * (UL[4] - real(0.5) * rL * (uL[0] * uL[0] + uL[1] * uL[1] + uL[2] * uL[2]));
  const real pR = ph.gm1 * (UR[4] - real(0.5) * rR * (uR[0] * uR[0] + uR[1] * uR[1] + uR[2] * uR[2]));
  const real HL = (UL[4] + pL) * iL, HR = (UR[4] + pR) * iR;
  const real sL = sqrt(rL), sR = sqrt(rR);
  const real is = real(1) / (sL + sR);
  const real rt = sL * sR;
  real ut[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) ut[i] = (sL * uL[i] + sR * uR[i]) * is;
  const real Ht = (sL * HL + sR * HR) * is;
  const real q2 = ut[0] * ut[0] + ut[1] * ut[1] + ut[2] * ut[2];
  const real c2 = ph.gm1 * (Ht - real(0.5) * q2);
  const real ct = sqrt(c2);
  const real ic2 = real(1) / c2;
  const real unt = ut[0] * n[0] + ut[1] * n[1] + ut[2] * n[2];
  const real dr = rR - rL, dp = pR - pL;
  const real du[3] = {uR[0] - uL[0], uR[1] - uL[1], uR[2] - uL[2]};
  const real dun = du[0] * n[0] + du[1] * n[1] + du[2] * n[2];
  const real a1 = real(0.5) * (dp - rt * ct * dun) * ic2;
  const real a5 = real(0.5) * (dp + rt * ct * dun) * ic2;
  const real a2 = dr - dp * ic2;
  const real l1 = fabs(unt - ct), l2 = fabs(unt), l5 = fabs(unt + ct);
  const real w1 = l1 * a1, w5 = l5 * a5, w2 = l2 * a2;
  real dis[5];
  dis[0] = w1 + w5 + w2;
  real udu = 0;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const real sh = du[i] - dun * n[i];
    dis[1 + i] = w1 * (ut[i] - ct * n[i]) + w5 * (ut[i] + ct * n[i]) + w2 * ut[i] + l2 * rt * sh;
    udu += ut[i] * sh;
  }
  dis[4] = w1 * (Ht - unt * ct) + w5 * (Ht + unt * ct) + w2 * real(0.5) * q2 + l2 * rt * udu;
#pragma unroll
  for (int v = 0; v < 5; ++v) F[v] = real(0.5) * (FL[v] + FR[v]) - real(0.5) * dis[v];
}

// Viscous flux Fv[i][v] from U and the gradient of the conserved variables G[i][v], with
// dynamic viscosity mu and heat-flux coefficient kappa (on d(p/rho)).
template <typename real>
__device__ __forceinline__ void visc_flux_mk(const real U[5], const real G[3][5], real gm1, real mu, real kappa,
                                             real Fv[3][5]) {
  const real ir = real(1) / U[0];
  const real u[3] = {U[1] * ir, U[2] * ir, U[3] * ir};
  const real e = U[4] * ir;
  real du[3][3], dT[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll
    for (int j = 0; j < 3; ++j) du[i][j] = (G[i][1 + j] - u[j] * G[i][0]) * ir;
    const real de = (G[i][4] - e * G[i][0]) * ir;
    dT[i] = gm1 * (de - dot3(u[0], du[i][0], u[1], du[i][1], u[2], du[i][2]));
  }
  const real lam = real(-2.0 / 3.0) * mu * (du[0][0] + du[1][1] + du[2][2]);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    real tau[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) tau[j] = mu * (du[j][i] + du[i][j]) + (i == j ? lam : real(0));
    Fv[i][0] = 0;
    Fv[i][1] = tau[0];
    Fv[i][2] = tau[1];
    Fv[i][3] = tau[2];
    Fv[i][4] = tau[0] * u[0] + tau[1] * u[1] + tau[2] * u[2] + kappa * dT[i];
  }
}

template <typename real>
__device__ __forceinline__ void visc_flux(const real U[5], const real G[3][5], const Phys<real> &ph, real Fv[3][5]) {
  visc_flux_mk(U, G, ph.gm1, ph.mu, ph.kappa, Fv);
}

// ------------------------------------------------------------------------------------------
// Memory accesses by reuse
// ------------------------------------------------------------------------------------------
// Loads of data that a kernel reads once in all: the face buffers and face geometry in the face
// kernels (each entry belongs to one face), the RK register in the volume kernels (also stored that
// way). Non-temporal, they leave the caches to what is read again: the metric terms, which the fused
// pre-pass reloads, and the face results, which both neighbours read. Only where a wave's runs of
// RUN values are whole 128-byte lines or halves: shorter or ragged runs share lines with their
// neighbours, and a line dropped after its first use is fetched again. Two LSRK45 steps (us): 40^3
// p=3 FP64 6515 -> 6342 with the face values and gradients, -> 6306 with the face geometry, -> 6256
// with the register, FP32 form 4944 -> 4890; 16^3 p=7 FP64 2732 -> 2575, FP32 2040 -> 1937; but with
// ragged runs 27x25x29 p=2 FP64 (72 bytes) 1183 -> 1331, 13x11x17 p=5 FP32 (144) 524 -> 541. The same
// hint on the metric terms or on the face results, stored or loaded, loses at 40^3 p=3 (6573, 6520,
// 6600 against 6342).
template <int RUN, typename T>
constexpr bool kWholeRun = RUN * (int)sizeof(T) % 128 == 0 || RUN * (int)sizeof(T) == 64;
template <int RUN, typename T>
__device__ __forceinline__ T load_once(const T *p) {
  if constexpr (kWholeRun<RUN, T>) return __builtin_nontemporal_load(p);
  else return *p;
}
template <int RUN, typename T>
__device__ __forceinline__ void store_once(T v, T *p) {
  if constexpr (kWholeRun<RUN, T>) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// ------------------------------------------------------------------------------------------
// Fused epilogue of the volume kernels: the source term and the RK register update of one
// point, in double precision.
// ------------------------------------------------------------------------------------------

// Body force g per unit mass (the source term S of Eq. (3)): component v of
// (0, rho g, m . g) from the point's state X.
__device__ __forceinline__ double body_force(const StageArgs &st, const double X[5], int v) {
  if (!st.force || v == 0) return 0.0;
  if (v < 4) return X[0] * st.g[v - 1];
  return dot3(X[1], st.g[0], X[2], st.g[1], X[3], st.g[2]);
}

// x: the state the stage was evaluated on; R: its residual; r1, r2: the registers' old values.
//   LSRK45:   dU <- a dU + dt R; U <- x + b dU                       (out0 = U, reg1 = dU, which the
//                                                                     last stage does not store)
//   RK4:      acc <- acc + w R; S <- Q + c dt R, or at the last stage Q <- Q + dt acc
//                                                (out0 = Q, reg1 = acc, reg2 = S)
//   SSP(10,4) (out0 = q1 = U, reg1 = q2): stages 0-3 and 5-8 take a forward-Euler step
//             q1 <- q1 + dt/6 R (stage 0 also sets q2 <- q1); stage 4 then combines
//             q2 <- q2/25 + 9/25 q1, q1 <- 15 q2 - 5 q1; stage 9 sets q1 <- q2 + 3/5 q1 + dt/10 R.
// Returns the value of the state the next stage is evaluated on (RK4: S, or Q after the last
// stage; the others: U), which the volume kernel's fused pre-pass of the next stage uses.
template <int NS>
__device__ __forceinline__ double rk_store(const StageArgs &st, int64_t o, double x, double R, double r1,
                                           double r2, double *out0, double *reg1, double *reg2) {
  if (st.mode == kModeResidual) {
    out0[o] = R;
    return 0.0;
  }
  if (st.mode == kModeLSRK) {
    const double du = fma(st.a, r1, st.dt * R);
    const double u = fma(st.b, du, x);
    if (!st.last) store_once<NS>(du, &reg1[o]);
    out0[o] = u;
    return u;
  }
  if (st.mode == kModeRK4) {
    const double acc = fma(st.w, R, r1);
    if (!st.last) {
      const double sn = fma(st.cdt, R, r2);
      store_once<NS>(acc, &reg1[o]);
      reg2[o] = sn;
      return sn;
    }
    const double q = fma(st.dt, acc, r2);
    out0[o] = q;
    return q;
  }
  if (st.stage == 9) {
    const double q = fma(st.dt / 10, R, fma(0.6, x, r1));
    out0[o] = q;
    return q;
  }
  const double q1 = fma(st.dt / 6, R, x);
  if (st.stage == 4) {
    const double q2 = fma(9.0 / 25, q1, r1 / 25);
    const double q = fma(15.0, q2, -5 * q1);
    reg1[o] = q2;
    out0[o] = q;
    return q;
  }
  if (st.stage == 0) reg1[o] = x;
  out0[o] = q1;
  return q1;
}

// ------------------------------------------------------------------------------------------
// Kernel configuration
// ------------------------------------------------------------------------------------------
template <int P>
struct Cfg {
  static constexpr int N = P + 1;
  static constexpr int NS = N * N * N;
  static constexpr int NFP = N * N;
  static constexpr int NF = 6 * NFP;
  static constexpr int EPB = (256 / NS) > 64 ? 64 : ((256 / NS) > 0 ? (256 / NS) : 1);  // elements per block
  static constexpr int BLOCK = EPB * NS;
  // the second tile choice: half of EPB; where EPB is one element whose points do not fill
  // whole waves (p = 5: 216 points in 4 waves, p = 6: 343 in 6), two elements per block, which
  // fill 7 and 11 waves
  static constexpr int EPB2 = EPB > 1 ? EPB / 2 : (NS % 64 != 0 && 2 * NS <= 1024 ? 2 : 1);
};

// Occupancy targets (waves per SIMD) per kernel and degree; 0 lets the compiler decide. From
// p = 2 on the FP64 volume kernels ask for 4 (at most 128 VGPRs): left alone the compiler takes
// up to 165 (3 waves; 2 for some) to hoist LDS reads, and the kernels are short of waves, not of
// loads in flight. Spills in bytes per lane: BR2 12 at p = 3 without the fused pre-pass, 20 and 28
// at p = 6 with one element per block (with and without it); LDG 12 at p = 3 without it and at p = 4
// and 5 with it, 20 and 28 at p = 6; with an eddy viscosity 12 at p = 3 both ways (LDG with it 20),
// 12 and 20 at p = 6; none elsewhere. The FP32 form's volume kernel with the fused pre-pass asks
// for 5: it fits 96 VGPRs at p = 2, 4, 5 and 6 (13x11x17 p=5 channel: 56.3 -> 52.1 us; 2431
// blocks then take two rounds of the chip instead of three; p = 6 with two elements per block
// spills 12 bytes); at p = 3 the viscous kernel takes 98 and runs 4, which is what its LDS with the
// metric terms allows. Without the pre-pass 96 spill (36 -> 48 us there), so it asks for 4 at p = 5
// and the compiler's choice is 4 elsewhere; at p = 7 a block is eight waves and a fifth wave per
// SIMD does not fit another.
#ifndef FR_WPE_PREPASS
#define FR_WPE_PREPASS(P) 0
#endif
#ifndef FR_WPE_FACE
#define FR_WPE_FACE(P) 0
#endif
#ifndef FR_WPE_VOLUME
#define FR_WPE_VOLUME(P, SGS, PRE) ((P) >= 2 ? 4 : 0)
#endif
// The LDG face kernel. Its LDS allows 2 waves at p = 1 and 7, 2.5 at p = 3, 3 elsewhere. It asks for
// 3 up to p = 5 (with an eddy viscosity p = 5 spills 32 bytes per lane) and for 2 above: at p = 6 it
// takes 150 VGPRs and runs 3, with an eddy viscosity 176 and one block of six waves per CU.
#ifndef FR_WPE_LDG
#define FR_WPE_LDG(P) ((P) <= 5 ? 3 : 2)
#endif
// The feature kernel: left alone the compiler takes 130 VGPRs at p = 6, two too many for 4 waves (us:
// 343 elements 13.8 -> 11.0, 3375 85.7 -> 66.7), and 97 at p = 7, where its LDS allows 6 waves (4096
// elements 75.8 -> 62.0).
#ifndef FR_WPE_FEATURES
#define FR_WPE_FEATURES(P) ((P) == 7 ? 6 : (P) == 6 ? 4 : 0)
#endif
#ifndef FR_WPE_VOLUME32
#define FR_WPE_VOLUME32(P, PRE) ((P) == 7 || ((P) == 5 && !(PRE)) ? 4 : ((P) >= 2 && (PRE) ? 5 : 0))
#endif
#define FR_WPE_ATTR(w) __attribute__((amdgpu_waves_per_eu((w) > 0 ? (w) : 1, (w) > 0 ? 8 : 8)))

// Whether `extra` more bytes of LDS per block leave the blocks a CU can hold unchanged: a block
// of `threads` threads using `bytes` of the CU's 160 KB (and at most 32 waves per CU).
constexpr int lds_blocks(int bytes, int threads) {
  const int by_lds = (160 * 1024) / bytes, by_waves = 32 / ((threads + 63) / 64);
  return by_lds < by_waves ? by_lds : by_waves;
}
constexpr bool lds_copy_fits(int bytes, int extra, int threads) {
  return lds_blocks(bytes + extra, threads) == lds_blocks(bytes, threads);
}

// The 1-D operators as kernel arguments; W, the folded divergence, only in FP64 (the FP32 components
// keep their traces).
template <typename real>
struct OpsT {
  real D[kMaxN * kMaxN];
  real lm[kMaxN];
  real lp[kMaxN];
  real gcL[kMaxN];
  real gcR[kMaxN];
};
template <>
struct OpsT<double> {
  double D[kMaxN * kMaxN];
  double lm[kMaxN];
  double lp[kMaxN];
  double gcL[kMaxN];
  double gcR[kMaxN];
  double W[kMaxN * kMaxN];
};

// Entry i of the operator entries a volume kernel keeps in LDS: D [N][N], gcL [N], gcR [N] and, in
// FP64, W [N][N] (kOpEntries of them).
template <int N>
constexpr int kOpEntries = 2 * N * N + 2 * N;
template <int N, typename real>
__device__ __forceinline__ real op_entry(const OpsT<real> &ops, int i) {
  const real *tab = reinterpret_cast<const real *>(&ops);
  constexpr bool HAS_W = sizeof(real) == 8;
  constexpr int oL = kMaxN * kMaxN + 2 * kMaxN, oR = oL + kMaxN, oW = oR + kMaxN;
  static_assert(sizeof(OpsT<real>) == (oW + (HAS_W ? kMaxN * kMaxN : 0)) * sizeof(real), "the table's members in order");
  return tab[i < N * N ? i : (i < N * N + N ? oL + i - N * N : (!HAS_W || i < N * N + 2 * N ? oR + i - N * N - N : oW + i - N * N - 2 * N))];
}

// Barrier between the LDS phases of an element's threads. Where an element's points fill whole
// waves or a wave holds whole elements (N_s = 1, 8, 64), only lanes of one wave exchange data:
// a wave's LDS instructions execute in order, so ordering the compiler's accesses is enough and
// the block's waves run on independently. Otherwise a block barrier.
template <int NS>
constexpr bool kWaveElement = 64 % NS == 0;
template <int NS>
__device__ __forceinline__ void elem_sync() {
  if constexpr (kWaveElement<NS>) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// Stores to the per-face-point buffers, which are written once and read once by the next
// kernel, as runs of NFP entries per value. They are non-temporal (+2.8% per stage at 64^3
// p=3) except where a run is shorter than a 128-byte line and does not divide it (doubles at
// p = 2, floats at p = 2 and 4): there consecutive runs share lines, and plain stores let L2
// merge the pieces (the p = 2 pre-pass 3.56 -> 1.52 ms at 80^3).
// MERGE: plain stores also for runs longer than a line that end inside one (p = 4, 5, 6). The
// pre-pass and the BR2 face kernels' interior faces take them: at 52^3 p = 4 FP64 1.14 -> 1.04 ms and
// 0.98 -> 0.90, at 43^3 p = 5 FP32 form 0.64 -> 0.59 and 0.48 -> 0.47. The fused tail does not: there
// they measured 1.57 -> 1.62 ms and 1.27 -> 1.28; nor does the LDG face kernel (not measured there).
// Wall faces and the FP32 form's mass flux are stored non-temporally whatever their runs: one
// value of ten at most, or the few faces of a wall. Face values at p = 0 and 1: see write_traces.
template <int NFP, bool MERGE = false, typename T>
__device__ __forceinline__ void face_store(T v, T *p) {
  constexpr int run = NFP * (int)sizeof(T);
  if constexpr (run % 128 == 0 || 128 % run == 0 || (run > 128 && !MERGE)) {
    __builtin_nontemporal_store(v, p);
  } else {
    *p = v;
  }
}

// A thread's point index along xi_2 within its element. With one element per block and N*N = 64
// points per xi_2-plane (p = 7), each wavefront covers exactly one plane, so the index is the same
// on every lane; saying so lets the compiler keep the operator row D[i2][.] in scalar registers.
template <int N, int EPB>
__device__ __forceinline__ int plane_index(int t) {
  if constexpr (N * N == 64 && EPB == 1) return __builtin_amdgcn_readfirstlane(t / (N * N));
  else return t / (N * N);
}

// Interpolation to both faces normal to direction d: the sums over the line through their face
// point (a, b), c along it, of lm[c] src[point c] and lp[c] src[point c], the line read once for the
// two. d must be the same on every lane of the wavefront (the p = 7 kernels give each wavefront
// one direction's 64 lines); it picks one of three loops whose LDS strides are constants.
// * In ascending c (ROT false, and d = 2 always) lm and lp are read through scalar loads. For
//   d = 0 and 1 the lines' common stride (8 or 64 entries) then puts 8 lanes of a wavefront on
//   one LDS bank at every step (16 for doubles): an 8-way conflict.
// * With ROT, a lane of d = 0 reads its whole line (contiguous) with 16-byte loads, two for
//   floats and four for doubles, and sums it in ascending c; src must then be 16-byte aligned.
//   For d = 1 lane (a, b) starts at c = b and wraps around (mod 8): every step then reads 64
//   different banks for floats, and 32 different 8-byte bank pairs per half-wavefront for
//   doubles. The weights of the rotated order come from rot, an LDS table [l(-1), l(-1), l(+1),
//   l(+1)] (rot_entry) where they are contiguous.
// A form's kernels all take the same ROT, and the sums are written with fma (left to the
// compiler, a sum whose last addition is moved behind a branch stays unfused in one kernel and not
// in another), so fused and separate stages keep the same sums. The
// FP32 form's p = 7 kernels take it (32^3: the pre-pass, at 6.5 conflict cycles per LDS
// instruction, went from 0.66 to 0.56 ms with one face per task); the FP64 ones do not: there the
// rotated sums cost the fused volume kernel more than they saved (1.74 -> 1.80 ms), and their
// table would cost the pre-pass, whose two blocks fill the LDS exactly, one of them.
template <int N, typename C>
__device__ __forceinline__ C rot_entry(const C *lm, const C *lp, int i) {
  return i < 2 * N ? lm[i % N] : lp[i % N];
}
template <int N, bool ROT = false, typename T, typename C>
__device__ __forceinline__ void face_sums_uniform(int d, int a, int b, const T *src, const C *lm, const C *lp, T &lo,
                                                  T &hi, const C *rot = nullptr) {
  constexpr bool R = ROT && N == 8;  // the rotation is worked out for lines of eight points
  lo = hi = 0;
  if (R && d == 0) {
    constexpr int K = 16 / (int)sizeof(T);
    using V = T __attribute__((ext_vector_type(K)));
    const V *q = reinterpret_cast<const V *>(src + N * (a + N * b));
#pragma unroll
    for (int j = 0; j < N / K; ++j) {
      const V x = q[j];
#pragma unroll
      for (int k = 0; k < K; ++k) {
        lo = fma(lm[j * K + k], x[k], lo);
        hi = fma(lp[j * K + k], x[k], hi);
      }
    }
  } else if (R && d == 1) {
    const int r = b & (N - 1);
    const C *w = rot + r;
    const T *q = src + a + N * N * b;
#pragma unroll
    for (int s = 0; s < N; ++s) {
      const T x = q[((s + r) & (N - 1)) * N];
      lo = fma(w[s], x, lo);
      hi = fma(w[2 * N + s], x, hi);
    }
  } else {
    const int base = d == 0 ? N * (a + N * b) : (d == 1 ? a + N * N * b : a + N * b);
    if (d == 0) {
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const T x = src[base + c];
        lo = fma(lm[c], x, lo);
        hi = fma(lp[c], x, hi);
      }
    } else if (d == 1) {
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const T x = src[base + c * N];
        lo = fma(lm[c], x, lo);
        hi = fma(lp[c], x, hi);
      }
    } else {
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const T x = src[base + c * N * N];
        lo = fma(lm[c], x, lo);
        hi = fma(lp[c], x, hi);
      }
    }
  }
}

// One wavefront per face of the element (64 face points, one per lane): p = 7 with one element
// per block, where the kernels take their face loops as wave-uniform (value, face) tasks.
template <int NFP, int EPB>
constexpr bool kWavePerFace = NFP == 64 && EPB == 1;

// The face values of NV point-ordered element arrays (array v at src + v N_s): every line of
// points normal to a pair of faces is read once and gives the values at both its ends, with
// uniform weights (scalar registers). Items are (GV arrays, line) over the element's threads t,
// one direction after the other, so the line's LDS strides are constants and consecutive lanes
// store consecutive points of a face. GV: few arrays per item where an item per line would leave
// many threads idle (N^2 lines of NV / GV items over N^3 threads). dst: the element's first face
// entry, [6][nval][NFP]; array v goes to its entry slot(v), which steps by one within an item.
// PIECES: plain stores (see kPieceElems).
template <int N, int NV, int GV, bool MERGE, bool PIECES, typename T, typename C, typename Slot>
__device__ __forceinline__ void trace_lines(int t, const T *src, const C *lm, const C *lp, T *dst, int nval, Slot slot) {
  constexpr int NFP = N * N, NS = N * N * N, ITEMS = NV / GV * NFP;
  static_assert(NV % GV == 0, "arrays per item");
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    for (int q = t; q < ITEMS; q += NS) {
      const int grp = q / NFP, kk = q - grp * NFP;
      const T *x = src + grp * (GV * NS) + (d == 0 ? N * kk : (d == 1 ? kk % N + NFP * (kk / N) : kk));
      T *out = dst + (2 * d * nval + slot(grp * GV)) * NFP + kk;
#pragma unroll
      for (int v = 0; v < GV; ++v) {
        T lo = 0, hi = 0;
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const T y = x[v * NS + c * (d == 0 ? 1 : (d == 1 ? N : NFP))];
          lo = fma(lm[c], y, lo);
          hi = fma(lp[c], y, hi);
        }
        if constexpr (PIECES) {
          out[v * NFP] = lo;
          out[(nval + v) * NFP] = hi;
        } else {
          face_store<NFP, MERGE>(lo, &out[v * NFP]);
          face_store<NFP, MERGE>(hi, &out[(nval + v) * NFP]);
        }
      }
    }
  }
}
// At p = 0 and 1 a run is 4 to 32 bytes, a piece of a line that an item fills over several of its
// stores, for both ends of its lines in turn. Stored non-temporally the pieces go to memory as
// pieces; through the cache the lines leave whole, which is the better on all but small meshes.
// kPieceElems: the element count up to which p = 1 stores non-temporally all the same. Two LSRK45
// steps (us), non-temporal / through the cache: p = 0 FP64 8000 elements 193 / 169, 24389 657 / 307,
// 54872 1576 / 533; FP32 form 8000 137 / 148, 24389 426 / 269, 54872 1017 / 388; p = 1 FP64 3375
// 183 / 193, 5832 278 / 250, 15625 600 / 412, 29791 1007 / 736; FP32 form 3375 161 / 178, 5832
// 246 / 245, 15625 542 / 374, 29791 962 / 678.
constexpr int64_t kPieceElems = 5500;
template <int N, int NV, int GV, bool MERGE = false, typename T, typename C, typename Slot>
__device__ __forceinline__ void write_traces(int64_t E, int t, const T *src, const C *lm, const C *lp, T *dst, int nval,
                                             Slot slot) {
  if constexpr (N <= 2) {
    if (N == 1 || E > kPieceElems) {
      // (the empty statements keep the compiler from joining the two branches' stores as plain ones)
      asm volatile("" ::: "memory");
      trace_lines<N, NV, GV, MERGE, true>(t, src, lm, lp, dst, nval, slot);
      asm volatile("" ::: "memory");
      return;
    }
  }
  trace_lines<N, NV, GV, MERGE, false>(t, src, lm, lp, dst, nval, slot);
}
// Arrays per item for 20 arrays: 5 where (20 / 5) N^2 items fill the N^3 threads, else 1.
template <int N>
constexpr int kTraceGroup = N == 1 || N == 2 || N == 4 ? 5 : 1;
