// Generated by gen_expansions.py -- do not edit.
// Cartesian expansion kernels for orders 0..4 (see the generator's docstring).
#pragma once
#include "softening.h"
namespace sfmm {
template <int P> struct Exp;
template <> struct Exp<0> {
  static constexpr int P = 0;
  static constexpr int NQ = 1;   // mass moments, |a| <= P
  static constexpr int NL = 4;   // local coefficients: H then P
  __device__ __forceinline__ static void p2m_add(const double* b, double m, double* Q) {
    double mb[1];
    mb[0] = 1.0;
    Q[0] = fma(m, mb[0], Q[0]);
  }
  static constexpr int FLOPS_P2M = 2;
  __device__ __forceinline__ static void m2m_add(const double* g, const double* Qc, double* Q) {
    double mg[1];
    mg[0] = 1.0;
    Q[0] = (Q[0] + Qc[0]);
  }
  static constexpr int FLOPS_M2M = 1;
  __device__ __forceinline__ static void m2l_add(const double* r, const double* Q, double* local) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[4];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    {
      double s = D[1] * Q[0];
      local[0] += s;
    }
    {
      double s = D[2] * Q[0];
      local[1] += s;
    }
    {
      double s = D[3] * Q[0];
      local[2] += s;
    }
    {
      double s = D[0] * Q[0];
      local[3] += s;
    }
  }
  static constexpr int FLOPS_M2L = 24;  // + one rsqrt
  __device__ __forceinline__ static void m2l_add_f32(const float* r, const float* Q, double* local, bool ok = true) {
    const float r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const float rinv = ok ? __frsqrt_rn(r2) : 0.0f;
    const float rinv2 = rinv * rinv;
    float D[4];
    D[0] = rinv;
    const float sn1 = rinv2 * -1.0f;
    D[1] = (1.0f * r[0] * D[0]) * sn1;
    D[2] = (1.0f * r[1] * D[0]) * sn1;
    D[3] = (1.0f * r[2] * D[0]) * sn1;
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[1] * Q[0];
      local[0] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[2] * Q[0];
      local[1] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[3] * Q[0];
      local[2] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[0] * Q[0];
      local[3] += (double)s;
    }
  }
  static constexpr int NQR = 1;   // independent moments
  static constexpr int NLR = 4;  // S then X
  __device__ __forceinline__ static void reduce(const double* Q, double* Qr) {
    Qr[0] = Q[0];
  }
  __device__ __forceinline__ static void m2l_h(const double* r, const double* Qr, double* lr, bool ok) {
    const double r2 = fma(r[0], r[0], fma(r[1], r[1], r[2] * r[2]));
    const double ri = rsqrt_refined(r2);
    const double rinv = ok && r2 < __builtin_inf() ? ri : 0.0;
    const double s = rinv * rinv;
    const double w[3] = {r[0] * s, r[1] * s, r[2] * s};
    const double R0_000 = rinv;
    const double R1_000 = -1.0 * rinv;
    lr[0] = fma(R0_000, Qr[0], lr[0]);
    const double R0_100 = w[0] * R1_000;
    lr[1] = fma(R0_100, Qr[0], lr[1]);
    const double R0_010 = w[1] * R1_000;
    lr[2] = fma(R0_010, Qr[0], lr[2]);
    const double R0_001 = w[2] * R1_000;
    lr[3] = fma(R0_001, Qr[0], lr[3]);
  }
  static constexpr int FLOPS_M2L_H = 21;  // + one refined rsqrt
  __device__ __forceinline__ static void expand(const double* lr, double* local) {
    double t[4];
    t[0] = lr[0];
    local[3] = t[0];
    t[1] = lr[1];
    local[0] = t[1];
    t[2] = lr[2];
    local[1] = t[2];
    t[3] = lr[3];
    local[2] = t[3];
  }
  __device__ __forceinline__ static void m2l_pair(const double* r, const double* QS,
                                                    const double* QTs, double* local,
                                                    double* outS) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[4];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    {
      double s = D[1] * QS[0];
      local[0] += s;
    }
    {
      double s = D[2] * QS[0];
      local[1] += s;
    }
    {
      double s = D[3] * QS[0];
      local[2] += s;
    }
    {
      double s = D[0] * QS[0];
      local[3] += s;
    }
    {
      double s = D[1] * QTs[0];
      unsafeAtomicAdd(&outS[0], -s);
    }
    {
      double s = D[2] * QTs[0];
      unsafeAtomicAdd(&outS[1], -s);
    }
    {
      double s = D[3] * QTs[0];
      unsafeAtomicAdd(&outS[2], -s);
    }
    {
      double s = D[0] * QTs[0];
      unsafeAtomicAdd(&outS[3], s);
    }
  }
  static constexpr int FLOPS_M2L_PAIR = 32;  // both directions, + one rsqrt
  __device__ __forceinline__ static void l2l(const double* h, double* local) {
    double mh[1];
    mh[0] = 1.0;
    local[0] = local[0];
    local[1] = local[1];
    local[2] = local[2];
    local[3] = local[3];
  }
  static constexpr int FLOPS_L2L = 0;
  __device__ __forceinline__ static void l2p(const double* a, const double* local, double* f, double& phi) {
    double ma[1];
    ma[0] = 1.0;
    f[0] += local[0];
    f[1] += local[1];
    f[2] += local[2];
    phi += local[3];
  }
  static constexpr int FLOPS_L2P = 4;
};
template <> struct Exp<1> {
  static constexpr int P = 1;
  static constexpr int NQ = 4;   // mass moments, |a| <= P
  static constexpr int NL = 13;   // local coefficients: H then P
  __device__ __forceinline__ static void p2m_add(const double* b, double m, double* Q) {
    double mb[4];
    mb[0] = 1.0;
    mb[1] = mb[0] * b[0];
    mb[2] = mb[0] * b[1];
    mb[3] = mb[0] * b[2];
    Q[0] = fma(m, mb[0], Q[0]);
    Q[1] = fma(m, mb[1], Q[1]);
    Q[2] = fma(m, mb[2], Q[2]);
    Q[3] = fma(m, mb[3], Q[3]);
  }
  static constexpr int FLOPS_P2M = 11;
  __device__ __forceinline__ static void m2m_add(const double* g, const double* Qc, double* Q) {
    double mg[4];
    mg[0] = 1.0;
    mg[1] = mg[0] * g[0];
    mg[2] = mg[0] * g[1];
    mg[3] = mg[0] * g[2];
    Q[0] = (Q[0] + Qc[0]);
    Q[1] = (fma(Qc[0], mg[1], Q[1]) + Qc[1]);
    Q[2] = (fma(Qc[0], mg[2], Q[2]) + Qc[2]);
    Q[3] = (fma(Qc[0], mg[3], Q[3]) + Qc[3]);
  }
  static constexpr int FLOPS_M2M = 13;
  __device__ __forceinline__ static void m2l_add(const double* r, const double* Q, double* local) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[10];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    const double sn2 = rinv2 * -0.5;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    D[4] = (6.0 * r[0] * D[1] + 2.0 * D[0]) * sn2;
    D[5] = (3.0 * r[0] * D[2] + 3.0 * r[1] * D[1]) * sn2;
    D[6] = (3.0 * r[0] * D[3] + 3.0 * r[2] * D[1]) * sn2;
    D[7] = (6.0 * r[1] * D[2] + 2.0 * D[0]) * sn2;
    D[8] = (3.0 * r[1] * D[3] + 3.0 * r[2] * D[2]) * sn2;
    D[9] = (6.0 * r[2] * D[3] + 2.0 * D[0]) * sn2;
    {
      double s = D[1] * Q[0];
      local[10] -= s;
      s = fma(D[4], Q[1], s);
      s = fma(D[5], Q[2], s);
      s = fma(D[6], Q[3], s);
      local[0] += s;
    }
    {
      double s = D[2] * Q[0];
      local[11] -= s;
      s = fma(D[5], Q[1], s);
      s = fma(D[7], Q[2], s);
      s = fma(D[8], Q[3], s);
      local[1] += s;
    }
    {
      double s = D[3] * Q[0];
      local[12] -= s;
      s = fma(D[6], Q[1], s);
      s = fma(D[8], Q[2], s);
      s = fma(D[9], Q[3], s);
      local[2] += s;
    }
    {
      double s = D[4] * Q[0];
      local[3] -= s;
    }
    {
      double s = D[5] * Q[0];
      local[4] -= s;
    }
    {
      double s = D[6] * Q[0];
      local[5] -= s;
    }
    {
      double s = D[7] * Q[0];
      local[6] -= s;
    }
    {
      double s = D[8] * Q[0];
      local[7] -= s;
    }
    {
      double s = D[9] * Q[0];
      local[8] -= s;
    }
    {
      double s = D[0] * Q[0];
      s = fma(D[1], Q[1], s);
      s = fma(D[2], Q[2], s);
      s = fma(D[3], Q[3], s);
      local[9] += s;
    }
  }
  static constexpr int FLOPS_M2L = 97;  // + one rsqrt
  __device__ __forceinline__ static void m2l_add_f32(const float* r, const float* Q, double* local, bool ok = true) {
    const float r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const float rinv = ok ? __frsqrt_rn(r2) : 0.0f;
    const float rinv2 = rinv * rinv;
    float D[10];
    D[0] = rinv;
    const float sn1 = rinv2 * -1.0f;
    const float sn2 = rinv2 * -0.5f;
    D[1] = (1.0f * r[0] * D[0]) * sn1;
    D[2] = (1.0f * r[1] * D[0]) * sn1;
    D[3] = (1.0f * r[2] * D[0]) * sn1;
    D[4] = (6.0f * r[0] * D[1] + 2.0f * D[0]) * sn2;
    D[5] = (3.0f * r[0] * D[2] + 3.0f * r[1] * D[1]) * sn2;
    D[6] = (3.0f * r[0] * D[3] + 3.0f * r[2] * D[1]) * sn2;
    D[7] = (6.0f * r[1] * D[2] + 2.0f * D[0]) * sn2;
    D[8] = (3.0f * r[1] * D[3] + 3.0f * r[2] * D[2]) * sn2;
    D[9] = (6.0f * r[2] * D[3] + 2.0f * D[0]) * sn2;
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[1] * Q[0];
      local[10] -= (double)s;
      s = fmaf(D[4], Q[1], s);
      s = fmaf(D[5], Q[2], s);
      s = fmaf(D[6], Q[3], s);
      local[0] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[2] * Q[0];
      local[11] -= (double)s;
      s = fmaf(D[5], Q[1], s);
      s = fmaf(D[7], Q[2], s);
      s = fmaf(D[8], Q[3], s);
      local[1] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[3] * Q[0];
      local[12] -= (double)s;
      s = fmaf(D[6], Q[1], s);
      s = fmaf(D[8], Q[2], s);
      s = fmaf(D[9], Q[3], s);
      local[2] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[4] * Q[0];
      local[3] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[5] * Q[0];
      local[4] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[6] * Q[0];
      local[5] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[7] * Q[0];
      local[6] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[8] * Q[0];
      local[7] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[9] * Q[0];
      local[8] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[0] * Q[0];
      s = fmaf(D[1], Q[1], s);
      s = fmaf(D[2], Q[2], s);
      s = fmaf(D[3], Q[3], s);
      local[9] += (double)s;
    }
  }
  static constexpr int NQR = 4;   // independent moments
  static constexpr int NLR = 12;  // S then X
  __device__ __forceinline__ static void reduce(const double* Q, double* Qr) {
    Qr[0] = Q[0];
    Qr[1] = Q[1];
    Qr[2] = Q[2];
    Qr[3] = Q[3];
  }
  __device__ __forceinline__ static void m2l_h(const double* r, const double* Qr, double* lr, bool ok) {
    const double r2 = fma(r[0], r[0], fma(r[1], r[1], r[2] * r[2]));
    const double ri = rsqrt_refined(r2);
    const double rinv = ok && r2 < __builtin_inf() ? ri : 0.0;
    const double s = rinv * rinv;
    const double w[3] = {r[0] * s, r[1] * s, r[2] * s};
    const double R0_000 = rinv;
    const double R1_000 = -1.0 * rinv;
    const double R2_000 = 3.0 * rinv;
    lr[0] = fma(R0_000, Qr[0], lr[0]);
    const double R0_100 = w[0] * R1_000;
    lr[0] = fma(R0_100, Qr[1], lr[0]);
    lr[1] = fma(R0_100, Qr[0], lr[1]);
    const double R0_010 = w[1] * R1_000;
    lr[0] = fma(R0_010, Qr[2], lr[0]);
    lr[2] = fma(R0_010, Qr[0], lr[2]);
    const double R0_001 = w[2] * R1_000;
    lr[0] = fma(R0_001, Qr[3], lr[0]);
    lr[3] = fma(R0_001, Qr[0], lr[3]);
    const double R1_100 = w[0] * R2_000;
    const double T1_000 = s * R1_000;
    const double R0_200 = fma(w[0], R1_100, T1_000);
    lr[4] = fma(R0_200, Qr[1], lr[4]);
    lr[7] = fma(R0_200, Qr[0], lr[7]);
    const double R1_010 = w[1] * R2_000;
    const double R0_110 = w[0] * R1_010;
    lr[4] = fma(R0_110, Qr[2], lr[4]);
    lr[5] = fma(R0_110, Qr[1], lr[5]);
    lr[8] = fma(R0_110, Qr[0], lr[8]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_101 = w[2] * R1_100;
    lr[4] = fma(R0_101, Qr[3], lr[4]);
    lr[6] = fma(R0_101, Qr[1], lr[6]);
    lr[9] = fma(R0_101, Qr[0], lr[9]);
    const double R0_020 = fma(w[1], R1_010, T1_000);
    lr[5] = fma(R0_020, Qr[2], lr[5]);
    lr[10] = fma(R0_020, Qr[0], lr[10]);
    const double R0_011 = w[2] * R1_010;
    lr[5] = fma(R0_011, Qr[3], lr[5]);
    lr[6] = fma(R0_011, Qr[2], lr[6]);
    lr[11] = fma(R0_011, Qr[0], lr[11]);
    const double R0_002 = -(R0_200 + R0_020);
    lr[6] = fma(R0_002, Qr[3], lr[6]);
  }
  static constexpr int FLOPS_M2L_H = 67;  // + one refined rsqrt
  __device__ __forceinline__ static void expand(const double* lr, double* local) {
    double t[10];
    t[0] = lr[0];
    local[9] = t[0];
    t[1] = -lr[1];
    local[10] = t[1];
    t[2] = -lr[2];
    local[11] = t[2];
    t[3] = -lr[3];
    local[12] = t[3];
    t[1] = (lr[1] + lr[4]);
    local[0] = t[1];
    t[2] = (lr[2] + lr[5]);
    local[1] = t[2];
    t[3] = (lr[3] + lr[6]);
    local[2] = t[3];
    t[4] = -lr[7];
    local[3] = t[4];
    t[5] = -lr[8];
    local[4] = t[5];
    t[6] = -lr[9];
    local[5] = t[6];
    t[7] = -lr[10];
    local[6] = t[7];
    t[8] = -lr[11];
    local[7] = t[8];
    t[9] = -(t[4] + t[7]);
    local[8] = t[9];
  }
  __device__ __forceinline__ static void m2l_pair(const double* r, const double* QS,
                                                    const double* QTs, double* local,
                                                    double* outS) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[10];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    const double sn2 = rinv2 * -0.5;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    D[4] = (6.0 * r[0] * D[1] + 2.0 * D[0]) * sn2;
    D[5] = (3.0 * r[0] * D[2] + 3.0 * r[1] * D[1]) * sn2;
    D[6] = (3.0 * r[0] * D[3] + 3.0 * r[2] * D[1]) * sn2;
    D[7] = (6.0 * r[1] * D[2] + 2.0 * D[0]) * sn2;
    D[8] = (3.0 * r[1] * D[3] + 3.0 * r[2] * D[2]) * sn2;
    D[9] = (6.0 * r[2] * D[3] + 2.0 * D[0]) * sn2;
    {
      double s = D[1] * QS[0];
      local[10] -= s;
      s = fma(D[4], QS[1], s);
      s = fma(D[5], QS[2], s);
      s = fma(D[6], QS[3], s);
      local[0] += s;
    }
    {
      double s = D[2] * QS[0];
      local[11] -= s;
      s = fma(D[5], QS[1], s);
      s = fma(D[7], QS[2], s);
      s = fma(D[8], QS[3], s);
      local[1] += s;
    }
    {
      double s = D[3] * QS[0];
      local[12] -= s;
      s = fma(D[6], QS[1], s);
      s = fma(D[8], QS[2], s);
      s = fma(D[9], QS[3], s);
      local[2] += s;
    }
    {
      double s = D[4] * QS[0];
      local[3] -= s;
    }
    {
      double s = D[5] * QS[0];
      local[4] -= s;
    }
    {
      double s = D[6] * QS[0];
      local[5] -= s;
    }
    {
      double s = D[7] * QS[0];
      local[6] -= s;
    }
    {
      double s = D[8] * QS[0];
      local[7] -= s;
    }
    {
      double s = D[9] * QS[0];
      local[8] -= s;
    }
    {
      double s = D[0] * QS[0];
      s = fma(D[1], QS[1], s);
      s = fma(D[2], QS[2], s);
      s = fma(D[3], QS[3], s);
      local[9] += s;
    }
    {
      double s = D[1] * QTs[0];
      unsafeAtomicAdd(&outS[10], s);
      s = fma(D[4], QTs[1], s);
      s = fma(D[5], QTs[2], s);
      s = fma(D[6], QTs[3], s);
      unsafeAtomicAdd(&outS[0], -s);
    }
    {
      double s = D[2] * QTs[0];
      unsafeAtomicAdd(&outS[11], s);
      s = fma(D[5], QTs[1], s);
      s = fma(D[7], QTs[2], s);
      s = fma(D[8], QTs[3], s);
      unsafeAtomicAdd(&outS[1], -s);
    }
    {
      double s = D[3] * QTs[0];
      unsafeAtomicAdd(&outS[12], s);
      s = fma(D[6], QTs[1], s);
      s = fma(D[8], QTs[2], s);
      s = fma(D[9], QTs[3], s);
      unsafeAtomicAdd(&outS[2], -s);
    }
    {
      double s = D[4] * QTs[0];
      unsafeAtomicAdd(&outS[3], -s);
    }
    {
      double s = D[5] * QTs[0];
      unsafeAtomicAdd(&outS[4], -s);
    }
    {
      double s = D[6] * QTs[0];
      unsafeAtomicAdd(&outS[5], -s);
    }
    {
      double s = D[7] * QTs[0];
      unsafeAtomicAdd(&outS[6], -s);
    }
    {
      double s = D[8] * QTs[0];
      unsafeAtomicAdd(&outS[7], -s);
    }
    {
      double s = D[9] * QTs[0];
      unsafeAtomicAdd(&outS[8], -s);
    }
    {
      double s = D[0] * QTs[0];
      s = fma(D[1], QTs[1], s);
      s = fma(D[2], QTs[2], s);
      s = fma(D[3], QTs[3], s);
      unsafeAtomicAdd(&outS[9], s);
    }
  }
  static constexpr int FLOPS_M2L_PAIR = 144;  // both directions, + one rsqrt
  __device__ __forceinline__ static void l2l(const double* h, double* local) {
    double mh[4];
    mh[0] = 1.0;
    mh[1] = mh[0] * h[0];
    mh[2] = mh[0] * h[1];
    mh[3] = mh[0] * h[2];
    local[0] = fma(local[5], mh[3], fma(local[4], mh[2], fma(local[3], mh[1], local[0])));
    local[1] = fma(local[7], mh[3], fma(local[6], mh[2], fma(local[4], mh[1], local[1])));
    local[2] = fma(local[8], mh[3], fma(local[7], mh[2], fma(local[5], mh[1], local[2])));
    local[3] = local[3];
    local[4] = local[4];
    local[5] = local[5];
    local[6] = local[6];
    local[7] = local[7];
    local[8] = local[8];
    local[9] = fma(local[12], mh[3], fma(local[11], mh[2], fma(local[10], mh[1], local[9])));
    local[10] = local[10];
    local[11] = local[11];
    local[12] = local[12];
  }
  static constexpr int FLOPS_L2L = 27;
  __device__ __forceinline__ static void l2p(const double* a, const double* local, double* f, double& phi) {
    double ma[4];
    ma[0] = 1.0;
    ma[1] = ma[0] * a[0];
    ma[2] = ma[0] * a[1];
    ma[3] = ma[0] * a[2];
    f[0] += fma(local[5], ma[3], fma(local[4], ma[2], fma(local[3], ma[1], local[0])));
    f[1] += fma(local[7], ma[3], fma(local[6], ma[2], fma(local[4], ma[1], local[1])));
    f[2] += fma(local[8], ma[3], fma(local[7], ma[2], fma(local[5], ma[1], local[2])));
    phi += fma(local[12], ma[3], fma(local[11], ma[2], fma(local[10], ma[1], local[9])));
  }
  static constexpr int FLOPS_L2P = 31;
};
template <> struct Exp<2> {
  static constexpr int P = 2;
  static constexpr int NQ = 10;   // mass moments, |a| <= P
  static constexpr int NL = 29;   // local coefficients: H then P
  __device__ __forceinline__ static void p2m_add(const double* b, double m, double* Q) {
    double mb[10];
    mb[0] = 1.0;
    mb[1] = mb[0] * b[0];
    mb[2] = mb[0] * b[1];
    mb[3] = mb[0] * b[2];
    mb[4] = mb[1] * (b[0] * 0.5);
    mb[5] = mb[2] * b[0];
    mb[6] = mb[3] * b[0];
    mb[7] = mb[2] * (b[1] * 0.5);
    mb[8] = mb[3] * b[1];
    mb[9] = mb[3] * (b[2] * 0.5);
    Q[0] = fma(m, mb[0], Q[0]);
    Q[1] = fma(m, mb[1], Q[1]);
    Q[2] = fma(m, mb[2], Q[2]);
    Q[3] = fma(m, mb[3], Q[3]);
    Q[4] = fma(m, mb[4], Q[4]);
    Q[5] = fma(m, mb[5], Q[5]);
    Q[6] = fma(m, mb[6], Q[6]);
    Q[7] = fma(m, mb[7], Q[7]);
    Q[8] = fma(m, mb[8], Q[8]);
    Q[9] = fma(m, mb[9], Q[9]);
  }
  static constexpr int FLOPS_P2M = 32;
  __device__ __forceinline__ static void m2m_add(const double* g, const double* Qc, double* Q) {
    double mg[10];
    mg[0] = 1.0;
    mg[1] = mg[0] * g[0];
    mg[2] = mg[0] * g[1];
    mg[3] = mg[0] * g[2];
    mg[4] = mg[1] * (g[0] * 0.5);
    mg[5] = mg[2] * g[0];
    mg[6] = mg[3] * g[0];
    mg[7] = mg[2] * (g[1] * 0.5);
    mg[8] = mg[3] * g[1];
    mg[9] = mg[3] * (g[2] * 0.5);
    Q[0] = (Q[0] + Qc[0]);
    Q[1] = (fma(Qc[0], mg[1], Q[1]) + Qc[1]);
    Q[2] = (fma(Qc[0], mg[2], Q[2]) + Qc[2]);
    Q[3] = (fma(Qc[0], mg[3], Q[3]) + Qc[3]);
    Q[4] = (fma(Qc[1], mg[1], fma(Qc[0], mg[4], Q[4])) + Qc[4]);
    Q[5] = (fma(Qc[2], mg[1], fma(Qc[1], mg[2], fma(Qc[0], mg[5], Q[5]))) + Qc[5]);
    Q[6] = (fma(Qc[3], mg[1], fma(Qc[1], mg[3], fma(Qc[0], mg[6], Q[6]))) + Qc[6]);
    Q[7] = (fma(Qc[2], mg[2], fma(Qc[0], mg[7], Q[7])) + Qc[7]);
    Q[8] = (fma(Qc[3], mg[2], fma(Qc[2], mg[3], fma(Qc[0], mg[8], Q[8]))) + Qc[8]);
    Q[9] = (fma(Qc[3], mg[3], fma(Qc[0], mg[9], Q[9])) + Qc[9]);
  }
  static constexpr int FLOPS_M2M = 58;
  __device__ __forceinline__ static void m2l_add(const double* r, const double* Q, double* local) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[20];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    const double sn2 = rinv2 * -0.5;
    const double sn3 = rinv2 * -0.3333333333333333;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    D[4] = (6.0 * r[0] * D[1] + 2.0 * D[0]) * sn2;
    D[5] = (3.0 * r[0] * D[2] + 3.0 * r[1] * D[1]) * sn2;
    D[6] = (3.0 * r[0] * D[3] + 3.0 * r[2] * D[1]) * sn2;
    D[7] = (6.0 * r[1] * D[2] + 2.0 * D[0]) * sn2;
    D[8] = (3.0 * r[1] * D[3] + 3.0 * r[2] * D[2]) * sn2;
    D[9] = (6.0 * r[2] * D[3] + 2.0 * D[0]) * sn2;
    D[10] = (15.0 * r[0] * D[4] + 12.0 * D[1]) * sn3;
    D[11] = (10.0 * r[0] * D[5] + 4.0 * D[2] + 5.0 * r[1] * D[4]) * sn3;
    D[12] = (10.0 * r[0] * D[6] + 4.0 * D[3] + 5.0 * r[2] * D[4]) * sn3;
    D[13] = (5.0 * r[0] * D[7] + 10.0 * r[1] * D[5] + 4.0 * D[1]) * sn3;
    D[14] = (5.0 * r[0] * D[8] + 5.0 * r[1] * D[6] + 5.0 * r[2] * D[5]) * sn3;
    D[15] = (5.0 * r[0] * D[9] + 10.0 * r[2] * D[6] + 4.0 * D[1]) * sn3;
    D[16] = (15.0 * r[1] * D[7] + 12.0 * D[2]) * sn3;
    D[17] = (10.0 * r[1] * D[8] + 4.0 * D[3] + 5.0 * r[2] * D[7]) * sn3;
    D[18] = (5.0 * r[1] * D[9] + 10.0 * r[2] * D[8] + 4.0 * D[2]) * sn3;
    D[19] = (15.0 * r[2] * D[9] + 12.0 * D[3]) * sn3;
    {
      double s = D[1] * Q[0];
      s = fma(D[4], Q[1], s);
      s = fma(D[5], Q[2], s);
      s = fma(D[6], Q[3], s);
      local[20] -= s;
      s = fma(D[10], Q[4], s);
      s = fma(D[11], Q[5], s);
      s = fma(D[12], Q[6], s);
      s = fma(D[13], Q[7], s);
      s = fma(D[14], Q[8], s);
      s = fma(D[15], Q[9], s);
      local[0] += s;
    }
    {
      double s = D[2] * Q[0];
      s = fma(D[5], Q[1], s);
      s = fma(D[7], Q[2], s);
      s = fma(D[8], Q[3], s);
      local[21] -= s;
      s = fma(D[11], Q[4], s);
      s = fma(D[13], Q[5], s);
      s = fma(D[14], Q[6], s);
      s = fma(D[16], Q[7], s);
      s = fma(D[17], Q[8], s);
      s = fma(D[18], Q[9], s);
      local[1] += s;
    }
    {
      double s = D[3] * Q[0];
      s = fma(D[6], Q[1], s);
      s = fma(D[8], Q[2], s);
      s = fma(D[9], Q[3], s);
      local[22] -= s;
      s = fma(D[12], Q[4], s);
      s = fma(D[14], Q[5], s);
      s = fma(D[15], Q[6], s);
      s = fma(D[17], Q[7], s);
      s = fma(D[18], Q[8], s);
      s = fma(D[19], Q[9], s);
      local[2] += s;
    }
    {
      double s = D[4] * Q[0];
      local[23] += s;
      s = fma(D[10], Q[1], s);
      s = fma(D[11], Q[2], s);
      s = fma(D[12], Q[3], s);
      local[3] -= s;
    }
    {
      double s = D[5] * Q[0];
      local[24] += s;
      s = fma(D[11], Q[1], s);
      s = fma(D[13], Q[2], s);
      s = fma(D[14], Q[3], s);
      local[4] -= s;
    }
    {
      double s = D[6] * Q[0];
      local[25] += s;
      s = fma(D[12], Q[1], s);
      s = fma(D[14], Q[2], s);
      s = fma(D[15], Q[3], s);
      local[5] -= s;
    }
    {
      double s = D[7] * Q[0];
      local[26] += s;
      s = fma(D[13], Q[1], s);
      s = fma(D[16], Q[2], s);
      s = fma(D[17], Q[3], s);
      local[6] -= s;
    }
    {
      double s = D[8] * Q[0];
      local[27] += s;
      s = fma(D[14], Q[1], s);
      s = fma(D[17], Q[2], s);
      s = fma(D[18], Q[3], s);
      local[7] -= s;
    }
    {
      double s = D[9] * Q[0];
      local[28] += s;
      s = fma(D[15], Q[1], s);
      s = fma(D[18], Q[2], s);
      s = fma(D[19], Q[3], s);
      local[8] -= s;
    }
    {
      double s = D[10] * Q[0];
      local[9] += s;
    }
    {
      double s = D[11] * Q[0];
      local[10] += s;
    }
    {
      double s = D[12] * Q[0];
      local[11] += s;
    }
    {
      double s = D[13] * Q[0];
      local[12] += s;
    }
    {
      double s = D[14] * Q[0];
      local[13] += s;
    }
    {
      double s = D[15] * Q[0];
      local[14] += s;
    }
    {
      double s = D[16] * Q[0];
      local[15] += s;
    }
    {
      double s = D[17] * Q[0];
      local[16] += s;
    }
    {
      double s = D[18] * Q[0];
      local[17] += s;
    }
    {
      double s = D[19] * Q[0];
      local[18] += s;
    }
    {
      double s = D[0] * Q[0];
      s = fma(D[1], Q[1], s);
      s = fma(D[2], Q[2], s);
      s = fma(D[3], Q[3], s);
      s = fma(D[4], Q[4], s);
      s = fma(D[5], Q[5], s);
      s = fma(D[6], Q[6], s);
      s = fma(D[7], Q[7], s);
      s = fma(D[8], Q[8], s);
      s = fma(D[9], Q[9], s);
      local[19] += s;
    }
  }
  static constexpr int FLOPS_M2L = 280;  // + one rsqrt
  __device__ __forceinline__ static void m2l_add_f32(const float* r, const float* Q, double* local, bool ok = true) {
    const float r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const float rinv = ok ? __frsqrt_rn(r2) : 0.0f;
    const float rinv2 = rinv * rinv;
    float D[20];
    D[0] = rinv;
    const float sn1 = rinv2 * -1.0f;
    const float sn2 = rinv2 * -0.5f;
    const float sn3 = rinv2 * -0.3333333333333333f;
    D[1] = (1.0f * r[0] * D[0]) * sn1;
    D[2] = (1.0f * r[1] * D[0]) * sn1;
    D[3] = (1.0f * r[2] * D[0]) * sn1;
    D[4] = (6.0f * r[0] * D[1] + 2.0f * D[0]) * sn2;
    D[5] = (3.0f * r[0] * D[2] + 3.0f * r[1] * D[1]) * sn2;
    D[6] = (3.0f * r[0] * D[3] + 3.0f * r[2] * D[1]) * sn2;
    D[7] = (6.0f * r[1] * D[2] + 2.0f * D[0]) * sn2;
    D[8] = (3.0f * r[1] * D[3] + 3.0f * r[2] * D[2]) * sn2;
    D[9] = (6.0f * r[2] * D[3] + 2.0f * D[0]) * sn2;
    D[10] = (15.0f * r[0] * D[4] + 12.0f * D[1]) * sn3;
    D[11] = (10.0f * r[0] * D[5] + 4.0f * D[2] + 5.0f * r[1] * D[4]) * sn3;
    D[12] = (10.0f * r[0] * D[6] + 4.0f * D[3] + 5.0f * r[2] * D[4]) * sn3;
    D[13] = (5.0f * r[0] * D[7] + 10.0f * r[1] * D[5] + 4.0f * D[1]) * sn3;
    D[14] = (5.0f * r[0] * D[8] + 5.0f * r[1] * D[6] + 5.0f * r[2] * D[5]) * sn3;
    D[15] = (5.0f * r[0] * D[9] + 10.0f * r[2] * D[6] + 4.0f * D[1]) * sn3;
    D[16] = (15.0f * r[1] * D[7] + 12.0f * D[2]) * sn3;
    D[17] = (10.0f * r[1] * D[8] + 4.0f * D[3] + 5.0f * r[2] * D[7]) * sn3;
    D[18] = (5.0f * r[1] * D[9] + 10.0f * r[2] * D[8] + 4.0f * D[2]) * sn3;
    D[19] = (15.0f * r[2] * D[9] + 12.0f * D[3]) * sn3;
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[1] * Q[0];
      s = fmaf(D[4], Q[1], s);
      s = fmaf(D[5], Q[2], s);
      s = fmaf(D[6], Q[3], s);
      local[20] -= (double)s;
      s = fmaf(D[10], Q[4], s);
      s = fmaf(D[11], Q[5], s);
      s = fmaf(D[12], Q[6], s);
      s = fmaf(D[13], Q[7], s);
      s = fmaf(D[14], Q[8], s);
      s = fmaf(D[15], Q[9], s);
      local[0] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[2] * Q[0];
      s = fmaf(D[5], Q[1], s);
      s = fmaf(D[7], Q[2], s);
      s = fmaf(D[8], Q[3], s);
      local[21] -= (double)s;
      s = fmaf(D[11], Q[4], s);
      s = fmaf(D[13], Q[5], s);
      s = fmaf(D[14], Q[6], s);
      s = fmaf(D[16], Q[7], s);
      s = fmaf(D[17], Q[8], s);
      s = fmaf(D[18], Q[9], s);
      local[1] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[3] * Q[0];
      s = fmaf(D[6], Q[1], s);
      s = fmaf(D[8], Q[2], s);
      s = fmaf(D[9], Q[3], s);
      local[22] -= (double)s;
      s = fmaf(D[12], Q[4], s);
      s = fmaf(D[14], Q[5], s);
      s = fmaf(D[15], Q[6], s);
      s = fmaf(D[17], Q[7], s);
      s = fmaf(D[18], Q[8], s);
      s = fmaf(D[19], Q[9], s);
      local[2] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[4] * Q[0];
      local[23] += (double)s;
      s = fmaf(D[10], Q[1], s);
      s = fmaf(D[11], Q[2], s);
      s = fmaf(D[12], Q[3], s);
      local[3] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[5] * Q[0];
      local[24] += (double)s;
      s = fmaf(D[11], Q[1], s);
      s = fmaf(D[13], Q[2], s);
      s = fmaf(D[14], Q[3], s);
      local[4] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[6] * Q[0];
      local[25] += (double)s;
      s = fmaf(D[12], Q[1], s);
      s = fmaf(D[14], Q[2], s);
      s = fmaf(D[15], Q[3], s);
      local[5] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[7] * Q[0];
      local[26] += (double)s;
      s = fmaf(D[13], Q[1], s);
      s = fmaf(D[16], Q[2], s);
      s = fmaf(D[17], Q[3], s);
      local[6] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[8] * Q[0];
      local[27] += (double)s;
      s = fmaf(D[14], Q[1], s);
      s = fmaf(D[17], Q[2], s);
      s = fmaf(D[18], Q[3], s);
      local[7] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[9] * Q[0];
      local[28] += (double)s;
      s = fmaf(D[15], Q[1], s);
      s = fmaf(D[18], Q[2], s);
      s = fmaf(D[19], Q[3], s);
      local[8] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[10] * Q[0];
      local[9] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[11] * Q[0];
      local[10] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[12] * Q[0];
      local[11] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[13] * Q[0];
      local[12] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[14] * Q[0];
      local[13] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[15] * Q[0];
      local[14] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[16] * Q[0];
      local[15] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[17] * Q[0];
      local[16] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[18] * Q[0];
      local[17] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[19] * Q[0];
      local[18] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[0] * Q[0];
      s = fmaf(D[1], Q[1], s);
      s = fmaf(D[2], Q[2], s);
      s = fmaf(D[3], Q[3], s);
      s = fmaf(D[4], Q[4], s);
      s = fmaf(D[5], Q[5], s);
      s = fmaf(D[6], Q[6], s);
      s = fmaf(D[7], Q[7], s);
      s = fmaf(D[8], Q[8], s);
      s = fmaf(D[9], Q[9], s);
      local[19] += (double)s;
    }
  }
  static constexpr int NQR = 9;   // independent moments
  static constexpr int NLR = 24;  // S then X
  __device__ __forceinline__ static void reduce(const double* Q, double* Qr) {
    Qr[0] = Q[0];
    Qr[1] = Q[1];
    Qr[2] = Q[2];
    Qr[3] = Q[3];
    Qr[4] = Q[4] - Q[9];
    Qr[5] = Q[5];
    Qr[6] = Q[6];
    Qr[7] = Q[7] - Q[9];
    Qr[8] = Q[8];
  }
  __device__ __forceinline__ static void m2l_h(const double* r, const double* Qr, double* lr, bool ok) {
    const double r2 = fma(r[0], r[0], fma(r[1], r[1], r[2] * r[2]));
    const double ri = rsqrt_refined(r2);
    const double rinv = ok && r2 < __builtin_inf() ? ri : 0.0;
    const double s = rinv * rinv;
    const double w[3] = {r[0] * s, r[1] * s, r[2] * s};
    const double R0_000 = rinv;
    const double R1_000 = -1.0 * rinv;
    const double R2_000 = 3.0 * rinv;
    const double R3_000 = -15.0 * rinv;
    lr[0] = fma(R0_000, Qr[0], lr[0]);
    const double R0_100 = w[0] * R1_000;
    lr[0] = fma(R0_100, Qr[1], lr[0]);
    lr[1] = fma(R0_100, Qr[0], lr[1]);
    const double R0_010 = w[1] * R1_000;
    lr[0] = fma(R0_010, Qr[2], lr[0]);
    lr[2] = fma(R0_010, Qr[0], lr[2]);
    const double R0_001 = w[2] * R1_000;
    lr[0] = fma(R0_001, Qr[3], lr[0]);
    lr[3] = fma(R0_001, Qr[0], lr[3]);
    const double R1_100 = w[0] * R2_000;
    const double T1_000 = s * R1_000;
    const double R0_200 = fma(w[0], R1_100, T1_000);
    lr[0] = fma(R0_200, Qr[4], lr[0]);
    lr[1] = fma(R0_200, Qr[1], lr[1]);
    lr[4] = fma(R0_200, Qr[0], lr[4]);
    const double R1_010 = w[1] * R2_000;
    const double R0_110 = w[0] * R1_010;
    lr[0] = fma(R0_110, Qr[5], lr[0]);
    lr[1] = fma(R0_110, Qr[2], lr[1]);
    lr[2] = fma(R0_110, Qr[1], lr[2]);
    lr[5] = fma(R0_110, Qr[0], lr[5]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_101 = w[2] * R1_100;
    lr[0] = fma(R0_101, Qr[6], lr[0]);
    lr[1] = fma(R0_101, Qr[3], lr[1]);
    lr[3] = fma(R0_101, Qr[1], lr[3]);
    lr[6] = fma(R0_101, Qr[0], lr[6]);
    const double R0_020 = fma(w[1], R1_010, T1_000);
    lr[0] = fma(R0_020, Qr[7], lr[0]);
    lr[2] = fma(R0_020, Qr[2], lr[2]);
    lr[7] = fma(R0_020, Qr[0], lr[7]);
    const double R0_011 = w[2] * R1_010;
    lr[0] = fma(R0_011, Qr[8], lr[0]);
    lr[2] = fma(R0_011, Qr[3], lr[2]);
    lr[3] = fma(R0_011, Qr[2], lr[3]);
    lr[8] = fma(R0_011, Qr[0], lr[8]);
    const double R0_002 = -(R0_200 + R0_020);
    lr[3] = fma(R0_002, Qr[3], lr[3]);
    __builtin_amdgcn_sched_barrier(0);
    const double R2_100 = w[0] * R3_000;
    const double T2_000 = s * R2_000;
    const double R1_200 = fma(w[0], R2_100, T2_000);
    const double T1_100 = s * R1_100;
    const double R0_300 = fma(w[0], R1_200, 2.0 * T1_100);
    lr[9] = fma(R0_300, Qr[4], lr[9]);
    lr[12] = fma(R0_300, Qr[1], lr[12]);
    lr[17] = fma(R0_300, Qr[0], lr[17]);
    const double R2_010 = w[1] * R3_000;
    const double R1_110 = w[0] * R2_010;
    const double T1_010 = s * R1_010;
    const double R0_210 = fma(w[0], R1_110, T1_010);
    lr[9] = fma(R0_210, Qr[5], lr[9]);
    lr[10] = fma(R0_210, Qr[4], lr[10]);
    lr[12] = fma(R0_210, Qr[2], lr[12]);
    lr[13] = fma(R0_210, Qr[1], lr[13]);
    lr[18] = fma(R0_210, Qr[0], lr[18]);
    const double R0_201 = w[2] * R1_200;
    lr[9] = fma(R0_201, Qr[6], lr[9]);
    lr[11] = fma(R0_201, Qr[4], lr[11]);
    lr[12] = fma(R0_201, Qr[3], lr[12]);
    lr[14] = fma(R0_201, Qr[1], lr[14]);
    lr[19] = fma(R0_201, Qr[0], lr[19]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_120 = fma(w[1], R1_110, T1_100);
    lr[9] = fma(R0_120, Qr[7], lr[9]);
    lr[10] = fma(R0_120, Qr[5], lr[10]);
    lr[13] = fma(R0_120, Qr[2], lr[13]);
    lr[15] = fma(R0_120, Qr[1], lr[15]);
    lr[20] = fma(R0_120, Qr[0], lr[20]);
    const double R0_111 = w[2] * R1_110;
    lr[9] = fma(R0_111, Qr[8], lr[9]);
    lr[10] = fma(R0_111, Qr[6], lr[10]);
    lr[11] = fma(R0_111, Qr[5], lr[11]);
    lr[13] = fma(R0_111, Qr[3], lr[13]);
    lr[14] = fma(R0_111, Qr[2], lr[14]);
    lr[16] = fma(R0_111, Qr[1], lr[16]);
    lr[21] = fma(R0_111, Qr[0], lr[21]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_102 = -(R0_300 + R0_120);
    lr[11] = fma(R0_102, Qr[6], lr[11]);
    lr[14] = fma(R0_102, Qr[3], lr[14]);
    const double R1_020 = fma(w[1], R2_010, T2_000);
    const double R0_030 = fma(w[1], R1_020, 2.0 * T1_010);
    lr[10] = fma(R0_030, Qr[7], lr[10]);
    lr[15] = fma(R0_030, Qr[2], lr[15]);
    lr[22] = fma(R0_030, Qr[0], lr[22]);
    const double R0_021 = w[2] * R1_020;
    lr[10] = fma(R0_021, Qr[8], lr[10]);
    lr[11] = fma(R0_021, Qr[7], lr[11]);
    lr[15] = fma(R0_021, Qr[3], lr[15]);
    lr[16] = fma(R0_021, Qr[2], lr[16]);
    lr[23] = fma(R0_021, Qr[0], lr[23]);
    const double R0_012 = -(R0_210 + R0_030);
    lr[11] = fma(R0_012, Qr[8], lr[11]);
    lr[16] = fma(R0_012, Qr[3], lr[16]);
  }
  static constexpr int FLOPS_M2L_H = 177;  // + one refined rsqrt
  __device__ __forceinline__ static void expand(const double* lr, double* local) {
    double t[20];
    t[0] = lr[0];
    local[19] = t[0];
    t[1] = -lr[1];
    local[20] = t[1];
    t[2] = -lr[2];
    local[21] = t[2];
    t[3] = -lr[3];
    local[22] = t[3];
    t[4] = lr[4];
    local[23] = t[4];
    t[5] = lr[5];
    local[24] = t[5];
    t[6] = lr[6];
    local[25] = t[6];
    t[7] = lr[7];
    local[26] = t[7];
    t[8] = lr[8];
    local[27] = t[8];
    t[9] = -(t[4] + t[7]);
    local[28] = t[9];
    t[1] = (lr[1] + lr[9]);
    local[0] = t[1];
    t[2] = (lr[2] + lr[10]);
    local[1] = t[2];
    t[3] = (lr[3] + lr[11]);
    local[2] = t[3];
    t[4] = -(lr[4] + lr[12]);
    local[3] = t[4];
    t[5] = -(lr[5] + lr[13]);
    local[4] = t[5];
    t[6] = -(lr[6] + lr[14]);
    local[5] = t[6];
    t[7] = -(lr[7] + lr[15]);
    local[6] = t[7];
    t[8] = -(lr[8] + lr[16]);
    local[7] = t[8];
    t[9] = -(t[4] + t[7]);
    local[8] = t[9];
    t[10] = lr[17];
    local[9] = t[10];
    t[11] = lr[18];
    local[10] = t[11];
    t[12] = lr[19];
    local[11] = t[12];
    t[13] = lr[20];
    local[12] = t[13];
    t[14] = lr[21];
    local[13] = t[14];
    t[15] = -(t[10] + t[13]);
    local[14] = t[15];
    t[16] = lr[22];
    local[15] = t[16];
    t[17] = lr[23];
    local[16] = t[17];
    t[18] = -(t[11] + t[16]);
    local[17] = t[18];
    t[19] = -(t[12] + t[17]);
    local[18] = t[19];
  }
  __device__ __forceinline__ static void m2l_pair(const double* r, const double* QS,
                                                    const double* QTs, double* local,
                                                    double* outS) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[20];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    const double sn2 = rinv2 * -0.5;
    const double sn3 = rinv2 * -0.3333333333333333;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    D[4] = (6.0 * r[0] * D[1] + 2.0 * D[0]) * sn2;
    D[5] = (3.0 * r[0] * D[2] + 3.0 * r[1] * D[1]) * sn2;
    D[6] = (3.0 * r[0] * D[3] + 3.0 * r[2] * D[1]) * sn2;
    D[7] = (6.0 * r[1] * D[2] + 2.0 * D[0]) * sn2;
    D[8] = (3.0 * r[1] * D[3] + 3.0 * r[2] * D[2]) * sn2;
    D[9] = (6.0 * r[2] * D[3] + 2.0 * D[0]) * sn2;
    D[10] = (15.0 * r[0] * D[4] + 12.0 * D[1]) * sn3;
    D[11] = (10.0 * r[0] * D[5] + 4.0 * D[2] + 5.0 * r[1] * D[4]) * sn3;
    D[12] = (10.0 * r[0] * D[6] + 4.0 * D[3] + 5.0 * r[2] * D[4]) * sn3;
    D[13] = (5.0 * r[0] * D[7] + 10.0 * r[1] * D[5] + 4.0 * D[1]) * sn3;
    D[14] = (5.0 * r[0] * D[8] + 5.0 * r[1] * D[6] + 5.0 * r[2] * D[5]) * sn3;
    D[15] = (5.0 * r[0] * D[9] + 10.0 * r[2] * D[6] + 4.0 * D[1]) * sn3;
    D[16] = (15.0 * r[1] * D[7] + 12.0 * D[2]) * sn3;
    D[17] = (10.0 * r[1] * D[8] + 4.0 * D[3] + 5.0 * r[2] * D[7]) * sn3;
    D[18] = (5.0 * r[1] * D[9] + 10.0 * r[2] * D[8] + 4.0 * D[2]) * sn3;
    D[19] = (15.0 * r[2] * D[9] + 12.0 * D[3]) * sn3;
    {
      double s = D[1] * QS[0];
      s = fma(D[4], QS[1], s);
      s = fma(D[5], QS[2], s);
      s = fma(D[6], QS[3], s);
      local[20] -= s;
      s = fma(D[10], QS[4], s);
      s = fma(D[11], QS[5], s);
      s = fma(D[12], QS[6], s);
      s = fma(D[13], QS[7], s);
      s = fma(D[14], QS[8], s);
      s = fma(D[15], QS[9], s);
      local[0] += s;
    }
    {
      double s = D[2] * QS[0];
      s = fma(D[5], QS[1], s);
      s = fma(D[7], QS[2], s);
      s = fma(D[8], QS[3], s);
      local[21] -= s;
      s = fma(D[11], QS[4], s);
      s = fma(D[13], QS[5], s);
      s = fma(D[14], QS[6], s);
      s = fma(D[16], QS[7], s);
      s = fma(D[17], QS[8], s);
      s = fma(D[18], QS[9], s);
      local[1] += s;
    }
    {
      double s = D[3] * QS[0];
      s = fma(D[6], QS[1], s);
      s = fma(D[8], QS[2], s);
      s = fma(D[9], QS[3], s);
      local[22] -= s;
      s = fma(D[12], QS[4], s);
      s = fma(D[14], QS[5], s);
      s = fma(D[15], QS[6], s);
      s = fma(D[17], QS[7], s);
      s = fma(D[18], QS[8], s);
      s = fma(D[19], QS[9], s);
      local[2] += s;
    }
    {
      double s = D[4] * QS[0];
      local[23] += s;
      s = fma(D[10], QS[1], s);
      s = fma(D[11], QS[2], s);
      s = fma(D[12], QS[3], s);
      local[3] -= s;
    }
    {
      double s = D[5] * QS[0];
      local[24] += s;
      s = fma(D[11], QS[1], s);
      s = fma(D[13], QS[2], s);
      s = fma(D[14], QS[3], s);
      local[4] -= s;
    }
    {
      double s = D[6] * QS[0];
      local[25] += s;
      s = fma(D[12], QS[1], s);
      s = fma(D[14], QS[2], s);
      s = fma(D[15], QS[3], s);
      local[5] -= s;
    }
    {
      double s = D[7] * QS[0];
      local[26] += s;
      s = fma(D[13], QS[1], s);
      s = fma(D[16], QS[2], s);
      s = fma(D[17], QS[3], s);
      local[6] -= s;
    }
    {
      double s = D[8] * QS[0];
      local[27] += s;
      s = fma(D[14], QS[1], s);
      s = fma(D[17], QS[2], s);
      s = fma(D[18], QS[3], s);
      local[7] -= s;
    }
    {
      double s = D[9] * QS[0];
      local[28] += s;
      s = fma(D[15], QS[1], s);
      s = fma(D[18], QS[2], s);
      s = fma(D[19], QS[3], s);
      local[8] -= s;
    }
    {
      double s = D[10] * QS[0];
      local[9] += s;
    }
    {
      double s = D[11] * QS[0];
      local[10] += s;
    }
    {
      double s = D[12] * QS[0];
      local[11] += s;
    }
    {
      double s = D[13] * QS[0];
      local[12] += s;
    }
    {
      double s = D[14] * QS[0];
      local[13] += s;
    }
    {
      double s = D[15] * QS[0];
      local[14] += s;
    }
    {
      double s = D[16] * QS[0];
      local[15] += s;
    }
    {
      double s = D[17] * QS[0];
      local[16] += s;
    }
    {
      double s = D[18] * QS[0];
      local[17] += s;
    }
    {
      double s = D[19] * QS[0];
      local[18] += s;
    }
    {
      double s = D[0] * QS[0];
      s = fma(D[1], QS[1], s);
      s = fma(D[2], QS[2], s);
      s = fma(D[3], QS[3], s);
      s = fma(D[4], QS[4], s);
      s = fma(D[5], QS[5], s);
      s = fma(D[6], QS[6], s);
      s = fma(D[7], QS[7], s);
      s = fma(D[8], QS[8], s);
      s = fma(D[9], QS[9], s);
      local[19] += s;
    }
    {
      double s = D[1] * QTs[0];
      s = fma(D[4], QTs[1], s);
      s = fma(D[5], QTs[2], s);
      s = fma(D[6], QTs[3], s);
      unsafeAtomicAdd(&outS[20], s);
      s = fma(D[10], QTs[4], s);
      s = fma(D[11], QTs[5], s);
      s = fma(D[12], QTs[6], s);
      s = fma(D[13], QTs[7], s);
      s = fma(D[14], QTs[8], s);
      s = fma(D[15], QTs[9], s);
      unsafeAtomicAdd(&outS[0], -s);
    }
    {
      double s = D[2] * QTs[0];
      s = fma(D[5], QTs[1], s);
      s = fma(D[7], QTs[2], s);
      s = fma(D[8], QTs[3], s);
      unsafeAtomicAdd(&outS[21], s);
      s = fma(D[11], QTs[4], s);
      s = fma(D[13], QTs[5], s);
      s = fma(D[14], QTs[6], s);
      s = fma(D[16], QTs[7], s);
      s = fma(D[17], QTs[8], s);
      s = fma(D[18], QTs[9], s);
      unsafeAtomicAdd(&outS[1], -s);
    }
    {
      double s = D[3] * QTs[0];
      s = fma(D[6], QTs[1], s);
      s = fma(D[8], QTs[2], s);
      s = fma(D[9], QTs[3], s);
      unsafeAtomicAdd(&outS[22], s);
      s = fma(D[12], QTs[4], s);
      s = fma(D[14], QTs[5], s);
      s = fma(D[15], QTs[6], s);
      s = fma(D[17], QTs[7], s);
      s = fma(D[18], QTs[8], s);
      s = fma(D[19], QTs[9], s);
      unsafeAtomicAdd(&outS[2], -s);
    }
    {
      double s = D[4] * QTs[0];
      unsafeAtomicAdd(&outS[23], s);
      s = fma(D[10], QTs[1], s);
      s = fma(D[11], QTs[2], s);
      s = fma(D[12], QTs[3], s);
      unsafeAtomicAdd(&outS[3], -s);
    }
    {
      double s = D[5] * QTs[0];
      unsafeAtomicAdd(&outS[24], s);
      s = fma(D[11], QTs[1], s);
      s = fma(D[13], QTs[2], s);
      s = fma(D[14], QTs[3], s);
      unsafeAtomicAdd(&outS[4], -s);
    }
    {
      double s = D[6] * QTs[0];
      unsafeAtomicAdd(&outS[25], s);
      s = fma(D[12], QTs[1], s);
      s = fma(D[14], QTs[2], s);
      s = fma(D[15], QTs[3], s);
      unsafeAtomicAdd(&outS[5], -s);
    }
    {
      double s = D[7] * QTs[0];
      unsafeAtomicAdd(&outS[26], s);
      s = fma(D[13], QTs[1], s);
      s = fma(D[16], QTs[2], s);
      s = fma(D[17], QTs[3], s);
      unsafeAtomicAdd(&outS[6], -s);
    }
    {
      double s = D[8] * QTs[0];
      unsafeAtomicAdd(&outS[27], s);
      s = fma(D[14], QTs[1], s);
      s = fma(D[17], QTs[2], s);
      s = fma(D[18], QTs[3], s);
      unsafeAtomicAdd(&outS[7], -s);
    }
    {
      double s = D[9] * QTs[0];
      unsafeAtomicAdd(&outS[28], s);
      s = fma(D[15], QTs[1], s);
      s = fma(D[18], QTs[2], s);
      s = fma(D[19], QTs[3], s);
      unsafeAtomicAdd(&outS[8], -s);
    }
    {
      double s = D[10] * QTs[0];
      unsafeAtomicAdd(&outS[9], -s);
    }
    {
      double s = D[11] * QTs[0];
      unsafeAtomicAdd(&outS[10], -s);
    }
    {
      double s = D[12] * QTs[0];
      unsafeAtomicAdd(&outS[11], -s);
    }
    {
      double s = D[13] * QTs[0];
      unsafeAtomicAdd(&outS[12], -s);
    }
    {
      double s = D[14] * QTs[0];
      unsafeAtomicAdd(&outS[13], -s);
    }
    {
      double s = D[15] * QTs[0];
      unsafeAtomicAdd(&outS[14], -s);
    }
    {
      double s = D[16] * QTs[0];
      unsafeAtomicAdd(&outS[15], -s);
    }
    {
      double s = D[17] * QTs[0];
      unsafeAtomicAdd(&outS[16], -s);
    }
    {
      double s = D[18] * QTs[0];
      unsafeAtomicAdd(&outS[17], -s);
    }
    {
      double s = D[19] * QTs[0];
      unsafeAtomicAdd(&outS[18], -s);
    }
    {
      double s = D[0] * QTs[0];
      s = fma(D[1], QTs[1], s);
      s = fma(D[2], QTs[2], s);
      s = fma(D[3], QTs[3], s);
      s = fma(D[4], QTs[4], s);
      s = fma(D[5], QTs[5], s);
      s = fma(D[6], QTs[6], s);
      s = fma(D[7], QTs[7], s);
      s = fma(D[8], QTs[8], s);
      s = fma(D[9], QTs[9], s);
      unsafeAtomicAdd(&outS[19], s);
    }
  }
  static constexpr int FLOPS_M2L_PAIR = 437;  // both directions, + one rsqrt
  __device__ __forceinline__ static void l2l(const double* h, double* local) {
    double mh[10];
    mh[0] = 1.0;
    mh[1] = mh[0] * h[0];
    mh[2] = mh[0] * h[1];
    mh[3] = mh[0] * h[2];
    mh[4] = mh[1] * (h[0] * 0.5);
    mh[5] = mh[2] * h[0];
    mh[6] = mh[3] * h[0];
    mh[7] = mh[2] * (h[1] * 0.5);
    mh[8] = mh[3] * h[1];
    mh[9] = mh[3] * (h[2] * 0.5);
    local[0] = fma(local[14], mh[9], fma(local[13], mh[8], fma(local[12], mh[7], fma(local[11], mh[6], fma(local[10], mh[5], fma(local[9], mh[4], fma(local[5], mh[3], fma(local[4], mh[2], fma(local[3], mh[1], local[0])))))))));
    local[1] = fma(local[17], mh[9], fma(local[16], mh[8], fma(local[15], mh[7], fma(local[13], mh[6], fma(local[12], mh[5], fma(local[10], mh[4], fma(local[7], mh[3], fma(local[6], mh[2], fma(local[4], mh[1], local[1])))))))));
    local[2] = fma(local[18], mh[9], fma(local[17], mh[8], fma(local[16], mh[7], fma(local[14], mh[6], fma(local[13], mh[5], fma(local[11], mh[4], fma(local[8], mh[3], fma(local[7], mh[2], fma(local[5], mh[1], local[2])))))))));
    local[3] = fma(local[11], mh[3], fma(local[10], mh[2], fma(local[9], mh[1], local[3])));
    local[4] = fma(local[13], mh[3], fma(local[12], mh[2], fma(local[10], mh[1], local[4])));
    local[5] = fma(local[14], mh[3], fma(local[13], mh[2], fma(local[11], mh[1], local[5])));
    local[6] = fma(local[16], mh[3], fma(local[15], mh[2], fma(local[12], mh[1], local[6])));
    local[7] = fma(local[17], mh[3], fma(local[16], mh[2], fma(local[13], mh[1], local[7])));
    local[8] = fma(local[18], mh[3], fma(local[17], mh[2], fma(local[14], mh[1], local[8])));
    local[9] = local[9];
    local[10] = local[10];
    local[11] = local[11];
    local[12] = local[12];
    local[13] = local[13];
    local[14] = local[14];
    local[15] = local[15];
    local[16] = local[16];
    local[17] = local[17];
    local[18] = local[18];
    local[19] = fma(local[28], mh[9], fma(local[27], mh[8], fma(local[26], mh[7], fma(local[25], mh[6], fma(local[24], mh[5], fma(local[23], mh[4], fma(local[22], mh[3], fma(local[21], mh[2], fma(local[20], mh[1], local[19])))))))));
    local[20] = fma(local[25], mh[3], fma(local[24], mh[2], fma(local[23], mh[1], local[20])));
    local[21] = fma(local[27], mh[3], fma(local[26], mh[2], fma(local[24], mh[1], local[21])));
    local[22] = fma(local[28], mh[3], fma(local[27], mh[2], fma(local[25], mh[1], local[22])));
    local[23] = local[23];
    local[24] = local[24];
    local[25] = local[25];
    local[26] = local[26];
    local[27] = local[27];
    local[28] = local[28];
  }
  static constexpr int FLOPS_L2L = 138;
  __device__ __forceinline__ static void l2p(const double* a, const double* local, double* f, double& phi) {
    double ma[10];
    ma[0] = 1.0;
    ma[1] = ma[0] * a[0];
    ma[2] = ma[0] * a[1];
    ma[3] = ma[0] * a[2];
    ma[4] = ma[1] * (a[0] * 0.5);
    ma[5] = ma[2] * a[0];
    ma[6] = ma[3] * a[0];
    ma[7] = ma[2] * (a[1] * 0.5);
    ma[8] = ma[3] * a[1];
    ma[9] = ma[3] * (a[2] * 0.5);
    f[0] += fma(local[14], ma[9], fma(local[13], ma[8], fma(local[12], ma[7], fma(local[11], ma[6], fma(local[10], ma[5], fma(local[9], ma[4], fma(local[5], ma[3], fma(local[4], ma[2], fma(local[3], ma[1], local[0])))))))));
    f[1] += fma(local[17], ma[9], fma(local[16], ma[8], fma(local[15], ma[7], fma(local[13], ma[6], fma(local[12], ma[5], fma(local[10], ma[4], fma(local[7], ma[3], fma(local[6], ma[2], fma(local[4], ma[1], local[1])))))))));
    f[2] += fma(local[18], ma[9], fma(local[17], ma[8], fma(local[16], ma[7], fma(local[14], ma[6], fma(local[13], ma[5], fma(local[11], ma[4], fma(local[8], ma[3], fma(local[7], ma[2], fma(local[5], ma[1], local[2])))))))));
    phi += fma(local[28], ma[9], fma(local[27], ma[8], fma(local[26], ma[7], fma(local[25], ma[6], fma(local[24], ma[5], fma(local[23], ma[4], fma(local[22], ma[3], fma(local[21], ma[2], fma(local[20], ma[1], local[19])))))))));
  }
  static constexpr int FLOPS_L2P = 88;
};
template <> struct Exp<3> {
  static constexpr int P = 3;
  static constexpr int NQ = 20;   // mass moments, |a| <= P
  static constexpr int NL = 54;   // local coefficients: H then P
  __device__ __forceinline__ static void p2m_add(const double* b, double m, double* Q) {
    double mb[20];
    mb[0] = 1.0;
    mb[1] = mb[0] * b[0];
    mb[2] = mb[0] * b[1];
    mb[3] = mb[0] * b[2];
    mb[4] = mb[1] * (b[0] * 0.5);
    mb[5] = mb[2] * b[0];
    mb[6] = mb[3] * b[0];
    mb[7] = mb[2] * (b[1] * 0.5);
    mb[8] = mb[3] * b[1];
    mb[9] = mb[3] * (b[2] * 0.5);
    mb[10] = mb[4] * (b[0] * 0.3333333333333333);
    mb[11] = mb[5] * (b[0] * 0.5);
    mb[12] = mb[6] * (b[0] * 0.5);
    mb[13] = mb[7] * b[0];
    mb[14] = mb[8] * b[0];
    mb[15] = mb[9] * b[0];
    mb[16] = mb[7] * (b[1] * 0.3333333333333333);
    mb[17] = mb[8] * (b[1] * 0.5);
    mb[18] = mb[9] * b[1];
    mb[19] = mb[9] * (b[2] * 0.3333333333333333);
    Q[0] = fma(m, mb[0], Q[0]);
    Q[1] = fma(m, mb[1], Q[1]);
    Q[2] = fma(m, mb[2], Q[2]);
    Q[3] = fma(m, mb[3], Q[3]);
    Q[4] = fma(m, mb[4], Q[4]);
    Q[5] = fma(m, mb[5], Q[5]);
    Q[6] = fma(m, mb[6], Q[6]);
    Q[7] = fma(m, mb[7], Q[7]);
    Q[8] = fma(m, mb[8], Q[8]);
    Q[9] = fma(m, mb[9], Q[9]);
    Q[10] = fma(m, mb[10], Q[10]);
    Q[11] = fma(m, mb[11], Q[11]);
    Q[12] = fma(m, mb[12], Q[12]);
    Q[13] = fma(m, mb[13], Q[13]);
    Q[14] = fma(m, mb[14], Q[14]);
    Q[15] = fma(m, mb[15], Q[15]);
    Q[16] = fma(m, mb[16], Q[16]);
    Q[17] = fma(m, mb[17], Q[17]);
    Q[18] = fma(m, mb[18], Q[18]);
    Q[19] = fma(m, mb[19], Q[19]);
  }
  static constexpr int FLOPS_P2M = 68;
  __device__ __forceinline__ static void m2m_add(const double* g, const double* Qc, double* Q) {
    double mg[20];
    mg[0] = 1.0;
    mg[1] = mg[0] * g[0];
    mg[2] = mg[0] * g[1];
    mg[3] = mg[0] * g[2];
    mg[4] = mg[1] * (g[0] * 0.5);
    mg[5] = mg[2] * g[0];
    mg[6] = mg[3] * g[0];
    mg[7] = mg[2] * (g[1] * 0.5);
    mg[8] = mg[3] * g[1];
    mg[9] = mg[3] * (g[2] * 0.5);
    mg[10] = mg[4] * (g[0] * 0.3333333333333333);
    mg[11] = mg[5] * (g[0] * 0.5);
    mg[12] = mg[6] * (g[0] * 0.5);
    mg[13] = mg[7] * g[0];
    mg[14] = mg[8] * g[0];
    mg[15] = mg[9] * g[0];
    mg[16] = mg[7] * (g[1] * 0.3333333333333333);
    mg[17] = mg[8] * (g[1] * 0.5);
    mg[18] = mg[9] * g[1];
    mg[19] = mg[9] * (g[2] * 0.3333333333333333);
    Q[0] = (Q[0] + Qc[0]);
    Q[1] = (fma(Qc[0], mg[1], Q[1]) + Qc[1]);
    Q[2] = (fma(Qc[0], mg[2], Q[2]) + Qc[2]);
    Q[3] = (fma(Qc[0], mg[3], Q[3]) + Qc[3]);
    Q[4] = (fma(Qc[1], mg[1], fma(Qc[0], mg[4], Q[4])) + Qc[4]);
    Q[5] = (fma(Qc[2], mg[1], fma(Qc[1], mg[2], fma(Qc[0], mg[5], Q[5]))) + Qc[5]);
    Q[6] = (fma(Qc[3], mg[1], fma(Qc[1], mg[3], fma(Qc[0], mg[6], Q[6]))) + Qc[6]);
    Q[7] = (fma(Qc[2], mg[2], fma(Qc[0], mg[7], Q[7])) + Qc[7]);
    Q[8] = (fma(Qc[3], mg[2], fma(Qc[2], mg[3], fma(Qc[0], mg[8], Q[8]))) + Qc[8]);
    Q[9] = (fma(Qc[3], mg[3], fma(Qc[0], mg[9], Q[9])) + Qc[9]);
    Q[10] = (fma(Qc[4], mg[1], fma(Qc[1], mg[4], fma(Qc[0], mg[10], Q[10]))) + Qc[10]);
    Q[11] = (fma(Qc[5], mg[1], fma(Qc[4], mg[2], fma(Qc[2], mg[4], fma(Qc[1], mg[5], fma(Qc[0], mg[11], Q[11]))))) + Qc[11]);
    Q[12] = (fma(Qc[6], mg[1], fma(Qc[4], mg[3], fma(Qc[3], mg[4], fma(Qc[1], mg[6], fma(Qc[0], mg[12], Q[12]))))) + Qc[12]);
    Q[13] = (fma(Qc[7], mg[1], fma(Qc[5], mg[2], fma(Qc[2], mg[5], fma(Qc[1], mg[7], fma(Qc[0], mg[13], Q[13]))))) + Qc[13]);
    Q[14] = (fma(Qc[8], mg[1], fma(Qc[6], mg[2], fma(Qc[5], mg[3], fma(Qc[3], mg[5], fma(Qc[2], mg[6], fma(Qc[1], mg[8], fma(Qc[0], mg[14], Q[14]))))))) + Qc[14]);
    Q[15] = (fma(Qc[9], mg[1], fma(Qc[6], mg[3], fma(Qc[3], mg[6], fma(Qc[1], mg[9], fma(Qc[0], mg[15], Q[15]))))) + Qc[15]);
    Q[16] = (fma(Qc[7], mg[2], fma(Qc[2], mg[7], fma(Qc[0], mg[16], Q[16]))) + Qc[16]);
    Q[17] = (fma(Qc[8], mg[2], fma(Qc[7], mg[3], fma(Qc[3], mg[7], fma(Qc[2], mg[8], fma(Qc[0], mg[17], Q[17]))))) + Qc[17]);
    Q[18] = (fma(Qc[9], mg[2], fma(Qc[8], mg[3], fma(Qc[3], mg[8], fma(Qc[2], mg[9], fma(Qc[0], mg[18], Q[18]))))) + Qc[18]);
    Q[19] = (fma(Qc[9], mg[3], fma(Qc[3], mg[9], fma(Qc[0], mg[19], Q[19]))) + Qc[19]);
  }
  static constexpr int FLOPS_M2M = 176;
  __device__ __forceinline__ static void m2l_add(const double* r, const double* Q, double* local) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[35];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    const double sn2 = rinv2 * -0.5;
    const double sn3 = rinv2 * -0.3333333333333333;
    const double sn4 = rinv2 * -0.25;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    D[4] = (6.0 * r[0] * D[1] + 2.0 * D[0]) * sn2;
    D[5] = (3.0 * r[0] * D[2] + 3.0 * r[1] * D[1]) * sn2;
    D[6] = (3.0 * r[0] * D[3] + 3.0 * r[2] * D[1]) * sn2;
    D[7] = (6.0 * r[1] * D[2] + 2.0 * D[0]) * sn2;
    D[8] = (3.0 * r[1] * D[3] + 3.0 * r[2] * D[2]) * sn2;
    D[9] = (6.0 * r[2] * D[3] + 2.0 * D[0]) * sn2;
    D[10] = (15.0 * r[0] * D[4] + 12.0 * D[1]) * sn3;
    D[11] = (10.0 * r[0] * D[5] + 4.0 * D[2] + 5.0 * r[1] * D[4]) * sn3;
    D[12] = (10.0 * r[0] * D[6] + 4.0 * D[3] + 5.0 * r[2] * D[4]) * sn3;
    D[13] = (5.0 * r[0] * D[7] + 10.0 * r[1] * D[5] + 4.0 * D[1]) * sn3;
    D[14] = (5.0 * r[0] * D[8] + 5.0 * r[1] * D[6] + 5.0 * r[2] * D[5]) * sn3;
    D[15] = (5.0 * r[0] * D[9] + 10.0 * r[2] * D[6] + 4.0 * D[1]) * sn3;
    D[16] = (15.0 * r[1] * D[7] + 12.0 * D[2]) * sn3;
    D[17] = (10.0 * r[1] * D[8] + 4.0 * D[3] + 5.0 * r[2] * D[7]) * sn3;
    D[18] = (5.0 * r[1] * D[9] + 10.0 * r[2] * D[8] + 4.0 * D[2]) * sn3;
    D[19] = (15.0 * r[2] * D[9] + 12.0 * D[3]) * sn3;
    D[20] = (28.0 * r[0] * D[10] + 36.0 * D[4]) * sn4;
    D[21] = (21.0 * r[0] * D[11] + 18.0 * D[5] + 7.0 * r[1] * D[10]) * sn4;
    D[22] = (21.0 * r[0] * D[12] + 18.0 * D[6] + 7.0 * r[2] * D[10]) * sn4;
    D[23] = (14.0 * r[0] * D[13] + 6.0 * D[7] + 14.0 * r[1] * D[11] + 6.0 * D[4]) * sn4;
    D[24] = (14.0 * r[0] * D[14] + 6.0 * D[8] + 7.0 * r[1] * D[12] + 7.0 * r[2] * D[11]) * sn4;
    D[25] = (14.0 * r[0] * D[15] + 6.0 * D[9] + 14.0 * r[2] * D[12] + 6.0 * D[4]) * sn4;
    D[26] = (7.0 * r[0] * D[16] + 21.0 * r[1] * D[13] + 18.0 * D[5]) * sn4;
    D[27] = (7.0 * r[0] * D[17] + 14.0 * r[1] * D[14] + 6.0 * D[6] + 7.0 * r[2] * D[13]) * sn4;
    D[28] = (7.0 * r[0] * D[18] + 7.0 * r[1] * D[15] + 14.0 * r[2] * D[14] + 6.0 * D[5]) * sn4;
    D[29] = (7.0 * r[0] * D[19] + 21.0 * r[2] * D[15] + 18.0 * D[6]) * sn4;
    D[30] = (28.0 * r[1] * D[16] + 36.0 * D[7]) * sn4;
    D[31] = (21.0 * r[1] * D[17] + 18.0 * D[8] + 7.0 * r[2] * D[16]) * sn4;
    D[32] = (14.0 * r[1] * D[18] + 6.0 * D[9] + 14.0 * r[2] * D[17] + 6.0 * D[7]) * sn4;
    D[33] = (7.0 * r[1] * D[19] + 21.0 * r[2] * D[18] + 18.0 * D[8]) * sn4;
    D[34] = (28.0 * r[2] * D[19] + 36.0 * D[9]) * sn4;
    {
      double s = D[1] * Q[0];
      s = fma(D[4], Q[1], s);
      s = fma(D[5], Q[2], s);
      s = fma(D[6], Q[3], s);
      s = fma(D[10], Q[4], s);
      s = fma(D[11], Q[5], s);
      s = fma(D[12], Q[6], s);
      s = fma(D[13], Q[7], s);
      s = fma(D[14], Q[8], s);
      s = fma(D[15], Q[9], s);
      local[35] -= s;
      s = fma(D[20], Q[10], s);
      s = fma(D[21], Q[11], s);
      s = fma(D[22], Q[12], s);
      s = fma(D[23], Q[13], s);
      s = fma(D[24], Q[14], s);
      s = fma(D[25], Q[15], s);
      s = fma(D[26], Q[16], s);
      s = fma(D[27], Q[17], s);
      s = fma(D[28], Q[18], s);
      s = fma(D[29], Q[19], s);
      local[0] += s;
    }
    {
      double s = D[2] * Q[0];
      s = fma(D[5], Q[1], s);
      s = fma(D[7], Q[2], s);
      s = fma(D[8], Q[3], s);
      s = fma(D[11], Q[4], s);
      s = fma(D[13], Q[5], s);
      s = fma(D[14], Q[6], s);
      s = fma(D[16], Q[7], s);
      s = fma(D[17], Q[8], s);
      s = fma(D[18], Q[9], s);
      local[36] -= s;
      s = fma(D[21], Q[10], s);
      s = fma(D[23], Q[11], s);
      s = fma(D[24], Q[12], s);
      s = fma(D[26], Q[13], s);
      s = fma(D[27], Q[14], s);
      s = fma(D[28], Q[15], s);
      s = fma(D[30], Q[16], s);
      s = fma(D[31], Q[17], s);
      s = fma(D[32], Q[18], s);
      s = fma(D[33], Q[19], s);
      local[1] += s;
    }
    {
      double s = D[3] * Q[0];
      s = fma(D[6], Q[1], s);
      s = fma(D[8], Q[2], s);
      s = fma(D[9], Q[3], s);
      s = fma(D[12], Q[4], s);
      s = fma(D[14], Q[5], s);
      s = fma(D[15], Q[6], s);
      s = fma(D[17], Q[7], s);
      s = fma(D[18], Q[8], s);
      s = fma(D[19], Q[9], s);
      local[37] -= s;
      s = fma(D[22], Q[10], s);
      s = fma(D[24], Q[11], s);
      s = fma(D[25], Q[12], s);
      s = fma(D[27], Q[13], s);
      s = fma(D[28], Q[14], s);
      s = fma(D[29], Q[15], s);
      s = fma(D[31], Q[16], s);
      s = fma(D[32], Q[17], s);
      s = fma(D[33], Q[18], s);
      s = fma(D[34], Q[19], s);
      local[2] += s;
    }
    {
      double s = D[4] * Q[0];
      s = fma(D[10], Q[1], s);
      s = fma(D[11], Q[2], s);
      s = fma(D[12], Q[3], s);
      local[38] += s;
      s = fma(D[20], Q[4], s);
      s = fma(D[21], Q[5], s);
      s = fma(D[22], Q[6], s);
      s = fma(D[23], Q[7], s);
      s = fma(D[24], Q[8], s);
      s = fma(D[25], Q[9], s);
      local[3] -= s;
    }
    {
      double s = D[5] * Q[0];
      s = fma(D[11], Q[1], s);
      s = fma(D[13], Q[2], s);
      s = fma(D[14], Q[3], s);
      local[39] += s;
      s = fma(D[21], Q[4], s);
      s = fma(D[23], Q[5], s);
      s = fma(D[24], Q[6], s);
      s = fma(D[26], Q[7], s);
      s = fma(D[27], Q[8], s);
      s = fma(D[28], Q[9], s);
      local[4] -= s;
    }
    {
      double s = D[6] * Q[0];
      s = fma(D[12], Q[1], s);
      s = fma(D[14], Q[2], s);
      s = fma(D[15], Q[3], s);
      local[40] += s;
      s = fma(D[22], Q[4], s);
      s = fma(D[24], Q[5], s);
      s = fma(D[25], Q[6], s);
      s = fma(D[27], Q[7], s);
      s = fma(D[28], Q[8], s);
      s = fma(D[29], Q[9], s);
      local[5] -= s;
    }
    {
      double s = D[7] * Q[0];
      s = fma(D[13], Q[1], s);
      s = fma(D[16], Q[2], s);
      s = fma(D[17], Q[3], s);
      local[41] += s;
      s = fma(D[23], Q[4], s);
      s = fma(D[26], Q[5], s);
      s = fma(D[27], Q[6], s);
      s = fma(D[30], Q[7], s);
      s = fma(D[31], Q[8], s);
      s = fma(D[32], Q[9], s);
      local[6] -= s;
    }
    {
      double s = D[8] * Q[0];
      s = fma(D[14], Q[1], s);
      s = fma(D[17], Q[2], s);
      s = fma(D[18], Q[3], s);
      local[42] += s;
      s = fma(D[24], Q[4], s);
      s = fma(D[27], Q[5], s);
      s = fma(D[28], Q[6], s);
      s = fma(D[31], Q[7], s);
      s = fma(D[32], Q[8], s);
      s = fma(D[33], Q[9], s);
      local[7] -= s;
    }
    {
      double s = D[9] * Q[0];
      s = fma(D[15], Q[1], s);
      s = fma(D[18], Q[2], s);
      s = fma(D[19], Q[3], s);
      local[43] += s;
      s = fma(D[25], Q[4], s);
      s = fma(D[28], Q[5], s);
      s = fma(D[29], Q[6], s);
      s = fma(D[32], Q[7], s);
      s = fma(D[33], Q[8], s);
      s = fma(D[34], Q[9], s);
      local[8] -= s;
    }
    {
      double s = D[10] * Q[0];
      local[44] -= s;
      s = fma(D[20], Q[1], s);
      s = fma(D[21], Q[2], s);
      s = fma(D[22], Q[3], s);
      local[9] += s;
    }
    {
      double s = D[11] * Q[0];
      local[45] -= s;
      s = fma(D[21], Q[1], s);
      s = fma(D[23], Q[2], s);
      s = fma(D[24], Q[3], s);
      local[10] += s;
    }
    {
      double s = D[12] * Q[0];
      local[46] -= s;
      s = fma(D[22], Q[1], s);
      s = fma(D[24], Q[2], s);
      s = fma(D[25], Q[3], s);
      local[11] += s;
    }
    {
      double s = D[13] * Q[0];
      local[47] -= s;
      s = fma(D[23], Q[1], s);
      s = fma(D[26], Q[2], s);
      s = fma(D[27], Q[3], s);
      local[12] += s;
    }
    {
      double s = D[14] * Q[0];
      local[48] -= s;
      s = fma(D[24], Q[1], s);
      s = fma(D[27], Q[2], s);
      s = fma(D[28], Q[3], s);
      local[13] += s;
    }
    {
      double s = D[15] * Q[0];
      local[49] -= s;
      s = fma(D[25], Q[1], s);
      s = fma(D[28], Q[2], s);
      s = fma(D[29], Q[3], s);
      local[14] += s;
    }
    {
      double s = D[16] * Q[0];
      local[50] -= s;
      s = fma(D[26], Q[1], s);
      s = fma(D[30], Q[2], s);
      s = fma(D[31], Q[3], s);
      local[15] += s;
    }
    {
      double s = D[17] * Q[0];
      local[51] -= s;
      s = fma(D[27], Q[1], s);
      s = fma(D[31], Q[2], s);
      s = fma(D[32], Q[3], s);
      local[16] += s;
    }
    {
      double s = D[18] * Q[0];
      local[52] -= s;
      s = fma(D[28], Q[1], s);
      s = fma(D[32], Q[2], s);
      s = fma(D[33], Q[3], s);
      local[17] += s;
    }
    {
      double s = D[19] * Q[0];
      local[53] -= s;
      s = fma(D[29], Q[1], s);
      s = fma(D[33], Q[2], s);
      s = fma(D[34], Q[3], s);
      local[18] += s;
    }
    {
      double s = D[20] * Q[0];
      local[19] -= s;
    }
    {
      double s = D[21] * Q[0];
      local[20] -= s;
    }
    {
      double s = D[22] * Q[0];
      local[21] -= s;
    }
    {
      double s = D[23] * Q[0];
      local[22] -= s;
    }
    {
      double s = D[24] * Q[0];
      local[23] -= s;
    }
    {
      double s = D[25] * Q[0];
      local[24] -= s;
    }
    {
      double s = D[26] * Q[0];
      local[25] -= s;
    }
    {
      double s = D[27] * Q[0];
      local[26] -= s;
    }
    {
      double s = D[28] * Q[0];
      local[27] -= s;
    }
    {
      double s = D[29] * Q[0];
      local[28] -= s;
    }
    {
      double s = D[30] * Q[0];
      local[29] -= s;
    }
    {
      double s = D[31] * Q[0];
      local[30] -= s;
    }
    {
      double s = D[32] * Q[0];
      local[31] -= s;
    }
    {
      double s = D[33] * Q[0];
      local[32] -= s;
    }
    {
      double s = D[34] * Q[0];
      local[33] -= s;
    }
    {
      double s = D[0] * Q[0];
      s = fma(D[1], Q[1], s);
      s = fma(D[2], Q[2], s);
      s = fma(D[3], Q[3], s);
      s = fma(D[4], Q[4], s);
      s = fma(D[5], Q[5], s);
      s = fma(D[6], Q[6], s);
      s = fma(D[7], Q[7], s);
      s = fma(D[8], Q[8], s);
      s = fma(D[9], Q[9], s);
      s = fma(D[10], Q[10], s);
      s = fma(D[11], Q[11], s);
      s = fma(D[12], Q[12], s);
      s = fma(D[13], Q[13], s);
      s = fma(D[14], Q[14], s);
      s = fma(D[15], Q[15], s);
      s = fma(D[16], Q[16], s);
      s = fma(D[17], Q[17], s);
      s = fma(D[18], Q[18], s);
      s = fma(D[19], Q[19], s);
      local[34] += s;
    }
  }
  static constexpr int FLOPS_M2L = 659;  // + one rsqrt
  __device__ __forceinline__ static void m2l_add_f32(const float* r, const float* Q, double* local, bool ok = true) {
    const float r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const float rinv = ok ? __frsqrt_rn(r2) : 0.0f;
    const float rinv2 = rinv * rinv;
    float D[35];
    D[0] = rinv;
    const float sn1 = rinv2 * -1.0f;
    const float sn2 = rinv2 * -0.5f;
    const float sn3 = rinv2 * -0.3333333333333333f;
    const float sn4 = rinv2 * -0.25f;
    D[1] = (1.0f * r[0] * D[0]) * sn1;
    D[2] = (1.0f * r[1] * D[0]) * sn1;
    D[3] = (1.0f * r[2] * D[0]) * sn1;
    D[4] = (6.0f * r[0] * D[1] + 2.0f * D[0]) * sn2;
    D[5] = (3.0f * r[0] * D[2] + 3.0f * r[1] * D[1]) * sn2;
    D[6] = (3.0f * r[0] * D[3] + 3.0f * r[2] * D[1]) * sn2;
    D[7] = (6.0f * r[1] * D[2] + 2.0f * D[0]) * sn2;
    D[8] = (3.0f * r[1] * D[3] + 3.0f * r[2] * D[2]) * sn2;
    D[9] = (6.0f * r[2] * D[3] + 2.0f * D[0]) * sn2;
    D[10] = (15.0f * r[0] * D[4] + 12.0f * D[1]) * sn3;
    D[11] = (10.0f * r[0] * D[5] + 4.0f * D[2] + 5.0f * r[1] * D[4]) * sn3;
    D[12] = (10.0f * r[0] * D[6] + 4.0f * D[3] + 5.0f * r[2] * D[4]) * sn3;
    D[13] = (5.0f * r[0] * D[7] + 10.0f * r[1] * D[5] + 4.0f * D[1]) * sn3;
    D[14] = (5.0f * r[0] * D[8] + 5.0f * r[1] * D[6] + 5.0f * r[2] * D[5]) * sn3;
    D[15] = (5.0f * r[0] * D[9] + 10.0f * r[2] * D[6] + 4.0f * D[1]) * sn3;
    D[16] = (15.0f * r[1] * D[7] + 12.0f * D[2]) * sn3;
    D[17] = (10.0f * r[1] * D[8] + 4.0f * D[3] + 5.0f * r[2] * D[7]) * sn3;
    D[18] = (5.0f * r[1] * D[9] + 10.0f * r[2] * D[8] + 4.0f * D[2]) * sn3;
    D[19] = (15.0f * r[2] * D[9] + 12.0f * D[3]) * sn3;
    D[20] = (28.0f * r[0] * D[10] + 36.0f * D[4]) * sn4;
    D[21] = (21.0f * r[0] * D[11] + 18.0f * D[5] + 7.0f * r[1] * D[10]) * sn4;
    D[22] = (21.0f * r[0] * D[12] + 18.0f * D[6] + 7.0f * r[2] * D[10]) * sn4;
    D[23] = (14.0f * r[0] * D[13] + 6.0f * D[7] + 14.0f * r[1] * D[11] + 6.0f * D[4]) * sn4;
    D[24] = (14.0f * r[0] * D[14] + 6.0f * D[8] + 7.0f * r[1] * D[12] + 7.0f * r[2] * D[11]) * sn4;
    D[25] = (14.0f * r[0] * D[15] + 6.0f * D[9] + 14.0f * r[2] * D[12] + 6.0f * D[4]) * sn4;
    D[26] = (7.0f * r[0] * D[16] + 21.0f * r[1] * D[13] + 18.0f * D[5]) * sn4;
    D[27] = (7.0f * r[0] * D[17] + 14.0f * r[1] * D[14] + 6.0f * D[6] + 7.0f * r[2] * D[13]) * sn4;
    D[28] = (7.0f * r[0] * D[18] + 7.0f * r[1] * D[15] + 14.0f * r[2] * D[14] + 6.0f * D[5]) * sn4;
    D[29] = (7.0f * r[0] * D[19] + 21.0f * r[2] * D[15] + 18.0f * D[6]) * sn4;
    D[30] = (28.0f * r[1] * D[16] + 36.0f * D[7]) * sn4;
    D[31] = (21.0f * r[1] * D[17] + 18.0f * D[8] + 7.0f * r[2] * D[16]) * sn4;
    D[32] = (14.0f * r[1] * D[18] + 6.0f * D[9] + 14.0f * r[2] * D[17] + 6.0f * D[7]) * sn4;
    D[33] = (7.0f * r[1] * D[19] + 21.0f * r[2] * D[18] + 18.0f * D[8]) * sn4;
    D[34] = (28.0f * r[2] * D[19] + 36.0f * D[9]) * sn4;
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[1] * Q[0];
      s = fmaf(D[4], Q[1], s);
      s = fmaf(D[5], Q[2], s);
      s = fmaf(D[6], Q[3], s);
      s = fmaf(D[10], Q[4], s);
      s = fmaf(D[11], Q[5], s);
      s = fmaf(D[12], Q[6], s);
      s = fmaf(D[13], Q[7], s);
      s = fmaf(D[14], Q[8], s);
      s = fmaf(D[15], Q[9], s);
      local[35] -= (double)s;
      s = fmaf(D[20], Q[10], s);
      s = fmaf(D[21], Q[11], s);
      s = fmaf(D[22], Q[12], s);
      s = fmaf(D[23], Q[13], s);
      s = fmaf(D[24], Q[14], s);
      s = fmaf(D[25], Q[15], s);
      s = fmaf(D[26], Q[16], s);
      s = fmaf(D[27], Q[17], s);
      s = fmaf(D[28], Q[18], s);
      s = fmaf(D[29], Q[19], s);
      local[0] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[2] * Q[0];
      s = fmaf(D[5], Q[1], s);
      s = fmaf(D[7], Q[2], s);
      s = fmaf(D[8], Q[3], s);
      s = fmaf(D[11], Q[4], s);
      s = fmaf(D[13], Q[5], s);
      s = fmaf(D[14], Q[6], s);
      s = fmaf(D[16], Q[7], s);
      s = fmaf(D[17], Q[8], s);
      s = fmaf(D[18], Q[9], s);
      local[36] -= (double)s;
      s = fmaf(D[21], Q[10], s);
      s = fmaf(D[23], Q[11], s);
      s = fmaf(D[24], Q[12], s);
      s = fmaf(D[26], Q[13], s);
      s = fmaf(D[27], Q[14], s);
      s = fmaf(D[28], Q[15], s);
      s = fmaf(D[30], Q[16], s);
      s = fmaf(D[31], Q[17], s);
      s = fmaf(D[32], Q[18], s);
      s = fmaf(D[33], Q[19], s);
      local[1] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[3] * Q[0];
      s = fmaf(D[6], Q[1], s);
      s = fmaf(D[8], Q[2], s);
      s = fmaf(D[9], Q[3], s);
      s = fmaf(D[12], Q[4], s);
      s = fmaf(D[14], Q[5], s);
      s = fmaf(D[15], Q[6], s);
      s = fmaf(D[17], Q[7], s);
      s = fmaf(D[18], Q[8], s);
      s = fmaf(D[19], Q[9], s);
      local[37] -= (double)s;
      s = fmaf(D[22], Q[10], s);
      s = fmaf(D[24], Q[11], s);
      s = fmaf(D[25], Q[12], s);
      s = fmaf(D[27], Q[13], s);
      s = fmaf(D[28], Q[14], s);
      s = fmaf(D[29], Q[15], s);
      s = fmaf(D[31], Q[16], s);
      s = fmaf(D[32], Q[17], s);
      s = fmaf(D[33], Q[18], s);
      s = fmaf(D[34], Q[19], s);
      local[2] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[4] * Q[0];
      s = fmaf(D[10], Q[1], s);
      s = fmaf(D[11], Q[2], s);
      s = fmaf(D[12], Q[3], s);
      local[38] += (double)s;
      s = fmaf(D[20], Q[4], s);
      s = fmaf(D[21], Q[5], s);
      s = fmaf(D[22], Q[6], s);
      s = fmaf(D[23], Q[7], s);
      s = fmaf(D[24], Q[8], s);
      s = fmaf(D[25], Q[9], s);
      local[3] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[5] * Q[0];
      s = fmaf(D[11], Q[1], s);
      s = fmaf(D[13], Q[2], s);
      s = fmaf(D[14], Q[3], s);
      local[39] += (double)s;
      s = fmaf(D[21], Q[4], s);
      s = fmaf(D[23], Q[5], s);
      s = fmaf(D[24], Q[6], s);
      s = fmaf(D[26], Q[7], s);
      s = fmaf(D[27], Q[8], s);
      s = fmaf(D[28], Q[9], s);
      local[4] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[6] * Q[0];
      s = fmaf(D[12], Q[1], s);
      s = fmaf(D[14], Q[2], s);
      s = fmaf(D[15], Q[3], s);
      local[40] += (double)s;
      s = fmaf(D[22], Q[4], s);
      s = fmaf(D[24], Q[5], s);
      s = fmaf(D[25], Q[6], s);
      s = fmaf(D[27], Q[7], s);
      s = fmaf(D[28], Q[8], s);
      s = fmaf(D[29], Q[9], s);
      local[5] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[7] * Q[0];
      s = fmaf(D[13], Q[1], s);
      s = fmaf(D[16], Q[2], s);
      s = fmaf(D[17], Q[3], s);
      local[41] += (double)s;
      s = fmaf(D[23], Q[4], s);
      s = fmaf(D[26], Q[5], s);
      s = fmaf(D[27], Q[6], s);
      s = fmaf(D[30], Q[7], s);
      s = fmaf(D[31], Q[8], s);
      s = fmaf(D[32], Q[9], s);
      local[6] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[8] * Q[0];
      s = fmaf(D[14], Q[1], s);
      s = fmaf(D[17], Q[2], s);
      s = fmaf(D[18], Q[3], s);
      local[42] += (double)s;
      s = fmaf(D[24], Q[4], s);
      s = fmaf(D[27], Q[5], s);
      s = fmaf(D[28], Q[6], s);
      s = fmaf(D[31], Q[7], s);
      s = fmaf(D[32], Q[8], s);
      s = fmaf(D[33], Q[9], s);
      local[7] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[9] * Q[0];
      s = fmaf(D[15], Q[1], s);
      s = fmaf(D[18], Q[2], s);
      s = fmaf(D[19], Q[3], s);
      local[43] += (double)s;
      s = fmaf(D[25], Q[4], s);
      s = fmaf(D[28], Q[5], s);
      s = fmaf(D[29], Q[6], s);
      s = fmaf(D[32], Q[7], s);
      s = fmaf(D[33], Q[8], s);
      s = fmaf(D[34], Q[9], s);
      local[8] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[10] * Q[0];
      local[44] -= (double)s;
      s = fmaf(D[20], Q[1], s);
      s = fmaf(D[21], Q[2], s);
      s = fmaf(D[22], Q[3], s);
      local[9] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[11] * Q[0];
      local[45] -= (double)s;
      s = fmaf(D[21], Q[1], s);
      s = fmaf(D[23], Q[2], s);
      s = fmaf(D[24], Q[3], s);
      local[10] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[12] * Q[0];
      local[46] -= (double)s;
      s = fmaf(D[22], Q[1], s);
      s = fmaf(D[24], Q[2], s);
      s = fmaf(D[25], Q[3], s);
      local[11] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[13] * Q[0];
      local[47] -= (double)s;
      s = fmaf(D[23], Q[1], s);
      s = fmaf(D[26], Q[2], s);
      s = fmaf(D[27], Q[3], s);
      local[12] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[14] * Q[0];
      local[48] -= (double)s;
      s = fmaf(D[24], Q[1], s);
      s = fmaf(D[27], Q[2], s);
      s = fmaf(D[28], Q[3], s);
      local[13] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[15] * Q[0];
      local[49] -= (double)s;
      s = fmaf(D[25], Q[1], s);
      s = fmaf(D[28], Q[2], s);
      s = fmaf(D[29], Q[3], s);
      local[14] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[16] * Q[0];
      local[50] -= (double)s;
      s = fmaf(D[26], Q[1], s);
      s = fmaf(D[30], Q[2], s);
      s = fmaf(D[31], Q[3], s);
      local[15] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[17] * Q[0];
      local[51] -= (double)s;
      s = fmaf(D[27], Q[1], s);
      s = fmaf(D[31], Q[2], s);
      s = fmaf(D[32], Q[3], s);
      local[16] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[18] * Q[0];
      local[52] -= (double)s;
      s = fmaf(D[28], Q[1], s);
      s = fmaf(D[32], Q[2], s);
      s = fmaf(D[33], Q[3], s);
      local[17] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[19] * Q[0];
      local[53] -= (double)s;
      s = fmaf(D[29], Q[1], s);
      s = fmaf(D[33], Q[2], s);
      s = fmaf(D[34], Q[3], s);
      local[18] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[20] * Q[0];
      local[19] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[21] * Q[0];
      local[20] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[22] * Q[0];
      local[21] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[23] * Q[0];
      local[22] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[24] * Q[0];
      local[23] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[25] * Q[0];
      local[24] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[26] * Q[0];
      local[25] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[27] * Q[0];
      local[26] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[28] * Q[0];
      local[27] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[29] * Q[0];
      local[28] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[30] * Q[0];
      local[29] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[31] * Q[0];
      local[30] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[32] * Q[0];
      local[31] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[33] * Q[0];
      local[32] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[34] * Q[0];
      local[33] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[0] * Q[0];
      s = fmaf(D[1], Q[1], s);
      s = fmaf(D[2], Q[2], s);
      s = fmaf(D[3], Q[3], s);
      s = fmaf(D[4], Q[4], s);
      s = fmaf(D[5], Q[5], s);
      s = fmaf(D[6], Q[6], s);
      s = fmaf(D[7], Q[7], s);
      s = fmaf(D[8], Q[8], s);
      s = fmaf(D[9], Q[9], s);
      s = fmaf(D[10], Q[10], s);
      s = fmaf(D[11], Q[11], s);
      s = fmaf(D[12], Q[12], s);
      s = fmaf(D[13], Q[13], s);
      s = fmaf(D[14], Q[14], s);
      s = fmaf(D[15], Q[15], s);
      s = fmaf(D[16], Q[16], s);
      s = fmaf(D[17], Q[17], s);
      s = fmaf(D[18], Q[18], s);
      s = fmaf(D[19], Q[19], s);
      local[34] += (double)s;
    }
  }
  static constexpr int NQR = 16;   // independent moments
  static constexpr int NLR = 40;  // S then X
  __device__ __forceinline__ static void reduce(const double* Q, double* Qr) {
    Qr[0] = Q[0];
    Qr[1] = Q[1];
    Qr[2] = Q[2];
    Qr[3] = Q[3];
    Qr[4] = Q[4] - Q[9];
    Qr[5] = Q[5];
    Qr[6] = Q[6];
    Qr[7] = Q[7] - Q[9];
    Qr[8] = Q[8];
    Qr[9] = Q[10] - Q[15];
    Qr[10] = Q[11] - Q[18];
    Qr[11] = Q[12] - Q[19];
    Qr[12] = Q[13] - Q[15];
    Qr[13] = Q[14];
    Qr[14] = Q[16] - Q[18];
    Qr[15] = Q[17] - Q[19];
  }
  __device__ __forceinline__ static void m2l_h(const double* r, const double* Qr, double* lr, bool ok) {
    const double r2 = fma(r[0], r[0], fma(r[1], r[1], r[2] * r[2]));
    const double ri = rsqrt_refined(r2);
    const double rinv = ok && r2 < __builtin_inf() ? ri : 0.0;
    const double s = rinv * rinv;
    const double w[3] = {r[0] * s, r[1] * s, r[2] * s};
    const double R0_000 = rinv;
    const double R1_000 = -1.0 * rinv;
    const double R2_000 = 3.0 * rinv;
    const double R3_000 = -15.0 * rinv;
    const double R4_000 = 105.0 * rinv;
    lr[0] = fma(R0_000, Qr[0], lr[0]);
    const double R0_100 = w[0] * R1_000;
    lr[0] = fma(R0_100, Qr[1], lr[0]);
    lr[1] = fma(R0_100, Qr[0], lr[1]);
    const double R0_010 = w[1] * R1_000;
    lr[0] = fma(R0_010, Qr[2], lr[0]);
    lr[2] = fma(R0_010, Qr[0], lr[2]);
    const double R0_001 = w[2] * R1_000;
    lr[0] = fma(R0_001, Qr[3], lr[0]);
    lr[3] = fma(R0_001, Qr[0], lr[3]);
    const double R1_100 = w[0] * R2_000;
    const double T1_000 = s * R1_000;
    const double R0_200 = fma(w[0], R1_100, T1_000);
    lr[0] = fma(R0_200, Qr[4], lr[0]);
    lr[1] = fma(R0_200, Qr[1], lr[1]);
    lr[4] = fma(R0_200, Qr[0], lr[4]);
    const double R1_010 = w[1] * R2_000;
    const double R0_110 = w[0] * R1_010;
    lr[0] = fma(R0_110, Qr[5], lr[0]);
    lr[1] = fma(R0_110, Qr[2], lr[1]);
    lr[2] = fma(R0_110, Qr[1], lr[2]);
    lr[5] = fma(R0_110, Qr[0], lr[5]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_101 = w[2] * R1_100;
    lr[0] = fma(R0_101, Qr[6], lr[0]);
    lr[1] = fma(R0_101, Qr[3], lr[1]);
    lr[3] = fma(R0_101, Qr[1], lr[3]);
    lr[6] = fma(R0_101, Qr[0], lr[6]);
    const double R0_020 = fma(w[1], R1_010, T1_000);
    lr[0] = fma(R0_020, Qr[7], lr[0]);
    lr[2] = fma(R0_020, Qr[2], lr[2]);
    lr[7] = fma(R0_020, Qr[0], lr[7]);
    const double R0_011 = w[2] * R1_010;
    lr[0] = fma(R0_011, Qr[8], lr[0]);
    lr[2] = fma(R0_011, Qr[3], lr[2]);
    lr[3] = fma(R0_011, Qr[2], lr[3]);
    lr[8] = fma(R0_011, Qr[0], lr[8]);
    const double R0_002 = -(R0_200 + R0_020);
    lr[3] = fma(R0_002, Qr[3], lr[3]);
    __builtin_amdgcn_sched_barrier(0);
    const double R2_100 = w[0] * R3_000;
    const double T2_000 = s * R2_000;
    const double R1_200 = fma(w[0], R2_100, T2_000);
    const double T1_100 = s * R1_100;
    const double R0_300 = fma(w[0], R1_200, 2.0 * T1_100);
    lr[0] = fma(R0_300, Qr[9], lr[0]);
    lr[1] = fma(R0_300, Qr[4], lr[1]);
    lr[4] = fma(R0_300, Qr[1], lr[4]);
    lr[9] = fma(R0_300, Qr[0], lr[9]);
    const double R2_010 = w[1] * R3_000;
    const double R1_110 = w[0] * R2_010;
    const double T1_010 = s * R1_010;
    const double R0_210 = fma(w[0], R1_110, T1_010);
    lr[0] = fma(R0_210, Qr[10], lr[0]);
    lr[1] = fma(R0_210, Qr[5], lr[1]);
    lr[2] = fma(R0_210, Qr[4], lr[2]);
    lr[4] = fma(R0_210, Qr[2], lr[4]);
    lr[5] = fma(R0_210, Qr[1], lr[5]);
    lr[10] = fma(R0_210, Qr[0], lr[10]);
    const double R0_201 = w[2] * R1_200;
    lr[0] = fma(R0_201, Qr[11], lr[0]);
    lr[1] = fma(R0_201, Qr[6], lr[1]);
    lr[3] = fma(R0_201, Qr[4], lr[3]);
    lr[4] = fma(R0_201, Qr[3], lr[4]);
    lr[6] = fma(R0_201, Qr[1], lr[6]);
    lr[11] = fma(R0_201, Qr[0], lr[11]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_120 = fma(w[1], R1_110, T1_100);
    lr[0] = fma(R0_120, Qr[12], lr[0]);
    lr[1] = fma(R0_120, Qr[7], lr[1]);
    lr[2] = fma(R0_120, Qr[5], lr[2]);
    lr[5] = fma(R0_120, Qr[2], lr[5]);
    lr[7] = fma(R0_120, Qr[1], lr[7]);
    lr[12] = fma(R0_120, Qr[0], lr[12]);
    const double R0_111 = w[2] * R1_110;
    lr[0] = fma(R0_111, Qr[13], lr[0]);
    lr[1] = fma(R0_111, Qr[8], lr[1]);
    lr[2] = fma(R0_111, Qr[6], lr[2]);
    lr[3] = fma(R0_111, Qr[5], lr[3]);
    lr[5] = fma(R0_111, Qr[3], lr[5]);
    lr[6] = fma(R0_111, Qr[2], lr[6]);
    lr[8] = fma(R0_111, Qr[1], lr[8]);
    lr[13] = fma(R0_111, Qr[0], lr[13]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_102 = -(R0_300 + R0_120);
    lr[3] = fma(R0_102, Qr[6], lr[3]);
    lr[6] = fma(R0_102, Qr[3], lr[6]);
    const double R1_020 = fma(w[1], R2_010, T2_000);
    const double R0_030 = fma(w[1], R1_020, 2.0 * T1_010);
    lr[0] = fma(R0_030, Qr[14], lr[0]);
    lr[2] = fma(R0_030, Qr[7], lr[2]);
    lr[7] = fma(R0_030, Qr[2], lr[7]);
    lr[14] = fma(R0_030, Qr[0], lr[14]);
    const double R0_021 = w[2] * R1_020;
    lr[0] = fma(R0_021, Qr[15], lr[0]);
    lr[2] = fma(R0_021, Qr[8], lr[2]);
    lr[3] = fma(R0_021, Qr[7], lr[3]);
    lr[7] = fma(R0_021, Qr[3], lr[7]);
    lr[8] = fma(R0_021, Qr[2], lr[8]);
    lr[15] = fma(R0_021, Qr[0], lr[15]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_012 = -(R0_210 + R0_030);
    lr[3] = fma(R0_012, Qr[8], lr[3]);
    lr[8] = fma(R0_012, Qr[3], lr[8]);
    const double R3_100 = w[0] * R4_000;
    const double T3_000 = s * R3_000;
    const double R2_200 = fma(w[0], R3_100, T3_000);
    const double T2_100 = s * R2_100;
    const double R1_300 = fma(w[0], R2_200, 2.0 * T2_100);
    const double T1_200 = s * R1_200;
    const double R0_400 = fma(w[0], R1_300, 3.0 * T1_200);
    lr[16] = fma(R0_400, Qr[9], lr[16]);
    lr[19] = fma(R0_400, Qr[4], lr[19]);
    lr[24] = fma(R0_400, Qr[1], lr[24]);
    lr[31] = fma(R0_400, Qr[0], lr[31]);
    const double R3_010 = w[1] * R4_000;
    const double R2_110 = w[0] * R3_010;
    const double T2_010 = s * R2_010;
    const double R1_210 = fma(w[0], R2_110, T2_010);
    const double T1_110 = s * R1_110;
    const double R0_310 = fma(w[0], R1_210, 2.0 * T1_110);
    lr[16] = fma(R0_310, Qr[10], lr[16]);
    lr[17] = fma(R0_310, Qr[9], lr[17]);
    lr[19] = fma(R0_310, Qr[5], lr[19]);
    lr[20] = fma(R0_310, Qr[4], lr[20]);
    lr[24] = fma(R0_310, Qr[2], lr[24]);
    lr[25] = fma(R0_310, Qr[1], lr[25]);
    lr[32] = fma(R0_310, Qr[0], lr[32]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_301 = w[2] * R1_300;
    lr[16] = fma(R0_301, Qr[11], lr[16]);
    lr[18] = fma(R0_301, Qr[9], lr[18]);
    lr[19] = fma(R0_301, Qr[6], lr[19]);
    lr[21] = fma(R0_301, Qr[4], lr[21]);
    lr[24] = fma(R0_301, Qr[3], lr[24]);
    lr[26] = fma(R0_301, Qr[1], lr[26]);
    lr[33] = fma(R0_301, Qr[0], lr[33]);
    const double R1_120 = fma(w[1], R2_110, T2_100);
    const double T1_020 = s * R1_020;
    const double R0_220 = fma(w[0], R1_120, T1_020);
    lr[16] = fma(R0_220, Qr[12], lr[16]);
    lr[17] = fma(R0_220, Qr[10], lr[17]);
    lr[19] = fma(R0_220, Qr[7], lr[19]);
    lr[20] = fma(R0_220, Qr[5], lr[20]);
    lr[22] = fma(R0_220, Qr[4], lr[22]);
    lr[25] = fma(R0_220, Qr[2], lr[25]);
    lr[27] = fma(R0_220, Qr[1], lr[27]);
    lr[34] = fma(R0_220, Qr[0], lr[34]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_211 = w[2] * R1_210;
    lr[16] = fma(R0_211, Qr[13], lr[16]);
    lr[17] = fma(R0_211, Qr[11], lr[17]);
    lr[18] = fma(R0_211, Qr[10], lr[18]);
    lr[19] = fma(R0_211, Qr[8], lr[19]);
    lr[20] = fma(R0_211, Qr[6], lr[20]);
    lr[21] = fma(R0_211, Qr[5], lr[21]);
    lr[23] = fma(R0_211, Qr[4], lr[23]);
    lr[25] = fma(R0_211, Qr[3], lr[25]);
    lr[26] = fma(R0_211, Qr[2], lr[26]);
    lr[28] = fma(R0_211, Qr[1], lr[28]);
    lr[35] = fma(R0_211, Qr[0], lr[35]);
    const double R0_202 = -(R0_400 + R0_220);
    lr[18] = fma(R0_202, Qr[11], lr[18]);
    lr[21] = fma(R0_202, Qr[6], lr[21]);
    lr[26] = fma(R0_202, Qr[3], lr[26]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_130 = fma(w[1], R1_120, 2.0 * T1_110);
    lr[16] = fma(R0_130, Qr[14], lr[16]);
    lr[17] = fma(R0_130, Qr[12], lr[17]);
    lr[20] = fma(R0_130, Qr[7], lr[20]);
    lr[22] = fma(R0_130, Qr[5], lr[22]);
    lr[27] = fma(R0_130, Qr[2], lr[27]);
    lr[29] = fma(R0_130, Qr[1], lr[29]);
    lr[36] = fma(R0_130, Qr[0], lr[36]);
    const double R0_121 = w[2] * R1_120;
    lr[16] = fma(R0_121, Qr[15], lr[16]);
    lr[17] = fma(R0_121, Qr[13], lr[17]);
    lr[18] = fma(R0_121, Qr[12], lr[18]);
    lr[20] = fma(R0_121, Qr[8], lr[20]);
    lr[21] = fma(R0_121, Qr[7], lr[21]);
    lr[22] = fma(R0_121, Qr[6], lr[22]);
    lr[23] = fma(R0_121, Qr[5], lr[23]);
    lr[27] = fma(R0_121, Qr[3], lr[27]);
    lr[28] = fma(R0_121, Qr[2], lr[28]);
    lr[30] = fma(R0_121, Qr[1], lr[30]);
    lr[37] = fma(R0_121, Qr[0], lr[37]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_112 = -(R0_310 + R0_130);
    lr[18] = fma(R0_112, Qr[13], lr[18]);
    lr[21] = fma(R0_112, Qr[8], lr[21]);
    lr[23] = fma(R0_112, Qr[6], lr[23]);
    lr[28] = fma(R0_112, Qr[3], lr[28]);
    const double R2_020 = fma(w[1], R3_010, T3_000);
    const double R1_030 = fma(w[1], R2_020, 2.0 * T2_010);
    const double R0_040 = fma(w[1], R1_030, 3.0 * T1_020);
    lr[17] = fma(R0_040, Qr[14], lr[17]);
    lr[22] = fma(R0_040, Qr[7], lr[22]);
    lr[29] = fma(R0_040, Qr[2], lr[29]);
    lr[38] = fma(R0_040, Qr[0], lr[38]);
    const double R0_031 = w[2] * R1_030;
    lr[17] = fma(R0_031, Qr[15], lr[17]);
    lr[18] = fma(R0_031, Qr[14], lr[18]);
    lr[22] = fma(R0_031, Qr[8], lr[22]);
    lr[23] = fma(R0_031, Qr[7], lr[23]);
    lr[29] = fma(R0_031, Qr[3], lr[29]);
    lr[30] = fma(R0_031, Qr[2], lr[30]);
    lr[39] = fma(R0_031, Qr[0], lr[39]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_022 = -(R0_220 + R0_040);
    lr[18] = fma(R0_022, Qr[15], lr[18]);
    lr[23] = fma(R0_022, Qr[8], lr[23]);
    lr[30] = fma(R0_022, Qr[3], lr[30]);
  }
  static constexpr int FLOPS_M2L_H = 388;  // + one refined rsqrt
  __device__ __forceinline__ static void expand(const double* lr, double* local) {
    double t[35];
    t[0] = lr[0];
    local[34] = t[0];
    t[1] = -lr[1];
    local[35] = t[1];
    t[2] = -lr[2];
    local[36] = t[2];
    t[3] = -lr[3];
    local[37] = t[3];
    t[4] = lr[4];
    local[38] = t[4];
    t[5] = lr[5];
    local[39] = t[5];
    t[6] = lr[6];
    local[40] = t[6];
    t[7] = lr[7];
    local[41] = t[7];
    t[8] = lr[8];
    local[42] = t[8];
    t[9] = -(t[4] + t[7]);
    local[43] = t[9];
    t[10] = -lr[9];
    local[44] = t[10];
    t[11] = -lr[10];
    local[45] = t[11];
    t[12] = -lr[11];
    local[46] = t[12];
    t[13] = -lr[12];
    local[47] = t[13];
    t[14] = -lr[13];
    local[48] = t[14];
    t[15] = -(t[10] + t[13]);
    local[49] = t[15];
    t[16] = -lr[14];
    local[50] = t[16];
    t[17] = -lr[15];
    local[51] = t[17];
    t[18] = -(t[11] + t[16]);
    local[52] = t[18];
    t[19] = -(t[12] + t[17]);
    local[53] = t[19];
    t[1] = (lr[1] + lr[16]);
    local[0] = t[1];
    t[2] = (lr[2] + lr[17]);
    local[1] = t[2];
    t[3] = (lr[3] + lr[18]);
    local[2] = t[3];
    t[4] = -(lr[4] + lr[19]);
    local[3] = t[4];
    t[5] = -(lr[5] + lr[20]);
    local[4] = t[5];
    t[6] = -(lr[6] + lr[21]);
    local[5] = t[6];
    t[7] = -(lr[7] + lr[22]);
    local[6] = t[7];
    t[8] = -(lr[8] + lr[23]);
    local[7] = t[8];
    t[9] = -(t[4] + t[7]);
    local[8] = t[9];
    t[10] = (lr[9] + lr[24]);
    local[9] = t[10];
    t[11] = (lr[10] + lr[25]);
    local[10] = t[11];
    t[12] = (lr[11] + lr[26]);
    local[11] = t[12];
    t[13] = (lr[12] + lr[27]);
    local[12] = t[13];
    t[14] = (lr[13] + lr[28]);
    local[13] = t[14];
    t[15] = -(t[10] + t[13]);
    local[14] = t[15];
    t[16] = (lr[14] + lr[29]);
    local[15] = t[16];
    t[17] = (lr[15] + lr[30]);
    local[16] = t[17];
    t[18] = -(t[11] + t[16]);
    local[17] = t[18];
    t[19] = -(t[12] + t[17]);
    local[18] = t[19];
    t[20] = -lr[31];
    local[19] = t[20];
    t[21] = -lr[32];
    local[20] = t[21];
    t[22] = -lr[33];
    local[21] = t[22];
    t[23] = -lr[34];
    local[22] = t[23];
    t[24] = -lr[35];
    local[23] = t[24];
    t[25] = -(t[20] + t[23]);
    local[24] = t[25];
    t[26] = -lr[36];
    local[25] = t[26];
    t[27] = -lr[37];
    local[26] = t[27];
    t[28] = -(t[21] + t[26]);
    local[27] = t[28];
    t[29] = -(t[22] + t[27]);
    local[28] = t[29];
    t[30] = -lr[38];
    local[29] = t[30];
    t[31] = -lr[39];
    local[30] = t[31];
    t[32] = -(t[23] + t[30]);
    local[31] = t[32];
    t[33] = -(t[24] + t[31]);
    local[32] = t[33];
    t[34] = -(t[25] + t[32]);
    local[33] = t[34];
  }
  __device__ __forceinline__ static void m2l_pair(const double* r, const double* QS,
                                                    const double* QTs, double* local,
                                                    double* outS) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[35];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    const double sn2 = rinv2 * -0.5;
    const double sn3 = rinv2 * -0.3333333333333333;
    const double sn4 = rinv2 * -0.25;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    D[4] = (6.0 * r[0] * D[1] + 2.0 * D[0]) * sn2;
    D[5] = (3.0 * r[0] * D[2] + 3.0 * r[1] * D[1]) * sn2;
    D[6] = (3.0 * r[0] * D[3] + 3.0 * r[2] * D[1]) * sn2;
    D[7] = (6.0 * r[1] * D[2] + 2.0 * D[0]) * sn2;
    D[8] = (3.0 * r[1] * D[3] + 3.0 * r[2] * D[2]) * sn2;
    D[9] = (6.0 * r[2] * D[3] + 2.0 * D[0]) * sn2;
    D[10] = (15.0 * r[0] * D[4] + 12.0 * D[1]) * sn3;
    D[11] = (10.0 * r[0] * D[5] + 4.0 * D[2] + 5.0 * r[1] * D[4]) * sn3;
    D[12] = (10.0 * r[0] * D[6] + 4.0 * D[3] + 5.0 * r[2] * D[4]) * sn3;
    D[13] = (5.0 * r[0] * D[7] + 10.0 * r[1] * D[5] + 4.0 * D[1]) * sn3;
    D[14] = (5.0 * r[0] * D[8] + 5.0 * r[1] * D[6] + 5.0 * r[2] * D[5]) * sn3;
    D[15] = (5.0 * r[0] * D[9] + 10.0 * r[2] * D[6] + 4.0 * D[1]) * sn3;
    D[16] = (15.0 * r[1] * D[7] + 12.0 * D[2]) * sn3;
    D[17] = (10.0 * r[1] * D[8] + 4.0 * D[3] + 5.0 * r[2] * D[7]) * sn3;
    D[18] = (5.0 * r[1] * D[9] + 10.0 * r[2] * D[8] + 4.0 * D[2]) * sn3;
    D[19] = (15.0 * r[2] * D[9] + 12.0 * D[3]) * sn3;
    D[20] = (28.0 * r[0] * D[10] + 36.0 * D[4]) * sn4;
    D[21] = (21.0 * r[0] * D[11] + 18.0 * D[5] + 7.0 * r[1] * D[10]) * sn4;
    D[22] = (21.0 * r[0] * D[12] + 18.0 * D[6] + 7.0 * r[2] * D[10]) * sn4;
    D[23] = (14.0 * r[0] * D[13] + 6.0 * D[7] + 14.0 * r[1] * D[11] + 6.0 * D[4]) * sn4;
    D[24] = (14.0 * r[0] * D[14] + 6.0 * D[8] + 7.0 * r[1] * D[12] + 7.0 * r[2] * D[11]) * sn4;
    D[25] = (14.0 * r[0] * D[15] + 6.0 * D[9] + 14.0 * r[2] * D[12] + 6.0 * D[4]) * sn4;
    D[26] = (7.0 * r[0] * D[16] + 21.0 * r[1] * D[13] + 18.0 * D[5]) * sn4;
    D[27] = (7.0 * r[0] * D[17] + 14.0 * r[1] * D[14] + 6.0 * D[6] + 7.0 * r[2] * D[13]) * sn4;
    D[28] = (7.0 * r[0] * D[18] + 7.0 * r[1] * D[15] + 14.0 * r[2] * D[14] + 6.0 * D[5]) * sn4;
    D[29] = (7.0 * r[0] * D[19] + 21.0 * r[2] * D[15] + 18.0 * D[6]) * sn4;
    D[30] = (28.0 * r[1] * D[16] + 36.0 * D[7]) * sn4;
    D[31] = (21.0 * r[1] * D[17] + 18.0 * D[8] + 7.0 * r[2] * D[16]) * sn4;
    D[32] = (14.0 * r[1] * D[18] + 6.0 * D[9] + 14.0 * r[2] * D[17] + 6.0 * D[7]) * sn4;
    D[33] = (7.0 * r[1] * D[19] + 21.0 * r[2] * D[18] + 18.0 * D[8]) * sn4;
    D[34] = (28.0 * r[2] * D[19] + 36.0 * D[9]) * sn4;
    {
      double s = D[1] * QS[0];
      s = fma(D[4], QS[1], s);
      s = fma(D[5], QS[2], s);
      s = fma(D[6], QS[3], s);
      s = fma(D[10], QS[4], s);
      s = fma(D[11], QS[5], s);
      s = fma(D[12], QS[6], s);
      s = fma(D[13], QS[7], s);
      s = fma(D[14], QS[8], s);
      s = fma(D[15], QS[9], s);
      local[35] -= s;
      s = fma(D[20], QS[10], s);
      s = fma(D[21], QS[11], s);
      s = fma(D[22], QS[12], s);
      s = fma(D[23], QS[13], s);
      s = fma(D[24], QS[14], s);
      s = fma(D[25], QS[15], s);
      s = fma(D[26], QS[16], s);
      s = fma(D[27], QS[17], s);
      s = fma(D[28], QS[18], s);
      s = fma(D[29], QS[19], s);
      local[0] += s;
    }
    {
      double s = D[2] * QS[0];
      s = fma(D[5], QS[1], s);
      s = fma(D[7], QS[2], s);
      s = fma(D[8], QS[3], s);
      s = fma(D[11], QS[4], s);
      s = fma(D[13], QS[5], s);
      s = fma(D[14], QS[6], s);
      s = fma(D[16], QS[7], s);
      s = fma(D[17], QS[8], s);
      s = fma(D[18], QS[9], s);
      local[36] -= s;
      s = fma(D[21], QS[10], s);
      s = fma(D[23], QS[11], s);
      s = fma(D[24], QS[12], s);
      s = fma(D[26], QS[13], s);
      s = fma(D[27], QS[14], s);
      s = fma(D[28], QS[15], s);
      s = fma(D[30], QS[16], s);
      s = fma(D[31], QS[17], s);
      s = fma(D[32], QS[18], s);
      s = fma(D[33], QS[19], s);
      local[1] += s;
    }
    {
      double s = D[3] * QS[0];
      s = fma(D[6], QS[1], s);
      s = fma(D[8], QS[2], s);
      s = fma(D[9], QS[3], s);
      s = fma(D[12], QS[4], s);
      s = fma(D[14], QS[5], s);
      s = fma(D[15], QS[6], s);
      s = fma(D[17], QS[7], s);
      s = fma(D[18], QS[8], s);
      s = fma(D[19], QS[9], s);
      local[37] -= s;
      s = fma(D[22], QS[10], s);
      s = fma(D[24], QS[11], s);
      s = fma(D[25], QS[12], s);
      s = fma(D[27], QS[13], s);
      s = fma(D[28], QS[14], s);
      s = fma(D[29], QS[15], s);
      s = fma(D[31], QS[16], s);
      s = fma(D[32], QS[17], s);
      s = fma(D[33], QS[18], s);
      s = fma(D[34], QS[19], s);
      local[2] += s;
    }
    {
      double s = D[4] * QS[0];
      s = fma(D[10], QS[1], s);
      s = fma(D[11], QS[2], s);
      s = fma(D[12], QS[3], s);
      local[38] += s;
      s = fma(D[20], QS[4], s);
      s = fma(D[21], QS[5], s);
      s = fma(D[22], QS[6], s);
      s = fma(D[23], QS[7], s);
      s = fma(D[24], QS[8], s);
      s = fma(D[25], QS[9], s);
      local[3] -= s;
    }
    {
      double s = D[5] * QS[0];
      s = fma(D[11], QS[1], s);
      s = fma(D[13], QS[2], s);
      s = fma(D[14], QS[3], s);
      local[39] += s;
      s = fma(D[21], QS[4], s);
      s = fma(D[23], QS[5], s);
      s = fma(D[24], QS[6], s);
      s = fma(D[26], QS[7], s);
      s = fma(D[27], QS[8], s);
      s = fma(D[28], QS[9], s);
      local[4] -= s;
    }
    {
      double s = D[6] * QS[0];
      s = fma(D[12], QS[1], s);
      s = fma(D[14], QS[2], s);
      s = fma(D[15], QS[3], s);
      local[40] += s;
      s = fma(D[22], QS[4], s);
      s = fma(D[24], QS[5], s);
      s = fma(D[25], QS[6], s);
      s = fma(D[27], QS[7], s);
      s = fma(D[28], QS[8], s);
      s = fma(D[29], QS[9], s);
      local[5] -= s;
    }
    {
      double s = D[7] * QS[0];
      s = fma(D[13], QS[1], s);
      s = fma(D[16], QS[2], s);
      s = fma(D[17], QS[3], s);
      local[41] += s;
      s = fma(D[23], QS[4], s);
      s = fma(D[26], QS[5], s);
      s = fma(D[27], QS[6], s);
      s = fma(D[30], QS[7], s);
      s = fma(D[31], QS[8], s);
      s = fma(D[32], QS[9], s);
      local[6] -= s;
    }
    {
      double s = D[8] * QS[0];
      s = fma(D[14], QS[1], s);
      s = fma(D[17], QS[2], s);
      s = fma(D[18], QS[3], s);
      local[42] += s;
      s = fma(D[24], QS[4], s);
      s = fma(D[27], QS[5], s);
      s = fma(D[28], QS[6], s);
      s = fma(D[31], QS[7], s);
      s = fma(D[32], QS[8], s);
      s = fma(D[33], QS[9], s);
      local[7] -= s;
    }
    {
      double s = D[9] * QS[0];
      s = fma(D[15], QS[1], s);
      s = fma(D[18], QS[2], s);
      s = fma(D[19], QS[3], s);
      local[43] += s;
      s = fma(D[25], QS[4], s);
      s = fma(D[28], QS[5], s);
      s = fma(D[29], QS[6], s);
      s = fma(D[32], QS[7], s);
      s = fma(D[33], QS[8], s);
      s = fma(D[34], QS[9], s);
      local[8] -= s;
    }
    {
      double s = D[10] * QS[0];
      local[44] -= s;
      s = fma(D[20], QS[1], s);
      s = fma(D[21], QS[2], s);
      s = fma(D[22], QS[3], s);
      local[9] += s;
    }
    {
      double s = D[11] * QS[0];
      local[45] -= s;
      s = fma(D[21], QS[1], s);
      s = fma(D[23], QS[2], s);
      s = fma(D[24], QS[3], s);
      local[10] += s;
    }
    {
      double s = D[12] * QS[0];
      local[46] -= s;
      s = fma(D[22], QS[1], s);
      s = fma(D[24], QS[2], s);
      s = fma(D[25], QS[3], s);
      local[11] += s;
    }
    {
      double s = D[13] * QS[0];
      local[47] -= s;
      s = fma(D[23], QS[1], s);
      s = fma(D[26], QS[2], s);
      s = fma(D[27], QS[3], s);
      local[12] += s;
    }
    {
      double s = D[14] * QS[0];
      local[48] -= s;
      s = fma(D[24], QS[1], s);
      s = fma(D[27], QS[2], s);
      s = fma(D[28], QS[3], s);
      local[13] += s;
    }
    {
      double s = D[15] * QS[0];
      local[49] -= s;
      s = fma(D[25], QS[1], s);
      s = fma(D[28], QS[2], s);
      s = fma(D[29], QS[3], s);
      local[14] += s;
    }
    {
      double s = D[16] * QS[0];
      local[50] -= s;
      s = fma(D[26], QS[1], s);
      s = fma(D[30], QS[2], s);
      s = fma(D[31], QS[3], s);
      local[15] += s;
    }
    {
      double s = D[17] * QS[0];
      local[51] -= s;
      s = fma(D[27], QS[1], s);
      s = fma(D[31], QS[2], s);
      s = fma(D[32], QS[3], s);
      local[16] += s;
    }
    {
      double s = D[18] * QS[0];
      local[52] -= s;
      s = fma(D[28], QS[1], s);
      s = fma(D[32], QS[2], s);
      s = fma(D[33], QS[3], s);
      local[17] += s;
    }
    {
      double s = D[19] * QS[0];
      local[53] -= s;
      s = fma(D[29], QS[1], s);
      s = fma(D[33], QS[2], s);
      s = fma(D[34], QS[3], s);
      local[18] += s;
    }
    {
      double s = D[20] * QS[0];
      local[19] -= s;
    }
    {
      double s = D[21] * QS[0];
      local[20] -= s;
    }
    {
      double s = D[22] * QS[0];
      local[21] -= s;
    }
    {
      double s = D[23] * QS[0];
      local[22] -= s;
    }
    {
      double s = D[24] * QS[0];
      local[23] -= s;
    }
    {
      double s = D[25] * QS[0];
      local[24] -= s;
    }
    {
      double s = D[26] * QS[0];
      local[25] -= s;
    }
    {
      double s = D[27] * QS[0];
      local[26] -= s;
    }
    {
      double s = D[28] * QS[0];
      local[27] -= s;
    }
    {
      double s = D[29] * QS[0];
      local[28] -= s;
    }
    {
      double s = D[30] * QS[0];
      local[29] -= s;
    }
    {
      double s = D[31] * QS[0];
      local[30] -= s;
    }
    {
      double s = D[32] * QS[0];
      local[31] -= s;
    }
    {
      double s = D[33] * QS[0];
      local[32] -= s;
    }
    {
      double s = D[34] * QS[0];
      local[33] -= s;
    }
    {
      double s = D[0] * QS[0];
      s = fma(D[1], QS[1], s);
      s = fma(D[2], QS[2], s);
      s = fma(D[3], QS[3], s);
      s = fma(D[4], QS[4], s);
      s = fma(D[5], QS[5], s);
      s = fma(D[6], QS[6], s);
      s = fma(D[7], QS[7], s);
      s = fma(D[8], QS[8], s);
      s = fma(D[9], QS[9], s);
      s = fma(D[10], QS[10], s);
      s = fma(D[11], QS[11], s);
      s = fma(D[12], QS[12], s);
      s = fma(D[13], QS[13], s);
      s = fma(D[14], QS[14], s);
      s = fma(D[15], QS[15], s);
      s = fma(D[16], QS[16], s);
      s = fma(D[17], QS[17], s);
      s = fma(D[18], QS[18], s);
      s = fma(D[19], QS[19], s);
      local[34] += s;
    }
    {
      double s = D[1] * QTs[0];
      s = fma(D[4], QTs[1], s);
      s = fma(D[5], QTs[2], s);
      s = fma(D[6], QTs[3], s);
      s = fma(D[10], QTs[4], s);
      s = fma(D[11], QTs[5], s);
      s = fma(D[12], QTs[6], s);
      s = fma(D[13], QTs[7], s);
      s = fma(D[14], QTs[8], s);
      s = fma(D[15], QTs[9], s);
      unsafeAtomicAdd(&outS[35], s);
      s = fma(D[20], QTs[10], s);
      s = fma(D[21], QTs[11], s);
      s = fma(D[22], QTs[12], s);
      s = fma(D[23], QTs[13], s);
      s = fma(D[24], QTs[14], s);
      s = fma(D[25], QTs[15], s);
      s = fma(D[26], QTs[16], s);
      s = fma(D[27], QTs[17], s);
      s = fma(D[28], QTs[18], s);
      s = fma(D[29], QTs[19], s);
      unsafeAtomicAdd(&outS[0], -s);
    }
    {
      double s = D[2] * QTs[0];
      s = fma(D[5], QTs[1], s);
      s = fma(D[7], QTs[2], s);
      s = fma(D[8], QTs[3], s);
      s = fma(D[11], QTs[4], s);
      s = fma(D[13], QTs[5], s);
      s = fma(D[14], QTs[6], s);
      s = fma(D[16], QTs[7], s);
      s = fma(D[17], QTs[8], s);
      s = fma(D[18], QTs[9], s);
      unsafeAtomicAdd(&outS[36], s);
      s = fma(D[21], QTs[10], s);
      s = fma(D[23], QTs[11], s);
      s = fma(D[24], QTs[12], s);
      s = fma(D[26], QTs[13], s);
      s = fma(D[27], QTs[14], s);
      s = fma(D[28], QTs[15], s);
      s = fma(D[30], QTs[16], s);
      s = fma(D[31], QTs[17], s);
      s = fma(D[32], QTs[18], s);
      s = fma(D[33], QTs[19], s);
      unsafeAtomicAdd(&outS[1], -s);
    }
    {
      double s = D[3] * QTs[0];
      s = fma(D[6], QTs[1], s);
      s = fma(D[8], QTs[2], s);
      s = fma(D[9], QTs[3], s);
      s = fma(D[12], QTs[4], s);
      s = fma(D[14], QTs[5], s);
      s = fma(D[15], QTs[6], s);
      s = fma(D[17], QTs[7], s);
      s = fma(D[18], QTs[8], s);
      s = fma(D[19], QTs[9], s);
      unsafeAtomicAdd(&outS[37], s);
      s = fma(D[22], QTs[10], s);
      s = fma(D[24], QTs[11], s);
      s = fma(D[25], QTs[12], s);
      s = fma(D[27], QTs[13], s);
      s = fma(D[28], QTs[14], s);
      s = fma(D[29], QTs[15], s);
      s = fma(D[31], QTs[16], s);
      s = fma(D[32], QTs[17], s);
      s = fma(D[33], QTs[18], s);
      s = fma(D[34], QTs[19], s);
      unsafeAtomicAdd(&outS[2], -s);
    }
    {
      double s = D[4] * QTs[0];
      s = fma(D[10], QTs[1], s);
      s = fma(D[11], QTs[2], s);
      s = fma(D[12], QTs[3], s);
      unsafeAtomicAdd(&outS[38], s);
      s = fma(D[20], QTs[4], s);
      s = fma(D[21], QTs[5], s);
      s = fma(D[22], QTs[6], s);
      s = fma(D[23], QTs[7], s);
      s = fma(D[24], QTs[8], s);
      s = fma(D[25], QTs[9], s);
      unsafeAtomicAdd(&outS[3], -s);
    }
    {
      double s = D[5] * QTs[0];
      s = fma(D[11], QTs[1], s);
      s = fma(D[13], QTs[2], s);
      s = fma(D[14], QTs[3], s);
      unsafeAtomicAdd(&outS[39], s);
      s = fma(D[21], QTs[4], s);
      s = fma(D[23], QTs[5], s);
      s = fma(D[24], QTs[6], s);
      s = fma(D[26], QTs[7], s);
      s = fma(D[27], QTs[8], s);
      s = fma(D[28], QTs[9], s);
      unsafeAtomicAdd(&outS[4], -s);
    }
    {
      double s = D[6] * QTs[0];
      s = fma(D[12], QTs[1], s);
      s = fma(D[14], QTs[2], s);
      s = fma(D[15], QTs[3], s);
      unsafeAtomicAdd(&outS[40], s);
      s = fma(D[22], QTs[4], s);
      s = fma(D[24], QTs[5], s);
      s = fma(D[25], QTs[6], s);
      s = fma(D[27], QTs[7], s);
      s = fma(D[28], QTs[8], s);
      s = fma(D[29], QTs[9], s);
      unsafeAtomicAdd(&outS[5], -s);
    }
    {
      double s = D[7] * QTs[0];
      s = fma(D[13], QTs[1], s);
      s = fma(D[16], QTs[2], s);
      s = fma(D[17], QTs[3], s);
      unsafeAtomicAdd(&outS[41], s);
      s = fma(D[23], QTs[4], s);
      s = fma(D[26], QTs[5], s);
      s = fma(D[27], QTs[6], s);
      s = fma(D[30], QTs[7], s);
      s = fma(D[31], QTs[8], s);
      s = fma(D[32], QTs[9], s);
      unsafeAtomicAdd(&outS[6], -s);
    }
    {
      double s = D[8] * QTs[0];
      s = fma(D[14], QTs[1], s);
      s = fma(D[17], QTs[2], s);
      s = fma(D[18], QTs[3], s);
      unsafeAtomicAdd(&outS[42], s);
      s = fma(D[24], QTs[4], s);
      s = fma(D[27], QTs[5], s);
      s = fma(D[28], QTs[6], s);
      s = fma(D[31], QTs[7], s);
      s = fma(D[32], QTs[8], s);
      s = fma(D[33], QTs[9], s);
      unsafeAtomicAdd(&outS[7], -s);
    }
    {
      double s = D[9] * QTs[0];
      s = fma(D[15], QTs[1], s);
      s = fma(D[18], QTs[2], s);
      s = fma(D[19], QTs[3], s);
      unsafeAtomicAdd(&outS[43], s);
      s = fma(D[25], QTs[4], s);
      s = fma(D[28], QTs[5], s);
      s = fma(D[29], QTs[6], s);
      s = fma(D[32], QTs[7], s);
      s = fma(D[33], QTs[8], s);
      s = fma(D[34], QTs[9], s);
      unsafeAtomicAdd(&outS[8], -s);
    }
    {
      double s = D[10] * QTs[0];
      unsafeAtomicAdd(&outS[44], s);
      s = fma(D[20], QTs[1], s);
      s = fma(D[21], QTs[2], s);
      s = fma(D[22], QTs[3], s);
      unsafeAtomicAdd(&outS[9], -s);
    }
    {
      double s = D[11] * QTs[0];
      unsafeAtomicAdd(&outS[45], s);
      s = fma(D[21], QTs[1], s);
      s = fma(D[23], QTs[2], s);
      s = fma(D[24], QTs[3], s);
      unsafeAtomicAdd(&outS[10], -s);
    }
    {
      double s = D[12] * QTs[0];
      unsafeAtomicAdd(&outS[46], s);
      s = fma(D[22], QTs[1], s);
      s = fma(D[24], QTs[2], s);
      s = fma(D[25], QTs[3], s);
      unsafeAtomicAdd(&outS[11], -s);
    }
    {
      double s = D[13] * QTs[0];
      unsafeAtomicAdd(&outS[47], s);
      s = fma(D[23], QTs[1], s);
      s = fma(D[26], QTs[2], s);
      s = fma(D[27], QTs[3], s);
      unsafeAtomicAdd(&outS[12], -s);
    }
    {
      double s = D[14] * QTs[0];
      unsafeAtomicAdd(&outS[48], s);
      s = fma(D[24], QTs[1], s);
      s = fma(D[27], QTs[2], s);
      s = fma(D[28], QTs[3], s);
      unsafeAtomicAdd(&outS[13], -s);
    }
    {
      double s = D[15] * QTs[0];
      unsafeAtomicAdd(&outS[49], s);
      s = fma(D[25], QTs[1], s);
      s = fma(D[28], QTs[2], s);
      s = fma(D[29], QTs[3], s);
      unsafeAtomicAdd(&outS[14], -s);
    }
    {
      double s = D[16] * QTs[0];
      unsafeAtomicAdd(&outS[50], s);
      s = fma(D[26], QTs[1], s);
      s = fma(D[30], QTs[2], s);
      s = fma(D[31], QTs[3], s);
      unsafeAtomicAdd(&outS[15], -s);
    }
    {
      double s = D[17] * QTs[0];
      unsafeAtomicAdd(&outS[51], s);
      s = fma(D[27], QTs[1], s);
      s = fma(D[31], QTs[2], s);
      s = fma(D[32], QTs[3], s);
      unsafeAtomicAdd(&outS[16], -s);
    }
    {
      double s = D[18] * QTs[0];
      unsafeAtomicAdd(&outS[52], s);
      s = fma(D[28], QTs[1], s);
      s = fma(D[32], QTs[2], s);
      s = fma(D[33], QTs[3], s);
      unsafeAtomicAdd(&outS[17], -s);
    }
    {
      double s = D[19] * QTs[0];
      unsafeAtomicAdd(&outS[53], s);
      s = fma(D[29], QTs[1], s);
      s = fma(D[33], QTs[2], s);
      s = fma(D[34], QTs[3], s);
      unsafeAtomicAdd(&outS[18], -s);
    }
    {
      double s = D[20] * QTs[0];
      unsafeAtomicAdd(&outS[19], -s);
    }
    {
      double s = D[21] * QTs[0];
      unsafeAtomicAdd(&outS[20], -s);
    }
    {
      double s = D[22] * QTs[0];
      unsafeAtomicAdd(&outS[21], -s);
    }
    {
      double s = D[23] * QTs[0];
      unsafeAtomicAdd(&outS[22], -s);
    }
    {
      double s = D[24] * QTs[0];
      unsafeAtomicAdd(&outS[23], -s);
    }
    {
      double s = D[25] * QTs[0];
      unsafeAtomicAdd(&outS[24], -s);
    }
    {
      double s = D[26] * QTs[0];
      unsafeAtomicAdd(&outS[25], -s);
    }
    {
      double s = D[27] * QTs[0];
      unsafeAtomicAdd(&outS[26], -s);
    }
    {
      double s = D[28] * QTs[0];
      unsafeAtomicAdd(&outS[27], -s);
    }
    {
      double s = D[29] * QTs[0];
      unsafeAtomicAdd(&outS[28], -s);
    }
    {
      double s = D[30] * QTs[0];
      unsafeAtomicAdd(&outS[29], -s);
    }
    {
      double s = D[31] * QTs[0];
      unsafeAtomicAdd(&outS[30], -s);
    }
    {
      double s = D[32] * QTs[0];
      unsafeAtomicAdd(&outS[31], -s);
    }
    {
      double s = D[33] * QTs[0];
      unsafeAtomicAdd(&outS[32], -s);
    }
    {
      double s = D[34] * QTs[0];
      unsafeAtomicAdd(&outS[33], -s);
    }
    {
      double s = D[0] * QTs[0];
      s = fma(D[1], QTs[1], s);
      s = fma(D[2], QTs[2], s);
      s = fma(D[3], QTs[3], s);
      s = fma(D[4], QTs[4], s);
      s = fma(D[5], QTs[5], s);
      s = fma(D[6], QTs[6], s);
      s = fma(D[7], QTs[7], s);
      s = fma(D[8], QTs[8], s);
      s = fma(D[9], QTs[9], s);
      s = fma(D[10], QTs[10], s);
      s = fma(D[11], QTs[11], s);
      s = fma(D[12], QTs[12], s);
      s = fma(D[13], QTs[13], s);
      s = fma(D[14], QTs[14], s);
      s = fma(D[15], QTs[15], s);
      s = fma(D[16], QTs[16], s);
      s = fma(D[17], QTs[17], s);
      s = fma(D[18], QTs[18], s);
      s = fma(D[19], QTs[19], s);
      unsafeAtomicAdd(&outS[34], s);
    }
  }
  static constexpr int FLOPS_M2L_PAIR = 1068;  // both directions, + one rsqrt
  __device__ __forceinline__ static void l2l(const double* h, double* local) {
    double mh[20];
    mh[0] = 1.0;
    mh[1] = mh[0] * h[0];
    mh[2] = mh[0] * h[1];
    mh[3] = mh[0] * h[2];
    mh[4] = mh[1] * (h[0] * 0.5);
    mh[5] = mh[2] * h[0];
    mh[6] = mh[3] * h[0];
    mh[7] = mh[2] * (h[1] * 0.5);
    mh[8] = mh[3] * h[1];
    mh[9] = mh[3] * (h[2] * 0.5);
    mh[10] = mh[4] * (h[0] * 0.3333333333333333);
    mh[11] = mh[5] * (h[0] * 0.5);
    mh[12] = mh[6] * (h[0] * 0.5);
    mh[13] = mh[7] * h[0];
    mh[14] = mh[8] * h[0];
    mh[15] = mh[9] * h[0];
    mh[16] = mh[7] * (h[1] * 0.3333333333333333);
    mh[17] = mh[8] * (h[1] * 0.5);
    mh[18] = mh[9] * h[1];
    mh[19] = mh[9] * (h[2] * 0.3333333333333333);
    local[0] = fma(local[28], mh[19], fma(local[27], mh[18], fma(local[26], mh[17], fma(local[25], mh[16], fma(local[24], mh[15], fma(local[23], mh[14], fma(local[22], mh[13], fma(local[21], mh[12], fma(local[20], mh[11], fma(local[19], mh[10], fma(local[14], mh[9], fma(local[13], mh[8], fma(local[12], mh[7], fma(local[11], mh[6], fma(local[10], mh[5], fma(local[9], mh[4], fma(local[5], mh[3], fma(local[4], mh[2], fma(local[3], mh[1], local[0])))))))))))))))))));
    local[1] = fma(local[32], mh[19], fma(local[31], mh[18], fma(local[30], mh[17], fma(local[29], mh[16], fma(local[27], mh[15], fma(local[26], mh[14], fma(local[25], mh[13], fma(local[23], mh[12], fma(local[22], mh[11], fma(local[20], mh[10], fma(local[17], mh[9], fma(local[16], mh[8], fma(local[15], mh[7], fma(local[13], mh[6], fma(local[12], mh[5], fma(local[10], mh[4], fma(local[7], mh[3], fma(local[6], mh[2], fma(local[4], mh[1], local[1])))))))))))))))))));
    local[2] = fma(local[33], mh[19], fma(local[32], mh[18], fma(local[31], mh[17], fma(local[30], mh[16], fma(local[28], mh[15], fma(local[27], mh[14], fma(local[26], mh[13], fma(local[24], mh[12], fma(local[23], mh[11], fma(local[21], mh[10], fma(local[18], mh[9], fma(local[17], mh[8], fma(local[16], mh[7], fma(local[14], mh[6], fma(local[13], mh[5], fma(local[11], mh[4], fma(local[8], mh[3], fma(local[7], mh[2], fma(local[5], mh[1], local[2])))))))))))))))))));
    local[3] = fma(local[24], mh[9], fma(local[23], mh[8], fma(local[22], mh[7], fma(local[21], mh[6], fma(local[20], mh[5], fma(local[19], mh[4], fma(local[11], mh[3], fma(local[10], mh[2], fma(local[9], mh[1], local[3])))))))));
    local[4] = fma(local[27], mh[9], fma(local[26], mh[8], fma(local[25], mh[7], fma(local[23], mh[6], fma(local[22], mh[5], fma(local[20], mh[4], fma(local[13], mh[3], fma(local[12], mh[2], fma(local[10], mh[1], local[4])))))))));
    local[5] = fma(local[28], mh[9], fma(local[27], mh[8], fma(local[26], mh[7], fma(local[24], mh[6], fma(local[23], mh[5], fma(local[21], mh[4], fma(local[14], mh[3], fma(local[13], mh[2], fma(local[11], mh[1], local[5])))))))));
    local[6] = fma(local[31], mh[9], fma(local[30], mh[8], fma(local[29], mh[7], fma(local[26], mh[6], fma(local[25], mh[5], fma(local[22], mh[4], fma(local[16], mh[3], fma(local[15], mh[2], fma(local[12], mh[1], local[6])))))))));
    local[7] = fma(local[32], mh[9], fma(local[31], mh[8], fma(local[30], mh[7], fma(local[27], mh[6], fma(local[26], mh[5], fma(local[23], mh[4], fma(local[17], mh[3], fma(local[16], mh[2], fma(local[13], mh[1], local[7])))))))));
    local[8] = fma(local[33], mh[9], fma(local[32], mh[8], fma(local[31], mh[7], fma(local[28], mh[6], fma(local[27], mh[5], fma(local[24], mh[4], fma(local[18], mh[3], fma(local[17], mh[2], fma(local[14], mh[1], local[8])))))))));
    local[9] = fma(local[21], mh[3], fma(local[20], mh[2], fma(local[19], mh[1], local[9])));
    local[10] = fma(local[23], mh[3], fma(local[22], mh[2], fma(local[20], mh[1], local[10])));
    local[11] = fma(local[24], mh[3], fma(local[23], mh[2], fma(local[21], mh[1], local[11])));
    local[12] = fma(local[26], mh[3], fma(local[25], mh[2], fma(local[22], mh[1], local[12])));
    local[13] = fma(local[27], mh[3], fma(local[26], mh[2], fma(local[23], mh[1], local[13])));
    local[14] = fma(local[28], mh[3], fma(local[27], mh[2], fma(local[24], mh[1], local[14])));
    local[15] = fma(local[30], mh[3], fma(local[29], mh[2], fma(local[25], mh[1], local[15])));
    local[16] = fma(local[31], mh[3], fma(local[30], mh[2], fma(local[26], mh[1], local[16])));
    local[17] = fma(local[32], mh[3], fma(local[31], mh[2], fma(local[27], mh[1], local[17])));
    local[18] = fma(local[33], mh[3], fma(local[32], mh[2], fma(local[28], mh[1], local[18])));
    local[19] = local[19];
    local[20] = local[20];
    local[21] = local[21];
    local[22] = local[22];
    local[23] = local[23];
    local[24] = local[24];
    local[25] = local[25];
    local[26] = local[26];
    local[27] = local[27];
    local[28] = local[28];
    local[29] = local[29];
    local[30] = local[30];
    local[31] = local[31];
    local[32] = local[32];
    local[33] = local[33];
    local[34] = fma(local[53], mh[19], fma(local[52], mh[18], fma(local[51], mh[17], fma(local[50], mh[16], fma(local[49], mh[15], fma(local[48], mh[14], fma(local[47], mh[13], fma(local[46], mh[12], fma(local[45], mh[11], fma(local[44], mh[10], fma(local[43], mh[9], fma(local[42], mh[8], fma(local[41], mh[7], fma(local[40], mh[6], fma(local[39], mh[5], fma(local[38], mh[4], fma(local[37], mh[3], fma(local[36], mh[2], fma(local[35], mh[1], local[34])))))))))))))))))));
    local[35] = fma(local[49], mh[9], fma(local[48], mh[8], fma(local[47], mh[7], fma(local[46], mh[6], fma(local[45], mh[5], fma(local[44], mh[4], fma(local[40], mh[3], fma(local[39], mh[2], fma(local[38], mh[1], local[35])))))))));
    local[36] = fma(local[52], mh[9], fma(local[51], mh[8], fma(local[50], mh[7], fma(local[48], mh[6], fma(local[47], mh[5], fma(local[45], mh[4], fma(local[42], mh[3], fma(local[41], mh[2], fma(local[39], mh[1], local[36])))))))));
    local[37] = fma(local[53], mh[9], fma(local[52], mh[8], fma(local[51], mh[7], fma(local[49], mh[6], fma(local[48], mh[5], fma(local[46], mh[4], fma(local[43], mh[3], fma(local[42], mh[2], fma(local[40], mh[1], local[37])))))))));
    local[38] = fma(local[46], mh[3], fma(local[45], mh[2], fma(local[44], mh[1], local[38])));
    local[39] = fma(local[48], mh[3], fma(local[47], mh[2], fma(local[45], mh[1], local[39])));
    local[40] = fma(local[49], mh[3], fma(local[48], mh[2], fma(local[46], mh[1], local[40])));
    local[41] = fma(local[51], mh[3], fma(local[50], mh[2], fma(local[47], mh[1], local[41])));
    local[42] = fma(local[52], mh[3], fma(local[51], mh[2], fma(local[48], mh[1], local[42])));
    local[43] = fma(local[53], mh[3], fma(local[52], mh[2], fma(local[49], mh[1], local[43])));
    local[44] = local[44];
    local[45] = local[45];
    local[46] = local[46];
    local[47] = local[47];
    local[48] = local[48];
    local[49] = local[49];
    local[50] = local[50];
    local[51] = local[51];
    local[52] = local[52];
    local[53] = local[53];
  }
  static constexpr int FLOPS_L2L = 438;
  __device__ __forceinline__ static void l2p(const double* a, const double* local, double* f, double& phi) {
    double ma[20];
    ma[0] = 1.0;
    ma[1] = ma[0] * a[0];
    ma[2] = ma[0] * a[1];
    ma[3] = ma[0] * a[2];
    ma[4] = ma[1] * (a[0] * 0.5);
    ma[5] = ma[2] * a[0];
    ma[6] = ma[3] * a[0];
    ma[7] = ma[2] * (a[1] * 0.5);
    ma[8] = ma[3] * a[1];
    ma[9] = ma[3] * (a[2] * 0.5);
    ma[10] = ma[4] * (a[0] * 0.3333333333333333);
    ma[11] = ma[5] * (a[0] * 0.5);
    ma[12] = ma[6] * (a[0] * 0.5);
    ma[13] = ma[7] * a[0];
    ma[14] = ma[8] * a[0];
    ma[15] = ma[9] * a[0];
    ma[16] = ma[7] * (a[1] * 0.3333333333333333);
    ma[17] = ma[8] * (a[1] * 0.5);
    ma[18] = ma[9] * a[1];
    ma[19] = ma[9] * (a[2] * 0.3333333333333333);
    f[0] += fma(local[28], ma[19], fma(local[27], ma[18], fma(local[26], ma[17], fma(local[25], ma[16], fma(local[24], ma[15], fma(local[23], ma[14], fma(local[22], ma[13], fma(local[21], ma[12], fma(local[20], ma[11], fma(local[19], ma[10], fma(local[14], ma[9], fma(local[13], ma[8], fma(local[12], ma[7], fma(local[11], ma[6], fma(local[10], ma[5], fma(local[9], ma[4], fma(local[5], ma[3], fma(local[4], ma[2], fma(local[3], ma[1], local[0])))))))))))))))))));
    f[1] += fma(local[32], ma[19], fma(local[31], ma[18], fma(local[30], ma[17], fma(local[29], ma[16], fma(local[27], ma[15], fma(local[26], ma[14], fma(local[25], ma[13], fma(local[23], ma[12], fma(local[22], ma[11], fma(local[20], ma[10], fma(local[17], ma[9], fma(local[16], ma[8], fma(local[15], ma[7], fma(local[13], ma[6], fma(local[12], ma[5], fma(local[10], ma[4], fma(local[7], ma[3], fma(local[6], ma[2], fma(local[4], ma[1], local[1])))))))))))))))))));
    f[2] += fma(local[33], ma[19], fma(local[32], ma[18], fma(local[31], ma[17], fma(local[30], ma[16], fma(local[28], ma[15], fma(local[27], ma[14], fma(local[26], ma[13], fma(local[24], ma[12], fma(local[23], ma[11], fma(local[21], ma[10], fma(local[18], ma[9], fma(local[17], ma[8], fma(local[16], ma[7], fma(local[14], ma[6], fma(local[13], ma[5], fma(local[11], ma[4], fma(local[8], ma[3], fma(local[7], ma[2], fma(local[5], ma[1], local[2])))))))))))))))))));
    phi += fma(local[53], ma[19], fma(local[52], ma[18], fma(local[51], ma[17], fma(local[50], ma[16], fma(local[49], ma[15], fma(local[48], ma[14], fma(local[47], ma[13], fma(local[46], ma[12], fma(local[45], ma[11], fma(local[44], ma[10], fma(local[43], ma[9], fma(local[42], ma[8], fma(local[41], ma[7], fma(local[40], ma[6], fma(local[39], ma[5], fma(local[38], ma[4], fma(local[37], ma[3], fma(local[36], ma[2], fma(local[35], ma[1], local[34])))))))))))))))))));
  }
  static constexpr int FLOPS_L2P = 184;
};
template <> struct Exp<4> {
  static constexpr int P = 4;
  static constexpr int NQ = 35;   // mass moments, |a| <= P
  static constexpr int NL = 90;   // local coefficients: H then P
  __device__ __forceinline__ static void p2m_add(const double* b, double m, double* Q) {
    double mb[35];
    mb[0] = 1.0;
    mb[1] = mb[0] * b[0];
    mb[2] = mb[0] * b[1];
    mb[3] = mb[0] * b[2];
    mb[4] = mb[1] * (b[0] * 0.5);
    mb[5] = mb[2] * b[0];
    mb[6] = mb[3] * b[0];
    mb[7] = mb[2] * (b[1] * 0.5);
    mb[8] = mb[3] * b[1];
    mb[9] = mb[3] * (b[2] * 0.5);
    mb[10] = mb[4] * (b[0] * 0.3333333333333333);
    mb[11] = mb[5] * (b[0] * 0.5);
    mb[12] = mb[6] * (b[0] * 0.5);
    mb[13] = mb[7] * b[0];
    mb[14] = mb[8] * b[0];
    mb[15] = mb[9] * b[0];
    mb[16] = mb[7] * (b[1] * 0.3333333333333333);
    mb[17] = mb[8] * (b[1] * 0.5);
    mb[18] = mb[9] * b[1];
    mb[19] = mb[9] * (b[2] * 0.3333333333333333);
    mb[20] = mb[10] * (b[0] * 0.25);
    mb[21] = mb[11] * (b[0] * 0.3333333333333333);
    mb[22] = mb[12] * (b[0] * 0.3333333333333333);
    mb[23] = mb[13] * (b[0] * 0.5);
    mb[24] = mb[14] * (b[0] * 0.5);
    mb[25] = mb[15] * (b[0] * 0.5);
    mb[26] = mb[16] * b[0];
    mb[27] = mb[17] * b[0];
    mb[28] = mb[18] * b[0];
    mb[29] = mb[19] * b[0];
    mb[30] = mb[16] * (b[1] * 0.25);
    mb[31] = mb[17] * (b[1] * 0.3333333333333333);
    mb[32] = mb[18] * (b[1] * 0.5);
    mb[33] = mb[19] * b[1];
    mb[34] = mb[19] * (b[2] * 0.25);
    Q[0] = fma(m, mb[0], Q[0]);
    Q[1] = fma(m, mb[1], Q[1]);
    Q[2] = fma(m, mb[2], Q[2]);
    Q[3] = fma(m, mb[3], Q[3]);
    Q[4] = fma(m, mb[4], Q[4]);
    Q[5] = fma(m, mb[5], Q[5]);
    Q[6] = fma(m, mb[6], Q[6]);
    Q[7] = fma(m, mb[7], Q[7]);
    Q[8] = fma(m, mb[8], Q[8]);
    Q[9] = fma(m, mb[9], Q[9]);
    Q[10] = fma(m, mb[10], Q[10]);
    Q[11] = fma(m, mb[11], Q[11]);
    Q[12] = fma(m, mb[12], Q[12]);
    Q[13] = fma(m, mb[13], Q[13]);
    Q[14] = fma(m, mb[14], Q[14]);
    Q[15] = fma(m, mb[15], Q[15]);
    Q[16] = fma(m, mb[16], Q[16]);
    Q[17] = fma(m, mb[17], Q[17]);
    Q[18] = fma(m, mb[18], Q[18]);
    Q[19] = fma(m, mb[19], Q[19]);
    Q[20] = fma(m, mb[20], Q[20]);
    Q[21] = fma(m, mb[21], Q[21]);
    Q[22] = fma(m, mb[22], Q[22]);
    Q[23] = fma(m, mb[23], Q[23]);
    Q[24] = fma(m, mb[24], Q[24]);
    Q[25] = fma(m, mb[25], Q[25]);
    Q[26] = fma(m, mb[26], Q[26]);
    Q[27] = fma(m, mb[27], Q[27]);
    Q[28] = fma(m, mb[28], Q[28]);
    Q[29] = fma(m, mb[29], Q[29]);
    Q[30] = fma(m, mb[30], Q[30]);
    Q[31] = fma(m, mb[31], Q[31]);
    Q[32] = fma(m, mb[32], Q[32]);
    Q[33] = fma(m, mb[33], Q[33]);
    Q[34] = fma(m, mb[34], Q[34]);
  }
  static constexpr int FLOPS_P2M = 123;
  __device__ __forceinline__ static void m2m_add(const double* g, const double* Qc, double* Q) {
    double mg[35];
    mg[0] = 1.0;
    mg[1] = mg[0] * g[0];
    mg[2] = mg[0] * g[1];
    mg[3] = mg[0] * g[2];
    mg[4] = mg[1] * (g[0] * 0.5);
    mg[5] = mg[2] * g[0];
    mg[6] = mg[3] * g[0];
    mg[7] = mg[2] * (g[1] * 0.5);
    mg[8] = mg[3] * g[1];
    mg[9] = mg[3] * (g[2] * 0.5);
    mg[10] = mg[4] * (g[0] * 0.3333333333333333);
    mg[11] = mg[5] * (g[0] * 0.5);
    mg[12] = mg[6] * (g[0] * 0.5);
    mg[13] = mg[7] * g[0];
    mg[14] = mg[8] * g[0];
    mg[15] = mg[9] * g[0];
    mg[16] = mg[7] * (g[1] * 0.3333333333333333);
    mg[17] = mg[8] * (g[1] * 0.5);
    mg[18] = mg[9] * g[1];
    mg[19] = mg[9] * (g[2] * 0.3333333333333333);
    mg[20] = mg[10] * (g[0] * 0.25);
    mg[21] = mg[11] * (g[0] * 0.3333333333333333);
    mg[22] = mg[12] * (g[0] * 0.3333333333333333);
    mg[23] = mg[13] * (g[0] * 0.5);
    mg[24] = mg[14] * (g[0] * 0.5);
    mg[25] = mg[15] * (g[0] * 0.5);
    mg[26] = mg[16] * g[0];
    mg[27] = mg[17] * g[0];
    mg[28] = mg[18] * g[0];
    mg[29] = mg[19] * g[0];
    mg[30] = mg[16] * (g[1] * 0.25);
    mg[31] = mg[17] * (g[1] * 0.3333333333333333);
    mg[32] = mg[18] * (g[1] * 0.5);
    mg[33] = mg[19] * g[1];
    mg[34] = mg[19] * (g[2] * 0.25);
    Q[0] = (Q[0] + Qc[0]);
    Q[1] = (fma(Qc[0], mg[1], Q[1]) + Qc[1]);
    Q[2] = (fma(Qc[0], mg[2], Q[2]) + Qc[2]);
    Q[3] = (fma(Qc[0], mg[3], Q[3]) + Qc[3]);
    Q[4] = (fma(Qc[1], mg[1], fma(Qc[0], mg[4], Q[4])) + Qc[4]);
    Q[5] = (fma(Qc[2], mg[1], fma(Qc[1], mg[2], fma(Qc[0], mg[5], Q[5]))) + Qc[5]);
    Q[6] = (fma(Qc[3], mg[1], fma(Qc[1], mg[3], fma(Qc[0], mg[6], Q[6]))) + Qc[6]);
    Q[7] = (fma(Qc[2], mg[2], fma(Qc[0], mg[7], Q[7])) + Qc[7]);
    Q[8] = (fma(Qc[3], mg[2], fma(Qc[2], mg[3], fma(Qc[0], mg[8], Q[8]))) + Qc[8]);
    Q[9] = (fma(Qc[3], mg[3], fma(Qc[0], mg[9], Q[9])) + Qc[9]);
    Q[10] = (fma(Qc[4], mg[1], fma(Qc[1], mg[4], fma(Qc[0], mg[10], Q[10]))) + Qc[10]);
    Q[11] = (fma(Qc[5], mg[1], fma(Qc[4], mg[2], fma(Qc[2], mg[4], fma(Qc[1], mg[5], fma(Qc[0], mg[11], Q[11]))))) + Qc[11]);
    Q[12] = (fma(Qc[6], mg[1], fma(Qc[4], mg[3], fma(Qc[3], mg[4], fma(Qc[1], mg[6], fma(Qc[0], mg[12], Q[12]))))) + Qc[12]);
    Q[13] = (fma(Qc[7], mg[1], fma(Qc[5], mg[2], fma(Qc[2], mg[5], fma(Qc[1], mg[7], fma(Qc[0], mg[13], Q[13]))))) + Qc[13]);
    Q[14] = (fma(Qc[8], mg[1], fma(Qc[6], mg[2], fma(Qc[5], mg[3], fma(Qc[3], mg[5], fma(Qc[2], mg[6], fma(Qc[1], mg[8], fma(Qc[0], mg[14], Q[14]))))))) + Qc[14]);
    Q[15] = (fma(Qc[9], mg[1], fma(Qc[6], mg[3], fma(Qc[3], mg[6], fma(Qc[1], mg[9], fma(Qc[0], mg[15], Q[15]))))) + Qc[15]);
    Q[16] = (fma(Qc[7], mg[2], fma(Qc[2], mg[7], fma(Qc[0], mg[16], Q[16]))) + Qc[16]);
    Q[17] = (fma(Qc[8], mg[2], fma(Qc[7], mg[3], fma(Qc[3], mg[7], fma(Qc[2], mg[8], fma(Qc[0], mg[17], Q[17]))))) + Qc[17]);
    Q[18] = (fma(Qc[9], mg[2], fma(Qc[8], mg[3], fma(Qc[3], mg[8], fma(Qc[2], mg[9], fma(Qc[0], mg[18], Q[18]))))) + Qc[18]);
    Q[19] = (fma(Qc[9], mg[3], fma(Qc[3], mg[9], fma(Qc[0], mg[19], Q[19]))) + Qc[19]);
    Q[20] = (fma(Qc[10], mg[1], fma(Qc[4], mg[4], fma(Qc[1], mg[10], fma(Qc[0], mg[20], Q[20])))) + Qc[20]);
    Q[21] = (fma(Qc[11], mg[1], fma(Qc[10], mg[2], fma(Qc[5], mg[4], fma(Qc[4], mg[5], fma(Qc[2], mg[10], fma(Qc[1], mg[11], fma(Qc[0], mg[21], Q[21]))))))) + Qc[21]);
    Q[22] = (fma(Qc[12], mg[1], fma(Qc[10], mg[3], fma(Qc[6], mg[4], fma(Qc[4], mg[6], fma(Qc[3], mg[10], fma(Qc[1], mg[12], fma(Qc[0], mg[22], Q[22]))))))) + Qc[22]);
    Q[23] = (fma(Qc[13], mg[1], fma(Qc[11], mg[2], fma(Qc[7], mg[4], fma(Qc[5], mg[5], fma(Qc[4], mg[7], fma(Qc[2], mg[11], fma(Qc[1], mg[13], fma(Qc[0], mg[23], Q[23])))))))) + Qc[23]);
    Q[24] = (fma(Qc[14], mg[1], fma(Qc[12], mg[2], fma(Qc[11], mg[3], fma(Qc[8], mg[4], fma(Qc[6], mg[5], fma(Qc[5], mg[6], fma(Qc[4], mg[8], fma(Qc[3], mg[11], fma(Qc[2], mg[12], fma(Qc[1], mg[14], fma(Qc[0], mg[24], Q[24]))))))))))) + Qc[24]);
    Q[25] = (fma(Qc[15], mg[1], fma(Qc[12], mg[3], fma(Qc[9], mg[4], fma(Qc[6], mg[6], fma(Qc[4], mg[9], fma(Qc[3], mg[12], fma(Qc[1], mg[15], fma(Qc[0], mg[25], Q[25])))))))) + Qc[25]);
    Q[26] = (fma(Qc[16], mg[1], fma(Qc[13], mg[2], fma(Qc[7], mg[5], fma(Qc[5], mg[7], fma(Qc[2], mg[13], fma(Qc[1], mg[16], fma(Qc[0], mg[26], Q[26]))))))) + Qc[26]);
    Q[27] = (fma(Qc[17], mg[1], fma(Qc[14], mg[2], fma(Qc[13], mg[3], fma(Qc[8], mg[5], fma(Qc[7], mg[6], fma(Qc[6], mg[7], fma(Qc[5], mg[8], fma(Qc[3], mg[13], fma(Qc[2], mg[14], fma(Qc[1], mg[17], fma(Qc[0], mg[27], Q[27]))))))))))) + Qc[27]);
    Q[28] = (fma(Qc[18], mg[1], fma(Qc[15], mg[2], fma(Qc[14], mg[3], fma(Qc[9], mg[5], fma(Qc[8], mg[6], fma(Qc[6], mg[8], fma(Qc[5], mg[9], fma(Qc[3], mg[14], fma(Qc[2], mg[15], fma(Qc[1], mg[18], fma(Qc[0], mg[28], Q[28]))))))))))) + Qc[28]);
    Q[29] = (fma(Qc[19], mg[1], fma(Qc[15], mg[3], fma(Qc[9], mg[6], fma(Qc[6], mg[9], fma(Qc[3], mg[15], fma(Qc[1], mg[19], fma(Qc[0], mg[29], Q[29]))))))) + Qc[29]);
    Q[30] = (fma(Qc[16], mg[2], fma(Qc[7], mg[7], fma(Qc[2], mg[16], fma(Qc[0], mg[30], Q[30])))) + Qc[30]);
    Q[31] = (fma(Qc[17], mg[2], fma(Qc[16], mg[3], fma(Qc[8], mg[7], fma(Qc[7], mg[8], fma(Qc[3], mg[16], fma(Qc[2], mg[17], fma(Qc[0], mg[31], Q[31]))))))) + Qc[31]);
    Q[32] = (fma(Qc[18], mg[2], fma(Qc[17], mg[3], fma(Qc[9], mg[7], fma(Qc[8], mg[8], fma(Qc[7], mg[9], fma(Qc[3], mg[17], fma(Qc[2], mg[18], fma(Qc[0], mg[32], Q[32])))))))) + Qc[32]);
    Q[33] = (fma(Qc[19], mg[2], fma(Qc[18], mg[3], fma(Qc[9], mg[8], fma(Qc[8], mg[9], fma(Qc[3], mg[18], fma(Qc[2], mg[19], fma(Qc[0], mg[33], Q[33]))))))) + Qc[33]);
    Q[34] = (fma(Qc[19], mg[3], fma(Qc[9], mg[9], fma(Qc[3], mg[19], fma(Qc[0], mg[34], Q[34])))) + Qc[34]);
  }
  static constexpr int FLOPS_M2M = 438;
  __device__ __forceinline__ static void m2l_add(const double* r, const double* Q, double* local) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[56];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    const double sn2 = rinv2 * -0.5;
    const double sn3 = rinv2 * -0.3333333333333333;
    const double sn4 = rinv2 * -0.25;
    const double sn5 = rinv2 * -0.2;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    D[4] = (6.0 * r[0] * D[1] + 2.0 * D[0]) * sn2;
    D[5] = (3.0 * r[0] * D[2] + 3.0 * r[1] * D[1]) * sn2;
    D[6] = (3.0 * r[0] * D[3] + 3.0 * r[2] * D[1]) * sn2;
    D[7] = (6.0 * r[1] * D[2] + 2.0 * D[0]) * sn2;
    D[8] = (3.0 * r[1] * D[3] + 3.0 * r[2] * D[2]) * sn2;
    D[9] = (6.0 * r[2] * D[3] + 2.0 * D[0]) * sn2;
    D[10] = (15.0 * r[0] * D[4] + 12.0 * D[1]) * sn3;
    D[11] = (10.0 * r[0] * D[5] + 4.0 * D[2] + 5.0 * r[1] * D[4]) * sn3;
    D[12] = (10.0 * r[0] * D[6] + 4.0 * D[3] + 5.0 * r[2] * D[4]) * sn3;
    D[13] = (5.0 * r[0] * D[7] + 10.0 * r[1] * D[5] + 4.0 * D[1]) * sn3;
    D[14] = (5.0 * r[0] * D[8] + 5.0 * r[1] * D[6] + 5.0 * r[2] * D[5]) * sn3;
    D[15] = (5.0 * r[0] * D[9] + 10.0 * r[2] * D[6] + 4.0 * D[1]) * sn3;
    D[16] = (15.0 * r[1] * D[7] + 12.0 * D[2]) * sn3;
    D[17] = (10.0 * r[1] * D[8] + 4.0 * D[3] + 5.0 * r[2] * D[7]) * sn3;
    D[18] = (5.0 * r[1] * D[9] + 10.0 * r[2] * D[8] + 4.0 * D[2]) * sn3;
    D[19] = (15.0 * r[2] * D[9] + 12.0 * D[3]) * sn3;
    D[20] = (28.0 * r[0] * D[10] + 36.0 * D[4]) * sn4;
    D[21] = (21.0 * r[0] * D[11] + 18.0 * D[5] + 7.0 * r[1] * D[10]) * sn4;
    D[22] = (21.0 * r[0] * D[12] + 18.0 * D[6] + 7.0 * r[2] * D[10]) * sn4;
    D[23] = (14.0 * r[0] * D[13] + 6.0 * D[7] + 14.0 * r[1] * D[11] + 6.0 * D[4]) * sn4;
    D[24] = (14.0 * r[0] * D[14] + 6.0 * D[8] + 7.0 * r[1] * D[12] + 7.0 * r[2] * D[11]) * sn4;
    D[25] = (14.0 * r[0] * D[15] + 6.0 * D[9] + 14.0 * r[2] * D[12] + 6.0 * D[4]) * sn4;
    D[26] = (7.0 * r[0] * D[16] + 21.0 * r[1] * D[13] + 18.0 * D[5]) * sn4;
    D[27] = (7.0 * r[0] * D[17] + 14.0 * r[1] * D[14] + 6.0 * D[6] + 7.0 * r[2] * D[13]) * sn4;
    D[28] = (7.0 * r[0] * D[18] + 7.0 * r[1] * D[15] + 14.0 * r[2] * D[14] + 6.0 * D[5]) * sn4;
    D[29] = (7.0 * r[0] * D[19] + 21.0 * r[2] * D[15] + 18.0 * D[6]) * sn4;
    D[30] = (28.0 * r[1] * D[16] + 36.0 * D[7]) * sn4;
    D[31] = (21.0 * r[1] * D[17] + 18.0 * D[8] + 7.0 * r[2] * D[16]) * sn4;
    D[32] = (14.0 * r[1] * D[18] + 6.0 * D[9] + 14.0 * r[2] * D[17] + 6.0 * D[7]) * sn4;
    D[33] = (7.0 * r[1] * D[19] + 21.0 * r[2] * D[18] + 18.0 * D[8]) * sn4;
    D[34] = (28.0 * r[2] * D[19] + 36.0 * D[9]) * sn4;
    D[35] = (45.0 * r[0] * D[20] + 80.0 * D[10]) * sn5;
    D[36] = (36.0 * r[0] * D[21] + 48.0 * D[11] + 9.0 * r[1] * D[20]) * sn5;
    D[37] = (36.0 * r[0] * D[22] + 48.0 * D[12] + 9.0 * r[2] * D[20]) * sn5;
    D[38] = (27.0 * r[0] * D[23] + 24.0 * D[13] + 18.0 * r[1] * D[21] + 8.0 * D[10]) * sn5;
    D[39] = (27.0 * r[0] * D[24] + 24.0 * D[14] + 9.0 * r[1] * D[22] + 9.0 * r[2] * D[21]) * sn5;
    D[40] = (27.0 * r[0] * D[25] + 24.0 * D[15] + 18.0 * r[2] * D[22] + 8.0 * D[10]) * sn5;
    D[41] = (18.0 * r[0] * D[26] + 8.0 * D[16] + 27.0 * r[1] * D[23] + 24.0 * D[11]) * sn5;
    D[42] = (18.0 * r[0] * D[27] + 8.0 * D[17] + 18.0 * r[1] * D[24] + 8.0 * D[12] + 9.0 * r[2] * D[23]) * sn5;
    D[43] = (18.0 * r[0] * D[28] + 8.0 * D[18] + 9.0 * r[1] * D[25] + 18.0 * r[2] * D[24] + 8.0 * D[11]) * sn5;
    D[44] = (18.0 * r[0] * D[29] + 8.0 * D[19] + 27.0 * r[2] * D[25] + 24.0 * D[12]) * sn5;
    D[45] = (9.0 * r[0] * D[30] + 36.0 * r[1] * D[26] + 48.0 * D[13]) * sn5;
    D[46] = (9.0 * r[0] * D[31] + 27.0 * r[1] * D[27] + 24.0 * D[14] + 9.0 * r[2] * D[26]) * sn5;
    D[47] = (9.0 * r[0] * D[32] + 18.0 * r[1] * D[28] + 8.0 * D[15] + 18.0 * r[2] * D[27] + 8.0 * D[13]) * sn5;
    D[48] = (9.0 * r[0] * D[33] + 9.0 * r[1] * D[29] + 27.0 * r[2] * D[28] + 24.0 * D[14]) * sn5;
    D[49] = (9.0 * r[0] * D[34] + 36.0 * r[2] * D[29] + 48.0 * D[15]) * sn5;
    D[50] = (45.0 * r[1] * D[30] + 80.0 * D[16]) * sn5;
    D[51] = (36.0 * r[1] * D[31] + 48.0 * D[17] + 9.0 * r[2] * D[30]) * sn5;
    D[52] = (27.0 * r[1] * D[32] + 24.0 * D[18] + 18.0 * r[2] * D[31] + 8.0 * D[16]) * sn5;
    D[53] = (18.0 * r[1] * D[33] + 8.0 * D[19] + 27.0 * r[2] * D[32] + 24.0 * D[17]) * sn5;
    D[54] = (9.0 * r[1] * D[34] + 36.0 * r[2] * D[33] + 48.0 * D[18]) * sn5;
    D[55] = (45.0 * r[2] * D[34] + 80.0 * D[19]) * sn5;
    {
      double s = D[1] * Q[0];
      s = fma(D[4], Q[1], s);
      s = fma(D[5], Q[2], s);
      s = fma(D[6], Q[3], s);
      s = fma(D[10], Q[4], s);
      s = fma(D[11], Q[5], s);
      s = fma(D[12], Q[6], s);
      s = fma(D[13], Q[7], s);
      s = fma(D[14], Q[8], s);
      s = fma(D[15], Q[9], s);
      s = fma(D[20], Q[10], s);
      s = fma(D[21], Q[11], s);
      s = fma(D[22], Q[12], s);
      s = fma(D[23], Q[13], s);
      s = fma(D[24], Q[14], s);
      s = fma(D[25], Q[15], s);
      s = fma(D[26], Q[16], s);
      s = fma(D[27], Q[17], s);
      s = fma(D[28], Q[18], s);
      s = fma(D[29], Q[19], s);
      local[56] -= s;
      s = fma(D[35], Q[20], s);
      s = fma(D[36], Q[21], s);
      s = fma(D[37], Q[22], s);
      s = fma(D[38], Q[23], s);
      s = fma(D[39], Q[24], s);
      s = fma(D[40], Q[25], s);
      s = fma(D[41], Q[26], s);
      s = fma(D[42], Q[27], s);
      s = fma(D[43], Q[28], s);
      s = fma(D[44], Q[29], s);
      s = fma(D[45], Q[30], s);
      s = fma(D[46], Q[31], s);
      s = fma(D[47], Q[32], s);
      s = fma(D[48], Q[33], s);
      s = fma(D[49], Q[34], s);
      local[0] += s;
    }
    {
      double s = D[2] * Q[0];
      s = fma(D[5], Q[1], s);
      s = fma(D[7], Q[2], s);
      s = fma(D[8], Q[3], s);
      s = fma(D[11], Q[4], s);
      s = fma(D[13], Q[5], s);
      s = fma(D[14], Q[6], s);
      s = fma(D[16], Q[7], s);
      s = fma(D[17], Q[8], s);
      s = fma(D[18], Q[9], s);
      s = fma(D[21], Q[10], s);
      s = fma(D[23], Q[11], s);
      s = fma(D[24], Q[12], s);
      s = fma(D[26], Q[13], s);
      s = fma(D[27], Q[14], s);
      s = fma(D[28], Q[15], s);
      s = fma(D[30], Q[16], s);
      s = fma(D[31], Q[17], s);
      s = fma(D[32], Q[18], s);
      s = fma(D[33], Q[19], s);
      local[57] -= s;
      s = fma(D[36], Q[20], s);
      s = fma(D[38], Q[21], s);
      s = fma(D[39], Q[22], s);
      s = fma(D[41], Q[23], s);
      s = fma(D[42], Q[24], s);
      s = fma(D[43], Q[25], s);
      s = fma(D[45], Q[26], s);
      s = fma(D[46], Q[27], s);
      s = fma(D[47], Q[28], s);
      s = fma(D[48], Q[29], s);
      s = fma(D[50], Q[30], s);
      s = fma(D[51], Q[31], s);
      s = fma(D[52], Q[32], s);
      s = fma(D[53], Q[33], s);
      s = fma(D[54], Q[34], s);
      local[1] += s;
    }
    {
      double s = D[3] * Q[0];
      s = fma(D[6], Q[1], s);
      s = fma(D[8], Q[2], s);
      s = fma(D[9], Q[3], s);
      s = fma(D[12], Q[4], s);
      s = fma(D[14], Q[5], s);
      s = fma(D[15], Q[6], s);
      s = fma(D[17], Q[7], s);
      s = fma(D[18], Q[8], s);
      s = fma(D[19], Q[9], s);
      s = fma(D[22], Q[10], s);
      s = fma(D[24], Q[11], s);
      s = fma(D[25], Q[12], s);
      s = fma(D[27], Q[13], s);
      s = fma(D[28], Q[14], s);
      s = fma(D[29], Q[15], s);
      s = fma(D[31], Q[16], s);
      s = fma(D[32], Q[17], s);
      s = fma(D[33], Q[18], s);
      s = fma(D[34], Q[19], s);
      local[58] -= s;
      s = fma(D[37], Q[20], s);
      s = fma(D[39], Q[21], s);
      s = fma(D[40], Q[22], s);
      s = fma(D[42], Q[23], s);
      s = fma(D[43], Q[24], s);
      s = fma(D[44], Q[25], s);
      s = fma(D[46], Q[26], s);
      s = fma(D[47], Q[27], s);
      s = fma(D[48], Q[28], s);
      s = fma(D[49], Q[29], s);
      s = fma(D[51], Q[30], s);
      s = fma(D[52], Q[31], s);
      s = fma(D[53], Q[32], s);
      s = fma(D[54], Q[33], s);
      s = fma(D[55], Q[34], s);
      local[2] += s;
    }
    {
      double s = D[4] * Q[0];
      s = fma(D[10], Q[1], s);
      s = fma(D[11], Q[2], s);
      s = fma(D[12], Q[3], s);
      s = fma(D[20], Q[4], s);
      s = fma(D[21], Q[5], s);
      s = fma(D[22], Q[6], s);
      s = fma(D[23], Q[7], s);
      s = fma(D[24], Q[8], s);
      s = fma(D[25], Q[9], s);
      local[59] += s;
      s = fma(D[35], Q[10], s);
      s = fma(D[36], Q[11], s);
      s = fma(D[37], Q[12], s);
      s = fma(D[38], Q[13], s);
      s = fma(D[39], Q[14], s);
      s = fma(D[40], Q[15], s);
      s = fma(D[41], Q[16], s);
      s = fma(D[42], Q[17], s);
      s = fma(D[43], Q[18], s);
      s = fma(D[44], Q[19], s);
      local[3] -= s;
    }
    {
      double s = D[5] * Q[0];
      s = fma(D[11], Q[1], s);
      s = fma(D[13], Q[2], s);
      s = fma(D[14], Q[3], s);
      s = fma(D[21], Q[4], s);
      s = fma(D[23], Q[5], s);
      s = fma(D[24], Q[6], s);
      s = fma(D[26], Q[7], s);
      s = fma(D[27], Q[8], s);
      s = fma(D[28], Q[9], s);
      local[60] += s;
      s = fma(D[36], Q[10], s);
      s = fma(D[38], Q[11], s);
      s = fma(D[39], Q[12], s);
      s = fma(D[41], Q[13], s);
      s = fma(D[42], Q[14], s);
      s = fma(D[43], Q[15], s);
      s = fma(D[45], Q[16], s);
      s = fma(D[46], Q[17], s);
      s = fma(D[47], Q[18], s);
      s = fma(D[48], Q[19], s);
      local[4] -= s;
    }
    {
      double s = D[6] * Q[0];
      s = fma(D[12], Q[1], s);
      s = fma(D[14], Q[2], s);
      s = fma(D[15], Q[3], s);
      s = fma(D[22], Q[4], s);
      s = fma(D[24], Q[5], s);
      s = fma(D[25], Q[6], s);
      s = fma(D[27], Q[7], s);
      s = fma(D[28], Q[8], s);
      s = fma(D[29], Q[9], s);
      local[61] += s;
      s = fma(D[37], Q[10], s);
      s = fma(D[39], Q[11], s);
      s = fma(D[40], Q[12], s);
      s = fma(D[42], Q[13], s);
      s = fma(D[43], Q[14], s);
      s = fma(D[44], Q[15], s);
      s = fma(D[46], Q[16], s);
      s = fma(D[47], Q[17], s);
      s = fma(D[48], Q[18], s);
      s = fma(D[49], Q[19], s);
      local[5] -= s;
    }
    {
      double s = D[7] * Q[0];
      s = fma(D[13], Q[1], s);
      s = fma(D[16], Q[2], s);
      s = fma(D[17], Q[3], s);
      s = fma(D[23], Q[4], s);
      s = fma(D[26], Q[5], s);
      s = fma(D[27], Q[6], s);
      s = fma(D[30], Q[7], s);
      s = fma(D[31], Q[8], s);
      s = fma(D[32], Q[9], s);
      local[62] += s;
      s = fma(D[38], Q[10], s);
      s = fma(D[41], Q[11], s);
      s = fma(D[42], Q[12], s);
      s = fma(D[45], Q[13], s);
      s = fma(D[46], Q[14], s);
      s = fma(D[47], Q[15], s);
      s = fma(D[50], Q[16], s);
      s = fma(D[51], Q[17], s);
      s = fma(D[52], Q[18], s);
      s = fma(D[53], Q[19], s);
      local[6] -= s;
    }
    {
      double s = D[8] * Q[0];
      s = fma(D[14], Q[1], s);
      s = fma(D[17], Q[2], s);
      s = fma(D[18], Q[3], s);
      s = fma(D[24], Q[4], s);
      s = fma(D[27], Q[5], s);
      s = fma(D[28], Q[6], s);
      s = fma(D[31], Q[7], s);
      s = fma(D[32], Q[8], s);
      s = fma(D[33], Q[9], s);
      local[63] += s;
      s = fma(D[39], Q[10], s);
      s = fma(D[42], Q[11], s);
      s = fma(D[43], Q[12], s);
      s = fma(D[46], Q[13], s);
      s = fma(D[47], Q[14], s);
      s = fma(D[48], Q[15], s);
      s = fma(D[51], Q[16], s);
      s = fma(D[52], Q[17], s);
      s = fma(D[53], Q[18], s);
      s = fma(D[54], Q[19], s);
      local[7] -= s;
    }
    {
      double s = D[9] * Q[0];
      s = fma(D[15], Q[1], s);
      s = fma(D[18], Q[2], s);
      s = fma(D[19], Q[3], s);
      s = fma(D[25], Q[4], s);
      s = fma(D[28], Q[5], s);
      s = fma(D[29], Q[6], s);
      s = fma(D[32], Q[7], s);
      s = fma(D[33], Q[8], s);
      s = fma(D[34], Q[9], s);
      local[64] += s;
      s = fma(D[40], Q[10], s);
      s = fma(D[43], Q[11], s);
      s = fma(D[44], Q[12], s);
      s = fma(D[47], Q[13], s);
      s = fma(D[48], Q[14], s);
      s = fma(D[49], Q[15], s);
      s = fma(D[52], Q[16], s);
      s = fma(D[53], Q[17], s);
      s = fma(D[54], Q[18], s);
      s = fma(D[55], Q[19], s);
      local[8] -= s;
    }
    {
      double s = D[10] * Q[0];
      s = fma(D[20], Q[1], s);
      s = fma(D[21], Q[2], s);
      s = fma(D[22], Q[3], s);
      local[65] -= s;
      s = fma(D[35], Q[4], s);
      s = fma(D[36], Q[5], s);
      s = fma(D[37], Q[6], s);
      s = fma(D[38], Q[7], s);
      s = fma(D[39], Q[8], s);
      s = fma(D[40], Q[9], s);
      local[9] += s;
    }
    {
      double s = D[11] * Q[0];
      s = fma(D[21], Q[1], s);
      s = fma(D[23], Q[2], s);
      s = fma(D[24], Q[3], s);
      local[66] -= s;
      s = fma(D[36], Q[4], s);
      s = fma(D[38], Q[5], s);
      s = fma(D[39], Q[6], s);
      s = fma(D[41], Q[7], s);
      s = fma(D[42], Q[8], s);
      s = fma(D[43], Q[9], s);
      local[10] += s;
    }
    {
      double s = D[12] * Q[0];
      s = fma(D[22], Q[1], s);
      s = fma(D[24], Q[2], s);
      s = fma(D[25], Q[3], s);
      local[67] -= s;
      s = fma(D[37], Q[4], s);
      s = fma(D[39], Q[5], s);
      s = fma(D[40], Q[6], s);
      s = fma(D[42], Q[7], s);
      s = fma(D[43], Q[8], s);
      s = fma(D[44], Q[9], s);
      local[11] += s;
    }
    {
      double s = D[13] * Q[0];
      s = fma(D[23], Q[1], s);
      s = fma(D[26], Q[2], s);
      s = fma(D[27], Q[3], s);
      local[68] -= s;
      s = fma(D[38], Q[4], s);
      s = fma(D[41], Q[5], s);
      s = fma(D[42], Q[6], s);
      s = fma(D[45], Q[7], s);
      s = fma(D[46], Q[8], s);
      s = fma(D[47], Q[9], s);
      local[12] += s;
    }
    {
      double s = D[14] * Q[0];
      s = fma(D[24], Q[1], s);
      s = fma(D[27], Q[2], s);
      s = fma(D[28], Q[3], s);
      local[69] -= s;
      s = fma(D[39], Q[4], s);
      s = fma(D[42], Q[5], s);
      s = fma(D[43], Q[6], s);
      s = fma(D[46], Q[7], s);
      s = fma(D[47], Q[8], s);
      s = fma(D[48], Q[9], s);
      local[13] += s;
    }
    {
      double s = D[15] * Q[0];
      s = fma(D[25], Q[1], s);
      s = fma(D[28], Q[2], s);
      s = fma(D[29], Q[3], s);
      local[70] -= s;
      s = fma(D[40], Q[4], s);
      s = fma(D[43], Q[5], s);
      s = fma(D[44], Q[6], s);
      s = fma(D[47], Q[7], s);
      s = fma(D[48], Q[8], s);
      s = fma(D[49], Q[9], s);
      local[14] += s;
    }
    {
      double s = D[16] * Q[0];
      s = fma(D[26], Q[1], s);
      s = fma(D[30], Q[2], s);
      s = fma(D[31], Q[3], s);
      local[71] -= s;
      s = fma(D[41], Q[4], s);
      s = fma(D[45], Q[5], s);
      s = fma(D[46], Q[6], s);
      s = fma(D[50], Q[7], s);
      s = fma(D[51], Q[8], s);
      s = fma(D[52], Q[9], s);
      local[15] += s;
    }
    {
      double s = D[17] * Q[0];
      s = fma(D[27], Q[1], s);
      s = fma(D[31], Q[2], s);
      s = fma(D[32], Q[3], s);
      local[72] -= s;
      s = fma(D[42], Q[4], s);
      s = fma(D[46], Q[5], s);
      s = fma(D[47], Q[6], s);
      s = fma(D[51], Q[7], s);
      s = fma(D[52], Q[8], s);
      s = fma(D[53], Q[9], s);
      local[16] += s;
    }
    {
      double s = D[18] * Q[0];
      s = fma(D[28], Q[1], s);
      s = fma(D[32], Q[2], s);
      s = fma(D[33], Q[3], s);
      local[73] -= s;
      s = fma(D[43], Q[4], s);
      s = fma(D[47], Q[5], s);
      s = fma(D[48], Q[6], s);
      s = fma(D[52], Q[7], s);
      s = fma(D[53], Q[8], s);
      s = fma(D[54], Q[9], s);
      local[17] += s;
    }
    {
      double s = D[19] * Q[0];
      s = fma(D[29], Q[1], s);
      s = fma(D[33], Q[2], s);
      s = fma(D[34], Q[3], s);
      local[74] -= s;
      s = fma(D[44], Q[4], s);
      s = fma(D[48], Q[5], s);
      s = fma(D[49], Q[6], s);
      s = fma(D[53], Q[7], s);
      s = fma(D[54], Q[8], s);
      s = fma(D[55], Q[9], s);
      local[18] += s;
    }
    {
      double s = D[20] * Q[0];
      local[75] += s;
      s = fma(D[35], Q[1], s);
      s = fma(D[36], Q[2], s);
      s = fma(D[37], Q[3], s);
      local[19] -= s;
    }
    {
      double s = D[21] * Q[0];
      local[76] += s;
      s = fma(D[36], Q[1], s);
      s = fma(D[38], Q[2], s);
      s = fma(D[39], Q[3], s);
      local[20] -= s;
    }
    {
      double s = D[22] * Q[0];
      local[77] += s;
      s = fma(D[37], Q[1], s);
      s = fma(D[39], Q[2], s);
      s = fma(D[40], Q[3], s);
      local[21] -= s;
    }
    {
      double s = D[23] * Q[0];
      local[78] += s;
      s = fma(D[38], Q[1], s);
      s = fma(D[41], Q[2], s);
      s = fma(D[42], Q[3], s);
      local[22] -= s;
    }
    {
      double s = D[24] * Q[0];
      local[79] += s;
      s = fma(D[39], Q[1], s);
      s = fma(D[42], Q[2], s);
      s = fma(D[43], Q[3], s);
      local[23] -= s;
    }
    {
      double s = D[25] * Q[0];
      local[80] += s;
      s = fma(D[40], Q[1], s);
      s = fma(D[43], Q[2], s);
      s = fma(D[44], Q[3], s);
      local[24] -= s;
    }
    {
      double s = D[26] * Q[0];
      local[81] += s;
      s = fma(D[41], Q[1], s);
      s = fma(D[45], Q[2], s);
      s = fma(D[46], Q[3], s);
      local[25] -= s;
    }
    {
      double s = D[27] * Q[0];
      local[82] += s;
      s = fma(D[42], Q[1], s);
      s = fma(D[46], Q[2], s);
      s = fma(D[47], Q[3], s);
      local[26] -= s;
    }
    {
      double s = D[28] * Q[0];
      local[83] += s;
      s = fma(D[43], Q[1], s);
      s = fma(D[47], Q[2], s);
      s = fma(D[48], Q[3], s);
      local[27] -= s;
    }
    {
      double s = D[29] * Q[0];
      local[84] += s;
      s = fma(D[44], Q[1], s);
      s = fma(D[48], Q[2], s);
      s = fma(D[49], Q[3], s);
      local[28] -= s;
    }
    {
      double s = D[30] * Q[0];
      local[85] += s;
      s = fma(D[45], Q[1], s);
      s = fma(D[50], Q[2], s);
      s = fma(D[51], Q[3], s);
      local[29] -= s;
    }
    {
      double s = D[31] * Q[0];
      local[86] += s;
      s = fma(D[46], Q[1], s);
      s = fma(D[51], Q[2], s);
      s = fma(D[52], Q[3], s);
      local[30] -= s;
    }
    {
      double s = D[32] * Q[0];
      local[87] += s;
      s = fma(D[47], Q[1], s);
      s = fma(D[52], Q[2], s);
      s = fma(D[53], Q[3], s);
      local[31] -= s;
    }
    {
      double s = D[33] * Q[0];
      local[88] += s;
      s = fma(D[48], Q[1], s);
      s = fma(D[53], Q[2], s);
      s = fma(D[54], Q[3], s);
      local[32] -= s;
    }
    {
      double s = D[34] * Q[0];
      local[89] += s;
      s = fma(D[49], Q[1], s);
      s = fma(D[54], Q[2], s);
      s = fma(D[55], Q[3], s);
      local[33] -= s;
    }
    {
      double s = D[35] * Q[0];
      local[34] += s;
    }
    {
      double s = D[36] * Q[0];
      local[35] += s;
    }
    {
      double s = D[37] * Q[0];
      local[36] += s;
    }
    {
      double s = D[38] * Q[0];
      local[37] += s;
    }
    {
      double s = D[39] * Q[0];
      local[38] += s;
    }
    {
      double s = D[40] * Q[0];
      local[39] += s;
    }
    {
      double s = D[41] * Q[0];
      local[40] += s;
    }
    {
      double s = D[42] * Q[0];
      local[41] += s;
    }
    {
      double s = D[43] * Q[0];
      local[42] += s;
    }
    {
      double s = D[44] * Q[0];
      local[43] += s;
    }
    {
      double s = D[45] * Q[0];
      local[44] += s;
    }
    {
      double s = D[46] * Q[0];
      local[45] += s;
    }
    {
      double s = D[47] * Q[0];
      local[46] += s;
    }
    {
      double s = D[48] * Q[0];
      local[47] += s;
    }
    {
      double s = D[49] * Q[0];
      local[48] += s;
    }
    {
      double s = D[50] * Q[0];
      local[49] += s;
    }
    {
      double s = D[51] * Q[0];
      local[50] += s;
    }
    {
      double s = D[52] * Q[0];
      local[51] += s;
    }
    {
      double s = D[53] * Q[0];
      local[52] += s;
    }
    {
      double s = D[54] * Q[0];
      local[53] += s;
    }
    {
      double s = D[55] * Q[0];
      local[54] += s;
    }
    {
      double s = D[0] * Q[0];
      s = fma(D[1], Q[1], s);
      s = fma(D[2], Q[2], s);
      s = fma(D[3], Q[3], s);
      s = fma(D[4], Q[4], s);
      s = fma(D[5], Q[5], s);
      s = fma(D[6], Q[6], s);
      s = fma(D[7], Q[7], s);
      s = fma(D[8], Q[8], s);
      s = fma(D[9], Q[9], s);
      s = fma(D[10], Q[10], s);
      s = fma(D[11], Q[11], s);
      s = fma(D[12], Q[12], s);
      s = fma(D[13], Q[13], s);
      s = fma(D[14], Q[14], s);
      s = fma(D[15], Q[15], s);
      s = fma(D[16], Q[16], s);
      s = fma(D[17], Q[17], s);
      s = fma(D[18], Q[18], s);
      s = fma(D[19], Q[19], s);
      s = fma(D[20], Q[20], s);
      s = fma(D[21], Q[21], s);
      s = fma(D[22], Q[22], s);
      s = fma(D[23], Q[23], s);
      s = fma(D[24], Q[24], s);
      s = fma(D[25], Q[25], s);
      s = fma(D[26], Q[26], s);
      s = fma(D[27], Q[27], s);
      s = fma(D[28], Q[28], s);
      s = fma(D[29], Q[29], s);
      s = fma(D[30], Q[30], s);
      s = fma(D[31], Q[31], s);
      s = fma(D[32], Q[32], s);
      s = fma(D[33], Q[33], s);
      s = fma(D[34], Q[34], s);
      local[55] += s;
    }
  }
  static constexpr int FLOPS_M2L = 1362;  // + one rsqrt
  __device__ __forceinline__ static void m2l_add_f32(const float* r, const float* Q, double* local, bool ok = true) {
    const float r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const float rinv = ok ? __frsqrt_rn(r2) : 0.0f;
    const float rinv2 = rinv * rinv;
    float D[56];
    D[0] = rinv;
    const float sn1 = rinv2 * -1.0f;
    const float sn2 = rinv2 * -0.5f;
    const float sn3 = rinv2 * -0.3333333333333333f;
    const float sn4 = rinv2 * -0.25f;
    const float sn5 = rinv2 * -0.2f;
    D[1] = (1.0f * r[0] * D[0]) * sn1;
    D[2] = (1.0f * r[1] * D[0]) * sn1;
    D[3] = (1.0f * r[2] * D[0]) * sn1;
    D[4] = (6.0f * r[0] * D[1] + 2.0f * D[0]) * sn2;
    D[5] = (3.0f * r[0] * D[2] + 3.0f * r[1] * D[1]) * sn2;
    D[6] = (3.0f * r[0] * D[3] + 3.0f * r[2] * D[1]) * sn2;
    D[7] = (6.0f * r[1] * D[2] + 2.0f * D[0]) * sn2;
    D[8] = (3.0f * r[1] * D[3] + 3.0f * r[2] * D[2]) * sn2;
    D[9] = (6.0f * r[2] * D[3] + 2.0f * D[0]) * sn2;
    D[10] = (15.0f * r[0] * D[4] + 12.0f * D[1]) * sn3;
    D[11] = (10.0f * r[0] * D[5] + 4.0f * D[2] + 5.0f * r[1] * D[4]) * sn3;
    D[12] = (10.0f * r[0] * D[6] + 4.0f * D[3] + 5.0f * r[2] * D[4]) * sn3;
    D[13] = (5.0f * r[0] * D[7] + 10.0f * r[1] * D[5] + 4.0f * D[1]) * sn3;
    D[14] = (5.0f * r[0] * D[8] + 5.0f * r[1] * D[6] + 5.0f * r[2] * D[5]) * sn3;
    D[15] = (5.0f * r[0] * D[9] + 10.0f * r[2] * D[6] + 4.0f * D[1]) * sn3;
    D[16] = (15.0f * r[1] * D[7] + 12.0f * D[2]) * sn3;
    D[17] = (10.0f * r[1] * D[8] + 4.0f * D[3] + 5.0f * r[2] * D[7]) * sn3;
    D[18] = (5.0f * r[1] * D[9] + 10.0f * r[2] * D[8] + 4.0f * D[2]) * sn3;
    D[19] = (15.0f * r[2] * D[9] + 12.0f * D[3]) * sn3;
    D[20] = (28.0f * r[0] * D[10] + 36.0f * D[4]) * sn4;
    D[21] = (21.0f * r[0] * D[11] + 18.0f * D[5] + 7.0f * r[1] * D[10]) * sn4;
    D[22] = (21.0f * r[0] * D[12] + 18.0f * D[6] + 7.0f * r[2] * D[10]) * sn4;
    D[23] = (14.0f * r[0] * D[13] + 6.0f * D[7] + 14.0f * r[1] * D[11] + 6.0f * D[4]) * sn4;
    D[24] = (14.0f * r[0] * D[14] + 6.0f * D[8] + 7.0f * r[1] * D[12] + 7.0f * r[2] * D[11]) * sn4;
    D[25] = (14.0f * r[0] * D[15] + 6.0f * D[9] + 14.0f * r[2] * D[12] + 6.0f * D[4]) * sn4;
    D[26] = (7.0f * r[0] * D[16] + 21.0f * r[1] * D[13] + 18.0f * D[5]) * sn4;
    D[27] = (7.0f * r[0] * D[17] + 14.0f * r[1] * D[14] + 6.0f * D[6] + 7.0f * r[2] * D[13]) * sn4;
    D[28] = (7.0f * r[0] * D[18] + 7.0f * r[1] * D[15] + 14.0f * r[2] * D[14] + 6.0f * D[5]) * sn4;
    D[29] = (7.0f * r[0] * D[19] + 21.0f * r[2] * D[15] + 18.0f * D[6]) * sn4;
    D[30] = (28.0f * r[1] * D[16] + 36.0f * D[7]) * sn4;
    D[31] = (21.0f * r[1] * D[17] + 18.0f * D[8] + 7.0f * r[2] * D[16]) * sn4;
    D[32] = (14.0f * r[1] * D[18] + 6.0f * D[9] + 14.0f * r[2] * D[17] + 6.0f * D[7]) * sn4;
    D[33] = (7.0f * r[1] * D[19] + 21.0f * r[2] * D[18] + 18.0f * D[8]) * sn4;
    D[34] = (28.0f * r[2] * D[19] + 36.0f * D[9]) * sn4;
    D[35] = (45.0f * r[0] * D[20] + 80.0f * D[10]) * sn5;
    D[36] = (36.0f * r[0] * D[21] + 48.0f * D[11] + 9.0f * r[1] * D[20]) * sn5;
    D[37] = (36.0f * r[0] * D[22] + 48.0f * D[12] + 9.0f * r[2] * D[20]) * sn5;
    D[38] = (27.0f * r[0] * D[23] + 24.0f * D[13] + 18.0f * r[1] * D[21] + 8.0f * D[10]) * sn5;
    D[39] = (27.0f * r[0] * D[24] + 24.0f * D[14] + 9.0f * r[1] * D[22] + 9.0f * r[2] * D[21]) * sn5;
    D[40] = (27.0f * r[0] * D[25] + 24.0f * D[15] + 18.0f * r[2] * D[22] + 8.0f * D[10]) * sn5;
    D[41] = (18.0f * r[0] * D[26] + 8.0f * D[16] + 27.0f * r[1] * D[23] + 24.0f * D[11]) * sn5;
    D[42] = (18.0f * r[0] * D[27] + 8.0f * D[17] + 18.0f * r[1] * D[24] + 8.0f * D[12] + 9.0f * r[2] * D[23]) * sn5;
    D[43] = (18.0f * r[0] * D[28] + 8.0f * D[18] + 9.0f * r[1] * D[25] + 18.0f * r[2] * D[24] + 8.0f * D[11]) * sn5;
    D[44] = (18.0f * r[0] * D[29] + 8.0f * D[19] + 27.0f * r[2] * D[25] + 24.0f * D[12]) * sn5;
    D[45] = (9.0f * r[0] * D[30] + 36.0f * r[1] * D[26] + 48.0f * D[13]) * sn5;
    D[46] = (9.0f * r[0] * D[31] + 27.0f * r[1] * D[27] + 24.0f * D[14] + 9.0f * r[2] * D[26]) * sn5;
    D[47] = (9.0f * r[0] * D[32] + 18.0f * r[1] * D[28] + 8.0f * D[15] + 18.0f * r[2] * D[27] + 8.0f * D[13]) * sn5;
    D[48] = (9.0f * r[0] * D[33] + 9.0f * r[1] * D[29] + 27.0f * r[2] * D[28] + 24.0f * D[14]) * sn5;
    D[49] = (9.0f * r[0] * D[34] + 36.0f * r[2] * D[29] + 48.0f * D[15]) * sn5;
    D[50] = (45.0f * r[1] * D[30] + 80.0f * D[16]) * sn5;
    D[51] = (36.0f * r[1] * D[31] + 48.0f * D[17] + 9.0f * r[2] * D[30]) * sn5;
    D[52] = (27.0f * r[1] * D[32] + 24.0f * D[18] + 18.0f * r[2] * D[31] + 8.0f * D[16]) * sn5;
    D[53] = (18.0f * r[1] * D[33] + 8.0f * D[19] + 27.0f * r[2] * D[32] + 24.0f * D[17]) * sn5;
    D[54] = (9.0f * r[1] * D[34] + 36.0f * r[2] * D[33] + 48.0f * D[18]) * sn5;
    D[55] = (45.0f * r[2] * D[34] + 80.0f * D[19]) * sn5;
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[1] * Q[0];
      s = fmaf(D[4], Q[1], s);
      s = fmaf(D[5], Q[2], s);
      s = fmaf(D[6], Q[3], s);
      s = fmaf(D[10], Q[4], s);
      s = fmaf(D[11], Q[5], s);
      s = fmaf(D[12], Q[6], s);
      s = fmaf(D[13], Q[7], s);
      s = fmaf(D[14], Q[8], s);
      s = fmaf(D[15], Q[9], s);
      s = fmaf(D[20], Q[10], s);
      s = fmaf(D[21], Q[11], s);
      s = fmaf(D[22], Q[12], s);
      s = fmaf(D[23], Q[13], s);
      s = fmaf(D[24], Q[14], s);
      s = fmaf(D[25], Q[15], s);
      s = fmaf(D[26], Q[16], s);
      s = fmaf(D[27], Q[17], s);
      s = fmaf(D[28], Q[18], s);
      s = fmaf(D[29], Q[19], s);
      local[56] -= (double)s;
      s = fmaf(D[35], Q[20], s);
      s = fmaf(D[36], Q[21], s);
      s = fmaf(D[37], Q[22], s);
      s = fmaf(D[38], Q[23], s);
      s = fmaf(D[39], Q[24], s);
      s = fmaf(D[40], Q[25], s);
      s = fmaf(D[41], Q[26], s);
      s = fmaf(D[42], Q[27], s);
      s = fmaf(D[43], Q[28], s);
      s = fmaf(D[44], Q[29], s);
      s = fmaf(D[45], Q[30], s);
      s = fmaf(D[46], Q[31], s);
      s = fmaf(D[47], Q[32], s);
      s = fmaf(D[48], Q[33], s);
      s = fmaf(D[49], Q[34], s);
      local[0] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[2] * Q[0];
      s = fmaf(D[5], Q[1], s);
      s = fmaf(D[7], Q[2], s);
      s = fmaf(D[8], Q[3], s);
      s = fmaf(D[11], Q[4], s);
      s = fmaf(D[13], Q[5], s);
      s = fmaf(D[14], Q[6], s);
      s = fmaf(D[16], Q[7], s);
      s = fmaf(D[17], Q[8], s);
      s = fmaf(D[18], Q[9], s);
      s = fmaf(D[21], Q[10], s);
      s = fmaf(D[23], Q[11], s);
      s = fmaf(D[24], Q[12], s);
      s = fmaf(D[26], Q[13], s);
      s = fmaf(D[27], Q[14], s);
      s = fmaf(D[28], Q[15], s);
      s = fmaf(D[30], Q[16], s);
      s = fmaf(D[31], Q[17], s);
      s = fmaf(D[32], Q[18], s);
      s = fmaf(D[33], Q[19], s);
      local[57] -= (double)s;
      s = fmaf(D[36], Q[20], s);
      s = fmaf(D[38], Q[21], s);
      s = fmaf(D[39], Q[22], s);
      s = fmaf(D[41], Q[23], s);
      s = fmaf(D[42], Q[24], s);
      s = fmaf(D[43], Q[25], s);
      s = fmaf(D[45], Q[26], s);
      s = fmaf(D[46], Q[27], s);
      s = fmaf(D[47], Q[28], s);
      s = fmaf(D[48], Q[29], s);
      s = fmaf(D[50], Q[30], s);
      s = fmaf(D[51], Q[31], s);
      s = fmaf(D[52], Q[32], s);
      s = fmaf(D[53], Q[33], s);
      s = fmaf(D[54], Q[34], s);
      local[1] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[3] * Q[0];
      s = fmaf(D[6], Q[1], s);
      s = fmaf(D[8], Q[2], s);
      s = fmaf(D[9], Q[3], s);
      s = fmaf(D[12], Q[4], s);
      s = fmaf(D[14], Q[5], s);
      s = fmaf(D[15], Q[6], s);
      s = fmaf(D[17], Q[7], s);
      s = fmaf(D[18], Q[8], s);
      s = fmaf(D[19], Q[9], s);
      s = fmaf(D[22], Q[10], s);
      s = fmaf(D[24], Q[11], s);
      s = fmaf(D[25], Q[12], s);
      s = fmaf(D[27], Q[13], s);
      s = fmaf(D[28], Q[14], s);
      s = fmaf(D[29], Q[15], s);
      s = fmaf(D[31], Q[16], s);
      s = fmaf(D[32], Q[17], s);
      s = fmaf(D[33], Q[18], s);
      s = fmaf(D[34], Q[19], s);
      local[58] -= (double)s;
      s = fmaf(D[37], Q[20], s);
      s = fmaf(D[39], Q[21], s);
      s = fmaf(D[40], Q[22], s);
      s = fmaf(D[42], Q[23], s);
      s = fmaf(D[43], Q[24], s);
      s = fmaf(D[44], Q[25], s);
      s = fmaf(D[46], Q[26], s);
      s = fmaf(D[47], Q[27], s);
      s = fmaf(D[48], Q[28], s);
      s = fmaf(D[49], Q[29], s);
      s = fmaf(D[51], Q[30], s);
      s = fmaf(D[52], Q[31], s);
      s = fmaf(D[53], Q[32], s);
      s = fmaf(D[54], Q[33], s);
      s = fmaf(D[55], Q[34], s);
      local[2] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[4] * Q[0];
      s = fmaf(D[10], Q[1], s);
      s = fmaf(D[11], Q[2], s);
      s = fmaf(D[12], Q[3], s);
      s = fmaf(D[20], Q[4], s);
      s = fmaf(D[21], Q[5], s);
      s = fmaf(D[22], Q[6], s);
      s = fmaf(D[23], Q[7], s);
      s = fmaf(D[24], Q[8], s);
      s = fmaf(D[25], Q[9], s);
      local[59] += (double)s;
      s = fmaf(D[35], Q[10], s);
      s = fmaf(D[36], Q[11], s);
      s = fmaf(D[37], Q[12], s);
      s = fmaf(D[38], Q[13], s);
      s = fmaf(D[39], Q[14], s);
      s = fmaf(D[40], Q[15], s);
      s = fmaf(D[41], Q[16], s);
      s = fmaf(D[42], Q[17], s);
      s = fmaf(D[43], Q[18], s);
      s = fmaf(D[44], Q[19], s);
      local[3] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[5] * Q[0];
      s = fmaf(D[11], Q[1], s);
      s = fmaf(D[13], Q[2], s);
      s = fmaf(D[14], Q[3], s);
      s = fmaf(D[21], Q[4], s);
      s = fmaf(D[23], Q[5], s);
      s = fmaf(D[24], Q[6], s);
      s = fmaf(D[26], Q[7], s);
      s = fmaf(D[27], Q[8], s);
      s = fmaf(D[28], Q[9], s);
      local[60] += (double)s;
      s = fmaf(D[36], Q[10], s);
      s = fmaf(D[38], Q[11], s);
      s = fmaf(D[39], Q[12], s);
      s = fmaf(D[41], Q[13], s);
      s = fmaf(D[42], Q[14], s);
      s = fmaf(D[43], Q[15], s);
      s = fmaf(D[45], Q[16], s);
      s = fmaf(D[46], Q[17], s);
      s = fmaf(D[47], Q[18], s);
      s = fmaf(D[48], Q[19], s);
      local[4] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[6] * Q[0];
      s = fmaf(D[12], Q[1], s);
      s = fmaf(D[14], Q[2], s);
      s = fmaf(D[15], Q[3], s);
      s = fmaf(D[22], Q[4], s);
      s = fmaf(D[24], Q[5], s);
      s = fmaf(D[25], Q[6], s);
      s = fmaf(D[27], Q[7], s);
      s = fmaf(D[28], Q[8], s);
      s = fmaf(D[29], Q[9], s);
      local[61] += (double)s;
      s = fmaf(D[37], Q[10], s);
      s = fmaf(D[39], Q[11], s);
      s = fmaf(D[40], Q[12], s);
      s = fmaf(D[42], Q[13], s);
      s = fmaf(D[43], Q[14], s);
      s = fmaf(D[44], Q[15], s);
      s = fmaf(D[46], Q[16], s);
      s = fmaf(D[47], Q[17], s);
      s = fmaf(D[48], Q[18], s);
      s = fmaf(D[49], Q[19], s);
      local[5] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[7] * Q[0];
      s = fmaf(D[13], Q[1], s);
      s = fmaf(D[16], Q[2], s);
      s = fmaf(D[17], Q[3], s);
      s = fmaf(D[23], Q[4], s);
      s = fmaf(D[26], Q[5], s);
      s = fmaf(D[27], Q[6], s);
      s = fmaf(D[30], Q[7], s);
      s = fmaf(D[31], Q[8], s);
      s = fmaf(D[32], Q[9], s);
      local[62] += (double)s;
      s = fmaf(D[38], Q[10], s);
      s = fmaf(D[41], Q[11], s);
      s = fmaf(D[42], Q[12], s);
      s = fmaf(D[45], Q[13], s);
      s = fmaf(D[46], Q[14], s);
      s = fmaf(D[47], Q[15], s);
      s = fmaf(D[50], Q[16], s);
      s = fmaf(D[51], Q[17], s);
      s = fmaf(D[52], Q[18], s);
      s = fmaf(D[53], Q[19], s);
      local[6] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[8] * Q[0];
      s = fmaf(D[14], Q[1], s);
      s = fmaf(D[17], Q[2], s);
      s = fmaf(D[18], Q[3], s);
      s = fmaf(D[24], Q[4], s);
      s = fmaf(D[27], Q[5], s);
      s = fmaf(D[28], Q[6], s);
      s = fmaf(D[31], Q[7], s);
      s = fmaf(D[32], Q[8], s);
      s = fmaf(D[33], Q[9], s);
      local[63] += (double)s;
      s = fmaf(D[39], Q[10], s);
      s = fmaf(D[42], Q[11], s);
      s = fmaf(D[43], Q[12], s);
      s = fmaf(D[46], Q[13], s);
      s = fmaf(D[47], Q[14], s);
      s = fmaf(D[48], Q[15], s);
      s = fmaf(D[51], Q[16], s);
      s = fmaf(D[52], Q[17], s);
      s = fmaf(D[53], Q[18], s);
      s = fmaf(D[54], Q[19], s);
      local[7] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[9] * Q[0];
      s = fmaf(D[15], Q[1], s);
      s = fmaf(D[18], Q[2], s);
      s = fmaf(D[19], Q[3], s);
      s = fmaf(D[25], Q[4], s);
      s = fmaf(D[28], Q[5], s);
      s = fmaf(D[29], Q[6], s);
      s = fmaf(D[32], Q[7], s);
      s = fmaf(D[33], Q[8], s);
      s = fmaf(D[34], Q[9], s);
      local[64] += (double)s;
      s = fmaf(D[40], Q[10], s);
      s = fmaf(D[43], Q[11], s);
      s = fmaf(D[44], Q[12], s);
      s = fmaf(D[47], Q[13], s);
      s = fmaf(D[48], Q[14], s);
      s = fmaf(D[49], Q[15], s);
      s = fmaf(D[52], Q[16], s);
      s = fmaf(D[53], Q[17], s);
      s = fmaf(D[54], Q[18], s);
      s = fmaf(D[55], Q[19], s);
      local[8] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[10] * Q[0];
      s = fmaf(D[20], Q[1], s);
      s = fmaf(D[21], Q[2], s);
      s = fmaf(D[22], Q[3], s);
      local[65] -= (double)s;
      s = fmaf(D[35], Q[4], s);
      s = fmaf(D[36], Q[5], s);
      s = fmaf(D[37], Q[6], s);
      s = fmaf(D[38], Q[7], s);
      s = fmaf(D[39], Q[8], s);
      s = fmaf(D[40], Q[9], s);
      local[9] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[11] * Q[0];
      s = fmaf(D[21], Q[1], s);
      s = fmaf(D[23], Q[2], s);
      s = fmaf(D[24], Q[3], s);
      local[66] -= (double)s;
      s = fmaf(D[36], Q[4], s);
      s = fmaf(D[38], Q[5], s);
      s = fmaf(D[39], Q[6], s);
      s = fmaf(D[41], Q[7], s);
      s = fmaf(D[42], Q[8], s);
      s = fmaf(D[43], Q[9], s);
      local[10] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[12] * Q[0];
      s = fmaf(D[22], Q[1], s);
      s = fmaf(D[24], Q[2], s);
      s = fmaf(D[25], Q[3], s);
      local[67] -= (double)s;
      s = fmaf(D[37], Q[4], s);
      s = fmaf(D[39], Q[5], s);
      s = fmaf(D[40], Q[6], s);
      s = fmaf(D[42], Q[7], s);
      s = fmaf(D[43], Q[8], s);
      s = fmaf(D[44], Q[9], s);
      local[11] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[13] * Q[0];
      s = fmaf(D[23], Q[1], s);
      s = fmaf(D[26], Q[2], s);
      s = fmaf(D[27], Q[3], s);
      local[68] -= (double)s;
      s = fmaf(D[38], Q[4], s);
      s = fmaf(D[41], Q[5], s);
      s = fmaf(D[42], Q[6], s);
      s = fmaf(D[45], Q[7], s);
      s = fmaf(D[46], Q[8], s);
      s = fmaf(D[47], Q[9], s);
      local[12] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[14] * Q[0];
      s = fmaf(D[24], Q[1], s);
      s = fmaf(D[27], Q[2], s);
      s = fmaf(D[28], Q[3], s);
      local[69] -= (double)s;
      s = fmaf(D[39], Q[4], s);
      s = fmaf(D[42], Q[5], s);
      s = fmaf(D[43], Q[6], s);
      s = fmaf(D[46], Q[7], s);
      s = fmaf(D[47], Q[8], s);
      s = fmaf(D[48], Q[9], s);
      local[13] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[15] * Q[0];
      s = fmaf(D[25], Q[1], s);
      s = fmaf(D[28], Q[2], s);
      s = fmaf(D[29], Q[3], s);
      local[70] -= (double)s;
      s = fmaf(D[40], Q[4], s);
      s = fmaf(D[43], Q[5], s);
      s = fmaf(D[44], Q[6], s);
      s = fmaf(D[47], Q[7], s);
      s = fmaf(D[48], Q[8], s);
      s = fmaf(D[49], Q[9], s);
      local[14] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[16] * Q[0];
      s = fmaf(D[26], Q[1], s);
      s = fmaf(D[30], Q[2], s);
      s = fmaf(D[31], Q[3], s);
      local[71] -= (double)s;
      s = fmaf(D[41], Q[4], s);
      s = fmaf(D[45], Q[5], s);
      s = fmaf(D[46], Q[6], s);
      s = fmaf(D[50], Q[7], s);
      s = fmaf(D[51], Q[8], s);
      s = fmaf(D[52], Q[9], s);
      local[15] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[17] * Q[0];
      s = fmaf(D[27], Q[1], s);
      s = fmaf(D[31], Q[2], s);
      s = fmaf(D[32], Q[3], s);
      local[72] -= (double)s;
      s = fmaf(D[42], Q[4], s);
      s = fmaf(D[46], Q[5], s);
      s = fmaf(D[47], Q[6], s);
      s = fmaf(D[51], Q[7], s);
      s = fmaf(D[52], Q[8], s);
      s = fmaf(D[53], Q[9], s);
      local[16] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[18] * Q[0];
      s = fmaf(D[28], Q[1], s);
      s = fmaf(D[32], Q[2], s);
      s = fmaf(D[33], Q[3], s);
      local[73] -= (double)s;
      s = fmaf(D[43], Q[4], s);
      s = fmaf(D[47], Q[5], s);
      s = fmaf(D[48], Q[6], s);
      s = fmaf(D[52], Q[7], s);
      s = fmaf(D[53], Q[8], s);
      s = fmaf(D[54], Q[9], s);
      local[17] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[19] * Q[0];
      s = fmaf(D[29], Q[1], s);
      s = fmaf(D[33], Q[2], s);
      s = fmaf(D[34], Q[3], s);
      local[74] -= (double)s;
      s = fmaf(D[44], Q[4], s);
      s = fmaf(D[48], Q[5], s);
      s = fmaf(D[49], Q[6], s);
      s = fmaf(D[53], Q[7], s);
      s = fmaf(D[54], Q[8], s);
      s = fmaf(D[55], Q[9], s);
      local[18] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[20] * Q[0];
      local[75] += (double)s;
      s = fmaf(D[35], Q[1], s);
      s = fmaf(D[36], Q[2], s);
      s = fmaf(D[37], Q[3], s);
      local[19] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[21] * Q[0];
      local[76] += (double)s;
      s = fmaf(D[36], Q[1], s);
      s = fmaf(D[38], Q[2], s);
      s = fmaf(D[39], Q[3], s);
      local[20] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[22] * Q[0];
      local[77] += (double)s;
      s = fmaf(D[37], Q[1], s);
      s = fmaf(D[39], Q[2], s);
      s = fmaf(D[40], Q[3], s);
      local[21] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[23] * Q[0];
      local[78] += (double)s;
      s = fmaf(D[38], Q[1], s);
      s = fmaf(D[41], Q[2], s);
      s = fmaf(D[42], Q[3], s);
      local[22] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[24] * Q[0];
      local[79] += (double)s;
      s = fmaf(D[39], Q[1], s);
      s = fmaf(D[42], Q[2], s);
      s = fmaf(D[43], Q[3], s);
      local[23] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[25] * Q[0];
      local[80] += (double)s;
      s = fmaf(D[40], Q[1], s);
      s = fmaf(D[43], Q[2], s);
      s = fmaf(D[44], Q[3], s);
      local[24] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[26] * Q[0];
      local[81] += (double)s;
      s = fmaf(D[41], Q[1], s);
      s = fmaf(D[45], Q[2], s);
      s = fmaf(D[46], Q[3], s);
      local[25] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[27] * Q[0];
      local[82] += (double)s;
      s = fmaf(D[42], Q[1], s);
      s = fmaf(D[46], Q[2], s);
      s = fmaf(D[47], Q[3], s);
      local[26] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[28] * Q[0];
      local[83] += (double)s;
      s = fmaf(D[43], Q[1], s);
      s = fmaf(D[47], Q[2], s);
      s = fmaf(D[48], Q[3], s);
      local[27] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[29] * Q[0];
      local[84] += (double)s;
      s = fmaf(D[44], Q[1], s);
      s = fmaf(D[48], Q[2], s);
      s = fmaf(D[49], Q[3], s);
      local[28] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[30] * Q[0];
      local[85] += (double)s;
      s = fmaf(D[45], Q[1], s);
      s = fmaf(D[50], Q[2], s);
      s = fmaf(D[51], Q[3], s);
      local[29] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[31] * Q[0];
      local[86] += (double)s;
      s = fmaf(D[46], Q[1], s);
      s = fmaf(D[51], Q[2], s);
      s = fmaf(D[52], Q[3], s);
      local[30] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[32] * Q[0];
      local[87] += (double)s;
      s = fmaf(D[47], Q[1], s);
      s = fmaf(D[52], Q[2], s);
      s = fmaf(D[53], Q[3], s);
      local[31] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[33] * Q[0];
      local[88] += (double)s;
      s = fmaf(D[48], Q[1], s);
      s = fmaf(D[53], Q[2], s);
      s = fmaf(D[54], Q[3], s);
      local[32] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[34] * Q[0];
      local[89] += (double)s;
      s = fmaf(D[49], Q[1], s);
      s = fmaf(D[54], Q[2], s);
      s = fmaf(D[55], Q[3], s);
      local[33] -= (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[35] * Q[0];
      local[34] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[36] * Q[0];
      local[35] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[37] * Q[0];
      local[36] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[38] * Q[0];
      local[37] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[39] * Q[0];
      local[38] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[40] * Q[0];
      local[39] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[41] * Q[0];
      local[40] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[42] * Q[0];
      local[41] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[43] * Q[0];
      local[42] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[44] * Q[0];
      local[43] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[45] * Q[0];
      local[44] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[46] * Q[0];
      local[45] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[47] * Q[0];
      local[46] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[48] * Q[0];
      local[47] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[49] * Q[0];
      local[48] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[50] * Q[0];
      local[49] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[51] * Q[0];
      local[50] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[52] * Q[0];
      local[51] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[53] * Q[0];
      local[52] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[54] * Q[0];
      local[53] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[55] * Q[0];
      local[54] += (double)s;
    }
    __builtin_amdgcn_sched_barrier(0);
    {
      float s = D[0] * Q[0];
      s = fmaf(D[1], Q[1], s);
      s = fmaf(D[2], Q[2], s);
      s = fmaf(D[3], Q[3], s);
      s = fmaf(D[4], Q[4], s);
      s = fmaf(D[5], Q[5], s);
      s = fmaf(D[6], Q[6], s);
      s = fmaf(D[7], Q[7], s);
      s = fmaf(D[8], Q[8], s);
      s = fmaf(D[9], Q[9], s);
      s = fmaf(D[10], Q[10], s);
      s = fmaf(D[11], Q[11], s);
      s = fmaf(D[12], Q[12], s);
      s = fmaf(D[13], Q[13], s);
      s = fmaf(D[14], Q[14], s);
      s = fmaf(D[15], Q[15], s);
      s = fmaf(D[16], Q[16], s);
      s = fmaf(D[17], Q[17], s);
      s = fmaf(D[18], Q[18], s);
      s = fmaf(D[19], Q[19], s);
      s = fmaf(D[20], Q[20], s);
      s = fmaf(D[21], Q[21], s);
      s = fmaf(D[22], Q[22], s);
      s = fmaf(D[23], Q[23], s);
      s = fmaf(D[24], Q[24], s);
      s = fmaf(D[25], Q[25], s);
      s = fmaf(D[26], Q[26], s);
      s = fmaf(D[27], Q[27], s);
      s = fmaf(D[28], Q[28], s);
      s = fmaf(D[29], Q[29], s);
      s = fmaf(D[30], Q[30], s);
      s = fmaf(D[31], Q[31], s);
      s = fmaf(D[32], Q[32], s);
      s = fmaf(D[33], Q[33], s);
      s = fmaf(D[34], Q[34], s);
      local[55] += (double)s;
    }
  }
  static constexpr int NQR = 25;   // independent moments
  static constexpr int NLR = 60;  // S then X
  __device__ __forceinline__ static void reduce(const double* Q, double* Qr) {
    Qr[0] = Q[0];
    Qr[1] = Q[1];
    Qr[2] = Q[2];
    Qr[3] = Q[3];
    Qr[4] = Q[4] - Q[9];
    Qr[5] = Q[5];
    Qr[6] = Q[6];
    Qr[7] = Q[7] - Q[9];
    Qr[8] = Q[8];
    Qr[9] = Q[10] - Q[15];
    Qr[10] = Q[11] - Q[18];
    Qr[11] = Q[12] - Q[19];
    Qr[12] = Q[13] - Q[15];
    Qr[13] = Q[14];
    Qr[14] = Q[16] - Q[18];
    Qr[15] = Q[17] - Q[19];
    Qr[16] = Q[20] - Q[25] + Q[34];
    Qr[17] = Q[21] - Q[28];
    Qr[18] = Q[22] - Q[29];
    Qr[19] = Q[23] - Q[25] + 2.0 * Q[34] - Q[32];
    Qr[20] = Q[24] - Q[33];
    Qr[21] = Q[26] - Q[28];
    Qr[22] = Q[27] - Q[29];
    Qr[23] = Q[30] - Q[32] + Q[34];
    Qr[24] = Q[31] - Q[33];
  }
  __device__ __forceinline__ static void m2l_h(const double* r, const double* Qr, double* lr, bool ok) {
    const double r2 = fma(r[0], r[0], fma(r[1], r[1], r[2] * r[2]));
    const double ri = rsqrt_refined(r2);
    const double rinv = ok && r2 < __builtin_inf() ? ri : 0.0;
    const double s = rinv * rinv;
    const double w[3] = {r[0] * s, r[1] * s, r[2] * s};
    const double R0_000 = rinv;
    const double R1_000 = -1.0 * rinv;
    const double R2_000 = 3.0 * rinv;
    const double R3_000 = -15.0 * rinv;
    const double R4_000 = 105.0 * rinv;
    const double R5_000 = -945.0 * rinv;
    lr[0] = fma(R0_000, Qr[0], lr[0]);
    const double R0_100 = w[0] * R1_000;
    lr[0] = fma(R0_100, Qr[1], lr[0]);
    lr[1] = fma(R0_100, Qr[0], lr[1]);
    const double R0_010 = w[1] * R1_000;
    lr[0] = fma(R0_010, Qr[2], lr[0]);
    lr[2] = fma(R0_010, Qr[0], lr[2]);
    const double R0_001 = w[2] * R1_000;
    lr[0] = fma(R0_001, Qr[3], lr[0]);
    lr[3] = fma(R0_001, Qr[0], lr[3]);
    const double R1_100 = w[0] * R2_000;
    const double T1_000 = s * R1_000;
    const double R0_200 = fma(w[0], R1_100, T1_000);
    lr[0] = fma(R0_200, Qr[4], lr[0]);
    lr[1] = fma(R0_200, Qr[1], lr[1]);
    lr[4] = fma(R0_200, Qr[0], lr[4]);
    const double R1_010 = w[1] * R2_000;
    const double R0_110 = w[0] * R1_010;
    lr[0] = fma(R0_110, Qr[5], lr[0]);
    lr[1] = fma(R0_110, Qr[2], lr[1]);
    lr[2] = fma(R0_110, Qr[1], lr[2]);
    lr[5] = fma(R0_110, Qr[0], lr[5]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_101 = w[2] * R1_100;
    lr[0] = fma(R0_101, Qr[6], lr[0]);
    lr[1] = fma(R0_101, Qr[3], lr[1]);
    lr[3] = fma(R0_101, Qr[1], lr[3]);
    lr[6] = fma(R0_101, Qr[0], lr[6]);
    const double R0_020 = fma(w[1], R1_010, T1_000);
    lr[0] = fma(R0_020, Qr[7], lr[0]);
    lr[2] = fma(R0_020, Qr[2], lr[2]);
    lr[7] = fma(R0_020, Qr[0], lr[7]);
    const double R0_011 = w[2] * R1_010;
    lr[0] = fma(R0_011, Qr[8], lr[0]);
    lr[2] = fma(R0_011, Qr[3], lr[2]);
    lr[3] = fma(R0_011, Qr[2], lr[3]);
    lr[8] = fma(R0_011, Qr[0], lr[8]);
    const double R0_002 = -(R0_200 + R0_020);
    lr[3] = fma(R0_002, Qr[3], lr[3]);
    __builtin_amdgcn_sched_barrier(0);
    const double R2_100 = w[0] * R3_000;
    const double T2_000 = s * R2_000;
    const double R1_200 = fma(w[0], R2_100, T2_000);
    const double T1_100 = s * R1_100;
    const double R0_300 = fma(w[0], R1_200, 2.0 * T1_100);
    lr[0] = fma(R0_300, Qr[9], lr[0]);
    lr[1] = fma(R0_300, Qr[4], lr[1]);
    lr[4] = fma(R0_300, Qr[1], lr[4]);
    lr[9] = fma(R0_300, Qr[0], lr[9]);
    const double R2_010 = w[1] * R3_000;
    const double R1_110 = w[0] * R2_010;
    const double T1_010 = s * R1_010;
    const double R0_210 = fma(w[0], R1_110, T1_010);
    lr[0] = fma(R0_210, Qr[10], lr[0]);
    lr[1] = fma(R0_210, Qr[5], lr[1]);
    lr[2] = fma(R0_210, Qr[4], lr[2]);
    lr[4] = fma(R0_210, Qr[2], lr[4]);
    lr[5] = fma(R0_210, Qr[1], lr[5]);
    lr[10] = fma(R0_210, Qr[0], lr[10]);
    const double R0_201 = w[2] * R1_200;
    lr[0] = fma(R0_201, Qr[11], lr[0]);
    lr[1] = fma(R0_201, Qr[6], lr[1]);
    lr[3] = fma(R0_201, Qr[4], lr[3]);
    lr[4] = fma(R0_201, Qr[3], lr[4]);
    lr[6] = fma(R0_201, Qr[1], lr[6]);
    lr[11] = fma(R0_201, Qr[0], lr[11]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_120 = fma(w[1], R1_110, T1_100);
    lr[0] = fma(R0_120, Qr[12], lr[0]);
    lr[1] = fma(R0_120, Qr[7], lr[1]);
    lr[2] = fma(R0_120, Qr[5], lr[2]);
    lr[5] = fma(R0_120, Qr[2], lr[5]);
    lr[7] = fma(R0_120, Qr[1], lr[7]);
    lr[12] = fma(R0_120, Qr[0], lr[12]);
    const double R0_111 = w[2] * R1_110;
    lr[0] = fma(R0_111, Qr[13], lr[0]);
    lr[1] = fma(R0_111, Qr[8], lr[1]);
    lr[2] = fma(R0_111, Qr[6], lr[2]);
    lr[3] = fma(R0_111, Qr[5], lr[3]);
    lr[5] = fma(R0_111, Qr[3], lr[5]);
    lr[6] = fma(R0_111, Qr[2], lr[6]);
    lr[8] = fma(R0_111, Qr[1], lr[8]);
    lr[13] = fma(R0_111, Qr[0], lr[13]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_102 = -(R0_300 + R0_120);
    lr[3] = fma(R0_102, Qr[6], lr[3]);
    lr[6] = fma(R0_102, Qr[3], lr[6]);
    const double R1_020 = fma(w[1], R2_010, T2_000);
    const double R0_030 = fma(w[1], R1_020, 2.0 * T1_010);
    lr[0] = fma(R0_030, Qr[14], lr[0]);
    lr[2] = fma(R0_030, Qr[7], lr[2]);
    lr[7] = fma(R0_030, Qr[2], lr[7]);
    lr[14] = fma(R0_030, Qr[0], lr[14]);
    const double R0_021 = w[2] * R1_020;
    lr[0] = fma(R0_021, Qr[15], lr[0]);
    lr[2] = fma(R0_021, Qr[8], lr[2]);
    lr[3] = fma(R0_021, Qr[7], lr[3]);
    lr[7] = fma(R0_021, Qr[3], lr[7]);
    lr[8] = fma(R0_021, Qr[2], lr[8]);
    lr[15] = fma(R0_021, Qr[0], lr[15]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_012 = -(R0_210 + R0_030);
    lr[3] = fma(R0_012, Qr[8], lr[3]);
    lr[8] = fma(R0_012, Qr[3], lr[8]);
    const double R3_100 = w[0] * R4_000;
    const double T3_000 = s * R3_000;
    const double R2_200 = fma(w[0], R3_100, T3_000);
    const double T2_100 = s * R2_100;
    const double R1_300 = fma(w[0], R2_200, 2.0 * T2_100);
    const double T1_200 = s * R1_200;
    const double R0_400 = fma(w[0], R1_300, 3.0 * T1_200);
    lr[0] = fma(R0_400, Qr[16], lr[0]);
    lr[1] = fma(R0_400, Qr[9], lr[1]);
    lr[4] = fma(R0_400, Qr[4], lr[4]);
    lr[9] = fma(R0_400, Qr[1], lr[9]);
    lr[16] = fma(R0_400, Qr[0], lr[16]);
    const double R3_010 = w[1] * R4_000;
    const double R2_110 = w[0] * R3_010;
    const double T2_010 = s * R2_010;
    const double R1_210 = fma(w[0], R2_110, T2_010);
    const double T1_110 = s * R1_110;
    const double R0_310 = fma(w[0], R1_210, 2.0 * T1_110);
    lr[0] = fma(R0_310, Qr[17], lr[0]);
    lr[1] = fma(R0_310, Qr[10], lr[1]);
    lr[2] = fma(R0_310, Qr[9], lr[2]);
    lr[4] = fma(R0_310, Qr[5], lr[4]);
    lr[5] = fma(R0_310, Qr[4], lr[5]);
    lr[9] = fma(R0_310, Qr[2], lr[9]);
    lr[10] = fma(R0_310, Qr[1], lr[10]);
    lr[17] = fma(R0_310, Qr[0], lr[17]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_301 = w[2] * R1_300;
    lr[0] = fma(R0_301, Qr[18], lr[0]);
    lr[1] = fma(R0_301, Qr[11], lr[1]);
    lr[3] = fma(R0_301, Qr[9], lr[3]);
    lr[4] = fma(R0_301, Qr[6], lr[4]);
    lr[6] = fma(R0_301, Qr[4], lr[6]);
    lr[9] = fma(R0_301, Qr[3], lr[9]);
    lr[11] = fma(R0_301, Qr[1], lr[11]);
    lr[18] = fma(R0_301, Qr[0], lr[18]);
    const double R1_120 = fma(w[1], R2_110, T2_100);
    const double T1_020 = s * R1_020;
    const double R0_220 = fma(w[0], R1_120, T1_020);
    lr[0] = fma(R0_220, Qr[19], lr[0]);
    lr[1] = fma(R0_220, Qr[12], lr[1]);
    lr[2] = fma(R0_220, Qr[10], lr[2]);
    lr[4] = fma(R0_220, Qr[7], lr[4]);
    lr[5] = fma(R0_220, Qr[5], lr[5]);
    lr[7] = fma(R0_220, Qr[4], lr[7]);
    lr[10] = fma(R0_220, Qr[2], lr[10]);
    lr[12] = fma(R0_220, Qr[1], lr[12]);
    lr[19] = fma(R0_220, Qr[0], lr[19]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_211 = w[2] * R1_210;
    lr[0] = fma(R0_211, Qr[20], lr[0]);
    lr[1] = fma(R0_211, Qr[13], lr[1]);
    lr[2] = fma(R0_211, Qr[11], lr[2]);
    lr[3] = fma(R0_211, Qr[10], lr[3]);
    lr[4] = fma(R0_211, Qr[8], lr[4]);
    lr[5] = fma(R0_211, Qr[6], lr[5]);
    lr[6] = fma(R0_211, Qr[5], lr[6]);
    lr[8] = fma(R0_211, Qr[4], lr[8]);
    lr[10] = fma(R0_211, Qr[3], lr[10]);
    lr[11] = fma(R0_211, Qr[2], lr[11]);
    lr[13] = fma(R0_211, Qr[1], lr[13]);
    lr[20] = fma(R0_211, Qr[0], lr[20]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_202 = -(R0_400 + R0_220);
    lr[3] = fma(R0_202, Qr[11], lr[3]);
    lr[6] = fma(R0_202, Qr[6], lr[6]);
    lr[11] = fma(R0_202, Qr[3], lr[11]);
    const double R0_130 = fma(w[1], R1_120, 2.0 * T1_110);
    lr[0] = fma(R0_130, Qr[21], lr[0]);
    lr[1] = fma(R0_130, Qr[14], lr[1]);
    lr[2] = fma(R0_130, Qr[12], lr[2]);
    lr[5] = fma(R0_130, Qr[7], lr[5]);
    lr[7] = fma(R0_130, Qr[5], lr[7]);
    lr[12] = fma(R0_130, Qr[2], lr[12]);
    lr[14] = fma(R0_130, Qr[1], lr[14]);
    lr[21] = fma(R0_130, Qr[0], lr[21]);
    const double R0_121 = w[2] * R1_120;
    lr[0] = fma(R0_121, Qr[22], lr[0]);
    lr[1] = fma(R0_121, Qr[15], lr[1]);
    lr[2] = fma(R0_121, Qr[13], lr[2]);
    lr[3] = fma(R0_121, Qr[12], lr[3]);
    lr[5] = fma(R0_121, Qr[8], lr[5]);
    lr[6] = fma(R0_121, Qr[7], lr[6]);
    lr[7] = fma(R0_121, Qr[6], lr[7]);
    lr[8] = fma(R0_121, Qr[5], lr[8]);
    lr[12] = fma(R0_121, Qr[3], lr[12]);
    lr[13] = fma(R0_121, Qr[2], lr[13]);
    lr[15] = fma(R0_121, Qr[1], lr[15]);
    lr[22] = fma(R0_121, Qr[0], lr[22]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_112 = -(R0_310 + R0_130);
    lr[3] = fma(R0_112, Qr[13], lr[3]);
    lr[6] = fma(R0_112, Qr[8], lr[6]);
    lr[8] = fma(R0_112, Qr[6], lr[8]);
    lr[13] = fma(R0_112, Qr[3], lr[13]);
    const double R2_020 = fma(w[1], R3_010, T3_000);
    const double R1_030 = fma(w[1], R2_020, 2.0 * T2_010);
    const double R0_040 = fma(w[1], R1_030, 3.0 * T1_020);
    lr[0] = fma(R0_040, Qr[23], lr[0]);
    lr[2] = fma(R0_040, Qr[14], lr[2]);
    lr[7] = fma(R0_040, Qr[7], lr[7]);
    lr[14] = fma(R0_040, Qr[2], lr[14]);
    lr[23] = fma(R0_040, Qr[0], lr[23]);
    const double R0_031 = w[2] * R1_030;
    lr[0] = fma(R0_031, Qr[24], lr[0]);
    lr[2] = fma(R0_031, Qr[15], lr[2]);
    lr[3] = fma(R0_031, Qr[14], lr[3]);
    lr[7] = fma(R0_031, Qr[8], lr[7]);
    lr[8] = fma(R0_031, Qr[7], lr[8]);
    lr[14] = fma(R0_031, Qr[3], lr[14]);
    lr[15] = fma(R0_031, Qr[2], lr[15]);
    lr[24] = fma(R0_031, Qr[0], lr[24]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_022 = -(R0_220 + R0_040);
    lr[3] = fma(R0_022, Qr[15], lr[3]);
    lr[8] = fma(R0_022, Qr[8], lr[8]);
    lr[15] = fma(R0_022, Qr[3], lr[15]);
    const double R4_100 = w[0] * R5_000;
    const double T4_000 = s * R4_000;
    const double R3_200 = fma(w[0], R4_100, T4_000);
    const double T3_100 = s * R3_100;
    const double R2_300 = fma(w[0], R3_200, 2.0 * T3_100);
    const double T2_200 = s * R2_200;
    const double R1_400 = fma(w[0], R2_300, 3.0 * T2_200);
    const double T1_300 = s * R1_300;
    const double R0_500 = fma(w[0], R1_400, 4.0 * T1_300);
    lr[25] = fma(R0_500, Qr[16], lr[25]);
    lr[28] = fma(R0_500, Qr[9], lr[28]);
    lr[33] = fma(R0_500, Qr[4], lr[33]);
    lr[40] = fma(R0_500, Qr[1], lr[40]);
    lr[49] = fma(R0_500, Qr[0], lr[49]);
    const double R4_010 = w[1] * R5_000;
    const double R3_110 = w[0] * R4_010;
    const double T3_010 = s * R3_010;
    const double R2_210 = fma(w[0], R3_110, T3_010);
    const double T2_110 = s * R2_110;
    const double R1_310 = fma(w[0], R2_210, 2.0 * T2_110);
    const double T1_210 = s * R1_210;
    const double R0_410 = fma(w[0], R1_310, 3.0 * T1_210);
    lr[25] = fma(R0_410, Qr[17], lr[25]);
    lr[26] = fma(R0_410, Qr[16], lr[26]);
    lr[28] = fma(R0_410, Qr[10], lr[28]);
    lr[29] = fma(R0_410, Qr[9], lr[29]);
    lr[33] = fma(R0_410, Qr[5], lr[33]);
    lr[34] = fma(R0_410, Qr[4], lr[34]);
    lr[40] = fma(R0_410, Qr[2], lr[40]);
    lr[41] = fma(R0_410, Qr[1], lr[41]);
    lr[50] = fma(R0_410, Qr[0], lr[50]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_401 = w[2] * R1_400;
    lr[25] = fma(R0_401, Qr[18], lr[25]);
    lr[27] = fma(R0_401, Qr[16], lr[27]);
    lr[28] = fma(R0_401, Qr[11], lr[28]);
    lr[30] = fma(R0_401, Qr[9], lr[30]);
    lr[33] = fma(R0_401, Qr[6], lr[33]);
    lr[35] = fma(R0_401, Qr[4], lr[35]);
    lr[40] = fma(R0_401, Qr[3], lr[40]);
    lr[42] = fma(R0_401, Qr[1], lr[42]);
    lr[51] = fma(R0_401, Qr[0], lr[51]);
    const double R2_120 = fma(w[1], R3_110, T3_100);
    const double T2_020 = s * R2_020;
    const double R1_220 = fma(w[0], R2_120, T2_020);
    const double T1_120 = s * R1_120;
    const double R0_320 = fma(w[0], R1_220, 2.0 * T1_120);
    lr[25] = fma(R0_320, Qr[19], lr[25]);
    lr[26] = fma(R0_320, Qr[17], lr[26]);
    lr[28] = fma(R0_320, Qr[12], lr[28]);
    lr[29] = fma(R0_320, Qr[10], lr[29]);
    lr[31] = fma(R0_320, Qr[9], lr[31]);
    lr[33] = fma(R0_320, Qr[7], lr[33]);
    lr[34] = fma(R0_320, Qr[5], lr[34]);
    lr[36] = fma(R0_320, Qr[4], lr[36]);
    lr[41] = fma(R0_320, Qr[2], lr[41]);
    lr[43] = fma(R0_320, Qr[1], lr[43]);
    lr[52] = fma(R0_320, Qr[0], lr[52]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_311 = w[2] * R1_310;
    lr[25] = fma(R0_311, Qr[20], lr[25]);
    lr[26] = fma(R0_311, Qr[18], lr[26]);
    lr[27] = fma(R0_311, Qr[17], lr[27]);
    lr[28] = fma(R0_311, Qr[13], lr[28]);
    lr[29] = fma(R0_311, Qr[11], lr[29]);
    lr[30] = fma(R0_311, Qr[10], lr[30]);
    lr[32] = fma(R0_311, Qr[9], lr[32]);
    lr[33] = fma(R0_311, Qr[8], lr[33]);
    lr[34] = fma(R0_311, Qr[6], lr[34]);
    lr[35] = fma(R0_311, Qr[5], lr[35]);
    lr[37] = fma(R0_311, Qr[4], lr[37]);
    lr[41] = fma(R0_311, Qr[3], lr[41]);
    lr[42] = fma(R0_311, Qr[2], lr[42]);
    lr[44] = fma(R0_311, Qr[1], lr[44]);
    lr[53] = fma(R0_311, Qr[0], lr[53]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_302 = -(R0_500 + R0_320);
    lr[27] = fma(R0_302, Qr[18], lr[27]);
    lr[30] = fma(R0_302, Qr[11], lr[30]);
    lr[35] = fma(R0_302, Qr[6], lr[35]);
    lr[42] = fma(R0_302, Qr[3], lr[42]);
    const double R0_230 = fma(w[1], R1_220, 2.0 * T1_210);
    lr[25] = fma(R0_230, Qr[21], lr[25]);
    lr[26] = fma(R0_230, Qr[19], lr[26]);
    lr[28] = fma(R0_230, Qr[14], lr[28]);
    lr[29] = fma(R0_230, Qr[12], lr[29]);
    lr[31] = fma(R0_230, Qr[10], lr[31]);
    lr[34] = fma(R0_230, Qr[7], lr[34]);
    lr[36] = fma(R0_230, Qr[5], lr[36]);
    lr[38] = fma(R0_230, Qr[4], lr[38]);
    lr[43] = fma(R0_230, Qr[2], lr[43]);
    lr[45] = fma(R0_230, Qr[1], lr[45]);
    lr[54] = fma(R0_230, Qr[0], lr[54]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_221 = w[2] * R1_220;
    lr[25] = fma(R0_221, Qr[22], lr[25]);
    lr[26] = fma(R0_221, Qr[20], lr[26]);
    lr[27] = fma(R0_221, Qr[19], lr[27]);
    lr[28] = fma(R0_221, Qr[15], lr[28]);
    lr[29] = fma(R0_221, Qr[13], lr[29]);
    lr[30] = fma(R0_221, Qr[12], lr[30]);
    lr[31] = fma(R0_221, Qr[11], lr[31]);
    lr[32] = fma(R0_221, Qr[10], lr[32]);
    lr[34] = fma(R0_221, Qr[8], lr[34]);
    lr[35] = fma(R0_221, Qr[7], lr[35]);
    lr[36] = fma(R0_221, Qr[6], lr[36]);
    lr[37] = fma(R0_221, Qr[5], lr[37]);
    lr[39] = fma(R0_221, Qr[4], lr[39]);
    lr[43] = fma(R0_221, Qr[3], lr[43]);
    lr[44] = fma(R0_221, Qr[2], lr[44]);
    lr[46] = fma(R0_221, Qr[1], lr[46]);
    lr[55] = fma(R0_221, Qr[0], lr[55]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_212 = -(R0_410 + R0_230);
    lr[27] = fma(R0_212, Qr[20], lr[27]);
    lr[30] = fma(R0_212, Qr[13], lr[30]);
    lr[32] = fma(R0_212, Qr[11], lr[32]);
    lr[35] = fma(R0_212, Qr[8], lr[35]);
    lr[37] = fma(R0_212, Qr[6], lr[37]);
    lr[44] = fma(R0_212, Qr[3], lr[44]);
    const double R1_130 = fma(w[1], R2_120, 2.0 * T2_110);
    const double R0_140 = fma(w[1], R1_130, 3.0 * T1_120);
    lr[25] = fma(R0_140, Qr[23], lr[25]);
    lr[26] = fma(R0_140, Qr[21], lr[26]);
    lr[29] = fma(R0_140, Qr[14], lr[29]);
    lr[31] = fma(R0_140, Qr[12], lr[31]);
    lr[36] = fma(R0_140, Qr[7], lr[36]);
    lr[38] = fma(R0_140, Qr[5], lr[38]);
    lr[45] = fma(R0_140, Qr[2], lr[45]);
    lr[47] = fma(R0_140, Qr[1], lr[47]);
    lr[56] = fma(R0_140, Qr[0], lr[56]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_131 = w[2] * R1_130;
    lr[25] = fma(R0_131, Qr[24], lr[25]);
    lr[26] = fma(R0_131, Qr[22], lr[26]);
    lr[27] = fma(R0_131, Qr[21], lr[27]);
    lr[29] = fma(R0_131, Qr[15], lr[29]);
    lr[30] = fma(R0_131, Qr[14], lr[30]);
    lr[31] = fma(R0_131, Qr[13], lr[31]);
    lr[32] = fma(R0_131, Qr[12], lr[32]);
    lr[36] = fma(R0_131, Qr[8], lr[36]);
    lr[37] = fma(R0_131, Qr[7], lr[37]);
    lr[38] = fma(R0_131, Qr[6], lr[38]);
    lr[39] = fma(R0_131, Qr[5], lr[39]);
    lr[45] = fma(R0_131, Qr[3], lr[45]);
    lr[46] = fma(R0_131, Qr[2], lr[46]);
    lr[48] = fma(R0_131, Qr[1], lr[48]);
    lr[57] = fma(R0_131, Qr[0], lr[57]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_122 = -(R0_320 + R0_140);
    lr[27] = fma(R0_122, Qr[22], lr[27]);
    lr[30] = fma(R0_122, Qr[15], lr[30]);
    lr[32] = fma(R0_122, Qr[13], lr[32]);
    lr[37] = fma(R0_122, Qr[8], lr[37]);
    lr[39] = fma(R0_122, Qr[6], lr[39]);
    lr[46] = fma(R0_122, Qr[3], lr[46]);
    const double R3_020 = fma(w[1], R4_010, T4_000);
    const double R2_030 = fma(w[1], R3_020, 2.0 * T3_010);
    const double R1_040 = fma(w[1], R2_030, 3.0 * T2_020);
    const double T1_030 = s * R1_030;
    const double R0_050 = fma(w[1], R1_040, 4.0 * T1_030);
    lr[26] = fma(R0_050, Qr[23], lr[26]);
    lr[31] = fma(R0_050, Qr[14], lr[31]);
    lr[38] = fma(R0_050, Qr[7], lr[38]);
    lr[47] = fma(R0_050, Qr[2], lr[47]);
    lr[58] = fma(R0_050, Qr[0], lr[58]);
    const double R0_041 = w[2] * R1_040;
    lr[26] = fma(R0_041, Qr[24], lr[26]);
    lr[27] = fma(R0_041, Qr[23], lr[27]);
    lr[31] = fma(R0_041, Qr[15], lr[31]);
    lr[32] = fma(R0_041, Qr[14], lr[32]);
    lr[38] = fma(R0_041, Qr[8], lr[38]);
    lr[39] = fma(R0_041, Qr[7], lr[39]);
    lr[47] = fma(R0_041, Qr[3], lr[47]);
    lr[48] = fma(R0_041, Qr[2], lr[48]);
    lr[59] = fma(R0_041, Qr[0], lr[59]);
    __builtin_amdgcn_sched_barrier(0);
    const double R0_032 = -(R0_230 + R0_050);
    lr[27] = fma(R0_032, Qr[24], lr[27]);
    lr[32] = fma(R0_032, Qr[15], lr[32]);
    lr[39] = fma(R0_032, Qr[8], lr[39]);
    lr[48] = fma(R0_032, Qr[3], lr[48]);
  }
  static constexpr int FLOPS_M2L_H = 745;  // + one refined rsqrt
  __device__ __forceinline__ static void expand(const double* lr, double* local) {
    double t[56];
    t[0] = lr[0];
    local[55] = t[0];
    t[1] = -lr[1];
    local[56] = t[1];
    t[2] = -lr[2];
    local[57] = t[2];
    t[3] = -lr[3];
    local[58] = t[3];
    t[4] = lr[4];
    local[59] = t[4];
    t[5] = lr[5];
    local[60] = t[5];
    t[6] = lr[6];
    local[61] = t[6];
    t[7] = lr[7];
    local[62] = t[7];
    t[8] = lr[8];
    local[63] = t[8];
    t[9] = -(t[4] + t[7]);
    local[64] = t[9];
    t[10] = -lr[9];
    local[65] = t[10];
    t[11] = -lr[10];
    local[66] = t[11];
    t[12] = -lr[11];
    local[67] = t[12];
    t[13] = -lr[12];
    local[68] = t[13];
    t[14] = -lr[13];
    local[69] = t[14];
    t[15] = -(t[10] + t[13]);
    local[70] = t[15];
    t[16] = -lr[14];
    local[71] = t[16];
    t[17] = -lr[15];
    local[72] = t[17];
    t[18] = -(t[11] + t[16]);
    local[73] = t[18];
    t[19] = -(t[12] + t[17]);
    local[74] = t[19];
    t[20] = lr[16];
    local[75] = t[20];
    t[21] = lr[17];
    local[76] = t[21];
    t[22] = lr[18];
    local[77] = t[22];
    t[23] = lr[19];
    local[78] = t[23];
    t[24] = lr[20];
    local[79] = t[24];
    t[25] = -(t[20] + t[23]);
    local[80] = t[25];
    t[26] = lr[21];
    local[81] = t[26];
    t[27] = lr[22];
    local[82] = t[27];
    t[28] = -(t[21] + t[26]);
    local[83] = t[28];
    t[29] = -(t[22] + t[27]);
    local[84] = t[29];
    t[30] = lr[23];
    local[85] = t[30];
    t[31] = lr[24];
    local[86] = t[31];
    t[32] = -(t[23] + t[30]);
    local[87] = t[32];
    t[33] = -(t[24] + t[31]);
    local[88] = t[33];
    t[34] = -(t[25] + t[32]);
    local[89] = t[34];
    t[1] = (lr[1] + lr[25]);
    local[0] = t[1];
    t[2] = (lr[2] + lr[26]);
    local[1] = t[2];
    t[3] = (lr[3] + lr[27]);
    local[2] = t[3];
    t[4] = -(lr[4] + lr[28]);
    local[3] = t[4];
    t[5] = -(lr[5] + lr[29]);
    local[4] = t[5];
    t[6] = -(lr[6] + lr[30]);
    local[5] = t[6];
    t[7] = -(lr[7] + lr[31]);
    local[6] = t[7];
    t[8] = -(lr[8] + lr[32]);
    local[7] = t[8];
    t[9] = -(t[4] + t[7]);
    local[8] = t[9];
    t[10] = (lr[9] + lr[33]);
    local[9] = t[10];
    t[11] = (lr[10] + lr[34]);
    local[10] = t[11];
    t[12] = (lr[11] + lr[35]);
    local[11] = t[12];
    t[13] = (lr[12] + lr[36]);
    local[12] = t[13];
    t[14] = (lr[13] + lr[37]);
    local[13] = t[14];
    t[15] = -(t[10] + t[13]);
    local[14] = t[15];
    t[16] = (lr[14] + lr[38]);
    local[15] = t[16];
    t[17] = (lr[15] + lr[39]);
    local[16] = t[17];
    t[18] = -(t[11] + t[16]);
    local[17] = t[18];
    t[19] = -(t[12] + t[17]);
    local[18] = t[19];
    t[20] = -(lr[16] + lr[40]);
    local[19] = t[20];
    t[21] = -(lr[17] + lr[41]);
    local[20] = t[21];
    t[22] = -(lr[18] + lr[42]);
    local[21] = t[22];
    t[23] = -(lr[19] + lr[43]);
    local[22] = t[23];
    t[24] = -(lr[20] + lr[44]);
    local[23] = t[24];
    t[25] = -(t[20] + t[23]);
    local[24] = t[25];
    t[26] = -(lr[21] + lr[45]);
    local[25] = t[26];
    t[27] = -(lr[22] + lr[46]);
    local[26] = t[27];
    t[28] = -(t[21] + t[26]);
    local[27] = t[28];
    t[29] = -(t[22] + t[27]);
    local[28] = t[29];
    t[30] = -(lr[23] + lr[47]);
    local[29] = t[30];
    t[31] = -(lr[24] + lr[48]);
    local[30] = t[31];
    t[32] = -(t[23] + t[30]);
    local[31] = t[32];
    t[33] = -(t[24] + t[31]);
    local[32] = t[33];
    t[34] = -(t[25] + t[32]);
    local[33] = t[34];
    t[35] = lr[49];
    local[34] = t[35];
    t[36] = lr[50];
    local[35] = t[36];
    t[37] = lr[51];
    local[36] = t[37];
    t[38] = lr[52];
    local[37] = t[38];
    t[39] = lr[53];
    local[38] = t[39];
    t[40] = -(t[35] + t[38]);
    local[39] = t[40];
    t[41] = lr[54];
    local[40] = t[41];
    t[42] = lr[55];
    local[41] = t[42];
    t[43] = -(t[36] + t[41]);
    local[42] = t[43];
    t[44] = -(t[37] + t[42]);
    local[43] = t[44];
    t[45] = lr[56];
    local[44] = t[45];
    t[46] = lr[57];
    local[45] = t[46];
    t[47] = -(t[38] + t[45]);
    local[46] = t[47];
    t[48] = -(t[39] + t[46]);
    local[47] = t[48];
    t[49] = -(t[40] + t[47]);
    local[48] = t[49];
    t[50] = lr[58];
    local[49] = t[50];
    t[51] = lr[59];
    local[50] = t[51];
    t[52] = -(t[41] + t[50]);
    local[51] = t[52];
    t[53] = -(t[42] + t[51]);
    local[52] = t[53];
    t[54] = -(t[43] + t[52]);
    local[53] = t[54];
    t[55] = -(t[44] + t[53]);
    local[54] = t[55];
  }
  __device__ __forceinline__ static void m2l_pair(const double* r, const double* QS,
                                                    const double* QTs, double* local,
                                                    double* outS) {
    const double r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    const double rinv = rsqrt(r2);
    const double rinv2 = rinv * rinv;
    double D[56];
    D[0] = rinv;
    const double sn1 = rinv2 * -1.0;
    const double sn2 = rinv2 * -0.5;
    const double sn3 = rinv2 * -0.3333333333333333;
    const double sn4 = rinv2 * -0.25;
    const double sn5 = rinv2 * -0.2;
    D[1] = (1.0 * r[0] * D[0]) * sn1;
    D[2] = (1.0 * r[1] * D[0]) * sn1;
    D[3] = (1.0 * r[2] * D[0]) * sn1;
    D[4] = (6.0 * r[0] * D[1] + 2.0 * D[0]) * sn2;
    D[5] = (3.0 * r[0] * D[2] + 3.0 * r[1] * D[1]) * sn2;
    D[6] = (3.0 * r[0] * D[3] + 3.0 * r[2] * D[1]) * sn2;
    D[7] = (6.0 * r[1] * D[2] + 2.0 * D[0]) * sn2;
    D[8] = (3.0 * r[1] * D[3] + 3.0 * r[2] * D[2]) * sn2;
    D[9] = (6.0 * r[2] * D[3] + 2.0 * D[0]) * sn2;
    D[10] = (15.0 * r[0] * D[4] + 12.0 * D[1]) * sn3;
    D[11] = (10.0 * r[0] * D[5] + 4.0 * D[2] + 5.0 * r[1] * D[4]) * sn3;
    D[12] = (10.0 * r[0] * D[6] + 4.0 * D[3] + 5.0 * r[2] * D[4]) * sn3;
    D[13] = (5.0 * r[0] * D[7] + 10.0 * r[1] * D[5] + 4.0 * D[1]) * sn3;
    D[14] = (5.0 * r[0] * D[8] + 5.0 * r[1] * D[6] + 5.0 * r[2] * D[5]) * sn3;
    D[15] = (5.0 * r[0] * D[9] + 10.0 * r[2] * D[6] + 4.0 * D[1]) * sn3;
    D[16] = (15.0 * r[1] * D[7] + 12.0 * D[2]) * sn3;
    D[17] = (10.0 * r[1] * D[8] + 4.0 * D[3] + 5.0 * r[2] * D[7]) * sn3;
    D[18] = (5.0 * r[1] * D[9] + 10.0 * r[2] * D[8] + 4.0 * D[2]) * sn3;
    D[19] = (15.0 * r[2] * D[9] + 12.0 * D[3]) * sn3;
    D[20] = (28.0 * r[0] * D[10] + 36.0 * D[4]) * sn4;
    D[21] = (21.0 * r[0] * D[11] + 18.0 * D[5] + 7.0 * r[1] * D[10]) * sn4;
    D[22] = (21.0 * r[0] * D[12] + 18.0 * D[6] + 7.0 * r[2] * D[10]) * sn4;
    D[23] = (14.0 * r[0] * D[13] + 6.0 * D[7] + 14.0 * r[1] * D[11] + 6.0 * D[4]) * sn4;
    D[24] = (14.0 * r[0] * D[14] + 6.0 * D[8] + 7.0 * r[1] * D[12] + 7.0 * r[2] * D[11]) * sn4;
    D[25] = (14.0 * r[0] * D[15] + 6.0 * D[9] + 14.0 * r[2] * D[12] + 6.0 * D[4]) * sn4;
    D[26] = (7.0 * r[0] * D[16] + 21.0 * r[1] * D[13] + 18.0 * D[5]) * sn4;
    D[27] = (7.0 * r[0] * D[17] + 14.0 * r[1] * D[14] + 6.0 * D[6] + 7.0 * r[2] * D[13]) * sn4;
    D[28] = (7.0 * r[0] * D[18] + 7.0 * r[1] * D[15] + 14.0 * r[2] * D[14] + 6.0 * D[5]) * sn4;
    D[29] = (7.0 * r[0] * D[19] + 21.0 * r[2] * D[15] + 18.0 * D[6]) * sn4;
    D[30] = (28.0 * r[1] * D[16] + 36.0 * D[7]) * sn4;
    D[31] = (21.0 * r[1] * D[17] + 18.0 * D[8] + 7.0 * r[2] * D[16]) * sn4;
    D[32] = (14.0 * r[1] * D[18] + 6.0 * D[9] + 14.0 * r[2] * D[17] + 6.0 * D[7]) * sn4;
    D[33] = (7.0 * r[1] * D[19] + 21.0 * r[2] * D[18] + 18.0 * D[8]) * sn4;
    D[34] = (28.0 * r[2] * D[19] + 36.0 * D[9]) * sn4;
    D[35] = (45.0 * r[0] * D[20] + 80.0 * D[10]) * sn5;
    D[36] = (36.0 * r[0] * D[21] + 48.0 * D[11] + 9.0 * r[1] * D[20]) * sn5;
    D[37] = (36.0 * r[0] * D[22] + 48.0 * D[12] + 9.0 * r[2] * D[20]) * sn5;
    D[38] = (27.0 * r[0] * D[23] + 24.0 * D[13] + 18.0 * r[1] * D[21] + 8.0 * D[10]) * sn5;
    D[39] = (27.0 * r[0] * D[24] + 24.0 * D[14] + 9.0 * r[1] * D[22] + 9.0 * r[2] * D[21]) * sn5;
    D[40] = (27.0 * r[0] * D[25] + 24.0 * D[15] + 18.0 * r[2] * D[22] + 8.0 * D[10]) * sn5;
    D[41] = (18.0 * r[0] * D[26] + 8.0 * D[16] + 27.0 * r[1] * D[23] + 24.0 * D[11]) * sn5;
    D[42] = (18.0 * r[0] * D[27] + 8.0 * D[17] + 18.0 * r[1] * D[24] + 8.0 * D[12] + 9.0 * r[2] * D[23]) * sn5;
    D[43] = (18.0 * r[0] * D[28] + 8.0 * D[18] + 9.0 * r[1] * D[25] + 18.0 * r[2] * D[24] + 8.0 * D[11]) * sn5;
    D[44] = (18.0 * r[0] * D[29] + 8.0 * D[19] + 27.0 * r[2] * D[25] + 24.0 * D[12]) * sn5;
    D[45] = (9.0 * r[0] * D[30] + 36.0 * r[1] * D[26] + 48.0 * D[13]) * sn5;
    D[46] = (9.0 * r[0] * D[31] + 27.0 * r[1] * D[27] + 24.0 * D[14] + 9.0 * r[2] * D[26]) * sn5;
    D[47] = (9.0 * r[0] * D[32] + 18.0 * r[1] * D[28] + 8.0 * D[15] + 18.0 * r[2] * D[27] + 8.0 * D[13]) * sn5;
    D[48] = (9.0 * r[0] * D[33] + 9.0 * r[1] * D[29] + 27.0 * r[2] * D[28] + 24.0 * D[14]) * sn5;
    D[49] = (9.0 * r[0] * D[34] + 36.0 * r[2] * D[29] + 48.0 * D[15]) * sn5;
    D[50] = (45.0 * r[1] * D[30] + 80.0 * D[16]) * sn5;
    D[51] = (36.0 * r[1] * D[31] + 48.0 * D[17] + 9.0 * r[2] * D[30]) * sn5;
    D[52] = (27.0 * r[1] * D[32] + 24.0 * D[18] + 18.0 * r[2] * D[31] + 8.0 * D[16]) * sn5;
    D[53] = (18.0 * r[1] * D[33] + 8.0 * D[19] + 27.0 * r[2] * D[32] + 24.0 * D[17]) * sn5;
    D[54] = (9.0 * r[1] * D[34] + 36.0 * r[2] * D[33] + 48.0 * D[18]) * sn5;
    D[55] = (45.0 * r[2] * D[34] + 80.0 * D[19]) * sn5;
    {
      double s = D[1] * QS[0];
      s = fma(D[4], QS[1], s);
      s = fma(D[5], QS[2], s);
      s = fma(D[6], QS[3], s);
      s = fma(D[10], QS[4], s);
      s = fma(D[11], QS[5], s);
      s = fma(D[12], QS[6], s);
      s = fma(D[13], QS[7], s);
      s = fma(D[14], QS[8], s);
      s = fma(D[15], QS[9], s);
      s = fma(D[20], QS[10], s);
      s = fma(D[21], QS[11], s);
      s = fma(D[22], QS[12], s);
      s = fma(D[23], QS[13], s);
      s = fma(D[24], QS[14], s);
      s = fma(D[25], QS[15], s);
      s = fma(D[26], QS[16], s);
      s = fma(D[27], QS[17], s);
      s = fma(D[28], QS[18], s);
      s = fma(D[29], QS[19], s);
      local[56] -= s;
      s = fma(D[35], QS[20], s);
      s = fma(D[36], QS[21], s);
      s = fma(D[37], QS[22], s);
      s = fma(D[38], QS[23], s);
      s = fma(D[39], QS[24], s);
      s = fma(D[40], QS[25], s);
      s = fma(D[41], QS[26], s);
      s = fma(D[42], QS[27], s);
      s = fma(D[43], QS[28], s);
      s = fma(D[44], QS[29], s);
      s = fma(D[45], QS[30], s);
      s = fma(D[46], QS[31], s);
      s = fma(D[47], QS[32], s);
      s = fma(D[48], QS[33], s);
      s = fma(D[49], QS[34], s);
      local[0] += s;
    }
    {
      double s = D[2] * QS[0];
      s = fma(D[5], QS[1], s);
      s = fma(D[7], QS[2], s);
      s = fma(D[8], QS[3], s);
      s = fma(D[11], QS[4], s);
      s = fma(D[13], QS[5], s);
      s = fma(D[14], QS[6], s);
      s = fma(D[16], QS[7], s);
      s = fma(D[17], QS[8], s);
      s = fma(D[18], QS[9], s);
      s = fma(D[21], QS[10], s);
      s = fma(D[23], QS[11], s);
      s = fma(D[24], QS[12], s);
      s = fma(D[26], QS[13], s);
      s = fma(D[27], QS[14], s);
      s = fma(D[28], QS[15], s);
      s = fma(D[30], QS[16], s);
      s = fma(D[31], QS[17], s);
      s = fma(D[32], QS[18], s);
      s = fma(D[33], QS[19], s);
      local[57] -= s;
      s = fma(D[36], QS[20], s);
      s = fma(D[38], QS[21], s);
      s = fma(D[39], QS[22], s);
      s = fma(D[41], QS[23], s);
      s = fma(D[42], QS[24], s);
      s = fma(D[43], QS[25], s);
      s = fma(D[45], QS[26], s);
      s = fma(D[46], QS[27], s);
      s = fma(D[47], QS[28], s);
      s = fma(D[48], QS[29], s);
      s = fma(D[50], QS[30], s);
      s = fma(D[51], QS[31], s);
      s = fma(D[52], QS[32], s);
      s = fma(D[53], QS[33], s);
      s = fma(D[54], QS[34], s);
      local[1] += s;
    }
    {
      double s = D[3] * QS[0];
      s = fma(D[6], QS[1], s);
      s = fma(D[8], QS[2], s);
      s = fma(D[9], QS[3], s);
      s = fma(D[12], QS[4], s);
      s = fma(D[14], QS[5], s);
      s = fma(D[15], QS[6], s);
      s = fma(D[17], QS[7], s);
      s = fma(D[18], QS[8], s);
      s = fma(D[19], QS[9], s);
      s = fma(D[22], QS[10], s);
      s = fma(D[24], QS[11], s);
      s = fma(D[25], QS[12], s);
      s = fma(D[27], QS[13], s);
      s = fma(D[28], QS[14], s);
      s = fma(D[29], QS[15], s);
      s = fma(D[31], QS[16], s);
      s = fma(D[32], QS[17], s);
      s = fma(D[33], QS[18], s);
      s = fma(D[34], QS[19], s);
      local[58] -= s;
      s = fma(D[37], QS[20], s);
      s = fma(D[39], QS[21], s);
      s = fma(D[40], QS[22], s);
      s = fma(D[42], QS[23], s);
      s = fma(D[43], QS[24], s);
      s = fma(D[44], QS[25], s);
      s = fma(D[46], QS[26], s);
      s = fma(D[47], QS[27], s);
      s = fma(D[48], QS[28], s);
      s = fma(D[49], QS[29], s);
      s = fma(D[51], QS[30], s);
      s = fma(D[52], QS[31], s);
      s = fma(D[53], QS[32], s);
      s = fma(D[54], QS[33], s);
      s = fma(D[55], QS[34], s);
      local[2] += s;
    }
    {
      double s = D[4] * QS[0];
      s = fma(D[10], QS[1], s);
      s = fma(D[11], QS[2], s);
      s = fma(D[12], QS[3], s);
      s = fma(D[20], QS[4], s);
      s = fma(D[21], QS[5], s);
      s = fma(D[22], QS[6], s);
      s = fma(D[23], QS[7], s);
      s = fma(D[24], QS[8], s);
      s = fma(D[25], QS[9], s);
      local[59] += s;
      s = fma(D[35], QS[10], s);
      s = fma(D[36], QS[11], s);
      s = fma(D[37], QS[12], s);
      s = fma(D[38], QS[13], s);
      s = fma(D[39], QS[14], s);
      s = fma(D[40], QS[15], s);
      s = fma(D[41], QS[16], s);
      s = fma(D[42], QS[17], s);
      s = fma(D[43], QS[18], s);
      s = fma(D[44], QS[19], s);
      local[3] -= s;
    }
    {
      double s = D[5] * QS[0];
      s = fma(D[11], QS[1], s);
      s = fma(D[13], QS[2], s);
      s = fma(D[14], QS[3], s);
      s = fma(D[21], QS[4], s);
      s = fma(D[23], QS[5], s);
      s = fma(D[24], QS[6], s);
      s = fma(D[26], QS[7], s);
      s = fma(D[27], QS[8], s);
      s = fma(D[28], QS[9], s);
      local[60] += s;
      s = fma(D[36], QS[10], s);
      s = fma(D[38], QS[11], s);
      s = fma(D[39], QS[12], s);
      s = fma(D[41], QS[13], s);
      s = fma(D[42], QS[14], s);
      s = fma(D[43], QS[15], s);
      s = fma(D[45], QS[16], s);
      s = fma(D[46], QS[17], s);
      s = fma(D[47], QS[18], s);
      s = fma(D[48], QS[19], s);
      local[4] -= s;
    }
    {
      double s = D[6] * QS[0];
      s = fma(D[12], QS[1], s);
      s = fma(D[14], QS[2], s);
      s = fma(D[15], QS[3], s);
      s = fma(D[22], QS[4], s);
      s = fma(D[24], QS[5], s);
      s = fma(D[25], QS[6], s);
      s = fma(D[27], QS[7], s);
      s = fma(D[28], QS[8], s);
      s = fma(D[29], QS[9], s);
      local[61] += s;
      s = fma(D[37], QS[10], s);
      s = fma(D[39], QS[11], s);
      s = fma(D[40], QS[12], s);
      s = fma(D[42], QS[13], s);
      s = fma(D[43], QS[14], s);
      s = fma(D[44], QS[15], s);
      s = fma(D[46], QS[16], s);
      s = fma(D[47], QS[17], s);
      s = fma(D[48], QS[18], s);
      s = fma(D[49], QS[19], s);
      local[5] -= s;
    }
    {
      double s = D[7] * QS[0];
      s = fma(D[13], QS[1], s);
      s = fma(D[16], QS[2], s);
      s = fma(D[17], QS[3], s);
      s = fma(D[23], QS[4], s);
      s = fma(D[26], QS[5], s);
      s = fma(D[27], QS[6], s);
      s = fma(D[30], QS[7], s);
      s = fma(D[31], QS[8], s);
      s = fma(D[32], QS[9], s);
      local[62] += s;
      s = fma(D[38], QS[10], s);
      s = fma(D[41], QS[11], s);
      s = fma(D[42], QS[12], s);
      s = fma(D[45], QS[13], s);
      s = fma(D[46], QS[14], s);
      s = fma(D[47], QS[15], s);
      s = fma(D[50], QS[16], s);
      s = fma(D[51], QS[17], s);
      s = fma(D[52], QS[18], s);
      s = fma(D[53], QS[19], s);
      local[6] -= s;
    }
    {
      double s = D[8] * QS[0];
      s = fma(D[14], QS[1], s);
      s = fma(D[17], QS[2], s);
      s = fma(D[18], QS[3], s);
      s = fma(D[24], QS[4], s);
      s = fma(D[27], QS[5], s);
      s = fma(D[28], QS[6], s);
      s = fma(D[31], QS[7], s);
      s = fma(D[32], QS[8], s);
      s = fma(D[33], QS[9], s);
      local[63] += s;
      s = fma(D[39], QS[10], s);
      s = fma(D[42], QS[11], s);
      s = fma(D[43], QS[12], s);
      s = fma(D[46], QS[13], s);
      s = fma(D[47], QS[14], s);
      s = fma(D[48], QS[15], s);
      s = fma(D[51], QS[16], s);
      s = fma(D[52], QS[17], s);
      s = fma(D[53], QS[18], s);
      s = fma(D[54], QS[19], s);
      local[7] -= s;
    }
    {
      double s = D[9] * QS[0];
      s = fma(D[15], QS[1], s);
      s = fma(D[18], QS[2], s);
      s = fma(D[19], QS[3], s);
      s = fma(D[25], QS[4], s);
      s = fma(D[28], QS[5], s);
      s = fma(D[29], QS[6], s);
      s = fma(D[32], QS[7], s);
      s = fma(D[33], QS[8], s);
      s = fma(D[34], QS[9], s);
      local[64] += s;
      s = fma(D[40], QS[10], s);
      s = fma(D[43], QS[11], s);
      s = fma(D[44], QS[12], s);
      s = fma(D[47], QS[13], s);
      s = fma(D[48], QS[14], s);
      s = fma(D[49], QS[15], s);
      s = fma(D[52], QS[16], s);
      s = fma(D[53], QS[17], s);
      s = fma(D[54], QS[18], s);
      s = fma(D[55], QS[19], s);
      local[8] -= s;
    }
    {
      double s = D[10] * QS[0];
      s = fma(D[20], QS[1], s);
      s = fma(D[21], QS[2], s);
      s = fma(D[22], QS[3], s);
      local[65] -= s;
      s = fma(D[35], QS[4], s);
      s = fma(D[36], QS[5], s);
      s = fma(D[37], QS[6], s);
      s = fma(D[38], QS[7], s);
      s = fma(D[39], QS[8], s);
      s = fma(D[40], QS[9], s);
      local[9] += s;
    }
    {
      double s = D[11] * QS[0];
      s = fma(D[21], QS[1], s);
      s = fma(D[23], QS[2], s);
      s = fma(D[24], QS[3], s);
      local[66] -= s;
      s = fma(D[36], QS[4], s);
      s = fma(D[38], QS[5], s);
      s = fma(D[39], QS[6], s);
      s = fma(D[41], QS[7], s);
      s = fma(D[42], QS[8], s);
      s = fma(D[43], QS[9], s);
      local[10] += s;
    }
    {
      double s = D[12] * QS[0];
      s = fma(D[22], QS[1], s);
      s = fma(D[24], QS[2], s);
      s = fma(D[25], QS[3], s);
      local[67] -= s;
      s = fma(D[37], QS[4], s);
      s = fma(D[39], QS[5], s);
      s = fma(D[40], QS[6], s);
      s = fma(D[42], QS[7], s);
      s = fma(D[43], QS[8], s);
      s = fma(D[44], QS[9], s);
      local[11] += s;
    }
    {
      double s = D[13] * QS[0];
      s = fma(D[23], QS[1], s);
      s = fma(D[26], QS[2], s);
      s = fma(D[27], QS[3], s);
      local[68] -= s;
      s = fma(D[38], QS[4], s);
      s = fma(D[41], QS[5], s);
      s = fma(D[42], QS[6], s);
      s = fma(D[45], QS[7], s);
      s = fma(D[46], QS[8], s);
      s = fma(D[47], QS[9], s);
      local[12] += s;
    }
    {
      double s = D[14] * QS[0];
      s = fma(D[24], QS[1], s);
      s = fma(D[27], QS[2], s);
      s = fma(D[28], QS[3], s);
      local[69] -= s;
      s = fma(D[39], QS[4], s);
      s = fma(D[42], QS[5], s);
      s = fma(D[43], QS[6], s);
      s = fma(D[46], QS[7], s);
      s = fma(D[47], QS[8], s);
      s = fma(D[48], QS[9], s);
      local[13] += s;
    }
    {
      double s = D[15] * QS[0];
      s = fma(D[25], QS[1], s);
      s = fma(D[28], QS[2], s);
      s = fma(D[29], QS[3], s);
      local[70] -= s;
      s = fma(D[40], QS[4], s);
      s = fma(D[43], QS[5], s);
      s = fma(D[44], QS[6], s);
      s = fma(D[47], QS[7], s);
      s = fma(D[48], QS[8], s);
      s = fma(D[49], QS[9], s);
      local[14] += s;
    }
    {
      double s = D[16] * QS[0];
      s = fma(D[26], QS[1], s);
      s = fma(D[30], QS[2], s);
      s = fma(D[31], QS[3], s);
      local[71] -= s;
      s = fma(D[41], QS[4], s);
      s = fma(D[45], QS[5], s);
      s = fma(D[46], QS[6], s);
      s = fma(D[50], QS[7], s);
      s = fma(D[51], QS[8], s);
      s = fma(D[52], QS[9], s);
      local[15] += s;
    }
    {
      double s = D[17] * QS[0];
      s = fma(D[27], QS[1], s);
      s = fma(D[31], QS[2], s);
      s = fma(D[32], QS[3], s);
      local[72] -= s;
      s = fma(D[42], QS[4], s);
      s = fma(D[46], QS[5], s);
      s = fma(D[47], QS[6], s);
      s = fma(D[51], QS[7], s);
      s = fma(D[52], QS[8], s);
      s = fma(D[53], QS[9], s);
      local[16] += s;
    }
    {
      double s = D[18] * QS[0];
      s = fma(D[28], QS[1], s);
      s = fma(D[32], QS[2], s);
      s = fma(D[33], QS[3], s);
      local[73] -= s;
      s = fma(D[43], QS[4], s);
      s = fma(D[47], QS[5], s);
      s = fma(D[48], QS[6], s);
      s = fma(D[52], QS[7], s);
      s = fma(D[53], QS[8], s);
      s = fma(D[54], QS[9], s);
      local[17] += s;
    }
    {
      double s = D[19] * QS[0];
      s = fma(D[29], QS[1], s);
      s = fma(D[33], QS[2], s);
      s = fma(D[34], QS[3], s);
      local[74] -= s;
      s = fma(D[44], QS[4], s);
      s = fma(D[48], QS[5], s);
      s = fma(D[49], QS[6], s);
      s = fma(D[53], QS[7], s);
      s = fma(D[54], QS[8], s);
      s = fma(D[55], QS[9], s);
      local[18] += s;
    }
    {
      double s = D[20] * QS[0];
      local[75] += s;
      s = fma(D[35], QS[1], s);
      s = fma(D[36], QS[2], s);
      s = fma(D[37], QS[3], s);
      local[19] -= s;
    }
    {
      double s = D[21] * QS[0];
      local[76] += s;
      s = fma(D[36], QS[1], s);
      s = fma(D[38], QS[2], s);
      s = fma(D[39], QS[3], s);
      local[20] -= s;
    }
    {
      double s = D[22] * QS[0];
      local[77] += s;
      s = fma(D[37], QS[1], s);
      s = fma(D[39], QS[2], s);
      s = fma(D[40], QS[3], s);
      local[21] -= s;
    }
    {
      double s = D[23] * QS[0];
      local[78] += s;
      s = fma(D[38], QS[1], s);
      s = fma(D[41], QS[2], s);
      s = fma(D[42], QS[3], s);
      local[22] -= s;
    }
    {
      double s = D[24] * QS[0];
      local[79] += s;
      s = fma(D[39], QS[1], s);
      s = fma(D[42], QS[2], s);
      s = fma(D[43], QS[3], s);
      local[23] -= s;
    }
    {
      double s = D[25] * QS[0];
      local[80] += s;
      s = fma(D[40], QS[1], s);
      s = fma(D[43], QS[2], s);
      s = fma(D[44], QS[3], s);
      local[24] -= s;
    }
    {
      double s = D[26] * QS[0];
      local[81] += s;
      s = fma(D[41], QS[1], s);
      s = fma(D[45], QS[2], s);
      s = fma(D[46], QS[3], s);
      local[25] -= s;
    }
    {
      double s = D[27] * QS[0];
      local[82] += s;
      s = fma(D[42], QS[1], s);
      s = fma(D[46], QS[2], s);
      s = fma(D[47], QS[3], s);
      local[26] -= s;
    }
    {
      double s = D[28] * QS[0];
      local[83] += s;
      s = fma(D[43], QS[1], s);
      s = fma(D[47], QS[2], s);
      s = fma(D[48], QS[3], s);
      local[27] -= s;
    }
    {
      double s = D[29] * QS[0];
      local[84] += s;
      s = fma(D[44], QS[1], s);
      s = fma(D[48], QS[2], s);
      s = fma(D[49], QS[3], s);
      local[28] -= s;
    }
    {
      double s = D[30] * QS[0];
      local[85] += s;
      s = fma(D[45], QS[1], s);
      s = fma(D[50], QS[2], s);
      s = fma(D[51], QS[3], s);
      local[29] -= s;
    }
    {
      double s = D[31] * QS[0];
      local[86] += s;
      s = fma(D[46], QS[1], s);
      s = fma(D[51], QS[2], s);
      s = fma(D[52], QS[3], s);
      local[30] -= s;
    }
    {
      double s = D[32] * QS[0];
      local[87] += s;
      s = fma(D[47], QS[1], s);
      s = fma(D[52], QS[2], s);
      s = fma(D[53], QS[3], s);
      local[31] -= s;
    }
    {
      double s = D[33] * QS[0];
      local[88] += s;
      s = fma(D[48], QS[1], s);
      s = fma(D[53], QS[2], s);
      s = fma(D[54], QS[3], s);
      local[32] -= s;
    }
    {
      double s = D[34] * QS[0];
      local[89] += s;
      s = fma(D[49], QS[1], s);
      s = fma(D[54], QS[2], s);
      s = fma(D[55], QS[3], s);
      local[33] -= s;
    }
    {
      double s = D[35] * QS[0];
      local[34] += s;
    }
    {
      double s = D[36] * QS[0];
      local[35] += s;
    }
    {
      double s = D[37] * QS[0];
      local[36] += s;
    }
    {
      double s = D[38] * QS[0];
      local[37] += s;
    }
    {
      double s = D[39] * QS[0];
      local[38] += s;
    }
    {
      double s = D[40] * QS[0];
      local[39] += s;
    }
    {
      double s = D[41] * QS[0];
      local[40] += s;
    }
    {
      double s = D[42] * QS[0];
      local[41] += s;
    }
    {
      double s = D[43] * QS[0];
      local[42] += s;
    }
    {
      double s = D[44] * QS[0];
      local[43] += s;
    }
    {
      double s = D[45] * QS[0];
      local[44] += s;
    }
    {
      double s = D[46] * QS[0];
      local[45] += s;
    }
    {
      double s = D[47] * QS[0];
      local[46] += s;
    }
    {
      double s = D[48] * QS[0];
      local[47] += s;
    }
    {
      double s = D[49] * QS[0];
      local[48] += s;
    }
    {
      double s = D[50] * QS[0];
      local[49] += s;
    }
    {
      double s = D[51] * QS[0];
      local[50] += s;
    }
    {
      double s = D[52] * QS[0];
      local[51] += s;
    }
    {
      double s = D[53] * QS[0];
      local[52] += s;
    }
    {
      double s = D[54] * QS[0];
      local[53] += s;
    }
    {
      double s = D[55] * QS[0];
      local[54] += s;
    }
    {
      double s = D[0] * QS[0];
      s = fma(D[1], QS[1], s);
      s = fma(D[2], QS[2], s);
      s = fma(D[3], QS[3], s);
      s = fma(D[4], QS[4], s);
      s = fma(D[5], QS[5], s);
      s = fma(D[6], QS[6], s);
      s = fma(D[7], QS[7], s);
      s = fma(D[8], QS[8], s);
      s = fma(D[9], QS[9], s);
      s = fma(D[10], QS[10], s);
      s = fma(D[11], QS[11], s);
      s = fma(D[12], QS[12], s);
      s = fma(D[13], QS[13], s);
      s = fma(D[14], QS[14], s);
      s = fma(D[15], QS[15], s);
      s = fma(D[16], QS[16], s);
      s = fma(D[17], QS[17], s);
      s = fma(D[18], QS[18], s);
      s = fma(D[19], QS[19], s);
      s = fma(D[20], QS[20], s);
      s = fma(D[21], QS[21], s);
      s = fma(D[22], QS[22], s);
      s = fma(D[23], QS[23], s);
      s = fma(D[24], QS[24], s);
      s = fma(D[25], QS[25], s);
      s = fma(D[26], QS[26], s);
      s = fma(D[27], QS[27], s);
      s = fma(D[28], QS[28], s);
      s = fma(D[29], QS[29], s);
      s = fma(D[30], QS[30], s);
      s = fma(D[31], QS[31], s);
      s = fma(D[32], QS[32], s);
      s = fma(D[33], QS[33], s);
      s = fma(D[34], QS[34], s);
      local[55] += s;
    }
    {
      double s = D[1] * QTs[0];
      s = fma(D[4], QTs[1], s);
      s = fma(D[5], QTs[2], s);
      s = fma(D[6], QTs[3], s);
      s = fma(D[10], QTs[4], s);
      s = fma(D[11], QTs[5], s);
      s = fma(D[12], QTs[6], s);
      s = fma(D[13], QTs[7], s);
      s = fma(D[14], QTs[8], s);
      s = fma(D[15], QTs[9], s);
      s = fma(D[20], QTs[10], s);
      s = fma(D[21], QTs[11], s);
      s = fma(D[22], QTs[12], s);
      s = fma(D[23], QTs[13], s);
      s = fma(D[24], QTs[14], s);
      s = fma(D[25], QTs[15], s);
      s = fma(D[26], QTs[16], s);
      s = fma(D[27], QTs[17], s);
      s = fma(D[28], QTs[18], s);
      s = fma(D[29], QTs[19], s);
      unsafeAtomicAdd(&outS[56], s);
      s = fma(D[35], QTs[20], s);
      s = fma(D[36], QTs[21], s);
      s = fma(D[37], QTs[22], s);
      s = fma(D[38], QTs[23], s);
      s = fma(D[39], QTs[24], s);
      s = fma(D[40], QTs[25], s);
      s = fma(D[41], QTs[26], s);
      s = fma(D[42], QTs[27], s);
      s = fma(D[43], QTs[28], s);
      s = fma(D[44], QTs[29], s);
      s = fma(D[45], QTs[30], s);
      s = fma(D[46], QTs[31], s);
      s = fma(D[47], QTs[32], s);
      s = fma(D[48], QTs[33], s);
      s = fma(D[49], QTs[34], s);
      unsafeAtomicAdd(&outS[0], -s);
    }
    {
      double s = D[2] * QTs[0];
      s = fma(D[5], QTs[1], s);
      s = fma(D[7], QTs[2], s);
      s = fma(D[8], QTs[3], s);
      s = fma(D[11], QTs[4], s);
      s = fma(D[13], QTs[5], s);
      s = fma(D[14], QTs[6], s);
      s = fma(D[16], QTs[7], s);
      s = fma(D[17], QTs[8], s);
      s = fma(D[18], QTs[9], s);
      s = fma(D[21], QTs[10], s);
      s = fma(D[23], QTs[11], s);
      s = fma(D[24], QTs[12], s);
      s = fma(D[26], QTs[13], s);
      s = fma(D[27], QTs[14], s);
      s = fma(D[28], QTs[15], s);
      s = fma(D[30], QTs[16], s);
      s = fma(D[31], QTs[17], s);
      s = fma(D[32], QTs[18], s);
      s = fma(D[33], QTs[19], s);
      unsafeAtomicAdd(&outS[57], s);
      s = fma(D[36], QTs[20], s);
      s = fma(D[38], QTs[21], s);
      s = fma(D[39], QTs[22], s);
      s = fma(D[41], QTs[23], s);
      s = fma(D[42], QTs[24], s);
      s = fma(D[43], QTs[25], s);
      s = fma(D[45], QTs[26], s);
      s = fma(D[46], QTs[27], s);
      s = fma(D[47], QTs[28], s);
      s = fma(D[48], QTs[29], s);
      s = fma(D[50], QTs[30], s);
      s = fma(D[51], QTs[31], s);
      s = fma(D[52], QTs[32], s);
      s = fma(D[53], QTs[33], s);
      s = fma(D[54], QTs[34], s);
      unsafeAtomicAdd(&outS[1], -s);
    }
    {
      double s = D[3] * QTs[0];
      s = fma(D[6], QTs[1], s);
      s = fma(D[8], QTs[2], s);
      s = fma(D[9], QTs[3], s);
      s = fma(D[12], QTs[4], s);
      s = fma(D[14], QTs[5], s);
      s = fma(D[15], QTs[6], s);
      s = fma(D[17], QTs[7], s);
      s = fma(D[18], QTs[8], s);
      s = fma(D[19], QTs[9], s);
      s = fma(D[22], QTs[10], s);
      s = fma(D[24], QTs[11], s);
      s = fma(D[25], QTs[12], s);
      s = fma(D[27], QTs[13], s);
      s = fma(D[28], QTs[14], s);
      s = fma(D[29], QTs[15], s);
      s = fma(D[31], QTs[16], s);
      s = fma(D[32], QTs[17], s);
      s = fma(D[33], QTs[18], s);
      s = fma(D[34], QTs[19], s);
      unsafeAtomicAdd(&outS[58], s);
      s = fma(D[37], QTs[20], s);
      s = fma(D[39], QTs[21], s);
      s = fma(D[40], QTs[22], s);
      s = fma(D[42], QTs[23], s);
      s = fma(D[43], QTs[24], s);
      s = fma(D[44], QTs[25], s);
      s = fma(D[46], QTs[26], s);
      s = fma(D[47], QTs[27], s);
      s = fma(D[48], QTs[28], s);
      s = fma(D[49], QTs[29], s);
      s = fma(D[51], QTs[30], s);
      s = fma(D[52], QTs[31], s);
      s = fma(D[53], QTs[32], s);
      s = fma(D[54], QTs[33], s);
      s = fma(D[55], QTs[34], s);
      unsafeAtomicAdd(&outS[2], -s);
    }
    {
      double s = D[4] * QTs[0];
      s = fma(D[10], QTs[1], s);
      s = fma(D[11], QTs[2], s);
      s = fma(D[12], QTs[3], s);
      s = fma(D[20], QTs[4], s);
      s = fma(D[21], QTs[5], s);
      s = fma(D[22], QTs[6], s);
      s = fma(D[23], QTs[7], s);
      s = fma(D[24], QTs[8], s);
      s = fma(D[25], QTs[9], s);
      unsafeAtomicAdd(&outS[59], s);
      s = fma(D[35], QTs[10], s);
      s = fma(D[36], QTs[11], s);
      s = fma(D[37], QTs[12], s);
      s = fma(D[38], QTs[13], s);
      s = fma(D[39], QTs[14], s);
      s = fma(D[40], QTs[15], s);
      s = fma(D[41], QTs[16], s);
      s = fma(D[42], QTs[17], s);
      s = fma(D[43], QTs[18], s);
      s = fma(D[44], QTs[19], s);
      unsafeAtomicAdd(&outS[3], -s);
    }
    {
      double s = D[5] * QTs[0];
      s = fma(D[11], QTs[1], s);
      s = fma(D[13], QTs[2], s);
      s = fma(D[14], QTs[3], s);
      s = fma(D[21], QTs[4], s);
      s = fma(D[23], QTs[5], s);
      s = fma(D[24], QTs[6], s);
      s = fma(D[26], QTs[7], s);
      s = fma(D[27], QTs[8], s);
      s = fma(D[28], QTs[9], s);
      unsafeAtomicAdd(&outS[60], s);
      s = fma(D[36], QTs[10], s);
      s = fma(D[38], QTs[11], s);
      s = fma(D[39], QTs[12], s);
      s = fma(D[41], QTs[13], s);
      s = fma(D[42], QTs[14], s);
      s = fma(D[43], QTs[15], s);
      s = fma(D[45], QTs[16], s);
      s = fma(D[46], QTs[17], s);
      s = fma(D[47], QTs[18], s);
      s = fma(D[48], QTs[19], s);
      unsafeAtomicAdd(&outS[4], -s);
    }
    {
      double s = D[6] * QTs[0];
      s = fma(D[12], QTs[1], s);
      s = fma(D[14], QTs[2], s);
      s = fma(D[15], QTs[3], s);
      s = fma(D[22], QTs[4], s);
      s = fma(D[24], QTs[5], s);
      s = fma(D[25], QTs[6], s);
      s = fma(D[27], QTs[7], s);
      s = fma(D[28], QTs[8], s);
      s = fma(D[29], QTs[9], s);
      unsafeAtomicAdd(&outS[61], s);
      s = fma(D[37], QTs[10], s);
      s = fma(D[39], QTs[11], s);
      s = fma(D[40], QTs[12], s);
      s = fma(D[42], QTs[13], s);
      s = fma(D[43], QTs[14], s);
      s = fma(D[44], QTs[15], s);
      s = fma(D[46], QTs[16], s);
      s = fma(D[47], QTs[17], s);
      s = fma(D[48], QTs[18], s);
      s = fma(D[49], QTs[19], s);
      unsafeAtomicAdd(&outS[5], -s);
    }
    {
      double s = D[7] * QTs[0];
      s = fma(D[13], QTs[1], s);
      s = fma(D[16], QTs[2], s);
      s = fma(D[17], QTs[3], s);
      s = fma(D[23], QTs[4], s);
      s = fma(D[26], QTs[5], s);
      s = fma(D[27], QTs[6], s);
      s = fma(D[30], QTs[7], s);
      s = fma(D[31], QTs[8], s);
      s = fma(D[32], QTs[9], s);
      unsafeAtomicAdd(&outS[62], s);
      s = fma(D[38], QTs[10], s);
      s = fma(D[41], QTs[11], s);
      s = fma(D[42], QTs[12], s);
      s = fma(D[45], QTs[13], s);
      s = fma(D[46], QTs[14], s);
      s = fma(D[47], QTs[15], s);
      s = fma(D[50], QTs[16], s);
      s = fma(D[51], QTs[17], s);
      s = fma(D[52], QTs[18], s);
      s = fma(D[53], QTs[19], s);
      unsafeAtomicAdd(&outS[6], -s);
    }
    {
      double s = D[8] * QTs[0];
      s = fma(D[14], QTs[1], s);
      s = fma(D[17], QTs[2], s);
      s = fma(D[18], QTs[3], s);
      s = fma(D[24], QTs[4], s);
      s = fma(D[27], QTs[5], s);
      s = fma(D[28], QTs[6], s);
      s = fma(D[31], QTs[7], s);
      s = fma(D[32], QTs[8], s);
      s = fma(D[33], QTs[9], s);
      unsafeAtomicAdd(&outS[63], s);
      s = fma(D[39], QTs[10], s);
      s = fma(D[42], QTs[11], s);
      s = fma(D[43], QTs[12], s);
      s = fma(D[46], QTs[13], s);
      s = fma(D[47], QTs[14], s);
      s = fma(D[48], QTs[15], s);
      s = fma(D[51], QTs[16], s);
      s = fma(D[52], QTs[17], s);
      s = fma(D[53], QTs[18], s);
      s = fma(D[54], QTs[19], s);
      unsafeAtomicAdd(&outS[7], -s);
    }
    {
      double s = D[9] * QTs[0];
      s = fma(D[15], QTs[1], s);
      s = fma(D[18], QTs[2], s);
      s = fma(D[19], QTs[3], s);
      s = fma(D[25], QTs[4], s);
      s = fma(D[28], QTs[5], s);
      s = fma(D[29], QTs[6], s);
      s = fma(D[32], QTs[7], s);
      s = fma(D[33], QTs[8], s);
      s = fma(D[34], QTs[9], s);
      unsafeAtomicAdd(&outS[64], s);
      s = fma(D[40], QTs[10], s);
      s = fma(D[43], QTs[11], s);
      s = fma(D[44], QTs[12], s);
      s = fma(D[47], QTs[13], s);
      s = fma(D[48], QTs[14], s);
      s = fma(D[49], QTs[15], s);
      s = fma(D[52], QTs[16], s);
      s = fma(D[53], QTs[17], s);
      s = fma(D[54], QTs[18], s);
      s = fma(D[55], QTs[19], s);
      unsafeAtomicAdd(&outS[8], -s);
    }
    {
      double s = D[10] * QTs[0];
      s = fma(D[20], QTs[1], s);
      s = fma(D[21], QTs[2], s);
      s = fma(D[22], QTs[3], s);
      unsafeAtomicAdd(&outS[65], s);
      s = fma(D[35], QTs[4], s);
      s = fma(D[36], QTs[5], s);
      s = fma(D[37], QTs[6], s);
      s = fma(D[38], QTs[7], s);
      s = fma(D[39], QTs[8], s);
      s = fma(D[40], QTs[9], s);
      unsafeAtomicAdd(&outS[9], -s);
    }
    {
      double s = D[11] * QTs[0];
      s = fma(D[21], QTs[1], s);
      s = fma(D[23], QTs[2], s);
      s = fma(D[24], QTs[3], s);
      unsafeAtomicAdd(&outS[66], s);
      s = fma(D[36], QTs[4], s);
      s = fma(D[38], QTs[5], s);
      s = fma(D[39], QTs[6], s);
      s = fma(D[41], QTs[7], s);
      s = fma(D[42], QTs[8], s);
      s = fma(D[43], QTs[9], s);
      unsafeAtomicAdd(&outS[10], -s);
    }
    {
      double s = D[12] * QTs[0];
      s = fma(D[22], QTs[1], s);
      s = fma(D[24], QTs[2], s);
      s = fma(D[25], QTs[3], s);
      unsafeAtomicAdd(&outS[67], s);
      s = fma(D[37], QTs[4], s);
      s = fma(D[39], QTs[5], s);
      s = fma(D[40], QTs[6], s);
      s = fma(D[42], QTs[7], s);
      s = fma(D[43], QTs[8], s);
      s = fma(D[44], QTs[9], s);
      unsafeAtomicAdd(&outS[11], -s);
    }
    {
      double s = D[13] * QTs[0];
      s = fma(D[23], QTs[1], s);
      s = fma(D[26], QTs[2], s);
      s = fma(D[27], QTs[3], s);
      unsafeAtomicAdd(&outS[68], s);
      s = fma(D[38], QTs[4], s);
      s = fma(D[41], QTs[5], s);
      s = fma(D[42], QTs[6], s);
      s = fma(D[45], QTs[7], s);
      s = fma(D[46], QTs[8], s);
      s = fma(D[47], QTs[9], s);
      unsafeAtomicAdd(&outS[12], -s);
    }
    {
      double s = D[14] * QTs[0];
      s = fma(D[24], QTs[1], s);
      s = fma(D[27], QTs[2], s);
      s = fma(D[28], QTs[3], s);
      unsafeAtomicAdd(&outS[69], s);
      s = fma(D[39], QTs[4], s);
      s = fma(D[42], QTs[5], s);
      s = fma(D[43], QTs[6], s);
      s = fma(D[46], QTs[7], s);
      s = fma(D[47], QTs[8], s);
      s = fma(D[48], QTs[9], s);
      unsafeAtomicAdd(&outS[13], -s);
    }
    {
      double s = D[15] * QTs[0];
      s = fma(D[25], QTs[1], s);
      s = fma(D[28], QTs[2], s);
      s = fma(D[29], QTs[3], s);
      unsafeAtomicAdd(&outS[70], s);
      s = fma(D[40], QTs[4], s);
      s = fma(D[43], QTs[5], s);
      s = fma(D[44], QTs[6], s);
      s = fma(D[47], QTs[7], s);
      s = fma(D[48], QTs[8], s);
      s = fma(D[49], QTs[9], s);
      unsafeAtomicAdd(&outS[14], -s);
    }
    {
      double s = D[16] * QTs[0];
      s = fma(D[26], QTs[1], s);
      s = fma(D[30], QTs[2], s);
      s = fma(D[31], QTs[3], s);
      unsafeAtomicAdd(&outS[71], s);
      s = fma(D[41], QTs[4], s);
      s = fma(D[45], QTs[5], s);
      s = fma(D[46], QTs[6], s);
      s = fma(D[50], QTs[7], s);
      s = fma(D[51], QTs[8], s);
      s = fma(D[52], QTs[9], s);
      unsafeAtomicAdd(&outS[15], -s);
    }
    {
      double s = D[17] * QTs[0];
      s = fma(D[27], QTs[1], s);
      s = fma(D[31], QTs[2], s);
      s = fma(D[32], QTs[3], s);
      unsafeAtomicAdd(&outS[72], s);
      s = fma(D[42], QTs[4], s);
      s = fma(D[46], QTs[5], s);
      s = fma(D[47], QTs[6], s);
      s = fma(D[51], QTs[7], s);
      s = fma(D[52], QTs[8], s);
      s = fma(D[53], QTs[9], s);
      unsafeAtomicAdd(&outS[16], -s);
    }
    {
      double s = D[18] * QTs[0];
      s = fma(D[28], QTs[1], s);
      s = fma(D[32], QTs[2], s);
      s = fma(D[33], QTs[3], s);
      unsafeAtomicAdd(&outS[73], s);
      s = fma(D[43], QTs[4], s);
      s = fma(D[47], QTs[5], s);
      s = fma(D[48], QTs[6], s);
      s = fma(D[52], QTs[7], s);
      s = fma(D[53], QTs[8], s);
      s = fma(D[54], QTs[9], s);
      unsafeAtomicAdd(&outS[17], -s);
    }
    {
      double s = D[19] * QTs[0];
      s = fma(D[29], QTs[1], s);
      s = fma(D[33], QTs[2], s);
      s = fma(D[34], QTs[3], s);
      unsafeAtomicAdd(&outS[74], s);
      s = fma(D[44], QTs[4], s);
      s = fma(D[48], QTs[5], s);
      s = fma(D[49], QTs[6], s);
      s = fma(D[53], QTs[7], s);
      s = fma(D[54], QTs[8], s);
      s = fma(D[55], QTs[9], s);
      unsafeAtomicAdd(&outS[18], -s);
    }
    {
      double s = D[20] * QTs[0];
      unsafeAtomicAdd(&outS[75], s);
      s = fma(D[35], QTs[1], s);
      s = fma(D[36], QTs[2], s);
      s = fma(D[37], QTs[3], s);
      unsafeAtomicAdd(&outS[19], -s);
    }
    {
      double s = D[21] * QTs[0];
      unsafeAtomicAdd(&outS[76], s);
      s = fma(D[36], QTs[1], s);
      s = fma(D[38], QTs[2], s);
      s = fma(D[39], QTs[3], s);
      unsafeAtomicAdd(&outS[20], -s);
    }
    {
      double s = D[22] * QTs[0];
      unsafeAtomicAdd(&outS[77], s);
      s = fma(D[37], QTs[1], s);
      s = fma(D[39], QTs[2], s);
      s = fma(D[40], QTs[3], s);
      unsafeAtomicAdd(&outS[21], -s);
    }
    {
      double s = D[23] * QTs[0];
      unsafeAtomicAdd(&outS[78], s);
      s = fma(D[38], QTs[1], s);
      s = fma(D[41], QTs[2], s);
      s = fma(D[42], QTs[3], s);
      unsafeAtomicAdd(&outS[22], -s);
    }
    {
      double s = D[24] * QTs[0];
      unsafeAtomicAdd(&outS[79], s);
      s = fma(D[39], QTs[1], s);
      s = fma(D[42], QTs[2], s);
      s = fma(D[43], QTs[3], s);
      unsafeAtomicAdd(&outS[23], -s);
    }
    {
      double s = D[25] * QTs[0];
      unsafeAtomicAdd(&outS[80], s);
      s = fma(D[40], QTs[1], s);
      s = fma(D[43], QTs[2], s);
      s = fma(D[44], QTs[3], s);
      unsafeAtomicAdd(&outS[24], -s);
    }
    {
      double s = D[26] * QTs[0];
      unsafeAtomicAdd(&outS[81], s);
      s = fma(D[41], QTs[1], s);
      s = fma(D[45], QTs[2], s);
      s = fma(D[46], QTs[3], s);
      unsafeAtomicAdd(&outS[25], -s);
    }
    {
      double s = D[27] * QTs[0];
      unsafeAtomicAdd(&outS[82], s);
      s = fma(D[42], QTs[1], s);
      s = fma(D[46], QTs[2], s);
      s = fma(D[47], QTs[3], s);
      unsafeAtomicAdd(&outS[26], -s);
    }
    {
      double s = D[28] * QTs[0];
      unsafeAtomicAdd(&outS[83], s);
      s = fma(D[43], QTs[1], s);
      s = fma(D[47], QTs[2], s);
      s = fma(D[48], QTs[3], s);
      unsafeAtomicAdd(&outS[27], -s);
    }
    {
      double s = D[29] * QTs[0];
      unsafeAtomicAdd(&outS[84], s);
      s = fma(D[44], QTs[1], s);
      s = fma(D[48], QTs[2], s);
      s = fma(D[49], QTs[3], s);
      unsafeAtomicAdd(&outS[28], -s);
    }
    {
      double s = D[30] * QTs[0];
      unsafeAtomicAdd(&outS[85], s);
      s = fma(D[45], QTs[1], s);
      s = fma(D[50], QTs[2], s);
      s = fma(D[51], QTs[3], s);
      unsafeAtomicAdd(&outS[29], -s);
    }
    {
      double s = D[31] * QTs[0];
      unsafeAtomicAdd(&outS[86], s);
      s = fma(D[46], QTs[1], s);
      s = fma(D[51], QTs[2], s);
      s = fma(D[52], QTs[3], s);
      unsafeAtomicAdd(&outS[30], -s);
    }
    {
      double s = D[32] * QTs[0];
      unsafeAtomicAdd(&outS[87], s);
      s = fma(D[47], QTs[1], s);
      s = fma(D[52], QTs[2], s);
      s = fma(D[53], QTs[3], s);
      unsafeAtomicAdd(&outS[31], -s);
    }
    {
      double s = D[33] * QTs[0];
      unsafeAtomicAdd(&outS[88], s);
      s = fma(D[48], QTs[1], s);
      s = fma(D[53], QTs[2], s);
      s = fma(D[54], QTs[3], s);
      unsafeAtomicAdd(&outS[32], -s);
    }
    {
      double s = D[34] * QTs[0];
      unsafeAtomicAdd(&outS[89], s);
      s = fma(D[49], QTs[1], s);
      s = fma(D[54], QTs[2], s);
      s = fma(D[55], QTs[3], s);
      unsafeAtomicAdd(&outS[33], -s);
    }
    {
      double s = D[35] * QTs[0];
      unsafeAtomicAdd(&outS[34], -s);
    }
    {
      double s = D[36] * QTs[0];
      unsafeAtomicAdd(&outS[35], -s);
    }
    {
      double s = D[37] * QTs[0];
      unsafeAtomicAdd(&outS[36], -s);
    }
    {
      double s = D[38] * QTs[0];
      unsafeAtomicAdd(&outS[37], -s);
    }
    {
      double s = D[39] * QTs[0];
      unsafeAtomicAdd(&outS[38], -s);
    }
    {
      double s = D[40] * QTs[0];
      unsafeAtomicAdd(&outS[39], -s);
    }
    {
      double s = D[41] * QTs[0];
      unsafeAtomicAdd(&outS[40], -s);
    }
    {
      double s = D[42] * QTs[0];
      unsafeAtomicAdd(&outS[41], -s);
    }
    {
      double s = D[43] * QTs[0];
      unsafeAtomicAdd(&outS[42], -s);
    }
    {
      double s = D[44] * QTs[0];
      unsafeAtomicAdd(&outS[43], -s);
    }
    {
      double s = D[45] * QTs[0];
      unsafeAtomicAdd(&outS[44], -s);
    }
    {
      double s = D[46] * QTs[0];
      unsafeAtomicAdd(&outS[45], -s);
    }
    {
      double s = D[47] * QTs[0];
      unsafeAtomicAdd(&outS[46], -s);
    }
    {
      double s = D[48] * QTs[0];
      unsafeAtomicAdd(&outS[47], -s);
    }
    {
      double s = D[49] * QTs[0];
      unsafeAtomicAdd(&outS[48], -s);
    }
    {
      double s = D[50] * QTs[0];
      unsafeAtomicAdd(&outS[49], -s);
    }
    {
      double s = D[51] * QTs[0];
      unsafeAtomicAdd(&outS[50], -s);
    }
    {
      double s = D[52] * QTs[0];
      unsafeAtomicAdd(&outS[51], -s);
    }
    {
      double s = D[53] * QTs[0];
      unsafeAtomicAdd(&outS[52], -s);
    }
    {
      double s = D[54] * QTs[0];
      unsafeAtomicAdd(&outS[53], -s);
    }
    {
      double s = D[55] * QTs[0];
      unsafeAtomicAdd(&outS[54], -s);
    }
    {
      double s = D[0] * QTs[0];
      s = fma(D[1], QTs[1], s);
      s = fma(D[2], QTs[2], s);
      s = fma(D[3], QTs[3], s);
      s = fma(D[4], QTs[4], s);
      s = fma(D[5], QTs[5], s);
      s = fma(D[6], QTs[6], s);
      s = fma(D[7], QTs[7], s);
      s = fma(D[8], QTs[8], s);
      s = fma(D[9], QTs[9], s);
      s = fma(D[10], QTs[10], s);
      s = fma(D[11], QTs[11], s);
      s = fma(D[12], QTs[12], s);
      s = fma(D[13], QTs[13], s);
      s = fma(D[14], QTs[14], s);
      s = fma(D[15], QTs[15], s);
      s = fma(D[16], QTs[16], s);
      s = fma(D[17], QTs[17], s);
      s = fma(D[18], QTs[18], s);
      s = fma(D[19], QTs[19], s);
      s = fma(D[20], QTs[20], s);
      s = fma(D[21], QTs[21], s);
      s = fma(D[22], QTs[22], s);
      s = fma(D[23], QTs[23], s);
      s = fma(D[24], QTs[24], s);
      s = fma(D[25], QTs[25], s);
      s = fma(D[26], QTs[26], s);
      s = fma(D[27], QTs[27], s);
      s = fma(D[28], QTs[28], s);
      s = fma(D[29], QTs[29], s);
      s = fma(D[30], QTs[30], s);
      s = fma(D[31], QTs[31], s);
      s = fma(D[32], QTs[32], s);
      s = fma(D[33], QTs[33], s);
      s = fma(D[34], QTs[34], s);
      unsafeAtomicAdd(&outS[55], s);
    }
  }
  static constexpr int FLOPS_M2L_PAIR = 2278;  // both directions, + one rsqrt
  __device__ __forceinline__ static void l2l(const double* h, double* local) {
    double mh[35];
    mh[0] = 1.0;
    mh[1] = mh[0] * h[0];
    mh[2] = mh[0] * h[1];
    mh[3] = mh[0] * h[2];
    mh[4] = mh[1] * (h[0] * 0.5);
    mh[5] = mh[2] * h[0];
    mh[6] = mh[3] * h[0];
    mh[7] = mh[2] * (h[1] * 0.5);
    mh[8] = mh[3] * h[1];
    mh[9] = mh[3] * (h[2] * 0.5);
    mh[10] = mh[4] * (h[0] * 0.3333333333333333);
    mh[11] = mh[5] * (h[0] * 0.5);
    mh[12] = mh[6] * (h[0] * 0.5);
    mh[13] = mh[7] * h[0];
    mh[14] = mh[8] * h[0];
    mh[15] = mh[9] * h[0];
    mh[16] = mh[7] * (h[1] * 0.3333333333333333);
    mh[17] = mh[8] * (h[1] * 0.5);
    mh[18] = mh[9] * h[1];
    mh[19] = mh[9] * (h[2] * 0.3333333333333333);
    mh[20] = mh[10] * (h[0] * 0.25);
    mh[21] = mh[11] * (h[0] * 0.3333333333333333);
    mh[22] = mh[12] * (h[0] * 0.3333333333333333);
    mh[23] = mh[13] * (h[0] * 0.5);
    mh[24] = mh[14] * (h[0] * 0.5);
    mh[25] = mh[15] * (h[0] * 0.5);
    mh[26] = mh[16] * h[0];
    mh[27] = mh[17] * h[0];
    mh[28] = mh[18] * h[0];
    mh[29] = mh[19] * h[0];
    mh[30] = mh[16] * (h[1] * 0.25);
    mh[31] = mh[17] * (h[1] * 0.3333333333333333);
    mh[32] = mh[18] * (h[1] * 0.5);
    mh[33] = mh[19] * h[1];
    mh[34] = mh[19] * (h[2] * 0.25);
    local[0] = fma(local[48], mh[34], fma(local[47], mh[33], fma(local[46], mh[32], fma(local[45], mh[31], fma(local[44], mh[30], fma(local[43], mh[29], fma(local[42], mh[28], fma(local[41], mh[27], fma(local[40], mh[26], fma(local[39], mh[25], fma(local[38], mh[24], fma(local[37], mh[23], fma(local[36], mh[22], fma(local[35], mh[21], fma(local[34], mh[20], fma(local[28], mh[19], fma(local[27], mh[18], fma(local[26], mh[17], fma(local[25], mh[16], fma(local[24], mh[15], fma(local[23], mh[14], fma(local[22], mh[13], fma(local[21], mh[12], fma(local[20], mh[11], fma(local[19], mh[10], fma(local[14], mh[9], fma(local[13], mh[8], fma(local[12], mh[7], fma(local[11], mh[6], fma(local[10], mh[5], fma(local[9], mh[4], fma(local[5], mh[3], fma(local[4], mh[2], fma(local[3], mh[1], local[0]))))))))))))))))))))))))))))))))));
    local[1] = fma(local[53], mh[34], fma(local[52], mh[33], fma(local[51], mh[32], fma(local[50], mh[31], fma(local[49], mh[30], fma(local[47], mh[29], fma(local[46], mh[28], fma(local[45], mh[27], fma(local[44], mh[26], fma(local[42], mh[25], fma(local[41], mh[24], fma(local[40], mh[23], fma(local[38], mh[22], fma(local[37], mh[21], fma(local[35], mh[20], fma(local[32], mh[19], fma(local[31], mh[18], fma(local[30], mh[17], fma(local[29], mh[16], fma(local[27], mh[15], fma(local[26], mh[14], fma(local[25], mh[13], fma(local[23], mh[12], fma(local[22], mh[11], fma(local[20], mh[10], fma(local[17], mh[9], fma(local[16], mh[8], fma(local[15], mh[7], fma(local[13], mh[6], fma(local[12], mh[5], fma(local[10], mh[4], fma(local[7], mh[3], fma(local[6], mh[2], fma(local[4], mh[1], local[1]))))))))))))))))))))))))))))))))));
    local[2] = fma(local[54], mh[34], fma(local[53], mh[33], fma(local[52], mh[32], fma(local[51], mh[31], fma(local[50], mh[30], fma(local[48], mh[29], fma(local[47], mh[28], fma(local[46], mh[27], fma(local[45], mh[26], fma(local[43], mh[25], fma(local[42], mh[24], fma(local[41], mh[23], fma(local[39], mh[22], fma(local[38], mh[21], fma(local[36], mh[20], fma(local[33], mh[19], fma(local[32], mh[18], fma(local[31], mh[17], fma(local[30], mh[16], fma(local[28], mh[15], fma(local[27], mh[14], fma(local[26], mh[13], fma(local[24], mh[12], fma(local[23], mh[11], fma(local[21], mh[10], fma(local[18], mh[9], fma(local[17], mh[8], fma(local[16], mh[7], fma(local[14], mh[6], fma(local[13], mh[5], fma(local[11], mh[4], fma(local[8], mh[3], fma(local[7], mh[2], fma(local[5], mh[1], local[2]))))))))))))))))))))))))))))))))));
    local[3] = fma(local[43], mh[19], fma(local[42], mh[18], fma(local[41], mh[17], fma(local[40], mh[16], fma(local[39], mh[15], fma(local[38], mh[14], fma(local[37], mh[13], fma(local[36], mh[12], fma(local[35], mh[11], fma(local[34], mh[10], fma(local[24], mh[9], fma(local[23], mh[8], fma(local[22], mh[7], fma(local[21], mh[6], fma(local[20], mh[5], fma(local[19], mh[4], fma(local[11], mh[3], fma(local[10], mh[2], fma(local[9], mh[1], local[3])))))))))))))))))));
    local[4] = fma(local[47], mh[19], fma(local[46], mh[18], fma(local[45], mh[17], fma(local[44], mh[16], fma(local[42], mh[15], fma(local[41], mh[14], fma(local[40], mh[13], fma(local[38], mh[12], fma(local[37], mh[11], fma(local[35], mh[10], fma(local[27], mh[9], fma(local[26], mh[8], fma(local[25], mh[7], fma(local[23], mh[6], fma(local[22], mh[5], fma(local[20], mh[4], fma(local[13], mh[3], fma(local[12], mh[2], fma(local[10], mh[1], local[4])))))))))))))))))));
    local[5] = fma(local[48], mh[19], fma(local[47], mh[18], fma(local[46], mh[17], fma(local[45], mh[16], fma(local[43], mh[15], fma(local[42], mh[14], fma(local[41], mh[13], fma(local[39], mh[12], fma(local[38], mh[11], fma(local[36], mh[10], fma(local[28], mh[9], fma(local[27], mh[8], fma(local[26], mh[7], fma(local[24], mh[6], fma(local[23], mh[5], fma(local[21], mh[4], fma(local[14], mh[3], fma(local[13], mh[2], fma(local[11], mh[1], local[5])))))))))))))))))));
    local[6] = fma(local[52], mh[19], fma(local[51], mh[18], fma(local[50], mh[17], fma(local[49], mh[16], fma(local[46], mh[15], fma(local[45], mh[14], fma(local[44], mh[13], fma(local[41], mh[12], fma(local[40], mh[11], fma(local[37], mh[10], fma(local[31], mh[9], fma(local[30], mh[8], fma(local[29], mh[7], fma(local[26], mh[6], fma(local[25], mh[5], fma(local[22], mh[4], fma(local[16], mh[3], fma(local[15], mh[2], fma(local[12], mh[1], local[6])))))))))))))))))));
    local[7] = fma(local[53], mh[19], fma(local[52], mh[18], fma(local[51], mh[17], fma(local[50], mh[16], fma(local[47], mh[15], fma(local[46], mh[14], fma(local[45], mh[13], fma(local[42], mh[12], fma(local[41], mh[11], fma(local[38], mh[10], fma(local[32], mh[9], fma(local[31], mh[8], fma(local[30], mh[7], fma(local[27], mh[6], fma(local[26], mh[5], fma(local[23], mh[4], fma(local[17], mh[3], fma(local[16], mh[2], fma(local[13], mh[1], local[7])))))))))))))))))));
    local[8] = fma(local[54], mh[19], fma(local[53], mh[18], fma(local[52], mh[17], fma(local[51], mh[16], fma(local[48], mh[15], fma(local[47], mh[14], fma(local[46], mh[13], fma(local[43], mh[12], fma(local[42], mh[11], fma(local[39], mh[10], fma(local[33], mh[9], fma(local[32], mh[8], fma(local[31], mh[7], fma(local[28], mh[6], fma(local[27], mh[5], fma(local[24], mh[4], fma(local[18], mh[3], fma(local[17], mh[2], fma(local[14], mh[1], local[8])))))))))))))))))));
    local[9] = fma(local[39], mh[9], fma(local[38], mh[8], fma(local[37], mh[7], fma(local[36], mh[6], fma(local[35], mh[5], fma(local[34], mh[4], fma(local[21], mh[3], fma(local[20], mh[2], fma(local[19], mh[1], local[9])))))))));
    local[10] = fma(local[42], mh[9], fma(local[41], mh[8], fma(local[40], mh[7], fma(local[38], mh[6], fma(local[37], mh[5], fma(local[35], mh[4], fma(local[23], mh[3], fma(local[22], mh[2], fma(local[20], mh[1], local[10])))))))));
    local[11] = fma(local[43], mh[9], fma(local[42], mh[8], fma(local[41], mh[7], fma(local[39], mh[6], fma(local[38], mh[5], fma(local[36], mh[4], fma(local[24], mh[3], fma(local[23], mh[2], fma(local[21], mh[1], local[11])))))))));
    local[12] = fma(local[46], mh[9], fma(local[45], mh[8], fma(local[44], mh[7], fma(local[41], mh[6], fma(local[40], mh[5], fma(local[37], mh[4], fma(local[26], mh[3], fma(local[25], mh[2], fma(local[22], mh[1], local[12])))))))));
    local[13] = fma(local[47], mh[9], fma(local[46], mh[8], fma(local[45], mh[7], fma(local[42], mh[6], fma(local[41], mh[5], fma(local[38], mh[4], fma(local[27], mh[3], fma(local[26], mh[2], fma(local[23], mh[1], local[13])))))))));
    local[14] = fma(local[48], mh[9], fma(local[47], mh[8], fma(local[46], mh[7], fma(local[43], mh[6], fma(local[42], mh[5], fma(local[39], mh[4], fma(local[28], mh[3], fma(local[27], mh[2], fma(local[24], mh[1], local[14])))))))));
    local[15] = fma(local[51], mh[9], fma(local[50], mh[8], fma(local[49], mh[7], fma(local[45], mh[6], fma(local[44], mh[5], fma(local[40], mh[4], fma(local[30], mh[3], fma(local[29], mh[2], fma(local[25], mh[1], local[15])))))))));
    local[16] = fma(local[52], mh[9], fma(local[51], mh[8], fma(local[50], mh[7], fma(local[46], mh[6], fma(local[45], mh[5], fma(local[41], mh[4], fma(local[31], mh[3], fma(local[30], mh[2], fma(local[26], mh[1], local[16])))))))));
    local[17] = fma(local[53], mh[9], fma(local[52], mh[8], fma(local[51], mh[7], fma(local[47], mh[6], fma(local[46], mh[5], fma(local[42], mh[4], fma(local[32], mh[3], fma(local[31], mh[2], fma(local[27], mh[1], local[17])))))))));
    local[18] = fma(local[54], mh[9], fma(local[53], mh[8], fma(local[52], mh[7], fma(local[48], mh[6], fma(local[47], mh[5], fma(local[43], mh[4], fma(local[33], mh[3], fma(local[32], mh[2], fma(local[28], mh[1], local[18])))))))));
    local[19] = fma(local[36], mh[3], fma(local[35], mh[2], fma(local[34], mh[1], local[19])));
    local[20] = fma(local[38], mh[3], fma(local[37], mh[2], fma(local[35], mh[1], local[20])));
    local[21] = fma(local[39], mh[3], fma(local[38], mh[2], fma(local[36], mh[1], local[21])));
    local[22] = fma(local[41], mh[3], fma(local[40], mh[2], fma(local[37], mh[1], local[22])));
    local[23] = fma(local[42], mh[3], fma(local[41], mh[2], fma(local[38], mh[1], local[23])));
    local[24] = fma(local[43], mh[3], fma(local[42], mh[2], fma(local[39], mh[1], local[24])));
    local[25] = fma(local[45], mh[3], fma(local[44], mh[2], fma(local[40], mh[1], local[25])));
    local[26] = fma(local[46], mh[3], fma(local[45], mh[2], fma(local[41], mh[1], local[26])));
    local[27] = fma(local[47], mh[3], fma(local[46], mh[2], fma(local[42], mh[1], local[27])));
    local[28] = fma(local[48], mh[3], fma(local[47], mh[2], fma(local[43], mh[1], local[28])));
    local[29] = fma(local[50], mh[3], fma(local[49], mh[2], fma(local[44], mh[1], local[29])));
    local[30] = fma(local[51], mh[3], fma(local[50], mh[2], fma(local[45], mh[1], local[30])));
    local[31] = fma(local[52], mh[3], fma(local[51], mh[2], fma(local[46], mh[1], local[31])));
    local[32] = fma(local[53], mh[3], fma(local[52], mh[2], fma(local[47], mh[1], local[32])));
    local[33] = fma(local[54], mh[3], fma(local[53], mh[2], fma(local[48], mh[1], local[33])));
    local[34] = local[34];
    local[35] = local[35];
    local[36] = local[36];
    local[37] = local[37];
    local[38] = local[38];
    local[39] = local[39];
    local[40] = local[40];
    local[41] = local[41];
    local[42] = local[42];
    local[43] = local[43];
    local[44] = local[44];
    local[45] = local[45];
    local[46] = local[46];
    local[47] = local[47];
    local[48] = local[48];
    local[49] = local[49];
    local[50] = local[50];
    local[51] = local[51];
    local[52] = local[52];
    local[53] = local[53];
    local[54] = local[54];
    local[55] = fma(local[89], mh[34], fma(local[88], mh[33], fma(local[87], mh[32], fma(local[86], mh[31], fma(local[85], mh[30], fma(local[84], mh[29], fma(local[83], mh[28], fma(local[82], mh[27], fma(local[81], mh[26], fma(local[80], mh[25], fma(local[79], mh[24], fma(local[78], mh[23], fma(local[77], mh[22], fma(local[76], mh[21], fma(local[75], mh[20], fma(local[74], mh[19], fma(local[73], mh[18], fma(local[72], mh[17], fma(local[71], mh[16], fma(local[70], mh[15], fma(local[69], mh[14], fma(local[68], mh[13], fma(local[67], mh[12], fma(local[66], mh[11], fma(local[65], mh[10], fma(local[64], mh[9], fma(local[63], mh[8], fma(local[62], mh[7], fma(local[61], mh[6], fma(local[60], mh[5], fma(local[59], mh[4], fma(local[58], mh[3], fma(local[57], mh[2], fma(local[56], mh[1], local[55]))))))))))))))))))))))))))))))))));
    local[56] = fma(local[84], mh[19], fma(local[83], mh[18], fma(local[82], mh[17], fma(local[81], mh[16], fma(local[80], mh[15], fma(local[79], mh[14], fma(local[78], mh[13], fma(local[77], mh[12], fma(local[76], mh[11], fma(local[75], mh[10], fma(local[70], mh[9], fma(local[69], mh[8], fma(local[68], mh[7], fma(local[67], mh[6], fma(local[66], mh[5], fma(local[65], mh[4], fma(local[61], mh[3], fma(local[60], mh[2], fma(local[59], mh[1], local[56])))))))))))))))))));
    local[57] = fma(local[88], mh[19], fma(local[87], mh[18], fma(local[86], mh[17], fma(local[85], mh[16], fma(local[83], mh[15], fma(local[82], mh[14], fma(local[81], mh[13], fma(local[79], mh[12], fma(local[78], mh[11], fma(local[76], mh[10], fma(local[73], mh[9], fma(local[72], mh[8], fma(local[71], mh[7], fma(local[69], mh[6], fma(local[68], mh[5], fma(local[66], mh[4], fma(local[63], mh[3], fma(local[62], mh[2], fma(local[60], mh[1], local[57])))))))))))))))))));
    local[58] = fma(local[89], mh[19], fma(local[88], mh[18], fma(local[87], mh[17], fma(local[86], mh[16], fma(local[84], mh[15], fma(local[83], mh[14], fma(local[82], mh[13], fma(local[80], mh[12], fma(local[79], mh[11], fma(local[77], mh[10], fma(local[74], mh[9], fma(local[73], mh[8], fma(local[72], mh[7], fma(local[70], mh[6], fma(local[69], mh[5], fma(local[67], mh[4], fma(local[64], mh[3], fma(local[63], mh[2], fma(local[61], mh[1], local[58])))))))))))))))))));
    local[59] = fma(local[80], mh[9], fma(local[79], mh[8], fma(local[78], mh[7], fma(local[77], mh[6], fma(local[76], mh[5], fma(local[75], mh[4], fma(local[67], mh[3], fma(local[66], mh[2], fma(local[65], mh[1], local[59])))))))));
    local[60] = fma(local[83], mh[9], fma(local[82], mh[8], fma(local[81], mh[7], fma(local[79], mh[6], fma(local[78], mh[5], fma(local[76], mh[4], fma(local[69], mh[3], fma(local[68], mh[2], fma(local[66], mh[1], local[60])))))))));
    local[61] = fma(local[84], mh[9], fma(local[83], mh[8], fma(local[82], mh[7], fma(local[80], mh[6], fma(local[79], mh[5], fma(local[77], mh[4], fma(local[70], mh[3], fma(local[69], mh[2], fma(local[67], mh[1], local[61])))))))));
    local[62] = fma(local[87], mh[9], fma(local[86], mh[8], fma(local[85], mh[7], fma(local[82], mh[6], fma(local[81], mh[5], fma(local[78], mh[4], fma(local[72], mh[3], fma(local[71], mh[2], fma(local[68], mh[1], local[62])))))))));
    local[63] = fma(local[88], mh[9], fma(local[87], mh[8], fma(local[86], mh[7], fma(local[83], mh[6], fma(local[82], mh[5], fma(local[79], mh[4], fma(local[73], mh[3], fma(local[72], mh[2], fma(local[69], mh[1], local[63])))))))));
    local[64] = fma(local[89], mh[9], fma(local[88], mh[8], fma(local[87], mh[7], fma(local[84], mh[6], fma(local[83], mh[5], fma(local[80], mh[4], fma(local[74], mh[3], fma(local[73], mh[2], fma(local[70], mh[1], local[64])))))))));
    local[65] = fma(local[77], mh[3], fma(local[76], mh[2], fma(local[75], mh[1], local[65])));
    local[66] = fma(local[79], mh[3], fma(local[78], mh[2], fma(local[76], mh[1], local[66])));
    local[67] = fma(local[80], mh[3], fma(local[79], mh[2], fma(local[77], mh[1], local[67])));
    local[68] = fma(local[82], mh[3], fma(local[81], mh[2], fma(local[78], mh[1], local[68])));
    local[69] = fma(local[83], mh[3], fma(local[82], mh[2], fma(local[79], mh[1], local[69])));
    local[70] = fma(local[84], mh[3], fma(local[83], mh[2], fma(local[80], mh[1], local[70])));
    local[71] = fma(local[86], mh[3], fma(local[85], mh[2], fma(local[81], mh[1], local[71])));
    local[72] = fma(local[87], mh[3], fma(local[86], mh[2], fma(local[82], mh[1], local[72])));
    local[73] = fma(local[88], mh[3], fma(local[87], mh[2], fma(local[83], mh[1], local[73])));
    local[74] = fma(local[89], mh[3], fma(local[88], mh[2], fma(local[84], mh[1], local[74])));
    local[75] = local[75];
    local[76] = local[76];
    local[77] = local[77];
    local[78] = local[78];
    local[79] = local[79];
    local[80] = local[80];
    local[81] = local[81];
    local[82] = local[82];
    local[83] = local[83];
    local[84] = local[84];
    local[85] = local[85];
    local[86] = local[86];
    local[87] = local[87];
    local[88] = local[88];
    local[89] = local[89];
  }
  static constexpr int FLOPS_L2L = 1105;
  __device__ __forceinline__ static void l2p(const double* a, const double* local, double* f, double& phi) {
    double ma[35];
    ma[0] = 1.0;
    ma[1] = ma[0] * a[0];
    ma[2] = ma[0] * a[1];
    ma[3] = ma[0] * a[2];
    ma[4] = ma[1] * (a[0] * 0.5);
    ma[5] = ma[2] * a[0];
    ma[6] = ma[3] * a[0];
    ma[7] = ma[2] * (a[1] * 0.5);
    ma[8] = ma[3] * a[1];
    ma[9] = ma[3] * (a[2] * 0.5);
    ma[10] = ma[4] * (a[0] * 0.3333333333333333);
    ma[11] = ma[5] * (a[0] * 0.5);
    ma[12] = ma[6] * (a[0] * 0.5);
    ma[13] = ma[7] * a[0];
    ma[14] = ma[8] * a[0];
    ma[15] = ma[9] * a[0];
    ma[16] = ma[7] * (a[1] * 0.3333333333333333);
    ma[17] = ma[8] * (a[1] * 0.5);
    ma[18] = ma[9] * a[1];
    ma[19] = ma[9] * (a[2] * 0.3333333333333333);
    ma[20] = ma[10] * (a[0] * 0.25);
    ma[21] = ma[11] * (a[0] * 0.3333333333333333);
    ma[22] = ma[12] * (a[0] * 0.3333333333333333);
    ma[23] = ma[13] * (a[0] * 0.5);
    ma[24] = ma[14] * (a[0] * 0.5);
    ma[25] = ma[15] * (a[0] * 0.5);
    ma[26] = ma[16] * a[0];
    ma[27] = ma[17] * a[0];
    ma[28] = ma[18] * a[0];
    ma[29] = ma[19] * a[0];
    ma[30] = ma[16] * (a[1] * 0.25);
    ma[31] = ma[17] * (a[1] * 0.3333333333333333);
    ma[32] = ma[18] * (a[1] * 0.5);
    ma[33] = ma[19] * a[1];
    ma[34] = ma[19] * (a[2] * 0.25);
    f[0] += fma(local[48], ma[34], fma(local[47], ma[33], fma(local[46], ma[32], fma(local[45], ma[31], fma(local[44], ma[30], fma(local[43], ma[29], fma(local[42], ma[28], fma(local[41], ma[27], fma(local[40], ma[26], fma(local[39], ma[25], fma(local[38], ma[24], fma(local[37], ma[23], fma(local[36], ma[22], fma(local[35], ma[21], fma(local[34], ma[20], fma(local[28], ma[19], fma(local[27], ma[18], fma(local[26], ma[17], fma(local[25], ma[16], fma(local[24], ma[15], fma(local[23], ma[14], fma(local[22], ma[13], fma(local[21], ma[12], fma(local[20], ma[11], fma(local[19], ma[10], fma(local[14], ma[9], fma(local[13], ma[8], fma(local[12], ma[7], fma(local[11], ma[6], fma(local[10], ma[5], fma(local[9], ma[4], fma(local[5], ma[3], fma(local[4], ma[2], fma(local[3], ma[1], local[0]))))))))))))))))))))))))))))))))));
    f[1] += fma(local[53], ma[34], fma(local[52], ma[33], fma(local[51], ma[32], fma(local[50], ma[31], fma(local[49], ma[30], fma(local[47], ma[29], fma(local[46], ma[28], fma(local[45], ma[27], fma(local[44], ma[26], fma(local[42], ma[25], fma(local[41], ma[24], fma(local[40], ma[23], fma(local[38], ma[22], fma(local[37], ma[21], fma(local[35], ma[20], fma(local[32], ma[19], fma(local[31], ma[18], fma(local[30], ma[17], fma(local[29], ma[16], fma(local[27], ma[15], fma(local[26], ma[14], fma(local[25], ma[13], fma(local[23], ma[12], fma(local[22], ma[11], fma(local[20], ma[10], fma(local[17], ma[9], fma(local[16], ma[8], fma(local[15], ma[7], fma(local[13], ma[6], fma(local[12], ma[5], fma(local[10], ma[4], fma(local[7], ma[3], fma(local[6], ma[2], fma(local[4], ma[1], local[1]))))))))))))))))))))))))))))))))));
    f[2] += fma(local[54], ma[34], fma(local[53], ma[33], fma(local[52], ma[32], fma(local[51], ma[31], fma(local[50], ma[30], fma(local[48], ma[29], fma(local[47], ma[28], fma(local[46], ma[27], fma(local[45], ma[26], fma(local[43], ma[25], fma(local[42], ma[24], fma(local[41], ma[23], fma(local[39], ma[22], fma(local[38], ma[21], fma(local[36], ma[20], fma(local[33], ma[19], fma(local[32], ma[18], fma(local[31], ma[17], fma(local[30], ma[16], fma(local[28], ma[15], fma(local[27], ma[14], fma(local[26], ma[13], fma(local[24], ma[12], fma(local[23], ma[11], fma(local[21], ma[10], fma(local[18], ma[9], fma(local[17], ma[8], fma(local[16], ma[7], fma(local[14], ma[6], fma(local[13], ma[5], fma(local[11], ma[4], fma(local[8], ma[3], fma(local[7], ma[2], fma(local[5], ma[1], local[2]))))))))))))))))))))))))))))))))));
    phi += fma(local[89], ma[34], fma(local[88], ma[33], fma(local[87], ma[32], fma(local[86], ma[31], fma(local[85], ma[30], fma(local[84], ma[29], fma(local[83], ma[28], fma(local[82], ma[27], fma(local[81], ma[26], fma(local[80], ma[25], fma(local[79], ma[24], fma(local[78], ma[23], fma(local[77], ma[22], fma(local[76], ma[21], fma(local[75], ma[20], fma(local[74], ma[19], fma(local[73], ma[18], fma(local[72], ma[17], fma(local[71], ma[16], fma(local[70], ma[15], fma(local[69], ma[14], fma(local[68], ma[13], fma(local[67], ma[12], fma(local[66], ma[11], fma(local[65], ma[10], fma(local[64], ma[9], fma(local[63], ma[8], fma(local[62], ma[7], fma(local[61], ma[6], fma(local[60], ma[5], fma(local[59], ma[4], fma(local[58], ma[3], fma(local[57], ma[2], fma(local[56], ma[1], local[55]))))))))))))))))))))))))))))))))));
  }
  static constexpr int FLOPS_L2P = 329;
};
}  // namespace sfmm
