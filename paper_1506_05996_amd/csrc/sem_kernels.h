// HIP kernels of the spectral-element solver for gfx950 (wave64, LDS-staged).
// Included once, by sem_device.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "sem_internal.h"

namespace sem {

// elements per workgroup of the operator kernel: about 128 lanes per group
template <int N>
constexpr int ax_epb() {
  return (64 / ((N + 1) * (N + 1))) > 0 ? (64 / ((N + 1) * (N + 1))) : 1;
}

// Elements per workgroup of the line-phase operator kernel and of the
// restriction: as many as fill whole waves where one element leaves many of its
// lanes idle ((N + 1)^2 lanes each: N = 5 uses 36 of 64 alone, 252 of 256 by
// sevens).  Measured on 6 M local nodes, factors rebuilt, one element (two at
// N = 4) / packed: N = 4 54.8 / 49.8 us FP64, 32.7 / 29.9 FP32; N = 5 63.8 / 47.0,
// 39.7 / 29.8; N = 6 55.6 / 51.3, 32.6 / 30.5; N = 8 63.1 / 52.1, 37.3 / 30.2.
// From N = 9 the lines' LDS buffers bound the elements in flight, and wider
// workgroups only wait more at their barriers (N = 9 by threes 58.9 / 96.0, by
// fives 71.5; N = 11 by twos 76.5 / 87.3; N = 13 by twos 67.9 / 80.2).  With stored
// factors (GEO false) N = 6 stays alone: 42.9 / 46.8 us FP64 at 22^3, 26.8 / 27.8 FP32.
template <int N, bool GEO = true>
constexpr int line_epb() {
  return N == 2 ? 7 : N == 3 ? 4 : N == 4 ? 5 : N == 5 ? 7 : N == 6 ? (GEO ? 5 : 1) : N == 8 ? 3 : 1;
}

// The sum of the corrections likewise, but for N = 4: pairs 87 us, fives 90 us
// (FP32 fine preconditioner; it moves bytes, and its LDS stage limits it).
template <int N>
constexpr int sum_epb() {
  return N == 4 ? 2 : line_epb<N>();
}

__device__ __forceinline__ void unpack_coef(int32_t code, int& ai, int& aj, int& ak) {
  ai = (int32_t)((uint32_t)code << 22) >> 22;
  aj = (int32_t)((uint32_t)code << 12) >> 22;
  ak = (int32_t)((uint32_t)code << 2) >> 22;
}

__device__ __forceinline__ int node_class(int x, int N) { return x == 0 ? 0 : (x == N ? 2 : 1); }

// Constant coefficients of the model problem c u - div(kappa grad u) = s
// (eq. (pde)): the operator is kappa times the stiffness action plus c times
// the mass term.  With GLL quadrature the element mass is diagonal, m_{ijk;e}
// at each node (Section 2.4), so its assembly is the lumped mass m_N: the
// kernels add c m_N u_N where each global node's value is written.
// With one kappa_e and c_e per element (Algorithm 2), the element kernel
// applies them to its own local values instead: kappa_e r + c_e m_{ijk;e} u.
template <typename T>
struct OpCoef {
  T kap, cm;
  const T* mN;  // lumped mass [n_global]; read only when cm != 0
  int scaled;   // constant coefficients other than kappa = 1, c = 0
  const T* ke;  // per element: kappa_e [E] (NULL: constant coefficients)
  const T* ce;  // per element: c_e [E]
  const T* mL;  // per element: local mass m_{ijk;e} [E][(N+1)^3], read where c_e != 0
  const T* kn;  // per node: kappa_{ijk;e} [E][(N+1)^3], read by the kernel that rebuilds G
                // (the stored factors carry kappa already); NULL otherwise
};

template <typename T>
__device__ __forceinline__ T op_value(const OpCoef<T>& oc, T stiff, int64_t g, T ug) {
  if (!oc.scaled) return stiff;
  T v = oc.kap * stiff;
  if (oc.cm != T(0)) v += oc.cm * oc.mN[g] * ug;
  return v;
}

// A node's share of u^T A u from one element: u times the element's own value,
// so that the scalar product needs no assembled vector (u is 0 on the Dirichlet
// set, where the operator's result is masked).  With constant coefficients the
// mass term is added at assembly; the element that owns the node counts it.
// kappa multiplies v ahead of u: u is about 1 / kappa times v's final size, and their
// product alone would leave the FP64 range where the energy does not.
template <typename T>
__device__ __forceinline__ double local_energy(const OpCoef<T>& oc, T v, T u, int64_t g, bool owned) {
  if (!oc.scaled) return (double)u * (double)v;
  double d = (double)u * ((double)oc.kap * (double)v);
  if (oc.cm != T(0) && owned) d += (double)oc.cm * (double)oc.mN[g] * (double)u * (double)u;
  return d;
}

// element e's kappa_e, c_e (1, 0 without per-element coefficients), read
// once per element before its results are stored
template <typename T>
struct ElemCoef {
  T k, c;
};

template <typename T>
__device__ __forceinline__ ElemCoef<T> elem_coef(const OpCoef<T>& oc, int64_t e) {
  if (oc.ke == nullptr) return ElemCoef<T>{T(1), T(0)};
  return ElemCoef<T>{oc.ke[e], oc.ce[e]};
}

// local value of element e at local node `loc` with per-element coefficients
template <typename T>
__device__ __forceinline__ T elem_value(const OpCoef<T>& oc, const ElemCoef<T>& ec, int64_t e, int64_t nloc, int loc,
                                        T stiff, T ul) {
  if (oc.ke == nullptr) return stiff;
  T v = ec.k * stiff;
  if (ec.c != T(0)) v += ec.c * oc.mL[e * nloc + loc] * ul;
  return v;
}

// ---------------------------------------------------------------------------
// Operator kernel, eq. (R) / Algorithm 2.  One (N+1)^2-lane group per element:
// lane (i,j) keeps the k-pencil of u and of the result in registers, the
// xi/eta contractions go through one LDS plane at a time.  Global ids come
// from the element's entity records (scatter of eq. (scatter) fused into the
// load); interior results go straight to y, shared-node results to the work
// array w that the gather kernel sums.
// ---------------------------------------------------------------------------
// value a[k] of a register array for a wave-uniform runtime index k
template <typename T, int M>
__device__ __forceinline__ T pick(const T (&a)[M], int k) {
  T r = a[0];
#pragma unroll
  for (int m = 1; m < M; ++m) r = (m == k) ? a[m] : r;
  return r;
}

// Sum of v over a workgroup of NT lanes in a fixed order (deterministic):
// wave shuffles when NT is a multiple of 64, else a tree in LDS (red[NT]).
// Every lane of the workgroup must call it; lane 0 gets the result.
template <int NT>
__device__ __forceinline__ double group_sum(double v, double* red) {
  const int tid = threadIdx.x;
  if constexpr (NT % 64 == 0) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((tid & 63) == 0) red[tid >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (tid == 0)
      for (int q = 0; q < NT / 64; ++q) s += red[q];
    return s;
  } else {
    constexpr int P2 = NT >= 512 ? 512 : NT >= 256 ? 256 : NT >= 128 ? 128 : NT >= 64 ? 64 : NT >= 32 ? 32 : NT >= 16 ? 16 : 8;
    red[tid] = v;
    __syncthreads();
    if (tid < NT - P2) red[tid] += red[tid + P2];
    __syncthreads();
    for (int h = P2 / 2; h > 0; h >>= 1) {
      if (tid < h) red[tid] += red[tid + h];
      __syncthreads();
    }
    return red[0];
  }
}

// global id and work slot of lane (i, j)'s node in plane k, from the records
struct NodeAddr {
  int g, w, flags;
};

__device__ __forceinline__ NodeAddr node_addr(const int32_t* __restrict__ rec, int64_t e, int cx, int cy, int k,
                                              int i, int j, int N) {
  const int32_t* r = rec + ((e * kClasses + cx + 3 * cy + 9 * node_class(k, N)) * kRecInts);
  int ai, aj, ak;
  unpack_coef(r[1], ai, aj, ak);
  const int off = ai * i + aj * j + ak * k;
  return NodeAddr{r[0] + off, r[2] + off, r[3]};
}

// Workgroups are dealt to the 8 XCDs round-robin (workgroup b on XCD b % 8):
// give each XCD one contiguous run of the traversal order so that elements
// that share faces, edges and vertices meet in the same L2.
__device__ __forceinline__ int64_t xcd_position(int64_t b, int64_t nlogical) {
  const int64_t per = (nlogical + 7) / 8;
  return (b & 7) * per + (b >> 3);
}

inline int64_t xcd_grid(int64_t nlogical) { return ((nlogical + 7) / 8) * 8; }

// GEO = false: the factors G are read from memory (6 per node).  GEO = true:
// they are rebuilt at every node from the element's 8 vertices (the r' kernel
// of Section 5.1 and Table 3, which trades the factor stream for arithmetic): the columns of
// the Jacobian of the trilinear map, c0 = dx/dxi etc., their cross products
// a0 = c1 x c2, a1 = c2 x c0, a2 = c0 x c1 (the rows of det J . J^-1), and
// G_ab = rho_i rho_j rho_k (a_a . a_b) / det J with det J = c0 . a0, the same
// rho rho rho |J| (J^T J)^-1 as the stored factors.  In that case G points to
// the vertex coordinates [E][8][3] and tq to the GLL points and weights [2][N+1].
// KN (with GEO): kappa per node (oc.kn) scales the rebuilt factors at its node;
// the element's values are staged in LDS next to u.
// 1/d for a positive, normal d: hardware reciprocal refined by Newton steps
// (two in FP64, one in FP32): within about an ulp of the rounded quotient
__device__ __forceinline__ double recip_pos(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
  return __builtin_fma(y, __builtin_fma(-d, y, 1.0), y);
}

__device__ __forceinline__ float recip_pos(float d) {
  const float y = __builtin_amdgcn_rcpf(d);
  return __builtin_fmaf(y, __builtin_fmaf(-d, y, 1.0f), y);
}

template <int N, typename T, int EPB, bool GEO = false, bool KN = false>
__global__ void __launch_bounds__(EPB*(N + 1) * (N + 1))
__attribute__((amdgpu_waves_per_eu(N <= 9 ? (GEO && sizeof(T) == 8 ? 3 : 4) : 1, 8)))
ax_kernel(const T* __restrict__ u, T* __restrict__ y, T* __restrict__ w, const T* __restrict__ G,
          const int32_t* __restrict__ rec, const T* __restrict__ Dg, const uint8_t* __restrict__ dir,
          const int32_t* __restrict__ order, int64_t E, double* __restrict__ dpart, const T* __restrict__ tq,
          OpCoef<T> oc) {
  constexpr int n1 = N + 1, P = n1 * n1, NN = P * n1;
  __shared__ T sD[P];
  __shared__ double sRed[EPB * P];
  __shared__ T sU[EPB][NN];  // the element's gathered u, all planes
  __shared__ T sA[EPB][P];
  __shared__ T sB[EPB][P];
  __shared__ T sK[KN ? EPB : 1][KN ? NN : 1];  // KN: the element's kappa per node
  const int tid = threadIdx.x;
  const int le = tid / P, ij = tid - le * P;
  const int i = ij % n1, j = ij / n1;
  const int64_t pos = xcd_position(blockIdx.x, (E + EPB - 1) / EPB) * EPB + le;
  const bool valid = pos < E;
  const int64_t e = valid ? order[pos] : 0;
  const int cx = node_class(i, N), cy = node_class(j, N);
  // The lane's k-pencil crosses three entity records (k = 0, interior k,
  // k = N).  Loads go out in dependency order with no wait between them:
  // records, then the factors of plane 0, then all u values, then D.
  const int4* rp = reinterpret_cast<const int4*>(rec) + e * kClasses + cx + 3 * cy;
  const int4 r0 = rp[0], r1 = rp[9], r2 = rp[18];
  // factors of plane k in registers, plane k+1 prefetched during plane k
  const T* Ge = G + (GEO ? e * 24 : e * 6 * NN + ij);
  T g0 = 0, g1 = 0, g2 = 0, g3 = 0, g4 = 0, g5 = 0;
  // GEO: the lane's k-independent parts of the Jacobian columns,
  // c0 = f0(zeta) P0 + f1(zeta) P1, c1 = f0(zeta) Q0 + f1(zeta) Q1, c2 = C2
  T P0[3], P1[3], Q0[3], Q1[3], C2[3], rij = 0;
  if constexpr (GEO) {
    const T ti = tq[i], tj = tq[j];
    const T f0i = T(0.5) * (T(1) - ti), f1i = T(0.5) * (T(1) + ti);
    const T f0j = T(0.5) * (T(1) - tj), f1j = T(0.5) * (T(1) + tj);
    rij = tq[n1 + i] * tq[n1 + j];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      // x(a, b, c) = Ge[(a + 2 b + 4 c) * 3 + q]
      P0[q] = T(0.5) * ((Ge[1 * 3 + q] - Ge[0 * 3 + q]) * f0j + (Ge[3 * 3 + q] - Ge[2 * 3 + q]) * f1j);
      P1[q] = T(0.5) * ((Ge[5 * 3 + q] - Ge[4 * 3 + q]) * f0j + (Ge[7 * 3 + q] - Ge[6 * 3 + q]) * f1j);
      Q0[q] = T(0.5) * ((Ge[2 * 3 + q] - Ge[0 * 3 + q]) * f0i + (Ge[3 * 3 + q] - Ge[1 * 3 + q]) * f1i);
      Q1[q] = T(0.5) * ((Ge[6 * 3 + q] - Ge[4 * 3 + q]) * f0i + (Ge[7 * 3 + q] - Ge[5 * 3 + q]) * f1i);
      C2[q] = T(0.5) * ((Ge[4 * 3 + q] - Ge[0 * 3 + q]) * f0i * f0j + (Ge[5 * 3 + q] - Ge[1 * 3 + q]) * f1i * f0j +
                        (Ge[6 * 3 + q] - Ge[2 * 3 + q]) * f0i * f1j + (Ge[7 * 3 + q] - Ge[3 * 3 + q]) * f1i * f1j);
    }
  } else {
    g0 = Ge[0 * NN];
    g1 = Ge[1 * NN];
    g2 = Ge[2 * NN];
    g3 = Ge[3 * NN];
    g4 = Ge[4 * NN];
    g5 = Ge[5 * NN];
  }
  T rw[n1];
  T uv[n1];  // the lane's own pencil of u (GEO: also used for the zeta derivative)
  {
#pragma unroll
    for (int k = 0; k < n1; ++k) {
      const int4 r = k == 0 ? r0 : (k == N ? r2 : r1);
      int ai, aj, ak;
      unpack_coef(r.y, ai, aj, ak);
      uv[k] = u[r.x + ai * i + aj * j + ak * k];
    }
    for (int x = tid; x < P; x += EPB * P) sD[x] = Dg[x];
#pragma unroll
    for (int k = 0; k < n1; ++k) {
      sU[le][k * P + ij] = valid ? uv[k] : T(0);
      rw[k] = T(0);
    }
    if constexpr (KN) {
#pragma unroll
      for (int k = 0; k < n1; ++k) sK[le][k * P + ij] = valid ? oc.kn[e * NN + k * P + ij] : T(1);
    }
  }
  __syncthreads();
  // FP64 rebuilt-factor form: the lane's two columns of D stay in registers
  // (fewer LDS reads for the transposed contractions; the other forms keep
  // their register budget for the factor stream)
  constexpr bool kDc = GEO && sizeof(T) == 8;
  T Dci[kDc ? n1 : 1], Dcj[kDc ? n1 : 1];
  if constexpr (kDc) {
#pragma unroll
    for (int m = 0; m < n1; ++m) {
      Dci[m] = sD[m * n1 + i];
      Dcj[m] = sD[m * n1 + j];
    }
  }
#pragma unroll 1
  for (int k = 0; k < n1; ++k) {
    T h0 = 0, h1 = 0, h2 = 0, h3 = 0, h4 = 0, h5 = 0;
    if constexpr (GEO) {
      const T tk = tq[k];  // wave-uniform
      const T f0k = T(0.5) * (T(1) - tk), f1k = T(0.5) * (T(1) + tk);
      T c0[3], c1[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        c0[q] = f0k * P0[q] + f1k * P1[q];
        c1[q] = f0k * Q0[q] + f1k * Q1[q];
      }
      const T a0x = c1[1] * C2[2] - c1[2] * C2[1], a0y = c1[2] * C2[0] - c1[0] * C2[2], a0z = c1[0] * C2[1] - c1[1] * C2[0];
      const T a1x = C2[1] * c0[2] - C2[2] * c0[1], a1y = C2[2] * c0[0] - C2[0] * c0[2], a1z = C2[0] * c0[1] - C2[1] * c0[0];
      const T a2x = c0[1] * c1[2] - c0[2] * c1[1], a2y = c0[2] * c1[0] - c0[0] * c1[2], a2z = c0[0] * c1[1] - c0[1] * c1[0];
      const T det = c0[0] * a0x + c0[1] * a0y + c0[2] * a0z;
      T sc = rij * tq[n1 + k] * recip_pos(det);
      if constexpr (KN) sc *= sK[le][k * P + ij];  // kappa at the node (eq. (R))
      g0 = sc * (a0x * a0x + a0y * a0y + a0z * a0z);
      g1 = sc * (a0x * a1x + a0y * a1y + a0z * a1z);
      g2 = sc * (a0x * a2x + a0y * a2y + a0z * a2z);
      g3 = sc * (a1x * a1x + a1y * a1y + a1z * a1z);
      g4 = sc * (a1x * a2x + a1y * a2y + a1z * a2z);
      g5 = sc * (a2x * a2x + a2y * a2y + a2z * a2z);
    } else {
      const T* Gn = Ge + (k + 1 < n1 ? k + 1 : 0) * P;
      h0 = Gn[0 * NN];
      h1 = Gn[1 * NN];
      h2 = Gn[2 * NN];
      h3 = Gn[3 * NN];
      h4 = Gn[4 * NN];
      h5 = Gn[5 * NN];
    }
    const T* Dk = Dg + k * n1;  // wave-uniform: scalar loads
    const T* su = &sU[le][k * P];
    T ur = 0, us = 0, ut = 0;
#pragma unroll
    for (int m = 0; m < n1; ++m) {
      ur += sD[i * n1 + m] * su[j * n1 + m];
      us += sD[j * n1 + m] * su[m * n1 + i];
      ut += Dk[m] * (GEO ? uv[m] : sU[le][m * P + ij]);
    }
    const T A = g0 * ur + g1 * us + g2 * ut;
    const T B = g1 * ur + g3 * us + g4 * ut;
    const T C = g2 * ur + g4 * us + g5 * ut;
    sA[le][ij] = A;
    sB[le][ij] = B;
#pragma unroll
    for (int m = 0; m < n1; ++m) rw[m] += Dk[m] * C;
    __syncthreads();
    T acc = 0;
#pragma unroll
    for (int m = 0; m < n1; ++m) {
      T dmi, dmj;
      if constexpr (kDc) {
        dmi = Dci[m];
        dmj = Dcj[m];
      } else {
        dmi = sD[m * n1 + i];
        dmj = sD[m * n1 + j];
      }
      acc += dmi * sA[le][j * n1 + m] + dmj * sB[le][m * n1 + i];
    }
#pragma unroll
    for (int m = 0; m < n1; ++m) rw[m] = (m == k) ? rw[m] + acc : rw[m];
    __syncthreads();
    if constexpr (!GEO) {
      g0 = h0;
      g1 = h1;
      g2 = h2;
      g3 = h3;
      g4 = h4;
      g5 = h5;
    }
  }
  // interior results straight to y, shared ones to the work array; with dpart,
  // this workgroup's share of u^T A u, node by node: a loop of its own over the
  // kept values takes 6 to 66 more VGPRs here (N = 7 FP64 spills 29), which costs
  // waves whether or not dpart is there (factors rebuilt, loop / node by node: N = 2
  // at 48^3 34.1 / 31.6 us FP64, N = 7 at 24^3 66.0 / 60.5 FP64, N = 15 at 10^3
  // 52.0 / 44.9 FP32)
  double dacc = 0.0;
  if (valid) {
    const bool masked_interior = rec[(e * kClasses + kInteriorClass) * kRecInts + 3] & kFlagMaskedInterior;
    const ElemCoef<T> ec = elem_coef(oc, e);
#pragma unroll
    for (int k = 0; k < n1; ++k) {
      const int4 r = k == 0 ? r0 : (k == N ? r2 : r1);
      int ai, aj, ak;
      unpack_coef(r.y, ai, aj, ak);
      const int off = ai * i + aj * j + ak * k;
      const T uk = ((r.w & kFlagInterior) || oc.ke != nullptr || dpart != nullptr) ? sU[le][k * P + ij] : T(0);
      const T v = elem_value(oc, ec, e, NN, k * P + ij, rw[k], uk);
      if (r.w & kFlagInterior)
        y[r.x + off] = (masked_interior && dir[r.x + off]) ? T(0) : op_value(oc, v, r.x + off, uk);
      else
        w[r.z + off] = v;
      if (dpart != nullptr) dacc += local_energy(oc, v, uk, r.x + off, r.w & kFlagOwned);
    }
  }
  if (dpart != nullptr) {
    const double t = group_sum<EPB * P>(dacc, sRed);
    if (tid == 0) dpart[blockIdx.x] = t;
  }
}


// ---------------------------------------------------------------------------
// One 1D contraction of a line of n1 = N + 1 values by a matrix A with
// A[N-q][N-m] = -A[q][m] (the GLL derivative matrix D and D^T: the points are
// symmetric about 0).  With e_m = x_m + x_{N-m} and o_m = x_m - x_{N-m}
// (m < H = n1/2), the outputs q and N-q are E + O and O - E, E = sum_m
// Ap[q][m] e_m (+ A[q][H] x_H for odd n1), O = sum_m Am[q][m] o_m, so a line
// costs H (n1 + 1) multiply-adds instead of n1^2.  tb: rows q < H of
// [Ap[q][0..H-1], A[q][H] (odd n1), Am[q][0..H-1]], then for odd n1 the middle
// output's Am[H][0..H-1] (read with wave-uniform addresses).  ld(m) reads
// entry m of the line, st(q, v) writes output q; every read comes first, so
// the output may overwrite the line.
// Whether the line-phase operator kernel contracts its lines by output pairs:
// FP32 everywhere (N = 15 0.171 -> 0.151 ms at 20^3), FP64 at N = 4 and 5, whose
// tables fit the scalar registers, and from N = 9, with the zeta pairs below.  An
// application by rows / by pairs, FP64: N = 4 at 36^3 53.3 / 50.8 us, N = 5 at 28^3
// 43.7 / 41.3, N = 9 at 16^3 46.3 / 44.8; N = 8 at 18^3 42.0 / 42.5, and at N = 3 and 6
// the element kernel alone is no faster.  At N = 7 (with the zeta pairs) 697 us at
// 56^3 against 693 by single rows, and a heat step on 10 x 10 x 125 elements 10.70
// against 10.44 ms.
template <int N, typename T>
constexpr bool line_pairs_on() {
  return sizeof(T) == 4 || N == 4 || N == 5 || N >= 9;
}

// Whether the pencil's nodes k and N-k are processed together (the zeta
// derivative and the zeta part of D^T C by output pairs as well): from N = 10
// (N = 15 at 20^3: 0.303-0.308 -> 0.288-0.289 ms FP64, 0.150-0.154 -> 0.139 ms FP32),
// and at N = 7 and 9, whose pencils have no middle node: without / with on 6 M
// local nodes N = 7 27.0 / 26.4 us FP32; N = 9 57.4 / 55.6 FP64, 35.1 / 33.0 FP32.
// With a middle node FP64 runs out of registers (N = 6 50 / 58, N = 8 51 / 77), and
// shorter pencils gain nothing.  N = 7 FP32 with stored factors and an element's
// coefficients is slower with them (see pair_rows).
template <int N, typename T, bool GEO>
constexpr bool zeta_pairs_on() {
  return line_pairs_on<N, T>() && (N >= 10 || (N == 7 && GEO) || N == 9);
}

template <int n1>
constexpr int dsplit_size() {
  return (n1 / 2) * (2 * (n1 / 2) + n1 % 2) + (n1 % 2) * (n1 / 2);
}

// Rows of D that the line loops hold at a time.  A row comes by scalar loads, and
// a loop over single rows waits for each one.  The pairs' tables fit the scalar
// registers whole in FP32 up to N = 10 and in FP64 up to N = 5; larger ones are
// taken by two rows (all rows at N = 15: 65 us).  Row by row (the other orders in FP64) the
// forward loops hold four rows, which costs scalar registers only, and the
// transposed ones all of them where a line is short.  Element kernel on 6 M local
// nodes, factors rebuilt, one row at a time / so: FP64 N = 3 46.6 / 45.1 us, N = 6
// 52.5 / 49.3, N = 7 46.4 / 44.6, N = 11 75.8 / 72.3, N = 15 54.6 / 50.5; FP32 N = 4 30.7 / 28.9, N = 5
// 30.5 / 28.0, N = 6 31.4 / 28.4, N = 7 28.9 / 27.0, N = 8 30.9 / 29.3, N = 15 32.5 / 30.9.
// With stored factors N = 7 FP32 keeps single rows and no zeta pairs: an element's
// coefficients on 20^3 elements 30.4 us with both, 31.7 with the rows alone, 28.1 so.
constexpr int kForwardRows = 4;
constexpr int transposed_rows(int N) { return N <= 3 ? N + 1 : 1; }
template <typename T, bool GEO>
constexpr int pair_rows(int n1) {
  if (!GEO && n1 == 8) return 1;
  return n1 <= (sizeof(T) == 4 ? 11 : 6) ? (n1 + 1) / 2 : 2;
}

template <int n1, typename T, bool GEO, typename Ld, typename St>
__device__ __forceinline__ void line_pairs(const T* __restrict__ tb, Ld ld, St st) {
  constexpr int H = n1 / 2, OD = n1 % 2, RW = 2 * H + OD;
  constexpr int ROWS = pair_rows<T, GEO>(n1);
  T e[H], o[H], xm = T(0);
#pragma unroll
  for (int m = 0; m < H; ++m) {
    const T l = ld(m), r = ld(n1 - 1 - m);
    e[m] = l + r;
    o[m] = l - r;
  }
  if constexpr (OD) xm = ld(H);
#pragma unroll ROWS
  for (int q = 0; q < H; ++q) {
    const T* row = tb + q * RW;
    T E = 0, O = 0;
#pragma unroll
    for (int m = 0; m < H; ++m) E += row[m] * e[m];
    if constexpr (OD) E += row[H] * xm;
#pragma unroll
    for (int m = 0; m < H; ++m) O += row[H + OD + m] * o[m];
    st(q, E + O);
    st(n1 - 1 - q, O - E);
  }
  if constexpr (OD) {
    const T* row = tb + H * RW;
    T O = 0;
#pragma unroll
    for (int m = 0; m < H; ++m) O += row[m] * o[m];
    st(H, O);
  }
}

// ---------------------------------------------------------------------------
// Operator kernel by line phases, eq. (R) / Algorithm 2.  Each 1D contraction
// is done by lanes that own whole lines of the element, so the derivative
// matrix is wave-uniform (scalar registers) and every line is read from LDS
// once per contraction instead of once per output node:
//   eta lines    (lane (i, k)):  u_s = D u along eta          -> Z
//   xi lines     (lane (j, k)):  u_r = D u along xi, in place -> X
//   pencils      (lane (i, j)):  u_t = D u along zeta in registers; the factors
//                G (stored, or rebuilt from the vertices); A -> X, B -> Z in
//                place; the zeta part of the transposed sum D^T C in registers
//   xi, eta lines: D^T A along xi in place in X, D^T B along eta in place in Z
//   pencils:     result = zeta part + X + Z at the lane's nodes
// Two padded LDS buffers per element (line stride N + 2, plane stride
// (N + 1)(N + 2)); lanes of one element read distinct banks along all three
// directions.  Same arguments, results and epilogue as ax_kernel.
// ---------------------------------------------------------------------------
template <int N, typename T, int EPB, bool GEO = false, bool KN = false>
__global__ void __launch_bounds__(EPB*(N + 1) * (N + 1))
__attribute__((amdgpu_waves_per_eu(N <= 9 ? 4 : 1, 8)))
ax_line_kernel(const T* __restrict__ u, T* __restrict__ y, T* __restrict__ w, const T* __restrict__ G,
               const int32_t* __restrict__ rec, const T* __restrict__ Dg, const uint8_t* __restrict__ dir,
               const int32_t* __restrict__ order, int64_t E, double* __restrict__ dpart, const T* __restrict__ tq,
               OpCoef<T> oc) {
  constexpr int n1 = N + 1, P = n1 * n1, NN = P * n1;
  constexpr int LS = n1 + 1, PS = n1 * LS, BS = n1 * PS;
  constexpr int TROWS = transposed_rows(N);
  constexpr bool PAIRS = line_pairs_on<N, T>(), ZPAIRS = zeta_pairs_on<N, T, GEO>();
  __shared__ T sX[EPB][BS];
  __shared__ T sZ[EPB][BS];
  __shared__ double sRed[EPB * P];
  const int tid = threadIdx.x;
  const int le = tid / P, ij = tid - le * P;
  const int a = ij % n1, b = ij / n1;  // pencil (i, j) = (a, b); lines (., k = b)
  const int64_t pos = xcd_position(blockIdx.x, (E + EPB - 1) / EPB) * EPB + le;
  const bool valid = pos < E;
  const int64_t e = valid ? order[pos] : 0;
  const int cx = node_class(a, N), cy = node_class(b, N);
  const int4* rp = reinterpret_cast<const int4*>(rec) + e * kClasses + cx + 3 * cy;
  const int4 r0 = rp[0], r1 = rp[9], r2 = rp[18];
  const T* Ge = G + (GEO ? e * 24 : e * 6 * NN + ij);
  // Rebuilt factors: along the lane's pencil (i, j) the Jacobian columns are
  // dx/dxi = f0(t) P0 + f1(t) P1, dx/deta = f0(t) Q0 + f1(t) Q1 (f0,1 = (1 -+ t)/2)
  // and dx/dzeta = C2 (no t), so the cofactor rows a0 = dx/deta x C2 and
  // a1 = C2 x dx/dxi are linear in t and a2 = dx/dxi x dx/deta is quadratic:
  // a0 = A0 + t A1, a1 = B0 + t B1, a2 = Z0 + t (Z1 + t Z2), and
  // |J| = a2 . C2 = d0 + t (d1 + t d2).
  T A0[3], A1[3], B0[3], B1[3], Z0[3], Z1[3], Z2[3], d0 = 0, d1 = 0, d2 = 0, rij = 0;
  if constexpr (GEO) {
    const T ti = tq[a], tj = tq[b];
    const T f0i = T(0.5) * (T(1) - ti), f1i = T(0.5) * (T(1) + ti);
    const T f0j = T(0.5) * (T(1) - tj), f1j = T(0.5) * (T(1) + tj);
    rij = tq[n1 + a] * tq[n1 + b];
    T P0[3], P1[3], Q0[3], Q1[3], C2[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      P0[q] = T(0.5) * ((Ge[1 * 3 + q] - Ge[0 * 3 + q]) * f0j + (Ge[3 * 3 + q] - Ge[2 * 3 + q]) * f1j);
      P1[q] = T(0.5) * ((Ge[5 * 3 + q] - Ge[4 * 3 + q]) * f0j + (Ge[7 * 3 + q] - Ge[6 * 3 + q]) * f1j);
      Q0[q] = T(0.5) * ((Ge[2 * 3 + q] - Ge[0 * 3 + q]) * f0i + (Ge[3 * 3 + q] - Ge[1 * 3 + q]) * f1i);
      Q1[q] = T(0.5) * ((Ge[6 * 3 + q] - Ge[4 * 3 + q]) * f0i + (Ge[7 * 3 + q] - Ge[5 * 3 + q]) * f1i);
      C2[q] = T(0.5) * ((Ge[4 * 3 + q] - Ge[0 * 3 + q]) * f0i * f0j + (Ge[5 * 3 + q] - Ge[1 * 3 + q]) * f1i * f0j +
                        (Ge[6 * 3 + q] - Ge[2 * 3 + q]) * f0i * f1j + (Ge[7 * 3 + q] - Ge[3 * 3 + q]) * f1i * f1j);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int q1 = (q + 1) % 3, q2 = (q + 2) % 3;
      const T x0 = Q0[q1] * C2[q2] - Q0[q2] * C2[q1], x1 = Q1[q1] * C2[q2] - Q1[q2] * C2[q1];
      const T y0 = C2[q1] * P0[q2] - C2[q2] * P0[q1], y1 = C2[q1] * P1[q2] - C2[q2] * P1[q1];
      const T z00 = P0[q1] * Q0[q2] - P0[q2] * Q0[q1], z11 = P1[q1] * Q1[q2] - P1[q2] * Q1[q1];
      const T z01 = (P0[q1] * Q1[q2] - P0[q2] * Q1[q1]) + (P1[q1] * Q0[q2] - P1[q2] * Q0[q1]);
      A0[q] = T(0.5) * (x0 + x1);
      A1[q] = T(0.5) * (x1 - x0);
      B0[q] = T(0.5) * (y0 + y1);
      B1[q] = T(0.5) * (y1 - y0);
      Z0[q] = T(0.25) * (z00 + z01 + z11);
      Z1[q] = T(0.5) * (z11 - z00);
      Z2[q] = T(0.25) * (z00 - z01 + z11);
    }
    d0 = Z0[0] * C2[0] + Z0[1] * C2[1] + Z0[2] * C2[2];
    d1 = Z1[0] * C2[0] + Z1[1] * C2[1] + Z1[2] * C2[2];
    d2 = Z2[0] * C2[0] + Z2[1] * C2[1] + Z2[2] * C2[2];
  }
  T uv[n1];
#pragma unroll
  for (int k = 0; k < n1; ++k) {
    const int4 r = k == 0 ? r0 : (k == N ? r2 : r1);
    int ai, aj, ak;
    unpack_coef(r.y, ai, aj, ak);
    uv[k] = valid ? u[r.x + ai * a + aj * b + ak * k] : T(0);
  }
  T kv[KN ? n1 : 1];
  if constexpr (KN) {
#pragma unroll
    for (int k = 0; k < n1; ++k) kv[k] = valid ? oc.kn[e * NN + k * P + ij] : T(1);
  }
  T* X = sX[le];
  T* Z = sZ[le];
#pragma unroll
  for (int k = 0; k < n1; ++k) X[k * PS + b * LS + a] = uv[k];
  __syncthreads();
  // Line contractions: by output pairs (line_pairs, with the even/odd split of
  // D and of D^T stored after D), or row by row with the full D (the form
  // that keeps more independent accumulators; see line_pairs_on); the line
  // sits in registers.
  const T* Dsp = Dg + n1 * n1;             // D
  const T* DTsp = Dsp + dsplit_size<n1>();  // D^T
  if constexpr (PAIRS) {
    // eta lines: lane (i = a, k = b)
    line_pairs<n1, T, GEO>(Dsp, [&](int m) { return X[b * PS + m * LS + a]; },
                      [&](int q, T v) { Z[b * PS + q * LS + a] = v; });
    __syncthreads();
    // xi lines: lane (j = a, k = b), in place
    line_pairs<n1, T, GEO>(Dsp, [&](int m) { return X[b * PS + a * LS + m]; },
                      [&](int q, T v) { X[b * PS + a * LS + q] = v; });
    __syncthreads();
  } else {
    // Forward contractions loop over the output index q with row q of D in
    // scalar registers (one row live at a time).
    {  // eta lines: lane (i = a, k = b)
      T v[n1];
#pragma unroll
      for (int m = 0; m < n1; ++m) v[m] = X[b * PS + m * LS + a];
#pragma unroll kForwardRows
      for (int q = 0; q < n1; ++q) {
        const T* Dq = Dg + q * n1;
        T s = 0;
#pragma unroll
        for (int m = 0; m < n1; ++m) s += Dq[m] * v[m];
        Z[b * PS + q * LS + a] = s;
      }
    }
    __syncthreads();
    {  // xi lines: lane (j = a, k = b), in place
      T v[n1];
#pragma unroll
      for (int m = 0; m < n1; ++m) v[m] = X[b * PS + a * LS + m];
#pragma unroll kForwardRows
      for (int q = 0; q < n1; ++q) {
        const T* Dq = Dg + q * n1;
        T s = 0;
#pragma unroll
        for (int m = 0; m < n1; ++m) s += Dq[m] * v[m];
        X[b * PS + a * LS + q] = s;
      }
    }
    __syncthreads();
  }
  T rw[n1];
#pragma unroll
  for (int k = 0; k < n1; ++k) rw[k] = T(0);
  if constexpr (ZPAIRS) {
    // nodes k and N-k of the pencil together: their zeta derivatives are one
    // output pair of line_pairs on u, and the zeta part of D^T C takes
    // C_k - C_{N-k} against the even part of row k of D and C_k + C_{N-k}
    // against the odd part (rw_m = SE_m + SO_m, rw_{N-m} = SE_m - SO_m)
    constexpr int H = n1 / 2, OD = n1 % 2, RW = 2 * H + OD;
    T ue[H], uo[H], SE[H], SO[H], SM = T(0);
#pragma unroll
    for (int m = 0; m < H; ++m) {
      ue[m] = uv[m] + uv[N - m];
      uo[m] = uv[m] - uv[N - m];
      SE[m] = SO[m] = T(0);
    }
    // A and B of node k to X and Z in place; returns C
    auto node = [&](int k, T ut) -> T {
      const int o = k * PS + b * LS + a;
      const T ur = X[o], us = Z[o];
      T A, B, C;
      if constexpr (GEO) {
        const T tk = tq[k];
        const T a0x = A0[0] + tk * A1[0], a0y = A0[1] + tk * A1[1], a0z = A0[2] + tk * A1[2];
        const T a1x = B0[0] + tk * B1[0], a1y = B0[1] + tk * B1[1], a1z = B0[2] + tk * B1[2];
        const T a2x = Z0[0] + tk * (Z1[0] + tk * Z2[0]), a2y = Z0[1] + tk * (Z1[1] + tk * Z2[1]),
                a2z = Z0[2] + tk * (Z1[2] + tk * Z2[2]);
        const T det = d0 + tk * (d1 + tk * d2);
        T sc = rij * tq[n1 + k] * recip_pos(det);
        if constexpr (KN) sc *= pick(kv, k);  // kappa at the node (eq. (R))
        // G = sc M M^T (M: rows a0, a1, a2): (A, B, C) = sc M (M^T grad u)
        const T vx = ur * a0x + us * a1x + ut * a2x, vy = ur * a0y + us * a1y + ut * a2y,
                vz = ur * a0z + us * a1z + ut * a2z;
        A = sc * (a0x * vx + a0y * vy + a0z * vz);
        B = sc * (a1x * vx + a1y * vy + a1z * vz);
        C = sc * (a2x * vx + a2y * vy + a2z * vz);
      } else {
        const T* Gk = Ge + k * P;
        const T g0 = Gk[0 * NN], g1 = Gk[1 * NN], g2 = Gk[2 * NN], g3 = Gk[3 * NN], g4 = Gk[4 * NN], g5 = Gk[5 * NN];
        A = g0 * ur + g1 * us + g2 * ut;
        B = g1 * ur + g3 * us + g4 * ut;
        C = g2 * ur + g4 * us + g5 * ut;
      }
      X[o] = A;
      Z[o] = B;
      return C;
    };
#pragma unroll 1
    for (int k = 0; k < H; ++k) {
      const T* row = Dsp + k * RW;  // wave-uniform: scalar loads
      T E = 0, O = 0;
#pragma unroll
      for (int m = 0; m < H; ++m) E += row[m] * ue[m];
      if constexpr (OD) E += row[H] * uv[H];
#pragma unroll
      for (int m = 0; m < H; ++m) O += row[H + OD + m] * uo[m];
      const T C1 = node(k, E + O), C2 = node(N - k, O - E);
      const T cd = C1 - C2, cs = C1 + C2;
#pragma unroll
      for (int m = 0; m < H; ++m) {
        SE[m] += row[m] * cd;
        SO[m] += row[H + OD + m] * cs;
      }
      if constexpr (OD) SM += row[H] * cd;
    }
    if constexpr (OD) {  // the middle node (its row of D is odd)
      const T* row = Dsp + H * RW;
      T O = 0;
#pragma unroll
      for (int m = 0; m < H; ++m) O += row[m] * uo[m];
      const T C = node(H, O);
#pragma unroll
      for (int m = 0; m < H; ++m) SO[m] += row[m] * C;
      rw[H] = SM;
    }
#pragma unroll
    for (int m = 0; m < H; ++m) {
      rw[m] = SE[m] + SO[m];
      rw[N - m] = SE[m] - SO[m];
    }
  } else {
#pragma unroll 1
    for (int k = 0; k < n1; ++k) {
      const T* Dk = Dg + k * n1;  // wave-uniform: scalar loads
      const int o = k * PS + b * LS + a;
      const T ur = X[o], us = Z[o];
      T ut = 0;
#pragma unroll
      for (int m = 0; m < n1; ++m) ut += Dk[m] * uv[m];
      T A, B, C;
      if constexpr (GEO) {
        const T tk = tq[k];
        const T a0x = A0[0] + tk * A1[0], a0y = A0[1] + tk * A1[1], a0z = A0[2] + tk * A1[2];
        const T a1x = B0[0] + tk * B1[0], a1y = B0[1] + tk * B1[1], a1z = B0[2] + tk * B1[2];
        const T a2x = Z0[0] + tk * (Z1[0] + tk * Z2[0]), a2y = Z0[1] + tk * (Z1[1] + tk * Z2[1]),
                a2z = Z0[2] + tk * (Z1[2] + tk * Z2[2]);
        const T det = d0 + tk * (d1 + tk * d2);
        T sc = rij * tq[n1 + k] * recip_pos(det);
        if constexpr (KN) sc *= pick(kv, k);  // kappa at the node (eq. (R))
        // G = sc M M^T (M: rows a0, a1, a2): (A, B, C) = sc M (M^T grad u)
        const T vx = ur * a0x + us * a1x + ut * a2x, vy = ur * a0y + us * a1y + ut * a2y,
                vz = ur * a0z + us * a1z + ut * a2z;
        A = sc * (a0x * vx + a0y * vy + a0z * vz);
        B = sc * (a1x * vx + a1y * vy + a1z * vz);
        C = sc * (a2x * vx + a2y * vy + a2z * vz);
      } else {
        const T* Gk = Ge + k * P;
        const T g0 = Gk[0 * NN], g1 = Gk[1 * NN], g2 = Gk[2 * NN], g3 = Gk[3 * NN], g4 = Gk[4 * NN], g5 = Gk[5 * NN];
        A = g0 * ur + g1 * us + g2 * ut;
        B = g1 * ur + g3 * us + g4 * ut;
        C = g2 * ur + g4 * us + g5 * ut;
      }
      X[o] = A;
      Z[o] = B;
#pragma unroll
      for (int m = 0; m < n1; ++m) rw[m] += Dk[m] * C;
    }
  }
  __syncthreads();
  // transposed xi lines (lane (j = a, k = b)) and eta lines (lane (i = a, k = b)), in place
  if constexpr (PAIRS) {
    line_pairs<n1, T, GEO>(DTsp, [&](int m) { return X[b * PS + a * LS + m]; },
                      [&](int q, T v) { X[b * PS + a * LS + q] = v; });
    line_pairs<n1, T, GEO>(DTsp, [&](int m) { return Z[b * PS + m * LS + a]; },
                      [&](int q, T v) { Z[b * PS + q * LS + a] = v; });
  } else {
    // loop over the input index m: row m of D in scalar registers scales line
    // entry m into all outputs; the results overwrite the line after the loop
    T sx[n1], sz[n1];
#pragma unroll
    for (int q = 0; q < n1; ++q) sx[q] = sz[q] = T(0);
#pragma unroll TROWS
    for (int m = 0; m < n1; ++m) {
      const T* Dm = Dg + m * n1;
      const T vx = X[b * PS + a * LS + m], vz = Z[b * PS + m * LS + a];
#pragma unroll
      for (int q = 0; q < n1; ++q) {
        sx[q] += Dm[q] * vx;
        sz[q] += Dm[q] * vz;
      }
    }
#pragma unroll
    for (int q = 0; q < n1; ++q) {
      X[b * PS + a * LS + q] = sx[q];
      Z[b * PS + q * LS + a] = sz[q];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < n1; ++k) rw[k] += X[k * PS + b * LS + a] + Z[k * PS + b * LS + a];
  double dacc = 0.0;
  if (valid) {
    const bool masked_interior = rec[(e * kClasses + kInteriorClass) * kRecInts + 3] & kFlagMaskedInterior;
    const ElemCoef<T> ec = elem_coef(oc, e);
    // the pencil's records read again (cached) rather than kept live through the contractions
    int64_t ro = e * kClasses + cx + 3 * cy;
    asm volatile("" : "+v"(ro));
    const int4* rq = reinterpret_cast<const int4*>(rec) + ro;
    const int4 q0 = rq[0], q1 = rq[9], q2 = rq[18];
#pragma unroll
    for (int k = 0; k < n1; ++k) {
      const int4 r = k == 0 ? q0 : (k == N ? q2 : q1);
      int ai, aj, ak;
      unpack_coef(r.y, ai, aj, ak);
      const int off = ai * a + aj * b + ak * k;
      const T uk = uv[k];
      const T v = elem_value(oc, ec, e, NN, k * P + ij, rw[k], uk);
      if (r.w & kFlagInterior)
        y[r.x + off] = (masked_interior && dir[r.x + off]) ? T(0) : op_value(oc, v, r.x + off, uk);
      else
        w[r.z + off] = v;
      rw[k] = v;
    }
    if (dpart != nullptr) {
#pragma unroll
      for (int k = 0; k < n1; ++k) {
        const int4 r = k == 0 ? q0 : (k == N ? q2 : q1);
        int ai, aj, ak;
        unpack_coef(r.y, ai, aj, ak);
        dacc += local_energy(oc, rw[k], uv[k], r.x + ai * a + aj * b + ak * k, r.w & kFlagOwned);
      }
    }
  }
  if (dpart != nullptr) {
    const double t = group_sum<EPB * P>(dacc, sRed);
    if (tid == 0) dpart[blockIdx.x] = t;
  }
}

// ---------------------------------------------------------------------------
// Operator at N = 15 on matrix cores (v_mfma_f64_16x16x4f64 in FP64,
// v_mfma_f32_16x16x4_f32 in FP32: the same operand layout).  One
// workgroup of four waves per element (16^3 nodes).  MFMA operand layout for
// a 16x16 product with K = 4: lane l supplies A[l%16][l/16] and B[l/16][l%16]
// and receives D[4r + l/16][l%16] (FP64) or D[4(l/16) + r][l%16] (FP32) in
// accumulator register r = 0..3.
//   1. zeta derivative  UT = D (16x16) x U (16 x 256 columns (j,i)), 4 tiles per wave
//   2. per plane k (4 planes per wave): UR = U_k D^T, US = D U_k, the factors
//      G at the lane's 4 nodes, A, B, C; then W_k = A_k D + D^T B_k
//   3. zeta transpose  W += D^T (16x16) x C (16 x 256), 4 tiles per wave, and the
//      results go to y (element interiors) or the work array (shared nodes).
// D is held in registers in both operand layouts (4 + 4 values per lane).
typedef double sem_d4 __attribute__((ext_vector_type(4)));
typedef float sem_f4 __attribute__((ext_vector_type(4)));
template <typename T> struct Mfma4;
template <> struct Mfma4<double> {
  typedef sem_d4 V;
  static __device__ __forceinline__ V fma(double a, double b, V c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
};
template <> struct Mfma4<float> {
  typedef sem_f4 V;
  static __device__ __forceinline__ V fma(float a, float b, V c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
};

template <typename T>

__global__ void __launch_bounds__(256)
ax_mfma15_kernel(const T* __restrict__ u, T* __restrict__ y, T* __restrict__ w,
                 const T* __restrict__ G, const int32_t* __restrict__ rec, const T* __restrict__ Dg,
                 const uint8_t* __restrict__ dir, const int32_t* __restrict__ order, int64_t E,
                 double* __restrict__ dpart, OpCoef<T> oc) {
  typedef typename Mfma4<T>::V V;
  constexpr int N = 15, n1 = 16, P = 256, NN = 4096;
  __shared__ T sU[NN];        // u, later the xi/eta part of the result
  __shared__ T sT[NN];        // zeta derivative of u, later C
  __shared__ __attribute__((aligned(16))) T sS[4][2][P];  // per-wave A_k, B_k; at the end the reduction
  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63;
  const int lr = l & 15, lq = l >> 4;
  // row of the 16x16 result held in accumulator register r: interleaved in FP64
  // (4r + l/16), blocked in FP32 (4(l/16) + r)
  auto orow = [lq](int r) { return std::is_same<T, double>::value ? 4 * r + lq : 4 * lq + r; };
  const int64_t pos = xcd_position(blockIdx.x, E);
  if (pos >= E) {  // whole workgroup
    if (dpart != nullptr && tid == 0) dpart[blockIdx.x] = 0.0;
    return;
  }
  const int64_t e = order[pos];
  // gather: lane tid owns the k-pencil of node (i, j) = (tid % 16, tid / 16)
  {
    const int i0 = tid & 15, j0 = tid >> 4;
    const int cx = node_class(i0, N), cy = node_class(j0, N);
    const int4* rp = reinterpret_cast<const int4*>(rec) + e * kClasses + cx + 3 * cy;
    const int4 r0 = rp[0], r1 = rp[9], r2 = rp[18];
    T uv[n1];
#pragma unroll
    for (int k = 0; k < n1; ++k) {
      const int4 r = k == 0 ? r0 : (k == N ? r2 : r1);
      int ai, aj, ak;
      unpack_coef(r.y, ai, aj, ak);
      uv[k] = u[r.x + ai * i0 + aj * j0 + ak * k];
    }
#pragma unroll
    for (int k = 0; k < n1; ++k) sU[k * P + tid] = uv[k];
  }
  T DA[4], DB[4];  // DA[s] = D[lr][4s+lq] (A layout of D), DB[s] = D[4s+lq][lr] (B layout)
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    DA[s] = Dg[lr * n1 + 4 * s + lq];
    DB[s] = Dg[(4 * s + lq) * n1 + lr];
  }
  __syncthreads();
  // 1. UT[k'][col] = sum_k D[k'][k] U[k][col]
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int t = wave * 4 + q;
    V acc = {0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = Mfma4<T>::fma(DA[s], sU[(4 * s + lq) * P + t * 16 + lr], acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) sT[orow(r) * P + t * 16 + lr] = acc[r];
  }
  __syncthreads();
  // 2. planes
  const T* Ge = G + e * 6 * NN;
  V W[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int k = wave * 4 + q;
    const T* Uk = sU + k * P;
    V ur = {0, 0, 0, 0}, us = {0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      ur = Mfma4<T>::fma(Uk[lr * n1 + 4 * s + lq], DA[s], ur);  // U_k D^T
      us = Mfma4<T>::fma(DA[s], Uk[(4 * s + lq) * n1 + lr], us);  // D U_k
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int node = k * P + orow(r) * n1 + lr;
      const T ut = sT[node];
      const T g0 = Ge[0 * NN + node], g1 = Ge[1 * NN + node], g2 = Ge[2 * NN + node];
      const T g3 = Ge[3 * NN + node], g4 = Ge[4 * NN + node], g5 = Ge[5 * NN + node];
      const T A = g0 * ur[r] + g1 * us[r] + g2 * ut;
      const T B = g1 * ur[r] + g3 * us[r] + g4 * ut;
      const T C = g2 * ur[r] + g4 * us[r] + g5 * ut;
      sS[wave][0][orow(r) * n1 + lr] = A;
      sS[wave][1][orow(r) * n1 + lr] = B;
      sT[node] = C;  // plane k of the zeta derivative is no longer needed
    }
    __syncthreads();
    V wk = {0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      wk = Mfma4<T>::fma(sS[wave][0][lr * n1 + 4 * s + lq], DB[s], wk);  // A_k D
      wk = Mfma4<T>::fma(DB[s], sS[wave][1][(4 * s + lq) * n1 + lr], wk);  // D^T B_k
    }
    W[q] = wk;
    __syncthreads();
  }
  // xi/eta part of the result into sU (u is no longer read)
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) sU[(wave * 4 + q) * P + orow(r) * n1 + lr] = W[q][r];
  __syncthreads();
  // 3. zeta transpose and output: tile t = row j of every plane
  const bool masked_interior = rec[(e * kClasses + kInteriorClass) * kRecInts + 3] & kFlagMaskedInterior;
  const ElemCoef<T> ec = elem_coef(oc, e);
  double dacc = 0.0;  // share of u^T A u, with dpart
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int t = wave * 4 + q;
    V acc = {0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = Mfma4<T>::fma(DB[s], sT[(4 * s + lq) * P + t * 16 + lr], acc);
    const int j = t, i = lr, cx = node_class(i, N), cy = node_class(j, N);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int k = orow(r);
      const NodeAddr a = node_addr(rec, e, cx, cy, k, i, j, N);
      const T ug = (dpart != nullptr || oc.scaled || oc.ke != nullptr) ? u[a.g] : T(0);
      const T v = elem_value(oc, ec, e, NN, k * P + j * n1 + i, acc[r] + sU[k * P + j * n1 + i], ug);
      if (a.flags & kFlagInterior)
        y[a.g] = (masked_interior && dir[a.g]) ? T(0) : op_value(oc, v, a.g, ug);
      else
        w[a.w] = v;
      if (dpart != nullptr) dacc += local_energy(oc, v, ug, a.g, a.flags & kFlagOwned);
    }
  }
  if (dpart != nullptr) {
    __syncthreads();  // sS is reused for the reduction (FP64: 2 x 80 KB fills the CU's LDS exactly)
    const double tsum = group_sum<256>(dacc, reinterpret_cast<double*>(&sS[0][0][0]));
    if (tid == 0) dpart[blockIdx.x] = tsum;
  }
}

// ---------------------------------------------------------------------------
// Gather of the shared nodes (eq. (gather)): one lane per shared global node,
// copies summed in ascending element order.
// ---------------------------------------------------------------------------
struct SharedNodes {
  const int32_t *vinc_off, *einc_off;
  const uint8_t *fcount, *dir;
  int64_t V, base_f, base_i;  // vertices, first face node, first interior node
  int m;                      // N - 1
  int64_t wedge_off, wvert_off;
};

template <typename T>
__device__ __forceinline__ T shared_sum(const T* __restrict__ w, const SharedNodes& sn, int64_t g) {
  T s = 0;
  if (g >= sn.base_f) {  // face node (most shared nodes): both slots read, the second kept on interior faces
    const uint32_t mm = (uint32_t)sn.m * (uint32_t)sn.m, q = (uint32_t)(g - sn.base_f), f = q / mm, r = q - f * mm;
    const T s0 = w[2 * (int64_t)f * mm + r], s1 = w[(2 * (int64_t)f + 1) * mm + r];
    s = sn.fcount[f] == 2 ? s0 + s1 : s0;
  } else if (g < sn.V) {
    for (int32_t q = sn.vinc_off[g]; q < sn.vinc_off[g + 1]; ++q) s += w[sn.wvert_off + q];
  } else {
    const uint32_t q = (uint32_t)(g - sn.V), ed = q / (uint32_t)sn.m, r = q - ed * (uint32_t)sn.m;
    for (int32_t x = sn.einc_off[ed]; x < sn.einc_off[ed + 1]; ++x) s += w[sn.wedge_off + (int64_t)x * sn.m + r];
  }
  return s;
}

// Dirichlet nodes zeroed.  As the operator's last step (oc.scaled) it also
// applies kappa and the mass term at the shared nodes of u; as the
// preconditioner's assembly it only sums.
template <typename T>
__global__ void __launch_bounds__(256)
gs_kernel(T* __restrict__ y, const T* __restrict__ w, SharedNodes sn, OpCoef<T> oc, const T* __restrict__ u) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= sn.base_i) return;
  const uint8_t dg = sn.dir[g];  // issued with the slots' loads
  const T s = shared_sum(w, sn, g);
  y[g] = dg ? T(0) : op_value(oc, s, g, oc.scaled ? u[g] : T(0));
}

// PCG's last step at the shared nodes: z gathered from the work array, then
// x += alpha p and p = z + beta p (schwarz_sum_kernel does the interiors), so
// that z is never stored.  start: p = z alone.
template <typename T>
__global__ void __launch_bounds__(256)
gs_px_kernel(T* __restrict__ x, T* __restrict__ p, const T* __restrict__ w, SharedNodes sn,
             const double* __restrict__ sc, int start) {
  if (sc[6] != 0.0 || !isfinite(sc[3])) return;  // whole grid: schwarz_sum_kernel did nothing either
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= sn.base_i) return;
  const T al = (T)sc[2], beta = (T)sc[3];
  const uint8_t dg = sn.dir[g];
  T pg = 0, xg = 0;
  if (!start) {
    pg = p[g];
    xg = x[g];
  }
  const T s = shared_sum(w, sn, g);
  const T z = dg ? T(0) : s;
  if (start) {
    p[g] = z;
  } else {
    x[g] = xg + al * pg;
    p[g] = z + beta * pg;
  }
}

// a step of PCG breaks down on p^T A p <= 0 or an alpha that is not finite, or on
// the beta before it (0 at the first step), which made no new p
__device__ __forceinline__ bool step_breaks(double pAp, double alpha, const double* __restrict__ sc) {
  return !(pAp > 0.0) || !isfinite(alpha) || !isfinite(sc[3]);
}

// sum of n partial sums by every workgroup of a consuming kernel (one wave or
// more, any size): the same order, so the same value, in each
template <int NT>
__device__ __forceinline__ double all_partials(const double* __restrict__ part, int n, double* red) {
  constexpr int W = (NT + 63) / 64;
  double s = 0.0;
  for (int q = threadIdx.x; q < n; q += NT) s += part[q];
  // lanes past the workgroup's end count as zero
  for (int o = 32; o > 0; o >>= 1) {
    const double t = __shfl_xor(s, o);
    s += ((int)(threadIdx.x ^ o) < NT) ? t : 0.0;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  double t = 0.0;
#pragma unroll
  for (int q = 0; q < W; ++q) t += red[q];
  __syncthreads();
  return t;
}

// PCG's r -= alpha A p at the shared nodes: A p gathered from the work array
// (with the coefficients, as gs_kernel; u = p), not stored.  alpha comes from
// sc[2], or, with na > 0, from the na partial sums of p . A p (every workgroup
// sums them; block 0 also stores the scalars, and the breakdown flag, which this
// kernel does not read).
template <typename T>
__global__ void __launch_bounds__(256)
gs_r_kernel(T* __restrict__ r, const T* __restrict__ w, SharedNodes sn, OpCoef<T> oc, const T* __restrict__ u,
            double* __restrict__ sc, int rz, const double* __restrict__ apart, int na) {
  __shared__ double sRed[256 / 64];
  T al;
  if (na > 0) {
    const double t = all_partials<256>(apart, na, sRed), a = sc[rz] / t;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      sc[1] = t;
      sc[2] = a;
      if (step_breaks(t, a, sc)) sc[6] = 1.0;
    }
    al = (T)a;
  } else {
    al = (T)sc[2];
  }
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= sn.base_i) return;
  const uint8_t dg = sn.dir[g];
  const T rg = r[g];
  const T s = shared_sum(w, sn, g);
  const T Ap = dg ? T(0) : op_value(oc, s, g, oc.scaled ? u[g] : T(0));
  r[g] = rg - al * Ap;
}

// ---------------------------------------------------------------------------
// Fine patch solve, eq. (z), one workgroup per subdomain.  The (N+3)^3 patch
// is gathered through I^p into LDS; each of the six 1D contractions is done
// by lanes that own a whole pencil in registers (one LDS read and one write
// per node and pass); the diagonal scaling 1/(kappa 4 (lambda_a/h_x^2 +
// lambda_b/h_y^2 + lambda_c/h_z^2) + c) is fused into the zeta pass.  The
// correction at the element's own nodes goes to zc; the slots outside the
// element go to the consumer layout of the element that holds them (zx).
// ---------------------------------------------------------------------------
// Patches per workgroup: each patch has m^2 pencils (m = N + 3), one per
// lane in each pass; several patches share a workgroup so that the lanes in use
// come close to a multiple of 64 (N = 7: 5 x 100 of 512), within ~64 KB of LDS
// in FP64.
template <int N>
constexpr int fdm_ppb() {
  return N == 2 ? 5 : N == 3 ? 7 : N == 4 ? 5 : N == 6 ? 3 : N == 7 ? 5 : N == 9 ? 3 : N == 10 ? 3 : N == 11 ? 2 : 1;
}

template <int N>
constexpr int fdm_threads() {
  return ((fdm_ppb<N>() * (N + 3) * (N + 3) + 63) / 64) * 64;
}

// One 1D pass of the fast diagonalisation on a lane's pencil.  The extended
// pencil is symmetric under a -> m-1-a, so every column of S is even or odd:
// with ho = m/2 pairs (a, m-1-a) and he = m - ho even columns, the pencil's
// transform takes the pair sums x_a + x_{m-1-a} against the even columns and
// the differences against the odd ones (about half the products of a full
// m x m pass).  Transformed coefficients sit in the order (even columns
// ascending, odd columns ascending).  Sp holds, for a < ho, row a as
// S[a][even j] (j < he) then S[a][odd j] (j < ho), and for odd m the middle
// row S[ho][even j]; rows are read with wave-uniform addresses (scalar loads
// feeding the FMAs) in a rolled loop, so S is not hoisted into registers.
//   pencil_St: out = S^T x     (x in LDS, stride apart)
//   pencil_S:  y = S v          (y in LDS)
template <int m, typename T>
__device__ __forceinline__ void pencil_St(const T* __restrict__ Sp, const T* x, int stride, T (&out)[m]) {
  constexpr int ho = m / 2, he = m - ho;
#pragma unroll
  for (int b = 0; b < m; ++b) out[b] = T(0);
#pragma unroll 1
  for (int a = 0; a < ho; ++a) {
    const T xl = x[a * stride], xr = x[(m - 1 - a) * stride];
    const T ps = xl + xr, ms = xl - xr;
    const T* sr = Sp + a * m;
#pragma unroll
    for (int j = 0; j < he; ++j) out[j] += sr[j] * ps;
#pragma unroll
    for (int j = 0; j < ho; ++j) out[he + j] += sr[he + j] * ms;
  }
  if constexpr (m % 2 == 1) {
    const T xc = x[ho * stride];
    const T* sr = Sp + ho * m;
#pragma unroll
    for (int j = 0; j < he; ++j) out[j] += sr[j] * xc;
  }
}

template <int m, typename T>
__device__ __forceinline__ void pencil_S(const T* __restrict__ Sp, const T (&v)[m], T* y, int stride) {
  constexpr int ho = m / 2, he = m - ho;
#pragma unroll 1
  for (int a = 0; a < ho; ++a) {
    const T* sr = Sp + a * m;
    T ev = T(0), od = T(0);
#pragma unroll
    for (int j = 0; j < he; ++j) ev += sr[j] * v[j];
#pragma unroll
    for (int j = 0; j < ho; ++j) od += sr[he + j] * v[he + j];
    y[a * stride] = ev + od;
    y[(m - 1 - a) * stride] = ev - od;
  }
  if constexpr (m % 2 == 1) {
    const T* sr = Sp + ho * m;
    T ev = T(0);
#pragma unroll
    for (int j = 0; j < he; ++j) ev += sr[j] * v[j];
    y[ho * stride] = ev;
  }
}

// The patch's node ids and consumer slots as records rather than tables with an
// entry per slot: along each axis a patch index is below, on, inside, on or past
// the element (patch_class 0..4), and within one of the 125 classes of (a, b, c) the
// global id is affine (pidx [E][125]: base, packed strides, kPatchNull); the
// outside slots' destinations are affine on each of the 26 faces, edges and corners
// (pdst [E][26]).  Set-up derives both from the tables and checks every slot.  At
// N = 7 a patch then reads 1.2 KB of indices instead of 6.0 KB, in the same two
// dependent loads, and the index arithmetic of 64 slots is mostly a wave's and not
// its lanes'.  Fine preconditioner, tables / records: N = 5 126 / 103 us on 6 M local
// nodes FP64, N = 6 118 / 93, N = 8 91 / 83, N = 15 95 / 88.  Below N = 5 a plane
// fills less than half a wave and the records are no smaller than the tables (N = 4
// FP32 90 / 96, N = 3 126 / 137, N = 2 55 / 84): those orders keep the tables.
template <int N>
constexpr bool patch_records_on() {
  return N >= kPatchRecordsFrom;
}

__device__ __host__ constexpr int patch_class(int a, int N) {
  return a <= 1 ? a : (a <= N ? 2 : (a == N + 1 ? 3 : 4));
}

template <int N, typename T>
__global__ void __launch_bounds__(fdm_threads<N>()) __attribute__((amdgpu_waves_per_eu(N <= 8 ? 8 : 4, 8)))
fdm_kernel(const T* __restrict__ r, T* __restrict__ zc, T* __restrict__ zx, const int32_t* __restrict__ pidx,
           const int32_t* __restrict__ pdst, const T* __restrict__ S,
           const T* __restrict__ lam, const T* __restrict__ hg, const int32_t* __restrict__ order, int64_t E,
           T kap, T cm, const T* __restrict__ ke, const T* __restrict__ ce, double* __restrict__ epart) {
  constexpr bool REC = patch_records_on<N>();
  constexpr int m = N + 3, MM = m * m, MMM = MM * m, PPB = fdm_ppb<N>(), NT = fdm_threads<N>();
  constexpr int NN = (N + 1) * (N + 1) * (N + 1), R = (PPB * MMM + NT - 1) / NT;
  __shared__ T X[PPB * MMM];
  __shared__ T sL[m];
  __shared__ int sE[PPB];  // element of each patch slot, -1 past the end
  __shared__ double sRed[NT / 64];
  const int tid = threadIdx.x;
  const int64_t pos0 = xcd_position(blockIdx.x, (E + PPB - 1) / PPB) * PPB;
  if (pos0 >= E) {  // whole workgroup
    if (epart != nullptr && tid == 0) epart[blockIdx.x] = 0.0;
    return;
  }
  if (tid < PPB) sE[tid] = pos0 + tid < E ? order[pos0 + tid] : -1;
  if (tid < m) sL[tid] = lam[tid];
  __syncthreads();
  if constexpr (REC) {
    // lane (a, b) of a patch owns the column (a, b, 0..m-1): five records, one
    // per class of c, then all residual loads, then the LDS stores
    const int lq = tid / MM, ab = tid - lq * MM, a = ab % m, b = ab / m;
    const int64_t e = tid < PPB * MM ? sE[lq] : -1;
    if (e >= 0) {
      const int2* rp = reinterpret_cast<const int2*>(pidx) + e * 125 + patch_class(a, N) + 5 * patch_class(b, N);
      int2 rc[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) rc[q] = rp[25 * q];
      int32_t g[5], ak[5];
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        int ai, aj;
        unpack_coef(rc[q].y, ai, aj, ak[q]);
        g[q] = rc[q].x + ai * a + aj * b;
      }
      T rv[m];
#pragma unroll
      for (int c = 0; c < m; ++c) {
        const int q = patch_class(c, N);
        rv[c] = r[rc[q].y & kPatchNull ? 0 : g[q] + ak[q] * c];
      }
#pragma unroll
      for (int c = 0; c < m; ++c) X[lq * MMM + c * MM + ab] = rc[patch_class(c, N)].y & kPatchNull ? T(0) : rv[c];
    } else if (tid < PPB * MM) {
#pragma unroll
      for (int c = 0; c < m; ++c) X[lq * MMM + c * MM + ab] = T(0);
    }
  } else {
    // all index loads, then all residual loads, then the LDS stores
    int32_t gi[R];
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int x = tid + q * NT, lp = min(x / MMM, PPB - 1);
      const int64_t e = x < PPB * MMM ? sE[lp] : -1;
      gi[q] = e >= 0 ? pidx[e * MMM + (x - lp * MMM)] : -1;
    }
    T rv[R];
#pragma unroll
    for (int q = 0; q < R; ++q) rv[q] = r[gi[q] >= 0 ? gi[q] : 0];
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (tid + q * NT < PPB * MMM) X[tid + q * NT] = gi[q] >= 0 ? rv[q] : T(0);
  }
  __syncthreads();
  const bool act = tid < PPB * MM;
  const int lp = act ? tid / MM : 0, pl = tid - lp * MM;
  const int p0 = pl % m, p1 = pl / m;
  const int64_t e = act && sE[lp] >= 0 ? sE[lp] : 0;  // slots past the end run on zeros
  T* Xp = X + lp * MMM;
  T v[m], o[m];
  // pass 1: xi, S^T   (lane owns row (b = p0, c = p1))
  if (act) {
    T* row = Xp + p1 * MM + p0 * m;
    pencil_St<m, T>(S, row, 1, o);
#pragma unroll
    for (int a = 0; a < m; ++a) row[a] = o[a];
  }
  __syncthreads();
  // pass 2: eta, S^T  (lane owns column (a = p0, c = p1))
  if (act) {
    T* col = Xp + p1 * MM + p0;
    pencil_St<m, T>(S, col, m, o);
#pragma unroll
    for (int b = 0; b < m; ++b) col[b * m] = o[b];
  }
  __syncthreads();
  // pass 3: zeta, S^T, diagonal, S  (lane owns pencil (a = p0, b = p1)).  The volume
  // factor 8/(hx hy hz) is divided into kappa and c here, so that with epart, the
  // workgroup's share of r . z, y = S^T r the transformed residual gives
  // r_s . z_s = sum y^2 / diagonal from what is in registers, each product as large
  // as a node's share of r . z (y^2 over the diagonal without the factor left the
  // FP64 range where r . z does not).  Fine preconditioner at 40^3, N = 7, factor applied
  // to z at the end / so: 572 / 563 us FP64, 371 / 353 us FP32.
  double en = 0.0;
  if (act) {
    const T hx = hg[e * 3 + 0], hy = hg[e * 3 + 1], hz = hg[e * 3 + 2], vol = hx * hy * hz;
    const T ihx2 = T(0.5) / (hx * hx), ihy2 = T(0.5) / (hy * hy), ihz2 = T(0.5) / (hz * hz);  // 4 / h^2 over 8
    T kp = kap, c0 = cm;
    if (ke != nullptr) {  // the subdomain's own element's coefficients
      kp = ke[e];
      c0 = ce[e];
    }
    kp *= vol;
    c0 *= T(0.125) * vol;
    T* pen = Xp + p1 * m + p0;
    const T dab = sL[p0] * ihx2 + sL[p1] * ihy2;
    pencil_St<m, T>(S, pen, MM, o);
#pragma unroll
    for (int c = 0; c < m; ++c) {
      const T yc = o[c];
      o[c] = yc * recip_pos(kp * (dab + sL[c] * ihz2) + c0);
      if (epart != nullptr) en += (double)yc * (double)o[c];
    }
    pencil_S<m, T>(S, o, pen, MM);
  }
  if (epart != nullptr) {
    for (int q = 32; q > 0; q >>= 1) en += __shfl_xor(en, q);
    if ((tid & 63) == 0) sRed[tid >> 6] = en;
  }
  __syncthreads();
  if (epart != nullptr && tid == 0) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < NT / 64; ++q) t += sRed[q];
    epart[blockIdx.x] = t;
  }
  // pass 4: eta, S
  if (act) {
    T* col = Xp + p1 * MM + p0;
#pragma unroll
    for (int b = 0; b < m; ++b) v[b] = col[b * m];
    pencil_S<m, T>(S, v, col, m);
  }
  __syncthreads();
  // pass 5: xi, S
  if (act) {
    T* row = Xp + p1 * MM + p0 * m;
#pragma unroll
    for (int a = 0; a < m; ++a) v[a] = row[a];
    pencil_S<m, T>(S, v, row, 1);
  }
  __syncthreads();
  // Results out, driven by the destination: the element's own nodes to zc in
  // element-local order, the slots outside the element in their ordinal order
  // (grouped by entity: 6 face planes of (N+1)^2, the lower of the other two axes
  // fastest; 12 edge lines of N+1, edge 4 axis + side_lo + 2 side_hi; 8 corners),
  // so that a wave's stores land in one neighbour's consumer block.  NULL slots are
  // dropped.
  if constexpr (REC) {
    // A wave takes 64 nodes of one plane at a time (a layer k of the own nodes, or a
    // face of the outside slots), so that the patch, the plane and its record are
    // uniform and a lane only adds its in-plane offset; then the edges' and corners'
    // slots, a lane each.
    constexpr int n1 = N + 1, P1 = n1 * n1, CH = (P1 + 63) / 64, W = NT / 64, NE = 12 * n1 + 8;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int2* prec = reinterpret_cast<const int2*>(pdst);
    for (int t = wave; t < PPB * n1 * CH; t += W) {
      const int lq = t / (n1 * CH), k = t / CH - lq * n1, ij = (t % CH) * 64 + lane;
      const int eq = __builtin_amdgcn_readfirstlane(sE[lq]);
      if (eq < 0 || (P1 % 64 != 0 && ij >= P1)) continue;
      zc[(int64_t)eq * NN + k * P1 + ij] = X[lq * MMM + (ij % n1 + 1) + m * (ij / n1 + 1) + MM * (k + 1)];
    }
    for (int t = wave; t < PPB * 6 * CH; t += W) {
      const int lq = t / (6 * CH), f = t / CH - lq * 6, uv = (t % CH) * 64 + lane;
      const int eq = __builtin_amdgcn_readfirstlane(sE[lq]);
      if (eq < 0) continue;
      const int2 d = prec[(int64_t)eq * 26 + f];
      if (d.y & kPatchNull) continue;
      int su, sv, sw;
      unpack_coef(d.y, su, sv, sw);
      const int ax = f >> 1, s0 = (f & 1) ? m - 1 : 0;
      const int lu = ax == 0 ? m : 1, lv = ax == 2 ? m : MM, l0 = s0 * (ax == 0 ? 1 : (ax == 1 ? m : MM));
      if (P1 % 64 != 0 && uv >= P1) continue;
      const int u = uv % n1, v = uv / n1;
      zx[d.x + su * u + sv * v] = X[lq * MMM + l0 + lu * (u + 1) + lv * (v + 1)];
    }
    for (int x = tid; x < PPB * NE; x += NT) {
      const int lq = x / NE, o = x - lq * NE;
      const int eq = sE[lq];
      if (eq < 0) continue;
      const int g = o / n1, u = o < 12 * n1 ? o - g * n1 : 0, id = o < 12 * n1 ? g : o - 12 * n1;
      const int2 d = prec[(int64_t)eq * 26 + 6 + (o < 12 * n1 ? id : 12 + id)];
      if (d.y & kPatchNull) continue;
      int su, sv, sw;
      unpack_coef(d.y, su, sv, sw);
      int off;
      if (o < 12 * n1) {  // edge 4 axis + side_lo + 2 side_hi
        const int ax = id >> 2, slo = (id & 1) ? m - 1 : 0, shi = (id & 2) ? m - 1 : 0;
        off = ax == 0 ? 1 + u + m * slo + MM * shi : (ax == 1 ? slo + m * (1 + u) + MM * shi : slo + m * shi + MM * (1 + u));
      } else {
        off = ((id & 1) ? m - 1 : 0) + ((id & 2) ? m * (m - 1) : 0) + ((id & 4) ? MM * (m - 1) : 0);
      }
      zx[d.x + su * u] = X[lq * MMM + off];
    }
  } else {
    // a lane per slot, with a table entry each
    constexpr int n1 = N + 1, P1 = n1 * n1, NX = MMM - NN;
    // the lane's slots are recomputed here rather than kept live (in
    // registers) from the gather through the five passes
    int ts = tid;
    asm volatile("" : "+v"(ts));
    constexpr int RC = (PPB * NN + NT - 1) / NT, RO = (PPB * NX + NT - 1) / NT;
#pragma unroll
    for (int q = 0; q < RC; ++q) {
      const int x = ts + q * NT;
      if (x >= PPB * NN) break;
      const int lq = x / NN, t = x - lq * NN;
      const int i = t % n1, j = (t / n1) % n1, k = t / P1;
      const int64_t eq = sE[lq];
      if (eq >= 0) zc[eq * NN + t] = X[lq * MMM + (i + 1) + m * (j + 1) + MM * (k + 1)];
    }
    int32_t dq[RO];
#pragma unroll
    for (int q = 0; q < RO; ++q) {
      const int x = ts + q * NT, lq = min(x / NX, PPB - 1);
      dq[q] = (x < PPB * NX && sE[lq] >= 0) ? pdst[(int64_t)sE[lq] * NX + (x - lq * NX)] : -1;
    }
#pragma unroll
    for (int q = 0; q < RO; ++q) {
      if (dq[q] < 0) continue;
      const int x = ts + q * NT, lq = x / NX, o = x - lq * NX;
      int ca, cb, cc;  // slot coordinates (a, b, c)
      if (o < 6 * P1) {
        const int f = o / P1, t = o - f * P1, d = f >> 1, s = (f & 1) ? m - 1 : 0;
        const int u = 1 + t % n1, v = 1 + t / n1;
        ca = d == 0 ? s : u;
        cb = d == 1 ? s : (d == 0 ? u : v);
        cc = d == 2 ? s : v;
      } else if (o < 6 * P1 + 12 * n1) {
        const int y = o - 6 * P1, id = y / n1, ax = id >> 2, t = 1 + y % n1;
        const int slo = (id & 1) ? m - 1 : 0, shi = (id & 2) ? m - 1 : 0;
        ca = ax == 0 ? t : slo;
        cb = ax == 1 ? t : (ax == 0 ? slo : shi);
        cc = ax == 2 ? t : shi;
      } else {
        const int id = o - 6 * P1 - 12 * n1;
        ca = (id & 1) ? m - 1 : 0;
        cb = (id & 2) ? m - 1 : 0;
        cc = (id & 4) ? m - 1 : 0;
      }
      zx[dq[q]] = X[lq * MMM + ca + m * cb + MM * cc];
    }
  }
}

// ---------------------------------------------------------------------------
// Sum of the patch corrections and the coarse interpolation, element by element
// (the preconditioner's result before assembly).  Lane (i, j) of element e
// walks its k-pencil: the patch of e itself (zc) plus the corrections that the
// neighbouring patches left in e's consumer layout (zx: planes one layer in
// from each face, lines one layer in from both faces of each edge, corner
// points), then I Z at the nodes e owns.  Shared nodes go to the work array for
// the gather; element interiors (Dirichlet zeroed)
//   kSumZ:     straight to z;
//   kSumStart: to p (the first search direction);
//   kSumPx:    into PCG's updates x += alpha p, p = z + beta p, so that z is
//              never stored: beta is known before this kernel, since r . z is
//              the patch solves' and the coarse solve's energies.  beta comes
//              from sc[3], or, with nb > 0, from the nb partial sums themselves
//              (every workgroup sums them; block 0 also stores the scalars).
//              The breakdown flag is read here, so it is not raised here: waves of
//              one workgroup would see it at different times and part before the
//              barriers.  A beta that is not finite stays in sc[3], where gs_px_kernel
//              sees it, and the next step's alpha raises the flag.
// ---------------------------------------------------------------------------
enum : int { kSumZ = 0, kSumStart = 1, kSumPx = 2 };

template <int N, typename T, int EPB, int MODE>
__global__ void __launch_bounds__(EPB*(N + 1) * (N + 1))
schwarz_sum_kernel(T* __restrict__ z, T* __restrict__ x, T* __restrict__ w, const T* __restrict__ zc,
                   const T* __restrict__ zx, const int32_t* __restrict__ rec, const uint8_t* __restrict__ dir,
                   const int32_t* __restrict__ order, int64_t E, int use_fine, const double* __restrict__ Zv,
                   const double* __restrict__ phi, double* __restrict__ sc, int rz_in, int rz_out,
                   const double* __restrict__ bpart, int nb) {
  constexpr int n1 = N + 1, P = n1 * n1, NN = P * n1;
  constexpr int NX = (N + 3) * (N + 3) * (N + 3) - NN;
  constexpr int F0 = 0, E0 = 6 * P, C0 = 6 * P + 12 * n1;
  constexpr int RX = (NX + P - 1) / P;
  __shared__ T sX[EPB][NX];  // the element's consumer layout, staged with coalesced loads
  __shared__ double sPhi[2 * n1];
  __shared__ double sRed[(EPB * P + 63) / 64];
  const int tid = threadIdx.x;
  const int le = tid / P, ij = tid - le * P;
  const int i = ij % n1, j = ij / n1;
  T al = 0, beta = 0;
  if constexpr (MODE == kSumPx) {
    if (sc[6] != 0.0) return;  // whole grid
    if (nb > 0) {
      const double t = all_partials<EPB * P>(bpart, nb, sRed);
      const double bd = t / sc[rz_in];
      if (blockIdx.x == 0 && tid == 0) {
        sc[3] = bd;
        sc[rz_out] = t;
      }
      if (!isfinite(bd)) return;  // every workgroup alike
      beta = (T)bd;
    } else {
      beta = (T)sc[3];
    }
    al = (T)sc[2];
  }
  const int64_t pos = xcd_position(blockIdx.x, (E + EPB - 1) / EPB) * EPB + le;
  const bool valid = pos < E;
  const int64_t e = valid ? order[pos] : 0;
  const int cx = node_class(i, N), cy = node_class(j, N);
  const int4* rp = reinterpret_cast<const int4*>(rec) + e * kClasses + cx + 3 * cy;
  const int4 r0 = rp[0], r1 = rp[9], r2 = rp[18];
  const bool masked_interior = rec[(e * kClasses + kInteriorClass) * kRecInts + 3] & kFlagMaskedInterior;
  T cv[n1];
  if (use_fine) {
    const T* ze = zc + e * NN;
    const T* xe = zx + e * NX;
    T xv[RX];
#pragma unroll
    for (int q = 0; q < RX; ++q) xv[q] = (ij + q * P < NX) ? xe[ij + q * P] : T(0);
#pragma unroll
    for (int k = 0; k < n1; ++k) cv[k] = ze[ij + P * k];
#pragma unroll
    for (int q = 0; q < RX; ++q)
      if (ij + q * P < NX) sX[le][ij + q * P] = xv[q];
  }
  // kSumPx: p and x at the lane's interior nodes (1 <= k < N), loaded ahead of
  // the sum so that the loop's loads do not wait one by one
  T pk[n1], xk[n1];
  if (MODE == kSumPx && valid && (r1.w & kFlagInterior)) {
    int ai, aj, ak;
    unpack_coef(r1.y, ai, aj, ak);
    const int base = r1.x + ai * i + aj * j;
#pragma unroll
    for (int k = 1; k < N; ++k) {
      pk[k] = z[base + ak * k];
      xk[k] = x[base + ak * k];
    }
  }
  double zv[8];
  if (Zv != nullptr) {
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int cls = 2 * (c & 1) + 6 * ((c >> 1) & 1) + 18 * (c >> 2);
      zv[c] = Zv[rec[(e * kClasses + cls) * kRecInts]];
    }
    for (int x = tid; x < 2 * n1; x += EPB * P) sPhi[x] = phi[x];
  }
  __syncthreads();
  // I Z at (i, j, k) = Phi_0(t_k) zk0 + Phi_1(t_k) zk1, with zk0 / zk1 the
  // bilinear interpolation in (i, j) of the vertex values on the faces k = 0 / N
  double zk0 = 0.0, zk1 = 0.0;
  if (Zv != nullptr) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double wij = sPhi[(c & 1) * n1 + i] * sPhi[(c >> 1) * n1 + j];
      zk0 += wij * zv[c];
      zk1 += wij * zv[c + 4];
    }
  }
  const T* xs = sX[le];
  const bool li0 = i == 1, li1 = i == N - 1, lj0 = j == 1, lj1 = j == N - 1;
#pragma unroll
  for (int k = 0; k < n1; ++k) {
    if (!valid) break;
    const bool lk0 = k == 1, lk1 = k == N - 1;
    T v = 0;
    if (use_fine) {
      v = cv[k];
      if (li0) v += xs[F0 + 0 * P + j + n1 * k];
      if (li1) v += xs[F0 + 1 * P + j + n1 * k];
      if (lj0) v += xs[F0 + 2 * P + i + n1 * k];
      if (lj1) v += xs[F0 + 3 * P + i + n1 * k];
      if (lk0) v += xs[F0 + 4 * P + i + n1 * j];
      if (lk1) v += xs[F0 + 5 * P + i + n1 * j];
      // edge lines along x (sides of y, z), along y (sides of x, z), along z (sides of x, y)
      if (lj0 && lk0) v += xs[E0 + (0 + 0 + 0) * n1 + i];
      if (lj1 && lk0) v += xs[E0 + (0 + 1 + 0) * n1 + i];
      if (lj0 && lk1) v += xs[E0 + (0 + 0 + 2) * n1 + i];
      if (lj1 && lk1) v += xs[E0 + (0 + 1 + 2) * n1 + i];
      if (li0 && lk0) v += xs[E0 + (4 + 0 + 0) * n1 + j];
      if (li1 && lk0) v += xs[E0 + (4 + 1 + 0) * n1 + j];
      if (li0 && lk1) v += xs[E0 + (4 + 0 + 2) * n1 + j];
      if (li1 && lk1) v += xs[E0 + (4 + 1 + 2) * n1 + j];
      if (li0 && lj0) v += xs[E0 + (8 + 0 + 0) * n1 + k];
      if (li1 && lj0) v += xs[E0 + (8 + 1 + 0) * n1 + k];
      if (li0 && lj1) v += xs[E0 + (8 + 0 + 2) * n1 + k];
      if (li1 && lj1) v += xs[E0 + (8 + 1 + 2) * n1 + k];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const bool si = (c & 1) ? li1 : li0, sj = ((c >> 1) & 1) ? lj1 : lj0, sk = (c >> 2) ? lk1 : lk0;
        if (si && sj && sk) v += xs[C0 + c];
      }
    }
    const int4 rr = k == 0 ? r0 : (k == N ? r2 : r1);
    if (Zv != nullptr && (rr.w & kFlagOwned)) v += (T)(sPhi[k] * zk0 + sPhi[n1 + k] * zk1);
    int ai, aj, ak;
    unpack_coef(rr.y, ai, aj, ak);
    const int off = ai * i + aj * j + ak * k;
    if (rr.w & kFlagInterior) {
      const T zk = (masked_interior && dir[rr.x + off]) ? T(0) : v;
      if constexpr (MODE == kSumPx) {
        if (k > 0 && k < N) {  // always, at an interior node
          x[rr.x + off] = xk[k] + al * pk[k];
          z[rr.x + off] = zk + beta * pk[k];
        }
      } else {
        z[rr.x + off] = zk;
      }
    } else {
      w[rr.z + off] = v;
    }
  }
}

// Coarse restriction, per element: R_e[IJK] = sum over the nodes this element
// owns of Phi_I(t_i) Phi_J(t_j) Phi_K(t_k) r_N  (= (I^T r) once gathered).  The
// eight parts go, negated, to the coarse rows' own entries of the contribution
// vector (part_dst; -1: Dirichlet vertex), where the forward sweep sums them.
// UPDATE: PCG's r -= alpha A p, second half (gs_r_kernel has done the shared
// nodes): first the interiors of each element, A p from y; and over the nodes that
// the element owns (each global node once) the workgroup's share of r . r
// (rpart[block], 0 for the padding blocks); cvec may be NULL.  (All in one kernel,
// the owner summing the copies of its shared nodes, measured 69 against 40 us at
// 24^3, N = 7: 140 VGPRs and a serial tail at edges and vertices.)
template <int N, typename T, int EPB, bool UPDATE>
__global__ void __launch_bounds__(EPB*(N + 1) * (N + 1))
restrict_kernel(T* __restrict__ r, const T* __restrict__ y, const double* __restrict__ sc, double* __restrict__ cvec,
                const int32_t* __restrict__ part_dst, double* __restrict__ rpart, const int32_t* __restrict__ rec,
                const double* __restrict__ phi, const int32_t* __restrict__ order, int64_t E) {
  constexpr int n1 = N + 1, P = n1 * n1;
  constexpr int NV = UPDATE ? 9 : 8;  // eight parts, and r . r
  __shared__ double red[EPB][NV][P + 1];  // padded rows: the summing lanes read distinct banks
  __shared__ double sPhi[2 * n1];
  const int tid = threadIdx.x;
  const int le = tid / P, ij = tid - le * P;
  const int i = ij % n1, j = ij / n1;
  const int64_t pos = xcd_position(blockIdx.x, (E + EPB - 1) / EPB) * EPB + le;
  const bool valid = pos < E;
  const int64_t e = valid ? order[pos] : 0;
  for (int x = tid; x < 2 * n1; x += EPB * P) sPhi[x] = phi[x];
  const int cx = node_class(i, N), cy = node_class(j, N);
  const int4* rp = reinterpret_cast<const int4*>(rec) + e * kClasses + cx + 3 * cy;
  const int4 r0 = rp[0], r1 = rp[9], r2 = rp[18];
  const T al = UPDATE ? (T)sc[2] : T(0);
  const bool in = r1.w & kFlagInterior;  // the lane's nodes 1 <= k < N
  T rv[n1], wv[n1];
  int32_t gk[n1];  // global node ids fit in 32 bits; -1: not owned
#pragma unroll
  for (int k = 0; k < n1; ++k) {
    const int4 rr = k == 0 ? r0 : (k == N ? r2 : r1);
    int ai, aj, ak;
    unpack_coef(rr.y, ai, aj, ak);
    const bool own = valid && (rr.w & kFlagOwned);
    gk[k] = own ? rr.x + ai * i + aj * j + ak * k : -1;
    rv[k] = own ? r[gk[k]] : T(0);
    wv[k] = UPDATE && own && in && k > 0 && k < N ? y[gk[k]] : T(0);
  }
  __syncthreads();
  // the lane's share of corner c: Phi_ci(t_i) Phi_cj(t_j) sum_k Phi_ck(t_k) r_k
  double sk0 = 0.0, sk1 = 0.0, rsq = 0.0;
#pragma unroll
  for (int k = 0; k < n1; ++k) {
    if (gk[k] < 0) continue;
    T rn = rv[k];
    if (UPDATE) {
      rn -= al * wv[k];
      if (in && k > 0 && k < N) r[gk[k]] = rn;
    }
    const double v = (double)rn;
    rsq += v * v;
    sk0 += sPhi[k] * v;
    sk1 += sPhi[n1 + k] * v;
  }
#pragma unroll
  for (int c = 0; c < 8; ++c)
    red[le][c][ij] = sPhi[(c & 1) * n1 + i] * sPhi[((c >> 1) & 1) * n1 + j] * ((c >> 2) ? sk1 : sk0);
  if constexpr (UPDATE) red[le][8][ij] = rsq;
  __syncthreads();
  for (int q = tid; q < NV * EPB; q += EPB * P) {
    const int l = q / NV, c = q - NV * l;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int x = 0;
    for (; x + 3 < P; x += 4) {
      s0 += red[l][c][x];
      s1 += red[l][c][x + 1];
      s2 += red[l][c][x + 2];
      s3 += red[l][c][x + 3];
    }
    for (; x < P; ++x) s0 += red[l][c][x];
    const double t = (s0 + s1) + (s2 + s3);
    if (c == 8) {
      if constexpr (EPB == 1)
        rpart[blockIdx.x] = t;
      else
        red[l][NV - 1][P] = t;
    } else if (cvec != nullptr && pos - le + l < E) {
      const int32_t d = part_dst[(int64_t)order[pos - le + l] * 8 + c];
      if (d >= 0) cvec[d] = -t;
    }
  }
  if constexpr (UPDATE && EPB > 1) {
    __syncthreads();
    if (tid == 0) {
      double t = 0.0;
#pragma unroll
      for (int l = 0; l < EPB; ++l) t += red[l][NV - 1][P];
      rpart[blockIdx.x] = t;
    }
  }
}

// Nested-dissection solve of the coarse system, node by node in height order.
//   forward, height h (leaves first), node t with own rows I and boundary B:
//     y_I = R_I - (the children's contributions to I)
//     Z_I = S_t^-1 y_I,   c_t = W_t y_t + (the children's contributions to B)
//   backward, height h (roots first):
//     X_I = Z_I - W_t^T X_B
// c_t goes to the parent's rows, so a row sums one entry per child and not one
// per descendant.  All rows are independent within a height; sums run in a
// fixed order.
//
// One launch per height and direction; a workgroup takes 4 RW rows of one node
// (wave w: rows row + w RW ..), each lane two consecutive columns at a time.
// What bounds a launch of a small or middling mesh is latency, not bytes: the
// matrix loads of a chunk are issued before the node's vector is assembled, so
// that both are in flight together; the vector (the rows' entries forward, the
// ancestors' solution backward) passes through LDS in chunks of kCoarseStage.
// NARROW (rows of at most 128 entries): one load per row and lane.
constexpr int kCoarseStage = 1024;

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// sums of the entries of the U row slots g[u] (negative: none) of the
// contribution vector, each in order; all rows' loads go out together, W
// entries of each at a time
template <int U, int W>
__device__ __forceinline__ void row_entries(const double* __restrict__ cvec, const int32_t* __restrict__ rs_off,
                                            const int (&g)[U], double (&sum)[U]) {
  int32_t q0[U], n[U], most = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int gu = max(g[u], 0);
    q0[u] = rs_off[gu];
    n[u] = rs_off[gu + 1];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    n[u] = g[u] >= 0 ? n[u] - q0[u] : 0;
    most = max(most, n[u]);
    sum[u] = 0.0;
  }
  for (int32_t q = 0; q < most; q += W) {
    double v[U][W];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < W; ++i) v[u][i] = cvec[q0[u] + max(min(q + i, n[u] - 1), 0)];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < W; ++i) sum[u] += q + i < n[u] ? v[u][i] : 0.0;
  }
}

// sums over the wave of RW values per lane in a fixed tree: the rows are dealt
// to parts of the wave while lanes are added, so that lanes l with
// l % (64 / RW) == 0 end with the sum of row l / (64 / RW)
template <int RW>
__device__ __forceinline__ double wave_rows_sum(double (&a)[RW]) {
  const int lane = threadIdx.x & 63;
  if constexpr (RW == 1) {
    return wave_sum(a[0]);
  } else {
    const bool hi = (lane & 32) != 0;
    double v[RW / 2];
#pragma unroll
    for (int i = 0; i < RW / 2; ++i) {
      const double keep = hi ? a[i + RW / 2] : a[i], give = hi ? a[i] : a[i + RW / 2];
      v[i] = keep + __shfl_xor(give, 32);
    }
    if constexpr (RW == 2) {
      double s = v[0];
      for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o);
      return s;
    } else {
      const bool hi2 = (lane & 16) != 0;
      double w[RW / 4];
#pragma unroll
      for (int i = 0; i < RW / 4; ++i) {
        const double keep = hi2 ? v[i + RW / 4] : v[i], give = hi2 ? v[i] : v[i + RW / 4];
        w[i] = keep + __shfl_xor(give, 16);
      }
      if constexpr (RW == 4) {
        double s = w[0];
        for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o);
        return s;
      } else {
        const bool hi3 = (lane & 8) != 0;
        double s = (hi3 ? w[1] : w[0]) + __shfl_xor(hi3 ? w[0] : w[1], 8);
        for (int o = 4; o > 0; o >>= 1) s += __shfl_xor(s, o);
        return s;
      }
    }
  }
}

// the wave's RW dot products (rows r0 .. of the tile's matrix) against the
// node's vector, entries c + 256 u given by vec(c, end, v[U]); partial sums per lane in acc
template <int RW, bool NARROW, typename Vec>
__device__ __forceinline__ void coarse_tile_dots(const CoarseTile& t, const double* __restrict__ pool, int r0,
                                                 double* sv, double (&acc)[RW], Vec vec) {
  constexpr int NJ = NARROW ? 1 : 4;  // 16-byte loads per row and lane ahead of the vector
  const int lane = threadIdx.x & 63;
  const double* rp[RW];
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    rp[i] = pool + t.mat + (int64_t)min(r0 + i, t.rows - 1) * t.ld;  // rows past the node: read, not stored
    acc[i] = 0.0;
  }
  for (int c0 = 0; c0 < t.len; c0 += kCoarseStage) {
    const int cn = min(kCoarseStage, t.len - c0);
    double2 mv[RW][NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int c = 2 * lane + 128 * j;
#pragma unroll
      for (int i = 0; i < RW; ++i)
        mv[i][j] = c < cn ? *reinterpret_cast<const double2*>(rp[i] + c0 + c) : make_double2(0.0, 0.0);
    }
    if (c0 > 0) __syncthreads();  // the previous chunk is consumed
    {  // entries past the end are 0 (the padding of an odd row meets one)
      double v[NJ];
      vec(c0 + (int)threadIdx.x, c0 + cn, v);
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        if (!NARROW || threadIdx.x < 128) sv[threadIdx.x + 256 * j] = v[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int c = 2 * lane + 128 * j;
      if (c < cn) {
        const double2 v = *reinterpret_cast<const double2*>(sv + c);
#pragma unroll
        for (int i = 0; i < RW; ++i) acc[i] += mv[i][j].x * v.x + mv[i][j].y * v.y;
      }
    }
    if constexpr (!NARROW) {
#pragma unroll 2
      for (int c = 2 * lane + 128 * NJ; c < cn; c += 128) {
        const double2 v = *reinterpret_cast<const double2*>(sv + c);
#pragma unroll
        for (int i = 0; i < RW; ++i) {
          const double2 m = *reinterpret_cast<const double2*>(rp[i] + c0 + c);
          acc[i] += m.x * v.x + m.y * v.y;
        }
      }
    }
  }
}

// forward: rows of [S^-1; W]; rows < s give Z (in X; final, with the vertex
// values, where the node has no boundary), the others the node's contribution.
// The lowest launch has further workgroups (from n_tiles on) that sum the
// element parts of the rows of all higher nodes into those rows' first
// entries, so that the tiles above, each of which assembles its whole node,
// read one entry instead of eight.  With epart, each tile also leaves its share
// of R . Z, which by the block factorisation is the sum of y_t . S_t^-1 y_t.
template <int RW, bool NARROW>
__global__ void __launch_bounds__(256)
coarse_fwd_kernel(double* __restrict__ X, double* __restrict__ Zv, double* __restrict__ cvec,
                  const double* __restrict__ pool, const CoarseTile* __restrict__ tiles,
                  const int32_t* __restrict__ rs_off, const int32_t* __restrict__ cdst,
                  const int32_t* __restrict__ cvert, int n_tiles, const int32_t* __restrict__ pre_slot,
                  const int32_t* __restrict__ pre_row, int n_pre, double* __restrict__ epart) {
  __shared__ __attribute__((aligned(16))) double sv[NARROW ? 128 : kCoarseStage];
  if ((int)blockIdx.x >= n_tiles) {
    const int x = ((int)blockIdx.x - n_tiles) * 256 + (int)threadIdx.x;
    if (x >= n_pre) return;
    const int g[1] = {pre_slot[x]};
    double v[1];
    row_entries<1, 8>(cvec, rs_off, g, v);
    cvec[rs_off[pre_row[x]]] = v[0];
    return;
  }
  const CoarseTile t = tiles[blockIdx.x];
  const int lane = threadIdx.x & 63, r0 = t.row + (threadIdx.x >> 6) * RW;
  // the row whose sum this lane ends with (wave_rows_sum): its own entries and
  // where its result goes, loaded ahead of the products
  const int r = r0 + lane / (64 / RW);
  const bool mine = lane % (64 / RW) == 0 && r < t.rows;
  double c[1] = {0.0};
  int32_t dst = 0;
  if (mine) {
    const int g[1] = {t.src + r};
    if (r >= t.s || epart != nullptr) row_entries<1, 8>(cvec, rs_off, g, c);
    if (r >= t.s)
      dst = cdst[t.coff + r - t.s];
    else if (t.root)
      dst = cvert[t.off + r];
  }
  double acc[RW];
  coarse_tile_dots<RW, NARROW>(t, pool, r0, sv, acc, [&](int c, int end, auto& v) {
    constexpr int U = NARROW ? 1 : 4;
    int g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) g[u] = c + 256 * u < end ? t.src + c + 256 * u : -1;
    row_entries<U, NARROW ? 8 : 4>(cvec, rs_off, g, v);
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = -v[u];
  });
  const double v = wave_rows_sum<RW>(acc);
  double en = 0.0;
  if (mine) {
    if (r < t.s) {
      X[t.off + r] = v;
      if (t.root) Zv[dst] = v;
      en = -c[0] * v;
    } else {
      cvec[dst] = v + c[0];
    }
  }
  if (epart != nullptr) {
    __shared__ double sp[4];
    en = wave_sum(en);
    if (lane == 0) sp[threadIdx.x >> 6] = en;
    __syncthreads();
    if (threadIdx.x == 0) epart[blockIdx.x] = ((sp[0] + sp[1]) + sp[2]) + sp[3];
  }
}

// backward: rows of W^T, one per own vertex c of a node: X_c = Z_c - (W^T)_c . X_B
// (X_B final from the ancestors' launches), also to the vertex values
template <int RW, bool NARROW>
__global__ void __launch_bounds__(256)
coarse_bwd_kernel(double* __restrict__ X, double* __restrict__ Zv, const double* __restrict__ pool,
                  const CoarseTile* __restrict__ tiles, const int32_t* __restrict__ fb_idx,
                  const int32_t* __restrict__ cvert) {
  __shared__ __attribute__((aligned(16))) double sv[NARROW ? 128 : kCoarseStage];
  const CoarseTile t = tiles[blockIdx.x];
  const int lane = threadIdx.x & 63, r0 = t.row + (threadIdx.x >> 6) * RW;
  const int r = r0 + lane / (64 / RW);  // the row whose sum this lane ends with
  const bool mine = lane % (64 / RW) == 0 && r < t.rows;
  double z = 0.0;
  int32_t dst = 0;
  if (mine) {
    z = X[t.off + r];
    dst = cvert[t.off + r];
  }
  double acc[RW];
  coarse_tile_dots<RW, NARROW>(t, pool, r0, sv, acc, [&](int c, int end, auto& v) {
    constexpr int U = NARROW ? 1 : 4;
    int32_t x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = fb_idx[t.src + min(c + 256 * u, end - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = X[x[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = c + 256 * u < end ? v[u] : 0.0;
  });
  const double v = wave_rows_sum<RW>(acc);
  if (mine) {
    X[t.off + r] = z - v;
    Zv[dst] = z - v;
  }
}

// ---------------------------------------------------------------------------
// Aggregation AMG with a K-cycle on the coarse system (Section 4.1, "Algebraic
// multigrid"): CSR matrices per level (columns ascending), damped Jacobi with
// wd = omega / a_ii, restriction by aggregate sums (members ascending),
// prolongation by injection.  All scalars of the flexible-CG steps stay on the
// device, so a whole cycle can be captured in a graph.
// ---------------------------------------------------------------------------
// Jacobi sweep from zero and its residual in one pass: x = wd .* b,
// r = b - A x (x at the neighbours formed on the fly)
__global__ void __launch_bounds__(256)
amg_presmooth_kernel(double* __restrict__ x, double* __restrict__ r, const double* __restrict__ b,
                     const double* __restrict__ wd, const int32_t* __restrict__ off, const int32_t* __restrict__ col,
                     const double* __restrict__ val, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double acc = 0.0;
  for (int32_t q = off[i]; q < off[i + 1]; ++q) {
    const int32_t j = col[q];
    acc += val[q] * (wd[j] * b[j]);
  }
  x[i] = wd[i] * b[i];
  r[i] = b[i] - acc;
}

// w = A v
__global__ void __launch_bounds__(256)
amg_spmv_kernel(double* __restrict__ w, const double* __restrict__ v, const int32_t* __restrict__ off,
                const int32_t* __restrict__ col, const double* __restrict__ val, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double acc = 0.0;
  for (int32_t q = off[i]; q < off[i + 1]; ++q) acc += val[q] * v[col[q]];
  w[i] = acc;
}

// B[a] = sum of r over the members of aggregate a
__global__ void __launch_bounds__(256)
amg_restrict_kernel(double* __restrict__ B, const double* __restrict__ r, const int32_t* __restrict__ moff,
                    const int32_t* __restrict__ mem, int64_t nc) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= nc) return;
  double acc = 0.0;
  for (int32_t q = moff[a]; q < moff[a + 1]; ++q) acc += r[mem[q]];
  B[a] = acc;
}

// t = x + X[agg]  (coarse correction by injection)
__global__ void __launch_bounds__(256)
amg_prolong_kernel(double* __restrict__ t, const double* __restrict__ x, const double* __restrict__ X,
                   const int32_t* __restrict__ agg, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) t[i] = x[i] + X[agg[i]];
}

// x = t + wd .* (b - A t)  (Jacobi sweep after the coarse correction)
__global__ void __launch_bounds__(256)
amg_post_kernel(double* __restrict__ x, const double* __restrict__ t, const double* __restrict__ b,
                const int32_t* __restrict__ off, const int32_t* __restrict__ col, const double* __restrict__ val,
                const double* __restrict__ wd, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double acc = 0.0;
  for (int32_t q = off[i]; q < off[i + 1]; ++q) acc += val[q] * t[col[q]];
  x[i] = t[i] + wd[i] * (b[i] - acc);
}

// sc[idx + k] = a . b_k over n entries for the K vectors b_0..b_{K-1} (K <= 3),
// one workgroup, fixed summation order
template <int K>
__global__ void __launch_bounds__(1024)
amg_dots_kernel(double* __restrict__ sc, int idx, const double* __restrict__ a, const double* __restrict__ b0,
                const double* __restrict__ b1, const double* __restrict__ b2, int64_t n) {
  __shared__ double red[1024 / 64];
  double acc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 1024) {
    const double ai = a[i];
    acc[0] += ai * b0[i];
    if constexpr (K > 1) acc[1] += ai * b1[i];
    if constexpr (K > 2) acc[2] += ai * b2[i];
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const double t = group_sum<1024>(acc[k], red);
    if (threadIdx.x == 0) sc[idx + k] = t;
    __syncthreads();  // red is reused by the next sum
  }
}

// r2 = b - (rho / a1) w   with sc = {rho, a1, ...}
__global__ void __launch_bounds__(256)
amg_r2_kernel(double* __restrict__ r2, const double* __restrict__ b, const double* __restrict__ w,
              const double* __restrict__ sc, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) r2[i] = b[i] - (sc[0] / sc[1]) * w[i];
}

// two flexible-CG steps combined: x = (rho/a1) v + (a2/den) (v2 - (g/a1) v),
// den = be - g^2/a1, with sc = {rho, a1, g, be, a2}
__global__ void __launch_bounds__(256)
amg_combine_kernel(double* __restrict__ x, const double* __restrict__ v, const double* __restrict__ v2,
                   const double* __restrict__ sc, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double rho = sc[0], a1 = sc[1], g = sc[2], be = sc[3], a2 = sc[4];
  const double den = be - g * g / a1;
  x[i] = (rho / a1) * v[i] + (a2 / den) * (v2[i] - (g / a1) * v[i]);
}

// x = Ainv b, dense row-major n x n; one wave per row
__global__ void __launch_bounds__(256)
amg_gemv_kernel(double* __restrict__ x, const double* __restrict__ Ainv, const double* __restrict__ b, int64_t n) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= n) return;  // whole wave
  double acc = 0.0;
  for (int64_t k = lane; k < n; k += 64) acc += Ainv[row * n + k] * b[k];
  acc = wave_sum(acc);
  if (lane == 0) x[row] = acc;
}

// level-0 right-hand side: the element parts of the coarse residual at each
// free vertex (the first entries of its part slot, negated there)
__global__ void __launch_bounds__(256)
amg_in_kernel(double* __restrict__ B0, const double* __restrict__ cvec, const int32_t* __restrict__ rs_off,
              const int32_t* __restrict__ pslot, const int32_t* __restrict__ cvert,
              const int32_t* __restrict__ vinc_off, const int32_t* __restrict__ nd_of, int64_t n) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n) return;
  const int32_t c = nd_of[x], v = cvert[c], q0 = rs_off[pslot[c]];
  double s = 0.0;
  for (int32_t q = 0; q < vinc_off[v + 1] - vinc_off[v]; ++q) s += cvec[q0 + q];
  B0[x] = -s;
}

// vertex-indexed result (0 on Dirichlet vertices) from the level-0 solution;
// with epart, each workgroup's share of R . Z (B0: the level-0 right-hand side)
__global__ void __launch_bounds__(256)
amg_out_kernel(double* __restrict__ Zv, const double* __restrict__ X0, const double* __restrict__ B0,
               const int32_t* __restrict__ cidx, const int32_t* __restrict__ pos, int64_t V,
               double* __restrict__ epart) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double en = 0.0;
  if (v < V) {
    const int32_t c = cidx[v];
    const double z = c >= 0 ? X0[pos[c]] : 0.0;
    Zv[v] = z;
    if (epart != nullptr && c >= 0) en = B0[pos[c]] * z;
  }
  if (epart != nullptr) {
    __shared__ double red[256 / 64];
    const double t = group_sum<256>(en, red);
    if (threadIdx.x == 0) epart[blockIdx.x] = t;
  }
}

// a given coarse residual (vertex order) in place of the element parts: the
// whole value as the first element's part, zeros as the others'
__global__ void __launch_bounds__(256)
coarse_set_rhs_kernel(double* __restrict__ cvec, const double* __restrict__ Rv, const int32_t* __restrict__ rs_off,
                      const int32_t* __restrict__ pslot, const int32_t* __restrict__ cvert,
                      const int32_t* __restrict__ vinc_off, int64_t nc) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= nc) return;
  const int32_t v = cvert[c], q0 = rs_off[pslot[c]];
  for (int32_t q = 0; q < vinc_off[v + 1] - vinc_off[v]; ++q) cvec[q0 + q] = q == 0 ? -Rv[v] : 0.0;
}

// --- set-up of the coarse fronts (column-major f x f front F, leading dimension f)
// copy the lower triangle of the leading n x n block to the upper one
__global__ void symmetrize_kernel(double* __restrict__ A, int64_t n, int64_t ld) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= n * n) return;
  const int64_t r = x % n, c = x / n;
  if (r < c) A[r + c * ld] = A[c + r * ld];
}

// entries of A_c into the zeroed front
__global__ void front_scatter_kernel(double* __restrict__ F, const int32_t* __restrict__ pos,
                                     const double* __restrict__ val, int64_t n) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x < n) F[pos[x]] = val[x];
}

// F_IB = F_BI^T: F[c, s + k] = F[s + k, c] for c < s, k < b
__global__ void front_transpose_kernel(double* __restrict__ F, int64_t f, int64_t s, int64_t b) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= s * b) return;
  const int64_t c = x % s, k = x / s;
  F[c + (s + k) * f] = F[(s + k) + c * f];
}

// extend-add of a child's update matrix U (b x b, leading dimension b) into F
__global__ void front_extend_add_kernel(double* __restrict__ F, int64_t f, const double* __restrict__ U, int64_t b,
                                        const int32_t* __restrict__ map) {
  const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (x >= b * b) return;
  const int64_t i = x % b, j = x / b;
  F[map[i] + (int64_t)map[j] * f] += U[x];
}

// ---------------------------------------------------------------------------
// PCG vector kernels (Algorithm 1).  Reductions are two-pass with a fixed
// grid and a fixed tree order, so results are reproducible run to run.
// Scalars live on the device: sc[0] and sc[10] = z^T r of the last two steps in
// turn, sc[1] = p^T w, sc[2] = alpha, sc[3] = beta, sc[4] = r^T r, sc[6] =
// breakdown flag.
// ---------------------------------------------------------------------------
constexpr int kRedBlocks = 1024;
constexpr int kRedThreads = 256;

// two consecutive entries as one 16-byte (double) or 8-byte (float) access
template <typename T>
struct Pair2;
template <>
struct Pair2<double> {
  typedef double2 type;
};
template <>
struct Pair2<float> {
  typedef float2 type;
};


__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int q = 0; q < (int)(blockDim.x >> 6); ++q) s += sh[q];
  return s;
}

template <typename TA, typename TB>
__global__ void __launch_bounds__(kRedThreads)
dot_partial_kernel(const TA* __restrict__ a, const TB* __restrict__ b, double* __restrict__ part, int64_t n,
                   int pairs) {
  __shared__ double sh[kRedThreads / 64];
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  double s = 0.0;
  if (pairs) {
    typedef typename Pair2<TA>::type A2;
    typedef typename Pair2<TB>::type B2;
    const A2* a2 = reinterpret_cast<const A2*>(a);
    const B2* b2 = reinterpret_cast<const B2*>(b);
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n / 2; x += stride) {
      const A2 av = a2[x];
      const B2 bv = b2[x];
      s += (double)av.x * (double)bv.x;
      s += (double)av.y * (double)bv.y;
    }
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) s += (double)a[n - 1] * (double)b[n - 1];
  } else {
    for (int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; x < n; x += stride)
      s += (double)a[x] * (double)b[x];
  }
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// the scalars of one step of Algorithm 1 from a finished sum
//   mode 0: sc[dst] = sum;  mode 1: alpha = sc[rz_in] / sum (p^T w);
//   mode 2: beta = sum / sc[rz_in], sc[rz_out] = sum;
//   mode 3: sc[4] = sum (r^T r), also to the host with the breakdown flag
__device__ __forceinline__ void pcg_scalar(double s, double* sc, int dst, int mode, int rz_in, int rz_out,
                                           double* host) {
  if (mode == 1) {
    const double a = sc[rz_in] / s;
    if (step_breaks(s, a, sc)) sc[6] = 1.0;
    sc[1] = s;
    sc[2] = a;
  } else if (mode == 2) {
    const double bta = s / sc[rz_in];
    if (!isfinite(bta)) sc[6] = 1.0;
    sc[3] = bta;
    sc[rz_out] = s;
  } else if (mode == 3) {
    sc[4] = s;
    if (host != nullptr) {
      host[0] = s;
      host[1] = sc[6];
    }
  } else {
    sc[dst] = s;
  }
}

// One workgroup sums up to kOneSum partial sums, 8 loads per lane in flight.
// (Through chunk sums and a second launch it takes 10 us; alone 5 to 7.)
constexpr int64_t kOneSum = 65536;
constexpr int kFinalThreads = 1024;
__global__ void __launch_bounds__(kFinalThreads)
dot_final_kernel(const double* __restrict__ part, double* __restrict__ sc, int nparts, int dst, int mode, int rz_in,
                 int rz_out, double* __restrict__ host) {
  __shared__ double sh[kFinalThreads / 64];
  double a[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) a[u] = 0.0;
  for (int x = threadIdx.x; x < nparts; x += 8 * kFinalThreads)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = x + u * kFinalThreads;
      a[u] += q < nparts ? part[q] : 0.0;
    }
  const double s = block_sum(((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7])), sh);
  if (threadIdx.x == 0) pcg_scalar(s, sc, dst, mode, rz_in, rz_out, host);
}

// first stage of a reduction over many partial sums: block b sums the
// partials [b * chunk, (b + 1) * chunk) in a fixed order
__global__ void __launch_bounds__(kRedThreads)
sum_chunks_kernel(const double* __restrict__ in, double* __restrict__ out, int64_t n, int64_t chunk) {
  __shared__ double sh[kRedThreads / 64];
  const int64_t b0 = (int64_t)blockIdx.x * chunk, b1 = b0 + chunk < n ? b0 + chunk : n;
  double s = 0.0;
  for (int64_t x = b0 + threadIdx.x; x < b1; x += blockDim.x) s += in[x];
  s = block_sum(s, sh);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// x += alpha p (this iteration's alpha); p = z + beta p: PCG's last step where
// there is no preconditioner (z = r).  Nothing once the breakdown flag is set (x
// keeps its last finite iterate).
// With `pairs`, entries go two at a time (all pointers 16-byte aligned, a
// single odd tail entry handled by thread 0 of block 0).
template <typename T>
__global__ void __launch_bounds__(256)
update_px_kernel(T* __restrict__ x, T* __restrict__ p, const T* __restrict__ z, const double* __restrict__ sc,
                 int64_t n, int pairs) {
  if (sc[6] != 0.0) return;  // whole grid
  typedef typename Pair2<T>::type T2;
  const T al = (T)sc[2];
  const T beta = (T)sc[3];
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  if (pairs) {
    T2* x2 = reinterpret_cast<T2*>(x);
    T2* p2 = reinterpret_cast<T2*>(p);
    const T2* z2 = reinterpret_cast<const T2*>(z);
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n / 2; q += stride) {
      const T2 pq = p2[q], zq = z2[q];
      T2 xq = x2[q], pn;
      xq.x += al * pq.x;
      xq.y += al * pq.y;
      pn.x = zq.x + beta * pq.x;
      pn.y = zq.y + beta * pq.y;
      x2[q] = xq;
      p2[q] = pn;
    }
    if ((n & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
      const T pq = p[n - 1];
      x[n - 1] += al * pq;
      p[n - 1] = z[n - 1] + beta * pq;
    }
  } else {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += stride) {
      const T pq = p[q];
      x[q] += al * pq;
      p[q] = z[q] + beta * pq;
    }
  }
}

// x += alpha p (the last iteration's deferred update; nothing after a breakdown)
template <typename T>
__global__ void __launch_bounds__(256)
update_x_kernel(T* __restrict__ x, const T* __restrict__ p, const double* __restrict__ sc, int64_t n) {
  if (sc[6] != 0.0) return;  // whole grid
  const T al = (T)sc[2];
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
    x[q] += al * p[q];
}

template <typename TD, typename TS>
__global__ void __launch_bounds__(256) copy_kernel(TD* __restrict__ d, const TS* __restrict__ s, int64_t n) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
    d[q] = (TD)s[q];
}

// Bandwidth probes (copy, triad, read) over n doubles as double2 pairs with a
// grid-stride loop: the on-device ceiling that the streaming kernels of the
// solver are compared with.  n is even and the pointers are 16-byte aligned.
__global__ void __launch_bounds__(256) stream_copy_kernel(double2* __restrict__ b, const double2* __restrict__ a,
                                                          int64_t n2) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n2; q += (int64_t)gridDim.x * blockDim.x)
    b[q] = a[q];
}

__global__ void __launch_bounds__(256) stream_triad_kernel(double2* __restrict__ c, const double2* __restrict__ a,
                                                           const double2* __restrict__ b, double s, int64_t n2) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n2; q += (int64_t)gridDim.x * blockDim.x) {
    const double2 x = a[q], y = b[q];
    c[q] = make_double2(x.x + s * y.x, x.y + s * y.y);
  }
}

__global__ void __launch_bounds__(256) stream_read_kernel(const double2* __restrict__ a, int64_t n2,
                                                          double* __restrict__ part) {
  double v = 0.0;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n2; q += (int64_t)gridDim.x * blockDim.x) {
    const double2 x = a[q];
    v += x.x + x.y;
  }
  __shared__ double red[4];
  const double t = group_sum<256>(v, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// Right-hand side of one backward Euler step of the heat equation (Section
// 6.2): b_N = m_N (u_N / dt + q_N) on free nodes, 0 on Dirichlet nodes
// (q = NULL: no source).
__global__ void __launch_bounds__(256)
heat_rhs_kernel(double* __restrict__ b, const double* __restrict__ u, const double* __restrict__ q,
                const double* __restrict__ mN, const uint8_t* __restrict__ dir, double dt, int64_t n) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < n) b[g] = dir[g] ? 0.0 : mN[g] * (u[g] / dt + (q != nullptr ? q[g] : 0.0));
}

template <typename T>
__global__ void __launch_bounds__(256) fill_kernel(T* __restrict__ d, T v, int64_t n) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
    d[q] = v;
}

// r = b - Ax (FP64) on the free nodes, 0 on the Dirichlet set (Ax = NULL:
// r = b there), with partial sums of r^T r
__global__ void __launch_bounds__(kRedThreads)
residual_kernel(double* __restrict__ r, const double* __restrict__ b, const double* __restrict__ Ax,
                const uint8_t* __restrict__ dir, double* __restrict__ part, int64_t n) {
  __shared__ double sh[kRedThreads / 64];
  double s = 0.0;
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
    const double v = dir[q] ? 0.0 : b[q] - (Ax != nullptr ? Ax[q] : 0.0);
    r[q] = v;
    s += v * v;
  }
  s = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// f32 = (float)(r64 * scale)
__global__ void __launch_bounds__(256)
scale_to_f32_kernel(float* __restrict__ d, const double* __restrict__ s, double scale, int64_t n) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
    d[q] = (float)(s[q] * scale);
}

// x64 += scale * d32
__global__ void __launch_bounds__(256)
axpy_f32_kernel(double* __restrict__ x, const float* __restrict__ d, double scale, int64_t n) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
    x[q] += scale * (double)d[q];
}

}  // namespace sem
