// Device code shared by the kernels: memory access helpers, activations and
// their derivatives, the chain rule of a layer and its adjoint, the input
// layer, the Navier-Stokes residuals.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include "ddpinn_internal.h"

namespace ddp {

typedef float v4f __attribute__((ext_vector_type(4)));

enum : int { M_PDE = 0, M_VALUE = 1, M_GRAD = 2 };

__device__ __forceinline__ v4f zero4() { return v4f{0.f, 0.f, 0.f, 0.f}; }

// Accesses to device memory through the global address space: generic
// (flat) accesses would also count against the LDS wait counter, so every
// LDS wait would also wait for outstanding memory loads.
#define GLOBAL_AS __attribute__((address_space(1)))
// read-only for the whole launch (work items, subdomain descriptors): loads
// through the constant address space become scalar loads
#define CONST_AS __attribute__((address_space(4)))
__device__ __forceinline__ v4f ldg4(const float* p) { return *(const GLOBAL_AS v4f*)p; }
__device__ __forceinline__ float ldg(const float* p) { return *(const GLOBAL_AS float*)p; }
__device__ __forceinline__ void stg4(float* p, v4f v) { *(GLOBAL_AS v4f*)p = v; }
__device__ __forceinline__ void stg(float* p, float v) { *(GLOBAL_AS float*)p = v; }
// wave-uniform base + 32-bit per-lane byte offset: selects the scalar-base
// addressing form (one lane-offset register instead of a 64-bit address per lane)
__device__ __forceinline__ v4f ldg4u(const float* base, uint32_t off) {
  return *(const GLOBAL_AS v4f*)((const GLOBAL_AS char*)base + off);
}
__device__ __forceinline__ void stg4u(float* base, uint32_t off, v4f v) {
  *(GLOBAL_AS v4f*)((GLOBAL_AS char*)base + off) = v;
}

// sin and cos with full range reduction (device library)
__device__ __forceinline__ void sincos_f32(float z, float& s, float& c) { sincosf(z, &s, &c); }

// tanh without branches, from two textbook forms:
//   |x| < 0.4 : x * P(x^2), P = Maclaurin series of tanh(x)/x through the x^12
//               term (the first omitted term is below 4e-9 relative)
//   otherwise : sign(x) * (1 - 2 / (exp(2|x|) + 1)), hardware exp2 and rcp
// Within ~3 ulp of the exact value over the whole float range (the float32
// error of this scheme is pinned on the CPU).
__device__ __forceinline__ float tanh_f32(float x) {
  const float a = fabsf(x);
  const float u = x * x;
  float p = 3.5921280365724810e-3f;          //  21844/6081075
  p = fmaf(p, u, -8.8632355299021966e-3f);   // -1382/155925
  p = fmaf(p, u, 2.1869488536155203e-2f);    //  62/2835
  p = fmaf(p, u, -5.3968253968253968e-2f);   // -17/315
  p = fmaf(p, u, 1.3333333333333333e-1f);    //  2/15
  p = fmaf(p, u, -3.3333333333333333e-1f);   // -1/3
  p = fmaf(p, u, 1.f);
  const float small = x * p;
  const float e = __builtin_amdgcn_exp2f(a * 2.8853900817779268f);   // exp(2|x|)
  const float big = __builtin_copysignf(fmaf(-2.f, __builtin_amdgcn_rcpf(e + 1.f), 1.f), x);
  return a < 0.4f ? small : big;
}

enum : int { ACT_TANH = 0, ACT_SIN = 1 };

// activation sigma(z) and its first derivatives: tanh (section 2.1 networks)
// or sin (the paper's cylinder networks, section 3.2-3.3)
template <int ACT>
__device__ __forceinline__ void act_d2(float z, float& s, float& s1, float& s2) {
  if constexpr (ACT == ACT_SIN) {
    sincos_f32(z, s, s1);
    s2 = -s;
  } else {
    s = tanh_f32(z);
    s1 = 1.f - s * s;
    s2 = -2.f * s * s1;
  }
}

// SV: the argument is tanh(z0) itself (kept in the stash in place of z0);
// tanh's derivatives are polynomials in it, so tanh is not evaluated again
template <int ACT, bool SV>
__device__ __forceinline__ void act_d2s(float v, float& s, float& s1, float& s2) {
  if constexpr (SV && ACT == ACT_TANH) {
    s = v;
    s1 = 1.f - s * s;
    s2 = -2.f * s * s1;
  } else {
    act_d2<ACT>(v, s, s1, s2);
  }
}

template <int ACT>
__device__ __forceinline__ void act_d3(float z, float& s, float& s1, float& s2, float& s3) {
  if constexpr (ACT == ACT_SIN) {
    sincos_f32(z, s, s1);
    s2 = -s;
    s3 = -s1;
  } else {
    s = tanh_f32(z);
    s1 = 1.f - s * s;
    s2 = -2.f * s * s1;
    s3 = 2.f * s1 * (3.f * s * s - 1.f);
  }
}

template <int ACT, bool SV>
__device__ __forceinline__ void act_d3s(float v, float& s, float& s1, float& s2, float& s3) {
  if constexpr (SV && ACT == ACT_TANH) {
    s = v;
    s1 = 1.f - s * s;
    s2 = -2.f * s * s1;
    s3 = 2.f * s1 * (3.f * s * s - 1.f);
  } else {
    act_d3<ACT>(v, s, s1, s2, s3);
  }
}

// Channel layout of a tile in a given mode.
//   M_PDE  : CM = 2d+2 channels: 0 value, 1..d d/dx_j, d+1 d/dt, d+2..2d+1 d2/dx_j^2
//   M_GRAD : CM = d+1 channels: 0 value, 1..d d/dx_j
//   M_VALUE: CM = 1
// Column block of (channel c, point block pb) = c*NPB + pb.
template <int DIM, int NCB, int MODE>
struct ModeCfg {
  static constexpr int CF = 2 * DIM + 2;
  static constexpr int CM = MODE == M_PDE ? CF : (MODE == M_VALUE ? 1 : DIM + 1);
  static constexpr int NPB = NCB / CM;
  static constexpr int NPTS = 16 * NPB;
  static_assert(NCB % CM == 0, "column blocks must hold whole channel sets");
};

// ---------------------------------------------------------------------------
// activation: z -> h with the chain rule, in place on accumulator fragments
//   h = sigma(z0); h_j = s1 z_j; h_jj = s2 z_j^2 + s1 z_jj
//   s1, s2 = first and second derivative of sigma at z0
// ---------------------------------------------------------------------------
template <int DIM, int NCB, int MODE, int ACT>
__device__ __forceinline__ void act_forward(v4f (&a)[NCB]) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPB = M::NPB;
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float s, s1, s2;
      act_d2<ACT>(a[pb][i], s, s1, s2);
      if constexpr (MODE == M_PDE) {
#pragma unroll
        for (int jj = 0; jj < DIM; ++jj) {
          const float z1 = a[(1 + jj) * NPB + pb][i];
          const float z2 = a[(DIM + 2 + jj) * NPB + pb][i];
          a[(DIM + 2 + jj) * NPB + pb][i] = s2 * z1 * z1 + s1 * z2;
        }
#pragma unroll
        for (int jj = 0; jj <= DIM; ++jj) a[(1 + jj) * NPB + pb][i] *= s1;
      } else if constexpr (MODE == M_GRAD) {
#pragma unroll
        for (int jj = 0; jj < DIM; ++jj) a[(1 + jj) * NPB + pb][i] *= s1;
      }
      a[pb][i] = s;
    }
  }
}

// Adjoint of act_forward: hb (dL/dh) -> dL/dz in place; zs holds z.
//   zbar_jj = s1 hbar_jj
//   zbar_j  = s1 hbar_j + 2 s2 z_j hbar_jj      (spatial j; time: s1 hbar_t)
//   zbar_0  = s1 hbar_0 + s2 sum_j z_j hbar_j + sum_j (s3 z_j^2 + s2 z_jj) hbar_jj
//   with s1, s2, s3 the first three derivatives of the activation at z_0
template <int DIM, int NCB, int MODE, int ACT, bool SV = false>
__device__ __forceinline__ void act_adjoint(v4f (&hb)[NCB], const v4f (&zs)[NCB]) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPB = M::NPB;
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (MODE == M_PDE) {
        float s, s1, s2, s3;
        act_d3s<ACT, SV>(zs[pb][i], s, s1, s2, s3);
        float z0b = s1 * hb[pb][i];
#pragma unroll
        for (int jj = 0; jj <= DIM; ++jj) {
          const int c = (1 + jj) * NPB + pb;
          const float h1 = hb[c][i];
          z0b += s2 * zs[c][i] * h1;
          hb[c][i] = s1 * h1;
        }
#pragma unroll
        for (int jj = 0; jj < DIM; ++jj) {
          const int c1 = (1 + jj) * NPB + pb, c2 = (DIM + 2 + jj) * NPB + pb;
          const float h2 = hb[c2][i];
          const float z1 = zs[c1][i], z2 = zs[c2][i];
          hb[c2][i] = s1 * h2;
          hb[c1][i] += 2.f * s2 * z1 * h2;
          z0b += (s3 * z1 * z1 + s2 * z2) * h2;
        }
        hb[pb][i] = z0b;
      } else {
        float s, s1, s2;
        act_d2s<ACT, SV>(zs[pb][i], s, s1, s2);
        hb[pb][i] *= s1;
      }
    }
  }
}

// sum over the 16 lanes of a lane group (same g)
__device__ __forceinline__ float sum16(float v) {
  v += __shfl_xor(v, 8, 16);
  v += __shfl_xor(v, 4, 16);
  v += __shfl_xor(v, 2, 16);
  v += __shfl_xor(v, 1, 16);
  return v;
}

// sum over the four lane groups (same j)
__device__ __forceinline__ float sum_groups(float v) {
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

// ---------------------------------------------------------------------------
// shared forward pieces
// ---------------------------------------------------------------------------

// input layer: z0 = W1 xi + b1; z_j = W1[:, j] (first-derivative channels);
// second-derivative channels start at 0.  xin: LDS [points][D].
template <int DIM, int NCB, int MODE>
__device__ __forceinline__ void input_layer(v4f (&a)[NCB], const float* __restrict__ W1p,
                                            const float* __restrict__ b1p, const float* xin,
                                            int w, int g, int j) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int D = DIM + 1, NPB = M::NPB;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 16 * w + 4 * g + i;
    float wr[D];
#pragma unroll
    for (int q = 0; q < D; ++q) wr[q] = ldg(W1p + r * D + q);
    const float br = ldg(b1p + r);
#pragma unroll
    for (int pb = 0; pb < NPB; ++pb) {
      const float* xp = xin + (16 * pb + j) * D;
      float z = br;
#pragma unroll
      for (int q = 0; q < D; ++q) z += wr[q] * xp[q];
      a[pb][i] = z;
      if constexpr (MODE == M_PDE) {
#pragma unroll
        for (int jj = 0; jj <= DIM; ++jj) a[(1 + jj) * NPB + pb][i] = wr[jj];
#pragma unroll
        for (int jj = 0; jj < DIM; ++jj) a[(DIM + 2 + jj) * NPB + pb][i] = 0.f;
      } else if constexpr (MODE == M_GRAD) {
#pragma unroll
        for (int jj = 0; jj < DIM; ++jj) a[(1 + jj) * NPB + pb][i] = wr[jj];
      }
    }
  }
}

// add the bias to the value-channel column blocks
template <int NCB, int NPB>
__device__ __forceinline__ void add_bias(v4f (&a)[NCB], const float* __restrict__ b, int w, int g) {
  const v4f bv = ldg4(b + 16 * w + 4 * g);
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) a[pb] += bv;
}

// Navier-Stokes residuals r1..r_{d+1} (section 2.1) from the channel stack of
// one point; Y(c, o) = output o of channel c.
template <int DIM, typename F>
__device__ __forceinline__ void residuals(F Y, float nu, float (&r)[DIM + 1]) {
#pragma unroll
  for (int i = 0; i < DIM; ++i) {
    float conv = 0.f, lap = 0.f;
#pragma unroll
    for (int jj = 0; jj < DIM; ++jj) {
      conv += Y(0, jj) * Y(1 + jj, i);
      lap += Y(DIM + 2 + jj, i);
    }
    r[i] = Y(1 + DIM, i) + conv + Y(1 + i, DIM) - nu * lap;
  }
  float div = 0.f;
#pragma unroll
  for (int jj = 0; jj < DIM; ++jj) div += Y(1 + jj, jj);
  r[DIM] = div;
}

// ---------------------------------------------------------------------------
// Hidden-neuron positions.  A hidden layer's Wp positions are read by the four
// lane groups of a GEMM's K dimension in segments of Wp/4.  Neuron n sits at
// position (n / Kq) * (Wp/4) + n % Kq with Kq = ceil(W/4): the padding fills
// the tail of every segment, so the GEMMs stop after Kq K-steps instead of
// Wp/4.  This is a permutation of the hidden neurons with zero weights at the
// padded positions (whose activations are 0), so the network is unchanged.
// ---------------------------------------------------------------------------
__host__ __device__ inline int hid_pos(const Shape& sh, int n) { return (n / sh.Kq) * (sh.Wp / 4) + n % sh.Kq; }
__host__ __device__ inline int hid_neuron(const Shape& sh, int p) {
  const int seg = sh.Wp / 4, g = p / seg, s = p - g * seg, n = g * sh.Kq + s;
  return (s < sh.Kq && n < sh.W) ? n : -1;
}

}  // namespace ddp
