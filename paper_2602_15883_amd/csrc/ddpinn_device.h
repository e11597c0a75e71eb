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
// wave-uniform base + 32-bit per-lane byte offset: selects the scalar-base
// addressing form (one lane-offset register instead of a 64-bit address per lane)
__device__ __forceinline__ v4f ldg4u(const float* base, uint32_t off) {
  return *(const GLOBAL_AS v4f*)((const GLOBAL_AS char*)base + off);
}
__device__ __forceinline__ void stg4u(float* base, uint32_t off, v4f v) {
  *(GLOBAL_AS v4f*)((GLOBAL_AS char*)base + off) = v;
}

__device__ __forceinline__ float ldgu(const float* base, uint32_t off) {
  return *(const GLOBAL_AS float*)((const GLOBAL_AS char*)base + off);
}
__device__ __forceinline__ void stgu(float* base, uint32_t off, float v) {
  *(GLOBAL_AS float*)((GLOBAL_AS char*)base + off) = v;
}

// sin and cos of four values.  The device library's sincosf carries its reduction
// of large arguments inline: 0.5 KB of code and a branch per value, which, unrolled over a wave's fragments, made
// the sin kernels up to 480 KB (the instruction cache holds 64) and spill.
//   |z| <= 2^16 : r = z - k pi/2 in three fma steps (Cody and Waite; the first is
//                 exact), then the Maclaurin series of sin and cos on |r| <= pi/4 (first
//                 omitted terms 2e-9 and 1e-10)
//   otherwise   : k and r from z * 2/pi modulo 4 in double, in pieces of 28 bits of 2/pi whose
//                 products are exact (Payne and Hanek); one value after another in a
//                 loop, which no ordinary network enters
// Within 1.5 ulp of the exact values (the scheme is pinned on the CPU); RMS error on
// [-10, 10] 0.28 (sin) and 0.29 (cos) of 2^-24, the library's 0.30 and 0.31.
__device__ __forceinline__ void sincos_reduce_large(float z, float& r, int& k) {
  const double x = z;
  double p = 0;
  auto piece = [&](double c) {
    const double t = x * c;
    p += fma(-4.0, __builtin_rint(t * 0.25), t);
  };
  piece(0xa2f9836p-28);
  piece(0xe4e4415p-56);
  piece(0x29fc275p-84);
  piece(0x7d1f534p-112);
  piece(0xddc0db6p-140);
  piece(0x295993cp-168);
  piece(0x439041fp-196);
  piece(0xe5163abp-224);
  const double q = __builtin_rint(p);
  k = (int)q;
  r = (float)((p - q) * 1.5707963267948966);
}
__device__ __forceinline__ void sincos4(v4f z, v4f& s, v4f& c) {
  v4f r;
  int k[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float q = __builtin_rintf(z[i] * 0.63661977236758134f);
    r[i] = fmaf(-q, -0x1.ee59dap-50f, fmaf(-q, -0x1.777a5cp-25f, fmaf(-q, 0x1.921fb6p+0f, z[i])));
    k[i] = (int)q;
  }
  const float m = fmaxf(fmaxf(fabsf(z[0]), fabsf(z[1])), fmaxf(fabsf(z[2]), fabsf(z[3])));
  if (__builtin_expect(m > 65536.f, 0)) {
#pragma clang loop unroll(disable)
    for (int t = 0; t < 4; ++t) {   // the four values rotate through the first place
      float r0 = r[0];
      if (fabsf(z[0]) > 65536.f) sincos_reduce_large(z[0], r0, k[0]);
      r[0] = r0;
      z = __builtin_shufflevector(z, z, 1, 2, 3, 0);
      r = __builtin_shufflevector(r, r, 1, 2, 3, 0);
      const int k0 = k[0];
      k[0] = k[1];
      k[1] = k[2];
      k[2] = k[3];
      k[3] = k0;
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float x = r[i], u = x * x;
    float p = 2.7557319223985893e-6f;       // 1/9!
    p = fmaf(u, p, -1.9841269841269841e-4f);
    p = fmaf(u, p, 8.3333333333333333e-3f);
    p = fmaf(u, p, -1.6666666666666667e-1f);
    const float sr = fmaf(x * u, p, x);
    float q = -2.7557319223985888e-7f;      // -1/10!
    q = fmaf(u, q, 2.4801587301587302e-5f);
    q = fmaf(u, q, -1.3888888888888889e-3f);
    q = fmaf(u, q, 4.1666666666666667e-2f);
    q = fmaf(u, q, -0.5f);
    const float cr = fmaf(u, q, 1.f);
    // odd quarter turns exchange the two; the signs are bit 1 of k and of k + 1
    const float a = (k[i] & 1) ? cr : sr, b = (k[i] & 1) ? sr : cr;
    s[i] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a) ^ ((uint32_t)(k[i] & 2) << 30));
    c[i] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, b) ^ ((uint32_t)((k[i] + 1) & 2) << 30));
  }
}

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

// activation sigma and its first derivatives: tanh (section 2.1 networks) or
// sin (the paper's cylinder networks, section 3.2-3.3), four values at a time.
// SV: the argument is tanh(z0) itself (kept in the stash in place of z0);
// tanh's derivatives are polynomials in it, so tanh is not evaluated again
template <int ACT, bool SV = false>
__device__ __forceinline__ void act4(v4f z, v4f& s, v4f& s1, v4f& s2) {
  if constexpr (ACT == ACT_SIN) {
    sincos4(z, s, s1);
    s2 = -s;
  } else {
    if constexpr (SV) {
      s = z;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) s[i] = tanh_f32(z[i]);
    }
    s1 = 1.f - s * s;
    s2 = -2.f * s * s1;
  }
}

// the third derivative from the lower ones
template <int ACT>
__device__ __forceinline__ v4f act_third(v4f s, v4f s1) {
  if constexpr (ACT == ACT_SIN) return -s1;
  else return 2.f * s1 * (3.f * s * s - 1.f);
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
    v4f s, s1, s2;
    act4<ACT>(a[pb], s, s1, s2);
    a[pb] = s;
    if constexpr (MODE == M_PDE) {
#pragma unroll
      for (int jj = 0; jj < DIM; ++jj) {
        const v4f z1 = a[(1 + jj) * NPB + pb];
        v4f& z2 = a[(DIM + 2 + jj) * NPB + pb];
        z2 = s2 * z1 * z1 + s1 * z2;
      }
    }
    if constexpr (MODE != M_VALUE) {
#pragma unroll
      for (int jj = 0; jj < M::CM - 1 && jj <= DIM; ++jj) a[(1 + jj) * NPB + pb] *= s1;
    }
  }
}

// Adjoint of act_forward: hb (dL/dh) -> dL/dz in place; zs holds z.
//   zbar_jj = s1 hbar_jj
//   zbar_j  = s1 hbar_j + 2 s2 z_j hbar_jj      (spatial j; time: s1 hbar_t)
//   zbar_0  = s1 hbar_0 + s2 sum_j z_j hbar_j + sum_j (s3 z_j^2 + s2 z_jj) hbar_jj
//   with s1, s2, s3 the first three derivatives of the activation at z_0
template <int DIM, int NCB, int MODE, int ACT>
__device__ __forceinline__ void act_adjoint(v4f (&hb)[NCB], const v4f (&zs)[NCB]) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPB = M::NPB;
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    v4f s, s1, s2;
    act4<ACT>(zs[pb], s, s1, s2);
    v4f z0b = s1 * hb[pb];
    if constexpr (MODE == M_PDE) {
      const v4f s3 = act_third<ACT>(s, s1);
#pragma unroll
      for (int jj = 0; jj <= DIM; ++jj) {
        const int c = (1 + jj) * NPB + pb;
        const v4f h1 = hb[c];
        z0b += s2 * zs[c] * h1;
        hb[c] = s1 * h1;
      }
#pragma unroll
      for (int jj = 0; jj < DIM; ++jj) {
        const int c1 = (1 + jj) * NPB + pb, c2 = (DIM + 2 + jj) * NPB + pb;
        const v4f h2 = hb[c2], z1 = zs[c1], z2 = zs[c2];
        hb[c2] = s1 * h2;
        hb[c1] += 2.f * s2 * z1 * h2;
        z0b += (s3 * z1 * z1 + s2 * z2) * h2;
      }
    }
    hb[pb] = z0b;
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
// Hidden-neuron positions (fp32 kernels; on triples Kq = Wp/4 and every neuron is at
// its own position).  A hidden layer's Wp positions are read by the four
// lane groups of a GEMM's K dimension in segments of Wp/4.  Neuron n sits at
// position (n / Kq) * (Wp/4) + n % Kq with Kq = ceil(W/4): the padding fills
// the tail of every segment, so the GEMMs stop after Kq K-steps instead of
// Wp/4.  This is a permutation of the hidden neurons with zero weights at the
// padded positions (whose activations are 0), so the network is unchanged.
// ---------------------------------------------------------------------------
__host__ __device__ inline int hid_neuron(const Shape& sh, int p) {
  const int seg = sh.Wp / 4, g = p / seg, s = p - g * seg, n = g * sh.Kq + s;
  return (s < sh.Kq && n < sh.W) ? n : -1;
}

}  // namespace ddp
