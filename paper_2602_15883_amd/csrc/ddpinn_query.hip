// Network forward of the routed query, the interface exchange and the
// evaluation, on bf16 matrix instructions with fp32 operands (ddpinn_split.h).
#include "ddpinn_split.h"

namespace ddp {

// forward of one staged tile (points in xin) through all layers; outputs in ys.
// One LDS stack: every wave's products read it before any wave overwrites it.
template <int DIM, int NCB, int MODE, int ACT, int R>
__device__ __forceinline__ void split_forward(const Shape& sh, const float* fr, char* lds, const SplitQueryLds& L,
                                              int rb0, int w, int lane, int tid, int nthr) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int D = DIM + 1;
  const int g = lane >> 4, j = lane & 15, Wp = sh.Wp, NW = sh.NW, KB = (NW + 1) >> 1;
  const LaneSlots ls = lane_slots(lane);
  const uint32_t lane16 = (uint32_t)lane * 16u;
  const float* xin = reinterpret_cast<const float*>(lds + L.xin);
  v4f acc[R][NCB];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    input_layer<DIM, NCB, MODE>(acc[r], fr + sh.f_w1, fr + sh.f_b, xin, rb0 + r, g, j);
    act_forward<DIM, NCB, MODE, ACT>(acc[r]);
  }
  for (int l = 2; l <= sh.H; ++l) {
    const float* wf = fr + sh.f_hid3 + (size_t)(l - 2) * sh.hid3_layer + (size_t)rb0 * KB * 3 * kFragFloats;
    Frags<R> f;
    load_frags<R>(wf, KB, 0, lane16, f);
    v4f bias[R];
#pragma unroll
    for (int r = 0; r < R; ++r) bias[r] = ldg4(fr + sh.f_b + (l - 1) * Wp + 16 * (rb0 + r) + 4 * g);
    stack_store<R, NCB>(lds, rb0, NW, ls, acc);
    __syncthreads();
    gemm_neurons<R, NCB>(wf, lds, NW, ls, lane16, f, acc);
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int pb = 0; pb < M::NPB; ++pb) acc[r][pb] += bias[r];
      act_forward<DIM, NCB, MODE, ACT>(acc[r]);
    }
    __syncthreads();
  }
  float* part = reinterpret_cast<float*>(lds);
  output_partials<D, R, NCB>(part, fr + sh.f_wo, Wp, rb0, w, g, j, acc);
  __syncthreads();
  output_sum<DIM, NCB, MODE>(part, 4 * sh.NWV, fr + sh.f_bo, reinterpret_cast<float*>(lds + L.ys), tid, nthr);
  __syncthreads();
}

// Up to 128 neurons and one column block per channel (SMALL): the weight
// fragments and the bias of the next layer are requested before the current one's
// products, so that a layer's chain holds no fetch from L2 or beyond.
template <int DIM, int NCB, int MODE, int ACT>
__device__ __forceinline__ void split_forward_small(const Shape& sh, const float* fr, char* lds, const SplitQueryLds& L,
                                                    int w, int lane, int tid, int nthr) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int D = DIM + 1, NKB = kMaxWaves / 2;
  const int g = lane >> 4, j = lane & 15, Wp = sh.Wp, NW = sh.NW, KB = (NW + 1) >> 1, H = sh.H;
  const LaneSlots ls = lane_slots(lane);
  const uint32_t lane16 = (uint32_t)lane * 16u;
  const float* xin = reinterpret_cast<const float*>(lds + L.xin);
  const float* wf = fr + sh.f_hid3 + (size_t)w * KB * 3 * kFragFloats;
  const float* bf = fr + sh.f_b + 16 * w + 4 * g;
  LayerFrags<NKB> f, fn;
  v4f acc[1][NCB], bias, biasn = zero4();
  input_layer<DIM, NCB, MODE>(acc[0], fr + sh.f_w1, fr + sh.f_b, xin, w, g, j);
  if (H > 1) {
    load_layer<NKB>(wf, KB, lane16, fn);
    biasn = ldg4(bf + Wp);
  }
  act_forward<DIM, NCB, MODE, ACT>(acc[0]);
  for (int l = 2; l <= H; ++l) {
    f = fn;
    bias = biasn;
    if (l < H) {
      load_layer<NKB>(wf + (size_t)(l - 1) * sh.hid3_layer, KB, lane16, fn);
      biasn = ldg4(bf + (size_t)l * Wp);
    }
    stack_store<1, NCB>(lds, w, NW, ls, acc);
    __syncthreads();
    gemm_layer<NCB, NKB>(lds, NW, ls, f, acc);
#pragma unroll
    for (int pb = 0; pb < M::NPB; ++pb) acc[0][pb] += bias;
    act_forward<DIM, NCB, MODE, ACT>(acc[0]);
    __syncthreads();
  }
  float* part = reinterpret_cast<float*>(lds);
  output_partials<D, 1, NCB>(part, fr + sh.f_wo, Wp, w, w, g, j, acc);
  __syncthreads();
  output_sum<DIM, NCB, MODE>(part, 4 * sh.NWV, fr + sh.f_bo, reinterpret_cast<float*>(lds + L.ys), tid, nthr);
  __syncthreads();
}

// WIDE: above 128 neurons (eight waves, some with two row blocks)
template <int DIM, int NCB, int MODE, int ACT, int WIDE, bool AHEAD = true>
__device__ __forceinline__ void split_forward_any(const Shape& sh, const float* fr, char* lds, const SplitQueryLds& L,
                                                  int w, int lane, int tid, int nthr) {
  if constexpr (WIDE) {
    const int rb0 = split_rb0(w, sh.NW, sh.NWV);
    if (split_rb0(w + 1, sh.NW, sh.NWV) - rb0 == 2)
      split_forward<DIM, NCB, MODE, ACT, 2>(sh, fr, lds, L, rb0, w, lane, tid, nthr);
    else split_forward<DIM, NCB, MODE, ACT, 1>(sh, fr, lds, L, rb0, w, lane, tid, nthr);
  } else if constexpr (NCB <= 3 && AHEAD) {
    split_forward_small<DIM, NCB, MODE, ACT>(sh, fr, lds, L, w, lane, tid, nthr);
  } else {
    split_forward<DIM, NCB, MODE, ACT, 1>(sh, fr, lds, L, w, w, lane, tid, nthr);
  }
}

// SMALL: one 16-point block per channel of the mode instead of CF column
// blocks, which halves (gradient mode) or divides by six (value mode) the
// work on a tile's critical path; for requests too small to fill the chip
// (450 points of 2D 8x100: 37.3 us with the weights fetched as they are needed, 34.4 so).
// The others run four waves per SIMD and are bound by the matrix units, whose products the other
// waves' activations and splits overlap: uvpw at 200,000 points, 16 networks 2D 8x100, 606 us with routing
// (products 229 at the rate of a large bf16 product); fp32 matrix instructions 1,026.
// SMALL = 2 (values): the same tiles with the weights fetched as they are needed, in half the
// registers, for requests that fill more of the chip.
template <int DIM, int MODE, int ACT, int SMALL, int WIDE>
__global__ __launch_bounds__(512, WIDE || SMALL == 1 ? 2 : 4) void split_query_kernel(const QueryArgs a) {
  constexpr int D = DIM + 1, CF = 2 * DIM + 2;
  constexpr int CMODE = MODE == M_VALUE ? 1 : (MODE == M_GRAD ? DIM + 1 : CF);
  constexpr int NCB = SMALL ? CMODE : CF;
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPTS = M::NPTS, NCOL = 16 * NCB;
  extern __shared__ __align__(16) char qlds[];
  const Shape& sh = a.sh;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SplitQueryLds L = split_query_lds(D, sh.NW, sh.NWV, NCB);
  const float* ys = reinterpret_cast<const float*>(qlds + L.ys);
  float* xin = reinterpret_cast<float*>(qlds + L.xin);
  int32_t* pidx = reinterpret_cast<int32_t*>(qlds + L.pidx);

  // tiles: for routed queries, subdomain s holds points [offsets[s], offsets[s]+counts[s])
  const int nsub = a.counts ? a.n_sub : 1;
  int64_t total = 0;
  for (int s = 0; s < nsub; ++s) {
    const int64_t c = a.counts ? a.counts[s] : a.n;
    total += (c + NPTS - 1) / NPTS;
  }
  // Tiles are ordered by subdomain.  Workgroups are dispatched to the eight
  // XCDs round-robin (workgroup b on XCD b mod 8), each XCD with its own L2:
  // with a grid that is a multiple of 8, XCD x takes the x-th eighth of the
  // tiles, so each L2 holds the weights of a few subdomains, not all.
  int64_t t0 = blockIdx.x, tend = total, tstep = gridDim.x;
  if (gridDim.x >= 16 && (gridDim.x & 7) == 0) {
    const int64_t x = blockIdx.x & 7;
    t0 = x * total / 8 + (blockIdx.x >> 3);
    tend = (x + 1) * total / 8;
    tstep = gridDim.x >> 3;
  }
  for (int64_t t = t0; t < tend; t += tstep) {
    int s = 0;
    int64_t tl = t, c = 0;
    for (; s < nsub; ++s) {
      c = a.counts ? a.counts[s] : a.n;
      const int64_t nt = (c + NPTS - 1) / NPTS;
      if (tl < nt) break;
      tl -= nt;
    }
    const int sub = a.counts ? s : a.sub;
    const int64_t base = (a.counts ? a.offsets[s] : 0) + tl * NPTS;
    const int cnt = (int)((c - tl * NPTS) < NPTS ? (c - tl * NPTS) : NPTS);
    for (int k = tid; k < NPTS; k += nthr)
      pidx[k] = (k < cnt) ? (a.perm ? a.perm[base + k] : (int32_t)(base + k)) : -1;
    __syncthreads();
    for (int k = tid; k < NPTS * D; k += nthr) {
      const int pt = k / D;
      xin[k] = pidx[pt] >= 0 ? a.x[(size_t)pidx[pt] * D + (k - pt * D)] : 0.f;
    }
    __syncthreads();
    split_forward_any<DIM, NCB, MODE, ACT, WIDE, SMALL != 2>(sh, a.subs[sub].frag, qlds, L, w, lane, tid, nthr);
    for (int k = tid; k < NPTS; k += nthr) {
      if (pidx[k] < 0) continue;
      const int64_t q = pidx[k];
      const int pb = k >> 4, jj = k & 15;
      auto Y = [&](int ch, int o) { return ys[o * NCOL + (ch * M::NPB + pb) * 16 + jj]; };
      if (a.what == Q_VALUE) {
        for (int o = 0; o < D; ++o) a.out[q * D + o] = Y(0, o);
      } else if (a.what == Q_UVPW) {
        if constexpr (MODE == M_GRAD && DIM == 2) {
          a.out[q * 4 + 0] = Y(0, 0);
          a.out[q * 4 + 1] = Y(0, 1);
          a.out[q * 4 + 2] = Y(0, 2);
          a.out[q * 4 + 3] = Y(1, 1) - Y(2, 0);   // v_x - u_y
        }
      } else if (a.what == Q_CHANNELS) {
        if constexpr (MODE == M_PDE)
          for (int ch = 0; ch < CF; ++ch)
            for (int o = 0; o < D; ++o) a.out[(q * CF + ch) * D + o] = Y(ch, o);
      } else {
        if constexpr (MODE == M_PDE) {
          float r[D];
          residuals<DIM>(Y, a.nu, r);
          for (int k = 0; k < D; ++k) a.out[q * D + k] = r[k];
        }
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// exchange: neighbour values at ghost points, anchor-normalised pressure.  One
// tile per face or a few: a tile's chain of layers bounds it (48 faces of 2,000 points, 2D 6x64: 72
// us on fp32 matrix instructions, 48 so; the products alone take 13).
// ---------------------------------------------------------------------------
template <int DIM, int ACT, int WIDE>
__global__ __launch_bounds__(512, WIDE ? 2 : 4) void split_exchange_kernel(const ExchangeArgs a) {
  constexpr int D = DIM + 1, CF = 2 * DIM + 2, NCB = CF, NCOL = 16 * NCB;
  extern __shared__ __align__(16) char qlds[];
  const Shape& sh = a.sh;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SplitQueryLds L = split_query_lds(D, sh.NW, sh.NWV, NCB);
  const float* ys = reinterpret_cast<const float*>(qlds + L.ys);
  float* xin = reinterpret_cast<float*>(qlds + L.xin);
  for (int t = blockIdx.x; t < a.n_items; t += gridDim.x) {
    const ExchangeItem it = a.items[t];
    const SubDev& ra = a.subs[it.a];
    const int half = NCOL / 2;
    for (int k = tid; k < NCOL * D; k += nthr) {
      const int pt = k / D, q = k - pt * D;
      float v = 0.f;
      if (it.paired) {
        const int pp = pt < half ? pt : pt - half;
        if (pp < it.count) {
          const float* gx = ra.gh_x + (size_t)(it.start + pp) * D;
          v = (pt < half) ? gx[q] : (q < DIM ? a.x_anc[q] : gx[DIM]);
        }
      } else if (pt < it.count) {
        v = ra.gh_x[(size_t)(it.start + pt) * D + q];
      }
      xin[k] = v;
    }
    __syncthreads();
    split_forward_any<DIM, NCB, M_VALUE, ACT, WIDE>(sh, a.subs[it.b].frag, qlds, L, w, lane, tid, nthr);
    float* tg = a.targets[it.a];
    for (int k = tid; k < it.count; k += nthr) {
      for (int o = 0; o < D; ++o) {
        float v = ys[o * NCOL + k];
        if (o == DIM && it.paired) v -= ys[o * NCOL + half + k];
        tg[(size_t)(it.start + k) * D + o] = v;
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// instances: one dimension per translation unit
// ---------------------------------------------------------------------------
template <int DIM, int MODE, int SMALL, int WIDE>
static const void* ptr_act(int act) {
  return act == ACT_SIN ? (const void*)split_query_kernel<DIM, MODE, ACT_SIN, SMALL, WIDE>
                        : (const void*)split_query_kernel<DIM, MODE, ACT_TANH, SMALL, WIDE>;
}
template <int DIM, int WIDE>
static const void* ptr_mode(int mode, int act, int small) {
  if constexpr (!WIDE) {
    if (mode == M_VALUE && small == 2) return ptr_act<DIM, M_VALUE, 2, WIDE>(act);
  }
  if (mode == M_VALUE) return small ? ptr_act<DIM, M_VALUE, 1, WIDE>(act) : ptr_act<DIM, M_VALUE, 0, WIDE>(act);
  if (mode == M_GRAD) {
    // only 2D has a gradient-mode query (u, v, p, omega)
    if constexpr (DIM == 2) return small ? ptr_act<DIM, M_GRAD, 1, WIDE>(act) : ptr_act<DIM, M_GRAD, 0, WIDE>(act);
  }
  return ptr_act<DIM, M_PDE, 0, WIDE>(act);
}
template <int DIM>
const void* split_query_ptr(int mode, int act, int small, int NW) {
  return NW > kMaxWaves ? ptr_mode<DIM, 1>(mode, act, small) : ptr_mode<DIM, 0>(mode, act, small);
}
template <int DIM>
const void* split_exchange_ptr(int act, int NW) {
  const bool sin = act == ACT_SIN;
  if (NW > kMaxWaves) return sin ? (const void*)split_exchange_kernel<DIM, ACT_SIN, 1> : (const void*)split_exchange_kernel<DIM, ACT_TANH, 1>;
  return sin ? (const void*)split_exchange_kernel<DIM, ACT_SIN, 0> : (const void*)split_exchange_kernel<DIM, ACT_TANH, 0>;
}
template const void* split_query_ptr<DDP_DIM>(int, int, int, int);
template const void* split_exchange_ptr<DDP_DIM>(int, int);

}  // namespace ddp
