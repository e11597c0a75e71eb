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
// products, so that a layer's chain holds no fetch from L2 or beyond.  NKB: K blocks held
// (all four for every network, the copies of unused ones cost 2D 6x48, 4,000 points 12.7 us against 10.9).
template <int DIM, int NCB, int MODE, int ACT, int NKB>
__device__ __forceinline__ void split_forward_small(const Shape& sh, const float* fr, char* lds, const SplitQueryLds& L,
                                                    int w, int lane, int tid, int nthr) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int D = DIM + 1;
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

// One or two row blocks, in one wave: a layer's result is, split, the operand of the next
// layer's products as it lies in the wave's registers (lane (g, j): neurons 4g + i of each block,
// column j), so that nothing goes through LDS and no wave waits for another.  With two, lane
// groups 1 and 2 hold the second block first (k_neuron's order: the weight rows are taken so).
// One block: through the stack, a wave has too few products to cover it (2D 6x16, 4,000 points: uvpw
// 14.9 us, 8.5 so, fp32 matrix instructions 11.7; values 10.2, 6.8, 8.1).  Two blocks, full tiles: the stacks
// of 3D tiles fill the LDS at 10 waves per compute unit (3D 6x17: residuals of 300,000 points 310 us, 183
// so, 254 on fp32 matrix instructions; 1,000,000 values 232, 153, 197).
template <int DIM, int NCB, int MODE, int ACT, int R>
__device__ __forceinline__ void split_forward_alone(const Shape& sh, const float* fr, char* lds, const SplitQueryLds& L,
                                                    int lane, int tid, int nthr) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int D = DIM + 1;
  const int g = lane >> 4, j = lane & 15, H = sh.H, Wp = 16 * R;
  const int flip = R == 2 ? slot_half(g) : 0;              // block r of the lane's results is r ^ flip
  // byte offset of the weight row that the lane fetches for block r
  uint32_t row[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    row[r] = (uint32_t)lane * 16u + (R == 2 ? (uint32_t)(r ^ slot_half(j >> 2)) * 12u * kFragFloats : 0u);
  const float* xin = reinterpret_cast<const float*>(lds + L.xin);
  const float* wf = fr + sh.f_hid3;
  const float* bf = fr + sh.f_b + 4 * g;
  v4f acc[R][NCB], bias[R];
  Frags<R> f;   // of the next layer
  auto load = [&](int l) {
    const float* wl = wf + (size_t)(l - 2) * sh.hid3_layer;
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int p = 0; p < 3; ++p) f.a[r][p] = ldg4u(wl + p * kFragFloats, row[r]);
      bias[r] = ldg4(bf + (size_t)(l - 1) * Wp + 16 * (r ^ flip));
    }
  };
#pragma unroll
  for (int r = 0; r < R; ++r)
    input_layer<DIM, NCB, MODE>(acc[r], fr + sh.f_w1, fr + sh.f_b, xin, r ^ flip, g, j);
  if (H > 1) load(2);
#pragma unroll
  for (int r = 0; r < R; ++r) act_forward<DIM, NCB, MODE, ACT>(acc[r]);
  for (int l = 2; l <= H; ++l) {
    const Frags<R> a = f;
    v4f b[R];
#pragma unroll
    for (int r = 0; r < R; ++r) b[r] = bias[r];
    if (l < H) load(l + 1);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      v2u h[R][3];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        split4(acc[r][cb], h[r]);
        acc[r][cb] = zero4();
      }
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if constexpr (R == 2) {
            typedef uint32_t v4u __attribute__((ext_vector_type(4)));
            const v4u u = __builtin_shufflevector(h[0][kPartB[q]], h[1][kPartB[q]], 0, 1, 2, 3);
            acc[r][cb] = mfma32(__builtin_bit_cast(v8h, a.a[r][kPartA[q]]), __builtin_bit_cast(v8h, u), acc[r][cb]);
          } else {
            const v8s a8 = __builtin_bit_cast(v8s, a.a[r][kPartA[q]]);
            acc[r][cb] = mfma16(__builtin_shufflevector(a8, a8, 0, 1, 2, 3), __builtin_bit_cast(v4s, h[r][kPartB[q]]), acc[r][cb]);
          }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
      for (int pb = 0; pb < M::NPB; ++pb) acc[r][pb] += b[r];
      act_forward<DIM, NCB, MODE, ACT>(acc[r]);
    }
  }
  // output layer: each block's sum on its own and over the lane groups in the order in which
  // output_partials and output_sum take them, so that a point's result is the same in every tile
  float* ys = reinterpret_cast<float*>(lds + L.ys);
#pragma unroll
  for (int o = 0; o < D; ++o) {
    v4f wo[R];
#pragma unroll
    for (int r = 0; r < R; ++r) wo[r] = ldg4(fr + sh.f_wo + o * Wp + 16 * (r ^ flip) + 4 * g);
    const float bo = ldg(fr + sh.f_bo + o);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      float t[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        t[r] = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) t[r] = fmaf(wo[r][i], acc[r][cb][i], t[r]);
      }
      float y = group_sum(R == 2 && flip ? t[R - 1] : t[0]);
      if constexpr (R == 2) y += group_sum(flip ? t[0] : t[1]);
      if (cb < M::NPB) y += bo;
      if (g == 0) ys[(o * NCB + cb) * 16 + j] = y;
    }
  }
  __syncthreads();
}

// How the waves share the row blocks: one each; above 128 neurons eight waves, some with two;
// one wave with one block, or two, in all.  (Instances of their own: a branch on the last ones in the first costs its
// registers, 3D 6x100, 300,000 values 313 -> 321 us.)
enum : int { ROWS_EACH = 0, ROWS_WIDE = 1, ROWS_ONE = 2, ROWS_TWO = 3 };
constexpr bool rows_alone(int rows) { return rows == ROWS_ONE || rows == ROWS_TWO; }
// waves per SIMD that the registers have to leave room for
constexpr int waves_per_simd(int rows, int small) {
  return rows == ROWS_WIDE || (rows == ROWS_EACH && small == 1) ? 2 : rows == ROWS_TWO ? 3 : 4;
}
template <int DIM, int NCB, int MODE, int ACT, int ROWS, bool AHEAD = true>
__device__ __forceinline__ void split_forward_any(const Shape& sh, const float* fr, char* lds, const SplitQueryLds& L,
                                                  int w, int lane, int tid, int nthr) {
  if constexpr (rows_alone(ROWS)) {
    split_forward_alone<DIM, NCB, MODE, ACT, ROWS == ROWS_TWO ? 2 : 1>(sh, fr, lds, L, lane, tid, nthr);
  } else if constexpr (ROWS == ROWS_WIDE) {
    const int rb0 = split_rb0(w, sh.NW, sh.NWV);
    if (split_rb0(w + 1, sh.NW, sh.NWV) - rb0 == 2)
      split_forward<DIM, NCB, MODE, ACT, 2>(sh, fr, lds, L, rb0, w, lane, tid, nthr);
    else split_forward<DIM, NCB, MODE, ACT, 1>(sh, fr, lds, L, rb0, w, lane, tid, nthr);
  } else if constexpr (NCB <= 3 && AHEAD) {
    if (sh.NW <= 2) split_forward_small<DIM, NCB, MODE, ACT, 1>(sh, fr, lds, L, w, lane, tid, nthr);
    else if (sh.NW <= 4) split_forward_small<DIM, NCB, MODE, ACT, 2>(sh, fr, lds, L, w, lane, tid, nthr);
    else split_forward_small<DIM, NCB, MODE, ACT, kMaxWaves / 2>(sh, fr, lds, L, w, lane, tid, nthr);
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
template <int DIM, int MODE, int ACT, int SMALL, int ROWS>
__global__ __launch_bounds__(rows_alone(ROWS) ? 64 : 512, waves_per_simd(ROWS, SMALL))
void split_query_kernel(const QueryArgs a) {
  constexpr int D = DIM + 1, CF = 2 * DIM + 2;
  constexpr int CMODE = MODE == M_VALUE ? 1 : (MODE == M_GRAD ? DIM + 1 : CF);
  constexpr int NCB = SMALL ? CMODE : CF;
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPTS = M::NPTS, NCOL = 16 * NCB;
  extern __shared__ __align__(16) char qlds[];
  const Shape& sh = a.sh;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SplitQueryLds L = split_query_lds(D, sh.NW, sh.NWV, NCB, rows_alone(ROWS));
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
    split_forward_any<DIM, NCB, MODE, ACT, ROWS, SMALL != 2>(sh, a.subs[sub].frag, qlds, L, w, lane, tid, nthr);
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
template <int DIM, int ACT, int ROWS>
__global__ __launch_bounds__(ROWS == ROWS_ONE ? 64 : 512, waves_per_simd(ROWS, 0)) void split_exchange_kernel(const ExchangeArgs a) {
  constexpr int D = DIM + 1, CF = 2 * DIM + 2, NCB = CF, NCOL = 16 * NCB;
  extern __shared__ __align__(16) char qlds[];
  const Shape& sh = a.sh;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SplitQueryLds L = split_query_lds(D, sh.NW, sh.NWV, NCB, rows_alone(ROWS));
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
    split_forward_any<DIM, NCB, M_VALUE, ACT, ROWS>(sh, a.subs[it.b].frag, qlds, L, w, lane, tid, nthr);
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
template <int DIM, int MODE, int SMALL, int ROWS>
static const void* ptr_act(int act) {
  return act == ACT_SIN ? (const void*)split_query_kernel<DIM, MODE, ACT_SIN, SMALL, ROWS>
                        : (const void*)split_query_kernel<DIM, MODE, ACT_TANH, SMALL, ROWS>;
}
template <int DIM, int ROWS>
static const void* ptr_mode(int mode, int act, int small) {
  if constexpr (ROWS == ROWS_EACH) {
    if (mode == M_VALUE && small == 2) return ptr_act<DIM, M_VALUE, 2, ROWS>(act);
  }
  if constexpr (ROWS != ROWS_TWO) {
    if (mode == M_VALUE && small) return ptr_act<DIM, M_VALUE, 1, ROWS>(act);
    if constexpr (DIM == 2)
      if (mode == M_GRAD && small) return ptr_act<DIM, M_GRAD, 1, ROWS>(act);
  }
  if (mode == M_VALUE) return ptr_act<DIM, M_VALUE, 0, ROWS>(act);
  // only 2D has a gradient-mode query (u, v, p, omega)
  if constexpr (DIM == 2)
    if (mode == M_GRAD) return ptr_act<DIM, M_GRAD, 0, ROWS>(act);
  return ptr_act<DIM, M_PDE, 0, ROWS>(act);
}
template <int DIM>
const void* split_query_ptr(int mode, int act, int small, int NW) {
  if (NW == 1) return ptr_mode<DIM, ROWS_ONE>(mode, act, small);
  if (small == 3) return ptr_mode<DIM, ROWS_TWO>(mode, act, 0);   // (two row blocks)
  return NW > kMaxWaves ? ptr_mode<DIM, ROWS_WIDE>(mode, act, small) : ptr_mode<DIM, ROWS_EACH>(mode, act, small);
}
template <int DIM, int ROWS>
static const void* ptr_exchange(int act) {
  return act == ACT_SIN ? (const void*)split_exchange_kernel<DIM, ACT_SIN, ROWS> : (const void*)split_exchange_kernel<DIM, ACT_TANH, ROWS>;
}
template <int DIM>
const void* split_exchange_ptr(int act, int NW) {
  if (NW == 1) return ptr_exchange<DIM, ROWS_ONE>(act);
  return NW > kMaxWaves ? ptr_exchange<DIM, ROWS_WIDE>(act) : ptr_exchange<DIM, ROWS_EACH>(act);
}
template const void* split_query_ptr<DDP_DIM>(int, int, int, int);
template const void* split_exchange_ptr<DDP_DIM>(int, int);

}  // namespace ddp
