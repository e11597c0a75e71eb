// Kernels on FP32 MFMA 16x16x4 for the networks whose activation stack of bf16
// triples (ddpinn_split.h) does not fit in the LDS: 3D above 208 neurons.  A wave
// owns two row blocks, w and w + 8, and runs them one after the other; the step
// holds its backward operands for half of a tile's columns at a time.
//
//   Each hidden layer is Z = W_l H (all channels at once, N = 16*NCB columns).
//   The A operand (weights) streams from a fragment-ordered copy in global
//   memory (L2 resident); the B operand (activations) is staged in LDS.  The
//   chain rule runs in registers on the accumulator fragment: lane (g, j) holds
//   rows 16rb+4g+i (i = 0..3) of column 16cb+j, so every channel of a (neuron,
//   point) pair sits in one lane.  Backward: pre-activations z of every layer are
//   stashed per tile in a per-workgroup global ring; dW_l = Zbar H_{l-1}^T (K =
//   columns) and Hbar_{l-1} = W_l^T Zbar run on MFMA.
#include "ddpinn_device.h"

namespace ddp {

__device__ __forceinline__ v4f mfma4(float a, float b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// GEMMs on FP32 MFMA 16x16x4
//
// K index of MFMA step s in lane group g (g = lane/16): kmap(s, g) = g*Wq + s
// with Wq = Wp/4, so that 4 consecutive steps of one lane read 4 contiguous
// floats (one ds_read_b128).  The weight fragments are laid out with the same
// map:  frag[((w*K4 + s4)*64 + lane)*4 + q] = W[16w + lane%16][kmap(4 s4 + q, lane/16)].
// ---------------------------------------------------------------------------

// acc[cb] += A(16 rows of this wave) * B(LDS [16*NCB cols][S], K = Wp)
template <int NCB>
__device__ __forceinline__ void mfma_step(const v4f a, const float* bb, int S, int s4, v4f (&acc)[NCB]) {
  v4f b[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) b[cb] = *reinterpret_cast<const v4f*>(bb + cb * 16 * S + 4 * s4);
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[cb] = mfma4(a[q], b[cb][q], acc[cb]);
}

// the last, partial chunk: only its first KT K-steps hold neurons
template <int NCB>
__device__ __forceinline__ void mfma_tail(const v4f a, const float* bb, int S, int s4, int KT, v4f (&acc)[NCB]) {
  v4f b[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) b[cb] = *reinterpret_cast<const v4f*>(bb + cb * 16 * S + 4 * s4);
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) acc[cb] = mfma4(a[0], b[cb][0], acc[cb]);
  if (KT > 1) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[cb] = mfma4(a[1], b[cb][1], acc[cb]);
  }
  if (KT > 2) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[cb] = mfma4(a[2], b[cb][2], acc[cb]);
  }
}

// K = 4*K4 + KT steps: K4 full chunks of four, then KT (0..3) more.  The weight
// fragment of the next chunk is in flight while the MFMAs of the current one
// run; chunks past the last re-read the last one.
template <int NCB>
__device__ __forceinline__ void gemm_rows(const float* __restrict__ afrag, const float* bufB,
                                          int S, int K4, int g, int j, int lane,
                                          v4f (&acc)[NCB], int KT) {
  const int KC = K4 + (KT ? 1 : 0);   // chunks per row block (4*KC = Wp/4, a lane group's segment)
  const float* bb = bufB + j * S + g * (4 * KC);
  const uint32_t lo = (uint32_t)lane * 16u;
  auto frag = [&](int c) { return ldg4u(afrag + (c < KC ? c : KC - 1) * 256, lo); };
  v4f a0 = frag(0);
  v4f a1 = frag(1);
  int s4 = 0;
  // a0, a1: the fragments of chunks s4 and s4 + 1
  for (; s4 + 2 <= K4; s4 += 2) {
    mfma_step<NCB>(a0, bb, S, s4, acc);
    a0 = frag(s4 + 2);
    mfma_step<NCB>(a1, bb, S, s4 + 1, acc);
    a1 = frag(s4 + 3);
  }
  if (s4 < K4) {
    mfma_step<NCB>(a0, bb, S, s4, acc);
    a0 = a1;
    ++s4;
  }
  if (KT) mfma_tail<NCB>(a0, bb, S, s4, KT, acc);
}

// dw[t] += sum_col Zbar[16w + m][col] * Hprev[16(nb0+t) + n][col], t < NNB
//   Zbar from bufG ([col][neuron], stride S); Hprev from bufHb ([neuron][col], stride S2)
//   Column of step (s4, q) in lane group g: 16*s4 + 4*g + q.  The four groups
//   then read Zbar rows 4*S apart (S = Wp + 4 = 4 mod 16, so 16 banks apart):
//   the 64 lanes of one A read hit 64 distinct banks; a group's B read is 4
//   contiguous columns of a neuron row (one ds_read_b128).
template <int NCB, int NNB>
__device__ __forceinline__ void gemm_dw(const float* bufG, int S, const float* bufHb, int S2,
                                        int w, int g, int j, int nb0, v4f (&dw)[4]) {
  const float* ab = bufG + (4 * g) * S + 16 * w + j;
  const float* bb = bufHb + (16 * nb0 + j) * S2 + 4 * g;
  for (int s4 = 0; s4 < NCB; ++s4) {
    float a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = ab[(16 * s4 + q) * S];
    v4f b[NNB];
#pragma unroll
    for (int t = 0; t < NNB; ++t) b[t] = *reinterpret_cast<const v4f*>(bb + t * 16 * S2 + 16 * s4);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int t = 0; t < NNB; ++t) dw[t] = mfma4(a[q], b[t][q], dw[t]);
  }
}


// store an accumulator fragment into the forward LDS layout [col][neuron]
template <int NCB>
__device__ __forceinline__ void store_fwd(float* buf, int S, const v4f (&a)[NCB], int w, int g, int j) {
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
    *reinterpret_cast<v4f*>(buf + (16 * cb + j) * S + 16 * w + 4 * g) = a[cb];
}


// output layer: ys[o][col] = W_{H+1}[o] . h[col] (+ b_{H+1}[o] on value columns)
template <int DIM, int NCB, int MODE>
__device__ __forceinline__ void output_layer(const float* bufH, int S, int Wp,
                                             const float* __restrict__ Wop, const float* __restrict__ bop,
                                             float* ys, int tid, int nthr) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int D = DIM + 1, NCOL = 16 * NCB;
  for (int idx = tid; idx < D * NCOL; idx += nthr) {
    const int o = idx / NCOL, col = idx - o * NCOL;
    const float* hr = bufH + col * S;
    const float* wo = Wop + o * Wp;
    float acc = 0.f;
    for (int n = 0; n < Wp; n += 4) {
      const v4f h4 = *reinterpret_cast<const v4f*>(hr + n);
      const v4f w4 = ldg4(wo + n);
      acc += h4[0] * w4[0];
      acc += h4[1] * w4[1];
      acc += h4[2] * w4[2];
      acc += h4[3] * w4[3];
    }
    if (col < 16 * M::NPB) acc += ldg(bop + o);
    ys[o * NCOL + col] = acc;
  }
}

// ---------------------------------------------------------------------------
// LDS plan of the step kernel (floats)
// ---------------------------------------------------------------------------
struct StepLds {
  int S, S2, NCOL;
  int bufH, bufG, ys, yb, xin, acc1, dbacc, red, sched, total;
};

// The forward keeps one activation stack [NCOL][S] at bufG (row stride S = Wp + 4:
// the rows that one operand read or store touches fall in distinct banks); the
// backward holds Zbar [NCOL/2][S] at bufG and H_{l-1} [Wp][NCOL/2 + 4] at bufH for
// one half of the tile's columns at a time.
__host__ __device__ inline StepLds step_lds(int D, int Wp, int H, int NCB) {
  StepLds L;
  L.NCOL = 16 * NCB;
  L.S = Wp + 4;
  L.S2 = L.NCOL / 2 + 4;
  const int zh = ((L.NCOL / 2) * L.S + 3) & ~3;
  const int bwd = zh + Wp * L.S2;
  const int fwd = L.NCOL * L.S;
  int o = 0;
  L.bufG = o;
  L.bufH = o + zh;
  o += ((fwd > bwd ? fwd : bwd) + 3) & ~3;
  L.ys = o;   o += (D * L.NCOL + 3) & ~3;
  L.yb = o;   o += (D * L.NCOL + 3) & ~3;
  L.xin = o;  o += (L.NCOL * D + 3) & ~3;
  L.acc1 = o; o += (Wp * D + 3) & ~3;
  L.dbacc = o; o += (H * Wp + 3) & ~3;
  L.red = o;  o += 64;
  L.sched = o; o += 4;
  L.total = o;
  return L;
}

// ---------------------------------------------------------------------------
// Backward pieces of one row block, for workgroups whose waves own two row
// blocks (the one-row-block path runs the same steps inline)
// ---------------------------------------------------------------------------

// hbar_H = W_{H+1}^T ybar for the rows of row block rb
template <int D, int NCB>
__device__ __forceinline__ void out_adjoint_rows(v4f (&acc)[NCB], const float* __restrict__ Wop, const float* yb,
                                                 int Wp, int rb, int g, int j) {
  constexpr int NCOL = 16 * NCB;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 16 * rb + 4 * g + i;
    float wo[D];
#pragma unroll
    for (int o = 0; o < D; ++o) wo[o] = ldg(Wop + o * Wp + r);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      float s = 0.f;
#pragma unroll
      for (int o = 0; o < D; ++o) s += wo[o] * yb[o * NCOL + 16 * cb + j];
      acc[cb][i] = s;
    }
  }
}

// layer l, row block rb: zbar from hbar (acc, in place) and z_l (zs); db_l;
// at l = 1 the input-layer gradient dW1
template <int DIM, int NCB, int MODE, int ACT>
__device__ __forceinline__ void adjoint_rows(v4f (&acc)[NCB], const v4f (&zs)[NCB], float* dbacc, float* acc1,
                                             const float* xin, int Wp, int rb, int l, int g, int j) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int D = DIM + 1;
  act_adjoint<DIM, NCB, MODE, ACT>(acc, zs);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float s = 0.f;
#pragma unroll
    for (int pb = 0; pb < M::NPB; ++pb) s += acc[pb][i];
    s = sum16(s);
    if (j == 0) dbacc[(l - 1) * Wp + 16 * rb + 4 * g + i] += s;
  }
  if (l != 1) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 16 * rb + 4 * g + i;
    float v[D];
#pragma unroll
    for (int q = 0; q < D; ++q) v[q] = 0.f;
#pragma unroll
    for (int pb = 0; pb < M::NPB; ++pb) {
      const float* xp = xin + (16 * pb + j) * D;
#pragma unroll
      for (int q = 0; q < D; ++q) {
        v[q] += acc[pb][i] * xp[q];
        if constexpr (MODE == M_PDE) v[q] += acc[(1 + q) * M::NPB + pb][i];
      }
    }
#pragma unroll
    for (int q = 0; q < D; ++q) {
      const float s = sum16(v[q]);
      if (j == 0) acc1[r * D + q] += s;
    }
  }
}

// h = act(z) of a stashed pre-activation stack, only the column blocks
// [CB0, CB0 + NCBH), written to the neuron-major LDS layout of that half
template <int DIM, int NCB, int MODE, int ACT, int CB0, int NCBH>
__device__ __forceinline__ void act_store_bwd_cols(float* buf, int S2, const v4f (&z)[NCB], int rb, int g, int j) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPB = M::NPB;
  auto put = [](float* row, int cb, float v) {
    if (cb >= CB0 && cb < CB0 + NCBH) row[16 * (cb - CB0)] = v;
  };
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    if constexpr (MODE != M_PDE) {
      if (pb < CB0 || pb >= CB0 + NCBH) continue;
    }
    v4f s, s1, s2;
    act4<ACT>(z[pb], s, s1, s2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float* row = buf + (16 * rb + 4 * g + i) * S2 + j;
      put(row, pb, s[i]);
      if constexpr (MODE == M_PDE) {
#pragma unroll
        for (int jj = 0; jj <= DIM; ++jj) put(row, (1 + jj) * NPB + pb, s1[i] * z[(1 + jj) * NPB + pb][i]);
#pragma unroll
        for (int jj = 0; jj < DIM; ++jj) {
          const float z1 = z[(1 + jj) * NPB + pb][i];
          put(row, (DIM + 2 + jj) * NPB + pb, s2[i] * z1 * z1 + s1[i] * z[(DIM + 2 + jj) * NPB + pb][i]);
        }
      }
    }
  }
}

// dW_l += Zbar_l H_{l-1}^T over the (row block, column block) tiles
// [t0, t1) of the layer, row-major, into the layer's block sw of the
// segment's slab.  A tile reads only LDS (the Zbar rows of its row block, the
// H rows of its column block), so any wave can take any tile: the NW*NW tiles
// are cut into equal contiguous runs, one per wave, which balances the SIMDs
// whatever row blocks their waves own (one writer per slab float still).
// Up to four tiles of one row block share the A operand.  The old slab values
// of a group are requested one group ahead (during the previous group's
// GEMM), so two groups' GEMMs cover the read's latency.
template <int NCB>
__device__ __forceinline__ void dw_tiles(float* sw, bool first, const float* bufG, int S, const float* bufH, int S2,
                                         int NW, int t0, int t1, int g, int j, uint32_t lo16) {
  auto group = [&](int t, int& rb, int& nb0) {
    rb = t / NW;
    nb0 = t - rb * NW;
    const int n = NW - nb0 < 4 ? NW - nb0 : 4;
    return n < t1 - t ? n : t1 - t;
  };
  v4f oldn[4];
  if (t0 < t1) {
    int rb, nb0;
    const int nnb = group(t0, rb, nb0);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      oldn[q] = (q < nnb && !first) ? ldg4u(sw + (size_t)(rb * NW + nb0 + q) * 256, lo16) : zero4();
  }
  for (int t = t0; t < t1;) {
    int rb, nb0;
    const int nnb = group(t, rb, nb0);
    v4f old[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) old[q] = oldn[q];
    if (t + nnb < t1 && !first) {
      int rb2, nb2;
      const int n2 = group(t + nnb, rb2, nb2);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        oldn[q] = q < n2 ? ldg4u(sw + (size_t)(rb2 * NW + nb2 + q) * 256, lo16) : zero4();
    }
    v4f dw[4] = {zero4(), zero4(), zero4(), zero4()};
    switch (nnb) {
      case 4: gemm_dw<NCB, 4>(bufG, S, bufH, S2, rb, g, j, nb0, dw); break;
      case 3: gemm_dw<NCB, 3>(bufG, S, bufH, S2, rb, g, j, nb0, dw); break;
      case 2: gemm_dw<NCB, 2>(bufG, S, bufH, S2, rb, g, j, nb0, dw); break;
      default: gemm_dw<NCB, 1>(bufG, S, bufH, S2, rb, g, j, nb0, dw); break;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < nnb) stg4u(sw + (size_t)(rb * NW + nb0 + q) * 256, lo16, old[q] + dw[q]);
    t += nnb;
  }
}

// ---------------------------------------------------------------------------
// Fused step kernel: persistent over this workgroup's item range.
// ---------------------------------------------------------------------------
template <int DIM, int ACT>
__global__ __launch_bounds__(512) void step_kernel(const StepArgs args) {
  constexpr int D = DIM + 1;
  constexpr int CF = 2 * DIM + 2;
  constexpr int NCB = CF;
  constexpr int RPW = 2;   // row blocks per wave
  constexpr int NCOL = 16 * NCB;
  using MP = ModeCfg<DIM, NCB, M_PDE>;
  using MV = ModeCfg<DIM, NCB, M_VALUE>;
  extern __shared__ float lds[];

  const Shape& sh = args.sh;
  const int Wp = sh.Wp, NW = sh.NW, NWV = sh.NWV, H = sh.H;
  const int K4 = sh.Kq >> 2, KT = sh.Kq & 3;   // K-steps of the hidden GEMMs: 4*K4 + KT
  const int tid = threadIdx.x, nthr = blockDim.x;
  // the wave index is uniform across a wave: keeping it in a scalar register
  // lets every per-wave address (weights, stash, slab) be a scalar base plus
  // the lane offset instead of a 64-bit vector address per use
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, j = lane & 15;
  const StepLds L = step_lds(D, Wp, H, NCB);
  float* bufH = lds + L.bufH;
  float* bufG = lds + L.bufG;
  float* ys = lds + L.ys;
  float* yb = lds + L.yb;
  float* xin = lds + L.xin;
  float* acc1 = lds + L.acc1;
  float* dbacc = lds + L.dbacc;
  float* red = lds + L.red;
  const int S = L.S, S2 = L.S2;
  // dW tiles of this wave (two-row-block kernels): the layer's NW*NW tiles in
  // contiguous runs whose lengths even out each wave's work between two
  // barriers.  A row block of Hbar costs NW dW tiles in multiply-adds (both
  // run over the same columns), and its share of the per-row-block VALU work
  // around the GEMMs (recomputing h, the adjoint) adds about a quarter of
  // that; so a wave with fewer Hbar row blocks takes more dW tiles: wave v's
  // share is (9/4 NW^2 - 5/4 NWV * NW * rows(v)) / NWV, rows(v) its row
  // blocks.  cut(v) is the sum of the shares of waves < v, with rows counted in halves.
  auto dw_cut = [&](int v) {
    const int ne = NW - NWV;
    const int hb = 2 * v + 2 * (v < ne ? v : ne);
    return (18 * NW * NW * v - 5 * NW * NWV * hb) / (8 * NWV);
  };
  const int dw_t0 = dw_cut(w), dw_t1 = dw_cut(w + 1);

  // row blocks of this wave: w, and w + NWV when there are more than NWV
  const int nrb = w + NWV < NW ? 2 : 1;
  // stash: H pre-activation stacks per row block; a wave's second row block
  // is NWV blocks further
  float* stash_w = args.stash + (size_t)blockIdx.x * args.stash_per_wg + (size_t)w * H * NCB * 256;
  const size_t stash_rb = (size_t)NWV * H * NCB * 256;
  const uint32_t lo16 = (uint32_t)lane * 16u;   // this lane's byte offset in a 1 KiB wave fragment
  const float nu = args.nu;
  const bool prio = args.prio != 0;   // raise the younger waves' priority for their GEMMs

  // segment accumulators; dW_{H+1} entry tid + r*nthr is thread tid's
  float lacc[6];
  float dwo[RPW], dbo = 0.f;
#pragma unroll
  for (int r = 0; r < RPW; ++r) dwo[r] = 0.f;

  // Item ranges: range blockIdx.x, or, with a counter, ranges taken in turn
  // until none is left (workgroups that share a compute unit do not progress
  // at the same rate, so a static split would leave the slower one last).
  int* s_range = reinterpret_cast<int*>(lds + L.sched);
  int range = blockIdx.x;
  for (;;) {
  if (args.counter) {
    __syncthreads();   // every thread has read the previous range index
    if (tid == 0) *s_range = atomicAdd(args.counter, 1);
    __syncthreads();
    range = *s_range;
  }
  if (range >= args.n_ranges) break;
  const int it0 = ((const CONST_AS int32_t*)args.wg_begin)[range];
  const int it1 = ((const CONST_AS int32_t*)args.wg_begin)[range + 1];
  for (int it = it0; it < it1; ++it) {
    __syncthreads();   // the previous tile's readers of xin/acc1 are done
    const CONST_AS Item& ir = ((const CONST_AS Item*)args.items)[it];
    Item item;
    item.sub = ir.sub;
    item.kind = ir.kind;
    item.start = ir.start;
    item.count = ir.count;
    item.slab = ir.slab;
    item.flags = ir.flags;
    const CONST_AS SubDev& sd = ((const CONST_AS SubDev*)args.subs)[item.sub];
    const float* fr = sd.frag;
    const float* W1p = fr + sh.f_w1;
    const float* bp = fr + sh.f_b;
    const float* Wop = fr + sh.f_wo;
    const float* bop = fr + sh.f_bo;
    const bool pde = item.kind == ITEM_PDE;

    if (item.flags & ITEM_FIRST) {
#pragma unroll
      for (int k = 0; k < 6; ++k) lacc[k] = 0.f;
#pragma unroll
      for (int r = 0; r < RPW; ++r) dwo[r] = 0.f;
      dbo = 0.f;
      for (int k = tid; k < Wp * D; k += nthr) acc1[k] = 0.f;
      for (int k = tid; k < H * Wp; k += nthr) dbacc[k] = 0.f;
    }

    // ---- stage the tile's input points into LDS
    if (pde) {
      for (int k = tid; k < MP::NPTS * D; k += nthr) {
        const int pt = k / D;
        xin[k] = (pt < item.count) ? ldg(sd.pde_x + (size_t)(item.start + pt) * D + (k - pt * D)) : 0.f;
      }
    } else {
      for (int k = tid; k < NCOL * D; k += nthr) {
        const int pt = k / D, q = k - pt * D;
        float v = 0.f;
        if (pt < item.count) {
          int idx = item.start + pt;
          if (idx < sd.n_obs) v = ldg(sd.obs_x + (size_t)idx * D + q);
          else if ((idx -= sd.n_obs) < sd.n_gh) v = ldg(sd.gh_x + (size_t)idx * D + q);
          else v = ldg(sd.anc_x + (size_t)(idx - sd.n_gh) * D + q);
        }
        xin[k] = v;
      }
    }
    __syncthreads();

    v4f acc[NCB];
    // ---- forward: input layer.
    // two row blocks per wave, one activation stack: every wave's GEMMs read
    // the stack before any wave overwrites it; the first block's
    // pre-activations wait in the stash meanwhile
    float* hin = bufG;
    for (int r = 0; r < nrb; ++r) {
      const int rb = w + r * NWV;
      float* st = stash_w + r * stash_rb;
      if (pde) input_layer<DIM, NCB, M_PDE>(acc, W1p, bp, xin, rb, g, j);
      else input_layer<DIM, NCB, M_VALUE>(acc, W1p, bp, xin, rb, g, j);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) stg4u(st + (0 * NCB + cb) * 256, lo16, acc[cb]);
      if (pde) act_forward<DIM, NCB, M_PDE, ACT>(acc);
      else act_forward<DIM, NCB, M_VALUE, ACT>(acc);
      store_fwd<NCB>(hin, S, acc, rb, g, j);
    }
    __syncthreads();
    for (int l = 2; l <= H; ++l) {
      const float* Wl = fr + sh.f_hid + (size_t)(l - 2) * 2 * Wp * Wp;
      for (int r = 0; r < nrb; ++r) {
        const int rb = w + r * NWV;
        float* st = stash_w + r * stash_rb;
        const float* Wf = Wl + (size_t)rb * 16 * Wp;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[cb] = zero4();
        if (prio && w >= (NWV >> 1)) __builtin_amdgcn_s_setprio(2);
        gemm_rows<NCB>(Wf, hin, S, K4, g, j, lane, acc, KT);
        __builtin_amdgcn_s_setprio(0);
        if (pde) add_bias<NCB, MP::NPB>(acc, bp + (l - 1) * Wp, rb, g);
        else add_bias<NCB, MV::NPB>(acc, bp + (l - 1) * Wp, rb, g);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) stg4u(st + ((l - 1) * NCB + cb) * 256, lo16, acc[cb]);
      }
      __syncthreads();
      for (int r = nrb - 1; r >= 0; --r) {
        if (r != nrb - 1) {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) acc[cb] = ldg4u(stash_w + r * stash_rb + ((l - 1) * NCB + cb) * 256, lo16);
        }
        if (pde) act_forward<DIM, NCB, M_PDE, ACT>(acc);
        else act_forward<DIM, NCB, M_VALUE, ACT>(acc);
        store_fwd<NCB>(hin, S, acc, w + r * NWV, g, j);
      }
      __syncthreads();
    }
    // ---- output layer (h_H is in hin)
    if (pde) output_layer<DIM, NCB, M_PDE>(hin, S, Wp, Wop, bop, ys, tid, nthr);
    else output_layer<DIM, NCB, M_VALUE>(hin, S, Wp, Wop, bop, ys, tid, nthr);
    __syncthreads();

    // ---- residuals, losses and output seeds ybar = dL/dy
    if (pde) {
      if (tid < MP::NPTS) {
        const int pb = tid >> 4, jj = tid & 15;
        auto col = [&](int c) { return (c * MP::NPB + pb) * 16 + jj; };
        auto Y = [&](int c, int o) { return ys[o * NCOL + col(c)]; };
        float r[D];
        residuals<DIM>(Y, nu, r);
        const bool valid = tid < item.count;
        float sq = 0.f;
        float rb[D];
#pragma unroll
        for (int k = 0; k < D; ++k) {
          if (!valid) r[k] = 0.f;
          sq += r[k] * r[k];
          rb[k] = 2.f * sd.lam[1] * sd.inv_n[0] * r[k];
        }
        lacc[1] += sq;
        // dL/dy for every channel (derivative of sum_k rb_k r_k / 2 ...)
#pragma unroll
        for (int i = 0; i < DIM; ++i) {
          float s = 0.f;
#pragma unroll
          for (int k = 0; k < DIM; ++k) s += rb[k] * Y(1 + i, k);
          yb[i * NCOL + col(0)] = s;                              // u_i
#pragma unroll
          for (int jx = 0; jx < DIM; ++jx) {
            yb[i * NCOL + col(1 + jx)] = rb[i] * Y(0, jx) + (i == jx ? rb[DIM] : 0.f);   // d_j u_i
            yb[i * NCOL + col(DIM + 2 + jx)] = -nu * rb[i];                               // d_jj u_i
          }
          yb[i * NCOL + col(1 + DIM)] = rb[i];                     // d_t u_i
        }
        yb[DIM * NCOL + col(0)] = 0.f;                             // p
#pragma unroll
        for (int jx = 0; jx < DIM; ++jx) {
          yb[DIM * NCOL + col(1 + jx)] = rb[jx];                   // d_j p
          yb[DIM * NCOL + col(DIM + 2 + jx)] = 0.f;
        }
        yb[DIM * NCOL + col(1 + DIM)] = 0.f;
      }
    } else {
      // one column per point; a workgroup may have fewer threads than columns
      for (int col = tid; col < NCOL; col += nthr) {
        float e[D];
#pragma unroll
        for (int o = 0; o < D; ++o) e[o] = 0.f;
        if (col < item.count) {
          int idx = item.start + col;
          float y[D];
#pragma unroll
          for (int o = 0; o < D; ++o) y[o] = ys[o * NCOL + col];
          if (idx < sd.n_obs) {
            float sq = 0.f;
#pragma unroll
            for (int i = 0; i < DIM; ++i) {
              const float d0 = y[i] - ldg(sd.obs_u + (size_t)idx * DIM + i);
              sq += sd.cw[i] * d0 * d0;
              e[i] = 2.f * sd.lam[0] * sd.inv_n[1] * sd.cw[i] * d0;
            }
            lacc[0] += sq;
          } else if ((idx -= sd.n_obs) < sd.n_gh) {
            float sq = 0.f;
            const float* tg = sd.gh_up + (size_t)idx * D;
#pragma unroll
            for (int i = 0; i < DIM; ++i) {
              const float d0 = y[i] - tg[i];
              sq += sd.cw[i] * d0 * d0;
              e[i] = 2.f * sd.lam[2] * sd.inv_n[2] * sd.cw[i] * d0;
            }
            lacc[2] += sq;
            const float dp = y[DIM] - tg[DIM];
            if (sd.gh_kind[idx]) {
              lacc[4] += dp * dp;
              e[DIM] = 2.f * sd.lam[4] * sd.inv_n[2] * dp;
            } else {
              lacc[3] += dp * dp;
              e[DIM] = 2.f * sd.lam[3] * sd.inv_n[2] * dp;
            }
          } else {
            idx -= sd.n_gh;
            const float dp = y[DIM] - ldg(sd.anc_p + idx);
            lacc[5] += dp * dp;
            e[DIM] = 2.f * sd.lam[5] * sd.inv_n[3] * dp;
          }
        }
#pragma unroll
        for (int o = 0; o < D; ++o) yb[o * NCOL + col] = e[o];
      }
    }
    __syncthreads();

    {
      // ---- two row blocks per wave (more than 8 row blocks): the same steps
      // per row block.  Only one block's zbar fits in registers across a
      // barrier, so the first block's waits in its own stash slot (z_l of
      // that block is dead once its adjoint has run).
      v4f zs[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
        zs[cb] = ldg4u(stash_w + ((H - 1) * NCB + cb) * 256, lo16);
      {
        const int npb = pde ? MP::NPB : MV::NPB;
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
          const int idx = tid + r * nthr;
          if (idx < D * Wp) {
            const int o = idx / Wp, n = idx - o * Wp;
            float s = 0.f;
            for (int col = 0; col < NCOL; ++col) s += yb[o * NCOL + col] * hin[col * S + n];
            dwo[r] += s;
          }
        }
        if (tid < D) {
          float s = 0.f;
          for (int col = 0; col < 16 * npb; ++col) s += yb[tid * NCOL + col];
          dbo += s;
        }
      }
      const bool raise = prio && w >= (NWV >> 1);   // wave priority for the GEMMs, as in the forward
      for (int r = 0; r < nrb; ++r) {
        const int rb = w + r * NWV;
        float* st = stash_w + r * stash_rb;
        if (r > 0) {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) zs[cb] = ldg4u(st + ((H - 1) * NCB + cb) * 256, lo16);
        }
        out_adjoint_rows<D, NCB>(acc, Wop, yb, Wp, rb, g, j);
        if (pde) adjoint_rows<DIM, NCB, M_PDE, ACT>(acc, zs, dbacc, acc1, xin, Wp, rb, H, g, j);
        else adjoint_rows<DIM, NCB, M_VALUE, ACT>(acc, zs, dbacc, acc1, xin, Wp, rb, H, g, j);
        if (H > 1) {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) stg4u(st + ((H - 1) * NCB + cb) * 256, lo16, acc[cb]);
        }
      }
      // The tile's columns in two halves (Zbar and H_{l-1} of one half fit
      // in LDS at a time; the GEMMs are separable over columns).  Every
      // block's zbar and hbar wait in its own stash slot between barriers.
      constexpr int NCBH = NCB / 2;
      for (int l = H; l >= 2; --l) {
        float* sw = args.slabs + (size_t)item.slab * sh.slab_floats + sh.s_hid + (size_t)(l - 2) * Wp * Wp;
        const size_t zl = (size_t)(l - 1) * NCB * 256, zp = (size_t)(l - 2) * NCB * 256;
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
          // this half's Zbar_l of both row blocks: the wave's own stash
          // slots, so they are requested before the barrier (which only
          // guards the LDS stacks)
          v4f t[NCBH];
          v4f tz[2][NCBH];
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            if (r < nrb) {
#pragma unroll
              for (int c = 0; c < NCBH; ++c)
                tz[r][c] = ldg4u(stash_w + r * stash_rb + zl + ((size_t)hh * NCBH + c) * 256, lo16);
            }
          }
          __syncthreads();
#pragma unroll
          for (int r = 0; r < 2; ++r)
            if (r < nrb) store_fwd<NCBH>(bufG, S, tz[r], w + r * NWV, g, j);
          // H_{l-1} of this half, recomputed from z_{l-1}
          for (int r = 0; r < nrb; ++r) {
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) zs[cb] = ldg4u(stash_w + r * stash_rb + zp + cb * 256, lo16);
            if (hh == 0) {
              if (pde) act_store_bwd_cols<DIM, NCB, M_PDE, ACT, 0, NCBH>(bufH, S2, zs, w + r * NWV, g, j);
              else act_store_bwd_cols<DIM, NCB, M_VALUE, ACT, 0, NCBH>(bufH, S2, zs, w + r * NWV, g, j);
            } else {
              if (pde) act_store_bwd_cols<DIM, NCB, M_PDE, ACT, NCBH, NCBH>(bufH, S2, zs, w + r * NWV, g, j);
              else act_store_bwd_cols<DIM, NCB, M_VALUE, ACT, NCBH, NCBH>(bufH, S2, zs, w + r * NWV, g, j);
            }
          }
          __syncthreads();
          if (raise) __builtin_amdgcn_s_setprio(2);
          dw_tiles<NCBH>(sw, (item.flags & ITEM_FIRST) && hh == 0, bufG, S, bufH, S2, NW, dw_t0, dw_t1, g, j,
                         lo16);
          // Hbar_{l-1} of this half into the stash slot of Zbar_l (consumed)
          const float* WTl = fr + sh.f_hid + (size_t)(l - 2) * 2 * Wp * Wp + (size_t)Wp * Wp;
          for (int r = 0; r < nrb; ++r) {
            const int rb = w + r * NWV;
#pragma unroll
            for (int c = 0; c < NCBH; ++c) t[c] = zero4();
            const float* WT = WTl + (size_t)rb * 16 * Wp;
            gemm_rows<NCBH>(WT, bufG, S, K4, g, j, lane, t, KT);
            float* st = stash_w + r * stash_rb + zl + (size_t)hh * NCBH * 256;
#pragma unroll
            for (int c = 0; c < NCBH; ++c) stg4u(st + c * 256, lo16, t[c]);
          }
          __builtin_amdgcn_s_setprio(0);
        }
        // adjoint of layer l-1 per block; zbar_{l-1} replaces z_{l-1}
        for (int r = 0; r < nrb; ++r) {
          const int rb = w + r * NWV;
          float* st = stash_w + r * stash_rb;
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) acc[cb] = ldg4u(st + zl + cb * 256, lo16);
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) zs[cb] = ldg4u(st + zp + cb * 256, lo16);
          if (pde) adjoint_rows<DIM, NCB, M_PDE, ACT>(acc, zs, dbacc, acc1, xin, Wp, rb, l - 1, g, j);
          else adjoint_rows<DIM, NCB, M_VALUE, ACT>(acc, zs, dbacc, acc1, xin, Wp, rb, l - 1, g, j);
          if (l > 2) {
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) stg4u(st + zp + cb * 256, lo16, acc[cb]);
          }
        }
      }
    }

    // ---- end of segment: write the accumulated gradient pieces and losses
    if (item.flags & ITEM_LAST) {
      __syncthreads();
      float* slab = args.slabs + (size_t)item.slab * sh.slab_floats;
      for (int k = tid; k < Wp * D; k += nthr) slab[sh.s_w1 + k] = acc1[k];
      for (int k = tid; k < H * Wp; k += nthr) slab[sh.s_b + k] = dbacc[k];
#pragma unroll
      for (int r = 0; r < RPW; ++r)
        if (tid + r * nthr < D * Wp) slab[sh.s_wo + tid + r * nthr] = dwo[r];
      if (tid < 4) slab[sh.s_bo + tid] = (tid < D) ? dbo : 0.f;
      // loss partials: wave sums, then across waves
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        float v = lacc[k];
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
        if (lane == 0) red[w * 8 + k] = v;
      }
      __syncthreads();
      if (tid < 8) {
        float v = 0.f;
        if (tid < 6)
          for (int q = 0; q < NWV; ++q) v += red[q * 8 + tid];
        slab[sh.s_loss + tid] = v;
      }
      __syncthreads();
    }
  }
  if (!args.counter) break;
  }
}


struct QueryLds { int S, NCOL, bufH, ys, xin, pidx, total; };
__host__ __device__ inline QueryLds query_lds(int D, int Wp, int NCB) {
  QueryLds L;
  L.NCOL = 16 * NCB;
  L.S = Wp + 4;
  int o = 0;
  L.bufH = o; o += (L.NCOL * L.S + 3) & ~3;
  L.ys = o;   o += (D * L.NCOL + 3) & ~3;
  L.xin = o;  o += (L.NCOL * D + 3) & ~3;
  L.pidx = o; o += L.NCOL;
  L.total = o;
  return L;
}

// forward of one staged tile (points in xin) through all layers; output in ys.
// Wave w computes row block w and row block w + NWV; one LDS
// stack, so every block's accumulators wait in registers until all waves have
// read the stack.
template <int DIM, int NCB, int MODE, int ACT>
__device__ __forceinline__ void forward_tile(const Shape& sh, const float* fr, float* bufH, float* ys,
                                             const float* xin, int S, int tid, int nthr, int w, int g,
                                             int j, int lane) {
  using M = ModeCfg<DIM, NCB, MODE>;
  const int Wp = sh.Wp, H = sh.H, K4 = sh.Kq >> 2, KT = sh.Kq & 3, NWV = sh.NWV;
  constexpr int RPW = 2;
  const int nrb = w + NWV < sh.NW ? 2 : 1;
  v4f acc[RPW][NCB];
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    if (r >= nrb) break;
    input_layer<DIM, NCB, MODE>(acc[r], fr + sh.f_w1, fr + sh.f_b, xin, w + r * NWV, g, j);
    act_forward<DIM, NCB, MODE, ACT>(acc[r]);
    store_fwd<NCB>(bufH, S, acc[r], w + r * NWV, g, j);
  }
  __syncthreads();
  for (int l = 2; l <= H; ++l) {
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      if (r >= nrb) break;
      const int rb = w + r * NWV;
      const float* Wf = fr + sh.f_hid + (size_t)(l - 2) * 2 * Wp * Wp + (size_t)rb * 16 * Wp;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) acc[r][cb] = zero4();
      gemm_rows<NCB>(Wf, bufH, S, K4, g, j, lane, acc[r], KT);
      add_bias<NCB, M::NPB>(acc[r], fr + sh.f_b + (l - 1) * Wp, rb, g);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      if (r >= nrb) break;
      act_forward<DIM, NCB, MODE, ACT>(acc[r]);
      store_fwd<NCB>(bufH, S, acc[r], w + r * NWV, g, j);
    }
    __syncthreads();
  }
  output_layer<DIM, NCB, MODE>(bufH, S, Wp, fr + sh.f_wo, fr + sh.f_bo, ys, tid, nthr);
  __syncthreads();
}

// SMALL: one 16-point block instead of CF column blocks (value mode); for
// requests too small to fill the chip (32,000 values of 6x224: 217 us, 330 with full tiles; 6x256: 254 and 370).
template <int DIM, int MODE, int ACT, int SMALL>
__global__ __launch_bounds__(512) void query_kernel(const QueryArgs a) {
  constexpr int D = DIM + 1, CF = 2 * DIM + 2;
  constexpr int NCB = SMALL ? 1 : CF;
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPTS = M::NPTS, NCOL = 16 * NCB;
  extern __shared__ float lds[];
  const Shape& sh = a.sh;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, w = tid >> 6, g = lane >> 4, j = lane & 15;
  const QueryLds L = query_lds(D, sh.Wp, NCB);
  float* bufH = lds + L.bufH;
  float* ys = lds + L.ys;
  float* xin = lds + L.xin;
  int32_t* pidx = reinterpret_cast<int32_t*>(lds + L.pidx);

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
    for (int k = tid; k < NCOL * D; k += nthr) {
      const int pt = k / D;
      float v = 0.f;
      if (pt < NPTS && pidx[pt] >= 0) v = a.x[(size_t)pidx[pt] * D + (k - pt * D)];
      xin[k] = v;
    }
    __syncthreads();
    forward_tile<DIM, NCB, MODE, ACT>(sh, a.subs[sub].frag, bufH, ys, xin, L.S, tid, nthr, w, g, j, lane);
    for (int k = tid; k < NPTS; k += nthr) {
      if (pidx[k] < 0) continue;
      const int64_t q = pidx[k];
      const int pb = k >> 4, jj = k & 15;
      auto Y = [&](int ch, int o) { return ys[o * NCOL + (ch * M::NPB + pb) * 16 + jj]; };
      if (a.what == Q_VALUE) {
        for (int o = 0; o < D; ++o) a.out[q * D + o] = Y(0, o);
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
// exchange: neighbour values at ghost points, anchor-normalised pressure
// ---------------------------------------------------------------------------
template <int DIM, int ACT>
__global__ __launch_bounds__(512) void exchange_kernel(const ExchangeArgs a) {
  constexpr int D = DIM + 1, CF = 2 * DIM + 2, NCB = CF, NCOL = 16 * NCB;
  extern __shared__ float lds[];
  const Shape& sh = a.sh;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, w = tid >> 6, g = lane >> 4, j = lane & 15;
  const QueryLds L = query_lds(D, sh.Wp, NCB);
  float* bufH = lds + L.bufH;
  float* ys = lds + L.ys;
  float* xin = lds + L.xin;
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
    forward_tile<DIM, NCB, M_VALUE, ACT>(sh, a.subs[it.b].frag, bufH, ys, xin, L.S, tid, nthr, w, g, j, lane);
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
// instances
// ---------------------------------------------------------------------------
int wide_step_lds_floats(const Shape& sh) {
  const int NCB = 2 * sh.dim + 2;
  return step_lds(sh.D, sh.Wp, sh.H, NCB).total;
}
int wide_query_lds_floats(const Shape& sh, int small) {
  return query_lds(sh.D, sh.Wp, small ? sh.dim + 1 : 2 * sh.dim + 2).total;
}

const void* wide_step_ptr(int act) {
  return act == ACT_SIN ? (const void*)step_kernel<3, ACT_SIN> : (const void*)step_kernel<3, ACT_TANH>;
}
const void* wide_query_ptr(int mode, int act, int small) {
  if (mode == M_VALUE) {
    if (small) return act == ACT_SIN ? (const void*)query_kernel<3, M_VALUE, ACT_SIN, 1> : (const void*)query_kernel<3, M_VALUE, ACT_TANH, 1>;
    return act == ACT_SIN ? (const void*)query_kernel<3, M_VALUE, ACT_SIN, 0> : (const void*)query_kernel<3, M_VALUE, ACT_TANH, 0>;
  }
  return act == ACT_SIN ? (const void*)query_kernel<3, M_PDE, ACT_SIN, 0> : (const void*)query_kernel<3, M_PDE, ACT_TANH, 0>;
}
const void* wide_exchange_ptr(int act) {
  return act == ACT_SIN ? (const void*)exchange_kernel<3, ACT_SIN> : (const void*)exchange_kernel<3, ACT_TANH>;
}

}  // namespace ddp
