// The fused training step on bf16 matrix instructions with fp32 operands
// (ddpinn_split.h): forward with derivative channels, residuals, losses,
// adjoint and weight gradients of one tile of points after another.
//
// A workgroup of up to eight waves takes a tile through the whole step; a wave owns
// one row block of 16 neurons of every layer (two where there are more row blocks than waves)
// and all columns of the tile.
//
// What bounds it: the matrix units, whose clock the power limit sets (one 16x16x32 product
// takes 16 cycles, 6.8 ns on zeros and 8.2 to 9.9 ns on real values with all units busy),
// and the phases in which both waves of a SIMD are outside their products. 3D 8x128,
// 250,000 points: products 4.2 ms at 8.2 ns, measured 8.5 ms (fp32 matrix instructions 12.0
// ms); of its cycles 48 % hold a product, 33 % the issue of vector instructions.
// 3D 8x200 sin, 600,000 points: 104 -> 55 ms; 2D 8x100, 100,000: 3.20 -> 2.26 ms.
//
// Transposed tiles.  The activations enter the matrix instructions as the first
// operand and the weights as the second, so a wave's accumulator fragment
// acc[r][cb] holds, in lane (g, j) (g = lane / 16, j = lane % 16), neuron j of the
// row block and columns 16 cb + 4g + i (i = 0..3).  Every channel of a (neuron,
// point) pair sits in one lane, sums over a tile's columns stay in the lane (and
// the four groups), and, for the weight gradient
//   dW_l[m][n] = sum_col Zbar_l[m][col] H_{l-1}[n][col],
// a wave's own rows of H_{l-1}, split, are its operand as they lie in the registers.
// So only Zbar_l is in LDS in the backward (only H_{l-1} in the forward): one
// stack of 6 bytes per value, and two barriers per layer; between them a wave runs its
// recomputation of h, its share of dW and of Hbar_{l-1} = W_l^T Zbar_l and its adjoint on
// its own, so that one wave's vector work overlaps another's matrix work.
//
// The LDS stack.  Unit (row block, column blocks 2 kc and 2 kc + 1, part): 1 KiB,
// slot (g, j) of 16 bytes at 16 g + (j ^ c(g)): the lane's four columns of each of the two
// column blocks (the even one first for g = 0, 3, second for g = 1, 2).  A
// contraction over columns reads a slot as it lies (ds_read_b128); a contraction over neurons uses
// the transposing read (ds_read_b64_tr_b16), which gives a lane one column and four neurons, once per
// row block.
#include <type_traits>

#include "ddpinn_split.h"

namespace ddp {

__device__ __forceinline__ v4s lds_read_tr(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS v4s*)(const LDS_AS char*)p);
}

// byte offset of a unit from the stack's first
template <int NCB>
__device__ __forceinline__ constexpr int unit_at(int kc, int p) { return (3 * kc + p) * 2 * kUnit; }
template <int NCB>
struct Stack {
  static constexpr int kRow = NCB / 2 * 3 * 2 * kUnit;   // bytes of a row block
};

// A lane's byte offsets: where it stores its columns of an even and of an odd column
// block; its slot; and its transposing reads of the even and of the odd column
// block, of the two row blocks in the K order of the weight fragments
// (k_neuron: the odd row block first for lane groups 1 and 2) and of one alone.
struct StepSlots { uint32_t put[2], slot, tr[2][2], tr1[2]; };
template <int NCB>
__device__ __forceinline__ StepSlots step_slots(int lane) {
  const LaneSlots ls = lane_slots(lane);
  const int h = slot_half(lane >> 4);
  StepSlots s;
  s.slot = ls.pair;
  s.put[0] = ls.pair + ls.half;
  s.put[1] = ls.pair + 8u - ls.half;
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    s.tr1[o] = ls.pair_tr + (o ? 8u - ls.half_tr : ls.half_tr);
    s.tr[o][0] = s.tr1[o] + (uint32_t)(h ? Stack<NCB>::kRow : 0);
    s.tr[o][1] = s.tr1[o] + (uint32_t)(h ? 0 : Stack<NCB>::kRow);
  }
  return s;
}

// one fragment (column block cb), split, into the row block's units at st
template <int NCB>
__device__ __forceinline__ void put_cb(char* st, const StepSlots& ss, int cb, v4f v) {
  v2u p[3];
  split4(v, p);
#pragma unroll
  for (int q = 0; q < 3; ++q) *reinterpret_cast<v2u*>(st + ss.put[cb & 1] + unit_at<NCB>(cb >> 1, q)) = p[q];
}
template <int R, int NCB>
__device__ __forceinline__ void put_rows(char* st, const StepSlots& ss, const v4f (&a)[R][NCB]) {
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) put_cb<NCB>(st + r * Stack<NCB>::kRow, ss, cb, a[r][cb]);
}

// acc[r][cb] = (weights of the wave's row blocks) x (stack), transposed tile.  f: the weight
// fragments of the first K block; the next block's are requested before the
// products of the current one, into the other of two sets (copies between them would
// take issue slots from the products).
// One LDS read is issued behind each matrix instruction: a burst of the twelve of a
// pair of column blocks, which all waves issue at the same time, holds up the products behind it.
// 192 products per wave, two waves per SIMD (6,220 cycles of the matrix unit): bursts 8,170
// cycles, two reads every two products 7,500, one read behind each 7,020.
template <int R, int NCB>
__device__ __forceinline__ void gemm_neurons_t(const float* wf, const char* st, int NW, const StepSlots& ss,
                                               uint32_t lane16, Frags<R>& f, v4f (&acc)[R][NCB]) {
  constexpr int NC = NCB / 2;
  const int KF = NW >> 1, KB = (NW + 1) >> 1;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[r][cb] = zero4();
  const char* at[2][2];
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int h = 0; h < 2; ++h) at[o][h] = st + ss.tr[o][h];
  auto join = [](v4s lo, v4s hi) { return __builtin_bit_cast(v8h, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)); };
  v8h a[2][2][3];
  if (KF > 0) {
#pragma unroll
    for (int o = 0; o < 2; ++o)
#pragma unroll
      for (int p = 0; p < 3; ++p) a[0][o][p] = join(lds_read_tr(at[o][0] + unit_at<NCB>(0, p)), lds_read_tr(at[o][1] + unit_at<NCB>(0, p)));
  }
  Frags<R> f2;
  auto block = [&](Frags<R>& cur, Frags<R>& nxt, int kb, auto par) {
    constexpr int P = NC & 1 ? decltype(par)::value : 0;
    uint32_t lo = lane16;
    asm volatile("" : "+v"(lo));   // (scalar bases)
    load_frags<R>(wf, KB, kb + 1 < KB ? kb + 1 : kb, lo, nxt);   // (the last one again at the end)
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) {
      if (kc + 1 == NC) {
        // the next K block; from the last one back to the first
        const int step = kb + 1 < KF ? 2 * Stack<NCB>::kRow : -(KF - 1) * 2 * Stack<NCB>::kRow;
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
          for (int h = 0; h < 2; ++h) at[o][h] += step;
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        v4s lo, hi;
#pragma unroll
        for (int o = 0; o < 2; ++o) {
#pragma unroll
          for (int r = 0; r < R; ++r)
            acc[r][2 * kc + o] = mfma32(a[(kc + P) & 1][o][kPartB[q]], __builtin_bit_cast(v8h, cur.a[r][kPartA[q]]), acc[r][2 * kc + o]);
          (o ? hi : lo) = lds_read_tr(at[q & 1][o] + unit_at<NCB>(kc + 1 < NC ? kc + 1 : 0, kPartB[q >> 1]));
          __builtin_amdgcn_sched_barrier(0);
        }
        a[(kc + 1 + P) & 1][q & 1][kPartB[q >> 1]] = join(lo, hi);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  int kb = 0;
  for (; kb + 2 <= KF; kb += 2) {
    block(f, f2, kb, std::integral_constant<int, 0>{});
    block(f2, f, kb + 1, std::integral_constant<int, 1>{});
  }
  if (kb < KF) {
    block(f, f2, kb, std::integral_constant<int, 0>{});
    f = f2;
  }
  if (NW & 1) {   // a last K block of 16 neurons
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) {
      v4s a4[2][3];
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int p = 0; p < 3; ++p) a4[o][p] = lds_read_tr(st + KF * 2 * Stack<NCB>::kRow + ss.tr1[o] + unit_at<NCB>(kc, p));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 6; ++q) {
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const v8s w8 = __builtin_bit_cast(v8s, f.a[r][kPartA[q]]);
            acc[r][2 * kc + o] = mfma16(a4[o][kPartB[q]], __builtin_shufflevector(w8, w8, 0, 1, 2, 3), acc[r][2 * kc + o]);
          }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
}

// output layer: ys[o][col] = W_{H+1}[o] . h[col] (+ b_{H+1}[o] on value columns);
// column blocks in turn over the waves
template <int D, int NCB>
__device__ __forceinline__ void output_t(const float* wof, const char* st, int NW, const StepSlots& ss, uint32_t lane16,
                                         const float* bop, int nvb, float* ys, int w, int NWV, int g, int j) {
  constexpr int NCOL = 16 * NCB;
  const int KF = NW >> 1, KB = (NW + 1) >> 1;
  for (int cb = w; cb < NCB; cb += NWV) {
    const char* sc = st + unit_at<NCB>(cb >> 1, 0);
    const uint32_t t0 = cb & 1 ? ss.tr[1][0] : ss.tr[0][0], t1 = cb & 1 ? ss.tr[1][1] : ss.tr[0][1];
    v4f y = zero4();
    for (int kb = 0; kb < KB; ++kb, sc += 2 * Stack<NCB>::kRow) {
      Frags<1> f;
      load_frags<1>(wof, KB, kb, lane16, f);
      if (kb < KF) {
        v8h a[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const v4s lo = lds_read_tr(sc + t0 + unit_at<NCB>(0, p)), hi = lds_read_tr(sc + t1 + unit_at<NCB>(0, p));
          a[p] = __builtin_bit_cast(v8h, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) y = mfma32(a[kPartB[q]], __builtin_bit_cast(v8h, f.a[0][kPartA[q]]), y);
      } else {
        const uint32_t t = cb & 1 ? ss.tr1[1] : ss.tr1[0];
        v4s a[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) a[p] = lds_read_tr(sc + t + unit_at<NCB>(0, p));
#pragma unroll
        for (int q = 0; q < 6; ++q) {
          const v8s w8 = __builtin_bit_cast(v8s, f.a[0][kPartA[q]]);
          y = mfma16(a[kPartB[q]], __builtin_shufflevector(w8, w8, 0, 1, 2, 3), y);
        }
      }
    }
    if (j < D) {
      if (cb < nvb) y += ldg(bop + j);
      *reinterpret_cast<v4f*>(ys + j * NCOL + 16 * cb + 4 * g) = y;
    }
  }
}

// What the stash keeps of a layer, per row block: the pre-activations z_c of the
// derivative channels and, in place of z_0, what the derivatives of the activation at z_0
// are polynomials in: tanh(z_0), or sin(z_0) and, in further blocks, cos(z_0), so that neither is
// evaluated again in the backward.  Value tiles with sin keep z_0 itself (every
// column block is a value there).
template <int PBP, int ACT, int NCB>
struct Keep {
  static constexpr int kMore = ACT == ACT_SIN ? PBP : 0;
  static constexpr int kBlocks = NCB + kMore;   // 1 KiB wave fragments per row block
};

// the first three derivatives of the activation at z_0 of point block pb
template <int ACT, int NCB, int MODE, int NZ>
__device__ __forceinline__ void derivs(const v4f (&z)[NZ], int pb, v4f& s, v4f& s1, v4f& s2, v4f& s3) {
  if constexpr (ACT == ACT_SIN && MODE == M_PDE) {
    s = z[pb];
    s1 = z[NCB + pb];
    s2 = -s;
  } else {
    act4<ACT, true>(z[pb], s, s1, s2);
  }
  s3 = act_third<ACT>(s, s1);
}

// z -> h in place; keep(block, fragment) takes what the backward needs
template <int DIM, int NCB, int MODE, int ACT, typename F>
__device__ __forceinline__ void activate_row(v4f (&a)[NCB], F keep) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPB = M::NPB;
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    v4f s, s1, s2;
    act4<ACT>(a[pb], s, s1, s2);
    if constexpr (ACT == ACT_SIN && MODE == M_VALUE) keep(pb, a[pb]);
    else keep(pb, s);
    a[pb] = s;
    if constexpr (MODE == M_PDE) {
      if constexpr (ACT == ACT_SIN) keep(NCB + pb, s1);
#pragma unroll
      for (int jj = 0; jj <= DIM; ++jj) {
        const int c1 = (1 + jj) * NPB + pb, c2 = (DIM + 2 + jj) * NPB + pb;
        keep(c1, a[c1]);
        if (jj < DIM) {
          keep(c2, a[c2]);
          a[c2] = s2 * a[c1] * a[c1] + s1 * a[c2];
        }
        a[c1] *= s1;
      }
    }
  }
}

// Adjoint of activate_row: hb (dL/dh) -> dL/dz in place.
//   zbar_jj = s1 hbar_jj
//   zbar_j  = s1 hbar_j + 2 s2 z_j hbar_jj      (spatial j; time: s1 hbar_t)
//   zbar_0  = s1 hbar_0 + s2 sum_j z_j hbar_j + sum_j (s3 z_j^2 + s2 z_jj) hbar_jj
template <int DIM, int NCB, int MODE, int ACT, int NZ>
__device__ __forceinline__ void adjoint_row(v4f (&hb)[NCB], const v4f (&z)[NZ]) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPB = M::NPB;
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    v4f s, s1, s2, s3;
    derivs<ACT, NCB, MODE>(z, pb, s, s1, s2, s3);
    v4f z0 = s1 * hb[pb];
    if constexpr (MODE == M_PDE) {
#pragma unroll
      for (int jj = 0; jj <= DIM; ++jj) {
        const int c1 = (1 + jj) * NPB + pb, c2 = (DIM + 2 + jj) * NPB + pb;
        const v4f h1 = hb[c1], z1 = z[c1];
        z0 += s2 * z1 * h1;
        hb[c1] = s1 * h1;
        if (jj < DIM) {
          const v4f h2 = hb[c2];
          hb[c2] = s1 * h2;
          hb[c1] += 2.f * s2 * z1 * h2;
          z0 += (s3 * z1 * z1 + s2 * z[c2]) * h2;
        }
      }
    }
    hb[pb] = z0;
  }
}

// h of the kept values, split, as the operand of a contraction over columns; a
// pair of column blocks at a time
template <int DIM, int NCB, int MODE, int ACT, int NZ>
__device__ __forceinline__ void h_operand(const v4f (&z)[NZ], bool swap, v8h (&ha)[NCB / 2][3]) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPB = M::NPB;
  v4f s1[NPB], s2[NPB];   // (value mode: unused)
  auto h_of = [&](int cb) -> v4f {
    const int c = cb / NPB, pb = cb - c * NPB;
    if (c == 0) {
      v4f s, a1, a2, a3;
      derivs<ACT, NCB, MODE>(z, pb, s, a1, a2, a3);
      if constexpr (MODE == M_PDE) {
        s1[pb] = a1;
        s2[pb] = a2;
      }
      return s;
    }
    if constexpr (MODE == M_PDE) {
      if (c <= DIM + 1) return s1[pb] * z[cb];
      const v4f z1 = z[(c - DIM - 1) * NPB + pb];
      return s2[pb] * z1 * z1 + s1[pb] * z[cb];
    }
    return zero4();
  };
#pragma unroll
  for (int kc = 0; kc < NCB / 2; ++kc) {
    v2u e[3], o[3];
    split4(h_of(2 * kc), e);
    split4(h_of(2 * kc + 1), o);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      typedef uint32_t v4u __attribute__((ext_vector_type(4)));
      const v4u u = {swap ? o[p][0] : e[p][0], swap ? o[p][1] : e[p][1], swap ? e[p][0] : o[p][0], swap ? e[p][1] : o[p][1]};
      ha[kc][p] = __builtin_bit_cast(v8h, u);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// dW of one row block n of H (ha) against two row blocks m of Zbar at a time, added to the slab (sw:
// tiles [NW][64 lanes][4] of row block n; lane (g, j): neuron 4g + i of n, neuron
// j of m).  The old slab values are requested before the products they are added to; one LDS
// read behind every two products (192 of them, two waves per SIMD: 8,120 cycles with
// the reads of a column pair in a burst, 7,610 so).
template <int NCB>
__device__ __forceinline__ void gemm_columns_t(const v8h (&ha)[NCB / 2][3], const char* st, int NW, const StepSlots& ss,
                                               uint32_t lane16, float* sw, bool first) {
  constexpr int NC = NCB / 2;
  const char* base = st + ss.slot;
  v8h b[2][2][3];
  auto read = [&](const char* row, int kc, int t, int p) {
    return *reinterpret_cast<const v8h*>(row + t * Stack<NCB>::kRow + unit_at<NCB>(kc, p));
  };
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int p = 0; p < 3; ++p) b[0][t][p] = read(NW > 1 ? base : base - t * Stack<NCB>::kRow, 0, t, p);
  auto pair = [&](int mb, auto par) {
    constexpr int P = NC & 1 ? decltype(par)::value : 0;
    uint32_t lo = lane16;
    asm volatile("" : "+v"(lo));   // (scalar bases)
    v4f old[2], dw[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) old[t] = first ? zero4() : ldg4u(sw + (size_t)(mb + t) * 256, lo);
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) {
      // the next pair; past the last one the last two row blocks (an odd last one is done from them)
      const char* nx = kc + 1 < NC ? base : base + (mb + 4 <= NW ? 2 : NW - 2 - mb) * Stack<NCB>::kRow;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 6; ++q) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
          dw[t] = mfma32(ha[kc][kPartA[q]], b[(kc + P) & 1][t][kPartB[q]], (kc == 0 && q == 0) ? zero4() : dw[t]);
        b[(kc + 1 + P) & 1][q & 1][kPartB[q >> 1]] = read(nx, kc + 1 < NC ? kc + 1 : 0, q & 1, kPartB[q >> 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) stg4u(sw + (size_t)(mb + t) * 256, lo, old[t] + dw[t]);
    base += (mb + 4 <= NW ? 2 : NW - 2 - mb) * Stack<NCB>::kRow;
  };
  int mb = 0;
  for (; mb + 4 <= NW; mb += 4) {
    pair(mb, std::integral_constant<int, 0>{});
    pair(mb + 2, std::integral_constant<int, 1>{});
  }
  if (mb + 2 <= NW) {
    pair(mb, std::integral_constant<int, 0>{});
    mb += 2;
  }
  if (mb < NW) {   // an odd last row block
    const char* row = st + ss.slot + mb * Stack<NCB>::kRow;
    const v4f old = first ? zero4() : ldg4u(sw + (size_t)mb * 256, lane16);
    v4f dw = zero4();
#pragma unroll
    for (int kc = 0; kc < NC; ++kc) {
      v8h c[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) c[p] = read(row, kc, 0, p);
#pragma unroll
      for (int q = 0; q < 6; ++q) dw = mfma32(ha[kc][kPartA[q]], c[kPartB[q]], dw);
    }
    stg4u(sw + (size_t)mb * 256, lane16, old + dw);
  }
}

// input layer: z0 = W1 xi + b1 and the seeded channels, transposed tile
template <int DIM, int NCB, int MODE>
__device__ __forceinline__ void input_layer_t(v4f (&a)[NCB], const float* __restrict__ W1p,
                                              const float* __restrict__ b1p, const float* xin, int rb, int g, int j) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int D = DIM + 1, NPB = M::NPB;
  const int r = 16 * rb + j;
  float wr[D];
#pragma unroll
  for (int q = 0; q < D; ++q) wr[q] = ldg(W1p + r * D + q);
  const float br = ldg(b1p + r);
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float* xp = xin + (16 * pb + 4 * g + i) * D;
      float z = br;
#pragma unroll
      for (int q = 0; q < D; ++q) z += wr[q] * xp[q];
      a[pb][i] = z;
    }
    if constexpr (MODE == M_PDE) {
#pragma unroll
      for (int jj = 0; jj <= DIM; ++jj) a[(1 + jj) * NPB + pb] = v4f{wr[jj], wr[jj], wr[jj], wr[jj]};
#pragma unroll
      for (int jj = 0; jj < DIM; ++jj) a[(DIM + 2 + jj) * NPB + pb] = zero4();
    }
  }
}

// one tile after another of this workgroup's item ranges, for a wave of R row blocks
template <int DIM, int PBP, int ACT, int R, int WIDE>
__device__ __forceinline__ void step_tiles(const StepArgs& args, char* lds, int rb0, int w) {
  constexpr int D = DIM + 1;
  constexpr int CF = 2 * DIM + 2;
  constexpr int NCB = CF * PBP;
  constexpr int NCOL = 16 * NCB;
  using MP = ModeCfg<DIM, NCB, M_PDE>;
  using MV = ModeCfg<DIM, NCB, M_VALUE>;
  constexpr int NZ = Keep<PBP, ACT, NCB>::kBlocks;
  // one row block and tanh: layer H's values stay in registers, not in the stash
  constexpr bool KEEP_H = R == 1 && ACT == ACT_TANH;

  const Shape& sh = args.sh;
  const int Wp = sh.Wp, NW = sh.NW, H = sh.H, KB = (NW + 1) >> 1;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, g = lane >> 4, j = lane & 15;
  // Byte offsets of the lane's memory accesses, on top of wave-uniform bases.
  // fresh() hides their values from loop-invariant code motion, which would otherwise keep
  // a 64-bit address per access in registers for the whole loop, and spill them.
  uint32_t lane16 = (uint32_t)lane * 16u, j4 = (uint32_t)j * 4u;
  auto fresh = [&] { asm volatile("" : "+v"(lane16), "+v"(j4)); };
  const StepSlots ss = step_slots<NCB>(lane);
  const bool swap = slot_half(g);
  const SplitStepLds L = split_step_lds(D, NW, NCB);
  float* ys = reinterpret_cast<float*>(lds + L.ys);
  float* xin = reinterpret_cast<float*>(lds + L.xin);
  char* mine = lds + rb0 * Stack<NCB>::kRow;   // the wave's row blocks in the stack
  // dW row blocks of the wave: its own, but some second ones go to a wave with one block on
  // another SIMD (wave v is on SIMD v mod 4).  Of ne = NW - NWS waves with two blocks, ne mod 4
  // leave the SIMDs uneven; the second blocks of the first 1, 2, 1 of those 1, 2, 3
  // waves move by as many waves.  Ten row blocks: 5 of them per SIMD between two
  // barriers of the backward (Hbar and dW), instead of 6, 6, 4, 4; 2D 6x150 sin, 500,000 points:
  // 15.5 -> 14.8 ms.
  int dw2 = R > 1 ? rb0 + 1 : -1;   // the second dW row block, or none
  if constexpr (WIDE) {
    const int ne = NW - sh.NWS, m = ne & 3, n_move = m == 2 ? 2 : m ? 1 : 0;
    const int v = R > 1 ? w : w - m;   // the wave whose second block it is about
    if (v >= ne - m && v < ne - m + n_move) dw2 = R > 1 ? -1 : split_rb0(v, NW, sh.NWS) + 1;
  }
  // stash: (layer, row block, block), 1 KiB wave fragments
  float* stash = args.stash + (size_t)blockIdx.x * args.stash_per_wg + (size_t)rb0 * NZ * 256;
  const size_t stash_l = (size_t)NW * NZ * 256;
  const float nu = args.nu;
  const bool prio = args.prio != 0;   // favour a wave in its matrix phases over one in its vector phases

  float lacc[6], dbo = 0.f;

  int* s_range = reinterpret_cast<int*>(ys);
  int range = blockIdx.x;
  for (;;) {
    if (args.counter) {
      // ranges in turn: co-resident workgroups do not progress at the same rate
      __syncthreads();
      if (tid == 0) *s_range = atomicAdd(args.counter, 1);
      __syncthreads();
      range = __builtin_amdgcn_readfirstlane(*s_range);
    }
    if (range >= args.n_ranges) break;
    const int it0 = ((const CONST_AS int32_t*)args.wg_begin)[range];
    const int it1 = ((const CONST_AS int32_t*)args.wg_begin)[range + 1];
    for (int it = it0; it < it1; ++it) {
      __syncthreads();   // the previous tile's readers of xin, ys and the stack are done
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
      const float* bp = fr + sh.f_b;
      const float* Wop = fr + sh.f_wo;
      const bool pde = item.kind == ITEM_PDE;
      const bool first = item.flags & ITEM_FIRST;
      float* slab = args.slabs + (size_t)item.slab * sh.slab_floats;

      if (first) {
#pragma unroll
        for (int k = 0; k < 6; ++k) lacc[k] = 0.f;
        dbo = 0.f;
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

      // ---- forward
      fresh();
      v4f acc[R][NCB];
      const int nvb = pde ? MP::NPB : MV::NPB;   // value-channel column blocks
      // z_l in acc -> h_l, and what the backward needs of z_l into the stash
      auto activate = [&](int l) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          float* st = stash + (size_t)(l - 1) * stash_l + (size_t)r * NZ * 256;
          auto keep = [&](int b, v4f v) { stg4u(st + b * 256, lane16, v); };
          if (pde) activate_row<DIM, NCB, M_PDE, ACT>(acc[r], keep);
          else activate_row<DIM, NCB, M_VALUE, ACT>(acc[r], keep);
        }
      };
      v4f zl[KEEP_H ? NZ : 1];   // of layer H
      auto activate_last = [&] {
        if constexpr (KEEP_H) {
          auto keep = [&](int b, v4f v) { zl[b] = v; };
          if (pde) activate_row<DIM, NCB, M_PDE, ACT>(acc[0], keep);
          else activate_row<DIM, NCB, M_VALUE, ACT>(acc[0], keep);
        } else {
          activate(H);
        }
      };
      const float* wf = fr + sh.f_hid3 + (size_t)rb0 * KB * 3 * kFragFloats;   // of W_2
      Frags<R> f;   // weight fragments and bias of the next contraction over neurons
      float bias[R];
      auto load_bias = [&](int l) {
#pragma unroll
        for (int r = 0; r < R; ++r) bias[r] = ldgu(bp + (l - 1) * Wp + 16 * (rb0 + r), j4);
      };
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (pde) input_layer_t<DIM, NCB, M_PDE>(acc[r], fr + sh.f_w1, bp, xin, rb0 + r, g, j);
        else input_layer_t<DIM, NCB, M_VALUE>(acc[r], fr + sh.f_w1, bp, xin, rb0 + r, g, j);
      }
      if (H > 1) {
        load_frags<R>(wf, KB, 0, lane16, f);
        load_bias(2);
        activate(1);
      } else {
        activate_last();
      }
      for (int l = 2; l <= H; ++l) {
        fresh();
        put_rows<R, NCB>(mine, ss, acc);
        __syncthreads();
        if (prio) __builtin_amdgcn_s_setprio(1);
        gemm_neurons_t<R, NCB>(wf + (size_t)(l - 2) * sh.hid3_layer, lds, NW, ss, lane16, f, acc);
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
            if (cb < nvb) acc[r][cb] += bias[r];
        if (l < H) {
          load_frags<R>(wf + (size_t)(l - 1) * sh.hid3_layer, KB, 0, lane16, f);
          load_bias(l + 1);
          activate(l);
        } else {
          activate_last();
        }
        __syncthreads();
      }

      // ---- output layer
      put_rows<R, NCB>(mine, ss, acc);
      __syncthreads();
      output_t<D, NCB>(fr + sh.f_wo3, lds, NW, ss, lane16, fr + sh.f_bo, nvb, ys, w, sh.NWS, g, j);
      __syncthreads();

      // ---- residuals, losses and output seeds ybar = dL/dy, in place of y
      // (every column belongs to one thread)
      if (pde) {
        if (tid < MP::NPTS) {
          const int pb = tid >> 4, jj = tid & 15;
          auto at = [&](int c, int o) -> float& { return ys[o * NCOL + (c * MP::NPB + pb) * 16 + jj]; };
          float y[CF][D];
#pragma unroll
          for (int c = 0; c < CF; ++c)
#pragma unroll
            for (int o = 0; o < D; ++o) y[c][o] = at(c, o);
          auto Y = [&](int c, int o) { return y[c][o]; };
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
#pragma unroll
          for (int i = 0; i < DIM; ++i) {
            float s = 0.f;
#pragma unroll
            for (int k = 0; k < DIM; ++k) s += rb[k] * Y(1 + i, k);
            at(0, i) = s;                                                    // u_i
#pragma unroll
            for (int jx = 0; jx < DIM; ++jx) {
              at(1 + jx, i) = rb[i] * Y(0, jx) + (i == jx ? rb[DIM] : 0.f);  // d_j u_i
              at(DIM + 2 + jx, i) = -nu * rb[i];                             // d_jj u_i
            }
            at(1 + DIM, i) = rb[i];                                          // d_t u_i
          }
          at(0, DIM) = 0.f;                                                  // p
#pragma unroll
          for (int jx = 0; jx < DIM; ++jx) {
            at(1 + jx, DIM) = rb[jx];                                        // d_j p
            at(DIM + 2 + jx, DIM) = 0.f;
          }
          at(1 + DIM, DIM) = 0.f;
        }
      } else {
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
          for (int o = 0; o < D; ++o) ys[o * NCOL + col] = e[o];
        }
      }
      __syncthreads();

      // ---- output layer adjoint: dW_{H+1} (h_H is in acc), db_{H+1}, hbar_H.
      // The small gradients (dW_{H+1}, db_l, dW_1) are summed over the tile's
      // columns and added to the slab by the lanes g = 0.
      {
        float* so = slab + sh.s_wo + 16 * rb0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          v4f hb[NCB];
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) hb[cb] = zero4();
#pragma unroll(WIDE ? 1 : D)   // (unrolled, ys is read for all outputs at once: with two row blocks, registers spill)
          for (int o = 0; o < D; ++o) {
            const float old = (g == 0 && !first) ? ldgu(so + o * Wp + 16 * r, j4) : 0.f;
            const float wo = ldgu(Wop + o * Wp + 16 * (rb0 + r), j4);
            float s = 0.f, b = 0.f;
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
              const v4f yv = *reinterpret_cast<const v4f*>(ys + o * NCOL + 16 * cb + 4 * g);
              if (r == 0 && cb < nvb) b += (yv[0] + yv[1]) + (yv[2] + yv[3]);
              s += (yv[0] * acc[r][cb][0] + yv[1] * acc[r][cb][1]) + (yv[2] * acc[r][cb][2] + yv[3] * acc[r][cb][3]);
              hb[cb] += wo * yv;
            }
            s = group_sum(s);
            if (g == 0) stgu(so + o * Wp + 16 * r, j4, old + s);
            if (r == 0) {
              b = group_sum(b);
              if (tid == o) dbo += b;
              asm volatile("" : "+v"(dbo));   // now: its terms would be kept until the tile's end
            }
          }
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) acc[r][cb] = hb[cb];
        }
      }
      auto load_z = [&](int l, int r, v4f (&z)[NZ]) {   // of layer l, row block rb0 + r
        const float* st = stash + (ptrdiff_t)(l - 1) * (ptrdiff_t)stash_l + (ptrdiff_t)r * NZ * 256;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) z[cb] = ldg4u(st + cb * 256, lane16);
#pragma unroll
        for (int cb = NCB; cb < NZ; ++cb)
          if (pde) z[cb] = ldg4u(st + cb * 256, lane16);
      };
      // adjoint of layer l, row block r: acc[r] = hbar_l -> zbar_l; db_l and, at l = 1, dW_1
      auto adjoint = [&](int l, int r, const v4f (&z)[NZ]) {
        float* sb = slab + sh.s_b + (size_t)(l - 1) * Wp + 16 * (rb0 + r);
        const float old = (g == 0 && !first) ? ldgu(sb, j4) : 0.f;
        if (pde) adjoint_row<DIM, NCB, M_PDE, ACT>(acc[r], z);
        else adjoint_row<DIM, NCB, M_VALUE, ACT>(acc[r], z);
        float s = 0.f;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          if (cb < nvb) s += (acc[r][cb][0] + acc[r][cb][1]) + (acc[r][cb][2] + acc[r][cb][3]);
        s = group_sum(s);
        if (g == 0) stgu(sb, j4, old + s);
        if (l > 1) return;
        // dW1[n][q] += sum_pts zbar0 xi_q + zbar_q (first-derivative channel q)
        float* s1 = slab + sh.s_w1 + (size_t)(16 * (rb0 + r)) * D;
        float v[D];
#pragma unroll
        for (int q = 0; q < D; ++q) v[q] = 0.f;
        if (pde) {
#pragma unroll
          for (int pb = 0; pb < MP::NPB; ++pb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float* xp = xin + (16 * pb + 4 * g + i) * D;
#pragma unroll
              for (int q = 0; q < D; ++q) v[q] += acc[r][pb][i] * xp[q] + acc[r][(1 + q) * MP::NPB + pb][i];
            }
        } else {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float* xp = xin + (16 * cb + 4 * g + i) * D;
#pragma unroll
              for (int q = 0; q < D; ++q) v[q] += acc[r][cb][i] * xp[q];
            }
        }
#pragma unroll
        for (int q = 0; q < D; ++q) {
          const float t = group_sum(v[q]);
          if (g == 0) stgu(s1 + q, j4 * D, (first ? 0.f : ldgu(s1 + q, j4 * D)) + t);
        }
      };
      if constexpr (KEEP_H) {
        adjoint(H, 0, zl);
      } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          v4f z[NZ];
          load_z(H, r, z);
          adjoint(H, r, z);
        }
      }

      // ---- hidden layer adjoints
      const float* wt = wf + sh.hid3_layer / 2;   // of W_2^T
      for (int l = H; l >= 2; --l) {
        fresh();
        // loads ahead of the barriers: z_{l-1} (of the first row block) and weights
        v4f z[NZ];
        load_z(l - 1, 0, z);
        __syncthreads();   // every reader of the stack (layer l + 1; the output layer) is done
        put_rows<R, NCB>(mine, ss, acc);
        __syncthreads();
        load_frags<R>(wt + (size_t)(l - 2) * sh.hid3_layer, KB, 0, lane16, f);
        for (int n = rb0; n >= 0;) {
          v8h ha[NCB / 2][3];
          if (pde) h_operand<DIM, NCB, M_PDE, ACT>(z, swap, ha);
          else h_operand<DIM, NCB, M_VALUE, ACT>(z, swap, ha);
          const int next = WIDE && n == rb0 ? dw2 : -1;
          if (WIDE && dw2 >= 0) load_z(l - 1, next >= 0 ? next - rb0 : 0, z);   // of the next one, at last again of the first
          if (prio) __builtin_amdgcn_s_setprio(1);
          gemm_columns_t<NCB>(ha, lds, NW, ss, lane16,
                              slab + sh.s_hid + (size_t)(l - 2) * Wp * Wp + (size_t)n * NW * 256, first);
          __builtin_amdgcn_s_setprio(0);
          if (!WIDE) break;
          n = next;
        }
        if (prio) __builtin_amdgcn_s_setprio(1);
        gemm_neurons_t<R, NCB>(wt + (size_t)(l - 2) * sh.hid3_layer, lds, NW, ss, lane16, f, acc);   // Hbar_{l-1}
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (r > 0) load_z(l - 1, r, z);
          adjoint(l - 1, r, z);
        }
      }

      // ---- end of segment: output bias gradient and loss sums
      if (item.flags & ITEM_LAST) {
        __syncthreads();
        if (tid < 4) slab[sh.s_bo + tid] = (tid < D) ? dbo : 0.f;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          float v = lacc[k];
          for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
          if (lane == 0) ys[w * 8 + k] = v;
        }
        __syncthreads();
        if (tid < 8) {
          float v = 0.f;
          if (tid < 6)
            for (int q = 0; q < sh.NWS; ++q) v += ys[q * 8 + tid];
          slab[sh.s_loss + tid] = v;
        }
      }
    }
    if (!args.counter) break;
  }
}

// Two waves per SIMD (256 registers each); the 32-point tiles have twice the
// columns and at most four waves, one per SIMD.  WIDE: fewer waves than row blocks (the first
// NW - NWS of them own two): above 128 neurons, and workgroups of four waves,
// two per compute unit.
template <int DIM, int PBP, int ACT, int WIDE>
__global__ __launch_bounds__(PBP == 1 ? 512 : 256, PBP == 1 ? 2 : 1) void split_step_kernel(const StepArgs args) {
  extern __shared__ __align__(16) char slds[];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if constexpr (WIDE) {
    const int rb0 = split_rb0(w, args.sh.NW, args.sh.NWS);
    // both branches meet the same barriers
    if (w < args.sh.NW - args.sh.NWS) step_tiles<DIM, PBP, ACT, 2, 1>(args, slds, rb0, w);
    else step_tiles<DIM, PBP, ACT, 1, 1>(args, slds, rb0, w);
  } else {
    step_tiles<DIM, PBP, ACT, 1, 0>(args, slds, w, w);
  }
}

// ---------------------------------------------------------------------------
// instances: one dimension and activation per translation unit
// ---------------------------------------------------------------------------
template <int DIM, int ACT>
const void* split_step_ptr(int tile_points, int NW, int NWS) {
  if (tile_points == 32) return NW <= 4 ? (const void*)split_step_kernel<DIM, 2, ACT, 0> : nullptr;
  return NW > NWS ? (const void*)split_step_kernel<DIM, 1, ACT, 1> : (const void*)split_step_kernel<DIM, 1, ACT, 0>;
}
template const void* split_step_ptr<DDP_DIM, DDP_ACT>(int, int, int);

}  // namespace ddp
