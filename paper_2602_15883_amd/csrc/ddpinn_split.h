// Contractions over the hidden neurons and over a tile's columns on bf16
// matrix instructions, with fp32 inputs kept exactly.
//
// Every fp32 operand x is written as x = h + m + l with h = bf16(x),
// m = bf16(x - h), l = x - h - m (round to nearest even): 8 + 8 + 8 significand
// bits hold all 24 of x, so the split itself loses nothing (see Range).  Of the nine partial products
// the six of weight 2^-16 and above are formed, smallest first,
//   l.h, h.l, m.m, m.h, h.m, h.h,
// on v_mfma_f32_16x16x32_bf16 into one fp32 accumulator; the three left out
// (m.l, l.m, l.l) are below 2^-25 of the product.  One instruction adds 32
// products with one rounding of the accumulator, where the fp32 instruction
// (16x16x4) rounds for every four, so the result is closer to the exact sum than
// the fp32 instruction's: relative error (2-norm) 0.92e-7 against 1.44e-7 at
// K = 64, 1.5e-7 against 2.0e-7 at K = 128, 2.1e-7 against 2.7e-7 at K = 224
// (Gaussian weights times tanh values, against a 64-bit sum).  The rate on
// MI355X is 2207 / 6 = 368 TFLOP/s of fp32 products against 149 for the fp32
// instruction (both measured, all compute units).
//
// Range.  No operand is scaled.  The split is exact from 2^-110 in magnitude (below, a third part
// can be under bf16's smallest, 2^-133, and what is under it is lost: an absolute error of less than
// 2^-133 per operand, where fp32 holds down to 2^-149).  A weight is exact up to the largest fp32; of the
// other operands one above 2^128 - 2^119 (3.396e38), which rounds to a bf16 infinity, gives NaN, and so does any
// infinite operand (inf - inf in the split), where fp32 arithmetic might give an infinity or saturate.
//
// The kernels keep the operands of one side, the activations (or Zbar), in an LDS
// stack of parts, 6 bytes per value, and stream the weights as fragments.  A stack
// unit holds, for two blocks of 16, 64 slots of 16 bytes in lane order: slot (g, j) (g = lane / 16,
// j = lane % 16) at 16 g + (j ^ c(g)), c = 0, 12, 4, 8; the even block's 8 bytes (four bf16 of
// an accumulator fragment) come first for g = 0, 3 and second for g = 1, 2, so
// a result goes to LDS without any exchange between lanes.  LDS serves 16-byte reads
// 16 lanes at a time (of two lane groups g = 2k, 2k + 1: j in 0..3, 12..15 of one and 4..11
// of the other) and 8-byte ones 32 at a time; with this placement a read of a slot
// (ds_read_b128) and a transposing read (ds_read_b64_tr_b16) both touch every bank
// once.  Measured on one compute unit: 263 bytes/clock for the 16-byte reads and 248 for the
// transposing ones, against 138 for pairs of 8-byte reads from units of 512 bytes.
//
// Here: the queries and the exchange.  A wave owns R row blocks of 16 neurons; its
// accumulator fragment acc[r][cb] holds, in lane (g, j), neurons 4g + i (i = 0..3) of
// the row block and column 16 cb + j.  Two row blocks 2 kb, 2 kb + 1 (K block kb) share
// units, one per (kb, column block, part); a slot is then a lane's 8 K values of a contraction
// over neurons, and the weight fragments use the same order of neurons (k_neuron).
// The last row block of an odd number has units of 512 bytes, slot (g, j) of 8
// bytes at 16 g + (j ^ 4 g).  The training step has its tiles transposed (ddpinn_step.hip).
#pragma once
#include <type_traits>

#include "ddpinn_device.h"

namespace ddp {

typedef __bf16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v2h __attribute__((ext_vector_type(2)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
#define LDS_AS __attribute__((address_space(3)))

constexpr int kUnit = 512;            // bytes of a (row block, column block, part)
constexpr int kUnits3 = 3 * kUnit;    // the three parts of a (row block, column block)
constexpr int kFragFloats = 256;      // a weight fragment: 64 lanes x 8 bf16, in floats

// placement of lane group g's slots (see above)
__host__ __device__ __forceinline__ int slot_xor(int g) { return (0x84c0 >> (4 * g)) & 15; }   // 0, 12, 4, 8
__host__ __device__ __forceinline__ int slot_half(int g) { return (g == 1 || g == 2) ? 1 : 0; }
// neuron (within K block kb, 0..31) of K slot e of lane group g
__host__ __device__ __forceinline__ int k_neuron(int g, int e) { return 16 * ((e >> 2) ^ slot_half(g)) + 4 * g + (e & 3); }

// a lane's byte offsets within the units: 16-byte slots of a pair of row
// blocks, 8-byte slots of a row block that stands alone; plain and transposing
struct LaneSlots { uint32_t pair, half, alone, pair_tr, half_tr; };
__device__ __forceinline__ LaneSlots lane_slots(int lane) {
  const int g = lane >> 4, j = lane & 15;
  LaneSlots s;
  s.pair = (uint32_t)(16 * g + (j ^ slot_xor(g))) * 16u;
  s.half = (uint32_t)slot_half(g) * 8u;            // of the even row block; the odd one's is 8 - half
  s.alone = (uint32_t)(16 * g + (j ^ (4 * g))) * 8u;
  // transposing read: lane i of group gp fetches four values of the slot (i % 4, 4 gp +
  // i / 4) and receives value i of the slots' sixteen, for 4 gp .. 4 gp + 3
  const int col = 4 * g + ((lane >> 2) & 3), gq = lane & 3;
  s.pair_tr = (uint32_t)(16 * gq + (col ^ slot_xor(gq))) * 16u;
  s.half_tr = (uint32_t)slot_half(gq) * 8u;
  return s;
}

// two floats -> their bf16 (packed) and, in place, the remainders
__device__ __forceinline__ uint32_t split_step(float& a, float& b) {
  const v2h h = __builtin_convertvector(v2f{a, b}, v2h);
  const uint32_t u = __builtin_bit_cast(uint32_t, h);
  a -= __builtin_bit_cast(float, u << 16);
  b -= __builtin_bit_cast(float, u & 0xffff0000u);
  return u;
}
// The first step for the weight copies: a finite operand that would round to a bf16 infinity
// takes the largest bf16 instead (its remainder fits the other parts).
__device__ __forceinline__ uint32_t split_first(float& a, float& b) {
  constexpr float top = 0x1.fep+127f;
  float x = a > top ? top : a < -top ? -top : a, y = b > top ? top : b < -top ? -top : b;
  const float dx = a - x, dy = b - y;
  const uint32_t u = split_step(x, y);
  a = x + dx;
  b = y + dy;
  return u;
}
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const v2h h = __builtin_convertvector(v2f{a, b}, v2h);
  return __builtin_bit_cast(uint32_t, h);
}

// x = p[0] + p[1] + p[2], exactly
__device__ __forceinline__ void split4(v4f x, v2u (&p)[3]) {
  float a = x[0], b = x[1], c = x[2], d = x[3];
  p[0] = v2u{split_step(a, b), split_step(c, d)};
  p[1] = v2u{split_step(a, b), split_step(c, d)};
  p[2] = v2u{pack_bf16(a, b), pack_bf16(c, d)};
}

__device__ __forceinline__ v4f mfma32(v8h a, v8h b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ v4f mfma16(v4s a, v4s b, v4f c) {
  return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

// sum over the four lane groups, in every lane
__device__ __forceinline__ float group_sum(float v) {
  v += __shfl_xor(v, 16, 64);
  v += __shfl_xor(v, 32, 64);
  return v;
}

// parts of the two operands of the q-th product, smallest products first
__device__ constexpr int kPartA[6] = {2, 0, 1, 1, 0, 0};
__device__ constexpr int kPartB[6] = {0, 2, 1, 0, 1, 0};

// Row block rb of a stack of NW: byte offset of its first unit and the bytes from one
// (column block, part) to the next; alone: the last of an odd number.
template <int NCB>
__device__ __forceinline__ uint32_t stack_row(int rb, int NW, bool& alone) {
  alone = (NW & 1) && rb == NW - 1;
  return (uint32_t)((rb >> 1) * NCB * 2 * kUnits3);
}

// where a lane stores a row block: byte address of (column block 0, part 0), and
// the bytes from one (column block, part) to the next
template <int NCB>
__device__ __forceinline__ char* stack_row_slot(char* st, int rb, int NW, const LaneSlots& ls, bool& alone) {
  char* base = st + stack_row<NCB>(rb, NW, alone);
  return base + (alone ? ls.alone : ls.pair + ((rb & 1) ? 8u - ls.half : ls.half));
}
// one fragment (column block cb of the row block at base), split
template <int U>
__device__ __forceinline__ void stack_put(char* base, int cb, v4f v) {
  v2u p[3];
  split4(v, p);
#pragma unroll
  for (int q = 0; q < 3; ++q) *reinterpret_cast<v2u*>(base + (cb * 3 + q) * U) = p[q];
}

// one row block of a layer (fp32, accumulator order) into the LDS stack
template <int NCB>
__device__ __forceinline__ void stack_store_row(char* st, int rb, int NW, const LaneSlots& ls, const v4f (&a)[NCB]) {
  bool alone;
  char* base = stack_row_slot<NCB>(st, rb, NW, ls, alone);
  if (alone) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) stack_put<kUnit>(base, cb, a[cb]);
  } else {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) stack_put<2 * kUnit>(base, cb, a[cb]);
  }
}
template <int R, int NCB>
__device__ __forceinline__ void stack_store(char* st, int rb0, int NW, const LaneSlots& ls, const v4f (&a)[R][NCB]) {
#pragma unroll
  for (int r = 0; r < R; ++r) stack_store_row<NCB>(st, rb0 + r, NW, ls, a[r]);
}

// Weight fragments of the wave's row blocks for K block kb ([row block][K
// block][part][lane][8 bf16], KB = ceil(NW / 2) K blocks per row block).
// Memory operations complete in order, so a load issued after others (stores
// among them) waits for them too: the callers request the first fragments before the
// stores and the long-latency loads that precede their use.
template <int R>
struct Frags { v4f a[R][3]; };
template <int R>
__device__ __forceinline__ void load_frags(const float* wf, int KB, int kb, uint32_t lane16, Frags<R>& f) {
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int p = 0; p < 3; ++p) f.a[r][p] = ldg4u(wf + (size_t)((r * KB + kb) * 3 + p) * kFragFloats, lane16);
}

// stack operands of CG column blocks of one K block
template <int CG>
__device__ __forceinline__ void stack_operand(const char* sp, int c0, v8h (&b)[CG][3]) {
#pragma unroll
  for (int c = 0; c < CG; ++c)
#pragma unroll
    for (int p = 0; p < 3; ++p) b[c][p] = *reinterpret_cast<const v8h*>(sp + ((c0 + c) * 3 + p) * 2 * kUnit);
}

// the six products of one K block for CG column blocks from c0
template <int R, int NCB, int CG>
__device__ __forceinline__ void products32(const v4f (&a)[R][3], const v8h (&b)[CG][3], int c0, v4f (&acc)[R][NCB]) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int q = 0; q < 6; ++q) {
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
      for (int r = 0; r < R; ++r)
        acc[r][c0 + c] = mfma32(__builtin_bit_cast(v8h, a[r][kPartA[q]]), b[c][kPartB[q]], acc[r][c0 + c]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// a last K block of 16 neurons (sp: its units plus the lane's slot)
template <int R, int NCB, int CG>
__device__ __forceinline__ void products16(const v4f (&a)[R][3], const char* sp, v4f (&acc)[R][NCB]) {
#pragma unroll
  for (int c0 = 0; c0 < NCB; c0 += CG) {
    v4s b4[CG][3];
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
      for (int p = 0; p < 3; ++p) b4[c][p] = *reinterpret_cast<const v4s*>(sp + ((c0 + c) * 3 + p) * kUnit);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
#pragma unroll
      for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const v8s a8 = __builtin_bit_cast(v8s, a[r][kPartA[q]]);
          acc[r][c0 + c] = mfma16(__builtin_shufflevector(a8, a8, 0, 1, 2, 3), b4[c][kPartB[q]], acc[r][c0 + c]);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// acc[r][cb] = rows of the wave's row blocks of (weights x stack), K = all NW
// row blocks of the stack.  f: the weight fragments of the first K block; the next
// block's are requested before the products of the current one, and so are the
// stack operands of the next CG column blocks, one LDS read at a time between the products (a
// burst of them, which all waves issue at the same time, holds up the products
// behind it); nothing is copied between the two sets.  Residuals of 30,000 3D points,
// 8x128: 300 us with bursts, 289 so.
template <int R, int NCB>
__device__ __forceinline__ void gemm_neurons(const float* wf, const char* st, int NW, const LaneSlots& ls,
                                             uint32_t lane16, Frags<R>& f, v4f (&acc)[R][NCB]) {
  constexpr int CG = NCB % 2 == 0 ? 2 : 1;   // column blocks in flight
  constexpr int NG = NCB / CG;
  constexpr int kNext = NCB * 2 * kUnits3;   // bytes from one K block to the next
  const int KF = NW >> 1, KB = (NW + 1) >> 1;
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[r][cb] = zero4();
  const char* sp = st + ls.pair;
  v8h b[2][CG][3];
  if (KF > 0) stack_operand<CG>(sp, 0, b[0]);
  Frags<R> f2;
  auto block = [&](Frags<R>& cur, Frags<R>& nxt, int kb, auto par) {
    constexpr int P = NG & 1 ? decltype(par)::value : 0;
    uint32_t lo = lane16;
    asm volatile("" : "+v"(lo));   // (scalar bases)
    load_frags<R>(wf, KB, kb + 1 < KB ? kb + 1 : kb, lo, nxt);   // (the last one again at the end)
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      const int c0 = gi + 1 < NG ? (gi + 1) * CG : 0;
      if (gi + 1 == NG) sp += kb + 1 < KF ? kNext : 0;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int q = 0; q < 6; ++q) {
#pragma unroll
        for (int c = 0; c < CG; ++c)
#pragma unroll
          for (int r = 0; r < R; ++r)
            acc[r][gi * CG + c] = mfma32(__builtin_bit_cast(v8h, cur.a[r][kPartA[q]]), b[(gi + P) & 1][c][kPartB[q]], acc[r][gi * CG + c]);
        if (q < 3 * CG) {
          const int c = q % CG, p = kPartB[q / CG];
          b[(gi + 1 + P) & 1][c][p] = *reinterpret_cast<const v8h*>(sp + ((c0 + c) * 3 + p) * 2 * kUnit);
        }
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
  if (KF > 0) sp += kNext;
  if (NW & 1) products16<R, NCB, CG>(f.a, sp + ls.alone - ls.pair, acc);
}

// The same for one row block and few column blocks, with all the layer's weight
// fragments in f (KB <= NKB): for launches too small to cover the latency of
// fetching them as they are needed.
template <int NKB>
struct LayerFrags { v4f a[NKB][1][3]; };
template <int NKB>
__device__ __forceinline__ void load_layer(const float* wf, int KB, uint32_t lane16, LayerFrags<NKB>& f) {
#pragma unroll
  for (int k = 0; k < NKB; ++k)
    if (k < KB) {
#pragma unroll
      for (int p = 0; p < 3; ++p) f.a[k][0][p] = ldg4u(wf + (size_t)(k * 3 + p) * kFragFloats, lane16);
    }
}
template <int NCB, int NKB>
__device__ __forceinline__ void gemm_layer(const char* st, int NW, const LaneSlots& ls, const LayerFrags<NKB>& f,
                                           v4f (&acc)[1][NCB]) {
  const int KF = NW >> 1;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) acc[0][cb] = zero4();
#pragma unroll
  for (int kb = 0; kb < NKB; ++kb) {
    const char* sp = st + kb * NCB * 2 * kUnits3;
    if (kb < KF) {
      v8h b[NCB][3];
      stack_operand<NCB>(sp + ls.pair, 0, b);
      products32<1, NCB, NCB>(f.a[kb], b, 0, acc);
    } else if (kb == KF && (NW & 1)) {
      products16<1, NCB, NCB>(f.a[kb], sp + ls.alone, acc);
    }
  }
}

// Output layer: this wave's share of ys[o][col] = W_{H+1}[o] . h[col], one
// partial sum per lane group, into part[(4 w + g)][o][col] (LDS); the h of the
// last hidden layer never goes to LDS.
template <int D, int R, int NCB>
__device__ __forceinline__ void output_partials(float* part, const float* Wop, int Wp, int rb0, int w, int g, int j,
                                                const v4f (&a)[R][NCB]) {
  constexpr int NCOL = 16 * NCB;
#pragma unroll
  for (int o = 0; o < D; ++o) {
    v4f wo[R];
#pragma unroll
    for (int r = 0; r < R; ++r) wo[r] = ldg4(Wop + o * Wp + 16 * (rb0 + r) + 4 * g);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      float s = 0.f;
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) s = fmaf(wo[r][i], a[r][cb][i], s);
      part[((4 * w + g) * D + o) * NCOL + 16 * cb + j] = s;
    }
  }
}

// ys = sum of the waves' partials (in order), plus the bias on value columns
template <int DIM, int NCB, int MODE>
__device__ __forceinline__ void output_sum(const float* part, int n_part, const float* bop, float* ys, int tid,
                                           int nthr) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int D = DIM + 1, NCOL = 16 * NCB;
  for (int idx = tid; idx < D * NCOL; idx += nthr) {
    const int o = idx / NCOL, col = idx - o * NCOL;
    float s = 0.f;
    for (int q = 0; q < n_part; q += 4)
      s += (part[q * D * NCOL + idx] + part[(q + 1) * D * NCOL + idx]) +
           (part[(q + 2) * D * NCOL + idx] + part[(q + 3) * D * NCOL + idx]);
    if (col < 16 * M::NPB) s += ldg(bop + o);
    ys[idx] = s;
  }
}

// LDS of a query workgroup, in bytes.  The activation stack also takes, once
// the last hidden layer's products have read it, the output layer's partial
// sums (at most 1 KiB per row block and column block) and the outputs ys behind them.
// alone: one wave has all row blocks and needs neither stack nor partial sums.
struct SplitQueryLds { int part_floats, stack, ys, xin, pidx, total; };
__host__ __device__ inline SplitQueryLds split_query_lds(int D, int NW, int NWV, int NCB, bool alone) {
  SplitQueryLds L;
  const int NCOL = 16 * NCB;
  L.part_floats = alone ? 0 : 4 * NWV * D * NCOL;
  L.stack = 0;
  L.ys = 4 * L.part_floats;
  int o = alone ? 4 * D * NCOL : NW * NCB * kUnits3;
  L.xin = o;  o += 4 * NCOL * D;
  L.pidx = o; o += 4 * NCOL;
  L.total = o;
  return L;
}

// LDS of a step workgroup, in bytes.  ys holds the outputs, then (in place) the
// loss seeds ybar; it also takes the loss sums at the end of a segment and the
// index of the item range.
struct SplitStepLds { int ys, xin, total; };
__host__ __device__ inline SplitStepLds split_step_lds(int D, int NW, int NCB) {
  SplitStepLds L;
  const int NCOL = 16 * NCB;
  int o = NW * NCB * kUnits3;
  L.ys = o;  o += 4 * D * NCOL;
  L.xin = o; o += 4 * D * NCOL;
  L.total = o;
  return L;
}

// first row block of wave w: one each, and a second one for the first NW - NWV waves
__host__ __device__ __forceinline__ int split_rb0(int w, int NW, int NWV) { return w + (w < NW - NWV ? w : NW - NWV); }

}  // namespace ddp
