// The fused training step on bf16 matrix instructions with fp32 operands
// (ddpinn_split.h): forward with derivative channels, residuals, losses,
// adjoint and weight gradients of one tile of points after another.
//
// A workgroup of up to four waves takes a tile through the whole step; wave w owns
// the row blocks [rb0(w), rb0(w+1)) of every layer (two per wave up to 128
// neurons, three or four above), all columns of the tile.  Two row blocks per
// wave halve what the waves read from LDS against one: at one row block the LDS
// reads of a contraction take as long as its matrix instructions, at two half as
// long.  One activation stack is in LDS at a time:
//   forward, layer l:   H_{l-1} -> Z_l = W_l H_{l-1} -> chain rule -> H_l
//   backward, layer l:  Zbar_l  -> Hbar_{l-1} = W_l^T Zbar_l; every wave keeps the
//                       operand fragments of its own Zbar_l rows in registers
//                       H_{l-1} -> dW_l = Zbar_l H_{l-1}^T
// so that the stack (6 bytes per value: 73 KiB for a 2D tile at 128 neurons, 96 KiB in 3D) leaves room
// for two workgroups per compute unit in 2D, whose matrix and vector phases then
// overlap.
#include <type_traits>

#include "ddpinn_split.h"

namespace ddp {

// sum over the 16 lanes of a lane group, in every lane
__device__ __forceinline__ float row_sum(float v) {
  auto rot = [](float x, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value,
                                                                 0xf, 0xf, false));
  };
  v += rot(v, std::integral_constant<int, 0x128>{});   // row_ror:8
  v += rot(v, std::integral_constant<int, 0x124>{});
  v += rot(v, std::integral_constant<int, 0x122>{});
  v += rot(v, std::integral_constant<int, 0x121>{});
  return v;
}
__device__ __forceinline__ v4f row_sum4(v4f v) { return v4f{row_sum(v[0]), row_sum(v[1]), row_sum(v[2]), row_sum(v[3])}; }

__device__ __forceinline__ v4s lds_read_tr(const char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS v4s*)(const LDS_AS char*)p);
}

// operand of a contraction over columns: one row block, column blocks 2 kc and
// 2 kc + 1, one part; p: the unit of column block 2 kc plus the lane's slot,
// stride: bytes from one column block's unit to the next
__device__ __forceinline__ v8h col_operand(const char* p, int stride) {
  const v4s lo = lds_read_tr(p), hi = lds_read_tr(p + stride);
  return __builtin_bit_cast(v8h, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// the wave's own row blocks of the stack as operands of a contraction over columns
template <int R, int NCB>
__device__ __forceinline__ void own_operands(const char* st, int rb0, int NW, const LaneSlots& ls, v8h (&za)[R][NCB / 2][3]) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    bool alone;
    const char* base = st + stack_row<NCB>(rb0 + r, NW, alone);
    base += alone ? ls.alone_tr : ls.pair_tr + (((rb0 + r) & 1) ? 8u - ls.half_tr : ls.half_tr);
    const int u = alone ? kUnit : 2 * kUnit;
#pragma unroll
    for (int kc = 0; kc < NCB / 2; ++kc)
#pragma unroll
      for (int p = 0; p < 3; ++p) za[r][kc][p] = col_operand(base + (6 * kc + p) * u, 3 * u);
  }
}

// dw = the wave's dW rows times NT row blocks of H (base[t]: their units), over the
// tile's columns
template <int R, int NCB, int NT, int U>
__device__ __forceinline__ void dw_group(const v8h (&za)[R][NCB / 2][3], const char* const (&base)[NT], v4f (&dw)[R][NT]) {
#pragma unroll
  for (int kc = 0; kc < NCB / 2; ++kc) {
    v8h b[NT][3];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int p = 0; p < 3; ++p) b[t][p] = col_operand(base[t] + (6 * kc + p) * U, 3 * U);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < R; ++r)
          dw[r][t] = mfma32(za[r][kc][kPartA[q]], b[t][kPartB[q]], (kc == 0 && q == 0) ? zero4() : dw[r][t]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// dW of the wave's row blocks, two column blocks (row blocks of H) at a time, added
// to the slab (sw: tiles [row block][NW][64 lanes][4] from the wave's first row
// block); the old slab values are requested before the products they are added to
template <int R, int NCB>
__device__ __forceinline__ void gemm_columns(const v8h (&za)[R][NCB / 2][3], const char* st, int NW, const LaneSlots& ls,
                                             uint32_t lane16, float* sw, bool first) {
  constexpr int kNext = NCB * 2 * kUnits3;
  auto add = [&](int nb, auto nt, auto unit, const char* const (&base)[decltype(nt)::value]) {
    constexpr int NT = decltype(nt)::value;
    v4f old[R][NT], dw[R][NT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) old[r][t] = first ? zero4() : ldg4u(sw + (size_t)(r * NW + nb + t) * 256, lane16);
    dw_group<R, NCB, NT, decltype(unit)::value>(za, base, dw);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) stg4u(sw + (size_t)(r * NW + nb + t) * 256, lane16, old[r][t] + dw[r][t]);
  };
  const char* base[2] = {st + ls.pair_tr + ls.half_tr, st + ls.pair_tr + 8 - ls.half_tr};
  int nb = 0;
  for (; nb + 2 <= NW; nb += 2) {
    const char* const bt[2] = {base[0], base[1]};
    add(nb, std::integral_constant<int, 2>{}, std::integral_constant<int, 2 * kUnit>{}, bt);
    base[0] += kNext;
    base[1] += kNext;
  }
  if (nb < NW) {
    const char* const bt[1] = {st + (nb >> 1) * kNext + ls.alone_tr};
    add(nb, std::integral_constant<int, 1>{}, std::integral_constant<int, kUnit>{}, bt);
  }
}

// h of a pre-activation stack (SV: tanh(z0) in place of z0)
template <int DIM, int NCB, int MODE, int ACT, bool SV>
__device__ __forceinline__ void act_recompute(const v4f (&z)[NCB], v4f (&h)[NCB]) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPB = M::NPB;
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float s, s1, s2;
      act_d2s<ACT, SV>(z[pb][i], s, s1, s2);
      h[pb][i] = s;
      if constexpr (MODE == M_PDE) {
#pragma unroll
        for (int jj = 0; jj <= DIM; ++jj) h[(1 + jj) * NPB + pb][i] = s1 * z[(1 + jj) * NPB + pb][i];
#pragma unroll
        for (int jj = 0; jj < DIM; ++jj) {
          const float z1 = z[(1 + jj) * NPB + pb][i];
          h[(DIM + 2 + jj) * NPB + pb][i] = s2 * z1 * z1 + s1 * z[(DIM + 2 + jj) * NPB + pb][i];
        }
      }
    }
}

// h of a stashed pre-activation stack (SV: tanh(z0) in place of z0), one channel
// at a time straight into the LDS stack (few values live at once)
template <int DIM, int NCB, int MODE, int ACT, bool SV, int U>
__device__ __forceinline__ void act_store(char* base, const v4f (&z)[NCB]) {
  using M = ModeCfg<DIM, NCB, MODE>;
  constexpr int NPB = M::NPB;
#pragma unroll
  for (int pb = 0; pb < NPB; ++pb) {
    v4f sv, s1, s2;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float a0, a1, a2;
      act_d2s<ACT, SV>(z[pb][i], a0, a1, a2);
      sv[i] = a0;
      s1[i] = a1;
      s2[i] = a2;
    }
    stack_put<U>(base, pb, sv);
    if constexpr (MODE == M_PDE) {
#pragma unroll
      for (int jj = 0; jj <= DIM; ++jj) stack_put<U>(base, (1 + jj) * NPB + pb, s1 * z[(1 + jj) * NPB + pb]);
#pragma unroll
      for (int jj = 0; jj < DIM; ++jj) {
        const v4f z1 = z[(1 + jj) * NPB + pb];
        stack_put<U>(base, (DIM + 2 + jj) * NPB + pb, s2 * z1 * z1 + s1 * z[(DIM + 2 + jj) * NPB + pb]);
      }
    }
  }
}

// one tile after another of this workgroup's item ranges, for a wave of R row blocks
template <int DIM, int PBP, int ACT, int R>
__device__ __forceinline__ void step_tiles(const StepArgs& args, char* lds, int rb0, int w) {
  constexpr int D = DIM + 1;
  constexpr int CF = 2 * DIM + 2;
  constexpr int NCB = CF * PBP;
  constexpr int NCOL = 16 * NCB;
  using MP = ModeCfg<DIM, NCB, M_PDE>;
  using MV = ModeCfg<DIM, NCB, M_VALUE>;
  constexpr bool LEAN = NCB > 6;   // few registers to spare: h one channel at a time
  constexpr bool SV = ACT == ACT_TANH;   // the stash keeps tanh(z0) in place of z0

  const Shape& sh = args.sh;
  const int Wp = sh.Wp, NW = sh.NW, H = sh.H, KB = (NW + 1) >> 1;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int lane = tid & 63, g = lane >> 4, j = lane & 15;
  const uint32_t lane16 = (uint32_t)lane * 16u;
  const LaneSlots ls = lane_slots(lane);
  const SplitStepLds L = split_step_lds(D, NW, NCB);
  float* ys = reinterpret_cast<float*>(lds + L.ys);
  float* xin = reinterpret_cast<float*>(lds + L.xin);
  float* part = reinterpret_cast<float*>(lds);
  // stash: z of (layer, row block, column block), 1 KiB wave fragments
  float* stash = args.stash + (size_t)blockIdx.x * args.stash_per_wg + (size_t)rb0 * NCB * 256;
  const size_t stash_l = (size_t)NW * NCB * 256;
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

      // ---- forward.  The stash keeps the pre-activations of layers 1..H-1 for
      // the adjoint (z_H stays in registers); with tanh its value channel keeps tanh(z0), in which the
      // derivatives of tanh are polynomials.
      v4f acc[R][NCB];
      const int nvb = pde ? MP::NPB : MV::NPB;   // value-channel column blocks
      // z_l in acc -> stash, then h_l in acc
      v4f zl[R][NCB];   // z_H
      auto activate = [&](int l) {
        float* st = stash + (size_t)(l - 1) * stash_l;
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
            if (!SV || cb >= nvb) stg4u(st + (r * NCB + cb) * 256, lane16, acc[r][cb]);
          if (pde) act_forward<DIM, NCB, M_PDE, ACT>(acc[r]);
          else act_forward<DIM, NCB, M_VALUE, ACT>(acc[r]);
          if (SV) {
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
              if (cb < nvb) stg4u(st + (r * NCB + cb) * 256, lane16, acc[r][cb]);
          }
        }
      };
      auto activate_last = [&] {   // z_H in acc -> zl, h_H in acc
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) zl[r][cb] = acc[r][cb];
          if (pde) act_forward<DIM, NCB, M_PDE, ACT>(acc[r]);
          else act_forward<DIM, NCB, M_VALUE, ACT>(acc[r]);
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
            if (SV && cb < nvb) zl[r][cb] = acc[r][cb];
        }
      };
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (pde) input_layer<DIM, NCB, M_PDE>(acc[r], fr + sh.f_w1, bp, xin, rb0 + r, g, j);
        else input_layer<DIM, NCB, M_VALUE>(acc[r], fr + sh.f_w1, bp, xin, rb0 + r, g, j);
      }
      const float* wf = fr + sh.f_hid3 + (size_t)rb0 * KB * 3 * kFragFloats;   // of W_2
      Frags<R> f;   // weight fragments and bias of the next contraction over neurons
      v4f bias[R];
      auto load_bias = [&](int l) {
#pragma unroll
        for (int r = 0; r < R; ++r) bias[r] = ldg4(bp + (l - 1) * Wp + 16 * (rb0 + r) + 4 * g);
      };
      if (H > 1) {
        load_frags<R>(wf, KB, 0, lane16, f);
        load_bias(2);
      }
      if (H > 1) activate(1);
      else activate_last();
      for (int l = 2; l <= H; ++l) {
        stack_store<R, NCB>(lds, rb0, NW, ls, acc);
        __syncthreads();
        if (prio) __builtin_amdgcn_s_setprio(1);
        gemm_neurons<R, NCB, true>(wf + (size_t)(l - 2) * sh.hid3_layer, lds, NW, ls, lane16, f, acc);
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
            if (cb < nvb) acc[r][cb] += bias[r];
        if (l < H) {
          load_frags<R>(wf + (size_t)(l - 1) * sh.hid3_layer, KB, 0, lane16, f);
          load_bias(l + 1);
        }
        if (l < H) activate(l);
        else activate_last();
        __syncthreads();
      }

      // ---- output layer
      output_partials<D, R, NCB>(part, Wop, Wp, rb0, w, g, j, acc);
      __syncthreads();
      if (pde) output_sum<DIM, NCB, M_PDE>(part, 4 * sh.NWV, fr + sh.f_bo, ys, tid, nthr);
      else output_sum<DIM, NCB, M_VALUE>(part, 4 * sh.NWV, fr + sh.f_bo, ys, tid, nthr);
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
      // columns and added to the slab by the lanes j = 0.
      auto load_z = [&](int l, int r, v4f (&z)[NCB]) {
        const float* st = stash + (size_t)(l - 1) * stash_l + (size_t)r * NCB * 256;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) z[cb] = ldg4u(st + cb * 256, lane16);
      };
      {
        float* so = slab + sh.s_wo + 16 * rb0 + 4 * g;
        v4f hb[R][NCB];
#pragma unroll
        for (int o = 0; o < D; ++o) {
          v4f old[R], wo[R], s[R];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            old[r] = (j == 0 && !first) ? ldg4(so + o * Wp + 16 * r) : zero4();
            wo[r] = ldg4(Wop + o * Wp + 16 * (rb0 + r) + 4 * g);
            s[r] = zero4();
          }
          float b = 0.f;
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            const float yv = ys[o * NCOL + 16 * cb + j];
            if (cb < nvb) b += yv;
#pragma unroll
            for (int r = 0; r < R; ++r) {
              s[r] += yv * acc[r][cb];
              hb[r][cb] = o == 0 ? wo[r] * yv : hb[r][cb] + wo[r] * yv;
            }
          }
#pragma unroll
          for (int r = 0; r < R; ++r) {
            s[r] = row_sum4(s[r]);
            if (j == 0) stg4(so + o * Wp + 16 * r, old[r] + s[r]);
          }
          b = row_sum(b);
          if (tid == o) dbo += b;
          asm volatile("" : "+v"(dbo));   // now: its terms would be kept until the tile's end
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) acc[r][cb] = hb[r][cb];
      }
      // Layer l, one row block after another: H_l into the LDS stack (below H);
      // acc = hbar_l -> zbar_l; db_l and, at l = 1, dW_1.
      auto adjoint = [&](int l, v4f (&zn)[NCB], auto last) {   // zn: z_l of the first row block, if not last
        float* sb = slab + sh.s_b + (size_t)(l - 1) * Wp + 16 * rb0 + 4 * g;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          v4f zs[NCB];
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) zs[cb] = decltype(last)::value ? zl[r][cb] : zn[cb];
          const v4f old = (j == 0 && !first) ? ldg4(sb + 16 * r) : zero4();
          if constexpr (!decltype(last)::value) {
            bool alone;
            char* base = stack_row_slot<NCB>(lds, rb0 + r, NW, ls, alone);
            if constexpr (LEAN) {
              if (alone) {
                if (pde) act_store<DIM, NCB, M_PDE, ACT, SV, kUnit>(base, zs);
                else act_store<DIM, NCB, M_VALUE, ACT, SV, kUnit>(base, zs);
              } else {
                if (pde) act_store<DIM, NCB, M_PDE, ACT, SV, 2 * kUnit>(base, zs);
                else act_store<DIM, NCB, M_VALUE, ACT, SV, 2 * kUnit>(base, zs);
              }
            } else {
              v4f h[NCB];
              if (pde) act_recompute<DIM, NCB, M_PDE, ACT, SV>(zs, h);
              else act_recompute<DIM, NCB, M_VALUE, ACT, SV>(zs, h);
              stack_store_row<NCB>(lds, rb0 + r, NW, ls, h);
            }
          }
          if (pde) act_adjoint<DIM, NCB, M_PDE, ACT, SV>(acc[r], zs);
          else act_adjoint<DIM, NCB, M_VALUE, ACT, SV>(acc[r], zs);
          v4f s = zero4();
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
            if (cb < nvb) s += acc[r][cb];
          s = row_sum4(s);
          if (r + 1 < R && !decltype(last)::value) load_z(l, r + 1, zn);
          if (j == 0) stg4(sb + 16 * r, old + s);
        }
        if (l > 1) return;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          // dW1[n][q] += sum_pts zbar0 xi_q + zbar_q (first-derivative channel q)
          float* s1 = slab + sh.s_w1 + (size_t)(16 * (rb0 + r) + 4 * g) * D;
          v4f o1[D], v[D];
#pragma unroll
          for (int q = 0; q < D; ++q) {
            o1[q] = (j == 0 && !first) ? ldg4(s1 + 4 * q) : zero4();
            v[q] = zero4();
          }
          if (pde) {
#pragma unroll
            for (int pb = 0; pb < MP::NPB; ++pb)
#pragma unroll
              for (int q = 0; q < D; ++q)
                v[q] += acc[r][pb] * xin[(16 * pb + j) * D + q] + acc[r][(1 + q) * MP::NPB + pb];
          } else {
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
              for (int q = 0; q < D; ++q) v[q] += acc[r][cb] * xin[(16 * cb + j) * D + q];
          }
#pragma unroll
          for (int q = 0; q < D; ++q) v[q] = row_sum4(v[q]);
          if (j == 0) {
            float t[4 * D];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
              for (int q = 0; q < D; ++q) t[i * D + q] = v[q][i];
#pragma unroll
            for (int q = 0; q < D; ++q) stg4(s1 + 4 * q, o1[q] + v4f{t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]});
          }
        }
      };
      const float* wt = wf + sh.hid3_layer / 2;   // of W_2^T
      if (H > 1) load_frags<R>(wt + (size_t)(H - 2) * sh.hid3_layer, KB, 0, lane16, f);
      {
        v4f none[NCB];
        adjoint(H, none, std::true_type{});
      }

      // ---- hidden layer adjoints
      for (int l = H; l >= 2; --l) {
        if (l < H) load_frags<R>(wt + (size_t)(l - 2) * sh.hid3_layer, KB, 0, lane16, f);
        __syncthreads();   // every reader of the stack (dW_{l+1}; the output partials) is done
        stack_store<R, NCB>(lds, rb0, NW, ls, acc);
        __syncthreads();
        v4f zn[NCB];   // z_{l-1} of the first row block
        load_z(l - 1, 0, zn);
        if (prio) __builtin_amdgcn_s_setprio(1);
        gemm_neurons<R, NCB, true>(wt + (size_t)(l - 2) * sh.hid3_layer, lds, NW, ls, lane16, f, acc);   // Hbar_{l-1}
        __builtin_amdgcn_s_setprio(0);
        v8h za[R][NCB / 2][3];
        own_operands<R, NCB>(lds, rb0, NW, ls, za);
        __syncthreads();
        adjoint(l - 1, zn, std::false_type{});
        __syncthreads();
        if (prio) __builtin_amdgcn_s_setprio(1);
        gemm_columns<R, NCB>(za, lds, NW, ls, lane16,
                             slab + sh.s_hid + (size_t)(l - 2) * Wp * Wp + (size_t)rb0 * NW * 256, first);
        __builtin_amdgcn_s_setprio(0);
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
            for (int q = 0; q < sh.NWV; ++q) v += ys[q * 8 + tid];
          slab[sh.s_loss + tid] = v;
        }
      }
    }
    if (!args.counter) break;
  }
}

// Two waves per SIMD (256 registers each); the 32-point tiles have twice the
// columns and at most four waves, one per SIMD.
template <int DIM, int PBP, int ACT>
__global__ __launch_bounds__(PBP == 1 ? 512 : 256, PBP == 1 ? 2 : 1) void split_step_kernel(const StepArgs args) {
  extern __shared__ __align__(16) char slds[];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  step_tiles<DIM, PBP, ACT, 1>(args, slds, w, w);
}

// ---------------------------------------------------------------------------
// instances: one dimension and activation per translation unit
// ---------------------------------------------------------------------------
template <int DIM, int ACT>
const void* split_step_ptr(int tile_points, int NW) {
  if (tile_points == 32) return NW <= 4 ? (const void*)split_step_kernel<DIM, 2, ACT> : nullptr;
  return (const void*)split_step_kernel<DIM, 1, ACT>;
}
template const void* split_step_ptr<DDP_DIM, DDP_ACT>(int, int);

}  // namespace ddp
