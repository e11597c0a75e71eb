// Kernels around the networks, and the launchers: weight copies, gradient
// reduction and Adam, query routing, evaluation metrics (arXiv 2602.15883,
// sections 2.1, 2.2 and 3).  The network kernels are in ddpinn_step.hip (the fused
// training step), ddpinn_query.hip (query and exchange) and ddpinn_wide.hip (all three for
// 3D networks above 208 neurons).
//
// Gradients: each workgroup of the step accumulates its contribution in a
// private slab (one per (workgroup, subdomain) segment); the slabs are summed in
// a fixed order here.  No float atomics: every slab float has one writer lane and
// the sum order is fixed, so results are bitwise reproducible.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "ddpinn_split.h"

namespace ddp {

// ---------------------------------------------------------------------------
// prep: fragment-ordered copies of the weights (hidden neurons at their
// positions, zeros at padded positions)
// ---------------------------------------------------------------------------
// threads: one per float ahead of f_hid3, then one per pair of bf16 triples
__host__ __device__ inline int64_t prep_threads(const Shape& sh) {
  const int64_t KB = (sh.NW + 1) / 2;
  return sh.f_hid3 + (sh.s3 ? (2 * (sh.H - 1) * sh.NW + 1) * KB * 256 : 0);
}

__global__ void prep_kernel(const PrepArgs a) {
  const Shape& sh = a.sh;
  const int s = blockIdx.y;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  // (strided: one counter per subdomain can be more than the threads of a small network's copies)
  if (s == 0)
    for (int64_t k = idx; k < a.n_counters; k += (int64_t)gridDim.x * blockDim.x) a.counters[k] = 0;
  const float* th = a.subs[s].theta;
  float* fr = a.subs[s].frag;
  const int W = sh.W, Wp = sh.Wp, D = sh.D, H = sh.H;
  float v = 0.f;
  if (idx >= sh.f_hid3) {
    // bf16 triples of two neighbouring K slots of a hidden layer
    if (idx >= prep_threads(sh)) return;
    const int KB = (sh.NW + 1) >> 1, per = sh.NW * KB * 256;   // pairs of one matrix
    int e = (int)(idx - sh.f_hid3);
    const int m = e / per;
    e -= m * per;
    const bool out = m == 2 * (H - 1);   // W_{H+1}: its D rows
    const int l = out ? H + 1 : 2 + (m >> 1), trans = out ? 0 : m & 1;
    const int e2 = e & 3, lane = (e >> 2) & 63, t = e >> 8, kb = t % KB, rb = t / KB;
    const int r = out ? ((lane & 15) < D ? lane & 15 : -1) : hid_neuron(sh, 16 * rb + (lane & 15));
    float x[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      // a last row block alone keeps its neurons in the first four K slots
      const int g = lane >> 4, s8 = 2 * e2 + q, alone = (sh.NW & 1) && kb == KB - 1;
      const int k = hid_neuron(sh, 32 * kb + (alone ? 16 * (s8 >> 2) + 4 * g + (s8 & 3) : k_neuron(g, s8)));
      x[q] = (r >= 0 && k >= 0) ? (trans ? th[sh.p_w[l] + (int64_t)k * W + r] : th[sh.p_w[l] + (int64_t)r * W + k]) : 0.f;
    }
    uint32_t* o = reinterpret_cast<uint32_t*>(fr + sh.f_hid3) + (size_t)m * per * 3 + (size_t)t * 768 + lane * 4 + e2;
    o[0] = split_first(x[0], x[1]);
    o[256] = split_step(x[0], x[1]);
    o[512] = pack_bf16(x[0], x[1]);
    return;
  }
  if (idx < sh.f_w1) {
    const int64_t per = 2LL * Wp * Wp;
    const int l = 2 + (int)(idx / per);
    const int64_t rem = idx - (int64_t)(l - 2) * per;
    const bool trans = rem >= (int64_t)Wp * Wp;
    const int e = (int)(trans ? rem - (int64_t)Wp * Wp : rem);
    const int q = e & 3, lane = (e >> 2) & 63, t = e >> 8;
    const int K4 = Wp / 16;
    const int s4 = t % K4, w = t / K4;
    const int k = hid_neuron(sh, (lane >> 4) * (Wp / 4) + 4 * s4 + q);
    const int r = hid_neuron(sh, 16 * w + (lane & 15));
    if (r >= 0 && k >= 0) v = trans ? th[sh.p_w[l] + (int64_t)k * W + r] : th[sh.p_w[l] + (int64_t)r * W + k];
  } else if (idx < sh.f_b) {
    const int e = (int)(idx - sh.f_w1), p = e / D, q = e - p * D, r = hid_neuron(sh, p);
    if (r >= 0) v = th[sh.p_w[1] + (int64_t)r * D + q];
  } else if (idx < sh.f_wo) {
    const int e = (int)(idx - sh.f_b), l = 1 + e / Wp, r = hid_neuron(sh, e % Wp);
    if (r >= 0) v = th[sh.p_b[l] + r];
  } else if (idx < sh.f_bo) {
    const int e = (int)(idx - sh.f_wo), o = e / Wp, n = hid_neuron(sh, e % Wp);
    if (n >= 0) v = th[sh.p_w[H + 1] + (int64_t)o * W + n];
  } else if (idx < sh.f_bo + 4) {
    const int o = (int)(idx - sh.f_bo);
    if (o < D) v = th[sh.p_b[H + 1] + o];
  }
  fr[idx] = v;
}

// ---------------------------------------------------------------------------
// Gradient reduction and Adam.  One launch: the slabs of a subdomain are
// summed in a fixed order (a wave takes every kReduceGroups-th chunk of kSlabChunk slabs, then
// the waves' sums) in 64 bits and rounded once: the slabs largely cancel, and a sum in 32 bits
// was up to three quarters of a gradient's error (2D 4x32, 200,000 points, 512 slabs: 1.6e-7 of the
// gradient's norm, 0.84e-7 so; 3D 5x96, 20,000 points: 1.34 and 0.85e-7).  Without clipping Adam
// follows in the same thread, which also writes the parameter's kernel copies, so that neither
// the gradient nor theta is read again.
// With clipping a second launch applies Adam, each block adding up the same
// norm from the blocks' sums of squares.
// A block takes 64 consecutive slab positions (256 bytes of each slab); the kernel
// is bound by the reads of the slabs, of which a wave has sixteen in flight
// (2D 4x50, 2,000 points, 128 slabs of 58 KB: slab sum 4.8, gradient 9.9, Adam 4.7 and copies
// 4.1 us as four launches, 5.8 us so; 3D 8x200, 256 slabs of 1.2 MB: 64 us).
// ---------------------------------------------------------------------------

// row and column positions of element e of a layer's dW in the slab: tiles [row
// block][column block][64 lanes][4], lane (g, j): row 4g + i, column j; the
// kernels on triples keep the transpose so
__device__ __forceinline__ void slab_tile_rc(const Shape& sh, int e, int& r, int& c) {
  const int lane = (e >> 2) & 63, t = e >> 8, w = t / sh.NW, nb = t - w * sh.NW;
  const int a = 16 * w + 4 * (lane >> 4) + (e & 3), b = 16 * nb + (lane & 15);
  r = sh.s3 ? b : a;
  c = sh.s3 ? a : b;
}

// packed parameter at a slab position (-1: padding or a loss sum)
__device__ __forceinline__ int64_t slab_param(const Shape& sh, int64_t pos) {
  const int W = sh.W, Wp = sh.Wp, D = sh.D;
  if (pos < sh.s_b) {                          // dW_l in accumulator order
    const int per = Wp * Wp, l = 2 + (int)(pos / per);
    const int e = (int)(pos - (int64_t)(l - 2) * per);
    int rp, cp;
    slab_tile_rc(sh, e, rp, cp);
    const int r = hid_neuron(sh, rp), c = hid_neuron(sh, cp);
    return r >= 0 && c >= 0 ? sh.p_w[l] + (int64_t)r * W + c : -1;
  }
  if (pos < sh.s_w1) {
    const int e = (int)(pos - sh.s_b), l = e / Wp, r = hid_neuron(sh, e - l * Wp);
    return r >= 0 ? sh.p_b[l + 1] + r : -1;
  }
  if (pos < sh.s_wo) {
    const int e = (int)(pos - sh.s_w1), q = e / D, r = hid_neuron(sh, q);
    return r >= 0 ? (int64_t)r * D + (e - q * D) : -1;
  }
  if (pos < sh.s_bo) {
    const int e = (int)(pos - sh.s_wo), o = e / Wp, n = hid_neuron(sh, e - o * Wp);
    return n >= 0 ? sh.p_w[sh.H + 1] + (int64_t)o * W + n : -1;
  }
  return pos < sh.s_bo + D ? sh.p_b[sh.H + 1] + (pos - sh.s_bo) : -1;
}

// The copies that queries and exchanges read of the parameter at slab position pos
// (prep_kernel's layout).  The step's own copies (the transposed ones and W_{H+1}'s triples) are
// rebuilt by prep_kernel at the start of every step.
__device__ __forceinline__ void write_copies(const Shape& sh, float* fr, int64_t pos, float v) {
  const int Wp = sh.Wp;
  if (pos >= sh.s_b) {
    // biases, W_1, W_{H+1} and b_{H+1} have the same order in both buffers
    const int64_t o = pos < sh.s_w1 ? sh.f_b + (pos - sh.s_b) : pos < sh.s_wo ? sh.f_w1 + (pos - sh.s_w1)
                    : pos < sh.s_bo ? sh.f_wo + (pos - sh.s_wo) : sh.f_bo + (pos - sh.s_bo);
    fr[o] = v;
    return;
  }
  const int per = Wp * Wp, li = (int)(pos / per), e = (int)(pos - (int64_t)li * per);
  int r, c;
  slab_tile_rc(sh, e, r, c);
  if (!sh.s3) {
    const int seg = Wp / 4, g = c / seg, q = c - g * seg;
    fr[sh.f_hid + (int64_t)li * 2 * per + (((int64_t)(r >> 4) * (Wp / 16) + (q >> 2)) * 64 + 16 * g + (r & 15)) * 4 + (q & 3)] = v;
    return;
  }
  float x = v, y = 0.f;
  uint32_t part[3];
  part[0] = split_first(x, y);
  part[1] = split_step(x, y);
  part[2] = pack_bf16(x, y);
  const int KB = (sh.NW + 1) >> 1, kb = c >> 5, n = c & 31, g = (n >> 2) & 3;
  const int alone = (sh.NW & 1) && kb == KB - 1;
  const int slot = 4 * ((n >> 4) ^ (alone ? 0 : slot_half(g))) + (n & 3);
  uint16_t* o = reinterpret_cast<uint16_t*>(fr + sh.f_hid3 + (int64_t)li * sh.hid3_layer) +
                ((int64_t)((r >> 4) * KB + kb) * 3 * 64 + 16 * g + (r & 15)) * 8 + slot;
  o[0] = (uint16_t)part[0];
  o[512] = (uint16_t)part[1];
  o[1024] = (uint16_t)part[2];
}

// Adam on parameter p (slab position pos) with gradient g
__device__ __forceinline__ void adam_update(const ReduceArgs& a, const SubDev& sd, int64_t p, int64_t pos, float g) {
  const float m = a.beta1 * sd.m[p] + (1.f - a.beta1) * g;
  const float v = a.beta2 * sd.v[p] + (1.f - a.beta2) * g * g;
  sd.m[p] = m;
  sd.v[p] = v;
  const float c1 = 1.f - powf(a.beta1, (float)a.t);
  const float c2 = 1.f - powf(a.beta2, (float)a.t);
  float* th = const_cast<float*>(sd.theta);
  const float x = th[p] - a.lr * (m / c1) / (sqrtf(v / c2) + a.eps);
  th[p] = x;
  write_copies(a.sh, sd.frag, pos, x);
}

constexpr int kReduceGroups = 8;   // waves of a block
constexpr int kReducePos = kWave;  // slab positions of a block

__global__ __launch_bounds__(kReduceGroups * kReducePos) void reduce_kernel(const ReduceArgs a) {
  const Shape& sh = a.sh;
  const int s = blockIdx.y, lane = threadIdx.x % kReducePos;
  const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kReducePos);   // the wave
  const int64_t pos = (int64_t)blockIdx.x * kReducePos + lane;
  const int k0 = a.seg_begin[s], k1 = a.seg_begin[s + 1];
  __shared__ double part[kReduceGroups][kReducePos];
  double acc = 0.0;
  auto add = [&](int c0, auto whole) {
    float v[kSlabChunk];
#pragma unroll
    for (int q = 0; q < kSlabChunk; ++q) {   // (past the last slab the last one, which is not added)
      const int k = decltype(whole)::value || c0 + q < k1 ? c0 + q : k1 - 1;
      v[q] = ldg(a.slabs + (size_t)k * sh.slab_floats + pos);
    }
    if (!decltype(whole)::value) {
#pragma unroll
      for (int q = 0; q < kSlabChunk; ++q) v[q] = c0 + q < k1 ? v[q] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < kSlabChunk; q += 4)
      acc += ((double)v[q] + (double)v[q + 1]) + ((double)v[q + 2] + (double)v[q + 3]);
  };
  int c0 = k0 + grp * kSlabChunk;
  for (; c0 + kSlabChunk <= k1; c0 += kReduceGroups * kSlabChunk) add(c0, std::true_type{});
  if (c0 < k1) add(c0, std::false_type{});
  part[grp][lane] = acc;
  __syncthreads();
  if (grp != 0) return;   // one wave from here on
  acc = 0.0;
#pragma unroll
  for (int q = 0; q < kReduceGroups; ++q) acc += part[q][lane];
  const float tot = (float)acc;
  const SubDev& sd = a.subs[s];
  const int64_t p = slab_param(sh, pos);
  if (p >= 0) {
    a.gbuf[(size_t)s * sh.P + p] = tot;
    if (a.grad_out) a.grad_out[(size_t)s * sh.P + p] = tot;
    if (a.update && a.clip <= 0.f) adam_update(a, sd, p, pos, tot);
  }
  if (a.clip > 0.f) {
    float q = p >= 0 ? tot * tot : 0.f;
    for (int o = 32; o > 0; o >>= 1) q += __shfl_xor(q, o, 64);
    if (lane == 0) a.normpart[(size_t)s * gridDim.x + blockIdx.x] = q;
  }
  // losses (s_loss is a multiple of kReducePos)
  if (pos - lane != sh.s_loss) return;
  float L[7];
  for (int q = 0; q < 6; ++q) L[q] = __shfl(tot, q, 64);
  if (lane != 0) return;
  L[0] *= sd.inv_n[1];
  L[1] *= sd.inv_n[0];
  L[2] *= sd.inv_n[2];
  L[3] *= sd.inv_n[2];
  L[4] *= sd.inv_n[2];
  L[5] *= sd.inv_n[3];
  L[6] = sd.lam[0] * L[0] + sd.lam[1] * L[1] + sd.lam[2] * L[2] + sd.lam[3] * L[3] +
         sd.lam[4] * L[4] + sd.lam[5] * L[5];
  for (int q = 0; q < 7; ++q) {
    a.loss_ws[s * 8 + q] = L[q];
    if (a.loss_out) a.loss_out[s * 7 + q] = L[q];
  }
  a.loss_ws[s * 8 + 7] = 0.f;
}

// Adam on the clipped gradient: every block adds up the subdomain's norm from
// the reduce blocks' sums of squares (the same order in each), then updates its positions
__global__ __launch_bounds__(256) void clip_adam_kernel(const ReduceArgs a, int nblk) {
  const Shape& sh = a.sh;
  const int s = blockIdx.y;
  __shared__ float red[256];
  float v = 0.f;
  for (int k = threadIdx.x; k < nblk; k += blockDim.x) v += a.normpart[(size_t)s * nblk + k];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int o = blockDim.x / 2; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  const float nrm = sqrtf(red[0]);
  const float scale = nrm > a.clip ? a.clip / nrm : 1.f;
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (!a.update || pos >= sh.slab_floats) return;
  const int64_t p = slab_param(sh, pos);
  if (p >= 0) adam_update(a, a.subs[s], p, pos, a.gbuf[(size_t)s * sh.P + p] * scale);
}

// ---------------------------------------------------------------------------
// query: routing (bin points by subdomain box) and grouped forward
// ---------------------------------------------------------------------------
__global__ void route_zero_kernel(int32_t* counts, int32_t* cursor, int n_sub) {
  for (int s = threadIdx.x; s < n_sub; s += blockDim.x) { counts[s] = 0; cursor[s] = 0; }
}

// Routing is a counting sort by subdomain.  Points are counted in a per-block
// LDS histogram and each block adds its counts to the global ones with one
// atomic per subdomain; the scatter reserves a contiguous slot range per
// (block, subdomain) the same way.  (Global atomics per point serialise on
// the few subdomain counters.)
constexpr int kRouteBlock = 256;

// The boxes are read from LDS (staged once per block): a point tests up to
// n_sub boxes in turn, and each test read from global memory cost its latency.
// 32 bytes each; more boxes are read from global memory, one latency per box and point (16
// boxes: 450 points 14.7 us from there, 9.7 us from LDS; count of 200,000 points 24.0 and 18.1)
constexpr int kRouteLdsSubs = 512;

__device__ __forceinline__ const float* stage_boxes(const RouteArgs& a, float* lbox) {
  if (a.n_sub > kRouteLdsSubs) return a.boxes;
  for (int k = threadIdx.x; k < 8 * a.n_sub; k += blockDim.x) lbox[k] = a.boxes[k];
  return lbox;
}

__device__ __forceinline__ int route_point(const RouteArgs& a, const float* boxes, int64_t i) {
  const float* x = a.x + i * a.D;
  const float c[4] = {x[0], x[1], x[2], a.D > 3 ? x[3] : 0.f};
  for (int s = 0; s < a.n_sub; ++s) {
    const float* lo = boxes + s * 8;
    const float* hi = lo + 4;
    bool in = true;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      in &= q >= a.D || ((c[q] >= lo[q]) && (c[q] < hi[q] || (c[q] == hi[q] && hi[q] == a.gmax[q])));
    if (in) return s;
  }
  return -1;
}

// offsets = exclusive sums of counts, by one wave
__device__ __forceinline__ void route_offsets(const int* counts, int n_sub, int* offsets) {
  if (threadIdx.x >= 64) return;
  int base = 0;
  for (int s0 = 0; s0 < n_sub; s0 += 64) {
    const int s = s0 + threadIdx.x, c = s < n_sub ? counts[s] : 0;
    int v = c;
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(v, o, 64);
      if ((int)threadIdx.x >= o) v += u;
    }
    if (s < n_sub) offsets[s] = base + v - c;
    base += __shfl(v, 63, 64);
  }
  if (threadIdx.x == 0) offsets[n_sub] = base;
}

__global__ __launch_bounds__(kRouteBlock) void route_count_kernel(const RouteArgs a) {
  extern __shared__ int hist[];   // [n_sub], then the boxes
  for (int s = threadIdx.x; s < a.n_sub; s += blockDim.x) hist[s] = 0;
  const float* boxes = stage_boxes(a, reinterpret_cast<float*>(hist + a.n_sub));
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < a.n) {
    const int found = route_point(a, boxes, i);
    a.sub_id[i] = found;
    if (found >= 0) atomicAdd(&hist[found], 1);
    else
      for (int q = 0; q < a.out_cols; ++q) a.out[i * a.out_cols + q] = __builtin_nanf("");
  }
  __syncthreads();
  for (int s = threadIdx.x; s < a.n_sub; s += blockDim.x)
    if (hist[s]) atomicAdd(a.counts + s, hist[s]);
}

// every block takes the offsets from the counts itself; block 0 writes them out
__global__ __launch_bounds__(kRouteBlock) void route_scatter_kernel(const RouteArgs a) {
  extern __shared__ int sh[];   // hist[n_sub], base[n_sub + 1]
  int* hist = sh;
  int* base = sh + a.n_sub;
  for (int s = threadIdx.x; s < a.n_sub; s += blockDim.x) hist[s] = 0;
  route_offsets(a.counts, a.n_sub, base);
  __syncthreads();
  if (blockIdx.x == 0)
    for (int s = threadIdx.x; s <= a.n_sub; s += blockDim.x) a.offsets[s] = base[s];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int s = (i < a.n) ? a.sub_id[i] : -1;
  const int rank = (s >= 0) ? atomicAdd(&hist[s], 1) : 0;
  __syncthreads();
  for (int q = threadIdx.x; q < a.n_sub; q += blockDim.x)
    if (hist[q]) base[q] += atomicAdd(a.cursor + q, hist[q]);
  __syncthreads();
  if (s >= 0) a.perm[base[s] + rank] = (int32_t)i;
}

// A small query routed by one workgroup: subdomain of every point, counts,
// offsets and the permutation from one launch instead of four.  Each thread
// keeps the subdomains of its points in registers between the two passes.
constexpr int kRouteSmallThreads = 1024;
constexpr int kRouteSmallPerThread = 8;
constexpr int kRouteSmallMax = kRouteSmallThreads * kRouteSmallPerThread;   // points

__global__ __launch_bounds__(kRouteSmallThreads) void route_small_kernel(const RouteArgs a) {
  extern __shared__ int sh[];   // hist[n_sub], base[n_sub + 1], then the boxes
  int* hist = sh;
  int* base = sh + a.n_sub;
  for (int s = threadIdx.x; s < a.n_sub; s += blockDim.x) hist[s] = 0;
  const float* boxes = stage_boxes(a, reinterpret_cast<float*>(base + a.n_sub + 1));
  __syncthreads();
  int sid[kRouteSmallPerThread];
#pragma unroll
  for (int k = 0; k < kRouteSmallPerThread; ++k) {
    const int64_t i = threadIdx.x + (int64_t)k * kRouteSmallThreads;
    sid[k] = -1;
    if (i < a.n) {
      const int found = route_point(a, boxes, i);
      sid[k] = found;
      a.sub_id[i] = found;
      if (found >= 0) atomicAdd(&hist[found], 1);
      else
        for (int q = 0; q < a.out_cols; ++q) a.out[i * a.out_cols + q] = __builtin_nanf("");
    }
  }
  __syncthreads();
  route_offsets(hist, a.n_sub, base);
  __syncthreads();
  for (int s = threadIdx.x; s <= a.n_sub; s += blockDim.x) {
    a.offsets[s] = base[s];
    if (s < a.n_sub) a.counts[s] = hist[s];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kRouteSmallPerThread; ++k)
    if (sid[k] >= 0) a.perm[atomicAdd(&base[sid[k]], 1)] = (int32_t)(threadIdx.x + k * kRouteSmallThreads);
}

// ---------------------------------------------------------------------------
// evaluation post-processing (stitched field, master anchor pinning,
// per-snapshot pressure-mean removal, relative L2 errors)
// ---------------------------------------------------------------------------
__global__ void anchor_points_kernel(const float* x, int64_t n, int D, float a0, float a1, float a2, float* xa) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float an[3] = {a0, a1, a2};
  for (int q = 0; q < D - 1; ++q) xa[i * D + q] = an[q];
  xa[i * D + D - 1] = x[i * D + D - 1];   // the point's own time
}

// routed counts kept only for master subdomains (the anchor pass skips the rest)
__global__ void master_counts_kernel(const SubDev* subs, const int32_t* counts, int n_sub, int32_t* out) {
  for (int s = threadIdx.x; s < n_sub; s += blockDim.x) out[s] = subs[s].is_master ? counts[s] : 0;
}

__device__ __forceinline__ float block_sum256(float v, float* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  const float r = red[0];
  __syncthreads();
  return r;
}

// processed pressure of point i: p - p(x_anc, t) on master subdomains
__device__ __forceinline__ float eval_p(const EvalArgs& a, int64_t i) {
  const int D = a.D;
  float p = a.pred[i * D + D - 1];
  const int s = a.sub_id[i];
  if (s >= 0 && a.subs[s].is_master) p -= a.pa[i * D + D - 1];
  return p;
}

__global__ void eval_means_kernel(const EvalArgs a) {
  __shared__ float red[256];
  const int k = blockIdx.y;
  const int64_t b0 = a.snap_off[k], b1 = a.snap_off[k + 1];
  const int64_t lo = b0 + (int64_t)blockIdx.x * kEvalChunk;
  const int64_t hi = min(b1, lo + kEvalChunk);
  float sp = 0.f, sr = 0.f;
  for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) {
    sp += eval_p(a, i);
    sr += a.ref[i * a.D + a.D - 1];
  }
  sp = block_sum256(sp, red);
  sr = block_sum256(sr, red);
  if (threadIdx.x == 0) {
    a.mpart[((size_t)k * a.nblk + blockIdx.x) * 2 + 0] = sp;
    a.mpart[((size_t)k * a.nblk + blockIdx.x) * 2 + 1] = sr;
  }
}

__global__ void eval_err_kernel(const EvalArgs a) {
  __shared__ float red[256];
  const int k = blockIdx.y, D = a.D, dim = D - 1;
  const int64_t b0 = a.snap_off[k], b1 = a.snap_off[k + 1];
  float mp = 0.f, mr = 0.f;
  for (int b = 0; b < a.nblk; ++b) {
    mp += a.mpart[((size_t)k * a.nblk + b) * 2 + 0];
    mr += a.mpart[((size_t)k * a.nblk + b) * 2 + 1];
  }
  if (b1 > b0) {
    mp /= (float)(b1 - b0);
    mr /= (float)(b1 - b0);
  }
  const int64_t lo = b0 + (int64_t)blockIdx.x * kEvalChunk;
  const int64_t hi = min(b1, lo + kEvalChunk);
  float num[4] = {0.f, 0.f, 0.f, 0.f}, den[4] = {0.f, 0.f, 0.f, 0.f};
  for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) {
    for (int q = 0; q < dim; ++q) {
      const float r = a.ref[i * D + q], e = a.pred[i * D + q] - r;
      num[q] += e * e;
      den[q] += r * r;
    }
    const float r = a.ref[i * D + dim] - mr;
    const float e = (eval_p(a, i) - mp) - r;
    num[dim] += e * e;
    den[dim] += r * r;
  }
  float* out = a.epart + ((size_t)k * a.nblk + blockIdx.x) * 2 * (D + 1);
  for (int q = 0; q < D; ++q) {
    const float vn = block_sum256(num[q], red);
    const float vd = block_sum256(den[q], red);
    if (threadIdx.x == 0) {
      out[2 * q] = vn;
      out[2 * q + 1] = vd;
    }
  }
}

// err[q] (velocity components), err[dim] (velocity vector), err[dim+1] (p).
// One block; each thread sums a fixed share of the chunk sums and the shares
// are added in a fixed order.  (One thread took 329 us for the 8,000 chunk sums of
// 1,000,000 points; 2,000,000 take 8.4 us so.)
__global__ __launch_bounds__(256) void eval_final_kernel(const EvalArgs a) {
  __shared__ float red[256];
  const int D = a.D, dim = D - 1, n = a.n_snap * a.nblk;
  float num[4] = {0.f, 0.f, 0.f, 0.f}, den[4] = {0.f, 0.f, 0.f, 0.f};
  for (int k = threadIdx.x; k < n; k += blockDim.x) {
    const float* e = a.epart + (size_t)k * 2 * (D + 1);
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < D) {
        num[q] += e[2 * q];
        den[q] += e[2 * q + 1];
      }
  }
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (q < D) {
      num[q] = block_sum256(num[q], red);
      den[q] = block_sum256(den[q], red);
    }
  if (threadIdx.x != 0) return;
  float nv = 0.f, dv = 0.f;
  for (int q = 0; q < dim; ++q) {
    a.err_out[q] = sqrtf(num[q] / den[q]);
    nv += num[q];
    dv += den[q];
  }
  a.err_out[dim] = sqrtf(nv / dv);
  a.err_out[dim + 1] = sqrtf(num[dim] / den[dim]);
}

hipError_t launch_anchor_points(const float* x, int64_t n, int D, const float* x_anc, float* xa, hipStream_t s) {
  const unsigned nb = (unsigned)((n + 255) / 256);
  if (nb)
    hipLaunchKernelGGL(anchor_points_kernel, dim3(nb), dim3(256), 0, s, x, n, D, x_anc[0], D > 2 ? x_anc[1] : 0.f,
                       D > 3 ? x_anc[2] : 0.f, xa);
  return hipGetLastError();
}

hipError_t launch_master_counts(const SubDev* subs, const int32_t* counts, int n_sub, int32_t* out, hipStream_t s) {
  hipLaunchKernelGGL(master_counts_kernel, dim3(1), dim3(256), 0, s, subs, counts, n_sub, out);
  return hipGetLastError();
}

hipError_t launch_evaluate(const EvalArgs& a, hipStream_t s) {
  const dim3 grid(a.nblk, a.n_snap);
  hipLaunchKernelGGL(eval_means_kernel, grid, dim3(256), 0, s, a);
  hipLaunchKernelGGL(eval_err_kernel, grid, dim3(256), 0, s, a);
  hipLaunchKernelGGL(eval_final_kernel, dim3(1), dim3(256), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int step_value_points(int dim, int tile_points) {
  return 16 * (2 * dim + 2) * (tile_points / 16);
}

// LDS of a compute unit
constexpr int kLdsBytes = 160 * 1024;

// The kernels on triples serve every network whose stack fits: where both kinds ran, the fp32 ones
// were slower at every width (3D 8x200, 600,000 points: 104 against 55 ms per step; 2D 4x50,
// 2,000 points: 69 against 47 us).
bool split_fits(int dim, int NW) {
  const int NCB = 2 * dim + 2;
  return std::max(split_query_lds(dim + 1, NW, std::min(NW, 8), NCB, false).total, split_step_lds(dim + 1, NW, NCB).total) <= kLdsBytes;
}

static const void* split_step_any(int dim, int tile_points, int act, int NW, int NWS) {
  if (dim == 2) return act == ACT_SIN ? split_step_ptr<2, ACT_SIN>(tile_points, NW, NWS) : split_step_ptr<2, ACT_TANH>(tile_points, NW, NWS);
  return act == ACT_SIN ? split_step_ptr<3, ACT_SIN>(tile_points, NW, NWS) : split_step_ptr<3, ACT_TANH>(tile_points, NW, NWS);
}
static const void* split_query_any(int dim, int mode, int act, int small, int NW) {
  return dim == 2 ? split_query_ptr<2>(mode, act, small, NW) : split_query_ptr<3>(mode, act, small, NW);
}
static const void* split_exchange_any(int dim, int act, int NW) {
  return dim == 2 ? split_exchange_ptr<2>(act, NW) : split_exchange_ptr<3>(act, NW);
}

// Five or six row blocks, whose stack fits in the LDS twice: the step can run two
// workgroups of four waves per compute unit in place of one of five or six waves,
// which leaves SIMDs with a single wave.  With seven or eight (2D; 3D does not fit) the two ways are
// within 1 % (2D 8x128 at 4 layers, 100,000 points: 1.20 and 1.21 ms per step) or the one is faster
// (2D 2x112, 50,000 points: 0.25 against 0.26 ms).
bool step_halves(const Shape& sh) {
  return sh.s3 && sh.NW > 4 && sh.NW <= 6 && 2 * split_step_lds(sh.D, sh.NW, 2 * sh.dim + 2).total <= kLdsBytes;
}

int step_lds_floats(const Shape& sh, int tile_points) {
  if (sh.s3) return split_step_lds(sh.D, sh.NW, (2 * sh.dim + 2) * (tile_points / 16)).total / 4;
  return wide_step_lds_floats(sh);
}

int query_waves(const Shape& sh, int small) { return small == 3 ? 1 : sh.NWV; }

int query_lds_floats(const Shape& sh, int small) {
  if (sh.s3)
    return split_query_lds(sh.D, sh.NW, sh.NWV, small == 1 || small == 2 ? sh.dim + 1 : 2 * sh.dim + 2, query_waves(sh, small) == 1).total / 4;
  return wide_query_lds_floats(sh, small);
}

const void* step_kernel_ptr(const Shape& sh, int tile_points) {
  if (sh.s3) return split_step_any(sh.dim, tile_points, sh.act, sh.NW, sh.NWS);
  return tile_points == 16 ? wide_step_ptr(sh.act) : nullptr;
}
const void* prep_kernel_ptr() { return (const void*)prep_kernel; }
const void* reduce_kernel_ptr() { return (const void*)reduce_kernel; }
const void* clip_adam_kernel_ptr() { return (const void*)clip_adam_kernel; }

void grid_prep(const PrepArgs& a, dim3* grid, dim3* block) {
  *block = dim3(256);
  *grid = dim3((unsigned)((prep_threads(a.sh) + 255) / 256), (unsigned)a.n_sub);
}
int reduce_blocks(const Shape& sh) { return (int)(sh.slab_floats / kReducePos); }
void grid_reduce(const ReduceArgs& a, dim3* grid, dim3* block) {
  *block = dim3(kReduceGroups * kReducePos);
  *grid = dim3((unsigned)reduce_blocks(a.sh), (unsigned)a.n_sub);
}
void grid_clip_adam(const ReduceArgs& a, dim3* grid, dim3* block) {
  *block = dim3(256);
  *grid = dim3((unsigned)((a.sh.slab_floats + 255) / 256), (unsigned)a.n_sub);
}

hipError_t launch_prep(const PrepArgs& a, hipStream_t s) {
  dim3 grid, block;
  grid_prep(a, &grid, &block);
  hipLaunchKernelGGL(prep_kernel, grid, block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_step(const StepArgs& a, int tile_points, int n_wg, hipStream_t s) {
  const size_t lds = (size_t)a.lds_floats * sizeof(float);
  const void* k = step_kernel_ptr(a.sh, tile_points);
  if (!k) return hipErrorInvalidValue;
  const dim3 block(a.sh.NWS * 64);
  void* args[] = {const_cast<StepArgs*>(&a)};
  return hipLaunchKernel(k, dim3(n_wg), block, args, lds, s);
}

// Routed-query scratch held by the library, for callers that cannot
// allocate (pinn_query_noalloc).  Every GPU the library runs on holds its own
// copy for the life of the process.  Host code never passes this name to a
// kernel: the name is a host-side stand-in; the device address comes from
// noalloc_scratch_address, resolved once per device with that device current.
static __device__ __align__(256) char scratch[kNoallocScratchBytes];

hipError_t noalloc_scratch_address(void** ptr) { return hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch)); }

// the same launch with events tied to the dispatch itself: e0 takes the
// kernel's start and e1 its end time stamp (either may be null)
hipError_t launch_step_timed(const StepArgs& a, int tile_points, int n_wg, hipStream_t s, hipEvent_t e0,
                             hipEvent_t e1) {
  const size_t lds = (size_t)a.lds_floats * sizeof(float);
  const void* k = step_kernel_ptr(a.sh, tile_points);
  if (!k) return hipErrorInvalidValue;
  const dim3 block(a.sh.NWS * 64);
  void* args[] = {const_cast<StepArgs*>(&a)};
  return hipExtLaunchKernel(k, dim3(n_wg), block, args, lds, s, e0, e1, 0);
}

hipError_t launch_reduce(const ReduceArgs& a, hipStream_t s) {
  dim3 grid, block;
  grid_reduce(a, &grid, &block);
  hipLaunchKernelGGL(reduce_kernel, grid, block, 0, s, a);
  if (a.clip > 0.f) {
    grid_clip_adam(a, &grid, &block);
    hipLaunchKernelGGL(clip_adam_kernel, grid, block, 0, s, a, reduce_blocks(a.sh));
  }
  return hipGetLastError();
}

hipError_t launch_route(const RouteArgs& a, hipStream_t s) {
  const size_t box = a.n_sub <= kRouteLdsSubs ? 32 * (size_t)a.n_sub : 0, h = sizeof(int) * (size_t)a.n_sub;
  if (a.n <= kRouteSmallMax) {
    hipLaunchKernelGGL(route_small_kernel, dim3(1), dim3(kRouteSmallThreads), 2 * h + 4 + box, s, a);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(route_zero_kernel, dim3(1), dim3(256), 0, s, a.counts, a.cursor, a.n_sub);
  const unsigned nb = (unsigned)((a.n + kRouteBlock - 1) / kRouteBlock);
  if (nb) hipLaunchKernelGGL(route_count_kernel, dim3(nb), dim3(kRouteBlock), h + box, s, a);
  if (nb) hipLaunchKernelGGL(route_scatter_kernel, dim3(nb), dim3(kRouteBlock), 2 * h + 4, s, a);
  return hipGetLastError();
}

const void* query_kernel_ptr(const Shape& sh, int what, int small) {
  const int mode = (what == Q_VALUE) ? M_VALUE : (what == Q_UVPW ? M_GRAD : M_PDE);
  return sh.s3 ? split_query_any(sh.dim, mode, sh.act, small, sh.NW) : wide_query_ptr(mode, sh.act, small);
}
const void* exchange_kernel_ptr(const Shape& sh) {
  return sh.s3 ? split_exchange_any(sh.dim, sh.act, sh.NW) : wide_exchange_ptr(sh.act);
}

hipError_t launch_query(const QueryArgs& a, int n_wg, hipStream_t s) {
  if (n_wg >= 16) n_wg &= ~7;   // a multiple of the XCD count (see query_kernel)
  const size_t lds = (size_t)a.lds_floats * sizeof(float);
  const dim3 block(query_waves(a.sh, a.small) * 64);
  void* args[] = {const_cast<QueryArgs*>(&a)};
  return hipLaunchKernel(query_kernel_ptr(a.sh, a.what, a.small), dim3(n_wg), block, args, lds, s);
}

hipError_t launch_exchange(const ExchangeArgs& a, int n_wg, hipStream_t s) {
  const size_t lds = (size_t)a.lds_floats * sizeof(float);
  const dim3 block(a.sh.NWV * 64);
  void* args[] = {const_cast<ExchangeArgs*>(&a)};
  return hipLaunchKernel(exchange_kernel_ptr(a.sh), dim3(n_wg), block, args, lds, s);
}

// LDS above 64 KiB must be allowed per kernel before launch.
hipError_t set_lds_limits(int bytes) {
  hipError_t e = hipSuccess;
  auto allow = [&](const void* k) {
    const hipError_t r = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (r != hipSuccess) e = r;
  };
  for (int dim = 2; dim <= 3; ++dim)
    for (int act = ACT_TANH; act <= ACT_SIN; ++act) {
      allow(split_step_any(dim, 32, act, 4, 4));
      for (int nw : {8, 13}) allow(split_step_any(dim, 16, act, nw, 8));
      for (int nw : {8, 16}) {
        for (int mode : {M_PDE, M_VALUE, M_GRAD}) {
          allow(split_query_any(dim, mode, act, 0, nw));
          allow(split_query_any(dim, mode, act, 1, nw));
        }
        allow(split_exchange_any(dim, act, nw));
      }
      allow(wide_step_ptr(act));
      for (int small = 0; small <= 1; ++small) {
        allow(wide_query_ptr(M_VALUE, act, small));
        allow(wide_query_ptr(M_PDE, act, small));
      }
      allow(wide_exchange_ptr(act));
    }
  return e;
}

}  // namespace ddp
