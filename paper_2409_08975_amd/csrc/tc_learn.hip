// Learned importance proposal (an extension: the paper samples the centre
// edge with probability w_e / W; here with q_e / Q, q_e = w_e * h_e, and
// corrects each sample by Q / h_e, which keeps the estimate unbiased for any
// h >= 1).
//
//   k_features     per scan position p, eight window features of the centre
//                  edge (sizes of its in- and out-windows and of the path
//                  weight, the spans of the two windows relative to delta,
//                  the multi-edge counts of (u, v) and (v, u) around t, and
//                  the mean squared degree of the windows' far endpoints from
//                  prefix sums, k_deg2_*), stored as bfloat16.
//   k_mlp_forward  g = sigmoid(w3 . relu(W2 relu(W1 f + b1) + b2) + b3) for
//                  32 edges per wavefront: both hidden layers on MFMA
//                  (bfloat16 operands, float32 accumulation).  The
//                  accumulator layout of one layer is fed to the next as its
//                  B operand without a trip through LDS: within one MFMA the
//                  order of the contraction index is free, so the weights are
//                  loaded in the order in which each lane holds the
//                  activations.
//   k_mlp_grad     mean binary cross-entropy against y = [X > 0] (or the
//                  soft label min(1, X / cap)) and its
//                  gradient, per block (fixed row-to-block assignment):
//                  the same forward, dH1 = W2^T dZ2 on MFMA from registers,
//                  and the weight gradients dW2 = dZ2 H1^T and
//                  [dW1 | db1] = dZ1 [F | 1]^T on MFMA after an LDS
//                  transpose that puts edges on the contraction index.
//   k_mlp_reduce   sums the block partials in block order (deterministic),
//                  then either stores the gradient or takes an Adam step.
//   k_quantize     h_int = max(1, floor((eps + (1 - eps) g) 2^s + 1/2)),
//                  s = clamp(63 - bitlen(W), 1, 16), in float32 with no
//                  contraction, so the integer decision is reproducible;
//                  optionally g is first divided by its maximum over the
//                  edges (k_score_max), so that the scores span [0, 1].
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "tc_device.h"
#include "tc_internal.h"

namespace tc {

// parameter vector: W1 [64][8], b1 [64], W2 [64][64], b2 [64], w3 [64], b3
constexpr int kIn = 8, kHid = 64;
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kHid * kIn;
constexpr int kOffW2 = kOffB1 + kHid;
constexpr int kOffB2 = kOffW2 + kHid * kHid;
constexpr int kOffW3 = kOffB2 + kHid;
constexpr int kOffB3 = kOffW3 + kHid;
constexpr int kNParams = kOffB3 + 1;  // 4801
static_assert(kNParams == TC_MLP_PARAMS, "parameter count");

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// bfloat16 bits of a float, round to nearest even (NaN stays NaN)
// bfloat16 rounded to nearest even (the conversion instruction; single
// precision denormals are kept, so it agrees with the rounding rule on every
// value but NaN), NaN made quiet keeping its top bits; a select, not a
// branch, so a wavefront never splits here
__device__ __forceinline__ uint16_t bf16_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  const uint16_t rne = __builtin_bit_cast(uint16_t, (__bf16)f);
  return (u & 0x7FFFFFFFu) > 0x7F800000u ? (uint16_t)((u >> 16) | 0x40u) : rne;
}
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// two values rounded to nearest even in one instruction (a NaN stays a NaN):
// a in the low half, b in the high half
__device__ __forceinline__ uint32_t bf16x2_bits(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float bf16_val(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ float bf16_round(float f) { return bf16_val(bf16_bits(f)); }

// Row (within a 32-row block) of accumulator register v of a lane in half h
// (h = lane / 32) for the 32x32 MFMA output layout; the column is lane % 32.
__device__ __forceinline__ int drow(int v, int h) { return 8 * (v >> 2) + 4 * h + (v & 3); }

// Row of the input held at position s (0..7) of K-chunk kc = 2 * rb + c by a
// lane in half h, when a layer's output block rb feeds the next layer.
__device__ __forceinline__ int krow(int kc, int s, int h) {
  return 32 * (kc >> 1) + drow(8 * (kc & 1) + s, h);
}

__device__ __forceinline__ bf16x8 pack8(const uint16_t (&e)[8]) {
  s16x8 v;
#pragma unroll
  for (int s = 0; s < 8; ++s) v[s] = (short)e[s];
  return __builtin_bit_cast(bf16x8, v);
}

// ---------------------------------------------------------------- features --
// Squared (capped) degree of the far endpoint of each adjacency entry: the
// source of an in-CSR entry (its in-degree) or the target of an out-CSR
// entry (its out-degree).  Capping at 2^16 - 1 keeps a window's sum below
// 2^63, so window sums taken from wrapping 64-bit prefix sums are exact, and
// lets the gathered degrees be kept as 16-bit words between the two passes
// of the scan: the second pass reads 2 bytes per entry instead of repeating
// the gather.
constexpr int kPBlock = 256, kPItems = 8, kPTile = kPBlock * kPItems;

// per tile: the capped degrees and the wrapping sum of their squares.
// Kernels that gather through the graph's vertex ids leave a rejected graph
// (non-zero build status) alone.
__global__ __launch_bounds__(kPBlock) void k_deg2_tiles(const int32_t* __restrict__ end,
                                                       const uint32_t* __restrict__ off,
                                                       int64_t m, uint4* __restrict__ deg,
                                                       uint64_t* __restrict__ tile_sums,
                                                       const uint32_t* __restrict__ gstatus) {
  if (*gstatus) return;
  __shared__ uint64_t s_w[kPBlock / kWave];
  const int64_t p0 = (int64_t)blockIdx.x * kPTile + (int64_t)threadIdx.x * kPItems;
  uint32_t d[kPItems];
#pragma unroll
  for (int j = 0; j < kPItems; ++j) {
    uint2 o{0, 0};
    if (p0 + j < m) __builtin_memcpy(&o, off + end[p0 + j], sizeof(o));  // off[x], off[x + 1]
    d[j] = o.y - o.x;
  }
  uint64_t s = 0;
#pragma unroll
  for (int j = 0; j < kPItems; ++j) {
    d[j] = d[j] < 65535u ? d[j] : 65535u;
    s += (uint64_t)d[j] * d[j];
  }
  if (p0 < m)  // whole groups of eight: the scratch is padded to them
    deg[p0 / kPItems] = make_uint4(d[0] | d[1] << 16, d[2] | d[3] << 16, d[4] | d[5] << 16,
                                   d[6] | d[7] << 16);
  s = wave_sum64(s);
  if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t t = 0;
    for (int w = 0; w < kPBlock / kWave; ++w) t += s_w[w];
    tile_sums[blockIdx.x] = t;
  }
}

// one block: exclusive wrapping scan of the tile sums (in place)
__global__ __launch_bounds__(1024) void k_deg2_scan_tiles(uint64_t* __restrict__ tile_sums,
                                                          int64_t ntiles) {
  __shared__ uint64_t s_w[16];
  __shared__ uint64_t s_carry;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < ntiles; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const uint64_t v = i < ntiles ? tile_sums[i] : 0;
    const uint64_t inc = wave_inclusive_scan(v);
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    uint64_t pre = s_carry;
    for (int w = 0; w < wave; ++w) pre += s_w[w];
    if (i < ntiles) tile_sums[i] = pre + inc - v;
    __syncthreads();
    if (threadIdx.x == 1023) s_carry = pre + inc;
    __syncthreads();
  }
}

// Per tile: inclusive prefix sums (wrapping) of the squared degrees.  With T
// (the out-CSR) each is stored beside the entry's time, ps[2 i] and
// ps[2 i + 1]: a window's last entry then gives its sum and its latest time
// in one access.
template <bool T>
__global__ __launch_bounds__(kPBlock) void k_deg2_apply(const uint4* __restrict__ deg, int64_t m,
                                                       const uint64_t* __restrict__ tile_off,
                                                       const int64_t* __restrict__ t_col,
                                                       uint64_t* __restrict__ ps,
                                                       const uint32_t* __restrict__ gstatus) {
  if (*gstatus) return;
  __shared__ uint64_t s_w[kPBlock / kWave];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t p0 = (int64_t)blockIdx.x * kPTile + (int64_t)threadIdx.x * kPItems;
  uint4 q{0, 0, 0, 0};
  if (p0 < m) q = deg[p0 / kPItems];
  int64_t t[kPItems];
#pragma unroll
  for (int j = 0; j < kPItems; ++j) t[j] = T && p0 + j < m ? t_col[p0 + j] : 0;
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
  uint64_t v[kPItems];
  uint64_t s = 0;
#pragma unroll
  for (int j = 0; j < kPItems; ++j) {
    const uint64_t d = (w[j >> 1] >> (16 * (j & 1))) & 0xFFFFu;
    s += d * d;
    v[j] = s;
  }
  const uint64_t inc = wave_inclusive_scan(s);
  if (lane == 63) s_w[wave] = inc;
  __syncthreads();
  uint64_t run = tile_off[blockIdx.x] + inc - s;
  for (int k = 0; k < wave; ++k) run += s_w[k];
#pragma unroll
  for (int j = 0; j < kPItems; ++j) {
    if (p0 + j >= m) break;
    if (T)
      reinterpret_cast<ulonglong2*>(ps)[p0 + j] = make_ulonglong2(run + v[j], (uint64_t)t[j]);
    else
      ps[p0 + j] = run + v[j];
  }
}

// [start, end) of the run of `key` given the slot at its home position
__device__ __forceinline__ void run_from(const PairSlot* __restrict__ tab, int log2cap,
                                         uint64_t key, PairSlot sl, uint32_t* start,
                                         uint32_t* end) {
  const uint64_t mask = (1ull << log2cap) - 1;
  uint64_t h = pair_hash(key, log2cap);
  *start = *end = 0;
  for (uint64_t probe = 0; probe <= mask; ++probe) {
    if (sl.key == key) {
      *start = sl.start;
      *end = sl.end;
      return;
    }
    if (sl.key == kPairEmpty) return;
    h = (h + 1) & mask;
    sl = tab[h];
  }
}

// The random reads of an edge bound this kernel: the run-table slots of
// (u, v) and (v, u), the runs' times, and the ends of v's window.  The first
// four are issued together, the window's last entry holds its time and its
// prefix sum in one place, and the (u, v) run of a single edge is the edge
// itself, so its times are not read.  On the 2*10^7-edge graph: 2.21 -> 1.86 ms
// (the prefix sums before it: 0.71 -> 0.56 ms).
__global__ __launch_bounds__(256) void k_features(
    const int32_t* __restrict__ out_src, const int32_t* __restrict__ out_dst,
    const int64_t* __restrict__ out_t, const int64_t* __restrict__ in_t,
    const int64_t* __restrict__ pair_t, const int64_t* __restrict__ pair_skip,
    const PairSlot* __restrict__ pair_hash_tab, int32_t pair_hash_log2,
    const uint32_t* __restrict__ lo_in, const uint32_t* __restrict__ a,
    const uint32_t* __restrict__ lo_out, const uint32_t* __restrict__ b,
    const uint64_t* __restrict__ ps_in, const ulonglong2* __restrict__ ps_out, int64_t delta,
    int64_t m, uint4* __restrict__ feat, const uint32_t* __restrict__ gstatus) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= m || *gstatus) return;
  const int32_t u = out_src[p], v = out_dst[p];
  const int64_t t = out_t[p];
  const uint32_t ap = a[p], bp = b[p], li = lo_in[p], lo = lo_out[p];
  const uint64_t kuv = pair_key((uint32_t)u, (uint32_t)v), kvu = pair_key((uint32_t)v, (uint32_t)u);
  const PairSlot suv = pair_hash_tab[pair_hash(kuv, pair_hash_log2)];
  const PairSlot svu = pair_hash_tab[pair_hash(kvu, pair_hash_log2)];
  const ulonglong2 none = make_ulonglong2(0, 0);
  const ulonglong2 last = bp ? ps_out[lo + bp - 1] : none;  // {sum, time} at the window's end
  const uint64_t before_out = bp && lo ? ps_out[lo - 1].x : 0;
  const uint64_t sum_in = ap ? ps_in[li + ap - 1] - (li ? ps_in[li - 1] : 0) : 0;
  const int64_t first_t = ap ? in_t[li] : 0;
  float f[8];
  f[0] = log1pf((float)ap);
  f[1] = log1pf((float)bp);
  f[2] = log1pf((float)((uint64_t)ap * (uint64_t)bp));
  f[3] = (ap > 0 && delta > 0) ? (float)(t - first_t) / (float)delta : 0.0f;
  f[4] = (bp > 0 && delta > 0) ? (float)((int64_t)last.y - t) / (float)delta : 0.0f;
  // multi-edge counts in [t - delta, t + delta] (integer times: "from
  // t - delta on" is "after t - delta - 1")
  uint32_t r0, r1, w0, w1;
  run_from(pair_hash_tab, pair_hash_log2, kuv, suv, &r0, &r1);
  uint32_t n_uv = 1;
  if (r1 - r0 > 1) {
    run_window(pair_t, pair_skip, m, r0, r1, t - delta - 1, t + delta, &w0, &w1);
    n_uv = w1 - w0;
  }
  f[5] = log1pf((float)n_uv);
  run_from(pair_hash_tab, pair_hash_log2, kvu, svu, &r0, &r1);
  uint32_t n_vu = 0;
  if (r1 > r0) {
    run_window(pair_t, pair_skip, m, r0, r1, t - delta - 1, t + delta, &w0, &w1);
    n_vu = w1 - w0;
  }
  f[6] = log1pf((float)n_vu);
  // mean squared degree of the window ends (exact wrapping window sums)
  const double m_in = ap ? (double)sum_in / (double)ap : 0.0;
  const double m_out = bp ? (double)(last.x - before_out) / (double)bp : 0.0;
  f[7] = (float)(0.5 * log1p(m_in * m_out));
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    w[i] = (uint32_t)bf16_bits(f[2 * i]) | ((uint32_t)bf16_bits(f[2 * i + 1]) << 16);
  feat[p] = make_uint4(w[0], w[1], w[2], w[3]);
}

// ------------------------------------------------------------ MLP pieces --
// Per-lane operand registers of the two MFMA layers.
struct MlpOps {
  s16x4 w1[2];      // layer 1, output block rb: W1[32 rb + i][4 h + s]
  bf16x8 w2[2][4];  // layer 2, output block ob, K-chunk kc: W2[32 ob + i][krow(kc, s, h)]
};

// four consecutive parameters (no alignment beyond a float's is assumed)
struct F4 {
  float v[4];
};
__device__ __forceinline__ F4 load4(const float* __restrict__ p) {
  F4 r;
  __builtin_memcpy(&r, p, sizeof(r));
  return r;
}

__device__ void load_ops(const float* __restrict__ P, int lane, MlpOps* o) {
  const int i = lane & 31, h = lane >> 5;
  F4 q1[2], q2[2][4][2];  // every load issued before the first conversion
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) q1[rb] = load4(P + kOffW1 + (32 * rb + i) * kIn + 4 * h);
#pragma unroll
  for (int ob = 0; ob < 2; ++ob)
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
#pragma unroll
      for (int g = 0; g < 2; ++g)  // krow is consecutive over s = 4 g .. 4 g + 3
        q2[ob][kc][g] = load4(P + kOffW2 + (32 * ob + i) * kHid + krow(kc, 4 * g, h));
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    s16x4 v;
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = (short)bf16_bits(q1[rb].v[s]);
    o->w1[rb] = v;
  }
#pragma unroll
  for (int ob = 0; ob < 2; ++ob)
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) {
      uint16_t e[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) e[s] = bf16_bits(q2[ob][kc][s >> 2].v[s & 3]);
      o->w2[ob][kc] = pack8(e);
    }
}

// small vectors in LDS: b1, b2 (float32), w3 (bfloat16-rounded), b3
struct MlpVecs {
  float b1[kHid], b2[kHid], w3[kHid], b3;
};

__device__ void load_vecs(const float* __restrict__ P, MlpVecs* s) {
  for (int i = threadIdx.x; i < kHid; i += blockDim.x) {
    s->b1[i] = P[kOffB1 + i];
    s->b2[i] = P[kOffB2 + i];
    s->w3[i] = bf16_round(P[kOffW3 + i]);
  }
  if (threadIdx.x == 0) s->b3 = P[kOffB3];
}

struct Fwd {
  f32x16 z1[2], z2[2];
  bf16x8 h1[4];  // layer-2 B operand chunks (relu(z1) in bfloat16)
  uint32_t h2[2][8];  // relu(z2) in bfloat16, two per word
  float z3;
};

// max(x, 0), 0 for NaN, as one instruction: the median of x, 0 and `inf`, a
// register that holds +inf without the compiler knowing it (fmaxf, and a
// median it can see through, take two: a maximum first quietens a signalling
// NaN that its operand might hold)
__device__ __forceinline__ float opaque_inf() {
  float v;
  asm("v_mov_b32 %0, 0x7f800000" : "=v"(v));
  return v;
}
__device__ __forceinline__ float reluf(float x, float inf) {
  return __builtin_amdgcn_fmed3f(x, 0.0f, inf);
}

// relu of an accumulator block, rounded to bfloat16: two K-chunks of the next
// layer's B operand
__device__ __forceinline__ void relu_pack(const f32x16& z, float inf, bf16x8* out) {
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    uint32_t q[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      q[e] = bf16x2_bits(reluf(z[8 * c + 2 * e], inf), reluf(z[8 * c + 2 * e + 1], inf));
    out[c] = __builtin_bit_cast(bf16x8, uint4{q[0], q[1], q[2], q[3]});
  }
}

// forward of 32 edges; fb = features 4h..4h+3 of edge lane % 32
__device__ __forceinline__ void mlp_fwd(const MlpOps& o, const MlpVecs& sv, s16x4 fb, int h,
                                        Fwd* r) {
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    f32x16 c;
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = sv.b1[32 * rb + drow(v, h)];
    r->z1[rb] = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(o.w1[rb], fb, c, 0, 0, 0);
  }
  const float inf = opaque_inf();
  relu_pack(r->z1[0], inf, &r->h1[0]);
  relu_pack(r->z1[1], inf, &r->h1[2]);
  float part = 0.0f;
#pragma unroll
  for (int ob = 0; ob < 2; ++ob) {
    f32x16 c;
#pragma unroll
    for (int v = 0; v < 16; ++v) c[v] = sv.b2[32 * ob + drow(v, h)];
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.w2[ob][kc], r->h1[kc], c, 0, 0, 0);
    r->z2[ob] = c;
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const uint32_t pr = bf16x2_bits(reluf(c[v], inf), reluf(c[v + 1], inf));
      r->h2[ob][v >> 1] = pr;
      part += sv.w3[32 * ob + drow(v, h)] * __uint_as_float(pr << 16);
      part += sv.w3[32 * ob + drow(v + 1, h)] * __uint_as_float(pr & 0xFFFF0000u);
    }
  }
  part += __shfl_xor(part, 32, kWave);
  r->z3 = part + sv.b3;
}

__device__ __forceinline__ float sigmoidf(float z) { return 1.0f / (1.0f + expf(-z)); }
__device__ __forceinline__ s16x4 load_feat4(const uint16_t* __restrict__ feat, int64_t row, int h) {
  const uint2 q = *reinterpret_cast<const uint2*>(feat + row * kIn + 4 * h);
  s16x4 v;
  v[0] = (short)(q.x & 0xFFFF);
  v[1] = (short)(q.x >> 16);
  v[2] = (short)(q.y & 0xFFFF);
  v[3] = (short)(q.y >> 16);
  return v;
}

constexpr int kAhead = 4;

// g for n rows of features (inference).  The two MFMA layers need 320 cycles
// of matrix core per 32 rows; what bounded the kernel was the vector and LDS
// work beside them: biases and w3 read from LDS in every tile and moved into
// the accumulators, and the last layer's dot product.  Here the biases stay in
// registers as the MFMAs' C operand (D is a different register block, so
// nothing is copied), and the dot product is one more MFMA chain whose A
// operand has w3 in row 0; per 32 rows the vector unit is left with the ReLUs,
// the roundings and one sigmoid.  The operands leave two wavefronts per SIMD,
// so each keeps the features of its next kAhead tiles in flight.  2*10^7
// rows: 511 -> 293 us (640 TFLOP/s); 345 us with one tile in flight.
__global__ __launch_bounds__(256, 2) void k_mlp_forward(const float* __restrict__ P,
                                                        const uint16_t* __restrict__ feat,
                                                        int64_t n, float* __restrict__ g) {
  MlpOps o;
  const int lane = threadIdx.x & 63, h = lane >> 5, i = lane & 31;
  load_ops(P, lane, &o);
  f32x16 c1[2], c2[2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      c1[b][v] = P[kOffB1 + 32 * b + drow(v, h)];
      c2[b][v] = P[kOffB2 + 32 * b + drow(v, h)];
    }
  bf16x8 w3[4];  // A operand of the last layer: row 0 is w3, the others are zero
#pragma unroll
  for (int kc = 0; kc < 4; ++kc) {
    uint16_t e[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) e[s] = i == 0 ? bf16_bits(P[kOffW3 + krow(kc, s, h)]) : (uint16_t)0;
    w3[kc] = pack8(e);
  }
  const float b3 = P[kOffB3];
  const float inf = opaque_inf();
  const int64_t tiles = (n + 31) / 32;
  const int64_t wstride = (int64_t)gridDim.x * (blockDim.x / kWave);
  // the wavefront index is uniform across its lanes, so the tile loop
  // branches as a whole
  const int64_t wave_id = (int64_t)blockIdx.x * (blockDim.x / kWave) + uni(threadIdx.x >> 6);
  auto rows_of = [&](int64_t tile) -> s16x4 {
    const int64_t row = tile * 32 + i;
    return tile < tiles && row < n ? load_feat4(feat, row, h) : s16x4{0, 0, 0, 0};
  };
  // kAhead tiles are in flight while kAhead are computed (2,048 wavefronts of
  // one 512-byte tile each would leave the memory latency uncovered)
  s16x4 next[kAhead];
#pragma unroll
  for (int q = 0; q < kAhead; ++q) next[q] = rows_of(wave_id + q * wstride);
  for (int64_t t0 = wave_id; t0 < tiles; t0 += kAhead * wstride) {
    s16x4 cur[kAhead];
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      cur[q] = next[q];
      next[q] = rows_of(t0 + (kAhead + q) * wstride);
    }
#pragma unroll
    for (int q = 0; q < kAhead; ++q) {
      const int64_t tile = t0 + q * wstride;
      if (tile >= tiles) break;  // uniform over the wavefront
      bf16x8 x[4];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const f32x16 z = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(o.w1[b], cur[q], c1[b], 0, 0, 0);
        relu_pack(z, inf, &x[2 * b]);
      }
      bf16x8 y[4];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        f32x16 z = c2[b];
#pragma unroll
        for (int kc = 0; kc < 4; ++kc)
          z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(o.w2[b][kc], x[kc], z, 0, 0, 0);
        relu_pack(z, inf, &y[2 * b]);
      }
      f32x16 d = f32x16{};
#pragma unroll
      for (int kc = 0; kc < 4; ++kc)
        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w3[kc], y[kc], d, 0, 0, 0);
      const int64_t row = tile * 32 + i;
      if (h == 0 && row < n) g[row] = sigmoidf(d[0] + b3);  // row 0 of column i
    }
  }
}

// ------------------------------------------------------------ gradients ----
constexpr int kGradBlock = 256;
constexpr int kGradWaves = kGradBlock / kWave;
constexpr int kTS = 40;  // LDS row stride (bfloat16 entries) of a 64 x 32 tile

struct GradLds {
  MlpVecs sv;
  // W2 in bfloat16 as MFMA A operands, eight entries of a lane together at
  // ((block 4 + kc) 2 + h) 32 + i: W2[32 ob + i][krow(kc, 0..7, h)] for the
  // forward layer and W2[krow(kc, 0..7, h)][32 kb + i] for dH1 = W2^T dZ2
  bf16x8 w2f[2 * 4 * 2 * 32], w2t[2 * 4 * 2 * 32];
  alignas(16) uint16_t dz2[kGradWaves][kHid * kTS];
  alignas(16) uint16_t h1[kGradWaves][kHid * kTS];
  alignas(16) uint16_t dz1[kGradWaves][kHid * kTS];
  alignas(16) uint16_t f[kGradWaves][32 * 8];
  alignas(16) float red[kGradWaves][kNParams + 1];
};

// Label row of item i of the current batch: index = (mul * (start + i) + add)
// mod n of the label arrays (a bijection of [0, n) when gcd(mul, n) = 1).
struct BatchMap {
  uint64_t mul, base, n;  // base = (mul * start + add) mod n
  double inv_n;
  uint32_t count;
  uint64_t n_feat;  // feature rows; labels whose row is outside are ignored
  float label_cap;  // 0: y = [X > 0]; else y = min(1, X / label_cap)
};

static BatchMap batch_map(uint64_t mul, uint64_t add, uint64_t n, uint64_t start, uint32_t count,
                          uint64_t n_feat, float label_cap) {
  return BatchMap{mul, (mul * start + add) % n, n, 1.0 / (double)n, count, n_feat, label_cap};
}

// x = base + mul i stays below 2^53 (mul < n < 2^31 and i < 2^20 in training;
// mul = 1 otherwise), so its binary64 quotient by n is off by at most one.
__device__ __forceinline__ uint64_t batch_index(const BatchMap& bm, uint64_t i) {
  const uint64_t x = bm.base + bm.mul * i;
  int64_t r = (int64_t)(x - (uint64_t)((double)x * bm.inv_n) * bm.n);
  if (r < 0) r += (int64_t)bm.n;
  if (r >= (int64_t)bm.n) r -= (int64_t)bm.n;
  return (uint64_t)r;
}

// The label of lane i of a tile: its feature half-row and target.
struct Label {
  s16x4 fb;
  float y;
  bool valid;
};

__device__ __forceinline__ Label load_label(const BatchMap& bm, const uint16_t* __restrict__ feat,
                                            const uint32_t* __restrict__ rows,
                                            const uint64_t* __restrict__ X, uint32_t tile,
                                            uint32_t tiles, int i, int h) {
  const uint32_t item = tile * 32 + i;
  Label l{s16x4{0, 0, 0, 0}, 0.0f, false};
  if (tile < tiles && item < bm.count) {
    const uint64_t idx = batch_index(bm, item);
    const int64_t row = rows ? (int64_t)rows[idx] : (int64_t)idx;
    const uint64_t xv = X[idx];
    l.valid = (uint64_t)row < bm.n_feat;
    if (l.valid) l.fb = load_feat4(feat, row, h);
    l.y = bm.label_cap > 0.0f ? fminf(1.0f, __fdiv_rn((float)xv, bm.label_cap))
                              : (xv != 0 ? 1.0f : 0.0f);
  }
  return l;
}

// Sum over the 32 lanes of each half of 64 values per lane, spread out: at
// step OFF a lane keeps half of its values and adds the copies of them that
// lane i ^ OFF holds, so the 64 sums cost 92 additions and 94 selects instead of
// 320 additions (a DPP step adds both candidates and selects afterwards), each
// formed by the same tree as a butterfly over the lanes.  Lane i is left with
// the sums of values 2 i and 2 i + 1 in val[0] and val[1].  Inside a row of 16
// lanes the other lane's value is a DPP operand (rotations by 8, by 12 or 4,
// quad permutations); rows are exchanged by a bpermute.
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(
      0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, true));
}
// CLO brings lane i + OFF of the row to a lane with (i & OFF) = 0, CHI lane
// i - OFF to the others
template <int OFF, int CLO, int CHI>
__device__ __forceinline__ void half_sum_step(float (&val)[64], int i) {
  const bool up = (i & OFF) != 0;
#pragma unroll
  for (int k = 0; k < 2 * OFF; ++k) {
    const float lo = val[k] + dpp_f32<CLO>(val[k]);
    const float hi = val[k + 2 * OFF] + dpp_f32<CHI>(val[k + 2 * OFF]);
    val[k] = up ? hi : lo;
  }
}
__device__ __forceinline__ void half_sums64(float (&val)[64], int i) {
#pragma unroll
  for (int k = 0; k < 32; ++k) {
    const bool up = (i & 16) != 0;
    const float send = up ? val[k] : val[k + 32];
    const float keep = up ? val[k + 32] : val[k];
    val[k] = keep + __shfl_xor(send, 16, kWave);
  }
  half_sum_step<8, 0x128, 0x128>(val, i);
  half_sum_step<4, 0x12C, 0x124>(val, i);
  half_sum_step<2, 0x4E, 0x4E>(val, i);
  half_sum_step<1, 0xB1, 0xB1>(val, i);
}

// Partial loss and gradient of one block over its tiles of the batch; the
// tile-to-block assignment depends only on the launch shape.  A batch of
// 8,192 labels is one tile per wavefront on 64 blocks, so the launch is as
// long as one wavefront's chain of label gathers, layers and sums: the first
// tile's labels are fetched before the parameters, the sums over a tile's 32
// edges are spread over the lanes, and every operand is read as 16-byte
// words.  At 8,192 labels 37.3 -> 13.2 us.
__global__ __launch_bounds__(kGradBlock) void k_mlp_grad(const float* __restrict__ P,
                                                         const uint16_t* __restrict__ feat,
                                                         const uint32_t* __restrict__ rows,
                                                         const uint64_t* __restrict__ X,
                                                         BatchMap bm,
                                                         float* __restrict__ partial) {
  extern __shared__ char s_raw[];
  GradLds& L = *reinterpret_cast<GradLds*>(s_raw);
  const int lane = threadIdx.x & 63, h = lane >> 5, i = lane & 31;
  const int wave = (int)uni(threadIdx.x >> 6);
  const uint32_t tiles = (bm.count + 31) / 32;
  const uint32_t first = blockIdx.x * kGradWaves + wave;
  Label lab = load_label(bm, feat, rows, X, first, tiles, i, h);
  load_vecs(P, &L.sv);
  // every operand is read from memory once per block
  constexpr int kSlots = 2 * 4 * 2 * 32 / kGradBlock;
  F4 qf[kSlots][2];
  float qt[kSlots][8];
  F4 q1[2];
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    const int sl = q * kGradBlock + threadIdx.x;
    const int si = sl & 31, sh = (sl >> 5) & 1, kc = (sl >> 6) & 3, b = sl >> 8;
#pragma unroll
    for (int g = 0; g < 2; ++g)  // krow is consecutive over s = 4 g .. 4 g + 3
      qf[q][g] = load4(P + kOffW2 + (32 * b + si) * kHid + krow(kc, 4 * g, sh));
#pragma unroll
    for (int s = 0; s < 8; ++s) qt[q][s] = P[kOffW2 + krow(kc, s, sh) * kHid + 32 * b + si];
  }
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) q1[rb] = load4(P + kOffW1 + (32 * rb + i) * kIn + 4 * h);
#pragma unroll
  for (int q = 0; q < kSlots; ++q) {
    uint16_t ef[8], et[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      ef[s] = bf16_bits(qf[q][s >> 2].v[s & 3]);
      et[s] = bf16_bits(qt[q][s]);
    }
    L.w2f[q * kGradBlock + threadIdx.x] = pack8(ef);
    L.w2t[q * kGradBlock + threadIdx.x] = pack8(et);
  }
  MlpOps o;
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    s16x4 v;
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = (short)bf16_bits(q1[rb].v[s]);
    o.w1[rb] = v;
  }
  __syncthreads();
#pragma unroll
  for (int ob = 0; ob < 2; ++ob)
#pragma unroll
    for (int kc = 0; kc < 4; ++kc) o.w2[ob][kc] = L.w2f[((ob * 4 + kc) * 2 + h) * 32 + i];
  const float inv_n = 1.0f / (float)bm.count;
  f32x16 gW2[2][2], gW1[2];
#pragma unroll
  for (int a2 = 0; a2 < 2; ++a2) {
    gW1[a2] = f32x16{};
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2) gW2[a2][b2] = f32x16{};
  }
  float gb3 = 0.0f, loss = 0.0f;
  float g32[2] = {0.0f, 0.0f};  // this lane's two of the w3 and b2 gradients (half_sums64)
  uint16_t* tdz2 = L.dz2[wave];
  uint16_t* th1 = L.h1[wave];
  uint16_t* tdz1 = L.dz1[wave];
  uint16_t* tf = L.f[wave];
  const uint32_t stride = gridDim.x * kGradWaves;
  for (uint32_t tile = first; tile < tiles; tile += stride) {  // uniform over the wavefront
    const s16x4 fb = lab.fb;
    const bool valid = lab.valid;
    const float y = lab.y;
    if (tile + stride < tiles) lab = load_label(bm, feat, rows, X, tile + stride, tiles, i, h);
    Fwd r;
    mlp_fwd(o, L.sv, fb, h, &r);
    const float gz = sigmoidf(r.z3);
    const float dz3 = valid ? (gz - y) * inv_n : 0.0f;
    if (h == 0 && valid) {
      // the two softplus terms share log1p(exp(-|z|))
      const float tail = log1pf(expf(-fabsf(r.z3)));
      loss += y * (fmaxf(-r.z3, 0.0f) + tail) + (1.0f - y) * (fmaxf(r.z3, 0.0f) + tail);
      gb3 += dz3;
    }
    // layer 3 and dZ2 (registers, rows drow(v, h) of block ob, edge i); the
    // w3 and b2 gradients are summed over the tile's 32 edges right away
    bf16x8 dzc[4];  // dZ2 in bfloat16: the B operand of dH1
    float val[64];  // w3 terms, then b2 terms, 16 ob + v each
#pragma unroll
    for (int ob = 0; ob < 2; ++ob) {
      uint32_t pk[8];
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        float d[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          d[e] = r.z2[ob][v + e] > 0.0f ? L.sv.w3[32 * ob + drow(v + e, h)] * dz3 : 0.0f;
          val[32 + 16 * ob + v + e] = d[e];
        }
        const uint32_t pr = r.h2[ob][v >> 1];
        val[16 * ob + v] = dz3 * __uint_as_float(pr << 16);
        val[16 * ob + v + 1] = dz3 * __uint_as_float(pr & 0xFFFF0000u);
        pk[v >> 1] = bf16x2_bits(d[0], d[1]);
      }
#pragma unroll
      for (int c = 0; c < 2; ++c)
        dzc[2 * ob + c] = __builtin_bit_cast(
            bf16x8, uint4{pk[4 * c], pk[4 * c + 1], pk[4 * c + 2], pk[4 * c + 3]});
    }
    half_sums64(val, i);
    g32[0] += val[0];
    g32[1] += val[1];
    // dH1 = W2^T dZ2, then dZ1 = dH1 * [z1 > 0]
    // stage dZ2, H1, dZ1 and F with edges along rows for the weight gradients
    // (each wavefront its own tiles)
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      f32x16 c = f32x16{};
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(L.w2t[((kb * 4 + kc) * 2 + h) * 32 + i],
                                                    dzc[kc], c, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const int r0 = (32 * kb + drow(v, h)) * kTS + i, r1 = r0 + kTS;  // rows of v, v + 1
        const uint32_t pd = bf16x2_bits(r.z1[kb][v] > 0.0f ? c[v] : 0.0f,
                                        r.z1[kb][v + 1] > 0.0f ? c[v + 1] : 0.0f);
        const s16x8 ph = __builtin_bit_cast(s16x8, r.h1[2 * kb + (v >> 3)]);
        const s16x8 pz = __builtin_bit_cast(s16x8, dzc[2 * kb + (v >> 3)]);
        tdz1[r0] = (uint16_t)pd;
        tdz1[r1] = (uint16_t)(pd >> 16);
        th1[r0] = (uint16_t)ph[v & 7];
        th1[r1] = (uint16_t)ph[(v & 7) + 1];
        tdz2[r0] = (uint16_t)pz[v & 7];
        tdz2[r1] = (uint16_t)pz[(v & 7) + 1];
      }
    }
    {
      const uint2 q = {(uint32_t)(uint16_t)fb[0] | ((uint32_t)(uint16_t)fb[1] << 16),
                       (uint32_t)(uint16_t)fb[2] | ((uint32_t)(uint16_t)fb[3] << 16)};
      *reinterpret_cast<uint2*>(tf + i * 8 + 4 * h) = q;
    }
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();
    // dW2[32 ob + .][32 kb + .] += dZ2 H1^T and [dW1 | db1] += dZ1 [F | 1]^T,
    // contracting over the 32 edges (two K-chunks of 16)
#pragma unroll
    for (int e2 = 0; e2 < 2; ++e2) {
      const int col = 16 * e2 + 8 * h;
      bf16x8 Ad[2], Bh[2];
#pragma unroll
      for (int x2 = 0; x2 < 2; ++x2) {
        Ad[x2] = *reinterpret_cast<const bf16x8*>(tdz2 + (32 * x2 + i) * kTS + col);
        Bh[x2] = *reinterpret_cast<const bf16x8*>(th1 + (32 * x2 + i) * kTS + col);
      }
#pragma unroll
      for (int ob = 0; ob < 2; ++ob)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
          gW2[ob][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Ad[ob], Bh[kb], gW2[ob][kb], 0, 0, 0);
      // B of [F | 1]^T: column i < 8 is feature i of the edges, column 8 is 1
      uint16_t e[8];
#pragma unroll
      for (int s = 0; s < 8; ++s)
        e[s] = i < 8 ? tf[(col + s) * 8 + i] : (i == 8 ? (uint16_t)0x3F80u : (uint16_t)0);
      const bf16x8 Bf = pack8(e);
#pragma unroll
      for (int rb = 0; rb < 2; ++rb) {
        const bf16x8 A1 = *reinterpret_cast<const bf16x8*>(tdz1 + (32 * rb + i) * kTS + col);
        gW1[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A1, Bf, gW1[rb], 0, 0, 0);
      }
    }
    __threadfence_block();
    __builtin_amdgcn_wave_barrier();  // the next tile rewrites the staged ones
  }
  // per-wave partials into LDS, then the block sum in wave order
  float* red = L.red[wave];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int k = 2 * i + e, v = k & 15, ob = (k >> 4) & 1;
    red[(k & 32 ? kOffB2 : kOffW3) + 32 * ob + drow(v, h)] = g32[e];
  }
#pragma unroll
  for (int ob = 0; ob < 2; ++ob)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int rr = 32 * ob + drow(v, h);
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) red[kOffW2 + rr * kHid + 32 * kb + i] = gW2[ob][kb][v];
      if (i < 8) red[kOffW1 + rr * kIn + i] = gW1[ob][v];
      if (i == 8) red[kOffB1 + rr] = gW1[ob][v];
    }
  {
    float s3 = gb3, sl = loss;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      s3 += __shfl_xor(s3, off, kWave);
      sl += __shfl_xor(sl, off, kWave);
    }
    if (lane == 0) {
      red[kOffB3] = s3;
      red[kNParams] = sl;
    }
  }
  __syncthreads();
  // two parameters per thread and round (an even row length)
  static_assert((kNParams + 1) % 2 == 0, "pairs of a partial row");
  for (int j = threadIdx.x; j < (kNParams + 1) / 2; j += kGradBlock) {
    float2 s{0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < kGradWaves; ++w) {
      const float2 v = *reinterpret_cast<const float2*>(&L.red[w][2 * j]);
      s.x += v.x;
      s.y += v.y;
    }
    reinterpret_cast<float2*>(partial + (size_t)blockIdx.x * (kNParams + 1))[j] = s;
  }
}

size_t mlp_grad_lds_bytes() { return sizeof(GradLds); }

// Sum of the block partials in block order.  mode 0: grad[j] and *loss;
// mode 1: one Adam step on params with moments opt[0..n), opt[n..2n).
struct AdamArgs {
  float lr, beta1, beta2, eps;
  float omb1, omb2;  // 1 - beta, formed in binary64 and rounded once
  float bc1, bc2;    // 1 - beta^step
};

// One thread per parameter.  Its partials (1.2 MB over 64 blocks, mostly from
// other XCDs' writes) are fetched 32 at a time and added in block order: the
// launch takes two or three memory round trips instead of one per few
// blocks (64 blocks' partials: 16.6 -> 5.1 us).
constexpr int kReduceBlock = 64;
constexpr int kReduceGrid = (kNParams + kReduceBlock) / kReduceBlock;
__global__ __launch_bounds__(kReduceBlock) void k_mlp_reduce(
    const float* __restrict__ partial, int nblocks, int mode, float* __restrict__ grad,
    float* __restrict__ loss, float loss_scale, float* __restrict__ params,
    float* __restrict__ opt, AdamArgs ad) {
  const int j = blockIdx.x * kReduceBlock + threadIdx.x;
  if (j > kNParams || (j == kNParams && !loss)) return;
  const bool adam = mode == 1 && j < kNParams;
  const float o1 = adam ? opt[j] : 0.0f, o2 = adam ? opt[kNParams + j] : 0.0f;
  const float p0 = adam ? params[j] : 0.0f;
  float s = 0.0f;
  constexpr int kAtOnce = 32;
  for (int b0 = 0; b0 < nblocks; b0 += kAtOnce) {
    float v[kAtOnce];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q)
      v[q] = b0 + q < nblocks ? partial[(size_t)(b0 + q) * (kNParams + 1) + j] : 0.0f;
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q)
      if (b0 + q < nblocks) s += v[q];
  }
  if (j == kNParams) {
    // loss: sum over rows / batch size, scaled (e.g. 1 / batches per epoch)
    *loss += s * loss_scale;
    return;
  }
  if (mode == 0) {
    grad[j] = s;
    return;
  }
  const float mj = ad.beta1 * o1 + ad.omb1 * s;
  const float vj = ad.beta2 * o2 + ad.omb2 * (s * s);
  opt[j] = mj;
  opt[kNParams + j] = vj;
  const float mh = mj / ad.bc1, vh = vj / ad.bc2;
  params[j] = p0 - ad.lr * mh / (sqrtf(vh) + ad.eps);
}

__global__ void k_zero_f32(float* p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0f;
}

// ----------------------------------------------------------- quantisation --
// g clamped to [0, 1] (NaN read as 0)
__device__ __forceinline__ float clamp_score(float x) {
  if (!(x >= 0.0f)) x = 0.0f;
  return x > 1.0f ? 1.0f : x;
}

// max of the clamped scores (non-negative floats order like their bit patterns)
__global__ __launch_bounds__(256) void k_score_max(const float* __restrict__ g, int64_t m,
                                                   uint32_t* __restrict__ gmax_bits) {
  __shared__ uint32_t s_max;
  if (threadIdx.x == 0) s_max = 0u;
  __syncthreads();
  uint32_t b = 0u;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < m;
       p += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t v = __float_as_uint(clamp_score(g[p]));
    b = v > b ? v : b;
  }
  atomicMax(&s_max, b);
  __syncthreads();
  if (threadIdx.x == 0) atomicMax(gmax_bits, s_max);
}

__global__ void k_zero_u32(uint32_t* p) { *p = 0u; }

__global__ __launch_bounds__(256) void k_quantize(const float* __restrict__ g, int64_t m,
                                                  float eps, const uint64_t* __restrict__ S,
                                                  const float* __restrict__ gmax,
                                                  uint32_t* __restrict__ hq) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= m) return;
  const uint64_t W = S[m];
  const int bitlen = W ? 64 - __clzll((long long)W) : 0;
  int s = 63 - bitlen;
  s = s < 1 ? 1 : (s > 16 ? 16 : s);
  float x = clamp_score(g[p]);
  if (gmax) {
    const float gm = *gmax;
    if (gm > 0.0f) x = __fdiv_rn(x, gm);
  }
  const float one_m = __fsub_rn(1.0f, eps);
  const float hv = __fadd_rn(eps, __fmul_rn(one_m, x));
  const float hs = __fmul_rn(hv, (float)(1u << s));
  const float r = floorf(__fadd_rn(hs, 0.5f));
  const uint32_t v = (uint32_t)r;
  hq[p] = v < 1u ? 1u : v;
}

// ------------------------------------------------------------- host side --
static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// prefix sums of the in-CSR (8 bytes per entry) and of the out-CSR with the
// times beside them (16), the capped degrees (2, in groups of eight), tiles
struct FeatLayout {
  size_t ps_in, ps_out, deg, tiles, total;
  int64_t ntiles;
};

static FeatLayout feat_layout(int64_t m) {
  FeatLayout L;
  L.ntiles = (m + kPTile - 1) / kPTile;
  L.ps_in = 0;
  L.ps_out = L.ps_in + align256((size_t)m * 8 + 8);
  L.deg = L.ps_out + align256((size_t)m * 16);
  L.tiles = L.deg + align256((size_t)((m + kPItems - 1) / kPItems) * 16);
  L.total = L.tiles + align256((size_t)L.ntiles * 8 + 8);
  return L;
}

size_t features_workspace_bytes(int64_t m) { return feat_layout(m).total; }

tc_status edge_features(const tc_graph* g, const tc_weights* w, uint16_t* feat, void* ws,
                        size_t ws_bytes, hipStream_t st) {
  const int64_t m = g->m;
  const FeatLayout L = feat_layout(m);
  if (ws_bytes < L.total) return TC_E_WORKSPACE;
  if (m == 0) return TC_OK;
  char* base = (char*)ws;
  uint64_t* ps_in = (uint64_t*)(base + L.ps_in);
  uint64_t* ps_out = (uint64_t*)(base + L.ps_out);
  uint4* deg = (uint4*)(base + L.deg);
  uint64_t* tiles = (uint64_t*)(base + L.tiles);
  const uint32_t* gst = (const uint32_t*)g->status;
  const dim3 grid((unsigned)L.ntiles), block(kPBlock);
  for (int side = 0; side < 2; ++side) {
    hipLaunchKernelGGL(k_deg2_tiles, grid, block, 0, st,
                       (const int32_t*)(side == 0 ? g->in_src : g->out_dst),
                       (const uint32_t*)(side == 0 ? g->in_off : g->out_off), m, deg, tiles, gst);
    hipLaunchKernelGGL(k_deg2_scan_tiles, dim3(1), dim3(1024), 0, st, tiles, L.ntiles);
    if (side == 0)
      hipLaunchKernelGGL(k_deg2_apply<false>, grid, block, 0, st, (const uint4*)deg, m,
                         (const uint64_t*)tiles, (const int64_t*)nullptr, ps_in, gst);
    else
      hipLaunchKernelGGL(k_deg2_apply<true>, grid, block, 0, st, (const uint4*)deg, m,
                         (const uint64_t*)tiles, (const int64_t*)g->out_t, ps_out, gst);
  }
  {
    TimedLaunch tl("k_features", st);
    hipLaunchKernelGGL(k_features, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st,
                       (const int32_t*)g->out_src, (const int32_t*)g->out_dst,
                       (const int64_t*)g->out_t, (const int64_t*)g->in_t,
                       (const int64_t*)g->pair_t, (const int64_t*)g->pair_skip,
                       (const PairSlot*)g->pair_hash, g->pair_hash_log2, w->lo_in, w->a,
                       w->lo_out, w->b, (const uint64_t*)ps_in, (const ulonglong2*)ps_out,
                       w->delta, m, (uint4*)feat, gst);
  }
  return hipGetLastError() == hipSuccess ? TC_OK : TC_E_HIP;
}

tc_status mlp_forward(const float* params, const uint16_t* feat, int64_t n, float* g,
                      hipStream_t st) {
  if (n > 0) {
    const int64_t tiles = (n + 31) / 32;
    int64_t blocks = (tiles + 3) / 4;
    // two resident blocks per CU: each loads the operands once
    if (blocks > 512) blocks = 512;
    TimedLaunch tl("k_mlp_forward", st);
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)blocks), dim3(256), 0, st, params, feat, n, g);
  }
  return hipGetLastError() == hipSuccess ? TC_OK : TC_E_HIP;
}

int mlp_grad_blocks(int64_t count) {
  const int64_t tiles = (count + 31) / 32;
  int64_t b = (tiles + kGradWaves - 1) / kGradWaves;
  if (b > 512) b = 512;
  return b < 1 ? 1 : (int)b;
}

size_t mlp_workspace_bytes(int64_t batch) {
  return (size_t)mlp_grad_blocks(batch) * (kNParams + 1) * sizeof(float);
}

static tc_status launch_grad(const float* params, const uint16_t* feat, const uint32_t* rows,
                             const uint64_t* X, const BatchMap& bm, float* partial,
                             hipStream_t st) {
  const int nb = mlp_grad_blocks(bm.count);
  if (hipFuncSetAttribute((const void*)k_mlp_grad, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)sizeof(GradLds)) != hipSuccess)
    return TC_E_HIP;
  TimedLaunch tl("k_mlp_grad", st);
  hipLaunchKernelGGL(k_mlp_grad, dim3((unsigned)nb), dim3(kGradBlock), sizeof(GradLds), st,
                     params, feat, rows, X, bm, partial);
  return TC_OK;
}

tc_status mlp_grad(const float* params, const uint16_t* feat, int64_t n_feat, const uint32_t* rows,
                   const uint64_t* X, int64_t n, float label_cap, float* grad, float* loss,
                   void* ws, size_t ws_bytes, hipStream_t st) {
  if (ws_bytes < mlp_workspace_bytes(n)) return TC_E_WORKSPACE;
  const BatchMap bm = batch_map(1, 0, (uint64_t)n, 0, (uint32_t)n, (uint64_t)n_feat, label_cap);
  float* partial = (float*)ws;
  tc_status s = launch_grad(params, feat, rows, X, bm, partial, st);
  if (s != TC_OK) return s;
  hipLaunchKernelGGL(k_zero_f32, dim3(1), dim3(64), 0, st, loss, 1);
  hipLaunchKernelGGL(k_mlp_reduce, dim3(kReduceGrid), dim3(kReduceBlock), 0, st,
                     (const float*)partial, mlp_grad_blocks(n), 0, grad, loss, 1.0f / (float)n,
                     (float*)nullptr, (float*)nullptr, AdamArgs{});
  return hipGetLastError() == hipSuccess ? TC_OK : TC_E_HIP;
}

static AdamArgs adam_args(int64_t step, float lr) {
  AdamArgs a;
  a.lr = lr;
  a.beta1 = 0.9f;
  a.beta2 = 0.999f;
  a.eps = 1e-8f;
  a.omb1 = (float)(1.0 - 0.9);
  a.omb2 = (float)(1.0 - 0.999);
  a.bc1 = (float)(1.0 - std::pow(0.9, (double)step));
  a.bc2 = (float)(1.0 - std::pow(0.999, (double)step));
  return a;
}

tc_status mlp_adam(float* params, float* opt, const float* grad, int64_t step, float lr,
                   hipStream_t st) {
  // the gradient is one "partial" of one block
  hipLaunchKernelGGL(k_mlp_reduce, dim3(kReduceGrid), dim3(kReduceBlock), 0, st, grad, 1, 1,
                     (float*)nullptr, (float*)nullptr, 0.0f, params, opt, adam_args(step, lr));
  return hipGetLastError() == hipSuccess ? TC_OK : TC_E_HIP;
}

static uint64_t gcd64(uint64_t a, uint64_t b) {
  while (b) {
    const uint64_t t = a % b;
    a = b;
    b = t;
  }
  return a;
}

tc_status mlp_train(float* params, float* opt, const uint16_t* feat, int64_t n_feat,
                    const uint32_t* rows, const uint64_t* X, int64_t n, float label_cap,
                    int32_t batch, int32_t epochs, float lr,
                    uint64_t seed, int64_t step0, float* loss_per_epoch, void* ws,
                    size_t ws_bytes, hipStream_t st) {
  if (ws_bytes < mlp_workspace_bytes(batch)) return TC_E_WORKSPACE;
  float* partial = (float*)ws;
  const int64_t nbatches = (n + batch - 1) / batch;
  if (loss_per_epoch)
    hipLaunchKernelGGL(k_zero_f32, dim3((epochs + 63) / 64), dim3(64), 0, st, loss_per_epoch,
                       epochs);
  int64_t step = step0;
  for (int32_t e = 0; e < epochs; ++e) {
    // a per-epoch bijection i -> (mul * i + add) mod n drawn from Philox
    const Words4 r = philox_block(seed, 0x4D4C5000u, (uint64_t)e, 0);
    uint64_t mul = n > 1 ? 1 + ((((uint64_t)r.x1 << 32) | r.x0) % (uint64_t)(n - 1)) : 1;
    while (gcd64(mul, (uint64_t)n) != 1) mul = mul + 1 < (uint64_t)n ? mul + 1 : 1;
    const uint64_t add = (((uint64_t)r.x3 << 32) | r.x2) % (uint64_t)n;
    for (int64_t bi = 0; bi < nbatches; ++bi) {
      const uint64_t start = (uint64_t)bi * (uint64_t)batch;
      const uint32_t count = (uint32_t)std::min<int64_t>(batch, n - (int64_t)start);
      const BatchMap bm =
          batch_map(mul, add, (uint64_t)n, start, count, (uint64_t)n_feat, label_cap);
      tc_status s = launch_grad(params, feat, rows, X, bm, partial, st);
      if (s != TC_OK) return s;
      ++step;
      hipLaunchKernelGGL(k_mlp_reduce, dim3(kReduceGrid), dim3(kReduceBlock), 0, st,
                         (const float*)partial, mlp_grad_blocks(count), 1, (float*)nullptr,
                         loss_per_epoch ? loss_per_epoch + e : (float*)nullptr,
                         1.0f / ((float)count * (float)nbatches), params, opt,
                         adam_args(step, lr));
    }
  }
  return hipGetLastError() == hipSuccess ? TC_OK : TC_E_HIP;
}

tc_status quantize_proposal(const tc_weights* w, const float* g, float eps, float* gmax,
                            uint32_t* hq, hipStream_t st) {
  const int64_t m = w->m;
  if (gmax) {
    hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(1), 0, st, (uint32_t*)gmax);
    if (m > 0) {
      int64_t blocks = (m + 255) / 256;
      if (blocks > 2048) blocks = 2048;
      hipLaunchKernelGGL(k_score_max, dim3((unsigned)blocks), dim3(256), 0, st, g, m,
                         (uint32_t*)gmax);
    }
  }
  if (m > 0)
    hipLaunchKernelGGL(k_quantize, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st, g, m, eps,
                       (const uint64_t*)w->S, (const float*)gmax, hq);
  return hipGetLastError() == hipSuccess ? TC_OK : TC_E_HIP;
}

}  // namespace tc
