// Temporal adjacency build: validation, stable LSD radix sorts and CSR
// offsets.  The canonical orders are (t, eid) -> (src, t, eid) for the
// out-lists, (dst, t, eid) for the in-lists and (src, dst, t, eid) for the
// per-pair lists; each later sort is a stable sort of the previous order, so
// timestamp ties keep increasing edge id (section III-A assumes time-sorted
// per-vertex lists; the tie order is this library's convention).
//
// Radix sort design (gfx950, wave64): every sort moves 16-byte edge
// records in tiles of 512 threads; the last pass of a vertex sort writes the
// graph's columns instead of records.  A pass is (1) per-tile digit
// histograms written tile-major (one contiguous row of counts per tile), (2)
// a column scan of that matrix that turns every count into the keys of its
// digit in the tiles before, (3) a scatter that ranks keys stably inside the
// tile with wavefront ballots (one ballot per digit bit gives the lanes
// sharing a digit), exchanges the tile through LDS into digit order and
// writes each digit run to its global slot with coalesced stores.  Digits
// have up to 11 bits: a pass costs about the same whatever its digit (the
// memory rate bounds it), so fewer, wider digits win as long as a tile still
// holds a few records per digit; the tile is as large as the LDS exchange
// allows for that reason.
//
// The whole build is one stream-ordered launch sequence: it allocates
// nothing, never waits on the device, and can be captured in a HIP graph.
// The validation result and the time range stay on the device; the time
// sort's passes read their plan from there (see BuildPlan).
#include <hip/hip_runtime.h>

#include "tc_device.h"
#include "tc_internal.h"
#include "tc_rules.h"

namespace tc {

constexpr int kSortBlock = 512;
constexpr int kSortWaves = kSortBlock / kWave;
constexpr uint32_t kXcds = 8;  // accelerator complex dies of an MI355X, each with its own L2
constexpr int kColChunk = 32;  // tiles per chunk of the histogram column scan
constexpr int kMaxDigit = 11;
constexpr int kMaxBins = 1 << kMaxDigit;
constexpr int kMinBins = 64;  // histogram rows are at least one 256-byte line
// Records per thread: tiles of 4,096 records, or of 2,048 where the larger
// ones would be too few to fill the CUs (1,000,001 edges: the build 262 us
// with small tiles, 280 with large; 2,000,001, where the small ones are past
// the one-launch column scan, 490 and 368).
constexpr int kItemsLarge = 8, kItemsSmall = 4;
constexpr int64_t kLargeFrom = (1 << 20) + 1;
static bool large_tiles(int64_t m) { return m >= kLargeFrom; }
static int64_t sort_tiles(int64_t m) {
  const int64_t t = (int64_t)kSortBlock * (large_tiles(m) ? kItemsLarge : kItemsSmall);
  return (m + t - 1) / t;
}

// XCD-aware tile order: workgroups are dealt to the XCDs round robin (block b
// to XCD b mod 8), and each XCD has its own L2.  Neighbouring tiles write
// neighbouring pieces of every digit run, so each XCD takes a contiguous range
// of the nb tiles: partial cache lines then meet in one L2 instead of being
// written back piecewise from several.
__device__ __forceinline__ uint32_t xcd_tile(uint32_t block, uint32_t nb) {
  const uint32_t xcd = block % kXcds, slot = block / kXcds;
  const uint32_t q = nb / kXcds, rem = nb % kXcds;
  return xcd * q + (xcd < rem ? xcd : rem) + slot;
}

static unsigned blocks_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

// ------------------------------------------------------------ validation ---
// What one block of the validation found; k_plan reduces them.
struct Found {
  uint64_t mn, mx;  // of order-preserving keys of the times
  uint32_t bad;
};
constexpr int kMaxFound = 1024;

// The validation, which also counts the low kMaxDigit bits of every time per
// sort tile (tile-major rows of kMaxBins): the first pass of the time sort
// takes its digit counts from these rows once t_min is known (k_start), so
// it needs no histogram read of its own.  Each block walks tiles blockIdx.x,
// blockIdx.x + gridDim.x, ...
// t is mapped to an order-preserving unsigned key (flip the sign bit)
template <int ITEMS>
__global__ __launch_bounds__(kSortBlock) void k_validate(const int32_t* __restrict__ src,
                                                         const int32_t* __restrict__ dst,
                                                         const int64_t* __restrict__ t, int64_t m,
                                                         int32_t n, Found* __restrict__ found,
                                                         uint32_t* __restrict__ hist) {
  const int64_t lim = (int64_t)1 << 62;
  uint64_t mn = ~0ull, mx = 0;
  uint32_t bad = 0;
  auto check = [&](int32_t s, int32_t d, int64_t tt) {
    if (s < 0 || s >= n || d < 0 || d >= n || tt >= lim || tt <= -lim) bad = 1;
    const uint64_t key = (uint64_t)tt ^ (1ull << 63);
    mn = key < mn ? key : mn;
    mx = key > mx ? key : mx;
  };
  __shared__ uint32_t s_h[kMaxBins];
  constexpr int kTile = kSortBlock * ITEMS;
  const int64_t ntiles = (m + kTile - 1) / kTile;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
#pragma unroll
    for (int q = 0; q < kMaxBins / kSortBlock; ++q) s_h[q * kSortBlock + threadIdx.x] = 0;
    __syncthreads();
    const int64_t start = tile * kTile;
    int32_t sv[ITEMS], dv[ITEMS];
    int64_t tv[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {  // the tile's loads issued together
      const int64_t i = start + (int64_t)r * kSortBlock + threadIdx.x;
      const bool in = i < m;
      sv[r] = in ? src[i] : 0;
      dv[r] = in ? dst[i] : 0;
      tv[r] = in ? t[i] : 0;
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      if (start + (int64_t)r * kSortBlock + threadIdx.x < m) {
        check(sv[r], dv[r], tv[r]);
        atomicAdd(&s_h[(uint32_t)(uint64_t)tv[r] & (kMaxBins - 1)], 1u);
      }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kMaxBins / kSortBlock; ++q)
      hist[tile * kMaxBins + q * kSortBlock + threadIdx.x] = s_h[q * kSortBlock + threadIdx.x];
    __syncthreads();  // the next tile clears s_h
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    uint64_t a = __shfl_xor(mn, off, kWave);
    uint64_t b = __shfl_xor(mx, off, kWave);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
    bad |= __shfl_xor(bad, off, kWave);
  }
  __shared__ uint64_t s_mn[kSortWaves], s_mx[kSortWaves];
  __shared__ uint32_t s_bad[kSortWaves];
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    s_mn[wave] = mn;
    s_mx[wave] = mx;
    s_bad[wave] = bad;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
      mn = s_mn[w] < mn ? s_mn[w] : mn;
      mx = s_mx[w] > mx ? s_mx[w] : mx;
      bad |= s_bad[w];
    }
    found[blockIdx.x] = Found{mn, mx, bad};
  }
}

// ------------------------------------------------------------ sort plan ---
// Every sort of the build moves whole 16-byte edge records.  The time sort
// sorts the records by t - t_min, which needs up to 63 bits: its low 32 bits
// are a word of the record, and the bits above them sit in the unused top
// bits of a vertex word where they fit there (PACKED: millisecond times of a
// few years, with vertex ids of up to 26 bits), so that the digits run over
// all of the value and no later step reads the input again.  A range too wide
// for that takes passes over the low word, then over the high word, re-keyed
// from the input by edge id (WIDE).  How many of the launched passes do work,
// their digit widths and their ping-pong buffers are decided on the device
// from the validated time range (k_plan), so the host enqueues the same
// launches whatever the data and never waits for the device: the build is one
// stream-ordered sequence that a HIP graph can capture.  A pass with no work
// leaves at once.
constexpr int kTimePasses = 6;  // 63 bits in digits of kMaxDigit, or two words of 32

struct BuildPlan {
  int64_t tmin, tmax;  // time range (0, 0 for an empty or rejected input)
  uint32_t bad;        // the validation set TC_F_RANGE: nothing after it runs
  int32_t wide;        // high-word passes, times read back from the input
  int32_t npass;       // passes of the time sort that do work (the first npass ones)
  int32_t high;        // first high-word pass of a wide range (else kTimePasses)
  int32_t shift[kTimePasses], dbits[kTimePasses];
};

__device__ __forceinline__ int bitlen_dev(uint64_t x) { return x ? 64 - __clzll(x) : 0; }

__host__ __device__ constexpr int digit_passes(int bits) {
  return (bits + kMaxDigit - 1) / kMaxDigit;
}

// digit widths as equal as possible (narrow ones first): fewer distinct
// digits per tile means longer runs in the scatter's output, and fewer partly
// written cache lines
__host__ __device__ inline void digit_plan(int bits, int npass, int i, int* shift, int* dbits) {
  int sh = 0;
  for (int q = 0; q < i; ++q) sh += (bits - sh) / (npass - q);
  *shift = sh;
  *dbits = (bits - sh) / (npass - i);
}

// row length of a pass's histogram matrix
__host__ __device__ constexpr int hist_bins(int dbits) {
  return (1 << dbits) < kMinBins ? kMinBins : 1 << dbits;
}

// one block of kMaxFound threads; also starts the counters of the build
__global__ __launch_bounds__(kMaxFound) void k_plan(const Found* __restrict__ found, int nfound,
                                                    int64_t m, int vbits,
                                                    BuildPlan* __restrict__ P,
                                                    uint32_t* __restrict__ status,
                                                    int64_t* __restrict__ t_range,
                                                    uint32_t* __restrict__ spill_count) {
  const int tid = threadIdx.x;
  uint64_t mn = ~0ull, mx = 0;
  uint32_t any = 0;
  if (tid < nfound) {
    const Found f = found[tid];
    mn = f.mn;
    mx = f.mx;
    any = f.bad;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint64_t a = __shfl_xor(mn, off, kWave), b = __shfl_xor(mx, off, kWave);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
    any |= __shfl_xor(any, off, kWave);
  }
  __shared__ Found s_f[kMaxFound / kWave];
  if ((tid & 63) == 0) s_f[tid >> 6] = Found{mn, mx, any};
  __syncthreads();
  if (tid != 0) return;
  for (int w = 1; w < kMaxFound / kWave; ++w) {
    mn = s_f[w].mn < mn ? s_f[w].mn : mn;
    mx = s_f[w].mx > mx ? s_f[w].mx : mx;
    any |= s_f[w].bad;
  }
  BuildPlan B;
  B.bad = any;
  B.tmin = B.tmax = 0;
  B.wide = 0;
  B.npass = 0;
  B.high = kTimePasses;
  for (int p = 0; p < kTimePasses; ++p) B.shift[p] = B.dbits[p] = 0;
  if (!B.bad && m > 0) {
    B.tmin = (int64_t)(mn ^ (1ull << 63));
    B.tmax = (int64_t)(mx ^ (1ull << 63));
    const int tbits = bitlen_dev((uint64_t)(B.tmax - B.tmin));
    B.wide = tbits > 64 - vbits ? 1 : 0;
    const int lo = B.wide ? 32 : tbits, hi = tbits - lo;
    const int nlo = digit_passes(lo), nhi = digit_passes(hi);
    for (int i = 0; i < nlo; ++i) digit_plan(lo, nlo, i, &B.shift[i], &B.dbits[i]);
    for (int i = 0; i < nhi; ++i) digit_plan(hi, nhi, i, &B.shift[nlo + i], &B.dbits[nlo + i]);
    B.npass = nlo + nhi;
    if (B.wide) B.high = nlo;
  }
  *P = B;
  *status = any ? TC_F_RANGE : 0u;
  *spill_count = 0;
  t_range[0] = B.tmin;  // for tc_graph
  t_range[1] = B.tmax;
}

// ------------------------------------------------------------ radix pass ---
// Re-keying of a 16-byte edge record between the sorts of the build:
//   RX_NONE  identity
//   RX_OUT   (t, eid, src, dst) -> (src, eid, dst, t)   out-CSR input
//   RX_PAIR  (a, eid, b, t) -> (b, eid, a, t): the in-CSR input from the
//            out-CSR one as it is loaded, and the pair-index input from the
//            in-CSR order
enum { RX_NONE = 0, RX_OUT = 1, RX_PAIR = 3 };
__device__ __forceinline__ uint4 rec_xform(const uint4& r, int xf) {
  if (xf == RX_OUT) return make_uint4(r.z, r.y, r.w, r.x);
  if (xf == RX_PAIR) return make_uint4(r.z, r.y, r.x, r.w);
  return r;
}

// The input edge columns (read by the first pass of the time sort, which
// builds each record (t - t_min, eid, src, dst) as it loads it, and by the
// first high-word pass of a wide range, which re-keys each record with the
// high word of t[eid] - t_min).
struct EdgeCols {
  const int32_t* src;
  const int32_t* dst;
  const int64_t* t;
};

// What a pass is and where it reads its records from (a template parameter:
// the choice costs the scatter registers when it is made at run time):
//   RP_COLS    first pass of the time sort, from the edge columns
//   RP_TIME    a later pass of the time sort, from the buffer before it
//   RP_VERTEX  a pass of a vertex sort, from a buffer
//   RP_INCOLS  first pass of the pair sort, from the in-list columns
enum { RP_COLS = 0, RP_TIME = 1, RP_VERTEX = 2, RP_INCOLS = 3 };

// The in-list columns as the pair sort's input: the 16-byte in-CSR records
// {src, eid, t} and the key column dst give the record (src, eid, dst,
// t - t_min) in in-CSR order, so no re-keyed copy of the in-CSR order is
// written for it.
struct InCols {
  const uint4* rec;
  const int32_t* key;
  const int32_t* src;  // the new key, for the histogram
};

// The bits of t - t_min above its low 32 travel in the top bits of one vertex
// word (zero when the range needs none or is wide): the word that holds dst
// in the time sort, and whichever word that becomes after it.
__host__ __device__ __forceinline__ uint32_t vertex_mask(int vbits) { return (1u << vbits) - 1u; }

// The time of a record (key, eid, other, low word of t - t_min)
__device__ __forceinline__ int64_t rec_time(const BuildPlan& P, const int64_t* __restrict__ t_in,
                                            const uint4& r, int vbits) {
  if (P.wide) return t_in[r.y];
  const uint32_t hi = (r.x >> vbits) | (r.z >> vbits);
  return P.tmin + (int64_t)(((uint64_t)hi << 32) | r.w);
}

// The graph columns that the last pass of a vertex sort writes in place of
// its sorted records: for output position i with record (key, eid, other,
// t - t_min), key[i], other[i], t[i], eid[i], optionally the 16-byte record
// {other, eid, t} and, every 16th position, the sampled time levels.
struct EmitCols {
  const BuildPlan* plan;  // time base, the wide-range flag and the validation
  const int64_t* t_in;    // input times, read by edge id for wide ranges
  int32_t* key;
  int32_t* other;
  int64_t* t;
  int32_t* eid;
  uint4* rec;      // or null
  int64_t* skip;   // or null
};

// One launched radix pass.  A vertex sort's passes are planned by the host
// (bit counts follow from n); with time >= 0 it is that pass of the time
// sort and everything below `out` is resolved on the device.
struct RecPass {
  const BuildPlan* plan;
  int time;         // pass of the time sort, or -1
  int vbits;
  const uint4* in;  // host-planned input
  uint4* out;       // host-planned output
  uint4* buf[2];    // time sort: the ping-pong buffers (the sort ends in buf[0])
  int shift, dbits;
  int xfin;         // re-keying of the input as it is loaded (host-planned passes)
  int xf1;          // re-keying of the time sort's last output
  EdgeCols ec;
  EmitCols E;       // k_radix_scatter<..., true>: the columns out of the last pass
  InCols ic;        // host-planned input from the in-list columns (ic.rec non-null)
};

struct PassCfg {
  bool active, wide, high;  // high: the pass that re-keys a wide range's records
  int shift, dbits, xfin, xf1, vbits;
  int64_t tmin;
  const uint4* in;
  uint4* out;
};

template <int KIND>
__device__ __forceinline__ PassCfg resolve(const RecPass& R) {
  PassCfg c;
  const BuildPlan& P = *R.plan;
  c.vbits = R.vbits;
  c.tmin = P.tmin;
  c.wide = P.wide != 0;
  c.high = false;
  if (KIND == RP_VERTEX || KIND == RP_INCOLS) {
    // a rejected input leaves the sorts' records undefined: nothing runs
    c.active = P.bad == 0;
    c.shift = R.shift;
    c.dbits = R.dbits;
    c.xfin = R.xfin;
    c.in = R.in;
    c.out = R.out;
    c.xf1 = RX_NONE;
    return c;
  }
  const int p = R.time, n = P.npass;
  c.xfin = RX_NONE;
  c.active = p < n && P.bad == 0;
  c.shift = P.shift[p];
  c.dbits = P.dbits[p];
  // pass p of n writes buf[(n - 1 - p) & 1], so the last one writes buf[0];
  // pass 0 reads the edge columns, the others the previous output
  c.out = R.buf[(n - 1 - p) & 1];
  c.in = R.buf[(n - p) & 1];
  c.high = p == P.high;
  c.xf1 = p == n - 1 ? R.xf1 : RX_NONE;
  return c;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 load_once(const uint4* p) {
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <int KIND>
__device__ __forceinline__ uint4 load_rec(const RecPass& R, const PassCfg& c, int64_t g) {
  if (KIND == RP_COLS) {
    const uint64_t dt = (uint64_t)(R.ec.t[g] - c.tmin);
    // a wide range's high word has no room here
    const uint32_t hi = c.wide ? 0u : (uint32_t)(dt >> 32) << c.vbits;
    return make_uint4((uint32_t)dt, (uint32_t)g, (uint32_t)R.ec.src[g],
                      (uint32_t)R.ec.dst[g] | hi);
  }
  if (KIND == RP_INCOLS) {
    const uint4 q = load_once(R.ic.rec + g);
    const uint64_t dt = (((uint64_t)q.w << 32) | q.z) - (uint64_t)c.tmin;
    const uint32_t hi = c.wide ? 0u : (uint32_t)(dt >> 32) << c.vbits;
    return make_uint4(q.x, q.y, (uint32_t)R.ic.key[g] | hi, (uint32_t)dt);
  }
  uint4 r = load_once(c.in + g);
  if (KIND == RP_TIME) {
    if (c.high) r.x = (uint32_t)((uint64_t)(R.ec.t[r.y] - c.tmin) >> 32);
    return r;
  }
  return rec_xform(r, c.xfin);
}

// the digit of a record: of its key word, or in the time sort of the whole
// t - t_min (low word, then the bits above dst)
template <int KIND>
__device__ __forceinline__ uint32_t digit_of(const PassCfg& c, uint32_t mask, uint32_t x,
                                             uint32_t w) {
  if (KIND == RP_VERTEX || KIND == RP_INCOLS) return (x >> c.shift) & mask;
  return (uint32_t)((((uint64_t)(w >> c.vbits) << 32) | x) >> c.shift) & mask;
}

// What the sorts start from, in one launch: the digit counts of the time
// sort's first pass from the validation's counts of the low bits (its digit is
// the low w <= kMaxDigit bits of t - t_min, shift 0, so digit d counts the low
// bits b with (b - t_min) mod 2^w = d); with no active time pass (every time
// equal) the records built from the edge columns, re-keyed like the last pass
// of the time sort would leave them; and the empty run table where runs are
// inserted one by one (cap slots, else 0).
__global__ __launch_bounds__(kSortBlock) void k_start(const uint32_t* __restrict__ low,
                                                      uint32_t* __restrict__ hist,
                                                      int64_t ntiles, EdgeCols ec, int64_t m,
                                                      const BuildPlan* __restrict__ plan,
                                                      uint4* __restrict__ out, int xf1,
                                                      uint4* __restrict__ tab, int64_t cap) {
  const int64_t first = (int64_t)blockIdx.x * kSortBlock + threadIdx.x;
  const int64_t all = (int64_t)gridDim.x * kSortBlock;
  for (int64_t i = first; i < cap; i += all) tab[i] = make_uint4(~0u, ~0u, 0u, 0u);
  if (plan->bad) return;
  if (plan->npass == 0) {
    for (int64_t i = first; i < m; i += all)
      out[i] = rec_xform(make_uint4(0u, (uint32_t)i, (uint32_t)ec.src[i], (uint32_t)ec.dst[i]),
                         xf1);
    return;
  }
  __shared__ uint32_t s_r[kMaxBins];
  const uint32_t W = 1u << plan->dbits[0], tm = (uint32_t)(uint64_t)plan->tmin;
  const int bins = hist_bins(plan->dbits[0]);
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
#pragma unroll
    for (int q = 0; q < kMaxBins / kSortBlock; ++q)
      s_r[q * kSortBlock + threadIdx.x] = low[tile * kMaxBins + q * kSortBlock + threadIdx.x];
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < (uint32_t)bins; d += kSortBlock) {
      uint32_t v = 0;
      if (d < W)
        for (uint32_t b = (d + tm) & (W - 1); b < (uint32_t)kMaxBins; b += W) v += s_r[b];
      hist[tile * bins + d] = v;
    }
    __syncthreads();  // the next row overwrites s_r
  }
}

// the re-keying of a vertex sort with no pass (n = 1): a[i] from in[i]
// (in == a allowed: every element is read and written by the same thread)
__global__ __launch_bounds__(256) void k_rec_xform(const uint4* in, int xfin, uint4* a, int64_t m,
                                                   uint4* __restrict__ out2, int xf2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) {
    const uint4 r = rec_xform(in[i], xfin);
    a[i] = r;
    if (out2) out2[i] = rec_xform(r, xf2);
  }
}

template <int ITEMS, int KIND>
__global__ __launch_bounds__(kSortBlock) void k_radix_hist(RecPass R, int64_t m,
                                                           uint32_t* __restrict__ hist) {
  __shared__ uint32_t s_h[kMaxBins];
  const PassCfg c = resolve<KIND>(R);
  if (!c.active) return;
  const uint32_t mask = (1u << c.dbits) - 1u;
  const int bins = hist_bins(c.dbits);
  constexpr int kTile = kSortBlock * ITEMS;
  // one tile per block, or several when the grid is smaller than the tile
  // count (the passes that are usually idle)
  const int64_t ntiles = (m + kTile - 1) / kTile;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    for (int d = threadIdx.x; d < bins; d += kSortBlock) s_h[d] = 0;
    __syncthreads();
    const int64_t start = tile * kTile;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const int64_t i = start + (int64_t)r * kSortBlock + threadIdx.x;
      if (i < m) {
        uint4 k;
        if (KIND == RP_INCOLS)
          k.x = (uint32_t)R.ic.src[i], k.w = 0;  // 4 bytes of it, not 16
        else
          k = load_rec<KIND>(R, c, i);
        atomicAdd(&s_h[digit_of<KIND>(c, mask, k.x, k.w)], 1u);
      }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < bins; d += kSortBlock) hist[tile * bins + d] = s_h[d];
    __syncthreads();  // the next tile clears s_h
  }
}

// The histograms of the in-CSR and the out-CSR sorts' first passes from one
// read of the time-ordered records (src, eid, dst, t) that both start from.
template <int ITEMS>
__global__ __launch_bounds__(kSortBlock) void k_radix_hist2(const uint4* __restrict__ in,
                                                            const BuildPlan* __restrict__ plan,
                                                            int dbits, int64_t m,
                                                            uint32_t* __restrict__ by_dst,
                                                            uint32_t* __restrict__ by_src) {
  if (plan->bad) return;
  __shared__ uint32_t s_h[2][kMaxBins];
  const uint32_t mask = (1u << dbits) - 1u;
  const int bins = hist_bins(dbits);
  for (int d = threadIdx.x; d < bins; d += kSortBlock) s_h[0][d] = s_h[1][d] = 0;
  __syncthreads();
  const int64_t start = (int64_t)blockIdx.x * (kSortBlock * ITEMS);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int64_t i = start + (int64_t)r * kSortBlock + threadIdx.x;
    if (i < m) {
      const uint4 k = load_once(in + i);
      atomicAdd(&s_h[0][k.z & mask], 1u);
      atomicAdd(&s_h[1][k.x & mask], 1u);
    }
  }
  __syncthreads();
  for (int d = threadIdx.x; d < bins; d += kSortBlock) {
    by_dst[(int64_t)blockIdx.x * bins + d] = s_h[0][d];
    by_src[(int64_t)blockIdx.x * bins + d] = s_h[1][d];
  }
}

// Column scan of the tile-major histogram: hist[t][d] becomes the number of
// keys of digit d in the tiles before t, and tot[d] the digit's total; the
// scatter adds the keys of smaller digits.  A launch costs 3 us, so up to
// kSelfScanTiles tiles the scatter's blocks each add up the columns
// themselves (20,001 edges: the build 120 -> 107 us; 60,001 edges in 30 tiles
// 158 -> 165), and up to kOneScanTiles it is one kernel (32 digits per block,
// the tiles spread over its threads).  Above, three kernels: per-chunk
// column sums, an exclusive scan of each digit's chunk sums (which also
// leaves the totals), and an in-place walk of every chunk.  Every access
// reads or writes whole row pieces.  The row length follows the pass's digit;
// a pass the plan leaves idle returns at once.
constexpr int kSelfScanTiles = 16, kOneScanTiles = 512;

struct PassBins {
  const BuildPlan* plan;
  int time;  // pass of the time sort, or -1
  int bins;  // row length of a vertex sort's pass
};
// row length of the pass, 0 if it is idle
__device__ __forceinline__ int pass_bins(const PassBins& G) {
  if (G.plan->bad) return 0;
  if (G.time < 0) return G.bins;
  return G.time < G.plan->npass ? hist_bins(G.plan->dbits[G.time]) : 0;
}

__global__ __launch_bounds__(1024) void k_col_one(uint32_t* __restrict__ hist, int ntiles,
                                                  uint32_t* __restrict__ tot, PassBins G) {
  const int bins = pass_bins(G);
  constexpr int kDig = 32, kParts = 1024 / kDig;
  constexpr int kRows = kOneScanTiles / kParts;
  if ((int)blockIdx.x * kDig >= bins) return;
  __shared__ uint32_t s_sum[kParts][kDig];
  const int dl = threadIdx.x % kDig, part = threadIdx.x / kDig;
  const int d = blockIdx.x * kDig + dl;
  const int per = (ntiles + kParts - 1) / kParts;  // at most kRows
  const int t0 = part * per;
  uint32_t v[kRows];
  uint32_t s = 0;
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    v[j] = j < per && t0 + j < ntiles ? hist[(int64_t)(t0 + j) * bins + d] : 0u;
    s += v[j];
  }
  s_sum[part][dl] = s;
  __syncthreads();
  uint32_t run = 0, all = 0;
  for (int p = 0; p < kParts; ++p) {
    const uint32_t x = s_sum[p][dl];
    run += p < part ? x : 0u;
    all += x;
  }
  if (part == 0) tot[d] = all;
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    if (j < per && t0 + j < ntiles) hist[(int64_t)(t0 + j) * bins + d] = run;
    run += v[j];
  }
}

__global__ __launch_bounds__(256) void k_col_sum(const uint32_t* __restrict__ hist,
                                                 int64_t ntiles, uint32_t* __restrict__ csum,
                                                 PassBins G) {
  const int bins = pass_bins(G);
  const int64_t t0 = (int64_t)blockIdx.x * kColChunk;
  for (int d = threadIdx.x; d < bins; d += 256) {
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < kColChunk; ++j) {
      // clamped index: every load is issued unconditionally
      const int64_t t = t0 + j < ntiles ? t0 + j : ntiles - 1;
      const uint32_t v = hist[t * bins + d];
      s += (t0 + j < ntiles) ? v : 0u;
    }
    csum[(int64_t)blockIdx.x * bins + d] = s;
  }
}

// one block per digit (blockIdx.x), chunks spread over the block's threads
__global__ __launch_bounds__(256) void k_col_scan(uint32_t* __restrict__ csum, int64_t nchunks,
                                                  uint32_t* __restrict__ tot, PassBins G) {
  const int bins = pass_bins(G);
  if ((int)blockIdx.x >= bins) return;
  __shared__ uint32_t s_w[256 / kWave];
  const int d = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (int64_t base = 0; base < nchunks; base += 256) {
    const int64_t c = base + threadIdx.x;
    const uint32_t v = c < nchunks ? csum[c * bins + d] : 0u;
    const uint32_t inc = wave_inclusive_scan(v);
    if (lane == 63) s_w[wave] = inc;
    __syncthreads();
    uint32_t off = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 256 / kWave; ++w) {
      off += w < wave ? s_w[w] : 0u;
      all += s_w[w];
    }
    if (c < nchunks) csum[c * bins + d] = carry + off + inc - v;
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) tot[d] = carry;
}

// one block per chunk: its threads walk the chunk's tiles
__global__ __launch_bounds__(256) void k_col_apply(uint32_t* __restrict__ hist, int64_t ntiles,
                                                   const uint32_t* __restrict__ csum,
                                                   PassBins G) {
  const int bins = pass_bins(G);
  const int64_t t0 = (int64_t)blockIdx.x * kColChunk;
  for (int d = threadIdx.x; d < bins; d += 256) {
    uint32_t run = csum[(int64_t)blockIdx.x * bins + d];
    uint32_t v[kColChunk];
#pragma unroll
    for (int j = 0; j < kColChunk; ++j) {
      const int64_t t = t0 + j < ntiles ? t0 + j : ntiles - 1;
      v[j] = hist[t * bins + d];
    }
#pragma unroll
    for (int j = 0; j < kColChunk; ++j) {
      if (t0 + j < ntiles) hist[(t0 + j) * bins + d] = run;
      run += v[j];
    }
  }
}

// the totals row, then the chunk sums
size_t col_scan_scratch_elems(int64_t ntiles, int bins) {
  return (size_t)bins * ((ntiles + kColChunk - 1) / kColChunk + 1);
}

static void col_scan(uint32_t* hist, int64_t ntiles, uint32_t* part, const PassBins& G,
                     hipStream_t st) {
  const unsigned bins = G.time < 0 ? (unsigned)G.bins : (unsigned)kMaxBins;
  if (ntiles <= kOneScanTiles) {
    hipLaunchKernelGGL(k_col_one, dim3((bins + 31) / 32), dim3(1024), 0, st, hist, (int)ntiles,
                       part, G);
    return;
  }
  const int64_t nchunks = (ntiles + kColChunk - 1) / kColChunk;
  uint32_t* csum = part + bins;
  hipLaunchKernelGGL(k_col_sum, dim3((unsigned)nchunks), dim3(256), 0, st,
                     (const uint32_t*)hist, ntiles, csum, G);
  hipLaunchKernelGGL(k_col_scan, dim3(bins), dim3(256), 0, st, csum, nchunks, part, G);
  hipLaunchKernelGGL(k_col_apply, dim3((unsigned)nchunks), dim3(256), 0, st, hist, ntiles,
                     (const uint32_t*)csum, G);
}

// the columns of one sorted record at output position i (see EmitCols)
__device__ __forceinline__ void emit_cols(const EmitCols& E, int vbits, int64_t m, int64_t i,
                                          uint4 r) {
  const int64_t te = rec_time(*E.plan, E.t_in, r, vbits);
  r.x &= vertex_mask(vbits);
  r.z &= vertex_mask(vbits);
  E.key[i] = (int32_t)r.x;
  E.other[i] = (int32_t)r.z;
  E.t[i] = te;
  E.eid[i] = (int32_t)r.y;
  if (E.rec) E.rec[i] = make_uint4(r.z, r.y, (uint32_t)te, (uint32_t)(te >> 32));
  if (E.skip && (i & 15) == 0) {
    const int64_t n1 = skip_level_len(m, 1), n2 = skip_level_len(m, 2);
    E.skip[i >> 4] = te;
    if ((i & 255) == 0) E.skip[n1 + (i >> 8)] = te;
    if ((i & 4095) == 0) E.skip[n1 + n2 + (i >> 12)] = te;
  }
}

// The scatter moves 32 bytes per record and runs at the rate of a large
// device copy (3*10^8 records by a 9-bit digit: 2.3 ms, 4.2 TB/s; 2*10^7 by a
// 10-bit digit 0.17 ms), so the sort's time is its passes and its histogram
// reads.  Against 8- and 9-bit digits in 1,536-record tiles (12 passes for
// 2*10^7 edges of 20-bit vertices and 22-bit times, now 8) the build went from
// 4.65 to 4.03 ms, 5*10^6 edges of millisecond times from 1.45 to 1.11 ms,
// and 3*10^8 edges from 55.8 to 50 ms.  Records are read past the caches'
// replacement order (non-temporal: 3% of the 2*10^7-edge build), which leaves
// the half-written lines of the digit runs in L2 until they are full.
// Tiles of 6,144 records exchanged half a record at a time needed 128
// registers and spills (twice the time per pass); 2,048-record tiles give the
// scatter 5-10% but pay more for four times the histogram rows.
template <int ITEMS, int KIND, bool EMIT>
__global__ __launch_bounds__(kSortBlock, ITEMS > 5 ? 4 : 6) void k_radix_scatter(
    RecPass R, int64_t m,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ tot) {
  // Each wavefront owns a contiguous eighth of the tile and ranks its keys
  // in order with ballots (no block barrier inside); one block-wide pass then
  // offsets every wavefront's digit counts by those of the wavefronts before
  // it, which keeps the pass stable.
  constexpr int kTile = kSortBlock * ITEMS;
  constexpr int kSub = kWave * ITEMS;  // entries per wavefront
  constexpr int kOwn = 4;              // digits per thread of the block-wide pass
  static_assert(kMaxBins <= kOwn * kSortBlock, "every digit has a thread");
  static_assert(2 * kTile < 65536, "16-bit tile positions");
  const PassCfg c = resolve<KIND>(R);
  if (!c.active) return;
  const int dbits = c.dbits;
  const uint32_t mask = (1u << dbits) - 1u;
  const int bins = hist_bins(dbits);
  // s_base[d]: global position of digit d's run minus its start in the tile
  // s_pos[w][d]: wavefront w's running count of digit d, then the position
  //              in the tile of w's first key of digit d (16 bits suffice);
  //              once every thread holds its records' positions, the same
  //              LDS exchanges the records
  constexpr int kPosBytes = kSortWaves * kMaxBins * 2, kXBytes = kTile * 16;
  __shared__ __align__(16) char s_mem[kPosBytes > kXBytes ? kPosBytes : kXBytes];
  __shared__ uint32_t s_base[kMaxBins];
  __shared__ uint64_t s_wsum[kSortWaves];
  uint16_t* const s_pos = reinterpret_cast<uint16_t*>(s_mem);
  uint4* const s_rec = reinterpret_cast<uint4*>(s_mem);
  const uint32_t nb = (uint32_t)((m + kTile - 1) / kTile);
  // One tile per block, or several when the grid is smaller (a multiple of 8
  // blocks then, for the passes that are usually idle).
  for (uint32_t vt = blockIdx.x; vt < nb; vt += gridDim.x) {
    // a thread index the compiler cannot carry over from the last tile: it
    // would keep every address formed from it in registers across the loop
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63, wave = (int)uni(threadIdx.x >> 6);
    uint16_t* const my_pos = s_pos + wave * bins;
    const uint32_t tile = xcd_tile(vt, nb);
    const int64_t start = (int64_t)tile * kTile;
    const int len = (int)((m - start) < kTile ? (m - start) : kTile);

    // the last tile is filled up with records of the largest digit: they rank
    // behind all of its own, so only the final writes need to leave them out
    uint4 key[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const int idx = wave * kSub + r * kWave + lane;
      key[r] = idx < len ? load_rec<KIND>(R, c, start + idx) : uint4{~0u, ~0u, ~0u, ~0u};
    }
    uint4 gb{0, 0, 0, 0}, tt{0, 0, 0, 0};  // digits kOwn tid ..: prefix over tiles, totals
    if (kOwn * tid < bins) {
      if (ITEMS == kItemsSmall && nb <= (uint32_t)kSelfScanTiles) {  // hist: plain counts
#pragma unroll 8
        for (uint32_t u = 0; u < nb; ++u) {
          const uint4 v = *reinterpret_cast<const uint4*>(hist + (int64_t)u * bins + kOwn * tid);
          tt.x += v.x, tt.y += v.y, tt.z += v.z, tt.w += v.w;
          const uint32_t f = u < tile ? ~0u : 0u;
          gb.x += v.x & f, gb.y += v.y & f, gb.z += v.z & f, gb.w += v.w & f;
        }
      } else {
        gb = *reinterpret_cast<const uint4*>(hist + (int64_t)tile * bins + kOwn * tid);
        tt = *reinterpret_cast<const uint4*>(tot + kOwn * tid);
      }
    }
    for (int i = tid; i < kSortWaves * bins / 8; i += kSortBlock)
      reinterpret_cast<uint4*>(s_mem)[i] = uint4{0, 0, 0, 0};
    __syncthreads();

    // lanes whose record r has the digit of this lane's: one ballot per bit,
    // the records of a thread side by side
    uint32_t dig[ITEMS], rank[ITEMS];
    uint64_t peers[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      dig[r] = digit_of<KIND>(c, mask, key[r].x, key[r].w);
      peers[r] = ~0ull;
    }
    for (int b = 0; b < dbits; ++b) {  // uniform
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        const bool bit = (dig[r] >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        peers[r] &= bit ? bb : ~bb;
      }
    }
    // rank among the wavefront's records of the same digit
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const uint32_t below = __builtin_amdgcn_mbcnt_hi(
          (uint32_t)(peers[r] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers[r], 0u));
      // read the running count before the leader of each digit group adds to it
      const uint32_t run = my_pos[dig[r]];
      rank[r] = run + below;
      __builtin_amdgcn_wave_barrier();
      if (below == 0) my_pos[dig[r]] = (uint16_t)(run + (uint32_t)__popcll(peers[r]));
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // thread tid owns digits kOwn tid ..: one scan over the block gives both
    // the keys of smaller digits (totals, above bit 16) and the digit's start
    // in the tile (counts, below)
    {
      // the counts of four digits as 16-bit halves (a tile's sums fit them)
      uint2 c2{0, 0};
      const bool own = kOwn * tid < bins;
      if (own)
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
          const uint2 v = *reinterpret_cast<const uint2*>(s_pos + w * bins + kOwn * tid);
          c2.x += v.x;
          c2.y += v.y;
        }
      const uint32_t cnt[kOwn] = {c2.x & 0xFFFFu, c2.x >> 16, c2.y & 0xFFFFu, c2.y >> 16};
      const uint32_t total[kOwn] = {tt.x, tt.y, tt.z, tt.w};
      const uint32_t before[kOwn] = {gb.x, gb.y, gb.z, gb.w};
      uint64_t s = 0;
#pragma unroll
      for (int j = 0; j < kOwn; ++j) s += ((uint64_t)total[j] << 16) + cnt[j];
      const uint64_t inc = wave_inclusive_scan(s);
      if (lane == 63) s_wsum[wave] = inc;
      __syncthreads();
      uint64_t run = inc - s;
#pragma unroll
      for (int w = 0; w < kSortWaves; ++w) run += w < wave ? s_wsum[w] : 0ull;
      if (own) {
        uint32_t pos[kOwn];
#pragma unroll
        for (int j = 0; j < kOwn; ++j) {
          const uint32_t off = (uint32_t)run & 0xFFFFu;
          // modulo 2^32; the sum with the tile position is exact
          s_base[kOwn * tid + j] = (uint32_t)(run >> 16) + before[j] - off;
          pos[j] = off;
          run += ((uint64_t)total[j] << 16) + cnt[j];
        }
        uint2 at{pos[0] | pos[1] << 16, pos[2] | pos[3] << 16};
#pragma unroll
        for (int w = 0; w < kSortWaves; ++w) {
          uint2* const sp = reinterpret_cast<uint2*>(s_pos + w * bins + kOwn * tid);
          const uint2 v = *sp;
          *sp = at;
          at.x += v.x;
          at.y += v.y;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
      rank[r] += my_pos[dig[r]];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) s_rec[rank[r]] = key[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const int i = r * kSortBlock + tid;
      if (i < len) {
        const uint4 k = s_rec[i];
        const int64_t gpos = (int64_t)(s_base[digit_of<KIND>(c, mask, k.x, k.w)] + (uint32_t)i);
        // the time sort's last pass re-keys the records for the next sort; a
        // vertex sort's last pass writes the graph's columns instead
        if (EMIT)
          emit_cols(R.E, c.vbits, m, gpos, k);
        else
          c.out[gpos] = rec_xform(k, c.xf1);
      }
    }
    __syncthreads();  // the next tile reuses the LDS
  }
}

// Histogram and scan scratch of the sorts.
struct SortScratch {
  uint32_t* hist;
  uint32_t* part;
  size_t part_elems;
  int vbits;
};

// One launched pass: histogram (unless its counts are there already), column
// scan, scatter.  `grid` blocks walk the tiles.
template <int ITEMS, int KIND>
void radix_pass(const RecPass& R, bool count, bool emit, int64_t m, unsigned grid,
                const SortScratch& sc, hipStream_t st) {
  const int64_t ntiles = (m + kSortBlock * ITEMS - 1) / (kSortBlock * ITEMS);
  const dim3 g(grid), b(kSortBlock);
  if constexpr (KIND != RP_COLS)
    if (count)
    hipLaunchKernelGGL((k_radix_hist<ITEMS, KIND>), g, b, 0, st, R, m, sc.hist);
  if (ITEMS != kItemsSmall || ntiles > kSelfScanTiles)
    col_scan(sc.hist, ntiles, sc.part,
             PassBins{R.plan, R.time, R.time < 0 ? hist_bins(R.dbits) : 0}, st);
  constexpr bool kVertex = KIND == RP_VERTEX || KIND == RP_INCOLS;
  const auto scatter = [&] {
    if (kVertex && emit)
      hipLaunchKernelGGL((k_radix_scatter<ITEMS, KIND, kVertex>), g, b, 0, st, R, m,
                         (const uint32_t*)sc.hist, (const uint32_t*)sc.part);
    else
      hipLaunchKernelGGL((k_radix_scatter<ITEMS, KIND, false>), g, b, 0, st, R, m,
                         (const uint32_t*)sc.hist, (const uint32_t*)sc.part);
  };
  if (R.time >= 0) {  // the plan may leave the pass idle: not timed
    scatter();
    return;
  }
  TimedLaunch tl("k_radix_scatter", st);
  scatter();
}

template <int KIND>
void radix_pass(const RecPass& R, bool count, bool emit, int64_t m, unsigned grid,
                const SortScratch& sc, hipStream_t st) {
  if (large_tiles(m))
    radix_pass<kItemsLarge, KIND>(R, count, emit, m, grid, sc, st);
  else
    radix_pass<kItemsSmall, KIND>(R, count, emit, m, grid, sc, st);
}

// width of pass p of a vertex sort: wide digits first, a narrow one last, so
// that the last pass, which writes four or five arrays, writes the longest
// runs
static int vertex_digit(int bits, int npass, int p) {
  int sh, db;
  digit_plan(bits, npass, npass - 1 - p, &sh, &db);
  return db;
}

// Host-planned stable sort of m records by the low `bits` bits of their
// first word (a vertex id), ping-ponging between k0 and k1; the last pass
// writes the columns E instead of the sorted records (returns 1).  With no
// pass (bits = 0) the records stay in k0, a second copy re-keyed by xf2 goes
// to `extra` if given, and the caller emits from k0 (returns 0).  Returns -1
// if the scan scratch is too small (nothing enqueued then).  With `in0` the
// first pass reads the records from there, re-keyed by xf_in as it loads
// them, and in0 is left as it was; with `ic` it reads them from the in-list
// columns (the caller passes ic only when the sort has a pass).  With `first`
// the first pass's histogram matrix is already there.
static int radix_sort(uint4* k0, uint4* k1, int64_t m, int bits, const SortScratch& sc,
                      hipStream_t st, uint4* extra, int xf2, const EmitCols& E, const uint4* in0,
                      int xf_in, const InCols* ic, uint32_t* first) {
  const int64_t ntiles = sort_tiles(m);
  if (sc.part_elems < col_scan_scratch_elems(ntiles, kMaxBins)) return -1;
  const int npass = digit_passes(bits);
  if (npass == 0) {
    if (extra || in0)
      hipLaunchKernelGGL(k_rec_xform, dim3(blocks_for(m, 256)), dim3(256), 0, st,
                         in0 ? in0 : (const uint4*)k0, in0 ? xf_in : (int)RX_NONE, k0, m, extra,
                         xf2);
    return 0;
  }
  int cur = 0, shift = 0;
  for (int p = 0; p < npass; ++p) {
    RecPass R{};
    R.plan = E.plan;
    R.time = -1;
    R.vbits = sc.vbits;
    R.in = p == 0 && in0 ? in0 : (cur ? k1 : k0);
    R.xfin = p == 0 && in0 ? xf_in : (int)RX_NONE;
    if (p == 0 && ic) R.ic = *ic;
    R.out = cur ? k0 : k1;
    R.shift = shift;
    R.dbits = vertex_digit(bits, npass, p);
    shift += R.dbits;
    const bool last = p + 1 == npass;
    if (last) R.E = E;
    SortScratch use = sc;
    const bool counted = p == 0 && first;
    if (counted) use.hist = first;
    if (R.ic.rec)
      radix_pass<RP_INCOLS>(R, !counted, last, m, (unsigned)ntiles, use, st);
    else
      radix_pass<RP_VERTEX>(R, !counted, last, m, (unsigned)ntiles, use, st);
    cur ^= 1;
  }
  return 1;
}

// The time sort: kTimePasses launched passes planned on the device (see
// BuildPlan).  It reads the edge columns and leaves the time-ordered records
// re-keyed by xf1 in b0.  Its first pass takes its digit counts from the
// validation (k_start, which also clears `cap` slots of the run table).
static bool time_sort(const BuildPlan* plan, const EdgeCols& ec, uint4* b0, uint4* b1, int64_t m,
                      const uint32_t* low, const SortScratch& sc, hipStream_t st, int xf1,
                      uint4* tab, int64_t cap) {
  const int64_t ntiles = sort_tiles(m);
  if (sc.part_elems < col_scan_scratch_elems(ntiles, kMaxBins)) return false;
  const int64_t sb = cap > 0 && ntiles < 256 ? 256 : ntiles;
  hipLaunchKernelGGL(k_start, dim3((unsigned)(sb < 2048 ? sb : 2048)), dim3(kSortBlock), 0, st,
                     low, sc.hist, ntiles, ec, m, plan, b0, xf1, tab, cap);
  for (int p = 0; p < kTimePasses; ++p) {
    RecPass R{};
    R.plan = plan;
    R.time = p;
    R.vbits = sc.vbits;
    R.buf[0] = b0;
    R.buf[1] = b1;
    R.xf1 = xf1;
    R.ec = ec;
    // the passes past 33 bits work only for ranges that wide
    const unsigned grid = (unsigned)(p >= 3 ? late_pass_blocks(ntiles) : ntiles);
    if (p == 0)
      radix_pass<RP_COLS>(R, false, false, m, grid, sc, st);
    else
      radix_pass<RP_TIME>(R, true, false, m, grid, sc, st);
  }
  return true;
}

// -------------------------------------------------------- columns/offsets ---
__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* __restrict__ a, int64_t n,
                                                  uint32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = v;
}

// ----------------------------------------------------- pair-run hash table ---
// Every maximal run of equal (src, dst) in the pair index is one entry of an
// open-addressing table (linear probing, Fibonacci hashing of the 64-bit key
// src << 32 | dst).  A slot is 16 bytes {key, run start, run end}, so a hit
// costs one 16-byte load.  The capacity is a power of two above 1.25 m, so
// the load factor stays below 0.8 and a probe always reaches an empty slot.
__global__ __launch_bounds__(256) void k_hash_clear(PairSlot* __restrict__ tab, int64_t cap) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < cap) {
    tab[i].key = kPairEmpty;
    tab[i].start = 0;
    tab[i].end = 0;
  }
}

// The pair index's sorted (src, dst) keys.
struct PairKeys {
  const uint32_t* src;
  const int32_t* dst;
  int64_t m;
  __device__ __forceinline__ uint64_t at(int64_t j) const {
    return pair_key(src[j], (uint32_t)dst[j]);
  }
  // whether position i, of key `key`, starts a run
  __device__ __forceinline__ bool head(int64_t i, uint64_t key) const {
    return i == 0 || at(i - 1) != key;
  }
  // where the run starting at i ends: galloping over the sorted keys, then
  // bisecting the last gap, so a run of length L costs O(log L) probes and
  // most runs (a single edge) one
  __device__ __forceinline__ int64_t run_end(int64_t i, uint64_t key) const {
    int64_t lo = i, hi, step = 1;  // at(lo) == key
    for (;;) {
      hi = lo + step;
      if (hi >= m || at(hi) != key) break;
      lo = hi;
      step <<= 1;
    }
    if (hi > m) hi = m;  // hi == m, or at(hi) != key
    while (hi - lo > 1) {
      const int64_t mid = lo + ((hi - lo) >> 1);
      if (at(mid) == key)
        lo = mid;
      else
        hi = mid;
    }
    return hi;
  }
};

// Linear probing from slot h: a compare-and-swap claims the slot's key, one
// 8-byte store fills the run.
__device__ __forceinline__ void table_insert(PairSlot* __restrict__ tab, int log2cap, uint64_t h,
                                             uint64_t key, uint32_t start, uint32_t end) {
  const uint64_t mask = (1ull << log2cap) - 1;
  for (uint64_t probe = 0; probe <= mask; ++probe) {
    const unsigned long long prev =
        atomicCAS((unsigned long long*)&tab[h].key, (unsigned long long)kPairEmpty,
                  (unsigned long long)key);
    if (prev == kPairEmpty) {
      *reinterpret_cast<uint2*>(&tab[h].start) = make_uint2(start, end);
      return;
    }
    h = (h + 1) & mask;
  }
}

// One thread per pair-index position, the first of a run inserts it.
__global__ __launch_bounds__(256) void k_hash_insert(PairKeys K, PairSlot* __restrict__ tab,
                                                     int log2cap,
                                                     const BuildPlan* __restrict__ plan) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= K.m || plan->bad) return;
  const uint64_t key = K.at(i);
  if (!K.head(i, key)) return;
  table_insert(tab, log2cap, pair_hash(key, log2cap), key, (uint32_t)i,
               (uint32_t)K.run_end(i, key));
}

// The table without random memory atomics.  A compare-and-swap on a random
// line and the store into it run at 1.4*10^10 per second (1.42 ms for the
// 2*10^7-edge graph, a third of its build); so the runs are first grouped by
// the table segment that their home slot lies in (one radix pass over them,
// in any order inside a group), then one block per segment places its runs
// by linear probing in LDS and writes the whole segment, empty slots
// included, as one stream.  A run that would probe past its segment's end is
// put aside and inserted into the following segment afterwards, when every
// slot from its home to the segment's end is taken, as a search expects.
// Same graph: 0.58 ms (0.21 the grouping scatter, 0.29 the segments), and no
// pass to clear the table.
//
// Segments have 2^14 slots (64 KB of LDS, two blocks per CU), or 2^15 where
// the groups would be more than kMaxGroups; the groups' count rows then bound
// the tables it serves (up to 2^27 slots: 10^8 edges).  Larger ones would
// take a second grouping pass, which costs what the atomics do, and below
// 2^21 slots (0.8*10^6 edges) the atomics' 25 us are less than three more
// launches: both take k_hash_insert, as graphs of few vertices do (few_pairs).
constexpr int kSegLog2 = 14, kMaxSegLog2 = 15, kMaxGroupLog2 = 12, kGroupFromLog2 = 21;
static_assert(1 << (kGroupFromLog2 - kSegLog2) >= kMinBins, "whole rows of the column scan");
constexpr int kMaxGroups = 1 << kMaxGroupLog2;
// 4,096 pair positions per grouping tile
constexpr int kRunBlock = 1024, kRunItems = 4, kRunTile = kRunBlock * kRunItems;

static int group_log2(int log2cap) {  // 0: not grouped
  if (log2cap < kGroupFromLog2 || log2cap > kMaxSegLog2 + kMaxGroupLog2) return 0;
  return log2cap - kSegLog2 < kMaxGroupLog2 ? log2cap - kSegLog2 : kMaxGroupLog2;
}
static int64_t run_tiles(int64_t m) { return (m + kRunTile - 1) / kRunTile; }

// The runs of a grouping tile: thread tid's positions start + 1024 r + tid, the
// key of each, and for the first of a run its group (else ~0)
struct RunTile {
  uint64_t key[kRunItems];
  uint32_t group[kRunItems];
  bool single[kRunItems];  // the next position has another key
  __device__ __forceinline__ void load(const PairKeys& K, int64_t start, int tid, int glog2) {
    uint64_t prev[kRunItems], next[kRunItems];
#pragma unroll
    for (int r = 0; r < kRunItems; ++r) {  // every load issued together
      const int64_t i = start + (int64_t)r * kRunBlock + tid;
      key[r] = i < K.m ? K.at(i) : 0;
      prev[r] = i > 0 && i < K.m ? K.at(i - 1) : ~0ull;
      next[r] = i + 1 < K.m ? K.at(i + 1) : ~0ull;  // no key (vertices are below 2^31)
    }
#pragma unroll
    for (int r = 0; r < kRunItems; ++r) {
      const bool head = start + (int64_t)r * kRunBlock + tid < K.m && prev[r] != key[r];
      group[r] = head ? (uint32_t)pair_hash(key[r], glog2) : ~0u;
      single[r] = next[r] != key[r];
    }
  }
};

// per-tile group counts
__global__ __launch_bounds__(kRunBlock) void k_run_hist(PairKeys K, int glog2,
                                                         uint32_t* __restrict__ hist,
                                                         const BuildPlan* __restrict__ plan) {
  if (plan->bad) return;
  __shared__ uint32_t s_n[kMaxGroups];
  const int groups = 1 << glog2, tid = threadIdx.x;
  for (int g = tid; g < groups; g += kRunBlock) s_n[g] = 0;
  __syncthreads();
  const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
  RunTile T;
  T.load(K, (int64_t)tile * kRunTile, tid, glog2);
#pragma unroll
  for (int r = 0; r < kRunItems; ++r)
    if (T.group[r] != ~0u) atomicAdd(&s_n[T.group[r]], 1u);
  __syncthreads();
  for (int g = tid; g < groups; g += kRunBlock) hist[(int64_t)tile * groups + g] = s_n[g];
}

// The runs {key, start, end} to their groups (hist: the group's runs in the
// tiles before, tot: group totals), staged in LDS so that a tile's runs of a
// group are written together.
__global__ __launch_bounds__(kRunBlock) void k_run_scatter(PairKeys K, int glog2,
                                                            const uint32_t* __restrict__ hist,
                                                            const uint32_t* __restrict__ tot,
                                                            uint4* __restrict__ list,
                                                            const BuildPlan* __restrict__ plan) {
  if (plan->bad) return;
  extern __shared__ __align__(16) char s_raw[];
  uint4* const s_rec = reinterpret_cast<uint4*>(s_raw);
  const int groups = 1 << glog2, tid = threadIdx.x;
  uint32_t* const s_off = reinterpret_cast<uint32_t*>(s_rec + kRunTile);  // counts, then starts
  uint32_t* const s_base = s_off + groups;
  __shared__ uint64_t s_w[kRunBlock / kWave];
  __shared__ uint32_t s_total;
  for (int g = tid; g < groups; g += kRunBlock) s_off[g] = 0;
  __syncthreads();
  const uint32_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const int64_t start = (int64_t)tile * kRunTile;
  RunTile T;
  T.load(K, start, tid, glog2);
  uint32_t rank[kRunItems];
#pragma unroll
  for (int r = 0; r < kRunItems; ++r)
    rank[r] = T.group[r] != ~0u ? atomicAdd(&s_off[T.group[r]], 1u) : 0u;
  __syncthreads();
  // thread tid's consecutive groups: one scan gives their starts in the list
  // (totals, above bit 16) and in the tile (counts, below)
  constexpr int kOwn = kMaxGroups / kRunBlock;
  const int own = (groups + kRunBlock - 1) / kRunBlock;  // at most kOwn
  uint32_t cnt[kOwn], t[kOwn];
  uint64_t sum = 0;
#pragma unroll
  for (int j = 0; j < kOwn; ++j) {
    const int g = own * tid + j;
    const bool in = j < own && g < groups;
    cnt[j] = in ? s_off[g] : 0u;
    t[j] = in ? tot[g] : 0u;
    sum += ((uint64_t)t[j] << 16) + cnt[j];
  }
  const uint64_t inc = wave_inclusive_scan(sum);
  if ((tid & 63) == 63) s_w[tid >> 6] = inc;
  __syncthreads();
  uint64_t run = inc - sum;
#pragma unroll
  for (int w = 0; w < kRunBlock / kWave; ++w) run += w < (tid >> 6) ? s_w[w] : 0ull;
#pragma unroll
  for (int j = 0; j < kOwn; ++j) {
    const int g = own * tid + j;
    if (j < own && g < groups) {
      const uint32_t off = (uint32_t)run & 0xFFFFu;
      s_off[g] = off;
      s_base[g] = (uint32_t)(run >> 16) + hist[(int64_t)tile * groups + g] - off;
    }
    run += ((uint64_t)t[j] << 16) + cnt[j];
  }
  if (tid == kRunBlock - 1) s_total = (uint32_t)run & 0xFFFFu;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRunItems; ++r)
    if (T.group[r] != ~0u) {
      const int64_t i = start + (int64_t)r * kRunBlock + tid;
      const int64_t end = T.single[r] ? i + 1 : K.run_end(i, T.key[r]);
      s_rec[s_off[T.group[r]] + rank[r]] = make_uint4((uint32_t)T.key[r],
                                                      (uint32_t)(T.key[r] >> 32), (uint32_t)i,
                                                      (uint32_t)end);
    }
  __syncthreads();
  for (uint32_t j = tid; j < s_total; j += kRunBlock) {
    const uint4 r = s_rec[j];
    list[s_base[pair_hash(((uint64_t)r.y << 32) | r.x, glog2)] + j] = r;
  }
}
static size_t run_scatter_lds(int glog2) { return (size_t)kRunTile * 16 + ((size_t)8 << glog2); }

constexpr int kSegBlock = 1024;
__global__ __launch_bounds__(kSegBlock) void k_table_segment(const uint4* __restrict__ list,
                                                             const uint32_t* __restrict__ tot,
                                                             int log2cap, int glog2,
                                                             uint4* __restrict__ tab,
                                                             uint32_t* __restrict__ spill,
                                                             uint32_t* __restrict__ spill_count,
                                                             const BuildPlan* __restrict__ plan) {
  extern __shared__ uint32_t s_slot[];  // per slot of the segment: its run, or ~0
  __shared__ uint32_t s_w[kSegBlock / kWave];
  const int tid = threadIdx.x, seg = blockIdx.x;
  const uint32_t slots = 1u << (log2cap - glog2);
  for (uint32_t q = tid; q < slots; q += kSegBlock) s_slot[q] = ~0u;
  uint32_t before = 0;  // runs of the groups below
  for (int g = tid; g < seg; g += kSegBlock) before += tot[g];
  before = lane_u32(scan_dpp(before), kWave - 1);
  if ((tid & 63) == 0) s_w[tid >> 6] = before;
  __syncthreads();
  uint32_t first = 0;
  for (int w = 0; w < kSegBlock / kWave; ++w) first += s_w[w];
  const bool bad = plan->bad != 0;  // a rejected input: an empty table
  const uint32_t n = bad ? 0u : tot[seg];
  for (uint32_t j = tid; j < n; j += kSegBlock) {
    const uint4 r = list[first + j];
    const uint64_t key = ((uint64_t)r.y << 32) | r.x;
    uint32_t q = (uint32_t)pair_hash(key, log2cap) & (slots - 1);
    while (q < slots && atomicCAS(&s_slot[q], ~0u, j) != ~0u) ++q;
    if (q == slots) spill[atomicAdd(spill_count, 1u)] = first + j;
  }
  __syncthreads();
  uint4* const out = tab + (uint64_t)seg * slots;
  for (uint32_t q = tid; q < slots; q += kSegBlock) {
    const uint32_t j = s_slot[q];
    out[q] = j == ~0u ? make_uint4(~0u, ~0u, 0u, 0u) : list[first + j];
  }
}

// the runs put aside, from the segment after their own
__global__ __launch_bounds__(256) void k_table_spill(const uint4* __restrict__ list,
                                                     const uint32_t* __restrict__ spill,
                                                     const uint32_t* __restrict__ spill_count,
                                                     int log2cap, int glog2,
                                                     PairSlot* __restrict__ tab) {
  const uint32_t n = *spill_count;
  const int shift = log2cap - glog2;
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
    const uint4 r = list[spill[i]];
    const uint64_t key = ((uint64_t)r.y << 32) | r.x;
    const uint64_t next = ((pair_hash(key, glog2) + 1) << shift) & ((1ull << log2cap) - 1);
    table_insert(tab, log2cap, next, key, r.z, r.w);
  }
}

int pair_hash_log2(int64_t m) {
  int lg = 4;
  while (((int64_t)1 << lg) < m + m / 4 + 1) ++lg;
  return lg;
}

// sorted records (key, eid, other, t - t_min) -> columns of one order, for a
// graph of a single vertex (its vertex sorts have no pass whose last one
// would write the columns).  The time is t_min + the record's time word and the
// bits above it in a vertex word (rec_time): with no vertex bits there is room
// for every range, so none is read back from the input.
// With `off` (n + 1 entries), also the CSR offsets of the sorted keys:
// off[v] = first position whose key is >= v, written by the thread of the
// position where the key passes v (grid of m + 1 threads).  With `skip`
// (the pair index), also the sampled levels skip_k[i] = t[16^k i], k = 1..3,
// from the times this pass writes anyway.  A rejected input (bad vertex id or
// time) writes nothing.
__global__ __launch_bounds__(256) void k_emit(const uint4* __restrict__ in, int64_t m,
                                              const BuildPlan* __restrict__ plan,
                                              const int64_t* __restrict__ t_in,
                                              int32_t* __restrict__ key_col,
                                              int32_t* __restrict__ other_col,
                                              int64_t* __restrict__ t_col,
                                              int32_t* __restrict__ eid_col,
                                              uint4* __restrict__ rec, int32_t n, int vbits,
                                              uint32_t* __restrict__ off,
                                              int64_t* __restrict__ skip) {
  if (plan->bad) return;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < m) {
    uint4 r = in[i];
    const int64_t te = rec_time(*plan, t_in, r, vbits);
    r.x &= vertex_mask(vbits);
    r.z &= vertex_mask(vbits);
    key_col[i] = (int32_t)r.x;
    other_col[i] = (int32_t)r.z;
    t_col[i] = te;
    eid_col[i] = (int32_t)r.y;
    if (rec) rec[i] = make_uint4(r.z, r.y, (uint32_t)te, (uint32_t)(te >> 32));
    if (skip && (i & 15) == 0) {
      const int64_t n1 = skip_level_len(m, 1), n2 = skip_level_len(m, 2);
      skip[i >> 4] = te;
      if ((i & 255) == 0) skip[n1 + (i >> 8)] = te;
      if ((i & 4095) == 0) skip[n1 + n2 + (i >> 12)] = te;
    }
  }
  if (off && i <= m) {
    const uint32_t vm = vertex_mask(vbits);
    const int64_t prev = (i == 0) ? -1 : (int64_t)(in[i - 1].x & vm);
    const int64_t cur = (i == m) ? (int64_t)n : (int64_t)(in[i].x & vm);
    for (int64_t v = prev + 1; v <= cur; ++v) off[v] = (uint32_t)i;
  }
}

// CSR offsets of both orders from their sorted key columns (blockIdx.y):
// off[v] = first position whose key is at least v, for v in [0, n].  Each
// thread takes kOffItems consecutive positions (two 16-byte loads where the
// column allows), so the launch has an eighth of the blocks a thread per
// position would need.
constexpr int kOffItems = 8;
struct OffCols {
  const int32_t* key[2];
  uint32_t* off[2];
};
__global__ __launch_bounds__(256) void k_offsets(OffCols C, int64_t m,
                                                 const BuildPlan* __restrict__ plan, int32_t n) {
  if (plan->bad) return;
  const int32_t* __restrict__ key = C.key[blockIdx.y];
  uint32_t* __restrict__ off = C.off[blockIdx.y];
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * kOffItems;
  if (i0 > m) return;
  int32_t k[kOffItems];
  if (i0 + kOffItems <= m && ((uintptr_t)key & 15) == 0) {
    const int4 a = *(const int4*)(key + i0), b = *(const int4*)(key + i0 + 4);
    k[0] = a.x, k[1] = a.y, k[2] = a.z, k[3] = a.w, k[4] = b.x, k[5] = b.y, k[6] = b.z,
    k[7] = b.w;
  } else {
#pragma unroll
    for (int j = 0; j < kOffItems; ++j) k[j] = i0 + j < m ? key[i0 + j] : n;
  }
  int64_t prev = i0 == 0 ? -1 : (int64_t)key[i0 - 1];
#pragma unroll
  for (int j = 0; j < kOffItems; ++j) {
    const int64_t i = i0 + j;
    if (i <= m) {
      const int64_t cur = i == m ? (int64_t)n : (int64_t)k[j];
      for (int64_t v = prev + 1; v <= cur; ++v) off[v] = (uint32_t)i;
      prev = cur;
    }
  }
}

// --------------------------------------------------------------- layout ----
static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct GraphLayout {
  size_t out_off, in_off, out_src, out_dst, out_eid, out_t, in_src, in_eid, in_dst, in_t,
      pair_dst, out_rec, in_rec, pair_eid, pair_t, pair_hash, pair_skip, status, found, trange,
      plan, low, hist, part, part_elems, spill_count,
      rr[4], total;
};

static GraphLayout graph_layout(int32_t n, int64_t m) {
  GraphLayout L;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o += align256(bytes ? bytes : 1);
    return at;
  };
  const size_t M = (size_t)m;
  // rows of the count matrices: never fewer than a smaller graph's, whose
  // smaller tiles can be more, so that a workspace serves every smaller graph
  const int64_t most = sort_tiles(kLargeFrom - 1);
  const int64_t ntiles = large_tiles(m) && sort_tiles(m) < most ? most : sort_tiles(m);
  L.out_off = take(((size_t)n + 1) * 4);
  L.in_off = take(((size_t)n + 1) * 4);
  L.out_src = take(M * 4);
  L.out_dst = take(M * 4);
  L.out_eid = take(M * 4);
  L.out_t = take(M * 8);
  L.in_src = take(M * 4);
  L.in_eid = take(M * 4);
  L.in_dst = take(M * 4);
  L.in_t = take(M * 8);
  L.pair_dst = take(M * 4);
  L.pair_eid = take(M * 4);
  L.pair_t = take(M * 8);
  L.out_rec = take(M * 16);
  L.in_rec = take(M * 16);
  L.pair_hash = take(sizeof(PairSlot) << pair_hash_log2(m));
  L.pair_skip =
      take((size_t)(skip_level_len(m, 1) + skip_level_len(m, 2) + skip_level_len(m, 3)) * 8);
  L.status = take(16);
  L.found = take(kMaxFound * sizeof(Found));
  L.trange = take(16);
  L.plan = take(sizeof(BuildPlan));
  // sort scratch: four 16-byte-record buffers
  for (int b = 0; b < 4; ++b) L.rr[b] = take((M + 1) * 16);
  L.low = take((size_t)kMaxBins * ntiles * 4);
  // (the grouping of the run table uses the same matrix and scan scratch)
  const int64_t groups = (int64_t)1 << group_log2(pair_hash_log2(m));
  const size_t rows = (size_t)kMaxBins * (size_t)ntiles, grows = (size_t)(groups * run_tiles(m));
  L.hist = take((rows > grows ? rows : grows) * 4);
  // scan scratch of the histogram column scan
  L.part_elems = col_scan_scratch_elems(ntiles, kMaxBins);
  const size_t gpart = col_scan_scratch_elems(run_tiles(m), (int)groups);
  if (gpart > L.part_elems) L.part_elems = gpart;
  L.spill_count = take(4);
  L.part = take(L.part_elems * 4);
  L.total = o;
  return L;
}

size_t graph_workspace_bytes(int32_t n, int64_t m) { return graph_layout(n, m).total; }

static int bitlen(uint64_t x) { return x ? 64 - __builtin_clzll(x) : 0; }

tc_status build_graph(int32_t n, int64_t m, const int32_t* src, const int32_t* dst,
                      const int64_t* t, void* ws, size_t ws_bytes, hipStream_t st, tc_graph* g) {
  GraphLayout L = graph_layout(n, m);
  if (ws_bytes < L.total) return TC_E_WORKSPACE;
  char* base = (char*)ws;
  g->n = n;
  g->m = m;
  g->out_off = (uint32_t*)(base + L.out_off);
  g->in_off = (uint32_t*)(base + L.in_off);
  g->out_src = (int32_t*)(base + L.out_src);
  g->out_dst = (int32_t*)(base + L.out_dst);
  g->out_eid = (int32_t*)(base + L.out_eid);
  g->out_t = (int64_t*)(base + L.out_t);
  g->in_src = (int32_t*)(base + L.in_src);
  g->in_eid = (int32_t*)(base + L.in_eid);
  g->in_dst = (int32_t*)(base + L.in_dst);
  g->in_t = (int64_t*)(base + L.in_t);
  g->pair_dst = (int32_t*)(base + L.pair_dst);
  g->pair_eid = (int32_t*)(base + L.pair_eid);
  g->pair_t = (int64_t*)(base + L.pair_t);
  g->status = (uint32_t*)(base + L.status);
  g->t_range = (int64_t*)(base + L.trange);
  g->pair_hash = (void*)(base + L.pair_hash);
  g->pair_hash_log2 = pair_hash_log2(m);
  g->pair_skip = (int64_t*)(base + L.pair_skip);
  g->out_rec = (void*)(base + L.out_rec);
  g->in_rec = (void*)(base + L.in_rec);
  Found* found = (Found*)(base + L.found);
  BuildPlan* plan = (BuildPlan*)(base + L.plan);
  uint32_t* low = (uint32_t*)(base + L.low);
  uint32_t* hist = (uint32_t*)(base + L.hist);
  uint32_t* part = (uint32_t*)(base + L.part);
  uint32_t* spill_count = (uint32_t*)(base + L.spill_count);

  const int vbits = bitlen((uint64_t)(n - 1));
  // validation and the sort plan, on the device
  const int64_t ntiles = sort_tiles(m);
  const int nfound = (int)(ntiles < kMaxFound ? ntiles : kMaxFound);
  if (m > 0)
    hipLaunchKernelGGL(large_tiles(m) ? k_validate<kItemsLarge> : k_validate<kItemsSmall>,
                       dim3((unsigned)nfound), dim3(kSortBlock), 0, st, src, dst, t, m, n, found,
                       low);
  hipLaunchKernelGGL(k_plan, dim3(1), dim3(kMaxFound), 0, st, (const Found*)found, nfound, m,
                     vbits, plan, g->status, g->t_range, spill_count);
  const int lg = g->pair_hash_log2, glog2 = few_pairs(n, m) ? 0 : group_log2(lg);
  const int64_t cap = (int64_t)1 << lg;
  if (m == 0) {
    hipLaunchKernelGGL(k_hash_clear, dim3(blocks_for(cap, 256)), dim3(256), 0, st,
                       (PairSlot*)g->pair_hash, cap);
    hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for((int64_t)n + 1, 256)), dim3(256), 0, st,
                       g->out_off, (int64_t)n + 1, 0u);
    hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for((int64_t)n + 1, 256)), dim3(256), 0, st,
                       g->in_off, (int64_t)n + 1, 0u);
    if (hipGetLastError() != hipSuccess) return TC_E_HIP;
    return TC_OK;
  }
  uint4* rr[4];
  for (int b = 0; b < 4; ++b) rr[b] = (uint4*)(base + L.rr[b]);
  // 1. time order, ending in rr[0] re-keyed as the out-CSR input
  const EdgeCols ec{src, dst, t};
  const SortScratch sc{hist, part, L.part_elems, vbits};
  if (!time_sort(plan, ec, rr[0], rr[1], m, (const uint32_t*)low, sc, st, RX_OUT,
                 (uint4*)g->pair_hash, glog2 == 0 ? cap : 0))
    return TC_E_WORKSPACE;
  // A vertex sort of rr[from] (spare rr[tmp]) whose last pass writes the
  // columns E; with no pass (n = 1) the records are emitted from rr[from].
  // With `in0` >= 0 the sort reads rr[in0] (re-keyed by xf_in) and leaves it
  // as it was, ping-ponging between rr[from] and rr[tmp]; with `ic` its first
  // pass reads the in-list columns instead of rr[from].
  auto sort_emit = [&](int from, int tmp, const EmitCols& E, uint32_t* off, int extra = -1,
                       int xf2 = RX_NONE, int in0 = -1, int xf_in = RX_NONE,
                       const InCols* ic = nullptr, uint32_t* first = nullptr) -> bool {
    const int w = radix_sort(rr[from], rr[tmp], m, vbits, sc, st,
                             extra < 0 ? (uint4*)nullptr : rr[extra], xf2, E,
                             in0 < 0 ? (const uint4*)nullptr : rr[in0], xf_in, ic, first);
    if (w < 0) return false;
    if (w == 0)
      hipLaunchKernelGGL(k_emit, dim3(blocks_for(m + 1, 256)), dim3(256), 0, st,
                         (const uint4*)rr[from], m, (const BuildPlan*)plan, t, E.key,
                         E.other, E.t, E.eid, E.rec, n, vbits, off, E.skip);
    return true;
  };
  // 2. in-CSR: the time order read from rr[0] with src and dst swapped
  //    ((src, eid, dst, t) -> (dst, eid, src, t)), stable by dst, written as
  //    the in-list columns.  With a single vertex (no pass) a copy of the
  //    records re-keyed for the pair index goes to rr[3] instead.
  const bool one = vbits == 0;
  if (!one) {
    // the first histograms of the in-CSR sort (hist) and of the out-CSR sort
    // (low, free now)
    const int db = vertex_digit(vbits, digit_passes(vbits), 0);
    hipLaunchKernelGGL(large_tiles(m) ? k_radix_hist2<kItemsLarge> : k_radix_hist2<kItemsSmall>,
                       dim3((unsigned)sort_tiles(m)), dim3(kSortBlock), 0, st,
                       (const uint4*)rr[0], (const BuildPlan*)plan, db, m, hist, low);
  }
  if (!sort_emit(2, 1,
                 EmitCols{plan, t, g->in_dst, g->in_src, g->in_t, g->in_eid, (uint4*)g->in_rec,
                          nullptr},
                 g->in_off, one ? 3 : -1, RX_PAIR, 0, RX_PAIR, nullptr, one ? nullptr : hist))
    return TC_E_WORKSPACE;
  // 3. pair index: the in-order (dst, t, eid), read from the in-list
  //    columns, stably by src; the pair sources go to the free buffer rr[2]
  int32_t* psrc = (int32_t*)rr[2];
  const InCols ic{(const uint4*)g->in_rec, g->in_dst, g->in_src};
  if (!sort_emit(3, 1,
                 EmitCols{plan, t, psrc, g->pair_dst, g->pair_t, g->pair_eid, nullptr,
                          g->pair_skip},
                 nullptr, -1, RX_NONE, -1, RX_NONE, one ? nullptr : &ic))
    return TC_E_WORKSPACE;
  // 4. the run table: grouped runs in rr[3] and the list of those put aside
  //    in rr[1] (both free until the out-CSR sort), or inserted one by one
  //    into the cleared table
  const PairKeys pk{(const uint32_t*)psrc, (const int32_t*)g->pair_dst, m};
  if (glog2 == 0) {
    hipLaunchKernelGGL(k_hash_insert, dim3(blocks_for(m, 256)), dim3(256), 0, st, pk,
                       (PairSlot*)g->pair_hash, lg, (const BuildPlan*)plan);
  } else {
    const int64_t rt = run_tiles(m);
    const int segs = 1 << glog2;
    const size_t lds = (size_t)4 << (lg - glog2);
    hipLaunchKernelGGL(k_run_hist, dim3((unsigned)rt), dim3(kRunBlock), 0, st, pk, glog2, hist,
                       (const BuildPlan*)plan);
    col_scan(hist, rt, part, PassBins{plan, -1, segs}, st);
    if (hipFuncSetAttribute((const void*)k_run_scatter,
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)run_scatter_lds(kMaxGroupLog2)) != hipSuccess)
      return TC_E_HIP;
    hipLaunchKernelGGL(k_run_scatter, dim3((unsigned)rt), dim3(kRunBlock),
                       run_scatter_lds(glog2), st, pk, glog2, (const uint32_t*)hist,
                       (const uint32_t*)part, rr[3], (const BuildPlan*)plan);
    if (hipFuncSetAttribute((const void*)k_table_segment,
                            hipFuncAttributeMaxDynamicSharedMemorySize, 4 << kMaxSegLog2) !=
        hipSuccess)
      return TC_E_HIP;
    hipLaunchKernelGGL(k_table_segment, dim3((unsigned)segs), dim3(kSegBlock), lds, st,
                       (const uint4*)rr[3], (const uint32_t*)part, lg, glog2,
                       (uint4*)g->pair_hash, (uint32_t*)rr[1], spill_count,
                       (const BuildPlan*)plan);
    hipLaunchKernelGGL(k_table_spill, dim3(64), dim3(256), 0, st, (const uint4*)rr[3],
                       (const uint32_t*)rr[1], (const uint32_t*)spill_count, lg, glog2,
                       (PairSlot*)g->pair_hash);
  }
  // 5. out-CSR: stable by src, from the time order in rr[0]
  if (!sort_emit(0, 1,
                 EmitCols{plan, t, g->out_src, g->out_dst, g->out_t, g->out_eid,
                          (uint4*)g->out_rec, nullptr},
                 g->out_off, -1, RX_NONE, -1, RX_NONE, nullptr, one ? nullptr : low))
    return TC_E_WORKSPACE;
  if (!one)
    hipLaunchKernelGGL(k_offsets, dim3(blocks_for((m + kOffItems) / kOffItems, 256), 2),
                       dim3(256), 0, st,
                       OffCols{{g->in_dst, g->out_src}, {g->in_off, g->out_off}}, m,
                       (const BuildPlan*)plan, n);
  if (hipGetLastError() != hipSuccess) return TC_E_HIP;
  return TC_OK;
}

}  // namespace tc
