// gr_beam_select: beam item step (paper Sections 6.1-6.3) on gfx950.
//
// Two kernels per call, or one for few beams over a short vocabulary (no host synchronisation, no allocation; everything lives in caller buffers):
//   k_rows         one pass over the logits.  A streamed row is read ONCE by a workgroup with 16-byte loads and kept in
//                  registers for the max, the fp64 sum-exp and the keys; the validity bits come straight from the mask
//                  row in memory.  A row with few valid children is gathered by one wavefront, which leaves all of its
//                  candidate scores.
//   k_select       one workgroup per request: top-W of the request's candidates by (score descending, flat index
//                  ascending).  It never sorts the W*V candidates: k_rows leaves the best candidate score of every 16th of a
//                  row; a histogram of these yields a threshold that at least W candidates reach, only what reaches
//                  it is read again (by finer keys that k_rows left too, which yield a higher threshold where the first lets
//                  too much through), and another histogram over that yields the few candidates that are sorted (the
//                  early-termination idea of Section 6.2: stop as soon as the survivors are fixed).  One CU draws some
//                  40 GB/s from memory it has not seen, so what counts is how few cache lines it has to touch.  If the
//                  survivors do not fit in LDS (thousands of equal scores) an exact MSB radix select over all candidates
//                  takes over.
//
// Arithmetic that decides beam order is fixed: m = fp32 max over valid logits, S = fp64 sum of
// exp(x - m), lse = fp32(m + log S), bias = score_in - lse (fp32), cand = bias + x (fp32), with no
// fused multiply-add in the last two operations.
#include <type_traits>
#include "gr_internal.hpp"

namespace {

constexpr int kGroups = 16;         // groups of a row's candidates; the best score of each is kept
// and, per row, this many floats of finer data behind them:
//   streamed row: 256 keys of 16 bits, one for every line of 32 consecutive logits of a block (how far its best score is below the row's);
//   gathered row with at most kScoreMax children: all of their scores;
//   gathered row with more: up to 256 such keys, one for every 8 << key_shift(n) consecutive children.
constexpr int kRowFloats = 240;
constexpr int kLines = 256;
constexpr int kScoreMax = kRowFloats;
constexpr int kWaveMax = 1024;      // a row with at most this many children is gathered by one wavefront, one with more by a workgroup
constexpr int kSelThreads = 1024;
constexpr int kListCap = 8192;      // survivors that fit in LDS
constexpr int kChunkCap = 4096;     // keys whose candidates are looked at again by the fast path
constexpr int kUnitCap = 8192;      // units of four candidates that are
constexpr int kFewMax = 192;        // candidates that are counted against each other
constexpr int kDirectQuads = 512;   // quads of scores of short gathered rows that are all taken at once
constexpr int kHistBins = 2048;
constexpr int kMaxMaskWords = 1024; // V <= 32768
constexpr int kBlockV = 8192;       // logits of a row that a workgroup holds in registers at a time
constexpr int kMaxW = 2048;
constexpr int kGroupCap = 2 * kListCap;  // key groups (floats in the list's place)
constexpr size_t kSelLdsBytes = (size_t)kListCap * 8 + (size_t)kUnitCap * 4 + (size_t)kHistBins * 4 + (size_t)kChunkCap * 4 + (size_t)kMaxW * 16;

enum { ROW_DEAD = 0, ROW_DENSE = 1, ROW_SPARSE = 2, ROW_DONE = 3 };      // low bits of row_info; the child count of a gathered row above them.  DONE (a
                                                                         // request's first row): k_rows has written the request's outputs

struct SelCtx {
  int B, W, V, depth, step;
  int row_threads;           // threads that stream a row: thread t holds tokens 4 (t + row_threads i) .. + 3 for all i
  int unit_shift;            // log2 of the units (float4 of logits) behind a key of a streamed row: 8 per block of kBlockV logits, to a power of two
  const char* blob;          // mask blob or nullptr
  const float* logits;
  const float* scores_in;
  const int32_t* prefix_in;
  const int32_t* range_in;
  int32_t* parent_out;
  int32_t* token_out;
  float* scores_out;
  int32_t* prefix_out;
  int32_t* range_out;
  int32_t* item_index_out;
  float* row_bias;           // workspace [B*W]
  int32_t* row_info;         // workspace [B*W]
  int32_t* row_start;        // workspace [B*W]: first child of a gathered row in the pair list (level 1) or in the table (level 2)
  float* row_group;          // workspace [B*W*kGroups]
  float* row_data;           // workspace [B*W*kRowFloats]
};

// four consecutive logits; a row begins at any multiple of 4 bytes
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(4)));

struct MaskView {
  const uint32_t* l0;
  const uint32_t* l1;
  const int32_t* off1;
  const int32_t* pair_off;
  const int32_t* pair_t2;
  const int32_t* pair_row;
  const int32_t* t3;
  int words;
  int64_t n_items;
  bool ok;                   // header matches the call (magic, V, depth)
};

__device__ __forceinline__ MaskView mask_view(const char* blob, int V, int depth) {
  const gr_mask_header* h = (const gr_mask_header*)blob;
  MaskView m;
  m.l0 = (const uint32_t*)(blob + h->off_l0);
  m.l1 = (const uint32_t*)(blob + h->off_l1);
  m.off1 = (const int32_t*)(blob + h->off_off1);
  m.pair_off = (const int32_t*)(blob + h->off_pair_off);
  m.pair_t2 = (const int32_t*)(blob + h->off_pair_t2);
  m.pair_row = (const int32_t*)(blob + h->off_pair_row);
  m.t3 = (const int32_t*)(blob + h->off_t3);
  m.words = h->words;
  m.n_items = h->n_items;
  m.ok = h->magic == GR_MASK_MAGIC && h->V == V && h->depth == depth;
  return m;
}

// The kernel's arguments, read where this stands and not before.
typedef const __attribute__((address_space(4))) SelCtx* LateArgs;
__device__ __forceinline__ LateArgs late_args() {
  LateArgs a = (LateArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return a;
}

// The valid children of a beam row (steps 1 and 2): entries [start, start + n) of the pair list or of the table.  A prefix
// or range that this mask could not have produced yields none instead of an out-of-bounds read.
__device__ __forceinline__ void row_children(const SelCtx& c, const MaskView& mv, int row, int* start, int* n) {
  *start = 0; *n = 0;
  if (!mv.ok) return;
  if (c.step == 1) {
    const int t1 = c.prefix_in[(size_t)row * c.depth];
    if (t1 >= 0 && t1 < c.V) { *start = mv.pair_off[t1]; *n = mv.pair_off[t1 + 1] - *start; }
  } else {
    const int lo = c.range_in[2 * (size_t)row], hi = c.range_in[2 * (size_t)row + 1];
    // (at most V: the place of a child and the unit it falls in are packed for no more)
    if (lo >= 0 && hi >= lo && (int64_t)hi <= mv.n_items && hi - lo <= c.V) { *start = lo; *n = hi - lo; }
  }
}
__device__ __forceinline__ const int32_t* child_list(const SelCtx& c, const MaskView& mv) { return c.step == 1 ? mv.pair_t2 : mv.t3; }

__device__ __forceinline__ int lower_bound_i32(const int32_t* a, int n, int key) {
  int lo = 0, hi = n;
  while (lo < hi) { int mid = (lo + hi) >> 1; if (a[mid] < key) lo = mid + 1; else hi = mid; }
  return lo;
}

// e^(x - ref) in fp64 for fp32 x <= ref (and not more than ~700 below it), about 2e-14 relative:
//   t = (x - ref) * 256/ln2 = n + f with n = rint(t), |f| <= 1/2, both from one addition of 1.5 * 2^52 (the sum's
//   low word then holds n); e^(x-ref) = 2^(n>>8) * 2^((n&255)/256) * 2^(f/256) with 2^(f/256) = c0 + f (c1 + f (c2 + f c3)):
//   the Taylor terms c_k = (ln2/256)^k / k! with the fourth one spread over c0 and c2 as its Chebyshev expansion on |f| <= 1/2
//   says (f^4 = f^2/4 - 1/128 + T_4(2 f)/128: what is left is below 2e-14).  The middle factor comes from a 256-entry table in
//   LDS whose high words have their index subtracted, so that one shift-and-add of n makes both factors at once.
//   Nine fp64 and three integer operations, all at the full rate (no rounding, conversion-to-integer or ldexp instruction);
//   the exponentials are what a streamed row costs beside its bytes.  The error is far below what the single fp32 rounding
//   of lse = m + log S can see.
// The constants live in scalar registers (set up once per kernel): left to itself the compiler
// re-materialises each 64-bit literal with vector moves next to every use.
struct ExpK { double c, magic, c0, c1, c2, c3; };
__device__ __forceinline__ ExpK exp_consts() {
  ExpK k = {0x1.71547652b82fep+8, 0x1.8p+52, 0x1.fffffffffff62p-1, 0x1.62e42fefa39efp-9, 0x1.ebfbe4e4d734ep-19, 0x1.c6b08d704a0c0p-29};
  asm volatile("" : "+s"(k.c), "+s"(k.magic), "+s"(k.c0), "+s"(k.c1), "+s"(k.c2), "+s"(k.c3));
  return k;
}
__constant__ double c_exp_tab[64] = {        // 2^(j/64), correctly rounded
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0};
constexpr int kExpTab = 256;
__device__ __forceinline__ void fill_exp_tab(double* tab, int threads) {      // (the caller's barrier publishes it)
  for (int j = threadIdx.x; j < kExpTab; j += threads) {
    const double q = (j & 1) ? ((j & 2) ? 0x1.02168143b0281p+0 : 0x1.00b1afa5abcbfp+0) : ((j & 2) ? 0x1.0163da9fb3335p+0 : 1.0);    // 2^((j & 3)/256)
    const double v = c_exp_tab[j >> 2] * q;
    tab[j] = __hiloint2double(__double2hiint(v) - (j << 12), __double2loint(v));
  }
}
// S + e^(x - ref); rc = -(double)ref * k.c; x must be >= ref - 600 (callers clamp: what is cut off is below 1e-260 of the sum)
__device__ __forceinline__ double exp_add(double S, float x, double rc, const double* tab, const ExpK& k) {
  const double t = fma((double)x, k.c, rc);
  const double u = t + k.magic;
  const uint32_t n = (uint32_t)__double2loint(u);
  const double f = t - (u - k.magic);
  double p = fma(f, k.c3, k.c2);
  p = fma(p, f, k.c1);
  p = fma(p, f, k.c0);
  const double tj = tab[n & (kExpTab - 1)];
  return fma(__hiloint2double(__double2hiint(tj) + (int)(n << 12), __double2loint(tj)), p, S);
}
__device__ __forceinline__ double exp_rel(float x, double rc, const double* tab, const ExpK& k) { return exp_add(0.0, x, rc, tab, k); }
// max without the NaN-quieting instructions fmaxf() drags in (NaN inputs are outside the contract)
__device__ __forceinline__ float max_raw(float a, float b) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Wavefront reductions: within rows of 16 lanes by DPP, across the four rows by lane reads (the result is wave-uniform).
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140, kXor8 = 0x128;       // (row_ror:8)
__device__ __forceinline__ float quad_max(float v) {
  v = max_raw(v, dpp_f32<kXor1>(v));
  return max_raw(v, dpp_f32<kXor2>(v));
}
__device__ __forceinline__ float lane_f32(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }
__device__ __forceinline__ float wave_max(float v) {
  v = quad_max(v);
  v = max_raw(v, dpp_f32<kHalfMirror>(v));
  v = max_raw(v, dpp_f32<kMirror>(v));
  return max_raw(max_raw(lane_f32(v, 0), lane_f32(v, 16)), max_raw(lane_f32(v, 32), lane_f32(v, 48)));
}
// The maximum over eight lanes of each of several values, in exchange steps (the first mirrored, so that every step stays inside the
// eight lanes) that each halve the values a lane still carries: `a` is carried on by lanes without the bit, `b` by lanes with it.
template <int CTRL>
__device__ __forceinline__ float half_max(float a, float b, bool bit) { return max_raw(bit ? b : a, dpp_f32<CTRL>(bit ? a : b)); }
// eight values: a lane ends with value 4 (bit 2) + 2 (bit 0) + (bit 1) of its number
__device__ __forceinline__ float best_of_eight(const float (&x)[8]) {
  const int lane = threadIdx.x;
  const bool b2 = lane & 4, b0 = lane & 1, b1 = lane & 2;
  float u[4], v[2];
#pragma unroll
  for (int i = 0; i < 4; i++) u[i] = half_max<kHalfMirror>(x[i], x[i + 4], b2);
#pragma unroll
  for (int i = 0; i < 2; i++) v[i] = half_max<kXor1>(u[i], u[i + 2], b0);
  return half_max<kXor2>(v[0], v[1], b1);
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane_f64(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<kXor1>(v);
  v += dpp_f64<kXor2>(v);
  v += dpp_f64<kHalfMirror>(v);
  v += dpp_f64<kMirror>(v);
  return (lane_f64(v, 0) + lane_f64(v, 16)) + (lane_f64(v, 32) + lane_f64(v, 48));
}
// inclusive prefix sum over the lanes
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);       // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);       // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);       // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);       // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);       // lane 15 of rows 0, 2 to rows 1, 3
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);       // lane 31 to rows 2, 3
  return v;
}

// lanes of the mask in front of this one
__device__ __forceinline__ uint32_t rank_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// sum over aligned groups of 1 << sh lanes, sh = 2 to 4
__device__ __forceinline__ int lanes_sum(int v, int sh) {
  v += __builtin_amdgcn_update_dpp(0, v, kXor1, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, kXor2, 0xf, 0xf, true);
  if (sh > 2) v += __builtin_amdgcn_update_dpp(0, v, kHalfMirror, 0xf, 0xf, true);
  if (sh > 3) v += __builtin_amdgcn_update_dpp(0, v, kMirror, 0xf, 0xf, true);
  return v;
}

// Workgroup reductions with ONE barrier each: the per-wavefront partials go to one of two slot sets, used
// alternately (every thread makes the same sequence of calls: `par` counts them), so a wavefront that is
// already writing the next reduction's partials cannot disturb a slower one that still reads this one's; the
// set after that is only written behind the next reduction's barrier.  s_red holds 2 * NWAVES entries.
template <int NWAVES>
__device__ __forceinline__ void block_max_min(float& mx, float& mn, float2* s_red, int& par) {
  mx = wave_max(mx);
  mn = -wave_max(-mn);
  float2* slot = s_red + (par++ & 1) * NWAVES;
  if (gr_lane() == 0) slot[threadIdx.x >> 6] = make_float2(mx, mn);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NWAVES; i++) { const float2 r = slot[i]; mx = fmaxf(mx, r.x); mn = fminf(mn, r.y); }
}
// exclusive prefix of v over the workgroup's threads (thread order), and the total
template <int NWAVES>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* total, uint32_t* s_red, int& par) {
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));                              // (k_rows: the comparisons below, made ahead of its loop over rows, took up its scalar registers)
  const int lane = gr_lane(), wave = tid >> 6;
  const uint32_t incl = wave_incl_scan(v);
  uint32_t* slot = s_red + (par++ & 1) * NWAVES;
  if (lane == 63) slot[wave] = incl;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NWAVES; i++) { const uint32_t t = slot[i]; if (i < wave) base += t; tot += t; }
  *total = tot;
  return base + incl - v;
}

__device__ __forceinline__ uint64_t composite(float score, uint32_t flat) {
  return ((uint64_t)gr_ordkey(score + 0.0f) << 32) | (uint64_t)(0xffffffffu - flat);     // (+0.0f: -0 and +0 are one score)
}

// Monotone (non-increasing in the score) histogram bin of a score below the best, `hi`; bins of one width.
__device__ __forceinline__ int key_bin(float hi, float scale, float score) {
  return (int)fminf(fmaxf((hi - score) * scale, 0.f), (float)(kHistBins - 1));
}

constexpr float kNoThreshold = -3.402823466e38f;       // the lowest float: every candidate reaches it

// Bins for thresholds, of the distance below the best score `hi` (monotone: a better score is never in a later bin), even in the logarithm:
// 128 to an octave over the 16 octaves below `range`, or below 4096 where that is wider.  So they are as fine for scores that
// lie close together as for scores far apart, and a few scores far below do not make the others' bins coarse.  What lies
// lower is in the last bin.
struct Bins {
  float hi;
  int base;
  __device__ __forceinline__ int of(float score) const {
    return min(max((int)(__float_as_uint(fmaxf(hi - score, 0.f)) >> 16) - base, 0), kHistBins - 1);
  }
  // a score that everything in bins 0..thr reaches (a little low: rounding may only let more through)
  __device__ __forceinline__ float floor_of(int thr) const {
    const float d = __uint_as_float((uint32_t)(thr + 1 + base) << 16);
    return thr < kHistBins - 1 ? hi - d - 1e-6f * (fabsf(hi) + d) : kNoThreshold;
  }
};
__device__ __forceinline__ Bins make_bins(float hi, float range) {
  return Bins{hi, (int)(__float_as_uint(fminf(range, 4096.f)) >> 16) - (kHistBins - 2)};
}

// Smallest bin t with at least `want` entries in bins 0..t (bin 0 = best scores); the last bin when there are fewer
// than `want` entries in total.  Done by the whole workgroup (every thread owns kHistBins / NT consecutive
// bins; one scan, one barrier inside): a serial walk by one wavefront over 32 bins per lane costs more than a
// microsecond.  Leaves the histogram cleared.  The caller puts a barrier behind it before reading *s_thr.  Returns the number of entries.
template <int NT>
__device__ __forceinline__ uint32_t hist_threshold_all(uint32_t* s_hist, uint32_t want, int* s_thr, uint32_t* s_redu, int& par) {
  constexpr int per = kHistBins / NT;
  const int tid = threadIdx.x;
  uint32_t h[per], local = 0;
#pragma unroll
  for (int k = 0; k < per; k++) { h[k] = s_hist[tid * per + k]; local += h[k]; s_hist[tid * per + k] = 0; }
  uint32_t total;
  const uint32_t below = block_excl_scan<NT / 64>(local, &total, s_redu, par);
  if (total < want) {
    if (tid == 0) *s_thr = kHistBins - 1;
  } else if (below < want && want <= below + local) {
    uint32_t acc = below;
    int bin = tid * per;
#pragma unroll
    for (int k = 0; k < per; k++) {
      acc += h[k];
      if (acc >= want) break;
      bin++;
    }
    *s_thr = bin;
  }
  return total;
}

// Histogram of the candidates' bins -> its exclusive prefix, in place, and in *s_thr the bin that holds the want-th candidate (the last one
// when there are fewer).  The caller puts a barrier behind it.  Returns the most candidates in one of this thread's bins.
template <int NT>
__device__ __forceinline__ uint32_t hist_prefix(uint32_t* s_hist, uint32_t want, int* s_thr, uint32_t* s_redu, int& par) {
  constexpr int per = kHistBins / NT;
  const int tid = threadIdx.x;
  uint32_t h[per], sum = 0, most = 0;
#pragma unroll
  for (int k = 0; k < per; k++) { h[k] = s_hist[tid * per + k]; sum += h[k]; most = max(most, h[k]); }
  uint32_t total;
  uint32_t run = block_excl_scan<NT / 64>(sum, &total, s_redu, par);
  if (tid == 0 && total < want) *s_thr = kHistBins - 1;
#pragma unroll
  for (int k = 0; k < per; k++) {
    s_hist[tid * per + k] = run;
    if (run < want && run + h[k] >= want) *s_thr = tid * per + k;
    run += h[k];
  }
  return most;
}
// Orders the m candidates of `list` (n in all) in bins up to `cut` (descending composite key = score descending, flat index ascending).
// Histogram bins are ordered by score, so a survivor's place is the number of survivors in better bins plus its rank inside its own
// (tiny) bin.  Counting sort by bin, then every survivor counts the larger keys of its bin.  Exact ties share a bin and are ranked
// by the key's flat-index half there.
template <int NT>
__device__ __forceinline__ void order_by_bins(uint64_t* list, uint64_t* tmp, uint32_t* s_hist, int n, int m, int cut, float hi, float scale) {
  auto bin_of = [&](uint64_t key) { return key_bin(hi, scale, gr_ordkey_inv((uint32_t)(key >> 32))); };
#pragma unroll 1
  for (int i = threadIdx.x; i < n; i += NT) {
    const uint64_t key = list[i];
    const int bin = bin_of(key);
    if (bin <= cut) tmp[atomicAdd(&s_hist[bin], 1u)] = key;            // the bin's counter now runs to the bin's end
  }
  __syncthreads();
#pragma unroll 1
  for (int q = threadIdx.x; q < m; q += NT) {
    const uint64_t key = tmp[q];
    const int bin = bin_of(key);
    const int s0 = bin ? (int)s_hist[bin - 1] : 0, s1 = (int)s_hist[bin];
    int cnt = 0;
    for (int j = s0; j < s1; j++) cnt += tmp[j] > key;
    list[s0 + cnt] = key;
  }
  __syncthreads();
}

// ------------------------------------------------------------------------------------------------
// Rows that are streamed in full: one workgroup per row.
// ------------------------------------------------------------------------------------------------
template <int NT>
struct RowLds {
  float q[NT / 64][kBlockV / (NT / 64) / 4];     // valid logits of a thinly populated block, per wavefront
  double tab[kExpTab];
  double s[2][NT / 64];                // per-wavefront sums and maxima, and the best logit behind every key; two sets, used in turn
  float m[2][NT / 64];                 // by successive rows
  float key[2][kLines];
  uint32_t mask[kMaxMaskWords];        // validity bits of a last-level row with many children
};

// What the workgroup of a request's only live row needs to select as well.
constexpr int kPickCap = 2432;         // candidates that reach the threshold
constexpr int kPickW = 1024;
struct PickLds {
  uint64_t list[kPickCap], tmp[kPickCap];
  uint32_t hist[kHistBins];
  uint32_t red[2 * 8];
  float top[8], low[8];                // per wavefront: the best logit, the logit down to which the threshold is looked for
  uint32_t others[8];                  // and whether it saw another live row of the request
  uint32_t n, crowded;
  int thr;
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
__device__ __forceinline__ float keep_if_bit(float x, uint32_t bits, int k) {        // x where bit k is set, else -inf
  const uint32_t mask = (uint32_t)((int32_t)(bits << (31 - k)) >> 31);
  return __uint_as_float((mask & __float_as_uint(x)) | (~mask & 0xff800000u));
}

// The 16-bit key of a score in a row: its distance to the row's best score, rounded down to 8 bits of mantissa (so that scores close
// together but far from 0 keep their order).  Larger scores have smaller or equal keys: what reaches a threshold T <= best has a
// key of at most key16(best, T).  The key of -inf is above those of all finite scores.
constexpr uint32_t kKeyLast = 0xfeffu;
__device__ __forceinline__ uint32_t key16(float best, float score) {
  const uint32_t k = __float_as_uint(best - score) >> 15;
  return score > -INFINITY ? min(k, kKeyLast) : kKeyLast + 1u;
}
// a score that one with this key is not below (the rounding of these differences is allowed for where a threshold is made of it)
__device__ __forceinline__ float key16_low(float best, uint32_t key) { return best - __uint_as_float((key + 1u) << 15); }

__device__ __forceinline__ void mark_dead(const SelCtx& c, int row) { c.row_info[row] = ROW_DEAD; }

// What a streamed row leaves, by one wavefront; keys: the best logit of every line.
__device__ __forceinline__ void row_leaves(const SelCtx& c, int row, float bias, float best, const float* keys) {
  const int tid = threadIdx.x & 63;
  if (tid == 0) { c.row_bias[row] = bias; c.row_info[row] = ROW_DENSE; }
  const float4 kl = *(const float4*)&keys[4 * tid];
  const float k0 = __fadd_rn(bias, kl.x), k1 = __fadd_rn(bias, kl.y), k2 = __fadd_rn(bias, kl.z), k3 = __fadd_rn(bias, kl.w);      // (bias is finite)
  uint2 packed;
  packed.x = key16(best, k0) | (key16(best, k1) << 16);
  packed.y = key16(best, k2) | (key16(best, k3) << 16);
  *(uint2*)(c.row_data + (size_t)row * kRowFloats + 2 * tid) = packed;
  const float group = quad_max(max_raw(max_raw(k0, k1), max_raw(k2, k3)));
  if ((tid & 3) == 0) c.row_group[(size_t)row * kGroups + (tid >> 2)] = group;
}

// Bound: HBM and, close behind, the fp64 exponentials: 8192 rows of 8192 logits take 53 us = 5.1 TB/s, of which the vector
// instructions alone are 34 us (650 a wavefront; with the 64-entry table, a polynomial term and an addition more per exponential, a
// barrier per reduction and a compare per validity bit it was 68 us).  Six workgroups a CU: 80 registers, no spills (seven: 66 us).
//
// `row` is live; t1 = first token of its prefix (level 1), [start, start + n_list) = its children where they were looked up
// (all wave-uniform).  Every wavefront works relative to its own maximum and the workgroup meets once: the first wavefront then joins
// the (max, sum) pairs and writes the row's results, while the others are free for the next row (or gone).
template <int NT>
__device__ __forceinline__ void row_dense(const SelCtx& c, const MaskView& mv, RowLds<NT>& L, int row, float s_in, int t1, int start, int n_list, int set) {
  constexpr int NV4 = kBlockV / 4 / NT, NWV = NT / 64;        // float4 per thread; wavefronts
  const int tid = threadIdx.x, wave = tid >> 6, V = c.V;
  const float* x = c.logits + (size_t)row * V;
  const int words = (V + 31) >> 5;
  const uint32_t* mrow = nullptr;                  // the row's validity bits: levels 0 and 1 from the mask, else made in LDS
  const bool all_valid = !c.blob;
  if (c.blob) {
    if (c.step == 0) mrow = mv.ok ? mv.l0 : nullptr;
    else if (c.step == 1) mrow = (mv.ok && t1 >= 0 && t1 < V) ? mv.l1 + (size_t)t1 * mv.words : nullptr;
    else {
      // the last level has no dense mask: the child list is set position by position in an empty LDS mask
      // (Section 6.1's sparse form applied to an existing mask)
      __syncthreads();
      for (int i = tid; i < words; i += NT) L.mask[i] = 0u;
      __syncthreads();
      for (int i = tid; i < n_list; i += NT) { const int v = mv.t3[start + i]; atomicOr(&L.mask[v >> 5], 1u << (v & 31)); }
      __syncthreads();
    }
    if (c.step < 2 && !mrow) {
      if (tid == 0) mark_dead(c, row);
      return;
    }
  }
  // loads past the end of the row or of its mask words return 0 (hardware bounds check); bits past V are 0
  const __amdgpu_buffer_rsrc_t rx = buffer_of(x, (uint32_t)(V & ~3) * 4), rm = buffer_of(mrow, (uint32_t)words * 4);
  const ExpK ek = exp_consts();
  float lmax[NV4], m = -INFINITY;                  // this thread's best valid logit of each load; the wavefront's of all
#pragma unroll
  for (int i = 0; i < NV4; i++) lmax[i] = -INFINITY;
  double S = 0.0;                                  // the wavefront's sum relative to m
  float xv[4 * NV4];
#pragma unroll 1
  for (int v0 = 0; v0 < V; v0 += kBlockV) {
    // ---- one block of the row: logits and validity bits requested together
    u32x4 xr[NV4];
    uint32_t mw[NV4];
#pragma unroll
    for (int i = 0; i < NV4; i++) xr[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, (v0 + 4 * tid) * 4 + i * (NT * 16), 0, 0);
    if (mrow) {
#pragma unroll
      for (int i = 0; i < NV4; i++) mw[i] = __builtin_amdgcn_raw_buffer_load_b32(rm, (v0 >> 5) * 4 + (tid >> 3) * 4 + i * (NT / 2), 0, 0);
    }
    // validity bits: bit 4 i + j <-> token v0 + 4 (tid + i * NT) + j
    uint32_t vbits = 0xffffffffu;
    const bool whole = all_valid && v0 + kBlockV <= V;
    if (!whole) {
      vbits = 0;
#pragma unroll
      for (int i = 0; i < NV4; i++) {
        const int v = v0 + 4 * (tid + i * NT);
        uint32_t w;
        if (mrow) w = mw[i] >> (4 * (tid & 7));
        else if (all_valid) { const int left = V - v; w = left >= 4 ? 0xfu : left > 0 ? (1u << left) - 1u : 0u; }
        else w = v < V ? L.mask[v >> 5] >> (v & 31) : 0u;
        vbits |= (w & 0xfu) << (4 * i);
      }
    }
    const int tail = (V >> 2) - (v0 >> 2);         // the float4 that the row ends in, when it is a part of one
    if ((V & 3) && tail >= 0 && tail < kBlockV / 4 && (tail & (NT - 1)) == tid) {
      u32x4 t = {0, 0, 0, 0};
      const float* xt = x + (V & ~3);
      t.x = __float_as_uint(xt[0]);
      if ((V & 3) > 1) t.y = __float_as_uint(xt[1]);
      if ((V & 3) > 2) t.z = __float_as_uint(xt[2]);
#pragma unroll
      for (int i = 0; i < NV4; i++) if (i == tail / NT) xr[i] = t;
    }
#pragma unroll
    for (int i = 0; i < NV4; i++) {
      xv[4 * i] = __uint_as_float(xr[i].x); xv[4 * i + 1] = __uint_as_float(xr[i].y);
      xv[4 * i + 2] = __uint_as_float(xr[i].z); xv[4 * i + 3] = __uint_as_float(xr[i].w);
    }
    // invalid entries become -inf: they lose every max and add nothing to the sum
    if (!whole) {
#pragma unroll
      for (int e = 0; e < 4 * NV4; e++) xv[e] = keep_if_bit(xv[e], vbits, e);
    }
    float bmax = -INFINITY;
#pragma unroll
    for (int i = 0; i < NV4; i++) {
      const float mi = max_raw(max_raw(xv[4 * i], xv[4 * i + 1]), max_raw(xv[4 * i + 2], xv[4 * i + 3]));
      lmax[i] = max_raw(lmax[i], mi);
      bmax = max_raw(bmax, mi);
    }
    const float mb = wave_max(bmax);
    if (!(mb > -INFINITY)) continue;               // (wave-uniform)
    const double rc = -(double)mb * ek.c;
    const float lo = mb - 600.f;
    double Sb = 0.0;
    // Thinly populated block (up to a quarter of the wavefront's logits are valid): the valid ones are packed into a
    // queue (lane order, so the sum is reproducible) and exponentiated with full lanes.
    bool packed = false;
    if (!whole) {
      const uint32_t mine = (uint32_t)__popc(vbits), incl = wave_incl_scan(mine);
      const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
      packed = total <= (uint32_t)(kBlockV / NWV / 4);
      if (packed) {
        float* q = L.q[wave];
        uint32_t pos = incl - mine;
#pragma unroll
        for (int e = 0; e < 4 * NV4; e++)
          if ((vbits >> e) & 1u) q[pos++] = xv[e];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
        for (uint32_t i = tid & 63; i < total; i += 64) Sb = exp_add(Sb, max_raw(q[i], lo), rc, L.tab, ek);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
    }
    if (!packed) {
#pragma unroll
      for (int i = 0; i < NV4; i++) {
        if (v0 + 4 * NT * i < V) {                 // (uniform)
#pragma unroll
          for (int j = 0; j < 4; j++) Sb = exp_add(Sb, max_raw(xv[4 * i + j], lo), rc, L.tab, ek);
        }
        // keep the four exponentials of a load together: hoisting the first halves of all costs a hundred registers
        asm volatile("" : "+v"(Sb)::"memory");
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (v0 > 0) {
      // join with the blocks before (-inf counts nothing: what is cut off at -600 is below 1e-260 of the sum)
      const float mn = max_raw(m, mb);
      const double rn = -(double)mn * ek.c;
      S = S * exp_rel(max_raw(m, mn - 600.f), rn, L.tab, ek);
      Sb = Sb * exp_rel(max_raw(mb, mn - 600.f), rn, L.tab, ek);
      m = mn;
    } else {
      m = mb;
    }
    S += Sb;
  }
  S = wave_sum(S);
  if ((tid & 63) == 0) { L.m[set][wave] = m; L.s[set][wave] = S; }
  // The best logit of every line = of eight neighbouring threads, for each of their NV4 loads.
  {
    const bool b2 = tid & 4, b0 = tid & 1, b1 = tid & 2;
    float* key = L.key[set] + (tid >> 3) * NV4;
    if constexpr (NV4 == 8) {
      key[4 * b2 + 2 * b0 + b1] = best_of_eight(lmax);
    } else {
      float v[2];
#pragma unroll
      for (int i = 0; i < 2; i++) v[i] = half_max<kHalfMirror>(lmax[i], lmax[i + 2], b2);
      float r = half_max<kXor1>(v[0], v[1], b0);
      r = max_raw(r, dpp_f32<kXor2>(r));
      if (!b1) key[2 * b2 + b0] = r;
    }
  }
  __syncthreads();
  if (wave != 0) return;
  const int lane = tid & 63;
  m = (lane < NWV) ? L.m[set][lane] : -INFINITY;
  S = (lane < NWV) ? L.s[set][lane] : 0.0;
  const float M = wave_max(m);
  if (!(M > -INFINITY)) {
    if (tid == 0) mark_dead(c, row);
    return;
  }
  const double T = wave_sum(S * exp_rel(max_raw(m, M - 600.f), -(double)M * ek.c, L.tab, ek));
  const float lse = (float)((double)M + log(T));
  const float bias = __fsub_rn(s_in, lse);
  const float best = __fadd_rn(bias, M);
  row_leaves(c, row, bias, best, L.key[set]);
}

// Level 0, where as a rule one row of a request is live, its first: this is that row.  Where the request's other rows are all dead, the workgroup, which holds
// all of the request's candidates in registers, selects the W best too, and k_select then only finds that it is done: a level-0
// step of 8 x 128 beams over 8192 tokens 18.0 -> 12.9 us, of 128 x 256 18.8 -> 13.6, of one x 16 over 256 13.4 -> 10.1.
//
// Bound: the chain of steps in one workgroup.  So the row's logits are asked for before it is known to be live; the threshold that W candidates
// reach is looked for among the logits, beside the exponentials (rounding a sum is monotone: what reaches a logit reaches its score); it is
// found among the best of every four where they are enough; candidates get their places a wavefront at a time, and few of them
// are counted against each other.  A call without and with these, us: one request x 16 beams over 256 tokens 10.1, 9.6; one x 128 over 8192 12.3, 11.3; 8 x 128
// with a mask 13.8, 12.6.
//
// The best of every four (by_load) for up to a sixth of the tokens: beyond that the threshold among them lets through many more than are wanted.  us by all
// candidates and by fours: 256 tokens x 64 beams 9.9, 10.4; 1024 x 256 11.0, 11.0; 4096 x 600 13.0, 12.6; 4096 x 512 12.3, 11.9; 8192 x 512 13.9, 12.6; but 4096 x 1024,
// where they did not fit the list and the request was left to k_select, 14.1, 23.8.  And only where four candidates for every beam, and some, fit the
// list, so that it holds them however alike the four are: 8192 x 1024 with the logits of a four as good as equal 16.0, 26.3
// (all different 15.3, 14.6), 8192 x 512, which four times fit, 13.9 (15.2 by all).
constexpr int kPickFew = 96;           // candidates that are counted against each other: 128 take as long as by bins or longer (300 tokens x 128 beams 10.9 us, 10.6 by bins)
template <int NT>
__device__ __forceinline__ void row_first(const SelCtx& c, const MaskView& mv, RowLds<NT>& L, PickLds& P, int row) {
  constexpr int NV4 = kBlockV / 4 / NT, NWV = NT / 64;        // float4 per thread; wavefronts
  static_assert(NV4 == 4 && NWV == 8 && kPickW <= 2 * NT && 4 * NT <= kPickCap, "a list of one load at least, two other rows to a thread");
  static_assert(kPickFew <= NT / 4, "four threads to a candidate that is counted");
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));                              // (what follows from it is not made ahead of the loop over rows and spilled)
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), V = c.V, words = (V + 31) >> 5;
  const float* x = c.logits + (size_t)row * V;
  const bool all_valid = !c.blob;
  const __amdgpu_buffer_rsrc_t rx = buffer_of(x, (uint32_t)(V & ~3) * 4);
  u32x4 xr[NV4];
  uint32_t mw[NV4];
#pragma unroll
  for (int i = 0; i < NV4; i++) xr[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, 16 * tid + i * (NT * 16), 0, 0);
  const float s_in = c.scores_in[row];
  float rival0 = -INFINITY, rival1 = -INFINITY;
  if (1 + tid < c.W) rival0 = c.scores_in[row + 1 + tid];
  if (1 + tid + NT < c.W) rival1 = c.scores_in[row + 1 + tid + NT];
  if (__builtin_expect(!all_valid && !mv.ok, 0)) {
    if (tid == 0) mark_dead(c, row);
    return;
  }
  if (!all_valid) {
    const __amdgpu_buffer_rsrc_t rm = buffer_of(mv.l0, (uint32_t)words * 4);
#pragma unroll
    for (int i = 0; i < NV4; i++) mw[i] = __builtin_amdgcn_raw_buffer_load_b32(rm, (tid >> 3) * 4 + i * (NT / 2), 0, 0);
  }
  fill_exp_tab(L.tab, NT);
  for (int i = tid; i < kHistBins; i += NT) P.hist[i] = 0;
  if (tid == 0) { P.n = 0; P.crowded = 0; }
  if (__builtin_expect(!(s_in > -INFINITY), 0)) {
    if (tid == 0) mark_dead(c, row);
    return;
  }
  const bool by_load = 6 * c.W <= V && 4 * c.W + 256 <= kPickCap;
  if (!by_load) __syncthreads();                             // (publishes the table and the empty histogram, while the logits are on their way)
  // validity bits and the row's tail as in row_dense
  uint32_t vbits = 0xffffu;
  const bool whole = all_valid && V == kBlockV;
  if (!whole) {
    vbits = 0;
#pragma unroll
    for (int i = 0; i < NV4; i++) {
      const int left = V - 4 * (tid + i * NT);
      const uint32_t w = !all_valid ? mw[i] >> (4 * (tid & 7)) : left >= 4 ? 0xfu : left > 0 ? (1u << left) - 1u : 0u;
      vbits |= (w & 0xfu) << (4 * i);
    }
  }
  const int tail = V >> 2;
  if ((V & 3) && (tail & (NT - 1)) == tid) {
    u32x4 t = {0, 0, 0, 0};
    const float* xt = x + (V & ~3);
    t.x = __float_as_uint(xt[0]);
    if ((V & 3) > 1) t.y = __float_as_uint(xt[1]);
    if ((V & 3) > 2) t.z = __float_as_uint(xt[2]);
#pragma unroll
    for (int i = 0; i < NV4; i++) if (i == tail / NT) xr[i] = t;
  }
  float xv[4 * NV4], best4[NV4];                             // best4: of each load
#pragma unroll
  for (int i = 0; i < NV4; i++) {
    xv[4 * i] = __uint_as_float(xr[i].x); xv[4 * i + 1] = __uint_as_float(xr[i].y);
    xv[4 * i + 2] = __uint_as_float(xr[i].z); xv[4 * i + 3] = __uint_as_float(xr[i].w);
  }
  if (!whole) {
#pragma unroll
    for (int e = 0; e < 4 * NV4; e++) xv[e] = keep_if_bit(xv[e], vbits, e);
  }
#pragma unroll
  for (int i = 0; i < NV4; i++) best4[i] = max_raw(max_raw(xv[4 * i], xv[4 * i + 1]), max_raw(xv[4 * i + 2], xv[4 * i + 3]));
  const float mb = wave_max(max_raw(max_raw(best4[0], best4[1]), max_raw(best4[2], best4[3])));
  // down to where the threshold is looked for: the worst of all where one load holds them (W may be most of them: 163 beams over 256
  // tokens gave up with the best of every four, 17.9 us instead of 11.2), else the worst of the threads' best of a load
  float low = INFINITY;
  if (V <= 4 * NT) {
#pragma unroll
    for (int j = 0; j < 4; j++) low = fminf(low, xv[j] > -INFINITY ? xv[j] : INFINITY);
  } else {
#pragma unroll
    for (int i = 0; i < NV4; i++) low = fminf(low, best4[i] > -INFINITY ? best4[i] : INFINITY);
  }
  low = -wave_max(-low);
  const bool any = __any(rival0 > -INFINITY || rival1 > -INFINITY);
  if (lane == 0) { P.top[wave] = mb; P.low[wave] = low; P.others[wave] = any; }
  float hi = 0.f, lo = 0.f;
  bool pick = true;
  Bins bins = {0.f, 0};
  auto look = [&]() __attribute__((always_inline)) {
    hi = wave_max(lane < NWV ? P.top[lane & (NWV - 1)] : -INFINITY);
    lo = -wave_max(lane < NWV ? -P.low[lane & (NWV - 1)] : -INFINITY);
    pick = !__any(lane < NWV && P.others[lane & (NWV - 1)]);
    bins = make_bins(hi, hi - lo);
  };
  if (by_load) {
    __syncthreads();                                         // (publishes the table and the empty histogram too)
    look();
    if (__builtin_expect(!(hi > -INFINITY), 0)) {
      if (tid == 0) mark_dead(c, row);
      return;
    }
    if (pick) {
#pragma unroll
      for (int i = 0; i < NV4; i++)
        if (best4[i] > -INFINITY) atomicAdd(&P.hist[bins.of(best4[i])], 1u);
    }
  }
  // the wavefront's sum relative to its own maximum, as in row_dense
  const ExpK ek = exp_consts();
  double S = 0.0;
  if (mb > -INFINITY) {
    const double rc = -(double)mb * ek.c;
    const float cap = mb - 600.f;
    bool packed = false;
    if (!whole) {
      const uint32_t mine = (uint32_t)__popc(vbits), incl = wave_incl_scan(mine);
      const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
      packed = total <= (uint32_t)(kBlockV / NWV / 4);
      if (packed) {
        float* q = L.q[wave];
        uint32_t pos = incl - mine;
#pragma unroll
        for (int e = 0; e < 4 * NV4; e++)
          if ((vbits >> e) & 1u) q[pos++] = xv[e];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
        for (uint32_t i = lane; i < total; i += 64) S = exp_add(S, max_raw(q[i], cap), rc, L.tab, ek);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
    }
    if (!packed) {
#pragma unroll
      for (int i = 0; i < NV4; i++) {
        if (4 * NT * i < V) {                      // (uniform)
#pragma unroll
          for (int j = 0; j < 4; j++) S = exp_add(S, max_raw(xv[4 * i + j], cap), rc, L.tab, ek);
        }
        asm volatile("" : "+v"(S)::"memory");
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  S = wave_sum(S);
  if (lane == 0) { L.m[0][wave] = mb; L.s[0][wave] = S; }
  __syncthreads();
  if (!by_load) {
    look();
    if (__builtin_expect(!(hi > -INFINITY), 0)) {
      if (tid == 0) mark_dead(c, row);
      return;
    }
    if (pick) {
#pragma unroll
      for (int e = 0; e < 4 * NV4; e++)
        if (xv[e] > -INFINITY) atomicAdd(&P.hist[bins.of(xv[e])], 1u);
    }
  }
  const float m_w = (lane < NWV) ? L.m[0][lane & (NWV - 1)] : -INFINITY;
  const double Sw = (lane < NWV) ? L.s[0][lane & (NWV - 1)] : 0.0;
  const double total_S = wave_sum(Sw * exp_rel(max_raw(m_w, hi - 600.f), -(double)hi * ek.c, L.tab, ek));
  const float lse = (float)((double)hi + log(total_S));
  const float bias = __fsub_rn(s_in, lse), best = __fadd_rn(bias, hi);
  // what the row leaves for k_select where it does not select
  auto leave = [&]() {
    {
      const bool b2 = tid & 4, b0 = tid & 1, b1 = tid & 2;
      float v[2];
#pragma unroll
      for (int i = 0; i < 2; i++) v[i] = half_max<kHalfMirror>(best4[i], best4[i + 2], b2);
      float r = half_max<kXor1>(v[0], v[1], b0);
      r = max_raw(r, dpp_f32<kXor2>(r));
      if (!b1) L.key[0][(tid >> 3) * NV4 + 2 * b2 + b0] = r;
    }
    __syncthreads();
    if (wave == 0) row_leaves(c, row, bias, best, L.key[0]);
  };
  if (__builtin_expect(!pick, 0)) { leave(); return; }
  int par = 0;
  if (!by_load) __syncthreads();
  uint32_t total = hist_threshold_all<NT>(P.hist, (uint32_t)c.W, &P.thr, P.red, par);
  __syncthreads();
  float T = bins.floor_of(P.thr);
  if (__builtin_expect(by_load && (T == kNoThreshold || total < (uint32_t)c.W), 0)) {        // (too few of them, or the W-th is among the lowest: all candidates)
#pragma unroll
    for (int e = 0; e < 4 * NV4; e++)
      if (xv[e] > -INFINITY) atomicAdd(&P.hist[bins.of(xv[e])], 1u);
    __syncthreads();
    total = hist_threshold_all<NT>(P.hist, (uint32_t)c.W, &P.thr, P.red, par);
    __syncthreads();
    T = bins.floor_of(P.thr);
  }
  if (__builtin_expect(T == kNoThreshold && total >= (uint32_t)c.W, 0)) { leave(); return; }        // (the W-th lies below lo)
  // what reaches it (all of fewer than W), in bins of one width
  if (T > kNoThreshold) T = __fadd_rn(bias, T);
  const float end = T == kNoThreshold ? __fadd_rn(bias, lo) : T, scale = best > end ? fminf((float)(kHistBins - 1) / (best - end), 1e30f) : 0.f;
  uint32_t in = 0;
#pragma unroll
  for (int e = 0; e < 4 * NV4; e++) {
    xv[e] = __fadd_rn(bias, xv[e]);                          // (scores from here on)
    in |= (xv[e] >= T ? 1u : 0u) << e;
  }
  const uint32_t count = (uint32_t)__popc(in), incl = wave_incl_scan(count);
  uint32_t at = 0;
  if (lane == 63) at = atomicAdd(&P.n, incl);
  at = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + incl - count;
#pragma unroll
  for (int e = 0; e < 4 * NV4; e++) {
    if (!((in >> e) & 1u)) continue;
    atomicAdd(&P.hist[key_bin(best, scale, xv[e])], 1u);
    if (at < (uint32_t)kPickCap) P.list[at] = composite(xv[e], (uint32_t)(4 * (tid + NT * (e / 4)) + (e & 3)));
    at++;
  }
  __syncthreads();
  const int n = (int)P.n;
  const LateArgs late = late_args();
  auto emit = [&](int j, bool some, uint64_t key) {
    const size_t o = (size_t)row + j;
    int32_t* po = late->prefix_out + o * late->depth;
    int token = -1, r_lo = 0, r_hi = 0;
    float score = -INFINITY;
    if (some) {
      token = (int)(0xffffffffu - (uint32_t)key);
      score = gr_ordkey_inv((uint32_t)(key >> 32));
      if (late->blob) { r_lo = mv.off1[token]; r_hi = mv.off1[token + 1]; }
    }
    late->parent_out[o] = some ? 0 : -1;
    late->token_out[o] = token;
    late->scores_out[o] = score;
    po[0] = token;
    for (int k = 1; k < late->depth; k++) po[k] = -1;
    late->range_out[2 * o] = r_lo;
    late->range_out[2 * o + 1] = r_hi;
    if (late->item_index_out) late->item_index_out[o] = -1;
  };
  if (tid == 0) c.row_info[row] = ROW_DONE;
  if (n <= kPickFew) {
    const int sh = n <= 32 ? 4 : n <= 64 ? 3 : 2, i = tid >> sh;
    uint64_t key = 0;
    int better = 0;
    if (i < n) {
      key = P.list[i];
#pragma unroll 4
      for (int j = tid & ((1 << sh) - 1); j < n; j += 1 << sh) better += P.list[j] > key;
    }
    better = lanes_sum(better, sh);
    if (i < n && (tid & ((1 << sh) - 1)) == 0) P.tmp[better] = key;
    __syncthreads();
    for (int j = tid; j < late->W; j += NT) emit(j, j < n, j < n ? P.tmp[j] : 0);
    return;
  }
  bool fits = n <= kPickCap;
  if (__builtin_expect(fits, 1)) {
    if (hist_prefix<NT>(P.hist, (uint32_t)c.W, &P.thr, P.red, par) > 128u) P.crowded = 1u;
    __syncthreads();
    fits = !P.crowded;
  }
  if (__builtin_expect(!fits, 0)) { leave(); return; }
  const int cut = P.thr, m = cut < kHistBins - 1 ? (int)P.hist[cut + 1] : n;
  __syncthreads();                                           // (the bin after the cut is read before any counter moves)
  order_by_bins<NT>(P.list, P.tmp, P.hist, n, m, cut, best, scale);
  for (int j = tid; j < late->W; j += NT) emit(j, j < m, j < m ? P.list[j] : 0);
}

// ------------------------------------------------------------------------------------------------
// Rows whose valid children are listed (Section 6.1's sparse form): only the valid logits are gathered, 512 at a time, by one
// wavefront or by the four of a workgroup.  A row with at most kScoreMax children leaves every candidate's score, its groups
// are of 16 children; one with more leaves a key for every few consecutive children, as a streamed row does for its lines:
// what is read again of it lies together in the child list and, where the list is dense, in the row.  (With 64 keys a row, of
// children 64 apart, k_select took 93 us where 256 beams of each of 16 requests had 8192 children, now 24 us.)
// ------------------------------------------------------------------------------------------------
constexpr int kPartU = 8, kPart = 64 * kPartU;
struct GatherPart {
  float x[kPartU];           // the last kPart logits of this wavefront (all of a short row), -inf past the end
  float m;                   // best logit of the wavefront
  double S;                  // the wavefront's sum relative to m
};
// log2 of the eights of consecutive children behind a key: at most kLines keys
__device__ __forceinline__ int key_shift(int n) { return n <= 8 * kLines ? 0 : 21 - __clz(n - 1); }
// keys of a row and log2 of the keys of a group (at most kGroups groups)
__device__ __forceinline__ int key_count(int n) { return ((n - 1) >> (3 + key_shift(n))) + 1; }
__device__ __forceinline__ int group_shift(int keys) { return keys <= 4 * kGroups ? 2 : keys <= 8 * kGroups ? 3 : 4; }

__device__ __forceinline__ void gather_part(GatherPart& g, const float* x, const int32_t* list, int n, int first, int step, const double* tab,
                                            const ExpK& ek, float* keys) {
  const int lane = threadIdx.x & 63, ks = key_shift(n);
  uint32_t tok[kPartU];      // (row and list at most 128 KB: 32-bit offsets from addresses that all lanes share)
  auto child = [&](int i) { return *(const uint32_t*)((const char*)list + 4u * (uint32_t)min(i + lane, n - 1)); };
  double S = 0.0;
  g.m = -INFINITY;
#pragma unroll
  for (int k = 0; k < kPartU; k++)
    if (first + 64 * k < n) tok[k] = child(first + 64 * k);
#pragma unroll 1
  for (int base = first; base < n; base += step) {
#pragma unroll
    for (int k = 0; k < kPartU; k++)
      if (base + 64 * k < n) g.x[k] = *(const float*)((const char*)x + 4u * tok[k]);       // (uniform; the rest becomes -inf below)
#pragma unroll
    for (int k = 0; k < kPartU; k++)
      if (base + step + 64 * k < n) tok[k] = child(base + step + 64 * k);
    float bmax = -INFINITY;
#pragma unroll
    for (int k = 0; k < kPartU; k++) {
      if (base + 64 * k + lane >= n) g.x[k] = -INFINITY;
      bmax = max_raw(bmax, g.x[k]);
    }
    if (n > kScoreMax) {
      // the best of children base + 64 k + 8 (lane / 8) .. + 7, then of as many eights of these as belong to a key
      float v = best_of_eight(g.x);
      const int k = (lane & 4) + 2 * (lane & 1) + ((lane >> 1) & 1);
      if (ks > 0) v = max_raw(v, dpp_f32<kXor8>(v));
      if (ks > 1) v = max_raw(v, __shfl_xor(v, 16, 64));
      if (ks > 2) v = max_raw(v, __shfl_xor(v, 32, 64));
      if (ks > 3) v = max_raw(v, dpp_f32<kXor2>(v));
      keys[((base >> 3) + 8 * k + (lane >> 3)) >> ks] = v;
    }
    const float mn = max_raw(g.m, wave_max(bmax)), lo = mn - 600.f;
    const double rn = -(double)mn * ek.c;
    if (mn > -INFINITY) {                                    // (before the first finite logit S is 0, and rn infinite)
      if (base > first) S = S * exp_rel(max_raw(g.m, lo), rn, tab, ek);
#pragma unroll
      for (int k = 0; k < kPartU; k++)
        if (base + 64 * k < n) S = exp_add(S, max_raw(g.x[k], lo), rn, tab, ek);     // (-inf adds less than 1e-260)
    }
    g.m = mn;
  }
  g.S = wave_sum(S);
}
// What a row leaves, from its (m, S), the logits of a short row and the best logits of a long one's keys; one wavefront.
__device__ __forceinline__ void gather_done(const SelCtx& c, const GatherPart& g, int row, float s_in, int start, int n, const float* keys) {
  const int lane = threadIdx.x & 63;
  if (!(g.m > -INFINITY)) {
    if (lane == 0) mark_dead(c, row);
    return;
  }
  const float lse = (float)((double)g.m + log(g.S));
  const float bias = __fsub_rn(s_in, lse);
  if (lane == 0) { c.row_bias[row] = bias; c.row_info[row] = ROW_SPARSE | (n << 2); c.row_start[row] = start; }
  float* data = c.row_data + (size_t)row * kRowFloats;
  float* group = c.row_group + (size_t)row * kGroups;
  if (n <= kScoreMax) {
#pragma unroll
    for (int k = 0; k < (kScoreMax + 63) / 64; k++) {
      if (64 * k < n) {
        const float score = (g.x[k] > -INFINITY) ? __fadd_rn(bias, g.x[k]) : -INFINITY;
        if (64 * k + lane < kScoreMax) data[64 * k + lane] = score;
        float best = quad_max(score);                        // of 16 children
        best = max_raw(best, dpp_f32<kHalfMirror>(best));
        best = max_raw(best, dpp_f32<kMirror>(best));
        if ((lane & 15) == 0) group[4 * k + (lane >> 4)] = best;
      }
    }
  } else {
    const int nk = key_count(n), gs = group_shift(nk) - 2;
    const float best = __fadd_rn(bias, g.m);
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; j++) v[j] = 4 * lane + j < nk ? __fadd_rn(bias, keys[4 * lane + j]) : -INFINITY;
    uint2 packed;
    packed.x = key16(best, v[0]) | (key16(best, v[1]) << 16);
    packed.y = key16(best, v[2]) | (key16(best, v[3]) << 16);
    *(uint2*)(data + 2 * lane) = packed;
    float top = max_raw(max_raw(v[0], v[1]), max_raw(v[2], v[3]));       // of the keys of a group: this lane's, or of two or four lanes
    if (gs > 0) top = max_raw(top, dpp_f32<kXor1>(top));
    if (gs > 1) top = max_raw(top, dpp_f32<kXor2>(top));
    if ((lane & ((1 << gs) - 1)) == 0 && (lane >> gs) < kGroups) group[lane >> gs] = top;
  }
}

// Levels 1 and 2 with a mask.  Bound: cache lines drawn at random (32 x 256 beams, V = 8192, Zipf table, level 1: 165 MB of lines
// in 46 us; what a row's children share no line with is wasted).  Lists up to 8192 children are gathered too: streaming the
// long ones needs a second kind of workgroup, and whatever share was streamed (above 512, 1024 or 2048 children) the call
// took as long.  Level 2, where nearly every row has one or two children, takes 10 us (19 us when every row also had a
// workgroup for the case that it has to be streamed).  Lists as long as the row are where streaming was ahead: 16 x 256 rows of
// 8192 children take 47 us (39 us streamed), 16 x 8 of them 14 us (15 us).
//
// A row per wavefront, then the workgroup's long rows by all of its wavefronts.
constexpr int kGatherWaves = 4;
constexpr int kDeal = 64;
__global__ void __launch_bounds__(kGatherWaves * 64, 8) k_rows_listed(SelCtx c) {
  __shared__ double s_tab[kExpTab], s_S[2][kGatherWaves];
  __shared__ float s_in4[kGatherWaves], s_m[2][kGatherWaves];
  __shared__ float s_own[kGatherWaves][kLines], s_keys[2][kLines];       // best logits of the keys of a wavefront's own row, of a workgroup's
  __shared__ int s_start[kGatherWaves], s_n[kGatherWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Long rows are neighbours, as a rule: of every 256 rows a workgroup takes four that are 64 apart.  (16 requests of 256 beams whose first
  // 64 have 8192 children: 41 us an item step, 65 with rows 16 apart.  Not further: rows from the four quarters of a batch of 49 MB of
  // logits took 16.7 us where these take 13.5.)
  auto row_of = [&](int w) { return (int)(blockIdx.x / kDeal * kDeal * kGatherWaves + blockIdx.x % kDeal) + kDeal * w; };
  const MaskView mv = mask_view(c.blob, c.V, c.depth);
  float s_in = -INFINITY;
  int start = 0, n = 0;
  const int own_row = row_of(wave);
  fill_exp_tab(s_tab, kGatherWaves * 64);
  if (own_row < c.B * c.W) {
    s_in = c.scores_in[own_row];
    row_children(c, mv, own_row, &start, &n);
    if (!(s_in > -INFINITY) || n == 0) {
      if (lane == 0) mark_dead(c, own_row);
      n = 0;
    }
  }
  if (lane == 0) { s_n[wave] = n; s_in4[wave] = s_in; s_start[wave] = start; }
  __syncthreads();
  const ExpK ek = exp_consts();
  const int32_t* list = child_list(c, mv);
  // where all rows are long, each wavefront keeps to its own all the same: it has as many parts to go through as with its share of all
  uint32_t joint = 0;                              // the rows that all wavefronts gather
#pragma unroll
  for (int w = 0; w < kGatherWaves; w++) joint |= (uint32_t)(s_n[w] > kWaveMax) << w;
  joint = __builtin_amdgcn_readfirstlane(joint);
  if (joint == (1u << kGatherWaves) - 1u) joint = 0;
  int set = 0;
  n = __builtin_amdgcn_readfirstlane(n);
  bool own = n > 0 && !((joint >> wave) & 1u);     // first this wavefront's own row, then those
#pragma unroll 1
  for (; own || joint; own = false) {
    const int w = own ? wave : __ffs(joint) - 1, nw = __builtin_amdgcn_readfirstlane(s_n[w]), sw = __builtin_amdgcn_readfirstlane(s_start[w]), row = row_of(w);
    if (!own) joint &= joint - 1;
    GatherPart g;
    float* keys = own ? s_own[wave] : s_keys[set];
    gather_part(g, c.logits + (size_t)row * c.V, list + sw, nw, own ? 0 : wave * kPart, own ? kPart : kGatherWaves * kPart, s_tab, ek, keys);
    if (!own) {
      if (lane == 0) { s_m[set][wave] = g.m; s_S[set][wave] = g.S; }
      __syncthreads();
      const int at = set;
      set ^= 1;
      if (wave != 0) continue;
      // (lane w joins wavefront w's pair; the sums meet in all lanes)
      const float mw = lane < kGatherWaves ? s_m[at][lane] : -INFINITY;
      g.m = wave_max(mw);
      if (g.m > -INFINITY)
        g.S = wave_sum((lane < kGatherWaves ? s_S[at][lane] : 0.0) * exp_rel(max_raw(mw, g.m - 600.f), -(double)g.m * ek.c, s_tab, ek));
    } else {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    gather_done(c, g, row, s_in4[w], sw, nw, keys);
  }
}

// All rows of request b, a row to a wavefront, for the workgroup that selects too; a row is too short to be shared out.
constexpr int kGatherRows = kSelThreads / 64, kGatherV = kPart;
__device__ __forceinline__ void gather_rows(const SelCtx& c, const MaskView& mv, int b, char* lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), row = b * c.W + wave;       // (what row `wave` of the request leaves goes to places of that number)
  double* tab = (double*)lds;
  float* keys = (float*)(tab + kExpTab) + wave * kLines;
  float s_in = -INFINITY;
  int start = 0, n = 0;
  if (wave < c.W) {
    s_in = c.scores_in[row];
    row_children(c, mv, row, &start, &n);
  }
  fill_exp_tab(tab, kSelThreads);
  __syncthreads();
  if (wave >= c.W) return;
  n = __builtin_amdgcn_readfirstlane(n);
  start = __builtin_amdgcn_readfirstlane(start);
  if (!(s_in > -INFINITY) || n == 0) {
    if ((threadIdx.x & 63) == 0) mark_dead(c, wave);
    return;
  }
  GatherPart g;
  const ExpK ek = exp_consts();
  gather_part(g, c.logits + (size_t)row * c.V, child_list(c, mv) + start, n, 0, kPart, tab, ek, keys);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  gather_done(c, g, wave, s_in, start, n, keys);
}

// Rows that are streamed, dealt to workgroups
//   one each: for calls whose rows are all streamed and, as a rule, all live;
//   every gridDim-th (STRIDE): for level 0, where as a rule one row of a request is live, its first: these rows are dealt first, then a
//   workgroup asks for the scores of all its other rows at once and turns to the live ones (8192 workgroups that only find a dead row
//   cost 16 us to dispatch; the live rows of 8 requests spread over 1021 workgroups 3 us more than at the front of 512, which is
//   two to a CU).  With so few rows at work a row is dealt to twice as many threads.
//   PICK: first rows may select as well.  They have a loop of their own: what the selection keeps in registers slows other rows down.  us where
//   all rows are live, here and in the kernel without PICK: 32 x 256 beams over 8192 tokens 72.0, 73.0; 8 x 128 21.7, 21.3; 64 x 128 over 1000
//   59.6, 58.8; 185 x 485 over 500 512, 507 (short rows that are many lose by the code beside them).
constexpr size_t kStrideGrid = 512;
template <bool STRIDE, int NT, bool PICK>
__global__ void __launch_bounds__(NT, STRIDE ? 4 : 6) k_rows(SelCtx c) {
  static_assert(STRIDE || !PICK, "requests are selected from at level 0 only");
  __shared__ RowLds<NT> L;
  __shared__ std::conditional_t<PICK, PickLds, char> P;
  const int tid = threadIdx.x, lane = tid & 63, rows = c.B * c.W;
  MaskView mv;
  mv.ok = false;
  if constexpr (!STRIDE) {
    const int row = blockIdx.x;
    const float s_in = c.scores_in[row];
    const int t1 = (c.blob && c.step == 1) ? c.prefix_in[(size_t)row * c.depth] : -1;
    if (c.blob) mv = mask_view(c.blob, c.V, c.depth);
    if (!(s_in > -INFINITY)) {
      if (tid == 0) mark_dead(c, row);
      return;
    }
    fill_exp_tab(L.tab, NT);
    int start = 0, n = 0;
    if (c.blob && c.step == 2) row_children(c, mv, row, &start, &n);
    __syncthreads();
    row_dense<NT>(c, mv, L, row, s_in, t1, start, n, 0);
  } else {
    c.step = 0;                                              // (no other level comes here: what those need of row_dense is left out)
    if (c.blob) mv = mask_view(c.blob, c.V, c.depth);
    bool filled = false;
    if constexpr (PICK) {
#pragma unroll 1
      for (int b = blockIdx.x; b < c.B; b += gridDim.x) {
        if (filled) __syncthreads();                         // (everybody is done with what the row before left in LDS)
        row_first<NT>(c, mv, L, P, b * c.W);
        filled = true;
      }
    }
    if (!filled) fill_exp_tab(L.tab, NT);
    __syncthreads();
    // the requests' first rows come first, then all others
    auto row_at = [&](int64_t at) {
      if (at < c.B) return (int)at * c.W;
      const int left = (int)at - c.B, b = left / (c.W - 1);
      return b * c.W + 1 + (left - b * (c.W - 1));
    };
    int set = 0;
    for (int64_t base = blockIdx.x; base < rows; base += (int64_t)gridDim.x * 64) {
      const int64_t at = base + (int64_t)lane * gridDim.x;
      const bool mine = at < rows && !(PICK && at < c.B);
      const int r = mine ? row_at(at) : 0;
      const float s = mine ? c.scores_in[r] : -INFINITY;
      if (tid < 64 && mine && !(s > -INFINITY)) mark_dead(c, r);
      uint64_t live = __ballot(s > -INFINITY);
      for (; live; live &= live - 1) {
        const int l = __ffsll((unsigned long long)live) - 1, row = __builtin_amdgcn_readlane(r, l);
        row_dense<NT>(c, mv, L, row, lane_f32(s, l), -1, 0, 0, set);
        set ^= 1;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------------
// Per-request selection.
// ------------------------------------------------------------------------------------------------
// A candidate's place in its row: the token in a streamed row, the position in the child list in a gathered one (the list is
// sorted, so both order the candidates of a row as its tokens do).
//
// Visit every finite candidate of request b.  f(score, w * V + place, pred) is called wave-convergently
// (pred = this lane holds a candidate); left0 = the place of what the request's first row left.  Rows given by bit masks are strided by the whole
// workgroup; rows given by child lists are taken one per wavefront.
template <bool LISTED, class F>
__device__ __forceinline__ void for_each_candidate(const SelCtx& c, const MaskView& mv, int b, size_t left0, F&& f) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  if (!LISTED && (!c.blob || c.step == 0)) {
    for (int w = 0; w < c.W; w++) {
      const int row = b * c.W + w;
      if (c.row_info[left0 + w] == ROW_DEAD) continue;
      const float bias = c.row_bias[left0 + w];
      const float* x = c.logits + (size_t)row * c.V;
      const uint32_t flat0 = (uint32_t)w * (uint32_t)c.V;
      for (int v0 = 0; v0 < c.V; v0 += blockDim.x) {
        const int v = v0 + threadIdx.x;
        const bool valid = v < c.V && (!c.blob || ((mv.l0[v >> 5] >> (v & 31)) & 1u));
        const float score = valid ? __fadd_rn(bias, x[v]) : -INFINITY;
        f(score, flat0 + v, score > -INFINITY);
      }
    }
  } else {
    for (int w = wave; w < c.W; w += nw) {
      const int row = b * c.W + w;
      if (c.row_info[left0 + w] == ROW_DEAD) continue;
      const float bias = c.row_bias[left0 + w];
      const float* x = c.logits + (size_t)row * c.V;
      const uint32_t flat0 = (uint32_t)w * (uint32_t)c.V;
      int start, n;
      row_children(c, mv, row, &start, &n);
      const int32_t* list = child_list(c, mv) + start;
      for (int i0 = 0; i0 < n; i0 += 64) {
        const int i = i0 + lane;
        const int v = i < n ? list[i] : 0;
        const float score = i < n ? __fadd_rn(bias, x[v]) : -INFINITY;
        f(score, flat0 + (LISTED ? i : v), score > -INFINITY);
      }
    }
  }
}

// Exact MSB radix select of the W best composite keys over ALL candidates (slow, always correct).
// Leaves the survivors in s_list and returns their number.
template <bool LISTED>
__device__ int radix_select_all(const SelCtx& c, const MaskView& mv, int b, size_t left0, uint64_t* s_list, uint32_t* s_hist) {
  __shared__ uint64_t s_prefix;
  __shared__ uint32_t s_need, s_bin, s_cnt;
  __shared__ int s_all;
  const int tid = threadIdx.x, lane = tid & 63;
  uint64_t prefix = 0;       // digits chosen so far (the top 64-shift bits of the W-th largest key)
  uint32_t need = (uint32_t)c.W;
  int shift = 64;            // number of key bits not yet fixed
  bool take_all = false;
  for (int pass = 0; pass < 6; pass++) {
    const int width = (pass < 5) ? 11 : 9;
    const int lo_shift = shift - width;
    const int nbins = 1 << width;
    for (int i = tid; i < nbins; i += kSelThreads) s_hist[i] = 0;
    __syncthreads();
    for_each_candidate<LISTED>(c, mv, b, left0, [&](float score, uint32_t flat, bool pred) {
      const uint64_t k = composite(score, flat);
      const bool in = pred && (pass == 0 || (k >> shift) == prefix);
      const uint32_t dgt = (uint32_t)(k >> lo_shift) & (uint32_t)(nbins - 1);
      // most lanes of a wave usually fall in the same bin on the leading digits: add them as one
      const uint64_t act = __ballot(in);
      if (act) {
        const int leader = __ffsll((unsigned long long)act) - 1;
        const uint32_t d0 = __shfl(dgt, leader, 64);
        const uint64_t same = __ballot(in && dgt == d0);
        if (lane == leader) atomicAdd(&s_hist[d0], (uint32_t)__popcll(same));
        if (in && dgt != d0) atomicAdd(&s_hist[dgt], 1u);
      }
    });
    __syncthreads();
    if (tid < 64) {
      // wave 0: find the bin that holds the need-th largest key
      const int per = nbins / 64;
      uint32_t local = 0;
      for (int i = 0; i < per; i++) local += s_hist[lane * per + i];
      uint32_t incl = local;   // inclusive suffix sum over lanes (higher lane = larger keys)
      for (int o = 1; o < 64; o <<= 1) {
        uint32_t v = __shfl_down(incl, o, 64);
        if (lane + o < 64) incl += v;
      }
      const uint32_t total = __shfl(incl, 0, 64);
      const uint32_t above = incl - local;
      if (total < need) {
        if (lane == 0) s_all = 1;           // fewer candidates than slots: keep them all
      } else if (above < need && need <= incl) {
        uint32_t acc = above;
        int bin = lane * per + per - 1;
        for (;; bin--) {
          const uint32_t h = s_hist[bin];
          if (acc + h >= need) break;
          acc += h;
        }
        s_prefix = (prefix << width) | (uint64_t)bin;
        s_need = need - acc;
        s_bin = s_hist[bin];
        s_all = 0;
      }
    }
    __syncthreads();
    if (s_all) { take_all = true; break; }
    prefix = s_prefix;
    need = s_need;
    shift = lo_shift;
    // everything above the bin (W - need keys) plus the bin itself fits in LDS: stop refining
    if ((uint32_t)c.W - need + s_bin <= (uint32_t)kListCap) break;
  }
  if (tid == 0) s_cnt = 0;
  __syncthreads();
  for_each_candidate<LISTED>(c, mv, b, left0, [&](float score, uint32_t flat, bool pred) {
    const uint64_t k = composite(score, flat);
    if (pred && (take_all || (k >> shift) >= prefix)) {
      const uint32_t idx = atomicAdd(&s_cnt, 1u);
      if (idx < (uint32_t)kListCap) s_list[idx] = k;
    }
  });
  __syncthreads();
  return min((int)s_cnt, kListCap);
}

// Bound: latency - a chain of some six memory round trips and a dozen barriers in one workgroup per request - and, with cold
// caches, the 40 GB/s at which one CU draws lines.  32 requests x 256 beams, V = 8192: 17 / 9 us at levels 1 / 2 (34 and 27 us when all
// 64 K chunk keys of a request were read and re-read chunks lay across eight lines); 4 us at level 0, where k_rows has selected as a rule.
// Code size is part of it: unrolled over registers this kernel was 81 KB and took up
// to twice as long, because each instruction line is fetched once per launch and used once; hence the rolled loops.
// LISTED: the call's rows are gathered ones (k_rows_listed), else streamed ones (k_rows); each is half of the code.
// GATHER: the workgroup gathers its request's rows itself, a wavefront a row, and no kernel runs in front of this one.
template <bool LISTED, bool GATHER>
__global__ void __launch_bounds__(kSelThreads) k_select(SelCtx c) {
  static_assert(LISTED || !GATHER, "streamed rows have kernels of their own");
  extern __shared__ __attribute__((aligned(16))) char smem[];
  uint64_t* s_list = (uint64_t*)smem;
  float* s_group = (float*)smem;                             // (before the list) best score of every group, or of every unit
  uint32_t* s_units = (uint32_t*)(s_list + kListCap);        // units that hold a candidate above the threshold: place in s_chunks << 8 | unit of the key
  uint64_t* s_tmp = (uint64_t*)s_units;                      // (after them) the survivors by bin
  constexpr int kTmpCap = kUnitCap / 2;
  uint32_t* s_hist = s_units + kUnitCap;
  uint32_t* s_chunks = s_hist + kHistBins;                   // row << 8 | key above the threshold, from the front; row << 8 | four scores, from the back
  float* s_rbias = (float*)(s_chunks + kChunkCap);           // per beam row of the request: bias,
  constexpr int kRows = GATHER ? kGatherRows : kMaxW;
  int32_t* s_rinfo = (int32_t*)(s_rbias + kRows);            // mode and child count,
  int32_t* s_ra = s_rinfo + kRows;                           // first child (gathered), first token (streamed, level 1) or table range start,
  float* s_rbest = (float*)(s_ra + kRows);                   // best score
  constexpr int NW = kSelThreads / 64;
  __shared__ float2 s_redf[2 * NW];
  __shared__ uint32_t s_redu[2 * NW], s_quads[NW];
  __shared__ uint32_t s_n, s_ng, s_nd, s_ns, s_nu, s_most;
  __shared__ int s_thr;
  int parf = 0, paru = 0;
  const int b = blockIdx.x, tid = threadIdx.x;
  const bool maybe_done = !LISTED && c.step == 0;
  const int first_info = maybe_done ? c.row_info[(size_t)b * c.W] : 0;
  MaskView mv;
  if (c.blob) mv = mask_view(c.blob, c.V, c.depth);
  if constexpr (GATHER) {
    // what the rows leave stays in LDS, which takes the workspace's place
    __shared__ __attribute__((aligned(16))) float s_data[kGatherRows * kRowFloats], s_groups[kGatherRows * kGroups], s_bias[kGatherRows];
    __shared__ int32_t s_info[kGatherRows], s_first[kGatherRows];
    c.row_data = s_data; c.row_group = s_groups; c.row_bias = s_bias; c.row_info = s_info; c.row_start = s_first;
    gather_rows(c, mv, b, smem);
    __syncthreads();                                         // (publishes the rows, and gives the rest of the LDS back)
  }

  // ---- the groups' best scores that k_rows left (two by two for more than 1024 beams)
  const size_t left0 = GATHER ? 0 : (size_t)b * c.W;         // where what they left of the request's first row lies
  const float* data = c.row_data + left0 * kRowFloats;
  const float4* group4 = (const float4*)(c.row_group + left0 * kGroups);
  const int32_t* info_b = c.row_info + left0;
  const int gsh = c.W * kGroups <= kGroupCap ? 4 : 3;        // log2 of the groups per row
  const int ngroups = c.W << gsh;
  float hi = -INFINITY, lo = INFINITY;                       // best and worst group
  // what k_rows left of a row beside them; asked for together with the groups (by themselves they are a round trip of their own, 0.5 us)
  struct Row { int info, a; float bias; };
  auto row_of = [&](int w) {
    const size_t row = (size_t)b * c.W + w;
    Row r;
    r.info = c.row_info[left0 + w]; r.bias = c.row_bias[left0 + w];
    r.a = 0;
    if (LISTED) r.a = c.row_start[left0 + w];
    else if (c.blob && c.step == 1) r.a = c.prefix_in[row * c.depth];
    else if (c.blob && c.step == 2) r.a = c.range_in[2 * row];
    return r;
  };
  auto keep_row = [&](int w, const Row& r) {
    s_rbias[w] = r.bias;
    s_rinfo[w] = r.info;
    s_ra[w] = r.a;
  };
  Row own = {ROW_DEAD, 0, 0.f};
  if (tid < c.W) own = row_of(tid);
#pragma unroll 2
  for (int q = tid; q < c.W * (kGroups / 4); q += kSelThreads) {
    const int w = q / (kGroups / 4), first = 4 * (q % (kGroups / 4)), info = info_b[w];
    float4 g = group4[q];
    const int ng = (info & 3) == ROW_DEAD ? 0 : LISTED && (info >> 2) <= kScoreMax ? ((info >> 2) + 15) >> 4 : kGroups;
    if (first >= ng) g.x = -INFINITY;
    if (first + 1 >= ng) g.y = -INFINITY;
    if (first + 2 >= ng) g.z = -INFINITY;
    if (first + 3 >= ng) g.w = -INFINITY;
    if (gsh == 4) *(float4*)&s_group[4 * q] = g;
    else *(float2*)&s_group[2 * q] = make_float2(fmaxf(g.x, g.y), fmaxf(g.z, g.w));
    const float best = quad_max(fmaxf(fmaxf(g.x, g.y), fmaxf(g.z, g.w)));      // (a row's groups are in four neighbouring lanes)
    if (first == 0) s_rbest[w] = best;
    hi = fmaxf(hi, best);
    auto low = [&](float v) { lo = fminf(lo, v > -INFINITY ? v : INFINITY); };
    low(g.x); low(g.y); low(g.z); low(g.w);
  }
  if (maybe_done && first_info == ROW_DONE) return;          // (asked for first, looked at here: nobody waits for it alone)
  // ---- the request's rows
  if (tid < c.W) keep_row(tid, own);
#pragma unroll 1
  for (int w = tid + kSelThreads; w < c.W; w += kSelThreads) keep_row(w, row_of(w));
  // quads of scores that they left, kNotShort for a row that is not a short one; and a bit for a dead row
  constexpr uint32_t kNotShort = 1u << 16, kSomeDead = 1u << 27;       // (1024 rows of at most 60 quads stay below the one, all of the one below the other)
  uint32_t own_quads = 0, quads_incl = 0;
  if (LISTED) {
    own_quads = (own.info & 3) == ROW_DEAD ? 0u : (own.info >> 2) <= kScoreMax ? (uint32_t)((own.info >> 2) + 3) >> 2 : kNotShort;
    quads_incl = wave_incl_scan(own_quads);
    const bool some_dead = __any((own.info & 3) == ROW_DEAD && tid < c.W);
    if (gr_lane() == 63) s_quads[tid >> 6] = quads_incl | (some_dead ? kSomeDead : 0u);
  }
  if (tid == 0) { s_n = 0; s_ng = 0; s_nd = 0; s_ns = 0; s_nu = 0; s_most = 0; }
  for (int i = tid; i < kHistBins; i += kSelThreads) s_hist[i] = 0;
  block_max_min<NW>(hi, lo, s_redf, parf);                   // (its barrier publishes the row table and the groups)

  int n = 0;
  bool few = false;
  if (hi > -INFINITY) {
    // Few scores of short gathered rows (the last level, as a rule): all of them are candidates, and the worst of the groups, which as many as
    // there are rows reach, is the threshold.  (Up to kDirectQuads: scores as good as equal are ranked one by one further down.  The
    // last level of 8 x 128 beams 9.7 -> 6.6 us, of one request x 16 beams 8.1 -> 5.3.)
    uint32_t per_wave = 0, sum = 0;
    if (LISTED) {
      per_wave = wave_incl_scan(gr_lane() < NW ? s_quads[gr_lane() & (NW - 1)] : 0u);
      sum = (uint32_t)__builtin_amdgcn_readlane((int)per_wave, 63);
    }
    const uint32_t quads = sum & (kSomeDead - 1u);
    const bool short_rows = LISTED && c.W <= kSelThreads && quads < kNotShort, direct = short_rows && quads <= (uint32_t)kDirectQuads;
    Bins bins = make_bins(hi, hi - lo);
    float T, scale;                                          // threshold; bins of one width down to it
    auto scale_to = [&](float t) { return t > kNoThreshold ? (hi > t ? fminf((float)(kHistBins - 1) / (hi - t), 1e30f) : 0.f) : 64.f; };
    bool fallback = false;
    int quarters = 0;
    const int ssh = 6 - gsh;                                 // log2 of the threads to a listed group
    uint32_t most = 0;
    // (an atomic per thread whose row is longer than those before it, not per key: lanes with values of their own go one by one)
    auto note_most = [&]() { if (most > 0 && most > *(volatile uint32_t*)&s_most) atomicMax(&s_most, most); };
    auto add = [&](bool front, int w, int key) {
      const uint32_t pos = atomicAdd(front ? &s_nd : &s_ns, 1u);
      if (pos < (uint32_t)kChunkCap) s_chunks[front ? pos : kChunkCap - 1 - pos] = ((uint32_t)w << 8) | (uint32_t)key;
    };
    auto take = [&](int w, int q, const float4& f) {         // the candidates of a short gathered row's quad
      const float v[4] = {f.x, f.y, f.z, f.w};
      const int left = (s_rinfo[w] >> 2) - 4 * q;            // (past the row's last wavefront of children nothing was written)
      // (places for the wavefront's candidates of all four at once: an atomic is waited for some 0.1 us)
      uint64_t in[4];
      uint32_t total = 0;
#pragma unroll
      for (int j = 0; j < 4; j++) { in[j] = __ballot(j < left && v[j] >= T); total += (uint32_t)__popcll(in[j]); }
      if (total == 0) return;
      const uint64_t here = __ballot(1);
      const int first = __ffsll((unsigned long long)here) - 1;
      uint32_t at = 0;
      if (gr_lane() == first) at = atomicAdd(&s_n, total);
      at = (uint32_t)__builtin_amdgcn_readlane((int)at, first);
#pragma unroll
      for (int j = 0; j < 4; j++) {
        if (j < left && v[j] >= T) {
          atomicAdd(&s_hist[key_bin(hi, scale, v[j])], 1u);
          const uint32_t pos = at + rank_below(in[j]);
          if (pos < (uint32_t)kListCap) s_list[pos] = composite(v[j], (uint32_t)w * (uint32_t)c.V + (uint32_t)(4 * q + j));
        }
        at += (uint32_t)__popcll(in[j]);
      }
    };
    auto quarter = [&](int i) { return ((int)s_units[i >> ssh] << ssh) + (i & ((1 << ssh) - 1)); };      // row << 6 | quarter of the row's 16 groups
    // the keys of a quarter group of a streamed or long gathered row: the first one's number, and how many
    auto quarter_keys = [&](const float* fine, int q, int info, int* key, int* num) {
      const int gs = !LISTED ? 4 : group_shift(key_count(info >> 2));
      *num = 1 << (gs - 2);
      *key = ((q >> 2) << gs) + ((q & 3) << (gs - 2));
      const uint2 k = *(const uint2*)(fine + 2 * (*key >> 2));
      return ((uint64_t)k.y << 32 | k.x) >> (16 * (*key & 3));
    };
    auto last_key = [&](int w) { return s_rbest[w] < T ? -1 : (int)key16(s_rbest[w], T); };
    if (direct) {
      const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
      const uint32_t quad0 = (wave ? (uint32_t)__builtin_amdgcn_readlane((int)per_wave, wave - 1) & (kSomeDead - 1u) : 0u) + quads_incl - own_quads;
      for (uint32_t k = 0; k < own_quads; k++) s_chunks[kChunkCap - 1 - (quad0 + k)] = ((uint32_t)tid << 8) | k;
      T = sum < kSomeDead ? lo : kNoThreshold;
      scale = scale_to(T);
      if (tid == 0) s_ns = quads;
      __syncthreads();                                       // (the list takes the groups' place)
      for (uint32_t i = tid; i < quads; i += kSelThreads) {
        const uint32_t ent = s_chunks[kChunkCap - 1 - i];
        const int w = (int)(ent >> 8), q = (int)(ent & 255u);
        take(w, q, *(const float4*)(data + (size_t)w * kRowFloats + 4 * q));
      }
    } else {
    // ---- threshold that at least W groups reach (no threshold when there are fewer)
#pragma unroll 1
    for (int i = tid; i < ngroups; i += kSelThreads)
      if (s_group[i] > -INFINITY) atomicAdd(&s_hist[bins.of(s_group[i])], 1u);
    __syncthreads();
    hist_threshold_all<kSelThreads>(s_hist, (uint32_t)c.W, &s_thr, s_redu, paru);
    __syncthreads();
    T = bins.floor_of(s_thr);
    scale = scale_to(T);
    // ---- groups that reach it
#pragma unroll 1
    for (int i = tid; i < ngroups; i += kSelThreads) {
      if (!(s_group[i] >= T)) continue;
      const uint32_t pos = atomicAdd(&s_ng, 1u);
      if (pos < (uint32_t)kUnitCap) s_units[pos] = (uint32_t)i;
    }
    __syncthreads();
    const int ng = (int)s_ng;
    fallback = ng > kUnitCap;
    quarters = min(ng, kUnitCap) << ssh;
    // ---- the finer keys behind them that reach it (four threads to a group, one round of loads for all).  Where all rows
    // left scores these are candidates at once, and nothing has to be read again: 15 thousand children of 128 beams 10.4 -> 8.7 us.
#pragma unroll 1
    for (int i = tid; i < quarters; i += kSelThreads) {
      const int at = quarter(i), w = at >> 6, q = at & 63, info = s_rinfo[w], cnt = info >> 2;
      const float* fine = data + (size_t)w * kRowFloats;
      if constexpr (!LISTED) {
        const uint2 k = *(const uint2*)(fine + 2 * q);
        const int last = last_key(w);
        if ((int)(k.x & 0xffffu) <= last) add(true, w, 4 * q);
        if ((int)(k.x >> 16) <= last) add(true, w, 4 * q + 1);
        if ((int)(k.y & 0xffffu) <= last) add(true, w, 4 * q + 2);
        if ((int)(k.y >> 16) <= last) add(true, w, 4 * q + 3);
      } else if (cnt <= kScoreMax) {
        // (the scores of a row's last wavefront of children are -inf past its end; past that they are not written)
        if (4 * q < cnt) {
          const float4 k = *(const float4*)(fine + 4 * q);
          if (fmaxf(fmaxf(k.x, k.y), fmaxf(k.z, k.w)) >= T) {
            add(false, w, q);
            if (short_rows) take(w, q, k);
          }
        }
      } else {
        const int last = last_key(w);
        int key, num;
        uint64_t keys = quarter_keys(fine, q, info, &key, &num);
#pragma unroll 1
        for (; num > 0; num--, key++, keys >>= 16)
          if ((int)(keys & 0xffffu) <= last) { add(true, w, key); most = max(most, (uint32_t)cnt); }
      }
    }
    }
    note_most();
    __syncthreads();
    int nd = (int)s_nd, ns = (int)s_ns;
    n = (int)s_n;
    const bool taken = short_rows && !fallback && n <= kListCap && ns <= kChunkCap;    // the list is complete
    // Few candidates count those that are better, several threads to one: no bins (16 beams, V = 256 9.1 -> 7.6 us at level 1; one request of 128 beams,
    // V = 8192, at level 2 10.6 -> 9.7, 30 of 40 beams 11.3 -> 10.0).  The work grows with the square of their number: at 192 some
    // 0.8 us, as long as the bins.
    few = taken && n <= kFewMax;
    if (few) {
      const int sh = n <= 64 ? 4 : n <= 128 ? 3 : 2, i = tid >> sh;
      uint64_t own_key = 0;
      if (i < n) own_key = s_list[i];
      int better = 0;
      if (i < n) {
#pragma unroll 4
        for (int j = tid & ((1 << sh) - 1); j < n; j += 1 << sh) better += s_list[j] > own_key;
      }
      better = lanes_sum(better, sh);
      if (i < n && (tid & ((1 << sh) - 1)) == 0) s_tmp[better] = own_key;
      __syncthreads();
    } else {
    if (!taken) {
    if (__builtin_expect(n > 0, 0)) {
      __syncthreads();
      for (int i = tid; i < kHistBins; i += kSelThreads) s_hist[i] = 0;
      if (tid == 0) s_n = 0;
      __syncthreads();
    }
    // Where the W best are many to a group (few beams far ahead of the others, long rows) the groups' threshold is too low and the
    // keys' own takes its place, which W of them reach: they are counted, then listed again.  The line: 32 requests of 128 beams, 8192
    // tokens, logits of width 6 and then 1 have 11 keys a beam above the groups' threshold and take 37 us without a mask, 54 us when
    // all of them are looked at; gathered keys cost more lines of memory each.
    if (__builtin_expect(!fallback && (nd + ns > kChunkCap || nd > c.W + (s_most > 0 ? 256 : 512)), 0)) {
      bins = make_bins(hi, hi - T);
#pragma unroll 1
      for (int pass = 0; pass < 2; pass++) {
        most = 0;
#pragma unroll 1
        for (int i = tid; i < quarters; i += kSelThreads) {
          const int at = quarter(i), w = at >> 6, q = at & 63, info = s_rinfo[w], cnt = info >> 2;
          const float* fine = data + (size_t)w * kRowFloats;
          if (!LISTED || cnt > kScoreMax) {
            const int last = last_key(w);
            int key, num;
            uint64_t keys = quarter_keys(fine, q, info, &key, &num);
#pragma unroll 1
            for (; num > 0; num--, key++, keys >>= 16) {
              if ((int)(keys & 0xffffu) > last) continue;
              if (pass == 0) atomicAdd(&s_hist[bins.of(key16_low(s_rbest[w], (uint32_t)keys & 0xffffu))], 1u);
              else { add(true, w, key); most = max(most, (uint32_t)cnt); }
            }
          } else if (4 * q < cnt) {
            const float4 f = *(const float4*)(fine + 4 * q);
            const float k = fmaxf(fmaxf(f.x, f.y), fmaxf(f.z, f.w));
            if (k >= T && pass == 0) atomicAdd(&s_hist[bins.of(k)], 1u);
            if (k >= T && pass == 1) add(false, w, q);
          }
        }
        if (pass == 1) note_most();
        __syncthreads();
        if (pass == 1) break;
        if (tid == 0) { s_nd = 0; s_ns = 0; s_most = 0; }
        hist_threshold_all<kSelThreads>(s_hist, (uint32_t)c.W, &s_thr, s_redu, paru);
        __syncthreads();
        T = fmaxf(T, bins.floor_of(s_thr));
      }
      nd = (int)s_nd; ns = (int)s_ns;
    }
    }
    // units of four candidates behind a key in front: float4 of logits, or consecutive children
    const int sh = LISTED ? 1 + key_shift((int)s_most) : c.unit_shift;
    fallback = fallback || nd + ns > kChunkCap;
    const int front_units = nd << sh;
    const int lsh = c.row_threads == 512 ? 2 : 3;            // log2 of a thread's loads per block of a streamed row
    auto unit_token = [&](int k, int e) {                    // first token of unit e of line k
      return 32 * (k >> lsh) + 4 * c.row_threads * (k & ((1 << lsh) - 1)) + 4 * (e & 7) + kBlockV * (e >> 3);
    };
    if (!fallback && !taken) {
      // ---- units behind them that hold a candidate above the threshold (as far as the logits tell: validity comes next).  Four
      // scores are a unit as they are.
      auto entry = [&](int u, int* w, int* k, int* e) {
        const uint32_t ent = s_chunks[u >> sh];
        *w = (int)(ent >> 8); *k = (int)(ent & 255u); *e = u & ((1 << sh) - 1);
      };
      auto keep = [&](int u) {
        const uint32_t pos = atomicAdd(&s_nu, 1u);
        if (pos < (uint32_t)kUnitCap) s_units[pos] = ((uint32_t)(u >> sh) << 8) | (uint32_t)(u & ((1 << sh) - 1));
      };
      // best logit of a gathered row's unit
      auto child_best = [&](int w, int k, int e) {
        const int cnt = s_rinfo[w] >> 2, ks = key_shift(cnt), at = (k << (3 + ks)) + 4 * e;
        const float* x = c.logits + ((size_t)b * c.W + w) * c.V;
        const int32_t* list = child_list(c, mv) + s_ra[w];
        if (e >= 2 << ks || at >= cnt) return -INFINITY;     // (rows of fewer children have fewer units behind a key)
        const float y0 = x[list[at]], y1 = x[list[min(at + 1, cnt - 1)]], y2 = x[list[min(at + 2, cnt - 1)]], y3 = x[list[min(at + 3, cnt - 1)]];
        return fmaxf(fmaxf(y0, y1), fmaxf(y2, y3));          // (a child taken twice changes nothing here)
      };
      // best valid logit of a streamed row's unit
      auto token_best = [&](int w, int k, int e) {
        const int v = unit_token(k, e);
        if (v >= c.V) return -INFINITY;
        const float* x = c.logits + ((size_t)b * c.W + w) * c.V;
        uint32_t bits = 0xfu;
        if (c.blob) bits = (c.step == 0 ? mv.l0 : mv.l1 + (size_t)s_ra[w] * mv.words)[v >> 5] >> (v & 31);
        f32x4u y;
        if (v + 3 < c.V) y = *(const f32x4u*)(x + v);
        else { y.x = x[v]; y.y = x[min(v + 1, c.V - 1)]; y.z = x[min(v + 2, c.V - 1)]; y.w = y.z; }
        // (past the row's end a mask has no bits; without one the last token is taken again, which changes nothing here)
        return fmaxf(fmaxf(bits & 1u ? y.x : -INFINITY, bits & 2u ? y.y : -INFINITY), fmaxf(bits & 4u ? y.z : -INFINITY, bits & 8u ? y.w : -INFINITY));
      };
      auto listed_units = [&](auto&& f) {                    // f(unit, its best score) for every unit in front, four at a time
        constexpr int U = 4;
#pragma unroll 1
        for (int base = tid; base < front_units; base += U * kSelThreads) {
          float best[U];
#pragma unroll
          for (int q = 0; q < U; q++) {
            const int u = base + q * kSelThreads;
            best[q] = -INFINITY;
            if (u < front_units) {
              int w, k, e;
              entry(u, &w, &k, &e);
              best[q] = __fadd_rn(s_rbias[w], child_best(w, k, e));
            }
          }
#pragma unroll
          for (int q = 0; q < U; q++)
            if (base + q * kSelThreads < front_units) f(base + q * kSelThreads, best[q]);
        }
      };
      // Fewer groups than W, as at level 0 where all candidates are one row's: the units themselves yield a threshold.  (Not where a streamed
      // row's validity is only looked up below; the best candidates of the first kGroupCap units are kept, beyond that they are
      // looked for again.)
      const bool countable = LISTED || !(c.blob && c.step == 2);
      const bool by_unit = countable && T == kNoThreshold && front_units >= c.W, kept = by_unit && front_units <= kGroupCap;
      if (by_unit) {
        bins = make_bins(hi, hi - T);
        auto count = [&](int u, float best) {
          if (u < min(front_units, kGroupCap)) s_group[u] = best;
          if (best >= T) atomicAdd(&s_hist[bins.of(best)], 1u);
        };
        constexpr int U = 2;
#pragma unroll 1
        for (int base = tid; !LISTED && base < front_units; base += U * kSelThreads) {
          float best[U];
#pragma unroll
          for (int q = 0; q < U; q++) {
            const int u = base + q * kSelThreads;
            best[q] = -INFINITY;
            if (u >= front_units) continue;
            int w, k, e;
            entry(u, &w, &k, &e);
            best[q] = token_best(w, k, e);
            best[q] = __fadd_rn(s_rbias[w], best[q]);
          }
#pragma unroll
          for (int q = 0; q < U; q++) count(base + q * kSelThreads, best[q]);
        }
        if constexpr (LISTED) listed_units(count);
        __syncthreads();
        hist_threshold_all<kSelThreads>(s_hist, (uint32_t)c.W, &s_thr, s_redu, paru);
        __syncthreads();
        T = fmaxf(T, bins.floor_of(s_thr));
      }
      if (kept) {
#pragma unroll 1
        for (int u = tid; u < front_units; u += kSelThreads)
          if (s_group[u] >= T) keep(u);
      } else if constexpr (!LISTED) {
        constexpr int U = 4;
#pragma unroll 1
        for (int base = tid; base < front_units; base += U * kSelThreads) {
          float best[U], bias[U];
#pragma unroll
          for (int q = 0; q < U; q++) {
            const int u = base + q * kSelThreads;
            best[q] = -INFINITY; bias[q] = 0.f;
            if (u < front_units) {
              int w, k, e;
              entry(u, &w, &k, &e);
              const int v = unit_token(k, e);
              const float* x = c.logits + ((size_t)b * c.W + w) * c.V;
              if (v + 3 < c.V) { const f32x4u t = *(const f32x4u*)(x + v); best[q] = fmaxf(fmaxf(t.x, t.y), fmaxf(t.z, t.w)); }
              else if (v < c.V) best[q] = INFINITY;        // (the row's last tokens are looked at one by one below)
              bias[q] = s_rbias[w];
            }
          }
#pragma unroll
          for (int q = 0; q < U; q++)
            if (__fadd_rn(bias[q], best[q]) >= T) keep(base + q * kSelThreads);
        }
      } else {
        listed_units([&](int u, float best) { if (best >= T) keep(u); });
      }
      __syncthreads();
      // more units than there is room for: the same, over those that reach the threshold
      if (__builtin_expect(s_nu > (uint32_t)kUnitCap && countable && !by_unit, 0)) {
        bins = make_bins(hi, hi - T);
#pragma unroll 1
        for (int pass = 0; pass < 2; pass++) {               // count, keep
#pragma unroll 1
          for (int u = tid; u < front_units; u += kSelThreads) {
            int w, k, e;
            entry(u, &w, &k, &e);
            const float best = __fadd_rn(s_rbias[w], LISTED ? child_best(w, k, e) : token_best(w, k, e));
            if (!(best >= T)) continue;
            if (pass == 0) atomicAdd(&s_hist[bins.of(best)], 1u);
            else keep(u);
          }
          __syncthreads();
          if (pass == 1) break;
          if (tid == 0) s_nu = 0;
          hist_threshold_all<kSelThreads>(s_hist, (uint32_t)c.W, &s_thr, s_redu, paru);
          __syncthreads();
          T = fmaxf(T, bins.floor_of(s_thr));
        }
      }
      fallback = s_nu > (uint32_t)kUnitCap;
    }
    if (!fallback) {
      // ---- their candidates, counted in bins of one width from the best score down to the threshold.  When they do not fit, the
      // bins still tell where the W best end, and a second round takes only those.
      const int nu = (int)s_nu, units = nu + ns;
      scale = scale_to(T);
      int cut = kHistBins - 1;
#pragma unroll 1
      for (int round = 0; round < 2; round++) {
#pragma unroll 1
        for (int i = taken && round == 0 ? units : tid; i < units; i += kSelThreads) {
          const uint32_t unit = i < nu ? s_units[i] : 0u;
          const uint32_t ent = s_chunks[i < nu ? (int)(unit >> 8) : kChunkCap - 1 - (i - nu)];
          const int w = (int)(ent >> 8), k = (int)(ent & 255u), cnt = s_rinfo[w] >> 2;
          const float* xrow = c.logits + ((size_t)b * c.W + w) * c.V;
          int place, end = cnt;                            // the unit's candidates: place .. place + 3, < end
          float bias = s_rbias[w], y[4];
          uint32_t bits = 0xfu;
          if (!LISTED) {
            place = unit_token(k, (int)(unit & 255u));
            end = c.V;
            if (c.blob && c.step == 0) bits = mv.l0[place >> 5] >> (place & 31);
            else if (c.blob && c.step == 1) bits = mv.l1[(size_t)s_ra[w] * mv.words + (place >> 5)] >> (place & 31);
#pragma unroll
            for (int j = 0; j < 4; j++) y[j] = xrow[min(place + j, c.V - 1)];
          } else if (i >= nu) {
            place = 4 * k;
            bias = 0.f;                                    // (these scores are complete)
            const float4 t = *(const float4*)(data + (size_t)w * kRowFloats + place);
            y[0] = t.x; y[1] = t.y; y[2] = t.z; y[3] = t.w;
          } else {
            place = (k << (3 + key_shift(cnt))) + 4 * (int)(unit & 255u);
            const int32_t* list = child_list(c, mv) + s_ra[w];
            int tok[4];
#pragma unroll
            for (int j = 0; j < 4; j++) tok[j] = list[min(place + j, cnt - 1)];
#pragma unroll
            for (int j = 0; j < 4; j++) y[j] = xrow[tok[j]];
          }
#pragma unroll
          for (int j = 0; j < 4; j++) {
            const int at = place + j;
            const float score = __fadd_rn(bias, y[j]);     // (with bias 0 unchanged but for -0, which composite() makes 0)
            if (at >= end || !((bits >> j) & 1u) || !(score >= T)) continue;
            if (!LISTED && c.blob && c.step == 2) {        // last level, streamed row: the candidate has to be in the row's child list
              const int32_t* list = mv.t3 + s_ra[w];
              const int len = c.range_in[2 * ((size_t)b * c.W + w) + 1] - s_ra[w], pos = lower_bound_i32(list, len, at);
              if (!(pos < len && list[pos] == at)) continue;
            }
            const int bin = key_bin(hi, scale, score);
            if (bin > cut) continue;
            if (round == 0) atomicAdd(&s_hist[bin], 1u);
            const uint32_t pos = atomicAdd(&s_n, 1u);
            if (pos < (uint32_t)kListCap) s_list[pos] = composite(score, (uint32_t)w * (uint32_t)c.V + (uint32_t)at);
          }
        }
        __syncthreads();
        n = (int)s_n;
        if (round == 0) {
          if (__builtin_expect(T == kNoThreshold && n <= kListCap && s_hist[kHistBins - 1] > 64u, 0)) {
            // (no threshold, and many lie below the bins: down to the worst of them)
            float mx = -INFINITY, mn = INFINITY;
            for (int i = tid; i < n; i += kSelThreads) mn = fminf(mn, gr_ordkey_inv((uint32_t)(s_list[i] >> 32)));
            __syncthreads();
            for (int i = tid; i < kHistBins; i += kSelThreads) s_hist[i] = 0;
            block_max_min<NW>(mx, mn, s_redf, parf);         // (its barrier: the histogram is clear)
            scale = hi > mn ? fminf((float)(kHistBins - 1) / (hi - mn), 1e30f) : 0.f;
            for (int i = tid; i < n; i += kSelThreads) atomicAdd(&s_hist[key_bin(hi, scale, gr_ordkey_inv((uint32_t)(s_list[i] >> 32)))], 1u);
            __syncthreads();
          }
          hist_prefix<kSelThreads>(s_hist, (uint32_t)c.W, &s_thr, s_redu, paru);
          if (n > kListCap && tid == 0) s_n = 0;
          __syncthreads();
          cut = s_thr;
        }
        if (n <= kListCap) break;
      }
      fallback = n > kListCap;
      int m = 0;                                             // survivors up to the W-th one's bin
      if (!fallback) {
        m = cut < kHistBins - 1 ? (int)s_hist[cut + 1] : n;
        fallback = m > kTmpCap;
      }
      if (!fallback) {
        __syncthreads();                                     // (s_hist[cut + 1] is read before any counter moves)
        order_by_bins<kSelThreads>(s_list, s_tmp, s_hist, n, m, cut, hi, scale);
        n = m;
      }
    }
    if (__builtin_expect(fallback, 0)) {
      __syncthreads();
      n = radix_select_all<LISTED>(c, mv, b, left0, s_list, s_hist);
      int n2 = 1;
      while (n2 < n) n2 <<= 1;
      for (int i = n + tid; i < n2; i += kSelThreads) s_list[i] = 0;   // 0 sorts after every real key
      __syncthreads();
      for (int k = 2; k <= n2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
          for (int i = tid; i < n2; i += kSelThreads) {
            const int ixj = i ^ j;
            if (ixj > i) {
              const uint64_t a = s_list[i], bb = s_list[ixj];
              const bool desc = (i & k) == 0;
              if (desc ? (a < bb) : (a > bb)) { s_list[i] = bb; s_list[ixj] = a; }
            }
          }
          __syncthreads();
        }
      }
    }
    }
  }

  // ---- level 1: which pair a survivor of a streamed row is = the valid tokens before it in its mask row, counted by four
  // lanes in one round of loads (a binary search in the child list is a dozen dependent ones)
  int32_t* s_rank = (int32_t*)s_hist;                        // [W] (kHistBins >= kMaxW)
  if (!LISTED && c.blob && c.step == 1) {
    for (int j0 = 0; j0 < min(n, c.W); j0 += kSelThreads / 4) {
      const int j = j0 + (tid >> 2), g = tid & 3;
      uint32_t cnt = 0;
      if (j < min(n, c.W)) {
        const uint32_t flat = 0xffffffffu - (uint32_t)s_list[j];
        const int w = (int)(flat / (uint32_t)c.V), tok = (int)(flat % (uint32_t)c.V);
        {
          const uint32_t* mrow = mv.l1 + (size_t)s_ra[w] * mv.words;
          const int full = tok >> 5;                         // whole words before the token's
          if (g == 0) cnt = (uint32_t)mv.pair_off[s_ra[w]] + (uint32_t)__popc(mrow[full] & ((1u << (tok & 31)) - 1u));
#pragma unroll 1
          for (int i = 4 * g; i < full; i += 16) {           // (reads at most three words past the row: the blob goes on there)
            const u32x4u q = *(const u32x4u*)(mrow + i);
            cnt += (uint32_t)__popc(q.x) + (i + 1 < full ? (uint32_t)__popc(q.y) : 0u) + (i + 2 < full ? (uint32_t)__popc(q.z) : 0u) +
                   (i + 3 < full ? (uint32_t)__popc(q.w) : 0u);
          }
        }
      }
      cnt += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)cnt, kXor1, 0xf, 0xf, true);
      cnt += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)cnt, kXor2, 0xf, 0xf, true);
      if (g == 0 && j < c.W) s_rank[j] = (int32_t)cnt;
    }
    __syncthreads();
  }

  // ---- write the new beam state, best first.  (The arguments are read again here: held from the start on, the scalar registers they
  // take are spilled and reloaded all through the kernel.)
  const LateArgs late = late_args();
  const uint64_t* best = few ? s_tmp : s_list;
  for (int j = tid; j < late->W; j += kSelThreads) {
    const size_t o = (size_t)b * late->W + j;
    int32_t* po = late->prefix_out + o * late->depth;
    for (int k = 0; k < late->depth; k++) po[k] = -1;
    int r_lo = 0, r_hi = 0, item = -1;
    if (j < n) {
      const uint64_t key = best[j];
      const uint32_t flat = 0xffffffffu - (uint32_t)key;
      const int parent = (int)(flat / (uint32_t)late->V), place = (int)(flat % (uint32_t)late->V);
      constexpr bool gathered = LISTED;
      int token = place;
      if (late->blob) {
        if (late->step == 0) {
          r_lo = mv.off1[token]; r_hi = mv.off1[token + 1];
        } else if (late->step == 1) {
          const int p = gathered ? s_ra[parent] + place : s_rank[j];
          if (gathered) token = mv.pair_t2[p];
          r_lo = mv.pair_row[p]; r_hi = mv.pair_row[p + 1];
        } else {
          const int first = s_ra[parent];
          r_lo = first + (gathered ? place : lower_bound_i32(mv.t3 + first, late->range_in[2 * ((size_t)b * late->W + parent) + 1] - first, token));
          if (gathered) token = mv.t3[r_lo];
          r_hi = r_lo + 1;
          item = r_lo;
        }
      }
      late->parent_out[o] = parent;
      late->token_out[o] = token;
      late->scores_out[o] = gr_ordkey_inv((uint32_t)(key >> 32));
      const size_t prow = (size_t)b * late->W + parent;
      for (int k = 0; k < late->step; k++) po[k] = late->prefix_in[prow * late->depth + k];
      po[late->step] = token;
    } else {
      late->parent_out[o] = -1;
      late->token_out[o] = -1;
      late->scores_out[o] = -INFINITY;
    }
    late->range_out[2 * o] = r_lo;
    late->range_out[2 * o + 1] = r_hi;
    if (late->item_index_out) late->item_index_out[o] = item;
  }
}

}  // namespace

extern "C" size_t gr_beam_select_workspace_bytes(int32_t B, int32_t W, int32_t V, int32_t depth) {
  if (B <= 0 || W <= 0 || V <= 0 || depth <= 0) return 0;
  const size_t rows = (size_t)B * W;
  return 3 * gr_align256(rows * 4) + gr_align256(rows * (kGroups + kRowFloats) * 4);
}

extern "C" gr_status gr_beam_select(const gr_select_params* p, void* workspace, size_t workspace_bytes, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!p) return GR_ERR_INVALID_ARG;
  if (p->B <= 0 || p->W <= 0 || p->V <= 0 || p->depth <= 0 || p->step < 0 || p->step >= p->depth) return GR_ERR_INVALID_ARG;
  if (!p->logits || !p->scores_in || !p->parent_out || !p->token_out || !p->scores_out || !p->prefix_out || !p->range_out)
    return GR_ERR_INVALID_ARG;
  if (p->step > 0 && (!p->prefix_in || (p->mask && !p->range_in))) return GR_ERR_INVALID_ARG;
  if (p->prefix_in && p->prefix_in == p->prefix_out) return GR_ERR_INVALID_ARG;
  if (p->range_in && p->range_in == p->range_out) return GR_ERR_INVALID_ARG;
  if (p->depth != 3 || p->W > 2048 || p->V > 32768 || (int64_t)p->W * p->V >= ((int64_t)1 << 31)) return GR_ERR_UNSUPPORTED;
  if ((int64_t)p->B * p->W >= ((int64_t)1 << 31)) return GR_ERR_UNSUPPORTED;
  if (!workspace || ((uintptr_t)workspace & 255)) return GR_ERR_INVALID_ARG;
  if (workspace_bytes < gr_beam_select_workspace_bytes(p->B, p->W, p->V, p->depth)) return GR_ERR_WORKSPACE_TOO_SMALL;

  SelCtx c;
  c.B = p->B; c.W = p->W; c.V = p->V; c.depth = p->depth; c.step = p->step;
  c.unit_shift = 3;
  while ((kBlockV >> 3) << c.unit_shift < p->V) c.unit_shift++;
  c.blob = (const char*)p->mask;
  c.logits = p->logits; c.scores_in = p->scores_in; c.prefix_in = p->prefix_in; c.range_in = p->range_in;
  c.parent_out = p->parent_out; c.token_out = p->token_out; c.scores_out = p->scores_out;
  c.prefix_out = p->prefix_out; c.range_out = p->range_out; c.item_index_out = p->item_index_out;
  const size_t rows = (size_t)p->B * p->W;
  char* ws = (char*)workspace;
  c.row_bias = (float*)ws;                 ws += gr_align256(rows * 4);
  c.row_info = (int32_t*)ws;               ws += gr_align256(rows * 4);
  c.row_start = (int32_t*)ws;              ws += gr_align256(rows * 4);
  c.row_group = (float*)ws;                ws += rows * kGroups * 4;       // (whole 64 bytes a row: row_data stays 16-byte aligned)
  c.row_data = (float*)ws;

  c.row_threads = p->step == 0 ? 512 : 256;
  // A workgroup that reads scores and selects as well writes its request's outputs while others may still read theirs: not where an output
  // lies on the incoming scores (k_select, a launch behind all readers, writes it then).  Levels 1 and 2 read a request's scores in its own
  // workgroup only, so there the scores may be the ones that came in.
  auto on_scores = [&](const void* out, size_t per_row) {
    return out && (uintptr_t)out < (uintptr_t)(p->scores_in + rows) && (uintptr_t)p->scores_in < (uintptr_t)out + rows * per_row * 4;
  };
  const bool others_on = on_scores(p->parent_out, 1) || on_scores(p->token_out, 1) || on_scores(p->prefix_out, (size_t)p->depth) || on_scores(p->range_out, 2) ||
                         on_scores(p->item_index_out, 1);
  const bool scores_on = on_scores(p->scores_out, 1);
  const bool pick = p->step == 0 && p->V <= kBlockV && p->W <= kPickW && !others_on && !scores_on;
  const bool listed = p->mask && p->step >= 1 && !(p->flags & GR_SELECT_FORCE_DENSE);
  // One kernel instead of two where every wavefront of the selecting workgroup has at most one row, and that row one round of loads (longer ones
  // are drawn faster by more CUs).  us of a level with two kernels and with one: one request x 16 beams, V = 256, 8 children a row 10.3, 9.4, 250 children 13.7,
  // 13.0; V = 512, 500 children 14.1, 13.5; 256 x 16 12.9, 9.7 and 17.8, 14.6; 300 x 4 16.6, 15.6; 8 x 4 10.5, 8.5.  But two rows a wavefront
  // (32 beams) 10.5, 12.0, and two rounds (1000 children of V = 1024, 16 beams) 15.4, 15.9.
  const bool gather = listed && p->W <= kGatherRows && p->V <= kGatherV && !others_on && (!scores_on || p->scores_out == p->scores_in);
  if (listed && !gather)
    hipLaunchKernelGGL(k_rows_listed, dim3((unsigned)((rows + kDeal * kGatherWaves - 1) / (kDeal * kGatherWaves) * kDeal)), dim3(kGatherWaves * 64), 0, stream, c);
  else if (pick)
    hipLaunchKernelGGL((k_rows<true, 512, true>), dim3((unsigned)(rows < kStrideGrid ? rows : kStrideGrid)), dim3(512), 0, stream, c);
  else if (p->step == 0)
    hipLaunchKernelGGL((k_rows<true, 512, false>), dim3((unsigned)(rows < kStrideGrid ? rows : kStrideGrid)), dim3(512), 0, stream, c);
  else if (!listed)
    hipLaunchKernelGGL((k_rows<false, 256, false>), dim3((unsigned)rows), dim3(256), 0, stream, c);
  const size_t lds = kSelLdsBytes - (gather ? (size_t)(kMaxW - kGatherRows) * 16 : 0);      // (the row tables are that much shorter)
#define GR_LAUNCH_SELECT(...)                                                                                         \
  do {                                                                                                                \
    if (const gr_status st = gr_allow_lds<k_select<__VA_ARGS__>>(lds)) return st;                                     \
    hipLaunchKernelGGL((k_select<__VA_ARGS__>), dim3(p->B), dim3(kSelThreads), lds, stream, c);                       \
  } while (0)
  if (gather) GR_LAUNCH_SELECT(true, true);
  else if (listed) GR_LAUNCH_SELECT(true, false);
  else GR_LAUNCH_SELECT(false, false);
#undef GR_LAUNCH_SELECT
  GR_HIP_TRY(hipGetLastError());
  return GR_OK;
}

// ------------------------------------------------------------------------------------------------
// gr_beam_select_noalloc: the same item step for callers that cannot allocate or hand in a workspace.
// The kernels' scratch memory (row bias / mode / first child, group maxima and keys) lives in a static device
// array; every GPU the library runs on holds its own copy at its own address, obtained once per device.
// ------------------------------------------------------------------------------------------------
namespace {
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
constexpr int kMaxDevices = 64;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
void* g_scratch_ptr[kMaxDevices];          // device address of `scratch` per device (0 = not looked up yet)
}  // namespace

extern "C" size_t gr_beam_select_noalloc_max_workspace_bytes(void) { return kStaticScratchBytes; }

extern "C" gr_status gr_beam_select_noalloc(const gr_select_params* p, void* stream_) {
  if (!p) return GR_ERR_INVALID_ARG;
  if (p->B <= 0 || p->W <= 0 || p->V <= 0 || p->depth <= 0) return GR_ERR_INVALID_ARG;
  if (gr_beam_select_workspace_bytes(p->B, p->W, p->V, p->depth) > kStaticScratchBytes) return GR_ERR_WORKSPACE_TOO_SMALL;
  int dev = -1;
  GR_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return GR_ERR_UNSUPPORTED;
  if (!g_scratch_ptr[dev]) {
    // (the array's name is only a host-side handle: its device address on the current device is asked for once)
    void* ptr = nullptr;
    GR_HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return GR_ERR_HIP;
    g_scratch_ptr[dev] = ptr;
  }
  // nothing in the workspace has to start at zero: a row's mode is always written by the call that reads it, and what else a call reads
  // of a row is used only where the mode says that it was written (a dead row's bias, start and groups are not)
  return gr_beam_select(p, g_scratch_ptr[dev], kStaticScratchBytes, stream_);
}

