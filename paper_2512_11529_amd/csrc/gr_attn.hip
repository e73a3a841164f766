// gr_beam_attn: shared-prefix beam attention on gfx950 (paper Sections 5.1, 5.2).
//
// Work unit = (request b, KV head h, block of query rows, L segment).  The W*g query rows that share
// KV head h of request b (g = Hq/Hkv) form the N side of a transposed score matrix
//     S^T[kv, q] = K[kv, :] . Q[q, :]          (v_mfma_f32_32x32x16_bf16, A = K tile from LDS, B = Q in registers)
// so that every lane owns ONE query column: the online-softmax max / sum / rescale are per-lane
// scalars and the exponentiated scores leave the accumulators already in the B-operand layout of
//     O^T[d, q] += V^T[d, kv] . P^T[kv, q]     (A = V tile read from LDS with the transposing ds_read_b64_tr_b16).
// Each prompt K/V tile is brought in once per workgroup (direct global -> LDS loads into unpadded, XOR-swizzled
// tiles) and used by all query rows of the block.  The unshared stage (each beam's own u decode tokens) and the merge
// run in the epilogue of one segment on the same per-lane state; when the prompt is split into
// segments, partial (max, sum, O) go to the workspace and k_attn_merge combines them.
#include <type_traits>
#include "gr_internal.hpp"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int KT = 64;        // kv tokens per LDS tile

// Dynamic LDS of k_beam_attn: K and V tiles, double-buffered; the Q hand-over, behind the tiles for workgroups of 8 wavefronts and in the V
// tiles' place for those of 4.  After the prompt loop a wavefront's 32 own-token rows take the K tiles' place (of K; Q's where 8 wavefronts hold
// 256 rows) and the V tiles' (of V; all tiles' there), and its 32 rows of output K's again.  All of it in unpadded, swizzled rows.  Behind it 256
// bytes per wave that loads issued only to bring lines into L2 write to.
// Workgroups whose two halves share the prompt (ks = 2): each half's tiles and a place for one more (a third V tile where the head size is 128), which
// takes half of Q at first and, after the loop, the second half's (maximum, sum).
constexpr int attn_tiles_bytes(int d) { return 4 * KT * d * 2; }
constexpr int attn_lds_used(int d, int mwg) { return attn_tiles_bytes(d) + (mwg == 256 ? mwg * d * 2 : 0); }
constexpr int attn_lds_bytes(int d, int mwg, int ks) {
  return ks == 2 ? 2 * 5 * KT * d * 2 : attn_lds_used(d, mwg) + mwg / 32 * 256;
}
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct AttnCtx {
  int B, W, Hq, Hkv, g, ND, u;
  int M;            // W * g query rows per (b, kv head)
  int MB;           // row blocks per (b, kv head)
  int nsplit;       // L segments per request
  int n_groups;     // B * Hkv * nsplit
  float rcp_hkv;    // 1 / Hkv, a little high: n * rcp_hkv is n / Hkv rounded down for 0 <= n < 512
  float rcp_g, rcp_u;       // 1 / g, 1 / max(u, 1)
  uint32_t inv_mb, inv_split, inv_hkv;       // for div_by
  float c;          // sm_scale * log2(e)
  float k_scale, v_scale;   // FP8 prompt cache: value = code * scale (1 for the bf16 cache)
  const uint16_t* q;
  const uint16_t* ks;
  const uint16_t* vs;
  const int32_t* cu;
  const uint16_t* ku;
  const uint16_t* vu;
  uint16_t* out;
  float* lse;
  float* part_o;    // [B, nsplit, Hkv, M rows in blocks of 32: D / 4, row, 4] fp32, unnormalised
  float* part_ml;   // [B, nsplit, Hkv, M, 2] (max in log2 domain, sum)
  const int32_t* order;   // [B] requests by decreasing prompt length, or nullptr (requests taken in index order)
  const int32_t* slot;    // [B, W, ND] row of the request's own-token block that holds (beam, token), or nullptr (= w * ND + t)
};

// The kernel's arguments, read where this stands and not before: what only rare or late code needs takes no scalar registers through the prompt loop.
typedef const __attribute__((address_space(4))) AttnCtx* LateArgs;
__device__ __forceinline__ LateArgs late_args() {
  LateArgs a = (LateArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return a;
}

// n / d and n % d for 0 <= n < 2^22 and a small runtime divisor, through a float reciprocal and one
// correction step (a handful of instructions where the generic 32-bit division takes dozens).
__device__ __forceinline__ void divmod_small(int n, int d, float rcp_d, int* q, int* r) {
  int qq = (int)((float)n * rcp_d);
  int rr = n - qq * d;
  if (rr >= d) { qq++; rr -= d; }
  if (rr < 0) { qq--; rr += d; }
  *q = qq; *r = rr;
}

// n / d for any n, with inv = (2^32 - 1) / d rounded down from the host: the product's high word is n / d or one less.  (In scalar registers; the generic
// division by a number from memory is three times as long, and a unit starts with four of them.)
constexpr uint32_t div_inv(uint32_t d) { return 0xffffffffu / d; }
__device__ __forceinline__ unsigned div_by(unsigned n, unsigned d, uint32_t inv) {
  const unsigned q = __umulhi(n, inv);
  return q + (n - q * d >= d ? 1u : 0u);
}
// r / g for 0 <= r < 2^22, with rcp = 1 / g rounded to nearest: (r + 1/2) / g is at least 1/(2g) from a whole number, and two roundings move it by less
// than (r + 1/2) / g * 2^-23 (1 + 2^-25) < 1/(2g).
__device__ __forceinline__ int small_div(int r, float rcp) { return (int)fmaf((float)r, rcp, 0.5f * rcp); }

__device__ __forceinline__ int wave_total(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);      // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);      // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);      // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);      // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);      // lane 15 of rows 0, 2 to rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);      // lane 31 to rows 2, 3
  return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ int rank_in(uint64_t mask) {     // lanes of the mask in front of this one
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}
// The request of rank `rank` by decreasing prompt length (ties by index), its first row and its length; every wavefront by itself, lane i
// with requests i and i + 64.  About 0.2 us, which the two dependent loads that it takes the place of (the order, then the
// request's rows) cost as well; a kernel for the order is 5.6 us in front of the call.
constexpr int kRankB = 128;
__device__ __forceinline__ int request_by_length(const int32_t* cu, int B, int rank, int lane, int* row0, int* len) {
  int first[2], l[2];
#pragma unroll
  for (int k = 0; k < 2; k++) {
    first[k] = 0; l[k] = -1;
    if (lane + 64 * k < B) { first[k] = cu[lane + 64 * k]; l[k] = cu[lane + 64 * k + 1] - first[k]; }
  }
  auto reach = [&](int n) { return __popcll(__ballot(l[0] >= n)) + __popcll(__ballot(l[1] >= n)); };
  int lo = 0, hi = 64;                                       // more than `rank` requests reach lo, not so many hi
  while (hi < 1 << 30 && reach(hi) > rank) { lo = hi; hi <<= 1; }
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (reach(mid) > rank) lo = mid; else hi = mid;
  }
  rank -= reach(hi);                                         // among those of length lo
  const uint64_t same0 = __ballot(l[0] == lo), same1 = __ballot(l[1] == lo);
  const bool upper = rank >= __popcll(same0);
  const uint64_t same = upper ? same1 : same0;
  rank -= upper ? __popcll(same0) : 0;
  const uint64_t it = __ballot(((same >> lane) & 1) && rank_in(same) == rank);
  const int at = __ffsll((unsigned long long)it) - 1;
  *row0 = __builtin_amdgcn_readlane(upper ? first[1] : first[0], at);
  *len = lo;
  return at + (upper ? 64 : 0);
}

// The larger of a value and the other half's (of lane ^ 32).
__device__ __forceinline__ float halves_max(float v) {
  const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1]));
}

// Per-tile building blocks.  A tile is KT = 64 prompt tokens; S^T of a tile is [64 kv x 32*NCB q]
// = 2 sub-tiles x NCB column blocks of 32x32 fp32 accumulators.
template <int D, int NCB>
struct AttnTile {
  // Prompt tiles arrive by direct global->LDS loads: a wave-level load writes 1 KiB of consecutive LDS (lane l -> bytes
  // 16 l ..), so tile rows cannot be padded.  Instead the 16-byte pieces of a row are stored permuted (piece p of row r
  // sits in slot p ^ swz(r); the lane that fills slot s fetches piece s ^ swz(r) from memory), chosen so that the
  // operand reads below hit every bank group once:
  //   K (ds_read_b128, 16 lanes = 16 consecutive rows, same piece): swz = r & 15 (256-byte rows) or (r >> 1) & 7 (128-byte rows);
  //   V (ds_read_b64_tr_b16, 32 lanes = 4 consecutive rows x 4 pieces):  swz = 4 (r & 3)  or  4 ((r >> 1) & 1).
  static constexpr int PPRW = D / 8;                                       // 16-byte pieces per row
  static __device__ __forceinline__ int swz_k(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
  static __device__ __forceinline__ int swz_v(int r) { return D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1); }
  // Per-lane LDS addresses of the operand reads of a tile at the start of LDS, fixed for the whole kernel: what tile slot, slab and
  // block add to them is known at compile time and goes into the instructions.
  struct Rd { int k[D / 16]; int v[D / 32]; };
  static __device__ __forceinline__ Rd make_rd(int lane, int lds_base) {
    const int G = lane >> 5, n32 = lane & 31;
    Rd r;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) r.k[ks] = lds_base + 2 * (n32 * D + ((2 * ks + G) ^ swz_k(n32)) * 8);
    const int vrow = 4 * G + ((lane & 15) >> 2);
#pragma unroll
    for (int db = 0; db < D / 32; db++)
      r.v[db] = lds_base + 2 * (vrow * D + ((4 * db + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ swz_v(vrow)) * 8 + 4 * (lane & 1));
    return r;
  }
  // K operand of 32 tokens `sub` and 16 dimensions `ks`; V^T operand of 16 tokens `slab` and 32 dimensions `db`
  static __device__ __forceinline__ bf16x8 read_k(int tile, const Rd& r, int sub, int ks) {         // `tile`: element offset in LDS
    typedef const u32x4 __attribute__((address_space(3))) * lds_u32x4;
    return __builtin_bit_cast(bf16x8, *(lds_u32x4)(uintptr_t)(uint32_t)(r.k[ks] + 2 * (tile + sub * 32 * D)));
  }
  static __device__ __forceinline__ bf16x8 read_v(int tile, const Rd& r, int slab, int db) {
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    typedef s16x4 __attribute__((address_space(3))) * lds_s16x4;
    const int at = r.v[db] + 2 * (tile + slab * 16 * D);
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)(uint32_t)at);
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(uintptr_t)(uint32_t)(at + 2 * 8 * D));
    s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
  }
  // S^T = K . Q^T from the K tile in LDS (A operand) and Q in registers (B operand)
  static __device__ __forceinline__ void qk(int sk, const bf16x8 (&qop)[NCB][D / 16], f32x16 (&s)[KT / 32][NCB],
                                            const Rd& rdo) {
#pragma unroll
    for (int sub = 0; sub < KT / 32; sub++)
#pragma unroll
      for (int cb = 0; cb < NCB; cb++)
#pragma unroll
        for (int i = 0; i < 16; i++) s[sub][cb][i] = 0.f;
    // operand reads run PF steps ahead of the MFMAs that consume them
    constexpr int N = (KT / 32) * (D / 16), PF = 4;
    bf16x8 a[N];
#pragma unroll
    for (int i = 0; i < PF; i++) a[i] = read_k(sk, rdo, i % 2, i / 2);
#pragma unroll
    for (int i = 0; i < N; i++) {
      if (i + PF < N) a[i + PF] = read_k(sk, rdo, (i + PF) % 2, (i + PF) / 2);
#pragma unroll
      for (int cb = 0; cb < NCB; cb++) s[i % 2][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], qop[cb][i / 2], s[i % 2][cb], 0, 0, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, PF, 0);
#pragma unroll
    for (int i = 0; i < N - PF; i++) {
      __builtin_amdgcn_sched_group_barrier(0x008, NCB, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, PF * NCB, 0);
  }

  // Per-lane maximum of a tile's scores for the lane's query column (both halves of the column).
  static __device__ __forceinline__ float colmax(const f32x16 (&s)[KT / 32][NCB]) {
    float mx = -INFINITY;
#pragma unroll
    for (int sub = 0; sub < KT / 32; sub++)
#pragma unroll
      for (int i = 0; i < 16; i += 2) mx = fmaxf(fmaxf(mx, s[sub][0][i]), s[sub][0][i + 1]);
    return halves_max(mx);
  }

  // One steady-state tile with the matrix and vector pipes kept busy together.  The wave issues, in this order,
  // the MFMAs of S(t+1) = K(t+1).Q^T and then those of O += V(t).P(t); between consecutive MFMAs it
  // exponentiates a fixed share of tile t's scores (their reference m2 is already decided), so that
  // the 32 quarter-rate exponentials per lane run in the shadow of the 32 MFMAs instead of after them.  P(t)'s quarters are
  // complete when the PV MFMAs come to them.  Instruction order is pinned chunk by chunk.
  // Measured at 32 x 4096 tokens x 256 beams, two wavefronts per SIMD: 507 us with the exponentials staged over three chunks, 515
  // with each finished in one; 8 x 2048 x 128 (one wavefront per SIMD, 1.1 us a tile): 40.1 against 41.4 us.  Operand reads 5 or 6
  // MFMAs ahead: no change.
  static constexpr int NQK = (KT / 32) * (D / 16), NPV = (KT / 16) * (D / 32), NMF = NQK + NPV;
  // All 32 exponentials are issued after this many MFMAs: as late as the last quarter of the probabilities, packed two chunks later, allows.  us with NPV / 2
  // and with this: 32 x 4096 x 256 beams 477.9, 472.6; 64 ragged requests of 512-8192 853, 845; 8 causal prompts of 1024-8192 1184, 1173.
  static constexpr int EXP_BY = NQK + NPV * 11 / 16;
  static constexpr int exps_after(int j) {                // exponentials finished once MFMA j's chunk has been issued
    const int t = (32 * (j + 1) + EXP_BY - 1) / EXP_BY;
    return j < 0 ? 0 : (t > 32 ? 32 : t);
  }
  // The workgroup meets before the tile's last HEAD MFMAs (0: after all), whose operands are in registers by then: loads for the tile after have landed, everybody has
  // read K(t+1) and V(t), and the next tile's first HEAD operands are read beside those MFMAs.  With the meeting between two tiles every wave of
  // the CU asked LDS for its first operands at once, with nothing to compute meanwhile: 8 causal prompts of 1024-8192 tokens 1210 -> 1189 us, 4 x 16384
  // x 512 beams in FP8 456.7 -> 452.7, 64 ragged requests of 512-8192 x 256 864 -> 853.  (4 MFMAs: 1189, 450, 860, but 32 x 4096 x 256 478 instead of
  // 476; 1: 1199, 456, 859.)
  // `between` is called in every chunk: the loads of tiles ahead are issued there, one every second MFMA (head size 64: every one).  Issued
  // together at the start of a tile they held all waves up while the CU's address unit worked them off: 32 x 4096 x 256 beams 486 -> 472 us, the 64
  // ragged requests 873 -> 849, 16 x 2000 x 200 beams of head size 64 21.4 -> 20.5.
  static constexpr int PF = 4;                           // operand reads run PF MFMAs ahead
  static constexpr int SPREAD = D == 128 ? 2 : 1;
  template <int HEAD, class F, class G>
  static __device__ __forceinline__ void fused(F&& between, G&& meet, bf16x8 (&head)[PF], int sk_after, int sk_next, int sv_cur, const bf16x8 (&qop)[NCB][D / 16],
                                               const f32x16 (&s_cur)[KT / 32][NCB], f32x16 (&s_next)[KT / 32][NCB],
                                               f32x16 (&o)[D / 32][NCB], float m2, float c, float& rs, bf16x8 (&pop)[KT / 16], const Rd& rdo) {
    static_assert(NCB == 1, "one column block per wave");
    auto rdk = [&](int i) { return read_k(sk_next, rdo, i % 2, i / 2); };
    auto rdv = [&](int i) { return read_v(sv_cur, rdo, i / (D / 32), i % (D / 32)); };
    bf16x8 a[NMF];
    float p[32], arg[32];                                   // (a few of each are alive at a time)
    rs = 0.f;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < PF; i++) a[i] = i < HEAD ? head[i < HEAD ? i : 0] : rdk(i);
#pragma unroll
    for (int e = 0; e < exps_after(0); e++) arg[e] = fmaf(s_cur[e / 16][0][e % 16], c, -m2);
#pragma unroll
    for (int j = 0; j < NMF; j++) {
      if (j == NMF - HEAD) meet();
      if (j + PF < NMF) a[j + PF] = (j + PF < NQK) ? rdk(j + PF) : rdv(j + PF - NQK);
      else if (j >= NMF - HEAD) head[j + HEAD - NMF] = read_k(sk_after, rdo, (j + HEAD - NMF) % 2, (j + HEAD - NMF) / 2);
      if (j < NQK) {
        s_next[j % 2][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j], qop[0][j / 2], j < 2 ? zero : s_next[j % 2][0], 0, 0, 0);
      } else {
        const int i = j - NQK;
        o[i % (D / 32)][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[j], pop[i / (D / 32)], o[i % (D / 32)][0], 0, 0, 0);
      }
      between(j);
      // the exponentials' arguments, the exponentials and their sums and packing are three stages, one chunk apart, so that none
      // waits for the one before
#pragma unroll
      for (int e = exps_after(j - 2); e < exps_after(j - 1); e++) rs += p[e];
#pragma unroll
      for (int e = exps_after(j - 1); e < exps_after(j); e++) p[e] = __builtin_amdgcn_exp2f(arg[e]);
#pragma unroll
      for (int e = exps_after(j); e < exps_after(j + 1); e++) arg[e] = fmaf(s_cur[e / 16][0][e % 16], c, -m2);
#pragma unroll
      for (int e = exps_after(j - 2); e < exps_after(j - 1); e++) {
        if (e % 8 == 7) {
          bf16x8 pk;
#pragma unroll
          for (int k = 0; k < 8; k += 2) {
            f32x2 two = {p[e - 7 + k], p[e - 7 + k + 1]};
            bf16x2 h = __builtin_convertvector(two, bf16x2);
            pk[k] = h[0];
            pk[k + 1] = h[1];
          }
          pop[e / 8] = pk;
        }
      }
      asm volatile("" : "+v"(rs));                           // the running sum is due here, not at the end of the tile
      __builtin_amdgcn_sched_barrier(0);
    }
    if (HEAD == 0) meet();
  }

  // A segment's first and last tile are searched for the columns' maxima before their probabilities are made, the tiles between only from where a
  // wavefront meets scores that rise: 16 vector instructions a tile and an exchange between lanes, in a loop bound by what it issues
  // beside the MFMAs.  Worth 3 %: 32 x 4096 tokens x 256 beams 509 -> 495 us, 4 x 16384 x 512 in FP8 467 -> 454, 4 causal prompts of 3000 278 -> 268.
  // The reference is the first tile's maximum.  Where a lane's half of a column of a later tile sums to more than kRaise = 2^kLazy, which no
  // column does without a score kLazy - 5 bits above its reference, the column gets a higher reference after that tile, a power of two
  // for which this sum lies between 1 and 2, and the wavefront searches from there on: the reference becomes the maximum before a tile's
  // probabilities are made, once it is exceeded by more than kLazy.  us with the search in every tile, with it from the first rise, and with
  // neither, but columns that rose by 48 bits in a tile computed again: 32 x 4096 x 256 beams 509, 495, 492, and with scores of eight times
  // the width that N(0,1) queries and keys give 535, 542, 860; 4 causal prompts of 3000 278, 268, 268 and 297, 302, 495.
  //   Precision, in the one tile of the rise: the best token's probability, which may be nearly all of the sum, is not 1 as with the true
  // maximum; O has it rounded to bf16 and the sum has not.  What the rounding changed of the tile's sum is kept and O scaled by it at the end.
  //   Range: O may have overflowed there although the result does not.  A wavefront that met a rise looks through its O at the end, and where
  // it finds that, or where a sum passed kTooHigh, it computes its columns again (k_beam_attn's `redo`).
  //   A wavefront whose first tile has a score above kWide searches from the start: the scores will rise, perhaps beyond kTooHigh.  N(0,1) queries
  // and keys stay below 10 there.  Without it, scores 32 times as wide were computed twice: 32 x 4096 x 256 825 -> 542 us, 4 causal prompts
  // of 3000 421 -> 300, 4 x 16384 x 512 in FP8 1147 -> 468; N(0,1) inputs within 1 %.
  static constexpr float kLazy = 8.0f, kRaise = 256.0f, kTooHigh = 0x1p100f, kWide = 16.0f;

  // The segment's last tile, which no scores follow: O += V . P with the exponentials of the next 16 tokens between the MFMAs of the present
  // ones.  V^T operand: d = 32*db + (lane%32), k slot e <-> token 16*s + 8*(e/4) + 4*G + e%4.
  static __device__ __forceinline__ void finish(int sv, const f32x16 (&s)[KT / 32][NCB], f32x16 (&o)[D / 32][NCB], float m2, float c, float& rs, const Rd& rdo) {
    static_assert(NCB == 1, "one column block per wave");
    constexpr int DB = D / 32, N = NPV, PF = 4, EPC = 8 / DB;
    auto rdv = [&](int i) { return read_v(sv, rdo, i / DB, i % DB); };
    bf16x8 a[N], pop[KT / 16];
    float p[32];
    rs = 0.f;
    auto exps = [&](int e0, int n) {
#pragma unroll
      for (int e = e0; e < e0 + n; e++) {
        p[e] = __builtin_amdgcn_exp2f(fmaf(s[e / 16][0][e % 16], c, -m2));
        rs += p[e];
      }
    };
    auto pack = [&](int t) {
#pragma unroll
      for (int k = 0; k < 8; k += 2) {
        const f32x2 two = {p[8 * t + k], p[8 * t + k + 1]};
        const bf16x2 h = __builtin_convertvector(two, bf16x2);
        pop[t][k] = h[0];
        pop[t][k + 1] = h[1];
      }
    };
#pragma unroll
    for (int i = 0; i < PF; i++) a[i] = rdv(i);
    exps(0, 8);
    pack(0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < N; i++) {
      const int t = i / DB, k = i % DB;
      if (i + PF < N) a[i + PF] = rdv(i + PF);
      o[k][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], pop[t], o[k][0], 0, 0, 0);
      if (t + 1 < KT / 16) {
        exps(8 * (t + 1) + EPC * k, EPC);
        if (k == DB - 1) pack(t + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
};

// CAUSAL = false: the decode step described above.  CAUSAL = true: causal self-attention over the packed prompts
// (the prefill that fills the shared cache, Sections 2.2.1 / 5.1) through the same tiles: request b's query rows are
// its own tokens (row r = token r / g, head r % g of the KV group), a row block only walks the K/V tiles up to its
// last token, scores of keys after a row's token are set to -inf on the tiles that straddle the diagonal, and there
// is no own-token stage and no L split.
// KV8 = true: the prompt K/V are FP8 E4M3 codes with one scale per tensor (value = code * scale).  The tiles are widened
// to bf16 (exactly) on their way into LDS: 8-byte loads into registers one tile ahead, four conversions per 16-byte piece,
// a ds_write into the same swizzled layout the direct loads fill.  The scales never touch the tiles: the K scale goes into
// the exponent scale of the prompt loop, whose references are in log2 units of the true scores, and at the end of the loop O is
// multiplied by v_scale: the bf16 own-token stage and the epilogue work in true units.
// KS = 2: two sets of NWAVES wavefronts hold the same query rows and take one half of the segment's tiles each, with tiles
// of their own in LDS; the second set's (maximum, sum, O) goes through LDS into the first's before the epilogue.  For launches of at
// most one 128-row workgroup per CU, whose SIMDs would otherwise hold one wavefront each and wait out every chain of its tile
// (1.1 us a tile and wavefront, 0.9 with a second one beside it).
// FIND = true: a workgroup finds out from the lengths which unit it is: CAUSAL = false, requests by decreasing prompt length (at most kRankB);
// CAUSAL = true, an XCD's row blocks heaviest first over all of its (request, KV head) pairs.  (Kernels of their own: the others took 0.3 us
// longer with that code to jump over.)
template <int D, int NCB, int NWAVES, bool CAUSAL, bool KV8, int KS, bool FIND>
__global__ void __launch_bounds__(NWAVES * 64 * KS) __attribute__((amdgpu_waves_per_eu(NCB == 1 ? 2 : 1, NCB == 1 ? 2 : 1)))
k_beam_attn(AttnCtx c) {
  using T = AttnTile<D, NCB>;
  constexpr int NT = NWAVES * 64;                // threads of a set
  static_assert(KS == 1 || (KS == 2 && NWAVES == 4 && !CAUSAL), "two sets of four wavefronts");
  constexpr int MWG = NWAVES * 32 * NCB;
  constexpr int PPR = D / 8;                     // 16-byte pieces per row
  constexpr int TILE = KT * D;                   // elements of one K or V tile (unpadded, swizzled rows)
  constexpr int NCHUNK = TILE * 2 / 1024;        // 1 KiB chunks (= wave-level loads) per tile
  constexpr int CPW = NCHUNK / NWAVES;           // chunks per wave and tile
  constexpr int RPC = 1024 / (D * 2);            // rows per chunk
  static_assert(NCHUNK % NWAVES == 0, "tile must divide over the waves");
  // Tiles in LDS: K(j) in s_k[slot], V(j) in s_v[slot], slot = (j + flip) % 2 (flip is chosen below so that the last tile is in slot 0: the main loop
  // then names its slots at compile time); where there are three V tiles (VS), V(j) in s_v[j % 3].  Then, for workgroups of 8 waves, which own the
  // CU's LDS anyway, a region of its own for the Q hand-over, so that the first tiles can be in flight while Q is staged; of 4 waves, K's only
  extern __shared__ __attribute__((aligned(1024))) uint16_t smem[];
  const int set = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
  // V tiles in LDS.  Two sets of a large head have three and ask for V two tiles ahead: their units are few, so that memory's latency is waited for, and with the
  // loads spread over the MFMAs one tile is not always enough.  us from HBM with two and three: 8 x 2048 x 128 beams 44.4, 41.9; 8 x 3000 x 128 59.6, 55.6
  // (from the caches 37.3, 38.1; head size 64: 16 x 2000 x 200 21.6, 21.9 and 20.6, 21.0).
  constexpr int VS = KS == 2 && D == 128 ? 3 : 2;
  uint16_t* s_tiles = smem + set * 5 * TILE;
  uint16_t* s_k = s_tiles;
  uint16_t* s_v = s_tiles + 2 * TILE;
  constexpr bool kQSeparate = NWAVES * KS == 8;
  // (workgroups of 4 waves meet between tiles: another one on the CU computes meanwhile, and waits for memory are longer the earlier a tile's loads have to
  // have landed; 16 prompts of 60-700 tokens 36.2 us with 3, 35.6)
  constexpr int HEAD = NWAVES * KS == 4 ? 0 : D == 128 ? 3 : 2;
  // K loads of a tile that go out before the references are settled and the first operands read.  Tiles of head size 64 are short: where long prompts are streamed
  // by about a workgroup per CU, every tile waits for the way from the meeting to its loads.  us with none and with these: 60 x 16384 tokens x 56 beams, 8
  // query and 2 KV heads, 180, 171; 128 x 8000 x 30 109, 105; 40 of 4000-12000 x 120, 8 heads, 207, 202.  64 x 8000 x 100, 8 heads, where a CU's two workgroups
  // compute in turn, 200, 202 (with all of K's 205).  Head size 128: 80 of 12768-18396 x 150, 2 heads, 400, 393, but 160 x 8000 x 120 256, 261: none there.
  constexpr int EARLY = !KV8 && !CAUSAL && D == 64 ? (KS == 2 ? CPW : 1) : 0;
  // Q's rows: behind the tiles, of two sets half of them behind either's; of 4 waves, in place of the V tiles
  static_assert(NWAVES == 8 || MWG * D == 2 * TILE, "Q fits the V tiles' place");
  auto q_at = [&](int row) { return KS == 2 ? 4 * TILE + row * D + (row >= MWG / 2 ? 5 * TILE - TILE : 0) : (kQSeparate ? 4 : 2) * TILE + row * D; };

  const int tid = (int)threadIdx.x % NT, wave = tid >> 6, lane = tid & 63, G = lane >> 5, n32 = lane & 31;

  // XCD-aware unit order: workgroups are dealt round-robin to the 8 XCDs, so ids congruent mod 8
  // share an L2.  The MB row blocks that read the same K/V stream get consecutive slots of one XCD.
  const unsigned id = blockIdx.x;
  const int xcd = (int)(id & 7u);
  const unsigned slot = id >> 3;
  const unsigned nth = div_by(slot, (unsigned)c.MB, c.inv_mb);
  int group = (int)nth * 8 + xcd;
  int mbi = (int)(slot - nth * (unsigned)c.MB);
  if (CAUSAL) mbi = c.MB - 1 - mbi;            // the blocks with the most keys to visit start first
  int len_l = 0, row0_l = 0;
  if constexpr (CAUSAL && FIND) {
    // Lane i knows pair xcd + 8 i.  Unit `slot` of the order by falling block number: its number mbi is the largest with more than `slot`
    // blocks of that number or above, and of the pairs that have such a block it is the one behind the rest.
    const int mine = xcd + 8 * lane;
    if (mine < c.n_groups) {
      const int bm = (int)((float)mine * c.rcp_hkv);         // (exact: see the host)
      row0_l = c.cu[bm];
      len_l = c.cu[bm + 1] - row0_l;
    }
    const int blocks = (len_l * c.g + MWG - 1) / MWG;
    auto from = [&](int m) { return wave_total(max(blocks - m, 0)); };
    int above = c.MB, rank = (int)slot;
    mbi = 0;
    while (above - mbi > 1) {
      const int mid = (mbi + above) >> 1, n = from(mid);
      if (n > (int)slot) mbi = mid;
      else { above = mid; rank = (int)slot - n; }
    }
    const uint64_t have = __ballot(blocks > mbi);
    const uint64_t it = __ballot(blocks > mbi && rank_in(have) == rank);
    if (it == 0) return;                       // (past the last unit)
    const int l = __ffsll((unsigned long long)it) - 1;
    group = xcd + 8 * l;
    row0_l = __builtin_amdgcn_readlane(row0_l, l);
    len_l = __builtin_amdgcn_readlane(len_l, l);
  }
  if (group >= c.n_groups) return;
  const unsigned gq = CAUSAL ? (unsigned)group : div_by((unsigned)group, (unsigned)c.nsplit, c.inv_split);
  const int sp = CAUSAL ? 0 : (int)((unsigned)group - gq * (unsigned)c.nsplit);
  const int bi = (int)div_by(gq, (unsigned)c.Hkv, c.inv_hkv);
  const unsigned kvh = gq - (unsigned)bi * (unsigned)c.Hkv;
  int b = c.order ? c.order[bi] : bi;
  if constexpr (!CAUSAL && FIND) b = request_by_length(c.cu, c.B, bi, lane, &row0_l, &len_l);
  const unsigned bu = (unsigned)b;                             // (for offsets: no sign to extend, which takes scalar registers)
  const int row0 = FIND ? row0_l : c.cu[b];
  const int Lb = FIND ? len_l : c.cu[b + 1] - row0;
  const int Mb = CAUSAL ? Lb * c.g : c.M;                      // query rows of this (request, KV head)
  if (CAUSAL && mbi * MWG >= Mb) return;                       // (before any barrier: the whole workgroup leaves)
  int chunk = CAUSAL ? Lb : (int)div_by((unsigned)Lb + (unsigned)c.nsplit - 1u, (unsigned)c.nsplit, c.inv_split);
  chunk = ((chunk + KT - 1) / KT) * KT;
  // The segment whose unit takes the beams' own tokens too: the first, which starts first, or the last where its wavefronts have fewer tiles (4
  // requests of 500-1500 tokens x 64 beams, 8 heads of 64: 13.9 -> 12.6 us).
  const int last_tiles = max(0, Lb - (c.nsplit - 1) * chunk + KT - 1) / KT;
  const int own_sp = (last_tiles + KS - 1) / KS < (chunk / KT + KS - 1) / KS ? c.nsplit - 1 : 0;
  int seg0 = CAUSAL ? 0 : min(Lb, sp * chunk);
  int seg1 = CAUSAL ? __builtin_amdgcn_readfirstlane(small_div(min((mbi + 1) * MWG, Mb) - 1, c.rcp_g)) + 1 : min(Lb, seg0 + chunk);
  int ntiles = (seg1 - seg0 + KT - 1) / KT, set1_idle = 0;     // set1_idle: barriers that the second set waits at beside its own
  if (KS == 2) {                                               // the first set takes the odd tile
    const int n0 = (ntiles + 1) / 2, n1 = ntiles - n0;
    set1_idle = n0 - n1;
    const int mid = min(seg1, seg0 + n0 * KT);
    if (set == 0) seg1 = mid; else seg0 = mid;
    ntiles = set == 0 ? n0 : n1;
  }
  const int flip = (ntiles - 1) & 1;

  static_assert(NCB == 1, "one column block per wave");
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int row_w = mbi * MWG + wave_u * 32;                   // the wave's first query row
  int qrow[NCB];       // local query row or -1
  qrow[0] = row_w + n32 < Mb ? row_w + n32 : -1;
  const int beam_q = small_div(max(qrow[0], 0), c.rcp_g);      // the query's beam, or token
  // causal mode: the last key a column may see, and the first token of the wave's 32 columns (tiles that end at or
  // before it need no masking).  Columns past the end of the request keep everything (their output is dropped).
  const int tokq = (CAUSAL && qrow[0] >= 0) ? beam_q : 0x7fffffff;
  const int wave_tok0 = CAUSAL ? __builtin_amdgcn_readfirstlane(small_div(row_w, c.rcp_g)) : 0x7fffffff;

  f32x16 o_acc[D / 32][NCB];
#pragma unroll
  for (int db = 0; db < D / 32; db++)
#pragma unroll
    for (int cb = 0; cb < NCB; cb++)
#pragma unroll
      for (int i = 0; i < 16; i++) o_acc[db][cb][i] = 0.f;
  float m_run[NCB], l_run[NCB];                                // reference of the exponentials in log2 units, and sum
#pragma unroll
  for (int cb = 0; cb < NCB; cb++) { m_run[cb] = -INFINITY; l_run[cb] = 0.f; }

  // ---- K/V tile staging: global -> LDS directly (no registers, no LDS store instructions).  Wave w fills chunks
  // w, w + NWAVES, ... of a tile: lane l of chunk ch writes LDS bytes 1024 ch + 16 l, i.e. slot l % PPR of row
  // ch * RPC + l / PPR, and therefore fetches piece slot ^ swz(row) of that row.  Rows past the end of the segment
  // (last tile only) re-read the last valid row: finite values that the -inf score mask (K) and zero probabilities
  // (V) make irrelevant.  The loads are issued from inline assembly so that the compiler, which cannot tell the
  // tile buffers apart, does not make every later LDS read wait for them; `all_landed` waits for all of this
  // wave's loads, and the barrier that follows publishes every wave's.
  constexpr int EB = KV8 ? 1 : 2;                            // bytes per stored K/V element
  const uint32_t tok_bytes = (uint32_t)c.Hkv * D * EB;      // bytes between consecutive tokens
  const float cp = KV8 ? c.c * c.k_scale : c.c;              // exponent scale of the prompt loop
  typename T::Rd rdo = T::make_rd(lane, (int)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)s_tiles);
  // this lane's byte offsets from the tile's first row, per chunk (rows up to `most`)
  auto tile_offsets = [&](uint32_t (&off)[CPW], bool is_k, int most) {
#pragma unroll
    for (int i = 0; i < CPW; i++) {
      const int row = (i * NWAVES + wave) * RPC + lane / PPR, slot = lane % PPR;
      off[i] = (uint32_t)min(row, most) * tok_bytes + (uint32_t)((slot ^ (is_k ? T::swz_k(row) : T::swz_v(row))) * 16);
    }
  };
  const uint32_t lds_k = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)s_k;
  const uint32_t lds_v = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)s_v;
  auto dma = [&](uint32_t lds_addr, const char* gbase, uint32_t off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(off), "s"(gbase) : "memory", "m0");
  };
  // Tiles are asked for in their order, the last one again and again: the next one's address goes up by a tile, and when it is the last one, the only
  // one that can be partial, the offsets become its own.  (Worked out from its number, with a look at how full it is, a tile's
  // addresses were half of what stood between the MFMAs of two tiles: 64 ragged requests of 512-8192 x 256 beams 856 -> 845 us, 32 x 4096 x 256 476 -> 470.)
  const int tl = ntiles - 1;
  const int last_row = seg1 - (seg0 + tl * KT) - 1;          // of the last tile
  const uint32_t tile_bytes = KT * tok_bytes;                // (a prompt of more than one tile: below 2^32)
  const size_t first_byte = ((size_t)(unsigned)(row0 + seg0) * (unsigned)c.Hkv + kvh) * D * EB;
  const char* k_at = (const char*)c.ks + first_byte;
  const char* v_at = (const char*)c.vs + first_byte;
  uint32_t koff[CPW], voff[CPW];
  auto tload_chunk = [&](bool is_k, int buf, int i) {
    dma((is_k ? lds_k : lds_v) + (uint32_t)(buf * (TILE * 2) + (i * NWAVES + wave_u) * 1024), is_k ? k_at : v_at, is_k ? koff[i] : voff[i]);
  };
  auto tload = [&](bool is_k, int buf) {
#pragma unroll
    for (int i = 0; i < CPW; i++) tload_chunk(is_k, buf, i);
  };
  auto all_landed = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
  // FP8 tiles: piece p = tid + i * NT of a tile = 8 codes of row p / PPR; registers one tile ahead
  constexpr int P8 = KT * PPR / NT;                          // pieces per thread and tile
  struct Stage8 { uint2 r[P8]; };
  uint32_t off8[P8];                                         // byte offsets of this thread's pieces inside a tile
#pragma unroll
  for (int i = 0; i < P8; i++) { const int p = tid + i * NT; off8[i] = (uint32_t)(p / PPR) * tok_bytes + (uint32_t)(p % PPR) * 8; }
  // (pieces past the segment's last row read as 0, by the loads' bounds check: the bytes from the tile's first row to the segment's end)
  uint32_t k_left = (uint32_t)(seg1 - seg0) * tok_bytes, v_left = k_left;
  auto gload8_piece = [&](bool is_k, int i) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 r = __builtin_amdgcn_raw_buffer_load_b64(
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(is_k ? k_at : v_at), 0, is_k ? k_left : v_left, 0x00020000), (int)off8[i], 0, 0);
    return make_uint2(r.x, r.y);
  };
  auto gload8 = [&](bool is_k) {
    Stage8 st;
#pragma unroll
    for (int i = 0; i < P8; i++) st.r[i] = gload8_piece(is_k, i);
    return st;
  };
  auto offsets_of_last = [&](bool is_k) {
    if (KV8) return;
    int most = last_row;
    // (decode: worked out when they are needed; ahead of the loop they took registers through it, and something was spilled.  The causal kernels have
    // those registers, and a call of 16 short prompts was 0.4 % slower so.)
    if (CAUSAL && most == KT - 1) return;
    if (!CAUSAL) asm volatile("" : "+v"(most));
    tile_offsets(is_k ? koff : voff, is_k, most);
  };
  // to the next tile, or back
  auto advance = [&](bool is_k, bool back) __attribute__((always_inline)) {
    (is_k ? k_at : v_at) += back ? -(ptrdiff_t)tile_bytes : (ptrdiff_t)tile_bytes;
    if (KV8) (is_k ? k_left : v_left) += back ? tile_bytes : 0u - tile_bytes;
  };
  // the address of tile `to`, from that of the one before
  auto go_to = [&](bool is_k, int to) {
    if (to <= tl) advance(is_k, false);
    if (to == tl) offsets_of_last(is_k);
  };
  auto widen8 = [](uint2 r) {
    const bf16x2 e01 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)r.x, 1.0f, false);
    const bf16x2 e23 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)r.x, 1.0f, true);
    const bf16x2 e45 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)r.y, 1.0f, false);
    const bf16x2 e67 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)r.y, 1.0f, true);
    uint4 v;
    v.x = __builtin_bit_cast(uint32_t, e01); v.y = __builtin_bit_cast(uint32_t, e23);
    v.z = __builtin_bit_cast(uint32_t, e45); v.w = __builtin_bit_cast(uint32_t, e67);
    return v;
  };
  // (a thread's pieces are 16 rows or a multiple apart, in the same place of each: one address for all)
  static_assert(NT / PPR % 16 == 0, "swizzles repeat every 16 rows");
  const int row8 = tid / PPR, k8_to = row8 * D + ((tid % PPR) ^ T::swz_k(row8)) * 8, v8_to = row8 * D + ((tid % PPR) ^ T::swz_v(row8)) * 8;
  auto lstore8_piece = [&](uint16_t* dst, bool is_k, uint2 codes, int i) {
    *(uint4*)(dst + (is_k ? k8_to : v8_to) + i * (NT / PPR) * D) = widen8(codes);
  };
  auto lstore8 = [&](uint16_t* dst, bool is_k, const Stage8& st) {
#pragma unroll
    for (int i = 0; i < P8; i++) lstore8_piece(dst, is_k, st.r[i], i);
  };
  Stage8 k8, v8;

  // ---- geometry of the unshared stage (one segment only): every beam's own u decode tokens go through
  // the same MFMA path as the prompt.  The 32 query columns of a wave belong to a handful of beams
  // (32/g of them when g divides 32).  Their K rows and V rows form private 32-row mini-tiles,
  // row rho = beam_local * u + token, which direct loads bring into the wave's own slice of LDS in the prompt tiles' layout;
  // S^T = K_u . Q^T is a full 32 x 32 block of which a column
  // keeps only its own beam's u rows (the rest are masked to -inf), and O^T += V_u^T . P^T follows.
  // Compared with per-lane dot products this reads each beam's rows once instead of once per query
  // head and replaces ~1000 VALU operations per lane by 16 MFMAs per wave.  The first mini-tile's K is
  // asked for while the last prompt tile is being processed, its V while the scores are made.  (Through registers the rows took 330
  // instructions of the last tile's critical path.)
  constexpr int UR = 32;                                 // rows of a mini-tile
  const bool may_own = !CAUSAL && set == 0 && (sp == 0 || sp == c.nsplit - 1) && c.u > 0;     // (known before the prompt's length is)
  const bool own_stage = may_own && sp == own_sp;
  int beam0 = 0, Ru = 0;                                 // the wave's first beam, and its beams' own rows
  if (may_own && row_w < Mb) {
    beam0 = __builtin_amdgcn_readfirstlane(small_div(row_w, c.rcp_g));
    Ru = (__builtin_amdgcn_readfirstlane(small_div(min(row_w + 31, Mb - 1), c.rcp_g)) - beam0 + 1) * c.u;
  }
  const int my_lo = (qrow[0] >= 0) ? (beam_q - beam0) * c.u : -1;                // this column's rows [my_lo, my_lo + u)
  // Byte offset in the request's own-token block of the row behind row pass * 32 + lane % 32 of the mini-tiles (past the last one: the first's)
  const uint32_t own_bytes = (uint32_t)c.Hkv * D * 2;
  auto own_row = [&](int pass) {
    const int rho = pass * UR + n32;
    int bl, tok;
    divmod_small(rho < Ru ? rho : 0, c.u, c.rcp_u, &bl, &tok);
    int prow = (beam0 + bl) * c.ND + tok;
    if (c.slot && Ru > 0) {                                // (an entry outside the block falls back to the beam's own row)
      const int sl = c.slot[(size_t)bu * (unsigned)(c.W * c.ND) + (unsigned)prow];
      prow = ((unsigned)sl < (unsigned)(c.W * c.ND)) ? sl : prow;
    }
    return (uint32_t)prow * own_bytes;
  };
  const char* ku_b = (const char*)(c.ku + ((size_t)bu * (unsigned)(c.W * c.ND) * (unsigned)c.Hkv + kvh) * D);        // this request's own-token caches
  const char* vu_b = (const char*)(c.vu + ((size_t)bu * (unsigned)(c.W * c.ND) * (unsigned)c.Hkv + kvh) * D);
  // element offsets from s_tiles of the wave's mini-tiles: K in place of the K tiles, which the last tile's step no longer reads, or of Q
  const int own_k = (NWAVES == 8 ? 4 * TILE : 0) + wave_u * UR * D, own_v = (NWAVES == 8 ? 0 : 2 * TILE) + wave_u * UR * D;
  auto uload = [&](bool is_k, uint32_t row_off, int rows) {               // the first `rows` rows of a mini-tile, and what else is in their 1 KiB chunks
#pragma unroll
    for (int i = 0; i < UR / RPC; i++) {
      if (i * RPC >= rows) break;                          // (wave-uniform)
      const int row = i * RPC + lane / PPR, piece = (lane % PPR) ^ (is_k ? T::swz_k(row) : T::swz_v(row));
      dma(lds_k + (uint32_t)((is_k ? own_k : own_v) * 2 + i * 1024), is_k ? ku_b : vu_b, (uint32_t)__shfl((int)row_off, row, 64) + (uint32_t)piece * 16);
    }
  };

  // The own-token rows are what the end of a unit waits for: they are asked for three tiles before the last one, one 4-byte load
  // per 128-byte line into LDS that nobody reads, so that the loads into their places, which are free with the last tile only, find them in L2.
  auto touch = [&](uint32_t dump, const void* gbase, uint32_t off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(dump), "v"(off), "s"(gbase) : "memory", "m0");
  };
  // (with three V tiles, two sets of head size 128: one tile before the last one, when the place of the V tile after that is free)
  const int touch_own = own_stage && Ru > 0 ? max(0, ntiles - (VS == 3 ? 2 : 4)) : 0x7fffffff;
  auto touch_own_rows = [&](int v_free, uint32_t row_off) {      // v_free: place of a V tile that nobody reads, of three
    uint32_t w = (uint32_t)wave_u;
    asm volatile("" : "+s"(w));                            // (worked out here, not kept in a register from the start on)
    const uint32_t dump = (VS == 3 ? lds_v + (uint32_t)v_free * (TILE * 2) : lds_k + (KS == 2 ? 4 * TILE * 2 : attn_lds_used(D, MWG))) + w * 256;
    const uint32_t off = row_off + (D == 128 ? 128 * G : 0);
    touch(dump, ku_b, off);
    touch(dump, vu_b, off);
  };

  // ---- Q: the workgroup's MWG query rows come into LDS like K tiles (a lane that reads its own row straight from memory touches 32 rows
  // with every load), rows past the last one as that one: their columns are dropped.
  {
    constexpr int NWG = NWAVES * KS, QPW = MWG / RPC / NWG;    // 1 KiB chunks per wave
    // this request's queries (decode: its W beams; prefill: its own tokens); offsets inside it fit 32 bits
    const char* q_b = (const char*)(c.q + ((CAUSAL ? (size_t)(unsigned)row0 : (size_t)bu * (unsigned)c.W) * (unsigned)c.Hq + kvh * (unsigned)c.g) * D);
    const int wg_wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const uint32_t lds_0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)smem;
    const uint32_t skip = (uint32_t)(c.Hq - c.g) * D * 2;      // from a beam's last row of this KV head to the next beam's first
#pragma unroll
    for (int i = 0; i < QPW; i++) {
      const int ch = i * NWG + wg_wave, rl = ch * RPC + lane / PPR, r = min(mbi * MWG + rl, Mb - 1);
      dma(lds_0 + (uint32_t)q_at(ch * RPC) * 2, q_b, (uint32_t)r * (D * 2) + (uint32_t)small_div(r, c.rcp_g) * skip + (uint32_t)(((lane % PPR) ^ T::swz_k(rl)) * 16));
    }
  }
  if (!KV8) {
    tile_offsets(koff, true, KT - 1);
    tile_offsets(voff, false, KT - 1);
    if (tl == 0) { offsets_of_last(true); offsets_of_last(false); }
  }
  // first prompt tiles: requested before anything waits on memory; V(0) once Q has left its place where Q has no LDS of its own.
  Stage8 k8b;
  if (KV8) {
    if (ntiles > 0) { k8 = gload8(true); v8 = gload8(false); go_to(true, 1); k8b = gload8(true); }
  } else if (ntiles > 0) {
    tload(true, flip);
    if (kQSeparate) tload(false, VS == 3 ? 0 : flip);
    go_to(true, 1);
    tload(true, flip ^ 1);
    if (VS == 3) { go_to(false, 1); tload(false, 1); }
  }
  // (Where there is a slot table its entries are waited for here, and with them, loads returning in order, every tile asked for before.  That is hidden: us a call
  // without and with a table: 1 x 256 tokens x 16 beams of head size 64 6.80, 6.79; 1 x 1531 x 128 16.8, 16.9; 8 x 2048 x 128 37.0, 37.1.  Asked for ahead of
  // Q, so that the first scores wait for Q and K(0) alone: 6.7, 16.8, 37.3, and 0.3 to 0.5 % more for a whole decode of 1 x 1531 x 128.)
  uint32_t prow0 = may_own ? own_row(0) : 0;
  // Q as B operands: lane holds query column n32 of the wave's block, d = 16*ks + 8*G + (0..7)
  bf16x8 qop[NCB][D / 16];
  {
    if (KV8 && kQSeparate && ntiles > 0) {
      lstore8(s_k + flip * TILE, true, k8); lstore8(s_v + (VS == 3 ? 0 : flip * TILE), false, v8); lstore8(s_k + (flip ^ 1) * TILE, true, k8b);
      go_to(true, 2); go_to(false, 1);
      k8 = gload8(true);
      v8 = gload8(false);
    }
    // (Q and K(0), which the first scores take; what was asked for after them may be on its way, but for calls with a slot table.  The FP8 codes that were waited for came after Q.)
    if (ntiles == 0) all_landed();
    else if (!KV8) asm volatile("s_waitcnt vmcnt(%0)" ::"i"((kQSeparate ? VS : 1) * CPW) : "memory");
    else if (!kQSeparate) all_landed();
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) qop[0][ks] = T::read_k(q_at(wave_u * 32) - (int)(s_tiles - smem), rdo, 0, ks);
    if (!kQSeparate) {
      __syncthreads();                               // the V tile slots may now be overwritten
      if (!KV8 && ntiles > 0) tload(false, flip);
      if (KV8 && ntiles > 0) {
        lstore8(s_k + flip * TILE, true, k8); lstore8(s_v + flip * TILE, false, v8); lstore8(s_k + (flip ^ 1) * TILE, true, k8b);
        go_to(true, 2); go_to(false, 1);
        k8 = gload8(true);
        v8 = gload8(false);
        __syncthreads();
      }
    }
  }

  float rounded = 0.f;                                 // what O has more of the sum than l_run, by rounding, in a tile of a rise
  bool rise = false, again = false;                    // some column's scores rose far above its reference; too far
  if (ntiles > 0) {
    // Pipeline: iteration t issues S(t+1) = K(t+1).Q^T together with the softmax of S(t), then O += V(t).P(t).
    // Meanwhile K(t+2) and V(t+1) are on their way into LDS, in the places of K(t) and V(t-1), which everybody had read when the
    // workgroup met near the end of the iteration before: one barrier per tile orders every buffer reuse.  Loads for tiles past the end are clamped to the
    // last tile (harmless re-reads; a duplicate K tile lands in a buffer nobody reads any more).

    // One steady-state iteration: tile t (scores in s_in) has a successor whose scores go to s_out.  The references are settled
    // first (raising them, and rescaling O and the running sum, is a rare wave-uniform branch), so that the tile's MFMAs and
    // exponentials form one straight-line block.
    float rs = 0.f;                                    // sum of the tile before
    bf16x8 pop[KT / 16];                               // the probabilities behind rs
    auto rescale = [&](float alpha) __attribute__((always_inline)) {
#pragma unroll
      for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) o_acc[db][0][i] *= alpha;
      l_run[0] *= alpha;
      rounded *= alpha;
    };
    auto rose = [&]() __attribute__((always_inline)) { return __any(!(rs <= T::kRaise)); };
    auto settle = [&]() __attribute__((always_inline)) {       // by the sum of the tile before
      if (KS == 2 ? __builtin_expect(!rise && rose(), 0) : !rise && rose()) {
        rise = true;
        const float r = halves_max(rs);
        again = again || __any(!(r <= T::kTooHigh));
        float in_o = 0.f;
#pragma unroll
        for (int e = 0; e < 32; e++) in_o += (float)pop[e / 8][e % 8];
        if (r > T::kRaise) rounded += in_o - rs;
        const float m_new = r > T::kRaise ? m_run[0] + (float)(__builtin_amdgcn_frexp_expf(r) - 1) : m_run[0];
        rescale(__builtin_amdgcn_exp2f(m_run[0] - m_new));
        m_run[0] = m_new;
      }
    };
    auto raise_to = [&](float mx) __attribute__((always_inline)) {       // by the maximum of this tile
      if (__any(mx > m_run[0] + T::kLazy)) {
        const float m_new = fmaxf(m_run[0], mx);
        rescale(__builtin_amdgcn_exp2f(m_run[0] - m_new));
        m_run[0] = m_new;
      }
    };
    auto causal_mask = [&](f32x16 (&s)[KT / 32][NCB], int tok0) {
#pragma unroll
      for (int sub = 0; sub < KT / 32; sub++)
#pragma unroll
        for (int i = 0; i < 16; i++) {
          const int kv = tok0 + sub * 32 + 8 * (i / 4) + 4 * G + (i % 4);
          s[sub][0][i] = (kv > tokq) ? -INFINITY : s[sub][0][i];
        }
    };
    // (inline assembly, so that no read of LDS is moved ahead of it; FP8 tiles are written by ds_write)
    auto meet = [&]() __attribute__((always_inline)) {
      if (KV8) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(VS == 3 ? CPW : 0) : "memory");      // (three V tiles: the last one asked for is not needed yet)
    };
    bf16x8 head[T::PF];
    constexpr int kAheadK = KV8 ? 3 : 2, kAheadV = KV8 ? 2 : VS - 1;       // step t asks for tiles t + kAhead
    const int seldom = min(tl - kAheadK, touch_own);
    int vs = 0;                                        // three V tiles: the place of V(t), which rdo.v has in it
    auto step = [&](auto slot_c, f32x16 (&s_in)[KT / 32][NCB], f32x16 (&s_out)[KT / 32][NCB], int t) {      // tile t in slot slot_c
      constexpr int slot = decltype(slot_c)::value;
      int v_to;
      auto ask = [&]() __attribute__((always_inline)) {
        v_to = VS == 3 ? (vs == 0 ? 2 : vs - 1) : slot ^ 1;
        advance(true, false);
        advance(false, false);
        if (__builtin_expect(t >= seldom, KS == 2)) {                               // (one test for what the last steps have to do)
          if (t == touch_own) touch_own_rows(v_to, prow0);
          if (t + kAheadK >= tl) { if (t + kAheadK > tl) advance(true, true); else offsets_of_last(true); }
          if (t + kAheadV >= tl) { if (t + kAheadV > tl) advance(false, true); else offsets_of_last(false); }
        }
#pragma unroll
        for (int i = 0; i < EARLY; i++) tload_chunk(true, slot, i);
      };
      if (EARLY > 0) ask();
      l_run[0] += rs;
      if (CAUSAL && seg0 + t * KT + KT - 1 > wave_tok0) causal_mask(s_in, seg0 + t * KT);       // (wave-uniform) past the wave's first token
      // (one branch where the tiles are many; two sets, whose kernels are short of registers, spilled with it: FP8 codes, 12 x 900 x 60 beams 21.4 us, 19.2)
      if (KS == 2) {
        settle();
        if (__builtin_expect(rise, 0)) raise_to(T::colmax(s_in) * cp);
      } else if (__builtin_expect(rise || rose(), 0)) {
        settle();
        raise_to(T::colmax(s_in) * cp);
      }
      if (EARLY == 0) ask();
      T::template fused<HEAD>([&](int j) __attribute__((always_inline)) {
        const int i = j / T::SPREAD + EARLY;
        if (KV8) {
          if (j % T::SPREAD || i >= 2 * P8) return;
          if (i < P8) {
            lstore8_piece(s_k + slot * TILE, true, k8.r[i], i);     // K(t+2) over K(t)
            k8.r[i] = gload8_piece(true, i);                        // K(t+3)
          } else {
            lstore8_piece(s_v + (VS == 3 ? (vs == 2 ? 0 : vs + 1) : slot ^ 1) * TILE, false, v8.r[i - P8], i - P8);       // V(t+1)
            v8.r[i - P8] = gload8_piece(false, i - P8);             // V(t+2)
          }
          return;
        }
        if (j % T::SPREAD || i >= 2 * CPW) return;
        if (i < CPW) tload_chunk(true, slot, i);               // K(t+2) over K(t)
        else tload_chunk(false, v_to, i - CPW);                // V(t+1), of three V tiles V(t+2), over V(t-1)
      }, meet, head, slot * TILE, (slot ^ 1) * TILE, (VS == 3 ? 2 : 2 + slot) * TILE, qop, s_in, s_out, o_acc, m_run[0], cp, rs, pop, rdo);
      if (VS == 3) {
        const int on = (vs == 2 ? -2 : 1) * (TILE * 2);
#pragma unroll
        for (int db = 0; db < D / 32; db++) rdo.v[db] += on;
        vs = vs == 2 ? 0 : vs + 1;
      }
    };
    // the last tile of the segment: the only one that can be partial, and it has no successor
    auto last = [&](f32x16 (&s_in)[KT / 32][NCB], int t) {
      l_run[0] += rs;
      settle();
      if (own_stage) uload(true, prow0, Ru);               // (into the place of K tiles that nobody reads any more)
      const int tok0 = seg0 + t * KT;
      if (tok0 + KT > seg1) {
#pragma unroll
        for (int sub = 0; sub < KT / 32; sub++)
#pragma unroll
          for (int i = 0; i < 16; i++) {
            const int kv = tok0 + sub * 32 + 8 * (i / 4) + 4 * G + (i % 4);
            s_in[sub][0][i] = (kv >= seg1) ? -INFINITY : s_in[sub][0][i];
          }
      }
      if (CAUSAL) causal_mask(s_in, tok0);
      const float top = T::colmax(s_in) * cp;
      if (t == 0) m_run[0] = top; else raise_to(top);
      T::finish(2 * TILE, s_in, o_acc, m_run[0], cp, rs, rdo);
      l_run[0] += rs;
      if (VS == 3) {
        all_landed();                                  // (the copy of the last V tile that came for nothing, before its place is used)
#pragma unroll
        for (int db = 0; db < D / 32; db++) rdo.v[db] -= vs * (TILE * 2);
      }
    };

    f32x16 s_a[KT / 32][NCB], s_b[KT / 32][NCB];      // ping-pong score accumulators: no copies
    T::qk(flip * TILE, qop, s_a, rdo);
    if (ntiles > 1) {
      if (CAUSAL && seg0 + KT - 1 > wave_tok0) causal_mask(s_a, seg0);
      m_run[0] = T::colmax(s_a) * cp;                  // (every column sees the segment's first token)
      rise = __any(m_run[0] > T::kWide);
    }
    meet();                                            // K(1) and V(0) are there
    if (ntiles > 1) {
#pragma unroll
      for (int i = 0; i < HEAD; i++) head[i] = T::read_k((flip ^ 1) * TILE, rdo, i % 2, i / 2);
    }
    // ntiles - 1 steps, then the last tile.  An odd step is peeled off first so that the loop runs
    // whole ping-pong pairs and the last tile is always in s_a.
    int t = 0;
    if (flip) {
      step(std::integral_constant<int, 1>(), s_a, s_b, 0);
#pragma unroll
      for (int sub = 0; sub < KT / 32; sub++)
#pragma unroll
        for (int cb = 0; cb < NCB; cb++) s_a[sub][cb] = s_b[sub][cb];
      t = 1;
    }
    for (; t + 1 < ntiles; t += 2) {
      step(std::integral_constant<int, 0>(), s_a, s_b, t);
      step(std::integral_constant<int, 1>(), s_b, s_a, t + 1);
    }
    last(s_a, t);
  }

  // KS = 2: the second set's O, as its lanes hold it, in place of its tiles (each wave's in the places of its mini-tiles: another may still compute its
  // columns again in its own), and its (maximum, sum) pairs
  uint16_t* s_set1 = smem + 5 * TILE;
  auto set1_o = [&](int e) { return (f32x4*)(s_set1 + (e < D / 16 ? own_k : own_v) + (e % (D / 16)) * 512) + lane; };
  float* s_set1_ml = (float*)(s_set1 + 4 * TILE);

  // ---- unshared stage (see its geometry above)
  if (KS == 2 && set == 1)
    for (int i = 0; i < set1_idle; i++) __syncthreads();
  if (KS == 2 || own_stage || ntiles > 0) __syncthreads(); // every wave is done with the prompt tiles
  // (m, l, O) joined by 32 rows in LDS, this wave's alone; the column sees row base + k where base + k is below `rows` (as unsigned numbers), and rows
  // from `used` on are seen by none.  The reference is the maximum of what the column has seen, so that the best own token's probability, which may
  // be nearly all of the sum, is 1 and not rounded.  before_v: what has to be done before V is read.
  auto mini_tile = [&](int base, unsigned rows, int used, float cs, float& m, float& l, auto&& before_v) {
    f32x16 su;
#pragma unroll
    for (int i = 0; i < 16; i++) su[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < D / 16; ks++) su = __builtin_amdgcn_mfma_f32_32x32x16_bf16(T::read_k(own_k, rdo, 0, ks), qop[0][ks], su, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 16; i++) su[i] = (unsigned)(base + 8 * (i / 4) + 4 * G + (i % 4)) < rows ? su[i] : -INFINITY;
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; i++) mx = fmaxf(mx, su[i]);
    mx = halves_max(mx) * cs;
    if (__any(mx > m)) {
      const float m_new = fmaxf(m, mx), alpha = __builtin_amdgcn_exp2f(m - m_new);      // (m_new is -inf while the column has seen no key at all)
      const float scale = mx > m ? alpha : 1.f;
      l *= scale;
      m = m_new;
#pragma unroll
      for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) o_acc[db][0][i] *= scale;
    }
    const float ref = m > -INFINITY ? m : 0.f;
    float pr[16], rsum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; i++) {
      pr[i] = __builtin_amdgcn_exp2f(fmaf(su[i], cs, -ref));
      rsum += pr[i];
    }
    l += rsum;
    bf16x8 pu[UR / 16];
#pragma unroll
    for (int t = 0; t < UR / 16; t++)
#pragma unroll
      for (int e = 0; e < 8; e++) pu[t][e] = (__bf16)pr[8 * t + e];
    before_v();
#pragma unroll
    for (int t = 0; t < UR / 16; t++) {
      if (t > 0 && used <= 16 * t) break;                  // (wave-uniform)
#pragma unroll
      for (int db = 0; db < D / 32; db++)
        o_acc[db][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(T::read_v(own_v, rdo, t, db), pu[t], o_acc[db][0], 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");                    // the mini-tiles are rewritten by the next pass
  };
  // The segment again for a wave with a column whose scores rose too fast or whose O overflowed: 32 tokens at a time through its mini-tiles,
  // maxima first.  It waits for
  // memory and computes by turns while the rest of the chip idles: 4 requests of 16384 tokens x 256 beams in which four wavefronts have to
  // take 571 us instead of 276 (1010 with the pieces fetched one after the other), one of 8000 x 128 49 instead of 29 (72).
  auto redo = [&]() {
    constexpr int UP = UR * PPR / 64;                      // 16-byte pieces per lane and tensor
    uint16_t* k32 = s_tiles + own_k;
    uint16_t* v32 = s_tiles + own_v;
    all_landed();                                          // (the own tokens' K, which is written over)
    const LateArgs late = late_args();
    const size_t first_byte = ((size_t)(unsigned)row0 * (unsigned)late->Hkv + kvh) * D * EB;
    const char* kbase = (const char*)late->ks + first_byte;
    const char* vbase = (const char*)late->vs + first_byte;
    m_run[0] = -INFINITY; l_run[0] = 0.f;
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
      for (int i = 0; i < 16; i++) o_acc[db][0][i] = 0.f;
#pragma unroll 1
    for (int tok0 = seg0; tok0 < seg1; tok0 += UR) {
      f32x4 kp[UP], vp[UP];                                // (as 16 bytes)
#pragma unroll
      for (int i = 0; i < UP; i++) {
        const int pi = lane + 64 * i, row = pi / PPR, col = (pi % PPR) * 8;
        const size_t off = (size_t)min(tok0 + row, seg1 - 1) * tok_bytes + (size_t)col * EB;
        if constexpr (KV8) {
          kp[i] = __builtin_bit_cast(f32x4, widen8(*(const uint2*)(kbase + off)));
          vp[i] = __builtin_bit_cast(f32x4, widen8(*(const uint2*)(vbase + off)));
        } else {
          kp[i] = *(const f32x4*)(kbase + off);
          vp[i] = *(const f32x4*)(vbase + off);
        }
      }
#pragma unroll
      for (int i = 0; i < UP; i++) {
        const int pi = lane + 64 * i, row = pi / PPR, piece = pi % PPR;
        *(f32x4*)(&k32[row * D + (piece ^ T::swz_k(row)) * 8]) = kp[i];
        *(f32x4*)(&v32[row * D + (piece ^ T::swz_v(row)) * 8]) = vp[i];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");                  // (the mini-tiles are this wave's alone, and LDS serves a wave in order)
      mini_tile(tok0, CAUSAL ? min((unsigned)seg1, (unsigned)tokq + 1u) : (unsigned)seg1, UR, cp, m_run[0], l_run[0], [] {});
    }
    if (own_stage) uload(true, prow0, Ru);                 // (fetched again)
  };
  if (__builtin_expect(rise, 0)) {
    float z = l_run[0] * 0.f;                              // (0 unless something is infinite or no number)
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
      for (int i = 0; i < 16; i++) z = fmaf(o_acc[db][0][i], 0.f, z);
    if (again || __any(!(z == 0.f))) {
      redo();
    } else {
      const float l = l_run[0] + __shfl_xor(l_run[0], 32, 64), more = rounded + __shfl_xor(rounded, 32, 64);
      const float scale = more == 0.f ? 1.f : l / (l + more);
#pragma unroll
      for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) o_acc[db][0][i] *= scale;
    }
  }
  if (KV8 && ntiles > 0) {                                 // prompt loop -> true units
#pragma unroll
    for (int db = 0; db < D / 32; db++)
#pragma unroll
      for (int i = 0; i < 16; i++) o_acc[db][0][i] *= c.v_scale;
  }
  if (KS == 2 && set == 1) {
#pragma unroll
    for (int e = 0; e < D / 8; e++) {
      const f32x4 v = {o_acc[e / 4][0][4 * (e % 4)], o_acc[e / 4][0][4 * (e % 4) + 1], o_acc[e / 4][0][4 * (e % 4) + 2], o_acc[e / 4][0][4 * (e % 4) + 3]};
      *set1_o(e) = v;
    }
    const f32x2 ml = {m_run[0], l_run[0]};
    *(f32x2*)(s_set1_ml + (wave * 64 + lane) * 2) = ml;
  }
  if (own_stage) {
    int tiles = ntiles;
    // (compared again in the kernels that have no scalar registers to keep the result of the comparison at the start of the unit in)
    if (!KV8 && NWAVES * KS == 4) asm volatile("" : "+s"(tiles));
    if (tiles == 0) uload(true, prow0, Ru);
    uint32_t row_off = prow0;
    for (int pass = 0; pass * UR < Ru; pass++) {
      const int used = Ru - pass * UR;                     // (V: whole halves of 16 rows, whose probabilities are 0 past the last one)
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");      // (K is there, and the pass before has read V)
      uload(false, row_off, min(UR, (used + 15) & ~15));
      mini_tile(pass * UR - my_lo, my_lo >= 0 ? (unsigned)c.u : 0u, used, c.c, m_run[0], l_run[0], [&] {
        if (used > UR) { row_off = own_row(pass + 1); uload(true, row_off, used - UR); }       // (K has been read)
        all_landed();
      });
    }
  }

  // ---- the second set's half of the segment joins the first's
  if (KS == 2) {
    __syncthreads();
    if (set == 1) return;
    const f32x2 ml = *(const f32x2*)(s_set1_ml + (wave * 64 + lane) * 2);
    const float m_new = fmaxf(m_run[0], ml.x);
    const bool any_key = m_new > -INFINITY;                // false only for a column that has seen no key at all
    const float a0 = any_key ? __builtin_amdgcn_exp2f(m_run[0] - m_new) : 1.f;
    const float a1 = any_key ? __builtin_amdgcn_exp2f(ml.x - m_new) : 0.f;
    l_run[0] = l_run[0] * a0 + ml.y * a1;
    m_run[0] = m_new;
#pragma unroll
    for (int e = 0; e < D / 8; e++) {
      const f32x4 v = *set1_o(e);
#pragma unroll
      for (int k = 0; k < 4; k++) o_acc[e / 4][0][4 * (e % 4) + k] = o_acc[e / 4][0][4 * (e % 4) + k] * a0 + v[k] * a1;
    }
  }

  // ---- epilogue: merge is already done in registers; normalise or write this segment's partials
  {
    const int r = qrow[0];
    const float m = m_run[0], l = l_run[0];
    const float l_tot = l + __shfl_xor(l, 32, 64);
    if (c.nsplit == 1) {
      // The wave's 32 rows x D outputs go through its own slice of LDS so that global memory sees whole
      // 256-byte rows (16 lanes x 16 bytes) instead of 8-byte pieces of 32 different rows per store.
      uint16_t* s_o = s_tiles + own_k;
      const float inv = (l_tot > 0.f) ? 1.0f / l_tot : 0.f;
#pragma unroll
      for (int db = 0; db < D / 32; db++)
#pragma unroll
        for (int q4 = 0; q4 < 4; q4++) {
          f32x2 a = {o_acc[db][0][4 * q4] * inv, o_acc[db][0][4 * q4 + 1] * inv};
          f32x2 bb = {o_acc[db][0][4 * q4 + 2] * inv, o_acc[db][0][4 * q4 + 3] * inv};
          bf16x2 ha = __builtin_convertvector(a, bf16x2), hb = __builtin_convertvector(bb, bf16x2);
          uint2 st;
          st.x = __builtin_bit_cast(uint32_t, ha);
          st.y = __builtin_bit_cast(uint32_t, hb);
          *(uint2*)(&s_o[n32 * D + ((4 * db + q4) ^ (n32 & (PPR - 1))) * 8 + 4 * G]) = st;
        }
      uint16_t* out_b = c.out + ((CAUSAL ? (size_t)(unsigned)row0 : (size_t)bu * (unsigned)c.W) * (unsigned)c.Hq + kvh * (unsigned)c.g) * D;
#pragma unroll
      for (int i = 0; i < 32 * PPR / 64; i++) {
        const int p = lane + 64 * i, rl = p / PPR, piece = p % PPR, rr = row_w + rl;
        const uint4 v = *(const uint4*)(&s_o[rl * D + (piece ^ (rl & (PPR - 1))) * 8]);
        if (rr < Mb) *(uint4*)(out_b + (uint32_t)((rr + small_div(rr, c.rcp_g) * (c.Hq - c.g)) * D + piece * 8)) = v;
      }
      if (c.lse && G == 0 && r >= 0)
        c.lse[((CAUSAL ? (size_t)(unsigned)row0 : (size_t)bu * (unsigned)c.W) + (unsigned)beam_q) * (unsigned)c.Hq + kvh * (unsigned)c.g + (unsigned)(r - beam_q * c.g)] = (l_tot > 0.f) ? (m + __builtin_amdgcn_logf(l_tot)) * kLn2 : -INFINITY;
    } else {
      // this segment's unnormalised fp32 partial O and (max, sum), as the lanes hold them (see k_attn_merge): every store is a run of whole lines.
      // (Staged through LDS into rows of D floats they took 2.1 us of a unit's 13.5.)
      const int first = mbi * MWG + wave_u * 32, left = min(32, Mb - first);       // the wave's rows
      const size_t row_p = (((size_t)bu * (unsigned)c.nsplit + (unsigned)sp) * (unsigned)c.Hkv + kvh) * (unsigned)c.M + (unsigned)first;
      if (r >= 0) {
        f32x4* part = (f32x4*)(c.part_o + row_p * D) + G * left + n32;
#pragma unroll
        for (int e = 0; e < D / 8; e++) {
          const f32x4 v = {o_acc[e / 4][0][4 * (e % 4)], o_acc[e / 4][0][4 * (e % 4) + 1], o_acc[e / 4][0][4 * (e % 4) + 2], o_acc[e / 4][0][4 * (e % 4) + 3]};
          part[2 * e * left] = v;
        }
        if (G == 0) {
          const f32x2 ml = {(l_tot > 0.f) ? m : -INFINITY, l_tot};
          *(f32x2*)(c.part_ml + (row_p + n32) * 2) = ml;
        }
      }
    }
  }
}

// Merge of the per-segment partials (Section 5.2 merge stage).  They lie as k_beam_attn's lanes hold them: per (request, segment, KV head) its M rows
// in blocks of up to 32, of a block first columns 0..3 of all its rows, then columns 4..7, and so on.  A lane takes four columns of a row; the
// eight rows of eight neighbouring lanes are a line, and the eight lanes of a row write 64 bytes of it.  The (max, sum) pairs
// and the partials of four segments are requested together, so a row waits for memory once per four segments.  Bound: the
// partials' bytes; 4096 rows x 5 segments of 128 (10.5 MB) take 4.3 us (6.7 us with 4-byte loads, one segment at a time).
template <int D>
__global__ void __launch_bounds__(256) k_attn_merge(AttnCtx c) {
  constexpr int RPW = 1024 / D;                            // rows per workgroup, of one (request, KV head) pair
  static_assert(RPW % 8 == 0 && 32 % RPW == 0, "whole lines of one block");
  const unsigned per_pair = ((unsigned)c.M + RPW - 1) / RPW, pair = blockIdx.x / per_pair;
  const int b = (int)(pair / (unsigned)c.Hkv), kvh = (int)(pair - (unsigned)b * (unsigned)c.Hkv);
  const int t = (int)threadIdx.x, piece = (t >> 3) % (D / 4), r = (int)(blockIdx.x - pair * per_pair) * RPW + (t & 7) + 8 * (t / (2 * D));
  if (r >= c.M) return;
  const int left = min(32, c.M - (r & ~31));               // rows of this row's block
  const size_t per_seg = (size_t)c.Hkv * c.M;              // rows of a segment of the request
  const size_t row0 = ((size_t)b * c.nsplit * c.Hkv + kvh) * c.M + r;
  const float* part = c.part_o + (row0 - (r & 31)) * D + 4 * (piece * left + (r & 31));
  float M2 = -INFINITY, L = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int U = 4;
#pragma unroll 1
  for (int s0 = 0; s0 < c.nsplit; s0 += U) {
    f32x2 ml[U];
    f32x4 o[U];
#pragma unroll
    for (int k = 0; k < U; k++) {
      const size_t skip = (size_t)min(s0 + k, c.nsplit - 1) * per_seg;
      ml[k] = *(const f32x2*)(c.part_ml + (row0 + skip) * 2);
      o[k] = *(const f32x4*)(part + skip * D);
    }
    float mx = M2;
#pragma unroll
    for (int k = 0; k < U; k++) {
      if (s0 + k >= c.nsplit) ml[k].y = 0.f;               // (a repeated segment counts nothing)
      if (ml[k].y > 0.f) mx = fmaxf(mx, ml[k].x);
    }
    if (!(mx > -INFINITY)) continue;
    const float alpha = __builtin_amdgcn_exp2f(M2 - mx);
    L *= alpha;
#pragma unroll
    for (int e = 0; e < 4; e++) acc[e] *= alpha;
#pragma unroll
    for (int k = 0; k < U; k++) {
      if (!(ml[k].y > 0.f)) continue;
      const float sc = __builtin_amdgcn_exp2f(ml[k].x - mx);
      L += ml[k].y * sc;
#pragma unroll
      for (int e = 0; e < 4; e++) acc[e] += o[k][e] * sc;
    }
    M2 = mx;
  }
  const float inv = (L > 0.f) ? 1.0f / L : 0.f;
  bf16x4 h;
#pragma unroll
  for (int e = 0; e < 4; e++) h[e] = (__bf16)(acc[e] * inv);
  const int w = (int)((unsigned)r / (unsigned)c.g);
  const size_t row = ((size_t)b * c.W + w) * c.Hq + kvh * c.g + (r - w * c.g);
  *(bf16x4*)(c.out + row * D + 4 * piece) = h;
  if (c.lse && piece == 0) c.lse[row] = (L > 0.f) ? (M2 + __builtin_amdgcn_logf(L)) * kLn2 : -INFINITY;
}

// Requests by decreasing prompt length (ties by index), so that the longest units are dispatched first
// and the tail of a ragged batch is made of short ones.  Rank by counting; B is at most kMaxOrderB.
constexpr int kMaxOrderB = 4096;
__global__ void __launch_bounds__(256) k_attn_order(const int32_t* cu, int B, int32_t* order) {
  __shared__ int s_len[kMaxOrderB];
  for (int i = threadIdx.x; i < B; i += 256) s_len[i] = cu[i + 1] - cu[i];
  __syncthreads();
  for (int i = threadIdx.x; i < B; i += 256) {
    const int li = s_len[i];
    int rank = 0;
    for (int j = 0; j < B; j++) rank += (s_len[j] > li) || (s_len[j] == li && j < i);
    order[rank] = i;
  }
}

// Host-side launch plan, fitted to measured sweeps over (B, L, W) on the MI355X.  8-wave workgroups of 256 query rows stage each
// K/V tile once per 256 rows and win for long prompts once there are at least 256 of them (one per CU); else, workgroups of 128 rows: two of
// 4 waves to a CU, or, where there is at most one per CU, one of 8 waves in two sets that share the prompt (ks = 2: 8 requests of
// 2048 tokens x 128 beams, 256 workgroups, 46.3 -> 41.8 us; 2 x 256 x 16 of head size 64 8.4 -> 7.7).
// Splitting the prompt into L segments costs fp32 partials through memory and the merge kernel.  With fewer workgroups than
// CUs, the number of segments is the one for which this sum is least, in us: for every round of workgroups of an XCD (32 CUs, one or two
// to a CU; a segment of a (request, KV head) pair stays on one XCD) 6 and 1.6 (head size 128) or 1.07 (64) for a tile of each
// set that a segment holds, 3.5 for the merge, and the partials written and read at 3 TB/s (64: 3.5).  Over 48 shapes of 400 to 12000 tokens it is 2 %
// above the best number on average (3.4 % without the rounds and with 4 TB/s): 2 requests of 8000 tokens x 200
// beams, 8 query and 2 KV heads of 64: 29.2 us with 9 segments, whose 36 pairs put 35 workgroups on some XCDs, 20.5 with 8; 4 x 2048 x 128 of 8
// heads of 64 20.9 with 8, 15.9 with 4; one of 800 x 128 of these 13.9, 13.7, 12.5, 11.5, 12.8 with 1 to 5.
// Up to two workgroups per CU are looked at: with one at most, long prompts whose pairs and row blocks are somewhat more than half of 256, or a third, left
// places empty: 9 of 2860-4376 x 195 beams of 16 query and 4 KV heads 97.4 us, now 74.4; 7 x 12959 x 66 178.7, 145.6; 12 of 1504-2443 x 39, 8 heads
// of 64, 23.2, 21.0; of 180 shapes none is more than 2 % slower.
//
// With 256 workgroups of 256 rows or more, 128 rows win nevertheless, us with 128 and 256 rows:
//   where they waste fewer rows of the last block (more than 5 %; 8 % for FP8 codes, which every workgroup widens for itself): 128 requests of
//     100-900 tokens x 200 beams, 32 query and 8 KV heads of 128: 319, 350 (FP8 329, 350); 48 of 512-8192 x 300, 8 heads of 64: 210, 271;
//   for prompts of up to 1024 tokens on average in more than one round: two workgroups to a CU cover each other's queries, own tokens and
//     output, which are 40 % of the life of a unit of 8 tiles: 64 x 512 x 128 96.8, 101.6; 32 x 1024 x 256 149.6, 153.9; 128 x 128 x 256 of
//     16 query and 2 KV heads 93, 103, of 8 and 2 heads of 64 28.3, 32.0.  But 64 x 1500 x 256 425, 421, 32 x 4096 x 256 504, 498, with FP8 codes
//     128 x 512 x 256 385, 373, and where queries and outputs are twice what the Infinity Cache holds 128 x 128 x 256 of 32 heads 223, 216.
struct AttnPlan { int mwg, nsplit, ks; bool many; };       // many: more workgroups than CUs before the choice of 128 rows for their own sake
int g_plan_rows = 0, g_plan_segments = 0;                  // gr_diag_attn_plan: 0 = use the rule below
AttnPlan plan_attn(const gr_attn_params* p, bool kv8) {
  const int g = p->Hq / p->Hkv;
  const int64_t M = (int64_t)p->W * g;
  AttnPlan plan;
  auto wants_sets = [&](const AttnPlan& q) {
    return q.mwg == 128 && p->max_L > KT && (int64_t)p->B * p->Hkv * ((M + 127) / 128) * q.nsplit <= 256 ? 2 : 1;
  };
  if (g_plan_rows) {                                        // a sweep asked for this tiling; keep at least one tile per segment
    const int64_t cap = p->max_L / KT;
    plan.mwg = g_plan_rows;
    plan.nsplit = (int)(g_plan_segments < cap ? g_plan_segments : (cap < 1 ? 1 : cap));
    plan.ks = wants_sets(plan);
    plan.many = (int64_t)p->B * p->Hkv * ((M + plan.mwg - 1) / plan.mwg) * plan.nsplit > 256;
    return plan;
  }
  const int64_t units256 = (int64_t)p->B * p->Hkv * ((M + 255) / 256);
  plan.mwg = (M <= 128 || units256 < 256) ? 128 : 256;     // 256-row workgroups only when they fill the chip by themselves
  const int64_t units = (int64_t)p->B * p->Hkv * ((M + plan.mwg - 1) / plan.mwg);
  plan.nsplit = 1;
  if (units < 256 && p->max_L > 4 * KT) {
    const int64_t want = (512 + units / 2) / units, cap = p->max_L / ((p->d == 64 ? 3 : 4) * KT);      // about two workgroups per CU; at least so many tiles per segment
    const int most = (int)(want < cap ? (want < 16 ? want : 16) : (cap < 16 ? cap : 16));
    const int tiles = (p->max_L + KT - 1) / KT;
    const double partial_us = 2.0 * p->B * p->W * p->Hq * p->d * 4 / (p->d == 64 ? 3.5e6 : 3e6);             // of one segment
    double least = 0;
    for (int n = 1; n <= most; n++) {
      const int ks = units * n <= 256 ? 2 : 1, per_set = ((tiles + n - 1) / n + ks - 1) / ks;
      const int64_t on_xcd = ((int64_t)p->B * p->Hkv * n + 7) / 8 * ((M + 127) / 128), rounds = (on_xcd + 64 / ks - 1) / (64 / ks);
      const double us = (double)rounds * (6.0 + (p->d == 64 ? 1.07 : 1.6) * per_set) + (n > 1 ? 3.5 + partial_us * n : 0.0);
      if (n == 1 || us < least) { least = us; plan.nsplit = n; }
    }
  }
  plan.many = units * plan.nsplit > 256;
  if (plan.mwg == 256) {
    const int64_t rows128 = (M + 127) / 128 * 128, rows256 = (M + 255) / 256 * 256;
    const bool fewer_rows = rows256 * 100 > rows128 * (kv8 ? 108 : 105);
    const bool short_prompts = !kv8 && p->total_L <= (int64_t)p->B * 1024 && units256 > 256 && (int64_t)p->B * p->W * p->Hq * p->d * 4 <= ((int64_t)400 << 20);
    if (fewer_rows || short_prompts) plan.mwg = 128;
  }
  plan.ks = wants_sets(plan);
  return plan;
}

// Ragged batches with more units than CUs are worth ordering by length (measured: 4 % on 128 requests of
// 512..8192 tokens); a uniform batch (total_L == B * max_L) is not touched.  Up to kRankB requests every workgroup finds its own by
// rank (FIND), beyond that a kernel of one workgroup writes the order first: 128 of 40-120 tokens x 30 beams, 32 query and 8 KV
// heads of 128, 36.9 us with that kernel, 33.2 without; 100 of 50-500 x 40, 8 and 2 heads of 64, 16.0, 12.6.
bool attn_wants_order(const gr_attn_params* p, const AttnPlan& plan) {
  return p->B >= 2 && p->B <= kMaxOrderB && p->total_L != (int64_t)p->B * p->max_L && plan.many;
}

}  // namespace

extern "C" gr_status gr_diag_attn_plan(int32_t rows_per_workgroup, int32_t l_segments) {
  if (rows_per_workgroup == 0 && l_segments == 0) { g_plan_rows = g_plan_segments = 0; return GR_OK; }
  if ((rows_per_workgroup != 128 && rows_per_workgroup != 256) || l_segments < 1 || l_segments > 16) return GR_ERR_INVALID_ARG;
  g_plan_rows = rows_per_workgroup; g_plan_segments = l_segments;
  return GR_OK;
}

extern "C" size_t gr_beam_attn_workspace_bytes(const gr_attn_params* p) {
  if (!p || p->B <= 0 || p->W <= 0 || p->Hq <= 0 || p->Hkv <= 0 || p->Hq % p->Hkv) return 0;
  const AttnPlan plan = plan_attn(p, false);               // (what it says about the workspace is the same for FP8 codes)
  size_t need = attn_wants_order(p, plan) ? gr_align256((size_t)p->B * 4) : 0;      // (up to kRankB requests: asked for as ever, and not used)
  if (plan.nsplit > 1) {
    const size_t rows = (size_t)p->B * plan.nsplit * p->W * p->Hq;
    need += gr_align256(rows * p->d * 4) + gr_align256(rows * 8);
  }
  return need;
}

namespace {
gr_status attn_run(const gr_attn_params* p, const int32_t* slot, bool kv8, float k_scale, float v_scale, void* workspace, size_t workspace_bytes,
                   void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!p) return GR_ERR_INVALID_ARG;
  if (kv8 && (!(k_scale > 0.f) || !(k_scale < INFINITY) || !(v_scale > 0.f) || !(v_scale < INFINITY))) return GR_ERR_INVALID_ARG;
  if (p->B <= 0 || p->W <= 0 || p->Hq <= 0 || p->Hkv <= 0 || p->d <= 0 || p->ND < 0 || p->u < 0 || p->u > p->ND)
    return GR_ERR_INVALID_ARG;
  if (p->max_L < 0 || p->total_L < 0 || p->total_L > (int64_t)p->max_L * p->B) return GR_ERR_INVALID_ARG;
  if (!p->q || !p->cu_seqlens || !p->out) return GR_ERR_INVALID_ARG;
  if (p->total_L > 0 && (!p->k_shared || !p->v_shared)) return GR_ERR_INVALID_ARG;
  if (p->u > 0 && (!p->k_unshared || !p->v_unshared)) return GR_ERR_INVALID_ARG;
  if (p->Hq % p->Hkv) return GR_ERR_INVALID_ARG;
  if ((((uintptr_t)p->q | (uintptr_t)p->k_shared | (uintptr_t)p->v_shared | (uintptr_t)p->k_unshared | (uintptr_t)p->v_unshared |
        (uintptr_t)p->out) & 15) || ((uintptr_t)p->cu_seqlens & 3) || ((uintptr_t)p->lse_out & 3) || ((uintptr_t)slot & 3))
    return GR_ERR_INVALID_ARG;                                                          // every tensor is moved in 16-byte pieces
  if (!(p->sm_scale > 0.f) || !(p->sm_scale < INFINITY)) return GR_ERR_INVALID_ARG;   // (also rejects NaN: the largest score is taken before it is scaled)
  if (p->d != 64 && p->d != 128) return GR_ERR_UNSUPPORTED;
  if (p->total_L >= ((int64_t)1 << 31)) return GR_ERR_UNSUPPORTED;
  if ((int64_t)p->max_L * p->Hkv * p->d * 2 >= ((int64_t)1 << 32)) return GR_ERR_UNSUPPORTED;   // one request's K (or V) must fit a buffer descriptor
  const int g = p->Hq / p->Hkv;
  if ((int64_t)p->W * g >= ((int64_t)1 << 22)) return GR_ERR_UNSUPPORTED;      // row indices go through small_div, whose bound is 2^22
  if ((int64_t)p->W * p->Hq * p->d >= ((int64_t)1 << 31) || (int64_t)p->W * p->ND * p->Hkv * p->d >= ((int64_t)1 << 31))
    return GR_ERR_UNSUPPORTED;                                                   // offsets inside one request fit 32 bits

  AttnCtx c;
  c.B = p->B; c.W = p->W; c.Hq = p->Hq; c.Hkv = p->Hkv; c.g = g; c.ND = p->ND; c.u = p->u;
  c.M = p->W * g;
  const AttnPlan plan = plan_attn(p, kv8);
  c.MB = (c.M + plan.mwg - 1) / plan.mwg;
  c.nsplit = plan.nsplit;
  c.n_groups = p->B * p->Hkv * c.nsplit;
  c.rcp_g = 1.0f / (float)g; c.rcp_u = 1.0f / (float)(p->u > 1 ? p->u : 1);
  c.inv_mb = div_inv((uint32_t)c.MB); c.inv_split = div_inv((uint32_t)c.nsplit); c.inv_hkv = div_inv((uint32_t)c.Hkv);
  c.c = p->sm_scale * kLog2e;
  c.k_scale = kv8 ? k_scale : 1.f; c.v_scale = kv8 ? v_scale : 1.f;
  c.q = (const uint16_t*)p->q; c.ks = (const uint16_t*)p->k_shared; c.vs = (const uint16_t*)p->v_shared;
  c.cu = p->cu_seqlens; c.ku = (const uint16_t*)p->k_unshared; c.vu = (const uint16_t*)p->v_unshared;
  c.out = (uint16_t*)p->out; c.lse = p->lse_out;
  c.part_o = nullptr; c.part_ml = nullptr; c.order = nullptr; c.slot = slot; c.rcp_hkv = 0.f;
  const size_t need = gr_beam_attn_workspace_bytes(p);
  const bool ordered = attn_wants_order(p, plan), find = ordered && p->B <= kRankB;       // (these have one set of wavefronts: two are for at most 256 workgroups)
  if (need > 0) {
    if (!workspace || ((uintptr_t)workspace & 255)) return GR_ERR_INVALID_ARG;
    if (workspace_bytes < need) return GR_ERR_WORKSPACE_TOO_SMALL;
    char* ws = (char*)workspace;
    if (ordered && !find) {
      hipLaunchKernelGGL(k_attn_order, dim3(1), dim3(256), 0, stream, p->cu_seqlens, p->B, (int32_t*)ws);
      c.order = (const int32_t*)ws;
    }
    if (ordered) ws += gr_align256((size_t)p->B * 4);
    if (c.nsplit > 1) {
      const size_t rows = (size_t)p->B * c.nsplit * p->W * p->Hq;
      c.part_o = (float*)ws;
      c.part_ml = (float*)(ws + gr_align256(rows * p->d * 4));
    }
  }
  const int64_t groups_padded = ((int64_t)c.n_groups + 7) / 8 * 8;
  const int64_t grid = groups_padded * c.MB;
  if (grid >= ((int64_t)1 << 31)) return GR_ERR_UNSUPPORTED;
  const size_t lds = attn_lds_bytes(p->d, plan.mwg, plan.ks);
#define GR_LAUNCH(...)                                                                                       \
  do {                                                                                                       \
    if (const gr_status st = gr_allow_lds<k_beam_attn<__VA_ARGS__>>(lds)) return st;                         \
    hipLaunchKernelGGL((k_beam_attn<__VA_ARGS__>), dim3((unsigned)grid), dim3(threads), lds, stream, c);     \
  } while (0)
#define GR_LAUNCH_ATTN(DD, NW_)                                                                              \
  do {                                                                                                       \
    if (find) { if (kv8) GR_LAUNCH(DD, 1, NW_, false, true, 1, true); else GR_LAUNCH(DD, 1, NW_, false, false, 1, true); }      \
    else { if (kv8) GR_LAUNCH(DD, 1, NW_, false, true, 1, false); else GR_LAUNCH(DD, 1, NW_, false, false, 1, false); }         \
  } while (0)
#define GR_LAUNCH_SETS(DD)                                                                                   \
  do { if (kv8) GR_LAUNCH(DD, 1, 4, false, true, 2, false); else GR_LAUNCH(DD, 1, 4, false, false, 2, false); } while (0)
  const unsigned threads = plan.mwg == 256 || plan.ks == 2 ? 512 : 256;
  if (p->d == 128) {
    if (plan.mwg == 256) GR_LAUNCH_ATTN(128, 8); else if (plan.ks == 2) GR_LAUNCH_SETS(128); else GR_LAUNCH_ATTN(128, 4);
  } else {
    if (plan.mwg == 256) GR_LAUNCH_ATTN(64, 8); else if (plan.ks == 2) GR_LAUNCH_SETS(64); else GR_LAUNCH_ATTN(64, 4);
  }
#undef GR_LAUNCH_SETS
#undef GR_LAUNCH_ATTN
  if (c.nsplit > 1) {
    const int rpw = 1024 / p->d;                           // rows per workgroup
    const unsigned mgrid = (unsigned)((int64_t)p->B * p->Hkv * ((c.M + rpw - 1) / rpw));
    if (p->d == 128) hipLaunchKernelGGL((k_attn_merge<128>), dim3(mgrid), dim3(256), 0, stream, c);
    else hipLaunchKernelGGL((k_attn_merge<64>), dim3(mgrid), dim3(256), 0, stream, c);
  }
  GR_HIP_TRY(hipGetLastError());
  return GR_OK;
}
}  // namespace

extern "C" gr_status gr_beam_attn(const gr_attn_params* p, void* workspace, size_t workspace_bytes, void* stream) {
  return attn_run(p, nullptr, false, 1.f, 1.f, workspace, workspace_bytes, stream);
}

// The same attention with the own-token caches read through a slot table: nothing is moved between decode steps, the
// table (gr_beam_slot_update) says which row of the request's block holds token t of beam w.
extern "C" gr_status gr_beam_attn_slots(const gr_attn_params* p, const int32_t* slot, void* workspace, size_t workspace_bytes, void* stream) {
  if (!slot) return GR_ERR_INVALID_ARG;
  return attn_run(p, slot, false, 1.f, 1.f, workspace, workspace_bytes, stream);
}

// The same attention over a prompt cache stored as FP8 E4M3 codes with one scale per tensor.
extern "C" gr_status gr_beam_attn_fp8kv(const gr_attn_fp8kv_params* p, void* workspace, size_t workspace_bytes, void* stream) {
  if (!p) return GR_ERR_INVALID_ARG;
  return attn_run(&p->attn, nullptr, true, p->k_scale, p->v_scale, workspace, workspace_bytes, stream);
}

// Causal prompt attention through the same kernel (CAUSAL = true).
extern "C" gr_status gr_prefill_attn(const gr_prefill_params* p, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!p) return GR_ERR_INVALID_ARG;
  if (p->B <= 0 || p->Hq <= 0 || p->Hkv <= 0 || p->d <= 0 || p->Hq % p->Hkv) return GR_ERR_INVALID_ARG;
  if (p->max_L < 0 || p->total_L < 0 || p->total_L > (int64_t)p->max_L * p->B) return GR_ERR_INVALID_ARG;
  if (!p->cu_seqlens) return GR_ERR_INVALID_ARG;
  if (p->total_L > 0 && (!p->q || !p->k || !p->v || !p->out)) return GR_ERR_INVALID_ARG;
  if ((((uintptr_t)p->q | (uintptr_t)p->k | (uintptr_t)p->v | (uintptr_t)p->out) & 15) || ((uintptr_t)p->cu_seqlens & 3) ||
      ((uintptr_t)p->lse_out & 3))
    return GR_ERR_INVALID_ARG;
  if (!(p->sm_scale > 0.f) || !(p->sm_scale < INFINITY)) return GR_ERR_INVALID_ARG;
  if (p->d != 64 && p->d != 128) return GR_ERR_UNSUPPORTED;
  if (p->total_L >= ((int64_t)1 << 31)) return GR_ERR_UNSUPPORTED;
  if ((int64_t)p->max_L * p->Hkv * p->d * 2 >= ((int64_t)1 << 32)) return GR_ERR_UNSUPPORTED;   // one request's K (or V) must fit a buffer descriptor
  const int g = p->Hq / p->Hkv;
  if ((int64_t)p->max_L * g >= ((int64_t)1 << 22)) return GR_ERR_UNSUPPORTED;                   // row indices go through small_div, whose bound is 2^22
  if ((int64_t)p->max_L * p->Hq * p->d >= ((int64_t)1 << 31)) return GR_ERR_UNSUPPORTED;        // offsets inside one request fit 32 bits
  if (p->total_L == 0 || p->max_L == 0) return GR_OK;

  AttnCtx c;
  c.B = p->B; c.W = 0; c.Hq = p->Hq; c.Hkv = p->Hkv; c.g = g; c.ND = 0; c.u = 0;
  c.M = p->max_L * g;                                        // the longest request's rows size the grid
  // 128 rows, two workgroups to a CU: one computes while the other waits for its queries or stores its output, which is most of
  // the life of a block of a short prompt.  256 rows stage every K/V tile half as often, which counts for long prompts of head size
  // 128, and for shorter ones where an XCD has one or two (prompt, KV head) pairs and 1.25 to 2 such blocks per CU (counted by
  // the tokens there are), so that the few heaviest blocks are what the call waits for.  us with 256 and 128 rows (32 query and 8 KV heads of 128 unless noted):
  // 1 x 1024 tokens 29.7, 22.3; 16 prompts of 62-512 38.2, 33.9; 4 x 1024 56, 49; 1 x 2048 55.1, 47.6; 16 x 2048 596, 579; 4 of
  // 190-1500 with 16 query and 4 KV heads 43.6, 36.7; but 1 x 4096 128, 138 and 8 of 1024-8192 1674, 1700; 2 x 2048 74.5, 77.9 and 1 to 4 x 2048 of 16 query and 2 KV heads 69-75, 75-79.  8 heads of 64:
  // 1 x 4096 71, 50; 16 x 4096 383, 344.
  const int64_t pairs = (int64_t)p->B * p->Hkv, rows_per_xcd = p->total_L * p->Hq / (pairs < 8 ? pairs : 8);
  const bool heavy = p->max_L > 2048 || (pairs <= 16 && rows_per_xcd > 40 * 256 && rows_per_xcd <= 64 * 256);
  const int mwg = p->d == 64 || !heavy || c.M <= 128 ? 128 : 256;
  c.MB = (c.M + mwg - 1) / mwg;
  c.nsplit = 1;
  c.n_groups = p->B * p->Hkv;
  c.rcp_g = 1.0f / (float)g; c.rcp_u = 1.f;
  c.inv_mb = div_inv((uint32_t)c.MB); c.inv_split = div_inv(1); c.inv_hkv = div_inv((uint32_t)c.Hkv);
  c.c = p->sm_scale * kLog2e;
  c.k_scale = 1.f; c.v_scale = 1.f;
  c.q = (const uint16_t*)p->q; c.ks = (const uint16_t*)p->k; c.vs = (const uint16_t*)p->v;
  c.cu = p->cu_seqlens; c.ku = nullptr; c.vu = nullptr;
  c.out = (uint16_t*)p->out; c.lse = p->lse_out;
  c.part_o = nullptr; c.part_ml = nullptr; c.order = nullptr; c.slot = nullptr;
  const int64_t groups_padded = ((int64_t)c.n_groups + 7) / 8 * 8;
  const int64_t grid = groups_padded * c.MB;
  // Row blocks dealt heaviest first over all pairs of an XCD: the blocks that prompts shorter than the longest do not have come last
  // (pair by pair they come first, and hold a place while they find that out), and the call ends with light blocks.  Against that stand
  // 0.4 us at the start of every block and K/V that is read again when it has left the L2.  So: where not all blocks have a place at once,
  //   an XCD's pairs times the rows of a token in each are at most 48 (head size 128) or 128 (64), or more, up to 64 with head size 128,
  //     where the prompts are on average shorter than two thirds of the longest, and
  //   the K/V of an XCD's pairs times the rows of a token take at most 24 MiB: 64 x 4500 tokens of 8 heads of 64 1647 us pair by pair, 2266 by
  //     weight, 32 x 3000 with 32 and 8 heads 1397, 1532, 48 of 960-1200 with 8 heads of 128 162, 188; but 32 x 3000 with 8 heads 405, 387.
  // 2400 shapes of 250 to 11000 tokens: where the rule deals by weight that takes 0.94 of pair by pair in the mean (head size 64 0.91, 128
  // 0.95), and in one of 90 more than 1.06.  us pair by pair, by weight: 16 prompts of 60-700 tokens, 32 query and 8 KV heads of 128, 44.7, 41.6; 8 of
  // 200-2000 136.7, 133; 10 of 300-1000 57.5, 55.8; 40 of 100-900, 8 and 2 heads, 47.2, 44.1; 8 heads of 64: 12 of 100-1000 18.9, 15.1, 16 of
  // 1000-4000 153, 140.  But 32 of 100-600, 32 and 8 heads of 128, 69, 78; 16 x 600 70, 74; 64 of 100-600, 16 and 2 heads, 68, 71.
  const int64_t rows_of_token = groups_padded / 8 * g;
  const bool uneven = p->total_L * 3 < (int64_t)p->B * p->max_L * 2;
  const bool by_weight = groups_padded <= 512 && grid > 512 && mwg == 128 && p->total_L * p->Hq * p->d <= (int64_t)48 << 20 &&
                         (rows_of_token <= (p->d == 64 ? 128 : 48) || (uneven && (p->d == 64 || rows_of_token <= 64)));
  c.rcp_hkv = 1.0f / (float)p->Hkv * 1.00001f;
  if (grid >= ((int64_t)1 << 31)) return GR_ERR_UNSUPPORTED;
  const size_t lds = attn_lds_bytes(p->d, mwg, 1);
  const unsigned threads = 2 * mwg;
  if (p->d == 128) {
    if (mwg == 256) GR_LAUNCH(128, 1, 8, true, false, 1, false);
    else if (by_weight) GR_LAUNCH(128, 1, 4, true, false, 1, true);
    else GR_LAUNCH(128, 1, 4, true, false, 1, false);
  } else {
    if (by_weight) GR_LAUNCH(64, 1, 4, true, false, 1, true); else GR_LAUNCH(64, 1, 4, true, false, 1, false);
  }
#undef GR_LAUNCH
  GR_HIP_TRY(hipGetLastError());
  return GR_OK;
}
