// gr_item_mask_build: valid-item mask blob from the sorted item table (paper Section 6.1).
//
// A row that starts a new first token contributes the row offsets of that token; a row that starts a new
// (t1,t2) pair contributes one entry of the sparse pair list (the CSR form of level 1, which is also the
// row index of level 2).  The first pass over the table counts the pairs of every block of rows, the
// second one places them; the two bit levels are then made from the finished pair list, one workgroup per first token.
//
// Bound: memory (the table twice, the second time mostly from the Infinity Cache, and what is written once): 10 M items at
// V = 8192 take 25 us (count: 4.7 TB/s) + 35 us (scatter: 230 MB) + 11 us (bits), against 44 + 5 (scan) + 222 us with rows
// taken in runs per thread (96-byte strides between lanes) and bits set by atomics in memory.
// Both passes bring a block's rows in with whole-line 16-byte loads through LDS and take rows lane by lane, so
// that every store is contiguous over the wavefront; a row's place in the pair list is a ballot rank.
#include <mutex>
#include "gr_internal.hpp"

namespace {

constexpr int kBuildThreads = 256;
constexpr int kRowsPerThread = 8;
constexpr int kRowsPerBlock = kBuildThreads * kRowsPerThread;
constexpr int kBuildWaves = kBuildThreads / 64;
constexpr int kBitThreads = 256;
// With more blocks of rows than this their counts are scanned by a kernel of its own (5 us and a launch at any size);
// below, every workgroup of the second pass adds up the counts in front of it (at most 32 KB of L2 reads, about 2 us).
constexpr int kSumBlocks = 8192;

// where the parts of the blob lie
struct MaskParts {
  gr_mask_header* head;
  uint32_t* l0;
  uint32_t* l1;
  int32_t* off1;
  int32_t* pair_off;
  int32_t* pair_t2;
  int32_t* pair_row;
  int32_t* t3;
};

// The block's rows as they lie in the table: s_rows[3 + 3 r + c] = column c of the block's row r; s_rows[0..2] = the row in
// front of the block (of the first block: tokens -1, which no valid row equals and every valid row follows).
__device__ __forceinline__ int stage_rows(const int32_t* items, int64_t n, int32_t* s_rows) {
  const int64_t first = (int64_t)blockIdx.x * kRowsPerBlock;
  const int rows = (int)(n - first < kRowsPerBlock ? n - first : kRowsPerBlock);
  const int32_t* src = items + 3 * first;
  const int ints = 3 * rows, t = threadIdx.x;
  if (((uintptr_t)src & 15) == 0) {                       // (blocks start at multiples of 24 KiB of the table)
    const int quads = ints >> 2;
    int4 q[3 * kRowsPerBlock / 4 / kBuildThreads];
#pragma unroll
    for (int k = 0; k < 3 * kRowsPerBlock / 4 / kBuildThreads; k++)
      if (t + k * kBuildThreads < quads) q[k] = ((const int4*)src)[t + k * kBuildThreads];
#pragma unroll
    for (int k = 0; k < 3 * kRowsPerBlock / 4 / kBuildThreads; k++) {
      const int i = t + k * kBuildThreads;
      if (i < quads) { int32_t* d = s_rows + 3 + 4 * i; d[0] = q[k].x; d[1] = q[k].y; d[2] = q[k].z; d[3] = q[k].w; }
    }
    const int i = 4 * quads + t;
    if (i < ints) s_rows[3 + i] = src[i];
  } else {
    for (int i = t; i < ints; i += kBuildThreads) s_rows[3 + i] = src[i];
  }
  if (t < 3) s_rows[t] = first > 0 ? src[t - 3] : -1;
  __syncthreads();
  return rows;
}

// row r of the block against the row in front of it; false when the table is not valid there
__device__ __forceinline__ bool row_ok_and_flags(const int32_t* s_rows, int r, int V, bool* new_t1, bool* new_pair) {
  const int32_t* p = s_rows + 3 * r;
  const int32_t pa = p[0], pb = p[1], pc = p[2], a = p[3], b = p[4], c = p[5];
  const bool ok = a >= 0 && a < V && b >= 0 && b < V && c >= 0 && c < V;
  // strictly increasing lexicographic order
  const bool gt = (a > pa) || (a == pa && (b > pb || (b == pb && c > pc)));
  *new_t1 = (a != pa);
  *new_pair = (a != pa) || (b != pb);
  return ok && gt;
}

// pass 1: validate rows, count pair starts per block; the sign bit of a block's count tells that its rows are not valid (so that no word
// has to be cleared before: a launch of its own, 5 us).  The first block also writes the header.
constexpr int32_t kBadBlock = (int32_t)0x80000000;
__global__ void __launch_bounds__(kBuildThreads) k_mask_count(const int32_t* items, int64_t n, int V, int32_t* block_counts, gr_mask_header* head, gr_mask_header h) {
  __shared__ int32_t s_rows[3 * kRowsPerBlock + 3];
  __shared__ int s_cnt[kBuildWaves];
  const int rows = stage_rows(items, n, s_rows);
  int cnt = 0;
  bool bad = false;
#pragma unroll
  for (int k = 0; k < kRowsPerThread; k++) {
    const int r = k * kBuildThreads + (int)threadIdx.x;
    bool t1 = false, pr = false;
    if (r < rows && !row_ok_and_flags(s_rows, r, V, &t1, &pr)) bad = true;
    cnt += __popcll(__ballot(pr));
  }
  if (__any(bad)) cnt |= kBadBlock;
  if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    int sum = 0, sign = 0;
#pragma unroll
    for (int w = 0; w < kBuildWaves; w++) { sum += s_cnt[w] & ~kBadBlock; sign |= s_cnt[w] & kBadBlock; }
    block_counts[blockIdx.x] = sum | sign;
    if (blockIdx.x == 0) *head = h;
  }
}

// Exclusive scan of the per-block counts by a single workgroup (large tables only, see kSumBlocks).  The sign bit of a sum tells that some
// block up to this one is not valid.
__global__ void __launch_bounds__(1024) k_mask_scan(int32_t* counts, int nblocks) {
  __shared__ int s_part[1024];
  __shared__ int s_first_bad;
  const int t = threadIdx.x;
  const int per = (nblocks + 1023) / 1024;
  const int lo = min(nblocks, t * per), hi = min(nblocks, lo + per);
  if (t == 0) s_first_bad = nblocks;
  __syncthreads();
  int sum = 0;
  for (int i = lo; i < hi; i++) {
    sum += counts[i] & ~kBadBlock;
    if (counts[i] < 0) atomicMin(&s_first_bad, i);
  }
  s_part[t] = sum;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {   // Hillis-Steele inclusive scan
    int v = (t >= o) ? s_part[t - o] : 0;
    __syncthreads();
    s_part[t] += v;
    __syncthreads();
  }
  int run = s_part[t] - sum;
  for (int i = lo; i < hi; i++) { int c = counts[i] & ~kBadBlock; counts[i] = run | (i >= s_first_bad ? kBadBlock : 0); run += c; }
}

// pass 2: scatter pairs, fill offsets, copy the third column
__global__ void __launch_bounds__(kBuildThreads) k_mask_scatter(const int32_t* items, int64_t n, int V, const int32_t* block_counts,
                                                                bool scanned, MaskParts m, int32_t* err, int32_t* host_err) {
  __shared__ int32_t s_rows[3 * kRowsPerBlock + 3];
  __shared__ int s_base[kBuildWaves], s_bad[kBuildWaves];
  __shared__ int s_cnt[kRowsPerThread * kBuildWaves + 1];  // pair starts of every 64 consecutive rows, then their exclusive prefix and sum
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  // pairs of all blocks in front of this one, and whether one of these or this one is not valid
  int part = 0, sign = 0;
  if (scanned) {
    if (t == 0) { sign = block_counts[blockIdx.x]; part = sign & ~kBadBlock; }
  } else {
    for (int i = 4 * t; i <= (int)blockIdx.x; i += 4 * kBuildThreads) {
      const int4 q = *(const int4*)(block_counts + i);     // (reads at most three counts past the last: inside the workspace)
      const int left = (int)blockIdx.x - i;
      sign |= q.x | (left > 0 ? q.y : 0) | (left > 1 ? q.z : 0) | (left > 2 ? q.w : 0);
      part += (left > 0 ? q.x & ~kBadBlock : 0) + (left > 1 ? q.y & ~kBadBlock : 0) + (left > 2 ? q.z & ~kBadBlock : 0) + (left > 3 ? q.w & ~kBadBlock : 0);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);
  const bool bad = __any(sign < 0);
  if (lane == 0) { s_base[wave] = part; s_bad[wave] = bad; }
  const int rows = stage_rows(items, n, s_rows);           // (its barrier publishes s_base)
  int base = 0, stop = 0;
#pragma unroll
  for (int w = 0; w < kBuildWaves; w++) { base += s_base[w]; stop |= s_bad[w]; }
  const int64_t first = (int64_t)blockIdx.x * kRowsPerBlock;
  if (t == 0 && first + rows == n) {                       // (the last block knows of all)
    *err = stop;
    if (host_err) *host_err = stop;
  }
  if (stop) return;   // (what lies behind bad rows could index out of bounds; the host reports GR_ERR_BAD_TABLE)
  bool nt1[kRowsPerThread], npr[kRowsPerThread];
  int rank[kRowsPerThread];
#pragma unroll
  for (int k = 0; k < kRowsPerThread; k++) {
    const int r = k * kBuildThreads + t;
    nt1[k] = npr[k] = false;
    if (r < rows) row_ok_and_flags(s_rows, r, V, &nt1[k], &npr[k]);
    const uint64_t starts = __ballot(npr[k]);
    rank[k] = __popcll(starts & (((uint64_t)1 << lane) - 1));
    if (lane == 0) s_cnt[k * kBuildWaves + wave] = __popcll(starts);
  }
  __syncthreads();
  if (wave == 0) {
    constexpr int N = kRowsPerThread * kBuildWaves;
    const int v = lane < N ? s_cnt[lane] : 0;
    int incl = v;
#pragma unroll
    for (int o = 1; o < N; o <<= 1) { const int x = __shfl_up(incl, o, 64); if (lane >= o) incl += x; }
    if (lane < N) s_cnt[lane] = incl - v;
    if (lane == N - 1) s_cnt[N] = incl;
  }
  __syncthreads();
  auto fill = [&](int tok0, int tok1, int from, int step, int row, int p) {
    for (int tok = tok0 + from; tok <= tok1; tok += step) { m.off1[tok] = row; m.pair_off[tok] = p; }
  };
#pragma unroll
  for (int k = 0; k < kRowsPerThread; k++) {
    const int r = k * kBuildThreads + t;
    const int p = base + s_cnt[k * kBuildWaves + wave] + rank[k];
    const int i = (int)(first + r);
    int tok0 = 0, tok1 = -1;                               // first tokens whose rows begin here
    if (r < rows) {
      m.t3[i] = s_rows[3 + 3 * r + 2];
      if (npr[k]) { m.pair_t2[p] = s_rows[3 + 3 * r + 1]; m.pair_row[p] = i; }
      if (nt1[k]) { tok0 = s_rows[3 * r] + 1; tok1 = s_rows[3 + 3 * r]; }
    }
    // few tokens are skipped as a rule; where many are, the wavefront writes them together
    const bool many = tok1 - tok0 >= 8;
    if (!many) fill(tok0, tok1, 0, 1, i, p);
    for (uint64_t todo = __ballot(many); todo; todo &= todo - 1) {
      const int l = __ffsll((unsigned long long)todo) - 1;
      fill(__shfl(tok0, l, 64), __shfl(tok1, l, 64), lane, 64, __shfl(i, l, 64), __shfl(p, l, 64));
    }
  }
  if (first + rows == n) {                                 // the last block closes the offsets
    const int total_pairs = base + s_cnt[kRowsPerThread * kBuildWaves];
    fill(s_rows[3 * rows] + 1, V, t, kBuildThreads, (int)n, total_pairs);
    if (t == 0) {
      m.pair_row[total_pairs] = (int32_t)n;
      m.head->n_pairs = total_pairs;
    }
  }
}

// pass 3: the bits.  The workgroup of first token t1 marks its second tokens in LDS, one byte each, and writes the row of
// level 1 once, whole (so the levels need no clearing, and no bit is set by an atomic operation: neighbours of the sorted list
// fall in one word, where the LDS would take them one after another).  Every 32nd workgroup also writes the word of level 0
// that its token begins.
__global__ void __launch_bounds__(kBitThreads) k_mask_bits(int V, MaskParts m, const int32_t* err) {
  extern __shared__ __attribute__((aligned(16))) uint4 s_mark[];        // a byte per token, `words` x 32
  const int words = (V + 31) >> 5, t1 = blockIdx.x, t = threadIdx.x;
  const int bad = *err, lo = m.pair_off[t1], hi = m.pair_off[t1 + 1];
  if (bad) return;
  constexpr int U = 4;
  int v[U];
  auto request = [&](int i0) {
#pragma unroll
    for (int k = 0; k < U; k++) v[k] = m.pair_t2[min(i0 + k * kBitThreads, hi - 1)];      // (a pair marked twice is marked)
  };
  if (lo + t < hi) request(lo + t);
  for (int i = t; i < 2 * words; i += kBitThreads) s_mark[i] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  for (int i0 = lo + t; i0 < hi; i0 += U * kBitThreads) {
#pragma unroll
    for (int k = 0; k < U; k++) ((uint8_t*)s_mark)[v[k]] = 1;
    if (i0 + U * kBitThreads < hi) request(i0 + U * kBitThreads);
  }
  __syncthreads();
  uint32_t* row = m.l1 + (size_t)t1 * words;
  for (int i = t; i < words; i += kBitThreads) {
    const uint4 a = s_mark[2 * i], b = s_mark[2 * i + 1];
    const uint32_t q[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t bits = 0;
#pragma unroll
    for (int k = 0; k < 8; k++) bits |= ((q[k] * 0x10204080u) >> 28) << (4 * k);     // bytes 0..3 of q -> bits 0..3
    row[i] = bits;
  }
  if ((t1 & 31) == 0 && t < 64) {
    const int tok = min(t1 + t, V - 1);
    const uint64_t some = __ballot(t < 32 && t1 + t < V && m.pair_off[tok + 1] > m.pair_off[tok]);
    if (t == 0) m.l0[t1 >> 5] = (uint32_t)some;
  }
}

// Words of host memory that the last block writes its verdict to, so that the call's end is one wait for the stream (a copy of four
// bytes to pageable memory is a kernel, a staging buffer and a second wait: 12 us of a call).  One page for the process, until it ends;
// a word belongs to one call at a time.  A call that finds none free copies the verdict from its workspace instead.
class VerdictWords {
 public:
  int take() {                                             // a word's number, or -1
    std::call_once(once_, [this] {
      void* p = nullptr;
      if (hipHostMalloc(&p, kWords * kStride, hipHostMallocPortable | hipHostMallocMapped | hipHostMallocCoherent) == hipSuccess) host_ = (char*)p;
      else (void)hipGetLastError();
    });
    if (!host_) return -1;
    uint64_t used = used_.load(std::memory_order_relaxed);
    while (~used) {
      const int w = __builtin_ctzll(~used);
      if (used_.compare_exchange_weak(used, used | (uint64_t)1 << w, std::memory_order_acquire)) return w;
    }
    return -1;
  }
  void give_back(int w) { used_.fetch_and(~((uint64_t)1 << w), std::memory_order_release); }
  volatile int32_t* host(int w) const { return (volatile int32_t*)(host_ + w * kStride); }
  int32_t* device(int w) const {                           // on the current device
    void* d = nullptr;
    if (hipHostGetDevicePointer(&d, host_ + w * kStride, 0) == hipSuccess) return (int32_t*)d;
    (void)hipGetLastError();
    return nullptr;
  }

 private:
  static constexpr int kWords = 64, kStride = 64;
  std::once_flag once_;
  std::atomic<uint64_t> used_{0};
  char* host_ = nullptr;
};
VerdictWords g_verdicts;

}  // namespace

extern "C" size_t gr_item_mask_bytes(int64_t n_items, int32_t depth, int32_t V) {
  if (n_items <= 0 || depth != 3 || V <= 0 || V > 32768) return 0;
  gr_mask_header h;
  gr_mask_layout(n_items, V, &h);
  return (size_t)h.total_bytes;
}

extern "C" size_t gr_item_mask_build_workspace_bytes(int64_t n_items, int32_t depth, int32_t V) {
  if (n_items <= 0 || depth != 3 || V <= 0) return 0;
  return 256 + gr_align256((size_t)((n_items + kRowsPerBlock - 1) / kRowsPerBlock) * 4);
}

extern "C" gr_status gr_item_mask_build(const int32_t* items_sorted, int64_t n_items, int32_t depth, int32_t V, void* mask_out,
                                        size_t mask_bytes, void* workspace, size_t workspace_bytes, void* stream_) {
  hipStream_t stream = (hipStream_t)stream_;
  if (!items_sorted || !mask_out || !workspace || n_items <= 0 || V <= 0) return GR_ERR_INVALID_ARG;
  if (depth != 3 || V > 32768 || n_items >= ((int64_t)1 << 31)) return GR_ERR_UNSUPPORTED;
  if (((uintptr_t)mask_out & 255) || ((uintptr_t)workspace & 255)) return GR_ERR_INVALID_ARG;
  gr_mask_header h;
  gr_mask_layout(n_items, V, &h);
  if (mask_bytes < (size_t)h.total_bytes) return GR_ERR_INVALID_ARG;
  if (workspace_bytes < gr_item_mask_build_workspace_bytes(n_items, depth, V)) return GR_ERR_WORKSPACE_TOO_SMALL;

  char* blob = (char*)mask_out;
  int32_t* err = (int32_t*)workspace;
  int32_t* counts = (int32_t*)((char*)workspace + 256);
  const int nblocks = (int)((n_items + kRowsPerBlock - 1) / kRowsPerBlock);
  const bool scanned = nblocks > kSumBlocks;
  MaskParts m;
  m.head = (gr_mask_header*)blob;
  m.l0 = (uint32_t*)(blob + h.off_l0);
  m.l1 = (uint32_t*)(blob + h.off_l1);
  m.off1 = (int32_t*)(blob + h.off_off1);
  m.pair_off = (int32_t*)(blob + h.off_pair_off);
  m.pair_t2 = (int32_t*)(blob + h.off_pair_t2);
  m.pair_row = (int32_t*)(blob + h.off_pair_row);
  m.t3 = (int32_t*)(blob + h.off_t3);

  const int word = g_verdicts.take();
  int32_t* host_err = word >= 0 ? g_verdicts.device(word) : nullptr;
  hipLaunchKernelGGL(k_mask_count, dim3(nblocks), dim3(kBuildThreads), 0, stream, items_sorted, n_items, V, counts, m.head, h);
  if (scanned) hipLaunchKernelGGL(k_mask_scan, dim3(1), dim3(1024), 0, stream, counts, nblocks);
  hipLaunchKernelGGL(k_mask_scatter, dim3(nblocks), dim3(kBuildThreads), 0, stream, items_sorted, n_items, V, counts, scanned, m, err, host_err);
  hipLaunchKernelGGL(k_mask_bits, dim3(V), dim3(kBitThreads), (size_t)h.words * 32, stream, V, m, err);
  hipError_t hip = hipGetLastError();
  int32_t verdict = 0;
  if (hip == hipSuccess && !host_err) hip = hipMemcpyAsync(&verdict, err, sizeof(int32_t), hipMemcpyDeviceToHost, stream);
  const hipError_t waited = hipStreamSynchronize(stream);  // (also after a failed launch: no kernel of this call writes the word later)
  if (host_err) verdict = *g_verdicts.host(word);
  if (word >= 0) g_verdicts.give_back(word);
  if (hip != hipSuccess || waited != hipSuccess) return GR_ERR_HIP;
  return verdict ? GR_ERR_BAD_TABLE : GR_OK;
}
