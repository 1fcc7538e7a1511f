// Salts (HMAC-SHA256) and chained block hashes on gfx950.
//
// Paper: per-principal salt sigma_p = HMAC_K(principal_id) (Sec. 4.1); block
// hashes chained h_j = H(h_{j-1}, tokens_j) (Sec. 2.1) with the salt at the
// root (Sec. 4.1) or at the divergence boundary k (Sec. 4.2).
//
// Execution model.  A chain is a strict sequence of SHA-256 compressions
// (h_j needs h_{j-1}), so all parallelism comes from the batch.  Two kernels:
//   * k_chains_lp: four waves per 64 requests, two lanes per request for
//     the rounds on two of them and for the message schedule on the other
//     two, which shortens every chain; for batches of at most two workgroups
//     per CU;
//   * k_chains_mixed: larger batches, ordered longest first: the longest
//     requests on lane-pair workgroups, the others on one lane each (a wave
//     advances 64 chains), so that the lanes of a wave carry similar block
//     counts and long chains start early.
//
// Per block a lane issues two compressions: (IV; h_{j-1} || T_j[0..7]) and
// (state; T_j[8..15] || padding of a 96-byte message).  Three cases leave
// that pattern:
//   * the first block of an unsalted chain: a 64-byte message T_0, whose
//     second compression is the constant padding block;
//   * the boundary block k > 0: a 128-byte message sigma || h_{k-1} || T_k,
//     three compressions, which its request alone spends further iterations on;
//   * the root-salted first block is the usual pattern with sigma in place of
//     h_{-1}.
//
// Token ids are little-endian int32 (4 bytes each, no separator); SHA-256
// words are big-endian, so each token word is byte-swapped on load.  Digests
// are stored as their big-endian byte serialisation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <thread>
#include <tuple>
#include <vector>

#include "common.h"
#include "sha256_cdna4.h"

namespace kvgov {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(4)));


// ---------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ void load_raw(const int32_t *p, u32x4 raw[4]) {
  const u32x4 *q = reinterpret_cast<const u32x4 *>(p);
#pragma unroll
  for (int i = 0; i < 4; ++i) raw[i] = q[i];
}

// Token prefetch.  T <- the block held in raw (block j), then raw <- block
// j + 1 (block j again when j is the last, so that the load is
// unconditional).  The scheduling barriers pin the load right after the last
// read of raw: it then writes raw's registers in place, and its latency hides
// behind a block's compressions.  (Issued before those reads, or under a
// condition, the load lands in temporaries that are copied into raw at once,
// which waits for it.)  Callers take the next block before storing the
// current digest: a wait for the load must not also wait for a store issued
// after it.
__device__ __forceinline__ void swap_block(const u32x4 raw[4], uint32_t T[16]);
__device__ __forceinline__ void take_block(u32x4 raw[4], uint32_t T[16], const int32_t *tp,
                                           int64_t j, int64_t nf) {
  swap_block(raw, T);
  __builtin_amdgcn_sched_barrier(0);
  load_raw(tp + 16 * (j + 1 < nf ? j + 1 : j), raw);
  __builtin_amdgcn_sched_barrier(0);
}

__device__ __forceinline__ void swap_block(const u32x4 raw[4], uint32_t T[16]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    T[4 * i + 0] = bswap(raw[i].x);
    T[4 * i + 1] = bswap(raw[i].y);
    T[4 * i + 2] = bswap(raw[i].z);
    T[4 * i + 3] = bswap(raw[i].w);
  }
}

__device__ __forceinline__ void store_digest(uint8_t *dst, const uint32_t H[8]) {
  u32x4 *q = reinterpret_cast<u32x4 *>(dst);
  q[0] = u32x4{bswap(H[0]), bswap(H[1]), bswap(H[2]), bswap(H[3])};
  q[1] = u32x4{bswap(H[4]), bswap(H[5]), bswap(H[6]), bswap(H[7])};
}

__device__ __forceinline__ void load_digest(const uint8_t *src, uint32_t H[8]) {
  const u32x4 *q = reinterpret_cast<const u32x4 *>(src);
  const u32x4 a = q[0], b = q[1];
  H[0] = bswap(a.x); H[1] = bswap(a.y); H[2] = bswap(a.z); H[3] = bswap(a.w);
  H[4] = bswap(b.x); H[5] = bswap(b.y); H[6] = bswap(b.z); H[7] = bswap(b.w);
}

// ---------------------------------------------------------------------------
// a1: salts
// ---------------------------------------------------------------------------

struct SaltArgs {
  uint32_t inner[8], outer[8];  // states after K ^ ipad and K ^ opad
  const uint8_t *ids;
  int32_t id_len;
  int32_t P;
  uint8_t *salts;
};

typedef uint32_t u32_any __attribute__((aligned(1)));  // a dword at any byte

// sigma_p = H((K ^ opad) || H((K ^ ipad) || id_p))   (RFC 2104 over SHA-256)
// The first compression of either hash takes only K, so the states after
// them are the caller's (two compressions on the host): a salt is then the
// id's blocks and one more, in sequence, and a launch of one wave is
// nothing but that sequence.  64 ids of 32 bytes: 17.9 us with all four
// compressions here and the ids read by bytes, 9.2 us so.
__global__ __launch_bounds__(64) void k_salts(SaltArgs a) {
  const int p = blockIdx.x * kWave + threadIdx.x;
  if (p >= a.P) return;
  const uint8_t *id = a.ids + (int64_t)p * a.id_len;
  const int L = a.id_len;
  uint32_t st[8], w[16];
#pragma unroll
  for (int i = 0; i < 8; ++i) st[i] = a.inner[i];
  const int nblk = (L + 9 + 63) / 64;  // id, 0x80, 64-bit length
  for (int blk = 0; blk < nblk; ++blk) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int at = blk * 64 + 4 * i;
      uint32_t word = 0;
      if (at + 4 <= L) {
        word = bswap(*reinterpret_cast<const u32_any *>(id + at));
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int pos = at + q;
          const uint32_t byte = pos < L ? (uint32_t)id[pos] : (pos == L ? 0x80u : 0u);
          word = (word << 8) | byte;
        }
      }
      w[i] = word;
    }
    if (blk == nblk - 1) {
      const uint64_t bits = (uint64_t)(64 + L) * 8u;
      w[14] = (uint32_t)(bits >> 32);
      w[15] = (uint32_t)bits;
    }
    compress(st, w);
  }
  uint32_t o[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    o[i] = a.outer[i];
    w[i] = st[i];
  }
  w[8] = 0x80000000u;
#pragma unroll
  for (int i = 9; i < 15; ++i) w[i] = 0;
  w[15] = (64 + 32) * 8;
  compress(o, w);
  store_digest(a.salts + (int64_t)p * 32, o);
}

// ---------------------------------------------------------------------------
// output layout: blk_offsets = exclusive prefix sum of len // 16 (minus the
// start block when resuming)
// ---------------------------------------------------------------------------

constexpr int kScanThreads = 1024;
constexpr int kScanItems = 4;  // consecutive requests per thread and step
constexpr int kScanStep = kScanThreads * kScanItems;

// blocks hashed for request r: full blocks from start[r] on (start NULL: 0)
__device__ __forceinline__ int64_t req_blocks(const int64_t *tok_offsets, const int32_t *start,
                                              int64_t r, int32_t *status) {
  const int64_t len = tok_offsets[r + 1] - tok_offsets[r];
  const int64_t j0 = start ? start[r] : 0;
  if (len < 0 || j0 < 0 || j0 > (len >> 4)) {
    latch(status, KVGOV_E_OFFSETS);
    return 0;
  }
  return (len >> 4) - j0;
}

// inclusive scan across the threads of a workgroup; *total is their sum
__device__ __forceinline__ int64_t block_inclusive_scan(int64_t v, int64_t *lds_waves,
                                                        int64_t *total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int64_t u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  if (lane == 63) lds_waves[wid] = v;
  __syncthreads();
  int64_t before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kScanThreads / 64; ++i) {
    before += i < wid ? lds_waves[i] : 0;
    all += lds_waves[i];
  }
  __syncthreads();
  *total = all;
  return v + before;
}

// blocks of requests [r0, r1), on every thread
__device__ __forceinline__ int64_t sum_blocks(const int64_t *tok_offsets, const int32_t *start,
                                              int64_t r0, int64_t r1, int32_t *status,
                                              int64_t *lds_waves) {
  int64_t s = 0, total;
#pragma unroll 8
  for (int64_t r = r0 + threadIdx.x; r < r1; r += kScanThreads)
    s += req_blocks(tok_offsets, start, r, status);
  block_inclusive_scan(s, lds_waves, &total);
  return total;
}

__global__ __launch_bounds__(kScanThreads) void k_blk_partial(const int64_t *tok_offsets,
                                                              const int32_t *start, int32_t n,
                                                              int64_t tile, int64_t *partial,
                                                              int32_t *status) {
  __shared__ int64_t lds[kScanThreads / 64];
  const int64_t r0 = (int64_t)blockIdx.x * tile, r1 = r0 + tile < n ? r0 + tile : n;
  const int64_t s = sum_blocks(tok_offsets, start, r0, r1, status, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// The offsets of `tile` requests per workgroup.  What lies before them is
// summed by the workgroup itself: from k_blk_partial's sums, or, for batches
// small enough that this takes less than another launch does, from the
// lengths (partial NULL, see block_offsets_impl).
__global__ __launch_bounds__(kScanThreads) void k_blk_write(const int64_t *tok_offsets,
                                                            const int32_t *start, int32_t n,
                                                            int64_t tile,
                                                            const int64_t *partial,
                                                            int64_t *blk_offsets,
                                                            int32_t *status) {
  __shared__ int64_t lds[kScanThreads / 64];
  const int64_t r0 = (int64_t)blockIdx.x * tile, r1 = r0 + tile < n ? r0 + tile : n;
  int64_t carry = 0, total;
  if (blockIdx.x > 0) {
    if (partial) {
      int64_t s = 0;
      for (int i = threadIdx.x; i < (int)blockIdx.x; i += kScanThreads) s += partial[i];
      block_inclusive_scan(s, lds, &carry);
    } else {
      carry = sum_blocks(tok_offsets, start, 0, r0, status, lds);
    }
  }
  for (int64_t b = r0; b < r1; b += kScanStep) {
    // each thread owns kScanItems consecutive requests
    const int64_t t0 = b + (int64_t)threadIdx.x * kScanItems;
    int64_t c[kScanItems];
    int64_t s = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      c[i] = t0 + i < r1 ? req_blocks(tok_offsets, start, t0 + i, status) : 0;
      s += c[i];
    }
    int64_t run = carry + block_inclusive_scan(s, lds, &total) - s;
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      const int64_t r = t0 + i;
      if (r < r1) blk_offsets[r] = run;
      run += c[i];
      if (r == n - 1) blk_offsets[n] = run;
    }
    carry += total;
  }
  if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0) blk_offsets[0] = 0;
}

// ---------------------------------------------------------------------------
// longest-first ordering: counting sort of requests by block count
// ---------------------------------------------------------------------------

constexpr int kOrderBuckets = 4096;  // block counts >= 4095 share the top bucket

// int32 of scratch that the order of n requests takes
constexpr int64_t order_scratch_ints(int64_t n) { return (int64_t)kOrderBuckets + 64 + n; }

// bucket of request r: the blocks it hashes, from the block offsets (any
// values are safe here; the chain kernels validate them)
__device__ __forceinline__ int order_bucket(const int64_t *blk_offsets, int32_t r) {
  const int64_t d = blk_offsets[r + 1] - blk_offsets[r];
  const int64_t nb = d > 0 ? d : 0;
  return (int)(nb < kOrderBuckets - 1 ? nb : kOrderBuckets - 1);
}

// Histogram and scatter work on tiles of kOrderTile requests per workgroup and
// count in LDS first, so global atomics are one per (tile, non-empty bucket):
// per-request atomics on a few hot bucket counters serialise (4 ms for a
// 1.25M-request batch).  Workgroups of four waves find room on a busy chip
// (other streams' kernels in flight) far sooner than workgroups of sixteen.
constexpr int kOrderThreads = 256;
// (16 requests per thread, half as many workgroups: histogram and scatter 8.6 +
// 9.7 us for 250,000 requests of one length, with 8 5.9 + 7.3; four per thread are no
// better and add global atomics.  1.25 M requests of many lengths: the same.)
constexpr int kOrderPerThread = 8;
constexpr int64_t kOrderTile = (int64_t)kOrderThreads * kOrderPerThread;

__global__ __launch_bounds__(kOrderThreads) void k_order_hist(const int64_t *blk_offsets,
                                                              int32_t n, int32_t *hist) {
  __shared__ int32_t h[kOrderBuckets];
  for (int i = threadIdx.x; i < kOrderBuckets; i += kOrderThreads) h[i] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kOrderTile;
#pragma unroll
  for (int k = 0; k < kOrderPerThread; ++k) {
    const int64_t r = base + (int64_t)k * kOrderThreads + threadIdx.x;
    if (r < n) atomicAdd(&h[order_bucket(blk_offsets, (int32_t)r)], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kOrderBuckets; i += kOrderThreads)
    if (h[i]) atomicAdd(&hist[i], h[i]);
}

// one workgroup: start[b] = number of requests in buckets above b (descending
// order), and *even = the request at place `lp_requests` is as long as the
// longest, within a 32nd.  A chain of waits in one workgroup: 4.6 us (with each
// thread summing the earlier threads' counts from LDS, 8.7).
__global__ __launch_bounds__(256) void k_order_scan(int32_t *hist, int32_t lp_requests,
                                                    int32_t *even) {
  __shared__ int32_t waves[256 / kWave];
  __shared__ int32_t longest, next;
  constexpr int per = kOrderBuckets / 256;
  const int t = threadIdx.x;
  if (t == 0) longest = next = -1;
  // thread t owns buckets kOrderBuckets-1-t*per down to kOrderBuckets-(t+1)*per,
  // so the highest buckets go to thread 0
  const int low = kOrderBuckets - (t + 1) * per;
  int32_t cnt[per], local = 0;
#pragma unroll
  for (int i = 0; i < per; ++i) {
    cnt[i] = hist[low + i];
    local += cnt[i];
  }
  int32_t before = local;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int32_t v = __shfl_up(before, d, kWave);
    if ((t & (kWave - 1)) >= d) before += v;
  }
  if ((t & (kWave - 1)) == kWave - 1) waves[t / kWave] = before;
  __syncthreads();
  before -= local;
  for (int w = 0; w < t / kWave; ++w) before += waves[w];
#pragma unroll
  for (int i = per - 1; i >= 0; --i) {
    hist[low + i] = before;
    if (cnt[i] > 0 && before == 0) longest = low + i;
    if (before <= lp_requests && lp_requests < before + cnt[i]) next = low + i;
    before += cnt[i];
  }
  __syncthreads();
  if (t == 0)
    *even = longest < kOrderBuckets - 1 && next >= 0 && next >= longest - longest / 32;
}

__global__ __launch_bounds__(kOrderThreads) void k_order_scatter(const int64_t *blk_offsets,
                                                                 int32_t n, int32_t *cursor,
                                                                 int32_t *order,
                                                                 int32_t *status) {
  __shared__ int32_t cnt[kOrderBuckets];
  __shared__ int32_t at[kOrderBuckets];
  for (int i = threadIdx.x; i < kOrderBuckets; i += kOrderThreads) cnt[i] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kOrderTile;
  int32_t bucket[kOrderPerThread], rank[kOrderPerThread];
#pragma unroll
  for (int k = 0; k < kOrderPerThread; ++k) {
    const int64_t r = base + (int64_t)k * kOrderThreads + threadIdx.x;
    bucket[k] = -1;
    if (r < n) {
      bucket[k] = order_bucket(blk_offsets, (int32_t)r);
      rank[k] = atomicAdd(&cnt[bucket[k]], 1);
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kOrderBuckets; i += kOrderThreads)
    if (cnt[i]) at[i] = atomicAdd(&cursor[i], cnt[i]);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kOrderPerThread; ++k) {
    if (bucket[k] >= 0) {
      const int64_t r = base + (int64_t)k * kOrderThreads + threadIdx.x;
      // the positions are 0 .. n-1 while the histogram is the batch's own
      const int32_t pos = at[bucket[k]] + rank[k];
      if ((uint32_t)pos < (uint32_t)n)
        order[pos] = (int32_t)r;
      else
        latch(status, KVGOV_E_INTERNAL);
    }
  }
}

__global__ __launch_bounds__(256) void k_fill_i32(int32_t *p, int64_t count, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < count) p[i] = v;
}

// ---------------------------------------------------------------------------
// a2/a3: chains
// ---------------------------------------------------------------------------

struct ChainArgs {
  const int32_t *tokens;
  int64_t n_tokens;
  const int64_t *tok_offsets;
  const int64_t *blk_offsets;
  const int32_t *principal;
  const uint8_t *salts;
  int32_t P;
  int32_t n;
  const int32_t *boundary_tok;
  uint8_t *hashes;
  int64_t n_blocks;
  const int32_t *order;  // NULL: request i on lane i
  const int32_t *even;   // with an order: no few requests are the longest
  int32_t *status;
  // chain extension: request r resumes at block start[r] from the parent
  // digest parents[r] (NULL: every chain starts at block 0)
  const int32_t *start;
  const uint8_t *parents;
  // workgroups from this one on are the second ones on their CUs (0: one per CU)
  int32_t second_from;
};

// Per-request set-up shared by both chain kernels.  Returns false (after
// latching the error) for a request that must write nothing.
struct ChainReq {
  const int32_t *tp;  // tokens of the first block hashed
  uint8_t *out;       // its output row
  int64_t nf;         // blocks to hash (full blocks from the start block on)
  int64_t j0;         // the start block (0 unless resuming)
  int64_t k;          // salted block (boundary mode), else -1
  int64_t kr;         // iteration (block kr + j0) of a boundary block still to
                      // hash with sigma || h, else -1
  uint32_t sig[8];    // salt as state words (salted modes)
  bool salted_root;   // block 0 carries the salt (root, or boundary k = 0)
};

template <int MODE>
__device__ __forceinline__ bool chain_setup(const ChainArgs &a, int32_t r, ChainReq &q) {
  // r comes from the ordering scratch when the batch is ordered: a value
  // outside the batch would mean that scratch was overwritten
  if ((uint32_t)r >= (uint32_t)a.n) {
    latch(a.status, KVGOV_E_INTERNAL);
    return false;
  }
  const int64_t t0 = a.tok_offsets[r], t1 = a.tok_offsets[r + 1];
  if (t0 < 0 || t1 < t0 || t1 > a.n_tokens) {
    latch(a.status, KVGOV_E_OFFSETS);
    return false;
  }
  const int64_t len = t1 - t0;
  const int64_t full = len >> 4;
  q.j0 = a.start ? a.start[r] : 0;
  if (q.j0 < 0 || q.j0 > full) {
    latch(a.status, KVGOV_E_OFFSETS);
    return false;
  }
  q.nf = full - q.j0;
  const int64_t b0 = a.blk_offsets[r];
  if (b0 < 0 || a.blk_offsets[r + 1] - b0 != q.nf || b0 + q.nf > a.n_blocks) {
    latch(a.status, KVGOV_E_OFFSETS);
    return false;
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) q.sig[i] = 0;
  if (MODE != KVGOV_NONE) {
    const int32_t p = a.principal[r];
    if (p < 0 || p >= a.P) {
      latch(a.status, KVGOV_E_PRINCIPAL);
      return false;
    }
    load_digest(a.salts + (int64_t)p * 32, q.sig);
  }
  q.k = -1;
  if (MODE == KVGOV_BOUNDARY) {
    const int32_t bt = a.boundary_tok[r];
    if (bt < 0 || bt > len) {
      latch(a.status, KVGOV_E_BOUNDARY);
      return false;
    }
    q.k = bt >> 4;
  }
  q.tp = a.tokens + t0 + 16 * q.j0;
  q.out = a.hashes + b0 * 32;
  q.salted_root = (MODE == KVGOV_ROOT) || (MODE == KVGOV_BOUNDARY && q.k == 0);
  q.kr = q.k > 0 && q.k >= q.j0 ? q.k - q.j0 : -1;
  return true;
}

// Padding words 8..15 of the second block of a 96-byte message.
__device__ __forceinline__ void pad96_tail(uint32_t w[16]) {
  w[8] = 0x80000000u;
#pragma unroll
  for (int q = 9; q < 15; ++q) w[q] = 0;
  w[15] = 96 * 8;
}

// One lane per request.  Every instruction of a compression (rounds and
// message schedule) is issued by the lane's wave.
//
// An iteration is two compressions: (IV; h || T[0..7]), then (state; T[8..15]
// || pad96).  A block of another pattern takes iterations of its own lane,
// with one compression each (the second one's result is not used), while the
// other lanes of the wave go on with theirs: the unsalted first block two, (IV;
// T) and (state; pad64), the boundary block three, (IV; sigma || h), (state;
// T) and (state; pad128).  So a request costs its wave one or two iterations
// more, wherever its boundary is.  (In one iteration for the whole wave, a
// wave of 64 boundaries ran three compressions in nearly every iteration:
// 262,144 chains of 32 blocks with uniform boundaries 2.24 ms, now 0.95, and
// 0.83 with root salts.)
// Unsalted chains have such a block at their start alone, so their two come before
// the loop, which is then the root-salted one's (50,000 chains of up to 200
// blocks 1,116 us with the test in the loop, 982 so, root-salted 975).
template <int MODE>
__device__ __forceinline__ void single_chain(const ChainArgs &a, int64_t i) {
  if (i >= a.n) return;
  const int32_t r = a.order ? a.order[i] : (int32_t)i;
  ChainReq q;
  if (!chain_setup<MODE>(a, r, q) || q.nf == 0) return;
  const int64_t nf = q.nf;

  // What the lane's next first compression is: a plain block's, or one of the
  // others' (sigma || h; the block's tokens; padding of `bits`).
  enum { kPlain, kSalt, kTokens, kPadding };
  int what = kPlain;
  uint32_t bits = 64 * 8;

  // H holds h_{j-1} as state words, or, between the compressions of a block of
  // another pattern, the state so far: the parent digest when resuming; a
  // root-salted first block (and k == 0 in boundary mode) is the usual
  // pattern with sigma in place of h_{-1}.
  uint32_t H[8];
  if (q.j0 > 0) {
    load_digest(a.parents + (int64_t)r * 32, H);
  } else if (q.salted_root) {
#pragma unroll
    for (int w = 0; w < 8; ++w) H[w] = q.sig[w];
  } else {
    set_iv(H);
    what = kTokens;
  }
  if (MODE == KVGOV_BOUNDARY && q.kr == 0) {
    what = kSalt;
    bits = 128 * 8;
  }

  u32x4 nxt[4];
  uint32_t T[16];  // tokens of block j
  load_raw(q.tp, nxt);
  take_block(nxt, T, q.tp, 0, nf);

  int64_t j = 0;  // block q.j0 + j of the chain
  const auto iteration = [&](bool other) __attribute__((always_inline)) {
    uint32_t st[8], w[16];
    if (!other) {
      set_iv(st);
#pragma unroll
      for (int x = 0; x < 8; ++x) { w[x] = H[x]; w[8 + x] = T[x]; }
    } else {
      const bool iv = what == kPlain || what == kSalt;
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        st[x] = iv ? kSha.H0[x] : H[x];
        const uint32_t lo = what == kSalt ? q.sig[x] : H[x];
        const uint32_t hi = what == kSalt ? H[x] : T[x];
        w[x] = what == kTokens ? T[x] : lo;
        w[8 + x] = what == kTokens ? T[8 + x] : hi;
        if (what == kPadding) {
          w[x] = x == 0 ? 0x80000000u : 0u;
          w[8 + x] = x == 7 ? bits : 0u;
        }
      }
    }
    compress(st, w);
    if (other) {
#pragma unroll
      for (int x = 0; x < 8; ++x) H[x] = st[x];
    }
#pragma unroll
    for (int x = 0; x < 8; ++x) w[x] = T[8 + x];
    pad96_tail(w);
    compress(st, w);
    if (!other) {
#pragma unroll
      for (int x = 0; x < 8; ++x) H[x] = st[x];
      // the next block's tokens before the digest store (see take_block)
      take_block(nxt, T, q.tp, j + 1 < nf ? j + 1 : j, nf);
      store_digest(q.out + j * 32, H);
      ++j;
    } else {
      const bool plain = what == kPlain;
      const bool ends = plain || what == kPadding;  // the block's digest is there
#pragma unroll
      for (int x = 0; x < 8; ++x) H[x] = plain ? st[x] : H[x];
      // a lane whose block goes on keeps its tokens, and loads the same again
      uint32_t N[16];
      swap_block(nxt, N);
      __builtin_amdgcn_sched_barrier(0);
      const int64_t at = ends ? j + 2 : j + 1;
      load_raw(q.tp + 16 * (at < nf ? at : nf - 1), nxt);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = 0; x < 16; ++x) T[x] = ends ? N[x] : T[x];
      if (ends) store_digest(q.out + j * 32, H);
      j += ends ? 1 : 0;
      what = ends ? kPlain : (what == kSalt ? kTokens : kPadding);
    }
    if (MODE == KVGOV_BOUNDARY && j == q.kr && what == kPlain) {
      what = kSalt;
      bits = 128 * 8;
    }
  };
  if (MODE == KVGOV_NONE) {  // the unsalted first block
    for (int k = 0; k < 2; ++k)
      if (j < nf && __any(what != kPlain)) iteration(true);
  }
  while (j < nf) iteration(MODE == KVGOV_BOUNDARY && __any(what != kPlain));
}

// ---------------------------------------------------------------------------
// lane-pair chain kernel
// ---------------------------------------------------------------------------
//
// A chain is latency-bound: the 64 rounds of a compression are a dependency
// chain, and a wave alone on its SIMD issues one instruction per ~4.16
// cycles, so what a block costs is the number of instructions its rounds
// waves issue, plus what they wait for.  This kernel takes the message
// schedule off the rounds lanes and splits each round over two lanes.
// Write A_t for the word a after round t and E_t for e (so b_t = A_{t-1},
// c_t = A_{t-2}, d_t = A_{t-3}, and likewise f, g, h from E).  A round is
//   E_{t+1} = A_{t-3} + T1_t,   T1_t = E_{t-3} + Sigma1(E_t) + Ch(E_t, E_{t-1}, E_{t-2}) + K_t + W_t
//   A_{t+1} = T1_t + Sigma0(A_t) + Maj(A_t, A_{t-1}, A_{t-2})
//           = E_{t+1} - A_{t-3} + Sigma0(A_t) + Maj(A_t, A_{t-1}, A_{t-2}).
// Each request has two adjacent lanes of a rounds wave: the E lane (even)
// produces the E words and the A lane (odd) the A words, two rounds behind:
// in step i the E lane computes E_{i+1} and the A lane A_{i-1}.  Both run the
// same nine instructions on their own last four words x0..x3 (E: E_i..E_{i-3};
// A: A_{i-2}..A_{i-5}), and each needs its partner's x1 (A_{i-3} resp.
// E_{i-1}), which one DPP quad swap delivers to both:
//   S  = rotr(x0,r1) ^ rotr(x0,r2) ^ rotr(x0,r3)   Sigma1(E_i)          | Sigma0(A_{i-2})
//   X  = bitop(x0, x1, m)                          E_i                  | ~(A_{i-2} ^ A_{i-3})
//   F  = choose(X, x1, x2)                         Ch(E_i, .., ..)      | Maj(A_{i-2}, .., ..)
//   Z  = (x3 ^ m) + kw + partner's x1              E_{i-3} + K_i + W_i  | ~A_{i-5} + 1 + E_{i-1}
//                                                  + A_{i-3}            |
//   x0 = S + F + Z                                 E_{i+1}              | A_{i-1}
// with per-lane rotation amounts, m = 0 (E) or ~0 (A), and kw = K + W on E
// lanes and 1 on A lanes (a row of their own in the LDS tables).  Choose with
// ~(a ^ b) as selector is Maj(a, b, c).  Z depends only on words from
// earlier steps, so it is formed one step ahead, and the DPP read is off the
// dependency chain (x0 -> rotates -> xor3 -> add3, and x0 -> X -> choose).
//
// The steps of a block.  C1 = (IV; h_{j-1} || T[0..7]), C2 = (state;
// T[8..15] || padding).
//   * C1's round 0 has a constant state: E_1 = K_0 + W_0 + constant, so C1
//     starts at step 1.  The A lane has nothing to compute in steps 0 and 1;
//     its x0 is set to the initial b, then a.
//   * The A lane finishes C1 (A_63, A_64) in steps 64 and 65, and the E lane
//     needs nothing of it for C2's rounds 0 and 1 but words that are two
//     steps old, so those two steps are C2's steps 0 and 1 at the same time.
//     The feed-forward of C1 (the state's words plus IV) is added to the
//     ring on the E lanes before step 0 and on the A lanes after step 1; what
//     a lane's Z takes from its partner's ring (or from its own, as x3) while
//     the two differ by that addition is made up in kw: C2's kw rows 0, 1, 2
//     hold + IV_3 + IV_7, + IV_2, + IV_1 for the E lanes, and rows 1 and 2
//     of the A lanes' row 1 - IV_4 and 1 - IV_3.
//   * C2 ends with the A lane's two steps of its own (64, 65).
// So a block is 63 + 66 steps, 129 x 9 instructions, and some 90 more (LDS
// reads, feed-forward, the message words of the next block, the store).
//
// The steps are two asm statements per block, with their LDS reads, waits and
// barriers inside: every four K + W words are one ds_read_b128 (tables
// [request][round], the row strides 4 words past a multiple of 16 banks),
// issued at least four steps before their first use into a ring of four quads, the quad a read
// overwrites having just been used.  Every instruction between two such points
// is eight bytes long or paired with another of four, from an eight-byte
// boundary on: a wave alone on its SIMD issues an instruction every 4.0
// cycles while the eight-byte ones lie on eight-byte boundaries and every 5.0
// cycles where they do not (the same 64 steps in a loop, 146 against 182
// cycles per four steps, as one four-byte s_nop is put before them), and a
// taken branch costs it 30 to 130 cycles.  With all of that a block takes
// 5,330 cycles, of which the steps are 4,640 and the 30 LDS reads 340 (11.5
// each); 4096 chains of 137 to 196 blocks take 0.472 ms.  Compiled code
// around shorter asm runs, with a wait for a whole group's reads at
// the head of each run, two-word reads, 132 steps and about 280 other
// instructions a block took 7,350 cycles, 0.622 ms.
//
// Workgroup: 64 requests, four waves.  Waves 0 and 1 run the rounds of 32
// requests each, waves 2 and 3 the message schedule, two lanes per request:
// C1's words 16..63 (which depend on h_{j-1}) in six groups of eight, one
// barrier each (a group takes the schedule waves about as long as the rounds
// waves take for eight steps, so groups of sixteen made the rounds wait:
// 0.542 against 0.530 ms), then the tables of block j + 1 that depend on
// tokens only.  All four waves meet seven barriers per iteration; trip
// counts are decided over all 64 requests.  A request that has ended keeps running on what its LDS
// rows hold and stores nothing.
//
// The boundary block k > 0 is a 128-byte message, three compressions: the
// iteration of that block takes (IV; sigma || h_{k-1}) and (.; T_k), and the
// request takes one more iteration for the padding block, as C2 from the
// saved state (its C1 is idle).  Only that request's chain is longer by one
// iteration, so requests of one workgroup with different boundaries do not
// add up.  (16,384 requests of ~60 blocks with uniform boundaries: 0.258 ms
// with a third compression, for the whole workgroup, in every iteration that
// holds some request's boundary block, two of three; 0.169 ms now.)

struct LpLds {
  uint32_t msg[kWave][20];        // words 0..15 of the first message (for the schedule)
  uint32_t kwm[kWave + 2][12];    // K + words 8..15 of it; then the A lanes', and a row
                                  // that is written and never read
  uint32_t c1[kWave + 1][52];     // K + W of the first compression, rounds 16..63
  uint32_t c2[2][kWave + 1][68];  // K + W of the second compression, by iteration parity
};
static_assert(sizeof(LpLds) % 16 == 0, "LpLds rows are read 16 bytes at a time");

typedef uint32_t lp_quad __attribute__((ext_vector_type(4)));

struct LpLane {
  uint32_t r1, r2, r3;  // rotation amounts of the lane's big sigma
  uint32_t m;           // 0 on E lanes, ~0 on A lanes
};

constexpr uint32_t c_rotr(uint32_t x, int n) { return (x >> n) | (x << (32 - n)); }

constexpr uint64_t kALanes = 0xAAAAAAAAAAAAAAAAull;  // lane mask of the A lanes

// the partner lane's x (adjacent lanes swap: DPP quad_perm [1,0,3,2])
__device__ __forceinline__ uint32_t lp_partner(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true);
}

// LDS byte address of a shared object, as the ds instructions take it
__device__ __forceinline__ uint32_t lds_addr(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p;
}

// One step.  On entry Z holds this step's Z; the step forms x0' (V) and the
// next step's Z (ZN) from KWN (the next step's x3 is this step's x2, and its
// partner's x1 is the partner's present x0).  Ordered so that no instruction
// waits on the one before it, except the first on the previous step's x0.
// The DPP source (X0) was written at least eight instructions earlier, so
// the DPP read needs no wait states.
#define KVGOV_LP_T "%[t1]", "%[t2]", "%[t3]", "%[xx]", "%[f]", "%[sg]"
#define KVGOV_LP_STEP(X0, X1, X2, Z, V, ZN, KWN, T1, T2, T3, XX, F, S)               \
  "v_alignbit_b32 " T1 ", " X0 ", " X0 ", %[r1]\n\t"                              \
  "v_alignbit_b32 " T2 ", " X0 ", " X0 ", %[r2]\n\t"                              \
  "v_bitop3_b32 " XX ", " X0 ", " X1 ", %[m] bitop3:0xd2\n\t"                     \
  "v_alignbit_b32 " T3 ", " X0 ", " X0 ", %[r3]\n\t"                              \
  "v_bitop3_b32 " F ", " XX ", " X1 ", " X2 " bitop3:0xca\n\t"                    \
  "v_bitop3_b32 " S ", " T1 ", " T2 ", " T3 " bitop3:0x96\n\t"                    \
  "v_xad_u32 " ZN ", " X2 ", %[m], " KWN "\n\t"                                   \
  "v_add3_u32 " V ", " S ", " F ", " Z "\n\t"                                     \
  "v_add_u32_dpp " ZN ", " X0 ", " ZN " quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
// the last step: no next Z
#define KVGOV_LP_LAST(X0, X1, X2, Z, V, T1, T2, T3, XX, F, S)                        \
  "v_alignbit_b32 " T1 ", " X0 ", " X0 ", %[r1]\n\t"                              \
  "v_alignbit_b32 " T2 ", " X0 ", " X0 ", %[r2]\n\t"                              \
  "v_bitop3_b32 " XX ", " X0 ", " X1 ", %[m] bitop3:0xd2\n\t"                     \
  "v_alignbit_b32 " T3 ", " X0 ", " X0 ", %[r3]\n\t"                              \
  "v_bitop3_b32 " F ", " XX ", " X1 ", " X2 " bitop3:0xca\n\t"                    \
  "v_bitop3_b32 " S ", " T1 ", " T2 ", " T3 " bitop3:0x96\n\t"                    \
  "v_add3_u32 " V ", " S ", " F ", " Z "\n\t"
#define KVGOV_LP_STEP_(...) KVGOV_LP_STEP(__VA_ARGS__)
#define KVGOV_LP_LAST_(...) KVGOV_LP_LAST(__VA_ARGS__)

// The four words x0..x3 live in a ring of four registers q0..q3: the k-th
// step of a run reads x0 from q[-k mod 4] and writes x0' over the dead x3;
// Z alternates between y0 and y1.
#define KVGOV_LP_R0(K) KVGOV_LP_STEP_("%[q0]", "%[q1]", "%[q2]", "%[y0]", "%[q3]", "%[y1]", K, KVGOV_LP_T)
#define KVGOV_LP_R1(K) KVGOV_LP_STEP_("%[q3]", "%[q0]", "%[q1]", "%[y1]", "%[q2]", "%[y0]", K, KVGOV_LP_T)
#define KVGOV_LP_R2(K) KVGOV_LP_STEP_("%[q2]", "%[q3]", "%[q0]", "%[y0]", "%[q1]", "%[y1]", K, KVGOV_LP_T)
#define KVGOV_LP_R3(K) KVGOV_LP_STEP_("%[q1]", "%[q2]", "%[q3]", "%[y1]", "%[q0]", "%[y0]", K, KVGOV_LP_T)

// K + W quads, in fixed registers so that their words have names: words
// 4n .. 4n + 3 of a compression sit in quad n % 4.  Taking a quad's words
// in four steps (step i takes the kw of step i + 1): in C1 step i is the
// ring's R[(i - 1) % 4], in C2 R[i % 4].
#define KVGOV_LP_P0 "v[96:99]"
#define KVGOV_LP_P1 "v[100:103]"
#define KVGOV_LP_P2 "v[104:107]"
#define KVGOV_LP_P3 "v[108:111]"
#define KVGOV_LP_C1_P0 KVGOV_LP_R2("v96") KVGOV_LP_R3("v97") KVGOV_LP_R0("v98") KVGOV_LP_R1("v99")
#define KVGOV_LP_C1_P1 KVGOV_LP_R2("v100") KVGOV_LP_R3("v101") KVGOV_LP_R0("v102") KVGOV_LP_R1("v103")
#define KVGOV_LP_C1_P2 KVGOV_LP_R2("v104") KVGOV_LP_R3("v105") KVGOV_LP_R0("v106") KVGOV_LP_R1("v107")
#define KVGOV_LP_C1_P3 KVGOV_LP_R2("v108") KVGOV_LP_R3("v109") KVGOV_LP_R0("v110") KVGOV_LP_R1("v111")
#define KVGOV_LP_C2_P0 KVGOV_LP_R3("v96") KVGOV_LP_R0("v97") KVGOV_LP_R1("v98") KVGOV_LP_R2("v99")
#define KVGOV_LP_C2_P1 KVGOV_LP_R3("v100") KVGOV_LP_R0("v101") KVGOV_LP_R1("v102") KVGOV_LP_R2("v103")
#define KVGOV_LP_C2_P2 KVGOV_LP_R3("v104") KVGOV_LP_R0("v105") KVGOV_LP_R1("v106") KVGOV_LP_R2("v107")
#define KVGOV_LP_C2_P3 KVGOV_LP_R3("v108") KVGOV_LP_R0("v109") KVGOV_LP_R1("v110") KVGOV_LP_R2("v111")
#define KVGOV_LP_RD(P, A, OFF) "ds_read_b128 " P ", %[" A "] offset:" #OFF "\n\t"
#define KVGOV_LP_WAIT(N) "s_waitcnt lgkmcnt(" #N ")\n\ts_nop 0\n\t"
#define KVGOV_LP_ALIGN ".p2align 3\n\t"
#define KVGOV_LP_BAR "s_waitcnt lgkmcnt(0)\n\ts_barrier\n\t"
#define KVGOV_LP_TEMPS                                                                     \
  [t1] "=&v"(t1), [t2] "=&v"(t2), [t3] "=&v"(t3), [xx] "=&v"(xx), [f] "=&v"(f), [sg] "=&v"(sg)
#define KVGOV_LP_ROLE [m] "v"(c.m), [r1] "v"(c.r1), [r2] "v"(c.r2), [r3] "v"(c.r3)

// C1, steps 1..63.  q = x0, x1, x2 of step 1 (q[3] is free), z its Z; kw[2..7]
// the K + W of rounds 2..7; a0 the value the A lanes' x0 takes after step 1.
// Reads words 8..15 at LDS address am and 16..63 at ac1, each group of these after
// the barrier that releases it (words 16.., 24.., 32.., 48..), and C2's
// words 0..11 at ac2 into p.  On return q[1], q[2], q[3], q[0] are x0..x3
// after step 63 and z the Z of step 64.
__device__ __forceinline__ void lp_c1(uint32_t q[4], uint32_t &z, const uint32_t kw[8], uint32_t a0,
                                      const LpLane &c, uint32_t am, uint32_t ac1, uint32_t ac2,
                                      lp_quad p[3]) {
  uint32_t y1, t1, t2, t3, xx, f, sg;
  asm volatile(
      KVGOV_LP_ALIGN
      KVGOV_LP_RD(KVGOV_LP_P2, "am", 0) KVGOV_LP_RD(KVGOV_LP_P3, "am", 16)
      KVGOV_LP_R0("%[k2]")                                                       // step 1
      "v_cndmask_b32_e64 %[q3], %[q3], %[a0], %[al]\n\t"
      KVGOV_LP_R1("%[k3]") KVGOV_LP_R2("%[k4]") KVGOV_LP_R3("%[k5]")             // 2..4
      KVGOV_LP_R0("%[k6]") KVGOV_LP_R1("%[k7]")                                  // 5, 6
      KVGOV_LP_WAIT(1) KVGOV_LP_C1_P2                                            // 7..10
      KVGOV_LP_BAR                                                               // 16..23
      KVGOV_LP_RD(KVGOV_LP_P0, "ac1", 0) KVGOV_LP_RD(KVGOV_LP_P1, "ac1", 16)
      KVGOV_LP_C1_P3                                                             // 11..14
      KVGOV_LP_WAIT(1) KVGOV_LP_C1_P0                                            // 15..18
      KVGOV_LP_BAR                                                               // 24..31
      KVGOV_LP_RD(KVGOV_LP_P2, "ac1", 32) KVGOV_LP_RD(KVGOV_LP_P3, "ac1", 48)
      KVGOV_LP_C1_P1                                                             // 19..22
      KVGOV_LP_WAIT(1) KVGOV_LP_C1_P2                                            // 23..26
      KVGOV_LP_BAR                                                               // 32..39
      KVGOV_LP_RD(KVGOV_LP_P0, "ac1", 64) KVGOV_LP_RD(KVGOV_LP_P1, "ac1", 80)
      KVGOV_LP_C1_P3                                                             // 27..30
      KVGOV_LP_WAIT(1) KVGOV_LP_C1_P0                                            // 31..34
      KVGOV_LP_BAR                                                               // 40..47
      KVGOV_LP_RD(KVGOV_LP_P2, "ac1", 96) KVGOV_LP_RD(KVGOV_LP_P3, "ac1", 112)
      KVGOV_LP_C1_P1                                                             // 35..38
      KVGOV_LP_WAIT(1) KVGOV_LP_C1_P2                                            // 39..42
      KVGOV_LP_BAR                                                               // 48..55
      KVGOV_LP_RD(KVGOV_LP_P0, "ac1", 128) KVGOV_LP_RD(KVGOV_LP_P1, "ac1", 144)
      KVGOV_LP_C1_P3                                                             // 43..46
      KVGOV_LP_WAIT(1) KVGOV_LP_C1_P0                                            // 47..50
      KVGOV_LP_BAR                                                               // 56..63
      KVGOV_LP_RD(KVGOV_LP_P2, "ac1", 160) KVGOV_LP_RD(KVGOV_LP_P3, "ac1", 176)
      KVGOV_LP_RD(KVGOV_LP_P0, "ac2", 0)
      KVGOV_LP_C1_P1                                                             // 51..54
      KVGOV_LP_RD(KVGOV_LP_P1, "ac2", 16)
      KVGOV_LP_WAIT(3) KVGOV_LP_C1_P2                                            // 55..58
      KVGOV_LP_RD(KVGOV_LP_P2, "ac2", 32)
      KVGOV_LP_WAIT(3) KVGOV_LP_C1_P3                                            // 59..62
      KVGOV_LP_WAIT(0) KVGOV_LP_R2("v96")                                        // 63
      : [q0] "+v"(q[0]), [q1] "+v"(q[1]), [q2] "+v"(q[2]), [q3] "=&v"(q[3]), [y0] "+v"(z),
        [y1] "=&v"(y1), KVGOV_LP_TEMPS, "=&{v[96:99]}"(p[0]), "=&{v[100:103]}"(p[1]),
        "=&{v[104:107]}"(p[2])
      : KVGOV_LP_ROLE, [k2] "v"(kw[2]), [k3] "v"(kw[3]), [k4] "v"(kw[4]), [k5] "v"(kw[5]),
        [k6] "v"(kw[6]), [k7] "v"(kw[7]), [a0] "v"(a0), [al] "s"(kALanes), [am] "v"(am),
        [ac1] "v"(ac1), [ac2] "v"(ac2)
      : "v108", "v109", "v110", "v111", "memory");
  z = y1;
}

// C2, steps 0..65.  s = the state's words (see the feed-forward above; the
// A lanes' still without it), z the Z of step 0, p the words 0..11.  fa =
// what the A lanes add after step 1 (0 on E lanes).  On return q holds x0..x3
// after step 63 and n0, n1 the A lanes' last two words; s holds the state
// C2 started from, but for the A lanes' s[3] without fa's fourth word.
__device__ __forceinline__ void lp_c2(uint32_t s[4], uint32_t z, const lp_quad p[3],
                                      const uint32_t fa[3], const LpLane &c, uint32_t ac2,
                                      uint32_t q[4], uint32_t &n0, uint32_t &n1) {
  uint32_t y1, x2, t1, t2, t3, xx, f, sg;
  lp_quad p0, p1, p2;
  asm volatile(
      KVGOV_LP_ALIGN
      KVGOV_LP_RD(KVGOV_LP_P3, "ac2", 48)
      // steps 0 and 1 (C1's 64 and 65 on the A lanes)
      KVGOV_LP_STEP_("%[s0]", "%[s1]", "%[s2]", "%[y0]", "%[q3]", "%[y1]", "v97", KVGOV_LP_T)
      KVGOV_LP_STEP_("%[q3]", "%[s0]", "%[s1]", "%[y1]", "%[q2]", "%[y0]", "v98", KVGOV_LP_T)
      "v_add_u32_e64 %[x2], %[s0], %[f2]\n\t"
      "v_add_u32_e64 %[q2], %[q2], %[f0]\n\t"
      "v_add_u32_e64 %[q3], %[q3], %[f1]\n\t"
      "v_cndmask_b32_e64 %[s3], %[s3], %[s1], %[al]\n\t"
      "v_cndmask_b32_e64 %[s2], %[s2], %[x2], %[al]\n\t"
      "v_cndmask_b32_e64 %[s1], %[s1], %[q3], %[al]\n\t"
      "v_cndmask_b32_e64 %[s0], %[s0], %[q2], %[al]\n\t"
      KVGOV_LP_STEP_("%[q2]", "%[q3]", "%[x2]", "%[y0]", "%[q1]", "%[y1]", "v99", KVGOV_LP_T)
      KVGOV_LP_RD(KVGOV_LP_P0, "ac2", 64)
      KVGOV_LP_R3("v100") KVGOV_LP_R0("v101") KVGOV_LP_R1("v102") KVGOV_LP_R2("v103")  // 3..6
      KVGOV_LP_RD(KVGOV_LP_P1, "ac2", 80)
      KVGOV_LP_C2_P2                                                             // 7..10
      KVGOV_LP_RD(KVGOV_LP_P2, "ac2", 96)
      KVGOV_LP_WAIT(2) KVGOV_LP_C2_P3                                            // 11..14
      KVGOV_LP_RD(KVGOV_LP_P3, "ac2", 112) KVGOV_LP_C2_P0                        // 15..18
      KVGOV_LP_RD(KVGOV_LP_P0, "ac2", 128) KVGOV_LP_WAIT(2) KVGOV_LP_C2_P1
      KVGOV_LP_RD(KVGOV_LP_P1, "ac2", 144) KVGOV_LP_C2_P2
      KVGOV_LP_RD(KVGOV_LP_P2, "ac2", 160) KVGOV_LP_WAIT(2) KVGOV_LP_C2_P3       // 27..30
      KVGOV_LP_RD(KVGOV_LP_P3, "ac2", 176) KVGOV_LP_C2_P0
      KVGOV_LP_RD(KVGOV_LP_P0, "ac2", 192) KVGOV_LP_WAIT(2) KVGOV_LP_C2_P1
      KVGOV_LP_RD(KVGOV_LP_P1, "ac2", 208) KVGOV_LP_C2_P2
      KVGOV_LP_RD(KVGOV_LP_P2, "ac2", 224) KVGOV_LP_WAIT(2) KVGOV_LP_C2_P3       // 43..46
      KVGOV_LP_RD(KVGOV_LP_P3, "ac2", 240) KVGOV_LP_C2_P0                        // 47..50
      KVGOV_LP_WAIT(1) KVGOV_LP_C2_P1 KVGOV_LP_C2_P2                             // 51..58
      KVGOV_LP_WAIT(0) KVGOV_LP_C2_P3                                            // 59..62
      KVGOV_LP_R3("1")                                                           // 63
      KVGOV_LP_STEP_("%[q0]", "%[q1]", "%[q2]", "%[y0]", "%[n0]", "%[y1]", "1", KVGOV_LP_T)
      KVGOV_LP_LAST_("%[n0]", "%[q0]", "%[q1]", "%[y1]", "%[n1]", KVGOV_LP_T)
      : [s0] "+v"(s[0]), [s1] "+v"(s[1]), [s2] "+v"(s[2]), [s3] "+v"(s[3]), [y0] "+v"(z),
        [y1] "=&v"(y1), [x2] "=&v"(x2), [q0] "=&v"(q[0]), [q1] "=&v"(q[1]), [q2] "=&v"(q[2]),
        [q3] "=&v"(q[3]), [n0] "=&v"(n0), [n1] "=&v"(n1), KVGOV_LP_TEMPS,
        "=&{v[96:99]}"(p0), "=&{v[100:103]}"(p1), "=&{v[104:107]}"(p2)
      : KVGOV_LP_ROLE, [f0] "v"(fa[0]), [f1] "v"(fa[1]), [f2] "v"(fa[2]), [al] "s"(kALanes),
        [ac2] "v"(ac2), "{v[96:99]}"(p[0]), "{v[100:103]}"(p[1]), "{v[104:107]}"(p[2])
      : "v108", "v109", "v110", "v111", "memory");
}

// Message schedule on a lane pair: lane p of the pair makes the words W[t],
// t = 16 + 2k + p, of step k, so a wave makes two words of 32 requests in
// about 15 instructions.  Both lanes keep a 16-word window in which lane p's
// logical word i at step k is W[2k + p + i], stored at w[(2k + i) & 15]: the
// four operands of W[t] (t - 16, t - 15, t - 7, t - 2: logical 0, 1, 9, 14)
// are then the same registers on both lanes.  After the step each lane takes
// its partner's new word with one DPP swap: lane 0 needs it as logical 15 of
// the next window (W[17 + 2k]), lane 1 as logical 13 (W[16 + 2k]); lane 1's
// logical 15 (W[18 + 2k], lane 0's next word) is set the same way one step
// later, before it is first read (as logical 9, four steps on).
// Word 2k of the row at LDS address `row` (already offset by p) receives
// K[t] + W[t]; kt = the lane's K.  Four steps are one asm statement of
// eight-byte instructions only (see KVGOV_LP_ALIGN): 13 per step and a write for
// two, with no wait state before a DPP read (two instructions after the write of
// what it reads): the first step's exchange is put between the second step's
// first instructions.  The rounds waves wait for the schedule at every group
// once a group takes it longer than eight steps take them, and then each barrier
// costs them some 70 cycles, however short the wait: 0.510 ms for the 4096
// chains above with a write per step, 0.468 so.
#define KVGOV_LP_SUM(W0, W1, W9, W14, KT, T, MID)                                   \
  "v_alignbit_b32 %[t1], " W1 ", " W1 ", 7\n\t"                                    \
  "v_alignbit_b32 %[t2], " W1 ", " W1 ", 18\n\t"                                   \
  MID                                                                              \
  "v_lshrrev_b32_e64 %[t3], 3, " W1 "\n\t"                                         \
  "v_alignbit_b32 %[t4], " W14 ", " W14 ", 17\n\t"                                 \
  "v_bitop3_b32 %[t1], %[t1], %[t2], %[t3] bitop3:0x96\n\t"                        \
  "v_alignbit_b32 %[t5], " W14 ", " W14 ", 19\n\t"                                 \
  "v_lshrrev_b32_e64 %[t6], 10, " W14 "\n\t"                                       \
  "v_add3_u32 " W0 ", %[t1], " W0 ", " W9 "\n\t"                                   \
  "v_bitop3_b32 %[t4], %[t4], %[t5], %[t6] bitop3:0x96\n\t"                        \
  "v_add_u32_e64 " W0 ", " W0 ", %[t4]\n\t"                                        \
  "v_add_u32_e64 " T ", " W0 ", " KT "\n\t"
// w[i0] holds the new word (logical 14 of the next window); w[i1] <- the
// partner's (logical 15; on lane 1 replaced before it is read), w[i15] on
// lane 1 <- the partner's (logical 13)
#define KVGOV_LP_SWAP(W0, W1, W15)                                                  \
  "v_mov_b32_dpp " W1 ", " W0 " quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t" \
  "v_cndmask_b32_e64 " W15 ", " W15 ", " W1 ", %[ol]\n\t"
#define KVGOV_LP_SCHED2(W0, W1, W2, W3, W9, W11, W14, W15, KA, KB, OA, OB)          \
  KVGOV_LP_SUM(W0, W1, W9, W14, KA, "%[t7]", "")                                   \
  KVGOV_LP_SUM(W2, W3, W11, W0, KB, "%[t1]", KVGOV_LP_SWAP(W0, W1, W15))           \
  "ds_write2_b32 %[row], %[t7], %[t1] offset0:" OA " offset1:" OB "\n\t"           \
  KVGOV_LP_SWAP(W2, W3, W1)

// Steps 4 G .. 4 G + 3; kt the lane's constants of these.
template <int G>
__device__ __forceinline__ void lp_pair4(uint32_t w[16], uint32_t row, const uint32_t *kt) {
  uint32_t t1, t2, t3, t4, t5, t6, t7;
  constexpr int b = (8 * G) & 15;  // the window's start: 0 or 8
#define KVGOV_LP_W(I) [w##I] "+v"(w[(b + I) & 15])
  asm volatile(KVGOV_LP_ALIGN
               KVGOV_LP_SCHED2("%[w0]", "%[w1]", "%[w2]", "%[w3]", "%[w9]", "%[w11]", "%[w14]",
                               "%[w15]", "%[k0]", "%[k1]", "%c[o0]", "%c[o1]")
               KVGOV_LP_SCHED2("%[w4]", "%[w5]", "%[w6]", "%[w7]", "%[w13]", "%[w15]", "%[w2]",
                               "%[w3]", "%[k2]", "%[k3]", "%c[o2]", "%c[o3]")
               : KVGOV_LP_W(0), KVGOV_LP_W(1), KVGOV_LP_W(2), KVGOV_LP_W(3), KVGOV_LP_W(4),
                 KVGOV_LP_W(5), KVGOV_LP_W(6), KVGOV_LP_W(7), KVGOV_LP_W(9), KVGOV_LP_W(11),
                 KVGOV_LP_W(13), KVGOV_LP_W(14), KVGOV_LP_W(15), [t1] "=&v"(t1), [t2] "=&v"(t2),
                 [t3] "=&v"(t3), [t4] "=&v"(t4), [t5] "=&v"(t5), [t6] "=&v"(t6), [t7] "=&v"(t7)
               : [k0] "v"(kt[0]), [k1] "v"(kt[1]), [k2] "v"(kt[2]), [k3] "v"(kt[3]),
                 [row] "v"(row), [ol] "s"(kALanes), [o0] "i"(8 * G), [o1] "i"(8 * G + 2),
                 [o2] "i"(8 * G + 4), [o3] "i"(8 * G + 6)
               : "memory");
#undef KVGOV_LP_W
}

// The schedule waves' barrier.  The compiler waits for the LDS accesses that it
// knows; lp_pair4's writes are inside asm, so their wait is here.
__device__ __forceinline__ void lp_sched_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __syncthreads();
}

// What a request does in iteration i of its workgroup.
enum LpBlock {
  kLpPlain,     // first (IV; h || T[0..7])      second (.; T[8..15] || pad96)
  kLpFirst,     // first (IV; T[0..15])          second (.; pad64)
  kLpBoundary,  // first (IV; sigma || h)        second (.; T[0..15])
  kLpPad        // first idle                    second (the boundary block's state; pad128)
};

// The tables of a request's next iteration that depend on tokens and
// constants: raw words and K + words of the first message except h (written
// by the rounds lanes), and K + W of all 64 rounds of the second message (all on
// both lanes of the pair; the schedule is split by parity).
__device__ __forceinline__ void lp_prepare(const uint32_t Tn[16], const uint32_t sig[8],
                                           LpBlock what, LpLds &L, int buf, int col, bool odd,
                                           const uint32_t kt[24]) {
  uint32_t m[16], w[16];
  lp_quad *raw = reinterpret_cast<lp_quad *>(L.msg[col]);
  lp_quad *kwm = reinterpret_cast<lp_quad *>(L.kwm[col]);
  // words 8..15 of the first message
  if (what == kLpPlain || what == kLpFirst) {
    const int o = what == kLpFirst ? 8 : 0;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      lp_quad r, k;
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        r[y] = o ? Tn[8 + 4 * x + y] : Tn[4 * x + y];
        k[y] = r[y] + kSha.K[8 + 4 * x + y];
      }
      raw[2 + x] = r;
      kwm[x] = k;
    }
  }
  if (what == kLpBoundary || what == kLpFirst) {
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      lp_quad r;
#pragma unroll
      for (int y = 0; y < 4; ++y) r[y] = what == kLpFirst ? Tn[4 * x + y] : sig[4 * x + y];
      raw[x] = r;
    }
  }
  // the second message
#pragma unroll
  for (int x = 0; x < 16; ++x) m[x] = 0;
  if (what == kLpPlain) {
#pragma unroll
    for (int x = 0; x < 8; ++x) m[x] = Tn[8 + x];
    pad96_tail(m);
  } else if (what == kLpBoundary) {
#pragma unroll
    for (int x = 0; x < 16; ++x) m[x] = Tn[x];
  } else {
    m[0] = 0x80000000u;
    m[15] = what == kLpFirst ? 64 * 8 : 128 * 8;
  }
  lp_quad *row = reinterpret_cast<lp_quad *>(L.c2[buf][col]);
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    lp_quad k;
#pragma unroll
    for (int y = 0; y < 4; ++y) k[y] = m[4 * x + y] + kSha.K[4 * x + y];
    if (x == 0) {  // the feed-forward of the first compression (see above)
      k[0] += kSha.H0[3] + kSha.H0[7];
      k[1] += kSha.H0[2];
      k[2] += kSha.H0[1];
    }
    row[x] = k;
  }
  // lane 1's window starts one word later; its logical 15 (W[16]) comes
  // from lane 0's first step
#pragma unroll
  for (int i = 0; i < 15; ++i) w[i] = odd ? m[i + 1] : m[i];
  w[15] = m[15];
  const uint32_t out = lds_addr(L.c2[buf][col] + 16 + (odd ? 1 : 0));
  lp_pair4<0>(w, out, kt);
  lp_pair4<1>(w, out, kt + 4);
  lp_pair4<2>(w, out, kt + 8);
  lp_pair4<3>(w, out, kt + 12);
  lp_pair4<4>(w, out, kt + 16);
  lp_pair4<5>(w, out, kt + 20);
}

// The A lane's Z and third word with which two steps from (c, d) of the
// state give it b and a: what a padding iteration starts from, see lp_pad.
__device__ __forceinline__ uint32_t lp_a_sum(uint32_t x0, uint32_t x1, uint32_t x2) {
  return big_sigma0(x0) + maj(x0, x1, x2);
}

// Before C2 of a padding iteration: the ring and Z as steps 64 and 65 of a C1
// with the saved state P (e..h on E lanes, a..d on A lanes) as its result
// would find them.  kw0 = C2's kw row 0.  The E lane's step 0 takes P as it
// is.  The A lane's ring must read c - IV_2, d - IV_3, and its two steps give
// b - IV_1 and a - IV_0 (the feed-forward comes after them): its Z, and x2
// (which only its own next Z takes, as x3, and step 0's majority), are
// solved for.
__device__ __forceinline__ void lp_pad(const uint32_t P[4], uint32_t kw0, bool a_lane,
                                       uint32_t s[4], uint32_t &z) {
  uint32_t o[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) o[x] = lp_partner(P[x]);
  if (a_lane) {
    const uint32_t a = P[0] - kSha.H0[0], b = P[1] - kSha.H0[1], cc = P[2] - kSha.H0[2],
                   d = P[3] - kSha.H0[3];
    // step 1: a = sum(b, c, d) + Z1, Z1 = ~x2 + (1 - IV_4) + e
    const uint32_t z1 = a - lp_a_sum(b, cc, d);
    const uint32_t x2 = ~(z1 - 1u + kSha.H0[4] - o[0]);
    s[0] = cc;
    s[1] = d;
    s[2] = x2;
    s[3] = 0;
    z = b - lp_a_sum(cc, d, x2);
  } else {
#pragma unroll
    for (int x = 0; x < 4; ++x) s[x] = P[x];
    z = P[3] + o[3] + kw0 - kSha.H0[3] - kSha.H0[7];
  }
}

// Workgroup `group` of the lane-pair kernel: requests group * 64 + 0..63 of
// the (ordered) batch.
template <int MODE>
__device__ __forceinline__ void lp_group(const ChainArgs &a, int32_t group, LpLds &L) {
  const int lane = threadIdx.x & (kWave - 1);
  // The wave's part: 0 and 1 rounds, 2 and 3 schedule.  Where two workgroups share a
  // CU, the waves of the second one start one SIMD further on in the order
  // that the first one's took, so that its waves 0 and 1 would meet a rounds
  // and a schedule wave; turned by three, its rounds waves meet the schedule
  // waves of the first (32,768 chains of 128 blocks: 0.633 -> 0.611 ms).
  const int turn = a.second_from > 0 && group >= a.second_from ? 3 : 0;
  const int wave = __builtin_amdgcn_readfirstlane((int)((threadIdx.x / kWave + turn) & 3));
  const bool sched_wave = wave >= 2;
  const bool odd = lane & 1;  // rounds: the A lane; schedule: the odd words' lane
  // the request (LDS row) of this lane within the workgroup
  const int mine = (wave & 1) * 32 + (lane >> 1);
  const int32_t base = group * kWave;
  const int32_t i = base + mine;

  ChainReq q{};
  bool ok = false;
  int32_t r = 0;
  if (i < a.n) {
    r = a.order ? a.order[i] : i;
    ok = chain_setup<MODE>(a, r, q);
  }
  const int64_t nf = ok ? q.nf : 0;
  const int64_t kb = ok && q.kr < nf ? q.kr : -1;  // the boundary block's iteration, else -1
  // iterations: the blocks, and the boundary block's padding
  const int64_t ni = nf + (MODE == KVGOV_BOUNDARY && kb >= 0 ? 1 : 0);

  // Trip count over all 64 requests: each wave's maximum through LDS (the
  // first words of the tables, before these are written).
  int64_t J = ni;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    const int64_t o = __shfl_xor(J, d, kWave);
    J = o > J ? o : J;
  }
  int64_t *trips = reinterpret_cast<int64_t *>(&L);
  if (lane == 0) trips[wave] = J;
  __syncthreads();
  J = trips[0] > trips[1] ? trips[0] : trips[1];
  __syncthreads();
  if (J == 0) return;  // every wave of the workgroup

  // the A lanes' rows
  for (int x = threadIdx.x; x < 12; x += blockDim.x) L.kwm[kWave][x] = 1u;
  for (int x = threadIdx.x; x < 52; x += blockDim.x) L.c1[kWave][x] = 1u;
  for (int x = threadIdx.x; x < 68; x += blockDim.x) {
    const uint32_t v = x == 1 ? 1u - kSha.H0[4] : (x == 2 ? 1u - kSha.H0[3] : 1u);
    L.c2[0][kWave][x] = v;
    L.c2[1][kWave][x] = v;
  }

  if (sched_wave) {
    // ---- schedule waves, two lanes per request
    uint32_t kt[24];  // the lane's round constants, K[16 + 2k + parity]
#pragma unroll
    for (int k = 0; k < 24; ++k) {
      kt[k] = odd ? kSha.K[17 + 2 * k] : kSha.K[16 + 2 * k];
      asm("" : "+v"(kt[k]));  // kept in a register
    }
    // tokens one block ahead: raw holds block `held` (lanes without blocks
    // read a valid dummy: some request of the workgroup has a block, so the
    // token array holds at least 16 tokens)
    u32x4 raw[4];
    const int32_t *tp = nf > 0 ? q.tp : a.tokens;
    const int64_t last = nf > 0 ? nf - 1 : 0;
    int64_t held = 0;
    load_raw(tp, raw);
    {
      uint32_t T0[16];
      swap_block(raw, T0);
      held = last < 1 ? last : 1;
      load_raw(tp + 16 * held, raw);
      // h_{j0-1}: the parent digest when resuming (in the second half of a
      // boundary block's first message), sigma for a salted root
      const bool resume = ok && q.j0 > 0, bnd0 = MODE == KVGOV_BOUNDARY && kb == 0;
      const bool root = ok && q.salted_root;
      uint32_t h[8];
#pragma unroll
      for (int x = 0; x < 8; ++x) h[x] = root ? q.sig[x] : 0u;
      if (resume && nf > 0) load_digest(a.parents + (int64_t)r * 32, h);
      if (nf > 0) {
        lp_prepare(T0, q.sig, bnd0 ? kLpBoundary : (resume || root ? kLpPlain : kLpFirst), L, 0,
                   mine, odd, kt);
        if (resume || root) {
#pragma unroll
          for (int x = 0; x < 8; ++x) {
            if (bnd0) {
              L.msg[mine][8 + x] = h[x];
              L.kwm[mine][x] = h[x] + kSha.K[8 + x];
            } else {
              L.msg[mine][x] = h[x];
            }
          }
        }
      }
    }
    lp_sched_barrier();
    const uint32_t row1 = lds_addr(L.c1[mine] + (odd ? 1 : 0));
    const uint32_t *msg = L.msg[mine] + (odd ? 1 : 0);
    uint32_t w[16];
#pragma unroll
    for (int x = 8; x < 15; ++x) w[x] = msg[x];
    w[15] = L.msg[mine][15];
    for (int64_t j = 0; j < J; ++j) {
#pragma unroll
      for (int x = 0; x < 8; ++x) w[x] = msg[x];
      if (MODE == KVGOV_BOUNDARY) {  // may hold h_{j-1}, which the rounds lanes wrote
#pragma unroll
        for (int x = 8; x < 15; ++x) w[x] = msg[x];
        w[15] = L.msg[mine][15];
      }
      lp_pair4<0>(w, row1, kt);
      lp_sched_barrier();
      lp_pair4<1>(w, row1, kt + 4);
      lp_sched_barrier();
      lp_pair4<2>(w, row1, kt + 8);
      lp_sched_barrier();
      lp_pair4<3>(w, row1, kt + 12);
      lp_sched_barrier();
      lp_pair4<4>(w, row1, kt + 16);
      lp_sched_barrier();
      lp_pair4<5>(w, row1, kt + 20);
      lp_sched_barrier();
      // iteration j + 1: its tokens (block `held`, unless it is a padding
      // iteration), and the load of the block after it
      const bool pad = MODE == KVGOV_BOUNDARY && kb >= 0 && j == kb;
      uint32_t Tn[16];
      swap_block(raw, Tn);
      __builtin_amdgcn_sched_barrier(0);
      if (!pad) held = held < last ? held + 1 : last;
      load_raw(tp + 16 * held, raw);
      __builtin_amdgcn_sched_barrier(0);
      if (j + 1 < ni) {
        const bool bnd = MODE == KVGOV_BOUNDARY && kb >= 0 && j + 1 == kb;
        lp_prepare(Tn, q.sig, MODE != KVGOV_BOUNDARY ? kLpPlain
                                                     : (pad ? kLpPad : (bnd ? kLpBoundary : kLpPlain)),
                   L, (int)((j + 1) & 1), mine, odd, kt);
      }
      if (MODE != KVGOV_BOUNDARY) {  // this pair's own writes
#pragma unroll
        for (int x = 8; x < 15; ++x) w[x] = msg[x];
        w[15] = L.msg[mine][15];
      }
      lp_sched_barrier();
    }
    return;
  }

  // ---- rounds waves
  const bool a_lane = odd;
  LpLane c;
  c.r1 = a_lane ? 2 : 6;
  c.r2 = a_lane ? 13 : 11;
  c.r3 = a_lane ? 22 : 25;
  c.m = a_lane ? ~0u : 0u;
  const int row = a_lane ? kWave : mine;
  const int half = a_lane ? 0 : 4;  // state words held: a..d = 0..3, e..h = 4..7
  // feed-forward of C1: added on E lanes before C2, on A lanes two steps on
  uint32_t fe[4], fa[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    fe[x] = a_lane ? 0u : kSha.H0[4 + x];
    fa[x] = a_lane ? kSha.H0[x] : 0u;
  }
  // step 1 of C1: E_1 = K_0 + W_0 + (h + Sigma1(e) + Ch(e, f, g) + d) on E
  // lanes; Z of step 1 = K_1 + W_1 + g + c
  constexpr uint32_t e0 = kSha.H0[4], f0 = kSha.H0[5], g0 = kSha.H0[6];
  constexpr uint32_t c_e1 = kSha.K[0] + kSha.H0[7] + kSha.H0[3] +
                            (c_rotr(e0, 6) ^ c_rotr(e0, 11) ^ c_rotr(e0, 25)) +
                            ((e0 & f0) ^ (~e0 & g0));
  constexpr uint32_t c_z1 = kSha.K[1] + g0 + kSha.H0[2];
  const uint32_t x1_0 = a_lane ? kSha.H0[2] : e0;  // x1, x2 of step 1
  const uint32_t x2_0 = a_lane ? kSha.H0[3] : f0;
  const uint32_t am = lds_addr(L.kwm[row]), ac1 = lds_addr(L.c1[row]);
  const uint32_t ac2_0 = lds_addr(L.c2[0][row]), ac2_1 = lds_addr(L.c2[1][row]);
  uint32_t sg[4];  // the lane's half of the salt (boundary mode)
#pragma unroll
  for (int x = 0; x < 4; ++x) sg[x] = MODE != KVGOV_BOUNDARY ? 0u : (a_lane ? q.sig[x] : q.sig[4 + x]);
  uint8_t *out = ok ? q.out + half * 4 : nullptr;
  uint32_t kd[4] = {c_e1, c_z1, kSha.K[2], kSha.K[3]};  // added to the partner's words
#pragma unroll
  for (int x = 0; x < 4; ++x) asm("" : "+v"(kd[x]));  // in registers: one DPP add each

  __syncthreads();  // the first iteration's tables
  // the schedule has time to spare, the rounds have none (the same batch: ->
  // 0.564 ms; no difference where a wave has its SIMD to itself)
  __builtin_amdgcn_s_setprio(2);
  // st: words 0..7 of the first message (A lanes 0..3, E lanes 4..7)
  uint32_t st[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) st[x] = L.msg[mine][half + x];
  uint32_t hold[4] = {0, 0, 0, 0};  // the boundary block's state (boundary mode)
  uint32_t k8[4];  // the lane's half of K[8..15] (boundary mode)
#pragma unroll
  for (int x = 0; x < 4; ++x) k8[x] = a_lane ? kSha.K[8 + x] : kSha.K[12 + x];
  // C1's start from words 0..7 of its message (E lanes take a..d from the partner)
  uint32_t kw[8], x0_1, z_1;
  const auto start = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t o = lp_partner(st[t]) + kd[t];
      if (t == 0) x0_1 = a_lane ? kSha.H0[1] : o;
      if (t == 1) z_1 = o;
      if (t >= 2) kw[t] = a_lane ? 1u : o;
      kw[4 + t] = a_lane ? 1u : st[t] + kSha.K[4 + t];
    }
  };
  start();
  for (int64_t j = 0; j < J; ++j) {
    const uint32_t ac2 = (j & 1) ? ac2_1 : ac2_0;
    uint32_t ring[4] = {x0_1, x1_0, x2_0, 0}, z = z_1, s[4], x[4], n0, n1;
    lp_quad p[3];
    lp_c1(ring, z, kw, kSha.H0[0], c, am, ac1, ac2, p);
    s[0] = ring[1] + fe[0];
    s[1] = ring[2] + fe[1];
    s[2] = ring[3] + fe[2];
    s[3] = ring[0] + fe[3];
    if (MODE == KVGOV_BOUNDARY) {
      const bool pad = kb >= 0 && j == kb + 1;
      if (__any(pad)) {
        uint32_t sp[4], zp;
        lp_pad(hold, p[0][0], a_lane, sp, zp);
#pragma unroll
        for (int t = 0; t < 4; ++t) s[t] = pad ? sp[t] : s[t];
        z = pad ? zp : z;
      }
    }
    lp_c2(s, z, p, fa, c, ac2, x, n0, n1);
    st[0] = (a_lane ? n1 : x[0]) + s[0];
    st[1] = (a_lane ? n0 : x[1]) + s[1];
    st[2] = (a_lane ? x[0] : x[2]) + s[2];
    st[3] = (a_lane ? x[1] : x[3]) + s[3] + fa[3];
    // h_j: words 0..7 of the next iteration's first message, or 8..15 when
    // that is the boundary block (words 0..7 are then the salt's)
    const bool hashed = MODE != KVGOV_BOUNDARY || j != kb;  // st is a digest
    if (j < ni && hashed) {
      *reinterpret_cast<u32x4 *>(out) = u32x4{bswap(st[0]), bswap(st[1]), bswap(st[2]), bswap(st[3])};
      out += 32;
    }
    if (MODE == KVGOV_BOUNDARY) {
      const bool bnd = kb >= 0 && j + 1 == kb;
      lp_quad kw8;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        hold[t] = hashed ? hold[t] : st[t];
        kw8[t] = st[t] + k8[t];
      }
      *reinterpret_cast<lp_quad *>(bnd ? L.kwm[mine] + half : L.kwm[kWave + 1]) = kw8;
      *reinterpret_cast<lp_quad *>(L.msg[mine] + half + (bnd ? 8 : 0)) =
          lp_quad{st[0], st[1], st[2], st[3]};
#pragma unroll
      for (int t = 0; t < 4; ++t) st[t] = bnd ? sg[t] : st[t];
    } else {
      *reinterpret_cast<lp_quad *>(L.msg[mine] + half) = lp_quad{st[0], st[1], st[2], st[3]};
    }
    // while the LDS writes complete
    start();
#pragma unroll
    for (int t = 2; t < 8; ++t) asm volatile("" : "+v"(kw[t]));
    __syncthreads();
  }
}

template <int MODE>
__global__ __launch_bounds__(4 * kWave) void k_chains_lp(ChainArgs a) {
  __shared__ __align__(16) LpLds L;
  lp_group<MODE>(a, blockIdx.x, L);
}

// Large ordered batches: the first `lp_groups` workgroups run the lane-pair
// path on the longest requests (the batch is ordered longest first), so
// that the longest chains finish sooner; the remaining workgroups run
// one lane per request on the rest.  Both in one launch, 256 lanes per
// workgroup.
// Where the rest's first request is as long as the longest, the lane pairs shorten
// nothing that the batch waits for, and take CUs that the rest would fill:
// then one lane per request for all of them (65,536 chains of 32 blocks 262 ->
// 206 us, 131,072 433 -> 382).
//
// Two workgroups share a CU, the second of them 256 (second_from) after the first.
// These second ones take their places in reverse, so that the CU with the longest
// first requests gets the shortest second ones; places past the batch's end have
// nothing to do.  (131,072 chains of up to 80 blocks 587 -> 444 us, 250,000
// lognormal ones 1,136 -> 1,075; with one workgroup per CU, the next one to whichever
// CU was free, 511 and 1,074.  Where the second ones are no more than the lane-pair
// workgroups, whose waves go first, they stay beside these: 65,536 lognormal prompts
// 5,120 us, in reverse 5,160.)
template <int MODE>
__global__ __launch_bounds__(256) void k_chains_mixed(ChainArgs a, int32_t lp_groups) {
  __shared__ __align__(16) LpLds L;
  if (*a.even) lp_groups = 0;
  int32_t place = blockIdx.x;
  if (a.second_from > 0 && place >= a.second_from && place < 2 * a.second_from)
    place = 3 * a.second_from - 1 - place;
  if (place < lp_groups)
    lp_group<MODE>(a, place, L);
  else
    single_chain<MODE>(a, (int64_t)lp_groups * kWave + (int64_t)(place - lp_groups) * 256 + threadIdx.x);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

static int cu_lds_bytes() {
  int dev = 0, v = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) !=
          hipSuccess ||
      v <= 0)
    v = 160 * 1024;
  return v;
}

// Dynamic LDS of a lane-pair workgroup so that at most `per_cu` of them
// share a CU.
static size_t lp_lds_reserve(int per_cu) {
  const size_t cu = (size_t)cu_lds_bytes();
  const size_t want = per_cu == 1 ? cu / 2 + 4096 : cu / 2 - 1024;
  return want > sizeof(LpLds) ? want - sizeof(LpLds) : 0;
}

// Lane-pair workgroups per CU for a batch of n requests: the lane-pair
// kernel shortens every chain but needs four waves per 64 requests, so it
// runs while the batch fits in one or two workgroups per CU (latency-bound
// batches); larger batches keep every SIMD busy with the single-wave kernel
// (0).
static int lp_slots(int32_t n) {
  if (n <= 0) return 0;
  const int64_t groups = ceil_div(n, (int64_t)kWave);
  const int64_t cus = device_cu_count();
  if (groups <= cus) return 1;
  if (groups <= 2 * cus) return 2;
  return 0;
}

int device_cu_count() {
  static std::mutex mu;
  static std::vector<int> cus;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  std::lock_guard<std::mutex> g(mu);
  if ((int)cus.size() <= dev) cus.resize(dev + 1, 0);
  if (cus[dev] == 0) {
    int v = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        v <= 0)
      v = 256;
    cus[dev] = v;
  }
  return cus[dev];
}

int stream_scratch(hipStream_t s, size_t bytes, void **ptr, std::unique_lock<std::mutex> &lk) {
  static std::mutex mu;
  // keyed by device and stream; hipStreamPerThread names a different stream
  // in every host thread, so the thread is part of its key
  using Key = std::tuple<int, hipStream_t, std::thread::id>;
  static std::map<Key, std::pair<void *, size_t>> bufs;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return KVGOV_E_HIP;
  const std::thread::id tid =
      s == hipStreamPerThread ? std::this_thread::get_id() : std::thread::id();
  lk = std::unique_lock<std::mutex>(mu);
  std::pair<void *, size_t> &b = bufs[Key(dev, s, tid)];
  if (b.second < bytes) {
    constexpr size_t kGrain = 64 * 1024;
    const size_t cap = (std::max(bytes, 2 * b.second) + kGrain - 1) / kGrain * kGrain;
    if (b.first) {
      // earlier calls on s may still read the old buffer
      const bool ok = hipStreamSynchronize(s) == hipSuccess && hipFree(b.first) == hipSuccess;
      b = {nullptr, 0};
      if (!ok) {
        lk.unlock();
        return KVGOV_E_HIP;
      }
    }
    void *p = nullptr;
    if (hipMalloc(&p, cap) != hipSuccess) {
      (void)hipGetLastError();  // not left for the next launch check
      lk.unlock();
      return KVGOV_E_NOMEM;
    }
    b = {p, cap};
  }
  *ptr = b.first;
  return KVGOV_OK;
}

// Scratch of the allocation-free hashing entry point: the longest-first
// order of a batch (histogram, then the order), order_scratch_ints(n) int32 for
// n up to KVGOV_NOALLOC_MAX_REQUESTS.  One copy per device, held until the
// process ends; host code reaches it only through the address that
// hipGetSymbolAddress returns on that device (the array's name is a host
// stand-in, not a device address).
constexpr int64_t kNoAllocScratchInts = order_scratch_ints(KVGOV_NOALLOC_MAX_REQUESTS);
static __device__ __align__(256) int32_t scratch[kNoAllocScratchInts];

// Device address of `scratch` on the current device, looked up once per
// device; NULL if the lookup fails.
static int32_t *noalloc_scratch() {
  static std::mutex mu;
  static std::vector<int32_t *> ptrs;
  static std::vector<char> looked_up;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return nullptr;
  std::lock_guard<std::mutex> g(mu);
  if ((int)ptrs.size() <= dev) {
    ptrs.resize(dev + 1, nullptr);
    looked_up.resize(dev + 1, 0);
  }
  if (!looked_up[dev]) {
    int32_t *ptr = nullptr;
    if (hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch)) != hipSuccess)
      return nullptr;  // not cached: a later call tries again
    ptrs[dev] = ptr;
    looked_up[dev] = 1;
  }
  return ptrs[dev];
}

}  // namespace kvgov

using namespace kvgov;

extern "C" {

const char *kvgov_strerror(int code) {
  switch (code) {
    case KVGOV_OK: return "ok";
    case KVGOV_E_INVAL: return "invalid argument";
    case KVGOV_E_UNSUPPORTED: return "unsupported argument (block size 16 and keys up to 64 bytes)";
    case KVGOV_E_OFFSETS: return "offsets not monotone, out of bounds, or not matching len // 16";
    case KVGOV_E_BOUNDARY: return "boundary_tok outside [0, len]";
    case KVGOV_E_PRINCIPAL: return "principal index outside [0, P)";
    case KVGOV_E_FULL: return "cache table full";
    case KVGOV_E_HIP: return "HIP runtime error";
    case KVGOV_E_NOMEM: return "device allocation failed";
    case KVGOV_E_CAPACITY: return "export buffer too small";
    case KVGOV_E_DEVICE: return "cache used with a different current device";
    case KVGOV_E_INTERNAL:
      return "internal invariant failed inside a kernel (bounded wait or scratch contents)";
    case KVGOV_E_TOO_LARGE:
      return "batch above KVGOV_NOALLOC_MAX_REQUESTS requests (allocation-free entry point)";
    default: return "unknown error code";
  }
}

int kvgov_version(void) { return (1 << 16) | 0; }

// One compression from the initial value on the host (salts: the blocks that
// hold K alone).  w is overwritten.
static void host_compress_iv(uint32_t out[8], uint32_t w[16]) {
  uint32_t s[8];
  for (int i = 0; i < 8; ++i) s[i] = kSha.H0[i];
  for (int t = 0; t < 64; ++t) {
    if (t >= 16) {
      const uint32_t a = w[(t - 2) & 15], b = w[(t - 15) & 15];
      w[t & 15] += (c_rotr(a, 17) ^ c_rotr(a, 19) ^ (a >> 10)) + w[(t - 7) & 15] +
                   (c_rotr(b, 7) ^ c_rotr(b, 18) ^ (b >> 3));
    }
    const uint32_t e = s[4], a = s[0];
    const uint32_t t1 = s[7] + (c_rotr(e, 6) ^ c_rotr(e, 11) ^ c_rotr(e, 25)) +
                        ((e & s[5]) ^ (~e & s[6])) + kSha.K[t] + w[t & 15];
    const uint32_t t2 = (c_rotr(a, 2) ^ c_rotr(a, 13) ^ c_rotr(a, 22)) +
                        ((a & s[1]) ^ (a & s[2]) ^ (s[1] & s[2]));
    for (int i = 7; i > 0; --i) s[i] = s[i - 1];
    s[4] += t1;
    s[0] = t1 + t2;
  }
  for (int i = 0; i < 8; ++i) out[i] = kSha.H0[i] + s[i];
  volatile uint32_t *wipe = s;
  for (int i = 0; i < 8; ++i) wipe[i] = 0;
}

int kvgov_salts(const uint8_t *K, size_t K_len, const uint8_t *principal_ids, int32_t id_len,
                int32_t P, uint8_t *salts, void *stream) {
  if (!K || K_len == 0 || P < 0 || id_len < 0 || id_len > KVGOV_MAX_ID_BYTES)
    return KVGOV_E_INVAL;
  if (K_len > KVGOV_MAX_KEY_BYTES) return KVGOV_E_UNSUPPORTED;
  if (P > 0 && (!salts || (!principal_ids && id_len > 0))) return KVGOV_E_INVAL;
  if (P > 0 && (reinterpret_cast<uintptr_t>(salts) & 3)) return KVGOV_E_INVAL;
  if (P == 0) return KVGOV_OK;
  SaltArgs a{};
  uint32_t key[16] = {}, w[16];
  for (size_t i = 0; i < K_len; ++i) key[i / 4] |= (uint32_t)K[i] << (24 - 8 * (i % 4));
  for (int i = 0; i < 16; ++i) w[i] = key[i] ^ 0x36363636u;
  host_compress_iv(a.inner, w);
  for (int i = 0; i < 16; ++i) w[i] = key[i] ^ 0x5c5c5c5cu;
  host_compress_iv(a.outer, w);
  a.ids = principal_ids;
  a.id_len = id_len;
  a.P = P;
  a.salts = salts;
  hipLaunchKernelGGL(k_salts, dim3((unsigned)ceil_div(P, kWave)), dim3(kWave), 0,
                     as_stream(stream), a);
  const int rc = launch_status();
  // the kernel argument was copied at launch
  volatile uint32_t *wipe[4] = {key, w, a.inner, a.outer};
  for (int k = 0; k < 4; ++k)
    for (int i = 0; i < (k < 2 ? 16 : 8); ++i) wipe[k][i] = 0;
  return rc;
}

// Batches whose offsets take one launch (see k_blk_write): calls in a row take
// 7.1 us at 4096 requests against 9.9 us in two launches (12.6 us in the three
// that this was), 8.3 against 9.8 at 16,384, 11.4 against 10.0 at 32,768.
constexpr int64_t kScanAlone = 16384;

static int block_offsets_impl(const int64_t *tok_offsets, const int32_t *start, int32_t n,
                              int32_t block_size, int64_t *blk_offsets, int32_t *status,
                              void *stream) {
  if (!tok_offsets || !blk_offsets || !status || n < 0) return KVGOV_E_INVAL;
  if (block_size != KVGOV_BLOCK_SIZE) return KVGOV_E_UNSUPPORTED;
  hipStream_t s = as_stream(stream);
  if (n <= kScanAlone) {
    const unsigned tiles = (unsigned)std::max<int64_t>(1, ceil_div(n, kScanStep));
    hipLaunchKernelGGL(k_blk_write, dim3(tiles), dim3(kScanThreads), 0, s, tok_offsets, start, n,
                       (int64_t)kScanStep, nullptr, blk_offsets, status);
    return launch_status();
  }
  // at most 4096 workgroups, whose sums the second launch adds up again
  const int64_t tile = ceil_div(n, (int64_t)kScanStep * 4096) * kScanStep;
  const int64_t tiles = ceil_div(n, tile);
  std::unique_lock<std::mutex> lk;
  void *scratch_p = nullptr;
  const int src = stream_scratch(s, (size_t)tiles * sizeof(int64_t), &scratch_p, lk);
  if (src != KVGOV_OK) return src;
  int64_t *partial = static_cast<int64_t *>(scratch_p);
  hipLaunchKernelGGL(k_blk_partial, dim3((unsigned)tiles), dim3(kScanThreads), 0, s,
                     tok_offsets, start, n, tile, partial, status);
  hipLaunchKernelGGL(k_blk_write, dim3((unsigned)tiles), dim3(kScanThreads), 0, s, tok_offsets,
                     start, n, tile, partial, blk_offsets, status);
  return launch_status();
}

int kvgov_block_offsets(const int64_t *tok_offsets, int32_t n, int32_t block_size,
                        int64_t *blk_offsets, int32_t *status, void *stream) {
  return block_offsets_impl(tok_offsets, nullptr, n, block_size, blk_offsets, status, stream);
}

int kvgov_resume_offsets(const int64_t *tok_offsets, const int32_t *start_block, int32_t n,
                         int32_t block_size, int64_t *blk_offsets, int32_t *status,
                         void *stream) {
  if (n > 0 && !start_block) return KVGOV_E_INVAL;
  return block_offsets_impl(tok_offsets, start_block, n, block_size, blk_offsets, status, stream);
}

// Longest-first order of a batch's requests (counting sort of their block
// counts) in `buf`: order_scratch_ints(n) int32 (the histogram, whether the
// longest lp_requests are like the rest, then the order).  Returns the order.
static const int32_t *order_requests(const int64_t *blk_offsets, int32_t n, int32_t lp_requests,
                                     int32_t *buf, int32_t *status, hipStream_t s) {
  int32_t *hist = buf;
  int32_t *order = buf + order_scratch_ints(0);
  hipLaunchKernelGGL(k_fill_i32, dim3(kOrderBuckets / 256), dim3(256), 0, s, hist,
                     (int64_t)kOrderBuckets, 0);
  const dim3 tiles((unsigned)ceil_div(n, kOrderTile));
  hipLaunchKernelGGL(k_order_hist, tiles, dim3(kOrderThreads), 0, s, blk_offsets, n, hist);
  hipLaunchKernelGGL(k_order_scan, dim3(1), dim3(256), 0, s, hist, lp_requests,
                     buf + kOrderBuckets);
  hipLaunchKernelGGL(k_order_scatter, tiles, dim3(kOrderThreads), 0, s, blk_offsets, n, hist,
                     order, status);
  return order;
}

// Events the next chain call of this host thread records around its chain
// kernel (kvgov_time_next_chain_kernel); taken and cleared by that call.
static thread_local hipEvent_t t_chain_events[2] = {nullptr, nullptr};

static int hash_chains_impl(const int32_t *tokens, int64_t n_tokens, const int64_t *tok_offsets,
                            int32_t n, const int32_t *principal, const uint8_t *salts, int32_t P,
                            int32_t mode, const int32_t *boundary_tok, int32_t block_size,
                            const int32_t *start, const uint8_t *parents,
                            const int64_t *blk_offsets, uint8_t *hashes, int64_t n_blocks,
                            int32_t *status, void *stream, bool noalloc) {
  const hipEvent_t ev_start = t_chain_events[0], ev_end = t_chain_events[1];
  t_chain_events[0] = t_chain_events[1] = nullptr;
  if (n < 0 || n_tokens < 0 || n_blocks < 0 || !status) return KVGOV_E_INVAL;
  if (mode != KVGOV_NONE && mode != KVGOV_ROOT && mode != KVGOV_BOUNDARY) return KVGOV_E_INVAL;
  if (block_size != KVGOV_BLOCK_SIZE) return KVGOV_E_UNSUPPORTED;
  if (n == 0) return KVGOV_OK;
  if (!tok_offsets || !blk_offsets || (n_tokens > 0 && !tokens) || (n_blocks > 0 && !hashes))
    return KVGOV_E_INVAL;
  if ((reinterpret_cast<uintptr_t>(tokens) & 3) || (reinterpret_cast<uintptr_t>(hashes) & 3))
    return KVGOV_E_INVAL;
  if (mode != KVGOV_NONE && (!principal || !salts || P <= 0)) return KVGOV_E_INVAL;
  if (mode == KVGOV_BOUNDARY && !boundary_tok) return KVGOV_E_INVAL;
  hipStream_t s = as_stream(stream);

  ChainArgs a{};
  a.tokens = tokens;
  a.n_tokens = n_tokens;
  a.tok_offsets = tok_offsets;
  a.blk_offsets = blk_offsets;
  a.principal = principal;
  a.salts = salts;
  a.P = P;
  a.n = n;
  a.boundary_tok = boundary_tok;
  a.hashes = hashes;
  a.n_blocks = n_blocks;
  a.status = status;
  a.order = nullptr;
  a.start = start;
  a.parents = parents;

  // Launch shape.  A chain wave is bound by its SIMD's issue rate, so it
  // should never share a SIMD while others sit idle.  The dispatcher stacks
  // the waves of concurrent launches on the same SIMDs, and the older wave
  // then takes nearly every issue slot, so the workgroups reserve LDS (unused
  // beyond the kernel's own) to bound how many share a CU.
  const int slots = lp_slots(n);
  std::unique_lock<std::mutex> lk;  // held while the ordered launch is enqueued
  if (slots) {
    // lane pairs: two rounds waves and two schedule waves per 64 requests,
    // one or two workgroups per CU; every request of the batch is resident
    // from the start, so the order of the requests does not matter
    const dim3 grid((unsigned)ceil_div(n, kWave));
    const size_t lds = lp_lds_reserve(slots);
    if (ev_start && hipEventRecord(ev_start, s) != hipSuccess) return KVGOV_E_HIP;
    const dim3 block(4 * kWave);
    a.second_from = slots == 2 ? device_cu_count() : 0;
    switch (mode) {
      case KVGOV_NONE: hipLaunchKernelGGL(k_chains_lp<KVGOV_NONE>, grid, block, lds, s, a); break;
      case KVGOV_ROOT: hipLaunchKernelGGL(k_chains_lp<KVGOV_ROOT>, grid, block, lds, s, a); break;
      default: hipLaunchKernelGGL(k_chains_lp<KVGOV_BOUNDARY>, grid, block, lds, s, a); break;
    }
  } else {
    // More than two lane-pair workgroups per CU: the batch has at least as
    // many waves (one lane per request) as the chip has SIMDs, and it is
    // ordered longest first (counting sort of block counts).  The longest
    // requests then run on lane-pair workgroups (one eighth of the CUs), the
    // rest one lane per request.
    // The ordering scratch: the library's fixed array for the
    // allocation-free entry point, else the stream's own scratch.
    int32_t *buf = nullptr;
    if (noalloc) {
      buf = noalloc_scratch();
      if (!buf) return KVGOV_E_HIP;
    } else {
      const size_t bytes = sizeof(int32_t) * (size_t)order_scratch_ints(n);
      void *p = nullptr;
      const int src = stream_scratch(s, bytes, &p, lk);
      if (src != KVGOV_OK) return src;
      buf = static_cast<int32_t *>(p);
    }
    const int32_t lp_groups = std::max(1, device_cu_count() / 8);
    a.order = order_requests(blk_offsets, n, lp_groups * kWave, buf, status, s);
    a.even = buf + kOrderBuckets;
    const int64_t rest = std::max<int64_t>(0, (int64_t)n - (int64_t)lp_groups * kWave);
    int64_t groups = lp_groups + ceil_div(rest, 4 * kWave);
    const int32_t cus = device_cu_count();
    if (groups > cus + lp_groups) {  // second ones beside more than the lane pairs
      a.second_from = cus;
      groups = std::max(groups, (int64_t)2 * cus);
    }
    const dim3 grid((unsigned)groups), block(4 * kWave);
    // two workgroups per CU: a second wave on each SIMD issues while the first
    // waits (250,000 chains of 32 blocks 0.695 -> 0.635 ms; one per CU was the
    // rule while a one-lane wave beside a lane-pair one slowed its chain, which
    // the rounds waves' priority prevents: 65,536 lognormal prompts 5.14 ->
    // 5.01 ms)
    const size_t lds = lp_lds_reserve(2);
    if (ev_start && hipEventRecord(ev_start, s) != hipSuccess) return KVGOV_E_HIP;
    switch (mode) {
      case KVGOV_NONE: hipLaunchKernelGGL(k_chains_mixed<KVGOV_NONE>, grid, block, lds, s, a, lp_groups); break;
      case KVGOV_ROOT: hipLaunchKernelGGL(k_chains_mixed<KVGOV_ROOT>, grid, block, lds, s, a, lp_groups); break;
      default: hipLaunchKernelGGL(k_chains_mixed<KVGOV_BOUNDARY>, grid, block, lds, s, a, lp_groups); break;
    }
  }
  int rc = launch_status();
  if (ev_end && hipEventRecord(ev_end, s) != hipSuccess && rc == KVGOV_OK) rc = KVGOV_E_HIP;
  return rc;
}

int kvgov_time_next_chain_kernel(void *start_event, void *end_event) {
  if ((start_event == nullptr) != (end_event == nullptr)) return KVGOV_E_INVAL;
  t_chain_events[0] = static_cast<hipEvent_t>(start_event);
  t_chain_events[1] = static_cast<hipEvent_t>(end_event);
  return KVGOV_OK;
}

int kvgov_hash_chains(const int32_t *tokens, int64_t n_tokens, const int64_t *tok_offsets,
                      int32_t n, const int32_t *principal, const uint8_t *salts, int32_t P,
                      int32_t mode, const int32_t *boundary_tok, int32_t block_size,
                      const int64_t *blk_offsets, uint8_t *hashes, int64_t n_blocks,
                      int32_t *status, void *stream) {
  return hash_chains_impl(tokens, n_tokens, tok_offsets, n, principal, salts, P, mode,
                          boundary_tok, block_size, nullptr, nullptr, blk_offsets, hashes,
                          n_blocks, status, stream, false);
}

int kvgov_hash_chains_noalloc(const int32_t *tokens, int64_t n_tokens,
                              const int64_t *tok_offsets, int32_t n, const int32_t *principal,
                              const uint8_t *salts, int32_t P, int32_t mode,
                              const int32_t *boundary_tok, int32_t block_size,
                              const int64_t *blk_offsets, uint8_t *hashes, int64_t n_blocks,
                              int32_t *status, void *stream) {
  if (n > KVGOV_NOALLOC_MAX_REQUESTS) return KVGOV_E_TOO_LARGE;
  return hash_chains_impl(tokens, n_tokens, tok_offsets, n, principal, salts, P, mode,
                          boundary_tok, block_size, nullptr, nullptr, blk_offsets, hashes,
                          n_blocks, status, stream, true);
}

int kvgov_hash_chains_resume(const int32_t *tokens, int64_t n_tokens, const int64_t *tok_offsets,
                             int32_t n, const int32_t *principal, const uint8_t *salts,
                             int32_t P, int32_t mode, const int32_t *boundary_tok,
                             int32_t block_size, const int32_t *start_block,
                             const uint8_t *parents, const int64_t *blk_offsets, uint8_t *hashes,
                             int64_t n_blocks, int32_t *status, void *stream) {
  if (n > 0 && (!start_block || !parents)) return KVGOV_E_INVAL;
  if (reinterpret_cast<uintptr_t>(parents) & 3) return KVGOV_E_INVAL;
  return hash_chains_impl(tokens, n_tokens, tok_offsets, n, principal, salts, P, mode,
                          boundary_tok, block_size, start_block, parents, blk_offsets, hashes,
                          n_blocks, status, stream, false);
}

}  // extern "C"
