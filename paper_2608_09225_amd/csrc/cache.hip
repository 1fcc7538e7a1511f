// Device-resident prefix-cache table: batched insert and first-miss lookup.
//
// Paper: a block prefix cache keys KV blocks by their chained block hash and
// resolves a request to the longest cached prefix, quantised to blocks; the
// prober learns the number of leading blocks matched (Sec. 2.1; Table
// tab:taxonomy, block prefix cache row).
//
// Layout (HBM):
//   keys [slots][32 B]  the stored keys; an empty slot holds 32 bytes 0xFF.
//                       Lookups read only this array, two slots (64 bytes of
//                       one line) at a time, and a probe sequence runs through
//                       the four slots of its 128-byte line before it leaves it.
//   tags [slots] u64    0 = empty, else (epoch << 32) | (claimant + 1): the
//                       insert call that claimed the slot and the index of the
//                       claiming key within that call's input.
//   meta                key count, per-call counters, latched error, and the
//                       tag and presence bit of the all-0xFF key, which cannot
//                       live in a slot because it is the empty pattern.
//
// Insert protocol (no fences, no waiting on other lanes).  A key walks its
// probe sequence; at each slot it reads the tag:
//   * empty          -> CAS the tag to (epoch, me); the winner writes the key
//                       into the slot and counts one new key.
//   * earlier epoch  -> the slot's key was written by an earlier kernel and is
//                       visible: compare all 256 bits.
//   * current epoch  -> the slot was claimed in this call; its key may not be
//                       written yet, so compare against the claimant's key in
//                       this call's input array instead.
// Equal -> already present, stop.  Otherwise move to the next slot.  Two
// copies of one key follow the same sequence and each slot changes state at
// most once, so exactly one copy claims a slot and the other finds it.
//
// Admission (lookup-then-insert in request order) runs the same insert and
// additionally lowers a slot claimed in the call to the smallest claiming
// row (atomicMin on the tag: the epoch bits are equal, so the minimum is the
// earliest row, i.e. the earliest request holding the key), and records per
// row which slot its key went to; a second kernel then decides per request
// what it sees: keys of earlier calls, and keys whose earliest row lies in an
// earlier request.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <new>

#include "table.h"

namespace kvgov {

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

// Arrays of a clear, in 16-byte units (a table has at least 16 slots): those of
// the table, and of the radix index that it belongs to.
struct FillArgs {
  u32x4 *ones[2];
  int64_t n_ones[2];
  u32x4 *zeros[3];
  int64_t n_zeros[3];
  CacheMeta *m;
};

// Bound by its writes.  Consecutive lanes write consecutive 16 bytes, four
// stores each: a clear of 2^20 slots 8.5 us and of 2^25 234 (a lane per slot,
// whose key is two stores of every other 16 bytes: 10.0 and 235; eight
// workgroups per CU that walk the arrays: 8.4 and 266).
__device__ __forceinline__ void fill(u32x4 *p, int64_t n, uint32_t v) {
  const u32x4 q = u32x4{v, v, v, v};
  const int64_t stride = (int64_t)gridDim.x * 1024;
  int64_t i = (int64_t)blockIdx.x * 1024 + threadIdx.x;
  for (; i + 768 < n; i += stride)
#pragma unroll
    for (int k = 0; k < 4; ++k) p[i + 256 * k] = q;
  for (int k = 0; k < 4; ++k)
    if (i + 256 * k < n) p[i + 256 * k] = q;
}

__global__ __launch_bounds__(256) void k_cache_fill(FillArgs a) {
  CacheMeta *m = a.m;
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < kCounterLanes; i += blockDim.x) {
      m->n_keys[i] = 0;
      m->new_keys[0][i] = 0;
      m->new_keys[1][i] = 0;
      m->n_edges[i] = 0;
    }
    if (threadIdx.x == 0) {
      m->exported = 0;
      m->erased = 0;
      m->marked = 0;
      m->radix_status = 0;
      m->ones_tag = 0;
      m->ones_rank = 0;
      m->status = 0;
      m->ones_present = 0;
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (a.n_ones[i]) fill(a.ones[i], a.n_ones[i], 0xFFFFFFFFu);
#pragma unroll
  for (int i = 0; i < 3; ++i)
    if (a.n_zeros[i]) fill(a.zeros[i], a.n_zeros[i], 0u);
}

// The depth of a key: its row within its request (clamped; only malformed
// interior offsets put it outside [0, n_blocks)).
__device__ __forceinline__ uint32_t row_depth(int64_t jj, int64_t n_blocks) {
  const int64_t most = n_blocks < 0x7FFFFFFF ? n_blocks : 0x7FFFFFFF;
  return (uint32_t)(jj < 0 ? 0 : (jj > most ? most : jj));
}

// Consecutive keys per wave chunk of k_chunk_insert.  Longer chunks mean fewer
// waves in flight at once, so that the copies of a key that many requests
// hold (a principal's shared prefix) reach its slot over a longer span and
// most of them find it claimed by a plain read instead of racing for it
// with compare-and-swaps on one address (measured: 256 beats 64, 128, 512; an
// admission of few rows takes shorter ones, see admit_chunk).
constexpr int kInsChunk = 256;

// The largest r in [0, n) with bo[r] <= f (bo non-decreasing in a valid
// batch; any answer in range is harmless otherwise, see k_chunk_insert).  Every
// lane of a wave searches the same f.
__device__ __forceinline__ int32_t find_request(const int64_t *bo, int32_t n, int64_t f) {
  int32_t a = 0, b = n - 1;
  while (a < b) {
    const int32_t mid = (a + b + 1) >> 1;
    if (bo[mid] <= f) a = mid; else b = mid - 1;
  }
  return a;
}

// Table sizes whose new keys are claimed without reading the tag first (see
// k_insert_req): where that gains by more than the spread at loads of 0.4 and 0.65.
// Batches of distinct keys that fill 0.4 of the table, read first / claimed first,
// us (from 2^21 slots with keys before tags): 2^18 slots 38.9 / 34.5, 2^19 50.4 /
// 45.2, 2^20 63.6 / 54.9, 2^21 80.9 / 78.3, 2^22 122 / 128, 2^23 338 / 308, 2^24
// 614 / 573; that fill 0.65: 2^20 140 / 132, 2^21 179 / 185, 2^22 240 / 258, 2^23
// 615 / 609.  Below 2^18 slots it gains by 2 to 3 us (2^17 37.7 / 34.3) and is
// not used.  Batches whose keys are there claim nothing, but their walk is slower
// with the claims' code in it: 2^20 40 / 41, 2^23 111 / 122, 2^24 236 / 257.  Past
// the home's bucket (with keys first, past the home) the slot is read again: where
// the table is fuller, the next slots are mostly taken (0.65 of 2^20 slots: 171 us
// with, 196 without).
__device__ __forceinline__ bool claims_first(uint64_t mask) {
  return mask >= (1ull << 23) - 1 || (mask >= (1ull << 18) - 1 && mask <= (1ull << 20) - 1);
}

// Insert walking the batch in chunks of `chunk` (a multiple of 64) consecutive rows
// per wave, 64 at a time: for batches whose requests are so long that a group per
// request would leave the chip idle (a flat key set given as one request), in
// the plain insert and as the admission's first half (ADMIT), which takes it for
// many short requests as well.  Before touching the
// table a key is compared with the key at the same block position of the
// previous request (requests that share a prefix - the same principal, or
// any principal below the boundary block - hold the same keys there): an
// equal earlier key makes this one a duplicate that needs no table access,
// so a prefix shared by thousands of requests costs a few table operations
// per key instead of thousands of atomics on one slot.  The request of each
// key comes from a window of 64 request starts (a search over lanes); the
// comparison is only an optimisation: skipping a key that equals an
// earlier key of the batch is always correct (the earlier one is inserted,
// or is itself a duplicate of an earlier one), and the compared position
// is checked to lie in the batch, so malformed interior offsets cannot
// cause a wrong result or an out-of-range read.  A row's request, and so
// its depth (its position in the request, which the recency rank holds),
// is exact: rows whose request lies past the window search for it.
//
// ADMIT: claims are lowered to the earliest row, and codes[f] records where
// row f's key went (kCodeDup for a key skipped as equal to the previous
// request's, which is in an earlier request by construction).
template <bool ADMIT>
__global__ __launch_bounds__(256) void k_chunk_insert(TableView t, const uint8_t *hashes,
                                                      const int64_t *blk_offsets, int32_t n,
                                                      int64_t n_blocks, uint32_t epoch,
                                                      uint32_t *codes, int chunk) {
  __shared__ uint32_t lds4[4];
  const int64_t lo = blk_offsets[0], hi = blk_offsets[n];
  const bool first = blockIdx.x == 0 && threadIdx.x == 0;
  if (blockIdx.x == 0 && threadIdx.x < kCounterLanes)
    t.meta->new_keys[(epoch + 1) & 1][threadIdx.x] = 0;  // counters of the next call
  if (lo < 0 || hi < lo || hi > n_blocks || hi - lo >= 0xFFFFFFFFll) {
    if (first) atomicCAS(&t.meta->status, 0, KVGOV_E_OFFSETS);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)gridDim.x * 4;
  const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  uint32_t added = 0;
  for (int64_t f0 = lo + wave * chunk; f0 < hi; f0 += waves * chunk) {
    const int64_t f1 = f0 + chunk < hi ? f0 + chunk : hi;
    int32_t rc = find_request(blk_offsets, n, f0);
    for (int64_t fb = f0; fb < f1; fb += 64) {
      // win[l] = start of request rc - 1 + l (clamped to [0, n])
      int32_t wi = rc - 1 + lane;
      wi = wi < 0 ? 0 : (wi > n ? n : wi);
      const int64_t win = blk_offsets[wi];
      const int64_t f = fb + lane;
      // pos: the largest l in [1, 63] with win[l] <= f
      int pos = 1;
#pragma unroll
      for (int step = 32; step >= 1; step >>= 1) {
        const int cand = pos + step;
        const int64_t v = __shfl(win, cand < 63 ? cand : 63, 64);
        if (cand <= 63 && v <= f) pos = cand;
      }
      int64_t b_r = __shfl(win, pos, 64);
      int64_t b_p = __shfl(win, pos - 1, 64);
      int32_t r = rc - 1 + pos;
      if (pos == 63) {
        // 64 rows can span more requests than the window reaches (requests
        // of one block or none): a row whose request starts past the window
        // finds it by binary search (its depth depends on it)
        const int32_t ne = rc + 63;
        if (ne < n && blk_offsets[ne] <= f) {
          r = find_request(blk_offsets, n, f);
          b_r = blk_offsets[r];
          b_p = blk_offsets[r - 1];
        }
      }
      if (f < f1) {
        const Key key = load_key(hashes + f * 32);
        bool dup = false;
        const int64_t jj = f - b_r;
        if (r >= 1 && jj >= 0 && jj < b_r - b_p && b_p + jj >= lo)
          dup = key_eq(key, load_key(hashes + (b_p + jj) * 32));
        uint32_t code = kCodeDup;
        const uint32_t depth = row_depth(jj, n_blocks);
        if (!dup) added += insert_key<ADMIT>(t, key, f, lo, hashes, epoch, &code, depth);
        if (ADMIT) codes[f] = code;
      }
      rc = __shfl(r, 63, 64);
    }
  }
  const uint32_t total = block_sum(added, lds4);
  if (threadIdx.x == 0 && total) {
    const int cl = blockIdx.x % kCounterLanes;
    atomicAdd(&t.meta->new_keys[epoch & 1][cl], (unsigned long long)total);
    atomicAdd(&t.meta->n_keys[cl], (unsigned long long)total);
  }
}

// The state of an insert by regions (below).
struct RegionState {
  uint32_t n_rest;  // rows in the rest list
  uint32_t bad;     // a malformed batch, or rows fewer than half of n_blocks
  // keys seen << 32 | of them repeated (or in the table), see k_region_sample: first
  // keys of evenly spread requests, and those chosen by the key; then rows
  unsigned long long spread, by_key, rows_spread, rows_by_key;
  // of the spread rows, those repeated alone
  unsigned long long rows_hot;

  // Does the batch go by requests?
  __device__ bool by_request() const {
    return bad || heads_repeat() || rows_repeat();
  }
  // Are first keys repeated, or in the table?
  __device__ bool heads_repeat() const { return repeats(spread, 8) || repeats(by_key, 8); }
  // Are other rows?
  __device__ bool rows_repeat() const { return repeats(rows_spread, 8) || repeats(rows_by_key, 160); }
  // Do few keys make up much of the batch?
  __device__ bool hot() const { return repeats(rows_hot, 8); }
  // one in `part` at least?
  static __device__ bool repeats(unsigned long long seen, uint32_t part) {
    return (seen & 0xFFFFFFFFu) * part > seen >> 32;
  }
};

// Lanes of an untracked admission up to which its groups take their rounds in turns.
constexpr int64_t kTurnLanes = 1 << 19;

// Rows of a request that its group of G lanes admits; the others are the walkers'
// (at least 64: of 64 consecutive rows, those past these are one request's).
template <int G>
constexpr int64_t kHeadRows = G < 16 ? 64 : 4 * G;

// Plain (set-union) insert with G lanes per request, which walk the
// request's rows G at a time.  Two comparisons keep keys that many requests
// share away from the table (a key skipped by either equals a row of the
// batch that lies before it, and the earliest row of any key is never
// skipped, so every key reaches the table):
//   * the previous request's row at the same depth (requests that share a
//     prefix and are adjacent, e.g. a prefix below the boundary block that
//     every request holds);
//   * the row at the same depth of an earlier request that starts with the
//     same key: the group's first lane inserts the request's first row
//     before the others start, and if the slot's tag names an earlier row
//     (the request that claimed the key, mostly the earliest one, since
//     workgroups start in request order) the group compares against the rows
//     that follow it.  Requests of one principal share the
//     root-salted prefix but are rarely adjacent.  (Lowering the tag to the
//     earliest first row with an atomic minimum, as admission does, measured
//     slower: 35.7 -> 36.6 us for the paper-shaped root-mode insert.)
// A key's rank holds its smallest depth, so on a table that tracks recency the
// second comparison stops at the end of that request, which a search of the
// offsets finds (the row past it lies in another request, at another depth).
// Without the second comparison, every request's prefix rows read and raised
// their keys' words: 66 us for the paper-shaped root-mode batch, 37 with it
// (46 for a second batch, whose prefix keys are of an earlier call: a tracked
// first row gives such a key this call's tag, so that later requests find an
// earlier one by it.  Untracked, reading the present keys costs less than the
// renewals: 20 against 25 us for a batch that is all present.)  Short requests save
// less by it than the search and the renewal cost, and their waves wait for those of
// the longer ones: on a table that tracks recency it is left out for requests of up
// to 8 rows and in batches of fewer than 16 on average (20,000 requests of 8 rows, 3
// of them one of 500 heads, present, 29 us and with it 32, of 16 rows, 6 of them
// heads, 41 and 40; 1 M lognormal ones of 3 on average, half of them 64 heads, 348
// and 435, present 213 and 276).
//
// Where the first key is new in this call, a chain's later keys are new as
// well, or of this call: these rows go to the compare-and-swap without reading
// the tag first, where that pays (claims_first).  The plain read fetches the
// tag's line into this XCD's cache, from which the other XCDs' claims take it
// again (270,000 random claims of 2^20 slots: 34 us with the read, 17
// without).  Rows that follow a key of an earlier call keep the read: they are
// mostly present (a batch that is all present: 20 us, 34 without the read).  So do
// a group's next rows once one was found (keys that are no chain's, 8 copies of
// each: 2^20 slots 48 us without this, 41 with, 2^23 214 and 162).
//
// KEYS: these rows look at a slot's key before its tag.  A present key then
// costs one line, not two, and a walk past other keys reads the line that holds
// them instead of their claimants' rows.  It pays where the tags are not cached as a
// whole, from 2^21 slots (tags first / keys first, us; P: all keys present, N:
// none, H: half): 2^20 slots, 270,000 keys N 39 / 43; 2^21, 1.05 M P 73 / 53, N
// 109 / 100, H 91 / 78; 2^22, 3.0 M P 230 / 171, N 333 / 297; 2^23, 5.9 M P 440
// / 324, N 783 / 681, H 585 / 480; 2^25, 8.4 M P 384 / 240, N 785 / 738, H 631 /
// 574.
// Each request inserts the rows [blk_offsets[r], blk_offsets[r + 1]) cut to
// the batch [blk_offsets[0], blk_offsets[n]); requests whose offsets are out
// of order insert nothing.  With non-decreasing offsets that is every row
// once.  Otherwise every row of the batch still lies in some request's
// range (take the last r with blk_offsets[r] <= row), so the table receives
// exactly the batch's keys.
//
// ADMIT: claims are lowered to the earliest row, tags of earlier calls stay (a
// key's tag says that it was there before the call), and codes[f] records
// where row f's key went, kCodeDup for a skipped row.  Its equal lies in an
// earlier request: the previous one, or, by the second comparison, a row
// before this request's first (a first key claimed by a later request is
// lowered, and that group compares with nothing).  (The chunked walk, which
// admission took for every batch before it had the second comparison: 73 us for
// 8192 requests of two paper-shaped batches; now 46.)  A group admits the first
// kHeadRows of its request; the workgroups from `walkers` on take the batch in
// chunks and admit the rows past them (admit_tails).  Without these a long
// request was a chain of rounds of one wave while the chip idled: 4096 lognormal
// prompts of up to 2048 blocks 276 us, now 120; 16 requests of 2048 rows 187 / 65;
// 64, of which one has 8192 rows, 376 / 124 (by chunks alone 110, 64 and 125).
// Where no request is that long they cost 0 to 4 us (4096 requests of 166 rows 44 /
// 48, by chunks alone 62).
//
// Requests that share a prefix and run at once would come to each of its slots
// together, and all with an atomic (a tag to lower, a recency word to raise); later
// ones find by a read that there is nothing left to do.  So a group starts its
// rounds at one that its number chooses: 4096 requests of 64 prefixes, tracked, new
// 55 / 51 us, present 70 / 58; 800 of 5, 300 rows each, untracked 52 / 42, tracked
// and present 59 / 47.  Untracked batches of more groups than run at once (kTurnLanes)
// keep the order, in which neighbours find their shared rows in the caches (60,000
// requests of 190 rows 414 us, in turns 425).
//
// admit_tails: a wave looks for its four windows' requests side by side, and a
// window that holds rows past a head holds them of the request of its first row
// alone (heads are as long as a window).  That request's first key mostly has its
// tag by then; where not, the second comparison is left out.
template <int G, bool TRACK>
__device__ __forceinline__ uint32_t admit_tails(const TableView &t, const uint8_t *hashes,
                                                const int64_t *blk_offsets, int32_t n,
                                                int64_t n_blocks, uint32_t epoch, uint32_t *codes,
                                                int64_t lo, int64_t hi, uint32_t walkers) {
  const int lane = threadIdx.x & 63;
  const int64_t waves = (int64_t)(gridDim.x - walkers) * 4;
  const int64_t wave = (int64_t)(blockIdx.x - walkers) * 4 + (threadIdx.x >> 6);
  constexpr int kWindow = 64, kPart = kWave * kWindow / kInsChunk;  // lanes per window's search
  uint32_t added = 0;
  int32_t known = -1;
  int64_t b_p = 0, n_p = 0, g0 = -1, g1 = 0;  // of request `known` (see k_insert_req)
  bool fresh = false;
  for (int64_t f0 = lo + wave * kInsChunk; f0 < hi; f0 += waves * kInsChunk) {
    // the windows' first rows' requests (find_request), side by side
    const int64_t w0 = f0 + (int64_t)(lane / kPart) * kWindow;
    int32_t a = 0;
    for (int32_t len = n, step; len > 1; len = step) {
      step = (len + kPart - 1) / kPart;
      const int64_t at = a + (int64_t)(lane % kPart) * step;
      const uint64_t le = __ballot(at < n && blk_offsets[at < n ? at : 0] <= w0) >>
                          (lane / kPart * kPart) & ((1u << kPart) - 1);
      a += (31 - __builtin_clz((uint32_t)le | 1u)) * step;
    }
    // and their rows past the head, if any (out of order: its group's)
    const int64_t wb = blk_offsets[a], we = blk_offsets[a + 1];
    const int64_t w1 = wb + kHeadRows<G> > w0 ? wb + kHeadRows<G> : w0;
    const int64_t w2 = we < w0 + kWindow ? we : w0 + kWindow;
    for (uint64_t todo = __ballot(wb >= lo && we <= hi && w1 < w2 && lane % kPart == 0); todo;
         todo &= todo - 1) {
      const int from = __builtin_ctzll(todo);
      const int32_t r = __shfl(a, from, 64);
      const int64_t b_r = __shfl(wb, from, 64), fb = __shfl(w0, from, 64);
      const int64_t first = __shfl(w1, from, 64), end = __shfl(w2, from, 64);
      if (r != known) {
        known = r;
        b_p = r >= 1 ? blk_offsets[r - 1] : 0;
        n_p = r >= 1 && b_p >= lo && b_p <= b_r ? b_r - b_p : 0;
        const Key head = load_key(hashes + b_r * 32);
        const int64_t slot = find_slot(t, head);
        const unsigned long long tag =
            slot >= 0 ? t.tags[slot] : (slot == -2 ? t.meta->ones_tag : 0ull);
        const bool now = (uint32_t)(tag >> 32) == epoch;
        const int64_t c = lo + (int64_t)(tag & 0xFFFFFFFFull) - 1;
        fresh = !TRACK && now && claims_first(t.mask);
        g0 = now && c >= lo && c < b_r ? c : -1;
        g1 = b_r;
        if (TRACK && g0 >= 0) {
          const int32_t q = find_request(blk_offsets, n, g0);
          if (blk_offsets[q] != g0) g0 = -1;
          if (blk_offsets[q + 1] < g1) g1 = blk_offsets[q + 1];
        }
      }
      const int64_t f = fb + lane;
      if (f >= first && f < end) {
        const int64_t jj = f - b_r;
        const Key key = load_key(hashes + f * 32);
        bool dup = jj < n_p && key_eq(key, load_key(hashes + (b_p + jj) * 32));
        if (!dup && g0 >= 0 && g0 + jj < g1) dup = key_eq(key, load_key(hashes + (g0 + jj) * 32));
        uint32_t code = kCodeDup;
        if (!dup)
          added += insert_key<true>(t, key, f, lo, hashes, epoch, &code,
                                    TRACK ? row_depth(jj, n_blocks) : kNoDepth, nullptr, false, fresh);
        codes[f] = code;
      }
    }
  }
  return added;
}

template <int G, bool ADMIT, bool TRACK, bool KEYS>
__global__ __launch_bounds__(256) void k_insert_req(TableView t, const uint8_t *hashes,
                                                    const int64_t *blk_offsets, int32_t n,
                                                    int64_t n_blocks, uint32_t epoch,
                                                    uint32_t *codes, uint32_t walkers,
                                                    const RegionState *st) {
  __shared__ uint32_t lds4[4];
  // a batch that may go by regions: does it, or is it the other launch's?
  if (st && (!st->by_request() || st->hot() == KEYS)) return;
  const bool repeats = st && !st->heads_repeat() && st->rows_repeat();  // no chains
  const int64_t lo = blk_offsets[0], hi = blk_offsets[n];
  if (blockIdx.x == 0 && threadIdx.x < kCounterLanes)
    t.meta->new_keys[(epoch + 1) & 1][threadIdx.x] = 0;  // counters of the next call
  if (lo < 0 || hi < lo || hi > n_blocks || hi - lo >= 0xFFFFFFFFll) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicCAS(&t.meta->status, 0, KVGOV_E_OFFSETS);
    return;
  }
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t r = gid / G;
  const int sub = (int)(gid % G);
  const int lane = threadIdx.x & 63;
  const int base = lane & ~(G - 1);
  uint32_t added = 0;
  // groups never straddle r < n (256 % G == 0); the block sum below needs
  // every thread, so out-of-range groups only skip the work
  if (ADMIT && blockIdx.x >= walkers) {
    added = admit_tails<G, TRACK>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, lo, hi,
                                  walkers);
  } else if (r < n) {
    const int64_t b_r = blk_offsets[r], b_e = blk_offsets[r + 1];
    const int64_t b_p = r >= 1 ? blk_offsets[r - 1] : 0;
    const int64_t b0 = b_r > lo ? b_r : lo;
    int64_t b1 = b_e < hi ? b_e : hi;
    if (ADMIT && b_r >= lo && b_e <= hi && b0 + kHeadRows<G> < b1) b1 = b0 + kHeadRows<G>;
    // the previous request's rows, when its range is in order and in the batch
    const int64_t n_p = r >= 1 && b_p >= lo && b_p <= b_r ? b_r - b_p : 0;
    if (b0 < b1) {
      // first row, by the group's first lane
      int64_t g0 = -1, g1 = hi;  // the earlier request's rows
      int fresh = 0;             // the first key is new in this call
      // the second comparison is made
      const bool seek = !TRACK || (b1 - b0 > 8 && n_blocks >= (int64_t)n * 16);
      if (sub == 0) {
        const int64_t jj = b0 - b_r;
        const Key key = load_key(hashes + b0 * 32);
        const bool dup = jj < n_p && key_eq(key, load_key(hashes + (b_p + jj) * 32));
        uint32_t code = kCodeDup;
        if (!dup) {
          unsigned long long claim = 0;
          added += insert_key<ADMIT>(t, key, b0, lo, hashes, epoch, &code,
                                     TRACK ? row_depth(jj, n_blocks) : kNoDepth, &claim,
                                     TRACK && !ADMIT && seek);
          fresh = !TRACK && !repeats && claims_first(t.mask) && (uint32_t)(claim >> 32) == epoch;
          const int64_t c = lo + (int64_t)(claim & 0xFFFFFFFFull) - 1;
          if (jj == 0 && (uint32_t)(claim >> 32) == epoch && c >= lo && c < b0 &&
              seek) {
            g0 = c;
            if (TRACK) {
              const int32_t q = find_request(blk_offsets, n, c);
              g1 = blk_offsets[q + 1] < hi ? blk_offsets[q + 1] : hi;
              if (blk_offsets[q] != c) g0 = -1;
            }
            if (ADMIT && g1 > b0) g1 = b0;
          }
        }
        if (ADMIT) codes[b0] = code;
      }
      g0 = __shfl(g0, base, 64);
      fresh = __shfl(fresh, base, 64);
      if (TRACK || ADMIT) g1 = __shfl(g1, base, 64);
      const int64_t rounds = (b1 - b0 + G - 2) / G;
      const int64_t turn =
          ADMIT && (TRACK || (int64_t)n * G <= kTurnLanes) && rounds > 1 ? (uint32_t)r % (uint32_t)rounds : 0;
      for (int64_t k = 0; k < rounds; ++k) {
        const int64_t at = k + turn < rounds ? k + turn : k + turn - rounds;
        const int64_t f = b0 + 1 + at * G + sub;
        if (f >= b1) continue;
        const int64_t jj = f - b_r;
        const Key key = load_key(hashes + f * 32);
        bool dup = jj < n_p && key_eq(key, load_key(hashes + (b_p + jj) * 32));
        if (!dup && g0 >= 0 && (!(TRACK || ADMIT) || g0 + jj < g1))
          dup = key_eq(key, load_key(hashes + (g0 + jj) * 32));
        uint32_t code = kCodeDup;
        uint32_t got = 1;
        if (!dup) {
          got = insert_key<ADMIT, KEYS>(t, key, f, lo, hashes, epoch, &code,
                                        TRACK ? row_depth(jj, n_blocks) : kNoDepth, nullptr, false,
                                        fresh != 0);
          added += got;
        }
        if (ADMIT) codes[f] = code;
        // a row that was there: no chain, or one that goes on as another's
        if (!TRACK && (__ballot(got == 0) & group_mask<G>(base))) fresh = 0;
      }
    }
  }
  const uint32_t total = block_sum(added, lds4);
  if (threadIdx.x == 0 && total) {
    const int cl = blockIdx.x % kCounterLanes;
    atomicAdd(&t.meta->new_keys[epoch & 1][cl], (unsigned long long)total);
    atomicAdd(&t.meta->n_keys[cl], (unsigned long long)total);
  }
}

// ---------------------------------------------------------------------------
// insert by regions: very large batches of new keys
// ---------------------------------------------------------------------------
//
// A key inserted on its own moves, at random places, its tag's line in and out
// and its 32 bytes, behind a compare-and-swap that waits for the line: 13.7 M
// new keys into 2^25 slots take k_insert_req 1.47 ms.  Taken region by region
// the tags are read once, in order, and claimed in LDS; what is moved instead
// is one entry of 8 bytes per row, to its region's list and back, and one
// random read of the row's key: 200 + 820 us, of which the 2.65 GB read and
// 0.66 GB written by k_region_insert are 670 us at a copy's rate (the random
// read fetches 128 bytes for each key's 32).
//   k_region_clear    counters, lists and sets of this call
//   k_region_sample   a look at the requests' first keys and at some rows: where
//                     many of them are shared, or in the table already, or the
//                     rows are fewer than half of n_blocks, k_insert_req is the
//                     better one (it keeps such rows off the table by
//                     comparisons, and finds present keys with one read each)
//                     and the kernels below end at once; otherwise k_insert_req
//                     does
//   k_region_lists    rows to their regions' lists
//   k_region_insert   region by region
//   k_list_insert     by insert_key: what the lists had no room for (keys that
//                     come many times) and rows whose probe sequence leaves
//                     their region
constexpr int kRegionLog2 = 14;
constexpr int kListThreads = 1024;
constexpr int kListItems = 16;  // rows per thread
constexpr int kListRows = kListThreads * kListItems;
constexpr int kMaxRegions = 4096;
constexpr int kMaxListed = 65000;  // entries of a region: an index fits 16 bits
constexpr int kSampleSlots = 8192;
constexpr int kSampled = 1024;      // requests looked at, evenly spread
constexpr int kSampledByKey = 2048;  // about as many, chosen by their first key
constexpr int kSampleRows = 64;      // one row of so many
constexpr int kSampleSets = 4;

struct RegionArgs {
  TableView t;
  const uint8_t *hashes;
  const int64_t *blk_offsets;
  int32_t n;
  int64_t n_blocks;
  uint32_t epoch;
  RegionState *st;
  uint32_t *cursor;             // per region: rows listed (may exceed cap)
  unsigned long long *sample;   // kSampleSets sets of kSampleSlots hashes
  unsigned long long *entries;  // per region: cap entries, (print << 46) | (home within the
                                // region << 32) | row; prints have 16 bits
  uint32_t *rest;               // rows for k_list_insert
  uint32_t cap;
  uint32_t regions;
  uint32_t key_mask, row_mask;  // of the hash bits that choose a request by its first key, a row by its
};

// The batch's rows, or none (an empty or malformed batch).
__device__ __forceinline__ bool region_rows(const RegionArgs &a, int64_t &lo, int64_t &hi) {
  lo = a.blk_offsets[0];
  hi = a.blk_offsets[a.n];
  return !(lo < 0 || hi < lo || hi > a.n_blocks || hi - lo >= 0xFFFFFFFFll);
}

__global__ __launch_bounds__(256) void k_region_clear(RegionArgs a) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < kSampleSets * kSampleSlots) a.sample[i] = 0;
  if (i < kMaxRegions) a.cursor[i] = 0;
  if (i == 0) *a.st = RegionState{};
}

// Was x in the set before?  (A set that is full where x belongs says no.)
__device__ __forceinline__ bool sample_twice(unsigned long long *set, uint64_t x) {
  x |= 1;  // never an empty slot; two keys that agree in 63 bits count as one
  uint32_t at = (uint32_t)(x >> 16) & (kSampleSlots - 1);  // not by the bits that choose
  for (int p = 0; p < 64; ++p, at = (at + 1) & (kSampleSlots - 1)) {
    // read first, from the caches: thousands of requests may hold one key
    unsigned long long was = set[at];
    if (was == 0) was = atomicCAS(&set[at], 0ull, (unsigned long long)x);
    if (was == 0) return false;
    if (was == x) return true;
  }
  return false;
}

// Two looks, for sharing of both kinds: kSampled requests evenly spread find
// few keys that many requests share (and keys that are in the table); all
// requests whose first key has zeros in some bits of its hash find groups of a
// few requests anywhere in the batch, which come into this sample together.
//
// Digests of a chain are shared from the first on or not at all, other keys may
// differ in the first row alone.  So a row of every kSampleRows is looked at in
// the same two ways.  Of a key's copies the second look sees one in 64: where
// all keys come twice, repeats are one in 128 of what it sees, and about there the
// two ways meet (14.7 M rows into 2^25 slots, by regions / by requests: two
// copies 1040 / 925 us, 16 870 / 490, 1024 1370 / 320, one key in all rows but the
// first 2960 / 195; all new 1140 / 1490).  A batch that then goes by requests
// claims no slot without a read, and where few keys make up much of it, tags are
// read before keys: a slot's key that an XCD's cache holds as it was before it was
// written sends every later copy to the compare-and-swap (1000 keys 890 us, 360
// by tags).
__device__ __forceinline__ void sample_look(const RegionArgs &a, unsigned long long *sets,
                                            const Key &key, bool spread, uint32_t mask,
                                            unsigned long long *cnt, unsigned long long *hot) {
  const uint64_t x = slot_hash(key);
  if (spread) {
    const bool twice = sample_twice(sets, x), there = twice || probe(a.t, key, true);
    atomicAdd(&cnt[0], 1ull << 32 | (there ? 1 : 0));
    if (hot) atomicAdd(hot, 1ull << 32 | (twice ? 1 : 0));
  }
  if (((uint32_t)(x >> 40) & mask) == 0) {
    const bool twice = sample_twice(sets + kSampleSlots, x);
    atomicAdd(&cnt[1], 1ull << 32 | (twice ? 1 : 0));
  }
}

// Is i, of n, one of kSampled that are evenly spread?
__device__ __forceinline__ bool is_spread(int64_t i, int64_t n) {
  return i == 0 || i * kSampled / n != (i - 1) * kSampled / n;
}

__global__ __launch_bounds__(kListThreads) void k_region_sample(RegionArgs a) {
  __shared__ unsigned long long cnt[kSampleSets + 1];
  int64_t lo, hi;
  const bool ok = region_rows(a, lo, hi);
  if (threadIdx.x < kSampleSets + 1) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * kListThreads + threadIdx.x;
  const int64_t b = i < a.n ? a.blk_offsets[i] : -1;
  if (ok && b >= lo && b < hi)
    sample_look(a, a.sample, load_key(a.hashes + b * 32), is_spread(i, a.n), a.key_mask, cnt,
                nullptr);
  // (scattered, as copies may be any number of rows apart, and a row of each
  // stretch that a plain multiple would choose never meets some of them)
  const int64_t looks = (hi - lo) / kSampleRows;
  if (ok && i < looks) {
    uint32_t x = (uint32_t)i * 0x9E3779B1u;
    x = (x ^ x >> 15) * 0x85EBCA77u;
    const int64_t f = lo + i * kSampleRows + (x ^ x >> 13) % kSampleRows;
    sample_look(a, a.sample + 2 * kSampleSlots, load_key(a.hashes + f * 32), is_spread(i, looks),
                a.row_mask, cnt + 2, cnt + kSampleSets);
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x < kCounterLanes)
      a.t.meta->new_keys[(a.epoch + 1) & 1][threadIdx.x] = 0;  // counters of the next call
    if (threadIdx.x == 0) {
      if (!ok) atomicCAS(&a.t.meta->status, 0, KVGOV_E_OFFSETS);
      a.st->bad = !ok || (hi - lo) * 2 < a.n_blocks;
    }
  }
  __syncthreads();
  unsigned long long *sums[kSampleSets + 1] = {&a.st->spread, &a.st->by_key, &a.st->rows_spread,
                                               &a.st->rows_by_key, &a.st->rows_hot};
#pragma unroll
  for (int k = 0; k < kSampleSets + 1; ++k)
    if (threadIdx.x == 64 * k && cnt[k]) atomicAdd(sums[k], cnt[k]);
}

// A workgroup sorts its 16384 rows by region in LDS, so that a region's entries
// leave together (written in the rows' order: 340 us instead of 205, 13.7 M
// rows).
__global__ __launch_bounds__(kListThreads) void k_region_lists(RegionArgs a) {
  constexpr int kPer = kMaxRegions / kListThreads;  // regions per thread
  // (print << 14 | home within the region) << 26 | row of the workgroup << 12 | region
  __shared__ unsigned long long sorted[kListRows];
  __shared__ uint32_t at[kMaxRegions];  // rows per region, then their first place
  __shared__ uint32_t wave_sum[kListThreads / 64];
  if (a.st->by_request()) return;
  int64_t lo, hi;
  if (!region_rows(a, lo, hi)) return;
  for (int64_t base = lo + (int64_t)blockIdx.x * kListRows; base < hi;
       base += (int64_t)gridDim.x * kListRows) {
    const int m = (int)(hi - base < kListRows ? hi - base : kListRows);
    for (uint32_t i = threadIdx.x; i < kMaxRegions; i += kListThreads) at[i] = 0;
    __syncthreads();
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    uint32_t what[kListItems], where[kListItems];  // (print, home); (region << 16) | rank
    constexpr int kBatch = 8;                      // rows in flight per thread
#pragma unroll
    for (int k0 = 0; k0 < kListItems; k0 += kBatch) {
      Key key[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int r = (k0 + k) * kListThreads + threadIdx.x;
        key[k] = load_key(a.hashes + (base + (r < m ? r : 0)) * 32);
      }
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int r = (k0 + k) * kListThreads + threadIdx.x;
        where[k0 + k] = kNone;
        if (r >= m) continue;
        if (key_is_empty_pattern(key[k])) {  // has no slot
          a.rest[atomicAdd(&a.st->n_rest, 1u)] = (uint32_t)(base - lo) + r;
          continue;
        }
        const uint64_t x = slot_hash(key[k]);
        const uint32_t home = (uint32_t)(x & a.t.mask), g = home >> kRegionLog2;
        what[k0 + k] = (uint32_t)(x >> 48) << kRegionLog2 | (home & ((1u << kRegionLog2) - 1));
        where[k0 + k] = g << 16 | atomicAdd(&at[g], 1u);
      }
    }
    __syncthreads();
    uint32_t cnt[kPer], sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      cnt[i] = at[threadIdx.x * kPer + i];
      sum += cnt[i];
    }
    uint32_t incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t v = __shfl_up(incl, d, 64);
      if ((int)(threadIdx.x & 63) >= d) incl += v;
    }
    if ((threadIdx.x & 63) == 63) wave_sum[threadIdx.x >> 6] = incl;
    __syncthreads();
    uint32_t start = incl - sum, listed = 0;
    for (int w = 0; w < kListThreads / 64; ++w) {
      if (w < (int)(threadIdx.x >> 6)) start += wave_sum[w];
      listed += wave_sum[w];
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      at[threadIdx.x * kPer + i] = start;
      start += cnt[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kListItems; ++k) {
      if (where[k] == kNone) continue;
      const uint32_t g = where[k] >> 16, r = k * kListThreads + threadIdx.x;
      sorted[at[g] + (where[k] & 0xFFFFu)] = (unsigned long long)what[k] << 26 | r << 12 | g;
    }
    __syncthreads();
    // from a place in `sorted` to the place in the region's list
    uint32_t got[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      got[i] = cnt[i] ? atomicAdd(&a.cursor[threadIdx.x * kPer + i], cnt[i]) : 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      at[threadIdx.x * kPer + i] = got[i] - at[threadIdx.x * kPer + i];
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < listed; i += kListThreads) {
      const unsigned long long e = sorted[i];
      const uint32_t g = (uint32_t)e & (kMaxRegions - 1), to = at[g] + i;
      const uint32_t row = (uint32_t)(base - lo) + ((uint32_t)(e >> 12) & (kListRows - 1));
      if (to < a.cap)
        a.entries[(uint64_t)g * a.cap + to] = e >> 26 << 32 | row;
      else
        a.rest[atomicAdd(&a.st->n_rest, 1u)] = row;
    }
    __syncthreads();
  }
}
static_assert(kListRows == 1 << 14 && kMaxRegions == 1 << 12, "an entry's fields");

// The claims need the rows' prints alone (16 bits of the hash that the home does
// not use): keys are read only where two prints meet, or a key of an earlier
// call.  Then the claimed slots are written in order, each key read from its
// row, and only where the tag is still free: a call of another stream may have
// taken it (the compare-and-swaps of neighbouring lanes share their lines: no
// slower than stores, 810 us either way).
__global__ __launch_bounds__(kListThreads) void k_region_insert(RegionArgs a) {
  constexpr int kSlots = 1 << kRegionLog2;
  constexpr uint32_t kOld = 0xFFFFFFFFu;  // a slot taken before
  __shared__ uint32_t claim[kSlots];      // 0, or (print << 16) | (place in the list + 1)
  __shared__ uint32_t added_sum;
  if (a.st->by_request()) return;
  const uint8_t *rows = a.hashes + a.blk_offsets[0] * 32;
  if (threadIdx.x == 0) added_sum = 0;
  uint32_t added = 0;
  for (uint32_t g = blockIdx.x; g < a.regions; g += gridDim.x) {
    const uint32_t cnt = a.cursor[g] < a.cap ? a.cursor[g] : a.cap;
    if (cnt == 0) continue;
    const uint64_t s0 = (uint64_t)g << kRegionLog2;
#pragma unroll
    for (int i = 0; i < kSlots / kListThreads; ++i) {
      const int s = i * kListThreads + threadIdx.x;
      claim[s] = a.t.tags[s0 + s] ? kOld : 0;
    }
    __syncthreads();
    const unsigned long long *list = a.entries + (uint64_t)g * a.cap;
    for (uint32_t e = threadIdx.x; e < cnt; e += kListThreads) {
      const unsigned long long ent = list[e];
      const uint32_t row = (uint32_t)ent, what = (uint32_t)(ent >> 32);
      const uint32_t home = what & (kSlots - 1), print = what >> kRegionLog2;
      for (uint32_t p = 0;; ++p) {
        const uint32_t bucket = (home >> 2) + (p >> 2);
        if (bucket >= kSlots / 4) {  // the sequence leaves the region
          a.rest[atomicAdd(&a.st->n_rest, 1u)] = row;
          break;
        }
        const uint32_t s = bucket << 2 | ((home + p) & 3);
        const uint32_t was = atomicCAS(&claim[s], 0u, print << 16 | (e + 1));
        if (was == 0) break;
        const bool old = was == kOld;
        if (!old && was >> 16 != print) continue;
        const Key other = old
                              ? Key{a.t.keys[2 * (s0 + s)], a.t.keys[2 * (s0 + s) + 1]}
                              : load_key(rows + (uint64_t)(uint32_t)list[(was & 0xFFFFu) - 1] * 32);
        if (key_eq(load_key(rows + (uint64_t)row * 32), other)) break;
      }
    }
    __syncthreads();
    constexpr int kBatch = 8;  // keys in flight per thread
    for (int i0 = 0; i0 < kSlots / kListThreads; i0 += kBatch) {
      uint32_t at[kBatch], row[kBatch];
      Key key[kBatch];
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        at[i] = claim[(i0 + i) * kListThreads + threadIdx.x];
        if (at[i] == kOld) at[i] = 0;
        row[i] = (uint32_t)list[at[i] ? (at[i] & 0xFFFFu) - 1 : 0];
      }
      // (a slot that is not claimed reads the list's first row)
#pragma unroll
      for (int i = 0; i < kBatch; ++i) key[i] = load_key(rows + (uint64_t)row[i] * 32);
#pragma unroll
      for (int i = 0; i < kBatch; ++i) {
        if (at[i] == 0) continue;
        const uint64_t s = s0 + (i0 + i) * kListThreads + threadIdx.x;
        const unsigned long long mine = (unsigned long long)a.epoch << 32 | (row[i] + 1);
        if (atomicCAS(&a.t.tags[s], 0ull, mine) != 0) {
          a.rest[atomicAdd(&a.st->n_rest, 1u)] = row[i];
          continue;
        }
        a.t.keys[2 * s] = key[i].lo;
        a.t.keys[2 * s + 1] = key[i].hi;
        ++added;
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) added += __shfl_xor(added, d, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0 && added) atomicAdd(&added_sum, added);
  __syncthreads();
  if (threadIdx.x == 0 && added_sum) {
    const int cl = blockIdx.x % kCounterLanes;
    atomicAdd(&a.t.meta->new_keys[a.epoch & 1][cl], (unsigned long long)added_sum);
    atomicAdd(&a.t.meta->n_keys[cl], (unsigned long long)added_sum);
  }
}

__global__ __launch_bounds__(256) void k_list_insert(RegionArgs a) {
  __shared__ uint32_t lds4[4];
  if (a.st->by_request()) return;
  const int64_t lo = a.blk_offsets[0];
  const uint32_t cnt = a.st->n_rest;
  uint32_t added = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < cnt; i += (uint64_t)gridDim.x * 256) {
    const int64_t f = lo + a.rest[i];
    uint32_t code;
    added += insert_key<false>(a.t, load_key(a.hashes + f * 32), f, lo, a.hashes, a.epoch, &code);
  }
  const uint32_t total = block_sum(added, lds4);
  if (threadIdx.x == 0 && total) {
    const int cl = blockIdx.x % kCounterLanes;
    atomicAdd(&a.t.meta->new_keys[a.epoch & 1][cl], (unsigned long long)total);
    atomicAdd(&a.t.meta->n_keys[cl], (unsigned long long)total);
  }
}

struct LookupArgs {
  TableView t;
  const uint8_t *hashes;
  const int64_t *blk_offsets;
  int32_t n;
  int64_t n_blocks;
  int32_t *hit_blocks;
};

// G lanes per request take G consecutive blocks at a time; a ballot over the
// group finds the first miss, and the group stops at the first chunk that
// holds one.  Several probes in flight per lane (over blocks past the first
// miss: 2 or 4 per lane) measured slower on the probe-heavy workload, whose
// lookup is bound by the lines it moves rather than by latency.
template <int G>
__global__ __launch_bounds__(256) void k_lookup(LookupArgs a) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t r = gid / G;
  if (r >= a.n) return;  // groups never straddle this test: 256 % G == 0
  const int sub = (int)(gid % G);
  const int lane = threadIdx.x & 63;
  const int base = lane & ~(G - 1);
  const uint64_t gmask = group_mask<G>(base);
  const int64_t b0 = a.blk_offsets[r], b1 = a.blk_offsets[r + 1];
  if (b0 < 0 || b1 < b0 || b1 > a.n_blocks) {
    if (sub == 0) {
      atomicCAS(&a.t.meta->status, 0, KVGOV_E_OFFSETS);
      a.hit_blocks[r] = 0;
    }
    return;
  }
  const bool ones = a.t.meta->ones_present != 0;
  const int64_t nf = b1 - b0;
  int64_t hit = nf;
  for (int64_t j0 = 0; j0 < nf; j0 += G) {
    const int64_t j = j0 + sub;
    bool miss = false;
    if (j < nf) miss = !probe(a.t, load_key(a.hashes + (b0 + j) * 32), ones);
    const uint64_t m = __ballot(miss) & gmask;
    if (m) {
      hit = j0 + (__builtin_ctzll(m) - base);
      break;
    }
  }
  if (sub == 0) a.hit_blocks[r] = (int32_t)hit;
}

struct AdmitArgs {
  TableView t;
  const int64_t *blk_offsets;
  int32_t n;
  int64_t n_blocks;
  uint32_t epoch;
  const uint32_t *codes;  // per row, from the insert
  int32_t *hit_blocks;
  int32_t *new_blocks;
};

// Second half of the admission: G lanes per request walk all of its rows G
// at a time.  Row f of request r (rows [b0, b1)) with key K:
//   visible to r  <=>  K was in the table before the call (a tag of an
//                      earlier epoch), or K's earliest row in the call lies
//                      before b0 (an earlier request holds it);
//   new for r     <=>  K's earliest row is f itself.
// hit_blocks[r] = first row not visible (relative to b0), new_blocks[r] =
// rows new for r.  The earliest rows are final: the insert has ended.
template <int G>
__global__ __launch_bounds__(256) void k_admit_scan(AdmitArgs a) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t r = gid / G;
  if (r >= a.n) return;  // groups never straddle this test: 256 % G == 0
  const int sub = (int)(gid % G);
  const int lane = threadIdx.x & 63;
  const int base = lane & ~(G - 1);
  const uint64_t gmask = group_mask<G>(base);
  const int64_t lo = a.blk_offsets[0], hi = a.blk_offsets[a.n];
  const int64_t b0 = a.blk_offsets[r], b1 = a.blk_offsets[r + 1];
  // the batch check of the insert (which then wrote no codes), and this
  // request's rows inside the batch
  if (lo < 0 || hi < lo || hi > a.n_blocks || hi - lo >= 0xFFFFFFFFll || b0 < lo || b1 < b0 ||
      b1 > hi) {
    if (sub == 0) {
      atomicCAS(&a.t.meta->status, 0, KVGOV_E_OFFSETS);
      a.hit_blocks[r] = 0;
      a.new_blocks[r] = 0;
    }
    return;
  }
  const int64_t nf = b1 - b0;
  int64_t hit = nf;
  uint32_t fresh = 0;
  for (int64_t j0 = 0; j0 < nf; j0 += G) {
    const int64_t j = j0 + sub;
    bool seen = true;
    if (j < nf) {
      const int64_t f = b0 + j;
      const uint32_t code = a.codes[f];
      if (code == kCodeFailed) {
        seen = false;
      } else if (code != kCodeDup) {
        const unsigned long long tag =
            code == kCodeOnes ? a.t.meta->ones_tag : a.t.tags[code & a.t.mask];
        if ((uint32_t)(tag >> 32) == a.epoch) {
          const int64_t first = lo + (int64_t)(tag & 0xFFFFFFFFull) - 1;
          seen = first < b0;
          fresh += first == f ? 1u : 0u;
        }
      }
    }
    const uint64_t m = __ballot(!seen) & gmask;
    if (m && hit == nf) hit = j0 + (__builtin_ctzll(m) - base);
  }
  // sum of `fresh` over the group
#pragma unroll
  for (int d = G / 2; d >= 1; d >>= 1) fresh += __shfl_xor(fresh, d, 64);
  if (sub == 0) {
    a.hit_blocks[r] = (int32_t)hit;
    a.new_blocks[r] = (int32_t)fresh;
  }
}

__global__ void k_export_begin(CacheMeta *m) { m->exported = 0; }

// One atomic per wave reserves the output rows of the wave's keys.
__device__ __forceinline__ void export_key(bool have, const u32x4 &lo, const u32x4 &hi,
                                           CacheMeta *m, uint8_t *out, int64_t cap) {
  const uint64_t mask = __ballot(have);
  if (!mask) return;
  const int lane = threadIdx.x & 63;
  const int leader = __builtin_ctzll(mask);
  unsigned long long base = 0;
  if (lane == leader) base = atomicAdd(&m->exported, (unsigned long long)__popcll(mask));
  base = __shfl(base, leader, 64);
  if (have) {
    const int64_t at = (int64_t)base + __popcll(mask & ((1ull << lane) - 1ull));
    if (at < cap) {
      u32x4 *q = reinterpret_cast<u32x4 *>(out + at * 32);
      q[0] = lo;
      q[1] = hi;
    }
  }
}

__global__ __launch_bounds__(256) void k_export(TableView t, uint8_t *out, int64_t cap) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  const int64_t slots = (int64_t)t.mask + 1;
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const u32x4 ones = u32x4{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
  if (blockIdx.x == 0 && threadIdx.x < 64)
    export_key(threadIdx.x == 0 && t.meta->ones_present != 0, ones, ones, t.meta, out, cap);
  // every lane of a wave runs the same number of iterations (ballot inside)
  const int64_t rounds = (slots + stride - 1) / stride;
  for (int64_t k = 0; k < rounds; ++k) {
    const int64_t s = gid + k * stride;
    const bool have = s < slots && t.tags[s] != 0;
    u32x4 lo = ones, hi = ones;
    if (have) {
      lo = t.keys[2 * s];
      hi = t.keys[2 * s + 1];
    }
    export_key(have, lo, hi, t.meta, out, cap);
  }
}

// ---------------------------------------------------------------------------
// maintenance: eviction by recency rank, erase, and the rebuild both end in
// ---------------------------------------------------------------------------

// Eviction keeps every key whose recency word (newer stamp first, then
// smaller depth) is at least a threshold.  Only the bits that differ between
// the table's words decide: the low bits of the stamp up to the highest that
// differs and the same of the depth half, put together (order kept), are a
// number of few bits: 2 calls of requests of up to 200 rows make 2 + 8.  A
// histogram of the top kRankDigit of these bits finds the digit at which the
// kept count crosses the budget, the next pass takes the next bits of the
// words with that digit, and so on.  Words of 0 (keys of calls that did not
// track) are the lowest class and take no part; their number is the table's
// less the others.
//
// One launch per pass: the workgroup that adds its counts last takes the
// decision.  (As eight passes of eight bits of the whole word, two launches
// each, over words gathered into a dense array, the select of a 2^20-slot
// table took 180 us of a 240 us evict; now 27 of 53.)
constexpr int kRankDigit = 11;
constexpr int kRankBins = 1 << kRankDigit;
constexpr int kRankThreads = 1024;
static_assert(kRankBins == 2 * kRankThreads, "two bins per thread in the decision");

struct SelectState {
  unsigned long long prefix;     // digits decided so far
  unsigned long long threshold;  // keep rank >= threshold once done
  unsigned long long budget;     // keys still allowed below the decided part
  unsigned long long ones_rank;  // the all-0xFF key's, if it is kept
  int32_t bits;                  // bits left to decide (kRankStart: none decided yet)
  int32_t done;
  int32_t ones_keep;
  uint32_t arrived;              // workgroups that have added their counts
};
constexpr int32_t kRankStart = 255;

// One workgroup's part of the recency words: which bits they have, and how
// many there are.
struct RankPart {
  unsigned long long any, all, used;  // or, and, number of the words other than 0
};
constexpr int kRankParts = 512;

__device__ __forceinline__ unsigned long long wave_or(unsigned long long v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v |= __shfl_xor(v, d, 64);
  return v;
}
__device__ __forceinline__ unsigned long long wave_and(unsigned long long v) {
  return ~wave_or(~v);
}

// The recency words' bits and number, a part per workgroup (added up by each
// workgroup of the select).  An empty slot's word is 0, so the tags are not
// read.  Workgroup 0 also starts the select.
__global__ __launch_bounds__(256) void k_rank_range(TableView t, SelectState *st, RankPart *parts,
                                                    unsigned int *hist, long long budget) {
  const int64_t slots = (int64_t)t.mask + 1;
  const int64_t stride = (int64_t)gridDim.x * 256;
  unsigned long long any = 0, all = ~0ull, used = 0;
#pragma unroll 8
  for (int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x; s < slots; s += stride) {
    const unsigned long long r = t.rank[s];
    any |= r;
    all &= r ? r : ~0ull;
    used += r ? 1 : 0;
  }
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      const unsigned long long r = t.meta->ones_present ? t.meta->ones_rank : 0ull;
      any |= r;
      all &= r ? r : ~0ull;
      used += r ? 1 : 0;
      st->prefix = 0;
      st->threshold = 0;
      st->budget = (unsigned long long)budget;
      st->bits = kRankStart;
      st->done = 0;
      st->arrived = 0;
    }
    for (int i = threadIdx.x; i < kRankBins; i += 256) hist[i] = 0;
  }
  __shared__ RankPart w[4];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) used += __shfl_xor(used, d, 64);
  any = wave_or(any);
  all = wave_and(all);
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = RankPart{any, all, used};
  __syncthreads();
  if (threadIdx.x == 0)
    parts[blockIdx.x] = RankPart{w[0].any | w[1].any | w[2].any | w[3].any,
                                 w[0].all & w[1].all & w[2].all & w[3].all,
                                 w[0].used + w[1].used + w[2].used + w[3].used};
}

// Which bits of the recency words differ, as the widths of the two halves.
struct RankBits {
  unsigned long long common;  // the bits above them, equal in every word
  unsigned long long used;    // words other than 0
  int cs, cd;                 // low bits of the stamp and of the depth half that decide
  __device__ __forceinline__ unsigned long long pack(unsigned long long r) const {
    return ((r >> 32) & ((1ull << cs) - 1)) << cd | (r & ((1ull << cd) - 1));
  }
  __device__ __forceinline__ unsigned long long unpack(unsigned long long c) const {
    return common | (c >> cd) << 32 | (c & ((1ull << cd) - 1));
  }
};

// From the parts, for every thread of a workgroup of kRankThreads.
__device__ __forceinline__ RankBits rank_bits(const RankPart *parts, int n_parts) {
  __shared__ RankPart w[kRankThreads / 64];
  RankPart p{0, ~0ull, 0};
  if ((int)threadIdx.x < n_parts) p = parts[threadIdx.x];
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) p.used += __shfl_xor(p.used, d, 64);
  p.any = wave_or(p.any);
  p.all = wave_and(p.all);
  if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = p;
  __syncthreads();
  unsigned long long any = 0, all = ~0ull;
  RankBits b;
  b.used = 0;
#pragma unroll
  for (int i = 0; i < kRankThreads / 64; ++i) {
    any |= w[i].any;
    all &= w[i].all;
    b.used += w[i].used;
  }
  const unsigned long long vary = any & ~all;
  const uint32_t hi = (uint32_t)(vary >> 32), lo = (uint32_t)vary;
  b.cs = hi ? 32 - __builtin_clz(hi) : 0;
  b.cd = lo ? 32 - __builtin_clz(lo) : 0;
  b.common = any & ~((((1ull << b.cs) - 1) << 32) | ((1ull << b.cd) - 1));
  return b;
}
static_assert(kRankParts <= kRankThreads, "a thread per part");

// The next digit: its histogram over the words that match the decided
// digits, and, in the workgroup that arrives last, the digit at which the
// kept count crosses the budget (keys with a higher digit are kept).  Leaves
// the histogram and the arrival count cleared for the next pass.
__global__ __launch_bounds__(kRankThreads) void k_rank_select(TableView t, SelectState *st,
                                                              const RankPart *parts, int n_parts,
                                                              unsigned int *hist) {
  __shared__ unsigned int h[kRankBins];
  __shared__ unsigned long long above[kRankThreads / 64];
  __shared__ int last;
  if (st->done) return;
  const int tid = threadIdx.x;
  const RankBits rb = rank_bits(parts, n_parts);
  const bool first = st->bits == kRankStart;
  const int left = first ? rb.cs + rb.cd : st->bits;
  const int width = left < kRankDigit ? left : kRankDigit;
  const int shift = left - width;
  const unsigned long long prefix = st->prefix, budget = st->budget;
  const int bins = 1 << width;
  for (int i = tid; i < bins; i += kRankThreads) h[i] = 0;
  __syncthreads();
  const auto count = [&](unsigned long long r) {
    if (!r) return;
    const unsigned long long c = rb.pack(r) >> shift;
    if ((c >> width) == prefix) atomicAdd(&h[c & (bins - 1)], 1u);
  };
  const int64_t slots = (int64_t)t.mask + 1;
  const int64_t stride = (int64_t)gridDim.x * kRankThreads;
#pragma unroll 4
  for (int64_t s = (int64_t)blockIdx.x * kRankThreads + tid; s < slots; s += stride)
    count(t.rank[s]);
  if (blockIdx.x == 0 && tid == 0 && t.meta->ones_present) count(t.meta->ones_rank);
  __syncthreads();
  // Each count is added by an atomic whose result is waited for, so it has
  // been performed before the workgroup counts itself as arrived, and the last
  // one takes the sums by atomics as well: no other memory passes between
  // workgroups, and no cache is written back (a fence per wave made the pass
  // take 47 us).
  unsigned int seen = 0;
  for (int i = tid; i < bins; i += kRankThreads)
    if (h[i]) seen |= atomicAdd(&hist[i], h[i]);
  asm volatile("s_waitcnt vmcnt(0)" ::"v"(seen) : "memory");
  __syncthreads();
  if (tid == 0) last = atomicAdd(&st->arrived, 1u) == gridDim.x - 1;
  __syncthreads();
  if (!last) return;

  // thread i owns bins 2i and 2i + 1; `over` = keys in higher bins
  unsigned int c[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int b = 2 * tid + k;
    c[k] = b < bins ? atomicExch(&hist[b], 0u) : 0u;
  }
  const int lane = tid & 63, wid = tid >> 6;
  unsigned long long inc = (unsigned long long)c[0] + c[1];  // this thread and higher lanes
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const unsigned long long u = __shfl_down(inc, d, 64);
    if (lane + d < 64) inc += u;
  }
  if (lane == 0) above[wid] = inc;
  __syncthreads();
  unsigned long long over = inc - c[0] - c[1];
  for (int i = 0; i < kRankThreads / 64; ++i) over += i > wid ? above[i] : 0ull;
  if (tid == 0) st->arrived = 0;
  if (first) {
    // first pass: everything fits, or everything but the words of 0
    unsigned long long keys = 0;
    for (int i = 0; i < kCounterLanes; ++i) keys += t.meta->n_keys[i];
    if (keys <= budget || rb.used <= budget) {
      if (tid == 0) {
        st->threshold = keys <= budget ? 0ull : 1ull;
        st->done = 1;
      }
      return;
    }
  }
  // the one bin with over <= budget < over + its count (a later pass's total
  // exceeds the budget as well: its digit did not fit as a whole)
#pragma unroll
  for (int k = 1; k >= 0; --k) {
    if (over <= budget && budget < over + c[k]) {
      const unsigned long long p = (prefix << width) | (unsigned long long)(2 * tid + k);
      st->prefix = p;
      st->budget = budget - over;
      st->bits = shift;
      if (shift == 0) {  // the whole class p does not fit: keep what ranks above it
        st->threshold = rb.unpack(p) + 1;
        st->done = 1;
      }
    }
    over += c[k];
  }
}

// Erase: a present key's recency word becomes kErased (counted once per key).
__global__ __launch_bounds__(256) void k_erase_mark(TableView t, const uint8_t *keys,
                                                    int64_t n) {
  __shared__ uint32_t lds4[4];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  uint32_t marked = 0;
  if (i < n) {
    const Key k = load_key(keys + i * 32);
    unsigned long long *w = nullptr;
    if (key_is_empty_pattern(k)) {
      if (t.meta->ones_present) w = &t.meta->ones_rank;
    } else {
      const int64_t slot = find_slot(t, k);
      if (slot >= 0) w = &t.rank[slot];
    }
    if (w && atomicExch(w, kErased) != kErased) marked = 1;
  }
  const uint32_t total = block_sum(marked, lds4);
  if (threadIdx.x == 0 && total) atomicAdd(&t.meta->marked, (unsigned long long)total);
}

// The rebuild.  A workgroup takes a region of kRegion slots, copies the
// region's kept keys and recency words to the scratch, close together from the
// region's own place on, and empties the region's occupied slots (the others
// are empty as they are); then every copy is inserted again.  No counter is
// shared, and a table at load 1/4 has a quarter of its slots written.  (With
// the copies packed over the whole table by one atomic per 4096 slots, the
// table emptied by a launch of its own, and 256 workgroups: 50 us for 2^20
// slots; now 24.)
constexpr int kRegion = 1024;

__global__ __launch_bounds__(256) void k_compact(TableView t, SelectState *st, int erase,
                                                 u32x4 *out_keys, unsigned long long *out_rank,
                                                 uint32_t *region_count) {
  __shared__ uint32_t wsum[4];
  const int64_t slots = (int64_t)t.mask + 1;
  const unsigned long long thr = erase ? 0ull : st->threshold;  // erase: all but the marked
  const u32x4 ones = u32x4{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
  constexpr int kItems = kRegion / 256;
  const int64_t b0 = (int64_t)blockIdx.x * kRegion;
  unsigned long long r[kItems], tag[kItems];
  uint32_t keep = 0, have = 0;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    const int64_t s = b0 + k * 256 + threadIdx.x;
    tag[k] = s < slots ? t.tags[s] : 0ull;
    r[k] = s < slots ? t.rank[s] : 0ull;
  }
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    have |= tag[k] != 0 ? 1u << k : 0u;
    keep |= tag[k] != 0 && r[k] != kErased && r[k] >= thr ? 1u << k : 0u;
  }
  // exclusive prefix of the kept counts over the workgroup
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t mine = __popc(keep);
  uint32_t inc = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = __shfl_up(inc, d, 64);
    if (lane >= d) inc += u;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    before += i < w ? wsum[i] : 0u;
    total += wsum[i];
  }
  int64_t o = b0 + before + inc - mine;
#pragma unroll
  for (int k = 0; k < kItems; ++k) {
    if (!(have & (1u << k))) continue;
    const int64_t s = b0 + k * 256 + threadIdx.x;
    if (keep & (1u << k)) {
      out_keys[2 * o] = t.keys[2 * s];
      out_keys[2 * o + 1] = t.keys[2 * s + 1];
      out_rank[o] = r[k];
      ++o;
    }
    t.keys[2 * s] = ones;
    t.keys[2 * s + 1] = ones;
    t.tags[s] = 0;
    t.rank[s] = 0;
  }
  if (threadIdx.x == 0) region_count[blockIdx.x] = total;
  // the all-0xFF key and the counters (the latched error and the export and
  // erase counts stay)
  if (blockIdx.x == 0) {
    CacheMeta *m = t.meta;
    for (int i = threadIdx.x; i < kCounterLanes; i += blockDim.x) {
      m->n_keys[i] = 0;
      m->new_keys[0][i] = 0;
      m->new_keys[1][i] = 0;
    }
    if (threadIdx.x == 0) {
      const unsigned long long q = m->ones_rank;
      st->ones_keep = m->ones_present && q != kErased && q >= thr;
      st->ones_rank = q;
      m->ones_tag = 0;
      m->ones_rank = 0;
      m->ones_present = 0;
      m->erased = m->marked;
      m->marked = 0;
    }
  }
}

// Inserts the kept keys again (all distinct) and restores their recency: a
// workgroup per region.  Bound by chains of waits, the longest probe sequence of
// each wave: in small tables a lane has one key at most, in large ones, which have
// regions enough to fill the chip, fewer threads go on to the region's next keys.
// Erase of one key with 256 / 512 / 1024 threads, us: 2^12 slots at load 0.8 140
// / - / 86, 2^16 166 / - / 104, 2^20 326 / 257 / 239, 2^22 708 / - / 767; at load
// 0.3 2^20 55 / 52 / 55, 2^22 153 / - / 163; at 0.02 2^20 26 / 26 / 28.
static int reinsert_threads(int64_t slots) {
  return slots <= 1 << 18 ? kRegion : slots <= 1 << 20 ? kRegion / 2 : kRegion / 4;
}

__global__ __launch_bounds__(kRegion) void k_reinsert(TableView t, const SelectState *st,
                                                      const uint8_t *keys,
                                                      const unsigned long long *rank,
                                                      const uint32_t *region_count,
                                                      uint32_t epoch) {
  __shared__ uint32_t sum;
  if (threadIdx.x == 0) sum = 0;
  __syncthreads();
  const int64_t b0 = (int64_t)blockIdx.x * kRegion;
  const int64_t n = b0 + region_count[blockIdx.x];
  uint32_t added = 0;
  for (int64_t i = b0 + threadIdx.x; i < n; i += blockDim.x) {
    uint32_t code = kCodeFailed;
    added += insert_key<false>(t, load_key(keys + i * 32), i, 0, keys, epoch, &code);
    if (code < kCodeFailed) t.rank[code] = rank[i];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && st->ones_keep) {
    t.meta->ones_tag = (unsigned long long)epoch << 32 | 1ull;
    t.meta->ones_present = 1;
    t.meta->ones_rank = st->ones_rank;
    ++added;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) added += __shfl_xor(added, d, 64);
  if ((threadIdx.x & 63) == 0 && added) atomicAdd(&sum, added);
  __syncthreads();
  if (threadIdx.x == 0 && sum)
    atomicAdd(&t.meta->n_keys[blockIdx.x % kCounterLanes], (unsigned long long)sum);
}

// Lanes per request for lookup: enough groups in flight to cover the chip
// (about 2^18 lanes), one lane each when the batch alone is that large; and,
// up to about 2^21 lanes, one lane per ~16 blocks of the average request,
// since a group walks its request's blocks G at a time and the longest
// request bounds the launch (a batch of long requests would otherwise wait on
// its longest one with one or two lanes).
//
// Batches of long requests (128 blocks or more on average) go to a full wave
// per request, up to 2^22 lanes: the launch then ends when the longest
// request's last round does, and a request of L blocks takes L / G rounds
// (65,536 requests averaging 208 blocks, at most 2048: 1.65 / 1.00 ms per
// lookup with 16 lanes per request, 1.34 / 0.75 ms with 64).  Short
// requests keep fewer lanes: their probes stop at the first miss, and spare
// lanes would only probe past it (1M probes of 8..64 blocks: 0.43 ms with 2
// lanes, 0.45 ms with 4).
static int lookup_group(int32_t n, int64_t n_blocks) {
  int g = 1;
  while (g < 64 && (int64_t)n * g * 2 <= (1 << 18)) g <<= 1;
  const int64_t avg = n > 0 ? n_blocks / n : 0;
  while (g < 64 && (int64_t)g * 16 <= avg && (int64_t)n * g * 2 <= (1 << 21)) g <<= 1;
  if (avg >= 128)
    while (g < 64 && (int64_t)n * g * 2 <= (1 << 22)) g <<= 1;
  return g;
}

}  // namespace kvgov

using namespace kvgov;

namespace {

int check_device(const kvgov_cache *c) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return KVGOV_E_HIP;
  return dev == c->device ? KVGOV_OK : KVGOV_E_DEVICE;
}

unsigned grid_for(int64_t work, int per_cu) {
  const int64_t cap = (int64_t)device_cu_count() * per_cu;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(work, 256), cap));
}

template <class T>
void raise_to(std::atomic<T> &most, T v) {
  T seen = most.load();
  while (seen < v && !most.compare_exchange_weak(seen, v)) {
  }
}

// Is the stream being captured, as far as is known?
bool is_capturing(hipStream_t s) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cap) == hipSuccess) return cap != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// The recency words are rewritten only if something may have written them
// since they were last cleared (a tracked insert or admission, an eviction,
// an erasure): on a table that never tracks, a clear writes 40 of its 48
// bytes per slot.  A captured clear empties nothing yet and runs on a table of
// any later state: it writes the words as well, and the clock goes on (an insert
// before its first run is not to meet its own epoch in an older tag).  Of a table
// that captured calls stamp, a clear sets the clock back to the last of these: the
// rows of a later call with the same epoch would be taken for the graph's own.
int enqueue_clear(kvgov_cache *c, hipStream_t s, const ClearMore &more = ClearMore{}) {
  FillArgs a{};
  a.m = c->view.meta;
  a.ones[0] = c->view.keys;
  a.n_ones[0] = c->slots * 2;
  a.zeros[0] = reinterpret_cast<u32x4 *>(c->view.tags);
  a.n_zeros[0] = c->slots / 2;
  const bool captured = is_capturing(s);
  if (captured || c->rank_dirty || c->graph_epoch) {
    a.zeros[1] = reinterpret_cast<u32x4 *>(c->view.rank);
    a.n_zeros[1] = c->slots / 2;
  }
  a.ones[1] = more.ones;
  a.n_ones[1] = more.n_ones;
  a.zeros[2] = more.zeros;
  a.n_zeros[2] = more.n_zeros;
  hipLaunchKernelGGL(k_cache_fill, dim3(grid_for((a.n_ones[0] + a.n_ones[1]) / 4, 1024)), dim3(256),
                     0, s, a);
  if (!captured) {
    c->rank_dirty = false;
    c->epoch = c->graph_epoch.load();
    if (!c->graph_epoch) c->max_rows = 0;
  }
  return launch_status();
}

// The plain insert takes a group of lanes per request while requests
// average at most this many rows (a group walks its request 64 rows at a
// time, so one request of 2^20 rows would take 16k steps of one wave), and
// the chunked walk above it.
constexpr int64_t kReqInsertMaxAvg = 4096;

// Lanes per request of the insert: about one lane per two rows of the average
// request, 4 to 64; in a batch small enough to be resident at once, a lane per
// row (a group then takes one round after its first row: 64 requests of 16
// rows 13.6 -> 9.8 us).  An admission's groups take what lanes the chip has, for the
// requests that are longer than the average (lognormal lengths of 6 rows on average:
// 300 requests 44 -> 34 us, 20,000 91 -> 57; equal ones the same either way).
template <bool ADMIT>
int insert_group(int32_t n, int64_t n_blocks) {
  const int64_t avg = n > 0 ? n_blocks / n : 0;
  int g = 4;
  while (g < 64 && (int64_t)g * 2 < avg) g <<= 1;
  while (g < 64 && g < avg && (int64_t)n * g * 2 <= (1 << 16)) g <<= 1;
  while (ADMIT && g < 64 && (int64_t)n * g * 2 <= (1 << 19)) g <<= 1;
  return g;
}

// k_chunk_insert: workgroups of 4 chunks, at most 16 per CU.
unsigned insert_grid(int64_t n_blocks, int chunk) {
  const int64_t groups = ceil_div(std::max<int64_t>(n_blocks, 1), (int64_t)chunk * 4);
  return (unsigned)std::min<int64_t>(groups, (int64_t)device_cu_count() * 16);
}

// A call that tracks recency is about to be enqueued: its depths are below
// n_blocks.
void note_tracked(kvgov_cache *c, int64_t n_blocks) {
  c->rank_dirty = true;
  raise_to(c->max_rows, n_blocks);
}

}  // namespace

uint32_t kvgov::next_epoch(kvgov_cache *c, hipStream_t s) {
  const uint32_t epoch = c->epoch.fetch_add(1) + 1;
  if (is_capturing(s)) raise_to(c->graph_epoch, epoch);
  return epoch;
}

int kvgov::cache_clear_with(kvgov_cache *c, hipStream_t s, const ClearMore &more) {
  return enqueue_clear(c, s, more);
}

// The table's state to the host: a kernel writes it to pinned memory.  A copy of
// these some hundred bytes into the caller's memory goes through the runtime's
// own staging and took 7 to 15 us longer: an admission that waits 104 us
// against 97, eviction and erase together 252 against 221.
__global__ __launch_bounds__(kWave) void k_report(uint32_t *to, const uint32_t *meta, int words) {
  for (int i = threadIdx.x; i < words; i += kWave) to[i] = meta[i];
}

namespace {

// Eight blocks of pinned memory for all tables, from the first call that waits
// to the process's end (an allocation for each table made its creation 45 us
// longer).  A ninth thread that reads at the same time copies, as does every
// one where there is no such memory.
class Reports {
 public:
  Reports() {
    const RelaxedCapture relaxed;
    void *p = nullptr;
    if (relaxed.ok() && hipHostMalloc(&p, kBlocks * sizeof(CacheMeta), hipHostMallocPortable) == hipSuccess)
      blocks_ = static_cast<CacheMeta *>(p);
    else
      (void)hipGetLastError();
  }
  CacheMeta *take() {
    if (!blocks_) return nullptr;
    for (int i = 0; i < kBlocks; ++i)
      if (!(used_.fetch_or(1u << i) >> i & 1u)) return blocks_ + i;
    return nullptr;
  }
  void give_back(CacheMeta *b) { used_.fetch_and(~(1u << (b - blocks_))); }

 private:
  static constexpr int kBlocks = 8;
  CacheMeta *blocks_ = nullptr;
  std::atomic<uint32_t> used_{0};
};

}  // namespace

int kvgov::cache_read_meta(kvgov_cache *c, CacheMeta *m, hipStream_t s, bool radix) {
  static Reports reports;
  const size_t bytes = radix ? sizeof(CacheMeta) : offsetof(CacheMeta, n_edges);
  CacheMeta *block = reports.take();
  int rc = KVGOV_OK;
  if (block) {
    hipLaunchKernelGGL(k_report, dim3(1), dim3(kWave), 0, s, reinterpret_cast<uint32_t *>(block),
                       reinterpret_cast<const uint32_t *>(c->view.meta), (int)(bytes / 4));
    rc = launch_status();
  } else if (hipMemcpyAsync(m, c->view.meta, bytes, hipMemcpyDeviceToHost, s) != hipSuccess) {
    rc = KVGOV_E_HIP;
  }
  if (rc == KVGOV_OK && hipStreamSynchronize(s) != hipSuccess) rc = KVGOV_E_HIP;
  if (block) {
    if (rc == KVGOV_OK) std::memcpy(m, block, bytes);
    reports.give_back(block);
  }
  return rc;
}

namespace {

// Maintenance scratch, in the stream's scratch buffer: selection state, the
// rank histogram, the regions' counts and room for every key of the table (32
// B key + 8 B recency each).  `lk` holds the scratch registry while the call
// enqueues its kernels; the stream runs its calls in order, so the buffer
// serves this call until its kernels end.
struct MaintScratch {
  SelectState *st = nullptr;
  RankPart *parts = nullptr;
  unsigned int *hist = nullptr;
  uint32_t *regions = nullptr;
  u32x4 *keys = nullptr;
  unsigned long long *rank = nullptr;
  std::unique_lock<std::mutex> lk;
};

unsigned region_grid(int64_t slots) { return (unsigned)ceil_div(slots, kRegion); }

int maint_alloc(kvgov_cache *c, hipStream_t s, MaintScratch &m) {
  const size_t off_parts = 256;
  static_assert(sizeof(SelectState) <= 256, "the state's part of the scratch");
  const size_t off_hist = off_parts + kRankParts * sizeof(RankPart);
  const size_t off_regions = off_hist + kRankBins * sizeof(unsigned int);
  const size_t off_keys = off_regions + ((size_t)region_grid(c->slots) * 4 + 255) / 256 * 256;
  const size_t off_rank = off_keys + (size_t)c->slots * 32;
  const size_t bytes = off_rank + (size_t)c->slots * 8;
  void *base = nullptr;
  const int rc = stream_scratch(s, bytes, &base, m.lk);
  if (rc != KVGOV_OK) return rc;
  uint8_t *b = static_cast<uint8_t *>(base);
  m.st = reinterpret_cast<SelectState *>(b);
  m.parts = reinterpret_cast<RankPart *>(b + off_parts);
  m.hist = reinterpret_cast<unsigned int *>(b + off_hist);
  m.regions = reinterpret_cast<uint32_t *>(b + off_regions);
  m.keys = reinterpret_cast<u32x4 *>(b + off_keys);
  m.rank = reinterpret_cast<unsigned long long *>(b + off_rank);
  return KVGOV_OK;
}

// Copies out what ranks at or above the selected threshold while emptying the
// table, and inserts the copies again; then reads the table's counters if
// asked (waiting for the stream).
int compact_rebuild(kvgov_cache *c, hipStream_t s, MaintScratch &m, int erase, CacheMeta *meta) {
  const uint32_t epoch = next_epoch(c, s);
  if (epoch == 0xFFFFFFFFu) return KVGOV_E_UNSUPPORTED;
  const dim3 grid(region_grid(c->slots)), block(256);
  hipLaunchKernelGGL(k_compact, grid, block, 0, s, c->view, m.st, erase, m.keys, m.rank,
                     m.regions);
  hipLaunchKernelGGL(k_reinsert, grid, dim3(reinsert_threads(c->slots)), 0, s, c->view, m.st,
                     reinterpret_cast<const uint8_t *>(m.keys), m.rank, m.regions, epoch);
  int rc = launch_status();
  m.lk.unlock();  // everything that uses the scratch is enqueued
  if (rc == KVGOV_OK && meta) {
    rc = cache_read_meta(c, meta, s);
    if (rc == KVGOV_OK) rc = meta->status;
  }
  return rc;
}

int bit_length(uint64_t v) { return v ? 64 - __builtin_clzll(v) : 0; }

// Keys added by insert call `epoch` (waits for the stream), and the latched
// error.
int read_new_keys(kvgov_cache *c, uint32_t epoch, int64_t *n_new, hipStream_t s) {
  CacheMeta m{};
  int rc = cache_read_meta(c, &m, s);
  if (rc != KVGOV_OK) return rc;
  int64_t added = 0;
  for (int i = 0; i < kCounterLanes; ++i) added += (int64_t)m.new_keys[epoch & 1][i];
  *n_new = added;
  return m.status;
}

template <int G, bool ADMIT, bool TRACK, bool KEYS>
void insert_req_group(const TableView &t, const uint8_t *hashes, const int64_t *blk_offsets,
                      int32_t n, int64_t n_blocks, uint32_t epoch, uint32_t *codes, hipStream_t s,
                      const RegionState *st) {
  const unsigned groups = (unsigned)std::max<int64_t>(1, ceil_div((int64_t)n * G, 256));
  const unsigned walkers = ADMIT && n_blocks > kHeadRows<G> ? insert_grid(n_blocks, kInsChunk) : 0;
  hipLaunchKernelGGL((k_insert_req<G, ADMIT, TRACK, KEYS>), dim3(groups + walkers), dim3(256), 0, s,
                     t, hashes, blk_offsets, n, n_blocks, epoch, codes, groups, st);
}

template <bool ADMIT, bool TRACK, bool KEYS>
void insert_req_launch(const TableView &t, const uint8_t *hashes, const int64_t *blk_offsets,
                       int32_t n, int64_t n_blocks, uint32_t epoch, uint32_t *codes, hipStream_t s,
                       const RegionState *st) {
  // (no request: only the batch check and the next call's counters)
  switch (n > 0 ? insert_group<ADMIT>(n, n_blocks) : 64) {
    case 4: insert_req_group<4, ADMIT, TRACK, KEYS>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, s, st); break;
    case 8: insert_req_group<8, ADMIT, TRACK, KEYS>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, s, st); break;
    case 16: insert_req_group<16, ADMIT, TRACK, KEYS>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, s, st); break;
    case 32: insert_req_group<32, ADMIT, TRACK, KEYS>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, s, st); break;
    default: insert_req_group<64, ADMIT, TRACK, KEYS>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, s, st); break;
  }
}

// Table sizes from which rows look at a slot's key before its tag (see
// k_insert_req).
constexpr uint64_t kKeysFirstSlots = (uint64_t)1 << 21;

template <bool ADMIT, bool TRACK>
void insert_req(const TableView &t, const uint8_t *hashes, const int64_t *blk_offsets, int32_t n,
                int64_t n_blocks, uint32_t epoch, uint32_t *codes, hipStream_t s) {
  if (!ADMIT && t.mask + 1 >= kKeysFirstSlots)
    insert_req_launch<ADMIT, TRACK, !ADMIT>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, s, nullptr);
  else
    insert_req_launch<ADMIT, TRACK, false>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, s, nullptr);
}

// Whether an insert may take k_insert_req (otherwise in chunks).
bool by_requests(int32_t n, int64_t n_blocks) {
  return n == 0 || n_blocks <= (int64_t)n * kReqInsertMaxAvg;
}

// Admissions of more and shorter requests than these go in chunks.  A group waits
// for the rounds of its wave's longest request; few requests get lanes enough for
// these (insert_group), of many most lanes would have no row.  Lognormal lengths, us
// by requests / in chunks: 200,000 of 6 on average 164 / 127, of 12 328 / 305, 1 M
// of 3 424 / 350, of 6 795 / 637; 2 M of one row, one in a hundred of 64, 756 / 491,
// all there 641 / 297.
// Equal ones are about the same either way (200,000 of 4 96 / 103, of 8 164 / 163,
// 500,000 of one 31 / 47); longer ones can share heads that are not the previous
// request's, which groups compare and chunks do not (200,000 of 16, half of them of
// 64 heads, 235 / 278).
constexpr int64_t kChunkAdmitAvg = 16;
constexpr int32_t kChunkAdmitMin = 1 << 16;

// Rows per wave of these: fewer rows than fill the chip take one or two rounds
// (100,000 of one row 21 us, 32 in chunks of 256; 200,000 of 2 71 / 76), but half of
// 3 M rows of 64 heads 290 / 277 (see kInsChunk).
int admit_chunk(int64_t n_blocks) {
  return n_blocks <= 1 << 18 ? kInsChunk / 4 : n_blocks <= 1 << 20 ? kInsChunk / 2 : kInsChunk;
}

// The insert of a call: by requests, or in chunks: few, long requests, where a group
// per request would leave the chip idle, and an admission's many short ones.  codes:
// ADMIT only.
template <bool ADMIT>
int insert_batch(const TableView &t, const uint8_t *hashes, const int64_t *blk_offsets, int32_t n,
                 int64_t n_blocks, uint32_t epoch, uint32_t *codes, hipStream_t s) {
  const bool many = ADMIT && n > kChunkAdmitMin && n_blocks < n * kChunkAdmitAvg;
  const int chunk = many ? admit_chunk(n_blocks) : kInsChunk;
  if (many || !by_requests(n, n_blocks))
    hipLaunchKernelGGL(k_chunk_insert<ADMIT>, dim3(insert_grid(n_blocks, chunk)), dim3(256), 0, s,
                       t, hashes, blk_offsets, n, n_blocks, epoch, codes, chunk);
  else if (t.track)
    insert_req<ADMIT, true>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, s);
  else
    insert_req<ADMIT, false>(t, hashes, blk_offsets, n, n_blocks, epoch, codes, s);
  return launch_status();
}

}  // namespace

namespace {

// Whether a batch may go by regions (us for new keys, by regions / by requests):
// 11.9 M rows into 2^25 slots 991 / 1064, 16.8 M 1293 / 1570, 23.7 M 1793 / 2652;
// but 8.4 M into 2^25 757 / 748, 16.8 M into 2^26 1529 / 1582.  Where the sample
// then finds the keys shared or present, the look and the kernels that end at
// once cost 30 to 45 us, 100 in a table that is 0.7 full (present keys: 16.8 M 617
// instead of 573, 23.7 M 1263 instead of 1165; shared ones 16.8 M 555 instead of
// 522), which is why smaller batches, whose gain is smaller, are left alone (8.4 M
// new keys into 2^24 slots 670 / 758, shared ones 309 / 279).  A batch of more rows than
// slots holds duplicates; the sample reads a line for each request, so
// requests are to be 32 rows long.
constexpr int64_t kRegionMinRows = (int64_t)10 << 20;

bool by_regions(const kvgov_cache *c, int32_t n, int64_t n_blocks) {
  return !c->view.track && n_blocks >= kRegionMinRows && n_blocks >= c->slots / 3 &&
         n_blocks <= c->slots && (c->slots >> kRegionLog2) <= kMaxRegions && n >= kSampled &&
         n_blocks / n >= 32 && n_blocks <= (int64_t)n * kReqInsertMaxAvg;
}

// The insert by regions, or, where its sample finds so, by requests.  False
// if it cannot have its scratch (then nothing is enqueued).
bool insert_regions(kvgov_cache *c, const uint8_t *hashes, const int64_t *blk_offsets, int32_t n,
                    int64_t n_blocks, uint32_t epoch, hipStream_t s, int *rc) {
  if (is_capturing(s)) return false;  // no memory may be allocated then
  RegionArgs a{c->view, hashes, blk_offsets, n, n_blocks, epoch};
  a.regions = (uint32_t)(c->slots >> kRegionLog2);
  // room for an even spread and ten standard deviations
  const double mean = (double)n_blocks / a.regions;
  a.cap = std::min((uint32_t)(mean + 10.0 * std::sqrt(mean) + 64.0), (uint32_t)kMaxListed);
  a.key_mask = 0;
  while (n / ((int64_t)a.key_mask + 1) >= 2 * kSampledByKey) a.key_mask = a.key_mask * 2 + 1;
  const int64_t looks = n_blocks / kSampleRows;
  a.row_mask = 0;
  while (looks / ((int64_t)a.row_mask + 1) >= 2 * kSampledByKey) a.row_mask = a.row_mask * 2 + 1;
  const size_t off_cursor = 256;
  const size_t off_sample = off_cursor + sizeof(uint32_t) * kMaxRegions;
  const size_t off_entries = off_sample + sizeof(unsigned long long) * kSampleSets * kSampleSlots;
  const size_t off_rest = off_entries + sizeof(unsigned long long) * a.regions * a.cap;
  const size_t bytes = off_rest + sizeof(uint32_t) * (size_t)n_blocks;
  std::unique_lock<std::mutex> lk;
  void *base = nullptr;
  const RelaxedCapture relaxed;
  if (!relaxed.ok() || stream_scratch(s, bytes, &base, lk) != KVGOV_OK) return false;
  uint8_t *b = static_cast<uint8_t *>(base);
  a.st = reinterpret_cast<RegionState *>(b);
  a.cursor = reinterpret_cast<uint32_t *>(b + off_cursor);
  a.sample = reinterpret_cast<unsigned long long *>(b + off_sample);
  a.entries = reinterpret_cast<unsigned long long *>(b + off_entries);
  a.rest = reinterpret_cast<uint32_t *>(b + off_rest);
  const unsigned cus = (unsigned)device_cu_count();
  const unsigned tiles = (unsigned)std::min<int64_t>(ceil_div(n_blocks, kListRows), cus);
  hipLaunchKernelGGL(k_region_clear, dim3(kSampleSets * kSampleSlots / 256), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_region_sample, dim3((unsigned)ceil_div(std::max<int64_t>(n, looks), kListThreads)),
                     dim3(kListThreads), 0, s, a);
  hipLaunchKernelGGL(k_region_lists, dim3(tiles), dim3(kListThreads), 0, s, a);
  hipLaunchKernelGGL(k_region_insert, dim3(std::min(a.regions, cus)), dim3(kListThreads), 0, s, a);
  hipLaunchKernelGGL(k_list_insert, dim3(cus * 4), dim3(256), 0, s, a);
  insert_req_launch<false, false, true>(c->view, hashes, blk_offsets, n, n_blocks, epoch, nullptr, s,
                                        a.st);
  insert_req_launch<false, false, false>(c->view, hashes, blk_offsets, n, n_blocks, epoch, nullptr, s,
                                         a.st);
  *rc = launch_status();
  return true;
}

}  // namespace

bool kvgov::cache_inserts_by_request(const kvgov_cache *c, int32_t n, int64_t n_blocks) {
  return by_requests(n, n_blocks) && !by_regions(c, n, n_blocks);
}

int kvgov::cache_insert_rows(kvgov_cache *c, const uint8_t *hashes, const int64_t *blk_offsets,
                             int32_t n, int64_t n_blocks, hipStream_t s, uint32_t *epoch) {
  *epoch = next_epoch(c, s);
  if (*epoch == 0xFFFFFFFFu) return KVGOV_E_UNSUPPORTED;  // 2^32 - 1 inserts since clear
  if (c->view.track) note_tracked(c, n_blocks);
  int rc = KVGOV_OK;
  if (by_regions(c, n, n_blocks) &&
      insert_regions(c, hashes, blk_offsets, n, n_blocks, *epoch, s, &rc))
    return rc;
  return insert_batch<false>(c->view, hashes, blk_offsets, n, n_blocks, *epoch, nullptr, s);
}

extern "C" {

int kvgov_cache_create(int32_t log2_slots, kvgov_cache **out) {
  if (!out || log2_slots < KVGOV_MIN_LOG2_SLOTS || log2_slots > KVGOV_MAX_LOG2_SLOTS)
    return KVGOV_E_INVAL;
  *out = nullptr;
  kvgov_cache *c = new (std::nothrow) kvgov_cache();
  if (!c) return KVGOV_E_NOMEM;
  if (hipGetDevice(&c->device) != hipSuccess) {
    delete c;
    return KVGOV_E_HIP;
  }
  c->log2_slots = log2_slots;
  c->slots = (int64_t)1 << log2_slots;
  c->view.mask = (uint64_t)c->slots - 1;
  void *keys = nullptr, *tags = nullptr, *rank = nullptr, *meta = nullptr;
  if (hipMalloc(&keys, (size_t)c->slots * 32) != hipSuccess ||
      hipMalloc(&tags, (size_t)c->slots * 8) != hipSuccess ||
      hipMalloc(&rank, (size_t)c->slots * 8) != hipSuccess ||
      hipMalloc(&meta, sizeof(CacheMeta)) != hipSuccess) {
    if (keys) (void)hipFree(keys);
    if (tags) (void)hipFree(tags);
    if (rank) (void)hipFree(rank);
    if (meta) (void)hipFree(meta);
    delete c;
    return KVGOV_E_NOMEM;
  }
  c->view.keys = static_cast<u32x4 *>(keys);
  c->view.tags = static_cast<unsigned long long *>(tags);
  c->view.rank = static_cast<unsigned long long *>(rank);
  c->view.track = 0;
  c->view.meta = static_cast<CacheMeta *>(meta);
  int rc = enqueue_clear(c, nullptr);
  if (rc == KVGOV_OK && hipStreamSynchronize(nullptr) != hipSuccess) rc = KVGOV_E_HIP;
  if (rc != KVGOV_OK) {
    kvgov_cache_destroy(c);
    return rc;
  }
  *out = c;
  return KVGOV_OK;
}

int kvgov_cache_destroy(kvgov_cache *c) {
  if (!c) return KVGOV_OK;
  int rc = KVGOV_OK;
  if (hipDeviceSynchronize() != hipSuccess) rc = KVGOV_E_HIP;
  if (hipFree(c->view.keys) != hipSuccess) rc = KVGOV_E_HIP;
  if (hipFree(c->view.tags) != hipSuccess) rc = KVGOV_E_HIP;
  if (hipFree(c->view.rank) != hipSuccess) rc = KVGOV_E_HIP;
  if (hipFree(c->view.meta) != hipSuccess) rc = KVGOV_E_HIP;
  delete c;
  return rc;
}

int kvgov_cache_clear(kvgov_cache *c, void *stream) {
  if (!c) return KVGOV_E_INVAL;
  int rc = check_device(c);
  if (rc != KVGOV_OK) return rc;
  return enqueue_clear(c, as_stream(stream));
}

int kvgov_cache_slots(const kvgov_cache *c, int64_t *slots) {
  if (!c || !slots) return KVGOV_E_INVAL;
  *slots = c->slots;
  return KVGOV_OK;
}

int kvgov_cache_insert(kvgov_cache *c, const uint8_t *hashes, const int64_t *blk_offsets,
                       int32_t n, int64_t n_blocks, int64_t *n_new, void *stream) {
  if (!c || !blk_offsets || n < 0 || n_blocks < 0 || (n_blocks > 0 && !hashes))
    return KVGOV_E_INVAL;
  if (reinterpret_cast<uintptr_t>(hashes) & 3) return KVGOV_E_INVAL;
  int rc = check_device(c);
  if (rc != KVGOV_OK) return rc;
  hipStream_t s = as_stream(stream);
  uint32_t epoch = 0;
  rc = cache_insert_rows(c, hashes, blk_offsets, n, n_blocks, s, &epoch);
  if (rc != KVGOV_OK || !n_new) return rc;
  return read_new_keys(c, epoch, n_new, s);
}

int kvgov_cache_lookup(kvgov_cache *c, const uint8_t *hashes, const int64_t *blk_offsets,
                       int32_t n, int64_t n_blocks, int32_t *hit_blocks, void *stream) {
  if (!c || !blk_offsets || n < 0 || n_blocks < 0 || (n_blocks > 0 && !hashes) ||
      (n > 0 && !hit_blocks))
    return KVGOV_E_INVAL;
  if (reinterpret_cast<uintptr_t>(hashes) & 3) return KVGOV_E_INVAL;
  int rc = check_device(c);
  if (rc != KVGOV_OK) return rc;
  if (n == 0) return KVGOV_OK;
  hipStream_t s = as_stream(stream);
  LookupArgs a{c->view, hashes, blk_offsets, n, n_blocks, hit_blocks};
  const int g = lookup_group(n, n_blocks);
  const dim3 grid((unsigned)ceil_div((int64_t)n * g, 256)), block(256);
  switch (g) {
    case 1: hipLaunchKernelGGL(k_lookup<1>, grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL(k_lookup<2>, grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL(k_lookup<4>, grid, block, 0, s, a); break;
    case 8: hipLaunchKernelGGL(k_lookup<8>, grid, block, 0, s, a); break;
    case 16: hipLaunchKernelGGL(k_lookup<16>, grid, block, 0, s, a); break;
    case 32: hipLaunchKernelGGL(k_lookup<32>, grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL(k_lookup<64>, grid, block, 0, s, a); break;
  }
  return launch_status();
}

// Lanes per request for the admission scan, which walks every row of a
// request: about one lane per 2 rows of the average request, 4 to 64.
static int admit_group(int32_t n, int64_t n_blocks) {
  const int64_t avg = n > 0 ? n_blocks / n : 0;
  int g = 4;
  while (g < 64 && (int64_t)g * 2 < avg) g <<= 1;
  return g;
}

int kvgov_cache_admit(kvgov_cache *c, const uint8_t *hashes, const int64_t *blk_offsets,
                      int32_t n, int64_t n_blocks, int32_t *hit_blocks, int32_t *new_blocks,
                      int64_t *n_new, void *stream) {
  if (!c || !blk_offsets || n < 0 || n_blocks < 0 || (n_blocks > 0 && !hashes) ||
      (n > 0 && (!hit_blocks || !new_blocks)))
    return KVGOV_E_INVAL;
  if (reinterpret_cast<uintptr_t>(hashes) & 3) return KVGOV_E_INVAL;
  int rc = check_device(c);
  if (rc != KVGOV_OK) return rc;
  if (n == 0) {
    if (n_new) *n_new = 0;
    return KVGOV_OK;
  }
  hipStream_t s = as_stream(stream);
  // per-row codes of the insert, in the stream's scratch (held while the two
  // kernels are enqueued)
  std::unique_lock<std::mutex> lk;
  void *scratch_p = nullptr;
  rc = stream_scratch(s, sizeof(uint32_t) * (size_t)std::max<int64_t>(n_blocks, 1), &scratch_p,
                      lk);
  if (rc != KVGOV_OK) return rc;
  uint32_t *codes = static_cast<uint32_t *>(scratch_p);
  const uint32_t epoch = next_epoch(c, s);
  if (epoch == 0xFFFFFFFFu) return KVGOV_E_UNSUPPORTED;
  if (c->view.track) note_tracked(c, n_blocks);
  rc = insert_batch<true>(c->view, hashes, blk_offsets, n, n_blocks, epoch, codes, s);
  if (rc != KVGOV_OK) return rc;
  AdmitArgs a{c->view, blk_offsets, n, n_blocks, epoch, codes, hit_blocks, new_blocks};
  const int g = admit_group(n, n_blocks);
  const dim3 grid((unsigned)ceil_div((int64_t)n * g, 256)), block(256);
  switch (g) {
    case 4: hipLaunchKernelGGL(k_admit_scan<4>, grid, block, 0, s, a); break;
    case 8: hipLaunchKernelGGL(k_admit_scan<8>, grid, block, 0, s, a); break;
    case 16: hipLaunchKernelGGL(k_admit_scan<16>, grid, block, 0, s, a); break;
    case 32: hipLaunchKernelGGL(k_admit_scan<32>, grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL(k_admit_scan<64>, grid, block, 0, s, a); break;
  }
  rc = launch_status();
  lk.unlock();
  if (rc != KVGOV_OK || !n_new) return rc;
  return read_new_keys(c, epoch, n_new, s);
}

int kvgov_cache_set_recency(kvgov_cache *c, int32_t on) {
  if (!c || (on != 0 && on != 1)) return KVGOV_E_INVAL;
  c->view.track = (uint32_t)on;
  return KVGOV_OK;
}

int kvgov_cache_evict(kvgov_cache *c, int64_t max_keys, int64_t *n_kept, void *stream) {
  if (!c || max_keys < 0) return KVGOV_E_INVAL;
  if (!c->view.track) return KVGOV_E_UNSUPPORTED;
  int rc = check_device(c);
  if (rc != KVGOV_OK) return rc;
  hipStream_t s = as_stream(stream);
  MaintScratch m;
  rc = maint_alloc(c, s, m);
  if (rc != KVGOV_OK) return rc;
  const int parts = (int)std::min<int64_t>(ceil_div(c->slots, 256 * 8), kRankParts);
  hipLaunchKernelGGL(k_rank_range, dim3(parts), dim3(256), 0, s, c->view, m.st, m.parts, m.hist,
                     (long long)max_keys);
  // enough passes for every bit that can differ: stamps up to the clock,
  // depths up to the largest tracked batch (a pass after the last needed one
  // ends at once); a captured eviction runs on tables of any later calls
  const int bits = is_capturing(s) ? 64
                                   : bit_length(c->epoch.load()) +
                                         bit_length((uint64_t)c->max_rows.load());
  const unsigned wgs = (unsigned)std::min<int64_t>(ceil_div(c->slots, kRankThreads * 8),
                                                   device_cu_count() * 2);
  for (int left = std::max(bits, 1); left > 0; left -= kRankDigit)
    hipLaunchKernelGGL(k_rank_select, dim3(wgs), dim3(kRankThreads), 0, s, c->view, m.st, m.parts,
                       parts, m.hist);
  c->rank_dirty = true;
  CacheMeta meta{};
  rc = compact_rebuild(c, s, m, 0, n_kept ? &meta : nullptr);
  if (rc == KVGOV_OK && n_kept) *n_kept = key_count(meta);
  return rc;
}

int kvgov_cache_erase(kvgov_cache *c, const uint8_t *keys, int64_t n_keys, int64_t *n_erased,
                      void *stream) {
  if (!c || n_keys < 0 || (n_keys > 0 && !keys)) return KVGOV_E_INVAL;
  if (reinterpret_cast<uintptr_t>(keys) & 3) return KVGOV_E_INVAL;
  int rc = check_device(c);
  if (rc != KVGOV_OK) return rc;
  hipStream_t s = as_stream(stream);
  MaintScratch m;
  rc = maint_alloc(c, s, m);
  if (rc != KVGOV_OK) return rc;
  if (n_keys > 0)
    hipLaunchKernelGGL(k_erase_mark, dim3((unsigned)ceil_div(n_keys, 256)), dim3(256), 0, s,
                       c->view, keys, n_keys);
  c->rank_dirty = true;
  CacheMeta meta{};
  rc = compact_rebuild(c, s, m, 1, n_erased ? &meta : nullptr);
  if (rc == KVGOV_OK && n_erased) *n_erased = (int64_t)meta.erased;
  return rc;
}

int kvgov_cache_count(kvgov_cache *c, int64_t *n_keys, void *stream) {
  if (!c || !n_keys) return KVGOV_E_INVAL;
  int rc = check_device(c);
  if (rc != KVGOV_OK) return rc;
  CacheMeta m{};
  rc = cache_read_meta(c, &m, as_stream(stream));
  if (rc != KVGOV_OK) return rc;
  *n_keys = key_count(m);
  return m.status;
}

int kvgov_cache_export(kvgov_cache *c, uint8_t *keys, int64_t cap, int64_t *n_keys,
                       void *stream) {
  if (!c || !n_keys || cap < 0 || (cap > 0 && !keys)) return KVGOV_E_INVAL;
  if (reinterpret_cast<uintptr_t>(keys) & 3) return KVGOV_E_INVAL;
  int rc = check_device(c);
  if (rc != KVGOV_OK) return rc;
  hipStream_t s = as_stream(stream);
  hipLaunchKernelGGL(k_export_begin, dim3(1), dim3(1), 0, s, c->view.meta);
  hipLaunchKernelGGL(k_export, dim3(grid_for(c->slots, 32)), dim3(256), 0, s, c->view, keys,
                     cap);
  rc = launch_status();
  if (rc != KVGOV_OK) return rc;
  CacheMeta m{};
  rc = cache_read_meta(c, &m, s);
  if (rc != KVGOV_OK) return rc;
  *n_keys = (int64_t)m.exported;
  return (int64_t)m.exported > cap ? KVGOV_E_CAPACITY : KVGOV_OK;
}

}  // extern "C"
