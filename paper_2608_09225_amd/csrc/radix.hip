// Token-granular prefix index: the radix-tree row of the paper's cache
// taxonomy (Table tab:taxonomy; Sec. 3.5: a radix tree reports the matched
// prefix length in tokens, finer than whole blocks), with the per-principal
// root of Sec. 4.1 (sigma_p as the root node gives each principal a disjoint
// tree).
//
// Structure: a trie whose nodes are
//   * block nodes: the chained digest h_j of a full block (the same keys as
//     the block prefix cache) and the roots (sigma_p, or 32 zero bytes for
//     the unsalted tree), stored in a block table (table.h); a node's id is
//     its slot index;
//   * token nodes: the prefixes of 1..15 tokens of a block below its parent
//     block node.  The first sequence to go below a block node leaves its
//     tokens there as the node's chain (one record of up to 15 tokens, one
//     compare-and-swap for all of its token nodes): the node of the chain's
//     first l tokens is (block node, l).  A sequence that leaves the chain, or
//     goes past its end, continues as edges (parent id, token) -> child in an
//     edge table of 64-bit keys; such a child's id is kEdgeBase + its edge
//     slot.
// A full block leads from the node of h_{j-1} to the node of h_j (through the
// block table: the 16th token is never a token node); a partial last block
// of an inserted sequence ends at a token node.  Match: the first block whose
// digest is absent gives the block depth m, and the longest walk over the
// chain and the edges below the node of h_{m-1} along the request's next
// tokens (at most 15) gives the rest: match = 16 m + steps.  The 16th step
// cannot exist: it would make block m present.
//
// Most blocks have one successor, so most token nodes are chains: 4096
// sequences of ~34 private blocks made 2.2 M edges, each a read, a
// compare-and-swap and a write at a random place of the edge table, one after
// the other along a block (236 us); as 147 k chains (46 us).
//
// Edge insert is one 64-bit compare-and-swap per edge (the key is the whole
// slot), so no lane ever reads a slot another lane is still writing.  A chain
// is claimed by a tag (call epoch, request); a lane of the same call that
// finds it claimed reads the claimant's tokens from the call's input, as the
// block table does with keys.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <new>

#include "table.h"

namespace kvgov {

constexpr unsigned long long kEdgeEmpty = ~0ull;
constexpr uint32_t kEdgeBase = 0x80000000u;  // id of the token node in edge slot e
constexpr uint32_t kOnesNode = 0x7FFFFFFFu;  // id of the all-0xFF block key (no slot)
constexpr uint32_t kNoNode = 0xFFFFFFFFu;
constexpr int kMaxLog2Radix = 30;           // keeps slot ids clear of the ids above
// Block tables up to this size keep chains, if there is memory for them: a token
// node of a chain has the id slot * 16 + l, below 2^30.  Larger ones (whose records
// would take another 72 bytes for each of 2^27 slots or more) have edges alone,
// and a block node's id is its slot.
constexpr int kMaxLog2Chains = 26;
constexpr int kChainMax = 15;

struct EdgeView {
  unsigned long long *keys;
  uint64_t mask;
  CacheMeta *meta;                 // the block table's: n_edges, radix_status
  unsigned long long *chain_tags;  // per block slot: 0, or (call epoch << 32) | (request + 1);
                                   // NULL: no chains
  u32x4 *chains;                   // per block slot: the token count, then up to 15 tokens
};

__device__ __forceinline__ uint64_t edge_hash(unsigned long long k) {
  uint64_t x = k * 0x9E3779B97F4A7C15ull;
  x ^= x >> 32;
  x *= 0xD6E8FEB86659FD93ull;
  x ^= x >> 32;
  return x;
}

__device__ __forceinline__ unsigned long long edge_key(uint32_t node, int32_t tok) {
  return ((unsigned long long)node << 32) | (uint32_t)tok;
}

// Child id of edge (node, tok), creating it if absent; kNoNode if the table
// is full (latched).  *added counts a created edge.
__device__ __forceinline__ uint32_t edge_insert(const EdgeView &e, uint32_t node, int32_t tok,
                                                uint32_t *added) {
  const unsigned long long key = edge_key(node, tok);
  uint64_t s = edge_hash(key) & e.mask;
  for (uint64_t p = 0; p <= e.mask; ++p) {
    unsigned long long cur = e.keys[s];
    if (cur == kEdgeEmpty) {
      cur = atomicCAS(&e.keys[s], kEdgeEmpty, key);
      if (cur == kEdgeEmpty) {
        ++*added;
        return kEdgeBase + (uint32_t)s;
      }
    }
    if (cur == key) return kEdgeBase + (uint32_t)s;
    s = (s + 1) & e.mask;
  }
  atomicCAS(&e.meta->radix_status, 0, KVGOV_E_FULL);
  return kNoNode;
}

__device__ __forceinline__ uint32_t edge_find(const EdgeView &e, uint32_t node, int32_t tok) {
  const unsigned long long key = edge_key(node, tok);
  uint64_t s = edge_hash(key) & e.mask;
  for (uint64_t p = 0; p <= e.mask; ++p) {
    const unsigned long long cur = e.keys[s];
    if (cur == key) return kEdgeBase + (uint32_t)s;
    if (cur == kEdgeEmpty) return kNoNode;
    s = (s + 1) & e.mask;
  }
  return kNoNode;
}

// Root keys into the block table (a row each; the insert protocol of
// table.h with `keys` as the call's input array).
__global__ __launch_bounds__(256) void k_radix_roots(TableView t, const uint8_t *keys,
                                                     int64_t count, uint32_t epoch) {
  uint32_t added = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count;
       i += (int64_t)gridDim.x * 256) {
    uint32_t code;
    added += insert_key<false>(t, load_key(keys + i * 32), i, 0, keys, epoch, &code, 0u);
  }
  if (added) atomicAdd(&t.meta->n_keys[blockIdx.x % kCounterLanes], (unsigned long long)added);
}

struct RadixArgs {
  TableView t;
  EdgeView e;
  const int32_t *tokens;
  int64_t n_tokens;
  const int64_t *tok_offsets;
  int32_t n;
  const int32_t *principal;
  const uint8_t *salts;  // ROOT: the roots; NONE: NULL (the zero root below)
  int32_t P;
  const uint8_t *zero_root;
  const uint8_t *hashes;
  const int64_t *blk_offsets;
  int64_t n_blocks;
  int32_t *match_len;  // match only
  uint32_t blk_epoch;  // insert only: the epoch of the call's block insert
};

// Request r's token range, full-block rows and root key, or false (latched).
struct RadixReq {
  int64_t t0, len, b0, nf;
  const uint8_t *root;
};

__device__ __forceinline__ bool radix_req(const RadixArgs &a, int64_t r, RadixReq &q) {
  q.t0 = a.tok_offsets[r];
  const int64_t t1 = a.tok_offsets[r + 1];
  q.b0 = a.blk_offsets[r];
  const int64_t b1 = a.blk_offsets[r + 1];
  q.len = t1 - q.t0;
  q.nf = b1 - q.b0;
  if (q.t0 < 0 || t1 < q.t0 || t1 > a.n_tokens || q.b0 < 0 || q.nf != (q.len >> 4) ||
      b1 > a.n_blocks) {
    atomicCAS(&a.e.meta->radix_status, 0, KVGOV_E_OFFSETS);
    return false;
  }
  if (a.salts) {
    const int32_t p = a.principal[r];
    if (p < 0 || p >= a.P) {
      atomicCAS(&a.e.meta->radix_status, 0, KVGOV_E_PRINCIPAL);
      return false;
    }
    q.root = a.salts + (int64_t)p * 32;
  } else {
    q.root = a.zero_root;
  }
  return true;
}

// The id of block node `slot` (find_slot's value) as a parent of edges.
__device__ __forceinline__ uint32_t node_id(const EdgeView &e, int64_t slot) {
  if (slot == -2) return kOnesNode;
  return e.chain_tags ? (uint32_t)slot * 16u : (uint32_t)slot;
}

// The slot that a row's key claimed with the tag `mine`, or -1 if another row
// or an earlier call holds the key: the claim lies on the key's probe sequence,
// before the first empty slot, so the tags alone tell, for as far as most
// sequences go; past that (a table that is nearly full) the key is looked
// for, which ends at the key.
__device__ __forceinline__ int64_t claimed_slot(const TableView &t, const Key &key,
                                                unsigned long long mine) {
  const uint64_t home = home_slot(key, t.mask);
  for (uint64_t p = 0; p < 8; ++p) {
    const uint64_t s = seq_slot(home, p, t.mask);
    const unsigned long long tag = t.tags[s];
    if (tag == mine) return (int64_t)s;
    if (tag == 0) return -1;
  }
  const int64_t slot = find_slot(t, key);
  return slot >= 0 && t.tags[slot] == mine ? slot : -1;
}

// A block's first 15 tokens (rem tokens from p on are the request's): 0 past
// its end.  A full block is four 16-byte loads.
__device__ __forceinline__ void load_tokens(const int32_t *p, int64_t rem, uint32_t tok[16]) {
  if (rem >= 16) {
    const u32x4 *v = reinterpret_cast<const u32x4 *>(p);
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const u32x4 w = v[x];
      tok[4 * x] = w.x;
      tok[4 * x + 1] = w.y;
      tok[4 * x + 2] = w.z;
      tok[4 * x + 3] = w.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kChainMax; ++i) tok[i] = i < rem ? (uint32_t)p[i] : 0u;
  }
}

// A chain's record: the token count, then the tokens.
__device__ __forceinline__ void load_chain(const u32x4 *rec, uint32_t c[16]) {
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const u32x4 v = rec[x];
    c[4 * x] = v.x;
    c[4 * x + 1] = v.y;
    c[4 * x + 2] = v.z;
    c[4 * x + 3] = v.w;
  }
}

// How many of the first n tokens agree.  (Compared as they come: two blocks of 16
// words held at once left five waves per SIMD of eight, and the walks along edges
// that follow wait for memory.)
__device__ __forceinline__ int same_tokens(const int32_t *p, const int32_t *q, int n) {
  int l = 0;
  for (; l + 4 <= n; l += 4) {
    const u32x4 v = *reinterpret_cast<const u32x4 *>(p + l);
    const u32x4 w = *reinterpret_cast<const u32x4 *>(q + l);
    if (v.x != w.x) return l;
    if (v.y != w.y) return l + 1;
    if (v.z != w.z) return l + 2;
    if (v.w != w.w) return l + 3;
  }
  while (l < n && p[l] == q[l]) ++l;
  return l;
}

// Inserts the token nodes of one (possibly partial) block below block node
// `slot`: record j of request r, rem tokens of the request at tp.  Returns
// the number of token nodes added.
__device__ __forceinline__ uint32_t insert_tokens(const RadixArgs &a, int64_t slot, int64_t r,
                                                  int64_t j, const int32_t *tp, int64_t rem) {
  const EdgeView &e = a.e;
  const int steps = (int)(rem < kChainMax ? rem : kChainMax);
  uint32_t added = 0;
  int l = 0;
  if (e.chain_tags && slot >= 0) {
    const unsigned long long mine =
        ((unsigned long long)a.blk_epoch << 32) | (unsigned long long)(r + 1);
    // read first: thousands of sequences may leave one node (65,536 sequences of
    // 24 tokens below the unsalted root: 871 us without the read, 165 with)
    unsigned long long tag = e.chain_tags[slot];
    u32x4 *rec = e.chains + slot * 4;
    if (tag == 0 && __hip_atomic_compare_exchange_strong(&e.chain_tags[slot], &tag, mine,
                                                         __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT)) {
      uint32_t tok[16];
      load_tokens(tp, rem, tok);
      rec[0] = u32x4{(uint32_t)steps, tok[0], tok[1], tok[2]};
#pragma unroll
      for (int q = 1; q < 4; ++q)
        rec[q] = u32x4{tok[4 * q - 1], tok[4 * q], tok[4 * q + 1], tok[4 * q + 2]};
      return (uint32_t)steps;
    }
    // the chain's tokens: claimed in this call, those of the same block of that
    // request (whose offsets the claimant found valid; a block that it does not
    // have, which only digests that are not its tokens' give, is an empty chain)
    const int32_t *chain = reinterpret_cast<const int32_t *>(rec) + 1;
    int64_t count;
    if ((uint32_t)(tag >> 32) == a.blk_epoch) {
      const int64_t q = (int64_t)(tag & 0xFFFFFFFFull) - 1;
      const int64_t t0 = a.tok_offsets[q];
      count = a.tok_offsets[q + 1] - t0 - 16 * j;
      chain = a.tokens + t0 + 16 * j;
    } else {
      count = chain[-1];
    }
    const int both = count < steps ? (int)(count < 0 ? 0 : count) : steps;
    l = same_tokens(tp, chain, both);
  }
  uint32_t node = node_id(e, slot) + (uint32_t)l;
  for (; l < steps && node != kNoNode; ++l) node = edge_insert(e, node, tp[l], &added);
  return added;
}

// Insert: G lanes per request, one (possibly partial) block each.  The token
// nodes of a full block j are fixed by h_j (its parent and its tokens), so
// only the row that claimed h_j in this call's block insert makes them: a
// block present before the call has them already, and every other row
// holding h_j would repeat them (thousands of rows of a shared prefix would
// otherwise contend on the same slots).  A partial last block has no digest
// and always makes its own.  A row that the block insert skipped, as equal to
// the previous request's row or to the row of the request that claimed its
// first key, claimed nothing: where that insert was by requests (BY_REQUEST)
// the same comparisons are made here first, and only the other rows look for
// their claim.  The parent's slot is mostly the neighbour lane's claim.
template <int G, bool BY_REQUEST>
__global__ __launch_bounds__(256) void k_radix_edges(RadixArgs a) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t r = gid / G;
  if (r >= a.n) return;
  const int sub = (int)(gid % G);
  const int base = (threadIdx.x & 63) & ~(G - 1);
  RadixReq q;
  if (!radix_req(a, r, q)) return;  // the whole group
  uint32_t added = 0;
  const int64_t nrec = (q.len + 15) >> 4;  // full blocks and a partial tail
  const int64_t lo = a.blk_offsets[0];
  const unsigned long long epoch = (unsigned long long)a.blk_epoch << 32;
  // the comparisons of the block insert (k_insert_req)
  int64_t b_p = 0, n_p = 0, g0 = -1;
  if (BY_REQUEST && q.nf > 0) {
    b_p = r >= 1 ? a.blk_offsets[r - 1] : 0;
    n_p = r >= 1 && b_p >= lo && b_p <= q.b0 ? q.b0 - b_p : 0;
    if (sub == 0 && q.b0 >= lo) {
      const Key key = load_key(a.hashes + q.b0 * 32);
      if (!(n_p > 0 && key_eq(key, load_key(a.hashes + b_p * 32)))) {
        const int64_t slot = find_slot(a.t, key);
        const unsigned long long tag =
            slot >= 0 ? a.t.tags[slot] : (slot == -2 ? a.t.meta->ones_tag : 0ull);
        const int64_t c = lo + (int64_t)(tag & 0xFFFFFFFFull) - 1;
        if ((tag >> 32) == a.blk_epoch && c >= lo && c < q.b0) g0 = c;
      }
    }
    g0 = __shfl(g0, base, 64);
  }
  int64_t before = -1;  // the claim of the row before this group's next lanes
  for (int64_t j0 = 0; j0 < nrec; j0 += G) {
    const int64_t j = j0 + sub;
    const int64_t f = q.b0 + j;
    int64_t slot = -1;  // this row's claim
    bool work = j < nrec;
    if (j < q.nf) {
      const Key key = load_key(a.hashes + f * 32);
      bool dup = false;
      if (BY_REQUEST && f >= lo) {
        dup = j < n_p && key_eq(key, load_key(a.hashes + (b_p + j) * 32));
        if (!dup && g0 >= 0 && j > 0) dup = key_eq(key, load_key(a.hashes + (g0 + j) * 32));
      }
      if (dup) {
        work = false;
      } else if (!key_is_empty_pattern(key)) {
        slot = claimed_slot(a.t, key, epoch | (unsigned long long)(f - lo + 1));
        work = slot >= 0;
      }
      // the all-0xFF digest has no tag: its token nodes are made again, which
      // changes nothing
    }
    int64_t parent = __shfl(slot, sub == 0 ? base : base + sub - 1, 64);
    if (sub == 0) parent = before;
    before = __shfl(slot, base + G - 1, 64);
    if (!work) continue;
    if (parent < 0)
      parent = find_slot(a.t, load_key(j == 0 ? q.root : a.hashes + (f - 1) * 32));
    if (parent == -1) {
      // the parent block was not inserted (a full table, latched there)
      atomicCAS(&a.e.meta->radix_status, 0, KVGOV_E_FULL);
      continue;
    }
    added += insert_tokens(a, parent, r, j, a.tokens + q.t0 + 16 * j, q.len - 16 * j);
  }
  if (added)
    atomicAdd(&a.e.meta->n_edges[blockIdx.x % kCounterLanes], (unsigned long long)added);
}

// Match: G lanes per request find the first absent block digest m (ballot),
// then one lane follows the chain and the edges below block node m - 1 (or the
// root).
template <int G>
__global__ __launch_bounds__(256) void k_radix_match(RadixArgs a) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t r = gid / G;
  if (r >= a.n) return;  // groups never straddle this test: 256 % G == 0
  const int sub = (int)(gid % G);
  const int lane = threadIdx.x & 63;
  const int base = lane & ~(G - 1);
  const uint64_t gmask = group_mask<G>(base);
  RadixReq q;
  if (!radix_req(a, r, q)) {
    if (sub == 0) a.match_len[r] = 0;
    return;
  }
  int64_t m = q.nf;
  int64_t slot = -1;    // of this lane's block
  int64_t parent = -1;  // of the last block found
  for (int64_t j0 = 0; j0 < q.nf; j0 += G) {
    const int64_t j = j0 + sub;
    slot = j < q.nf ? find_slot(a.t, load_key(a.hashes + (q.b0 + j) * 32)) : -1;
    const uint64_t mk = __ballot(slot == -1) & gmask;
    const int first = mk ? __builtin_ctzll(mk) - base : G;
    const int64_t found = __shfl(slot, base + (first > 0 ? first - 1 : 0), 64);
    if (first > 0) parent = found;
    if (mk) {
      m = j0 + first;
      break;
    }
  }
  if (sub != 0) return;
  if (m == 0) parent = find_slot(a.t, load_key(q.root));
  int64_t steps = 0;
  const int64_t rem = q.len - 16 * m;  // 0: a whole number of blocks, all found
  if (parent != -1 && rem > 0) {
    const int lim = (int)(rem < kChainMax ? rem : kChainMax);
    const int32_t *tp = a.tokens + q.t0 + 16 * m;
    bool below = true;  // the node has token nodes
    if (a.e.chain_tags && parent >= 0) {
      uint32_t tok[16], other[16];
      load_tokens(tp, rem, tok);
      load_chain(a.e.chains + parent * 4, other);
      below = a.e.chain_tags[parent] != 0;
      const int both = !below ? 0 : (lim < (int)other[0] ? lim : (int)other[0]);
      bool same = true;
#pragma unroll
      for (int i = 0; i < kChainMax; ++i) {
        same = same && i < both && tok[i] == other[1 + i];
        steps += same ? 1 : 0;
      }
    }
    uint32_t node = node_id(a.e, parent) + (uint32_t)steps;
    while (below && steps < lim) {
      node = edge_find(a.e, node, tp[steps]);
      if (node == kNoNode) break;
      ++steps;
    }
  }
  a.match_len[r] = (int32_t)(16 * m + steps);
}

}  // namespace kvgov

using namespace kvgov;

struct kvgov_radix {
  int device;
  kvgov_cache *blocks;
  EdgeView edges;
  int64_t edge_slots;
  uint8_t *zero_root;  // 32 zero bytes: the unsalted tree's root key
};

namespace {

int radix_check(const kvgov_radix *x) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return KVGOV_E_HIP;
  return dev == x->device ? KVGOV_OK : KVGOV_E_DEVICE;
}

// Empties the index: the block table's arrays, the token nodes' keys and, if
// there are chains, their tags, in one launch (2^20 block slots and 2^23 token
// nodes: 24.8 us as two, now 19.7).
int enqueue_radix_clear(kvgov_radix *x, hipStream_t s) {
  static_assert(kEdgeEmpty == ~0ull, "an empty token node is all ones");
  ClearMore more;
  more.ones = reinterpret_cast<u32x4 *>(x->edges.keys);
  more.n_ones = x->edge_slots / 2;
  if (x->edges.chain_tags) {
    more.zeros = reinterpret_cast<u32x4 *>(x->edges.chain_tags);
    more.n_zeros = x->blocks->slots / 2;
  }
  return cache_clear_with(x->blocks, s, more);
}

// Lanes per request: about one per two blocks of the average request, 4..64.
int radix_group(int32_t n, int64_t n_blocks) {
  const int64_t avg = n > 0 ? n_blocks / n : 0;
  int g = 4;
  while (g < 64 && (int64_t)g * 2 < avg) g <<= 1;
  return g;
}

// Shared argument checks of insert and match; fills the kernel arguments.
int radix_args(kvgov_radix *x, const int32_t *tokens, int64_t n_tokens,
               const int64_t *tok_offsets, int32_t n, const int32_t *principal,
               const uint8_t *salts, int32_t P, int32_t mode, const uint8_t *hashes,
               const int64_t *blk_offsets, int64_t n_blocks, RadixArgs &a) {
  if (!x || n < 0 || n_tokens < 0 || n_blocks < 0) return KVGOV_E_INVAL;
  if (mode == KVGOV_BOUNDARY) return KVGOV_E_UNSUPPORTED;
  if (mode != KVGOV_NONE && mode != KVGOV_ROOT) return KVGOV_E_INVAL;
  if (n > 0 && (!tok_offsets || !blk_offsets)) return KVGOV_E_INVAL;
  if ((n_tokens > 0 && !tokens) || (n_blocks > 0 && !hashes)) return KVGOV_E_INVAL;
  if (mode == KVGOV_ROOT && n > 0 && (!principal || !salts || P <= 0)) return KVGOV_E_INVAL;
  if ((reinterpret_cast<uintptr_t>(tokens) & 3) || (reinterpret_cast<uintptr_t>(hashes) & 3) ||
      (reinterpret_cast<uintptr_t>(salts) & 3))
    return KVGOV_E_INVAL;
  const int rc = radix_check(x);
  if (rc != KVGOV_OK) return rc;
  a = RadixArgs{};
  a.t = x->blocks->view;
  a.e = x->edges;
  a.tokens = tokens;
  a.n_tokens = n_tokens;
  a.tok_offsets = tok_offsets;
  a.n = n;
  a.principal = principal;
  a.salts = mode == KVGOV_ROOT ? salts : nullptr;
  a.P = P;
  a.zero_root = x->zero_root;
  a.hashes = hashes;
  a.blk_offsets = blk_offsets;
  a.n_blocks = n_blocks;
  return KVGOV_OK;
}

template <bool BY_REQUEST>
void radix_edges(const RadixArgs &a, int g, hipStream_t s) {
  const dim3 grid((unsigned)ceil_div((int64_t)a.n * g, 256)), block(256);
  switch (g) {
    case 4: hipLaunchKernelGGL((k_radix_edges<4, BY_REQUEST>), grid, block, 0, s, a); break;
    case 8: hipLaunchKernelGGL((k_radix_edges<8, BY_REQUEST>), grid, block, 0, s, a); break;
    case 16: hipLaunchKernelGGL((k_radix_edges<16, BY_REQUEST>), grid, block, 0, s, a); break;
    case 32: hipLaunchKernelGGL((k_radix_edges<32, BY_REQUEST>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((k_radix_edges<64, BY_REQUEST>), grid, block, 0, s, a); break;
  }
}

}  // namespace

extern "C" {

int kvgov_radix_create(int32_t log2_block_slots, int32_t log2_edge_slots, kvgov_radix **out) {
  if (!out || log2_block_slots < KVGOV_MIN_LOG2_SLOTS || log2_block_slots > kMaxLog2Radix ||
      log2_edge_slots < KVGOV_MIN_LOG2_SLOTS || log2_edge_slots > kMaxLog2Radix)
    return KVGOV_E_INVAL;
  *out = nullptr;
  kvgov_radix *x = new (std::nothrow) kvgov_radix();
  if (!x) return KVGOV_E_NOMEM;
  if (hipGetDevice(&x->device) != hipSuccess) {
    delete x;
    return KVGOV_E_HIP;
  }
  int rc = kvgov_cache_create(log2_block_slots, &x->blocks);
  if (rc != KVGOV_OK) {
    delete x;
    return rc;
  }
  x->edge_slots = (int64_t)1 << log2_edge_slots;
  x->edges.mask = (uint64_t)x->edge_slots - 1;
  void *keys = nullptr, *zero = nullptr, *ctags = nullptr, *chains = nullptr;
  if (hipMalloc(&keys, (size_t)x->edge_slots * 8) != hipSuccess ||
      hipMalloc(&zero, 32) != hipSuccess) {
    if (keys) (void)hipFree(keys);
    kvgov_cache_destroy(x->blocks);
    delete x;
    return KVGOV_E_NOMEM;
  }
  // where there is no memory for chains, edges alone
  if (log2_block_slots <= kMaxLog2Chains &&
      (hipMalloc(&ctags, (size_t)x->blocks->slots * 8) != hipSuccess ||
       hipMalloc(&chains, (size_t)x->blocks->slots * 64) != hipSuccess)) {
    (void)hipGetLastError();  // not left for the next launch check
    if (ctags) (void)hipFree(ctags);
    ctags = chains = nullptr;
  }
  x->edges.keys = static_cast<unsigned long long *>(keys);
  x->edges.meta = x->blocks->view.meta;
  x->zero_root = static_cast<uint8_t *>(zero);
  x->edges.chain_tags = static_cast<unsigned long long *>(ctags);
  x->edges.chains = static_cast<u32x4 *>(chains);
  rc = hipMemset(zero, 0, 32) == hipSuccess ? KVGOV_OK : KVGOV_E_HIP;
  if (rc == KVGOV_OK) rc = enqueue_radix_clear(x, nullptr);
  if (rc == KVGOV_OK && hipStreamSynchronize(nullptr) != hipSuccess) rc = KVGOV_E_HIP;
  if (rc != KVGOV_OK) {
    kvgov_radix_destroy(x);
    return rc;
  }
  *out = x;
  return KVGOV_OK;
}

int kvgov_radix_destroy(kvgov_radix *x) {
  if (!x) return KVGOV_OK;
  int rc = KVGOV_OK;
  if (hipDeviceSynchronize() != hipSuccess) rc = KVGOV_E_HIP;
  if (hipFree(x->edges.keys) != hipSuccess) rc = KVGOV_E_HIP;
  if (hipFree(x->zero_root) != hipSuccess) rc = KVGOV_E_HIP;
  if (hipFree(x->edges.chain_tags) != hipSuccess) rc = KVGOV_E_HIP;
  if (hipFree(x->edges.chains) != hipSuccess) rc = KVGOV_E_HIP;
  const int rb = kvgov_cache_destroy(x->blocks);
  if (rc == KVGOV_OK) rc = rb;
  delete x;
  return rc;
}

int kvgov_radix_clear(kvgov_radix *x, void *stream) {
  if (!x) return KVGOV_E_INVAL;
  int rc = radix_check(x);
  if (rc != KVGOV_OK) return rc;
  return enqueue_radix_clear(x, as_stream(stream));
}

int kvgov_radix_insert(kvgov_radix *x, const int32_t *tokens, int64_t n_tokens,
                       const int64_t *tok_offsets, int32_t n, const int32_t *principal,
                       const uint8_t *salts, int32_t P, int32_t mode, const uint8_t *hashes,
                       const int64_t *blk_offsets, int64_t n_blocks, void *stream) {
  RadixArgs a;
  int rc = radix_args(x, tokens, n_tokens, tok_offsets, n, principal, salts, P, mode, hashes,
                      blk_offsets, n_blocks, a);
  if (rc != KVGOV_OK || n == 0) return rc;
  hipStream_t s = as_stream(stream);
  // roots, then the full blocks' digests, then the edges below them
  kvgov_cache *c = x->blocks;
  const uint32_t epoch = next_epoch(c, s);
  if (epoch == 0xFFFFFFFFu) return KVGOV_E_UNSUPPORTED;
  const uint8_t *roots = mode == KVGOV_ROOT ? salts : x->zero_root;
  const int64_t n_roots = mode == KVGOV_ROOT ? P : 1;
  hipLaunchKernelGGL(k_radix_roots, dim3((unsigned)ceil_div(n_roots, 256)), dim3(256), 0, s,
                     c->view, roots, n_roots, epoch);
  rc = launch_status();
  if (rc != KVGOV_OK) return rc;
  rc = cache_insert_rows(c, hashes, blk_offsets, n, n_blocks, s, &a.blk_epoch);
  if (rc != KVGOV_OK) return rc;
  if (cache_inserts_by_request(c, n, n_blocks))
    radix_edges<true>(a, radix_group(n, n_blocks), s);
  else
    radix_edges<false>(a, radix_group(n, n_blocks), s);
  return launch_status();
}

int kvgov_radix_match(kvgov_radix *x, const int32_t *tokens, int64_t n_tokens,
                      const int64_t *tok_offsets, int32_t n, const int32_t *principal,
                      const uint8_t *salts, int32_t P, int32_t mode, const uint8_t *hashes,
                      const int64_t *blk_offsets, int64_t n_blocks, int32_t *match_len,
                      void *stream) {
  RadixArgs a;
  int rc = radix_args(x, tokens, n_tokens, tok_offsets, n, principal, salts, P, mode, hashes,
                      blk_offsets, n_blocks, a);
  if (rc != KVGOV_OK) return rc;
  if (n == 0) return KVGOV_OK;
  if (!match_len) return KVGOV_E_INVAL;
  a.match_len = match_len;
  hipStream_t s = as_stream(stream);
  const int g = radix_group(n, n_blocks) > 16 ? 64 : 16;
  const dim3 grid((unsigned)ceil_div((int64_t)n * g, 256)), block(256);
  if (g == 16)
    hipLaunchKernelGGL(k_radix_match<16>, grid, block, 0, s, a);
  else
    hipLaunchKernelGGL(k_radix_match<64>, grid, block, 0, s, a);
  return launch_status();
}

int kvgov_radix_stats(kvgov_radix *x, int64_t *block_nodes, int64_t *edges, void *stream) {
  if (!x || !block_nodes || !edges) return KVGOV_E_INVAL;
  int rc = radix_check(x);
  if (rc != KVGOV_OK) return rc;
  CacheMeta m{};
  rc = cache_read_meta(x->blocks, &m, as_stream(stream), true);
  if (rc != KVGOV_OK) return rc;
  int64_t e = 0;
  for (int i = 0; i < kCounterLanes; ++i) e += (int64_t)m.n_edges[i];
  *edges = e;
  *block_nodes = key_count(m);
  if (m.status != 0) return m.status;
  // token nodes of chains take no edge slot, but the index holds as many as it
  // has edge slots for
  if (m.radix_status == 0 && e > x->edge_slots) return KVGOV_E_FULL;
  return m.radix_status;
}

}  // extern "C"
