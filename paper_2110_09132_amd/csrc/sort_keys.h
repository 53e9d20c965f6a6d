// Sort keys of the coalesce and the sort of them, shared by coalesce.hip and bucket_sort.hip.
#pragma once

#include "common.h"

namespace emb {

// How a token's id becomes its sort key: the id itself; with row owners,
// owner << ib | id, which orders tokens by owner shard and by id inside it;
// with the vertical split as well, class << (ib + ob) | owner << ib | id, where
// class 0 marks the prior rows (the id occurs in the next batch) and 1 the
// delayed ones, so that the prior rows of every owner come first.
struct KeySpec {
  uint32_t V;                // ids in [0, V) take part
  const int32_t* row_owner;  // nullptr: the key is the id
  int32_t P;                 // owners in [0, P) take part
  int ib, ob;                // id bits and owner bits of a composite key
  uint32_t id_mask;          // key -> id
  uint32_t omask;            // (key >> ib) & omask -> owner
  int cls_shift;             // key >> cls_shift -> class (32: no class bit)
  const uint32_t* next_tab;  // set of the next batch's ids (nullptr: no split): one byte per
                             // row of [0, V) (next_bytemap), else a hash set of 2^(32 - tab_shift) slots
  bool next_bytemap;
  int tab_shift;
  const int32_t* next_ids;   // if given (and next_tab is not): the kernel builds the set in LDS from
  int T_next;                // these ids
  int G;                     // groups of the output: owners, times 2 with the split
  const int32_t* count_dev;  // if given: only the first *count_dev tokens take part
};

__device__ __forceinline__ int group_of(uint32_t key, const KeySpec& ks) {
  const int cls = static_cast<int>(static_cast<uint64_t>(key) >> ks.cls_shift);
  return cls * ks.P + static_cast<int>((key >> ks.ib) & ks.omask);
}

// Open-addressing hash set of ids (slot value id + 1, 0 = empty, linear probing).
__device__ __forceinline__ uint32_t tab_slot(uint32_t id, int shift) { return (id * 0x9E3779B1u) >> shift; }

__device__ __forceinline__ bool in_next(uint32_t id, const KeySpec& ks) {
  if (ks.next_bytemap) return reinterpret_cast<const uint8_t*>(ks.next_tab)[id] != 0;
  const uint32_t mask = 0xFFFFFFFFu >> ks.tab_shift;
  uint32_t slot = tab_slot(id, ks.tab_shift);
  for (uint32_t probe = 0; probe <= mask; ++probe) {
    const uint32_t v = ks.next_tab[slot];
    if (v == id + 1) return true;
    if (v == 0) return false;
    slot = (slot + 1) & mask;
  }
  return false;
}

constexpr int kRedTile = 128;  // sorted tokens per reduction workgroup: what tile_heads counts

// The bucket sort's part of the coalesce workspace (bucket_sort.hip).
struct BucketWs {
  uint32_t *tile_keys, *tile_vals;  // [T] each tile's tokens, ordered by bucket
  uint32_t *keys, *vals;            // [T] the sorted keys and positions (the result)
  uint32_t *tmp_keys, *tmp_vals;    // [T] for a bucket that does not fit in LDS
  uint32_t* n_valid;                // tokens that take part
  int32_t* span_count;              // cleared for the reduction
  int32_t* zero_counts;             // if given: P words cleared for the caller
  int P;
  uint32_t* tile_heads;             // [nred] first tokens of an id per kRedTile sorted tokens
  // set by the launch, in its words:
  uint32_t* splitters;              // ascending; one of padding at the end
  uint32_t* heavy;                  // buckets of one key (a bit each), and whether there is any
  uint16_t* starts;                 // per tile: where each bucket starts in it, and its token count
  int32_t* heavy_dst;               // per tile: where its tokens of each one-key bucket go
};
// The most tokens of the bucket sort's three configurations.
constexpr int kBucketFewTokens = 1 << 17, kBucketMidTokens = 1 << 18, kBucketMaxTokens = 5 << 17;
// The vertical split's set of next ids is built in LDS by each workgroup of the
// bucket sort's first kernel (a bit per row), up to these sizes: two launches
// (clear and insert, 6.5 us with their gaps) against reading the ids once per
// tile (split calls, 4096 tokens and next ids: 30.5 -> 27.1 us; 25000: 29.9 ->
// 31.3).  At 16384 ids it depends on whether they are in the caches, where a
// training step's next ids, just copied, need not be: 30.5 -> 28.5 us, but 44.5 ->
// 44.8 with rows of 4 KB that have passed through since; so half of that.  The
// set's up to 32 KB of LDS are measured with the smallest configuration only.
constexpr int64_t kLdsNextRows = 1 << 18;
constexpr int kLdsNextIds = 1 << 13;
inline bool bucket_next_in_lds(int64_t V, int T, int T_next) {
  return T <= kBucketFewTokens && V <= kLdsNextRows && T_next <= kLdsNextIds;
}
// Sorts T (1 .. kBucketMaxTokens) tokens by (key, position); key_bits: bits of
// the keys; words: 3/2 words per token (T rounded up to 1024) less T words.
void launch_bucket_sort(const int32_t* ids, int T, const KeySpec& ks, int key_bits, BucketWs ws, uint32_t* words,
                        int nred, int32_t* status, hipStream_t stream);

}  // namespace emb
