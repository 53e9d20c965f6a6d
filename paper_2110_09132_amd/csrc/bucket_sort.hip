// Sort of a batch's tokens by (key, position) for batches of up to
// kBucketMaxTokens tokens (a sample sort; Frazer & McKellar 1970), in two
// launches up to kBucketFewTokens tokens and three above.  The figures here are
// those of the smallest of the three configurations (BucketCfg, below).
//
//  1. bucket_split: every tile of 1024 tokens (2048 or 4096 in the larger
//     configurations) forms its keys, takes the same 512 (1024, 2048) sample
//     tokens of the batch, sorts their keys and keeps every second one as a
//     splitter (256, 512 or 1024 buckets of about equal size whatever the keys'
//     distribution; a key that fills a bucket by itself gets one of its own).
//     It then orders its tokens by bucket, stably, into its own part of a
//     scratch array and leaves where each bucket starts.
//  2. bucket_sort: one workgroup per bucket.  The tiles' starts tell it where
//     its tokens are, how many there are, and how many tokens the buckets
//     before it hold, so it needs nothing from the other workgroups.  It sorts
//     its tokens in LDS, writes them to their final places, and counts the
//     first tokens of each id for the reduction.  Buckets of one key need no
//     sort and can be long (a hot id): one more workgroup per tile copies its
//     tokens of those buckets.
//  3. bucket_copy, in the larger configurations: those copies in a launch of
//     their own, to the places that the buckets' workgroups have left.
// The result is the stable order by key, whatever the samples: they only
// decide how evenly the work is spread.
//
// The kernels are bound by latency (a chain of memory round trips, LDS steps
// and barriers; 64 tiles and 256 buckets for 65536 tokens), so what counts is
// how many dependent launches and round trips there are.  The radix sort of
// the same keys (key build, three passes, head count) takes five launches, its
// tiles waiting for each other in every pass.  Kernels of 65536 tokens of
// 24-bit keys, traced: 4.8 + 9.9 + 8.4 + 8.4 + 3.9 us -> 9.6 + 6.4 us; the
// owner-major call 57.8 -> 43.2 us, its 16384-token bf16 one 44.2 -> 31.7 us.
// Inside the first kernel (stamps): ids and owners 0.8 us (2.5 where every
// owner is a cache miss), the samples' sort 1.8, the bucket search 0.9, the
// ranking 1.5; inside the second: starts 0.6, tokens 0.6, the sort 1.8 (6 for a
// bucket of bunched keys), the writes 0.4.
#include "common.h"
#include "launch.h"
#include "sort_keys.h"

namespace emb {
namespace {

constexpr int kNT = 512;                      // threads of bucket_sort
constexpr int kNW = kNT / kWave;
constexpr int kMaxItems = 8;                  // tokens per thread of a bucket sorted in LDS
constexpr int kCap = kNT * kMaxItems;         // tokens of a bucket sorted in LDS, at most
constexpr uint32_t kCrowded = 64;             // tokens of one interval that make a bucket take radix passes
constexpr int kHeadWords = kCap / kRedTile + 2;

// 2^BITS buckets; tiles of ITEMS tokens per thread on NT threads.  COPYKERNEL:
// the tokens of one-key buckets are copied by a third launch instead of by more
// workgroups of the second.
template <int BITS, int NT, int ITEMS, int MAXTOKENS, bool COPYKERNEL>
struct BucketCfg {
  static constexpr bool kCopyKernel = COPYKERNEL;
  static constexpr int kThreads = NT, kBits = BITS, kItems = ITEMS;
  static constexpr int kBuckets = 1 << BITS;
  static constexpr int kSamples = 2 * kBuckets;
  static constexpr int kSampleItems = kSamples / NT;  // samples per thread
  static constexpr int kTile = NT * ITEMS;
  static constexpr int kMaxTokens = MAXTOKENS;
  static constexpr int kMaxTiles = MAXTOKENS / kTile;
  static constexpr int kTileSteps = kMaxTiles <= 128 ? 128 : 256;  // a power of two, for the search
  static constexpr int kRow = kBuckets + 8;           // half words of `starts` per tile
  static constexpr int kHeavyWords = kBuckets / 32;   // and one more: whether any bit is set
  // words of its own for T tokens: splitters, one-key bits, starts and, with the copy kernel, places
  static constexpr long long words(long long T) {
    return kBuckets + kHeavyWords + 1 + (T + kTile - 1) / kTile * (kRow / 2 + (COPYKERNEL ? kBuckets : 0));
  }
  static_assert(kSamples % NT == 0 && NT >= kBuckets && kMaxTiles <= kTileSteps && kTileSteps <= kNT, "whole shares");
};
// More tokens take more buckets: a bucket's share of the batch varies (its two
// samples' spacing), and one of more than kCap tokens is sorted slowly, so a
// bucket should hold about kCap / 8 on average.  More buckets cost the first
// kernel a longer sample sort and ranking in every tile (131072 tokens: 28 us
// with Few, 34 just above with Mid; 262144: 40 us with Mid, 55 with Many), and
// past Few's range the copies of one-key buckets by workgroups that each sum
// all tiles' starts cost more than a launch (524288 Zipf(1.3) tokens: 107 us
// against 65 with the copy kernel).
using Few = BucketCfg<8, 512, 2, kBucketFewTokens, false>;
using Mid = BucketCfg<9, 512, 4, kBucketMidTokens, true>;
using Many = BucketCfg<10, 1024, 4, kBucketMaxTokens, true>;
// They fit beside T words in 3/2 words per token, rounded up to 1024 tokens.
static_assert(Few::words(1) + 1 <= 1536 && Few::words(Few::kMaxTokens) <= Few::kMaxTokens / 2 &&
              Mid::words(Few::kMaxTokens + 1) <= Few::kMaxTokens / 2 && Mid::words(Mid::kMaxTokens) <= Mid::kMaxTokens / 2 &&
              Many::words(Mid::kMaxTokens + 1) <= Mid::kMaxTokens / 2 &&
              Many::words(kBucketMaxTokens) <= kBucketMaxTokens / 2, "the words fit the workspace");

// v of lane (lane ^ J), for a compile-time J: DPP moves inside rows of 16.
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  const int x = static_cast<int>(v);
  if constexpr (J == 1) return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, true));
  if constexpr (J == 2) return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, true));
  if constexpr (J == 4) {  // lanes reversed in groups of 8, then in groups of 4
    const int y = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, true);
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, y, 0x1B, 0xf, 0xf, true));
  }
  if constexpr (J == 8) return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, true));
  if constexpr (J == 16) return static_cast<uint32_t>(__builtin_amdgcn_ds_swizzle(x, 0x401F));
  return static_cast<uint32_t>(__shfl_xor(x, J, kWave));
}

// Ascending bitonic sort of IT * NT keys, element r * NT + thread in v[r].
template <int NT, int IT, int K, int J>
__device__ __forceinline__ void bitonic_merge(uint32_t (&v)[IT], uint32_t* buf) {
  const int tid = static_cast<int>(threadIdx.x);
  uint32_t other[IT];
  if constexpr (J >= NT) {
#pragma unroll
    for (int r = 0; r < IT; ++r) other[r] = v[r ^ (J / NT)];
  } else if constexpr (J < kWave) {
#pragma unroll
    for (int r = 0; r < IT; ++r) other[r] = lane_xor<J>(v[r]);
  } else {
#pragma unroll
    for (int r = 0; r < IT; ++r) buf[r * NT + tid] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < IT; ++r) other[r] = buf[r * NT + (tid ^ J)];
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < IT; ++r) {
    const int e = r * NT + tid;
    const bool keep_min = ((e & J) == 0) == ((e & K) == 0);
    v[r] = keep_min ? min(v[r], other[r]) : max(v[r], other[r]);
  }
  if constexpr (J > 1) bitonic_merge<NT, IT, K, J / 2>(v, buf);
}
template <int NT, int IT, int K>
__device__ __forceinline__ void bitonic_sort(uint32_t (&v)[IT], uint32_t* buf) {
  if constexpr (K > 2) bitonic_sort<NT, IT, K / 2>(v, buf);
  bitonic_merge<NT, IT, K, K / 2>(v, buf);
}

// Sample i's token: one at a scattered place of each of n equal shares
// of the batch (an even stride could meet a period of the tokens, such as the
// first token of every sentence).  The scattering is the first shift,
// multiplication and shift of xxHash32's final mix (Y. Collet's published
// specification; the multipliers are its primes 1 and 2) of i * prime 1 plus a
// constant, the low half of 2^64 / golden ratio.
__device__ __forceinline__ int sample_token(int i, int n, int Tc) {
  const int lo = static_cast<int>(static_cast<long long>(i) * Tc / n);
  const int hi = static_cast<int>(static_cast<long long>(i + 1) * Tc / n);
  uint32_t h = static_cast<uint32_t>(i) * 0x9E3779B1u + 0x7F4A7C15u;
  h ^= h >> 15;
  h *= 0x85EBCA77u;
  h ^= h >> 13;
  return lo + static_cast<int>((static_cast<uint64_t>(h) * static_cast<uint32_t>(max(hi - lo, 1))) >> 32);
}

// The bucket of a key: the number of splitters below it, or the next bucket if
// the key is a splitter at least twice (that bucket then holds this key alone).
// spl: kBuckets - 1 ascending splitters and one word of padding.
template <int kBuckets>
__device__ __forceinline__ uint32_t bucket_of(uint32_t key, const uint32_t* spl) {
  uint32_t pos = 0;
#pragma unroll
  for (uint32_t step = kBuckets / 2; step >= 1; step >>= 1)
    if (spl[pos + step - 1] < key) pos += step;
  if (pos < kBuckets - 1 && spl[pos] == key && spl[pos + 1] == key) ++pos;
  return pos;
}

template <class C>
__global__ __launch_bounds__(C::kThreads) void bucket_split_kernel(const int32_t* __restrict__ ids, int T, KeySpec ks,
                                                                   BucketWs ws, int nred, int32_t* status) {
  constexpr int NT = C::kThreads, NW = NT / kWave, kBuckets = C::kBuckets, kItems = C::kItems;
  constexpr int kSmp = C::kSampleItems, kAll = kItems + kSmp;
  __shared__ uint32_t buf[C::kSamples];
  __shared__ uint32_t spl[kBuckets];
  __shared__ uint32_t cnt[NW * kBuckets];
  __shared__ uint32_t dstart[kBuckets];
  __shared__ uint32_t wsum[NW];
  const int tid = static_cast<int>(threadIdx.x);
  const int w = tid / kWave;
  const int lane = static_cast<int>(lane_id());
  const int tile = static_cast<int>(blockIdx.x);
  const int Tc = ks.count_dev != nullptr ? min(max(*ks.count_dev, 0), T) : T;  // tokens that exist
  extern __shared__ uint32_t next_bits[];  // a bit per row that occurs in the next batch (ks.next_ids)
  // this thread's tokens, element (wave, round, lane) as the ranking walks them, and its samples
  int32_t id[kAll];
  int t[kAll];
#pragma unroll
  for (int r = 0; r < kItems; ++r) t[r] = tile * C::kTile + w * kItems * kWave + r * kWave + lane;
#pragma unroll
  for (int r = 0; r < kSmp; ++r) t[kItems + r] = sample_token(r * NT + tid, C::kSamples, Tc);
#pragma unroll
  for (int r = 0; r < kAll; ++r) id[r] = ids[min(t[r], T - 1)];
  uint32_t own[kAll], key[kAll];
  bool take[kAll];
  bool bad_id = false, bad_owner = false;
#pragma unroll
  for (int r = 0; r < kAll; ++r) {
    take[r] = id[r] >= 0 && static_cast<uint32_t>(id[r]) < ks.V;
    own[r] = 0;
    if (ks.row_owner != nullptr) own[r] = static_cast<uint32_t>(ks.row_owner[take[r] ? id[r] : 0]);
  }
  if (ks.next_ids != nullptr) {
    constexpr int kBatch = 8;  // next ids in flight per thread
    const int words = static_cast<int>((ks.V + 31) / 32);
    for (int i = tid; i < words; i += NT) next_bits[i] = 0;
    __syncthreads();
    for (int i0 = 0; i0 < ks.T_next; i0 += kBatch * NT) {
      int32_t nx[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) nx[k] = ks.next_ids[min(i0 + k * NT + tid, ks.T_next - 1)];
      // a look at all their words first: repeated ids (hot rows) then do not
      // queue on one word's atomic (past the end: the last id again)
      uint32_t seen[kBatch];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) seen[k] = next_bits[min(static_cast<uint32_t>(nx[k]), ks.V - 1) / 32];
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const uint32_t u = static_cast<uint32_t>(nx[k]);  // V < 2^31: a negative id is past every row
        const uint32_t bit = 1u << (u % 32);
        if (u < ks.V && (seen[k] & bit) == 0) atomicOr(&next_bits[u / 32], bit);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < kAll; ++r) {
    const bool exists = t[r] < Tc;
    const bool ownok = own[r] < static_cast<uint32_t>(ks.P);
    bad_id |= r < kItems && exists && !take[r];
    bad_owner |= r < kItems && exists && take[r] && !ownok;
    take[r] = exists && take[r] && ownok;
    key[r] = (own[r] << ks.ib) | static_cast<uint32_t>(id[r]);
    if (ks.next_ids != nullptr) {
      const uint32_t u = take[r] ? static_cast<uint32_t>(id[r]) : 0u;
      if (take[r] && ((next_bits[u / 32] >> (u % 32)) & 1u) == 0) key[r] |= 1u << ks.cls_shift;
    } else if (ks.next_tab != nullptr && take[r] && !in_next(static_cast<uint32_t>(id[r]), ks)) {
      key[r] |= 1u << ks.cls_shift;
    }
  }
  if (__any(bad_id) && lane == 0) raise_flag(status, EMB_DEV_ID_OUT_OF_RANGE);
  if (__any(bad_owner) && lane == 0) raise_flag(status, EMB_DEV_OWNER_OUT_OF_RANGE);
  // what the later kernels add to starts at zero
  for (int i = tile * NT + tid; i < nred; i += static_cast<int>(gridDim.x) * NT) ws.tile_heads[i] = 0;
  if (tile == 0 && tid == 0) *ws.span_count = 0;
  if (tile == 0 && ws.zero_counts != nullptr)
    for (int p = tid; p < ws.P; p += NT) ws.zero_counts[p] = 0;
  // the splitters: every second key of the sorted sample (a sample that takes no part sorts last)
  uint32_t s[kSmp];
#pragma unroll
  for (int r = 0; r < kSmp; ++r) s[r] = take[kItems + r] ? key[kItems + r] : 0xFFFFFFFFu;
  bitonic_sort<NT, kSmp, C::kSamples>(s, buf);
#pragma unroll
  for (int r = 0; r < kSmp; ++r) {
    const int e = r * NT + tid;
    if (e % 2 == 1) spl[e / 2] = e == C::kSamples - 1 ? 0xFFFFFFFFu : s[r];
  }
  __syncthreads();
  if (tile == 0) {  // for the second kernel: the splitters, and which buckets hold one key
    bool any = false;
    if (tid < kBuckets) {
      ws.splitters[tid] = spl[tid];
      const uint64_t m = __ballot(tid > 0 && spl[tid] == spl[max(tid - 1, 0)]);
      if (lane < 2) ws.heavy[w * 2 + lane] = static_cast<uint32_t>(m >> (32 * lane));
      any = m != 0;
    }
    any = __syncthreads_or(any ? 1 : 0) != 0;
    if (tid == 0) ws.heavy[C::kHeavyWords] = any ? 1u : 0u;
  }
  // this tile's tokens by bucket
  uint32_t dig[kItems], lpos[kItems];
  bool valid[kItems];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    valid[r] = take[r];
    dig[r] = bucket_of<kBuckets>(key[r], spl);
  }
  const uint32_t n = tile_stable_rank<NT, kItems, C::kBits>(dig, valid, kBuckets, C::kBits, cnt, dstart, wsum, lpos);
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    if (valid[r]) {
      const size_t at = static_cast<size_t>(tile) * C::kTile + lpos[r];
      ws.tile_keys[at] = key[r];
      ws.tile_vals[at] = static_cast<uint32_t>(t[r]);
    }
  }
  for (int b = tid; b <= kBuckets; b += NT)
    ws.starts[static_cast<size_t>(tile) * C::kRow + b] = static_cast<uint16_t>(b < kBuckets ? dstart[b] : n);
}

// LDS of the bucket sort.
template <class C>
struct BucketLds {
  int tpre[C::kTileSteps];   // bucket tokens in the tiles before
  int tsrc[C::kTileSteps];   // token j of the bucket, in tile t, is tile element tsrc[t] + j
  uint32_t wsum[kNW];
  int wcount[kNW], wlow[kNW];
  uint32_t hh[kHeadWords];   // heads per kRedTile sorted tokens, from the bucket's first
  uint32_t cnt[kCap + 1];    // per interval of keys: count, then start; the radix pass's counters
  uint32_t dstart[256];
  uint64_t mem[kCap];        // (key, token of the bucket), by interval; the radix pass's sorted keys
};

// Tile element of token j of the bucket: the last tile with tpre <= j.
template <class C>
__device__ __forceinline__ int bucket_source(const BucketLds<C>& l, int j) {
  int t = 0;
#pragma unroll
  for (int step = C::kTileSteps / 2; step >= 1; step >>= 1)
    if (l.tpre[t + step] <= j) t += step;
  return l.tsrc[t] + j;
}

// Sorts the bucket's n <= IT * kNT tokens in LDS; keys lie in [lo, lo + 2^wbits).
template <int IT, class C>
__device__ __forceinline__ void sort_bucket(BucketLds<C>& l, const BucketWs& ws, int T, int base, int n, uint32_t lo,
                                            int wbits) {
  const int tid = static_cast<int>(threadIdx.x);
  const int w = tid / kWave;
  uint32_t key[IT], val[IT], at[IT];
  bool valid[IT], head[IT];
  int j[IT];
#pragma unroll
  for (int r = 0; r < IT; ++r) {  // (wave, round, lane) order, as the ranking walks them
    j[r] = w * IT * kWave + r * kWave + static_cast<int>(lane_id());
    valid[r] = j[r] < n;
    const int src = min(bucket_source(l, min(j[r], n - 1)), T - 1);
    key[r] = ws.tile_keys[src];
    val[r] = ws.tile_vals[src];
  }
  bool radix = wbits <= 8;  // few distinct keys, perhaps with many tokens each
  if (!radix) {
    // kIntervals equal intervals of the key range, a token or two in each:
    // tokens go to their interval in any order, and each finds its place among
    // those of its interval by comparing (key, position) with all of them
    constexpr int kIntervals = IT * kNT;
    constexpr int kLog2 = IT == 1 ? 9 : IT == 2 ? 10 : IT == 4 ? 11 : 12;
    static_assert(kIntervals == 1 << kLog2, "a power of two");
    const int sh = max(wbits - kLog2, 0);
    for (int i = tid; i < kIntervals; i += kNT) l.cnt[i] = 0;
    __syncthreads();
    uint32_t iv[IT], arrival[IT];
    bool crowded = false;
#pragma unroll
    for (int r = 0; r < IT; ++r) {
      iv[r] = min((key[r] - lo) >> sh, static_cast<uint32_t>(kIntervals - 1));
      arrival[r] = valid[r] ? atomicAdd(&l.cnt[iv[r]], 1u) : 0u;
      crowded |= arrival[r] >= kCrowded;
    }
    radix = __syncthreads_or(crowded ? 1 : 0) != 0;  // keys bunched in a few intervals (a skewed tail)
    if (!radix) {
      block_exclusive_scan<kNT>(l.cnt, kIntervals, l.wsum);
      if (tid == 0) l.cnt[kIntervals] = static_cast<uint32_t>(n);
#pragma unroll
      for (int r = 0; r < IT; ++r)
        if (valid[r])
          l.mem[l.cnt[iv[r]] + arrival[r]] = (static_cast<uint64_t>(key[r]) << 32) | static_cast<uint32_t>(j[r]);
      __syncthreads();
#pragma unroll
      for (int r = 0; r < IT; ++r) {
        if (!valid[r]) continue;
        const uint64_t mine = (static_cast<uint64_t>(key[r]) << 32) | static_cast<uint32_t>(j[r]);
        const int s = static_cast<int>(l.cnt[iv[r]]), e = static_cast<int>(l.cnt[iv[r] + 1]);
        uint32_t below = 0;
        bool dup = false;
        for (int i = s; i < e; i += 4) {
          uint64_t m[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) m[q] = l.mem[min(i + q, e - 1)];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const bool less = i + q < e && m[q] < mine;
            below += less ? 1u : 0u;
            dup |= less && static_cast<uint32_t>(m[q] >> 32) == key[r];
          }
        }
        at[r] = static_cast<uint32_t>(s) + below;
        head[r] = !dup;
      }
    }
  }
  if (radix) {  // stable LSD passes in LDS
    const int npass = max((wbits + 7) / 8, 1);
    const int bits = (wbits + npass - 1) / npass;
    for (int p = 0; p < npass; ++p) {
      uint32_t dig[IT];
#pragma unroll
      for (int r = 0; r < IT; ++r) dig[r] = valid[r] ? ((key[r] - lo) >> (bits * p)) & ((1u << bits) - 1u) : 0u;
      (void)tile_stable_rank<kNT, IT, 8>(dig, valid, 1 << bits, bits, l.cnt, l.dstart, l.wsum, at);
#pragma unroll
      for (int r = 0; r < IT; ++r)
        if (valid[r]) l.mem[at[r]] = (static_cast<uint64_t>(key[r]) << 32) | val[r];
      __syncthreads();
      if (p + 1 < npass) {
#pragma unroll
        for (int r = 0; r < IT; ++r) {
          const uint64_t m = l.mem[j[r]];
          key[r] = static_cast<uint32_t>(m >> 32);
          val[r] = static_cast<uint32_t>(m);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < IT; ++r)
      head[r] = valid[r] && (at[r] == 0 || static_cast<uint32_t>(l.mem[at[r] - 1] >> 32) != key[r]);
  }
  const int first = base / kRedTile;
#pragma unroll
  for (int r = 0; r < IT; ++r) {
    const int pos = base + static_cast<int>(at[r]);
    if (!valid[r] || pos >= T) continue;
    ws.keys[pos] = key[r];
    ws.vals[pos] = val[r];
    if (head[r]) atomicAdd(&l.hh[pos / kRedTile - first], 1u);
  }
  __syncthreads();
  if (tid < kHeadWords && l.hh[tid] != 0 && first + tid <= (T - 1) / kRedTile) atomicAdd(&ws.tile_heads[first + tid], l.hh[tid]);
}

// A bucket of more than kCap tokens (rare: bucket_sorted in coalesce.hip says how
// rare, and what it costs): an LSD radix sort between the bucket's places in the
// result and in the scratch arrays, by this workgroup alone.
template <class C>
__device__ __forceinline__ void sort_long_bucket(BucketLds<C>& l, const BucketWs& ws, int T, int base, int n, uint32_t lo,
                                              int wbits) {
  n = min(n, T - base);
  const int tid = static_cast<int>(threadIdx.x);
  const int w = tid / kWave;
  uint32_t* run = reinterpret_cast<uint32_t*>(l.mem);  // [256]: where each digit's next token goes
  const int npass = max((wbits + 7) / 8, 1);
  for (int p = 0; p < npass; ++p) {
    const bool to_result = (npass - 1 - p) % 2 == 0;
    const uint32_t* ksrc = to_result ? ws.tmp_keys : ws.keys;
    const uint32_t* vsrc = to_result ? ws.tmp_vals : ws.vals;
    uint32_t* kdst = to_result ? ws.keys : ws.tmp_keys;
    uint32_t* vdst = to_result ? ws.vals : ws.tmp_vals;
    auto source = [&](int j) { return p == 0 ? min(bucket_source(l, j), T - 1) : base + j; };
    for (int d = tid; d < 256; d += kNT) run[d] = 0;
    __syncthreads();
    for (int j = tid; j < n; j += kNT) {
      const uint32_t k = p == 0 ? ws.tile_keys[source(j)] : ksrc[source(j)];
      atomicAdd(&run[((k - lo) >> (8 * p)) & 255u], 1u);
    }
    __syncthreads();
    block_exclusive_scan<kNT>(run, 256, l.wsum);
    for (int j0 = 0; j0 < n; j0 += kNT) {
      uint32_t dig[1], lpos[1];
      const int j = j0 + w * kWave + static_cast<int>(lane_id());
      const bool valid[1] = {j < n};
      const int src = source(min(j, n - 1));
      const uint32_t k = p == 0 ? ws.tile_keys[src] : ksrc[src];
      const uint32_t v = p == 0 ? ws.tile_vals[src] : vsrc[src];
      dig[0] = valid[0] ? ((k - lo) >> (8 * p)) & 255u : 0u;
      const uint32_t m = tile_stable_rank<kNT, 1, 8>(dig, valid, 256, 8, l.cnt, l.dstart, l.wsum, lpos);
      if (valid[0]) {
        const int pos = base + static_cast<int>(run[dig[0]] + (lpos[0] - l.dstart[dig[0]]));
        if (pos < T) {
          kdst[pos] = k;
          vdst[pos] = v;
        }
      }
      __syncthreads();
      for (int d = tid; d < 256; d += kNT) run[d] += (d < 255 ? l.dstart[d + 1] : m) - l.dstart[d];
      __syncthreads();
    }
    __threadfence_block();
    __syncthreads();
  }
  for (int j = tid; j < n; j += kNT)
    if (j == 0 || ws.keys[base + j] != ws.keys[base + j - 1]) atomicAdd(&ws.tile_heads[(base + j) / kRedTile], 1u);
}

// The tokens of one-key buckets in tile blockIdx.x, to the places the bucket's
// workgroup has left.
template <class C>
__global__ __launch_bounds__(C::kThreads) void bucket_copy_kernel(int T, BucketWs ws) {
  constexpr int NT = C::kThreads, kBuckets = C::kBuckets;
  __shared__ int row[kBuckets + 1];
  __shared__ int dst[kBuckets];
  if (ws.heavy[C::kHeavyWords] == 0) return;
  const int tid = static_cast<int>(threadIdx.x);
  const int t = static_cast<int>(blockIdx.x);
  const int most = min(C::kTile, T - t * C::kTile);
  for (int d = tid; d <= kBuckets; d += NT) {
    row[d] = min(static_cast<int>(ws.starts[static_cast<size_t>(t) * C::kRow + d]), most);
    if (d < kBuckets) {
      const bool heavy = (ws.heavy[d / 32] >> (d % 32)) & 1u;
      dst[d] = heavy ? ws.heavy_dst[static_cast<size_t>(t) * kBuckets + d] : -1;
    }
  }
  __syncthreads();
  const int n = row[kBuckets];
#pragma unroll
  for (int r = 0; r < C::kItems; ++r) {
    const int i = r * NT + tid;
    if (i >= n) break;
    int b = 0;  // the last bucket that starts at or before i
#pragma unroll
    for (int step = kBuckets / 2; step >= 1; step >>= 1)
      if (row[b + step] <= i) b += step;
    if (dst[b] < 0) continue;
    const int pos = dst[b] + i - row[b];
    if (pos < 0 || pos >= T) continue;
    ws.keys[pos] = ws.tile_keys[static_cast<size_t>(t) * C::kTile + i];
    ws.vals[pos] = ws.tile_vals[static_cast<size_t>(t) * C::kTile + i];
  }
}

// The tokens of one-key buckets in tile t, to their final places.
template <class C>
__device__ __forceinline__ void copy_heavy(BucketLds<C>& l, const BucketWs& ws, int T, int t, int ntiles) {
  constexpr int kBuckets = C::kBuckets, kParts = kNT > kBuckets ? kNT / kBuckets : 1, kBatch = 16;
  const int tid = static_cast<int>(threadIdx.x);
  int* dst = reinterpret_cast<int*>(l.mem);   // [kBuckets]: final place of element i of the tile, minus i
  int* part = dst + kBuckets;                 // [kParts][kBuckets]
  int* row = part + kParts * kBuckets;        // [kBuckets + 1]: this tile's starts
  static_assert((kParts + 2) * kBuckets + 1 <= 2 * kCap, "the copy's words fit");
  for (int i = tid; i < kParts * kBuckets; i += kNT) {
    const int d = i % kBuckets, p = i / kBuckets;
    int sum = 0;
    if ((ws.heavy[d / 32] >> (d % 32)) & 1u) {
      for (int q0 = p; q0 < ntiles; q0 += kParts * kBatch) {  // loads of kBatch tiles in flight
        int a[kBatch], e[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          const uint16_t* s = ws.starts + static_cast<size_t>(min(q0 + k * kParts, ntiles - 1)) * C::kRow + d;
          a[k] = s[0];
          e[k] = s[1];
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
          const int q = q0 + k * kParts;
          sum += q < ntiles ? a[k] + (q < t ? e[k] - a[k] : 0) : 0;
        }
      }
    }
    part[i] = sum;
  }
  const int most = min(C::kTile, T - t * C::kTile);
  for (int d = tid; d <= kBuckets; d += kNT)
    row[d] = min(static_cast<int>(ws.starts[static_cast<size_t>(t) * C::kRow + d]), most);
  __syncthreads();
  for (int d = tid; d < kBuckets; d += kNT) {
    int sum = -row[d];
#pragma unroll
    for (int p = 0; p < kParts; ++p) sum += part[p * kBuckets + d];
    dst[d] = ((ws.heavy[d / 32] >> (d % 32)) & 1u) ? sum : -1 - C::kTile;
  }
  __syncthreads();
  const int n = row[kBuckets];
  for (int i = tid; i < n; i += kNT) {
    int b = 0;  // the last bucket that starts at or before i
#pragma unroll
    for (int step = kBuckets / 2; step >= 1; step >>= 1)
      if (row[b + step] <= i) b += step;
    const int pos = dst[b] + i;
    if (pos < 0 || pos >= T) continue;
    ws.keys[pos] = ws.tile_keys[static_cast<size_t>(t) * C::kTile + i];
    ws.vals[pos] = ws.tile_vals[static_cast<size_t>(t) * C::kTile + i];
  }
}

// Workgroups 0 .. kBuckets - 1: one bucket each; the others: a tile's part of the one-key buckets.
template <class C>
__global__ __launch_bounds__(kNT) void bucket_sort_kernel(int T, int ntiles, int key_bits, BucketWs ws) {
  constexpr int kBuckets = C::kBuckets, kTileWaves = C::kTileSteps / kWave;
  __shared__ BucketLds<C> l;
  const int tid = static_cast<int>(threadIdx.x);
  const int w = tid / kWave;
  const int lane = static_cast<int>(lane_id());
  const int b = static_cast<int>(blockIdx.x);
  if (!C::kCopyKernel && b >= kBuckets) {
    if (ws.heavy[C::kHeavyWords] != 0) copy_heavy(l, ws, T, b - kBuckets, ntiles);
    return;
  }
  // the bucket's tokens per tile, and the tokens of earlier buckets
  int lo_t = 0, c = 0;
  if (tid < ntiles) {
    const uint16_t* s = ws.starts + static_cast<size_t>(tid) * C::kRow + b;
    lo_t = min(static_cast<int>(s[0]), C::kTile);
    c = max(min(static_cast<int>(s[1]), C::kTile) - lo_t, 0);
  }
  const uint32_t s_prev = ws.splitters[max(b - 1, 0)], s_this = ws.splitters[b];
  const bool heavy = (ws.heavy[b / 32] >> (b % 32)) & 1u;
  const int inc = static_cast<int>(wave_inclusive_scan(static_cast<uint32_t>(c)));
  const int lsum = static_cast<int>(wave_sum(static_cast<uint32_t>(lo_t)));
  if (lane == kWave - 1) {
    l.wcount[w] = inc;
    l.wlow[w] = lsum;
  }
  for (int i = tid; i < kHeadWords; i += kNT) l.hh[i] = 0;
  __syncthreads();
  int base = 0, n = 0, pre = inc - c;
#pragma unroll
  for (int q = 0; q < kTileWaves; ++q) {
    base += l.wlow[q];
    n += l.wcount[q];
    pre += q < w ? l.wcount[q] : 0;
  }
  if (tid < C::kTileSteps) {
    l.tpre[tid] = tid < ntiles ? pre : 0x7FFFFFFF;
    l.tsrc[tid] = tid * C::kTile + lo_t - pre;
  }
  if (b == kBuckets - 1 && tid == 0) *ws.n_valid = static_cast<uint32_t>(min(base + n, T));
  if (n == 0 || base >= T) return;  // (a bucket past the batch: only in a workspace overwritten meanwhile)
  if (heavy) {
    if (tid == 0) atomicAdd(&ws.tile_heads[base / kRedTile], 1u);
    if (C::kCopyKernel && tid < ntiles) ws.heavy_dst[static_cast<size_t>(tid) * kBuckets + b] = base + pre;
    return;
  }
  __syncthreads();
  // the bucket's keys lie in [lo, hi]
  const uint32_t lo = b == 0 ? 0u : s_prev + 1u;
  const uint32_t top = static_cast<uint32_t>((uint64_t{1} << key_bits) - 1u);
  const uint32_t hi = b == kBuckets - 1 ? top : min(s_this, top);
  const int wbits = hi > lo ? 32 - __clz(static_cast<int>(hi - lo)) : 0;
  if (n <= kNT)
    sort_bucket<1>(l, ws, T, base, n, lo, wbits);
  else if (n <= 2 * kNT)
    sort_bucket<2>(l, ws, T, base, n, lo, wbits);
  else if (n <= 4 * kNT)
    sort_bucket<4>(l, ws, T, base, n, lo, wbits);
  else if (n <= kCap)
    sort_bucket<8>(l, ws, T, base, n, lo, wbits);
  else
    sort_long_bucket(l, ws, T, base, n, lo, wbits);
}

}  // namespace

void launch_bucket_sort(const int32_t* ids, int T, const KeySpec& ks, int key_bits, BucketWs ws, uint32_t* words,
                        int nred, int32_t* status, hipStream_t stream) {
  const size_t next_lds = ks.next_ids != nullptr ? (ks.V + 31) / 32 * sizeof(uint32_t) : 0;
#define EMB_BUCKET(C)                                                                                               \
  do {                                                                                                              \
    const int ntiles = (T + C::kTile - 1) / C::kTile;                                                               \
    ws.splitters = words;                                                                                           \
    ws.heavy = words + C::kBuckets;                                                                                 \
    ws.starts = reinterpret_cast<uint16_t*>(words + C::kBuckets + C::kHeavyWords + 1);                              \
    ws.heavy_dst = reinterpret_cast<int32_t*>(words + C::kBuckets + C::kHeavyWords + 1 + ntiles * (C::kRow / 2));   \
    hipLaunchKernelGGL(bucket_split_kernel<C>, dim3(ntiles), dim3(C::kThreads), next_lds, stream, ids, T, ks, ws,   \
                       nred, status);                                                                               \
    hipLaunchKernelGGL(bucket_sort_kernel<C>, dim3(C::kBuckets + (C::kCopyKernel ? 0 : ntiles)), dim3(kNT), 0,      \
                       stream, T, ntiles, key_bits, ws);                                                            \
    if (C::kCopyKernel)                                                                                             \
      hipLaunchKernelGGL(bucket_copy_kernel<C>, dim3(ntiles), dim3(C::kThreads), 0, stream, T, ws);                 \
  } while (0)
  if (T <= Few::kMaxTokens)
    EMB_BUCKET(Few);
  else if (T <= Mid::kMaxTokens)
    EMB_BUCKET(Mid);
  else
    EMB_BUCKET(Many);
#undef EMB_BUCKET
}

}  // namespace emb
