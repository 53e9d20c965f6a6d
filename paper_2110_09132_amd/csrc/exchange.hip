// The receiver side of the sparse-gradient exchange (Sec. 4.1.1 / 4.1.2: the
// coalesced rows go to their owners with an AlltoAll; an owner sums what it
// receives for the same row), simulated on one device for P workers.
//
//  1. exchange_offsets: from the P send layouts (worker w's rows for owner p
//     at [send_offsets[w][p], send_offsets[w][p + 1])), where each block lands
//     at its receiver: owner-major, senders in order inside an owner.  One
//     workgroup; P <= 1024.
//  2. exchange_rows: a P x P block transpose of ids and rows.  Each row finds
//     its owner block by binary search over its sender's offsets, which each
//     workgroup first copies to LDS with the receivers' destinations.
// With few workers (kFusedWorkers) every workgroup of 2 works the destinations
// out for itself from the P x P block sizes, and the first leaves recv_offsets:
// one launch (8 workers x 500 rows of 256 bytes: 11.3 -> 8.5 us a call; 32 x 2000
// of 1 KB 38.1 -> 28.1; 8 x 65536 of 1 KB 210.8 -> 209.4).
// The merge of the received runs is the owner-major coalesce with a token
// count read on the device (the received total), in coalesce.hip.
#include "common.h"
#include "launch.h"

namespace emb {
namespace {

constexpr int kThreads = 1024;       // one thread per owner in exchange_offsets
constexpr int kRowThreads = 256;
constexpr int kRowsInFlight = 8;

// counts[w][p], from the offsets of sender w, clamped into [0, cap] and made monotone
__device__ __forceinline__ int block_count(const int32_t* __restrict__ offs, int P, int cap, int w, int p) {
  const int32_t* o = offs + static_cast<size_t>(w) * (P + 1);
  const int a = min(max(o[p], 0), cap);
  const int b = min(max(o[p + 1], a), cap);
  return b - a;
}

__global__ __launch_bounds__(kThreads) void exchange_offsets_kernel(const int32_t* __restrict__ send_offsets, int P,
                                                                    int cap, int32_t* __restrict__ recv_offsets,
                                                                    int32_t* __restrict__ recv_total) {
  __shared__ uint32_t base[kThreads];
  __shared__ uint32_t wsum[kThreads / kWave];
  const int p = threadIdx.x;
  uint32_t total = 0;
  if (p < P)
    for (int w = 0; w < P; ++w) total += static_cast<uint32_t>(block_count(send_offsets, P, cap, w, p));
  base[p] = total;
  __syncthreads();
  const uint32_t all = block_exclusive_scan<kThreads>(base, P, wsum);
  if (p < P) {
    uint32_t run = base[p];
    int32_t* r = recv_offsets + static_cast<size_t>(p) * (P + 1);
    for (int w = 0; w < P; ++w) {
      r[w] = static_cast<int32_t>(run);
      run += static_cast<uint32_t>(block_count(send_offsets, P, cap, w, p));
    }
    r[P] = static_cast<int32_t>(run);
  }
  if (p == 0) *recv_total = static_cast<int32_t>(all);
}

// exchange_rows works out the destinations itself for up to this many workers (a
// word or four per thread to load, and P of them to add up), and while its
// workgroups together read at most kFusedWords block sizes.  Where they read more, a
// launch of its own costs less: 32 workers x 50000 half-filled rows of 512 bytes,
// 25024 workgroups: 191 us with the destinations in each, 179 without; 20000 rows of
// 1 KB, 155 against 149; 12000 of 512 bytes, 6016 workgroups, 39.6 against 48.2.
constexpr int kFusedWorkers = 32;
constexpr long long kFusedWords = 8 << 20;
// In a launch of this many workgroups one that has no row first looks whether it has
// (8 workers x 130000 half-filled rows of 1 KB, 32504 workgroups: 236 -> 202 us); in
// smaller ones that round trip costs more (32 x 40000 half-filled rows of 128 bytes,
// 5024 workgroups: 36.6 -> 38.1).
constexpr unsigned kManyGroups = 8192;

// Row k of sender w (k < its sent rows) goes to receiver p, the owner block
// holding k, at recv_offsets[p][w] + (k - send_offsets[w][p]).  L lanes per row.
// kFused: the destinations are worked out here; kLook: see kManyGroups.
template <typename VecT, bool kFused, bool kLook>
__global__ __launch_bounds__(kRowThreads) void exchange_rows_kernel(
    const int32_t* __restrict__ send_ids, const VecT* __restrict__ send_rows, const int32_t* __restrict__ send_offsets,
    int P, int cap, int Dv, int log2L, int32_t* __restrict__ recv_offsets, int32_t* __restrict__ recv_total,
    int32_t* __restrict__ recv_ids, VecT* __restrict__ recv_rows) {
  // the sender's offsets, block sizes and destinations, once per workgroup in LDS
  // (a row then finds its block by a binary search in LDS, not in memory)
  __shared__ int32_t s_o[kThreads + 1];   // send_offsets[w][p]
  __shared__ int32_t s_cnt[kThreads];     // rows of block p (clamped)
  __shared__ int32_t s_dst[kThreads];     // where receiver p puts them: recv_offsets[p][w]
  const int L = 1 << log2L;
  const int rpw = kWave >> log2L;
  const int sub = static_cast<int>(lane_id()) >> log2L;
  const int cl = static_cast<int>(lane_id()) & (L - 1);
  const int w = blockIdx.y;  // the sender
  const int32_t* o = send_offsets + static_cast<size_t>(w) * (P + 1);
  const long long step = static_cast<long long>(rpw) * kRowsInFlight;
  if (kLook && blockIdx.x > 0 && blockIdx.x * (kRowThreads / kWave) * step >= min(max(o[P], 0), cap))
    return;  // no row for this workgroup (the first one leaves recv_offsets all the same)
  for (int p = threadIdx.x; p <= P; p += kRowThreads) {
    s_o[p] = o[p];
    if (p < P) {
      s_cnt[p] = block_count(send_offsets, P, cap, w, p);
      if (!kFused) s_dst[p] = recv_offsets[static_cast<size_t>(p) * (P + 1) + w];
    }
  }
  if constexpr (kFused) {
    __shared__ int32_t s_all[kFusedWorkers * kFusedWorkers];  // rows of sender i / P for owner i % P
    __shared__ int32_t s_tot[kFusedWorkers];                  // rows for each owner
    for (int i = threadIdx.x; i < P * P; i += kRowThreads) s_all[i] = block_count(send_offsets, P, cap, i / P, i % P);
    __syncthreads();
    const int p = static_cast<int>(threadIdx.x);
    int total = 0, before = 0;
    if (p < P) {
      for (int q = 0; q < P; ++q) {
        const int c = s_all[q * P + p];
        total += c;
        before += q < w ? c : 0;
      }
      s_tot[p] = total;
    }
    __syncthreads();
    if (p < P) {
      int base = 0;
      for (int q = 0; q < p; ++q) base += s_tot[q];
      s_dst[p] = base + before;
      if (blockIdx.x == 0 && w == 0) {
        int32_t* r = recv_offsets + static_cast<size_t>(p) * (P + 1);
        int run = base;
        for (int q = 0; q < P; ++q) {
          r[q] = run;
          run += s_all[q * P + p];
        }
        r[P] = run;
        if (p == P - 1) *recv_total = run;
      }
    }
  }
  __syncthreads();
  const int sent = min(max(s_o[P], 0), cap);
  const long long wave = (static_cast<long long>(blockIdx.x) * kRowThreads + threadIdx.x) / kWave;
  const long long nwaves = static_cast<long long>(gridDim.x) * (kRowThreads / kWave);
  for (long long r0 = wave * step; r0 < sent; r0 += nwaves * step) {
    int64_t dst[kRowsInFlight];
    int64_t src[kRowsInFlight];
#pragma unroll
    for (int u = 0; u < kRowsInFlight; ++u) {
      const long long k = r0 + u * rpw + sub;
      const int kc = static_cast<int>(k < sent ? k : sent - 1);
      // owner block of row kc: the last p with o[p] <= kc (offsets are ascending)
      int lo = 0, hi = P - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_o[mid] <= kc) lo = mid; else hi = mid - 1;
      }
      const int a = min(max(s_o[lo], 0), cap);
      const int off = kc - a;  // inside the block unless the offsets are malformed
      src[u] = static_cast<int64_t>(w) * cap + kc;
      dst[u] = (k < sent && off >= 0 && off < s_cnt[lo]) ? static_cast<int64_t>(s_dst[lo]) + off : -1;
    }
    if (cl == 0) {
#pragma unroll
      for (int u = 0; u < kRowsInFlight; ++u)
        if (dst[u] >= 0) recv_ids[dst[u]] = send_ids[src[u]];
    }
    for (int c = cl; c < Dv; c += L) {
      VecT v[kRowsInFlight];
#pragma unroll
      for (int u = 0; u < kRowsInFlight; ++u) v[u] = send_rows[static_cast<size_t>(src[u]) * Dv + c];
#pragma unroll
      for (int u = 0; u < kRowsInFlight; ++u)
        if (dst[u] >= 0) recv_rows[static_cast<size_t>(dst[u]) * Dv + c] = v[u];
    }
  }
}

}  // namespace

hipError_t launch_exchange(const int32_t* send_ids, const float* send_rows, const int32_t* send_offsets, int P,
                           int cap, int D, int32_t* recv_ids, float* recv_rows, int32_t* recv_offsets,
                           int32_t* recv_total, hipStream_t stream) {
  const auto al16 = [](const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
  const bool vec4 = (D % 4 == 0) && al16(send_rows) && al16(recv_rows);
  const int Dv = vec4 ? D / 4 : D;
  const RowLanes rl = row_lanes_for(Dv);
  const long long rows_per_block = static_cast<long long>(rl.rows_per_wave()) * kRowsInFlight * (kRowThreads / kWave);
  const dim3 grid(grid_for((cap + rows_per_block - 1) / rows_per_block, 65535), P);
  const bool look = grid.x * grid.y >= kManyGroups;
  const bool fused = cap > 0 && P <= kFusedWorkers && static_cast<long long>(grid.x) * P * P * P <= kFusedWords;
  if (!fused)
    hipLaunchKernelGGL(exchange_offsets_kernel, dim3(1), dim3(kThreads), 0, stream, send_offsets, P, cap, recv_offsets,
                       recv_total);
  if (cap == 0) return hipGetLastError();
#define EMB_EXCHANGE(VT, FUSED, LOOK)                                                                               \
  hipLaunchKernelGGL((exchange_rows_kernel<VT, FUSED, LOOK>), grid, dim3(kRowThreads), 0, stream, send_ids,         \
                     reinterpret_cast<const VT*>(send_rows), send_offsets, P, cap, Dv, rl.log2_lanes, recv_offsets, \
                     recv_total, recv_ids, reinterpret_cast<VT*>(recv_rows))
#define EMB_EXCHANGE_V(VT)                        \
  do {                                            \
    if (fused && look)                            \
      EMB_EXCHANGE(VT, true, true);               \
    else if (fused)                               \
      EMB_EXCHANGE(VT, true, false);              \
    else                                          \
      EMB_EXCHANGE(VT, false, false);             \
  } while (0)
  if (vec4)
    EMB_EXCHANGE_V(float4);
  else
    EMB_EXCHANGE_V(float);
#undef EMB_EXCHANGE_V
#undef EMB_EXCHANGE
  return hipGetLastError();
}

}  // namespace emb
