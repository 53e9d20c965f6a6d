// Pack the coalesced rows by owner shard (Sec. 4.1.1 / 4.1.2): the layout an
// AlltoAll of sparse gradients sends, one contiguous block per owner.
//
// A stable partition by owner is one radix pass whose digit is the owner
// (P <= 1024 owners plus one bin for rows that are not sent):
//  1. per-tile owner histograms (LDS atomics); the owner digit of every row
//     is kept, so the owner table is read once,
//  2. per tile: global base of each owner (sum of earlier tiles and owners) +
//     stable rank inside the tile (wave ballots, as in the sort) -> the send
//     slot of every row; ids are written there, the slot is kept for step 3;
//     tile 0 writes send_counts / send_offsets,
//  3. the rows are copied to their slots (contiguous row reads and writes).
// With few tiles and owners (all histograms a few words per thread) 2 and 3 are
// one kernel (pack_place): a workgroup takes a few consecutive rows of a tile,
// issues their loads, finds their slots meanwhile, and stores them there.  For
// small packs the launches and the round trips between them are most of the
// time: 7100 rows of 2 KB, 4 owners 19.5 -> 14.0 us a call, 200 of 256 bytes
// 18.9 -> 11.7, 63500 of 1 KB, 16 owners 37.7 -> 33.4.
#include "common.h"
#include "launch.h"

namespace emb {
namespace {

constexpr int kThreads = 256;
constexpr int kItems = 4;
constexpr int kTile = kThreads * kItems;  // rows per tile
constexpr int kMaxOwners = 1024;
constexpr int kBinsMax = kMaxOwners + 1;
constexpr int kRowsInFlight = 8;
// Slots and copy are one kernel up to these sizes: histogram words of all tiles,
// bins (its LDS, and so its workgroups per CU, grow with them), and tiles.  With
// 1025 bins it ran three workgroups per CU: 63500 rows of 1 KB, 16 owners, 38.9
// us against 33.4; at 391 tiles 53.8 us against 52.2 with separate kernels.
constexpr int kPlaceHistWords = 8192;
constexpr int kPlaceBins = 257;
constexpr int kPlaceTiles = 256;

__device__ __forceinline__ int clamp_rows(const int32_t* num_unique, int cap) {
  const int u = num_unique[0];
  return u < 0 ? 0 : (u > cap ? cap : u);
}

// Owner of a row, or P when the row is not sent.  The owner table is read
// at a clamped index so the load never depends on a branch.
__device__ __forceinline__ uint32_t owner_of(int32_t id, const int32_t* __restrict__ row_owner, int64_t V, int P,
                                             int& flags) {
  const bool id_ok = id >= 0 && id < V;
  const int32_t o = row_owner[id_ok ? id : 0];
  if (!id_ok) {
    flags |= EMB_DEV_ID_OUT_OF_RANGE;
    return static_cast<uint32_t>(P);
  }
  if (o < 0 || o >= P) {
    flags |= EMB_DEV_OWNER_OUT_OF_RANGE;
    return static_cast<uint32_t>(P);
  }
  return static_cast<uint32_t>(o);
}

__global__ __launch_bounds__(kThreads) void pack_hist_kernel(const int32_t* __restrict__ uniq_ids,
                                                             const int32_t* __restrict__ num_unique, int cap,
                                                             const int32_t* __restrict__ row_owner, int64_t V, int P,
                                                             uint32_t* __restrict__ tile_hist,
                                                             uint16_t* __restrict__ digit_of, int32_t* status) {
  __shared__ uint32_t h[kBinsMax];
  const int bins = P + 1;
  for (int i = threadIdx.x; i < bins; i += kThreads) h[i] = 0;
  __syncthreads();
  const int U = clamp_rows(num_unique, cap);
  const int base = blockIdx.x * kTile;
  int flags = 0;
  if (base < U) {
    int32_t id[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) id[r] = uniq_ids[min(base + r * kThreads + static_cast<int>(threadIdx.x), U - 1)];
    uint32_t d[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) d[r] = owner_of(id[r], row_owner, V, P, flags);
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      const int k = base + r * kThreads + static_cast<int>(threadIdx.x);
      if (k < U) {
        atomicAdd(&h[d[r]], 1u);
        digit_of[k] = static_cast<uint16_t>(d[r]);
      }
    }
  }
  if (flags != 0) raise_flag(status, flags);
  __syncthreads();
  for (int i = threadIdx.x; i < bins; i += kThreads) tile_hist[static_cast<size_t>(blockIdx.x) * bins + i] = h[i];
}

__global__ __launch_bounds__(kThreads) void pack_scatter_kernel(
    const int32_t* __restrict__ uniq_ids, const int32_t* __restrict__ num_unique, int cap,
    const uint16_t* __restrict__ digit_of, int P, int owner_bits, const uint32_t* __restrict__ tile_hist,
    int ntiles, int32_t* __restrict__ send_ids, int32_t* __restrict__ slot_of, int32_t* __restrict__ send_counts,
    int32_t* __restrict__ send_offsets) {
  __shared__ uint32_t cnt[(kThreads / kWave) * kBinsMax];
  __shared__ uint32_t dstart[kBinsMax], colall[kBinsMax], gbase[kBinsMax];
  __shared__ uint32_t red_all[kBinsMax], red_bef[kBinsMax];
  __shared__ uint32_t wsum[kThreads / kWave];
  const int bins = P + 1;
  const int tile = blockIdx.x;
  const int base = tile * kTile;
  const int w = threadIdx.x / kWave;
  const int U = clamp_rows(num_unique, cap);

  int32_t id[kItems];
  uint32_t dig[kItems], lpos[kItems];
  bool valid[kItems];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int k = base + w * kItems * kWave + r * kWave + static_cast<int>(lane_id());
    const int kc = max(min(k, U - 1), 0);
    valid[r] = k < U;
    id[r] = uniq_ids[kc];
    dig[r] = digit_of[kc];
    if (!valid[r]) dig[r] = 0u;
  }
  const uint32_t total =
      tile_global_bases<kThreads>(tile_hist, ntiles, tile, bins, colall, gbase, red_all, red_bef, wsum);
  tile_stable_rank<kThreads, kItems>(dig, valid, bins, owner_bits, cnt, dstart, wsum, lpos);
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const int k = base + w * kItems * kWave + r * kWave + static_cast<int>(lane_id());
    if (!valid[r]) continue;
    const uint32_t d = dig[r];
    if (d == static_cast<uint32_t>(P)) {
      slot_of[k] = -1;
    } else {
      const uint32_t dest = gbase[d] + (lpos[r] - dstart[d]);
      send_ids[dest] = id[r];
      slot_of[k] = static_cast<int32_t>(dest);
    }
  }
  if (tile == 0) {
    for (int p = threadIdx.x; p < P; p += kThreads) {
      send_counts[p] = static_cast<int32_t>(colall[p]);
      send_offsets[p] = static_cast<int32_t>(gbase[p]);  // tile 0: nothing before it
    }
    if (threadIdx.x == 0) send_offsets[P] = static_cast<int32_t>(total - colall[P]);
  }
}

template <typename VecT>
__global__ __launch_bounds__(kThreads) void pack_rows_kernel(const VecT* __restrict__ uniq_grad,
                                                             const int32_t* __restrict__ num_unique, int cap,
                                                             const int32_t* __restrict__ slot_of, int Dv, int log2L,
                                                             VecT* __restrict__ send_rows) {
  const int U = clamp_rows(num_unique, cap);
  const int L = 1 << log2L;
  const int rpw = kWave >> log2L;
  const int sub = lane_id() >> log2L;
  const int cl = lane_id() & (L - 1);
  const long long wave = (static_cast<long long>(blockIdx.x) * kThreads + threadIdx.x) / kWave;
  const long long nwaves = static_cast<long long>(gridDim.x) * (kThreads / kWave);
  const long long step = static_cast<long long>(rpw) * kRowsInFlight;
  for (long long r0 = wave * step; r0 < U; r0 += nwaves * step) {
    int32_t dst[kRowsInFlight];
#pragma unroll
    for (int u = 0; u < kRowsInFlight; ++u) {
      const long long k = r0 + u * rpw + sub;
      dst[u] = slot_of[k < U ? k : U - 1];
      if (k >= U) dst[u] = -1;
    }
    for (int c = cl; c < Dv; c += L) {
      VecT v[kRowsInFlight];
#pragma unroll
      for (int u = 0; u < kRowsInFlight; ++u) {
        const long long k = r0 + u * rpw + sub;
        v[u] = uniq_grad[static_cast<size_t>(k < U ? k : U - 1) * Dv + c];
      }
#pragma unroll
      for (int u = 0; u < kRowsInFlight; ++u)
        if (dst[u] >= 0) send_rows[static_cast<size_t>(dst[u]) * Dv + c] = v[u];
    }
  }
}

// Steps 2 and 3 for `rows` consecutive rows of a tile (a power of two, at most
// kThreads): their source is one contiguous run of rows * Dv vectors, which the
// threads walk in order whatever the width.
template <typename VecT>
__global__ __launch_bounds__(kThreads) void pack_place_kernel(
    const int32_t* __restrict__ uniq_ids, const VecT* __restrict__ uniq_grad, const int32_t* __restrict__ num_unique,
    int cap, const uint16_t* __restrict__ digit_of, int P, int owner_bits, const uint32_t* __restrict__ tile_hist,
    int ntiles, int Dv, int rows, int32_t* __restrict__ send_ids, VecT* __restrict__ send_rows,
    int32_t* __restrict__ send_counts, int32_t* __restrict__ send_offsets) {
  __shared__ uint32_t cnt[(kThreads / kWave) * kPlaceBins];
  __shared__ uint32_t dstart[kPlaceBins], colall[kPlaceBins], gbase[kPlaceBins];
  __shared__ uint32_t red_all[kPlaceBins], red_bef[kPlaceBins];
  __shared__ uint32_t before[kPlaceBins];  // rows of each owner in the tile before this workgroup's
  __shared__ uint32_t wsum[kThreads / kWave];
  __shared__ int32_t slot[kThreads];
  const int bins = P + 1;
  const int tid = static_cast<int>(threadIdx.x);
  const int r0 = static_cast<int>(blockIdx.x) * rows;
  const int U = clamp_rows(num_unique, cap);
  if (r0 >= U && blockIdx.x != 0) return;  // (the first workgroup writes the counts in any case)
  const int n = max(min(rows, U - r0), 0);
  const int tile = r0 / kTile;
  const int units = n * Dv;
  const VecT* src = uniq_grad + static_cast<size_t>(r0) * Dv;
  // the rows' loads first: nothing below depends on them
  VecT v[kRowsInFlight];
#pragma unroll
  for (int k = 0; k < kRowsInFlight; ++k) v[k] = units > 0 ? src[min(tid + k * kThreads, units - 1)] : VecT{};
  const int row = min(r0 + tid, max(U - 1, 0));
  const bool valid[1] = {tid < n};
  const int32_t id = uniq_ids[row];
  const uint32_t mine = min(static_cast<uint32_t>(digit_of[row]), static_cast<uint32_t>(P));
  uint32_t dig[1] = {valid[0] ? mine : 0u}, lpos[1];
  for (int d = tid; d < bins; d += kThreads) before[d] = 0;
  __syncthreads();
  for (int k = tile * kTile + tid; k < r0; k += kThreads)
    atomicAdd(&before[min(static_cast<uint32_t>(digit_of[k]), static_cast<uint32_t>(P))], 1u);
  const uint32_t total =
      tile_global_bases<kThreads>(tile_hist, ntiles, tile, bins, colall, gbase, red_all, red_bef, wsum);
  tile_stable_rank<kThreads, 1>(dig, valid, bins, owner_bits, cnt, dstart, wsum, lpos);
  int32_t dest = -1;
  if (valid[0] && dig[0] != static_cast<uint32_t>(P)) {
    const uint32_t d = dig[0];
    dest = static_cast<int32_t>(gbase[d] + before[d] + (lpos[0] - dstart[d]));
    if (dest >= cap) dest = -1;  // (only with a workspace overwritten meanwhile)
    if (dest >= 0) send_ids[dest] = id;
  }
  slot[tid] = dest;
  if (blockIdx.x == 0) {
    for (int p = tid; p < P; p += kThreads) {
      send_counts[p] = static_cast<int32_t>(colall[p]);
      send_offsets[p] = static_cast<int32_t>(gbase[p]);  // the first rows: nothing before them
    }
    if (tid == 0) send_offsets[P] = static_cast<int32_t>(total - colall[P]);
  }
  __syncthreads();
  for (int i0 = 0; i0 < units; i0 += kRowsInFlight * kThreads) {
    if (i0 > 0) {
#pragma unroll
      for (int k = 0; k < kRowsInFlight; ++k) v[k] = src[min(i0 + tid + k * kThreads, units - 1)];
    }
#pragma unroll
    for (int k = 0; k < kRowsInFlight; ++k) {
      const int i = i0 + tid + k * kThreads;
      if (i >= units) continue;
      const int r = i / Dv;
      const int to = slot[r];
      if (to >= 0) send_rows[static_cast<size_t>(to) * Dv + (i - r * Dv)] = v[k];
    }
  }
}

struct PackWs {
  uint32_t* tile_hist;
  int32_t* slot_of;
  uint16_t* digit_of;
  size_t bytes;
};

PackWs carve(void* base, int cap, int P) {
  Carver cv{static_cast<char*>(base)};
  const size_t ntiles = (static_cast<size_t>(cap) + kTile - 1) / kTile;
  PackWs w;
  w.tile_hist = cv.take<uint32_t>((ntiles > 0 ? ntiles : 1) * static_cast<size_t>(P + 1));
  w.slot_of = cv.take<int32_t>(static_cast<size_t>(cap > 0 ? cap : 1));
  w.digit_of = cv.take<uint16_t>(static_cast<size_t>(cap > 0 ? cap : 1));
  w.bytes = cv.size();
  return w;
}

__global__ void empty_pack_kernel(int P, int32_t* send_counts, int32_t* send_offsets) {
  for (int p = threadIdx.x; p <= P; p += blockDim.x) {
    if (p < P) send_counts[p] = 0;
    send_offsets[p] = 0;
  }
}

}  // namespace

size_t pack_workspace_bytes(int cap_rows, int P) { return carve(nullptr, cap_rows, P).bytes; }

hipError_t launch_pack(const int32_t* uniq_ids, const float* uniq_grad, const int32_t* num_unique, int cap_rows,
                       int D, const int32_t* row_owner, int64_t V, int P, int32_t* send_ids, float* send_rows,
                       int32_t* send_counts, int32_t* send_offsets, void* workspace, int32_t* status,
                       hipStream_t stream) {
  if (cap_rows == 0) {
    hipLaunchKernelGGL(empty_pack_kernel, dim3(1), dim3(256), 0, stream, P, send_counts, send_offsets);
    return hipGetLastError();
  }
  PackWs ws = carve(workspace, cap_rows, P);
  const int ntiles = (cap_rows + kTile - 1) / kTile;
  int owner_bits = 0;
  while ((1 << owner_bits) <= P) ++owner_bits;  // digits 0..P
  hipLaunchKernelGGL(pack_hist_kernel, dim3(ntiles), dim3(kThreads), 0, stream, uniq_ids, num_unique, cap_rows,
                     row_owner, V, P, ws.tile_hist, ws.digit_of, status);
  const bool vec4 = (D % 4 == 0) && (reinterpret_cast<uintptr_t>(uniq_grad) % 16 == 0) &&
                    (reinterpret_cast<uintptr_t>(send_rows) % 16 == 0);
  const int Dv = vec4 ? D / 4 : D;
  // every workgroup of the one-kernel form sums all tiles' histograms: worth a
  // launch and the slots' round trip while that is a few loads per thread
  if (P + 1 <= kPlaceBins && ntiles <= kPlaceTiles &&
      static_cast<long long>(ntiles) * (P + 1) <= kPlaceHistWords) {
    int rows = kThreads;  // about kRowsInFlight vectors per thread
    while (rows > 1 && static_cast<long long>(rows) * Dv > kRowsInFlight * kThreads) rows /= 2;
    const unsigned groups = static_cast<unsigned>((static_cast<long long>(cap_rows) + rows - 1) / rows);
    if (vec4)
      hipLaunchKernelGGL(pack_place_kernel<float4>, dim3(groups), dim3(kThreads), 0, stream, uniq_ids,
                         reinterpret_cast<const float4*>(uniq_grad), num_unique, cap_rows, ws.digit_of, P, owner_bits,
                         ws.tile_hist, ntiles, Dv, rows, send_ids, reinterpret_cast<float4*>(send_rows), send_counts,
                         send_offsets);
    else
      hipLaunchKernelGGL(pack_place_kernel<float>, dim3(groups), dim3(kThreads), 0, stream, uniq_ids, uniq_grad,
                         num_unique, cap_rows, ws.digit_of, P, owner_bits, ws.tile_hist, ntiles, Dv, rows, send_ids,
                         send_rows, send_counts, send_offsets);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(pack_scatter_kernel, dim3(ntiles), dim3(kThreads), 0, stream, uniq_ids, num_unique, cap_rows,
                     ws.digit_of, P, owner_bits, ws.tile_hist, ntiles, send_ids, ws.slot_of, send_counts,
                     send_offsets);
  const RowLanes rl = row_lanes_for(Dv);
  const long long rows_per_block = static_cast<long long>(rl.rows_per_wave()) * kRowsInFlight * (kThreads / kWave);
  const unsigned grid = grid_for((cap_rows + rows_per_block - 1) / rows_per_block, kMaxBlocks);
  if (vec4)
    hipLaunchKernelGGL(pack_rows_kernel<float4>, dim3(grid), dim3(kThreads), 0, stream,
                       reinterpret_cast<const float4*>(uniq_grad), num_unique, cap_rows, ws.slot_of, Dv,
                       rl.log2_lanes, reinterpret_cast<float4*>(send_rows));
  else
    hipLaunchKernelGGL(pack_rows_kernel<float>, dim3(grid), dim3(kThreads), 0, stream, uniq_grad, num_unique,
                       cap_rows, ws.slot_of, Dv, rl.log2_lanes, send_rows);
  return hipGetLastError();
}

}  // namespace emb
