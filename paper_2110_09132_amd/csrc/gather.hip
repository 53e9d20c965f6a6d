// Forward lookup (Sec. 4.1.1): out[t][:] = table[ids[t]][:].
//
// Each wave owns a contiguous range of output rows.  A row is handled by
// L = min(64, 2^ceil(log2(D / VEC))) lanes, so a wave covers 64 / L rows per
// step.  The ids of 64 rows come in one coalesced load (lane l holds the id of
// row l) and reach their lanes by shuffle; rows are processed in groups of
// kRowsInFlight steps, and the table loads of the next group are issued before
// the current group is stored (two register buffers used in turn), so each
// lane keeps two groups of independent 16-byte loads in flight.  Reads are whole table rows (cached: the
// update of the same step reads most of them again), writes contiguous rows (streaming stores).
#include <hip/hip_ext.h>

#include "common.h"
#include "launch.h"

namespace emb {
namespace {

constexpr int kThreads = 256;  // at most
constexpr int kRowsInFlight = 8;
// With fewer waves than this the launch spreads them out: workgroups of one
// wave, and wide rows' column steps over several of them.  2000 rows of 4 KB took
// 63 workgroups, each pulling 128 KB through one CU: 7.5 -> 6.1 us a call; 4000
// 8.6 -> 6.9, 8000 15.0 -> 11.7; 4200 rows of 256 bytes 4.0 -> 3.8.
// Rows that are not whole 128-byte lines share a line with the next wave's rows,
// which workgroups of one wave put on another XCD, whose L2 then writes its part of
// that line by itself: such rows are spread only where the column steps are split
// too, which pays all the same (3000 rows of 2053 floats 37.7 -> 22.1 us; but 5000 of
// 2052 13.5 -> 14.4, 5000 of 33 4.1 -> 4.4 with one wave per workgroup).
constexpr int kSpreadWaves = 1024;

// kWide: rows of more than one column step (Dv > 64).  The wave's column steps
// and row groups then run as one sequence of tiles, so that the loads of the
// next column step are in flight while the current one is stored (with few
// rows per wave, a single group per column step would otherwise wait for its
// loads step after step).
template <typename VecT, bool kWide>
__global__ __launch_bounds__(kThreads) void gather_kernel(const VecT* __restrict__ table, int64_t V, int Dv,
                                                          int log2L, const int32_t* __restrict__ ids, int T,
                                                          VecT* __restrict__ out, int32_t* status) {
  const int L = 1 << log2L;
  const int rpw = kWave >> log2L;
  const int lane = static_cast<int>(lane_id());
  const int sub = lane >> log2L;
  const int cl = lane & (L - 1);
  const int block_waves = static_cast<int>(blockDim.x) / kWave;
  const int wave = uniform(static_cast<int>(blockIdx.x) * block_waves + static_cast<int>(threadIdx.x / kWave));
  const int nwaves = static_cast<int>(gridDim.x) * block_waves;
  // rows of this wave: [r0, r1), a multiple of the rows one step covers
  const long long step_rows = static_cast<long long>(rpw) * kRowsInFlight;
  long long per = (static_cast<long long>(T) + nwaves - 1) / nwaves;
  per = (per + step_rows - 1) / step_rows * step_rows;
  const long long r0 = static_cast<long long>(wave) * per;
  const long long r1 = min(static_cast<long long>(T), r0 + per);
  bool bad = false;
  for (long long c0 = r0; c0 < r1; c0 += kWave) {  // 64 rows per id load
    const int n = static_cast<int>(min(static_cast<long long>(kWave), r1 - c0));
    const int32_t idreg = ids[min(c0 + lane, static_cast<long long>(T) - 1)];
    bad |= lane < n && (idreg < 0 || idreg >= V);
    // group g covers chunk rows [g * step_rows, (g + 1) * step_rows)
    const int ngroups = static_cast<int>((n + step_rows - 1) / step_rows);
    auto row_id = [&](int g, int u) {  // table row of this lane's row u of group g, -1 if none
      const int j = g * static_cast<int>(step_rows) + u * rpw + sub;
      const int id = __shfl(idreg, min(j, kWave - 1), kWave);
      return (j < n && id >= 0 && id < V) ? id : -1;
    };
    if constexpr (kWide) {
      // tiles (column step k: cb = k * L; row group g) in one sequence, two buffers in turn
      struct Tile {
        VecT v[kRowsInFlight];
        int id[kRowsInFlight];
        int c, g;
        bool live;
      } A, B;
      // (column steps blockIdx.y, blockIdx.y + gridDim.y, ... of this workgroup)
      const int part = static_cast<int>(blockIdx.y), parts = static_cast<int>(gridDim.y);
      const int nsteps = ((Dv + L - 1) / L - part + parts - 1) / parts;
      const int ntiles = nsteps * ngroups;
      int lk = 0, lg = 0, lq = 0;  // the next tile to load
      // a tile past the last one reads row 0 (one cached line) and is not stored
      auto load = [&](Tile& x) {
        x.live = lq < ntiles;
        x.g = x.live ? lg : 0;
        const int cb = (part + (x.live ? lk : 0) * parts) * L;
        x.c = min(cb + cl, Dv - 1);
        const bool cok = cb + cl < Dv;
#pragma unroll
        for (int u = 0; u < kRowsInFlight; ++u) {
          x.id[u] = x.live ? row_id(x.g, u) : -1;
          x.v[u] = table[static_cast<size_t>(x.id[u] < 0 ? 0 : x.id[u]) * Dv + x.c];
        }
        x.live = x.live && cok;
        ++lq;
        if (++lg == ngroups) {
          lg = 0;
          ++lk;
        }
      };
      auto store = [&](const Tile& x) {
        if (!x.live) return;
#pragma unroll
        for (int u = 0; u < kRowsInFlight; ++u) {
          const int j = x.g * static_cast<int>(step_rows) + u * rpw + sub;
          if (j < n) store_stream(&out[static_cast<size_t>(c0 + j) * Dv + x.c], x.id[u] < 0 ? VecT{} : x.v[u]);
        }
      };
      load(A);
      for (int q = 0; q < ntiles; q += 2) {
        load(B);
        store(A);
        load(A);
        store(B);
      }
      continue;
    }
    // column steps are uniform across the wave (the shuffles need every lane)
    for (int cb = 0; cb < Dv; cb += L) {
      const int c = min(cb + cl, Dv - 1);
      const bool cok = cb + cl < Dv;
      // two register buffers used in turn (every index is a compile-time
      // constant, and no loaded value is copied, so loads stay in flight)
      struct Group {
        VecT v[kRowsInFlight];
        int id[kRowsInFlight];
      } A, B;
      // loads are unconditional: past the last group they read row 0 and are not stored
      auto load = [&](int g, Group& x) {
#pragma unroll
        for (int u = 0; u < kRowsInFlight; ++u) {
          x.id[u] = row_id(g, u);
          x.v[u] = table[static_cast<size_t>(x.id[u] < 0 ? 0 : x.id[u]) * Dv + c];
        }
      };
      auto store = [&](int g, const Group& x) {
#pragma unroll
        for (int u = 0; u < kRowsInFlight; ++u) {
          const int j = g * static_cast<int>(step_rows) + u * rpw + sub;
          if (j < n && cok) store_stream(&out[static_cast<size_t>(c0 + j) * Dv + c], x.id[u] < 0 ? VecT{} : x.v[u]);
        }
      };
      load(0, A);
      for (int g = 0; g < ngroups; g += 2) {
        load(g + 1, B);
        store(g, A);
        load(g + 2, A);
        store(g + 1, B);
      }
    }
  }
  if (__any(bad) && lane_id() == 0) raise_flag(status, EMB_DEV_ID_OUT_OF_RANGE);
}

}  // namespace

hipError_t launch_gather(const float* table, int64_t V, int D, const int32_t* ids, int T, float* out,
                         int32_t* status, hipStream_t stream, hipEvent_t done) {
  if (T == 0) return done != nullptr ? hipEventRecord(done, stream) : hipSuccess;
  const bool vec4 = (D % 4 == 0) && (reinterpret_cast<uintptr_t>(table) % 16 == 0) &&
                    (reinterpret_cast<uintptr_t>(out) % 16 == 0);
  const int Dv = vec4 ? D / 4 : D;
  const RowLanes rl = row_lanes_for(Dv);
  const long long rows_per_wave = static_cast<long long>(rl.rows_per_wave()) * kRowsInFlight;
  const long long waves = (T + rows_per_wave - 1) / rows_per_wave;
  const bool wide = Dv > kWave;
  const bool lines = (static_cast<size_t>(D) * sizeof(float)) % 128 == 0;
  const bool spread = waves < kSpreadWaves && (lines || (wide && 2 * waves <= kSpreadWaves));
  const int threads = spread ? kWave : kThreads;
  const int parts = spread && wide ? static_cast<int>(grid_for(kSpreadWaves / waves, (Dv + kWave - 1) / kWave)) : 1;
  const dim3 grid(grid_for((waves * kWave + threads - 1) / threads, kMaxBlocks), parts);
  if (vec4) {
    const auto* tv = reinterpret_cast<const float4*>(table);
    auto* ov = reinterpret_cast<float4*>(out);
    if (wide)
      hipExtLaunchKernelGGL((gather_kernel<float4, true>), grid, dim3(threads), 0, stream, nullptr, done, 0, tv,
                            V, Dv, rl.log2_lanes, ids, T, ov, status);
    else
      hipExtLaunchKernelGGL((gather_kernel<float4, false>), grid, dim3(threads), 0, stream, nullptr, done, 0, tv,
                            V, Dv, rl.log2_lanes, ids, T, ov, status);
  } else {
    if (wide)
      hipExtLaunchKernelGGL((gather_kernel<float, true>), grid, dim3(threads), 0, stream, nullptr, done, 0,
                            table, V, Dv, rl.log2_lanes, ids, T, out, status);
    else
      hipExtLaunchKernelGGL((gather_kernel<float, false>), grid, dim3(threads), 0, stream, nullptr, done, 0,
                            table, V, Dv, rl.log2_lanes, ids, T, out, status);
  }
  return hipGetLastError();
}

}  // namespace emb
