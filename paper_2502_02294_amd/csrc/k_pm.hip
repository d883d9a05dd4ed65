// Particle-mesh kernels (Sec. 2.2): cell keys, a stable counting sort of the particles by
// their CIC base cell, the deterministic CIC deposit as a per-cell gather over the bins
// that can reach a cell, the mesh acceleration g = -grad(phi) (two-point central
// difference) and its CIC read-out, kick and drift (eq. dm_hamil: dx/dt = p/a^2,
// dp/dt = g), and the adjoints of all of them.
//
// CIC on cell centres: with s = x - 1/2, i0 = floor(s), w1 = s - i0, a particle puts
// weight (1-w1) in cell i0 and w1 in i0+1 per axis.  Cell c receives from particles whose
// base cell is c - o, o in {0,1}^3.  After the sort, the particles' upper weights w1 are gathered
// into bin order (float3 per particle); the deposit sums each bin's 8 corner weights in LDS and
// each cell adds its 8 corners, in a fixed order and with ascending particle id inside a bin:
// every sum is reproducible bit for bit without float atomics.
#include "dh_kernels.h"

namespace dh {

namespace {

constexpr int kScanThreads = 1024;
constexpr int kLargeSortBlocks = 512;   // two blocks of 64 KB of LDS per CU
constexpr int kLargeSortThreads = 1024;
constexpr int kScanTile = kScanThreads * 4;   // one 16-byte vector of counts a thread

__device__ __forceinline__ int wrapi(int j, int n) { return j & (n - 1); }

struct Cic {
  int i0[3];
  float w1[3];
};

__device__ __forceinline__ Cic cic_of(float x, float y, float z, int n) {
  Cic c;
  const float v[3] = {x, y, z};
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float s = v[d] - 0.5f;
    const float f = floorf(s);
    c.w1[d] = s - f;
    c.i0[d] = wrapi(static_cast<int>(f), n);
  }
  return c;
}

__device__ __forceinline__ float w1_of(float x) {
  const float s = x - 0.5f;
  return s - floorf(s);
}

__device__ __forceinline__ float wsel(float w1, int o) { return o ? w1 : 1.0f - w1; }

// acc[o] += val prod_d (o_d ? w1_d : 1 - w1_d), o = ox + 2 oy + 4 oz: the products are formed
// from z outwards, wx_o (wy_o (wz_o val)), so the 8 corners share their y-z factors (the
// vector deposit; the density deposit keeps its products (wx wy) wz, for which the compiler
// already shares the x-y factors: the shared form issues no fewer instructions there).
__device__ __forceinline__ void add_corners(float wx, float wy, float wz, float val,
                                            float (&acc)[8]) {
  const float z0 = (1.0f - wz) * val, z1 = wz * val;
  const float yz[4] = {(1.0f - wy) * z0, wy * z0, (1.0f - wy) * z1, wy * z1};
#pragma unroll
  for (int o = 0; o < 8; ++o) acc[o] = fmaf(wsel(wx, o & 1), yz[o >> 1], acc[o]);
}

// bin of particle i of sample s: s n^3 + CIC base cell
__device__ __forceinline__ uint32_t bin_of(const Cic& c, int n, int smp, long long nc) {
  return static_cast<uint32_t>(smp * nc + (c.i0[2] * n + c.i0[1]) * n + c.i0[0]);
}

__global__ void keys_kernel(const float* __restrict__ pos, uint32_t* __restrict__ key, int n,
                            long long np) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= np) return;
  pos += blockIdx.y * 3 * np;
  const Cic c = cic_of(pos[i], pos[np + i], pos[2 * np + i], n);
  key[blockIdx.y * np + i] = bin_of(c, n, blockIdx.y, np);
}

// Counts a particle of bin k and returns its arrival rank there.  Neighbouring particles that fall
// into one bin (in clustered states) are counted together: the first of a run of lanes adds the
// run's length (128^3 run to a = 0.29: kick and drift 54.6 -> 45.6 us a step; before clustering as
// with an atomic each).  All 64 lanes of the wave call it.
__device__ __forceinline__ uint32_t count_in_bin(uint32_t* count, uint32_t k) {
  const int lane = threadIdx.x & 63;
  const uint32_t below = __shfl_up(k, 1, 64);
  const uint64_t heads = __ballot(lane == 0 || k != below);
  const int head = 63 - __builtin_clzll(heads & (~0ULL >> (63 - lane)));
  const uint64_t after = heads >> lane >> 1;
  uint32_t base = 0;
  if (head == lane)
    base = atomicAdd(&count[k], after ? __builtin_ctzll(after) + 1u : 64u - lane);
  return __shfl(base, head, 64) + (lane - head);
}

__global__ void hist_kernel(const uint32_t* __restrict__ key, uint32_t* count,
                            uint32_t* __restrict__ rank, long long np) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= np) return;   // (np is a multiple of the block)
  rank[i] = count_in_bin(count, key[i]);
}

// Scans of the bin counts: 32-bit integer sums, so the grouping does not change a result.
constexpr int kScanWaves = kScanThreads / 64;

// inclusive scan over the 64 lanes of a wave
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t u = __shfl_up(v, off, 64);
    if (lane >= off) v += u;
  }
  return v;
}

// sum of v over the block (every thread receives it); sh[kScanWaves] is free before the call
__device__ __forceinline__ uint32_t block_add(uint32_t v, uint32_t* sh) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t t = 0;
#pragma unroll
  for (int k = 0; k < kScanWaves; ++k) t += sh[k];
  return t;
}

// sums[t] = sum of the counts of tile t
__global__ void __launch_bounds__(kScanThreads) scan_sums_kernel(const uint4* __restrict__ in,
                                                                 uint32_t* __restrict__ sums) {
  __shared__ uint32_t sh[kScanWaves];
  const uint4 v = in[blockIdx.x * kScanThreads + threadIdx.x];
  const uint32_t t = block_add(v.x + v.y + v.z + v.w, sh);
  if (threadIdx.x == 0) sums[blockIdx.x] = t;
}

// Exclusive scan of the bin counts, one block per tile: out[0..tiles kScanTile] = prefix sums
// and total.  What lies before its tile each block adds up itself: the tile sums (4 a thread at
// 256^3, from L2) or, for up to kScanDirect tiles (32^3), where another launch would cost more
// than it saves, the counts (in flight together: 4.6 us; 256 threads of 16 counts took 10.4).
// Also clears the list of large bins for the sort that follows.
constexpr int kScanDirect = 8;

__global__ void __launch_bounds__(kScanThreads) scan_kernel(const uint4* __restrict__ in,
                                                            const uint32_t* __restrict__ sums,
                                                            uint4* __restrict__ out, int tiles,
                                                            uint32_t* __restrict__ large) {
  __shared__ uint32_t sh[kScanWaves], shp[kScanWaves];
  const int t = blockIdx.x, wave = threadIdx.x >> 6;
  const int at = t * kScanThreads + threadIdx.x;
  const uint4 v = in[at];
  uint32_t part = 0;
  if (sums) {
    for (int i = threadIdx.x; i < t; i += kScanThreads) part += sums[i];
  } else {
#pragma unroll
    for (int k = 0; k < kScanDirect - 1; ++k) {
      const uint4 u = in[min(k, t) * kScanThreads + threadIdx.x];
      if (k < t) part += u.x + u.y + u.z + u.w;
    }
  }
  const uint32_t mine = v.x + v.y + v.z + v.w;
  const uint32_t inc = wave_inclusive_scan(mine);
  if ((threadIdx.x & 63) == 63) sh[wave] = inc;
  uint32_t run = block_add(part, shp) + inc - mine;   // its barrier also orders sh
#pragma unroll
  for (int k = 0; k < kScanWaves; ++k) run += k < wave ? sh[k] : 0u;
  out[at] = make_uint4(run, run + v.x, run + v.x + v.y, run + v.x + v.y + v.z);
  if (threadIdx.x == kScanThreads - 1 && t == tiles - 1)
    reinterpret_cast<uint32_t*>(out + static_cast<long long>(tiles) * kScanThreads)[0] = run + mine;
  if (threadIdx.x == 0 && t == 0) large[0] = 0u;
}

__global__ void scatter_kernel(const uint32_t* __restrict__ key, const uint32_t* __restrict__ rank,
                               const uint32_t* __restrict__ start, uint32_t* __restrict__ sorted,
                               long long np) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= np) return;
  sorted[start[key[i]] + rank[i]] = static_cast<uint32_t>(i);
}

// The atomics above fix each bin's size but not the order inside it; sorting each bin's ids
// ascending makes the layout a pure function of the keys.  A wave takes 64 consecutive bins,
// whose ids are one run of the list: it brings them to LDS, sorts every bin there (up to 8 ids
// by a lane in registers, more by all lanes, counting for each id the smaller ones), writes
// them back and gathers the positions, both coalesced over the run.  At 256^3 that is one pass
// of 100 us early on, where a pass per bin and a gather after it took 45 + 101 us; in a
// clustered state a lane alone sorted up to 32 ids through global memory (128^3 run to
// a = 0.29: 54 + 21 us a step on average).  Runs longer than kWaveIds go in several parts;
// bins of more than kWaveBin ids (dense halos gather thousands of particles in a cell) go to
// a list that bin_sort_large_kernel sorts one workgroup of 1024 threads per bin.  (In that run the
// two kernels take 44 + 15 us a step with bins of up to 256 left to the waves and 256 threads,
// 44 + 10 with 1024, 36 + 11 with bins of up to 128 and 32 + 14 with 64.)  (Moving the positions along
// with the ids in the scatter was slower: the scattered 16-byte writes cost more than the
// gather's scattered reads.)
constexpr uint32_t kWaveBin = 128;
constexpr uint32_t kWaveIds = 512;
constexpr int kLdsSort = 16384;   // ids a workgroup sorts in LDS (64 KB)

// Batcher's odd-even merge network for 8 keys (19 compare-exchanges)
__device__ __forceinline__ void sort8(uint32_t (&v)[8]) {
  constexpr int kNet[19][2] = {{0, 1}, {2, 3}, {4, 5}, {6, 7}, {0, 2}, {1, 3}, {4, 6},
                               {5, 7}, {1, 2}, {5, 6}, {0, 4}, {1, 5}, {2, 6}, {3, 7},
                               {2, 4}, {3, 5}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
  for (int k = 0; k < 19; ++k) {
    const uint32_t a = v[kNet[k][0]], b = v[kNet[k][1]];
    v[kNet[k][0]] = min(a, b);
    v[kNet[k][1]] = max(a, b);
  }
}

// upper CIC weights of particle id (global: sample id >> lnp) from per-sample [3][np] positions
__device__ __forceinline__ float3 gather_w1(const float* __restrict__ v, uint32_t id, int lnp) {
  const long long np = 1LL << lnp;
  const float* vs = v + (id >> lnp) * 3 * np;
  const long long loc = id & (np - 1);
  return make_float3(w1_of(vs[loc]), w1_of(vs[np + loc]), w1_of(vs[2 * np + loc]));
}

// orders the wave's LDS accesses (its lanes exchange ids through its own part of the LDS)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// sorts the k <= 64 R ids at s ascending, all lanes of the wave: an id's place is the number
// of smaller ones (ids are distinct)
template <int R>
__device__ __forceinline__ void wave_rank_sort(uint32_t* s, uint32_t k, int lane) {
  uint32_t v[R], rank[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint32_t i = lane + 64 * r;
    v[r] = i < k ? s[i] : 0u;
    rank[r] = 0;
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const uint32_t n = k > 64u * q ? min(k - 64u * q, 64u) : 0u;
    for (uint32_t j = 0; j < n; ++j) {
      const uint32_t u = __builtin_amdgcn_readlane(v[q], j);
#pragma unroll
      for (int r = 0; r < R; ++r) rank[r] += u < v[r] ? 1u : 0u;
    }
  }
  wave_sync();
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (lane + 64 * r < k) s[rank[r]] = v[r];
}

// (nbins is a multiple of 256.)  The counts are cleared for the next histogram.
__global__ void __launch_bounds__(256) bin_sort_gather_kernel(const uint32_t* __restrict__ start,
                                                              uint32_t* sorted,
                                                              const float* __restrict__ pos,
                                                              float3* __restrict__ sw1, int lnp,
                                                              uint32_t* __restrict__ count,
                                                              uint32_t* __restrict__ large,
                                                              bool keep_ids) {
  __shared__ uint32_t ids[4][kWaveIds];
  const int lane = threadIdx.x & 63;
  uint32_t* my = ids[threadIdx.x >> 6];
  const uint32_t b = blockIdx.x * 256u + threadIdx.x;
  const uint32_t lo = start[b], hi = start[b + 1];
  const uint32_t cnt = hi - lo;
  count[b] = 0;
  uint32_t run = __builtin_amdgcn_readfirstlane(lo);   // ids before it are done
  for (int first = 0; first < 64;) {
    // the bins from `first` on that fit into LDS together
    const uint64_t stop =
        __ballot(lane >= first && (hi - run > kWaveIds || cnt > kWaveBin)) >> first;
    const int fit = stop ? __builtin_ctzll(stop) : 64 - first;
    if (fit == 0) {
      // large[0] counts the entries large[1..]; the list order does not affect the result
      if (lane == first) large[1 + atomicAdd(&large[0], 1u)] = b;
      run = __shfl(hi, first, 64);
      ++first;
      continue;
    }
    const uint32_t end = __shfl(hi, first + fit - 1, 64);
    const uint32_t total = end - run;
    for (uint32_t i = lane; i < total; i += 64) my[i] = sorted[run + i];
    wave_sync();
    const bool mine = lane >= first && lane < first + fit;
    const uint32_t off = lo - run;
    if (mine && cnt >= 2 && cnt <= 8) {
      uint32_t v[8];
#pragma unroll
      for (uint32_t i = 0; i < 8; ++i) v[i] = i < cnt ? my[off + i] : 0xFFFFFFFFu;
      sort8(v);
#pragma unroll
      for (uint32_t i = 0; i < 8; ++i)
        if (i < cnt) my[off + i] = v[i];
    }
    for (uint64_t m = __ballot(mine && cnt > 8); m; m &= m - 1) {
      const int l = __builtin_ctzll(m);
      const uint32_t k = __shfl(cnt, l, 64);
      uint32_t* s = my + __shfl(off, l, 64);
      if (k <= 64)
        wave_rank_sort<1>(s, k, lane);
      else
        wave_rank_sort<2>(s, k, lane);
    }
    wave_sync();
    for (uint32_t i = lane; i < total; i += 64) {
      const uint32_t id = my[i];
      if (keep_ids) sorted[run + i] = id;
      sw1[run + i] = gather_w1(pos, id, lnp);
    }
    wave_sync();
    run = end;
    first += fit;
  }
}

// Ascending bitonic network over p = 2^m slots of which the first k hold data and the rest
// count as +infinity: every compare-exchange orders a lower index before a higher one (the
// first stage of each merge pairs i with its mirror), so a slot >= k is never written.
template <typename Get, typename Put>
__device__ void bitonic_ascending(uint32_t k, uint32_t p, Get get, Put put) {
  for (uint32_t size = 2; size <= p; size <<= 1) {
    for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
      for (uint32_t i = threadIdx.x; i < p; i += blockDim.x) {
        const uint32_t j = stride == (size >> 1) ? (i ^ (size - 1)) : (i ^ stride);
        if (j > i && j < k) {
          const uint32_t a = get(i), c = get(j);
          if (a > c) {
            put(i, c);
            put(j, a);
          }
        }
      }
      __syncthreads();
    }
  }
}

__global__ void __launch_bounds__(kLargeSortThreads) bin_sort_large_kernel(const uint32_t* __restrict__ start,
                                                             uint32_t* sorted,
                                                             const uint32_t* __restrict__ large,
                                                             const float* __restrict__ pos,
                                                             float3* __restrict__ sw1, int lnp) {
  __shared__ uint32_t sh[kLdsSort];
  const uint32_t count = large[0];
  for (uint32_t e = blockIdx.x; e < count; e += gridDim.x) {
    const uint32_t b = large[1 + e];
    const uint32_t lo = start[b], k = start[b + 1] - lo;
    uint32_t p = 1;
    while (p < k) p <<= 1;
    uint32_t* g = sorted + lo;
    if (k <= static_cast<uint32_t>(kLdsSort)) {
      for (uint32_t i = threadIdx.x; i < k; i += blockDim.x) sh[i] = g[i];
      __syncthreads();
      bitonic_ascending(k, p, [&](uint32_t i) { return sh[i]; },
                        [&](uint32_t i, uint32_t v) { sh[i] = v; });
      for (uint32_t i = threadIdx.x; i < k; i += blockDim.x) g[i] = sh[i];
    } else {
      bitonic_ascending(k, p, [&](uint32_t i) { return g[i]; },
                        [&](uint32_t i, uint32_t v) { g[i] = v; });
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < k; i += blockDim.x) sw1[lo + i] = gather_w1(pos, g[i], lnp);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------- deposit
// A block owns a column of TX x TY cells and walks along z.  For every plane of bins that
// reaches its cells one thread per bin of the plane (and of its low x and y halo) sums over the
// bin's particles, in ascending order, the 8 CIC corner weights (times the particle's vector
// for the vector deposit) and puts them into LDS:
//   W[o][b] = sum_{p in b} prod_d (o_d ? w1_d : 1 - w1_d),  o in {0,1}^3.
// A cell then adds W[o][c - o] over o in a fixed order; the corners with o_z = 1 wait in its
// registers for the next plane.  Each particle's weights are formed once per column that sees
// its bin (1.3 times) instead of once per cell, and the sums are reproducible bit for bit.
// What bounds it is the chain bounds -> particle -> sum of each bin, so the walk keeps the next
// planes' loads in flight; a block per tile of 32 x 4 x 4, which met that chain once per bin of
// a thread, took 183 us at 256^3 against 120 (345 MB: 2.9 TB/s), and 63 against 41 a step on
// average in a clustered 128^3 run; 32^3: 7.2 against 5.1.  Columns of 32 x 8: 130 at 256^3,
// 22 at 128^3 as here; longer walks leave the chip idle (see launch_columns).  Loading three or
// four particles ahead instead of two, or giving the bins of more to a second pass with full
// lanes: 5 to 20% slower.
// particles of a bin that its thread holds ahead of their plane
constexpr int kDepAhead = 2;

template <int TX, int TY>
struct DepCol {
  static constexpr int BX = TX + 1, BY = TY + 1;
  static constexpr int NB = BX * BY;                // bins of a plane
  static constexpr int NC = TX * TY;                // cells of a plane
  static constexpr int THREADS = (NB + 63) / 64 * 64;
};

// Bins of more than kCrowded particles (dense halos gather hundreds or thousands of
// particles in a cell) are summed by whole waves instead of one thread: the block lists them
// in LDS during pass 1 and its waves take them one each, every lane over a strided share of
// the bin's particles in ascending order, then a fixed butterfly across the wave, so the sums
// stay reproducible bit for bit and no thread loops over a crowded bin alone.
constexpr uint32_t kCrowded = 16;

template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true);
  return v + __builtin_bit_cast(float, o);
}

// Sums of v[0..8) over the 64 lanes of the wave, every lane receiving them: the butterfly
// v += v[lane ^ off], off = 32 ... 1, from 8 on in register moves (a rotation by off within 16
// lanes stands for the exchange once the wider levels have made the lanes repeat).
__device__ __forceinline__ void wave_sum(float (&v)[8]) {
#pragma unroll
  for (int off = 32; off >= 16; off >>= 1)
#pragma unroll
    for (int o = 0; o < 8; ++o) v[o] += __shfl_xor(v[o], off, 64);
#pragma unroll
  for (int o = 0; o < 8; ++o) {
    v[o] = dpp_add<0x128>(v[o]);   // row_ror:8
    v[o] = dpp_add<0x124>(v[o]);   // row_ror:4
    v[o] = dpp_add<0x4e>(v[o]);    // quad_perm [2,3,0,1]
    v[o] = dpp_add<0xb1>(v[o]);    // quad_perm [1,0,3,2]
  }
}

// acc[o] += prod_d (o_d ? w1_d : 1 - w1_d), the products formed as (wx wy) wz
__device__ __forceinline__ void add_weights(const float3& w, float (&acc)[8]) {
#pragma unroll
  for (int o = 0; o < 8; ++o)
    acc[o] = fmaf(wsel(w.x, o & 1) * wsel(w.y, (o >> 1) & 1), wsel(w.z, o >> 2), acc[o]);
}

// the sums of one particle of weights w: the CIC weights, or (VEC) these times its vector q
template <int NV>
__device__ __forceinline__ void add_particle(const float3& w, const float3& q,
                                             float (&acc)[NV][8]) {
  if constexpr (NV == 3) {
    add_corners(w.x, w.y, w.z, q.x, acc[0]);
    add_corners(w.x, w.y, w.z, q.y, acc[1]);
    add_corners(w.x, w.y, w.z, q.z, acc[2]);
  } else {
    add_weights(w, acc[0]);
  }
}

// Column walk over the cell planes [z0, z0 + planes) of the column at (x0, y0).  Loads run
// ahead of the sums: while a plane is summed, the first kDepAhead particles of the next
// planes' bins (D planes ahead) and the bounds of the one after are on their way.
// VEC: out[3][nc] += scale times the deposit of field[3][np], component by component through
// LDS; the vectors are read through the particle ids, one plane ahead (256^3: 330 us with 838 MB;
// gathering them into bin order first, as a pass per field, 102 + 321; a third of 960 threads
// for each component: 410).  Else out = field + m_dm times the deposit of the weights + offset.
template <int TX, int TY, bool VEC>
__global__ void __launch_bounds__((DepCol<TX, TY>::THREADS)) deposit_kernel(
    const uint32_t* __restrict__ start, const float3* __restrict__ sw1,
    const uint32_t* __restrict__ sorted, const float* __restrict__ field, long long stride,
    float m_dm, float offset, bool merged, float* __restrict__ out, int n, int planes,
    const StepScal* __restrict__ tab) {
  using T = DepCol<TX, TY>;
  constexpr int NV = VEC ? 3 : 1, A = kDepAhead;
  constexpr int D = VEC ? 1 : 2;         // planes between a particle's load and its use
  __shared__ float W[2][8 * T::NB];
  __shared__ int ncrowd[3];
  __shared__ uint16_t crowd[T::NB];
  __shared__ uint2 range[T::NB];
  if (!sample_active(tab, blockIdx.y)) return;
  const int tx = n / TX, ty = n / TY;
  const int t = blockIdx.x;
  const int x0 = t % tx * TX;
  const int y0 = t / tx % ty * TY;
  const int z0 = t / (tx * ty) * planes;
  const unsigned nn = n * n, nc = nn * n;
  const int b = threadIdx.x, lane = threadIdx.x & 63;
  start += static_cast<long long>(blockIdx.y) * nc;
  out += static_cast<long long>(blockIdx.y) * NV * nc;
  if (field) field += blockIdx.y * stride;
  float scale = m_dm;
  if (VEC) scale = merged ? tab[blockIdx.y].h_dm : tab[blockIdx.y].h_open;
  const int col = wrapi(y0 - 1 + b / T::BX, n) * n + wrapi(x0 - 1 + b % T::BX, n);
  // bounds of this thread's bin of plane k (cells z0 - 1 + k)
  const auto bounds = [&](int k) {
    if (b >= T::NB || k > planes) return make_uint2(0u, 0u);
    const uint32_t* s = start + (wrapi(z0 - 1 + k, n) * nn + col);
    return make_uint2(s[0], s[1]);
  };
  // particle i of a bin, or any where it has fewer
  const auto at = [](const uint2& r, int i) { return r.x + i < r.y ? r.x + i : 0u; };
  // the vector of the particle with global id g (the sample in the bits above nc)
  const auto vector_of = [&](uint32_t g) {
    const unsigned i = g & (nc - 1);
    return make_float3(field[i], field[nc + i], field[2 * nc + i]);
  };
  constexpr int R = D + 1 + VEC;   // planes whose bounds are known
  uint2 r[R];
#pragma unroll
  for (int d = 0; d < R; ++d) r[d] = bounds(d);
  float3 p[D][A], q[A];
  uint32_t id[A];
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int i = 0; i < A; ++i) p[d][i] = sw1[at(r[d], i)];
  if (VEC) {
#pragma unroll
    for (int i = 0; i < A; ++i) id[i] = sorted[at(r[0], i)];
#pragma unroll
    for (int i = 0; i < A; ++i) {
      q[i] = vector_of(id[i]);
      id[i] = sorted[at(r[1], i)];
    }
  }
  const int cx = b % TX, cy = b / TX;   // this thread's cell (b < NC)
  const int wat = (cy + 1) * T::BX + cx + 1;
  float ahead[NV][4];   // corners with o_z = 1, for the cell of the next plane
  if (threadIdx.x < 3) ncrowd[threadIdx.x] = 0;
  __syncthreads();
  for (int k = 0, step = 0; k <= planes; ++k) {
    float acc[NV][8];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int o = 0; o < 8; ++o) acc[v][o] = 0.0f;
    float3 p0[A], q0[A];
#pragma unroll
    for (int i = 0; i < A; ++i) {
      p0[i] = p[0][i];
      if (D == 2) p[0][i] = p[1][i];
      if (VEC) q0[i] = q[i];
    }
    const uint2 r0 = r[0];
#pragma unroll
    for (int d = 0; d + 1 < R; ++d) r[d] = r[d + 1];
    float before[NV];   // what the cell's sum is added to
    const unsigned c = (z0 - 1 + k) * nn + (y0 + cy) * n + (x0 + cx);
    if (k > 0 && b < T::NC) {
#pragma unroll
      for (int v = 0; v < NV; ++v)
        before[v] = VEC ? out[static_cast<long long>(v) * nc + c] : (field ? field[c] : 0.0f);
    }
    if (k + D <= planes) {
#pragma unroll
      for (int i = 0; i < A; ++i) {
        p[D - 1][i] = sw1[at(r[D - 1], i)];
        if (VEC) q[i] = vector_of(id[i]);
      }
      if (VEC) {
#pragma unroll
        for (int i = 0; i < A; ++i) id[i] = sorted[at(r[R - 2], i)];
      }
      r[R - 1] = bounds(k + R);
    }
    const bool crowded = r0.y - r0.x > kCrowded;
    if (crowded) {
      // the list order only decides which wave sums the bin
      const int e = atomicAdd(&ncrowd[k % 3], 1);
      crowd[e] = static_cast<uint16_t>(b);
      range[e] = r0;
    } else if (b < T::NB) {
#pragma unroll
      for (int i = 0; i < A; ++i)
        if (r0.x + i < r0.y) add_particle<NV>(p0[i], q0[i], acc);
      for (uint32_t j = r0.x + A; j < r0.y; j += A) {
#pragma unroll
        for (int i = 0; i < A; ++i) {
          const uint32_t ji = min(j + i, r0.y - 1);
          p0[i] = sw1[ji];
          if (VEC) q0[i] = vector_of(sorted[ji]);
        }
#pragma unroll
        for (int i = 0; i < A; ++i)
          if (j + i < r0.y) add_particle<NV>(p0[i], q0[i], acc);
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v, ++step) {
      float* w = W[step & 1];
      if (b < T::NB && !crowded) {
#pragma unroll
        for (int o = 0; o < 8; ++o) w[o * T::NB + b] = acc[v][o];
      }
      __syncthreads();
      const int count = ncrowd[k % 3];
      if (count > 0) {
        for (int e = b >> 6; e < count; e += T::THREADS / 64) {
          const int bin = crowd[e];
          const uint2 rc = range[e];
          float s[1][8];
#pragma unroll
          for (int o = 0; o < 8; ++o) s[0][o] = 0.0f;
          for (uint32_t j = rc.x + lane; j < rc.y; j += 64) {
            const float3 pj = sw1[j];
            if constexpr (VEC)
              add_corners(pj.x, pj.y, pj.z,
                          field[static_cast<long long>(v) * nc + (sorted[j] & (nc - 1))], s[0]);
            else
              add_weights(pj, s[0]);
          }
          wave_sum(s[0]);
          if (lane == 0) {
#pragma unroll
            for (int o = 0; o < 8; ++o) w[o * T::NB + bin] = s[0][o];
          }
        }
        __syncthreads();
      }
      if (v == NV - 1 && threadIdx.x == 0) ncrowd[(k + 2) % 3] = 0;
      if (b < T::NC) {
        if (k > 0) {
          float sum = 0.0f;
#pragma unroll
          for (int o = 0; o < 4; ++o) sum += w[o * T::NB + wat - (o >> 1) * T::BX - (o & 1)];
#pragma unroll
          for (int o = 0; o < 4; ++o) sum += ahead[v][o];
          if (VEC)
            out[static_cast<long long>(v) * nc + c] = fmaf(scale, sum, before[v]);
          else
            out[c] = before[v] + scale * sum + offset;
        }
#pragma unroll
        for (int o = 0; o < 4; ++o)
          ahead[v][o] = w[(4 + o) * T::NB + wat - (o >> 1) * T::BX - (o & 1)];
      }
    }
  }
}

// Cell c of one sample (at most 256^3, so 32-bit) from its x, y, z: n is a power of two.
struct GridIdx {
  unsigned n1, lg;   // n - 1, log2 n
  __device__ __forceinline__ unsigned at(unsigned x, unsigned y, unsigned z) const {
    return (((z & n1) << lg | (y & n1)) << lg) | (x & n1);
  }
};

// g[c] = -grad(phi) at c, for the read-outs on the particles (the cells' kernels form it from
// phi).  12 bytes a cell: with 16 this pass took 74 us at 256^3 against 65, kick and drift 275
// against 268.  A particle's own read-out from phi takes 32 loads, as rows or one by one, and
// 360 to 420 us.
__global__ void __launch_bounds__(256) grad_kernel(const float* __restrict__ phi,
                                                   float3* __restrict__ g, int lgn,
                                                   const StepScal* __restrict__ tab) {
  const unsigned c = blockIdx.x * blockDim.x + threadIdx.x;
  const unsigned nc = 1u << (3 * lgn);
  if (c >= nc || !sample_active(tab, blockIdx.y)) return;
  phi += static_cast<long long>(blockIdx.y) * nc;
  g += static_cast<long long>(blockIdx.y) * nc;
  const float4 v = mesh_g(phi, c, lgn);
  g[c] = make_float3(v.x, v.y, v.z);
}

__device__ __forceinline__ long long corner(const Cic& w, int ox, int oy, int oz, int n) {
  return (static_cast<long long>(wrapi(w.i0[2] + oz, n)) * n + wrapi(w.i0[1] + oy, n)) * n +
         wrapi(w.i0[0] + ox, n);
}

// CIC read-out of g at a particle
__device__ __forceinline__ void readout_g(const float3* __restrict__ g3, const Cic& w, int n,
                                          float out[3]) {
  out[0] = out[1] = out[2] = 0.0f;
#pragma unroll
  for (int oz = 0; oz < 2; ++oz)
#pragma unroll
    for (int oy = 0; oy < 2; ++oy)
#pragma unroll
      for (int ox = 0; ox < 2; ++ox) {
        const float3 g = g3[corner(w, ox, oy, oz, n)];
        const float ww = wsel(w.w1[0], ox) * wsel(w.w1[1], oy) * wsel(w.w1[2], oz);
        out[0] = fmaf(ww, g.x, out[0]);
        out[1] = fmaf(ww, g.y, out[1]);
        out[2] = fmaf(ww, g.z, out[2]);
      }
}

__global__ void __launch_bounds__(256) readout_g_kernel(const float3* __restrict__ g3,
                                                        const float* __restrict__ pos,
                                                        float* __restrict__ out, int n,
                                                        long long np) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= np) return;
  g3 += blockIdx.y * np;
  pos += blockIdx.y * 3 * np;
  out += blockIdx.y * 3 * np;
  const Cic w = cic_of(pos[i], pos[np + i], pos[2 * np + i], n);
  float g[3];
  readout_g(g3, w, n, g);
  out[i] = g[0];
  out[np + i] = g[1];
  out[2 * np + i] = g[2];
}

// Stars formed in a step, associated with the dark matter (Sec. 2.4.1): each particle's
// auxiliary field gains the CIC read-out of the step's new stars znew at its position.
// Samples that sit the step out are skipped.
__global__ void __launch_bounds__(256) star_readout_kernel(const float* __restrict__ znew,
                                                           const float* __restrict__ pos,
                                                           float* __restrict__ aux, int n,
                                                           long long np,
                                                           const StepScal* __restrict__ tab) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= np || !sample_active(tab, blockIdx.y)) return;
  znew += blockIdx.y * np;   // n^3 cells = n^3 particles per sample
  pos += blockIdx.y * 3 * np;
  aux += blockIdx.y * np;
  const Cic w = cic_of(pos[i], pos[np + i], pos[2 * np + i], n);
  float v = 0.0f;
#pragma unroll
  for (int oz = 0; oz < 2; ++oz)
#pragma unroll
    for (int oy = 0; oy < 2; ++oy)
#pragma unroll
      for (int ox = 0; ox < 2; ++ox)
        v = fmaf(wsel(w.w1[0], ox) * wsel(w.w1[1], oy) * wsel(w.w1[2], oz),
                 znew[corner(w, ox, oy, oz, n)], v);
  aux[i] += v;
}

__device__ __forceinline__ float wrap_pos(float x, float fn) {
  x -= fn * floorf(x / fn);
  if (x >= fn) x -= fn;
  return x;
}

// Opening half kick and drift of the dark matter, with the keys of the new positions.  With
// `prev`, the closing half kick of the sample's previous step (factor h_prev, same field and
// positions) is applied first: the two kicks are the separate roundings of kick_kernel
// followed by this kernel, fused into one pass over the particles.
// pos_in and pos may be the same array (in place): no __restrict__ on them
__global__ void __launch_bounds__(256) kick_drift_kernel(const float3* __restrict__ g3,
                                                         const float* pos_in, float* pos,
                                                         float* __restrict__ mom,
                                                         uint32_t* __restrict__ key,
                                                         float* __restrict__ mom_copy,
                                                         float* __restrict__ pos_copy, int n,
                                                         long long np, int prev,
                                                         const StepScal* __restrict__ tab,
                                                         uint32_t* count,
                                                         uint32_t* __restrict__ rank) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  const StepScal& sc = tab[blockIdx.y];
  if (i >= np) return;
  const int smp = blockIdx.y;
  g3 += smp * np;
  pos_in += smp * 3 * np;
  pos += smp * 3 * np;
  mom += smp * 3 * np;
  key += smp * np;
  if (mom_copy) mom_copy += smp * 3 * np;
  if (pos_copy) pos_copy += smp * 3 * np;
  if (count) rank += smp * np;
  if (!sc.active) {
    // the sort's histogram counts the sample's particles under the keys they have
    if (count) rank[i] = count_in_bin(count, key[i]);
    // a sample that sits the step out keeps its particles; the copies (the tape of the
    // reverse pass, which sorts them again) receive them unchanged
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const float xd = pos_in[d * np + i];
      if (pos != pos_in) pos[d * np + i] = xd;
      if (mom_copy) mom_copy[d * np + i] = mom[d * np + i];
      if (pos_copy) pos_copy[d * np + i] = xd;
    }
    return;
  }
  const float h = sc.h_open, drift_fac = sc.drift, hp = prev ? sc.h_prev : 0.0f;
  float x[3] = {pos_in[i], pos_in[np + i], pos_in[2 * np + i]};
  const Cic w = cic_of(x[0], x[1], x[2], n);
  float g[3];
  readout_g(g3, w, n, g);
  const float fn = static_cast<float>(n);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    float p = mom[d * np + i];
    if (prev) p = fmaf(hp, g[d], p);
    p = fmaf(h, g[d], p);
    mom[d * np + i] = p;
    x[d] = wrap_pos(x[d] + p * drift_fac, fn);
    pos[d * np + i] = x[d];
    if (mom_copy) mom_copy[d * np + i] = p;
    if (pos_copy) pos_copy[d * np + i] = x[d];
  }
  const Cic w2 = cic_of(x[0], x[1], x[2], n);
  const uint32_t k = bin_of(w2, n, smp, np);
  key[i] = k;
  // the sort's histogram (count zeroed beforehand): the arrival rank of the particle in its bin
  if (count) rank[i] = count_in_bin(count, k);
}

__global__ void __launch_bounds__(256) kick_kernel(const float3* __restrict__ g3,
                                                   const float* __restrict__ pos,
                                                   float* __restrict__ mom, int n, long long np,
                                                   const StepScal* __restrict__ tab) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  const StepScal& sc = tab[blockIdx.y];
  if (i >= np || !sc.active) return;
  const float h = sc.h_close;
  g3 += blockIdx.y * np;
  pos += blockIdx.y * 3 * np;
  mom += blockIdx.y * 3 * np;
  const Cic w = cic_of(pos[i], pos[np + i], pos[2 * np + i], n);
  float g[3];
  readout_g(g3, w, n, g);
#pragma unroll
  for (int d = 0; d < 3; ++d) mom[d * np + i] = fmaf(h, g[d], mom[d * np + i]);
}

// acc = sum_corners (dw/dx) (g_corner . lp): the kick's adjoint with respect to the position
__device__ __forceinline__ void kick_pos_acc(const float3* __restrict__ g3, const Cic& w,
                                             const float lp[3], int n, float acc[3]) {
  acc[0] = acc[1] = acc[2] = 0.0f;
#pragma unroll
  for (int oz = 0; oz < 2; ++oz)
#pragma unroll
    for (int oy = 0; oy < 2; ++oy)
#pragma unroll
      for (int ox = 0; ox < 2; ++ox) {
        const float3 g = g3[corner(w, ox, oy, oz, n)];
        const float gl = g.x * lp[0] + g.y * lp[1] + g.z * lp[2];
        const float wx = wsel(w.w1[0], ox), wy = wsel(w.w1[1], oy), wz = wsel(w.w1[2], oz);
        acc[0] += (ox ? 1.0f : -1.0f) * wy * wz * gl;
        acc[1] += wx * (oy ? 1.0f : -1.0f) * wz * gl;
        acc[2] += wx * wy * (oz ? 1.0f : -1.0f) * gl;
      }
}

// lam_x += h * sum_corners (dw/dx) (g_corner . lam_p)
__global__ void __launch_bounds__(256) kick_vjp_pos_kernel(const float3* __restrict__ g3,
                                                           const float* __restrict__ pos,
                                                           const float* __restrict__ lam_p,
                                                           bool merged, float* __restrict__ lam_x,
                                                           int n, long long np,
                                                           const StepScal* __restrict__ tab) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  const StepScal& sc = tab[blockIdx.y];
  if (i >= np || !sc.active) return;
  const float h = merged ? sc.h_dm : sc.h_open;
  g3 += blockIdx.y * np;
  pos += blockIdx.y * 3 * np;
  lam_p += blockIdx.y * 3 * np;
  lam_x += blockIdx.y * 3 * np;
  const Cic w = cic_of(pos[i], pos[np + i], pos[2 * np + i], n);
  const float lp[3] = {lam_p[i], lam_p[np + i], lam_p[2 * np + i]};
  float acc[3];
  kick_pos_acc(g3, w, lp, n, acc);
#pragma unroll
  for (int d = 0; d < 3; ++d) lam_x[d * np + i] = fmaf(h, acc[d], lam_x[d * np + i]);
}

// lam_x += mass * sum_corners lam_delta[corner] dw/dx
// With lam_p: first, with g3, the merged dark-matter kicks' adjoint with respect to the
// position (kick_vjp_pos_kernel, factor h_dm); last, lam_p += drift lam_x (the drift's
// adjoint, x1 = x0 + drift p).  With lam_rho (sample s at lam_rho + s rho_stride): lam_rho +=
// lam_delta on the cells, as many as particles, while the pass reads lam_delta anyway (a pass of
// its own took 40 us at 256^3).  One pass, the roundings of the separate kernels.
__global__ void __launch_bounds__(256) deposit_vjp_pos_kernel(const float* __restrict__ lam_delta,
                                                              const float* __restrict__ pos,
                                                              float mass, float* __restrict__ lam_x,
                                                              float* __restrict__ lam_p,
                                                              const float3* __restrict__ g3,
                                                              float* __restrict__ lam_rho,
                                                              long long rho_stride, int n,
                                                              long long np,
                                                              const StepScal* __restrict__ tab) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= np || !sample_active(tab, blockIdx.y)) return;
  lam_delta += blockIdx.y * np;
  pos += blockIdx.y * 3 * np;
  lam_x += blockIdx.y * 3 * np;
  if (lam_rho) lam_rho[blockIdx.y * rho_stride + i] += lam_delta[i];
  if (lam_p) lam_p += blockIdx.y * 3 * np;
  if (g3) g3 += blockIdx.y * np;
  const Cic w = cic_of(pos[i], pos[np + i], pos[2 * np + i], n);
  float lx0[3] = {lam_x[i], lam_x[np + i], lam_x[2 * np + i]};
  float lp[3] = {0.0f, 0.0f, 0.0f};
  if (lam_p) {
#pragma unroll
    for (int d = 0; d < 3; ++d) lp[d] = lam_p[d * np + i];
  }
  if (g3) {
    float ka[3];
    kick_pos_acc(g3, w, lp, n, ka);
    const float h = tab[blockIdx.y].h_dm;
#pragma unroll
    for (int d = 0; d < 3; ++d) lx0[d] = fmaf(h, ka[d], lx0[d]);
  }
  float acc[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int oz = 0; oz < 2; ++oz)
#pragma unroll
    for (int oy = 0; oy < 2; ++oy)
#pragma unroll
      for (int ox = 0; ox < 2; ++ox) {
        const float l = lam_delta[corner(w, ox, oy, oz, n)];
        const float wx = wsel(w.w1[0], ox), wy = wsel(w.w1[1], oy), wz = wsel(w.w1[2], oz);
        acc[0] += (ox ? 1.0f : -1.0f) * wy * wz * l;
        acc[1] += wx * (oy ? 1.0f : -1.0f) * wz * l;
        acc[2] += wx * wy * (oz ? 1.0f : -1.0f) * l;
      }
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float lx = fmaf(mass, acc[d], lx0[d]);
    lam_x[d * np + i] = lx;
    if (lam_p) lam_p[d * np + i] = fmaf(tab[blockIdx.y].drift, lx, lp[d]);
  }
}

__global__ void axpy_kernel(float* __restrict__ y, const float* __restrict__ x, float a,
                            long long count, long long ys, long long xs, bool by_drift,
                            const StepScal* __restrict__ tab) {
  const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i >= count || !sample_active(tab, blockIdx.y)) return;
  const float f = by_drift ? a * tab[blockIdx.y].drift : a;
  y[blockIdx.y * ys + i] = fmaf(f, x[blockIdx.y * xs + i], y[blockIdx.y * ys + i]);
}

// lam_phi[c] = lam_phi_in[c] + sum_d (lam_g_d[c + e_d] - lam_g_d[c - e_d]) / 2.
// FIRST: the terms of a first field lam_g0 come before those of lam_g, starting from 0 (the
// value the launch for lam_g0 alone would have passed in as lam_phi_in, rounded alike).
template <bool FIRST>
__global__ void __launch_bounds__(256) grad_vjp_kernel(const float* __restrict__ lam_g,
                                                       const float* __restrict__ lam_phi_in,
                                                       float* __restrict__ lam_phi, int n, int lgn,
                                                       const StepScal* __restrict__ tab,
                                                       const float* __restrict__ lam_g0) {
  const unsigned c = blockIdx.x * blockDim.x + threadIdx.x;
  const unsigned nc = 1u << (3 * lgn);
  if (c >= nc || !sample_active(tab, blockIdx.y)) return;
  lam_g += static_cast<long long>(blockIdx.y) * 3 * nc;
  if (lam_phi_in) lam_phi_in += static_cast<long long>(blockIdx.y) * nc;
  lam_phi += static_cast<long long>(blockIdx.y) * nc;
  const GridIdx gi{static_cast<unsigned>(n - 1), static_cast<unsigned>(lgn)};
  const unsigned ix = c & gi.n1, iy = (c >> lgn) & gi.n1, iz = c >> (2 * lgn);
  const float* lx = lam_g;
  const float* ly = lam_g + nc;
  const float* lz = lam_g + 2 * static_cast<long long>(nc);
  float v = lam_phi_in ? lam_phi_in[c] : 0.0f;
  if (FIRST) {
    lam_g0 += static_cast<long long>(blockIdx.y) * 3 * nc;
    const float* mx = lam_g0;
    const float* my = lam_g0 + nc;
    const float* mz = lam_g0 + 2 * static_cast<long long>(nc);
    v += 0.5f * (mx[gi.at(ix + 1, iy, iz)] - mx[gi.at(ix - 1, iy, iz)]);
    v += 0.5f * (my[gi.at(ix, iy + 1, iz)] - my[gi.at(ix, iy - 1, iz)]);
    v += 0.5f * (mz[gi.at(ix, iy, iz + 1)] - mz[gi.at(ix, iy, iz - 1)]);
  }
  v += 0.5f * (lx[gi.at(ix + 1, iy, iz)] - lx[gi.at(ix - 1, iy, iz)]);
  v += 0.5f * (ly[gi.at(ix, iy + 1, iz)] - ly[gi.at(ix, iy - 1, iz)]);
  v += 0.5f * (lz[gi.at(ix, iy, iz + 1)] - lz[gi.at(ix, iy, iz - 1)]);
  lam_phi[c] = v;
}

}  // namespace

long long large_bin_capacity(long long total) { return total / (kWaveBin + 1) + 1; }

size_t scan_block_count(long long nbins) {
  return static_cast<size_t>((nbins + kScanTile - 1) / kScanTile);
}

namespace {
int log2_ll(long long v) {
  int l = 0;
  while ((1LL << l) < v) ++l;
  return l;
}
dim3 per_sample(long long work, const Batch& b) { return dim3(blocks_for(work, 256), b.S); }
}  // namespace

void launch_keys(hipStream_t st, const float* pos, uint32_t* key, const Batch& b) {
  const long long np = b.nc();
  hipLaunchKernelGGL(keys_kernel, per_sample(np, b), dim3(256), 0, st, pos, key, b.n, np);
  DH_LAUNCH_CHECK();
}

void clear_counts(hipStream_t st, Bins& bins) {
  if (!bins.counting) return;
  launch_fill(st, reinterpret_cast<float*>(bins.count), 0.0f, bins.size);
  bins.counting = false;
}

void launch_sort(hipStream_t st, Bins& bins, const float* pos, const Batch& b, bool counted,
                 bool keep_ids) {
  const long long nbins = b.nc() * b.S, total = nbins;
  const int lnp = log2_ll(b.nc());
  if (!counted) {
    clear_counts(st, bins);
    bins.counting = true;
    hipLaunchKernelGGL(hist_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, st, bins.key,
                       bins.count, bins.rank, total);
    DH_LAUNCH_CHECK();
  }
  // (n is a power of two, 16 or more: whole tiles)
  const int tiles = static_cast<int>(scan_block_count(nbins));
  const bool direct = tiles <= kScanDirect;
  if (!direct) {
    hipLaunchKernelGGL(scan_sums_kernel, dim3(tiles), dim3(kScanThreads), 0, st,
                       reinterpret_cast<const uint4*>(bins.count), bins.block_sums);
    DH_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL(scan_kernel, dim3(tiles), dim3(kScanThreads), 0, st,
                     reinterpret_cast<const uint4*>(bins.count),
                     direct ? nullptr : bins.block_sums, reinterpret_cast<uint4*>(bins.start),
                     tiles, bins.large);
  DH_LAUNCH_CHECK();
  hipLaunchKernelGGL(scatter_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, st, bins.key,
                     bins.rank, bins.start, bins.sorted, total);
  DH_LAUNCH_CHECK();
  hipLaunchKernelGGL(bin_sort_gather_kernel, dim3(static_cast<unsigned>(nbins / 256)), dim3(256), 0,
                     st, bins.start, bins.sorted, pos, bins.sw1, lnp, bins.count, bins.large,
                     keep_ids);
  DH_LAUNCH_CHECK();
  bins.counting = false;
  hipLaunchKernelGGL(bin_sort_large_kernel, dim3(kLargeSortBlocks), dim3(kLargeSortThreads), 0, st, bins.start,
                     bins.sorted, bins.large, pos, bins.sw1, lnp);
  DH_LAUNCH_CHECK();
}

namespace {

template <int TX, int TY, bool VEC>
void launch_columns(hipStream_t st, const Bins& bins, const float* field, long long stride,
                    float m_dm, float offset, bool merged, float* out, const Batch& b) {
  using T = DepCol<TX, TY>;
  // longer walks read fewer halo planes, shorter ones fill the chip: 256^3 takes 129 / 120 / 123
  // us with 4 / 8 / 16 planes (16384 blocks with 8), 128^3 21.8 / 22.0 / 23.0 with 2 / 4 / 8
  // (4096 with 4; a clustered state 38 / 41 / 53, its vector deposit 59 / 54 / 59), 32^3 5.1 / 6.2 /
  // 8.3 with 1 / 2 / 4 (256 with 1)
  int planes = 8;
  while (planes > 1 && b.nc() * b.S / (T::NC * planes) < 4096) planes >>= 1;
  hipLaunchKernelGGL((deposit_kernel<TX, TY, VEC>),
                     dim3(static_cast<unsigned>(b.nc() / (T::NC * planes)), b.S),
                     dim3(T::THREADS), 0, st, bins.start, bins.sw1, bins.sorted,
                     field, stride, m_dm, offset, merged, out, b.n, planes, b.tab);
  DH_LAUNCH_CHECK();
}

// columns of 32 x 4 cells (16 x 8 at n = 16)
template <bool VEC>
void launch_columns(hipStream_t st, const Bins& bins, const float* field, long long stride,
                    float m_dm, float offset, bool merged, float* out, const Batch& b) {
  if (b.n >= 32)
    launch_columns<32, 4, VEC>(st, bins, field, stride, m_dm, offset, merged, out, b);
  else
    launch_columns<16, 8, VEC>(st, bins, field, stride, m_dm, offset, merged, out, b);
}

}  // namespace

void launch_deposit(hipStream_t st, const Bins& bins, const float* rho_gas,
                    long long rho_stride, float m_dm, float offset, float* out, const Batch& b) {
  launch_columns<false>(st, bins, rho_gas, rho_stride, m_dm, offset, false, out, b);
}

void launch_deposit_vec(hipStream_t st, const Bins& bins, const float* v, bool merged,
                        float* out_accum, const Batch& b) {
  if (!b.tab) throw ArgError("deposit_vec: step table required");
  launch_columns<true>(st, bins, v, 3 * b.nc(), 0.0f, 0.0f, merged, out_accum, b);
}

void launch_grad(hipStream_t st, const float* phi, float3* g3, const Batch& b) {
  hipLaunchKernelGGL(grad_kernel, per_sample(b.nc(), b), dim3(256), 0, st, phi, g3,
                     log2_ll(b.n), b.tab);
  DH_LAUNCH_CHECK();
}

void launch_readout_g(hipStream_t st, const float3* g3, const float* pos, float* out,
                      const Batch& b) {
  hipLaunchKernelGGL(readout_g_kernel, per_sample(b.nc(), b), dim3(256), 0, st, g3, pos, out, b.n,
                     b.nc());
  DH_LAUNCH_CHECK();
}

void launch_star_readout(hipStream_t st, const float* znew, const float* pos, float* aux,
                         const Batch& b) {
  hipLaunchKernelGGL(star_readout_kernel, per_sample(b.nc(), b), dim3(256), 0, st, znew, pos, aux,
                     b.n, b.nc(), b.tab);
  DH_LAUNCH_CHECK();
}

void launch_kick_drift(hipStream_t st, const float3* g3, const float* pos_in, float* pos,
                       float* mom, uint32_t* key, float* mom_copy, float* pos_copy, bool prev,
                       const Batch& b, Bins* count_into) {
  if (!b.tab) throw ArgError("kick_drift: step table required");
  if (count_into && key != count_into->key) throw ArgError("kick_drift: keys of another sort");
  uint32_t* count = count_into ? count_into->count : nullptr;
  uint32_t* rank = count_into ? count_into->rank : nullptr;
  if (count_into) {
    clear_counts(st, *count_into);
    count_into->counting = true;
  }
  hipLaunchKernelGGL(kick_drift_kernel, per_sample(b.nc(), b), dim3(256), 0, st, g3, pos_in, pos,
                     mom, key, mom_copy, pos_copy, b.n, b.nc(), prev ? 1 : 0, b.tab, count, rank);
  DH_LAUNCH_CHECK();
}

void launch_kick(hipStream_t st, const float3* g3, const float* pos, float* mom, const Batch& b) {
  if (!b.tab) throw ArgError("kick: step table required");
  hipLaunchKernelGGL(kick_kernel, per_sample(b.nc(), b), dim3(256), 0, st, g3, pos, mom, b.n,
                     b.nc(), b.tab);
  DH_LAUNCH_CHECK();
}

void launch_kick_vjp_pos(hipStream_t st, const float3* g3, const float* pos, const float* lam_p,
                         bool merged, float* lam_x, const Batch& b) {
  if (!b.tab) throw ArgError("kick adjoint: step table required");
  hipLaunchKernelGGL(kick_vjp_pos_kernel, per_sample(b.nc(), b), dim3(256), 0, st, g3, pos, lam_p,
                     merged, lam_x, b.n, b.nc(), b.tab);
  DH_LAUNCH_CHECK();
}

void launch_deposit_vjp_pos(hipStream_t st, const float* lam_delta, const float* pos, float mass,
                            float* lam_x, float* lam_p, const float3* g3, float* lam_rho,
                            long long rho_stride, const Batch& b) {
  if (lam_p && !b.tab) throw ArgError("deposit adjoint: step table required for the drift");
  if (g3 && !lam_p) throw ArgError("deposit adjoint: the kick term needs lam_p");
  hipLaunchKernelGGL(deposit_vjp_pos_kernel, per_sample(b.nc(), b), dim3(256), 0, st, lam_delta,
                     pos, mass, lam_x, lam_p, g3, lam_rho, rho_stride, b.n, b.nc(), b.tab);
  DH_LAUNCH_CHECK();
}

void launch_axpy(hipStream_t st, float* y, const float* x, float a, long long count, long long ys,
                 long long xs, bool by_drift, const Batch& b) {
  if (by_drift && !b.tab) throw ArgError("axpy: step table required");
  hipLaunchKernelGGL(axpy_kernel, per_sample(count, b), dim3(256), 0, st, y, x, a, count, ys, xs,
                     by_drift, b.tab);
  DH_LAUNCH_CHECK();
}

void launch_grad_vjp(hipStream_t st, const float* lam_g, const float* lam_phi_in, float* lam_phi,
                     const Batch& b) {
  hipLaunchKernelGGL(grad_vjp_kernel<false>, per_sample(b.nc(), b), dim3(256), 0, st, lam_g,
                     lam_phi_in, lam_phi, b.n, log2_ll(b.n), b.tab, nullptr);
  DH_LAUNCH_CHECK();
}

void launch_grad_vjp2(hipStream_t st, const float* lam_g0, const float* lam_g, float* lam_phi,
                      const Batch& b) {
  hipLaunchKernelGGL(grad_vjp_kernel<true>, per_sample(b.nc(), b), dim3(256), 0, st, lam_g,
                     nullptr, lam_phi, b.n, log2_ll(b.n), b.tab, lam_g0);
  DH_LAUNCH_CHECK();
}

}  // namespace dh
