// scan.hip -- exclusive prefix sum of per-segment hit counts (int32 counts -> int64 offsets), the compaction
// step that gives every punctured simplex its position in the face-id-sorted output.
#include "common.h"
#include "internal.h"

namespace ftk {

namespace {
constexpr int kThreads = 256;
constexpr int kItems = 8;
constexpr int kTile = kThreads * kItems;
// Up to this many counts one block scans in rounds of kOneThreads * kItems: three small launches and their gaps cost
// about 8 us, a round about 2 us and one launch.
constexpr int kOneThreads = 1024;
constexpr long long kOneBlock = 2 * kOneThreads * kItems;

template <int THREADS>
__device__ __forceinline__ long long block_excl_scan(long long v, long long* total) {
  __shared__ long long wsum[THREADS / kWave];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  long long x = v;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    long long o = __shfl_up(x, d, kWave);
    if (lane >= d) x += o;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  long long before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < THREADS / kWave; ++i) {
    if (i < w) before += wsum[i];
    all += wsum[i];
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

__global__ __launch_bounds__(kOneThreads) void scan_one(const int* __restrict__ in, long long* __restrict__ out,
                                                        long long n, long long base, long long* __restrict__ total) {
  for (long long b0 = 0; b0 < n; b0 += kOneThreads * kItems) {
    const long long first = b0 + threadIdx.x * kItems;
    int v[kItems];
    long long s = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      v[i] = first + i < n ? in[first + i] : 0;
      s += v[i];
    }
    long long all;
    long long run = base + block_excl_scan<kOneThreads>(s, &all);
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      if (first + i < n) out[first + i] = run;
      run += v[i];
    }
    base += all;
  }
  if (threadIdx.x == 0) *total = base;
}

// The kItems consecutive counts of a thread (0 past the end): two 16-byte loads inside the array when it is aligned for
// them (a plane of a ring need not be).  Bound by memory; 13M counts (4096^2 x 50): reduce 34 -> 12 us, down 102 -> 46 (3.4
// TB/s), and the block sums 21 -> 12 with 1024 threads.
__device__ __forceinline__ void load_items(const int* __restrict__ in, long long first, long long n, int (&v)[kItems]) {
  static_assert(kItems == 8, "two vectors of four");
  if (first + kItems <= n && ((uintptr_t)in & 15u) == 0) {
    const int4 a = *(const int4*)(in + first), b = *(const int4*)(in + first + 4);
    v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
  } else {
#pragma unroll
    for (int i = 0; i < kItems; ++i) v[i] = first + i < n ? in[first + i] : 0;
  }
}

__global__ __launch_bounds__(kThreads) void scan_reduce(const int* __restrict__ in, long long n,
                                                        long long* __restrict__ tmp) {
  const long long base = (long long)blockIdx.x * kTile + threadIdx.x * kItems;
  int v[kItems];
  load_items(in, base, n, v);
  long long s = 0;
#pragma unroll
  for (int i = 0; i < kItems; ++i) s += v[i];
  long long tot;
  block_excl_scan<kThreads>(s, &tot);
  if (threadIdx.x == 0) tmp[blockIdx.x] = tot;
}

// single block: tmp[0..nb) block sums -> exclusive offsets, total
__global__ __launch_bounds__(kOneThreads) void scan_blocks(long long* __restrict__ tmp, long long nb, long long carry,
                                                           long long* __restrict__ total) {
  for (long long b0 = 0; b0 < nb; b0 += kOneThreads) {
    long long i = b0 + threadIdx.x;
    long long v = i < nb ? tmp[i] : 0;
    long long tot;
    long long ex = block_excl_scan<kOneThreads>(v, &tot);
    if (i < nb) tmp[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) *total = carry;
}

__global__ __launch_bounds__(kThreads) void scan_down(const int* __restrict__ in, long long* __restrict__ out,
                                                      long long n, const long long* __restrict__ tmp) {
  const long long base = (long long)blockIdx.x * kTile + threadIdx.x * kItems;
  int v[kItems];
  load_items(in, base, n, v);
  long long s = 0;
#pragma unroll
  for (int i = 0; i < kItems; ++i) s += v[i];
  long long tot;
  long long run = tmp[blockIdx.x] + block_excl_scan<kThreads>(s, &tot);
  if (base + kItems <= n && ((uintptr_t)out & 15u) == 0) {
#pragma unroll
    for (int i = 0; i < kItems; i += 2) {
      *(longlong2*)(out + base + i) = make_longlong2(run, run + v[i]);
      run += v[i] + v[i + 1];
    }
  } else {
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      if (base + i < n) out[base + i] = run;
      run += v[i];
    }
  }
}
}  // namespace

size_t scan_tmp_elems(long long n) { return (size_t)((n + kTile - 1) / kTile) + 1; }

hipError_t launch_scan(const int* in, long long* out, long long n, long long* total, long long* tmp, hipStream_t s,
                       long long base) {
  if (n <= kOneBlock) {
    scan_one<<<1, kOneThreads, 0, s>>>(in, out, n, base, total);
    return hipGetLastError();
  }
  const long long nb = (n + kTile - 1) / kTile;
  scan_reduce<<<(unsigned)nb, kThreads, 0, s>>>(in, n, tmp);
  scan_blocks<<<1, kOneThreads, 0, s>>>(tmp, nb, base, total);
  scan_down<<<(unsigned)nb, kThreads, 0, s>>>(in, out, n, tmp);
  return hipGetLastError();
}

}  // namespace ftk
