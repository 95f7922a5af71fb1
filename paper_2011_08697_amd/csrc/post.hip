// post.hip -- trajectory post-processing on the device, after the tracking passes.
//
//   * Slicing at a time step (Sec. 3.2, "Ordinal and interval mesh elements"): the critical points of step t0 are
//     the punctured ordinal faces anchored at t0 (faces whose axis masks do not use the time axis).  Hits are
//     sorted by face id and face ids are t-major, so they form one contiguous range of the hit arrays.
//   * Per-trajectory attributes for filtering (Sec. 4.4, "Filtering"): number of points, time extent of their
//     spacetime positions, and the number of ends.  Under the symbolic perturbation every punctured face lies in
//     exactly two cells with one more punctured side each, unless it lies in a boundary hyperplane of the grid
//     (a coordinate equal to 0 with the axis unused, or equal to N - 1), where only one cell exists; so a
//     trajectory is a path with two boundary ends or a closed loop with none.
//   * Loop filtering: drop closed loops (a transient birth-death pair) whose time extent is below a threshold.
//   * Order of the points along each trajectory (cell neighbours, list ranking over a sparse ruling set), and the type
//     smoothing and run simplification that walk it (Sec. 4.4, "Simplification" and "Smoothing").
//
// All of it is bound by memory: streams over the hit arrays and single-entry gathers between them.  Flags over hits or
// positions are therefore kept as words of 64 with a prefix count per word (a rank costs two loads of a small array),
// and the face id -> index lookups of dense results read one entry per vertex.  Whole sequence (table, order, smoothing,
// simplification, filter, slice) on noise 1024^2 x 24, 44.8M points on 1.5M trajectories: 19.1 -> 7.3 ms.
#include <climits>

#include "common.h"
#include "internal.h"
#include "kuhn.h"

namespace ftk {

namespace {

template <int N>
constexpr int kFaceTypes = N == 2 ? 12 : 60;

// Extents (x, y, [z], t) of the grid and its number of vertices.
struct FaceSpace {
  int n;  // spatial dimension
  long long N[4];
  long long V;
  int T;  // face types per vertex
};

constexpr unsigned face_mask(int n, int ty, int k) { return n == 2 ? kTri2.m[ty][k] : kTet3.m[ty][k]; }

constexpr unsigned face_used_axes(int n, int ty) {
  unsigned u = 0;
  for (int k = 0; k < n; ++k) u |= face_mask(n, ty, k);
  return u;
}

// a / b for a, b >= 0: the 64-bit division is a long instruction sequence, so values of 32 bits take the short one
__device__ __forceinline__ long long quotient(long long a, long long b) {
  if (((a | b) >> 32) == 0) return (unsigned)a / (unsigned)b;
  return a / b;
}

// anchor coordinates c[0..N] (time last) of vertex v
template <int N>
__device__ __forceinline__ void vertex_decode(const FaceSpace& fs, long long v, long long* c) {
#pragma unroll
  for (int a = 0; a < N; ++a) {
    const long long q = quotient(v, fs.N[a]);
    c[a] = v - q * fs.N[a];
    v = q;
  }
  c[N] = v;
}

// first index in [0, n) with keys[i] >= v (keys ascending)
__device__ __forceinline__ long long lower_bound64(const long long* keys, long long n, long long v) {
  long long lo = 0, hi = n;
  while (lo < hi) {
    const long long mid = (lo + hi) >> 1;
    if (keys[mid] < v)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// ---------------------------------------------------------------------------------------------------------------
// Flags over hits or positions: one bit each in words of 64 (the ballot of the wavefront that decided them) and the
// number of set bits before each word.
// ---------------------------------------------------------------------------------------------------------------
struct Ranks {
  const unsigned long long* bits;
  const long long* base;
};

__device__ __forceinline__ unsigned long long below(int b) { return (1ull << b) - 1ull; }

__device__ __forceinline__ bool flagged(const Ranks& r, long long i) { return (r.bits[i >> 6] >> (i & 63)) & 1ull; }

// set flags before i
__device__ __forceinline__ long long rank_of(const Ranks& r, long long i) {
  return r.base[i >> 6] + __popcll(r.bits[i >> 6] & below((int)(i & 63)));
}

// stores the wavefront's flags as word i >> 6 (i: the thread's index, 64 consecutive ones per wavefront)
__device__ __forceinline__ void store_flags(bool f, long long i, long long n_words, unsigned long long* bits, int* cnt) {
  const unsigned long long m = __ballot(f);
  if ((threadIdx.x & 63) == 0 && (i >> 6) < n_words) {
    bits[i >> 6] = m;
    cnt[i >> 6] = __popcll(m);
  }
}

// ---------------------------------------------------------------------------------------------------------------
// Index of a face id in a sorted id array (hits, or trajectory labels).  Dense form: an entry per vertex (index of the
// vertex's first id, mask of its types), one load per lookup.  Sparse form: ids bucketed by vertex row (bucket b holds
// the ids in [b B, (b + 1) B) with B = T nx, bstart[b] is its first index), a search within the row.
// ---------------------------------------------------------------------------------------------------------------
template <int N>
struct Entry;
template <>
struct alignas(8) Entry<2> {
  unsigned first, mask;
};
template <>
struct alignas(16) Entry<3> {
  unsigned long long mask, first;
};

struct Ids {
  const long long* id;
  const void* entry;        // dense form: V entries
  long long V;
  const long long* bstart;  // sparse form
  long long nx;
};

template <int N, bool DENSE>
__device__ __forceinline__ long long find_id(const Ids& s, long long v, int ty) {
  if constexpr (DENSE) {
    const bool in = v >= 0 && v < s.V;
    const Entry<N> e = ((const Entry<N>*)s.entry)[in ? v : 0];
    const long long k = (long long)e.first + __popcll((unsigned long long)e.mask & below(ty));
    return in && ((e.mask >> ty) & 1u) ? k : -1;
  } else {
    if (v < 0 || v >= s.V) return -1;
    const long long f = v * kFaceTypes<N> + ty, b = quotient(v, s.nx);
    const long long lo = s.bstart[b], hi = s.bstart[b + 1];
    const long long k = lo + lower_bound64(s.id + lo, hi - lo, f);
    return (k < hi && s.id[k] == f) ? k : -1;
  }
}

template <int N, bool DENSE>
__device__ __forceinline__ long long find_id(const Ids& s, long long f) {
  if (f < 0) return -1;
  const long long v = f / kFaceTypes<N>;
  return find_id<N, DENSE>(s, v, (int)(f - v * kFaceTypes<N>));
}

// dense form (entries cleared beforehand): a vertex's first id writes its entry, the ids after it read from LDS
template <int N>
__global__ __launch_bounds__(256) void k_entries(const long long* __restrict__ id, long long n, long long V,
                                                 Entry<N>* __restrict__ entry) {
  constexpr int T = kFaceTypes<N>;
  __shared__ long long f[256 + T];  // f[0]: the id before the block's
  const long long i0 = (long long)blockIdx.x * 256;
  for (int k = threadIdx.x; k < 256 + T; k += 256) {
    const long long i = i0 + k - 1;
    f[k] = i >= 0 && i < n ? id[i] : -T;
  }
  __syncthreads();
  const int k = threadIdx.x + 1;
  const long long v = f[k] / T;
  if (i0 + threadIdx.x >= n || f[k] < 0 || v >= V || f[k - 1] >= v * T) return;
  unsigned long long mask = 0;
  for (int q = k; q < k + T && q < 256 + T; ++q) {
    const long long d = f[q] - v * T;
    if (d < 0 || d >= T) break;
    mask |= 1ull << d;
  }
  Entry<N> e;
  e.first = (unsigned)(i0 + threadIdx.x);
  e.mask = (decltype(e.mask))mask;
  entry[v] = e;
}

// sparse form
__global__ void k_buckets(const long long* __restrict__ id, long long n, long long B, long long n_buckets,
                          long long* __restrict__ bstart) {
  const long long b = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (b <= n_buckets) bstart[b] = lower_bound64(id, n, b * B);
}

// Per-trajectory (or per-run) accumulation.  Consecutive hits often belong to the same trajectory, so the lanes of
// a wave first combine over runs of equal keys (segmented reduction by shuffles) and only the first lane of each
// run goes to memory.  Lanes without a key pass a negative one of their own.  True for the lanes that head a run.
struct RunAcc {
  unsigned cnt;
  int mn, mx, ends;
};

__device__ __forceinline__ bool wave_run_reduce(long long key, RunAcc& a) {
  const int lane = threadIdx.x & 63;
  const long long prev = __shfl_up(key, 1);
  const bool head = lane == 0 || prev != key;
  const unsigned long long hb = __ballot(head);
  // lanes of this lane's run after it
  const unsigned long long later = lane == 63 ? 0ull : hb >> (lane + 1);
  const int left = later ? __ffsll((long long)later) - 1 : 63 - lane;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    if (!__ballot(left >= o)) break;
    const unsigned c2 = __shfl_down(a.cnt, o);
    const int mn2 = __shfl_down(a.mn, o), mx2 = __shfl_down(a.mx, o), e2 = __shfl_down(a.ends, o);
    if (o <= left) {
      a.cnt += c2;
      a.mn = min(a.mn, mn2);
      a.mx = max(a.mx, mx2);
      a.ends += e2;
    }
  }
  return head;
}

// A bound that other threads may improve meanwhile: an old value only costs a superfluous atomic.
__device__ __forceinline__ int seen(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__global__ void k_root_words(const long long* __restrict__ face_id, const long long* __restrict__ label, long long n,
                             unsigned long long* __restrict__ bits, int* __restrict__ cnt) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  store_flags(i < n && label[i] == face_id[i], i, (n + 63) >> 6, bits, cnt);
}

// (a lane per word here and in k_ruler_list: a lane per hit spends its time on launching waves without a flag)
__global__ void k_root_scatter(const long long* __restrict__ face_id, Ranks r, long long n_words, long long n_traj,
                               long long* __restrict__ roots, unsigned* __restrict__ status) {
  const long long w = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= n_words) return;
  long long j = r.base[w];
  for (unsigned long long m = r.bits[w]; m; m &= m - 1ull, ++j) {
    if (j < n_traj)
      roots[j] = face_id[(w << 6) + __ffsll((long long)m) - 1];
    else
      atomicOr(status, ST_INVARIANT);
  }
}

__global__ void k_traj_init(long long n_traj, unsigned long long* __restrict__ n_hits, int* __restrict__ t_min,
                            int* __restrict__ t_max, int* __restrict__ n_ends) {
  const long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_traj) return;
  n_hits[j] = 0;
  t_min[j] = 0x7f800000;  // +inf
  t_max[j] = 0;           // 0.0f: spacetime times are >= 0, so their bit patterns order like the values
  n_ends[j] = 0;
}

// The attributes of the trajectories: bound by the atomics, so they are combined first -- over runs of equal labels in
// a wavefront, then over kAccumItems hits per lane of the block in an LDS table (0.21 trajectories per hit are left of
// 0.40 runs on noise 1024^2 x 24) -- and a time bound goes to memory only where it improves the one seen.  Hits come in
// ascending time, so in their own order nearly every entry would raise t_max; the blocks take them in a scattered order
// (step has no factor in common with the grid), which leaves about the logarithm of a trajectory's entries.  44.8M hits:
// 1.98 -> 0.78 ms (1.58 in their own order and without the table, 1.04 without the table).
constexpr int kAccumItems = 4;
constexpr int kAccumSlots = 1024;
constexpr int kAccumProbes = 16;

template <int N, bool DENSE>
__global__ __launch_bounds__(256) void k_traj_accum(FaceSpace fs, const long long* __restrict__ face_id,
                                                    const long long* __restrict__ label,
                                                    const float* __restrict__ pos, long long n, Ids roots,
                                                    unsigned step, unsigned long long* __restrict__ n_hits,
                                                    int* __restrict__ t_min, int* __restrict__ t_max,
                                                    int* __restrict__ n_ends, unsigned* __restrict__ status) {
  __shared__ unsigned slot[kAccumSlots], cnt[kAccumSlots];  // trajectory (kFree: none), points
  __shared__ int mn[kAccumSlots], mx[kAccumSlots];
  constexpr unsigned kFree = 0xffffffffu;
  for (int k = threadIdx.x; k < kAccumSlots; k += 256) {
    slot[k] = kFree;
    cnt[k] = 0;
    mn[k] = 0x7f800000;
    mx[k] = 0;
  }
  __syncthreads();
  const unsigned block = (unsigned)((unsigned long long)blockIdx.x * step % gridDim.x);
  const long long i0 = (long long)block * (256 * kAccumItems) + threadIdx.x;
#pragma unroll 1
  for (int it = 0; it < kAccumItems; ++it) {
    const long long i = i0 + it * 256;
    long long key = -1 - (long long)(threadIdx.x & 63);
    RunAcc a = {0u, 0x7f800000, 0, 0};
    if (i < n) {
      const long long j = find_id<N, DENSE>(roots, label[i]);
      if (j < 0) {
        atomicOr(status, ST_INVARIANT);
      } else {
        key = j;
        const int tb = __float_as_int(pos[i * (N + 1) + N]);
        a.cnt = 1;
        a.mn = tb;
        a.mx = tb;
        // in a boundary hyperplane of the grid one cell holds the face
        const long long f = face_id[i], v = f / kFaceTypes<N>;
        const unsigned used = face_used_axes(N, (int)(f - v * kFaceTypes<N>));
        long long c[N + 1];
        vertex_decode<N>(fs, v, c);
        bool end = false;
#pragma unroll
        for (int x = 0; x <= N; ++x) end |= c[x] == fs.N[x] - 1 || (c[x] == 0 && !((used >> x) & 1u));
        a.ends = end ? 1 : 0;
      }
    }
    if (!wave_run_reduce(key, a) || key < 0) continue;
    if (a.ends) atomicAdd(&n_ends[key], a.ends);
    unsigned h = ((unsigned)key * 0x9e3779b1u) >> 22;
    static_assert(kAccumSlots == 1024, "the hash has 10 bits");
    bool kept = false;
    if (key < (long long)kFree) {
      for (int probe = 0; probe < kAccumProbes && !kept; ++probe) {
        const unsigned was = atomicCAS(&slot[h], kFree, (unsigned)key);
        kept = was == kFree || was == (unsigned)key;
        if (!kept) h = (h + 1) & (kAccumSlots - 1);
      }
    }
    if (kept) {
      atomicAdd(&cnt[h], a.cnt);
      atomicMin(&mn[h], a.mn);
      atomicMax(&mx[h], a.mx);
    } else {
      atomicAdd(&n_hits[key], (unsigned long long)a.cnt);
      atomicMin(&t_min[key], a.mn);
      atomicMax(&t_max[key], a.mx);
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kAccumSlots; k += 256) {
    const unsigned key = slot[k];
    if (key == kFree) continue;
    atomicAdd(&n_hits[key], (unsigned long long)cnt[k]);
    if (mn[k] < seen(&t_min[key])) atomicMin(&t_min[key], mn[k]);
    if (mx[k] > seen(&t_max[key])) atomicMax(&t_max[key], mx[k]);
  }
}

__global__ void k_slice_flags(FaceSpace fs, const long long* __restrict__ face_id, long long lo, long long hi,
                              int* __restrict__ flag) {
  const long long i = lo + (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= hi) return;
  const int ty = (int)(face_id[i] % fs.T);
  const unsigned tbit = 1u << fs.n;
  flag[i - lo] = (face_used_axes(fs.n, ty) & tbit) ? 0 : 1;
}

__global__ void k_slice_scatter(const int* __restrict__ flag, const long long* __restrict__ off, long long lo,
                                long long cnt, long long* __restrict__ idx) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < cnt && flag[k]) idx[off[k]] = lo + k;
}

// The trajectory of a hit by its label: the first steps of the search run over kSamples evenly spaced labels in LDS
// (64 KB, two blocks a CU), the last ones in memory; steps of fixed length, without branches.  1.5M labels, 44.8M hits:
// 0.93 -> 0.56 ms.
constexpr int kSamples = 8192;

__global__ __launch_bounds__(1024) void k_filter_loops(const long long* __restrict__ label, long long n,
                                                       const long long* __restrict__ roots, long long n_traj,
                                                       const int* __restrict__ t_min, const int* __restrict__ t_max,
                                                       const int* __restrict__ n_ends, float min_duration,
                                                       uint8_t* __restrict__ keep) {
  __shared__ long long sample[kSamples];
  long long stride = 1;
  while (stride * kSamples < n_traj) stride *= 2;
  for (int k = threadIdx.x; k < kSamples; k += blockDim.x) sample[k] = k * stride < n_traj ? roots[k * stride] : LLONG_MAX;
  __syncthreads();
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const long long L = label[i];
    int at = 0;  // the last sample not above L (the first label otherwise)
#pragma unroll
    for (int half = kSamples / 2; half > 0; half >>= 1) at += sample[at + half] <= L ? half : 0;
    long long j = at * stride;
    for (long long half = stride >> 1; half > 0; half >>= 1) {
      const long long k = j + half;
      j = k < n_traj && roots[k] <= L ? k : j;
    }
    bool k = true;
    if (j < n_traj && roots[j] == L && n_ends[j] == 0)
      k = !(__int_as_float(t_max[j]) - __int_as_float(t_min[j]) < min_duration);
    keep[i] = k ? 1 : 0;
  }
}

__global__ void k_range(FaceSpace fs, const long long* __restrict__ face_id, long long n, long long t0,
                        long long* __restrict__ out) {
  if (threadIdx.x != 0) return;
  long long plane_faces = fs.T;
  for (int a = 0; a < fs.n; ++a) plane_faces *= fs.N[a];
  out[0] = lower_bound64(face_id, n, t0 * plane_faces);
  out[1] = lower_bound64(face_id, n, (t0 + 1) * plane_faces);
}

// ---------------------------------------------------------------------------------------------------------------
// Order of the points along each trajectory.  The curve's piece in a cell is the segment between the cell's two
// punctured sides, so the neighbours of a hit are the other punctured side of each cell that holds it (at most
// two cells).  A face with axis masks (M_1..M_n) and unused axes R lies in the cells (R, M_1..M_n) anchored one
// step back along R and (M_1..M_n, R) at its own anchor when R is one axis; when R is empty, exactly one mask
// holds two axes {a, b} and the cells split it as (.., a, b, ..) or (.., b, a, ..) at the same anchor.  A cell
// (s_0..s_n) anchored at c drops vertex k to give a side: k = 0 moves the anchor to c + e(s_0) with masks
// (s_1..s_n); k = n + 1 keeps (s_0..s_{n-1}); an inner k merges s_{k-1} | s_k.
// ---------------------------------------------------------------------------------------------------------------

//
// All of it depends on the face type only, up to the vertex offset of the sides: build_sides lists, per type and cell,
// the n + 1 other sides and the axes along which the cell's anchor lies one step back.
template <int N>
struct Sides {
  unsigned char back[kFaceTypes<N>];                // of cell 0; cell 1 is anchored at the face's own anchor
  signed char d[kFaceTypes<N>][2][N + 1][N + 1];    // vertex offset of a side's anchor along each axis
  unsigned char type[kFaceTypes<N>][2][N + 1];
};

constexpr int type_of_masks(int n, const unsigned* m) {
  return n == 2 ? (int)kTri2Index.idx[m[0]][m[1]] : (int)kTet3Index.idx[m[0]][m[1]][m[2]];
}

template <int N>
constexpr Sides<N> build_sides() {
  Sides<N> r{};
  constexpr int D = N + 1;
  for (int ty = 0; ty < kFaceTypes<N>; ++ty) {
    const unsigned R = ((1u << D) - 1u) ^ face_used_axes(N, ty);
    r.back[ty] = (unsigned char)R;
    for (int cell = 0; cell < 2; ++cell) {
      unsigned s[4] = {0, 0, 0, 0};
      if (R) {
        for (int k = 0; k < N; ++k) s[cell == 0 ? k + 1 : k] = face_mask(N, ty, k);
        s[cell == 0 ? 0 : N] = R;
      } else {
        int o = 0;
        for (int k = 0; k < N; ++k) {
          const unsigned M = face_mask(N, ty, k);
          if (popc_c((int)M) == 2) {
            const unsigned lo = M & (0u - M), hi = M ^ lo;
            s[o++] = cell == 0 ? lo : hi;
            s[o++] = cell == 0 ? hi : lo;
          } else {
            s[o++] = M;
          }
        }
      }
      int n = 0;
      for (int k = 0; k <= D; ++k) {
        int off[4] = {0, 0, 0, 0};
        for (int a = 0; a < D; ++a) off[a] = (cell == 0 && ((R >> a) & 1u)) ? -1 : 0;
        unsigned m[4] = {0, 0, 0, 0};
        if (k == 0) {
          for (int a = 0; a < D; ++a) off[a] += (int)((s[0] >> a) & 1u);
          for (int q = 0; q < N; ++q) m[q] = s[q + 1];
        } else if (k == D) {
          for (int q = 0; q < N; ++q) m[q] = s[q];
        } else {
          int o = 0;
          for (int q = 0; q < D; ++q) {
            if (q == k - 1) {
              m[o++] = s[q] | s[q + 1];
              ++q;
            } else {
              m[o++] = s[q];
            }
          }
        }
        const int side = type_of_masks(N, m);
        bool self = side == ty;
        for (int a = 0; a < D; ++a) self = self && off[a] == 0;
        if (self) continue;
        for (int a = 0; a < D; ++a) r.d[ty][cell][n][a] = (signed char)off[a];
        r.type[ty][cell][n] = (unsigned char)side;
        ++n;
      }
    }
  }
  return r;
}
constexpr auto kSides2 = build_sides<2>();
constexpr auto kSides3 = build_sides<3>();

// A lookup per other side of the two cells (6 in 2D, 8 in 3D), with the vertex offsets of the sides in LDS; the loads of
// the dense form do not depend on each other.  Noise 1024^2 x 24: 2.85 -> 0.45 ms (searches in per-vertex buckets,
// sides decoded per hit with 64-bit divisions).
template <int N, bool DENSE>
__global__ __launch_bounds__(256) void k_neighbours(FaceSpace fs, long long n_hits, Ids hits, int2* __restrict__ nb,
                                                    unsigned* __restrict__ status) {
  constexpr int T = kFaceTypes<N>, K = N + 1, E = T * 2 * K;
  __shared__ long long sides[E];  // vertex offset * 64 + type
  __shared__ unsigned char back[T];
  for (int e = threadIdx.x; e < E; e += blockDim.x) {
    const int ty = e / (2 * K), cell = e / K & 1, k = e % K;
    long long d = 0;
    for (int a = N; a >= 0; --a)
      d = d * fs.N[a] + (N == 2 ? kSides2.d[ty % 12][cell][k % 3][a % 3] : kSides3.d[ty][cell][k][a]);
    sides[e] = d * 64 + (N == 2 ? kSides2.type[ty % 12][cell][k % 3] : kSides3.type[ty][cell][k]);
  }
  for (int t = threadIdx.x; t < T; t += blockDim.x) back[t] = N == 2 ? kSides2.back[t % 12] : kSides3.back[t];
  __syncthreads();
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_hits) return;
  const long long fid = hits.id[i], v = fid / T;
  const int ty = (int)(fid - v * T);
  long long c[N + 1];
  vertex_decode<N>(fs, v, c);
  const unsigned R = back[ty];
  bool inside[2] = {true, true};
#pragma unroll
  for (int a = 0; a <= N; ++a) {
    const long long c0 = c[a] - ((R >> a) & 1u);
    inside[0] &= c0 >= 0 && c0 <= fs.N[a] - 2;
    inside[1] &= c[a] <= fs.N[a] - 2;
  }
  long long h[2][K];
#pragma unroll
  for (int cell = 0; cell < 2; ++cell)
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const long long s = sides[(ty * 2 + cell) * K + k];
      // without branches, so that the loads are in flight together: outside the grid the face's own entry is read
      h[cell][k] = find_id<N, DENSE>(hits, inside[cell] ? v + (s >> 6) : v, (int)(s & 63));
    }
  int found[2] = {-1, -1};
  int nf = 0;
  bool bad = false;
#pragma unroll
  for (int cell = 0; cell < 2; ++cell) {
    if (!inside[cell]) continue;
    int hits_here = 0;
    long long other = -1;
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (h[cell][k] >= 0) {
        ++hits_here;
        other = h[cell][k];
      }
    if (hits_here != 1)
      bad = true;
    else if (nf++ == 0)
      found[0] = (int)other;
    else
      found[1] = (int)other;
  }
  if (bad || nf == 0) atomicOr(status, ST_INVARIANT);
  if (nf == 2 && found[1] < found[0]) {
    const int x = found[0];
    found[0] = found[1];
    found[1] = x;
  }
  nb[i] = make_int2(found[0], found[1]);
}

// A closed loop is cut between its label face (the root: smallest face id, so smallest index) and its neighbour
// with the larger face id; the walk then runs root, smaller neighbour, ..., larger neighbour.
template <int N, bool DENSE>
__global__ void k_cut_loops(const long long* __restrict__ roots, const int* __restrict__ n_ends, long long n_traj,
                            long long n_hits, Ids hits, int2* __restrict__ nb, unsigned* __restrict__ status) {
  const long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_traj || n_ends[j] != 0) return;
  const long long i = find_id<N, DENSE>(hits, roots[j]);
  if (i < 0) {
    atomicOr(status, ST_INVARIANT);
    return;
  }
  int2 q = nb[i];
  const int b = q.y;
  if (b < 0 || b >= n_hits) return;
  q.y = -1;
  nb[i] = q;
  int2 r = nb[b];
  if (r.x == (int)i) r.x = -1;
  if (r.y == (int)i) r.y = -1;
  nb[b] = r;
}

// List ranking by a sparse ruling set.  Rulers are the path ends and about one hit in kRulerEvery chosen by an
// integer hash of the index (the "lowbias32" mixer of C. Wellons).  The rulers are numbered (slots); arm 2 s + k of
// slot s leads along neighbour k of its hit.  Each arm walks to the next ruler and keeps (the arm that leads on from
// there, distance); an arm without a neighbour keeps itself at distance 0.  Pointer jumping on the arms finds the path
// ends, the rulers take their positions, and a second walk along the arms that lead away from the start writes the
// order: consecutive entries, where keeping (ruler, distance) per hit cost two scattered stores and a gather.
constexpr unsigned kRulerEvery = 32;

__device__ __forceinline__ unsigned mix32(unsigned x) {
  x ^= x >> 16;
  x *= 0x7feb352dU;
  x ^= x >> 15;
  x *= 0x846ca68bU;
  x ^= x >> 16;
  return x;
}

__device__ __forceinline__ bool is_ruler(int2 q, unsigned i) {
  return q.x < 0 || q.y < 0 || (mix32(i) & (kRulerEvery - 1u)) == 0u;
}

__global__ void k_ruler_words(const int2* __restrict__ nb, long long n_hits, unsigned long long* __restrict__ bits,
                              int* __restrict__ cnt) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  store_flags(i < n_hits && is_ruler(nb[i], (unsigned)i), i, (n_hits + 63) >> 6, bits, cnt);
}

__global__ void k_ruler_list(Ranks r, long long n_words, int* __restrict__ list) {
  const long long w = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= n_words) return;
  long long k = r.base[w];
  for (unsigned long long m = r.bits[w]; m; m &= m - 1ull) list[k++] = (int)((w << 6) + __ffsll((long long)m) - 1);
}

__device__ __forceinline__ unsigned long long arm_state(unsigned arm, unsigned dist) {
  return ((unsigned long long)dist << 32) | arm;
}

// Items per wavefront of the two walks: their lengths differ widely (a wavefront of fixed items would wait for the
// longest of 64), so a lane that is done takes the next item of its wavefront's share, as soon as kRefill lanes are.
constexpr int kWalkShare = 128;
constexpr int kRefill = 16;

__global__ __launch_bounds__(256) void k_walk(const int2* __restrict__ nb, Ranks rulers, const int* __restrict__ list,
                                              long long n_arms, int share, long long n_hits,
                                              unsigned long long* __restrict__ st, unsigned* __restrict__ status) {
  const int lane = threadIdx.x & 63;
  long long next = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * share;
  const long long end = min(next + share, n_arms);
  bool busy = false;
  long long arm = 0;
  int prev = 0, v = 0;
  unsigned dist = 0;
  for (;;) {
    const unsigned long long idle = __ballot(!busy);
    if (next < end && __popcll(idle) >= kRefill) {
      const long long mine = next + __popcll(idle & below(lane));
      if (!busy && mine < end) {
        const int R = list[mine >> 1];
        const int2 q = nb[R];
        const int first = (mine & 1) ? q.y : q.x;
        if (first < 0) {  // no neighbour this way: the ruler is a path end, its own far end at distance 0
          st[mine] = arm_state((unsigned)mine, 0);
        } else {
          arm = mine;
          prev = R;
          v = first;
          dist = 1;
          busy = true;
        }
      }
      next += __popcll(idle);
      continue;
    }
    if (idle == ~0ull) break;
    if (busy) {
      const int2 w = nb[v];
      const int s = w.x == prev ? 0 : 1;
      if ((s ? w.y : w.x) != prev || (long long)dist >= n_hits) {  // a walk cannot pass n_hits steps
        atomicOr(status, ST_INVARIANT);
        st[arm] = arm_state((unsigned)arm, 0);
        busy = false;
      } else if (is_ruler(w, (unsigned)v)) {
        st[arm] = arm_state(2u * (unsigned)rank_of(rulers, v) + (unsigned)(1 - s), dist);
        busy = false;
      } else {
        prev = v;
        v = s ? w.x : w.y;
        ++dist;
      }
    }
  }
}

// Pointer jumping over the listed arms (all of them when act is null), in place: a state is one 64-bit word that
// always names a true arm and distance further along the path, whichever of its values a reader meets, so a launch
// makes kJumps jumps per arm, and arms that are still open are listed for the next.  An arm is closed once the arm it
// names leads nowhere.  (Two buffers and one jump per launch: 9 launches and synchronisations, 2.7 ms, on noise
// 1024^2 x 24; 2 launches, 0.22 ms now.)
constexpr int kJumps = 8;
constexpr int kJumpThreads = 1024;

__global__ __launch_bounds__(kJumpThreads) void k_jump(const unsigned* __restrict__ act, long long n_act, long long n_hits,
                       unsigned long long* __restrict__ st, unsigned* __restrict__ next,
                       unsigned long long* __restrict__ next_n, unsigned* __restrict__ status) {
  const long long a = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  bool open = false;
  unsigned arm = 0;
  if (a < n_act) {
    arm = act ? act[a] : (unsigned)a;
    unsigned long long s = __hip_atomic_load(&st[arm], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    open = true;
    for (int it = 0; it < kJumps && open; ++it) {
      const unsigned c = (unsigned)s;
      const unsigned long long t = __hip_atomic_load(&st[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((unsigned)t == c) {
        open = false;
      } else {
        const unsigned long long D = (s >> 32) + (t >> 32);
        if (D > (unsigned long long)n_hits) {  // longer than the hit count: a cycle the loop cut did not open
          atomicOr(status, ST_INVARIANT);
          open = false;
        } else {
          s = arm_state((unsigned)t, (unsigned)D);
          __hip_atomic_store(&st[arm], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
  }
  // one addition to the list's length per block: from every wavefront they queue at its address
  __shared__ unsigned before[kJumpThreads / 64 + 1];
  __shared__ unsigned long long first;
  const int wave = threadIdx.x >> 6;
  const unsigned long long m = __ballot(open);
  if ((threadIdx.x & 63) == 0) before[wave + 1] = (unsigned)__popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    before[0] = 0;
    for (int k = 1; k <= kJumpThreads / 64; ++k) before[k] += before[k - 1];
    const unsigned all = before[kJumpThreads / 64];
    first = all ? atomicAdd(next_n, (unsigned long long)all) : 0ull;
  }
  __syncthreads();
  if (open) next[first + before[wave] + __popcll(m & below(threadIdx.x & 63))] = arm;
}

__global__ void k_count_to_int(const unsigned long long* __restrict__ n_points, long long n_traj,
                               int* __restrict__ out) {
  const long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n_traj) out[j] = (int)n_points[j];
}

// Position of each ruler: trajectory start + distance to its start end (the end with the smaller index, i.e. the
// smaller face id); the path length through the ruler must equal the trajectory's point count.  place = position * 2 +
// the arm that leads away from the start, ~0 for an error.
template <int N>
__global__ void k_place_rulers(const int* __restrict__ list, long long n_rulers, long long n_hits,
                               const unsigned long long* __restrict__ st, const long long* __restrict__ label,
                               Ids roots, const long long* __restrict__ offsets, long long* __restrict__ order,
                               unsigned* __restrict__ place, unsigned* __restrict__ status) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n_rulers) return;
  const unsigned long long s0 = st[2 * t], s1 = st[2 * t + 1];
  const int R = list[t], E0 = list[(unsigned)s0 >> 1], E1 = list[(unsigned)s1 >> 1];
  const long long D0 = (long long)(s0 >> 32), D1 = (long long)(s1 >> 32);
  const long long j = find_id<N, false>(roots, label[R]);
  unsigned p = 0xffffffffu;
  if (j >= 0) {
    const long long len = D0 + D1 + 1, rank = E0 < E1 ? D0 : D1;
    const long long lo = offsets[j], hi = offsets[j + 1];
    if (len == hi - lo && lo >= 0 && hi <= n_hits) {
      order[lo + rank] = R;
      p = 2u * (unsigned)(lo + rank) + (E0 < E1 ? 1u : 0u);
    }
  }
  place[t] = p;
  if (p == 0xffffffffu) atomicOr(status, ST_INVARIANT);
}

// Order of the hits between the rulers; *placed += their number.  The entries of a walk are held back until a group of
// four (32 bytes) is whole: stores of one entry reached memory one by one, 32 bytes each.  An order array that is not
// aligned to 16 bytes takes the four as single entries.
__global__ __launch_bounds__(256) void k_walk_order(const int2* __restrict__ nb, const int* __restrict__ list,
                                                    const unsigned* __restrict__ place, long long n_rulers, int share,
                                                    long long n_hits, long long* __restrict__ order,
                                                    unsigned long long* __restrict__ placed,
                                                    unsigned* __restrict__ status) {
  const int lane = threadIdx.x & 63;
  long long next = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * share;
  const long long end = min(next + share, n_rulers);
  const bool wide = ((uintptr_t)order & 15u) == 0;
  bool busy = false;
  int prev = 0, v = 0;
  unsigned p = 0;                  // position of v
  int h0 = 0, h1 = 0, h2 = 0;      // the three entries before p
  unsigned held = 0;               // of which this many are not stored
  unsigned count = 0;
  for (;;) {
    const unsigned long long idle = __ballot(!busy);
    if (next < end && __popcll(idle) >= kRefill) {
      const long long mine = next + __popcll(idle & below(lane));
      if (!busy && mine < end) {
        const unsigned at = place[mine];
        const int R = list[mine];
        const int2 q = nb[R];
        const int first = (at & 1u) ? q.y : q.x;
        if (at != 0xffffffffu && first >= 0) {
          p = (at >> 1) + 1;
          prev = R;
          v = first;
          held = 0;
          busy = true;
        }
      }
      next += __popcll(idle);
      continue;
    }
    if (idle == ~0ull) break;
    if (busy) {
      const int2 w = nb[v];
      const bool past = (long long)p >= n_hits;
      if (past) atomicOr(status, ST_INVARIANT);
      if (past || is_ruler(w, (unsigned)v)) {
        if (held > 2) order[p - 3] = h0;
        if (held > 1) order[p - 2] = h1;
        if (held > 0) order[p - 1] = h2;
        busy = false;
      } else {
        if ((p & 3u) == 3u) {
          if (held == 3 && wide) {
            struct alignas(16) Pair {
              long long a, b;
            };
            ((Pair*)(order + p - 3))[0] = Pair{h0, h1};
            ((Pair*)(order + p - 3))[1] = Pair{h2, v};
          } else {
            if (held > 2) order[p - 3] = h0;
            if (held > 1) order[p - 2] = h1;
            if (held > 0) order[p - 1] = h2;
            order[p] = v;
          }
          held = 0;
        } else {
          ++held;
        }
        h0 = h1;
        h1 = h2;
        h2 = v;
        ++p;
        ++count;
        const int nxt = w.x == prev ? w.y : w.x;
        prev = v;
        v = nxt;
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) count += __shfl_down(count, o);
  if (lane == 0 && count) atomicAdd(placed, (unsigned long long)count);
}

// ---------------------------------------------------------------------------------------------------------------
// Type smoothing and run simplification along the order (Sec. 4.4).  Position k of order[] belongs to trajectory
// j with offsets[j] <= k < offsets[j + 1]; a trajectory without ends is a closed loop.
// ---------------------------------------------------------------------------------------------------------------

struct Walk {
  const long long* order;
  const long long* offsets;
  const int* n_ends;
  Ranks starts;  // positions where a trajectory starts in order[]
  long long n_traj, n_hits;
};

// Trajectory starts in order[] as words: a search per word (the offsets ascend) in place of flags and their scan.
__global__ void k_starts(const long long* __restrict__ offsets, long long n_traj, long long n_words,
                         unsigned long long* __restrict__ bits, long long* __restrict__ base) {
  const long long w = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= n_words) return;
  const long long p0 = w << 6, j0 = lower_bound64(offsets, n_traj, p0);
  unsigned long long m = 0;
  for (long long j = j0; j < n_traj && j < j0 + 64; ++j) {
    const long long d = offsets[j] - p0;
    if (d < 0 || d >= 64) break;
    m |= 1ull << d;
  }
  bits[w] = m;
  base[w] = j0;
}

// trajectory of position k, its start and length; false for inconsistent offsets
__device__ __forceinline__ bool locate(const Walk& w, long long k, long long* j, long long* lo, long long* m) {
  const long long a = rank_of(w.starts, k) + (flagged(w.starts, k) ? 1 : 0) - 1;
  if (a < 0 || a >= w.n_traj) return false;
  *j = a;
  *lo = w.offsets[a];
  *m = w.offsets[a + 1] - *lo;
  return *lo >= 0 && *m > 0 && *lo + *m <= w.n_hits && k >= *lo && k < *lo + *m;
}

__device__ __forceinline__ long long hit_at(const Walk& w, long long q, unsigned* status) {
  const long long h = w.order[q];
  if (h < 0 || h >= w.n_hits) {
    atomicOr(status, ST_INVARIANT);
    return -1;
  }
  return h;
}

// The types of a block's positions and of `half` (at most kSmoothHalo) positions on either side are gathered once, into
// LDS; a window reaches outside only for larger halves and where it wraps around a loop.  44.8M points, half 2:
// 0.75 -> 0.47 ms, and 0.35 for the trajectory starts -> 0.03.
constexpr int kSmoothItems = 4;
constexpr int kSmoothSpan = 256 * kSmoothItems;
constexpr int kSmoothHalo = 64;

__global__ __launch_bounds__(256) void k_smooth(Walk w, const uint8_t* __restrict__ type_in, int half,
                                                uint8_t* __restrict__ type_out, unsigned* __restrict__ status) {
  __shared__ uint8_t tile[kSmoothSpan + 2 * kSmoothHalo];
  const long long k0 = (long long)blockIdx.x * kSmoothSpan;
  const int halo = min(half, kSmoothHalo);
  long long hit[kSmoothItems];
#pragma unroll
  for (int i = 0; i < kSmoothItems; ++i) {
    const long long k = k0 + i * 256 + threadIdx.x;
    hit[i] = k < w.n_hits ? hit_at(w, k, status) : -1;
  }
#pragma unroll
  for (int i = 0; i < kSmoothItems; ++i)
    tile[kSmoothHalo + i * 256 + threadIdx.x] = hit[i] >= 0 ? type_in[hit[i]] : (uint8_t)0;
  if ((int)threadIdx.x < 2 * halo) {
    const int d = (int)threadIdx.x < halo ? (int)threadIdx.x - halo : kSmoothSpan + (int)threadIdx.x - halo;
    const long long k = k0 + d;
    if (k >= 0 && k < w.n_hits) {
      const long long h = hit_at(w, k, status);
      tile[kSmoothHalo + d] = h >= 0 ? type_in[h] : (uint8_t)0;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kSmoothItems; ++i) {
    const long long k = k0 + i * 256 + threadIdx.x;
    if (k >= w.n_hits) continue;
    long long j, lo, m;
    if (!locate(w, k, &j, &lo, &m)) {
      atomicOr(status, ST_INVARIANT);
      continue;
    }
    if (hit[i] < 0) continue;
    const int own = tile[kSmoothHalo + (int)(k - k0)];
    int res = own;
    const long long r = k - lo;
    const bool loop = w.n_ends[j] == 0;
    const bool fits = loop ? m >= 2LL * half + 1 : (r - half >= 0 && r + half <= m - 1);
    if (fits && half > 0) {
      int common = -1;
      bool same = true;
      for (int dlt = -half; dlt <= half && same; ++dlt) {
        if (dlt == 0) continue;
        long long q = r + dlt;
        if (q < 0) q += m;  // loops only, and m > 2 half there
        if (q >= m) q -= m;
        const long long d = lo + q - k0;
        int tq;
        if (d >= -halo && d < kSmoothSpan + halo) {
          tq = tile[kSmoothHalo + (int)d];
        } else {
          const long long hq = hit_at(w, lo + q, status);
          if (hq < 0) return;
          tq = type_in[hq];
        }
        if (common < 0) common = tq;
        same = tq == common;
      }
      if (same && common >= 0 && common != own) res = common;
    }
    type_out[hit[i]] = (uint8_t)res;
  }
}

// Runs: position q starts one where its type differs from the previous position's (of a loop's first position: the
// loop's last), and at the start of a path.  Runs are numbered by their starts; the positions of a loop before its first
// start belong to its last run, which wraps around; a loop of one type has no start.
__global__ __launch_bounds__(256) void k_run_words(Walk w, const uint8_t* __restrict__ type_in, long long n_words,
                                                   unsigned long long* __restrict__ bits, int* __restrict__ cnt,
                                                   unsigned* __restrict__ status) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  long long j, lo, m;
  long long before = -1;  // the previous position
  int own = 0;
  bool ok = false, start = false;
  if (q < w.n_hits) {
    ok = locate(w, q, &j, &lo, &m);
    if (!ok) {
      atomicOr(status, ST_INVARIANT);
    } else {
      const long long h = hit_at(w, q, status);
      if (h >= 0) own = type_in[h];
      if (q > lo)
        before = q - 1;
      else if (w.n_ends[j] == 0)
        before = lo + m - 1;
      else
        start = true;
    }
  }
  int type_before = __shfl_up(own, 1);
  if (before >= 0 && (before != q - 1 || (threadIdx.x & 63) == 0)) {
    const long long h = hit_at(w, before, status);
    if (h >= 0) type_before = type_in[h];
  }
  if (before >= 0) start = own != type_before;
  store_flags(ok && start, q, n_words, bits, cnt);
}

// The run of position q and the first and last run of its trajectory (last < first: a loop of one type)
struct Run {
  long long run, first, last;
};

__device__ __forceinline__ Run run_at(const Ranks& runs, long long q, long long lo, long long m) {
  Run r;
  const long long k = rank_of(runs, q) + (flagged(runs, q) ? 1 : 0);
  r.first = rank_of(runs, lo);
  r.last = rank_of(runs, lo + m) - 1;
  r.run = k > r.first ? k - 1 : r.last;
  return r;
}

__global__ void k_run_init(const long long* __restrict__ n_runs, int* __restrict__ t_min, int* __restrict__ t_max) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= *n_runs) return;
  t_min[i] = 0x7f800000;
  t_max[i] = 0;
}

// Time bounds and type of each run.  Atomics also for a run that lies within one wavefront: plain stores beside them,
// into the same lines, took 1.39 ms where atomics alone take 0.54 (noise 1024^2 x 24, 15.8M runs).
__global__ __launch_bounds__(256) void k_run_stats(Walk w, int n, const float* __restrict__ pos,
                                                   const uint8_t* __restrict__ type_in, Ranks runs,
                                                   int* __restrict__ t_min, int* __restrict__ t_max,
                                                   uint8_t* __restrict__ run_type, unsigned* __restrict__ status) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  long long key = -1 - (long long)(threadIdx.x & 63);
  RunAcc a = {0u, 0x7f800000, 0, 0};
  long long j, lo, m;
  if (q < w.n_hits && locate(w, q, &j, &lo, &m)) {
    const long long h = hit_at(w, q, status);
    const Run r = run_at(runs, q, lo, m);
    if (h >= 0 && r.last >= r.first) {
      if (r.run < 0 || r.run >= w.n_hits) {
        atomicOr(status, ST_INVARIANT);
      } else {
        key = r.run;
        a.mn = a.mx = __float_as_int(pos[h * (n + 1) + n]);
        if (flagged(runs, q)) run_type[key] = type_in[h];
      }
    }
  }
  if (wave_run_reduce(key, a) && key >= 0) {
    atomicMin(&t_min[key], a.mn);
    atomicMax(&t_max[key], a.mx);
  }
}

// New type of each point: that of its run, decided from the neighbouring runs of its trajectory (0.83 ms with the
// decision in a pass of its own -> 0.56, noise 1024^2 x 24).
__global__ __launch_bounds__(256) void k_run_apply(Walk w, Ranks runs, const int* __restrict__ t_min,
                                                   const int* __restrict__ t_max,
                                                   const uint8_t* __restrict__ run_type, float theta,
                                                   const uint8_t* __restrict__ type_in,
                                                   uint8_t* __restrict__ type_out, unsigned* __restrict__ status) {
  const long long q = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= w.n_hits) return;
  long long j, lo, m;
  if (!locate(w, q, &j, &lo, &m)) return;
  const long long h = hit_at(w, q, status);
  if (h < 0) return;
  const Run r = run_at(runs, q, lo, m);
  if (r.last < r.first) {
    type_out[h] = type_in[h];
    return;
  }
  if (r.first < 0 || r.last >= w.n_hits || r.run < r.first || r.run > r.last) return;
  uint8_t res = run_type[r.run];
  long long pr = -1, nx = -1;
  if (r.last > r.first) {
    if (w.n_ends[j] == 0) {
      pr = r.run > r.first ? r.run - 1 : r.last;
      nx = r.run < r.last ? r.run + 1 : r.first;
    } else if (r.run > r.first && r.run < r.last) {
      pr = r.run - 1;
      nx = r.run + 1;
    }
  }
  if (pr >= 0) {
    const float ext = __int_as_float(t_max[r.run]) - __int_as_float(t_min[r.run]);
    const float ep = __int_as_float(t_max[pr]) - __int_as_float(t_min[pr]);
    const float en = __int_as_float(t_max[nx]) - __int_as_float(t_min[nx]);
    if (ext < theta && run_type[pr] == run_type[nx] && ep >= theta && en >= theta) res = run_type[pr];
  }
  type_out[h] = res;
}

unsigned blocks_for(long long n) { return (unsigned)((n + 255) / 256 > 0 ? (n + 255) / 256 : 1); }

FaceSpace make_space(int n, const int64_t* dims_with_t) {
  FaceSpace fs;
  fs.n = n;
  fs.V = 1;
  for (int a = 0; a < 4; ++a) fs.N[a] = 1;
  for (int a = 0; a <= n; ++a) {
    fs.N[a] = dims_with_t[a];
    fs.V *= dims_with_t[a];
  }
  fs.T = n == 2 ? 12 : 60;
  return fs;
}

// Items per wavefront of a walk: a full share once the chip is covered several times.
int walk_share(long long items) {
  const long long s = items / 8192 / 64 * 64;
  return (int)(s < 64 ? 64 : s > kWalkShare ? kWalkShare : s);
}

unsigned walk_blocks(long long items, int share) {
  const long long per = 4LL * share;
  return (unsigned)((items + per - 1) / per > 0 ? (items + per - 1) / per : 1);
}

// Odd to the grid (no common factor) and about 0.618 of it: consecutive blocks fall far apart.
unsigned scatter_step(unsigned blocks) {
  unsigned s = (unsigned)(blocks * 0.6180339887498949);
  if (s < 1) s = 1;
  for (;; ++s) {
    unsigned a = s, b = blocks;
    while (b) {
      const unsigned t = a % b;
      a = b;
      b = t;
    }
    if (a == 1) return s;
  }
}

template <int N>
hipError_t fill_entries(const long long* id, long long n, long long V, void* entry, hipStream_t s) {
  hipError_t e = hipMemsetAsync(entry, 0, sizeof(Entry<N>) * (size_t)V, s);
  if (e != hipSuccess) return e;
  k_entries<N><<<blocks_for(n), 256, 0, s>>>(id, n, V, (Entry<N>*)entry);
  return hipGetLastError();
}

// The lookup's table is built into `table`: entries (dense) or bucket starts.
template <int N>
hipError_t make_ids(const FaceSpace& fs, bool dense, const long long* id, long long n, void* table, Ids* out,
                    hipStream_t s) {
  Ids r;
  r.id = id;
  r.entry = dense ? table : nullptr;
  r.V = fs.V;
  r.bstart = dense ? nullptr : (const long long*)table;
  r.nx = fs.N[0];
  *out = r;
  if (dense) return fill_entries<N>(id, n, fs.V, table, s);
  const long long rows = fs.V / fs.N[0];
  k_buckets<<<blocks_for(rows + 1), 256, 0, s>>>(id, n, fs.T * fs.N[0], rows, (long long*)table);
  return hipGetLastError();
}

size_t entry_bytes(int n) { return n == 2 ? sizeof(Entry<2>) : sizeof(Entry<3>); }

size_t table_bytes(const FaceSpace& fs, bool dense) {
  return dense ? entry_bytes(fs.n) * (size_t)fs.V : sizeof(long long) * (size_t)(fs.V / fs.N[0] + 1);
}

// Entries per vertex pay while filling them (bytes per vertex) costs less than the searches they save (per hit); the
// bounds also keep the scratch of a call within 12 bytes per hit (table) and 128 (order).
bool dense_labels(const FaceSpace& fs, long long n_hits) {
  return (long long)entry_bytes(fs.n) * fs.V <= 12 * n_hits && n_hits <= INT_MAX;
}
bool dense_hits(const FaceSpace& fs, long long n_hits) { return (long long)entry_bytes(fs.n) * fs.V <= 128 * n_hits; }

template <int N>
hipError_t traj_table(const FaceSpace& fs, const long long* face_id, const long long* label, const float* pos,
                      long long n_hits, long long n_traj, const TableScratch& sc, long long* roots,
                      unsigned long long* hits, int* t_min, int* t_max, int* n_ends, long long* n_roots,
                      unsigned* status, hipStream_t s) {
  const long long nw = (n_hits + 63) / 64;
  k_root_words<<<blocks_for(n_hits), 256, 0, s>>>(face_id, label, n_hits, sc.bits, sc.cnt);
  hipError_t e = launch_scan(sc.cnt, sc.base, nw, n_roots, sc.scan_tmp, s);
  if (e != hipSuccess) return e;
  k_root_scatter<<<blocks_for(nw), 256, 0, s>>>(face_id, Ranks{sc.bits, sc.base}, nw, n_traj, roots, status);
  const bool dense = dense_labels(fs, n_hits);
  Ids ids;
  e = make_ids<N>(fs, dense, roots, n_traj, sc.table, &ids, s);
  if (e != hipSuccess) return e;
  const unsigned b = (unsigned)((n_hits + 256 * kAccumItems - 1) / (256 * kAccumItems)), step = scatter_step(b);
  auto* accum = dense ? k_traj_accum<N, true> : k_traj_accum<N, false>;
  accum<<<b, 256, 0, s>>>(fs, face_id, label, pos, n_hits, ids, step, hits, t_min, t_max, n_ends, status);
  return hipGetLastError();
}

}  // namespace

size_t traj_table_bytes(int n, const int64_t* dims_with_t, long long n_hits) {
  const FaceSpace fs = make_space(n, dims_with_t);
  return table_bytes(fs, dense_labels(fs, n_hits));
}
size_t order_hits_bytes(int n, const int64_t* dims_with_t, long long n_hits) {
  const FaceSpace fs = make_space(n, dims_with_t);
  return table_bytes(fs, dense_hits(fs, n_hits));
}
size_t order_labels_bytes(int n, const int64_t* dims_with_t) { return table_bytes(make_space(n, dims_with_t), false); }

hipError_t launch_traj_table(int n, const int64_t* dims_with_t, const long long* face_id, const long long* label,
                             const float* pos, long long n_hits, long long n_traj, const TableScratch& sc,
                             long long* roots, unsigned long long* hits, int* t_min, int* t_max, int* n_ends,
                             long long* n_roots, unsigned* status, hipStream_t s) {
  const FaceSpace fs = make_space(n, dims_with_t);
  k_traj_init<<<blocks_for(n_traj), 256, 0, s>>>(n_traj, hits, t_min, t_max, n_ends);
  if (n_hits == 0) return hipGetLastError();
  return n == 2 ? traj_table<2>(fs, face_id, label, pos, n_hits, n_traj, sc, roots, hits, t_min, t_max, n_ends, n_roots,
                                status, s)
                : traj_table<3>(fs, face_id, label, pos, n_hits, n_traj, sc, roots, hits, t_min, t_max, n_ends, n_roots,
                                status, s);
}

hipError_t launch_slice_range(int n, const int64_t* dims_with_t, const long long* face_id, long long n_hits,
                              long long t0, long long* range, hipStream_t s) {
  k_range<<<1, 64, 0, s>>>(make_space(n, dims_with_t), face_id, n_hits, t0, range);
  return hipGetLastError();
}

hipError_t launch_slice_compact(int n, const int64_t* dims_with_t, const long long* face_id, long long lo,
                                long long cnt, int* flag, long long* off, long long* total, long long* tmp,
                                long long* idx_out, bool scatter, hipStream_t s) {
  if (cnt <= 0) return hipSuccess;
  if (!scatter) {
    k_slice_flags<<<blocks_for(cnt), 256, 0, s>>>(make_space(n, dims_with_t), face_id, lo, lo + cnt, flag);
    return launch_scan(flag, off, cnt, total, tmp, s);
  }
  k_slice_scatter<<<blocks_for(cnt), 256, 0, s>>>(flag, off, lo, cnt, idx_out);
  return hipGetLastError();
}

hipError_t launch_filter_loops(const long long* label, long long n_hits, const long long* roots, long long n_traj,
                               const int* t_min, const int* t_max, const int* n_ends, float min_duration,
                               uint8_t* keep, hipStream_t s) {
  if (n_hits == 0) return hipSuccess;
  const long long blocks = (n_hits + 1023) / 1024;
  k_filter_loops<<<(unsigned)(blocks < 512 ? blocks : 512), 1024, 0, s>>>(label, n_hits, roots, n_traj, t_min, t_max,
                                                                          n_ends, min_duration, keep);
  return hipGetLastError();
}

namespace {

template <int N, bool DENSE>
void neighbours(const FaceSpace& fs, long long n_hits, const Ids& hits, const long long* roots, const int* n_ends,
                long long n_traj, int2* nb, unsigned* status, hipStream_t s) {
  k_neighbours<N, DENSE><<<blocks_for(n_hits), 256, 0, s>>>(fs, n_hits, hits, nb, status);
  k_cut_loops<N, DENSE><<<blocks_for(n_traj), 256, 0, s>>>(roots, n_ends, n_traj, n_hits, hits, nb, status);
}

template <int N>
hipError_t order_setup(const FaceSpace& fs, const long long* face_id, long long n_hits, const long long* roots,
                       const int* n_ends, long long n_traj, const OrderScratch& sc, unsigned* status, hipStream_t s) {
  const bool dense = dense_hits(fs, n_hits);
  Ids hits;
  hipError_t e = make_ids<N>(fs, dense, face_id, n_hits, sc.hits, &hits, s);
  if (e != hipSuccess) return e;
  if (dense)
    neighbours<N, true>(fs, n_hits, hits, roots, n_ends, n_traj, (int2*)sc.nb, status, s);
  else
    neighbours<N, false>(fs, n_hits, hits, roots, n_ends, n_traj, (int2*)sc.nb, status, s);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_order_setup(int n, const int64_t* dims_with_t, const long long* face_id, long long n_hits,
                              const long long* roots, const unsigned long long* n_points, const int* n_ends,
                              long long n_traj, const OrderScratch& sc, long long* n_rulers, long long* offsets,
                              unsigned* status, hipStream_t s) {
  const FaceSpace fs = make_space(n, dims_with_t);
  k_count_to_int<<<blocks_for(n_traj), 256, 0, s>>>(n_points, n_traj, sc.points);
  hipError_t e = launch_scan(sc.points, offsets, n_traj, offsets + n_traj, sc.scan_tmp, s);
  if (e != hipSuccess || n_hits == 0) return e;
  e = n == 2 ? order_setup<2>(fs, face_id, n_hits, roots, n_ends, n_traj, sc, status, s)
             : order_setup<3>(fs, face_id, n_hits, roots, n_ends, n_traj, sc, status, s);
  if (e != hipSuccess) return e;
  k_ruler_words<<<blocks_for(n_hits), 256, 0, s>>>((const int2*)sc.nb, n_hits, sc.bits, sc.cnt);
  return launch_scan(sc.cnt, sc.base, (n_hits + 63) / 64, n_rulers, sc.scan_tmp, s);
}

hipError_t launch_order_walk(const OrderScratch& sc, long long n_rulers, long long n_hits, int* list,
                             unsigned long long* st, unsigned* status, hipStream_t s) {
  if (n_rulers == 0) return hipSuccess;
  const Ranks rulers{sc.bits, sc.base};
  const long long nw = (n_hits + 63) / 64;
  k_ruler_list<<<blocks_for(nw), 256, 0, s>>>(rulers, nw, list);
  const int share = walk_share(2 * n_rulers);
  k_walk<<<walk_blocks(2 * n_rulers, share), 256, 0, s>>>((const int2*)sc.nb, rulers, list, 2 * n_rulers, share, n_hits,
                                                          st, status);
  return hipGetLastError();
}

hipError_t launch_order_jump(const unsigned* act, long long n_act, long long n_hits, unsigned long long* st,
                             unsigned* next, unsigned long long* next_n, unsigned* status, hipStream_t s) {
  if (n_act == 0) return hipSuccess;
  k_jump<<<(unsigned)((n_act + kJumpThreads - 1) / kJumpThreads), kJumpThreads, 0, s>>>(act, n_act, n_hits, st, next, next_n, status);
  return hipGetLastError();
}

hipError_t launch_order_place(int n, const int64_t* dims_with_t, const long long* label, long long n_hits,
                              const long long* roots, long long n_traj, const long long* offsets,
                              const OrderScratch& sc, const int* list, long long n_rulers,
                              const unsigned long long* st, unsigned* place, long long* order,
                              unsigned long long* placed, unsigned* status, hipStream_t s) {
  if (n_rulers == 0) return hipSuccess;
  const FaceSpace fs = make_space(n, dims_with_t);
  Ids ids;
  hipError_t e = n == 2 ? make_ids<2>(fs, false, roots, n_traj, sc.labels, &ids, s)
                        : make_ids<3>(fs, false, roots, n_traj, sc.labels, &ids, s);
  if (e != hipSuccess) return e;
  auto* rulers = n == 2 ? k_place_rulers<2> : k_place_rulers<3>;
  rulers<<<blocks_for(n_rulers), 256, 0, s>>>(list, n_rulers, n_hits, st, label, ids, offsets, order, place, status);
  const int share = walk_share(n_rulers);
  k_walk_order<<<walk_blocks(n_rulers, share), 256, 0, s>>>((const int2*)sc.nb, list, place, n_rulers, share, n_hits,
                                                            order, placed, status);
  return hipGetLastError();
}

namespace {

hipError_t make_walk(const long long* order, const long long* offsets, const int* n_ends, long long n_traj,
                     long long n_hits, unsigned long long* bits, long long* base, Walk* w, hipStream_t s) {
  const long long nw = (n_hits + 63) / 64;
  k_starts<<<blocks_for(nw), 256, 0, s>>>(offsets, n_traj, nw, bits, base);
  *w = Walk{order, offsets, n_ends, Ranks{bits, base}, n_traj, n_hits};
  return hipGetLastError();
}

}  // namespace

hipError_t launch_smooth(const long long* order, const long long* offsets, const int* n_ends, long long n_traj,
                         long long n_hits, const uint8_t* type_in, int half, unsigned long long* start_bits,
                         long long* start_base, uint8_t* type_out, unsigned* status, hipStream_t s) {
  if (n_hits == 0) return hipSuccess;
  Walk w;
  hipError_t e = make_walk(order, offsets, n_ends, n_traj, n_hits, start_bits, start_base, &w, s);
  if (e != hipSuccess) return e;
  k_smooth<<<(unsigned)((n_hits + kSmoothSpan - 1) / kSmoothSpan), 256, 0, s>>>(w, type_in, half, type_out, status);
  return hipGetLastError();
}

hipError_t launch_simplify(int n, const float* pos, const long long* order, const long long* offsets,
                           const int* n_ends, long long n_traj, long long n_hits, const uint8_t* type_in, float theta,
                           const RunScratch& sc, long long* n_runs, uint8_t* type_out, unsigned* status,
                           hipStream_t s) {
  if (n_hits == 0) return hipSuccess;
  Walk w;
  hipError_t e = make_walk(order, offsets, n_ends, n_traj, n_hits, sc.start_bits, sc.start_base, &w, s);
  if (e != hipSuccess) return e;
  const unsigned b = blocks_for(n_hits);
  const long long nw = n_hits / 64 + 1;  // the word of position n_hits too: a trajectory's last run is before its end
  k_run_words<<<blocks_for(64 * nw), 256, 0, s>>>(w, type_in, nw, sc.run_bits, sc.run_cnt, status);
  e = launch_scan(sc.run_cnt, sc.run_base, nw, n_runs, sc.scan_tmp, s);
  if (e != hipSuccess) return e;
  const Ranks runs{sc.run_bits, sc.run_base};
  k_run_init<<<b, 256, 0, s>>>(n_runs, sc.t_min, sc.t_max);
  k_run_stats<<<b, 256, 0, s>>>(w, n, pos, type_in, runs, sc.t_min, sc.t_max, sc.run_type, status);
  k_run_apply<<<b, 256, 0, s>>>(w, runs, sc.t_min, sc.t_max, sc.run_type, theta, type_in, type_out, status);
  return hipGetLastError();
}

}  // namespace ftk
