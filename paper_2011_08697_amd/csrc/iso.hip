// iso.hip -- isovolume tracking in 3D space + time (Sec. 6.1, two passes on the regular simplicial spacetime mesh;
// Alg. 1 right column).
//
// Mesh (Sec. 3.3): an edge anchored at vertex p with axis mask M (1..15; x = 1, y = 2, z = 4, t = 8) joins p and
// p + e(M); its id is g(p) * 15 + (M - 1) with the t-major vertex index g.  A pentachoron anchored at p with axis
// order (s1, s2, s3, s4) has the chain vertices p, p + e(s1), p + e(s1|s2), p + e(s1|s2|s3), p + e(1111).
//
//   iso_bits  -- the side of the level set of every vertex as one bit, 64 per word (a value equal to the isovalue
//                lies above it: the symbolic perturbation of a single entry is positive, Sec. 6.2).
//   iso_count -- one lane per word: crossings, tetrahedra (case I: one vertex on its side, 1 tetrahedron; case II: two,
//                3 tetrahedra), cubes with tetrahedra and runs of its 64 vertices, bit-parallel on the words of the 16
//                corners of their unit 4-cubes.
//   iso_runs_* - connected components of the vertices on one side of the level set, over runs of equal sides along x.
//   iso_emit  -- edge ids, intersection points p + mu e(M), mu = (c - f(p)) / (f(q) - f(p)), and the component of
//                every crossing, for the words that have any; the list of the cubes with tetrahedra.
//   iso_tess  -- per listed cube, its tetrahedra (indices of crossed edges): case I the four edges of the lone vertex
//                in chain order; case II the prism pair x triple split along the three monotone paths (staircase),
//                which matches on the quadrilateral shared with the neighbouring pentachoron.
//   iso_label -- the smallest edge id of each crossing's component.
//
// Isovolumes from vertex components.  An isovolume is a set of crossed edges connected through triangles (a triangle
// has no or two crossed edges; the crossed edges of one simplex are connected through its triangles).  The mesh of a
// box has no first cohomology, so the indicator of an isovolume -- two or no edges of every triangle -- is the
// coboundary of a vertex function that changes exactly across its edges.  Hence (1) the crossed edges between two
// vertex components belong to one isovolume (the function is constant on a component, so it differs on both or on
// none), (2) an isovolume joins one pair of components only (crossed edges of a triangle share a vertex, and their
// other ends are neighbours on one side), and (3) components and isovolumes form a tree.  Let v be the first vertex (in
// the global order) of a component other than that of vertex 0: its lower neighbours v - e(M) are all across the level
// and are neighbours of the lowest of them, so they lie in one component, whose first vertex is smaller.  The tree is
// rooted that way, and every isovolume is the one below exactly one component: of the two components that a crossed
// edge joins, the one whose first vertex is larger.  So an isovolume is named by that component, and there is one less
// of them than components.  The union-find runs on a few million runs instead of the crossed edges.
#include <utility>

#include "common.h"
#include "internal.h"
#include "kuhn.h"
#include "uf_cached.h"

namespace ftk {

namespace {


// chain corners of the 24 pentachoron types: corner k = s1 | ... | sk
struct PenCorners {
  unsigned char c[24][5];
};
constexpr PenCorners build_pen_corners() {
  PenCorners r{};
  for (int ty = 0; ty < 24; ++ty) {
    int acc = 0;
    r.c[ty][0] = 0;
    for (int k = 0; k < 4; ++k) {
      acc |= kPen3.m[ty][k];
      r.c[ty][k + 1] = (unsigned char)acc;
    }
  }
  return r;
}

struct IsoGrid {
  const float* f;
  int nx, ny, nz, nt;
  float c;
  const unsigned long long* bits;  // side of every vertex, one bit per vertex: row-major 64-vertex words
  int nwx;                         // words per row, ceil(nx / 64)
};

// Side of every vertex as one bit (a value equal to the isovalue counts as above), packed per 64 vertices of a row
// by a wave ballot: the passes that need the 16 corners of a 4-cube read these words (L2-resident, shared by
// neighbouring lanes) instead of 16 field values.  Non-finite values are reported here.
// Word k of the packed sides covers vertices 64 (k mod nwx) .. + 63 of grid row k / nwx (rows in (t, z, y) order).
// A wavefront packs kBitsWords consecutive words, their loads in flight together.
constexpr int kBitsWords = 4;
__global__ __launch_bounds__(256) void iso_bits(IsoGrid g, long long n_words, unsigned long long* __restrict__ bits,
                                                unsigned* __restrict__ status) {
  const int lane = threadIdx.x & 63;
  const long long k0 = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * kBitsWords;
  float v[kBitsWords];
  bool in[kBitsWords];
#pragma unroll
  for (int j = 0; j < kBitsWords; ++j) {
    const long long k = min(k0 + j, n_words - 1);
    const long long row = k / g.nwx;
    const int x = (int)(k - row * g.nwx) * 64 + lane;
    in[j] = k0 + j < n_words && x < g.nx;
    v[j] = g.f[row * g.nx + min(x, g.nx - 1)];
  }
  unsigned bad = 0;
#pragma unroll
  for (int j = 0; j < kBitsWords; ++j) {
    if (in[j] && !isfinite(v[j])) bad = ST_NONFINITE;
    const unsigned long long w = __ballot(in[j] && v[j] >= g.c);
    if (lane == 0 && k0 + j < n_words) bits[k0 + j] = w;
  }
  if (bad) atomicOr(status, bad);
}

typedef unsigned long long u64;

// Row of a word and which of its upper neighbours (y, z, t) are in the grid.
struct IsoRow {
  unsigned y, z, t;
  unsigned up;  // bit 0 y + 1, bit 1 z + 1, bit 2 t + 1
};
__device__ __forceinline__ IsoRow iso_row(const IsoGrid& g, unsigned r) {
  IsoRow q;
  q.y = r % (unsigned)g.ny;
  const unsigned zt = r / (unsigned)g.ny;
  q.z = zt % (unsigned)g.nz;
  q.t = zt / (unsigned)g.nz;
  q.up = (q.y + 1 < (unsigned)g.ny ? 1u : 0u) | (q.z + 1 < (unsigned)g.nz ? 2u : 0u) |
         (q.t + 1 < (unsigned)g.nt ? 4u : 0u);
  return q;
}
// Words from a row to the row at (dy, dz, dt) = the bits of m above it.
__device__ __forceinline__ long long row_step(const IsoGrid& g, int m) {
  return ((m & 1) + (((m >> 1) & 1) + (long long)((m >> 2) & 1) * g.nz) * g.ny) * (long long)g.nwx;
}
// Vertices of word column j inside the grid, and those with a neighbour at x + 1.
__device__ __forceinline__ u64 word_in(const IsoGrid& g, int j) {
  const int n = g.nx - 64 * j;
  return n >= 64 ? ~0ull : (1ull << n) - 1ull;
}
__device__ __forceinline__ u64 word_in_x1(const IsoGrid& g, int j) {
  const int n = g.nx - 64 * j - 1;
  return n >= 64 ? ~0ull : (n > 0 ? (1ull << n) - 1ull : 0ull);
}
// Positions where a run of equal sides starts, but the first.
__device__ __forceinline__ u64 run_starts(u64 w, u64 in) { return (w ^ (w << 1)) & in & ~1ull; }
__device__ __forceinline__ int run_at(u64 starts, int p) { return __popcll(starts & ((2ull << p) - 1ull)); }

// The sides of the 16 cube corners of a word's 64 vertices (corner mask x | y << 1 | z << 2 | t << 3) and which are in
// the grid.  One lane per word; the words of the row x and of the 7 rows above it.
struct IsoCorners {
  u64 s[16], in[16];
};
__device__ __forceinline__ void iso_corners(const IsoGrid& g, long long k, int j, unsigned up, IsoCorners& q) {
  u64 w[8], n[8];
  const bool more = j + 1 < g.nwx;
#pragma unroll
  for (int m = 0; m < 8; ++m) {  // rows past the grid: this row's words (dropped by in), all loads in flight together
    const long long a = k + ((m & ~(int)up) ? 0 : row_step(g, m));
    w[m] = g.bits[a];
    n[m] = g.bits[a + (more ? 1 : 0)];
  }
  const u64 in0 = word_in(g, j), in1 = word_in_x1(g, j);
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const bool ok = (m & ~(int)up) == 0;
    q.s[2 * m] = w[m];
    q.s[2 * m + 1] = (w[m] >> 1) | (more ? n[m] << 63 : 0ull);
    q.in[2 * m] = ok ? in0 : 0ull;
    q.in[2 * m + 1] = ok ? in1 : 0ull;
  }
}

// Tetrahedra of the isovolume in the pentachoron of type TY (Sec. 6.1): with k of its five chain vertices above the
// level, 1 for case I (k = 1 or 4), 3 for case II (k = 2 or 3), 0 otherwise; the chain corners are a compile-time
// mask, and the count per k is a nibble of 0x13310.
template <int TY>
__device__ __forceinline__ int pen_tets(unsigned above) {
  constexpr PenCorners kP = build_pen_corners();
  constexpr unsigned chain = 1u << kP.c[TY][0] | 1u << kP.c[TY][1] | 1u << kP.c[TY][2] | 1u << kP.c[TY][3] |
                             1u << kP.c[TY][4];
  return (int)((0x13310u >> (4u * (unsigned)__popc(above & chain))) & 15u);
}

template <int... TY>
__device__ __forceinline__ int pen_tets_all(std::integer_sequence<int, TY...>, unsigned above) {
  return (pen_tets<TY>(above) + ...);
}

// Tetrahedra of the pentachora of type TY of a word's vertices, added to n.
template <int TY>
__device__ __forceinline__ void pen_sum(const IsoCorners& q, const u64 (&s1)[16], const u64 (&c1)[16], u64 in, int& n) {
  constexpr PenCorners kP = build_pen_corners();
  // five sides added bit-sliced: s1, c1 hold those of corners 0, 15 and the first chain corner
  constexpr int a = kP.c[TY][1], b = kP.c[TY][2], c = kP.c[TY][3];
  const u64 s2 = s1[a] ^ q.s[b] ^ q.s[c];
  const u64 c2 = (s1[a] & q.s[b]) | (s1[a] & q.s[c]) | (q.s[b] & q.s[c]);
  const u64 two = (c1[a] ^ c2) & in;        // two or three above: case II
  const u64 one = (s2 ^ c1[a]) & ~two & in; // one or four above: case I
  n += __popcll(one) + 3 * __popcll(two);
}
template <int... TY>
__device__ __forceinline__ int pen_sum_all(std::integer_sequence<int, TY...>, const IsoCorners& q, u64 in) {
  u64 s1[16], c1[16];
#pragma unroll
  for (int a = 1; a < 16; a <<= 1) {
    s1[a] = q.s[0] ^ q.s[15] ^ q.s[a];
    c1[a] = (q.s[0] & q.s[15]) | (q.s[0] & q.s[a]) | (q.s[15] & q.s[a]);
  }
  int n = 0;
  (pen_sum<TY>(q, s1, c1, in, n), ...);
  return n;
}

// Counts per word, bit-parallel over its 64 vertices (bound by VALU issue).  Per vertex, with byte arrays whose group
// sums were scanned, the counts took 2.2 + 0.6 ms on 256^3 x 16; per word 0.13 + 0.13 ms.
__global__ __launch_bounds__(256) void iso_count(IsoGrid g, long long n_words, int* __restrict__ hcnt,
                                                 int* __restrict__ acnt, int* __restrict__ rcnt,
                                                 u64* __restrict__ n_tets) {
  __shared__ int s_tets;
  if (threadIdx.x == 0) s_tets = 0;
  __syncthreads();
  // a bounded grid: one addition to the common total per workgroup (they serialise)
  for (long long k = (long long)blockIdx.x * 256 + threadIdx.x; k < n_words; k += (long long)gridDim.x * 256) {
    const unsigned r = (unsigned)(k / g.nwx);
    const int j = (int)(k - (long long)r * g.nwx);
    IsoCorners q;
    iso_corners(g, k, j, iso_row(g, r).up, q);
    u64 any = q.s[0], all = ~0ull;
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      any |= q.s[c] & q.in[c];
      all &= q.s[c] | ~q.in[c];
    }
    int h = 0, a = 0;
    const u64 mixed = any & ~all & q.in[0];  // vertices with both sides among their corners
    if (mixed) {
#pragma unroll
      for (int c = 1; c < 16; ++c) h += __popcll((q.s[0] ^ q.s[c]) & q.in[c]);
      a = __popcll(mixed & q.in[15]);
      const int t = pen_sum_all(std::make_integer_sequence<int, 24>{}, q, q.in[15]);
      if (t) atomicAdd(&s_tets, t);
    }
    hcnt[k] = h;
    acnt[k] = a;
    rcnt[k] = 1 + __popcll(run_starts(q.s[0], q.in[0]));
  }
  __syncthreads();
  if (threadIdx.x == 0 && s_tets) atomicAdd(n_tets, (u64)s_tets);
}

// ---------------------------------------------------------------------------------------------------------------
// Components of the vertices on one side.  A node is a run of equal sides in a word, numbered in vertex order (rbase:
// first run of each word), so the root of a union-find tree, its smallest node, holds the component's first vertex.
// ---------------------------------------------------------------------------------------------------------------
// A run's parent: the run on its side before it along t, z, y or x that holds or precedes its first vertex, else
// itself (parents are smaller: a forest, flattened by uf_compress before the unions).
__global__ __launch_bounds__(256) void iso_runs_init(IsoGrid g, long long n_words, const long long* __restrict__ rbase,
                                                     unsigned* __restrict__ parent) {
  const long long k = (long long)blockIdx.x * 256 + threadIdx.x;
  if (k >= n_words) return;
  const unsigned r = (unsigned)(k / g.nwx);
  const int j = (int)(k - (long long)r * g.nwx);
  const IsoRow q = iso_row(g, r);
  const u64 in = word_in(g, j), w = g.bits[k];
  const long long at[3] = {q.t ? k - row_step(g, 4) : k, q.z ? k - row_step(g, 2) : k, q.y ? k - row_step(g, 1) : k};
  const bool ok[3] = {q.t != 0, q.z != 0, q.y != 0};
  u64 o[3];
  unsigned ob[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    o[a] = g.bits[at[a]];
    ob[a] = (unsigned)rbase[at[a]];
  }
  const unsigned b = (unsigned)rbase[k];
  const bool joins = j > 0 && ((g.bits[j > 0 ? k - 1 : k] >> 63) & 1ull) == (w & 1ull);
  u64 st = run_starts(w, in) | 1ull;
  for (unsigned n = b; st; ++n) {
    const int p = __ffsll((long long)st) - 1;
    st &= st - 1;
    unsigned par = p == 0 && joins ? b - 1u : n;
#pragma unroll
    for (int a = 2; a >= 0; --a)
      if (ok[a] && !(((o[a] ^ w) >> p) & 1ull)) par = ob[a] + (unsigned)run_at(run_starts(o[a], in), p);
    parent[n] = par;
  }
}

// The links between runs that the others do not imply.  The axes are taken in the order t, z, y, x.  Along t, z or y:
// one link per stretch of a word where both rows keep one side; along x: a word's last run and the next word's first.
// A link along a is implied, and left out, when at one of its vertices v the four vertices v, v + e(a), v + e(b),
// v + e(a) + e(b) are on one side for an earlier axis b (it then follows from the one at v + e(b) and the links along
// b).  Along t, the stretches that hold the first vertex of a run of the upper row are done by iso_runs_init.  Of several
// axes: only where every corner between is on the other side.  Inside the components nearly all links are implied, so
// what is left grows with the level set (256^3 x 16, 34 isovolumes: 0.6 ms with x first and no link from the
// initialisation counted, 0.20 now).
__global__ __launch_bounds__(256) void iso_runs_link(IsoGrid g, long long n_words, const long long* __restrict__ rbase,
                                                     unsigned* __restrict__ parent) {
  const long long k = (long long)blockIdx.x * 256 + threadIdx.x;
  if (k >= n_words) return;
  const unsigned r = (unsigned)(k / g.nwx);
  const int j = (int)(k - (long long)r * g.nwx);
  const unsigned up = iso_row(g, r).up;
  IsoCorners q;
  iso_corners(g, k, j, up, q);
  const bool more = j + 1 < g.nwx;
  const u64 w = q.s[0], in = q.in[0], st = run_starts(w, in);
  const unsigned b = (unsigned)rbase[k];
  if (more && !(((q.s[1] ^ w) >> 63) & 1ull)) {
    u64 implied = 0;
#pragma unroll
    for (int c = 1; c < 8; c <<= 1)
      if (up & (unsigned)c) implied |= ~(w ^ q.s[2 * c]) & ~(w ^ q.s[2 * c + 1]);
    if (!(implied >> 63)) {
      const unsigned nb = (unsigned)rbase[k + 1];
      uf_unite_cached(parent, nb - 1u, nb);
    }
  }
#pragma unroll
  for (int a = 4; a >= 1; a >>= 1) {  // row masks t, z, y
    if (!(up & (unsigned)a)) continue;
    const u64 same = ~(w ^ q.s[2 * a]) & in;
    u64 implied = 0;
    if (a == 4) implied = run_starts(q.s[8], in) | 1ull;
#pragma unroll
    for (int c = 4; c > a; c >>= 1)
      if (up & (unsigned)c) implied |= same & ~(w ^ q.s[2 * c]) & ~(w ^ q.s[2 * (a | c)]);
    u64 left = same;
    while (left) {
      const int p = __ffsll((long long)left) - 1;
      // the stretch from p: up to the next vertex off it or the next run
      const u64 stop = (~same | st) & ~((2ull << p) - 1ull);
      const u64 upto = stop ? (stop & (0ull - stop)) - 1ull : ~0ull;
      const u64 part = left & upto;
      left &= ~upto;
      if (part & implied) continue;
      const long long o = k + row_step(g, a);
      uf_unite_cached(parent, b + (unsigned)run_at(st, p),
                      (unsigned)rbase[o] + (unsigned)run_at(run_starts(q.s[2 * a], in), p));
    }
  }
#pragma unroll
  for (int M = 3; M < 16; ++M) {
    if ((M & (M - 1)) == 0) continue;
    u64 need = ~(w ^ q.s[M]) & q.in[M];
#pragma unroll
    for (int m = 1; m < M; ++m)
      if ((m & M) == m) need &= w ^ q.s[m];
    while (need) {
      const int p = __ffsll((long long)need) - 1;
      need &= need - 1;
      const int x = p + (M & 1);
      const long long o = k + row_step(g, M >> 1) + (x >> 6);
      const u64 ow = g.bits[o];
      uf_unite_cached(parent, b + (unsigned)run_at(st, p),
                      (unsigned)rbase[o] + (unsigned)run_at(run_starts(ow, word_in(g, j + (x >> 6))), x & 63));
    }
  }
}

// Every run's component (its root), the number of components, and the components' smallest edge ids cleared.
__global__ __launch_bounds__(256) void iso_runs_done(const unsigned* __restrict__ parent, long long n,
                                                     unsigned* __restrict__ comp, long long* __restrict__ first,
                                                     u64* __restrict__ roots) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  unsigned root = 0;
  if (i < n) {
    root = uf_find_plain(parent, (unsigned)i);
    comp[i] = root;
    first[i] = 0x7fffffffffffffffll;
  }
  const u64 b = __ballot(i < n && root == (unsigned)i);
  if (b && lane_id() == 0) atomicAdd(roots, (u64)__popcll(b));
}

// ---------------------------------------------------------------------------------------------------------------
// Emission.  A wavefront looks at the counts of kIsoEmitWords words and takes those with crossings one after another: lane =
// vertex for the crossing masks, offsets and cubes, then lane = crossing, so that ids, points and components go out in
// contiguous stores.  Bound by issue (about 340 vector and 280 scalar operations a word, 1.9 ms for the 1.6 M words with
// crossings of the 256^3 x 16 series; 16 or 32 words a wavefront: 2.0).
// ---------------------------------------------------------------------------------------------------------------
constexpr int kIsoEmitWords = 64;
struct IsoWave {
  unsigned short map[15 * 64];  // crossing j of the word -> vertex lane | mask << 6
  u64 starts[16];               // run starts and first run of the word's row and the 7 rows above it, at this word
  unsigned run[16];             // column and the next
};

__device__ __forceinline__ u64 lane_word(u64 v, int l) {
  return (u64)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, l) |
         (u64)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), l) << 32;
}

__global__ __launch_bounds__(256) void iso_emit(IsoGrid g, long long n_words, const int* __restrict__ hcnt,
                                                const long long* __restrict__ hbase,
                                                const long long* __restrict__ abase, const long long* __restrict__ rbase,
                                                const unsigned* __restrict__ comp, unsigned* __restrict__ vinfo,
                                                long long* __restrict__ edge_id, float* __restrict__ pos,
                                                unsigned* __restrict__ hcomp, long long* __restrict__ first,
                                                long long* __restrict__ list) {
  __shared__ IsoWave sw[4];
  __shared__ long long step[16];  // from a vertex to its corner M
  if (threadIdx.x < 16) {
    const long long M = threadIdx.x;
    step[M] = (M & 1) + ((M >> 1) & 1) * (long long)g.nx +
              (((M >> 2) & 1) + (M >> 3) * g.nz) * (long long)g.nx * (long long)g.ny;
  }
  __syncthreads();
  IsoWave& W = sw[threadIdx.x >> 6];
  const int lane = lane_id();
  const long long k0 = ((long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6))) * kIsoEmitWords;
  if (k0 >= n_words) return;
  // lane l: word k0 + l
  const long long kl = min(k0 + min(lane, kIsoEmitWords - 1), n_words - 1);
  const int hc = lane < kIsoEmitWords && k0 + lane < n_words ? hcnt[kl] : 0;
  const long long hb = hbase[kl], ab = abase[kl];
  const unsigned rl = (unsigned)(kl / g.nwx);
  const int jl = (int)(kl - (long long)rl * g.nwx);
  const IsoRow ql = iso_row(g, rl);
  const long long sx = g.nx, sxy = sx * g.ny, sxyz = sxy * g.nz;
  u64 todo = __ballot(hc > 0);
  if (!todo) return;
  // the 16 words around word e: lane 2 m + c = row m, column j + c, four lanes each for the components of their first
  // four runs (the sides of a word's runs alternate)
  auto around = [&](int e, u64& w, unsigned& rn) -> bool {
    const int j = __builtin_amdgcn_readlane(jl, e);
    const unsigned up = (unsigned)__builtin_amdgcn_readlane((int)ql.up, e);
    const int m = (lane >> 1) & 7, c = lane & 1;
    const bool inside = (m & ~(int)up) == 0 && (c == 0 || j + 1 < g.nwx);
    const long long a = k0 + e + (inside ? row_step(g, m) + c : 0);
    w = g.bits[a];
    rn = (unsigned)rbase[a];
    return inside;
  };
  u64 wl;
  unsigned rn;
  int e = __ffsll((long long)todo) - 1;
  bool inside = around(e, wl, rn);
  for (;;) {
    todo &= todo - 1;
    const int j = __builtin_amdgcn_readlane(jl, e), total = __builtin_amdgcn_readlane(hc, e);
    const unsigned up = (unsigned)__builtin_amdgcn_readlane((int)ql.up, e);
    const unsigned y = (unsigned)__builtin_amdgcn_readlane((int)ql.y, e), z = (unsigned)__builtin_amdgcn_readlane((int)ql.z, e);
    const unsigned t = (unsigned)__builtin_amdgcn_readlane((int)ql.t, e);
    const long long h0 = (long long)lane_word((u64)hb, e), a0 = (long long)lane_word((u64)ab, e);
    const u64 starts = run_starts(wl, word_in(g, j + (inside ? lane & 1 : 0)));
    const int runs = 1 + __popcll(starts), run = min(lane >> 4, runs - 1);
    const unsigned rcomp = comp[rn + (unsigned)run];
    // one component on each side among all of them: every crossing of the word is of one isovolume
    const bool over = (((unsigned)wl ^ (unsigned)run) & 1u) != 0;
    const u64 bo = __ballot(over), bu = __ballot(!over);
    const unsigned co = (unsigned)__builtin_amdgcn_readlane((int)rcomp, bo ? __ffsll((long long)bo) - 1 : 0);
    const unsigned cu = (unsigned)__builtin_amdgcn_readlane((int)rcomp, bu ? __ffsll((long long)bu) - 1 : 0);
    const bool single = __ballot(runs > 4 || rcomp != (over ? co : cu)) == 0;
    const u64 wz = inside ? wl : 0ull;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the previous word's reads of W are done
    __builtin_amdgcn_wave_barrier();
    if (lane < 16) {
      W.starts[lane] = starts;
      W.run[lane] = rn;
    }
    u64 s[16], valid[16];
    const u64 in0 = word_in(g, j), in1 = word_in_x1(g, j);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const bool ok = (m & ~(int)up) == 0;
      const u64 w = lane_word(wz, 2 * m);
      s[2 * m] = w;
      s[2 * m + 1] = (w >> 1) | (lane_word(wz, 2 * m + 1) << 63);
      valid[2 * m] = ok ? in0 : 0ull;
      valid[2 * m + 1] = ok ? in1 : 0ull;
    }
    unsigned m = 0;
    u64 any = s[0], all = s[0];
#pragma unroll
    for (int M = 1; M < 16; ++M) {
      any |= s[M];
      all &= s[M];
      m |= __builtin_amdgcn_inverse_ballot_w64((s[0] ^ s[M]) & valid[M]) ? 1u << (M - 1) : 0u;
    }
    const unsigned n = __popc(m);
    unsigned at = wave_incl_scan(n) - n;
    const long long v0 = ((long long)t * sxyz + (long long)z * sxy + (long long)y * sx) + 64ll * j;
    const unsigned info = at | m << 16;
    for (unsigned mm = m; mm; mm &= mm - 1u) W.map[at++] = (unsigned short)((unsigned)lane | (unsigned)__ffs((int)mm) << 6);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // Loads before stores: a load issued after a store waits for it too.  First this word's field values (for its first
    // 64 crossings), then the next word's words, then the stores.
    const float* F = g.f + v0;
    const int i_last = total - 1;
    unsigned ent = W.map[min(lane, i_last)];
    float f0 = F[ent & 63u], f1 = F[(ent & 63u) + step[ent >> 6]];
    const unsigned rc1 = max(co, cu);
    const long long seen = first[rc1];
    const int next = todo ? __ffsll((long long)todo) - 1 : e;
    inside = around(next, wl, rn);
    if (64 * j + lane < g.nx) vinfo[v0 + lane] = info;
    // cubes with tetrahedra: vertex and the sides of its corners (a corner's side differs where its edge is crossed)
    const u64 act = any & ~all & valid[15];
    if (__builtin_amdgcn_inverse_ballot_w64(act)) {
      const unsigned above = (m << 1) ^ (__builtin_amdgcn_inverse_ballot_w64(s[0]) ? 0xFFFFu : 0u);
      const long long a = a0 + __builtin_amdgcn_mbcnt_hi((unsigned)(act >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)act, 0u));
      list[a] = (long long)((u64)(v0 + lane) | (u64)above << 48);
    }
    const long long id0 = v0 * 15 - 1;
    const float fx = (float)(64 * j), fy = (float)(int)y, fz = (float)(int)z, ft = (float)(int)t;
    for (int i = lane;;) {
      const bool on = i < total;
      const int L = (int)(ent & 63u), M = (int)(ent >> 6);
      const int dx = M & 1, dy = (M >> 1) & 1, dz = (M >> 2) & 1, dt = M >> 3;
      const float mu = (g.c - f0) / (f1 - f0);
      const long long id = id0 + (L * 15 + M);
      unsigned rc = rc1;
      bool own = i == 0 && id < seen;
      if (!single) {
        const int x1 = L + dx, o = (M & ~1) | (x1 >> 6);
        rc = max(comp[W.run[0] + (unsigned)run_at(W.starts[0], L)],
                 comp[W.run[o] + (unsigned)run_at(W.starts[o], x1 & 63)]);
        // ids ascend with the lane: lane 0 stands for the wavefront's leading component
        const unsigned lead = (unsigned)__builtin_amdgcn_readfirstlane((int)rc);
        own = on && (rc != lead || lane == 0) && id < first[rc];
      }
      if (on) {
        edge_id[h0 + i] = id;
        if (pos)
          reinterpret_cast<float4*>(pos)[h0 + i] = make_float4((fx + (float)L) + mu * (float)dx, fy + mu * (float)dy,
                                                               fz + mu * (float)dz, ft + mu * (float)dt);
        hcomp[h0 + i] = rc;
        if (own) atomicMin(first + rc, id);
      }
      i += 64;
      if (i - lane >= total) break;
      ent = W.map[min(i, i_last)];
      f0 = F[ent & 63u];
      f1 = F[(ent & 63u) + step[ent >> 6]];
    }
    if (!todo) break;
    e = next;
  }
}

// Tessellation (Sec. 6.1).  In a pentachoron with k of its five chain vertices above the level, case I (one vertex on
// the smaller side) gives the tetrahedron of its four crossed edges, case II (two) the three tetrahedra of the prism
// between their crossed edges.  A wavefront takes 64 listed cubes: lane = cube for the corners' first hits and crossing
// masks and for listing its crossed pentachora, then lane = pentachoron, whose tetrahedra follow those of the lane
// before: they are staged in LDS and go out as contiguous 16-byte stores.  (One lane per cube with the 24 types unrolled
// ran every type for every wavefront and scattered each store over 64 lines: 2.86 against 1.52 ms on 256^3 x 16, 299 M
// tetrahedra, whose 4.8 GB are the bound; stored straight from the pentachoron lanes, 16 bytes each 48: 2.58 ms.)
struct IsoTess {
  uint2 corner[16][65];           // by corner, cube (padded: the lanes of a cube read different corners): first hit, mask
  unsigned short pen[24 * 64];    // crossed pentachora in output order: cube | type << 6
  int4 out[3 * 64];               // tetrahedra of 64 of them
};
// Chain corners of the 24 types as 4-bit fields, and for each set of chain positions above the level the positions on
// the smaller side (first, second) and the others, each in increasing order, as 3-bit fields.
struct IsoPenTables {
  unsigned chain[24], split[32];
};
constexpr IsoPenTables build_pen_tables() {
  IsoPenTables r{};
  const PenCorners c = build_pen_corners();
  for (int ty = 0; ty < 24; ++ty)
    for (int k = 0; k < 5; ++k) r.chain[ty] |= (unsigned)c.c[ty][k] << (4 * k);
  for (unsigned lm = 0; lm < 32; ++lm) {
    const unsigned mino = popc_c((int)lm) <= 2 ? lm : (~lm & 31u);
    unsigned a = 0, b = 2;  // fields 0, 1: smaller side; 2..5: the others
    for (unsigned p = 0; p < 5; ++p) {
      const unsigned f = (mino >> p) & 1u ? a++ : b++;
      if (f < 6) r.split[lm] |= p << (3 * f);
    }
    r.split[lm] |= (popc_c((int)mino) == 2 ? 1u : 0u) << 18;
  }
  return r;
}
__constant__ IsoPenTables kIsoPenTables = build_pen_tables();

// Crossed pentachora of a cube with sides `above`: types mixed, and the types of case II.
template <int... TY>
__device__ __forceinline__ void pen_sets(std::integer_sequence<int, TY...>, unsigned above, unsigned& mixed,
                                         unsigned& two) {
  auto one = [&](int ty, int tets) {
    mixed |= tets ? 1u << ty : 0u;
    two |= tets == 3 ? 1u << ty : 0u;
  };
  (one(TY, pen_tets<TY>(above)), ...);
}

// Tetrahedra of every 64 listed cubes (one workgroup of iso_tess).
__global__ __launch_bounds__(256) void iso_tess_count(const long long* __restrict__ list, long long n_list,
                                                      int* __restrict__ cnt) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  unsigned n = 0;
  if (i < n_list) n = (unsigned)pen_tets_all(std::make_integer_sequence<int, 24>{}, (unsigned)((u64)list[i] >> 48));
  n = wave_sum(n);
  if (lane_id() == 0 && i < n_list) cnt[i >> 6] = (int)n;
}

__global__ __launch_bounds__(64) void iso_tess(IsoGrid g, const long long* __restrict__ list,
                                               const long long* __restrict__ tbase, long long n_list,
                                               const unsigned* __restrict__ vinfo, const long long* __restrict__ hbase,
                                               int* __restrict__ tets) {
  __shared__ IsoTess W;
  __shared__ IsoPenTables tab;
  const int lane = threadIdx.x;
  if (lane < 24) tab.chain[lane] = kIsoPenTables.chain[lane];
  if (lane < 32) tab.split[lane] = kIsoPenTables.split[lane];
  const long long i0 = (long long)blockIdx.x * 64;
  const bool on = i0 + lane < n_list;
  const u64 ent = (u64)list[min(i0 + lane, n_list - 1)];
  const unsigned above = (unsigned)(ent >> 48);
  const long long v = (long long)(ent & 0xFFFFFFFFFFFFull);
  const long long row = v / g.nx;
  const int x = (int)(v - row * g.nx);
  // first hit and crossing mask of the cube's corners; a corner in a word without crossings anchors none, and what is
  // read for it is not used
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const long long r = row + ((m & 1) + (((m >> 1) & 1) + (long long)((m >> 2) & 1) * g.nz) * g.ny);
    const unsigned v0 = vinfo[r * g.nx + x], v1 = vinfo[r * g.nx + x + 1];
    const long long b0 = hbase[r * g.nwx + (x >> 6)], b1 = hbase[r * g.nwx + ((x + 1) >> 6)];
    W.corner[2 * m][lane] = make_uint2((unsigned)b0 + (v0 & 0xFFFFu), v0 >> 16);
    W.corner[2 * m + 1][lane] = make_uint2((unsigned)b1 + (v1 & 0xFFFFu), v1 >> 16);
  }
  unsigned mixed = 0, two = 0;
  pen_sets(std::make_integer_sequence<int, 24>{}, above, mixed, two);
  if (!on) mixed = 0;
  const unsigned incl = wave_incl_scan((unsigned)__popc(mixed));
  const int n_pen = __builtin_amdgcn_readlane((int)incl, 63);
  unsigned at = incl - (unsigned)__popc(mixed);
  for (unsigned m = mixed; m; m &= m - 1u) W.pen[at++] = (unsigned short)((unsigned)lane | ((unsigned)__ffs((int)m) - 1u) << 6);
  __syncthreads();
  int4* T = reinterpret_cast<int4*>(tets) + tbase[blockIdx.x];
  for (int p0 = 0; p0 < n_pen; p0 += 64) {
    const int p = p0 + lane;
    const unsigned pen = W.pen[min(p, n_pen - 1)];
    const unsigned c = pen & 63u, chain = tab.chain[pen >> 6];
    const unsigned side = (unsigned)__builtin_amdgcn_ds_bpermute((int)(c << 2), (int)above);
    unsigned lm = 0;
#pragma unroll
    for (int k = 0; k < 5; ++k) lm |= ((side >> ((chain >> (4 * k)) & 15u)) & 1u) << k;
    const unsigned sp = tab.split[lm];
    // hit index of the crossed edge between the chain positions in fields f and h
    auto edge = [&](int f, int h) -> int {
      const unsigned a = (sp >> (3 * f)) & 7u, b = (sp >> (3 * h)) & 7u;
      const unsigned ca = (chain >> (4u * min(a, b))) & 15u, M = ((chain >> (4u * max(a, b))) & 15u) ^ ca;
      const uint2 q = W.corner[ca][c];
      return (int)q.x + __popc(q.y & ((1u << (M - 1u)) - 1u));
    };
    const bool prism = (sp >> 18) & 1u;
    const unsigned mine = p < n_pen ? (prism ? 3u : 1u) : 0u, upto = wave_incl_scan(mine);
    // case I: the lone vertex with the others in chain order; case II: (p1, a0..a2), (p2, a0..a2)
    const int e0 = edge(0, 2), e1 = edge(0, 3), e2 = edge(0, 4);
    int4* const o = W.out + (upto - mine);
    if (mine == 1u) {
      o[0] = make_int4(e0, e1, e2, edge(0, 5));
    } else if (mine == 3u) {
      const int e3 = edge(1, 2), e4 = edge(1, 3), e5 = edge(1, 4);
      o[0] = make_int4(e0, e1, e2, e5);
      o[1] = make_int4(e0, e1, e4, e5);
      o[2] = make_int4(e0, e3, e4, e5);
    }
    __syncthreads();
    const int n = __builtin_amdgcn_readlane((int)upto, 63);
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (lane + 64 * q < n) T[lane + 64 * q] = W.out[lane + 64 * q];
    T += n;
    __syncthreads();  // the next 64 overwrite the staged ones
  }
}

__global__ __launch_bounds__(256) void iso_label(const unsigned* __restrict__ hcomp, const long long* __restrict__ first,
                                                 long long n, long long* __restrict__ label) {
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += (long long)gridDim.x * 256)
    label[i] = first[hcomp[i]];
}

unsigned blocks_of(long long n) { return (unsigned)((n + 255) / 256); }

}  // namespace

hipError_t launch_iso_count(const float* f, int nx, int ny, int nz, int nt, float c, unsigned long long* bits,
                            int* hcnt, int* acnt, int* rcnt, unsigned long long* n_tets, unsigned* status,
                            hipStream_t s) {
  const IsoGrid g{f, nx, ny, nz, nt, c, bits, (nx + 63) / 64};
  const long long n_words = (long long)nt * nz * ny * g.nwx;
  iso_bits<<<(unsigned)((n_words + 4 * kBitsWords - 1) / (4 * kBitsWords)), 256, 0, s>>>(g, n_words, bits, status);
  iso_count<<<blocks_of(n_words) < 2048u ? blocks_of(n_words) : 2048u, 256, 0, s>>>(g, n_words, hcnt, acnt, rcnt, n_tets);
  return hipGetLastError();
}

hipError_t launch_iso_components(int nx, int ny, int nz, int nt, const unsigned long long* bits,
                                 const long long* rbase, long long n_runs, unsigned* parent, unsigned* comp,
                                 long long* first, unsigned long long* n_comp, hipStream_t s) {
  const IsoGrid g{nullptr, nx, ny, nz, nt, 0.0f, bits, (nx + 63) / 64};
  const long long n_words = (long long)nt * nz * ny * g.nwx;
  iso_runs_init<<<blocks_of(n_words), 256, 0, s>>>(g, n_words, rbase, parent);
  const hipError_t e = launch_uf_compress(parent, n_runs, s);
  if (e != hipSuccess) return e;
  iso_runs_link<<<blocks_of(n_words), 256, 0, s>>>(g, n_words, rbase, parent);
  iso_runs_done<<<blocks_of(n_runs), 256, 0, s>>>(parent, n_runs, comp, first, n_comp);
  return hipGetLastError();
}

hipError_t launch_iso_emit(const float* f, int nx, int ny, int nz, int nt, float c, const unsigned long long* bits,
                           const int* hcnt, const long long* hbase, const long long* abase, const long long* rbase,
                           const unsigned* comp, long long n_hits, long long n_active, unsigned* vinfo,
                           long long* edge_id, float* pos, unsigned* hcomp, long long* first, long long* list,
                           int* tcnt, long long* tbase, long long* scan_tmp, int* tets, long long* label,
                           hipStream_t s) {
  const IsoGrid g{f, nx, ny, nz, nt, c, bits, (nx + 63) / 64};
  const long long n_words = (long long)nt * nz * ny * g.nwx;
  iso_emit<<<(unsigned)((n_words + 4 * kIsoEmitWords - 1) / (4 * kIsoEmitWords)), 256, 0, s>>>(
      g, n_words, hcnt, hbase, abase, rbase, comp, vinfo, edge_id, pos, hcomp, first, list);
  if (n_active > 0) {
    const long long groups = (n_active + 63) / 64;
    iso_tess_count<<<blocks_of(n_active), 256, 0, s>>>(list, n_active, tcnt);
    const hipError_t e = launch_scan(tcnt, tbase, groups, tbase + groups, scan_tmp, s);
    if (e != hipSuccess) return e;
    iso_tess<<<(unsigned)groups, 64, 0, s>>>(g, list, tbase, n_active, vinfo, hbase, tets);
  }
  const unsigned lb = blocks_of(n_hits);
  iso_label<<<lb < 8192u ? lb : 8192u, 256, 0, s>>>(hcomp, first, n_hits, label);
  return hipGetLastError();
}

}  // namespace ftk
