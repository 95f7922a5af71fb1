// vortex.hip -- quantum vortex surface tracking in 3D complex series (Sec. 5.1, two passes on the regular
// simplicial spacetime mesh; Alg. 1 middle column).
//
// The contour integral of the phase around a spacetime triangle, each edge's phase change wrapped into (-pi, pi],
// is 2 pi times the winding number of the image triangle (psi_0, psi_1, psi_2) around 0 (a straight segment that
// misses 0 turns by exactly the wrapped change).  So a triangle is positive when 0 lies inside its image: the
// puncture test of the 2-component field (Re psi, Im psi), decided exactly on quantised values with the symbolic
// perturbation (Sec. 4.3).  Its three cofactor signs are the SoS signs of the 2x2 determinants of the vertex pairs,
// i.e. of the triangle's edges, so one sign bit per spacetime edge is computed once and shared.
//
//   vx_edges -- one lane per vertex: SoS sign of det(q(p), q(p + e(M))) for the 15 edge masks M (bits x = 1, y = 2,
//               z = 4, t = 8), q = rint(psi * 2^s).
//   vx_tris  -- the 50 triangle types (M1, M2) anchored at each vertex (vertices p, p + e(a), p + e(b), a = M1,
//               b = M1 | M2): signs S01, S02 from the vertex's own edges, S12 from the edge (b ^ a) of p + e(a);
//               positive iff S12 == S01 and S02 != S01 (cofactor signs +S12, -S02, +S01 agree).  Counts per word of 64
//               vertices of a row and, per vertex, the triangles before it in its word.
//   vx_emit  -- triangle ids g * 50 + type, the vortex point from the exact cofactors (Eq. 2), and a parent with a
//               smaller index.
//   vx_link  -- the remaining links united.
// Links.  Under the perturbation every tetrahedron has no or two positive sides.  The positive sides of a pentachoron
// form one cycle through its tetrahedra (each lies in two of them), so uniting the two of every tetrahedron connects
// the positive sides of every pentachoron, which is what Sec. 5.1 asks for.  A tetrahedron (c; c1, c2, c3) has the sides
// (c + e(c1); c2, c3), (c; c1|c2, c3), (c; c1, c2|c3), (c; c1, c2): each link is found from its larger end, whose
// smaller partner lies at an anchor p - e(c1) (exactly one positive side among three) or at p itself with a smaller type
// (M1 split in two, or M2).
// Labels (smallest triangle id of each surface) come from the shared union-find passes.
#include "common.h"
#include "internal.h"
#include "kuhn.h"
#include "uf_cached.h"

namespace ftk {

namespace {

constexpr int kVxBX = 128;  // lanes per block along x: two words

typedef unsigned long long u64;

struct VxGrid {
  const float* psi;  // [nt][2][nz][ny][nx]
  int nx, ny, nz, nt;
  int nwx;           // words per row, ceil(nx / 64)
  float qscale;
};

__device__ __forceinline__ long long vx_vidx(const VxGrid& g, int x, int y, int z, int t) {
  return (((long long)t * g.nz + z) * g.ny + y) * g.nx + x;
}

// quantised component; flags non-finite and out-of-range values
__device__ __forceinline__ float vx_q(float f, float qscale, unsigned& st) {
  const float v = f * qscale;
  if (fabsf(v) < 2147483648.0f) return rintf(v);
  st |= isfinite(v) ? ST_RANGE : ST_NONFINITE;
  return 0.0f;
}

// Bit M - 1: the corner p + e(M) is in the grid.
__device__ __forceinline__ unsigned vx_corners(const VxGrid& g, int x, int y, int z, int t) {
  const unsigned no = (x + 1 < g.nx ? 0u : 1u) | (y + 1 < g.ny ? 0u : 2u) | (z + 1 < g.nz ? 0u : 4u) |
                      (t + 1 < g.nt ? 0u : 8u);
  // the masks that use axis x, y, z, t, as bits M - 1
  return 0x7FFFu & ~((no & 1u ? 0x5555u : 0u) | (no & 2u ? 0x6666u : 0u) | (no & 4u ? 0x7878u : 0u) |
                     (no & 8u ? 0x7F80u : 0u));
}

// One lane per vertex of a row; the x + 1 corners are the next lane's values (the column past the wavefront in one load
// for all rows and components).  Bound by the loads: 512 x 128 x 64 x 8, 0.74 -> 0.39 ms against 30 gathered values and
// 64-bit integer determinants per vertex.
__global__ __launch_bounds__(kVxBX) void vx_edges(VxGrid g, unsigned short* __restrict__ emask,
                                                   unsigned* __restrict__ status) {
  const int lane = threadIdx.x & 63;
  const int xw = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kVxBX + (threadIdx.x & ~63u)));
  if (xw >= g.nx) return;
  const int x = xw + lane, xc = min(x, g.nx - 1);
  const int y = blockIdx.y, z = blockIdx.z % g.nz, t = blockIdx.z / g.nz;
  const long long plane = (long long)g.nx * g.ny * g.nz;
  auto row = [&](int m, int c) -> long long {  // row (y, z, t) + the bits of m, clamped to the grid, component c
    const int cy = min(y + (m & 1), g.ny - 1), cz = min(z + ((m >> 1) & 1), g.nz - 1), ct = min(t + (m >> 2), g.nt - 1);
    return ((long long)ct * 2 + c) * plane + ((long long)cz * g.ny + cy) * g.nx;
  };
  float f[8][2];
#pragma unroll
  for (int m = 0; m < 8; ++m)
#pragma unroll
    for (int c = 0; c < 2; ++c) f[m][c] = g.psi[row(m, c) + xc];
  const float past = g.psi[row((lane >> 1) & 7, lane & 1) + min(xw + 64, g.nx - 1)];
  unsigned st = 0, st1 = 0;
  const float qp = vx_q(past, g.qscale, st1);
  float q[8][2];
#pragma unroll
  for (int m = 0; m < 8; ++m)
#pragma unroll
    for (int c = 0; c < 2; ++c) q[m][c] = vx_q(f[m][c], g.qscale, m == 0 ? st : st1);  // own values are reported
  const double a0 = q[0][0], a1 = q[0][1];
  unsigned neg = 0, zero = 0;
#pragma unroll
  for (int M = 1; M < 16; ++M) {
    const int m = M >> 1;
    const float b0f = (M & 1) ? from_next(q[m][0], lane_value(qp, 2 * m)) : q[m][0];
    const float b1f = (M & 1) ? from_next(q[m][1], lane_value(qp, 2 * m + 1)) : q[m][1];
    const double b0 = b0f, b1 = b1f;
    const double d = edge_det(a0, a1, b0, b1);
    neg |= (unsigned)edge_neg(d) & (1u << (M - 1));
    zero |= d == 0.0 ? 1u << (M - 1) : 0u;
  }
  if (__ballot(zero != 0u)) {
#pragma unroll
    for (int M = 1; M < 16; ++M) {
      const int m = M >> 1;
      const float b0f = (M & 1) ? from_next(q[m][0], lane_value(qp, 2 * m)) : q[m][0];
      const float b1f = (M & 1) ? from_next(q[m][1], lane_value(qp, 2 * m + 1)) : q[m][1];
      const unsigned tie = (unsigned)edge_tie(a1, b0f, b1f) & (1u << (M - 1));
      if ((zero >> (M - 1)) & 1u) neg = (neg & ~(1u << (M - 1))) | tie;
    }
  }
  if (x < g.nx) emask[vx_vidx(g, x, y, z, t)] = (unsigned short)(~neg & vx_corners(g, x, y, z, t));
  if (st && x < g.nx) atomicOr(status, st);
}

// The bits of w at the set bits of MASK, packed from bit K on.
template <unsigned MASK, int K = 0>
__device__ __forceinline__ unsigned packed(unsigned w) {
  if constexpr (MASK == 0) {
    return 0u;
  } else {
    constexpr int s = __builtin_ctz(MASK), n = __builtin_ctz(~(MASK >> s));
    constexpr unsigned run = ((1u << n) - 1u) << s;
    const unsigned at = s >= K ? w >> (s - K) : w << (K - s);
    return (at & (((1u << n) - 1u) << K)) | packed<(MASK & ~run), K + n>(w);
  }
}
constexpr unsigned disjoint_masks(int a) {  // bits M - 1 of the masks M disjoint from a
  unsigned r = 0;
  for (int M = 1; M < 16; ++M)
    if (!(M & a)) r |= 1u << (M - 1);
  return r;
}
constexpr int first_type(int a) {  // types with M1 < a
  int n = 0;
  for (int k = 0; k < 50; ++k) n += kTri3.m[k][0] < a;
  return n;
}
// Positive triangles with M1 = A and above, in type order: the types with one M1 are consecutive, by M2.  With the edge
// words e0 of the anchor and ea[A] of p + e(A), the three signs of (A, M2) are bit M2 - 1 of S01 (one bit, repeated),
// of e0 >> A (the edge A|M2 = A + M2) and of ea[A].
template <int A>
__device__ __forceinline__ u64 vx_positive(unsigned e0, const unsigned (&ea)[16], unsigned ok) {
  if constexpr (A >= 15) {
    return 0ull;
  } else {
    const unsigned s01 = 0u - ((e0 >> (A - 1)) & 1u);
    const unsigned w = ~(ea[A] ^ s01) & ((e0 >> A) ^ s01) & (ok >> A);
    return (u64)packed<disjoint_masks(A)>(w) << first_type(A) | vx_positive<A + 1>(e0, ea, ok);
  }
}

__global__ __launch_bounds__(kVxBX) void vx_tris(VxGrid g, const unsigned short* __restrict__ emask,
                                                  u64* __restrict__ tmask, unsigned short* __restrict__ before,
                                                  int* __restrict__ wcnt) {
  const int lane = threadIdx.x & 63;
  const int xw = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kVxBX + (threadIdx.x & ~63u)));
  if (xw >= g.nx) return;
  const int x = xw + lane, xc = min(x, g.nx - 1);
  const int y = blockIdx.y, z = blockIdx.z % g.nz, t = blockIdx.z / g.nz;
  auto row = [&](int m) -> long long {
    return vx_vidx(g, 0, min(y + (m & 1), g.ny - 1), min(z + ((m >> 1) & 1), g.nz - 1), min(t + (m >> 2), g.nt - 1));
  };
  // edge words of the corners; one outside the grid is not used (a triangle is tested only when its corner b, a superset
  // of a, is inside)
  unsigned ea[16];
#pragma unroll
  for (int m = 0; m < 8; ++m) ea[2 * m] = emask[row(m) + xc];
  const unsigned past = emask[row(lane & 7) + min(xw + 64, g.nx - 1)];
#pragma unroll
  for (int m = 0; m < 8; ++m) ea[2 * m + 1] = from_next(ea[2 * m], (unsigned)__builtin_amdgcn_readlane((int)past, m));
  const u64 m = x < g.nx ? vx_positive<1>(ea[0], ea, vx_corners(g, x, y, z, t)) : 0ull;
  const unsigned n = (unsigned)__popcll(m), incl = wave_incl_scan(n);
  if (x < g.nx) {
    const long long v = vx_vidx(g, x, y, z, t);
    tmask[v] = m;
    before[v] = (unsigned short)(incl - n);
  }
  if (lane == 63) wcnt[(((long long)t * g.nz + z) * g.ny + y) * g.nwx + (xw >> 6)] = (int)incl;
}

// Type tables for lane-dependent types, copied to LDS.
struct VxTables {
  unsigned char masks[50];      // M1 | M2 << 4
  unsigned char type[16 * 16];  // type of (M1, M2)
};
constexpr VxTables build_vx_tables() {
  VxTables r{};
  for (int k = 0; k < 50; ++k) r.masks[k] = (unsigned char)(kTri3.m[k][0] | kTri3.m[k][1] << 4);
  for (int a = 0; a < 16; ++a)
    for (int b = 0; b < 16; ++b) r.type[a * 16 + b] = (unsigned char)kTri3Index.idx[a][b];
  return r;
}
__constant__ VxTables kVxTables = build_vx_tables();

// A wavefront's word: per vertex its positive triangles and how many come before them.  (A list of the triangles in LDS,
// up to 50 per vertex, would halve the wavefronts per CU, and both passes below live from them.)
struct VxWave {
  u64 mask[64];
  unsigned short before[64];
};
// Vertex lane and type of the word's triangle i: the last vertex with at most i before it, and its (i - before)-th bit.
__device__ __forceinline__ void vx_find(const VxWave& W, unsigned i, unsigned& lane, unsigned& type) {
  unsigned l = 0;
#pragma unroll
  for (unsigned s = 32; s; s >>= 1)
    if (W.before[l + s] <= i) l += s;
  unsigned n = i - W.before[l], at = 0;
  u64 m = W.mask[l];
#pragma unroll
  for (unsigned s = 32; s; s >>= 1) {
    const unsigned c = (unsigned)__popcll(m & ((1ull << s) - 1ull));
    const bool up = n >= c;
    n -= up ? c : 0u;
    at += up ? s : 0u;
    m = up ? m >> s : m;
  }
  lane = l;
  type = at;
}

// What both passes over the triangles of a word need.
struct VxWord {
  int x0, y, z, t, n;
  long long v0, h0;  // first vertex, first hit
};
__device__ __forceinline__ bool vx_word(const VxGrid& g, long long k, long long n_words, const u64* __restrict__ tmask,
                                        const unsigned short* __restrict__ before, const int* __restrict__ wcnt,
                                        const long long* __restrict__ wbase, VxWave& W, VxWord& o) {
  if (k >= n_words) return false;
  o.n = wcnt[k];
  if (o.n == 0) return false;
  const int lane = lane_id();
  const unsigned r = (unsigned)(k / g.nwx);
  o.x0 = (int)(k - (long long)r * g.nwx) * 64;
  o.y = (int)(r % (unsigned)g.ny);
  o.z = (int)((r / (unsigned)g.ny) % (unsigned)g.nz);
  o.t = (int)(r / ((unsigned)g.ny * (unsigned)g.nz));
  o.v0 = (long long)r * g.nx + o.x0;
  o.h0 = wbase[k];
  const bool in = o.x0 + lane < g.nx;
  W.mask[lane] = in ? tmask[o.v0 + lane] : 0ull;
  W.before[lane] = in ? before[o.v0 + lane] : (unsigned short)0xFFFFu;
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return true;
}

// The smaller partner of triangle (p; M1, M2) in the tetrahedron (c; c1, M1, M2), c = p - e(c1), whose other three sides
// are anchored at c.
__device__ __forceinline__ unsigned vx_partner(const VxGrid& g, const VxTables& T, int x, int y, int z, int t,
                                               unsigned c1, unsigned M1, unsigned M2, const u64* __restrict__ tmask,
                                               const unsigned short* __restrict__ before,
                                               const long long* __restrict__ wbase) {
  const int cx = x - (int)(c1 & 1u);
  const long long r = ((long long)(t - (int)(c1 >> 3)) * g.nz + (z - (int)((c1 >> 2) & 1u))) * g.ny + (y - (int)((c1 >> 1) & 1u));
  const long long c = r * g.nx + cx;
  const u64 m = tmask[c];
  const unsigned base = (unsigned)wbase[r * g.nwx + (cx >> 6)] + before[c];
  const unsigned t1 = T.type[(c1 | M1) * 16 + M2], t2 = T.type[c1 * 16 + (M1 | M2)], t3 = T.type[c1 * 16 + M1];
  const unsigned ty = (m >> t1) & 1ull ? t1 : ((m >> t2) & 1ull ? t2 : t3);
  return base + (unsigned)__popcll(m & ((1ull << ty) - 1ull));
}

// One lane per positive triangle of a word.  The parent is a smaller partner: the one in the tetrahedron below along the
// lowest axis that the type leaves free, or else one of the same anchor (parents are smaller: a forest, flattened by
// uf_compress before vx_link).  512 x 128 x 64 x 8: 0.69 ms (one lane per vertex, writing its triangles one by one, 2.57).
__global__ __launch_bounds__(256) void vx_emit(VxGrid g, long long first, long long n_words, const u64* __restrict__ tmask,
                                               const unsigned short* __restrict__ before, const int* __restrict__ wcnt,
                                               const long long* __restrict__ wbase, long long* __restrict__ tri_id,
                                               float* __restrict__ pos, unsigned* __restrict__ parent) {
  __shared__ VxWave sw[4];
  __shared__ VxTables T;
  for (int i = threadIdx.x; i < (int)sizeof(VxTables); i += 256)
    ((unsigned char*)&T)[i] = ((const unsigned char*)&kVxTables)[i];
  __syncthreads();
  VxWave& W = sw[threadIdx.x >> 6];
  VxWord w;
  const long long k = first + (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (!vx_word(g, k, n_words, tmask, before, wcnt, wbase, W, w)) return;
  const long long plane = (long long)g.nx * g.ny * g.nz;
  const bool wide = ((uintptr_t)pos & 15u) == 0;
  for (int i = lane_id(); i < w.n; i += 64) {
    unsigned L, ty;
    vx_find(W, (unsigned)i, L, ty);
    const unsigned M1 = T.masks[ty] & 15u, M2 = T.masks[ty] >> 4, b = M1 | M2;
    const int x = w.x0 + (int)L, y = w.y, z = w.z, t = w.t;
    unsigned st = 0;
    auto value = [&](unsigned c, int comp) -> double {
      const long long o = ((long long)(t + (int)(c >> 3)) * 2 + comp) * plane +
                          ((long long)(z + (int)((c >> 2) & 1u)) * g.ny + (y + (int)((c >> 1) & 1u))) * g.nx + (x + (int)(c & 1u));
      return vx_q(g.psi[o], g.qscale, st);
    };
    const double p0 = value(0, 0), p1 = value(0, 1), q0 = value(M1, 0), q1 = value(M1, 1), r0 = value(b, 0), r1 = value(b, 1);
    const unsigned h = (unsigned)(w.h0 + i);
    unsigned par = h;
    const unsigned down = 15u & ~b & ((x > 0 ? 1u : 0u) | (y > 0 ? 2u : 0u) | (z > 0 ? 4u : 0u) | (t > 0 ? 8u : 0u));
    if (down) {
      par = vx_partner(g, T, x, y, z, t, down & (0u - down), M1, M2, tmask, before, wbase);
    } else {
      const u64 m = W.mask[L];
      auto same = [&](unsigned a, unsigned c) {  // the triangle (p; a, c), when positive
        const unsigned o = T.type[a * 16 + c];
        if ((m >> o) & 1ull) par = h - (unsigned)__popcll(m & ((1ull << ty) - (1ull << o)));
      };
      for (unsigned c = (M1 - 1u) & M1; c && par == h; c = (c - 1u) & M1) {
        same(c, (M1 ^ c) | M2);
        same(c, M1 ^ c);
      }
      for (unsigned c = (M2 - 1u) & M2; c && par == h; c = (c - 1u) & M2) same(M1, c);
    }
    // exact cofactors, each rounded once to binary64 (as edge_det); the nonzero ones share the puncture sign, so their
    // sum has no cancellation, and weights from one reciprocal carry a few roundings each (relative error below 2^-50,
    // far inside the binary32 points written)
    const double C0 = edge_det(q0, q1, r0, r1), C1 = -edge_det(p0, p1, r0, r1), C2 = edge_det(p0, p1, q0, q1);
    double mu0 = 1.0 / 3.0, mu1 = 1.0 / 3.0, mu2 = 1.0 / 3.0;
    if (C0 != 0.0 || C1 != 0.0 || C2 != 0.0) {
      const double rD = 1.0 / ((C0 + C1) + C2);
      mu0 = C0 * rD;
      mu1 = C1 * rD;
      mu2 = C2 * rD;
    }
    float out[4];
    const double c0[4] = {(double)x, (double)y, (double)z, (double)t};
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const double c1 = c0[a] + ((M1 >> a) & 1u), c2 = c0[a] + ((b >> a) & 1u);
      out[a] = (float)((mu0 * c0[a] + mu1 * c1) + mu2 * c2);
    }
    tri_id[h] = (w.v0 + L) * 50 + ty;
    parent[h] = par;
    if (pos) {
      if (wide) {
        reinterpret_cast<float4*>(pos)[h] = make_float4(out[0], out[1], out[2], out[3]);
      } else {
#pragma unroll
        for (int a = 0; a < 4; ++a) pos[(size_t)h * 4 + a] = out[a];
      }
    }
  }
}

// The links that are not a parent already, each from its larger end, one lane per positive triangle.  Bound by the
// latency of dependent loads, so the partners of a triangle are found together, then their parents read together: after
// uf_compress most of them agree with the triangle's own and are done; only the others are united.  512 x 128 x 64 x 8,
// 23 M triangles: 2.3 ms (partners one after another 5.5 ms; groups of the positive triangles of every 4-cube, each
// member united with its group's first and no forest before, 7.3 ms).
__global__ __launch_bounds__(256) void vx_link(VxGrid g, long long first, long long n_words, const u64* __restrict__ tmask,
                                               const unsigned short* __restrict__ before, const int* __restrict__ wcnt,
                                               const long long* __restrict__ wbase, unsigned* __restrict__ parent) {
  __shared__ VxWave sw[4];
  __shared__ VxTables T;
  for (int i = threadIdx.x; i < (int)sizeof(VxTables); i += 256)
    ((unsigned char*)&T)[i] = ((const unsigned char*)&kVxTables)[i];
  __syncthreads();
  VxWave& W = sw[threadIdx.x >> 6];
  VxWord w;
  const long long k = first + (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (!vx_word(g, k, n_words, tmask, before, wcnt, wbase, W, w)) return;
  for (int i = lane_id(); i < w.n; i += 64) {
    unsigned L, ty;
    vx_find(W, (unsigned)i, L, ty);
    const unsigned M1 = T.masks[ty] & 15u, M2 = T.masks[ty] >> 4;
    const int x = w.x0 + (int)L;
    const unsigned h = (unsigned)(w.h0 + i);
    const unsigned down =
        15u & ~(M1 | M2) & ((x > 0 ? 1u : 0u) | (w.y > 0 ? 2u : 0u) | (w.z > 0 ? 4u : 0u) | (w.t > 0 ? 8u : 0u));
    // two free axes at most: the lower one is the parent's, the higher one and both together are left
    constexpr int kSlots = 6;
    unsigned s[kSlots];
#pragma unroll
    for (int q = 0; q < kSlots; ++q) s[q] = h;
    int n = 2;
    const unsigned high = down & (down - 1u);
    if (high) {
      s[0] = vx_partner(g, T, x, w.y, w.z, w.t, high, M1, M2, tmask, before, wbase);
      s[1] = vx_partner(g, T, x, w.y, w.z, w.t, down, M1, M2, tmask, before, wbase);
    }
    const u64 m = W.mask[L];
    u64 rest = 0;  // same-anchor partners beyond the slots, by their distance (an anchor has at most 50 triangles)
    auto same = [&](unsigned a, unsigned c) {
      const unsigned o = T.type[a * 16 + c];
      if ((m >> o) & 1ull) {
        const unsigned v = h - (unsigned)__popcll(m & ((1ull << ty) - (1ull << o)));
#pragma unroll
        for (int q = 2; q < kSlots; ++q) s[q] = n == q ? v : s[q];
        if (n >= kSlots) rest |= 1ull << (h - v);
        ++n;
      }
    };
    for (unsigned c = (M1 - 1u) & M1; c; c = (c - 1u) & M1) {
      same(c, (M1 ^ c) | M2);
      same(c, M1 ^ c);
    }
    for (unsigned c = (M2 - 1u) & M2; c; c = (c - 1u) & M2) same(M1, c);
    unsigned p[kSlots];
    const unsigned ph = parent[h];
#pragma unroll
    for (int q = 0; q < kSlots; ++q) p[q] = parent[s[q]];
    unsigned r = ph;
    bool found = false;  // r is the triangle's root (as last found), not only its parent
#pragma unroll
    for (int q = 0; q < kSlots; ++q)
      if (p[q] != ph) {
        if (!found) r = uf_find_cached(parent, ph);
        found = true;
        r = uf_unite_into(parent, r, s[q]);
      }
    for (; rest; rest &= rest - 1) {
      if (!found) r = uf_find_cached(parent, ph);
      found = true;
      r = uf_unite_into(parent, r, h - ((unsigned)__ffsll((long long)rest) - 1u));
    }
  }
}

// Words of a launch of the passes over triangles: 64 lanes each, and a launch holds less than 2^32 lanes along x.
constexpr long long kVxLaunchWords = 1ll << 25;

dim3 vx_grid(const VxGrid& g) {
  return dim3((unsigned)((g.nx + kVxBX - 1) / kVxBX), (unsigned)g.ny, (unsigned)(g.nz * g.nt));
}

}  // namespace

hipError_t launch_vx_detect(const float* psi, int nx, int ny, int nz, int nt, float qscale, unsigned short* emask,
                            unsigned long long* tmask, unsigned short* before, int* wcnt, unsigned* status,
                            hipStream_t s) {
  const VxGrid g{psi, nx, ny, nz, nt, (nx + 63) / 64, qscale};
  vx_edges<<<vx_grid(g), kVxBX, 0, s>>>(g, emask, status);
  vx_tris<<<vx_grid(g), kVxBX, 0, s>>>(g, emask, tmask, before, wcnt);
  return hipGetLastError();
}

hipError_t launch_vx_emit(const float* psi, int nx, int ny, int nz, int nt, float qscale,
                          const unsigned long long* tmask, const unsigned short* before, const int* wcnt,
                          const long long* wbase, long long n_hits, long long* tri_id, float* pos, unsigned* parent,
                          hipStream_t s) {
  const VxGrid g{psi, nx, ny, nz, nt, (nx + 63) / 64, qscale};
  const long long n_words = (long long)nt * nz * ny * g.nwx;
  auto each = [&](auto launch) -> hipError_t {
    for (long long first = 0; first < n_words; first += kVxLaunchWords) {
      const long long words = n_words - first < kVxLaunchWords ? n_words - first : kVxLaunchWords;
      launch(first, (unsigned)((words + 3) / 4));
    }
    return hipGetLastError();
  };
  hipError_t e = each([&](long long first, unsigned blocks) {
    vx_emit<<<blocks, 256, 0, s>>>(g, first, n_words, tmask, before, wcnt, wbase, tri_id, pos, parent);
  });
  if (e == hipSuccess) e = launch_uf_compress(parent, n_hits, s);
  if (e != hipSuccess) return e;
  return each([&](long long first, unsigned blocks) {
    vx_link<<<blocks, 256, 0, s>>>(g, first, n_words, tmask, before, wcnt, wbase, parent);
  });
}

}  // namespace ftk
