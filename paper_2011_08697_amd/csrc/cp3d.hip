// cp3d.hip -- critical-point tracking in 3D space + time on gfx950.
//
// Mesh: the Kuhn subdivision of the (x, y, z, t) grid (Sec. 3.3): per vertex 15 edge, 50 triangle, 60 tetrahedron
// (the tested faces) and 24 pentachoron (cell) types.  A tetrahedron is punctured when the four signed cofactors of
// (v0 v1 v2 v3 ; 1 1 1 1) agree (Sec. 4.3, Eq. 2); each cofactor is, up to a fixed sign, the 3x3 determinant of the
// vectors of one of its triangles, so one SoS sign bit per triangle (50 per vertex, a 64-bit word) is computed and
// shared through LDS.
//
//   facts3d  -- one pass over the field: the sign facts of the quantised gradients over every 16 x 8 x 4 tile and step.
//   plan3d   -- the tile-steps that the facts of their two planes prove empty (most of them on smooth fields) are
//               marked; the others are listed as runs of consecutive steps of a tile.
//   detect3d -- one workgroup per listed run: gradients staged and quantised in LDS, triangle sign words of the tile
//               (+1 halo), 60 tetrahedron tests per anchor; writes a 60-bit puncture mask per vertex and the hit
//               count of every 16-vertex row segment.  Three blocks per CU (168 registers).
//   emit3d   -- face ids at their output indices from the segment prefixes, then one lane per hit: exact cofactors,
//               sublocation, Hessian type, and the union-find links of the hit's two pentachora (Alg. 1 pass 2).
#include "common.h"
#include "internal.h"

namespace ftk {

namespace {

constexpr int TX3 = 16, TY3 = 8, TZ3 = 4;
constexpr int SEG3 = 16;  // row segment width (x)

constexpr unsigned long long kTetUseX = types_using_axis(kTet3, 1);
constexpr unsigned long long kTetUseY = types_using_axis(kTet3, 2);
constexpr unsigned long long kTetUseZ = types_using_axis(kTet3, 4);
constexpr unsigned long long kTetUseT = types_using_axis(kTet3, 8);

// triangle types without the time axis (ordinal) and with it (interval)
struct TriSplit {
  int n_ord, n_int;
  unsigned char ord[50], itv[50];
};
constexpr TriSplit build_tri_split() {
  TriSplit r{};
  for (int i = 0; i < kTri3.count; ++i) {
    if ((kTri3.m[i][0] | kTri3.m[i][1]) & 8)
      r.itv[r.n_int++] = (unsigned char)i;
    else
      r.ord[r.n_ord++] = (unsigned char)i;
  }
  return r;
}
constexpr TriSplit kTriSplit = build_tri_split();
static_assert(kTriSplit.n_ord == 12 && kTriSplit.n_int == 38, "12 ordinal + 38 interval triangle types");

template <bool WIDE>
struct Q3;
template <>
struct Q3<false> {
  typedef float T;  // integers below 2^20, exact in binary32
};
template <>
struct Q3<true> {
  typedef long long T;
};

__device__ __forceinline__ long long fpl3(const Grid3& g, int t) { return g.f_ring ? t % g.f_ring : t; }
__device__ __forceinline__ long long mpl3(const Grid3& g, int t) { return g.m_ring ? t % g.m_ring : t; }

// Exact 3x3 determinant of columns a, b, c (rows = components): 64-bit when |entries| < 2^20, else 128-bit.
template <bool WIDE, typename Q>
__device__ __forceinline__ i128 det3x(const Q* a, const Q* b, const Q* c) {
  if (!WIDE) {
    long long m0 = (long long)b[1] * c[2] - (long long)b[2] * c[1];
    long long m1 = (long long)b[0] * c[2] - (long long)b[2] * c[0];
    long long m2 = (long long)b[0] * c[1] - (long long)b[1] * c[0];
    return (i128)((long long)a[0] * m0 - (long long)a[1] * m1 + (long long)a[2] * m2);
  }
  i128 m0 = (i128)b[1] * c[2] - (i128)b[2] * c[1];
  i128 m1 = (i128)b[0] * c[2] - (i128)b[2] * c[0];
  i128 m2 = (i128)b[0] * c[1] - (i128)b[1] * c[0];
  return (i128)a[0] * m0 - (i128)a[1] * m1 + (i128)a[2] * m2;
}

// SoS sign of the 3x3 determinant m[j][k] (row j = component, column k = vertex in index order), entry (j, k)
// perturbed by eps^(2^(3k+j)).  Expanding the perturbed determinant and ordering its terms by exponent, the sign
// is that of the first nonzero of
//   det, C00, C10, C20, C01, -m22, m12, C11, m22, -m02, C21, -m12, m02, C02, m21, -m11, -m20, -1
// with C_jk = (-1)^(j+k) times the 2x2 minor without row j and column k.  Returned as a bit: 1 for positive.
// (values passed by register: columns a = m[.][0], b = m[.][1], c = m[.][2])
__device__ __noinline__ unsigned sos3_tail(long long a0, long long a1, long long a2, long long b0, long long b1,
                                           long long b2, long long c0, long long c1, long long c2) {
  const i128 m00 = a0, m10 = a1, m20 = a2;
  const i128 m01 = b0, m11 = b1, m21 = b2;
  const i128 m02 = c0, m12 = c1, m22 = c2;
  i128 v;
  v = m11 * m22 - m12 * m21;          // C00
  if (v != 0) return v > 0;
  v = -(m01 * m22 - m02 * m21);       // C10
  if (v != 0) return v > 0;
  v = m01 * m12 - m02 * m11;          // C20
  if (v != 0) return v > 0;
  v = -(m10 * m22 - m12 * m20);       // C01
  if (v != 0) return v > 0;
  if (m22 != 0) return m22 < 0;       // -m22
  if (m12 != 0) return m12 > 0;       // m12
  v = m00 * m22 - m02 * m20;          // C11
  if (v != 0) return v > 0;
  // m22 == 0 here, so the next term (m22) vanishes
  if (m02 != 0) return m02 < 0;       // -m02
  v = -(m00 * m12 - m02 * m10);       // C21
  if (v != 0) return v > 0;
  // m12 == 0 and m02 == 0 here
  v = m10 * m21 - m11 * m20;          // C02
  if (v != 0) return v > 0;
  if (m21 != 0) return m21 > 0;       // m21
  if (m11 != 0) return m11 < 0;       // -m11
  if (m20 != 0) return m20 < 0;       // -m20
  return 0u;                          // -1
}

template <bool WIDE, typename Q>
__device__ __forceinline__ unsigned sos3_positive(const Q* a, const Q* b, const Q* c) {
  const i128 d = det3x<WIDE, Q>(a, b, c);
  if (d != 0) return d > 0;
  return sos3_tail(a[0], a[1], a[2], b[0], b[1], b[2], c[0], c[1], c[2]);
}

// The same sequence in binary64 for narrow entries (integers below 2^20): every term is an entry or a 2x2 minor,
// whose two products (below 2^40) and difference are exact in binary64.
__device__ __forceinline__ unsigned sos3_tail_f64(double m00, double m10, double m20, double m01, double m11,
                                                  double m21, double m02, double m12, double m22) {
  auto mn = [](double x, double y, double z, double w) { return __builtin_fma(x, y, -(z * w)); };  // exact
  double v;
  v = mn(m11, m22, m12, m21);         // C00
  if (v != 0.0) return v > 0.0;
  v = -mn(m01, m22, m02, m21);        // C10
  if (v != 0.0) return v > 0.0;
  v = mn(m01, m12, m02, m11);         // C20
  if (v != 0.0) return v > 0.0;
  v = -mn(m10, m22, m12, m20);        // C01
  if (v != 0.0) return v > 0.0;
  if (m22 != 0.0) return m22 < 0.0;   // -m22
  if (m12 != 0.0) return m12 > 0.0;   // m12
  v = mn(m00, m22, m02, m20);         // C11
  if (v != 0.0) return v > 0.0;
  if (m02 != 0.0) return m02 < 0.0;   // -m02 (m22 == 0 here)
  v = -mn(m00, m12, m02, m10);        // C21
  if (v != 0.0) return v > 0.0;
  v = mn(m10, m21, m11, m20);         // C02 (m12 == m02 == 0 here)
  if (v != 0.0) return v > 0.0;
  if (m21 != 0.0) return m21 > 0.0;   // m21
  if (m11 != 0.0) return m11 < 0.0;   // -m11
  if (m20 != 0.0) return m20 < 0.0;   // -m20
  return 0u;                          // -1
}

// Exact evaluation for narrow entries (below 2^20: minors below 2^41, terms below 2^61), then SoS.  A zero column
// makes the determinant vanish without evaluating it (frequent where gradients underflow the quantum); the
// sequence that follows runs in binary64, exactly.
__device__ __forceinline__ unsigned sos3_exact_narrow(float a0, float a1, float a2, float b0, float b1, float b2,
                                                      float c0, float c1, float c2) {
  const bool zero_col = (a0 == 0.0f && a1 == 0.0f && a2 == 0.0f) || (b0 == 0.0f && b1 == 0.0f && b2 == 0.0f) ||
                        (c0 == 0.0f && c1 == 0.0f && c2 == 0.0f);
  if (!zero_col) {
    const long long A0 = (long long)a0, A1 = (long long)a1, A2 = (long long)a2;
    const long long B0 = (long long)b0, B1 = (long long)b1, B2 = (long long)b2;
    const long long C0 = (long long)c0, C1 = (long long)c1, C2 = (long long)c2;
    const long long m0 = B1 * C2 - B2 * C1, m1 = B0 * C2 - B2 * C0, m2 = B0 * C1 - B1 * C0;
    const long long d = A0 * m0 - A1 * m1 + A2 * m2;
    if (d != 0) return d > 0;
  }
  return sos3_tail_f64(a0, a1, a2, b0, b1, b2, c0, c1, c2);
}

}  // namespace

// Compile-time triangle lists of the detection's four wavefronts: the 12 ordinal types, and the 38 interval types in two
// halves.
constexpr int kOrdN = 12, kItvHalf = 19;
template <int FIRST>
struct ItvList {
  static constexpr int n = kItvHalf;
  static constexpr int ti(int k) { return kTriSplit.itv[FIRST + k]; }
};
struct OrdList {
  static constexpr int n = kOrdN;
  static constexpr int ti(int k) { return kTriSplit.ord[k]; }
};
// Position of an ordinal type in their list (the words of plane t + 1 hold these only).
constexpr int ord_bit(int ti) {
  for (int k = 0; k < kOrdN; ++k)
    if (kTriSplit.ord[k] == ti) return k;
  return 0;
}

// ---------------------------------------------------------------------------------------------------------------
// Sign facts.  A tetrahedron anchored in a tile at step t has its vertices among the tile's anchors and their +1
// neighbours at the steps t and t + 1.  When on both planes one component has one strict sign at all of these vertices,
// it keeps that sign under the symbolic perturbation (its entries move by infinitesimals only), so the origin is outside
// every tetrahedron; with all vectors zero every triangle determinant takes the perturbation's last term (-1), so the
// four cofactor signs never agree.  Such a tile-step is empty: 94% of them on the 256^3 x 16 series of moving blobs.
//
// Facts are bits (2c / 2c + 1: component c > 0 / < 0 everywhere; 6: every vector zero), one byte for each of the eight
// parts of a tile that its lower neighbours need: byte c of a tile's word covers the anchors with x first (c & 1), y
// first (c & 2), z first (c & 4) only.  A tile's facts over its anchors and their +1 neighbours are the bytes c of the
// tiles at + c, combined.
//
// One wavefront per 64 x 8 x 4 vertices of a plane (four tiles), lane = x: each layer's rows are read once into
// registers (the layers before and after come with them), x neighbours by whole-wave DPP shifts with the two outer
// columns of the 32 rows in one load.  Bound by the rows read again for the halos: 256^3 x 16 in 0.30 ms; the same facts gathered by the
// detection's own tiles, which stage every plane in LDS, took 8 of its 10 ms.
// ---------------------------------------------------------------------------------------------------------------
namespace {

// Extrema of the three components over a set of vertices, and the facts they give.
struct Extrema3 {
  float mn[3], mx[3];
  __device__ __forceinline__ void set(const float (&q)[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) mn[c] = mx[c] = q[c];
  }
  __device__ __forceinline__ void add(const float (&q)[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      mn[c] = fminf(mn[c], q[c]);
      mx[c] = fmaxf(mx[c], q[c]);
    }
  }
  __device__ __forceinline__ float largest() const {
    return fmaxf(fmaxf(fmaxf(mx[0], -mn[0]), fmaxf(mx[1], -mn[1])), fmaxf(mx[2], -mn[2]));
  }
  __device__ __forceinline__ unsigned facts() const {
    unsigned f = largest() == 0.0f ? 64u : 0u;
#pragma unroll
    for (int c = 0; c < 3; ++c) f |= (mn[c] > 0.0f ? 1u << (2 * c) : 0u) | (mx[c] < 0.0f ? 2u << (2 * c) : 0u);
    return f;
  }
};

}  // namespace

__global__ __launch_bounds__(256) void facts3d(Grid3 g, int t_first, unsigned long long* __restrict__ facts,
                                               unsigned* __restrict__ status) {
  const int lane = threadIdx.x & 63;
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int ntx = (nx + TX3 - 1) / TX3, nty = (ny + TY3 - 1) / TY3, ntz = (nz + TZ3 - 1) / TZ3;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const long long yz = (long long)blockIdx.y * 4 + w;  // wavefronts of a workgroup are neighbours in y
  if (yz >= (long long)nty * ntz) return;
  const int ty = (int)(yz % nty), tz = (int)(yz / nty);
  const unsigned nxb = (unsigned)(nx + 63) / 64u;
  const int t = t_first + (int)(blockIdx.x / nxb);
  const int x0 = (int)(blockIdx.x % nxb) * 64, y0 = ty * TY3, z0 = tz * TZ3;
  const float* P = g.f + fpl3(g, t) * ((long long)nx * ny * nz);
  const int gx = x0 + lane;
  const unsigned xb = 4u * (unsigned)min(gx, nx - 1);
  const float one = g.qscale, half = 0.5f * g.qscale;  // powers of two: exact factors
  const int one_bits = __builtin_amdgcn_readfirstlane(__float_as_int(one));
  const int half_bits = __builtin_amdgcn_readfirstlane(__float_as_int(half));
  const float sx = (gx == 0 || gx == nx - 1) ? one : half;
  // rows at clamped (in-grid) coordinates: a clamped neighbour equals the edge value, which makes the difference the
  // one-sided one; only its factor differs
  auto row = [&](int y, int z) -> float {
    const long long r = (long long)min(max(z, 0), nz - 1) * ny + min(max(y, 0), ny - 1);
    return *(const float*)((const char*)(P + r * nx) + xb);
  };
  float side;  // lanes 0-31: column x0 - 1 of row (y0 + l % 8, z0 + l / 8); lanes 32-63: column x0 + 64
  {
    const int r = lane & 31;
    const long long o = (long long)min(z0 + (r >> 3), nz - 1) * ny + min(y0 + (r & 7), ny - 1);
    side = P[o * nx + (lane < 32 ? max(x0 - 1, 0) : min(x0 + 64, nx - 1))];
  }
  float prev[TY3], cur[TY3 + 2], next[TY3 + 2];
#pragma unroll
  for (int y = 0; y < TY3; ++y) prev[y] = row(y0 + y, z0 - 1);
#pragma unroll
  for (int y = 0; y < TY3 + 2; ++y) cur[y] = row(y0 - 1 + y, z0);
  Extrema3 all, zf, yf, yzf;  // the tile's rows; those of its first layer, first row of each layer, first row
  float nonfinite = 0.0f;
#pragma unroll
  for (int lz = 0; lz < TZ3; ++lz) {
#pragma unroll
    for (int y = 0; y < TY3 + 2; ++y) next[y] = row(y0 - 1 + y, z0 + lz + 1);
    const int z = z0 + lz;
    if (z < nz) {  // uniform
      const float sz = __int_as_float((z == 0 || z == nz - 1) ? one_bits : half_bits);
#pragma unroll
      for (int ly = 0; ly < TY3; ++ly) {
        const int y = y0 + ly;
        if (y < ny) {  // uniform
          const float f = cur[ly + 1];
          nonfinite = __builtin_fmaf(f, 0.0f, nonfinite);
          const float lo = from_prev(f, lane_value(side, lz * 8 + ly)), hi = from_next(f, lane_value(side, 32 + lz * 8 + ly));
          const float sy = __int_as_float((y == 0 || y == ny - 1) ? one_bits : half_bits);
          const float q[3] = {rintf((hi - lo) * sx), rintf((cur[ly + 2] - cur[ly]) * sy),
                              rintf((next[ly + 1] - prev[ly]) * sz)};
          if (lz == 0 && ly == 0) {
            all.set(q);
            yzf.set(q);
            yf.set(q);
          } else {
            all.add(q);
            if (ly == 0) yf.add(q);
          }
        }
      }
      if (lz == 0) zf = all;
    }
#pragma unroll
    for (int y = 0; y < TY3; ++y) prev[y] = cur[y + 1];
#pragma unroll
    for (int y = 0; y < TY3 + 2; ++y) cur[y] = next[y];
  }
  unsigned st = 0;
  const float big = all.largest();
  if (big >= 1048576.0f) st |= big >= 2199023255552.0f ? (ST_WIDE | ST_RANGE) : ST_WIDE;
  if (!(nonfinite == 0.0f)) st |= ST_NONFINITE;
  if (st) atomicOr(status, st);
  // fields of 8 bits: all rows, y first, z first, y and z first; lanes outside the grid do not count
  unsigned f = all.facts() | yf.facts() << 8 | zf.facts() << 16 | yzf.facts() << 24;
  if (gx >= nx) f = ~0u;
  unsigned r = f;  // over the 16 lanes of a tile, by rotations within them
  r &= (unsigned)__builtin_amdgcn_update_dpp(0, (int)r, 0x128, 0xf, 0xf, false);  // row_ror:8
  r &= (unsigned)__builtin_amdgcn_update_dpp(0, (int)r, 0x124, 0xf, 0xf, false);
  r &= (unsigned)__builtin_amdgcn_update_dpp(0, (int)r, 0x122, 0xf, 0xf, false);
  r &= (unsigned)__builtin_amdgcn_update_dpp(0, (int)r, 0x121, 0xf, 0xf, false);
  const int tx = x0 / TX3 + (lane >> 4);
  if ((lane & 15) == 0 && tx < ntx) {
    unsigned long long out = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) out |= (unsigned long long)((((c & 1) ? f : r) >> (8 * (c >> 1))) & 0x7Fu) << (8 * c);
    facts[((mpl3(g, t) * ntz + tz) * nty + ty) * ntx + tx] = out;
  }
}

// One lane per tile and `steps` steps: marks the tile's empty steps and lists the runs of the others (at most `most` steps
// each, none over the end of a lane's steps).  A lane takes its steps one after another, 0.5 to 5 us each,
// so that a lane with a whole series made long ones wait (8^3 x 8000: 4638 against 287 us a call, 32^3 x 2000: 3413 / 639).
constexpr int kPlanSteps = 16;
__global__ __launch_bounds__(256) void plan3d(Grid3 g, int steps, int most,
                                              const unsigned long long* __restrict__ facts,
                                              uint2* __restrict__ runs, unsigned long long* __restrict__ n_runs) {
  const int ntx = (g.nx + TX3 - 1) / TX3, nty = (g.ny + TY3 - 1) / TY3, ntz = (g.nz + TZ3 - 1) / TZ3;
  const long long tiles = (long long)ntx * nty * ntz;
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x, part = i / tiles, tile = i - part * tiles;
  const long long begin = g.t_begin + part * steps;
  if (begin >= g.t_end) return;
  const int t0 = (int)begin, t1 = min(t0 + steps, g.t_end);
  const int tx = (int)(tile % ntx), ty = (int)((tile / ntx) % nty), tz = (int)(tile / ((long long)ntx * nty));
  auto plane_facts = [&](int t) -> unsigned {
    unsigned f = 0x7Fu;
#pragma unroll
    for (int c = 0; c < 8; ++c) {  // clamped tiles, loads in flight together; tiles past the grid do not count
      const int x = tx + (c & 1), y = ty + ((c >> 1) & 1), z = tz + (c >> 2);
      const unsigned long long w =
          facts[((mpl3(g, t) * ntz + min(z, ntz - 1)) * nty + min(y, nty - 1)) * ntx + min(x, ntx - 1)];
      if (x < ntx && y < nty && z < ntz) f &= (unsigned)(w >> (8 * c));
    }
    return f;
  };
  unsigned here = plane_facts(t0);
  int start = -1;
  auto close = [&](int end) {
    if (start < 0) return;
    runs[atomicAdd(n_runs, 1ull)] = make_uint2((unsigned)tile, (unsigned)start | (unsigned)(end - start - 1) << 28);
    start = -1;
  };
  for (int t = t0; t < t1; ++t) {
    const unsigned there = t + 1 < g.nt ? plane_facts(t + 1) : 0x7Fu;
    const bool empty = (here & there) != 0u;
    g.cert[mpl3(g, t) * tiles + tile] = empty ? 1 : 0;
    if (empty || (start >= 0 && t - start == most)) close(t);
    if (!empty && start < 0) start = t;
    here = there;
  }
  close(t1);
}

// ---------------------------------------------------------------------------------------------------------------
// Pass 1: detection of the listed runs.  Persistent workgroups of 256 take them from a counter (their costs differ
// widely with the number of exact zeros).
//
// Inside a listed tile the facts decide again, now per anchor: an anchor whose unit 4-cube has a fact has no punctured
// tetrahedron, and a triangle word is needed only at the positions that another anchor's tests read.  The anchors left
// and the positions they need are listed in LDS, and the four wavefronts take the ordinal triangles of plane t, the two
// halves of the interval ones and the ordinal ones of plane t + 1 of every 64 of them, with dense lanes.  256^3 x 16:
// 1.04 ms at three wavefronts per SIMD, where a few values spill (1.19 when held to four, where more do); every triangle of every listed tile,
// in a static order of the runs, took 6.3 ms, and with the facts gathered by the same kernel 9.9 ms.
// ---------------------------------------------------------------------------------------------------------------
template <bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WIDE ? 2 : 3))) void detect3d(
    Grid3 g, const uint2* __restrict__ runs, const unsigned long long* __restrict__ n_runs,
    unsigned long long* __restrict__ taken, uint64_t* __restrict__ masks, int* __restrict__ seg_cnt,
    const unsigned* __restrict__ status) {
  if (!WIDE && (*status & ST_WIDE)) return;  // the caller runs the wide variant
  typedef typename Q3<WIDE>::T Q;
  constexpr int QX = TX3 + 2, QY = TY3 + 2, QZ = TZ3 + 2;  // quantised vectors: x0 .. x0+TX+1
  constexpr int WX = TX3 + 1, WY = TY3 + 1, WZ = TZ3 + 1;  // triangle words: x0 .. x0+TX
  constexpr int QN = QX * QY * QZ, WN = WX * WY * WZ, AN = TX3 * TY3 * TZ3;
  __shared__ Q qs[2][3][QN];
  __shared__ unsigned long long tw[WN];  // triangle words of plane t
  __shared__ unsigned short to[WN];      // ordinal triangles of plane t + 1
  __shared__ unsigned char qf[2][QN];    // sign facts of the vectors
  __shared__ unsigned long long left[AN / 64];  // anchors without a fact
  __shared__ unsigned short pos[WN], anc[AN];   // positions whose words are needed, anchors to be tested
  __shared__ int n_pos, n_anc, s_cnt[TY3 * TZ3];
  __shared__ unsigned long long s_item;
  __shared__ unsigned char s_tcor[50];  // triangle type -> corner a | corner b << 4
  static_assert(AN == 512, "two anchors a thread");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid < 50) s_tcor[tid] = (unsigned char)(kTri3.m[tid][0] | ((kTri3.m[tid][0] | kTri3.m[tid][1]) << 4));
  const int nx = g.nx, ny = g.ny, nz = g.nz, nt = g.nt;
  const int ntx = (nx + TX3 - 1) / TX3, nty = (ny + TY3 - 1) / TY3;
  const long long plane = (long long)nx * ny * nz;
  int bxl = 0, x0 = 0, y0 = 0, z0 = 0;  // the run's tile

  // Quantised gradients of plane tq into slot par.  fetch(): the thread's share of the plane's field block with a
  // one-cell halo, from clamped (in-grid) addresses into registers, all loads in flight together; halo cells
  // outside the grid hold copies of edge values, which diff3 never reads (one-sided differences at the first and
  // last index).  quantise(par): the block into the LDS of slot par (its previous plane is dead by then), the
  // stencils from LDS, then the quantised vectors into the slot and their facts (outside the grid: every fact).
  // Every thread reaches quantise() (it contains barriers).
  constexpr int SX = QX + 2, SY = QY + 2, SZ = QZ + 2, SN = SX * SY * SZ;
  constexpr int NS = (SN + 255) / 256, NE = (QN + 255) / 256;
  static_assert(SN * sizeof(float) <= sizeof(qs[0]), "staged field block exceeds the plane slot");
  float fv[NS];
  auto fetch = [&](int tq) {
    const float* src = g.f + fpl3(g, tq) * plane;
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      int e = tid + 256 * i;
      asm volatile("" : "+v"(e));  // opaque: the index math is redone per plane, not held in registers across steps
      const int lx = e % SX, r = e / SX, ly = r % SY, lz = r / SY;
      const int cx = min(max(x0 - 1 + lx, 0), nx - 1), cy = min(max(y0 - 1 + ly, 0), ny - 1);
      const int cz = min(max(z0 - 1 + lz, 0), nz - 1);
      fv[i] = src[((long long)cz * ny + cy) * nx + cx];
    }
  };
  auto quantise = [&](int par) {
    float* fb = reinterpret_cast<float*>(&qs[par][0][0]);
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int e = tid + 256 * i;
      if (e < SN) fb[e] = fv[i];
    }
    __syncthreads();
    Q q[NE][3];
    unsigned f[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      int e = tid + 256 * i;
      asm volatile("" : "+v"(e));
      q[i][0] = q[i][1] = q[i][2] = 0;
      f[i] = 0x7Fu;
      if (e < QN) {
        const int lx = e % QX, r = e / QX, ly = r % QY, lz = r / QY;
        const int gx = x0 + lx, gy = y0 + ly, gz = z0 + lz;
        if (gx < nx && gy < ny && gz < nz) {
          const float* c = fb + ((lz + 1) * SY + (ly + 1)) * SX + (lx + 1);
          const float c0 = c[0];
          const float v0 = quant(diff3(c[-1], c0, c[1], gx, nx), g.qscale);
          const float v1 = quant(diff3(c[-SX], c0, c[SX], gy, ny), g.qscale);
          const float v2 = quant(diff3(c[-SX * SY], c0, c[SX * SY], gz, nz), g.qscale);
          q[i][0] = (Q)v0;
          q[i][1] = (Q)v1;
          q[i][2] = (Q)v2;
          f[i] = (v0 > 0.0f ? 1u : 0u) | (v0 < 0.0f ? 2u : 0u) | (v1 > 0.0f ? 4u : 0u) | (v1 < 0.0f ? 8u : 0u) |
                 (v2 > 0.0f ? 16u : 0u) | (v2 < 0.0f ? 32u : 0u) |
                 ((v0 == 0.0f && v1 == 0.0f && v2 == 0.0f) ? 64u : 0u);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NE; ++i) {
      const int e = tid + 256 * i;
      if (e < QN) {
        qs[par][0][e] = q[i][0];
        qs[par][1][e] = q[i][1];
        qs[par][2][e] = q[i][2];
        qf[par][e] = (unsigned char)f[i];
      }
    }
  };

  // Signs of a list of triangle types anchored at position e of plane ap.  Triangle type (M1, M2) anchored at p has its
  // vertices at the corners 0, a = M1, b = M1|M2 of p's unit 4-cube (corner bit 0 x, 1 y, 2 z, 3 t; a corner with the t
  // bit lies in the other plane).  Narrow: det(c0, ca, cb) = (c0 x ca) . cb.  The cross product of two quantised vectors
  // (below 2^20) is exact in binary64 (components below 2^41) and shared by every triangle with the same corner a; the
  // dot product carries at most 3u sum |p_i| of rounding error, so |s| > 4e-16 sum |p_i| fixes the sign, as
  // |s| is then beyond it.  Undecided triangles (every vanishing determinant among them) take the exact integer
  // evaluation and SoS afterwards.  Returns bit ti of each positive type.
  auto signs = [&](int ap, int e, auto list) -> unsigned long long {
    constexpr int N = decltype(list)::n;
    const int op = ap ^ 1;
    const int wx = e % WX, r = e / WX, wy = r % WY, wz = r / WY;
    const int base = (wz * QY + wy) * QX + wx;
    auto at = [&](int cm, int comp) -> Q {
      return qs[(cm >> 3) ? op : ap][comp][base + (((cm >> 2) & 1) * QY + ((cm >> 1) & 1)) * QX + (cm & 1)];
    };
    unsigned long long w = 0;
    if constexpr (WIDE) {
      const Q q0[3] = {at(0, 0), at(0, 1), at(0, 2)};
#pragma unroll 1
      for (int k = 0; k < N; ++k) {
        const int ti = decltype(list)::ti(k);
        const int cc = s_tcor[ti], a = cc & 15, b = cc >> 4;
        const Q qa[3] = {at(a, 0), at(a, 1), at(a, 2)};
        const Q qb[3] = {at(b, 0), at(b, 1), at(b, 2)};
        w |= (unsigned long long)sos3_positive<true, Q>(q0, qa, qb) << ti;
      }
      return w;
    } else {
      const double u0 = at(0, 0), u1 = at(0, 1), u2 = at(0, 2);
      unsigned long long slow = 0;
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const int ti = decltype(list)::ti(k);
        const int a = kTri3.m[ti][0], b = a | kTri3.m[ti][1];
        const double a0 = at(a, 0), a1 = at(a, 1), a2 = at(a, 2);
        const double X0 = __builtin_fma(u1, a2, -(u2 * a1));
        const double X1 = __builtin_fma(u2, a0, -(u0 * a2));
        const double X2 = __builtin_fma(u0, a1, -(u1 * a0));
        const double b0 = at(b, 0), b1 = at(b, 1), b2 = at(b, 2);
        const double p0 = X0 * b0, p1 = X1 * b1, p2 = X2 * b2;
        const double sdet = (p0 + p1) + p2;
        const double bound = ((fabs(p0) + fabs(p1)) + fabs(p2)) * 4e-16;
        w |= (unsigned long long)(sdet > 0.0) << ti;
        slow |= (unsigned long long)!(fabs(sdet) > bound) << ti;
      }
      while (slow) {
        const int ti = __ffsll((long long)slow) - 1;
        slow &= slow - 1;
        const int cc = s_tcor[ti], a = cc & 15, b = cc >> 4;
        const unsigned bit = sos3_exact_narrow((float)u0, (float)u1, (float)u2, at(a, 0), at(a, 1), at(a, 2), at(b, 0),
                                               at(b, 1), at(b, 2));
        w = (w & ~(1ull << ti)) | ((unsigned long long)bit << ti);
      }
      return w;
    }
  };

  const unsigned long long n_items = *n_runs;
  for (;;) {
    __syncthreads();  // the previous run's tests are done with the LDS
    if (tid == 0) s_item = atomicAdd(taken, 1ull);
    __syncthreads();
    const unsigned long long item = s_item;
    if (item >= n_items) break;
    const uint2 run = runs[item];
    const int t0 = (int)(run.y & 0xFFFFFFFu), t1 = t0 + 1 + (int)(run.y >> 28);
    bxl = (int)(run.x % (unsigned)ntx);
    x0 = bxl * TX3;
    y0 = (int)((run.x / (unsigned)ntx) % (unsigned)nty) * TY3;
    z0 = (int)(run.x / ((unsigned)ntx * (unsigned)nty)) * TZ3;
    fetch(t0);
    quantise(t0 & 1);
    for (int t = t0; t < t1; ++t) {
      const int par = t & 1, nxp = par ^ 1;
      const bool has_next = t + 1 < nt;
      __syncthreads();  // previous tests done
      if (has_next) {
        fetch(t + 1);
        quantise(nxp);
      }
      if (tid == 0) n_pos = n_anc = 0;
      if (tid < TY3 * TZ3) s_cnt[tid] = 0;
      __syncthreads();  // quantised planes and facts visible

      // anchors without a fact; the masks of the others are zero
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int a = tid + 256 * h;
        const int lx = a % TX3, r = a / TX3, ly = r % TY3, lz = r / TY3;
        const int gx = x0 + lx, gy = y0 + ly, gz = z0 + lz;
        const bool in = gx < nx && gy < ny && gz < nz;
        const int q0 = (lz * QY + ly) * QX + lx;
        unsigned f = 0x7Fu;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int o = q0 + ((c >> 2) * QY + ((c >> 1) & 1)) * QX + (c & 1);
          f &= qf[par][o];
          if (has_next) f &= qf[nxp][o];
        }
        const bool test = in && f == 0u;
        if (in && !test) masks[((mpl3(g, t) * nz + gz) * ny + gy) * nx + gx] = 0ull;
        const unsigned long long b = __ballot(test);
        if (lane == 0) left[a >> 6] = b;
        if (b) {
          int at = 0;
          if (lane == 0) at = atomicAdd(&n_anc, __popcll(b));
          at = __builtin_amdgcn_readfirstlane(at);
          if (test) anc[at + __popcll(b & ((1ull << lane) - 1ull))] = (unsigned short)a;
        }
      }
      __syncthreads();
      const int na = n_anc;
      if (na > 0) {  // uniform
        // positions whose words the anchors read: p + e(M1), M1 of at most two axes
        for (int e0 = 0; e0 < WN; e0 += 256) {
          const int e = e0 + tid;
          const int wx = e % WX, r = e / WX, wy = r % WY, wz = r / WY;
          bool need = false;
#pragma unroll
          for (int c = 0; c < 7; ++c) {
            const int lx = wx - (c & 1), ly = wy - ((c >> 1) & 1), lz = wz - (c >> 2);
            if (e < WN && lx >= 0 && lx < TX3 && ly >= 0 && ly < TY3 && lz >= 0 && lz < TZ3) {
              const int a = (lz * TY3 + ly) * TX3 + lx;
              need = need || ((left[a >> 6] >> (a & 63)) & 1ull);
            }
          }
          const unsigned long long b = __ballot(need);
          if (b) {
            int at = 0;
            if (lane == 0) at = atomicAdd(&n_pos, __popcll(b));
            at = __builtin_amdgcn_readfirstlane(at);
            if (need) {
              pos[at + __popcll(b & ((1ull << lane) - 1ull))] = (unsigned short)e;
              tw[e] = 0ull;
              to[e] = 0;
            }
          }
        }
        __syncthreads();
        const int np = n_pos;
        // every wavefront its list of types, 64 positions at a time
        for (int i = lane; i < np; i += 64) {
          const int e = pos[i];
          unsigned long long w = 0;
          if (wave == 0) {
            w = signs(par, e, OrdList{});
          } else if (wave == 1) {
            if (has_next) w = signs(par, e, ItvList<0>{});
          } else if (wave == 2) {
            if (has_next) w = signs(par, e, ItvList<kItvHalf>{});
          } else if (has_next) {
            const unsigned long long v = signs(nxp, e, OrdList{});
            unsigned o = 0;
#pragma unroll
            for (int k = 0; k < kOrdN; ++k) o |= (unsigned)((v >> kTriSplit.ord[k]) & 1ull) << k;
            to[e] = (unsigned short)o;
          }
          if (wave < 3 && w) atomicOr(&tw[e], w);
        }
        __syncthreads();

        // 60 tetrahedron tests per listed anchor
        for (int i = tid; i < na; i += 256) {
          const int a = anc[i];
          const int lx = a % TX3, r = a / TX3, ly = r % TY3, lz = r / TY3;
          const int gx = x0 + lx, gy = y0 + ly, gz = z0 + lz;
          const int w0 = (lz * WY + ly) * WX + lx;
          unsigned long long W[8];  // neighbour p + e(cm), spatial masks; only masks with at most two axes are used
          unsigned O[8];            // the same at t + 1, ordinal types
#pragma unroll
          for (int cm = 0; cm < 8; ++cm) {
            const int o = w0 + ((cm >> 2) * WY + ((cm >> 1) & 1)) * WX + (cm & 1);
            W[cm] = __popc((unsigned)cm) <= 2 ? tw[o] : 0ull;
            O[cm] = (__popc((unsigned)cm) <= 1 && has_next) ? to[o] : 0u;
          }
          unsigned long long m = 0;
#pragma unroll
          for (int k = 0; k < 60; ++k) {
            const int m1 = kTet3.m[k][0], m2 = kTet3.m[k][1], m3 = kTet3.m[k][2];
            // sides opposite v0..v3: (p+e(M1); M2, M3), (p; M1|M2, M3), (p; M1, M2|M3), (p; M1, M2); cofactor signs
            // -S0, +S1, -S2, +S3: punctured iff S1 = S3 and S0, S2 differ from them
            const int t0i = kTri3Index.idx[m2][m3];
            const unsigned long long e0 = (m1 & 8) ? (unsigned long long)((O[m1 & 7] >> ord_bit(t0i)) & 1u)
                                                   : (W[m1 & 7] >> t0i) & 1ull;
            const unsigned long long e1 = (W[0] >> kTri3Index.idx[m1 | m2][m3]) & 1ull;
            const unsigned long long e2 = (W[0] >> kTri3Index.idx[m1][m2 | m3]) & 1ull;
            const unsigned long long e3 = (W[0] >> kTri3Index.idx[m1][m2]) & 1ull;
            m |= (((e1 == e3) & (e0 != e1) & (e2 != e1)) ? 1ull : 0ull) << k;
          }
          unsigned long long valid = (1ull << 60) - 1ull;
          if (gx == nx - 1) valid &= ~kTetUseX;
          if (gy == ny - 1) valid &= ~kTetUseY;
          if (gz == nz - 1) valid &= ~kTetUseZ;
          if (t == nt - 1) valid &= ~kTetUseT;
          m &= valid;
          masks[((mpl3(g, t) * nz + gz) * ny + gy) * nx + gx] = m;
          if (m) atomicAdd(&s_cnt[lz * TY3 + ly], __popcll(m));
        }
      }
      __syncthreads();
      if (tid < TY3 * TZ3) {
        const int gy = y0 + tid % TY3, gz = z0 + tid / TY3;
        if (gy < ny && gz < nz) seg_cnt[((mpl3(g, t) * nz + gz) * ny + gy) * g.nxt + bxl] = s_cnt[tid];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------------------------
// Emission + links: the ids listed from the masks, then one lane per hit.
// ---------------------------------------------------------------------------------------------------------------
namespace {

struct Field3 {
  const float* f;
  int nx, ny, nz;
  long long plane;
  int ring;  // steps stored as a ring of `ring` slots (0: step t at t)
  // Binary32 gradient (c) and Jacobian stencil J (row-major 3x3, J[a][b] = d grad_a / d x_b) of vertex (x, y, z, t),
  // the same operations as the detection's stencils.  The 25 field values of the stencil are read from clamped
  // (in-grid) addresses, all independent loads; the clamped ones are never used (diff3 takes one-sided differences
  // at the first and last index).
  __device__ __forceinline__ void stencil(int x, int y, int z, int t, float c[3], float J[9]) const {
    const float* P = f + (long long)(ring ? t % ring : t) * plane;
    auto at = [&](int dx, int dy, int dz) {
      const int xx = min(max(x + dx, 0), nx - 1), yy = min(max(y + dy, 0), ny - 1), zz = min(max(z + dz, 0), nz - 1);
      return P[((long long)zz * ny + yy) * nx + xx];
    };
    const int N[3] = {nx, ny, nz}, I[3] = {x, y, z};
    float v[3][3][3];  // v[dz+1][dy+1][dx+1] on the unit neighbourhood (corners unused)
    float far[3][2];   // f(x -+ 2 e_a)
#pragma unroll
    for (int dz = -1; dz <= 1; ++dz)
#pragma unroll
      for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
        for (int dx = -1; dx <= 1; ++dx)
          v[dz + 1][dy + 1][dx + 1] = (dx != 0 && dy != 0 && dz != 0) ? 0.0f : at(dx, dy, dz);
    far[0][0] = at(-2, 0, 0);
    far[0][1] = at(2, 0, 0);
    far[1][0] = at(0, -2, 0);
    far[1][1] = at(0, 2, 0);
    far[2][0] = at(0, 0, -2);
    far[2][1] = at(0, 0, 2);
    // value at offset d (|d|_inf <= 1, at most two nonzero) and at -+2 e_a
    auto val = [&](int dx, int dy, int dz) { return v[dz + 1][dy + 1][dx + 1]; };
    // gradient component a at the vertex offset by o = s e_b (s in {-1, 0, 1})
    auto grad_at = [&](int a, int b, int sgn) -> float {
      int o[3] = {0, 0, 0};
      o[b] = sgn;
      int lo[3] = {o[0], o[1], o[2]}, hi[3] = {o[0], o[1], o[2]};
      lo[a] -= 1;
      hi[a] += 1;
      float fl, fh;
      if (a == b && sgn != 0) {  // neighbours at o -+ e_a: the centre and the far value
        fl = sgn < 0 ? far[a][0] : val(0, 0, 0);
        fh = sgn < 0 ? val(0, 0, 0) : far[a][1];
      } else {
        fl = val(lo[0], lo[1], lo[2]);
        fh = val(hi[0], hi[1], hi[2]);
      }
      return diff3(fl, val(o[0], o[1], o[2]), fh, I[a] + o[a], N[a]);
    };
#pragma unroll
    for (int a = 0; a < 3; ++a) c[a] = grad_at(a, 0, 0);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b)
        J[a * 3 + b] = diff3(grad_at(a, b, -1), c[a], grad_at(a, b, 1), I[b], N[b]);
  }
};

// Binary64 classification of the gradient's Jacobian (the Hessian) in the reference order: H = (J + J^T) * 0.5,
// s1 = trace, s2 = sum of principal 2x2 minors, s3 = det (first-row expansion); Descartes' rule on (1, s1, s2, s3)
// counts negative eigenvalues (exact for the real-rooted characteristic polynomial of a symmetric matrix).
__device__ __noinline__ int classify3_fp64(double mu0, double mu1, double mu2, double mu3, const float* J0,
                                           const float* J1, const float* J2, const float* J3) {
  double Jc[9];
#pragma unroll
  for (int e = 0; e < 9; ++e) {
    double s = mu0 * (double)J0[e];
    s = s + mu1 * (double)J1[e];
    s = s + mu2 * (double)J2[e];
    s = s + mu3 * (double)J3[e];
    Jc[e] = s;
  }
  double H[9];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      double s = Jc[a * 3 + b] + Jc[b * 3 + a];
      H[a * 3 + b] = s * 0.5;
    }
  const double s1 = (H[0] + H[4]) + H[8];
  const double m01 = H[0] * H[4] - H[1] * H[3];
  const double m02 = H[0] * H[8] - H[2] * H[6];
  const double m12 = H[4] * H[8] - H[5] * H[7];
  const double s2 = (m01 + m02) + m12;
  const double c0 = H[4] * H[8] - H[5] * H[7];
  const double c1 = H[3] * H[8] - H[5] * H[6];
  const double c2 = H[3] * H[7] - H[4] * H[6];
  const double s3 = (H[0] * c0 - H[1] * c1) + H[2] * c2;
  if (s3 == 0) return T_DEG;
  int changes = 0;
  bool prev_neg = false;
  const double seq[3] = {s1, s2, s3};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    if (seq[i] == 0) continue;
    const bool neg = seq[i] < 0;
    if (neg != prev_neg) ++changes;
    prev_neg = neg;
  }
  return changes == 0 ? T_MIN : (changes == 1 ? T_SADDLE1 : (changes == 2 ? T_SADDLE2 : T_MAX));
}

}  // namespace

// Face ids of the hits, at their output indices: one wavefront looks at 64 tile-steps, takes the segments with hits of
// the tile-steps that were tested, four 16-vertex segments at a time, and numbers the hits of a segment by a scan over
// its lanes.  (One lane per vertex of every 64-vertex chunk with hits, each working its hits off one by one with a
// search for its index, left nearly all lanes idle: 1.48 + 0.22 against 0.07 + 0.15 ms for the 108,184 hits of the
// 256^3 x 16 series.)
__global__ __launch_bounds__(256) void emit3d_ids(Grid3 g, const uint64_t* __restrict__ masks,
                                                  const int* __restrict__ seg_cnt,
                                                  const long long* __restrict__ seg_off,
                                                  long long* __restrict__ face_id) {
  const int nx = g.nx, ny = g.ny, nz = g.nz;
  const int ntx = (nx + TX3 - 1) / TX3, nty = (ny + TY3 - 1) / TY3, ntz = (nz + TZ3 - 1) / TZ3;
  const long long tiles = (long long)ntx * nty * ntz, all = tiles * (g.t_end - g.t_begin);
  const int lane = threadIdx.x & 63;
  const long long first = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64;
  const long long mine = min(first + lane, all - 1);
  const int tl = g.t_begin + (int)(mine / tiles);
  const unsigned tile_l = (unsigned)(mine % tiles);
  const bool tested = first + lane < all && g.cert[mpl3(g, tl) * tiles + tile_l] == 0;
  unsigned long long todo = __ballot(tested);
  while (todo) {
    const int e = __ffsll((long long)todo) - 1;
    todo &= todo - 1;
    const unsigned tile = (unsigned)__builtin_amdgcn_readlane((int)tile_l, e);
    const int t = __builtin_amdgcn_readlane(tl, e);
    const int x0 = (int)(tile % (unsigned)ntx) * TX3;
    const int y0 = (int)((tile / (unsigned)ntx) % (unsigned)nty) * TY3;
    const int z0 = (int)(tile / ((unsigned)ntx * (unsigned)nty)) * TZ3;
    // lanes 0-31: the tile's segments
    const int sy = y0 + (lane & 7), sz = z0 + ((lane >> 3) & 3);
    const bool row_in = lane < TY3 * TZ3 && sy < ny && sz < nz;
    const long long seg = ((mpl3(g, t) * nz + min(sz, nz - 1)) * ny + min(sy, ny - 1)) * g.nxt + x0 / SEG3;
    const unsigned so = (unsigned)seg_off[seg];
    unsigned hit = (unsigned)__ballot(row_in && seg_cnt[seg] > 0);
    while (hit) {
      int sg = -1;  // this lane's segment among the next four
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int s = hit ? __ffs((int)hit) - 1 : -1;
        hit &= hit - 1u;
        if ((lane >> 4) == k) sg = s;
      }
      const int sc = max(sg, 0);
      const int x = x0 + (lane & 15), y = y0 + (sc & 7), z = z0 + (sc >> 3);
      const bool in = sg >= 0 && x < nx;
      const long long v = ((long long)z * ny + y) * nx + x;
      const unsigned long long m = in ? masks[mpl3(g, t) * ((long long)nx * ny * nz) + v] : 0ull;
      unsigned c = (unsigned)__popcll(m), incl = c;
      incl += (unsigned)__builtin_amdgcn_update_dpp(0, (int)incl, 0x111, 0xf, 0xf, false);  // row_shr:1, 2, 4, 8
      incl += (unsigned)__builtin_amdgcn_update_dpp(0, (int)incl, 0x112, 0xf, 0xf, false);
      incl += (unsigned)__builtin_amdgcn_update_dpp(0, (int)incl, 0x114, 0xf, 0xf, false);
      incl += (unsigned)__builtin_amdgcn_update_dpp(0, (int)incl, 0x118, 0xf, 0xf, false);
      unsigned at = (unsigned)__builtin_amdgcn_ds_bpermute(sc << 2, (int)so) + incl - c;
      const long long id0 = ((long long)t * ((long long)nx * ny * nz) + v) * 60;
      for (unsigned long long r = m; r; r &= r - 1) face_id[at++] = id0 + (__ffsll((long long)r) - 1);
    }
  }
}

// Records and links, one lane per hit.
template <bool WIDE>
__global__ __launch_bounds__(256) void emit3d(Grid3 g, const uint64_t* __restrict__ masks,
                                              const long long* __restrict__ seg_off, long long first, long long n_hits,
                                              Out3 o, unsigned* __restrict__ status,
                                              unsigned long long* __restrict__ cnt) {
  const int nx = g.nx, ny = g.ny, nz = g.nz, nt = g.nt, nxt = g.nxt;
  const int lane = threadIdx.x & 63;
  const long long plane = (long long)nx * ny * nz;
  // the puncture mask of vertex u: zero where its detection tile-step was certified (those masks are not written)
  const long long ntx = (nx + TX3 - 1) / TX3, nty = (ny + TY3 - 1) / TY3, ntz = (nz + TZ3 - 1) / TZ3;
  auto certified_at = [&](int ux, int uy, int uz, int ut) -> bool {
    return g.cert[((mpl3(g, ut) * ntz + uz / TZ3) * nty + uy / TY3) * ntx + ux / TX3] != 0;
  };
  unsigned st = 0;
  unsigned long long n_deg = 0, n_linked = 0;

  // first-hit index of vertex u (global coordinates, inside the grid): segment offset + hits of the earlier
  // vertices of its 16-vertex segment
  auto first_hit = [&](int ux, int uy, int uz, int ut) -> unsigned {
    const long long seg = ((mpl3(g, ut) * nz + uz) * ny + uy) * nxt + ux / SEG3;
    unsigned off = (unsigned)seg_off[seg];
    const long long ub = mpl3(g, ut) * plane + ((long long)uz * ny + uy) * nx;
    const int x0s = (ux / SEG3) * SEG3;
#pragma unroll
    for (int k = 0; k < SEG3 - 1; ++k) {  // independent loads (clamped index), counted below ux only
      const int xx = x0s + k;
      const unsigned long long mk = masks[ub + min(xx, nx - 1)];
      off += xx < ux ? (unsigned)__popcll(mk) : 0u;
    }
    return off;
  };
  auto mask_at = [&](int ux, int uy, int uz, int ut) -> unsigned long long {
    if (certified_at(ux, uy, uz, ut)) return 0ull;
    return masks[mpl3(g, ut) * plane + ((long long)uz * ny + uy) * nx + ux];
  };

  Field3 F{g.f, nx, ny, nz, plane, g.f_ring};
  const long long i_hit = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i_hit < n_hits) {
    {
      const unsigned idx = (unsigned)(first + i_hit);
      const long long id = o.face_id[idx];
      const long long gidx = id / 60;  // global index of the anchor
      const int ty = (int)(id - gidx * 60);
      const int t = (int)(gidx / plane);
      const long long vofs = gidx - (long long)t * plane;
      const int x = (int)(vofs % nx), y = (int)((vofs / nx) % ny), z = (int)(vofs / ((long long)nx * ny));
      const int m1 = kTet3.m[ty][0], m2 = kTet3.m[ty][1], m3 = kTet3.m[ty][2];
      int vx[4], vy[4], vz[4], vt[4];
      const int cm[4] = {0, m1, m1 | m2, m1 | m2 | m3};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        vx[i] = x + (cm[i] & 1);
        vy[i] = y + ((cm[i] >> 1) & 1);
        vz[i] = z + ((cm[i] >> 2) & 1);
        vt[i] = t + ((cm[i] >> 3) & 1);
      }
      long long q[4][3];
      float J[4][9];
      bool wide = false;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float gr[3];
        F.stencil(vx[i], vy[i], vz[i], vt[i], gr, J[i]);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const float rq = quant(gr[c], g.qscale);
          if (!(fabsf(rq) < 1048576.0f)) wide = true;
          q[i][c] = (long long)rq;
        }
      }
      // exact cofactors C_i = (-1)^(3+i) det(columns without i)
      i128 C[4];
      C[0] = -det3x<WIDE, long long>(q[1], q[2], q[3]);
      C[1] = det3x<WIDE, long long>(q[0], q[2], q[3]);
      C[2] = -det3x<WIDE, long long>(q[0], q[1], q[3]);
      C[3] = det3x<WIDE, long long>(q[0], q[1], q[2]);
      const i128 D = (C[0] + C[1]) + (C[2] + C[3]);
      unsigned fl = wide ? FL_WIDE : 0u;
      double mu64[4];
      if (D == 0) {
        fl |= FL_DEGENERATE;
        ++n_deg;
#pragma unroll
        for (int i = 0; i < 4; ++i) mu64[i] = 1.0 / 4.0;
      } else {
        const double dD = (double)D;
#pragma unroll
        for (int i = 0; i < 4; ++i) mu64[i] = (double)C[i] / dD;
      }
      const int type = classify3_fp64(mu64[0], mu64[1], mu64[2], mu64[3], J[0], J[1], J[2], J[3]);
      float pos[4], muo[4];
      if (g.precision == 0) {
        float mu32[4];
        if (D == 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) mu32[i] = 0.25f;
        } else {
          const float fD = (float)D;
#pragma unroll
          for (int i = 0; i < 4; ++i) mu32[i] = (float)C[i] / fD;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int* vc = c == 0 ? vx : (c == 1 ? vy : (c == 2 ? vz : vt));
          float s = mu32[0] * (float)vc[0];
          s = s + mu32[1] * (float)vc[1];
          s = s + mu32[2] * (float)vc[2];
          s = s + mu32[3] * (float)vc[3];
          pos[c] = s;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) muo[i] = mu32[i];
      } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int* vc = c == 0 ? vx : (c == 1 ? vy : (c == 2 ? vz : vt));
          double s = mu64[0] * (double)vc[0];
          s = s + mu64[1] * (double)vc[1];
          s = s + mu64[2] * (double)vc[2];
          s = s + mu64[3] * (double)vc[3];
          pos[c] = (float)s;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) muo[i] = (float)mu64[i];
      }
      if (o.pos)
#pragma unroll
        for (int c = 0; c < 4; ++c) o.pos[(size_t)idx * 4 + c] = pos[c];
      if (o.mu)
#pragma unroll
        for (int c = 0; c < 4; ++c) o.mu[(size_t)idx * 4 + c] = muo[c];
      if (o.type) o.type[idx] = (uint8_t)type;
      if (o.flags) o.flags[idx] = (uint8_t)fl;

      // ---- links: the (at most two) pentachora holding this tetrahedron.  A pentachoron with chain
      // (c1, c2, c3, c4) anchored at c has sides: drop w0 -> (c + e_c1; c2, c3, c4), drop w1 -> (c; c1|c2, c3, c4),
      // drop w2 -> (c; c1, c2|c3, c4), drop w3 -> (c; c1, c2, c3|c4), drop w4 -> (c; c1, c2, c3).
      unsigned p0 = idx, p1 = idx;
      int np = 0;
      auto visit_cell = [&](int cx, int cy, int cz, int ct, int c1, int c2, int c3, int c4) {
        const int fx = cx + (c1 & 1), fy = cy + ((c1 >> 1) & 1), fz = cz + ((c1 >> 2) & 1), ft = ct + ((c1 >> 3) & 1);
        const unsigned long long bm = mask_at(cx, cy, cz, ct);
        const unsigned long long fm = mask_at(fx, fy, fz, ft);
        int found = 0;
        unsigned other = 0xFFFFFFFFu;
#pragma unroll
        for (int s = 0; s < 5; ++s) {
          int ti;
          if (s == 0)
            ti = kTet3Index.idx[c2][c3][c4];
          else if (s == 1)
            ti = kTet3Index.idx[c1 | c2][c3][c4];
          else if (s == 2)
            ti = kTet3Index.idx[c1][c2 | c3][c4];
          else if (s == 3)
            ti = kTet3Index.idx[c1][c2][c3 | c4];
          else
            ti = kTet3Index.idx[c1][c2][c3];
          const unsigned long long um = s == 0 ? fm : bm;
          if ((um >> ti) & 1ull) {
            ++found;
            const unsigned hi = (s == 0 ? first_hit(fx, fy, fz, ft) : first_hit(cx, cy, cz, ct)) +
                                (unsigned)__popcll(um & ((1ull << ti) - 1ull));
            if (hi != idx) other = hi;
          }
        }
        if (found != 2 || other == 0xFFFFFFFFu) {
          st |= ST_INVARIANT;
          return;
        }
        if (np == 0)
          p0 = other;
        else
          p1 = other;
        ++np;
        if (other > idx) ++n_linked;
      };
      const int b = m1 | m2 | m3;
      const int N[4] = {nx, ny, nz, nt};
      const int P[4] = {x, y, z, t};
      if (__popc((unsigned)m1) == 1 && __popc((unsigned)m2) == 1 && __popc((unsigned)m3) == 1) {
        const int a = 15 & ~b;  // missing axis
        const int ai = __ffs(a) - 1;
        if (P[ai] >= 1)
          visit_cell(x - (a & 1), y - ((a >> 1) & 1), z - ((a >> 2) & 1), t - ((a >> 3) & 1), a, m1, m2, m3);
        if (P[ai] + 1 <= N[ai] - 1) visit_cell(x, y, z, t, m1, m2, m3, a);
      } else if (__popc((unsigned)m1) == 2) {
        const int lo = m1 & -m1, hi = m1 - lo;
        visit_cell(x, y, z, t, lo, hi, m2, m3);
        visit_cell(x, y, z, t, hi, lo, m2, m3);
      } else if (__popc((unsigned)m2) == 2) {
        const int lo = m2 & -m2, hi = m2 - lo;
        visit_cell(x, y, z, t, m1, lo, hi, m3);
        visit_cell(x, y, z, t, m1, hi, lo, m3);
      } else {
        const int lo = m3 & -m3, hi = m3 - lo;
        visit_cell(x, y, z, t, m1, m2, lo, hi);
        visit_cell(x, y, z, t, m1, m2, hi, lo);
      }
      unsigned par0 = idx, smaller = 0, big_small = 0;
      if (np > 0 && p0 < idx) {
        ++smaller;
        par0 = p0;
        big_small = p0;
      }
      if (np > 1 && p1 < idx) {
        ++smaller;
        if (p1 < par0) par0 = p1;
        if (p1 > big_small) big_small = p1;
      }
      o.parent[idx] = par0;
      if (smaller == 2) {
        unsigned long long slot = atomicAdd(&cnt[CNT_WORK], 1ull);
        o.work[slot] = make_uint2(idx, big_small);
      }
    }
  }
  unsigned long long s2 = wave_sum64(n_deg), s3 = wave_sum64(n_linked);
  if (lane == 0) {
    if (s2) atomicAdd(&cnt[CNT_DEGEN], s2);
    if (s3) atomicAdd(&cnt[CNT_LINKED], s3);
  }
  if (st) atomicOr(status, st);
}

// Blocks along x of a launch of facts3d (256 lanes each; a launch holds less than 2^32 lanes along x).
constexpr int kFactsBlocks = 1 << 23;

hipError_t launch_facts3d(const Grid3& g, int most, unsigned long long* facts, uint2* runs, unsigned long long* n_runs,
                          unsigned* status, hipStream_t s) {
  static_assert(kPlanSteps <= 16, "a run holds its steps less one in four bits");
  if (!g.cert || most < 1 || most > kPlanSteps) return hipErrorInvalidValue;
  const long long nty = (g.ny + TY3 - 1) / TY3, ntz = (g.nz + TZ3 - 1) / TZ3;
  const int t_last = g.t_end < g.nt ? g.t_end : g.nt - 1;  // plane after the last step's
  const int nxb = (g.nx + 63) / 64;
  const int planes = nxb < kFactsBlocks ? kFactsBlocks / nxb : 1;  // of a launch
  for (int t = g.t_begin; t <= t_last; t += planes) {
    const int n = t_last - t + 1 < planes ? t_last - t + 1 : planes;
    facts3d<<<dim3((unsigned)nxb * (unsigned)n, (unsigned)((nty * ntz + 3) / 4)), 256, 0, s>>>(g, t, facts, status);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // whole runs for a lane where there are several lanes to a tile
  const int steps = g.t_end - g.t_begin <= kPlanSteps ? kPlanSteps : kPlanSteps / most * most;
  const long long lanes = cert3_plane(g) * ((g.t_end - g.t_begin + steps - 1) / steps);
  plan3d<<<(unsigned)((lanes + 255) / 256), 256, 0, s>>>(g, steps, most, facts, runs, n_runs);
  return hipGetLastError();
}

hipError_t launch_detect3d(const Grid3& g, bool wide, const uint2* runs, const unsigned long long* n_runs,
                           unsigned long long* taken, uint64_t* masks, int* seg_cnt, const unsigned* status,
                           hipStream_t s) {
  const long long steps = cert3_plane(g) * (g.t_end - g.t_begin);
  const unsigned blocks = (unsigned)(steps < 768 ? steps : 768);  // three workgroups to a CU
  if (wide)
    detect3d<true><<<blocks, 256, 0, s>>>(g, runs, n_runs, taken, masks, seg_cnt, status);
  else
    detect3d<false><<<blocks, 256, 0, s>>>(g, runs, n_runs, taken, masks, seg_cnt, status);
  return hipGetLastError();
}

hipError_t launch_emit3d(const Grid3& g, bool wide, const uint64_t* masks, const int* seg_cnt,
                         const long long* seg_off, long long first, long long n_hits, const Out3& o, unsigned* status,
                         unsigned long long* cnt, hipStream_t s) {
  if (!g.cert) return hipErrorInvalidValue;  // the certified-tile flags are read with the masks
  if (n_hits <= 0) return hipSuccess;
  const long long steps = cert3_plane(g) * (g.t_end - g.t_begin);
  emit3d_ids<<<(unsigned)((steps + 255) / 256), 256, 0, s>>>(g, masks, seg_cnt, seg_off, o.face_id);
  const unsigned blocks = (unsigned)((n_hits + 255) / 256);
  if (wide)
    emit3d<true><<<blocks, 256, 0, s>>>(g, masks, seg_off, first, n_hits, o, status, cnt);
  else
    emit3d<false><<<blocks, 256, 0, s>>>(g, masks, seg_off, first, n_hits, o, status, cnt);
  return hipGetLastError();
}

}  // namespace ftk
