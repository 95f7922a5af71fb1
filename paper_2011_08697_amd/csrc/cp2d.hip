// cp2d.hip -- critical-point tracking in 2D space + time on gfx950.
//
// Mesh: the Kuhn subdivision of the (x, y, t) grid (Sec. 3.3): per vertex 7 edge types, 12 triangle types (the
// tested faces) and 6 tetrahedra (the cells).  Pass 1 of Alg. 1 (left column) tests every triangle: it is
// punctured when the origin is interior to the triangle of its (quantised) vertex vectors, i.e. when the three
// signed cofactors of (v0 v1 v2 ; 1 1 1) agree (Sec. 4.3, Eq. 2).  Each cofactor is, up to a fixed sign, the 2x2
// determinant of the two vertex vectors of one edge, so a sign bit is computed once per edge (7 per vertex) and
// shared by the triangles in registers.
//
// Kernels:
//   detect2d  -- one wavefront per 64 x 8 tile, marching through a slab of steps with the vectors of two planes in
//                registers: gradient (scalar input), quantisation, the 7 edge signs of every vertex as wave masks and
//                the 12 triangle tests of every anchor on them; writes a 12-bit puncture mask per vertex and the hit
//                count of every 64-vertex row segment.
//   emit2d    -- (dense or small results) one workgroup per 64 x 8 tile, marching through a slab of steps: prefix sums
//                give each hit its output index (face ids come out sorted), and a lane per hit computes the sublocation
//                (Eq. 2) from the exact cofactors, the Jacobian type (FP32 with certified FP64 fallback), and the
//                union-find links of the hit's two tetrahedra (Alg. 1 pass 2), united in LDS within the tile.
//   emit2d_ids, emit2d_sparse -- (sparse results) the face ids listed from the masks, then a lane per listed hit: the
//                same records, links into parents and link slots.
#include "common.h"
#include "internal.h"

namespace ftk {

namespace {

constexpr int TX = 64;

constexpr float kNarrow2 = 16777216.0f;  // 2^24: cofactors and their sum stay exact in binary64 below it

__device__ __forceinline__ int fpl(const Grid2& g, int t) { return g.f_ring ? t % g.f_ring : t; }
__device__ __forceinline__ int mpl(const Grid2& g, int t) { return g.m_ring ? t % g.m_ring : t; }

}  // namespace

// ---------------------------------------------------------------------------------------------------------------
// Pass 1: detection.
//
// A wavefront owns a tile of 64 x 8 anchors (lane = x) and marches it through the steps of a slab, with no LDS and no
// barrier: the quantised vectors of the planes t and t + 1 stay in registers (nine rows: the tile's and the one
// above), the x + 1 neighbour of a lane comes from a whole-wave DPP shift, and the one column past lane 63 is held
// lane-parallel (lane r + 1 = row r), so it costs one extra vector per plane and not one per row.  The field rows of
// the plane after next are in flight while a step is evaluated.
//
// The sign of an edge determinant is decided in binary64: a quantised component is the rounding of a binary32 value,
// so it has at most 24 significant bits at any magnitude, the product a1 b0 is exact and fma(a0, b1, -a1 b0) rounds
// the exact difference once -- its sign, zero included, is the exact one over the whole accepted range (|q| < 2^62).
// One variant therefore serves what the emission splits into a narrow and a 128-bit form.
//
// The sign of a determinant is the top bit of its high word, and the 12 triangle tests of an anchor are bit-parallel on
// words that these bits are spread into (TriSpread).  (Wave masks of the signs in scalar registers, with the tests as
// 64-bit scalar operations, were bound by scalar issue: 0.57 against 0.43 ms on 1024 x 1024 x 100.)
//
// Eight rows a wavefront need 160 registers (three wavefronts per SIMD); four rows run four wavefronts but load,
// quantise and test more halo (0.49 against 0.43 ms), and eight rows held to 128 registers spill (0.76 ms).
//
// Measured against tiles of 64 x 16 staged in LDS with one workgroup barrier per pass: 1024 x 1024 x 100 scalar noise
// 1.01 -> 0.43 ms, 4096 x 4096 x 50 vector 3.77 -> 2.25 ms, 1021 x 769 x 40 vector beyond 2^24 (then a narrow run and
// a 128-bit one) 0.69 -> 0.13 ms, 64 x 64 x 10 scalar 84 -> 9 us.
//
// A step whose vectors carry a sign fact over the tile skips the edges and the tests: when one component is of one
// strict sign at every vertex of both planes it keeps that sign under the symbolic perturbation (its entries move by
// infinitesimals only), so the origin is outside every triangle; with every vector zero each edge determinant takes
// the perturbation's last, negative term, so the three cofactor signs never agree.
//
// Bound: reading the field and writing the masks for sparse fields (4096 x 4096 x 50: 8.4 GB of them at 3.7 TB/s, 13.4 GB
// with the halos read again), VALU issue (about 75 operations a row and step) otherwise.
// ---------------------------------------------------------------------------------------------------------------
namespace {

constexpr int kDetRows = kDetectRows;      // anchor rows per wavefront
static_assert(8 % kDetRows == 0, "workgroups of 8, 16 and 32 rows are whole wavefronts");
constexpr int kDetVec = kDetRows + 1;      // rows of vectors
constexpr int kDetRaw = kDetRows + 3;      // scalar field rows behind them

typedef unsigned long long u64;

// v of lane i - 1 / i + 1 within the first 16 lanes (lanes without a source keep their own)
__device__ __forceinline__ float row_prev(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x111, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_next(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0x101, 0xf, 0xf, false));
}

// Field values of one plane behind the vectors of a tile.  Scalar: rows y0-1 .. y0+9 and, lane i = row y0-1+i, the
// columns x0-1, x0+63, x0+64, x0+65.  Vector: rows y0 .. y0+8 of both components and the column x0+64.
template <bool VEC>
struct DetRaw {
  float r[VEC ? 2 * kDetVec : kDetRaw];
  float h[VEC ? 2 : 4];
};
// Quantised vectors of one plane: q[row][component], the column x0+64 in h (lane r + 1 = row r).
struct DetPlane {
  float q[kDetVec][2];
  float h[2];
};

// Smallest of z and the magnitudes of the high words of two determinants, read as binary32: zero iff one of the
// determinants is zero (a nonzero one is an integer, whose high word is that of a value of at least one).
__device__ __forceinline__ float zero_seen(float z, double d, double e) {
  asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(z) : "v"(__double2hiint(d)), "v"(__double2hiint(e)));
  return z;
}

// The 12 triangle tests of an anchor run bit-parallel on three words with one bit per triangle type (M1, M2): E0, E1,
// E2 hold the sign of the edge opposite v0, v1, v2 -- the edges M2 of p + e(M1), M1|M2 of p and M1 of p.  The cofactor
// signs +S, -S, +S agree iff E0 = E2 != E1.  Each edge sign (a full lane mask) is spread over the types it serves by
// one and-or with a constant: fields of one word for E2 (bits 0-11) and E1 (bits 16-27) of the anchor's own edges, and
// the E0 bits of the anchors below it in x, y and t.
struct TriSpread {
  unsigned own[8];   // by edge mask: E2 bits, E1 bits << 16
  unsigned g[8];     // E0 bits at the anchor x - 1
  unsigned h[8];     // E0 bits at the anchor y - 1
  unsigned k[8];     // E0 bits at the anchor t - 1 (same x, y)
  unsigned gt[8];    // E0 bits at x - 1, t - 1
  unsigned ht[8];    // E0 bits at y - 1, t - 1
  unsigned gxy[8];   // E0 bits at x - 1, y - 1
};
constexpr TriSpread build_tri_spread() {
  TriSpread r{};
  for (int ty = 0; ty < 12; ++ty) {
    const int m1 = kTri2.m[ty][0], m2 = kTri2.m[ty][1];
    r.own[m1] |= 1u << ty;
    r.own[m1 | m2] |= 1u << (ty + 16);
    unsigned* at = m1 == 1 ? r.g : (m1 == 2 ? r.h : (m1 == 3 ? r.gxy : (m1 == 4 ? r.k : (m1 == 5 ? r.gt : r.ht))));
    at[m2] |= 1u << ty;
  }
  return r;
}
constexpr TriSpread kSpread = build_tri_spread();
constexpr unsigned kGOwn = kSpread.g[2] | kSpread.g[4] | kSpread.g[6] | kSpread.gt[2];  // E0 bits from x + 1, same row
constexpr unsigned kGXy = kSpread.gxy[4];                                                // from x + 1, y + 1
static_assert((kGOwn & kGXy) == 0 && kSpread.gxy[4] != 0, "distinct E0 bits in the word passed along x");
constexpr unsigned types_using(int axis) { return (unsigned)types_using_axis(kTri2, axis); }

__device__ __forceinline__ unsigned spread(int neg, unsigned bits, unsigned acc) { return ((unsigned)neg & bits) | acc; }

}  // namespace

template <bool VEC>
__device__ __forceinline__ void detect2d_wave(const Grid2& g, int TT, int bx, int y0, int bz,
                                              uint16_t* __restrict__ masks, int* __restrict__ seg_cnt,
                                              unsigned* __restrict__ status) {
  const int lane = lane_id();
  const int nx = g.nx, ny = g.ny, nt = g.nt;
  const int x0 = bx * TX, gx = x0 + lane;
  const int t0 = g.t_begin + bz * TT;
  const int t1 = min(t0 + TT, g.t_end);
  const long long plane = (long long)nx * ny;
  const unsigned xb = 4u * (unsigned)min(gx, nx - 1);  // byte offset in a row: 32-bit lane offsets to scalar addresses
  const long long row_bytes = 4ll * nx;
  // All loads use clamped (in-grid) addresses.  A clamped neighbour equals the value at the grid's edge, which turns
  // the central difference into the one-sided one there; only its factor differs.
  const float one = g.qscale, half = 0.5f * g.qscale;  // powers of two: exact factors
  const int one_bits = __builtin_amdgcn_readfirstlane(__float_as_int(one));  // scalar: chosen per row
  const int half_bits = __builtin_amdgcn_readfirstlane(__float_as_int(half));
  const float sx = (gx == 0 || gx == nx - 1) ? one : half;
  const float sxh = x0 + 64 == nx - 1 ? one : half;
  const int hy = y0 - 1 + lane;  // grid row of this lane's part of the column past the tile
  const float syh = (hy <= 0 || hy >= ny - 1) ? one : half;
  const int hyc = min(max(y0 - 1 + min(lane, kDetRaw - 1), 0), ny - 1);
  const u64 below = ~0ull >> (63 - min(63, nx - 1 - x0));            // lanes inside the grid
  const u64 h_in = x0 + 64 < nx ? ((1ull << min(kDetVec, ny - y0)) - 1ull) << 1 : 0ull;

  // The tile's first row, opaque to the compiler: what is derived from it per row (addresses, row masks) is redone
  // per step on the scalar unit and not held across steps, where it would not fit the scalar registers.
  auto first_row = [&]() -> int {
    int y = y0;
    asm volatile("" : "+s"(y));
    return y;
  };
  auto load = [&](int t, DetRaw<VEC>& w) {
    const int y0 = first_row();
    const float* P = g.f + (long long)fpl(g, t) * (VEC ? 2 * plane : plane);
    constexpr int first = VEC ? 0 : -1;  // rows y0 - 1 (scalar) or y0 (vector) and up
    const long long comp = plane * 4;
#pragma unroll
    for (int i = 0; i < (VEC ? kDetVec : kDetRaw); ++i) {
      const char* row = (const char*)P + (long long)min(max(y0 + first + i, 0), ny - 1) * row_bytes;
      if constexpr (VEC) {
        w.r[2 * i] = *(const float*)(row + xb);
        w.r[2 * i + 1] = *(const float*)(row + comp + xb);
      } else {
        w.r[i] = *(const float*)(row + xb);
      }
    }
    if constexpr (VEC) {
      const long long o = (long long)hyc * nx + min(x0 + 64, nx - 1);
      w.h[0] = P[o];
      w.h[1] = P[o + plane];
    } else {
      const float* H = P + (long long)hyc * nx;
      w.h[0] = H[max(x0 - 1, 0)];
      w.h[1] = H[min(x0 + 63, nx - 1)];
      w.h[2] = H[min(x0 + 64, nx - 1)];
      w.h[3] = H[min(x0 + 65, nx - 1)];
    }
  };

  unsigned st = 0;
  float nonfinite = 0.0f;  // NaN once an infinity or NaN was loaded
  // Quantised vectors of a loaded plane; returns its sign facts over the tile (bit 0 every x component > 0, bit 1
  // every one < 0, bits 2 and 3 the y component, bit 4 every vector zero).
  auto quantise = [&](const DetRaw<VEC>& w, DetPlane& p) -> unsigned {
    const int y0 = first_row();
    if constexpr (VEC) {
#pragma unroll
      for (int r = 0; r < kDetVec; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          nonfinite = __builtin_fmaf(w.r[2 * r + c], 0.0f, nonfinite);
          p.q[r][c] = rintf(w.r[2 * r + c] * one);
        }
      p.h[0] = rintf(w.h[0] * one);
      p.h[1] = rintf(w.h[1] * one);
    } else {
#pragma unroll
      for (int r = 0; r < kDetVec; ++r) {
        const float f = w.r[r + 1];
        nonfinite = __builtin_fmaf(f, 0.0f, nonfinite);
        const float lo = from_prev(f, lane_value(w.h[0], r + 1)), hi = from_next(f, lane_value(w.h[2], r + 1));
        const int y = y0 + r;
        p.q[r][0] = rintf((hi - lo) * sx);
        p.q[r][1] = rintf((w.r[r + 2] - w.r[r]) * __int_as_float((y == 0 || y >= ny - 1) ? one_bits : half_bits));
      }
      p.h[0] = rintf((w.h[3] - w.h[1]) * sxh);
      p.h[1] = rintf((row_next(w.h[2]) - row_prev(w.h[2])) * syh);
    }
    float mn[2] = {p.q[0][0], p.q[0][1]}, mx[2] = {p.q[0][0], p.q[0][1]};
#pragma unroll
    for (int r = 1; r < kDetVec; ++r)  // rows past the grid repeat its last row, or are zero (no fact then)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        mn[c] = fminf(mn[c], p.q[r][c]);
        mx[c] = fmaxf(mx[c], p.q[r][c]);
      }
    const float big = fmaxf(fmaxf(mx[0], -mn[0]), fmaxf(mx[1], -mn[1]));
    if (big >= kNarrow2) st |= big >= 4611686018427387904.0f ? (ST_WIDE | ST_RANGE) : ST_WIDE;
    const u64 off = ~below, hoff = ~h_in;  // lanes outside the grid
    const u64 p0 = (__ballot(mn[0] > 0.0f) | off) & (__ballot(p.h[0] > 0.0f) | hoff);
    const u64 n0 = (__ballot(mx[0] < 0.0f) | off) & (__ballot(p.h[0] < 0.0f) | hoff);
    const u64 p1 = (__ballot(mn[1] > 0.0f) | off) & (__ballot(p.h[1] > 0.0f) | hoff);
    const u64 n1 = (__ballot(mx[1] < 0.0f) | off) & (__ballot(p.h[1] < 0.0f) | hoff);
    const u64 z = ((__ballot(fmaxf(mx[0], -mn[0]) == 0.0f) & __ballot(fmaxf(mx[1], -mn[1]) == 0.0f)) | off) &
                  ((__ballot(p.h[0] == 0.0f) & __ballot(p.h[1] == 0.0f)) | hoff);
    const unsigned f = (p0 == ~0ull ? 1u : 0u) | (n0 == ~0ull ? 2u : 0u) | (p1 == ~0ull ? 4u : 0u) |
                       (n1 == ~0ull ? 8u : 0u) | (z == ~0ull ? 16u : 0u);
    return f;
  };

  // ~0 where the edge (a, b) is negative, ties by the perturbation
  auto edge = [&](double a0, double a1, double b0, double b1) -> int {
    const double d = edge_det(a0, a1, b0, b1);
    const int tie = edge_tie(a1, b0, b1), neg = edge_neg(d);
    return d == 0.0 ? tie : neg;
  };
  // Edge signs of plane t carried from one step to the next, already spread: the own word of the ordinal edges x, y, xy
  // of each row (row 8: x only) with a copy of the x and y signs in its free bits, and, lane-parallel, the y edges of
  // the column x0+64.
  constexpr int kBitX = 12, kBitY = 13;
  constexpr unsigned kOwnX = kSpread.own[1] | 1u << kBitX, kOwnY = kSpread.own[2] | 1u << kBitY, kOwnXY = kSpread.own[3];
  unsigned ord[kDetVec];
  int ohy = 0;
  auto ordinals = [&](const DetPlane& p) {
    double a0 = p.q[0][0], a1 = p.q[0][1];
    double c0 = from_next(p.q[0][0], lane_value(p.h[0], 1)), c1 = from_next(p.q[0][1], lane_value(p.h[1], 1));
    int nx_ = edge(a0, a1, c0, c1);
#pragma unroll
    for (int r = 0; r < kDetRows; ++r) {
      const double d0 = p.q[r + 1][0], d1 = p.q[r + 1][1];
      c0 = from_next(p.q[r + 1][0], lane_value(p.h[0], r + 2));
      c1 = from_next(p.q[r + 1][1], lane_value(p.h[1], r + 2));
      ord[r] = spread(nx_, kOwnX, spread(edge(a0, a1, d0, d1), kOwnY, spread(edge(a0, a1, c0, c1), kOwnXY, 0u)));
      nx_ = edge(d0, d1, c0, c1);
      a0 = d0;
      a1 = d1;
    }
    ord[kDetRows] = spread(nx_, kOwnX, 0u);
    ohy = edge(p.h[0], p.h[1], row_next(p.h[0]), row_next(p.h[1]));
  };

  DetRaw<VEC> raw;
  DetPlane A, B;
  load(t0, raw);
  unsigned factA = quantise(raw, A);
  if (t0 + 1 < nt) load(t0 + 1, raw);
  bool have_ord = false;  // ord and ohy hold plane t's edges
  const unsigned valid_x = gx < nx - 1 ? 0xFFFu : (gx < nx ? 0xFFFu & ~types_using(1) : 0u);
  for (int t = t0; t < t1; ++t) {
    const bool has_next = t + 1 < nt;
    unsigned factB = 31u;
    if (has_next) {
      factB = quantise(raw, B);
      if (t + 1 < t1 && t + 2 < nt) load(t + 2, raw);
    }
    const bool certified = (factA & factB) != 0u;  // uniform
    const int y0 = first_row();
    const long long seg0 = ((long long)mpl(g, t) * ny + y0) * g.nxt + bx;
    char* mrow = (char*)(masks + ((long long)mpl(g, t) * ny + y0) * nx);
    const unsigned mb = 2u * (unsigned)gx;
    int cnt = 0;  // lane r: hits of row r
    if (certified) {
#pragma unroll
      for (int r = 0; r < kDetRows; ++r) {
        if (y0 + r < ny && gx < nx) *(uint16_t*)(mrow + mb) = 0;
        mrow += row_bytes / 2;
      }
      have_ord = false;
    } else {
      if (!have_ord) ordinals(A);
      if (!has_next) B = A;  // no step t + 1: only the ordinal triangles are valid
      // the column x0+64, lane r + 1 = row r: the word its edges y, t, yt (and y of plane t + 1) pass to lane 63
      unsigned hg;
      {
        const double ha0 = A.h[0], ha1 = A.h[1], hb0 = B.h[0], hb1 = B.h[1];
        const double hn0 = row_next(B.h[0]), hn1 = row_next(B.h[1]);
        const int hby = edge(hb0, hb1, hn0, hn1);
        hg = spread(ohy, kSpread.g[2], 0u);
        hg = spread(edge(ha0, ha1, hb0, hb1), kSpread.g[4] | kGXy, hg);
        hg = spread(edge(ha0, ha1, hn0, hn1), kSpread.g[6], hg);
        hg = spread(hby, kSpread.gt[2], hg);
        ohy = hby;
      }
      // rolling over the rows: b, c = plane t+1 at (x, r), (x+1, r); d, f = at row r + 1; a, e = plane t at (x, r), r + 1
      double b0 = B.q[0][0], b1 = B.q[0][1];
      double c0 = from_next(B.q[0][0], lane_value(B.h[0], 1)), c1 = from_next(B.q[0][1], lane_value(B.h[1], 1));
      double a0 = A.q[0][0], a1 = A.q[0][1];
      int T = edge(a0, a1, b0, b1), XT = edge(a0, a1, c0, c1), bX = edge(b0, b1, c0, c1);
      unsigned e0_prev = 0, own_prev = 0;  // the row below, whose E0 still lacks the bits of this row
#pragma unroll
      for (int r = 0; r <= kDetRows; ++r) {
        // row r of the window: edges t, xt of plane t, x of plane t+1 (T, XT, bX); rows 0..7 also y, xy, yt, xyt
        int YT = 0, XYT = 0, bY = 0, bXY = 0, Tn = 0, XTn = 0, bXn = 0;
        if (r < kDetRows) {
          const double d0 = B.q[r + 1][0], d1 = B.q[r + 1][1];
          const double f0 = from_next(B.q[r + 1][0], lane_value(B.h[0], r + 2));
          const double f1 = from_next(B.q[r + 1][1], lane_value(B.h[1], r + 2));
          const double e0 = A.q[r + 1][0], e1 = A.q[r + 1][1];
          const double dYT = edge_det(a0, a1, d0, d1), dXYT = edge_det(a0, a1, f0, f1);
          const double dbY = edge_det(b0, b1, d0, d1), dbXY = edge_det(b0, b1, f0, f1);
          const double dbX = edge_det(d0, d1, f0, f1);
          const double dT = edge_det(e0, e1, d0, d1), dXT = edge_det(e0, e1, f0, f1);
          YT = edge_neg(dYT);
          XYT = edge_neg(dXYT);
          bY = edge_neg(dbY);
          bXY = edge_neg(dbXY);
          bXn = edge_neg(dbX);
          Tn = edge_neg(dT);
          XTn = edge_neg(dXT);
          float z = zero_seen(1.0f, dYT, dXYT);
          z = zero_seen(z, dbY, dbXY);
          z = zero_seen(z, dbX, dT);
          z = zero_seen(z, dXT, dXT);
          auto settle = [](int& neg, double d, int tie) { neg = d == 0.0 ? tie : neg; };
          if (__ballot(z == 0.0f)) {  // exact zeros are rare on generic data
            settle(YT, dYT, edge_tie(a1, d0, d1));
            settle(XYT, dXYT, edge_tie(a1, f0, f1));
            settle(bY, dbY, edge_tie(b1, d0, d1));
            settle(bXY, dbXY, edge_tie(b1, f0, f1));
            settle(bXn, dbX, edge_tie(d1, f0, f1));
            settle(Tn, dT, edge_tie(e1, d0, d1));
            settle(XTn, dXT, edge_tie(e1, f0, f1));
          }
          a0 = e0;
          a1 = e1;
          b0 = d0;
          b1 = d1;
        }
        const unsigned o = ord[r];
        // what the row's edges give to the anchors at x - 1 (and x - 1, y - 1)
        unsigned gw = ((o >> kBitY) & 1u) * kSpread.g[2];
        gw = spread(T, kSpread.g[4] | kGXy, gw);
        gw = spread(YT, kSpread.g[6], gw);
        gw = spread(bY, kSpread.gt[2], gw);
        gw = from_next(gw, (unsigned)__builtin_amdgcn_readlane((int)hg, r + 1));
        if (r > 0) {
          // the row below is complete with this row's x, t, xt (and x of plane t+1) edges
          unsigned hw = ((o >> kBitX) & 1u) * kSpread.h[1];
          hw = spread(T, kSpread.h[4], hw);
          hw = spread(XT, kSpread.h[5], hw);
          hw = spread(bX, kSpread.ht[1], hw);
          const unsigned E0 = e0_prev | (gw & kGXy) | hw;
          // uniform: types that need the next row or step (rows past the grid: none)
          const int y = y0 + r - 1;
          const unsigned vt = has_next ? 0xFFFu : 0xFFFu & ~types_using(4);
          const unsigned vy = y < ny - 1 ? 0xFFFu : (y < ny ? 0xFFFu & ~types_using(2) : 0u);
          const unsigned m = ~(E0 ^ own_prev) & ((own_prev >> 16) ^ E0) & valid_x & (vt & vy);
          if (__ballot(m != 0u)) {
            const unsigned n = wave_sum((unsigned)__popc(m));
            cnt |= __builtin_amdgcn_inverse_ballot_w64(1ull << (r - 1)) ? (int)n : 0;
          }
          if (y < ny && gx < nx) *(uint16_t*)(mrow + mb) = (uint16_t)m;
          mrow += row_bytes / 2;
        }
        if (r < kDetRows) {
          unsigned own = spread(T, kSpread.own[4], o);
          own = spread(XT, kSpread.own[5], own);
          own = spread(YT, kSpread.own[6], own);
          own_prev = spread(XYT, kSpread.own[7], own);
          unsigned kw = spread(bX, kSpread.k[1], gw & kGOwn);
          kw = spread(bY, kSpread.k[2], kw);
          e0_prev = spread(bXY, kSpread.k[3], kw);
          ord[r] = spread(bX, kOwnX, spread(bY, kOwnY, spread(bXY, kOwnXY, 0u)));
        } else {
          ord[r] = spread(bX, kOwnX, 0u);
        }
        T = Tn;
        XT = XTn;
        bX = bXn;
        __builtin_amdgcn_sched_barrier(0);  // rows are not interleaved: their registers would not fit
      }
      have_ord = true;
    }
    if (lane < kDetRows && y0 + lane < ny) seg_cnt[seg0 + (long long)lane * g.nxt] = cnt;
    A = B;
    factA = factB;
  }
  if (!(nonfinite == 0.0f)) st |= ST_NONFINITE;
  if (st) atomicOr(status, st);
}

// grid = (ceil(nx / 64), ceil(ny / rows per block), ceil(nt / TT)), block = 64 lanes x (rows per block / rows per wavefront) wavefronts
template <bool VEC>
__global__ __launch_bounds__(64 * 32 / kDetRows) __attribute__((amdgpu_waves_per_eu(3))) void detect2d(Grid2 g, int TT, uint16_t* __restrict__ masks,
                                                int* __restrict__ seg_cnt, unsigned* __restrict__ status) {
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int y0 = ((int)blockIdx.y * (int)(blockDim.x >> 6) + w) * kDetRows;
  if (y0 < g.ny) detect2d_wave<VEC>(g, TT, blockIdx.x, y0, blockIdx.z, masks, seg_cnt, status);
}

// ---------------------------------------------------------------------------------------------------------------
// Pass 1b: emission + pass 2 links.
// Same tiling as detection (64 x TY anchors, marching over a slab of TT steps).  The vector field of planes t and
// t+1 (gradient of the scalar, or the input vector) is kept in LDS with a 1-cell halo; quantised vectors and
// Jacobians of a hit's vertices are formed from it on the fly, with the same binary32 stencils as pass 1.  Each
// wavefront takes one row segment at a time and processes its hits hit-parallel (hit j of the segment on lane
// j mod 64), so output writes are contiguous.
// ---------------------------------------------------------------------------------------------------------------
namespace {

// Side tables of the triangle types, built at compile time.
// kTri2Pack[ty] = M1 | M2 << 4.  kTri2Cof[ty][k] describes the k-th tetrahedron holding a triangle of type ty
// (Alg. 1 pass 2; the cells holding a triangle, the side-of query of Sec. 3.2): bits 0-1 existence rule (1 always,
// 2 when p_a >= 1, 3 when p_a + 1 <= N_a - 1), bits 2-3 the axis a, then its three other sides as (anchor slot,
// type) in 7-bit fields.
enum { NB_SELF = 0, NB_MX, NB_PX, NB_MY, NB_PY, NB_MT, NB_PT };

struct Tri2Tables {
  unsigned char pack[12];
  unsigned cof[12][2];
};

constexpr int slot_minus(int ab) { return ab == 1 ? NB_MX : (ab == 2 ? NB_MY : NB_MT); }
constexpr int slot_plus(int ab) { return ab == 1 ? NB_PX : (ab == 2 ? NB_PY : NB_PT); }
constexpr int axis_of(int ab) { return ab == 1 ? 0 : (ab == 2 ? 1 : 2); }

// A tetrahedron with chain (c1, c2, c3) anchored at c has sides: drop w0 -> (c + e_c1; c2, c3),
// drop w1 -> (c; c1|c2, c3), drop w2 -> (c; c1, c2|c3), drop w3 -> (c; c1, c2).  at_minus: c = p - e_c1.
constexpr unsigned cof_word(int ty, bool at_minus, int rule, int axis, int c1, int c2, int c3) {
  const int first = at_minus ? NB_SELF : slot_plus(c1);
  const int base = at_minus ? slot_minus(c1) : NB_SELF;
  const int st[4] = {first, base, base, base};
  const int tt[4] = {kTri2Index.idx[c2][c3], kTri2Index.idx[c1 | c2][c3], kTri2Index.idx[c1][c2 | c3],
                     kTri2Index.idx[c1][c2]};
  unsigned w = (unsigned)rule | ((unsigned)axis << 2);
  int k = 0;
  for (int s = 0; s < 4; ++s) {
    if (st[s] == NB_SELF && tt[s] == ty) continue;  // the triangle itself
    w |= (unsigned)(st[s] | (tt[s] << 3)) << (4 + 7 * k);
    ++k;
  }
  return w;
}

constexpr Tri2Tables build_tri2_tables() {
  Tri2Tables r{};
  for (int ty = 0; ty < 12; ++ty) {
    const int m1 = kTri2.m[ty][0], m2 = kTri2.m[ty][1];
    r.pack[ty] = (unsigned char)(m1 | (m2 << 4));
    if (popc_c(m1) == 1 && popc_c(m2) == 1) {
      const int a = 7 & ~(m1 | m2);
      r.cof[ty][0] = cof_word(ty, true, 2, axis_of(a), a, m1, m2);
      r.cof[ty][1] = cof_word(ty, false, 3, axis_of(a), m1, m2, a);
    } else if (popc_c(m1) == 2) {
      const int lo = m1 & -m1, hi = m1 - lo;
      r.cof[ty][0] = cof_word(ty, false, 1, 0, lo, hi, m2);
      r.cof[ty][1] = cof_word(ty, false, 1, 0, hi, lo, m2);
    } else {
      const int lo = m2 & -m2, hi = m2 - lo;
      r.cof[ty][0] = cof_word(ty, false, 1, 0, m1, lo, hi);
      r.cof[ty][1] = cof_word(ty, false, 1, 0, m1, hi, lo);
    }
  }
  return r;
}
constexpr Tri2Tables kTri2Tab = build_tri2_tables();

// The same tables as 24 words for an LDS copy: word 2 ty + k = cof[ty][k] (bits 0-24), and pack[ty] in bits 25-31
// of word 2 ty.  Per-hit reads from LDS leave the vector memory counter to the stores, which a global table read
// would have to wait for.
struct Tri2Words {
  unsigned w[24];
};
constexpr Tri2Words build_tri2_words() {
  Tri2Words r{};
  for (int ty = 0; ty < 12; ++ty) {
    r.w[2 * ty] = kTri2Tab.cof[ty][0] | ((unsigned)kTri2Tab.pack[ty] << 25);
    r.w[2 * ty + 1] = kTri2Tab.cof[ty][1];
  }
  return r;
}
static_assert(build_tri2_words().w[0] >> 25 == kTri2Tab.pack[0], "pack field");
__constant__ Tri2Words kTri2WordsDev = build_tri2_words();

// Neighbour anchor slots (SELF, MX, PX, MY, PY, MT, PT) in 2-bit fields: column + 1 and row + 1 of the anchor.
constexpr unsigned kSlotCol = 0x1561u, kSlotRow = 0x1615u;

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

}  // namespace

// Local union-find in LDS over the hits of one tile and a run of consecutive steps (a chunk); the smallest local id
// (= smallest hit index) is the root.
__device__ __forceinline__ unsigned lfind(unsigned* lp, unsigned x) {
  unsigned p = lp[x];
  while (p != x) {
    unsigned gp = lp[p];
    if (gp != p) lp[x] = gp;
    x = p;
    p = gp;
  }
  return x;
}

__device__ __forceinline__ void lunite(unsigned* lp, unsigned a, unsigned b) {
  unsigned ra = lfind(lp, a), rb = lfind(lp, b);
  while (ra != rb) {
    if (ra < rb) {
      unsigned t = ra;
      ra = rb;
      rb = t;
    }
    unsigned old = atomicCAS(&lp[ra], ra, rb);
    if (old == ra) return;
    ra = lfind(lp, old);
    rb = lfind(lp, rb);
  }
}

// Union-find on the global parent array restricted to the hits of one workgroup's tile and slab: during emission
// nothing outside the workgroup reads or writes these parents, so workgroup-scope atomics (served by the CU's own
// caches) are coherent for them.
__device__ __forceinline__ unsigned wg_load(const unsigned* p, unsigned i) {
  return __hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ unsigned wg_find(unsigned* parent, unsigned x) {
  unsigned p = wg_load(parent, x);
  while (p != x) {
    const unsigned gp = wg_load(parent, p);
    if (gp != p) __hip_atomic_store(parent + x, gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    x = p;
    p = gp;
  }
  return x;
}

__device__ __forceinline__ void wg_unite(unsigned* parent, unsigned a, unsigned b) {
  unsigned ra = wg_find(parent, a), rb = wg_find(parent, b);
  while (ra != rb) {
    if (ra < rb) {
      const unsigned t = ra;
      ra = rb;
      rb = t;
    }
    unsigned expected = ra;
    if (__hip_atomic_compare_exchange_strong(parent + ra, &expected, rb, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP))
      return;
    ra = wg_find(parent, expected);
    rb = wg_find(parent, rb);
  }
}

// Edge list staging: links that leave the tile/chunk are collected in LDS and appended to the global list in
// batches (one global atomic per batch; same-address atomics serialise at one L2 channel).
constexpr int kEdgeStage = 496;

// Wave-aggregated append of (idx, partner) for the active lanes with want == true: one LDS add reserves the
// wave's slots; slots past the stage capacity go straight to the global list (one global add for them).
__device__ __forceinline__ void append_edge(bool want, unsigned idx, unsigned partner, uint2* stage, int* stage_n,
                                            int scap, uint2* work, unsigned long long* counter) {
  const unsigned long long bal = __ballot(want);
  if (bal == 0) return;
  const int lane = lane_id();
  const int leader = __ffsll((long long)bal) - 1;
  const int k = __popcll(bal);
  int pos = 0;
  if (lane == leader) pos = atomicAdd(stage_n, k);
  pos = __builtin_amdgcn_readlane(pos, leader);
  const int first_over = pos > scap ? pos : scap;  // first slot number routed to the global list
  const int n_over = pos + k - first_over;
  unsigned long long gpos = 0;
  if (n_over > 0) {
    if (lane == leader) gpos = atomicAdd(counter, (unsigned long long)n_over);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)gpos, leader);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(gpos >> 32), leader);
    gpos = ((unsigned long long)hi << 32) | lo;
  }
  if (want) {
    const int slot = pos + __popcll(bal & ((1ull << lane) - 1ull));
    const uint2 e = make_uint2(idx, partner);
    if (slot < scap)
      stage[slot] = e;
    else
      work[gpos + (unsigned long long)(slot - first_over)] = e;
  }
}

// Block-wide sum of a per-thread value (256 threads), returned on thread 0.
__device__ __forceinline__ unsigned long long block_sum256(unsigned long long v, unsigned long long* red) {
  v = wave_sum64(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  unsigned long long s = 0;
  if (threadIdx.x == 0) s = red[0] + red[1] + red[2] + red[3];
  return s;
}

// Record of one hit (Eq. 2, Sec. 4.1): exact cofactors of (v0 v1 v2 ; 1 1 1) from the quantised vectors qf of the
// triangle's vertices, barycentric coordinates mu, position, and the Jacobian type (FP32 with a certified error
// bound, else FP64); written at output index idx - o.gbase.  J holds the binary32 Jacobian stencil of each vertex.
template <bool WIDE>
__device__ __forceinline__ void hit_record2(const Grid2& g, const Out2& o, const float (&qf)[3][2],
                                            const float (&J)[3][4], bool wide, bool vector, int ax, int y, int t,
                                            int ty, int dx1, int dy1, int dt1, int dx2, int dy2, int dt2,
                                            unsigned idx, unsigned long long& n_fp64, unsigned long long& n_deg) {
  const long long plane = (long long)g.nx * g.ny;
  // exact cofactors of (v0 v1 v2 ; 1 1 1): C_i = (-1)^i det(columns without i)
  double Cd[3], Dd;
  bool degenerate;
  if (!WIDE) {
    // |q| < 2^24: every cofactor is an integer below 2^49 and D below 2^51, exact in binary64
    auto det2d = [](float a0, float a1, float b0, float b1) {
      const double p = (double)a1 * (double)b0;
      return __builtin_fma((double)a0, (double)b1, -p);
    };
    Cd[0] = det2d(qf[1][0], qf[1][1], qf[2][0], qf[2][1]);
    Cd[1] = -det2d(qf[0][0], qf[0][1], qf[2][0], qf[2][1]);
    Cd[2] = det2d(qf[0][0], qf[0][1], qf[1][0], qf[1][1]);
    Dd = (Cd[0] + Cd[1]) + Cd[2];
    degenerate = (Dd == 0.0);
  } else {
    long long q[3][2];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      q[i][0] = (long long)qf[i][0];
      q[i][1] = (long long)qf[i][1];
    }
    i128 C[3];
    C[0] = (i128)q[1][0] * q[2][1] - (i128)q[1][1] * q[2][0];
    C[1] = -((i128)q[0][0] * q[2][1] - (i128)q[0][1] * q[2][0]);
    C[2] = (i128)q[0][0] * q[1][1] - (i128)q[0][1] * q[1][0];
    const i128 D = C[0] + C[1] + C[2];
    degenerate = (D == 0);
#pragma unroll
    for (int i = 0; i < 3; ++i) Cd[i] = (double)C[i];
    Dd = (double)D;
  }
  unsigned fl = wide ? FL_WIDE : 0u;
  if (degenerate) {
    fl |= FL_DEGENERATE;
    ++n_deg;
  }
  float mu32[3];
  double mu64[3];
  int type = -1;
  if (g.precision == 0) {
    if (degenerate) {
      mu32[0] = mu32[1] = mu32[2] = 1.0f / 3.0f;
    } else {
      // hardware reciprocal (1 ulp): mu carries at most five roundings, inside the classifier's bound
      const float rD = __builtin_amdgcn_rcpf((float)Dd);
#pragma unroll
      for (int i = 0; i < 3; ++i) mu32[i] = (float)Cd[i] * rD;
    }
    type = classify2_fp32(mu32, J, vector);
  }
  if (g.precision != 0 || type < 0) {
    if (degenerate) {
      mu64[0] = mu64[1] = mu64[2] = 1.0 / 3.0;
    } else {
#pragma unroll
      for (int i = 0; i < 3; ++i) mu64[i] = Cd[i] / Dd;
    }
    type = classify2_fp64(mu64, J, vector);
    if (g.precision == 0) {
      fl |= FL_FP64;
      ++n_fp64;
    }
  }
  float pos[3], muo[3];
  const float cx0 = (float)ax, cy0 = (float)y, ct0 = (float)t;
  if (g.precision == 0) {
    float sx = mu32[0] * cx0;
    sx = sx + mu32[1] * (cx0 + dx1);
    sx = sx + mu32[2] * (cx0 + dx2);
    float sy = mu32[0] * cy0;
    sy = sy + mu32[1] * (cy0 + dy1);
    sy = sy + mu32[2] * (cy0 + dy2);
    float stt = mu32[0] * ct0;
    stt = stt + mu32[1] * (ct0 + dt1);
    stt = stt + mu32[2] * (ct0 + dt2);
    pos[0] = sx;
    pos[1] = sy;
    pos[2] = stt;
#pragma unroll
    for (int i = 0; i < 3; ++i) muo[i] = mu32[i];
  } else {
    const double X = ax, Y = y, T = t;
    double sx = mu64[0] * X;
    sx = sx + mu64[1] * (X + dx1);
    sx = sx + mu64[2] * (X + dx2);
    double sy = mu64[0] * Y;
    sy = sy + mu64[1] * (Y + dy1);
    sy = sy + mu64[2] * (Y + dy2);
    double stt = mu64[0] * T;
    stt = stt + mu64[1] * (T + dt1);
    stt = stt + mu64[2] * (T + dt2);
    pos[0] = (float)sx;
    pos[1] = (float)sy;
    pos[2] = (float)stt;
#pragma unroll
    for (int i = 0; i < 3; ++i) muo[i] = (float)mu64[i];
  }
  const long long agid = (long long)t * plane + (long long)y * g.nx + ax;
  const size_t oi = idx - o.gbase;
  if (o.face_id) o.face_id[oi] = agid * 12 + ty;  // null: listed already
  if (o.pos) {
    o.pos[oi * 3 + 0] = pos[0];
    o.pos[oi * 3 + 1] = pos[1];
    o.pos[oi * 3 + 2] = pos[2];
  }
  if (o.mu) {
    o.mu[oi * 3 + 0] = muo[0];
    o.mu[oi * 3 + 1] = muo[1];
    o.mu[oi * 3 + 2] = muo[2];
  }
  if (o.type) o.type[oi] = (uint8_t)type;
  if (o.flags) o.flags[oi] = (uint8_t)fl;
}

template <int TY, bool WIDE>
__device__ __forceinline__ void emit2d_tile(const Grid2& g, int TT, int bx, int by, int bz,
                                            const uint16_t* __restrict__ masks, const int* __restrict__ seg_cnt,
                                            const long long* __restrict__ seg_off, const Out2& o,
                                            unsigned* __restrict__ status,
                                            unsigned long long* __restrict__ cnt,
                                            unsigned long long* __restrict__ work_cnt) {
  constexpr int GW = TX + 3, GH = TY + 3;  // vector field: x0-1 .. x0+TX+1, y0-1 .. y0+TY+1
  constexpr int FW = TX + 5, FH = TY + 5;  // scalar field: x0-2 .. x0+TX+2
  constexpr int RW = TX + 2, RH = TY + 2;  // mask slices: x0-1 .. x0+TX, y0-1 .. y0+TY
  constexpr int CAP = 2048;                // local union-find capacity (hits)
  constexpr int MAXTT = kEmitSteps;        // step tables (TT <= kEmitSteps)
  __shared__ float2 gs[2][GH * GW];
  // Mask slices of steps t-1, t, t+1 (ring slot = step mod 3) over the tile's anchors with a one-anchor halo: hit
  // masks, first hit of each anchor relative to its row segment's first hit (left halo column: minus its hit
  // count, right halo column: the segment's total), and the segments' first hit indices.
  __shared__ unsigned short rm[3][RH * RW];
  __shared__ short rx[3][RH * RW];
  __shared__ unsigned rb[3][RH];
  __shared__ int s_slice[3];  // step held by each ring slot
  // hit j of the wave's current row -> anchor lane | type << 6; between hit phases the same LDS holds the scalar
  // field of a plane being loaded
  __shared__ __align__(16) unsigned short s_lane[4][12 * 64];
  static_assert(FH * FW * sizeof(float) <= sizeof(s_lane), "scalar plane staging exceeds the hit map");
  float* const fs = reinterpret_cast<float*>(&s_lane[0][0]);
  __shared__ unsigned lpar[CAP];
  // non-empty row segments of the current chunk in local-id order: first local id and first global hit index
  __shared__ unsigned s_segl[MAXTT * TY], s_segg[MAXTT * TY];
  __shared__ int s_nseg;
  __shared__ unsigned lbase[MAXTT][TY];  // local id of the first hit of (step t - t0, row)
  __shared__ unsigned s_rc[MAXTT][TY], s_ro[MAXTT][TY];  // hits and first hit index of (step t - t0, row)
  __shared__ int s_chunk_t0, s_chunk_n, s_flush, s_global, s_plane_lbase, s_plane_total;
  __shared__ int s_have[2];  // step held by each field buffer (-1: none)
  __shared__ uint2 s_stage[kEdgeStage];
  __shared__ int s_stage_n;
  __shared__ unsigned long long s_red[4];
  __shared__ unsigned s_cof[24];  // triangle side words (Tri2Words)

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int x0 = bx * TX, y0 = by * TY;
  const int t0 = g.t_begin + bz * TT;
  const int t1 = min(t0 + TT, g.t_end);
  const int nx = g.nx, ny = g.ny, nt = g.nt, nxt = g.nxt;
  const long long plane = (long long)nx * ny;
  const bool vector = g.kind != 0;
  // workgroup-local capacities: the LDS sizes, or tiny ones under the FTK_DEBUG_SMALL_LDS test hook
  const int cap = (g.debug & 1) ? 128 : CAP;
  const int scap = (g.debug & 1) ? 8 : kEdgeStage;
  unsigned st = 0;
  unsigned long long n_fp64 = 0, n_deg = 0, n_linked = 0;


  // vector field of plane t into gs[par] (field loads from clamped in-grid addresses, all in flight together).  Cells
  // outside the grid repeat the nearest vertex, so that a one-sided difference is the plain one at its full step.
  auto load_plane = [&](int t, int par) {
    if (!vector) {
      constexpr int NL = (FH * FW + 255) / 256;
      const float* src = g.f + (long long)fpl(g, t) * plane;
      float fv[NL];
      bool in[NL];
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        int e = tid + 256 * i;
        asm volatile("" : "+v"(e));  // opaque: the index math is redone per plane, not held across steps
        const int ly = e / FW, lx = e - ly * FW;
        const int gx = x0 - 2 + lx, gy = y0 - 2 + ly;
        in[i] = e < FH * FW && gx >= 0 && gx < nx && gy >= 0 && gy < ny;
        fv[i] = src[(long long)min(max(gy, 0), ny - 1) * nx + min(max(gx, 0), nx - 1)];
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int e = tid + 256 * i;
        if (e < FH * FW) fs[e] = in[i] ? fv[i] : 0.0f;
      }
      __syncthreads();
      for (int e = tid; e < GH * GW; e += 256) {
        int ly = e / GW, lx = e - ly * GW;
        const int gx = min(max(x0 - 1 + lx, 0), nx - 1), gy = min(max(y0 - 1 + ly, 0), ny - 1);
        const float* r = &fs[(gy - y0 + 2) * FW + (gx - x0 + 2)];
        gs[par][e] = make_float2(diff3(r[-1], r[0], r[1], gx, nx), diff3(r[-FW], r[0], r[FW], gy, ny));
      }
    } else {
      constexpr int NL = (GH * GW + 255) / 256;
      const float* su = g.f + (long long)fpl(g, t) * 2 * plane;
      const float* sv = su + plane;
      float f0[NL], f1[NL];
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        int e = tid + 256 * i;
        asm volatile("" : "+v"(e));
        const int ly = e / GW, lx = e - ly * GW;
        const int gx = x0 - 1 + lx, gy = y0 - 1 + ly;
        const long long k = (long long)min(max(gy, 0), ny - 1) * nx + min(max(gx, 0), nx - 1);
        f0[i] = su[k];
        f1[i] = sv[k];
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int e = tid + 256 * i;
        if (e < GH * GW) gs[par][e] = make_float2(f0[i], f1[i]);
      }
    }
  };

  // mask slice of step s (zero outside [0, nt)) into ring slot (s + 3) % 3
  auto load_slice = [&](int s) {
    constexpr int NL = (RH * RW + 255) / 256;
    const int slot = (s + 3) % 3;
    const bool ok = s >= 0 && s < nt;
    const long long mp = ok ? (long long)mpl(g, s) : 0;
    unsigned short mv[NL];
    bool in[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {  // clamped addresses, loads in flight together
      int e = tid + 256 * i;
      asm volatile("" : "+v"(e));
      const int r = e / RW, c = e - r * RW;
      const int y = y0 - 1 + r, x = x0 - 1 + c;
      in[i] = ok && e < RH * RW && y >= 0 && y < ny && x >= 0 && x < nx;
      mv[i] = masks[(mp * ny + min(max(y, 0), ny - 1)) * nx + min(max(x, 0), nx - 1)];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int e = tid + 256 * i;
      if (e < RH * RW) rm[slot][e] = in[i] ? mv[i] : (unsigned short)0;
    }
    if (tid < RH) {
      const int y = y0 - 1 + tid;
      rb[slot][tid] = (ok && y >= 0 && y < ny) ? (unsigned)seg_off[(mp * ny + y) * nxt + bx] : 0u;
    }
  };
  // per-anchor offsets of a loaded slice: one wavefront per row
  auto scan_slice = [&](int slot) {
    for (int r = wave; r < RH; r += 4) {
      const unsigned c = __popc((unsigned)rm[slot][r * RW + 1 + lane]);
      const unsigned incl = wave_incl_scan(c);
      rx[slot][r * RW + 1 + lane] = (short)(incl - c);
      if (lane == 63) rx[slot][r * RW + RW - 1] = (short)incl;
      if (lane == 0) rx[slot][r * RW] = (short)(-(int)__popc((unsigned)rm[slot][r * RW]));
    }
  };

  // Local root of x in the flushing chunk: a local id, or CAP + i once the set has been attached to the set of an
  // earlier chunk of this tile whose global root sits in stage slot i.
  auto lroot = [&](unsigned x) -> unsigned {
    for (;;) {
      const unsigned p = lpar[x];
      if (p == x || p >= (unsigned)CAP) return p;
      x = p;
    }
  };
  // Before the parents are written, each remaining local root r of segment k holds kRootTag + k (above every local
  // id and stage marker), so that its hit index s_segg[k] + (r - s_segl[k]) needs no search.
  constexpr unsigned kRootTag = 0x8000u;
  static_assert(CAP + kEdgeStage <= (int)kRootTag, "root tags above local ids and stage markers");
  // local id of a hit of the current chunk from its global index (segments are in increasing global order)
  auto seg_search = [&](const unsigned* key, unsigned v) -> int {
    int lo = 0, hi = s_nseg;  // last segment with key <= v
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (key[mid] <= v)
        lo = mid;
      else
        hi = mid;
    }
    return lo;
  };
  // Write the parent of every hit of the chunk.  Links staged as (earlier partner, hit) go from the chunk's first
  // step to an earlier chunk of this tile, whose parents are final: the hit's local set is attached to the
  // partner's global root (two such roots met by one set are united in place), and each hit of the chunk gets its
  // set's global root, or the hit index of its local root.  Attached links stay in the stage as no-op (R, R).
  auto flush = [&]() {
    __syncthreads();  // parents written so far by this workgroup are visible to it
    const int n = s_chunk_n, nseg = s_nseg;
    {
      // The chunk's local links: the hit loop made each hit's first smaller partner its parent (a forest: parents
      // point to smaller local ids) and left a second one in the entry's high half.  Take those out, point every
      // entry at its root (path halving), then unite the second partners through the shallow trees.
      unsigned sec[CAP / 256];
#pragma unroll
      for (int k = 0; k < CAP / 256; ++k) {
        const int i = tid + 256 * k;
        sec[k] = 0u;
        if (i < n) {
          const unsigned e = lpar[i];
          sec[k] = e >> 16;
          if (sec[k]) lpar[i] = e & 0xFFFFu;
        }
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < CAP / 256; ++k) {
        const int i = tid + 256 * k;
        if (i < n) lpar[i] = lfind(lpar, (unsigned)i);
      }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < CAP / 256; ++k)
        if (sec[k]) lunite(lpar, (unsigned)(tid + 256 * k), sec[k] - 1u);
      __syncthreads();
    }
    const int nst = s_stage_n < scap ? s_stage_n : scap;
    for (int i = tid; i < nst; i += 256) {
      const uint2 e = s_stage[i];
      if (e.x >= e.y) continue;  // (hit, smaller partner): for the global list
      // The partner's parent was written by an earlier flush of this workgroup: an ancestor of its set, which
      // serves as the attachment point (the load is in flight during the local search).
      const unsigned R = wg_load(o.parent, e.x);
      const int k = seg_search(s_segg, e.y);
      unsigned r = lroot(s_segl[k] + (e.y - s_segg[k]));
      s_stage[i] = make_uint2(R, R);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      for (;;) {
        if (r >= (unsigned)CAP) {
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
          wg_unite(o.parent, R, s_stage[r - CAP].x);
          break;
        }
        const unsigned old = atomicCAS(&lpar[r], r, (unsigned)(CAP + i));
        if (old == r) break;
        r = old >= (unsigned)CAP ? old : lroot(old);
      }
    }
    __syncthreads();
    for (int k = wave; k < nseg; k += 4) {
      const unsigned l0 = s_segl[k], l1 = k + 1 < nseg ? s_segl[k + 1] : (unsigned)n;
      for (unsigned li = l0 + lane; li < l1; li += 64)
        if (lpar[li] == li) lpar[li] = kRootTag + (unsigned)k;
    }
    __syncthreads();
    for (int k = wave; k < nseg; k += 4) {
      const unsigned l0 = s_segl[k], l1 = k + 1 < nseg ? s_segl[k + 1] : (unsigned)n, g0 = s_segg[k];
      for (unsigned li = l0 + lane; li < l1; li += 64) {
        unsigned x = li, p = lpar[li];
        while (p < (unsigned)CAP) {
          x = p;
          p = lpar[x];
        }
        unsigned target;
        if (p >= kRootTag) {
          const unsigned kr = p - kRootTag;
          target = s_segg[kr] + (x - s_segl[kr]);
        } else {
          target = s_stage[p - CAP].x;
        }
        o.parent[g0 + (li - l0)] = target;
      }
    }
  };
  // Move the staged links (hit, smaller partner) to the global list.  Links staged as (partner, hit) wait in the
  // stage for their chunk's flush (compacted to the front); attached ones, (R, R), are dropped.  One wavefront.
  auto drain = [&]() {
    __syncthreads();  // nobody reads the stage any more (a flush may just have)
    const int n = s_stage_n < scap ? s_stage_n : scap;  // slots past the capacity went to the list
    if (wave == 0) {
      unsigned n_out = 0;
      for (int b = 0; b < n; b += 64) {
        bool out = false;
        if (b + lane < n) {
          const uint2 e = s_stage[b + lane];
          out = e.x > e.y;
        }
        n_out += (unsigned)__popcll(__ballot(out));
      }
      unsigned long long gb = 0;
      if (lane == 0 && n_out) gb = atomicAdd(work_cnt, (unsigned long long)n_out);
      gb = ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(gb >> 32), 0) << 32) |
           (unsigned)__builtin_amdgcn_readlane((int)(unsigned)gb, 0);
      const unsigned long long below = (1ull << lane) - 1ull;
      unsigned wo = 0, wk = 0;
      for (int b = 0; b < n; b += 64) {
        uint2 e = make_uint2(0u, 0u);
        bool out = false, keep = false;
        if (b + lane < n) {
          e = s_stage[b + lane];
          out = e.x > e.y;
          keep = e.x < e.y;
        }
        const unsigned long long bo = __ballot(out), bk = __ballot(keep);
        if (out) o.work[gb + wo + (unsigned)__popcll(bo & below)] = e;
        if (keep) s_stage[wk + (unsigned)__popcll(bk & below)] = e;  // below b + 64: not read again
        wo += (unsigned)__popcll(bo);
        wk += (unsigned)__popcll(bk);
      }
      if (lane == 0) s_stage_n = (int)wk;
    }
    __syncthreads();
  };

  if (tid == 0) {
    s_chunk_t0 = t0;
    s_chunk_n = 0;
    s_nseg = 0;
    s_stage_n = 0;
    s_have[0] = s_have[1] = -1;
    s_slice[0] = s_slice[1] = s_slice[2] = -2;
  }
  if (tid < 24) s_cof[tid] = kTri2WordsDev.w[tid];
  // hit counts and offsets of this tile's row segments for all its steps, read once: empty steps are skipped
  // without touching their masks
  for (int i = tid; i < (t1 - t0) * TY; i += 256) {
    const int dt = i / TY, r = i - dt * TY, y = y0 + r;
    unsigned c = 0, b = 0;
    if (y < ny) {
      const long long k = ((long long)mpl(g, t0 + dt) * ny + y) * nxt + bx;
      c = (unsigned)seg_cnt[k];
      b = (unsigned)seg_off[k];
    }
    s_rc[dt][r] = c;
    s_ro[dt][r] = b;
  }
  __syncthreads();

  for (int t = t0; t < t1; ++t) {
    const int par = t & 1;
    {
      unsigned tot = 0;
#pragma unroll
      for (int r = 0; r < TY; ++r) tot += s_rc[t - t0][r];
      if (tot == 0) continue;  // uniform
    }
    __syncthreads();
    // ring slots still to be filled for steps t-1, t, t+1 (read before any slot is rewritten)
    const bool need_prev = s_slice[(t + 2) % 3] != t - 1;
    const bool need_cur = s_slice[t % 3] != t;
    const bool need_next = s_slice[(t + 1) % 3] != t + 1;
    if (tid == 0) {
      unsigned tot = 0;
      for (int r = 0; r < TY; ++r) tot += s_rc[t - t0][r];
      s_plane_total = (int)tot;
      s_flush = (s_chunk_n > 0 && (s_chunk_n + (int)tot > cap || t - s_chunk_t0 >= MAXTT)) ? 1 : 0;
    }
    __syncthreads();
    if (s_flush) {
      flush();
      __syncthreads();
      if (tid == 0) {
        s_chunk_n = 0;
        s_nseg = 0;
        s_chunk_t0 = t;
      }
      __syncthreads();
    }
    if (s_stage_n > scap / 2) drain();
    if (tid == 0) {
      const int tot = s_plane_total;
      if (tot > cap) {  // too many hits for the local structure: this step links through the global list only
        s_global = 1;
        s_chunk_t0 = t + 1;
        s_chunk_n = 0;
        s_nseg = 0;
      } else {
        s_global = 0;
        if (s_chunk_n == 0) s_chunk_t0 = t;
        s_plane_lbase = s_chunk_n;
        unsigned run = (unsigned)s_chunk_n;
        int ns = s_nseg;
        for (int r = 0; r < TY; ++r) {
          lbase[t - t0][r] = run;
          const unsigned c = s_rc[t - t0][r];
          if (c) {  // non-empty segments only: both keys strictly increase (rows past the grid have no base)
            s_segl[ns] = run;
            s_segg[ns] = s_ro[t - t0][r];
            ++ns;
          }
          run += c;
        }
        s_nseg = ns;
        s_chunk_n = (int)run;
      }
    }
    __syncthreads();
    const bool plane_global = s_global != 0;
    const int chunk_t0 = s_chunk_t0;
    if (s_plane_total == 0) continue;  // uniform: nothing anchored in this tile at this step
    if (!plane_global)
      for (int i = tid; i < s_plane_total; i += 256) lpar[s_plane_lbase + i] = (unsigned)(s_plane_lbase + i);
    // mask slices of steps t-1, t, t+1 (only those not held yet), then the vector field of steps t and t+1
    if (need_prev) load_slice(t - 1);
    if (need_cur) load_slice(t);
    if (need_next) load_slice(t + 1);
    __syncthreads();
    if (need_prev) scan_slice((t + 2) % 3);
    if (need_cur) scan_slice(t % 3);
    if (need_next) scan_slice((t + 1) % 3);
    if (tid == 0) {
      s_slice[(t + 2) % 3] = t - 1;
      s_slice[t % 3] = t;
      s_slice[(t + 1) % 3] = t + 1;
    }
    if (s_have[par] != t) {
      load_plane(t, par);
      __syncthreads();
      if (tid == 0) s_have[par] = t;
    }
    if (t + 1 < nt && s_have[par ^ 1] != t + 1) {
      load_plane(t + 1, par ^ 1);
      __syncthreads();
      if (tid == 0) s_have[par ^ 1] = t + 1;
    }
    __syncthreads();

    for (int ly = wave; ly < TY; ly += 4) {
      const int y = y0 + ly;
      if (y >= ny) break;
      const unsigned total = s_rc[t - t0][ly];
      if (total == 0) continue;
      const unsigned base = s_ro[t - t0][ly];
      const unsigned row_lbase = plane_global ? 0u : lbase[t - t0][ly];
      const int cur = t % 3;
      // ring slot of each neighbour anchor slot (2-bit fields, as kSlotCol)
      const unsigned rsw = (unsigned)cur * 0x155u | (unsigned)((t + 2) % 3) << 10 | (unsigned)((t + 1) % 3) << 12;
      // local id of a smaller partner = its hit index + (local base - first hit index) of its row segment: the
      // same anchor or x - 1 (this row), y - 1, or step t - 1 (read only when that segment is in this chunk)
      const unsigned d_self = row_lbase - base;
      const unsigned d_my = (!plane_global && ly > 0) ? lbase[t - t0][ly - 1] - s_ro[t - t0][ly - 1] : 0u;
      const unsigned d_mt = (!plane_global && t - 1 >= chunk_t0) ? lbase[t - 1 - t0][ly] - s_ro[t - 1 - t0][ly] : 0u;
      // link class per smaller-partner slot (2-bit fields): 0 united here, 1 global list, 2 staged for the flush
      const unsigned cls_mt = t - 1 >= chunk_t0 ? 0u : (t - 1 >= t0 ? 2u : 1u);
      const unsigned clw = (ly == 0 ? 1u << (2 * NB_MY) : 0u) | cls_mt << (2 * NB_MT);

      // hit -> (anchor lane, type) map of this row segment (wavefront-private)
      {
        const int a = (ly + 1) * RW + 1 + lane;
        unsigned m = rm[cur][a];
        unsigned k = (unsigned)rx[cur][a];
        while (m) {
          const unsigned ty = (unsigned)__ffs((int)m) - 1u;
          m &= m - 1u;
          s_lane[wave][k++] = (unsigned short)((unsigned)lane | (ty << 6));
        }
      }
      wave_lds_sync();

      for (unsigned j = lane; j < total; j += 64) {
        const unsigned ent = s_lane[wave][j];
        const int L = (int)(ent & 63u), ty = (int)(ent >> 6);
        const unsigned idx = base + j;
        const int ax = x0 + L;
        const unsigned w0 = s_cof[2 * ty], w1 = s_cof[2 * ty + 1];
        const unsigned pk = w0 >> 25;
        const int m1 = pk & 15, m2 = pk >> 4;
        // vertex offsets along x, y, t of v1 and v2
        const int dx1 = m1 & 1, dy1 = (m1 >> 1) & 1, dt1 = (m1 >> 2) & 1;
        const int dx2 = dx1 + (m2 & 1), dy2 = dy1 + ((m2 >> 1) & 1), dt2 = dt1 + ((m2 >> 2) & 1);
        const int lxs[3] = {L, L + dx1, L + dx2};
        const int lys[3] = {ly, ly + dy1, ly + dy2};
        const int dts[3] = {0, dt1, dt2};

        float qf[3][2];
        float J[3][4];
        bool wide = false;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          const float2* G = gs[par ^ dts[i]];
          const int c = (lys[i] + 1) * GW + (lxs[i] + 1);
          const float2 v = G[c];
          qf[i][0] = quant(v.x, g.qscale);
          qf[i][1] = quant(v.y, g.qscale);
          if constexpr (WIDE)  // the narrow variant only runs when every |q| < 2^24
            if (!(fabsf(qf[i][0]) < 2147483648.0f) || !(fabsf(qf[i][1]) < 2147483648.0f)) wide = true;
          const int gxv = x0 + lxs[i], gyv = y0 + lys[i];
          const float2 xl = G[c - 1], xh = G[c + 1], yl = G[c - GW], yh = G[c + GW];
          const float fx = gxv == 0 || gxv == nx - 1 ? 1.0f : 0.5f, fy = gyv == 0 || gyv == ny - 1 ? 1.0f : 0.5f;
          J[i][0] = (xh.x - xl.x) * fx;  // diff3: a product with 1 is exact
          J[i][1] = (yh.x - yl.x) * fy;
          J[i][2] = (xh.y - xl.y) * fx;
          J[i][3] = (yh.y - yl.y) * fy;
        }
        hit_record2<WIDE>(g, o, qf, J, wide, vector, ax, y, t, ty, dx1, dy1, dt1, dx2, dy2, dt2, idx, n_fp64,
                          n_deg);

        // ---- pass 2 links: each of the (at most two) tetrahedra holding this triangle has exactly one other
        // punctured side.  Each link is recorded by its larger endpoint: inside this tile and chunk it goes to the
        // LDS union-find, otherwise to the global edge list.
        // (branch-free: every neighbour lookup stays inside the ring slices)
        unsigned sm0 = 0, sm1 = 0;
        int sl0 = 0, sl1 = 0;
        int ns = 0;
        bool bad = false;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const unsigned w = k == 0 ? w0 : w1;
          const int rule = w & 3, axis = (w >> 2) & 3;
          const int pa = axis == 0 ? ax : (axis == 1 ? y : t);
          const int Na = axis == 0 ? nx : (axis == 1 ? ny : nt);
          const bool exists = !((rule == 2 && pa < 1) || (rule == 3 && pa + 1 > Na - 1));  // the cell is in the grid
          int found = 0, oslot = 0;
          unsigned other = 0;
#pragma unroll
          for (int sdx = 0; sdx < 3; ++sdx) {
            const unsigned f = (w >> (4 + 7 * sdx)) & 127u;
            const int slot = f & 7, tt = f >> 3;
            // ring slot, slice row and column of the neighbour anchor (bit fields: no branch on the slot)
            const unsigned s2 = (unsigned)slot * 2u;
            const int rs = (int)((rsw >> s2) & 3u);
            const int rr = ly + (int)((kSlotRow >> s2) & 3u);
            const int rc = L + (int)((kSlotCol >> s2) & 3u);
            const unsigned um = rm[rs][rr * RW + rc];
            const unsigned hit = (um >> tt) & 1u;
            const unsigned cand = rb[rs][rr] + (unsigned)(int)rx[rs][rr * RW + rc] + __popc(um & ((1u << tt) - 1u));
            found += (int)hit;
            other = hit ? cand : other;
            oslot = hit ? slot : oslot;
          }
          bad = bad || (exists && found != 1);
          const bool take = exists && found == 1 && other < idx;
          sm1 = (take && ns == 1) ? other : sm1;
          sl1 = (take && ns == 1) ? oslot : sl1;
          sm0 = (take && ns == 0) ? other : sm0;
          sl0 = (take && ns == 0) ? oslot : sl0;
          ns += take ? 1 : 0;
        }
        if (bad || t == g.debug_step) st |= ST_INVARIANT;
        n_linked += ns;
        // link class of each smaller partner: 0 united here (anchor in this tile and chunk), 1 global list,
        // 2 partner in an earlier chunk of this tile (staged as (partner, hit), attached at this chunk's flush);
        // -1 none
        int c0 = -1, c1 = -1;
        if (plane_global) {
          o.parent[idx] = idx;
          c0 = ns > 0 ? 1 : -1;
          c1 = ns > 1 ? 1 : -1;
        } else {
          const unsigned li = row_lbase + j;
          const unsigned clw_l = clw | (L == 0 ? 1u << (2 * NB_MX) : 0u);
          auto link_class = [&](int sl) -> int { return (int)((clw_l >> (2 * sl)) & 3u); };
          auto local_id = [&](unsigned other, int sl) -> unsigned {
            return other + (sl == NB_MY ? d_my : (sl == NB_MT ? d_mt : d_self));
          };
          c0 = ns > 0 ? link_class(sl0) : -1;
          c1 = ns > 1 ? link_class(sl1) : -1;
          // The first smaller partner of this chunk becomes the parent (parents point to smaller local ids: a
          // forest); a second one waits in the high half of the entry for the chunk's flush.  Only this lane writes
          // the entry, and nothing reads the chunk's entries before the flush.
          const unsigned l0 = local_id(sm0, sl0), l1 = local_id(sm1, sl1);
          lpar[li] = (c0 == 0 ? l0 : li) | (c1 == 0 ? (l1 + 1u) << 16 : 0u);
        }
        append_edge(c0 > 0, c0 == 2 ? sm0 : idx, c0 == 2 ? idx : sm0, s_stage, &s_stage_n, scap, o.work, work_cnt);
        append_edge(c1 > 0, c1 == 2 ? sm1 : idx, c1 == 2 ? idx : sm1, s_stage, &s_stage_n, scap, o.work, work_cnt);
      }
      wave_lds_sync();
    }
  }
  __syncthreads();
  flush();
  drain();
  unsigned long long s1 = block_sum256(n_fp64, s_red);
  unsigned long long s2 = block_sum256(n_deg, s_red);
  unsigned long long s3 = block_sum256(n_linked, s_red);
  if (tid == 0) {
    if (s1) atomicAdd(&cnt[CNT_FP64], s1);
    if (s2) atomicAdd(&cnt[CNT_DEGEN], s2);
    if (s3) atomicAdd(&cnt[CNT_LINKED], s3);
  }
  if (st) atomicOr(status, st);
}

// The narrow variant is held to 128 VGPRs so that four workgroups share a CU (its LDS allows four).
template <int TY, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WIDE ? 2 : 4))) void emit2d(Grid2 g, int TT, const uint16_t* __restrict__ masks,
                                              const int* __restrict__ seg_cnt, const long long* __restrict__ seg_off,
                                              Out2 o, unsigned* __restrict__ status,
                                              unsigned long long* __restrict__ cnt) {
  emit2d_tile<TY, WIDE>(g, TT, blockIdx.x, blockIdx.y, blockIdx.z, masks, seg_cnt, seg_off, o, status, cnt,
                        &cnt[CNT_WORK]);
}

// ---------------------------------------------------------------------------------------------------------------
// Sparse emission, for hits that are rare (a few per thousand vertices), where the tile-marching emission above pays a
// fixed cost per tile and step (ring loads, scans and barriers for a handful of hits).  Two launches: emit2d_ids lists the
// face ids from the masks of the non-empty row segments (straight into the result), and the hits are then taken a
// lane each, in full wavefronts.  A hit reads what it needs through the caches: its vertices' stencils, the masks of
// the anchors that hold the other sides of its cells, and a smaller partner's index by searching the partner's
// segment in the listed ids.  (A wavefront per segment, with its few hits in its lanes, waited a chain of loads per
// segment: vector 4096^2 x 50 780 -> 160 us, batch of 12 784 -> 183 us.)  No counter is shared: every link joins a
// hit to a smaller partner, so a hit with one or two smaller partners takes the first as its union-find parent (the
// parents then point to smaller indices and form a forest whose trees are connected parts of a trajectory; a tree's
// root is a hit with no smaller partner), and a hit with two writes the second to its own slot of the link array
// ((i, i) when absent), united afterwards by uf_hook_slots.  A trajectory is a path or a loop of hits (each lies in at
// most two cells), so the slot links (one per local maximum of the index along it) join all its trees.  The records are
// the same operations as in the tiled form (hit_record2), so both forms give identical outputs.
// ---------------------------------------------------------------------------------------------------------------
namespace {

// Binary32 vector of vertex (x, y) of field plane P (gradient of a scalar by the stencil of pass 1, or the vector
// itself) and its Jacobian stencil J: the same operations as the staged form.  Coordinates outside the grid are
// clamped; diff3 never uses those values (one-sided differences at the first and last index).
__device__ __forceinline__ void vertex_stencil2(const Grid2& g, int x, int y, int t, float2& v, float (&J)[4]) {
  const int nx = g.nx, ny = g.ny;
  const long long plane = (long long)nx * ny;
  auto cx = [&](int i) { return i < 0 ? 0 : (i >= nx ? nx - 1 : i); };
  auto cy = [&](int i) { return i < 0 ? 0 : (i >= ny ? ny - 1 : i); };
  float2 xl, xh, yl, yh;
  if (g.kind == 0) {
    const float* P = g.f + (long long)fpl(g, t) * plane;
    auto F = [&](int dx, int dy) { return P[(long long)cy(y + dy) * nx + cx(x + dx)]; };
    const float f00 = F(0, 0), fm0 = F(-1, 0), fp0 = F(1, 0), f0m = F(0, -1), f0p = F(0, 1);
    const float fmm0 = F(-2, 0), fpp0 = F(2, 0), f0mm = F(0, -2), f0pp = F(0, 2);
    const float fmm = F(-1, -1), fpm = F(1, -1), fmp = F(-1, 1), fpp = F(1, 1);
    const int xm = x - 1, xp = x + 1, ym = y - 1, yp = y + 1;
    v.x = diff3(fm0, f00, fp0, x, nx);
    v.y = diff3(f0m, f00, f0p, y, ny);
    xl = make_float2(diff3(fmm0, fm0, f00, xm, nx), diff3(fmm, fm0, fmp, y, ny));
    xh = make_float2(diff3(f00, fp0, fpp0, xp, nx), diff3(fpm, fp0, fpp, y, ny));
    yl = make_float2(diff3(fmm, f0m, fpm, x, nx), diff3(f0mm, f0m, f00, ym, ny));
    yh = make_float2(diff3(fmp, f0p, fpp, x, nx), diff3(f00, f0p, f0pp, yp, ny));
  } else {
    const float* U = g.f + (long long)fpl(g, t) * 2 * plane;
    const float* W = U + plane;
    auto V = [&](int dx, int dy) {
      const long long k = (long long)cy(y + dy) * nx + cx(x + dx);
      return make_float2(U[k], W[k]);
    };
    v = V(0, 0);
    xl = V(-1, 0);
    xh = V(1, 0);
    yl = V(0, -1);
    yh = V(0, 1);
  }
  J[0] = diff3(xl.x, v.x, xh.x, x, nx);
  J[1] = diff3(yl.x, v.x, yh.x, y, ny);
  J[2] = diff3(xl.y, v.y, xh.y, x, nx);
  J[3] = diff3(yl.y, v.y, yh.y, y, ny);
}

// a / b of indices: the 64-bit division is a long instruction sequence, so values of 32 bits take the short one
__device__ __forceinline__ long long index_div(long long a, int b) {
  if ((a >> 32) == 0) return (unsigned)a / (unsigned)b;
  return a / b;
}

// Hit idx, its face id listed.
template <bool WIDE>
__device__ __forceinline__ void emit2d_hit(const Grid2& g, unsigned idx, const unsigned* cof,
                                           const uint16_t* __restrict__ masks, const int* __restrict__ seg_cnt,
                                           const long long* __restrict__ seg_off, const Out2& o, unsigned& st,
                                           unsigned long long& n_fp64, unsigned long long& n_deg,
                                           unsigned long long& n_linked) {
  const int nx = g.nx, ny = g.ny, nt = g.nt;
  const long long* ids = o.face_id - o.gbase;  // by hit index
  const long long own = ids[idx], v = own / 12, row = index_div(v, nx);
  const int ty = (int)(own - v * 12), ax = (int)(v - row * nx), t = (int)index_div(row, ny), y = (int)(row - (long long)t * ny);
  const unsigned w0 = cof[2 * ty], w1 = cof[2 * ty + 1];
  const unsigned pk = w0 >> 25;
  const int m1 = pk & 15, m2 = pk >> 4;
  const int dx1 = m1 & 1, dy1 = (m1 >> 1) & 1, dt1 = (m1 >> 2) & 1;
  const int dx2 = dx1 + (m2 & 1), dy2 = dy1 + ((m2 >> 1) & 1), dt2 = dt1 + ((m2 >> 2) & 1);
  const int dxs[3] = {0, dx1, dx2}, dys[3] = {0, dy1, dy2}, dts[3] = {0, dt1, dt2};

  // links (Alg. 1 pass 2): the other punctured side of each tetrahedron holding the triangle; the larger end of each
  // link records it
  unsigned sm[2] = {0, 0};
  int ns = 0;
  bool bad = false;
  long long other[2] = {-1, -1};   // smaller partner of the cell
  long long seg[2] = {0, 0};       // and its row segment
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const unsigned w = k == 0 ? w0 : w1;
    const int rule = w & 3, axis = (w >> 2) & 3;
    const int pa = axis == 0 ? ax : (axis == 1 ? y : t);
    const int Na = axis == 0 ? nx : (axis == 1 ? ny : nt);
    const bool exists = !((rule == 2 && pa < 1) || (rule == 3 && pa + 1 > Na - 1));
    int found = 0;
    long long id = -1, sg = 0;
#pragma unroll
    for (int sdx = 0; sdx < 3; ++sdx) {
      const unsigned f = (w >> (4 + 7 * sdx)) & 127u;
      const int slot = f & 7, tt = f >> 3;
      const int xx = ax + (slot == NB_MX ? -1 : (slot == NB_PX ? 1 : 0));
      const int yy = y + (slot == NB_MY ? -1 : (slot == NB_PY ? 1 : 0));
      const int ts = t + (slot == NB_MT ? -1 : (slot == NB_PT ? 1 : 0));
      const bool in = xx >= 0 && xx < nx && yy >= 0 && yy < ny && ts >= 0 && ts < nt;
      // without a branch, so that the loads are in flight together: outside the grid the own mask is read
      const long long mr = in ? (long long)mpl(g, ts) * ny + yy : (long long)mpl(g, t) * ny + y;
      const unsigned um = masks[mr * nx + (in ? xx : ax)];
      const bool hit = in && ((um >> tt) & 1u);
      found += hit ? 1 : 0;
      id = hit ? (((long long)ts * ny + yy) * nx + xx) * 12 + tt : id;
      sg = hit ? mr * g.nxt + (xx >> 6) : sg;
    }
    bad = bad || (exists && found != 1);
    const bool take = exists && found == 1 && id < own;
    other[k] = take ? id : -1;
    seg[k] = sg;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (other[k] < 0) continue;
    unsigned lo = (unsigned)seg_off[seg[k]], hi = lo + (unsigned)seg_cnt[seg[k]];
    while (hi - lo > 1) {  // last id of the segment not above the partner's
      const unsigned mid = (lo + hi) >> 1;
      if (ids[mid] <= other[k])
        lo = mid;
      else
        hi = mid;
    }
    if (ns == 0)
      sm[0] = lo;
    else
      sm[1] = lo;
    ++ns;
  }
  if (bad || t == g.debug_step) st |= ST_INVARIANT;
  n_linked += ns;
  o.parent[idx] = ns > 0 ? sm[0] : idx;
  o.work[idx] = make_uint2(idx, ns > 1 ? sm[1] : idx);

  float qf[3][2];
  float J[3][4];
  bool wide = false;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    float2 u;
    vertex_stencil2(g, ax + dxs[i], y + dys[i], t + dts[i], u, J[i]);
    qf[i][0] = quant(u.x, g.qscale);
    qf[i][1] = quant(u.y, g.qscale);
    if constexpr (WIDE)
      if (!(fabsf(qf[i][0]) < 2147483648.0f) || !(fabsf(qf[i][1]) < 2147483648.0f)) wide = true;
  }
  Out2 rest = o;
  rest.face_id = nullptr;
  hit_record2<WIDE>(g, rest, qf, J, wide, g.kind != 0, ax, y, t, ty, dx1, dy1, dt1, dx2, dy2, dt2, idx, n_fp64, n_deg);
}

// Per-wavefront counters into the call's (or series') counters.
__device__ __forceinline__ void sparse_flush_counts(unsigned long long* cnt, unsigned long long& n_fp64,
                                                    unsigned long long& n_deg, unsigned long long& n_linked) {
  const unsigned long long a = wave_sum64(n_fp64), b = wave_sum64(n_deg), c = wave_sum64(n_linked);
  if (lane_id() == 0) {
    if (a) atomicAdd(&cnt[CNT_FP64], a);
    if (b) atomicAdd(&cnt[CNT_DEGEN], b);
    if (c) atomicAdd(&cnt[CNT_LINKED], c);
  }
  n_fp64 = n_deg = n_linked = 0;
}

// Face ids of the hits of segments [64 blk, 64 blk + 64) of the steps [t_begin, t_end): each lane reads one segment's
// count, the wavefront walks the non-empty ones, kIdsBatch mask rows in flight.
constexpr int kIdsBatch = 4;
__device__ __forceinline__ void emit2d_ids_block(const Grid2& g, long long blk, const uint16_t* __restrict__ masks,
                                                 const int* __restrict__ seg_cnt,
                                                 const long long* __restrict__ seg_off, const Out2& o) {
  const unsigned per_step = (unsigned)g.ny * (unsigned)g.nxt;  // segments per step
  const long long nseg = (long long)(g.t_end - g.t_begin) * per_step;
  const long long s0 = blk * 64;
  // step and in-step segment of the block's first segment; the block's 64 segments span at most a few steps
  const int tb = (int)(s0 / per_step);
  const unsigned rb0 = (unsigned)(s0 - (long long)tb * per_step);
  auto locate = [&](int b, int& t, unsigned& r) {
    t = tb;
    r = rb0 + (unsigned)b;
    while (r >= per_step) {
      r -= per_step;
      ++t;
    }
    t += g.t_begin;
  };
  int c = 0;
  unsigned first = 0;
  if (s0 + lane_id() < nseg) {
    int t;
    unsigned r;
    locate(lane_id(), t, r);
    const long long k = (long long)mpl(g, t) * per_step + r;
    c = seg_cnt[k];
    first = (unsigned)seg_off[k];
  }
  unsigned long long bal = __ballot(c > 0);
  while (bal) {
    unsigned m[kIdsBatch], base[kIdsBatch];
    long long id0[kIdsBatch];
#pragma unroll
    for (int q = 0; q < kIdsBatch; ++q) {
      m[q] = 0;
      base[q] = 0;
      id0[q] = 0;
      if (bal) {
        const int b = __ffsll((long long)bal) - 1;
        bal &= bal - 1ull;
        int t;
        unsigned r;
        locate(b, t, r);
        const int y = (int)(r / (unsigned)g.nxt), bx = (int)(r - (unsigned)y * (unsigned)g.nxt);
        const int x = bx * TX + lane_id();
        const unsigned mv = masks[((long long)mpl(g, t) * g.ny + y) * g.nx + min(x, g.nx - 1)];
        m[q] = x < g.nx ? mv : 0u;
        base[q] = (unsigned)__builtin_amdgcn_readlane((int)first, b);
        id0[q] = (((long long)t * g.ny + y) * g.nx + x) * 12;
      }
    }
#pragma unroll
    for (int q = 0; q < kIdsBatch; ++q) {
      const unsigned n = __popc(m[q]), incl = wave_incl_scan(n);
      unsigned k = base[q] + incl - n - o.gbase;
      for (unsigned w = m[q]; w; w &= w - 1u) o.face_id[k++] = id0[q] + __ffs((int)w) - 1;
    }
  }
}

// Wavefronts of the id lists: enough for eight per SIMD.
constexpr int kSparseWaves = 8192;

}  // namespace

__global__ __launch_bounds__(256) void emit2d_ids(Grid2 g, const uint16_t* __restrict__ masks,
                                                  const int* __restrict__ seg_cnt,
                                                  const long long* __restrict__ seg_off, Out2 o) {
  const long long nblk = ((long long)(g.t_end - g.t_begin) * g.ny * g.nxt + 63) / 64;
  const long long nw = (long long)gridDim.x * 4;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // wave-uniform: scalar loop state
  for (long long blk = (long long)blockIdx.x * 4 + wv; blk < nblk; blk += nw)
    emit2d_ids_block(g, blk, masks, seg_cnt, seg_off, o);
}

template <bool WIDE>
__global__ __launch_bounds__(256) void emit2d_sparse(Grid2 g, const uint16_t* __restrict__ masks,
                                                     const int* __restrict__ seg_cnt,
                                                     const long long* __restrict__ seg_off, long long n_hits, Out2 o,
                                                     unsigned* __restrict__ status,
                                                     unsigned long long* __restrict__ cnt) {
  __shared__ unsigned cof[24];
  __shared__ unsigned long long red[3][4];
  if (threadIdx.x < 24) cof[threadIdx.x] = kTri2WordsDev.w[threadIdx.x];
  __syncthreads();
  unsigned st = 0;
  unsigned long long n_fp64 = 0, n_deg = 0, n_linked = 0;
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n_hits; i += (long long)gridDim.x * 256)
    emit2d_hit<WIDE>(g, (unsigned)i, cof, masks, seg_cnt, seg_off, o, st, n_fp64, n_deg, n_linked);
  // one counter update per workgroup (same-address atomics serialise)
  const int w = threadIdx.x >> 6;
  const unsigned long long a = wave_sum64(n_fp64), b = wave_sum64(n_deg), c = wave_sum64(n_linked);
  if ((threadIdx.x & 63) == 0) {
    red[0][w] = a;
    red[1][w] = b;
    red[2][w] = c;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const int k = threadIdx.x;
    const unsigned long long v = red[k][0] + red[k][1] + red[k][2] + red[k][3];
    if (v) atomicAdd(&cnt[k == 0 ? CNT_FP64 : (k == 1 ? CNT_DEGEN : CNT_LINKED)], v);
  }
  if (st) atomicOr(status, st);
}

// ---------------------------------------------------------------------------------------------------------------
// Batched form: one persistent launch per stage for many independent series.  Workgroups pull (series, tile) items
// from a device counter; the item -> series map is a binary search over the per-series item prefix.
// ---------------------------------------------------------------------------------------------------------------
__device__ __forceinline__ int take_item(int* counter, int total, int* s_item) {
  __syncthreads();
  if (threadIdx.x == 0) *s_item = atomicAdd(counter, 1);
  __syncthreads();
  const int it = *s_item;
  return it < total ? it : -1;
}

__device__ __forceinline__ int series_of(const int* prefix, int nser, int item) {
  int lo = 0, hi = nser;  // prefix[lo] <= item < prefix[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (prefix[mid] <= item)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// Detection: every wavefront pulls its own items (its tiles are independent of its workgroup's).
template <bool VEC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void detect2d_batched(const Series2* __restrict__ S, const int* __restrict__ prefix,
                                                        int nser, int TT, int* counter, unsigned* status) {
  const int total = prefix[nser];
  for (;;) {
    int it = 0;
    if (lane_id() == 0) it = atomicAdd(counter, 1);
    it = __builtin_amdgcn_readfirstlane(it);
    if (it >= total) break;
    const int s = series_of(prefix, nser, it);
    const Grid2 g = S[s].g;
    const int local = it - prefix[s];
    const int tx = g.nxt, tyn = (g.ny + kDetRows - 1) / kDetRows;
    const int bx = local % tx, by = (local / tx) % tyn, bz = local / (tx * tyn);
    detect2d_wave<VEC>(g, TT, bx, by * kDetRows, bz, S[s].masks, S[s].seg_cnt, status);
  }
}

template <int TY, bool WIDE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WIDE ? 2 : 3))) void emit2d_batched(const Series2* __restrict__ S, const int* __restrict__ prefix,
                                                      int nser, int TT, int* counter, unsigned* status,
                                                      unsigned long long* work_cnt) {
  __shared__ int s_item;
  const int total = prefix[nser];
  for (;;) {
    const int it = take_item(counter, total, &s_item);
    if (it < 0) break;
    const int s = series_of(prefix, nser, it);
    const Grid2 g = S[s].g;
    const Out2 o = S[s].o;
    const int local = it - prefix[s];
    const int tx = g.nxt, tyn = (g.ny + TY - 1) / TY;
    const int bx = local % tx, by = (local / tx) % tyn, bz = local / (tx * tyn);
    emit2d_tile<TY, WIDE>(g, TT, bx, by, bz, S[s].masks, S[s].seg_cnt, S[s].seg_off, o, status, S[s].cnt,
                          work_cnt);
  }
}

// Batched sparse emission: blocks of 64 segments, then of 64 hits, of the series that take the sparse form, each
// concatenated (bprefix: per-series block prefix, zero blocks for the others); a wavefront's block -> series by binary
// search.
__device__ __forceinline__ int series_of_block(const long long* bprefix, int nser, long long B) {
  int lo = 0, hi = nser;  // bprefix[lo] <= B < bprefix[lo + 1]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (bprefix[mid] <= B)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

__global__ __launch_bounds__(256) void emit2d_ids_batched(const Series2* __restrict__ S,
                                                          const long long* __restrict__ bprefix, int nser) {
  const long long nblk = bprefix[nser];
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // wave-uniform: scalar loop state
  for (long long B = (long long)blockIdx.x * 4 + wv; B < nblk; B += (long long)gridDim.x * 4) {
    const int lo = series_of_block(bprefix, nser, B);
    const Grid2 g = S[lo].g;
    const Out2 o = S[lo].o;
    emit2d_ids_block(g, B - bprefix[lo], S[lo].masks, S[lo].seg_cnt, S[lo].seg_off, o);
  }
}

template <bool WIDE>
__global__ __launch_bounds__(256) void emit2d_sparse_batched(const Series2* __restrict__ S,
                                                             const long long* __restrict__ bprefix,
                                                             const unsigned* __restrict__ gbase, int nser,
                                                             unsigned* status) {
  __shared__ unsigned cof[24];
  if (threadIdx.x < 24) cof[threadIdx.x] = kTri2WordsDev.w[threadIdx.x];
  __syncthreads();
  const long long nblk = bprefix[nser];
  // consecutive blocks to one wavefront: it then meets few series, and counts each once
  const long long waves = (long long)gridDim.x * 4, share = (nblk + waves - 1) / waves;
  unsigned st = 0;
  unsigned long long n_fp64 = 0, n_deg = 0, n_linked = 0;
  int cur = -1;  // series whose counts are being gathered (flushed when the wavefront moves to another)
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));  // wave-uniform: scalar loop state
  const long long first = ((long long)blockIdx.x * 4 + wv) * share;
  for (long long B = first; B < min(first + share, nblk); ++B) {
    const int lo = series_of_block(bprefix, nser, B);
    if (lo != cur) {
      if (cur >= 0) sparse_flush_counts(S[cur].cnt, n_fp64, n_deg, n_linked);
      cur = lo;
    }
    const Grid2 g = S[lo].g;
    const Out2 o = S[lo].o;
    const long long idx = (long long)gbase[lo] + (B - bprefix[lo]) * 64 + lane_id();
    if (idx < (long long)gbase[lo + 1])
      emit2d_hit<WIDE>(g, (unsigned)idx, cof, S[lo].masks, S[lo].seg_cnt, S[lo].seg_off, o, st, n_fp64, n_deg, n_linked);
  }
  if (cur >= 0) sparse_flush_counts(S[cur].cnt, n_fp64, n_deg, n_linked);
  if (st) atomicOr(status, st);
}

// Emission of single steps (streaming): one step per launch, local union-find per step.
hipError_t launch_emit2d_steps(const Grid2& g, bool wide, const uint16_t* masks, const int* seg_cnt,
                               const long long* seg_off, const Out2& o, unsigned* status, unsigned long long* cnt,
                               hipStream_t s) {
  constexpr int TYE = 8;
  dim3 grid((unsigned)g.nxt, (unsigned)((g.ny + TYE - 1) / TYE), (unsigned)(g.t_end - g.t_begin));
  if (wide)
    emit2d<TYE, true><<<grid, 256, 0, s>>>(g, 1, masks, seg_cnt, seg_off, o, status, cnt);
  else
    emit2d<TYE, false><<<grid, 256, 0, s>>>(g, 1, masks, seg_cnt, seg_off, o, status, cnt);
  return hipGetLastError();
}

hipError_t launch_detect2d_batched(const Series2* S, const int* prefix, int nser, int total_items, int tt, int kind,
                                   int* counter, unsigned* status, hipStream_t s) {
  int blocks = (total_items + 3) / 4;
  if (blocks > 1024) blocks = 1024;  // four wavefronts per SIMD, of which its registers let three be resident
  if (blocks < 1) blocks = 1;
  if (kind != 0)
    detect2d_batched<true><<<blocks, 256, 0, s>>>(S, prefix, nser, tt, counter, status);
  else
    detect2d_batched<false><<<blocks, 256, 0, s>>>(S, prefix, nser, tt, counter, status);
  return hipGetLastError();
}

hipError_t launch_emit2d_batched(const Series2* S, const int* prefix, int nser, int total_items, bool wide,
                                 int* counter, unsigned* status, unsigned long long* work_cnt, hipStream_t s) {
  int blocks = total_items < 1536 ? total_items : 1536;
  if (blocks < 1) blocks = 1;
  if (wide)
    emit2d_batched<8, true><<<blocks, 256, 0, s>>>(S, prefix, nser, kEmitSteps, counter, status, work_cnt);
  else
    emit2d_batched<8, false><<<blocks, 256, 0, s>>>(S, prefix, nser, kEmitSteps, counter, status, work_cnt);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------------------------------------------
hipError_t launch_detect2d(const Grid2& g, int ty, int tt, uint16_t* masks, int* seg_cnt, unsigned* status,
                           hipStream_t s) {
  dim3 grid((unsigned)g.nxt, (unsigned)((g.ny + ty - 1) / ty), (unsigned)((g.t_end - g.t_begin + tt - 1) / tt));
  const unsigned threads = 64u * (unsigned)(ty / kDetRows);
  if (g.kind != 0)
    detect2d<true><<<grid, threads, 0, s>>>(g, tt, masks, seg_cnt, status);
  else
    detect2d<false><<<grid, threads, 0, s>>>(g, tt, masks, seg_cnt, status);
  return hipGetLastError();
}

hipError_t launch_emit2d(const Grid2& g, bool wide, int tt, const uint16_t* masks, const int* seg_cnt,
                         const long long* seg_off, const Out2& o, unsigned* status, unsigned long long* cnt,
                         hipStream_t s) {
  static_assert(kEmitSteps <= 32, "steps per emission tile exceed the tile's step tables");
  dim3 grid((unsigned)g.nxt, (unsigned)((g.ny + kEmitRows - 1) / kEmitRows),
            (unsigned)((g.t_end - g.t_begin + tt - 1) / tt));
  if (wide)
    emit2d<kEmitRows, true><<<grid, 256, 0, s>>>(g, tt, masks, seg_cnt, seg_off, o, status, cnt);
  else
    emit2d<kEmitRows, false><<<grid, 256, 0, s>>>(g, tt, masks, seg_cnt, seg_off, o, status, cnt);
  return hipGetLastError();
}

hipError_t launch_emit2d_sparse(const Grid2& g, bool wide, const uint16_t* masks, const int* seg_cnt,
                                const long long* seg_off, long long n_hits, const Out2& o, unsigned* status,
                                unsigned long long* cnt, hipStream_t s) {
  const long long nblk = ((long long)(g.t_end - g.t_begin) * g.ny * g.nxt + 63) / 64;
  long long blocks = (nblk + 3) / 4;
  if (blocks > kSparseWaves / 4) blocks = kSparseWaves / 4;
  if (blocks < 1) blocks = 1;
  emit2d_ids<<<(unsigned)blocks, 256, 0, s>>>(g, masks, seg_cnt, seg_off, o);
  long long hb = (n_hits + 255) / 256;
  if (hb > kSparseWaves / 4) hb = kSparseWaves / 4;
  if (hb < 1) hb = 1;
  auto* emit = wide ? emit2d_sparse<true> : emit2d_sparse<false>;
  emit<<<(unsigned)hb, 256, 0, s>>>(g, masks, seg_cnt, seg_off, n_hits, o, status, cnt);
  return hipGetLastError();
}

hipError_t launch_emit2d_sparse_batched(const Series2* S, const long long* seg_prefix, const long long* hit_prefix,
                                        const unsigned* gbase, int nser, long long seg_blocks, long long hit_blocks,
                                        bool wide, unsigned* status, hipStream_t s) {
  auto grid = [](long long waves) {
    const long long b = (waves + 3) / 4;
    return (unsigned)(b > kSparseWaves / 4 ? kSparseWaves / 4 : b < 1 ? 1 : b);
  };
  emit2d_ids_batched<<<grid(seg_blocks), 256, 0, s>>>(S, seg_prefix, nser);
  auto* emit = wide ? emit2d_sparse_batched<true> : emit2d_sparse_batched<false>;
  emit<<<grid(hit_blocks), 256, 0, s>>>(S, hit_prefix, gbase, nser, status);
  return hipGetLastError();
}

}  // namespace ftk
