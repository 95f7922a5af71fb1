// prism.hip -- critical-point tracking of a 2D vector field on an unstructured triangle mesh extruded in time
// (Sec. 3.2, prismatic subdivision; Sec. 4.2 two passes).
//
// Every mesh triangle v0 < v1 < v2 becomes, between steps t and t + 1, the prism a0 a1 a2 - b0 b1 b2 split by the
// staircase into a0 a1 a2 b2, a0 a1 b1 b2 and a0 b0 b1 b2 (global vertex order g = t nv + v); the quadrilateral of
// a mesh edge a < b is split along its monotone diagonal a - b'.  Faces of step t are numbered t * S + local,
// S = nf + 2 ne + 2 nf: the mesh triangle T (local T), the edge faces (a, b, b') and (a, a', b') of edge E (nf + 2E,
// +1), and the interior faces (v0, v1, v2') and (v0, v1', v2') of T (nf + 2 ne + 2T, +1); interval faces exist for
// t < nt - 1.
//
//   pm_signs -- the puncture test of a face needs the SoS signs of the determinants of its three vertex pairs, in global
//               order, and the faces share their pairs: (a, b) and (a, b') of an edge, (a, a') of a vertex.  Each
//               sign is found once, as a bit of the pair's word over the steps (lanes are steps, on a vertex-major copy
//               of the quantised field).
//   pm_faces -- one lane per face: its punctures of 64 steps from three such words, turned into words of 64 faces per
//               step (with their counts, whose scan gives the hits' offsets).
//   pm_emit  -- face ids, points from the exact cofactors (Eq. 2) in (x, y, t), identity parents; one lane per hit.
//   pm_unite_hits -- from the hits: the two punctured faces of each tetrahedron holding it are united (pm_unite,
//               one lane per (prism, step), for meshes with an edge of more than two triangles).
// Delaunay mesh of 200k vertices, 40 steps: 769 -> 305 us a call.
#include "common.h"
#include "internal.h"
#include "uf_cached.h"

namespace ftk {

namespace {

using u64 = unsigned long long;

struct PmMesh {
  const float* xy;      // [nv][2]
  const int* tri;       // [nf][3], ascending per row
  const int* edge;      // [ne][2], a < b, ascending
  const int* tri_edge;  // [nf][3]: edges (v0 v1), (v1 v2), (v0 v2)
  const float* field;   // [nt][2][nv]
  long long nv, nf, ne, S, FB;  // S faces in FB words of 64 a step
  int nt;
  float qscale;
};

// Punctured faces: face f of step t is bit f % 64 of word t FB + f / 64, its position p = t 64 FB + f.
struct PmHits {
  const u64* bits;
  const long long* base;  // hits before a word
};
__device__ __forceinline__ bool pm_hit(const PmHits& h, long long p) { return (h.bits[p >> 6] >> (p & 63)) & 1ull; }
__device__ __forceinline__ long long pm_index(const PmHits& h, long long p) {
  return h.base[p >> 6] + __popcll(h.bits[p >> 6] & ((1ull << (p & 63)) - 1ull));
}

// vertices (vertex, step offset) of local face f of a step, in global order
__device__ __forceinline__ void pm_face(const PmMesh& m, long long f, int* v, int* dt) {
  if (f < m.nf) {
    const int* a = m.tri + 3 * f;
    v[0] = a[0], v[1] = a[1], v[2] = a[2];
    dt[0] = dt[1] = dt[2] = 0;
  } else if (f < m.nf + 2 * m.ne) {
    const long long E = (f - m.nf) >> 1;
    const int up = (int)((f - m.nf) & 1);
    const int a = m.edge[2 * E], b = m.edge[2 * E + 1];
    v[0] = a, dt[0] = 0;
    v[1] = up ? a : b, dt[1] = up ? 1 : 0;
    v[2] = b, dt[2] = 1;
  } else {
    const long long T = (f - m.nf - 2 * m.ne) >> 1;
    const int up = (int)((f - m.nf - 2 * m.ne) & 1);
    const int* a = m.tri + 3 * T;
    v[0] = a[0], dt[0] = 0;
    v[1] = a[1], dt[1] = up;
    v[2] = a[2], dt[2] = 1;
  }
}

__device__ __forceinline__ void pm_q(const PmMesh& m, int v, int t, long long* q, unsigned& st) {
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const float x = m.field[((long long)t * 2 + c) * m.nv + v] * m.qscale;
    if (!isfinite(x)) {
      st |= ST_NONFINITE;
      q[c] = 0;
    } else if (!(fabsf(x) < 2147483648.0f)) {
      st |= ST_RANGE;
      q[c] = 0;
    } else {
      q[c] = (long long)rintf(x);
    }
  }
}

// The quantised field vertex-major, [nv][nt] pairs (u, v): the rows that pm_signs reads.  A workgroup moves a tile of
// 64 vertices x 16 steps through LDS: reads run along the vertices, writes along the steps of each vertex (128
// contiguous bytes).  *suspect becomes nonzero where a value is not finite or beyond 31 bits, of whichever vertex.
constexpr int kPmTV = 64, kPmTT = 16;
__device__ __forceinline__ bool pm_fits(float q) { return fabsf(q) < 2147483648.0f; }
__global__ __launch_bounds__(256) void pm_vertex_major(const float* __restrict__ field, long long nv, int nt,
                                                       float qscale, float2* __restrict__ ft,
                                                       unsigned* __restrict__ suspect) {
  __shared__ float tile[kPmTT][2][kPmTV + 1];
  const long long v0 = (long long)blockIdx.x * kPmTV;
  const int t0 = blockIdx.y * kPmTT;
  for (int e = threadIdx.x; e < kPmTT * 2 * kPmTV; e += 256) {
    const int dt = e / (2 * kPmTV), c = (e / kPmTV) & 1, dv = e % kPmTV;
    const long long v = v0 + dv;
    const int t = t0 + dt;
    const float q = (v < nv && t < nt) ? quant(field[(long long)(2 * t + c) * nv + v], qscale) : 0.0f;
    tile[dt][c][dv] = q;
    if (!pm_fits(q)) *suspect = 1u;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kPmTV * kPmTT; e += 256) {
    const int dv = e / kPmTT, dt = e % kPmTT;
    const long long v = v0 + dv;
    const int t = t0 + dt;
    if (v < nv && t < nt) ft[v * nt + t] = make_float2(tile[dt][0][dv], tile[dt][1][dv]);
  }
}

// Signs of the pairs (bit t: the determinant is negative): esign[chunk][edge] = words of (a, b) and (a, b'),
// vsign[chunk][vertex] = word of (a, a'), 64 steps a chunk; the bits of a next vertex beyond the last step mean nothing.
// The rows are the edges and then the vertices, taken as edges (v, v).  A wavefront's lanes are 64 >> log_p rows of
// 1 << log_p >= nt steps (one row when nt is larger), so a row's steps are read as one stretch; the rows of kPmBatch
// such reads are in flight together and their words leave in one store, kPmRounds batches a wavefront.  The status is
// found only when a value is suspect, on the edges, which reach every vertex of a triangle.  Bound by instruction issue.
// 200k vertices, 40 steps: 99 us, 433 for three determinants a face in 64-bit integers.
constexpr int kPmBatch = 4, kPmRounds = 4;
__global__ __launch_bounds__(256) void pm_signs(PmMesh m, const float2* __restrict__ ft, int log_p,
                                                const unsigned* __restrict__ suspect,
                                                ulonglong2* __restrict__ esign, u64* __restrict__ vsign,
                                                unsigned* __restrict__ status) {
  const int lane = threadIdx.x & 63, P = 1 << log_p, log_per = 6 - log_p, per = 1 << log_per;
  const int seg = lane >> log_p, tl = lane & (P - 1);
  const long long rows = m.ne + m.nv;
  const long long wave = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const u64 row_bits = P == 64 ? ~0ull : (1ull << P) - 1ull;
  const bool check = *suspect != 0;
  for (int round = 0; round < kPmRounds; ++round) {
    const long long r0 = (wave * kPmRounds + round) * (kPmBatch * per);
    if (r0 >= rows) break;
    int a[kPmBatch], b[kPmBatch];
#pragma unroll
    for (int k = 0; k < kPmBatch; ++k) {
      const long long r = min(r0 + k * per + seg, rows - 1);
      a[k] = b[k] = (int)(r - m.ne);
      if (r < m.ne) {
        const int2 e = ((const int2*)m.edge)[r];
        a[k] = e.x;
        b[k] = e.y;
      }
    }
    for (int t0 = 0, chunk = 0; t0 < m.nt; t0 += 64, ++chunk) {
      const int t = min(t0 + tl, m.nt - 1), t1 = min(t0 + 64, m.nt - 1);
      float2 qa[kPmBatch], qb[kPmBatch], past[kPmBatch];
#pragma unroll
      for (int k = 0; k < kPmBatch; ++k) {
        qa[k] = ft[(long long)a[k] * m.nt + t];
        qb[k] = ft[(long long)b[k] * m.nt + t];
      }
#pragma unroll
      for (int k = 0; k < kPmBatch; ++k) past[k] = qb[k];
      if (m.nt > 64) {
#pragma unroll
        for (int k = 0; k < kPmBatch; ++k) past[k] = ft[(long long)b[k] * m.nt + t1];
      }
      if (check) {
        unsigned st = 0;
        auto one = [&](float q) {
          if (!pm_fits(q)) st |= isfinite(q) ? ST_RANGE : ST_NONFINITE;
        };
#pragma unroll
        for (int k = 0; k < kPmBatch; ++k)
          if (r0 + k * per + seg < m.ne) {
            one(qa[k].x);
            one(qa[k].y);
            one(qb[k].x);
            one(qb[k].y);
          }
        if (st) atomicOr(status, st);
      }
      u64 wd = 0, we = 0;
#pragma unroll
      for (int k = 0; k < kPmBatch; ++k) {
        const double a0 = qa[k].x, a1 = qa[k].y, b0 = qb[k].x, b1 = qb[k].y;
        const double c0 = from_next(qb[k].x, past[k].x), c1 = from_next(qb[k].y, past[k].y);
        const double d = edge_det(a0, a1, b0, b1), e = edge_det(a0, a1, c0, c1);
        u64 md = __ballot(d < 0.0), me = __ballot(e < 0.0);
        if (__ballot(d == 0.0 || e == 0.0)) {
          md |= __ballot(d == 0.0 && edge_tie(a1, b0, b1) != 0);
          me |= __ballot(e == 0.0 && edge_tie(a1, c0, c1) != 0);
        }
        if ((lane >> log_per) == k) {  // lane l keeps the words of row r0 + l
          wd = md;
          we = me;
        }
      }
      const int shift = (lane & (per - 1)) << log_p;
      wd = (wd >> shift) & row_bits;
      we = (we >> shift) & row_bits;
      const long long r = r0 + lane;
      if (lane < kPmBatch * per && r < rows) {
        if (r < m.ne)
          esign[(long long)chunk * m.ne + r] = make_ulonglong2(wd, we);
        else
          vsign[(long long)chunk * m.nv + (r - m.ne)] = we;
      }
    }
  }
}

// Punctures of the faces, 512 of them a workgroup: the signs of a face's pairs (01), (02), (12), cofactor signs
// +S(12), -S(02), +S(01) agree.  The words over steps become words over faces in LDS.
constexpr int kPmGroups = 8;
__global__ __launch_bounds__(256) void pm_faces(PmMesh m, const ulonglong2* __restrict__ esign,
                                                const u64* __restrict__ vsign, u64* __restrict__ bits,
                                                int* __restrict__ cnt) {
  __shared__ u64 tile[64][kPmGroups];
  unsigned* half = (unsigned*)&tile[0][0];
  const long long b0 = (long long)blockIdx.x * kPmGroups;
  for (int t0 = 0, chunk = 0; t0 < m.nt; t0 += 64, ++chunk) {
    for (int k = threadIdx.x; k < 64 * kPmGroups; k += 256) (&tile[0][0])[k] = 0;
    __syncthreads();
    const ulonglong2* es = esign + (long long)chunk * m.ne;
    const u64* vs = vsign + (long long)chunk * m.nv;
    const bool more = t0 + 64 < m.nt;
    const int left = m.nt - t0;
    const u64 at = left >= 64 ? ~0ull : (1ull << left) - 1ull;           // steps with a face of one step
    const u64 between = left > 64 ? ~0ull : (1ull << (left - 1)) - 1ull;  // ... of two
    // the pair one step on: (a', b')
    auto next = [&](long long E) { return (es[E].x >> 1) | (more ? es[m.ne + E].x << 63 : 0ull); };
    for (int k = threadIdx.x; k < 64 * kPmGroups; k += 256) {
      const long long f = b0 * 64 + k;
      if (f >= m.S) break;
      u64 s01, s02, s12, steps = between;
      if (f < m.nf) {
        const int* te = m.tri_edge + 3 * f;
        s01 = es[te[0]].x, s12 = es[te[1]].x, s02 = es[te[2]].x;
        steps = at;
      } else if (f < m.nf + 2 * m.ne) {
        const long long E = (f - m.nf) >> 1;
        const ulonglong2 e = es[E];
        s02 = e.y;
        if ((f - m.nf) & 1) {  // (a, a', b')
          s01 = vs[m.edge[2 * E]];
          s12 = next(E);
        } else {  // (a, b, b')
          s01 = e.x;
          s12 = vs[m.edge[2 * E + 1]];
        }
      } else {
        const long long g = f - m.nf - 2 * m.ne;
        const int* te = m.tri_edge + 3 * (g >> 1);
        const ulonglong2 e = es[te[0]];
        s02 = es[te[2]].y;
        if (g & 1) {  // (v0, v1', v2')
          s01 = e.y;
          s12 = next(te[1]);
        } else {  // (v0, v1, v2')
          s01 = e.x;
          s12 = es[te[1]].y;
        }
      }
      for (u64 w = ~(s12 ^ s01) & (s02 ^ s01) & steps; w; w &= w - 1ull)
        atomicOr(&half[((__ffsll((long long)w) - 1) * kPmGroups + (k >> 6)) * 2 + ((k >> 5) & 1)], 1u << (k & 31));
    }
    __syncthreads();
    for (int k = threadIdx.x; k < min(left, 64) * kPmGroups; k += 256) {
      const long long b = b0 + k % kPmGroups;
      if (b < m.FB) {
        const u64 w = (&tile[0][0])[k];
        const long long o = (long long)(t0 + k / kPmGroups) * m.FB + b;
        bits[o] = w;
        cnt[o] = __popcll(w);
      }
    }
    __syncthreads();
  }
}

// position of hit i: the last word with at most i hits before it, and its (i - base)-th bit
__device__ __forceinline__ long long pm_find(const PmHits& h, long long n_words, long long i) {
  long long lo = 0, hi = n_words;  // first word with more than i hits before it
  while (lo < hi) {
    const long long mid = (lo + hi) >> 1;
    if (h.base[mid] <= i)
      lo = mid + 1;
    else
      hi = mid;
  }
  const long long w = lo - 1;
  unsigned n = (unsigned)(i - h.base[w]), at = 0;
  u64 b = h.bits[w];
#pragma unroll
  for (unsigned s = 32; s; s >>= 1) {
    const unsigned c = (unsigned)__popcll(b & ((1ull << s) - 1ull));
    const bool up = n >= c;
    n -= up ? c : 0u;
    at += up ? s : 0u;
    b = up ? b >> s : b;
  }
  return w * 64 + at;
}

__global__ void pm_emit(PmMesh m, PmHits h, long long n_hits, long long* __restrict__ face_id,
                        float* __restrict__ pos, unsigned* __restrict__ parent) {
  const long long o = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= n_hits) return;
  const long long p = pm_find(h, m.FB * m.nt, o);
  const int t = (int)(p / (m.FB * 64));
  const long long f = p - (long long)t * (m.FB * 64), id = (long long)t * m.S + f;
  int v[3], dt[3];
  pm_face(m, f, v, dt);
  unsigned st = 0;
  long long q[3][2];
#pragma unroll
  for (int i = 0; i < 3; ++i) pm_q(m, v[i], t + dt[i], q[i], st);
  const long long C0 = q[1][0] * q[2][1] - q[1][1] * q[2][0];
  const long long C1 = -(q[0][0] * q[2][1] - q[0][1] * q[2][0]);
  const long long C2 = q[0][0] * q[1][1] - q[0][1] * q[1][0];
  double mu[3] = {1.0 / 3.0, 1.0 / 3.0, 1.0 / 3.0};
  if (C0 != 0 || C1 != 0 || C2 != 0) {
    const double D = ((double)C0 + (double)C1) + (double)C2;
    mu[0] = (double)C0 / D;
    mu[1] = (double)C1 / D;
    mu[2] = (double)C2 / D;
  }
  face_id[o] = id;
  if (pos) {
    double x[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const double c[3] = {(double)m.xy[2 * v[i]], (double)m.xy[2 * v[i] + 1], (double)(t + dt[i])};
#pragma unroll
      for (int k = 0; k < 3; ++k) x[k] = i == 0 ? mu[0] * c[k] : x[k] + mu[i] * c[k];
    }
    pos[o * 3 + 0] = (float)x[0];
    pos[o * 3 + 1] = (float)x[1];
    pos[o * 3 + 2] = (float)x[2];
  }
  parent[o] = (unsigned)o;
}

// Positions of the sides of the three tetrahedra a0 a1 a2 b2, a0 a1 b1 b2, a0 b0 b1 b2 of the prism of
// triangle T between steps t and t + 1 (lower / upper edge and interior faces are +0 / +1).
__device__ __forceinline__ void pm_prism_tets(const PmMesh& m, long long T, int t, long long (&tet)[3][4]) {
  const long long step = m.FB * 64, base = (long long)t * step;
  const int* te = m.tri_edge + 3 * T;
  const long long e01 = base + m.nf + 2LL * te[0], e12 = base + m.nf + 2LL * te[1], e02 = base + m.nf + 2LL * te[2];
  const long long in = base + m.nf + 2 * m.ne + 2 * T;
  const long long ord0 = base + T, ord1 = base + step + T;
  const long long v[3][4] = {{ord0, in, e02, e12}, {e01, in, in + 1, e12 + 1}, {e01 + 1, e02 + 1, in + 1, ord1}};
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int j = 0; j < 4; ++j) tet[k][j] = v[k][j];
}

// From the hits (Alg. 1 pass 2 from the punctured faces' side): each tetrahedron of each prism holding the hit's face
// has exactly one other punctured side, united with it; any other count is an internal error.  Every tetrahedron with a
// punctured side is reached from its hits, so this is the all-prism pass below restricted to where it can act.  edge_tri:
// the (at most two) triangles of each mesh edge, -1 for none.
//
// SPREAD: eight lanes per hit, one for each tetrahedron of its at most two prisms (two idle).  Few hits leave the chip
// idle, so the time is that of one lane's loads (9k hits: 58 -> 31 us).  Otherwise one lane per hit, which decodes the hit
// once for all of them.
template <bool SPREAD>
__global__ void pm_unite_hits(PmMesh m, const int* __restrict__ edge_tri, PmHits h,
                              const long long* __restrict__ face_id, long long n_hits,
                              unsigned* __restrict__ parent, unsigned* __restrict__ status) {
  const long long tid = (long long)blockIdx.x * blockDim.x + threadIdx.x, i = SPREAD ? tid >> 3 : tid;
  if (i >= n_hits) return;
  const int t = (int)(face_id[i] / m.S);
  const long long f = face_id[i] - (long long)t * m.S, own = (long long)t * (m.FB * 64) + f;
  // prism `side` of the face: its triangle and step; false where there is none
  auto prism = [&](int side, long long& T, int& pt) -> bool {
    pt = t;
    if (f < m.nf) {  // a mesh triangle: bottom of the prism above it, top of the one below
      T = f;
      pt = t - side;
      return pt >= 0 && pt < m.nt - 1;
    }
    if (f < m.nf + 2 * m.ne) {  // an edge face: the prisms of the edge's triangles
      T = edge_tri[2 * ((f - m.nf) >> 1) + side];
      return T >= 0;
    }
    T = (f - m.nf - 2 * m.ne) >> 1;  // an interior face of one prism
    return side == 0;
  };
  auto unite = [&](const long long (&p)[4]) {
    bool mine = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) mine |= p[j] == own;
    if (!mine) return;
    int n = 0;
    long long other = -1;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (pm_hit(h, p[j])) {
        ++n;
        if (p[j] != own) other = p[j];
      }
    if (n == 2)
      uf_unite_cached(parent, (unsigned)i, (unsigned)pm_index(h, other));
    else
      atomicOr(status, ST_INVARIANT);
  };
  long long T, tet[3][4];
  int pt;
  if constexpr (SPREAD) {
    const int side = (int)(tid >> 2) & 1, k = (int)tid & 3;  // prism and tetrahedron
    if (k == 3 || !prism(side, T, pt)) return;
    pm_prism_tets(m, T, pt, tet);
    long long p[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = k == 0 ? tet[0][j] : k == 1 ? tet[1][j] : tet[2][j];
    unite(p);
  } else {
    for (int side = 0; side < 2; ++side) {
      if (!prism(side, T, pt)) continue;
      pm_prism_tets(m, T, pt, tet);
#pragma unroll
      for (int k = 0; k < 3; ++k) unite(tet[k]);
    }
  }
}

// One lane per (prism, step), for meshes with an edge of more than two triangles (no edge -> triangle table).
__global__ void pm_unite(PmMesh m, PmHits h, unsigned* __restrict__ parent, unsigned* __restrict__ status) {
  const long long T = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int t = blockIdx.y;
  if (T >= m.nf || t >= m.nt - 1) return;
  long long tet[3][4];
  pm_prism_tets(m, T, t, tet);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    long long i[4];
    int n = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (pm_hit(h, tet[k][j])) i[n++] = pm_index(h, tet[k][j]);
    if (n == 2)
      uf_unite_cached(parent, (unsigned)i[0], (unsigned)i[1]);
    else if (n != 0)
      atomicOr(status, ST_INVARIANT);
  }
}

}  // namespace

// Hits up to which the unions take eight lanes a hit.  One lane / eight
// lanes a hit, us a call on 20k vertices: white noise, 71k hits 150 / 140, 130k 175 / 169, 250k 200 / 211, 1.15M 434 / 544,
// 12M 3079 / 4328; waves, 23k 180 / 156, 75k 193 / 192, 261k 223 / 287.
constexpr long long kPmSpreadHits = 1 << 17;

static PmMesh pm_mesh(const float* xy, const int* tri, const int* edge, const int* tri_edge, const float* field,
                      long long nv, long long nf, long long ne, int nt, float qscale) {
  const long long S = nf + 2 * ne + 2 * nf;
  return PmMesh{xy, tri, edge, tri_edge, field, nv, nf, ne, S, (S + 63) / 64, nt, qscale};
}

hipError_t launch_pm_test(const float* xy, const int* tri, const int* edge, const int* tri_edge, const float* field,
                          long long nv, long long nf, long long ne, int nt, float qscale, const PmScratch& sc,
                          unsigned* suspect, unsigned* status, hipStream_t s) {
  const PmMesh m = pm_mesh(xy, tri, edge, tri_edge, field, nv, nf, ne, nt, qscale);
  float2* ft = (float2*)sc.rows;
  pm_vertex_major<<<dim3((unsigned)((nv + kPmTV - 1) / kPmTV), (unsigned)((nt + kPmTT - 1) / kPmTT)), 256, 0, s>>>(
      field, nv, nt, qscale, ft, suspect);
  int log_p = 2;  // at most 16 rows a read: 64 of a batch
  while (log_p < 6 && (1 << log_p) < nt) ++log_p;
  const long long per_block = 4ll * kPmRounds * kPmBatch * (64 >> log_p);
  pm_signs<<<(unsigned)((ne + nv + per_block - 1) / per_block), 256, 0, s>>>(m, ft, log_p, suspect, (ulonglong2*)sc.edge_signs,
                                                                             sc.vertex_signs, status);
  pm_faces<<<(unsigned)((m.FB + kPmGroups - 1) / kPmGroups), 256, 0, s>>>(m, (const ulonglong2*)sc.edge_signs,
                                                                          sc.vertex_signs, sc.bits, sc.cnt);
  return hipGetLastError();
}

hipError_t launch_pm_emit(const float* xy, const int* tri, const int* edge, const int* tri_edge, const int* edge_tri,
                          const float* field, long long nv, long long nf, long long ne, int nt, float qscale,
                          const PmScratch& sc, long long n_hits, long long* face_id, float* pos, unsigned* parent,
                          unsigned* status, hipStream_t s) {
  if (n_hits <= 0) return hipSuccess;
  const PmMesh m = pm_mesh(xy, tri, edge, tri_edge, field, nv, nf, ne, nt, qscale);
  const PmHits h{sc.bits, sc.base};
  const unsigned blocks = (unsigned)((n_hits + 255) / 256);
  pm_emit<<<blocks, 256, 0, s>>>(m, h, n_hits, face_id, pos, parent);
  if (edge_tri && n_hits <= kPmSpreadHits)
    pm_unite_hits<true><<<(unsigned)((n_hits + 31) / 32), 256, 0, s>>>(m, edge_tri, h, face_id, n_hits, parent, status);
  else if (edge_tri)
    pm_unite_hits<false><<<blocks, 256, 0, s>>>(m, edge_tri, h, face_id, n_hits, parent, status);
  else if (nt > 1)
    pm_unite<<<dim3((unsigned)((nf + 255) / 256), (unsigned)(nt - 1)), 256, 0, s>>>(m, h, parent, status);
  return hipGetLastError();
}

}  // namespace ftk
