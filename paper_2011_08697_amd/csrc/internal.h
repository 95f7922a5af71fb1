// internal.h -- host/device interface between the C ABI layer and the kernels (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ftk {

// 2D problem description passed by value to the kernels.
struct Grid2 {
  const float* f;
  int kind;       // 0 scalar, 1 vector (planar [t][2][y][x])
  int nx, ny, nt; // nt: number of steps of the series (a large value while a stream is still open)
  int nxt;        // row segments per row: ceil(nx / 64)
  float qscale;   // 2^quant_log2
  int precision;  // 0 FP32 + certified FP64 fallback, 1 FP64
  int t_begin, t_end;  // anchors processed by a launch: steps [t_begin, t_end)
  int f_ring;     // field planes stored as a ring of f_ring steps (step t at slot t % f_ring); 0: plane t at t
  int m_ring;     // same for the puncture masks and the per-segment counts/offsets
  int debug;      // FTK_DEBUG_* test hooks (0 in normal use)
  int debug_step; // step at which FTK_DEBUG_INVARIANT reports a bad cell (-1: none)
};

// 2D outputs (device pointers; pos/mu/type/flags may be null).
struct Out2 {
  unsigned gbase;    // global hit index of this series' first hit (outputs are indexed by global - gbase)
  long long* face_id;
  float* pos;
  float* mu;
  uint8_t* type;
  uint8_t* flags;
  unsigned* parent;  // union-find forest over global hit indices
  uint2* work;       // union edges that leave a tile/chunk (global hit, smaller partner)
  long long* label;  // labels (read by the batched label pass)
};

// One series of a batched call (device copy read by the persistent kernels).
struct Series2 {
  Grid2 g;
  Out2 o;
  uint16_t* masks;
  int* seg_cnt;
  long long* seg_off;
  unsigned long long* cnt;  // per-series counters (CNT_*)
  int wide;
  int pad;
};

// 3D problem description.
struct Grid3 {
  const float* f;
  int nx, ny, nz, nt;  // nt: number of steps of the series (a large value while a stream is still open)
  int nxt;
  float qscale;
  int precision;
  int t_begin = 0, t_end = 0;  // anchors processed by a launch: steps [t_begin, t_end)
  int f_ring = 0;  // field steps stored as a ring of f_ring steps (step t at slot t % f_ring); 0: step t at t
  int m_ring = 0;  // same for the puncture masks and the per-segment counts/offsets
  // One byte per detection tile-step (16 x 8 x 4 anchors at one step; stored like the masks, ring slots included):
  // 1 when the sign certificate proved the tile-step empty, whose masks are then not written (read them as zero).
  unsigned char* cert = nullptr;
};
// Number of detection tiles per step (cert entries per plane).
inline long long cert3_plane(const Grid3& g) {
  return (long long)((g.nx + 15) / 16) * ((g.ny + 7) / 8) * ((g.nz + 3) / 4);
}

struct Out3 {
  long long* face_id;
  float* pos;
  float* mu;
  uint8_t* type;
  uint8_t* flags;
  unsigned* parent;
  uint2* work;
};

constexpr int kDetectRows = 8;  // anchor rows of a detection wavefront
// Detection; ty: anchor rows per workgroup (8, 16 or 32), tt: steps per slab.  Sets ST_WIDE when a component reaches
// 2^24 (the emission then takes its 128-bit form) and ST_RANGE when one reaches 2^62.
hipError_t launch_detect2d(const Grid2& g, int ty, int tt, uint16_t* masks, int* seg_cnt, unsigned* status,
                           hipStream_t s);
// Tiled emission: workgroups of 64 x kEmitRows anchors marching through slabs of tt (at most kEmitSteps) steps.
constexpr int kEmitRows = 8, kEmitSteps = 16;
hipError_t launch_emit2d(const Grid2& g, bool wide, int tt, const uint16_t* masks, const int* seg_cnt,
                         const long long* seg_off, const Out2& o, unsigned* status, unsigned long long* cnt,
                         hipStream_t s);

// Sparse emission (ids of the non-empty row segments, then a lane per hit): same outputs as launch_emit2d, for fields
// with few hits per vertex.  Each hit writes its parent (its first smaller partner or itself) and its link slot
// o.work[i] ((i, i) when absent), united by launch_uf_hook_slots.
hipError_t launch_emit2d_sparse(const Grid2& g, bool wide, const uint16_t* masks, const int* seg_cnt,
                                const long long* seg_off, long long n_hits, const Out2& o, unsigned* status,
                                unsigned long long* cnt, hipStream_t s);
// Prefixes of the series' blocks of 64 segments and of 64 hits (no blocks: a series in the tiled form).
hipError_t launch_emit2d_sparse_batched(const Series2* S, const long long* seg_prefix, const long long* hit_prefix,
                                        const unsigned* gbase, int nser, long long seg_blocks, long long hit_blocks,
                                        bool wide, unsigned* status, hipStream_t s);

hipError_t launch_emit2d_steps(const Grid2& g, bool wide, const uint16_t* masks, const int* seg_cnt,
                               const long long* seg_off, const Out2& o, unsigned* status, unsigned long long* cnt,
                               hipStream_t s);
hipError_t launch_detect2d_batched(const Series2* S, const int* prefix, int nser, int total_items, int tt, int kind,
                                   int* counter, unsigned* status, hipStream_t s);
hipError_t launch_emit2d_batched(const Series2* S, const int* prefix, int nser, int total_items, bool wide,
                                 int* counter, unsigned* status, unsigned long long* work_cnt, hipStream_t s);
// Labels for concatenated series: hit i belongs to the series s with gbase[s] <= i < gbase[s+1].
hipError_t launch_uf_label_batched(unsigned* parent, const Series2* S, const unsigned* gbase, int nser, long long n,
                                   hipStream_t s);

// 3D detection of the steps [t_begin, t_end).  launch_facts3d marks the tile-steps proved empty (g.cert), lists the runs
// of the others (at most `most` <= 16 steps each; runs: cert3_plane entries per step, *n_runs counts up from its value)
// and reports non-finite and out-of-range values; launch_detect3d tests the listed runs and writes their masks and counts
// (the counts of the other tile-steps are the caller's to clear).  facts: cert3_plane words per plane, stored like the
// masks (ring slots included), planes t_begin .. t_end.  The narrow variant does nothing once ST_WIDE is set.
hipError_t launch_facts3d(const Grid3& g, int most, unsigned long long* facts, uint2* runs, unsigned long long* n_runs,
                          unsigned* status, hipStream_t s);
// taken: work counter, zero before the call.
hipError_t launch_detect3d(const Grid3& g, bool wide, const uint2* runs, const unsigned long long* n_runs,
                           unsigned long long* taken, uint64_t* masks, int* seg_cnt, const unsigned* status,
                           hipStream_t s);
// Emission of the n_hits hits of the steps [t_begin, t_end), whose output indices start at `first`.
hipError_t launch_emit3d(const Grid3& g, bool wide, const uint64_t* masks, const int* seg_cnt,
                         const long long* seg_off, long long first, long long n_hits, const Out3& o, unsigned* status,
                         unsigned long long* cnt, hipStream_t s);

// Exclusive scan of n int32 counts into int64 offsets; total written to *total (device).  tmp must hold
// scan_tmp_elems(n) int64 values.
size_t scan_tmp_elems(long long n);
hipError_t launch_scan(const int* in, long long* out, long long n, long long* total, long long* tmp, hipStream_t s,
                       long long base = 0);

// Trajectory post-processing (post.hip).
// Bytes of the lookup tables of a call (by vertex or by vertex row).
size_t traj_table_bytes(int n, const int64_t* dims_with_t, long long n_hits);
size_t order_hits_bytes(int n, const int64_t* dims_with_t, long long n_hits);
size_t order_labels_bytes(int n, const int64_t* dims_with_t);
// Words of 64 hits (ceil(n_hits / 64)): root flags, their counts and scan; table: traj_table_bytes.
struct TableScratch {
  unsigned long long* bits;
  int* cnt;
  long long *base, *scan_tmp;
  void* table;
};
hipError_t launch_traj_table(int n, const int64_t* dims_with_t, const long long* face_id, const long long* label,
                             const float* pos, long long n_hits, long long n_traj, const TableScratch& sc,
                             long long* roots, unsigned long long* hits, int* t_min, int* t_max, int* n_ends,
                             long long* n_roots, unsigned* status, hipStream_t s);
hipError_t launch_slice_range(int n, const int64_t* dims_with_t, const long long* face_id, long long n_hits,
                              long long t0, long long* range, hipStream_t s);
hipError_t launch_slice_compact(int n, const int64_t* dims_with_t, const long long* face_id, long long lo,
                                long long cnt, int* flag, long long* off, long long* total, long long* tmp,
                                long long* idx_out, bool scatter, hipStream_t s);
hipError_t launch_filter_loops(const long long* label, long long n_hits, const long long* roots, long long n_traj,
                               const int* t_min, const int* t_max, const int* n_ends, float min_duration,
                               uint8_t* keep, hipStream_t s);

// Order of the points along each trajectory.  setup: per-trajectory offsets (offsets[n_traj] = n_hits), cell
// neighbours nb ([n_hits][2] int32), loop cuts, ruler flags (words of 64 hits, as in TableScratch; *n_rulers = count).
// walk: the rulers' hits (list) and the states of their arms (st, 2 n_rulers), from walks to the next rulers.  jump:
// pointer jumping over the listed arms (act = null: all), still-open ones appended to next.  place: the rulers'
// positions (place, n_rulers) and order[]; *placed += the hits between the rulers.
struct OrderScratch {
  int* nb;
  unsigned long long* bits;
  int* cnt;
  long long* base;
  int* points;          // [n_traj]
  void *hits, *labels;  // order_hits_bytes, order_labels_bytes
  long long* scan_tmp;  // for the words and for n_traj
};
hipError_t launch_order_setup(int n, const int64_t* dims_with_t, const long long* face_id, long long n_hits,
                              const long long* roots, const unsigned long long* n_points, const int* n_ends,
                              long long n_traj, const OrderScratch& sc, long long* n_rulers, long long* offsets,
                              unsigned* status, hipStream_t s);
hipError_t launch_order_walk(const OrderScratch& sc, long long n_rulers, long long n_hits, int* list,
                             unsigned long long* st, unsigned* status, hipStream_t s);
hipError_t launch_order_jump(const unsigned* act, long long n_act, long long n_hits, unsigned long long* st,
                             unsigned* next, unsigned long long* next_n, unsigned* status, hipStream_t s);
hipError_t launch_order_place(int n, const int64_t* dims_with_t, const long long* label, long long n_hits,
                              const long long* roots, long long n_traj, const long long* offsets,
                              const OrderScratch& sc, const int* list, long long n_rulers,
                              const unsigned long long* st, unsigned* place, long long* order,
                              unsigned long long* placed, unsigned* status, hipStream_t s);
// Isovolume tracking (iso.hip).  Words of 64 vertices of a row (ceil(nx / 64) * ny * nz * nt of them) carry the sides
// (bits) and the counts of crossings, cubes with tetrahedra and runs of equal sides, whose exclusive scans are hbase,
// abase, rbase; *n_tets += the tetrahedra.
hipError_t launch_iso_count(const float* f, int nx, int ny, int nz, int nt, float c, unsigned long long* bits,
                            int* hcnt, int* acnt, int* rcnt, unsigned long long* n_tets, unsigned* status,
                            hipStream_t s);
// Component of every run (comp, n_runs; parent: scratch of n_runs), *n_comp += their number, first (n_runs) cleared.
hipError_t launch_iso_components(int nx, int ny, int nz, int nt, const unsigned long long* bits,
                                 const long long* rbase, long long n_runs, unsigned* parent, unsigned* comp,
                                 long long* first, unsigned long long* n_comp, hipStream_t s);
// Crossings with their points and labels, tetrahedra.  Scratch: vinfo (one word per vertex: hits before it in its word
// | crossing mask << 16), hcomp (n_hits), list (n_active cubes), and per 64 of them tcnt and tbase (one entry more), with
// scan_tmp for that many.
hipError_t launch_iso_emit(const float* f, int nx, int ny, int nz, int nt, float c, const unsigned long long* bits,
                           const int* hcnt, const long long* hbase, const long long* abase, const long long* rbase,
                           const unsigned* comp, long long n_hits, long long n_active, unsigned* vinfo,
                           long long* edge_id, float* pos, unsigned* hcomp, long long* first, long long* list,
                           int* tcnt, long long* tbase, long long* scan_tmp, int* tets, long long* label,
                           hipStream_t s);

// Quantum vortex surfaces (vortex.hip): edge signs, positive-triangle masks (tmask, 50 bits), the triangles before each
// vertex in its word of 64 vertices of a row, and the words' counts (ceil(nx / 64) * ny * nz * nt); then, with their
// scan wbase, triangle ids, points and the union-find forest.  Grids of (ceil(nx / 128), ny, nz * nt) blocks
// (ny, nz * nt <= 65535).
hipError_t launch_vx_detect(const float* psi, int nx, int ny, int nz, int nt, float qscale, unsigned short* emask,
                            unsigned long long* tmask, unsigned short* before, int* wcnt, unsigned* status,
                            hipStream_t s);
hipError_t launch_vx_emit(const float* psi, int nx, int ny, int nz, int nt, float qscale,
                          const unsigned long long* tmask, const unsigned short* before, const int* wcnt,
                          const long long* wbase, long long n_hits, long long* tri_id, float* pos, unsigned* parent,
                          hipStream_t s);
// Critical points on an extruded triangle mesh (prism.hip): words of 64 faces per step (ceil(S / 64) * nt of them) with
// their counts, whose scan is base (*suspect: a cleared word of scratch); then emission and the tetrahedron unions.
struct PmScratch {
  float* rows;                       // 2 nv nt: the quantised field, vertex-major
  unsigned long long* edge_signs;    // 2 ne ceil(nt / 64)
  unsigned long long* vertex_signs;  // nv ceil(nt / 64)
  unsigned long long* bits;
  int* cnt;
  long long* base;
};
hipError_t launch_pm_test(const float* xy, const int* tri, const int* edge, const int* tri_edge, const float* field,
                          long long nv, long long nf, long long ne, int nt, float qscale, const PmScratch& sc,
                          unsigned* suspect, unsigned* status, hipStream_t s);
// edge_tri: [ne][2] triangles of each edge (-1: none), or null for a mesh with an edge of more than two triangles
// (the unions then visit every prism).
hipError_t launch_pm_emit(const float* xy, const int* tri, const int* edge, const int* tri_edge, const int* edge_tri,
                          const float* field, long long nv, long long nf, long long ne, int nt, float qscale,
                          const PmScratch& sc, long long n_hits, long long* face_id, float* pos, unsigned* parent,
                          unsigned* status, hipStream_t s);
// Type smoothing and run simplification along an order (starts: words of 64 positions, as in RunScratch).
hipError_t launch_smooth(const long long* order, const long long* offsets, const int* n_ends, long long n_traj,
                         long long n_hits, const uint8_t* type_in, int half, unsigned long long* start_bits,
                         long long* start_base, uint8_t* type_out, unsigned* status, hipStream_t s);
// Words of 64 positions: trajectory starts (ceil(n_hits / 64)), run starts (one for position n_hits too); bounds and type
// of the runs (n_hits).
struct RunScratch {
  unsigned long long* start_bits;
  long long* start_base;
  unsigned long long* run_bits;
  int* run_cnt;
  long long *run_base, *scan_tmp;
  int *t_min, *t_max;
  uint8_t* run_type;
};
hipError_t launch_simplify(int n, const float* pos, const long long* order, const long long* offsets,
                           const int* n_ends, long long n_traj, long long n_hits, const uint8_t* type_in, float theta,
                           const RunScratch& sc, long long* n_runs, uint8_t* type_out, unsigned* status,
                           hipStream_t s);

// Union-find passes over n hits: extra unions from the work list, then labels = face_id of the root.
hipError_t launch_uf_hook(unsigned* parent, const uint2* work, const unsigned long long* work_count,
                          long long max_work, hipStream_t s);
// Compression of a forest whose parents all point to smaller indices (the sparse emission's), in one pass.
hipError_t launch_uf_compress(unsigned* parent, long long n, hipStream_t s);
// Unions of a link array with one slot per entry: entries (a, a) are empty.
hipError_t launch_uf_hook_slots(unsigned* parent, const uint2* slots, long long n_slots, hipStream_t s);
hipError_t launch_uf_label(unsigned* parent, const long long* face_id, long long* label, long long n,
                           unsigned long long* cnt, hipStream_t s);

}  // namespace ftk
