// Persistent iteration kernel: one launch runs many PNCG iterations, with the
// mesh tables and the vertex state of each block held in LDS and the blocks
// meeting twice per iteration through memory (persist.hip).
#pragma once

#include <cstdint>
#include <memory>
#include <vector>

#include "internal.h"

namespace pncg {

// A block of the persistent kernel hosts `vb` consecutive logical blocks of
// the per-iteration launches (the same slices of the incidence waves, tets
// and vertices, summed in the same order, so both forms give the same bits).
struct PersistBlock {
  int loc_off;            // into loc_v: own vertices first, then the others its tets touch
  int nown, nloc;
  int tet_off, ntet;      // into tet_e / tet_l
  int w0, nw;             // incidence waves
  int t0, nt;             // tets of the curvature pass
  int v0, nv;             // vertices of the curvature pass
};

// One tet of a chunk of incidence waves: the lanes, counted from the chunk's
// first, that its four corners' terms go to (kNone: a vertex of another chunk
// or block).
struct alignas(4) PersistEntry {
  unsigned short slot[4];
  unsigned short tet, pad;     // local tet
};

// Byte offsets of the arrays of a block in its dynamic LDS.  Local vertices
// [cap_loc]: x, m (mass), p, pg, fl (flags); own ones [cap_own]: xt, xb (list
// build positions), P (1 / diag), g (two copies, by iteration parity), ce
// (corner-entry range), run (row runs); the others: hv (global vertex).  Tets [cap_tet]: rec (record, kRec
// reals), tl (corners), te (global tet, where the records stay in memory).
// res: the corner terms of a chunk's lanes; seg: the row runs; tot: the sums of
// the row runs (by tet) or own vertices (by lane); lane: the block's lanes; wm:
// its waves (wave_last); rp: run partials of the pair entries [cap_rp][6]; dg:
// pairs of the curvature pass.
struct PersistLayout {
  unsigned x, m, xt, xb, P, tot, p, pg, g, rec, tl, te, hv, ce, lane, dt, dv, fl, res, seg, run, wm, rp, dg;
};

struct PersistArgs {
  int blocks, vb, grid;          // physical blocks, logical blocks in each, logical blocks in all
  const PersistBlock* blk;       // [blocks]
  const int* loc_v;              // global vertex of each local one
  const int* tet_e;              // global tet of each local one
  const ushort4* tet_l;          // its corners as local vertices
  const ushort2* lane;           // [64 nWaves] {local tet << 2 | corner or kNone, local vertex | kLaneLast}
  const ulonglong2* wave_last;   // [nWaves] {mask of the vertices' last lanes, first of them as a local vertex}
  // row runs: the lanes of one vertex within one row of 16 lanes of a wave
  const ushort2* seg;            // {last lane within the chunk, lanes before it}
  const ushort2* run;            // [nV] {first row run in the block, number}
  const int4* chunk;             // [blocks][chunks + 1] {first entry; first own vertex and row run in the
                                 // block; first row run of the block}
  const PersistEntry* entry;
  const unsigned short* dtet;    // [nT] local tet of each tet, in the block whose curvature pass takes it
  const unsigned short* dvert;   // [nV] local vertex of each vertex, likewise
  const uint8_t* lflag;          // [nV] vertex flags | kPairVertex
  // exchange buffers, three sets each (persist.hip)
  unsigned long long* slot_grad; // [3][8][grid]
  unsigned long long* slot_dir;  // [3][3][grid]
  unsigned long long* pgx;       // [3][nV][3]
  int* ring;                     // set of the next launch's first iteration
  long long limit;               // longest wait, in ticks of the 100 MHz clock (see Wait)
  int cap_own;                   // most own vertices of a block
  int chunks;                    // chunks of a block's waves
  int cap_rp, cap_dg;            // pair entries whose run partials, and pairs whose geometry, fit in LDS
  int elem_lds;                  // element records in LDS (else read from memory)
  PersistLayout at;
  size_t lds;                    // dynamic LDS of a block
};

constexpr unsigned short kNone = 0xffff;
constexpr unsigned short kLaneVert = 0x7fff, kLaneLast = 0x8000;   // vertex of a lane (kLaneVert: none); its last lane
constexpr int kMaxChunks = 8;
// Most chunks of a step's blocks; the adjoint takes kMaxChunks.  25 iterations,
// here and by launches: 907 and 977 us (118,000 tets float64) and 859 and 975
// us (179,000 mixed) with 6 chunks, 989 and 969 us (125,000 float64) and 1,047
// and 1,048 us (206,000 mixed) with 8.  CG iterations, 125,000 tets, 8 chunks:
// 8.9 and 10.5 ms.
constexpr int kStepChunks = 6;
constexpr int kRec = 12;              // reals of an element record in LDS (11, padded to 16 bytes)
constexpr int kRunPartials = 256;     // pair entries of a block with run partials in LDS
constexpr size_t kPairGeom = 88;      // bytes of a PairGeom (persist.hip); one wave of them per logical block
constexpr uint8_t kPairVertex = 4;    // corner of a surface triangle or edge (beside kFixed, kSurface)
// Dynamic LDS of a block: the 160 KiB of a compute unit less the kernels'
// static arrays (k_persist's 4,016 bytes at most, k_cg_persist's 2,256).
constexpr size_t kPersistLds = 160 * 1024 - 4016, kCgLds = 160 * 1024 - 2256;
constexpr int kPersistMaxIters = 512;  // iterations of one launch (the host looks at the error bits between launches)

// The adjoint's persistent CG kernel on the same tables.  Local vertices: x, z,
// p, w; own ones: q, diag, lam (3 doubles each), m, fl, run; the rest as in
// PersistLayout, with three values per slot.
struct CgLayout {
  unsigned x, z, p, w, q, diag, lam, m, res, tot, tl, hv, seg, run, wm, fl;
};
struct CgPersist {
  PersistArgs P;
  CgLayout at;
  size_t lds;
  int most;              // entries of the largest block's chunk
};

// A table that is filled after it is sized (a vector would write it twice).
template <typename T>
struct PersistTable {
  using value_type = T;
  std::unique_ptr<T[]> d;
  size_t n = 0;
  void resize(size_t m) { d.reset(new T[m]); n = m; }
  T* data() { return d.get(); }
  size_t size() const { return n; }
};
// Host-built tables of PersistArgs, and the layouts of the two element forms:
// [0] by tet, [1] by (tet, corner) lane for the corotated models.
struct PersistTables {
  std::vector<PersistBlock> blk;
  PersistTable<int> loc_v, tet_e;
  PersistTable<ushort4> tet_l;
  PersistTable<ushort2> lane, seg;
  std::vector<ushort2> run;
  PersistTable<ulonglong2> wave_last;
  std::vector<int4> chunk;
  PersistTable<PersistEntry> entry;
  PersistTable<unsigned short> dtet;
  std::vector<unsigned short> dvert;
  PersistArgs form[2];
  CgPersist cg;         // layout only
  bool ok[2], cg_ok;    // which can use them: a block's share fits in LDS
};
inline int persist_form(int model) { return model == kModelCorot ? 1 : 0; }
// Who asks for the tables: a step, by its element form, or the adjoint.
constexpr int kForAdjoint = 2;
// False, and no tables, where who asks (persist_form, kForAdjoint) could not use them.
bool persist_build(int nV, int nT, const int* tets, const std::vector<int>& inc, const std::vector<int>& inc_vert,
                   int grid, bool fp64, bool self, int who, PersistTables& T);
// Fill the exchange buffers with the empty mark and reset the ring.
void persist_clear(const PersistArgs& P, int nV, hipStream_t s);
// Iterations [k0, k0 + kPersistMaxIters) of a step, or up to its stop, pause or
// cap.  mode kModeNormal (k0 = 0, after launch_predict), kModeResume (after a
// list rebuild) or kModeContinue (after a launch that reached its own limit).
template <typename R>
void launch_persist(const Args<R>& A, const PersistArgs& P, int k0, int mode, hipStream_t s);
// Whether every block can be resident at once on the current device.
template <typename R>
hipError_t persist_fits(const PersistArgs& P, int model, bool self, int compute_units, bool* ok);

}  // namespace pncg
