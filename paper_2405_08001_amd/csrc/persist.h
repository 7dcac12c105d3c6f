// Persistent iteration kernel: one launch runs many PNCG iterations, with the
// mesh tables and the vertex state of each block held in LDS and the blocks
// meeting twice per iteration through memory (persist.hip).
#pragma once

#include <cstdint>
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

// Byte offsets of the arrays of a block in its dynamic LDS.  Local vertices
// [cap_loc]: x, m (mass), p, pg, fl (flags); own ones [cap_own]: xt, xb (list
// build positions), P (1 / diag), tot (element sums), g (two copies, by
// iteration parity), ce (corner-entry range); the others: hv (global vertex).
// Tets [cap_tet]: rec (record, kRec reals), tl (corners), te (global tet, where
// the records stay in memory).
struct PersistLayout {
  unsigned x, m, xt, xb, P, tot, p, pg, g, rec, tl, te, hv, ce, lane, dt, dv, fl;
};

struct PersistArgs {
  int blocks, vb, grid;          // physical blocks, logical blocks in each, logical blocks in all
  const PersistBlock* blk;       // [blocks]
  const int* loc_v;              // global vertex of each local one
  const int* tet_e;              // global tet of each local one
  const ushort4* tet_l;          // its corners as local vertices
  const ushort2* lane;           // [64 nWaves] {local tet << 2 | corner or kNone, local vertex | kLaneLast}
  const unsigned short* dtet;    // [nT] local tet of each tet, in the block whose curvature pass takes it
  const unsigned short* dvert;   // [nV] local vertex of each vertex, likewise
  const uint8_t* lflag;          // [nV] vertex flags | kPairVertex
  // exchange buffers, three sets each (persist.hip)
  unsigned long long* slot_grad; // [3][8][grid]
  unsigned long long* slot_dir;  // [3][3][grid]
  unsigned long long* pgx;       // [3][nV][3]
  int* ring;                     // set of the next launch's first iteration
  long long limit;               // longest wait, in ticks of the 100 MHz clock
  int cap_loc, cap_own, cap_tet, cap_lane, cap_dt, cap_dv;   // largest of each over the blocks
  int elem_lds;                  // element records in LDS (else read from memory)
  PersistLayout at;
  size_t lds;                    // dynamic LDS of a block
};

constexpr unsigned short kNone = 0xffff;
constexpr unsigned short kLaneVert = 0x7fff, kLaneLast = 0x8000;   // vertex of a lane (kLaneVert: none); its last lane
constexpr int kRec = 12;              // reals of an element record in LDS (11, padded to 16 bytes)
constexpr uint8_t kPairVertex = 4;    // corner of a surface triangle or edge (beside kFixed, kSurface)
constexpr size_t kPersistLds = 158 * 1024;   // of the 160 KiB of a compute unit, less the static arrays
constexpr int kPersistMaxIters = 512;  // iterations of one launch (the host looks at the error bits between launches)

// Host-built tables of PersistArgs; false where a block's share does not fit
// (then the step uses the per-iteration launches).
struct PersistTables {
  std::vector<PersistBlock> blk;
  std::vector<int> loc_v, tet_e;
  std::vector<ushort4> tet_l;
  std::vector<ushort2> lane;
  std::vector<unsigned short> dtet, dvert;
};
bool persist_build(int nV, int nT, const int* tets, const std::vector<int>& inc, const std::vector<int>& inc_vert,
                   int grid, bool fp64, bool self, PersistTables& T, PersistArgs& P);
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
