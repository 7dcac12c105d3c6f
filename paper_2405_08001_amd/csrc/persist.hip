// The PNCG iterations of a step in one launch (Algorithm 1, Sec. 4.1-4.4).
//
// What bounds it: an iteration is two passes over the mesh, each ended by a
// reduction over the whole device.  As two launches (solver_kernels.hip) it
// waits on dependent memory round trips: the partials, the incidence codes,
// the element records, the corner positions, the vertex arrays.  Here every
// block keeps its share in LDS for the whole step (the 256 compute units
// hold 40 MB), so a pass reads memory only for what other blocks changed: P g
// of the vertices it shares with them, and the reduction's partial sums.
//
// Split.  A block owns the vertices of its incidence waves and keeps x, p and
// P g of every vertex its tets touch, its own and its neighbours'.  Each
// block forms the direction p = -P g + beta p and the update x += alpha p of
// all of them, so only P g crosses blocks, once per iteration.
//
// Element terms.  The launches evaluate a tet in each of its four corners'
// lanes; here a block evaluates it once and leaves the corners' terms in LDS
// slots, one per incidence lane, which are then added per vertex in the order
// of the lanes' segmented sum (row_run_sum).  That takes 0.4 to 0.5 of the
// element arithmetic for more LDS traffic; the slots hold a chunk of the
// waves at a time where they do not all fit.  The corotated models keep the
// lanes (see the element pass).  Waves that have pair terms of their own leave
// the tets to the others.
//
// Meeting.  A block publishes its partial sums and P g with agent-scope
// stores and polls the other blocks' by agent-scope loads, one round trip per
// meeting.  Every 8-byte word is its own flag: a word that still holds the
// empty mark has not arrived.  There are three sets of words; iteration i of
// the context uses set i mod 3.  A block clears its words of set i - 1 after
// the first meeting of iteration i (every block has then passed the second
// meeting of i - 1, so nobody reads them), and waits for those stores before
// it publishes for the second meeting of i; a reader of set i + 2 has passed
// that meeting and so cannot see the old words.  The launch's first set was
// cleared by an earlier launch, the other two are cleared at its start.
// Measured on 256 blocks: 3.3 us for 3 sums, against 4.7 us through one
// gathering block per sum.
//
// Waits.  All blocks must be resident: the grid has at most one block per
// compute unit, and launches of several contexts of a process that would not
// fit beside each other take turns (UnitsHeld).  A wait is bounded by the clock
// all the same; a launch that runs out raises kErrSync, writes nothing, and the
// host runs the step again with the per-iteration launches, which give the same
// bits.
//
// Measured, us per pass: by launches, here with element terms by lane, by tet:
//   1,296 tets float64, 20 iterations           446   287   282
//   13,182 tets corotated mixed, 25             546   486   455 (by lane)
//   30,000 tets float64, 48                    1178   871   799
//   110,000-tet pile mixed, 2 frames of 25     1534  1003   952
//   21,000-tet pile float64, 2 frames of 25    1132   806   768
#include <cfloat>
#include <climits>

#include "iteration_common.h"
#include "persist_common.h"

namespace pncg {

namespace {

// one component of P g as a word (a float's upper half is zero, so it is never
// the empty mark)
__device__ __forceinline__ u64 pg_word(float a) { return (u64)(unsigned)__float_as_int(a); }
__device__ __forceinline__ u64 pg_word(double a) { return full(word(a)); }
__device__ __forceinline__ void from_word(u64 w, float& a) { a = lo_float(w); }
__device__ __forceinline__ void from_word(u64 w, double& a) { a = as_double(w); }

// padded 4-vector arrays shared between blocks during the launch (x and p of
// the pair vertices)
__device__ __forceinline__ V3<double> ld3_agent(const double4* a, int i) {
  const u64* p = reinterpret_cast<const u64*>(a + i);
  return mk3(as_double(ld_agent(p)), as_double(ld_agent(p + 1)), as_double(ld_agent(p + 2)));
}
__device__ __forceinline__ V3<float> ld3_agent(const float4* a, int i) {
  const u64* p = reinterpret_cast<const u64*>(a + i);
  const u64 w0 = ld_agent(p), w1 = ld_agent(p + 1);
  return mk3(lo_float(w0), hi_float(w0), lo_float(w1));
}
// one component
__device__ __forceinline__ void st1_agent(double4* a, int i, int j, double v) {
  st_agent(reinterpret_cast<u64*>(a + i) + j, word(v));
}
__device__ __forceinline__ void st1_agent(float4* a, int i, int j, float v) {
  __hip_atomic_store(reinterpret_cast<unsigned*>(a + i) + j, (unsigned)__float_as_int(v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

// Positions of pair corners, which may belong to any block: x_k as x_{k-1} +
// alpha p_k (lazy) or as stored by an earlier launch.
template <typename R>
struct PairPos {
  const double4* x;
  const R4<R>* p;
  double alpha;
  int lazy;
  __device__ __forceinline__ V3<double> operator()(int v) const {
    V3<double> r = ld3_agent(x, v);
    if (lazy) {
      const V3<R> q = ld3_agent(p, v);
      r = mk3(fma(alpha, double(q.x), r.x), fma(alpha, double(q.y), r.y), fma(alpha, double(q.z), r.z));
    }
    return r;
  }
};

// Scalars of the running iteration, the same in every block.
struct Run {
  double alpha, dE, dE0, D;            // first part
  double beta, gTp, gPg, gnorm, g0, n_active, Dx;   // direction part
  int a_up, exit, bad;
};

template <typename R>
struct KArgs {
  Args<R> A;
  PersistArgs P;
  int k0, mode;
};
template <typename R>
using KPtr = ArgPtr<KArgs<R>>;

template <typename R>
struct Elem {
  R B[9], vmu, vlam;
};
// record t of the block: in LDS (16-byte aligned) or in memory
template <typename R>
__device__ __forceinline__ Elem<R> element(KPtr<R> K, const unsigned char* lds, int t) {
  Elem<R> e;
  if (K->P.elem_lds) {
    const R* r = reinterpret_cast<const R*>(__builtin_assume_aligned(lds + K->P.at.rec + kRec * sizeof(R) * t, 16));
#pragma unroll
    for (int j = 0; j < 9; ++j) e.B[j] = r[j];
    e.vmu = r[9]; e.vlam = r[10];
  } else {
    const ElemRec<R>& r = K->A.elem[reinterpret_cast<const int*>(lds + K->P.at.te)[t]];
#pragma unroll
    for (int j = 0; j < 9; ++j) e.B[j] = r.B[j];
    e.vmu = r.vmu; e.vlam = r.vlam;
  }
  return e;
}

// Closest points of a pair (point-triangle or edge-edge) at `pos`; false if it
// is not active (pair_closest).
template <typename R, typename Pos>
__device__ __forceinline__ bool pair_at(const Args<R>& A, bool pt, const int (&iv)[4], const Pos& pos, Closest& c) {
  V3<double> X[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) X[i] = pos(iv[i]);
  c = pt ? closest_pt(X[0], X[1], X[2], X[3]) : closest_ee(X[0], X[1], X[2], X[3]);
  if (!(c.d > 0.0)) {
    raise_err(A.status, kErrPenetration);
    return false;
  }
  return c.d < A.dhat;
}

// sum_i c_i p_{k+1}(iv_i) of a pair, its corners in any block: P g as sent
// before the first meeting (it may still be on its way) and p_k as stored.
// All words are asked for at once.  False if the wait runs out.
template <typename R>
__device__ __forceinline__ bool pair_dir(const int (&iv)[4], const double (&c)[4], const u64* pgx, const R4<R>* pk, R beta,
                                         long long limit, V3<double>& sp) {
  u64 w[12];
  V3<R> p[4];
#pragma unroll
  for (int i = 0; i < 12; ++i) w[i] = ld_agent(pgx + 3 * (size_t)iv[i / 3] + i % 3);
#pragma unroll
  for (int i = 0; i < 4; ++i) p[i] = ld3_agent(pk, iv[i]);
  Wait t(limit);
  for (;;) {
    bool here = true;
#pragma unroll
    for (int i = 0; i < 12; ++i) {
      if (w[i] != kEmpty) continue;
      w[i] = ld_agent(pgx + 3 * (size_t)iv[i / 3] + i % 3);
      here = false;
    }
    if (here) break;
    if (t.over()) return false;
  }
  sp = mk3(0.0, 0.0, 0.0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    V3<R> g;
    from_word(w[3 * i], g.x); from_word(w[3 * i + 1], g.y); from_word(w[3 * i + 2], g.z);
    sp = fma3(c[i], cast3<double>(direction(g, p[i], beta)), sp);
  }
  return true;
}

// A pair of the curvature pass, its closest points found before the first
// meeting (v[0] < 0: not active).
struct PairGeom {
  double c[4], t[3], ca, cb;
  int v[4];
};
static_assert(sizeof(PairGeom) == kPairGeom, "PairGeom size");

// The arguments that the terms of a pair read.
template <typename R>
__device__ __forceinline__ Args<R> pair_args(KPtr<R> K) {
  Args<R> a;
  a.pv = K->A.pv;
  a.status = K->A.status;
  a.dhat = K->A.dhat;
  a.kappa = K->A.kappa;
  a.flags = K->A.flags;
  return a;
}

}  // namespace

// SELF: point-triangle / edge-edge pairs by the segmented scatter, each block
// evaluating its own vertices' entries (the sparse-contact form, see
// fused_pairs).
template <typename R, int M, bool SELF, int MAXT = 2 * GradBlock<R, M>::value>
__global__ void __launch_bounds__(MAXT) k_persist(KArgs<R>) {
  constexpr int GB = GradBlock<R, M>::value, DB = DirBlock<R, M>::value;
  constexpr int GW = GB / kWave, DW = DB / kWave;
  constexpr bool kTets = M != kModelCorot;   // element terms by tet, or by (tet, corner) lane
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ double sh[2 * 8 * 24];
  __shared__ double shg[8 * 4];
  __shared__ double planes[4 * kMaxPlanes];
  __shared__ int count[2];       // active pairs and planes, by iteration parity
  __shared__ u64 moved[2];       // largest squared displacement since the list build
  __shared__ Run run;
  __shared__ PersistBlock B;
  __shared__ int4 chk[kMaxChunks + 1];   // of each chunk: first entry, own vertex, row run
  __shared__ int ent[4];         // corner entries [b, e) of each logical block's vertices
  __shared__ int slot_id[2];     // partial index of each logical block: the blockIdx of the launch that has it
  __shared__ int busy[16];       // waves with pair work
  __shared__ int lblk[2][6];     // per logical block: incidence waves [b, e), tets [b, e), vertices [b, e)
  // thread, wave, and the wave's logical block within the block (vi) with the
  // thread's place in it (vt); taken anew by every phase
#define PHASE                                                                                          \
  const KPtr<R> K = kernel_args<KArgs<R>>();                                                                        \
  const int tid = fresh(threadIdx.x), BS = K->P.vb * GB, n = K->P.grid, vb = K->P.vb;                  \
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = vb * GW; \
  const int vi = wave >= GW ? 1 : 0, vt = tid - vi * GB;                                               \
  (void)lane, (void)vt, (void)nwaves, (void)n, (void)BS
#define LDS_AT(T, field) reinterpret_cast<T*>(lds + K->P.at.field)

  int k0, lp, set0, own0;
  PersistEntry entry0{};         // the thread's first entry of the first chunk
  // Pair work of the thread, fixed for the launch: corner pci of the pair with
  // corner vertices pw (the first corner entry that it evaluates), or, in the
  // last wave of a logical block where that one has few entries (early, their
  // number), the pair whose geometry it finds for the curvature pass.
  int4 pw = make_int4(0, 0, 0, 0);
  int pci = -1, early = 0;
  int erank = 0, efree = 0;      // place of the wave among those that share the tets (-1: has pair work), their number
  bool pending = false;          // x_k already lacks nothing, but stems from alpha_{k-1} p_k of this launch
  {
    PHASE;
    const bool leader = blockIdx.x == 0 && tid == 0;
    k0 = K->k0;
    const int mode = K->mode;
    // logical blocks lp vb + i of this block; the XCDs (workgroups are dealt
    // round-robin) get contiguous ranges where the grid divides evenly
    lp = (gridDim.x % kXcds) ? blockIdx.x : (blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
    const PersistBlock b = K->P.blk[lp];
    if (tid == 0) B = b;
    if (tid < 2) {
      const int L = lp * vb + min(tid, vb - 1);
      slot_id[tid] = (L % (n / kXcds)) * kXcds + L / (n / kXcds);
      const long long q[3] = {K->A.nWaves, K->A.nT, K->A.nV};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const long long per = (q[i] + n - 1) / n;
        lblk[tid][2 * i] = (int)min(L * per, q[i]);
        lblk[tid][2 * i + 1] = (int)min((L + 1) * per, q[i]);
      }
    }
    // ---- where to begin
    StepStatus* st = K->A.status;
    IterScal* scal = K->A.scal;
    if (tid < 4 * kMaxPlanes) planes[tid] = K->A.planes.p[tid >> 2][tid & 3];
    if (tid < 2) {
      count[tid] = 0;
      moved[tid] = 0;
    }
    if (tid == 0) {
      Run r{};
      if (k0 > 0) {
        const IterScal cur = scal[k0], prev = scal[k0 - 1];
        r.g0 = st->g0;
        r.dE = cur.dE; r.dE0 = cur.dE0; r.a_up = cur.a_up;
        r.D = mode == kModeResume ? 0.0 : cur.D;
        r.gTp = prev.gTp; r.gPg = prev.gPg;
      }
      run = r;
    }
    double D0 = 0.0;
    if (SELF && k0 == 0 && mode == kModeNormal && K->A.carry) {
      // a step that starts on an earlier step's list pauses for a rebuild if
      // x_0 has left it (as first_prologue does)
      for (int j = tid; j < n; j += BS) D0 = fmax(D0, K->A.part_dir[4 * j + 3]);
      D0 = wave_max(D0);
      if (lane == 0) sh[wave] = D0;
      __syncthreads();
      for (int w = 0; w < nwaves; ++w) D0 = fmax(D0, sh[w]);
    }
    const int pause = SELF && D0 > 0.5 * K->A.skin ? 1 : 0;
    if (leader && mode != kModeContinue) {
      IterScal& s = scal[k0];
      if (k0 == 0) {
        s.alpha = 0; s.dE = 0; s.dE0 = 0; s.a_up = 0;
      }
      s.D = 0; s.stop = 0; s.pause = pause;
      st->paused_at = pause ? 0 : -1;
      st->D = D0;
    }
    if (pause) return;

    // ---- tables and state into LDS
    set0 = *K->P.ring;
    const double4* xin = (k0 & 1) ? K->A.x1 : K->A.x0;
    const R4<R>* pin = (k0 & 1) ? K->A.p1 : K->A.p0;
    const int* lv = K->P.loc_v + b.loc_off;
    own0 = lv[0];   // own vertices are consecutive
    double *X = LDS_AT(double, x), *Ms = LDS_AT(double, m), *XT = LDS_AT(double, xt);
    R *Ps = LDS_AT(R, p), *G = LDS_AT(R, g);
    uint8_t* fl = LDS_AT(uint8_t, fl);
    for (int l = tid; l < b.nloc; l += BS) {
      const int v = lv[l];
      const V3<double> x = ld3(xin, v);
      X[3 * l] = x.x; X[3 * l + 1] = x.y; X[3 * l + 2] = x.z;
      const V3<R> p = ldr<R>(pin, v);
      Ps[3 * l] = p.x; Ps[3 * l + 1] = p.y; Ps[3 * l + 2] = p.z;
      Ms[l] = K->A.mass[v];
      fl[l] = K->P.lflag[v] | (K->A.vflag[v] & kFixed);
      if (l < b.nown) {
        const V3<double> xt = ld3(K->A.xt, v);
        XT[3 * l] = xt.x; XT[3 * l + 1] = xt.y; XT[3 * l + 2] = xt.z;
        // the gradient of iteration k0 - 1 (k0's goes to the other copy)
        const V3<R> g = ldr<R>(K->A.g, v);
        R* gp = G + 3 * ((k0 & 1) ? 0 : K->P.cap_own) + 3 * l;
        gp[0] = g.x; gp[1] = g.y; gp[2] = g.z;
        if (SELF) {
          double* XB = LDS_AT(double, xb);
          const V3<double> xb = ld3(K->A.xbuild, v);
          XB[3 * l] = xb.x; XB[3 * l + 1] = xb.y; XB[3 * l + 2] = xb.z;
          int* ce = LDS_AT(int, ce);
          ce[2 * l] = K->A.coff[v];
          ce[2 * l + 1] = K->A.coff[v + 1];
        }
      } else {
        LDS_AT(int, hv)[l - b.nown] = v;
      }
    }
    for (int t = tid; t < b.ntet; t += BS) {
      const int e = K->P.tet_e[b.tet_off + t];
      LDS_AT(ushort4, tl)[t] = K->P.tet_l[b.tet_off + t];
      if (K->P.elem_lds) {
        const ElemRec<R>& r = K->A.elem[e];
        R* d = LDS_AT(R, rec) + kRec * t;
#pragma unroll
        for (int j = 0; j < 9; ++j) d[j] = r.B[j];
        d[9] = r.vmu;
        d[10] = r.vlam;
      } else {
        LDS_AT(int, te)[t] = e;
      }
    }
    if constexpr (kTets) {
      const int nc = K->P.chunks;
      const int4* ck = K->P.chunk + lp * (nc + 1);
      if (tid <= nc) chk[tid] = ck[tid];
      for (int l = tid; l < b.nown; l += BS) LDS_AT(ushort2, run)[l] = K->P.run[own0 + l];
      const int s0 = ck[nc].w;
      for (int i = tid; i < ck[nc].z; i += BS) LDS_AT(ushort2, seg)[i] = K->P.seg[s0 + i];
    } else {
      for (int i = tid; i < b.nw * kWave; i += BS) LDS_AT(ushort2, lane)[i] = K->P.lane[(size_t)b.w0 * kWave + i];
    }
    for (int i = tid; i < b.nw; i += BS) LDS_AT(ulonglong2, wm)[i] = K->P.wave_last[b.w0 + i];
    for (int i = tid; i < b.nt; i += BS) LDS_AT(unsigned short, dt)[i] = K->P.dtet[b.t0 + i];
    for (int i = tid; i < b.nv; i += BS) LDS_AT(unsigned short, dv)[i] = K->P.dvert[b.v0 + i];
  }
  auto set_of = [&](int it) { return fresh_s(set0 + it - k0) % 3; };
  // clear this block's words of iteration it's set
  auto clear = [&](int it) {
    PHASE;
    const int s = set_of(it);
    if (tid < 8 * vb) st_agent(K->P.slot_grad + s * 8 * n + (tid & 7) * n + slot_id[tid >> 3], kEmpty);
    if (tid < 3 * vb) st_agent(K->P.slot_dir + s * 3 * n + (tid % 3) * n + slot_id[tid / 3], kEmpty);
    u64* w = K->P.pgx + 3 * ((size_t)s * K->A.nV + own0);
    for (int i = tid; i < 3 * B.nown; i += BS) st_agent(w + i, kEmpty);
  };
  __syncthreads();
  clear(k0 + 1);
  clear(k0 + 2);
  if constexpr (SELF) {
    PHASE;
    if (tid < vb) {
      const int wb = lblk[tid][0], we = lblk[tid][1];
      ent[2 * tid] = wb < we ? K->A.wrange[wb].x : 0;
      ent[2 * tid + 1] = wb < we ? K->A.wrange[we - 1].y : 0;
    }
    __syncthreads();
    if (tid == 0) {
      // a logical block without vertices has no entries: an empty range beside the other's
      if (vb == 2 && ent[2] >= ent[3]) ent[2] = ent[3] = ent[1];
      if (vb == 2 && ent[0] >= ent[1]) ent[0] = ent[1] = ent[2];
    }
    __syncthreads();
    const int e0 = ent[2 * vi], e1 = ent[2 * vi + 1];
    int j = e0 < e1 ? ((e0 >> 6) + (vt >> 6)) * kWave + lane : e1;
    if (j < e0 || j >= e1) j = -1;
    const int chunks = e0 < e1 ? ((e1 - 1) >> 6) - (e0 >> 6) + 1 : 0;
    const long long nq = min(K->A.ncand[0], K->A.cand_cap), pe = (4 * nq + n - 1) / n;
    const bool geom = K->P.cap_dg > 0 && pe <= kWave;
    // (one decision for the launch's blocks would not do: a block whose last
    // waves have entries of their own finds the geometry in the curvature pass)
    bool ge = geom && chunks < GW;
    if (vb == 2) {
      const int o0 = ent[2 - 2 * vi], o1 = ent[3 - 2 * vi];
      ge = ge && (o0 < o1 ? ((o1 - 1) >> 6) - (o0 >> 6) + 1 : 0) < GW;
    }
    early = ge ? (int)pe : 0;
    if (ge && vt >= GB - kWave) {
      const long long eb = (long long)(lp * vb + vi) * pe, ee = min(eb + pe, 4 * nq);
      j = eb + lane < ee ? (int)(eb + lane) : -1;
      if (j >= 0 && (K->A.cent[j] & 3) != 0) j = -1;
      // lanes without a pair
      LDS_AT(PairGeom, dg)[vi * kWave + lane].v[0] = -1;
    }
    if (j >= 0) {
      const int sl = K->A.cent[j];
      pci = sl & 3;
      pw = K->A.pv[sl >> 2];
    }
    const bool b = __any(pci >= 0);
    if (lane == 0) busy[wave] = b ? 1 : 0;
    __syncthreads();
    int before = 0, total = 0;
    for (int w = 0; w < nwaves; ++w) {
      const int f = 1 - busy[w];
      before += w < wave ? f : 0;
      total += f;
    }
    efree = __builtin_amdgcn_readfirstlane(total > 0 ? total : nwaves);
    erank = __builtin_amdgcn_readfirstlane(total == 0 ? wave : b ? -1 : before);
  } else {
    PHASE;
    efree = nwaves;
    erank = wave;
  }
  if constexpr (kTets) {
    PHASE;
    const int e = chk[0].x + erank * kWave + lane;
    if (erank >= 0 && e < chk[1].x) entry0 = K->P.entry[e];
  }

  int k = k0;
  int last_set = set0;      // set of the next launch
  for (;; ++k) {
    if (pending) {
      // ---- first part: alpha, dE and the stop, pause and cap tests
      PHASE;
      const bool leader = blockIdx.x == 0 && tid == 0;
      if (wave == 0) {
        double r[3];
        totals<3>(shg, n, 6u, r);
        if (lane == 0) {
          const double pHp = r[0], pmv = r[1], pmc = r[2];
          const double gTp = run.gTp;
          const double abar = pHp > 0.0 ? -gTp / pHp : HUGE_VAL;
          const double pm = (K->A.flags & 2u) ? pmc : pmv;
          const double aup = (K->A.has_prims && pm > 0.0) ? K->A.dhat / (2.0 * pm) : HUGE_VAL;
          const double alpha = fmin(aup, abar);
          const int hits = aup < abar ? 1 : 0;
          const double dE = predicted_dE(alpha, gTp, pHp);
          IterScal* o = K->A.scal + k;
          StepStatus* st = K->A.status;
          if (!isfinite(alpha)) {
            run.exit = 2;
            if (leader) {
              o->alpha = 0; o->dE = 0; o->dE0 = run.dE0; o->D = run.D; o->stop = 1; o->pause = 0; o->a_up = run.a_up + hits;
              st->stopped = 1; st->final_k = k - 1; st->iters = k - 1; st->reason = 3;
              st->gk = run.gnorm; st->dE0 = run.dE0; st->last_dE = run.dE; st->a_up_hits = run.a_up;
              st->n_active = run.n_active;
            }
          } else {
            const double dE0 = (k == 1) ? dE : run.dE0;
            const double D = fma(alpha, pmv, SELF ? run.Dx : run.D);
            int stop = 0, reason = 0;
            if (K->A.term == 0 && dE < K->A.eps * dE0) { stop = 1; reason = 0; }
            else if (k == K->A.iter_max) { stop = 1; reason = 2; }
            const int pause = (!stop && SELF && D > 0.5 * K->A.skin) ? 1 : 0;
            run.alpha = alpha; run.dE = dE; run.dE0 = dE0; run.D = D;
            run.a_up += hits;
            if (stop || pause || k - k0 >= kPersistMaxIters) run.exit = 1;
            if (leader) {
              o->alpha = alpha; o->dE = dE; o->dE0 = dE0; o->D = D; o->stop = stop; o->pause = pause; o->a_up = run.a_up;
              o->dir_stop = 0;
              if (stop) {
                st->stopped = 1; st->final_k = k; st->iters = k; st->reason = reason;
                st->gk = run.gnorm; st->dE0 = dE0; st->last_dE = dE; st->a_up_hits = run.a_up;
                st->n_active = run.n_active;
              }
              if (pause) st->paused_at = k;
              st->D = D;
            }
          }
        }
      }
      __syncthreads();
      if (run.exit == 2) {
        --k;            // x_{k-1} is the result
        break;
      }
      const double alpha = run.alpha;
      double* X = LDS_AT(double, x);
      const R* Ps = LDS_AT(R, p);
      for (int i = tid; i < 3 * B.nloc; i += BS) X[i] = fma(alpha, double(Ps[i]), X[i]);
      __syncthreads();
      if (run.exit) break;
    }

    // ---- pair terms of this block's vertices (block_pair_entries), and the
    // geometry of the curvature pass's pairs
    if constexpr (SELF) {
      PHASE;
      const PairPos<R> pos{((k & 1) != 0) != pending ? K->A.x1 : K->A.x0, (k & 1) ? K->A.p1 : K->A.p0, run.alpha,
                           pending ? 1 : 0};
      const Args<R> pa = pair_args(K);
      const int e0 = ent[2 * vi], e1 = ent[2 * vi + 1];
      if (e0 < e1) {
        const int base = ent[0], in_lds = ent[2 * vb - 1] - base <= K->P.cap_rp;
        const int m0 = (e0 >> 6) + (vt >> 6);
        for (int m = m0; m <= ((e1 - 1) >> 6); m += GW) {
          const int j = m * kWave + lane;
          const bool mine = j >= e0 && j < e1;
          double val[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
          int key = -1 - lane;
          if (mine) {
            int4 w = pw;
            int ci = pci;
            if (m != m0) {
              const int sl = K->A.cent[j];
              w = K->A.pv[sl >> 2];
              ci = sl & 3;
            }
            const int iv[4] = {w.x, w.y, w.z, w.w >= 0 ? w.w : ~w.w};
            Closest c;
            key = pick4(iv, ci);
            if (pair_at(pa, w.w >= 0, iv, pos, c)) {
              pair_grad_diag_corner(pa, c, ci, val);
              if (ci == 0) atomicAdd(&count[k & 1], 1);
            }
          }
          const bool last = seg_sum(key, val);
          if (mine && last) {
            double* o = in_lds ? LDS_AT(double, rp) + 6 * (j - base) : K->A.rp + 6 * (size_t)j;
#pragma unroll
            for (int i = 0; i < 6; ++i) o[i] = val[i];
          }
        }
      }
      if (early && vt >= GB - kWave && pci >= 0) {
        const int iv[4] = {pw.x, pw.y, pw.z, pw.w >= 0 ? pw.w : ~pw.w};
        Closest c;
        PairGeom* g = LDS_AT(PairGeom, dg) + vi * kWave + lane;
        const bool act = pair_at(pa, pw.w >= 0, iv, pos, c);
        g->v[0] = act ? iv[0] : -1;
        if (act) {
          pair_hess_coefs(pa, c.d, g->ca, g->cb);
#pragma unroll
          for (int i = 0; i < 4; ++i) { g->v[i] = iv[i]; g->c[i] = c.c[i]; }
          g->t[0] = c.t.x; g->t[1] = c.t.y; g->t[2] = c.t.z;
        }
      }
    }
    // ---- element gradient and diagonal, summed per vertex; then the vertex
    // terms (vertex_terms), one component to a thread: inertia, planes, pairs;
    // g, P g = g / diag and 1 / diag.
    for (int c = 0;; ++c) {
      {
        PHASE;
        const ushort4* tl = LDS_AT(ushort4, tl);
        const double* X = LDS_AT(double, x);
        if constexpr (kTets) {
          // each tet of the chunk once, its corners' terms to the lanes of
          // the chunk's vertices
          R* res = LDS_AT(R, res);
          const int e0 = chk[c].x + erank * kWave + lane, e1 = chk[c + 1].x;
          for (int e = e0; erank >= 0 && e < e1; e += efree * kWave) {
            const PersistEntry en = c == 0 && e == e0 ? entry0 : K->P.entry[e];
            const ushort4 v = tl[en.tet];
            const Elem<R> rec = element<R>(K, lds, en.tet);
            const Kin<R> kin = kinematics<R>(rec.B, at3(X, v.x), at3(X, v.y), at3(X, v.z), at3(X, v.w));
            bool ok = true;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
              const unsigned short to = en.slot[a];
              if (to == kNone) continue;
              V3<R> g, dg;
              if (!el_grad_diag<R, M>(kin, rec.vmu, rec.vlam, shape_vec(rec.B, a), g, dg)) {
                ok = false;
                g = mk3(R(0), R(0), R(0));
                dg = g;
              }
              R* o = res + 6 * to;
              o[0] = g.x; o[1] = g.y; o[2] = g.z; o[3] = dg.x; o[4] = dg.y; o[5] = dg.z;
            }
            if (!ok) raise_err(K->A.status, kErrInverted);
          }
        } else {
          // one (tet, corner) to a lane: the corotated terms' iteration count
          // is voted by the wave, so the waves keep the incidence's lanes
          const ushort2* lt = LDS_AT(ushort2, lane);
          R* tot = LDS_AT(R, tot);
          const int w0 = B.w0, we = lblk[vi][1];
          for (int w = lblk[vi][0] + (vt >> 6); w < we; w += GW) {
            const ushort2 ln = lt[(w - w0) * kWave + lane];
            const int l = ln.y & kLaneVert;
            R s[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
            if (ln.x != kNone) {
              const int t = ln.x >> 2;
              const ushort4 v = tl[t];
              const Elem<R> rec = element<R>(K, lds, t);
              const Kin<R> kin = kinematics<R>(rec.B, at3(X, v.x), at3(X, v.y), at3(X, v.z), at3(X, v.w));
              V3<R> g, dg;
              if (el_grad_diag<R, M>(kin, rec.vmu, rec.vlam, shape_vec(rec.B, ln.x & 3), g, dg)) {
                s[0] = g.x; s[1] = g.y; s[2] = g.z; s[3] = dg.x; s[4] = dg.y; s[5] = dg.z;
              } else {
                raise_err(K->A.status, kErrInverted);
              }
            }
            seg_sum(l, s);
            if (ln.y & kLaneLast) {
#pragma unroll
              for (int i = 0; i < 6; ++i) tot[6 * l + i] = s[i];
            }
          }
        }
      }
      __syncthreads();
      if constexpr (kTets) {
        // a vertex's lanes row by row, one value of one row to a thread
        PHASE;
        const ushort2* seg = LDS_AT(ushort2, seg);
        const R* res = LDS_AT(R, res);
        R* tot = LDS_AT(R, tot);
        const int t1 = 6 * chk[c + 1].z;
        for (int t = 6 * chk[c].z + tid; t < t1; t += BS) {
          const int q = t / 6;
          const ushort2 r = seg[q];
          tot[t] = row_run_sum<6>(res + (t - 6 * q), r.x, r.y);
        }
        __syncthreads();
      }
      PHASE;
      int i0 = 0, i1 = 3 * B.nown;
      if constexpr (kTets) {
        i0 = 3 * chk[c].y;
        i1 = 3 * chk[c + 1].y;
      }
      const double *X = LDS_AT(double, x), *XT = LDS_AT(double, xt), *Ms = LDS_AT(double, m);
      double* Pd = LDS_AT(double, P);
      R *pg = LDS_AT(R, pg), *G = LDS_AT(R, g) + ((k & 1) ? 3 * K->P.cap_own : 0);
      const uint8_t* fls = LDS_AT(uint8_t, fl);
      const double h2 = K->A.h2;
      u64* pgw = K->P.pgx + 3 * ((size_t)set_of(k) * K->A.nV + own0);
      for (int i = i0 + tid; i < i1; i += BS) {
        const int l = i / 3, j = i - 3 * l;
        const uint8_t fl = fls[l];
        const double m = Ms[l];
        R tg, td;
        if constexpr (kTets) {
          // the vertex's rows in turn
          const ushort2 r = LDS_AT(ushort2, run)[l];
          const R* tot = LDS_AT(R, tot) + 6 * r.x + j;
          tg = td = R(0);
          for (int q = 0; q < r.y; ++q) {
            tg += tot[6 * q];
            td += tot[6 * q + 3];
          }
        } else {
          const R* tot = LDS_AT(R, tot) + 6 * l;
          tg = tot[j];
          td = tot[3 + j];
        }
        double gd = vertex_g(h2, double(tg), m, X[i], XT[i]);
        double dd = vertex_diag(h2, double(td), m);
        if (fl & kSurface) {
          const V3<double> x = at3(X, l);
          for (int a = 0; a < K->A.planes.n; ++a) {
            const double* pl = planes + 4 * a;
            const double d = plane_dist(pl, x), dhat = K->A.dhat;
            if (d < dhat) {
              if (!(d > 0.0)) { raise_err(K->A.status, kErrPenetration); continue; }
              const double b1 = K->A.kappa * barrier_db(d, dhat), b2 = K->A.kappa * barrier_d2b(d, dhat);
              add_plane(b1, b2, pl[j], gd, dd);
              if (j == 0) atomicAdd(&count[k & 1], 1);
            }
          }
        }
        if constexpr (SELF) {
          const int* ce = LDS_AT(int, ce) + 2 * l;
          const int c0 = ce[0], c1 = ce[1];
          if (c0 < c1) {
            // the vertex's runs, one per 64-entry chunk (pair_partials_sum)
            const int base = ent[0], in_lds = ent[2 * vb - 1] - base <= K->P.cap_rp;
            double ga = 0.0, da = 0.0;
            for (int q = c0 >> 6; q * kWave < c1; ++q) {
              const int e = min(c1, (q + 1) * kWave) - 1;
              const double* rp = in_lds ? LDS_AT(double, rp) + 6 * (e - base) : K->A.rp + 6 * (size_t)e;
              ga += rp[j];
              da += rp[3 + j];
            }
            gd += ga;
            dd += da;
          }
          if ((fl & kSurface) && j == 0) {
            const double* XB = LDS_AT(double, xb);
            const V3<double> e = at3(X, l) - at3(XB, l);
            // the square (positive doubles order as their bits; the root is monotonic)
            const double e2 = dot(e, e);
            if (e2 > 0.0) atomicMax(&moved[k & 1], word(e2));
          }
          if (pending && (fl & kPairVertex)) st1_agent((k & 1) ? K->A.x1 : K->A.x0, own0 + l, j, X[i]);
        }
        if (fl & kFixed) {
          gd = 0.0;
          dd = 1.0;
        }
        const R gR = R(gd), pgR = R(gd / dd);
        G[i] = gR;
        pg[i] = pgR;
        Pd[i] = 1.0 / dd;
        st_agent(pgw + i, pg_word(pgR));
      }
      __syncthreads();
      if (!kTets || c + 1 >= K->P.chunks) break;
    }
    // ---- dot products for beta, each vertex at the lane its sum ended on
    {
      PHASE;
      const ulonglong2* wm = LDS_AT(ulonglong2, wm);
      const double* Pd = LDS_AT(double, P);
      const R *pg = LDS_AT(R, pg), *p = LDS_AT(R, p), *G = LDS_AT(R, g);
      const R *gn = G + ((k & 1) ? 3 * K->P.cap_own : 0), *go = G + ((k & 1) ? 0 : 3 * K->P.cap_own);
      double dots[6] = {0, 0, 0, 0, 0, 0};
      const int w0 = B.w0, we = lblk[vi][1];
      for (int w = lblk[vi][0] + (vt >> 6); w < we; w += GW) {
        const ulonglong2 m = wm[w - w0];   // last lanes of the wave's vertices, and the first of them
        if ((m.x >> lane) & 1) {
          const int i = 3 * ((int)m.y + __popcll(m.x & ((1ull << lane) - 1)));
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            add_beta_dots(double(gn[i + j]), double(pg[i + j]), double(go[i + j]), double(p[i + j]), Pd[i + j], dots);
          }
        }
      }
      // rows of 16 lanes: lane l of each row's first eight holds quantity l
      const double r = row_sums6(dots);
      if ((lane & 15) < 6) sh[wave * 24 + (lane >> 4) * 6 + (lane & 7)] = r;
    }
    __syncthreads();
    // ---- first meeting: the sums, and P g of the vertices shared with others
    {
      PHASE;
      const int s = set_of(k);
      u64* slots = K->P.slot_grad + s * 8 * n;
      if (tid < 8 * vb) {
        const int i = tid >> 3, q = tid & 7;
        double r;
        if (q < 6) {
          // the rows of a wave as wave_sum adds them, then the waves
          const double* h = sh + i * GW * 24 + q;
          r = (h[18] + h[12]) + (h[6] + h[0]);
          for (int w = 1; w < GW; ++w) r += (h[24 * w + 18] + h[24 * w + 12]) + (h[24 * w + 6] + h[24 * w]);
        } else {
          // counts and the maximum do not depend on the order: the block's go
          // with its first logical block
          r = i > 0 ? 0.0 : q == 6 ? double(count[k & 1]) : sqrt(as_double(moved[k & 1]));
        }
        st_agent(slots + q * n + slot_id[i], full(word(r)));
      }
      const u64* src = K->P.pgx + 3 * (size_t)s * K->A.nV;
      const int* hv = LDS_AT(int, hv);
      const int nh = 3 * (B.nloc - B.nown);
      R* pg = LDS_AT(R, pg) + 3 * B.nown;
      const u64* from[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int i = tid + u * BS;
        from[u] = i < nh ? src + 3 * (size_t)hv[i / 3] + i % 3 : nullptr;
      }
      const long long limit = K->P.limit;
      gather<8>(slots, n, 1u << 7, shg, nwaves, limit, &run.bad, [&]() {
        u64 w[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) w[u] = from[u] ? ld_agent(from[u]) : 0;
        bool all = true;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          if (!from[u]) continue;
          if (w[u] == kEmpty) {
            all = false;
          } else {
            from_word(w[u], pg[tid + u * BS]);
            from[u] = nullptr;
          }
        }
        return all;
      });
      // shares of more than two words per thread
      for (int i = tid + 2 * BS; i < nh; i += BS) {
        const u64* p = src + 3 * (size_t)hv[i / 3] + i % 3;
        u64 w = ld_agent(p);
        Wait t(limit);
        while (w == kEmpty) {
          if (run.bad || t.over()) { run.bad = 1; break; }
          w = ld_agent(p);
        }
        from_word(w, pg[i]);
      }
    }
    __syncthreads();
    // ---- direction part: beta, the restart and the gradient rules
    if (threadIdx.x < kWave) {
      PHASE;
      const bool leader = blockIdx.x == 0 && tid == 0;
      double r[8];
      totals<8>(shg, n, 1u << 7, r);
      if (lane == 0 && !run.bad) {
        const double gg = r[0], gPg = r[1];
        const double gnorm = sqrt(gg);
        const double g0 = k == 0 ? gnorm : run.g0;
        int dir_stop = 0, reason = 0, restart = 0;
        const int term = K->A.term;
        if ((term == 1 && gnorm <= K->A.eps * g0) || (term == 2 && gnorm <= K->A.eps)) { dir_stop = 1; reason = 1; }
        const double gPy = r[2], yp = r[3], yPy = r[4], pg = r[5];
        double beta = 0.0;
        if (k > 0) beta = beta_rule(K->A.flags, gPg, gPy, yp, yPy, pg, run.gPg, run.gTp);
        double gTp = direction_gTp(beta, pg, gPg);
        if (!(gTp < 0.0)) {
          restart = 1;
          beta = 0.0;
          gTp = -gPg;
        }
        if (!dir_stop && gTp == 0.0) { dir_stop = 1; reason = 3; }
        run.beta = beta; run.gTp = gTp; run.gPg = gPg; run.gnorm = gnorm; run.g0 = g0; run.n_active = r[6]; run.Dx = r[7];
        if (dir_stop) run.exit = 3;
        if (leader) {
          IterScal* o = K->A.scal + k;
          StepStatus* st = K->A.status;
          o->beta = beta; o->gTp = gTp; o->gnorm = gnorm; o->dir_stop = dir_stop; o->restart = restart; o->n_active = r[6];
          o->gPg = gPg;
          o->Dx = r[7];
          if (k == 0) st->g0 = gnorm;
          if (dir_stop) {
            st->stopped = 1; st->final_k = k; st->iters = k; st->reason = reason;
            st->gk = gnorm; st->dE0 = run.dE0; st->last_dE = run.dE; st->a_up_hits = run.a_up; st->n_active = r[6];
          }
        }
      }
    }
    __syncthreads();
    last_set = set_of(k + 1);
    if (run.bad || run.exit) break;
    if (threadIdx.x < 2) {
      // (published; the next iteration counts in the other one)
      if (threadIdx.x == 0) count[k & 1] = 0;
      else moved[k & 1] = 0;
    }
    // ---- p_{k+1} of every local vertex
    {
      PHASE;
      const R rb = R(run.beta);
      const R* pg = LDS_AT(R, pg);
      R* p = LDS_AT(R, p);
      const uint8_t* fl = LDS_AT(uint8_t, fl);
      for (int i = tid; i < 3 * B.nloc; i += BS) {
        const R q = fma(rb, p[i], -pg[i]);
        p[i] = q;
        if (SELF && i < 3 * B.nown && (fl[i / 3] & kPairVertex)) {
          const int l = i / 3;
          st1_agent((k & 1) ? K->A.p0 : K->A.p1, own0 + l, i - 3 * l, q);
        }
      }
    }
    if (k > k0) clear(k - 1);
    __syncthreads();
    // ---- p^T H p and the largest |p_v|
    double acc_pHp = 0.0, pmv = 0.0, pmc = 0.0;
    if (fresh(threadIdx.x) % GB < DB) {
      PHASE;
      constexpr bool kSplitPasses = DB > kSBlock;
      const double* X = LDS_AT(double, x);
      const R* p = LDS_AT(R, p);
      const bool tet_thread = !kSplitPasses || vt < kSBlock;
      double el = 0.0;
      if (tet_thread) {
        const unsigned short* dt = LDS_AT(unsigned short, dt);
        const ushort4* tl = LDS_AT(ushort4, tl);
        const int e1 = lblk[vi][3], t0 = B.t0;
        for (int e = lblk[vi][2] + vt; e < e1; e += kSBlock) {
          const int t = dt[e - t0];
          const ushort4 c = tl[t];
          const Elem<R> rec = element<R>(K, lds, t);
          const Kin<R> kin = kinematics<R>(rec.B, at3(X, c.x), at3(X, c.y), at3(X, c.z), at3(X, c.w));
          V3<R> d[3];
          dF_cols(rec.B, at3(p, c.x), at3(p, c.y), at3(p, c.z), at3(p, c.w), d);
          R ph = R(0);
          if (!el_pHp<R, M>(kin, rec.vmu, rec.vlam, d, ph)) raise_err(K->A.status, kErrInverted);
          el += double(ph);
        }
      }
      acc_pHp = K->A.h2 * el;
      if (!kSplitPasses || !tet_thread) {
        const unsigned short* dv = LDS_AT(unsigned short, dv);
        const double* Ms = LDS_AT(double, m);
        const uint8_t* fls = LDS_AT(uint8_t, fl);
        const int v1 = lblk[vi][5], v0 = B.v0;
        for (int v = lblk[vi][4] + (kSplitPasses ? vt - kSBlock : vt); v < v1; v += kSplitPasses ? DB - kSBlock : DB) {
          const int l = dv[v - v0];
          const V3<R> q = at3(p, l);
          const V3<double> pd = cast3<double>(q);
          const double p2 = dot(pd, pd);
          double vp = Ms[l] * p2;
          if (fls[l] & kSurface) {
            const V3<double> x = at3(X, l);
            for (int a = 0; a < K->A.planes.n; ++a) {
              const double* pl = planes + 4 * a;
              const double d = plane_dist(pl, x), dhat = K->A.dhat;
              if (d > 0.0 && d < dhat)
                vp = fma(plane_Hp(K->A.kappa, pl, d, dhat, pd), dot(mk3(pl[0], pl[1], pl[2]), pd), vp);
            }
          }
          const double pabs = sqrt(p2), pcomp = fmax(fabs(pd.x), fmax(fabs(pd.y), fabs(pd.z)));
          acc_pHp = sum_rounded(acc_pHp, vp);
          pmv = fmax(pmv, pabs);
          pmc = fmax(pmc, pcomp);
        }
      }
      if constexpr (SELF) {
        // the pairs of an even slice of the entry index (for_each_pair)
        const u64* src = K->P.pgx + 3 * (size_t)set_of(k) * K->A.nV;
        const R4<R>* pk = (k & 1) ? K->A.p1 : K->A.p0;
        const R rb = R(run.beta);
        const long long limit = K->P.limit;
        if (early) {
          if (vt < early) {
            const PairGeom* g = LDS_AT(PairGeom, dg) + vi * kWave + vt;
            const int iv[4] = {g->v[0], g->v[1], g->v[2], g->v[3]};
            if (iv[0] >= 0) {
              const double c[4] = {g->c[0], g->c[1], g->c[2], g->c[3]};
              V3<double> sp;
              if (!pair_dir<R>(iv, c, src, pk, rb, limit, sp)) run.bad = 1;
              acc_pHp += pair_pHp(g->ca, g->cb, sp, mk3(g->t[0], g->t[1], g->t[2]));
            }
          }
        } else {
          const Args<R> pa = pair_args(K);
          const PairPos<R> pos{((k & 1) != 0) != pending ? K->A.x1 : K->A.x0, pk, run.alpha, pending ? 1 : 0};
          const long long nq = min(K->A.ncand[0], K->A.cand_cap);
          const long long pe = (4 * nq + n - 1) / n;
          const long long eb = (long long)(lp * vb + vi) * pe, ee = min(eb + pe, 4 * nq);
          const int* cent = K->A.cent;
          for (long long j = eb + vt; j < ee; j += DB) {
            const int sl = cent[j];
            if ((sl & 3) != 0) continue;
            const int4 w = K->A.pv[sl >> 2];
            const int iv[4] = {w.x, w.y, w.z, w.w >= 0 ? w.w : ~w.w};
            Closest c;
            if (!pair_at(pa, w.w >= 0, iv, pos, c)) continue;
            double ca, cb;
            pair_hess_coefs(pa, c.d, ca, cb);
            V3<double> sp;
            if (!pair_dir<R>(iv, c.c, src, pk, rb, limit, sp)) run.bad = 1;
            acc_pHp += pair_pHp(ca, cb, sp, c.t);
          }
        }
      }
    }
    {
      const int lane = fresh(threadIdx.x) & (kWave - 1), wave = threadIdx.x >> 6;
      const double v[3] = {acc_pHp, pmv, pmc};
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const double r = i ? wave_max(v[i]) : wave_sum(v[i]);
        if (lane == 0) sh[wave * 3 + i] = r;
      }
    }
    // everything this block has stored (cleared words, x_k and p_{k+1} of the
    // pair vertices) has arrived before its second set of sums is published
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    {
      PHASE;
      u64* slots = K->P.slot_dir + set_of(k) * 3 * n;
      if (tid < 3 * vb) {
        const int i = tid / 3, q = tid - 3 * i;
        publish<3>(sh + i * GW * 3, q, DW, q > 0, slots + q * n + slot_id[i]);
      }
      // ---- second meeting
      gather<3>(slots, n, 6u, shg, nwaves, K->P.limit, &run.bad, []() { return true; });
    }
    __syncthreads();
    if (run.bad) break;
    pending = true;
  }
  PHASE;
  const bool leader = blockIdx.x == 0 && tid == 0;
  if (run.bad) {
    if (tid == 0) raise_err(K->A.status, kErrSync);
    return;
  }
  // ---- leave x_k, p_k and g_k (at the start of iteration k: g_{k-1}) as the
  // per-iteration launches do
  {
    double4* xo = (k & 1) ? K->A.x1 : K->A.x0;
    R4<R>* po = (k & 1) ? K->A.p1 : K->A.p0;
    const double* X = LDS_AT(double, x);
    const R *p = LDS_AT(R, p), *g = LDS_AT(R, g) + ((k & 1) ? 0 : 3 * K->P.cap_own);
    for (int l = tid; l < B.nown; l += BS) {
      st3(xo, own0 + l, at3(X, l));
      str<R>(po, own0 + l, at3(p, l));
      str<R>(K->A.g, own0 + l, at3(g, l));
    }
    // every block has read the ring: it was past a meeting before any could end
    if (leader) *K->P.ring = last_set;
  }
#undef LDS_AT
#undef PHASE
}

__global__ void __launch_bounds__(256) k_persist_clear(u64* a, long long na, u64* b, long long nb, u64* c, long long nc, int* ring) {
  const long long tid = (long long)blockIdx.x * 256 + threadIdx.x, stride = (long long)gridDim.x * 256;
  for (long long i = tid; i < na; i += stride) a[i] = kEmpty;
  for (long long i = tid; i < nb; i += stride) b[i] = kEmpty;
  for (long long i = tid; i < nc; i += stride) c[i] = kEmpty;
  if (tid == 0) *ring = 0;
}

void persist_clear(const PersistArgs& P, int nV, hipStream_t s) {
  hipLaunchKernelGGL(k_persist_clear, dim3(256), dim3(256), 0, s, P.slot_grad, 24LL * P.grid, P.slot_dir, 9LL * P.grid,
                     P.pgx, 9LL * nV, P.ring);
}

template <typename R>
void launch_persist(const Args<R>& A, const PersistArgs& P, int k0, int mode, hipStream_t s) {
  PNCG_BY_SCATTER(A.self, PNCG_BY_MODEL(A.model, hipLaunchKernelGGL((k_persist<R, M_, S_>), dim3(P.blocks),
                                                                    dim3(P.vb * GradBlock<R, M_>::value), P.lds, s,
                                                                    (KArgs<R>{A, P, k0, mode}))));
}

template <typename R>
hipError_t persist_fits(const PersistArgs& P, int model, bool self, int compute_units, bool* ok) {
  hipError_t e = hipSuccess;
  int per_cu = 0;
  PNCG_BY_SCATTER(self, PNCG_BY_MODEL(model, (e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                                                  &per_cu, k_persist<R, M_, S_>, P.vb * GradBlock<R, M_>::value, P.lds))));
  *ok = e == hipSuccess && per_cu >= 1 && P.blocks <= compute_units;
  return e;
}

template void launch_persist<float>(const Args<float>&, const PersistArgs&, int, int, hipStream_t);
template void launch_persist<double>(const Args<double>&, const PersistArgs&, int, int, hipStream_t);
template hipError_t persist_fits<float>(const PersistArgs&, int, bool, int, bool*);
template hipError_t persist_fits<double>(const PersistArgs&, int, bool, int, bool*);

}  // namespace pncg
