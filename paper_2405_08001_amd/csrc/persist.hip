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
// compute unit, and the host counts the compute units that such launches of
// the process hold.  A wait is bounded by the clock all the same; a launch
// that runs out raises kErrSync, writes nothing, and the host runs the step
// again with the per-iteration launches, which give the same bits.
#include <cfloat>
#include <climits>

#include "iteration_common.h"
#include "persist.h"

namespace pncg {

namespace {

typedef unsigned long long u64;
// a NaN that no arithmetic of the kernel produces; a value with these bits
// is published with its last bit flipped
constexpr u64 kEmpty = 0xfff8dead5eef0001ull;

__device__ __forceinline__ u64 ld_agent(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(u64* p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 full(u64 v) { return v == kEmpty ? v ^ 1 : v; }
__device__ __forceinline__ u64 word(double a) { return (u64)__double_as_longlong(a); }
__device__ __forceinline__ u64 word(float a, float b) {
  return (u64)(unsigned)__float_as_int(a) | ((u64)(unsigned)__float_as_int(b) << 32);
}
__device__ __forceinline__ double as_double(u64 w) { return __longlong_as_double((long long)w); }
__device__ __forceinline__ float lo_float(u64 w) { return __int_as_float((int)(unsigned)w); }
__device__ __forceinline__ float hi_float(u64 w) { return __int_as_float((int)(unsigned)(w >> 32)); }

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

// Watches the clock in a polling loop.
struct Wait {
  long long t0, limit;
  int n;
  __device__ __forceinline__ Wait(long long l) : t0(0), limit(l), n(0) {}
  // true when the wait has run out
  __device__ __forceinline__ bool over() {
    if ((++n & 63) != 0) return false;
    const long long t = wall_clock64();
    if (t0 == 0) t0 = t;
    return t - t0 > limit;
  }
};

// The kernel's arguments are read from the kernel argument segment where they
// are needed: kept in registers across the whole loop they would spill.  The
// empty asm statement hides from the compiler that the segment is the same
// each time.
template <typename R>
struct KArgs {
  Args<R> A;
  PersistArgs P;
  int k0, mode;
};
template <typename R>
using KPtr = const __attribute__((address_space(4))) KArgs<R>*;
template <typename R>
__device__ __forceinline__ KPtr<R> kargs() {
  unsigned long long p = (unsigned long long)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return (KPtr<R>)p;
}

// The same for a value in a vector or scalar register: what a phase derives
// from it is derived again in the next iteration instead of being kept.
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ int fresh_s(int x) {
  x = __builtin_amdgcn_readfirstlane(x);
  asm volatile("" : "+s"(x));
  return x;
}

template <typename T>
__device__ __forceinline__ V3<T> at3(const T* a, int l) { return mk3(a[3 * l], a[3 * l + 1], a[3 * l + 2]); }

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

// Publish quantity q of a logical block: sh holds the wave results [wave][N]
// of its nw waves, added (or compared) in wave order as block_reduce does.
template <int N>
__device__ __forceinline__ void publish(const double* sh, int q, int nw, bool mx, u64* slot) {
  double r = sh[q];
  for (int j = 1; j < nw; ++j) r = mx ? fmax(r, sh[j * N + q]) : r + sh[j * N + q];
  st_agent(slot, full(word(r)));
}

// Wait for the n partials of N quantities (slot [q][n]) and leave the wave
// sums [q][4] in sh: wave w of the four takes partials 64 w + lane and
// 256 + 64 w + lane, the order of reduce_partials.  The loads of a try, and
// those of other() (more words to wait for; true when they have arrived), are
// all in flight together.
template <int N, typename Other>
__device__ __forceinline__ void gather(const u64* slot, int n, unsigned maxmask, double* sh, int nwaves, long long limit,
                                       int* bad, Other&& other) {
  constexpr int T = (N * 4 + 6) / 7;   // tasks of a wave: at least seven waves share N * 4
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
  const int nw = min(4, (n + kWave - 1) / kWave), tasks = N * nw;
  u64 a[T], b[T];
  Wait w(limit);
  bool odone = false;
  for (;;) {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < T; ++i) {
      const int t = wave + i * nwaves;
      a[i] = b[i] = 0;
      if (t >= tasks) continue;
      const int q = t / nw, j = (t - q * nw) * kWave + lane;
      if (j < n) a[i] = ld_agent(slot + q * n + j);
      if (j + kSBlock < n) b[i] = ld_agent(slot + q * n + j + kSBlock);
    }
    if (!odone) odone = other();
#pragma unroll
    for (int i = 0; i < T; ++i) ok = ok && a[i] != kEmpty && b[i] != kEmpty;
    if (ok && odone) break;
    if (w.over()) {
      *bad = 1;
      break;
    }
  }
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int t = wave + i * nwaves;
    if (t >= tasks) continue;   // uniform over the wave
    const int q = t / nw, j = (t - q * nw) * kWave + lane;
    const bool mx = (maxmask >> q) & 1u;
    double v = 0.0;
    if (j < n) v = mx ? fmax(v, as_double(a[i])) : v + as_double(a[i]);
    if (j + kSBlock < n) v = mx ? fmax(v, as_double(b[i])) : v + as_double(b[i]);
    v = mx ? wave_max(v) : wave_sum(v);
    if (lane == 0) sh[q * 4 + (t - q * nw)] = v;
  }
}
// Totals of N quantities from the wave sums gather() left, by the first wave:
// lane q adds up quantity q, then every lane receives all.
template <int N>
__device__ __forceinline__ void totals(const double* sh, int n, unsigned maxmask, double (&r)[N]) {
  const int nw = min(4, (n + kWave - 1) / kWave), lane = threadIdx.x & (kWave - 1);
  double v = 0.0;
  if (lane < N) {
    const bool mx = (maxmask >> lane) & 1u;
    v = sh[lane * 4];
    for (int w = 1; w < nw; ++w) v = mx ? fmax(v, sh[lane * 4 + w]) : v + sh[lane * 4 + w];
  }
  const long long b = __double_as_longlong(v);
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const int lo = __builtin_amdgcn_readlane((int)b, q), hi = __builtin_amdgcn_readlane((int)(b >> 32), q);
    r[q] = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  }
}

}  // namespace

// SELF: point-triangle / edge-edge pairs by the segmented scatter, each block
// evaluating its own vertices' entries (the sparse-contact form, see
// fused_pairs).
template <typename R, int M, bool SELF, int MAXT = 2 * GradBlock<R, M>::value>
__global__ void __launch_bounds__(MAXT) k_persist(KArgs<R>) {
  constexpr int GB = GradBlock<R, M>::value, DB = DirBlock<R, M>::value;
  constexpr int GW = GB / kWave, DW = DB / kWave;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ double sh[2 * 8 * 8];
  __shared__ double shg[8 * 4];
  __shared__ Run run;
  __shared__ PersistBlock B;
  __shared__ int lblk[2][6];     // per logical block: incidence waves [b, e), tets [b, e), vertices [b, e)
  // thread, wave, and the wave's logical block within the block (vi) with the
  // thread's place in it (vt); taken anew by every phase
#define PHASE                                                                                          \
  const KPtr<R> K = kargs<R>();                                                                        \
  const int tid = fresh(threadIdx.x), BS = K->P.vb * GB, n = K->P.grid, vb = K->P.vb;                  \
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = vb * GW; \
  const int vi = wave >= GW ? 1 : 0, vt = tid - vi * GB;                                               \
  (void)lane, (void)vt, (void)nwaves, (void)n, (void)BS
#define LDS_AT(T, field) reinterpret_cast<T*>(lds + K->P.at.field)

  int k0, lp, set0, own0;
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
    for (int i = tid; i < b.nw * kWave; i += BS) LDS_AT(ushort2, lane)[i] = K->P.lane[(size_t)b.w0 * kWave + i];
    for (int i = tid; i < b.nt; i += BS) LDS_AT(unsigned short, dt)[i] = K->P.dtet[b.t0 + i];
    for (int i = tid; i < b.nv; i += BS) LDS_AT(unsigned short, dv)[i] = K->P.dvert[b.v0 + i];
  }
  // partial index of logical block i of this block: the blockIdx of the launch that has it
  auto slot_of = [&](int n, int vb, int i) {
    const int per = n / kXcds, L = fresh_s(lp) * vb + i;
    return (L % per) * kXcds + L / per;
  };
  auto set_of = [&](int it) { return fresh_s(set0 + it - k0) % 3; };
  // clear this block's words of iteration it's set
  auto clear = [&](int it) {
    PHASE;
    const int s = set_of(it);
    if (tid < 8 * vb) st_agent(K->P.slot_grad + s * 8 * n + (tid & 7) * n + slot_of(n, vb, tid >> 3), kEmpty);
    if (tid < 3 * vb) st_agent(K->P.slot_dir + s * 3 * n + (tid % 3) * n + slot_of(n, vb, tid / 3), kEmpty);
    u64* w = K->P.pgx + 3 * ((size_t)s * K->A.nV + own0);
    for (int i = tid; i < 3 * B.nown; i += BS) st_agent(w + i, kEmpty);
  };
  __syncthreads();
  clear(k0 + 1);
  clear(k0 + 2);

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
          const double dE = fma(-(0.5 * alpha * alpha), pHp, -(alpha * gTp));
          const double dmove = alpha * pmv;
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
            const double D = (SELF ? run.Dx : run.D) + dmove;
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

    // ---- pair terms of this block's vertices (block_pair_entries)
    double npair = 0.0;
    if constexpr (SELF) {
      PHASE;
      const PairPos<R> pos{((k & 1) != 0) != pending ? K->A.x1 : K->A.x0, (k & 1) ? K->A.p1 : K->A.p0, run.alpha,
                           pending ? 1 : 0};
      const int wb = lblk[vi][0], we = lblk[vi][1];
      if (wb < we) {
        const int2* wrange = K->A.wrange;
        const int e0 = wrange[wb].x, e1 = wrange[we - 1].y;
        if (e0 < e1) {
          const Args<R> pa = pair_args(K);
          const int* cent = K->A.cent;
          for (int m = (e0 >> 6) + (vt >> 6); m <= ((e1 - 1) >> 6); m += GW) {
            const int j = m * kWave + lane;
            const bool mine = j >= e0 && j < e1;
            double val[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            int key = -1 - lane;
            if (mine) {
              const int sl = cent[j];
              const int q = sl >> 2, ci = sl & 3;
              int iv[4];
              Closest c;
              const bool act = pair_closest(pa, q, pos, iv, c, -1);
              key = pick4(iv, ci);
              if (act) {
                pair_grad_diag_corner(pa, c, ci, val);
                if (ci == 0) npair += 1.0;
              }
            }
            const bool last = seg_sum(key, val);
            if (mine && last) {
              double* o = K->A.rp + 6 * (size_t)j;
#pragma unroll
              for (int i = 0; i < 6; ++i) o[i] = val[i];
            }
          }
        }
      }
    }
    // ---- element gradient and diagonal, summed per vertex
    {
      PHASE;
      const ushort2* lt = LDS_AT(ushort2, lane);
      const ushort4* tl = LDS_AT(ushort4, tl);
      const double* X = LDS_AT(double, x);
      R* tot = LDS_AT(R, tot);
      const int w0 = B.w0, we = lblk[vi][1];
      for (int w = lblk[vi][0] + (vt >> 6); w < we; w += GW) {
        const ushort2 ln = lt[(w - w0) * kWave + lane];
        const int l = ln.y & kLaneVert;
        R s[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
        if (ln.x != kNone) {
          const int t = ln.x >> 2;
          const ushort4 c = tl[t];
          const Elem<R> rec = element<R>(K, lds, t);
          const Kin<R> kin = kinematics<R>(rec.B, at3(X, c.x), at3(X, c.y), at3(X, c.z), at3(X, c.w));
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
    __syncthreads();
    // ---- vertex terms (vertex_terms), one component to a thread: inertia,
    // planes, pairs; g, P g = g / diag and 1 / diag.  The fused forms written
    // out are those the compiler chooses in the per-iteration launches.
    double nplane = 0.0, dx = 0.0;
    {
      PHASE;
      const double *X = LDS_AT(double, x), *XT = LDS_AT(double, xt), *Ms = LDS_AT(double, m);
      double* Pd = LDS_AT(double, P);
      const R* tot = LDS_AT(R, tot);
      R *pg = LDS_AT(R, pg), *G = LDS_AT(R, g) + ((k & 1) ? 3 * K->P.cap_own : 0);
      const uint8_t* fls = LDS_AT(uint8_t, fl);
      const double h2 = K->A.h2;
      u64* pgw = K->P.pgx + 3 * ((size_t)set_of(k) * K->A.nV + own0);
      for (int i = tid; i < 3 * B.nown; i += BS) {
        const int l = i / 3, j = i - 3 * l;
        const uint8_t fl = fls[l];
        const double m = Ms[l];
        double gd = fma(h2, double(tot[6 * l + j]), m * (X[i] - XT[i]));
        double dd = fma(h2, double(tot[6 * l + 3 + j]), m);
        if (fl & kSurface) {
          const V3<double> x = at3(X, l);
          for (int a = 0; a < K->A.planes.n; ++a) {
            const double pl[4] = {K->A.planes.p[a][0], K->A.planes.p[a][1], K->A.planes.p[a][2], K->A.planes.p[a][3]};
            const double d = plane_dist(pl, x), dhat = K->A.dhat;
            if (d < dhat) {
              if (!(d > 0.0)) { raise_err(K->A.status, kErrPenetration); continue; }
              const double b1 = K->A.kappa * barrier_db(d, dhat), b2 = K->A.kappa * barrier_d2b(d, dhat);
              const double nj = j == 0 ? pl[0] : j == 1 ? pl[1] : pl[2];
              gd = fma(b1, nj, gd);
              dd = fma(b2 * nj, nj, dd);
              if (j == 0) nplane += 1.0;
            }
          }
        }
        if constexpr (SELF) {
          const int* ce = LDS_AT(int, ce) + 2 * l;
          const int c0 = ce[0], c1 = ce[1];
          if (c0 < c1) {
            // the vertex's runs, one per 64-entry chunk (pair_partials_sum)
            double ga = 0.0, da = 0.0;
            for (int q = c0 >> 6; q * kWave < c1; ++q) {
              const double* rp = K->A.rp + 6 * (size_t)(min(c1, (q + 1) * kWave) - 1);
              ga += rp[j];
              da += rp[3 + j];
            }
            gd += ga;
            dd += da;
          }
          if ((fl & kSurface) && j == 0) {
            const double* XB = LDS_AT(double, xb);
            const double ex = X[i] - XB[i], ey = X[i + 1] - XB[i + 1], ez = X[i + 2] - XB[i + 2];
            dx = fmax(dx, sqrt(fma(ez, ez, fma(ex, ex, ey * ey))));
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
    }
    __syncthreads();
    // ---- dot products for beta, each vertex at the lane its sum ended on
    {
      PHASE;
      const ushort2* lt = LDS_AT(ushort2, lane);
      const double* Pd = LDS_AT(double, P);
      const R *pg = LDS_AT(R, pg), *p = LDS_AT(R, p), *G = LDS_AT(R, g);
      const R *gn = G + ((k & 1) ? 3 * K->P.cap_own : 0), *go = G + ((k & 1) ? 0 : 3 * K->P.cap_own);
      double dots[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      const int w0 = B.w0, we = lblk[vi][1];
      for (int w = lblk[vi][0] + (vt >> 6); w < we; w += GW) {
        const unsigned short c = lt[(w - w0) * kWave + lane].y;
        if (c & kLaneLast) {
          const int i = 3 * (c & kLaneVert);
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            const double g = double(gn[i + j]), pgj = double(pg[i + j]), pp = double(p[i + j]), P = Pd[i + j];
            const double y = g - double(go[i + j]);
            dots[0] = fma(g, g, dots[0]);
            dots[1] = fma(g, pgj, dots[1]);
            dots[2] = fma(g * P, y, dots[2]);
            dots[3] = fma(y, pp, dots[3]);
            dots[4] = fma(y * P, y, dots[4]);
            dots[5] = fma(pp, g, dots[5]);
          }
        }
      }
      dots[6] = nplane + npair;   // counts: exact in any order
      dots[7] = dx;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const double r = i == 7 ? wave_max(dots[i]) : wave_sum(dots[i]);
        if (lane == 0) sh[wave * 8 + i] = r;
      }
    }
    __syncthreads();
    // ---- first meeting: the sums, and P g of the vertices shared with others
    {
      PHASE;
      const int s = set_of(k);
      u64* slots = K->P.slot_grad + s * 8 * n;
      if (tid < 8 * vb) {
        const int i = tid >> 3, q = tid & 7;
        publish<8>(sh + i * GW * 8, q, GW, q == 7, slots + q * n + slot_of(n, vb, i));
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
        double gTp = fma(beta, pg, -gPg);
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
          const double px = q.x, py = q.y, pz = q.z;
          const double p2 = fma(pz, pz, fma(px, px, py * py));
          double vp = Ms[l] * p2;
          if (fls[l] & kSurface) {
            const V3<double> x = at3(X, l);
            for (int a = 0; a < K->A.planes.n; ++a) {
              const double pl[4] = {K->A.planes.p[a][0], K->A.planes.p[a][1], K->A.planes.p[a][2], K->A.planes.p[a][3]};
              const double d = plane_dist(pl, x), dhat = K->A.dhat;
              if (d > 0.0 && d < dhat) {
                const double np = fma(pl[2], pz, fma(pl[0], px, pl[1] * py));
                vp = fma(K->A.kappa * barrier_d2b(d, dhat) * np, np, vp);
              }
            }
          }
          const double pabs = sqrt(p2), pcomp = fmax(fabs(px), fmax(fabs(py), fabs(pz)));
          acc_pHp += vp;
          pmv = fmax(pmv, pabs);
          pmc = fmax(pmc, pcomp);
        }
      }
      if constexpr (SELF) {
        // the pairs of an even slice of the entry index (for_each_pair)
        const Args<R> pa = pair_args(K);
        const PairPos<R> pos{((k & 1) != 0) != pending ? K->A.x1 : K->A.x0, (k & 1) ? K->A.p1 : K->A.p0, run.alpha,
                             pending ? 1 : 0};
        const u64* src = K->P.pgx + 3 * (size_t)set_of(k) * K->A.nV;
        const R rb = R(run.beta);
        const long long nq = min(K->A.ncand[0], K->A.cand_cap);
        const long long pe = (4 * nq + n - 1) / n;
        const long long eb = (long long)(lp * vb + vi) * pe, ee = min(eb + pe, 4 * nq);
        const int* cent = K->A.cent;
        for (long long j = eb + vt; j < ee; j += DB) {
          const int sl = cent[j];
          if ((sl & 3) != 0) continue;
          int iv[4];
          Closest c;
          if (!pair_closest(pa, sl >> 2, pos, iv, c, -1)) continue;
          double ca, cb;
          pair_hess_coefs(pa, c.d, ca, cb);
          V3<double> sp = mk3(0.0, 0.0, 0.0);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            // every block has passed the first meeting, so P g of any vertex
            // has been sent; it may still be on its way
            u64 w[3];
            Wait t(K->P.limit);
            for (;;) {
              bool here = true;
#pragma unroll
              for (int q = 0; q < 3; ++q) { w[q] = ld_agent(src + 3 * (size_t)iv[i] + q); here = here && w[q] != kEmpty; }
              if (here) break;
              if (t.over()) { run.bad = 1; break; }
            }
            V3<R> pgv;
            from_word(w[0], pgv.x); from_word(w[1], pgv.y); from_word(w[2], pgv.z);
            const V3<R> q = direction(pgv, ld3_agent(pos.p, iv[i]), rb);
            sp = sp + c.c[i] * cast3<double>(q);
          }
          const double st = dot(sp, c.t);
          acc_pHp += ca * st * st + cb * dot(sp, sp);
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
        publish<3>(sh + i * GW * 3, q, DW, q > 0, slots + q * n + slot_of(n, vb, i));
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

bool persist_build(int nV, int nT, const int* tets, const std::vector<int>& inc, const std::vector<int>& inc_vert,
                   int grid, bool fp64, bool self, PersistTables& T, PersistArgs& P) {
  const int nWaves = (int)(inc.size() / kWave);
  P = PersistArgs{};
  P.grid = grid;
  P.vb = grid > 256 ? 2 : 1;
  P.blocks = grid / P.vb;
  T = PersistTables{};
  T.blk.resize(P.blocks);
  T.lane.assign(inc.size(), make_ushort2(kNone, kLaneVert));
  T.dtet.resize(nT);
  T.dvert.resize(nV);
  std::vector<int> vloc(nV, -1), vmark(nV, -1), tloc(nT, -1), tmark(nT, -1);
  auto slice = [&](long long n, int L, int& b, int& e) {
    const long long per = (n + grid - 1) / grid;
    b = (int)std::min<long long>(L * per, n);
    e = (int)std::min<long long>((L + 1) * per, n);
  };
  for (int p = 0; p < P.blocks; ++p) {
    PersistBlock& B = T.blk[p];
    int b0, e0, b1, e1;
    slice(nWaves, p * P.vb, b0, e0);
    slice(nWaves, p * P.vb + P.vb - 1, b1, e1);
    B.w0 = b0; B.nw = e1 - b0;
    slice(nT, p * P.vb, b0, e0);
    slice(nT, p * P.vb + P.vb - 1, b1, e1);
    B.t0 = b0; B.nt = e1 - b0;
    slice(nV, p * P.vb, b0, e0);
    slice(nV, p * P.vb + P.vb - 1, b1, e1);
    B.v0 = b0; B.nv = e1 - b0;
    B.loc_off = (int)T.loc_v.size();
    B.tet_off = (int)T.tet_e.size();
    int nl = 0, nt = 0;
    auto vertex = [&](int v) {
      if (vmark[v] != p) {
        vmark[v] = p;
        vloc[v] = nl++;
        T.loc_v.push_back(v);
      }
      return vloc[v];
    };
    // own vertices: those of the block's incidence waves, consecutive
    for (long long i = (long long)B.w0 * kWave; i < (long long)(B.w0 + B.nw) * kWave; ++i)
      if (inc_vert[i] >= 0) vertex(inc_vert[i]);
    B.nown = nl;
    auto tet = [&](int e) {
      if (tmark[e] != p) {
        tmark[e] = p;
        tloc[e] = nt++;
        T.tet_e.push_back(e);
        ushort4 c;
        c.x = (unsigned short)vertex(tets[4 * e]);
        c.y = (unsigned short)vertex(tets[4 * e + 1]);
        c.z = (unsigned short)vertex(tets[4 * e + 2]);
        c.w = (unsigned short)vertex(tets[4 * e + 3]);
        T.tet_l.push_back(c);
      }
      return tloc[e];
    };
    for (long long i = (long long)B.w0 * kWave; i < (long long)(B.w0 + B.nw) * kWave; ++i) {
      ushort2& l = T.lane[i];
      if (inc_vert[i] >= 0) {
        // a vertex's lanes are consecutive and within one wave
        const bool last = (i + 1) % kWave == 0 || inc_vert[i + 1] != inc_vert[i];
        l.y = (unsigned short)(vloc[inc_vert[i]] | (last ? kLaneLast : 0));
      }
      if (inc[i] >= 0) {
        const int t = tet(inc[i] >> 2);
        l.x = (unsigned short)(t << 2 | (inc[i] & 3));
      }
    }
    for (int e = B.t0; e < B.t0 + B.nt; ++e) T.dtet[e] = (unsigned short)tet(e);
    for (int v = B.v0; v < B.v0 + B.nv; ++v) T.dvert[v] = (unsigned short)vertex(v);
    B.nloc = nl;
    B.ntet = nt;
    // 16-bit local ids; a lane's words also hold the corner (two bits) and the last-lane mark
    if (nl >= kLaneVert || nt >= (kNone >> 2)) return false;
    P.cap_loc = std::max(P.cap_loc, nl);
    P.cap_own = std::max(P.cap_own, B.nown);
    P.cap_tet = std::max(P.cap_tet, nt);
    P.cap_lane = std::max(P.cap_lane, B.nw * kWave);
    P.cap_dt = std::max(P.cap_dt, B.nt);
    P.cap_dv = std::max(P.cap_dv, B.nv);
    if (24 * (size_t)nl > kPersistLds) return false;
  }
  T.loc_v.push_back(0);   // a block without vertices reads its first one
  // the layout of a block's LDS; element records in it if they fit
  const unsigned real = fp64 ? 8 : 4;
  for (int in_lds = 1; in_lds >= 0; --in_lds) {
    size_t o = 0;
    auto put = [&](unsigned& f, size_t bytes, size_t align) {
      o = (o + align - 1) / align * align;
      f = (unsigned)o;
      o += bytes;
    };
    PersistLayout& L = P.at;
    put(L.rec, in_lds ? kRec * real * (size_t)P.cap_tet : 0, 16);
    put(L.x, 24 * (size_t)P.cap_loc, 8);
    put(L.m, 8 * (size_t)P.cap_loc, 8);
    put(L.xt, 24 * (size_t)P.cap_own, 8);
    put(L.xb, self ? 24 * (size_t)P.cap_own : 0, 8);
    put(L.P, 24 * (size_t)P.cap_own, 8);
    put(L.tot, 6 * real * (size_t)P.cap_own, 8);
    put(L.p, 3 * real * (size_t)P.cap_loc, 8);
    put(L.pg, 3 * real * (size_t)P.cap_loc, 8);
    put(L.g, 6 * real * (size_t)P.cap_own, 8);
    put(L.tl, 8 * (size_t)P.cap_tet, 8);
    put(L.te, in_lds ? 0 : 4 * (size_t)P.cap_tet, 4);
    put(L.hv, 4 * (size_t)P.cap_loc, 4);
    put(L.ce, self ? 8 * (size_t)P.cap_own : 0, 4);
    put(L.lane, 4 * (size_t)P.cap_lane, 4);
    put(L.dt, 2 * (size_t)P.cap_dt, 2);
    put(L.dv, 2 * (size_t)P.cap_dv, 2);
    put(L.fl, P.cap_loc, 1);
    P.elem_lds = in_lds;
    P.lds = o;
    if (o <= kPersistLds) return true;
  }
  return false;
}

template void launch_persist<float>(const Args<float>&, const PersistArgs&, int, int, hipStream_t);
template void launch_persist<double>(const Args<double>&, const PersistArgs&, int, int, hipStream_t);
template hipError_t persist_fits<float>(const PersistArgs&, int, bool, int, bool*);
template hipError_t persist_fits<double>(const PersistArgs&, int, bool, int, bool*);

}  // namespace pncg
