// The CG iterations of the adjoint in one launch (k_cg_fused's arithmetic,
// without pair terms).
//
// What bounded it: k_cg_fused waits for dependent memory round trips (the
// partials, the incidence codes, the records, {z, w} and p of the corners) and
// evaluates each tet in the lanes of its four corners.  Here a block keeps z, p
// and w = diag^-1 H p of its vertices and its neighbours' in LDS, and a thread
// keeps the deformation gradient, its cofactors and the coefficients of its tet
// in registers for the whole solve (x does not move), so an iteration reads
// memory only for the w of vertices shared with other blocks and the six
// partial sums.  Blocks, sums and their order are those of persist.hip; the
// blocks meet once per iteration, which bounds it now (4 us of the 6.2 to 6.4).
// An iteration at 30,000 tets takes 6.4 us, 12.1 as launches; with the rest of
// the solve, 1,008 iterations take 6.5 and 12.2 ms.
//
// Meeting.  As in persist.hip, every word is its own flag and iteration i uses
// set i mod 3 of the exchange buffers.  A block clears its words of set i - 1
// after meeting i (every block has then published set i, so it has read all of
// i - 1) and waits for those stores before it publishes its sums of set i + 1;
// a reader of set i + 2 has those sums and so cannot see the old words.
//
// The solution goes to a buffer of its own: after a wait that ran out the host
// starts again from the caller's state with the per-iteration launches.
#include "adjoint.h"
#include "persist_common.h"

namespace pncg {

namespace {

constexpr int kCgThreads = 512;   // 256 registers to a thread; two tet passes at 110,000 tets
constexpr int kCgWaves = 4;       // waves of a k_cg_fused block, whose order of sums is kept

// What a thread keeps of a tet.
struct CgTet {
  Kin<double> kin;
  double B[9], a2, psi3, psi33;
  bool ok;
};

struct CgArgs {
  Args<double> A;
  AdjArgs C;
  PersistArgs P;
  CgLayout at;
  int k0;
};

// Sums over the partials of the launch before (part [grid][8]) as gather
// leaves them.
template <int N>
__device__ __forceinline__ void stored_sums(const double* part, int n, double* sh) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & (kWave - 1);
  const int nw = min(4, (n + kWave - 1) / kWave);
  for (int t = wave; t < N * nw; t += kCgThreads / kWave) {
    const int q = t / nw, w = t - q * nw, j = w * kWave + lane;
    double v = 0.0;
    if (j < n) v = v + part[8 * j + q];
    if (j + kSBlock < n) v = v + part[8 * (j + kSBlock) + q];
    v = wave_sum(v);
    if (lane == 0) sh[q * 4 + w] = v;
  }
}

}  // namespace

// ONE: a thread has at most one tet (the largest block's entries are one chunk
// of at most kCgThreads) and keeps it; otherwise the tets are formed again in
// each iteration (a kept one beside them would spill).
template <int M, bool ONE>
__global__ void __launch_bounds__(kCgThreads) k_cg_persist(CgArgs) {
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ double sh[2 * kCgWaves * 24];
  __shared__ double shg[7 * 4];
  __shared__ double planes[4 * kMaxPlanes];
  __shared__ struct {
    double alpha, beta;
    int exit, bad;
  } run;
  __shared__ PersistBlock B;
  __shared__ int4 chk[kMaxChunks + 1];
  __shared__ int slot_id[2], lblk[2][2];
#define PHASE                                                                                   \
  const ArgPtr<CgArgs> K = kernel_args<CgArgs>();                                               \
  const int tid = fresh(threadIdx.x), n = K->P.grid, vb = K->P.vb;                              \
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);          \
  (void)n, (void)vb, (void)lane, (void)wave
#define LDS_AT(T, field) reinterpret_cast<T*>(lds + K->at.field)
  int k0, set0, own0;
  {
    PHASE;
    k0 = K->k0;
    const int lp =
        (gridDim.x % kXcds) ? blockIdx.x : (blockIdx.x % kXcds) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
    const PersistBlock b = K->P.blk[lp];
    if (tid == 0) B = b;
    if (tid < 2) {
      const long long l = lp * vb + min(tid, vb - 1), nw = K->A.nWaves, per = (nw + n - 1) / n;
      slot_id[tid] = (int)((l % (n / kXcds)) * kXcds + l / (n / kXcds));
      lblk[tid][0] = (int)min(l * per, nw);
      lblk[tid][1] = (int)min((l + 1) * per, nw);
    }
    if (tid < 4 * kMaxPlanes) planes[tid] = K->A.planes.p[tid >> 2][tid & 3];
    if (tid == 0) run.bad = run.exit = 0;
    const int* lv = K->P.loc_v + b.loc_off;
    own0 = lv[0];   // own vertices are consecutive
    set0 = *K->P.ring;
    // state after launch k0 - 1
    double *X = LDS_AT(double, x), *Z = LDS_AT(double, z), *Pv = LDS_AT(double, p), *W = LDS_AT(double, w);
    const double4 *zw = K->C.zw[(k0 + 1) & 1], *pp = K->C.pbuf[(k0 + 1) & 1];
    for (int l = tid; l < b.nloc; l += kCgThreads) {
      const int v = lv[l];
      const V3<double> x = ld3(K->A.x0, v), z = ld3(zw, 2 * v), w = ld3(zw, 2 * v + 1);
      V3<double> p = mk3(0.0, 0.0, 0.0);
      if (k0 > 0) p = ld3(pp, v);
      X[3 * l] = x.x; X[3 * l + 1] = x.y; X[3 * l + 2] = x.z;
      Z[3 * l] = z.x; Z[3 * l + 1] = z.y; Z[3 * l + 2] = z.z;
      W[3 * l] = w.x; W[3 * l + 1] = w.y; W[3 * l + 2] = w.z;
      Pv[3 * l] = p.x; Pv[3 * l + 1] = p.y; Pv[3 * l + 2] = p.z;
      if (l < b.nown) {
        const V3<double> lam = ld3(k0 > 0 ? K->C.r : K->C.lam, v);
        double *L = LDS_AT(double, lam), *D = LDS_AT(double, diag);
        L[3 * l] = lam.x; L[3 * l + 1] = lam.y; L[3 * l + 2] = lam.z;
        LDS_AT(double, m)[l] = K->A.mass[v];
        LDS_AT(uint8_t, fl)[l] = K->A.vflag[v];
        for (int j = 0; j < 3; ++j) D[3 * l + j] = K->C.diag[3 * v + j];
        LDS_AT(ushort2, run)[l] = K->P.run[v];
      } else {
        LDS_AT(int, hv)[l - b.nown] = v;
      }
    }
    for (int t = tid; t < b.ntet; t += kCgThreads) LDS_AT(ushort4, tl)[t] = K->P.tet_l[b.tet_off + t];
    const int nc = K->P.chunks;
    const int4* ck = K->P.chunk + lp * (nc + 1);
    if (tid <= nc) chk[tid] = ck[tid];
    const int s0 = ck[nc].w;
    for (int i = tid; i < ck[nc].z; i += kCgThreads) LDS_AT(ushort2, seg)[i] = K->P.seg[s0 + i];
    for (int i = tid; i < b.nw; i += kCgThreads) LDS_AT(ulonglong2, wm)[i] = K->P.wave_last[b.w0 + i];
  }
  auto set_of = [&](int it) { return fresh_s(set0 + it - k0) % 3; };
  // clear this block's words of iteration it's set (those of the step kernel's
  // second meeting too: its next launch begins on one of these sets)
  auto clear = [&](int it) {
    PHASE;
    const int s = set_of(it);
    if (tid < 8 * vb) st_agent(K->P.slot_grad + s * 8 * n + (tid & 7) * n + slot_id[tid >> 3], kEmpty);
    if (tid < 3 * vb) st_agent(K->P.slot_dir + s * 3 * n + (tid % 3) * n + slot_id[tid / 3], kEmpty);
    u64* w = K->P.pgx + 3 * ((size_t)s * K->A.nV + own0);
    for (int i = tid; i < 3 * B.nown; i += kCgThreads) st_agent(w + i, kEmpty);
  };
  __syncthreads();
  clear(k0 + 1);
  clear(k0 + 2);
  auto tet_of = [&](int t) {
    const ArgPtr<CgArgs> K = kernel_args<CgArgs>();
    CgTet T;
    const ElemRec<double>& r = K->A.elem[K->P.tet_e[B.tet_off + t]];
#pragma unroll
    for (int j = 0; j < 9; ++j) T.B[j] = r.B[j];
    const ushort4 v = LDS_AT(ushort4, tl)[t];
    const double* X = LDS_AT(double, x);
    T.kin = kinematics<double>(T.B, at3(X, v.x), at3(X, v.y), at3(X, v.z), at3(X, v.w));
    T.ok = i23_ok<double, M>(T.kin);
    i23_coeffs<double, M>(T.kin, r.vmu, r.vlam, T.a2, T.psi3, T.psi33);
    return T;
  };
  auto corner_terms = [&](const CgTet& T, ushort4 v, const PersistEntry& en) {
    const ArgPtr<CgArgs> K = kernel_args<CgArgs>();
    const double* Pv = LDS_AT(double, p);
    double* res = LDS_AT(double, res);
    V3<double> d[3];
    dF_cols(T.B, at3(Pv, v.x), at3(Pv, v.y), at3(Pv, v.z), at3(Pv, v.w), d);
    const HpTet<double> hp = i23_Hp_tet(T.kin, T.psi33, d);
#pragma unroll
    for (int a = 0; a < 4; ++a) {
      const unsigned short to = en.slot[a];
      if (to == kNone) continue;
      V3<double> h = mk3(0.0, 0.0, 0.0);
      if (T.ok) h = i23_Hp_corner(T.kin, hp, T.a2, T.psi3, shape_vec(T.B, a));
      double* o = res + 3 * to;
      o[0] = h.x; o[1] = h.y; o[2] = h.z;
    }
    if (!T.ok) raise_err(K->A.status, kErrInverted);
  };
  PersistEntry en0{};
  CgTet T0{};
  ushort4 v0{};
  bool has0 = false;
  double bb = 0.0;
  {
    PHASE;
    if constexpr (ONE) {
      has0 = chk[0].x + tid < chk[1].x;
      if (has0) {
        en0 = K->P.entry[chk[0].x + tid];
        T0 = tet_of(en0.tet);
        v0 = LDS_AT(ushort4, tl)[en0.tet];
      }
    }
    stored_sums<7>(K->C.part_f, n, shg);
    if (k0 > 0) bb = K->C.status->bb;
  }
  __syncthreads();

  int k = k0;
  for (; k - k0 < kPersistMaxIters; ++k) {
    // ---- the stop rules, alpha and beta
    if (threadIdx.x < kWave) {
      PHASE;
      double r[7];
      totals<7>(shg, n, 0u, r);
      const double pq = r[0], rz = r[1], rr = r[2], rw = r[3], qz = r[4], qw = r[5];
      if (k == 0) bb = r[6];
      int reason = -1;
      double alpha = 0.0, beta = 0.0;
      if (rr <= K->C.tol2 * bb) {
        reason = 0;
      } else if (k > 0 && k - 1 >= K->C.max_iter) {
        reason = 1;
      } else if (k > 0) {
        if (!(pq > 0.0) || !isfinite(pq)) {
          reason = 2;
        } else {
          alpha = rz / pq;
          const double rz_new = cg_next_rz(alpha, rz, rw, qz, qw);
          beta = rz_new > 0.0 ? rz_new / rz : 0.0;
        }
      }
      if (lane == 0) {
        run.alpha = alpha;
        run.beta = beta;
        run.exit = reason >= 0;
      }
      if (blockIdx.x == 0 && tid == 0) {
        CgStatus* st = K->C.status;
        if (k == 0) st->bb = bb;
        if (reason >= 0) {
          st->iters = k > 0 ? k - 1 : 0;
          st->reason = reason;
          st->rr = reason == 2 ? 0.0 : rr;
          st->stopped = 1;
        }
      }
    }
    __syncthreads();
    if (run.exit) break;
    // ---- lambda_k, z_k and p_k
    {
      PHASE;
      const double alpha = run.alpha, beta = run.beta;
      double *Z = LDS_AT(double, z), *Pv = LDS_AT(double, p), *L = LDS_AT(double, lam);
      const double* W = LDS_AT(double, w);
      for (int i = tid; i < 3 * B.nloc; i += kCgThreads) {
        const double pp = Pv[i], z = fma(-alpha, W[i], Z[i]);
        Z[i] = z;
        Pv[i] = k == 0 ? z : fma(beta, pp, z);
        if (k > 0 && i < 3 * B.nown) L[i] = fma(alpha, pp, L[i]);
      }
    }
    __syncthreads();
    // ---- q = H p_k and w = q / diag of the own vertices
    for (int c = 0;; ++c) {
      {
        PHASE;
        if constexpr (ONE) {
          if (has0) corner_terms(T0, v0, en0);
        } else {
          for (int e = chk[c].x + tid; e < chk[c + 1].x; e += kCgThreads) {
            const PersistEntry en = K->P.entry[e];
            corner_terms(tet_of(en.tet), LDS_AT(ushort4, tl)[en.tet], en);
          }
        }
      }
      __syncthreads();
      {
        PHASE;
        const ushort2* seg = LDS_AT(ushort2, seg);
        const double* res = LDS_AT(double, res);
        double* tot = LDS_AT(double, tot);
        const int t1 = 3 * chk[c + 1].z;
        for (int t = 3 * chk[c].z + tid; t < t1; t += kCgThreads) {
          const int s = t / 3;
          const ushort2 r = seg[s];
          tot[t] = row_run_sum<3>(res + (t - 3 * s), r.x, r.y);
        }
      }
      // (the words cleared after the last meeting are out before any sums that
      // this block publishes from here on)
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      PHASE;
      const double *X = LDS_AT(double, x), *Pv = LDS_AT(double, p), *Ms = LDS_AT(double, m), *D = LDS_AT(double, diag);
      double *W = LDS_AT(double, w), *Q = LDS_AT(double, q);
      const double h2 = K->A.h2;
      u64* wx = K->P.pgx + 3 * ((size_t)set_of(k) * K->A.nV + own0);
      for (int i = 3 * chk[c].y + tid; i < 3 * chk[c + 1].y; i += kCgThreads) {
        const int l = i / 3, j = i - 3 * l;
        const uint8_t fl = LDS_AT(uint8_t, fl)[l];
        const ushort2 r = LDS_AT(ushort2, run)[l];
        const double* tr = LDS_AT(double, tot) + 3 * r.x + j;
        double s = 0.0;
        for (int u = 0; u < r.y; ++u) s += tr[3 * u];
        double q = fma(h2, s, Ms[l] * Pv[i]);
        if (fl & kSurface) {
          const V3<double> x = at3(X, l), p = at3(Pv, l);
          for (int a = 0; a < K->A.planes.n; ++a) {
            const double* pl = planes + 4 * a;
            const double d = plane_dist(pl, x), dhat = K->A.dhat;
            if (d > 0.0 && d < dhat)
              q = fma(plane_Hp(K->A.kappa, pl, d, dhat, p), pl[j], q);
          }
        }
        if (fl & kFixed) q = 0.0;
        const double w = q / D[i];
        Q[i] = q;
        W[i] = w;
        st_agent(wx + i, full(word(w)));
      }
      __syncthreads();
      if (ONE || c + 1 >= K->P.chunks) break;
    }
    // ---- the six sums, each vertex at the lane its sum ended on
    {
      PHASE;
      if (wave < vb * kCgWaves) {
        const double *Pv = LDS_AT(double, p), *Z = LDS_AT(double, z), *Q = LDS_AT(double, q), *D = LDS_AT(double, diag),
                     *W = LDS_AT(double, w);
        const ulonglong2* wm = LDS_AT(ulonglong2, wm);
        const int vi = wave / kCgWaves, w0 = B.w0, we = lblk[vi][1];
        double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        for (int w = lblk[vi][0] + wave % kCgWaves; w < we; w += kCgWaves) {
          const ulonglong2 m = wm[w - w0];
          if ((m.x >> lane) & 1) {
            const int l = (int)m.y + __popcll(m.x & ((1ull << lane) - 1));
            const V3<double> p = at3(Pv, l), q = at3(Q, l), z = at3(Z, l), d = at3(D, l), wq = at3(W, l);
            const V3<double> r = mk3(d.x * z.x, d.y * z.y, d.z * z.z);
            acc[0] += dot(p, q);
            acc[1] += dot(r, z);
            acc[2] += dot(r, r);
            acc[3] += dot(r, wq);
            acc[4] += dot(q, z);
            acc[5] += dot(q, wq);
          }
        }
        const double r = row_sums6(acc);
        if ((lane & 15) < 6) sh[wave * 24 + (lane >> 4) * 6 + (lane & 7)] = r;
      }
    }
    __syncthreads();
    // ---- the meeting: the sums, and w of the vertices shared with others
    {
      PHASE;
      const int s = set_of(k);
      u64* slots = K->P.slot_grad + s * 8 * n;
      if (tid < 8 * vb && (tid & 7) < 6) {
        const int i = tid >> 3, q = tid & 7;
        const double* h = sh + i * kCgWaves * 24 + q;
        double r = (h[18] + h[12]) + (h[6] + h[0]);
        for (int w = 1; w < kCgWaves; ++w) r += (h[24 * w + 18] + h[24 * w + 12]) + (h[24 * w + 6] + h[24 * w]);
        st_agent(slots + q * n + slot_id[i], full(word(r)));
        if (k - k0 + 1 == kPersistMaxIters) K->C.part_f[8 * slot_id[i] + q] = r;   // for the next launch
      }
      constexpr int kWords = 2;
      const u64* src = K->P.pgx + 3 * (size_t)s * K->A.nV;
      const int* hv = LDS_AT(int, hv);
      const int nh = 3 * (B.nloc - B.nown);
      double* wh = LDS_AT(double, w) + 3 * B.nown;
      const u64* from[kWords];
#pragma unroll
      for (int u = 0; u < kWords; ++u) {
        const int i = tid + u * kCgThreads;
        from[u] = i < nh ? src + 3 * (size_t)hv[i / 3] + i % 3 : nullptr;
      }
      const long long limit = K->P.limit;
      gather<6>(slots, n, 0u, shg, kCgThreads / kWave, limit, &run.bad, [&]() {
        u64 w[kWords];
#pragma unroll
        for (int u = 0; u < kWords; ++u) w[u] = from[u] ? ld_agent(from[u]) : 0;
        bool all = true;
#pragma unroll
        for (int u = 0; u < kWords; ++u) {
          if (!from[u]) continue;
          if (w[u] == kEmpty) {
            all = false;
          } else {
            wh[tid + u * kCgThreads] = as_double(w[u]);
            from[u] = nullptr;
          }
        }
        return all;
      });
      for (int i = tid + kWords * kCgThreads; i < nh; i += kCgThreads) {
        const u64* p = src + 3 * (size_t)hv[i / 3] + i % 3;
        u64 w = ld_agent(p);
        Wait t(limit);
        while (w == kEmpty) {
          if (run.bad || t.over()) {
            run.bad = 1;
            break;
          }
          w = ld_agent(p);
        }
        wh[i] = as_double(w);
      }
    }
    __syncthreads();
    if (run.bad) break;
    if (k > k0) clear(k - 1);
  }
  PHASE;
  if (run.bad) {
    if (tid == 0) K->C.status->sync = 1;
    return;
  }
  // lambda, and where the launch reached its own limit the state after launch k - 1
  const bool more = !run.exit;
  const double *L = LDS_AT(double, lam), *Z = LDS_AT(double, z), *W = LDS_AT(double, w), *Pv = LDS_AT(double, p);
  double4 *zw = K->C.zw[(k + 1) & 1], *pp = K->C.pbuf[(k + 1) & 1];
  for (int l = tid; l < B.nown; l += kCgThreads) {
    const int v = own0 + l;
    st3(K->C.r, v, at3(L, l));
    if (more) {
      st3(zw, 2 * v, at3(Z, l));
      st3(zw, 2 * v + 1, at3(W, l));
      st3(pp, v, at3(Pv, l));
    }
  }
  if (blockIdx.x == 0 && tid == 0) *K->P.ring = set_of(k);
#undef LDS_AT
#undef PHASE
}

// The kernel for a model and a mesh.
static void (*variant(int model, const CgPersist& P))(CgArgs) {
  const bool one = P.P.chunks == 1 && P.most <= kCgThreads;
  if (model == kModelSNH) return one ? k_cg_persist<kModelSNH, true> : k_cg_persist<kModelSNH, false>;
  return one ? k_cg_persist<kModelNH, true> : k_cg_persist<kModelNH, false>;
}

hipError_t cg_persist_fits(const CgPersist& P, int model, int compute_units, bool* ok) {
  int per_cu = 0;
  const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)variant(model, P), kCgThreads, P.lds);
  *ok = e == hipSuccess && per_cu >= 1 && P.P.blocks <= compute_units;
  return e;
}

void launch_cg_persist(const Args<double>& A, const AdjArgs& C, const CgPersist& P, int k0, hipStream_t s) {
  hipLaunchKernelGGL(variant(A.model, P), dim3(P.P.blocks), dim3(kCgThreads), P.lds, s, (CgArgs{A, C, P.P, P.at, k0}));
}

}  // namespace pncg
