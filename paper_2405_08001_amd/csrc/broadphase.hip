// Broad phase: candidate point-triangle and edge-edge pairs by an inflated
// axis-aligned box test in float64 over a uniform grid (the paper culls with
// a grid hash, Sec. 6; the grid changes speed, not the set).
//
//   PT (v, f): v a surface vertex not in f, and on every axis
//              min_f - r <= x_v <= max_f + r
//   EE (e1 < e2) without a shared vertex, on every axis
//              min_e1 - r <= max_e2  and  min_e2 <= max_e1 + r
//
// Grid entries (cell, item): every surface vertex in its cell, every
// triangle in each cell its r-inflated box touches, every edge in each cell
// its (r/2 + margin)-inflated box touches.  Entries are grouped by a hash of
// the cell; each entry's record (cell, item, exact float64 box, vertex ids)
// is stored contiguously per bucket.  Each entry is tested against others of
// its bucket so that a pair sharing a cell is seen once per shared cell.  A vertex lies in one cell, which is among the
// triangle's cells whenever the PT test holds; an edge pair is reported only
// in the cell holding the lower corner of the intersection of the two
// inflated boxes, which both edges touch.  So every pair is found exactly
// once, and the exact test above makes the final decision.
//
// The grid's cells are the caller's, 2^shift of them to a side (Broad).  The
// capacity of the entry arrays is counted in caller's cells, so which states
// fit does not depend on the shift; an item touches no more cells of the grid
// than caller's cells.
//
// The queries' lists are produced without any global counter: a counting pass
// stores the pair counts of every entry, an exclusive scan turns them into
// offsets (point-triangle counts of all entries first, then edge-edge), and a
// second pass writes the pairs.  The solver's list is emitted in one pass
// (k_pairs_emit) and put in order by its index.
#include <algorithm>
#include <climits>

#include "kernels.h"

namespace pncg {

namespace {

constexpr int kTile = kBlock * 16;
constexpr double kEdgeMargin = 1e-9;   // absolute slack of the edge culling boxes (m)

__device__ __forceinline__ int cell_coord(double p, double inv) {
  double c = floor(p * inv);
  c = fmin(fmax(c, -1048575.0), 1048575.0);
  return (int)c;
}
__device__ __forceinline__ int3 cell_of(V3<double> p, double inv, int shift) {
  return make_int3(cell_coord(p.x, inv) >> shift, cell_coord(p.y, inv) >> shift, cell_coord(p.z, inv) >> shift);
}
__device__ __forceinline__ long long cells_between(int3 a, int3 b) {
  return (long long)(b.x - a.x + 1) * (b.y - a.y + 1) * (b.z - a.z + 1);
}
__device__ __forceinline__ unsigned long long cell_key(int cx, int cy, int cz) {
  return ((unsigned long long)(cx + 1048576) << 42) | ((unsigned long long)(cy + 1048576) << 21) |
         (unsigned long long)(cz + 1048576);
}
// bucket of a cell in one half of the table: triangles use [0, tsize/2),
// edges [tsize/2, tsize)
__device__ __forceinline__ unsigned hash_key(unsigned long long k, int tsize, bool edge) {
  const unsigned cx = (unsigned)(k >> 42), cy = (unsigned)((k >> 21) & 0x1FFFFF), cz = (unsigned)(k & 0x1FFFFF);
  unsigned h = (cx * 73856093u) ^ (cy * 19349663u) ^ (cz * 83492791u);
  const unsigned half = (unsigned)tsize >> 1;
  return (h & (half - 1)) + (edge ? half : 0u);
}
__device__ __forceinline__ V3<double> ldx(const double4* x, int i) {
  double4 v = x[i];
  return mk3(v.x, v.y, v.z);
}
__device__ __forceinline__ V3<double> v4(double4 v) { return mk3(v.x, v.y, v.z); }
__device__ __forceinline__ V3<double> vmin3(V3<double> a, V3<double> b) { return mk3(fmin(a.x, b.x), fmin(a.y, b.y), fmin(a.z, b.z)); }
__device__ __forceinline__ V3<double> vmax3(V3<double> a, V3<double> b) { return mk3(fmax(a.x, b.x), fmax(a.y, b.y), fmax(a.z, b.z)); }

__device__ __forceinline__ bool in_sorted(const unsigned long long* keys, int n, unsigned long long k) {
  int lo = 0, hi = n;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (keys[mid] < k) lo = mid + 1; else hi = mid;
  }
  return lo < n && keys[lo] == k;
}

// --------------------------------------------------------------- scan
template <typename T>
__global__ void __launch_bounds__(kBlock) k_scan_reduce(const T* in, long long n, T* bsum) {
  __shared__ T sh[kBlock / kWave];
  const long long base = (long long)blockIdx.x * kTile;
  T s = 0;
  for (int i = threadIdx.x; i < kTile; i += kBlock) {
    long long j = base + i;
    if (j < n) s += in[j];
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, kWave);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    T t = 0;
    for (int w = 0; w < kBlock / kWave; ++w) t += sh[w];
    bsum[blockIdx.x] = t;
  }
}

// out[j] = exclusive prefix of in[j]; *total = sum (written by the last
// block).  Each block first adds up the sums of the blocks before it (bsum,
// from k_scan_reduce) in a fixed order, which takes the place of a separate
// launch that scans bsum.  RAW: it adds up their input instead.
template <typename T, bool RAW>
__global__ void __launch_bounds__(kBlock) k_scan_down(const T* in, long long n, const T* bsum, T* out, T* total) {
  __shared__ T sh[kBlock];
  __shared__ T sw[kBlock / kWave];
  T pre = 0;
  if constexpr (RAW) {
    // (kTile is a multiple of 8 kBlock: eight loads in flight)
    for (int j = threadIdx.x; j < (int)blockIdx.x * kTile; j += 8 * kBlock) {
      T u[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) u[i] = in[j + i * kBlock];
#pragma unroll
      for (int i = 0; i < 8; ++i) pre += u[i];
    }
  } else {
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kBlock) pre += bsum[b];
  }
  for (int o = kWave / 2; o > 0; o >>= 1) pre += __shfl_down(pre, o, kWave);
  if ((threadIdx.x & (kWave - 1)) == 0) sw[threadIdx.x / kWave] = pre;
  const long long base = (long long)blockIdx.x * kTile + (long long)threadIdx.x * 16;
  T v[16];
  T s = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    long long j = base + i;
    v[i] = j < n ? in[j] : 0;
    s += v[i];
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  T boff = 0;
#pragma unroll
  for (int w = 0; w < kBlock / kWave; ++w) boff += sw[w];
  for (int o = 1; o < kBlock; o <<= 1) {
    T u = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
    __syncthreads();
    sh[threadIdx.x] += u;
    __syncthreads();
  }
  T run = boff + sh[threadIdx.x] - s;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    long long j = base + i;
    if (j < n) out[j] = run;
    run += v[i];
  }
  if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == kBlock - 1) *total = run;
}

template <typename T>
void scan_exclusive(const T* in, long long n, T* out, T* total, T* scratch, hipStream_t s) {
  const int nb = (int)((n + kTile - 1) / kTile);
  // up to eight tiles the last block reads its predecessors' 28,672 values
  // in less time than the reduction's launch takes (about 6 us)
  if (nb <= 8) {
    hipLaunchKernelGGL((k_scan_down<T, true>), dim3(nb), dim3(kBlock), 0, s, in, n, (const T*)nullptr, out, total);
    return;
  }
  hipLaunchKernelGGL(k_scan_reduce<T>, dim3(nb), dim3(kBlock), 0, s, in, n, scratch);
  hipLaunchKernelGGL((k_scan_down<T, false>), dim3(nb), dim3(kBlock), 0, s, in, n, (const T*)scratch, out, total);
}

// ------------------------------------------------------------ grid build

// culling box of primitive i (0..nF-1 triangles, nF.. edges) with record lo,
// hi: what is inserted into the grid
__device__ __forceinline__ void cull_box(const Broad& B, int i, double r, V3<double> lo, V3<double> hi, V3<double>& cl,
                                         V3<double>& ch) {
  const double q = i >= B.nF ? 0.5 * r + kEdgeMargin : 0.0;
  cl = i >= B.nF ? mk3(lo.x - q, lo.y - q, lo.z - q) : lo;
  ch = i >= B.nF ? mk3(hi.x + q, hi.y + q, hi.z + q) : hi;
}

// Boxes of the items, and the entries of the grid: places for them (item_off,
// in the order in which blocks come, one reservation each) and each one's rank
// in its bucket, by bumping the bucket's counter.  Given a list counter, also
// empties the list.  One launch for boxes, counts and entries, where a scan of
// the counts for places in order took three more (bar of 15,360 tets: 25 -> 12 us,
// pile of 110,000: 43 -> 27 us, bound by the counters' atomics).
constexpr int kItems = 256;      // items of a block: a reservation costs 40 ns, one after the other
constexpr int kItemBlock = 1024;
constexpr int kItemLanes = 8;    // lanes that share an item's entries: a thread per item would make its 4 to 30 atomics or
                                 // record stores one behind the other

__device__ __forceinline__ int block_excl_scan(int v, int& total, int* sh);

struct ItemCells {
  int3 c0;
  unsigned nz, nyz;
  long long off, m;   // first entry, number of entries
};
// entries of an item, t by lane t mod kItemLanes of its group, z fastest, then
// y, then x: f(entry, cell key)
template <typename F>
__device__ __forceinline__ void item_entries(const ItemCells& c, int lane, F&& f) {
  for (long long t = lane; t < c.m; t += kItemLanes) {
    const unsigned cx = (unsigned)t / c.nyz, rem = (unsigned)t - cx * c.nyz, cy = rem / c.nz;
    f(c.off + t, cell_key(c.c0.x + (int)cx, c.c0.y + (int)cy, c.c0.z + (int)(rem - cy * c.nz)));
  }
}
// cells of the culling box of item i whose entries begin at off; those past the
// capacity are left out
__device__ __forceinline__ ItemCells item_cells(const Broad& B, V3<double> cl, V3<double> ch, double inv, long long off) {
  ItemCells c;
  const int3 c1 = cell_of(ch, inv, B.shift);
  c.c0 = cell_of(cl, inv, B.shift);
  c.nz = c1.z - c.c0.z + 1;
  c.nyz = (c1.y - c.c0.y + 1) * c.nz;
  c.off = off;
  c.m = max(0ll, min(cells_between(c.c0, c1), B.ent_cap - off));
  return c;
}

__global__ void __launch_bounds__(kItemBlock) k_items(Broad B, const double4* x, double inv, double r, long long* ncand) {
  __shared__ ItemCells cells[kItems];
  __shared__ long long wsum[kItems / kWave];
  __shared__ unsigned long long sbase;
  if (ncand && blockIdx.x == 0 && threadIdx.x == 0) {
    ncand[0] = 0;
    ncand[1] = -1;
  }
  const int n = B.nF + B.nE, i0 = blockIdx.x * kItems;
  const int i = i0 + threadIdx.x, lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const bool mine = threadIdx.x < kItems;
  long long cnt = 0, incl = 0;
  V3<double> cl = mk3(0.0, 0.0, 0.0), ch = cl;
  if (mine) {
    if (i < n) {
      V3<double> lo, hi;
      if (i < B.nF) {
        const V3<double> a = ldx(x, B.tris[3 * i]), b = ldx(x, B.tris[3 * i + 1]), c = ldx(x, B.tris[3 * i + 2]);
        const V3<double> mn = vmin3(vmin3(a, b), c), mx = vmax3(vmax3(a, b), c);
        lo = mk3(mn.x - r, mn.y - r, mn.z - r);
        hi = mk3(mx.x + r, mx.y + r, mx.z + r);
      } else {
        const int e = i - B.nF;
        const V3<double> a = ldx(x, B.edges[2 * e]), b = ldx(x, B.edges[2 * e + 1]);
        lo = vmin3(a, b);
        hi = vmax3(a, b);
      }
      B.item_lo[i] = make_double4(lo.x, lo.y, lo.z, 0.0);
      B.item_hi[i] = make_double4(hi.x, hi.y, hi.z, 0.0);
      cull_box(B, i, r, lo, hi, cl, ch);
      // entries are counted in caller's cells, up to a bound that no capacity
      // reaches and whose sums cannot overflow
      cnt = min(cells_between(cell_of(cl, inv, 0), cell_of(ch, inv, 0)), 1ll << 40);
    }
    incl = cnt;
    for (int o = 1; o < kWave; o <<= 1) {
      const long long u = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += u;
    }
    if (lane == kWave - 1) wsum[wave] = incl;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int w = 0; w < kItems / kWave; ++w) {
      const long long u = wsum[w];
      wsum[w] = t;
      t += u;
    }
    sbase = atomicAdd(B.resv, (unsigned long long)t);
  }
  __syncthreads();
  if (mine) {
    const long long off = (long long)sbase + wsum[wave] + incl - cnt;
    ItemCells c{};
    if (i < n) {
      B.item_off[i] = off;
      c = item_cells(B, cl, ch, inv, off);
    }
    cells[threadIdx.x] = c;
  }
  __syncthreads();
  for (int q = threadIdx.x / kItemLanes; q < kItems; q += kItemBlock / kItemLanes) {
    const bool edge = i0 + q >= B.nF;
    item_entries(cells[q], threadIdx.x & (kItemLanes - 1), [&](long long e, unsigned long long k) {
      B.ent_rank[e] = atomicAdd(&B.count[hash_key(k, B.tsize, edge)], 1);
    });
  }
}

// the slot after the last (slots are ints; a capacity beyond them counts
// caller's cells, not entries)
__device__ __forceinline__ int slot_end(const Broad& B) { return (int)min(B.ent_cap, (long long)INT_MAX); }

// Slots of the buckets: those of a tile of buckets are consecutive, and the
// tiles follow each other as their blocks come, triangles' from the first slot
// on, edges' up to the last.  Also empties the counters for the next build.
constexpr int kBucketsPer = 16;   // buckets of a thread
__global__ void __launch_bounds__(kBlock) k_bucket_alloc(Broad B, int tile) {
  __shared__ int sh[kBlock / kWave];
  __shared__ int sbase;
  const int h0 = blockIdx.x * tile, per = tile / kBlock, b0 = h0 + threadIdx.x * per;
  int c[kBucketsPer], s = 0;
#pragma unroll
  for (int i = 0; i < kBucketsPer; ++i) c[i] = i < per ? B.count[b0 + i] : 0;
#pragma unroll
  for (int i = 0; i < kBucketsPer; ++i) s += c[i];
  int total;
  int at = block_excl_scan(s, total, sh);
  if (threadIdx.x == 0) {
    const bool edge = h0 >= (B.tsize >> 1);
    const int before = (int)atomicAdd(B.resv + (edge ? 2 : 1), (unsigned long long)total);
    sbase = edge ? slot_end(B) - before - total : before;
  }
  __syncthreads();
  at += sbase;
#pragma unroll
  for (int i = 0; i < kBucketsPer; ++i) {
    if (i >= per) break;
    B.count[b0 + i] = 0;
    B.range[b0 + i] = make_int2(at, at + c[i]);
    at += c[i];
  }
}

// Group the entries by bucket and store each entry's full record there: its
// slot is the bucket's first plus the rank its counter gave it.  Also the words
// that later launches and the next build begin with: the edges' slots, the
// counters of the reservations and of the pair index (vcnt), and the build
// positions.
__global__ void __launch_bounds__(kBlock) k_bucket_fill(Broad B, const double4* x, double inv, double r, int* vcnt,
                                                        double4* xbuild) {
  const int n = B.nF + B.nE, lane = threadIdx.x & (kItemLanes - 1);
  const int tid = blockIdx.x * kBlock + threadIdx.x, stride = gridDim.x * kBlock;
  if (tid == 0) {
    B.totals[0] = (long long)B.resv[0];
    B.espan[0] = slot_end(B) - (long long)B.resv[2];
    B.espan[1] = slot_end(B);
    for (int j = 0; j < 3; ++j) B.resv[j] = 0;
  }
  if (vcnt)
    for (int v = tid; v < B.nV; v += stride) vcnt[v] = 0;
  if (xbuild)
    for (int v = tid; v < B.nV; v += stride) xbuild[v] = x[v];
  for (int i = tid / kItemLanes; i < n; i += stride / kItemLanes) {
    V3<double> cl, ch;
    const double4 ilo = B.item_lo[i], ihi = B.item_hi[i];
    cull_box(B, i, r, v4(ilo), v4(ihi), cl, ch);
    const bool edge = i >= B.nF;
    double4 lo = ilo, hi = ihi;
    int4 ids;
    if (!edge) {
      ids = make_int4(B.tris[3 * i], B.tris[3 * i + 1], B.tris[3 * i + 2], 0);
    } else {
      // an edge record holds its two end points (its box is their
      // component-wise min and max), so the exact distance of a pair reads
      // the staged records instead of gathering positions
      const int g = i - B.nF;
      ids = make_int4(B.edges[2 * g], B.edges[2 * g + 1], -1, 0);
      lo = x[ids.x];
      hi = x[ids.y];
    }
    item_entries(item_cells(B, cl, ch, inv, B.item_off[i]), lane, [&](long long e, unsigned long long k) {
      const int slot = B.range[hash_key(k, B.tsize, edge)].x + B.ent_rank[e];
      B.bkt_key[slot] = k;
      B.bkt_item[slot] = B.nSV + i;
      B.bkt_lo[slot] = lo;
      B.bkt_hi[slot] = hi;
      B.bkt_ids[slot] = ids;
    });
  }
}

// ------------------------------------------------------------------ pairs
// item ids: [0, nSV) surface vertices (surf order), [nSV, nSV + nF)
// triangles, [nSV + nF, ...) edges.
struct PairCtx {
  const double4* x;
  double inv, r, filter_d;
  int filter_obj;
};

// Records of a contiguous run of edge bucket slots held in LDS (an edge has
// two vertex ids; 34 KB, so that four blocks fit a compute unit).
constexpr int kSpan = 512;
struct SlotSpan {
  unsigned long long key[kSpan];
  int item[kSpan];
  int2 ids[kSpan];
  double lo[3][kSpan];
  double hi[3][kSpan];
};

// Record accessors: all slots from the LDS span, or all from global memory.
struct LdsRec {
  const SlotSpan& L;
  int base;
  __device__ __forceinline__ unsigned long long key(int t) const { return L.key[t - base]; }
  __device__ __forceinline__ int item(int t) const { return L.item[t - base]; }
  __device__ __forceinline__ int4 ids(int t) const {
    const int2 i = L.ids[t - base];
    return make_int4(i.x, i.y, -1, 0);
  }
  __device__ __forceinline__ V3<double> lo(int t) const {
    return mk3(L.lo[0][t - base], L.lo[1][t - base], L.lo[2][t - base]);
  }
  __device__ __forceinline__ V3<double> hi(int t) const {
    return mk3(L.hi[0][t - base], L.hi[1][t - base], L.hi[2][t - base]);
  }
};
struct GlobalRec {
  const Broad& B;
  __device__ __forceinline__ unsigned long long key(int t) const { return B.bkt_key[t]; }
  __device__ __forceinline__ int item(int t) const { return B.bkt_item[t]; }
  __device__ __forceinline__ int4 ids(int t) const { return B.bkt_ids[t]; }
  __device__ __forceinline__ V3<double> lo(int t) const { return v4(B.bkt_lo[t]); }
  __device__ __forceinline__ V3<double> hi(int t) const { return v4(B.bkt_hi[t]); }
};

// Point-triangle test of surface vertex v (position p, cell key) against
// the triangle entry in slot t.
__device__ __forceinline__ bool vertex_slot_pair(const Broad& B, const PairCtx& P, int v, V3<double> p,
                                                 unsigned long long key, int t, int2& out) {
  if (B.bkt_key[t] != key) return false;
  const int4 idB = B.bkt_ids[t];
  if (v == idB.x || v == idB.y || v == idB.z) return false;
  const V3<double> lo = v4(B.bkt_lo[t]), hi = v4(B.bkt_hi[t]);
  if (!(lo.x <= p.x && p.x <= hi.x && lo.y <= p.y && p.y <= hi.y && lo.z <= p.z && p.z <= hi.z)) return false;
  const int f = B.bkt_item[t] - B.nSV;
  // the distance filter first: it rejects most pairs in one step, while the
  // exclusion lookup is a chain of dependent loads (the filters commute)
  if (P.filter_d >= 0.0) {
    if (P.filter_obj && B.oid[v] != B.oid[idB.x]) return false;
    if (!(closest_pt(p, ldx(P.x, idB.x), ldx(P.x, idB.y), ldx(P.x, idB.z)).d < P.filter_d)) return false;
  }
  const unsigned long long pk = ((unsigned long long)(unsigned)v << 32) | (unsigned)f;
  if (B.n_excl_pt && in_sorted(B.excl_pt, B.n_excl_pt, pk)) return false;
  out = make_int2(v, f);
  return true;
}

// Exclusive prefix sum over a full wave by DPP lane moves: an inclusive
// scan within each row of 16 lanes (shifts by 1, 2, 4, 8), then lane 15 of
// rows 0 and 2 added to rows 1 and 3, then lane 31 to rows 2 and 3; the
// total is lane 63's.
__device__ __forceinline__ int wave_excl_scan(int v, int& total) {
  int x = v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
  total = __builtin_amdgcn_readlane(x, kWave - 1);
  return x - v;
}

// Point-triangle pairs of surface vertex w: one wave per vertex, one lane per
// slot of the vertex's triangle bucket.  FILL = false returns the count (in
// every lane); FILL = true writes the pairs from offset `o` in slot order.
template <bool FILL>
__device__ __forceinline__ int vertex_pairs_wave(const Broad& B, const PairCtx& P, int w, long long o, int2* out,
                                                 long long cap) {
  const int lane = threadIdx.x & (kWave - 1);
  const int v = B.surf[w];
  const V3<double> p = ldx(P.x, v);
  const int3 c = cell_of(p, P.inv, B.shift);
  const unsigned long long key = cell_key(c.x, c.y, c.z);
  const unsigned h = hash_key(key, B.tsize, false);
  const int2 sr = B.range[h];
  const int s0 = sr.x, s1 = sr.y;
  int count = 0;
  for (int t0 = s0; t0 < s1; t0 += kWave) {
    const int t = t0 + lane;
    int2 pr;
    const int hit = (t < s1 && vertex_slot_pair(B, P, v, p, key, t, pr)) ? 1 : 0;
    int tot;
    const int before = wave_excl_scan(hit, tot);
    if (FILL && hit) {
      const long long k = o + count + before;
      if (k < cap) out[k] = pr;
    }
    count += tot;
  }
  return count;
}

// Edge-edge pairs of edge slot s with the later edges of its cell.
template <typename Rec, typename Emit>
__device__ __forceinline__ void edge_pairs(const Broad& B, const PairCtx& P, const Rec& R, int s, Emit&& emit) {
  const int ebase = B.nSV + B.nF;
  const int ia = R.item(s);
  const unsigned long long key = R.key(s);
  const int2 sr = B.range[hash_key(key, B.tsize, true)];
  const int s0 = sr.x, s1 = sr.y;
  const V3<double> a0 = R.lo(s), a1 = R.hi(s);   // end points
  const V3<double> loA = vmin3(a0, a1), hiA = vmax3(a0, a1);
  const int4 idA = R.ids(s);
  const double r = P.r, q = 0.5 * P.r + kEdgeMargin;
  for (int t = s0; t < s1; ++t) {
    const int ib = R.item(t);
    if (ib <= ia || R.key(t) != key) continue;
    const int4 idB = R.ids(t);
    if (idA.x == idB.x || idA.x == idB.y || idA.y == idB.x || idA.y == idB.y) continue;
    const V3<double> b0 = R.lo(t), b1 = R.hi(t);
    const V3<double> lo = vmin3(b0, b1), hi = vmax3(b0, b1);
    // exact test with e1 = this (smaller) edge
    if (!((loA.x - r) <= hi.x && (loA.y - r) <= hi.y && (loA.z - r) <= hi.z)) continue;
    if (!(lo.x <= (hiA.x + r) && lo.y <= (hiA.y + r) && lo.z <= (hiA.z + r))) continue;
    // report only in the cell of the lower corner of the culling-box intersection
    const V3<double> corner = mk3(fmax(loA.x - q, lo.x - q), fmax(loA.y - q, lo.y - q), fmax(loA.z - q, lo.z - q));
    const int3 cc = cell_of(corner, P.inv, B.shift);
    if (cell_key(cc.x, cc.y, cc.z) != key) continue;
    const int e1 = ia - ebase, e2 = ib - ebase;
    // distance filter before the exclusion lookup (see vertex_slot_pair)
    if (P.filter_d >= 0.0) {
      if (P.filter_obj && B.oid[idA.x] != B.oid[idB.x]) continue;
      if (!(closest_ee(a0, a1, b0, b1).d < P.filter_d)) continue;
    }
    const unsigned long long pk = ((unsigned long long)(unsigned)e1 << 32) | (unsigned)e2;
    if (B.n_excl_ee && in_sorted(B.excl_ee, B.n_excl_ee, pk)) continue;
    emit(make_int2(e1, e2));
  }
}

// An edge's record, and that of slot s.
struct EdgeRec {
  unsigned long long key;
  int item;
  int4 ids;
  V3<double> a, b;   // end points
};
template <typename Rec>
__device__ __forceinline__ EdgeRec edge_rec(const Rec& R, int s) {
  return EdgeRec{R.key(s), R.item(s), R.ids(s), R.lo(s), R.hi(s)};
}

// Edge-edge test of edge E against slot t of its bucket, the pair reported
// once: e1 is the edge with the smaller item id, whose record takes the first
// place in the exact box test, the reporting-cell test and the distance (the
// same evaluation as edge_pairs from e1's side).  Emits (e1, ~e2).
template <typename Rec>
__device__ __forceinline__ bool edge_slot_pair_test(const Broad& B, const PairCtx& P, const Rec& R, const EdgeRec& E,
                                                    int t, int2& out) {
  const int ebase = B.nSV + B.nF;
  if (R.key(t) != E.key) return false;
  const int4 idT = R.ids(t);
  if (E.ids.x == idT.x || E.ids.x == idT.y || E.ids.y == idT.x || E.ids.y == idT.y) return false;
  const int item = R.item(t);
  const bool first = E.item < item;
  const V3<double> t0 = R.lo(t), t1 = R.hi(t);
  const V3<double> a0 = first ? E.a : t0, a1 = first ? E.b : t1, b0 = first ? t0 : E.a, b1 = first ? t1 : E.b;
  const V3<double> loA = vmin3(a0, a1), hiA = vmax3(a0, a1), lo = vmin3(b0, b1), hi = vmax3(b0, b1);
  const double r = P.r, q = 0.5 * P.r + kEdgeMargin;
  if (!((loA.x - r) <= hi.x && (loA.y - r) <= hi.y && (loA.z - r) <= hi.z)) return false;
  if (!(lo.x <= (hiA.x + r) && lo.y <= (hiA.y + r) && lo.z <= (hiA.z + r))) return false;
  const V3<double> corner = mk3(fmax(loA.x - q, lo.x - q), fmax(loA.y - q, lo.y - q), fmax(loA.z - q, lo.z - q));
  const int3 cc = cell_of(corner, P.inv, B.shift);
  if (cell_key(cc.x, cc.y, cc.z) != E.key) return false;
  const int e1 = (first ? E.item : item) - ebase, e2 = (first ? item : E.item) - ebase;
  if (P.filter_d >= 0.0) {
    if (P.filter_obj && B.oid[first ? E.ids.x : idT.x] != B.oid[first ? idT.x : E.ids.x]) return false;
    if (!(closest_ee(a0, a1, b0, b1).d < P.filter_d)) return false;
  }
  const unsigned long long pk = ((unsigned long long)(unsigned)e1 << 32) | (unsigned)e2;
  if (B.n_excl_ee && in_sorted(B.excl_ee, B.n_excl_ee, pk)) return false;
  out = make_int2(e1, ~e2);
  return true;
}

// The pairs of slot s with its bucket [r.x, r.y), each pair of the bucket at
// one of its two slots: slot i of n takes the n / 2 that follow it in the
// round, so the lanes' loops are equally long.
template <typename Rec, typename Emit>
__device__ __forceinline__ void edge_round(const Broad& B, const PairCtx& P, const Rec& R, int s, int2 r, Emit&& emit) {
  const EdgeRec E = edge_rec(R, s);
  const int n = r.y - r.x, i = s - r.x, m = (n - 1) / 2 + ((n & 1) == 0 && i < n / 2 ? 1 : 0);
  int t = s;
  for (int u = 0; u < m; ++u) {
    if (++t == r.y) t = r.x;
    int2 pr;
    if (edge_slot_pair_test(B, P, R, E, t, pr)) emit(pr);
  }
}

// Load the edge buckets covering slots [S, S + kBlock) into LDS; returns the
// first slot of the span, or -1 if the span does not fit.
__device__ __forceinline__ int load_span(const Broad& B, SlotSpan& L, long long S, long long E) {
  const int lo = B.range[hash_key(B.bkt_key[S], B.tsize, true)].x;
  const int hi = B.range[hash_key(B.bkt_key[E - 1], B.tsize, true)].y;
  const bool fits = hi - lo <= kSpan;
  if (fits) {
    for (int t = threadIdx.x; t < hi - lo; t += kBlock) {
      L.key[t] = B.bkt_key[lo + t];
      L.item[t] = B.bkt_item[lo + t];
      const int4 id = B.bkt_ids[lo + t];
      L.ids[t] = make_int2(id.x, id.y);
      const double4 a = B.bkt_lo[lo + t], b = B.bkt_hi[lo + t];
      L.lo[0][t] = a.x; L.lo[1][t] = a.y; L.lo[2][t] = a.z;
      L.hi[0][t] = b.x; L.hi[1][t] = b.y; L.hi[2][t] = b.z;
    }
  }
  __syncthreads();
  return fits ? lo : -1;
}

template <typename Emit>
__device__ __forceinline__ void edge_slot_pairs(const Broad& B, const PairCtx& P, const SlotSpan& L, int base, int s,
                                                Emit&& emit) {
  if (base >= 0) edge_pairs(B, P, LdsRec{L, base}, s, emit);
  else edge_pairs(B, P, GlobalRec{B}, s, emit);
}

// Work items: [0, nSV) surface vertices (point-triangle), then the edge slots
// [espan[0], espan[1]) (edge-edge).  part_cnt[w] = pairs of item w;
// every slot below work_cap is written, so no stale count survives.
__global__ void __launch_bounds__(kBlock) k_pairs_count(Broad B, PairCtx P) {
  __shared__ SlotSpan L;
  const long long e0 = B.espan[0], e1 = B.espan[1];
  const long long nw = B.nSV + (e1 - e0);
  // vertices: one wave each
  {
    const long long wid = ((long long)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const long long nwv = ((long long)gridDim.x * kBlock) >> 6;
    for (long long w = wid; w < B.nSV; w += nwv) {
      const int c = vertex_pairs_wave<false>(B, P, (int)w, 0, nullptr, 0);
      if ((threadIdx.x & (kWave - 1)) == 0) B.part_cnt[w] = c;
    }
  }
  // edge slots: a block takes kBlock consecutive slots and their buckets in LDS
  for (long long S = e0 + (long long)blockIdx.x * kBlock; S < e1; S += (long long)gridDim.x * kBlock) {
    const long long s = S + threadIdx.x;
    const int base = load_span(B, L, S, min(S + (long long)kBlock, e1));
    int c = 0;
    if (s < e1) edge_slot_pairs(B, P, L, base, (int)s, [&](int2) { ++c; });
    __syncthreads();
    if (s < e1) B.part_cnt[B.nSV + (s - e0)] = c;
  }
  for (long long w = nw + blockIdx.x * kBlock + threadIdx.x; w < B.work_cap; w += (long long)gridDim.x * kBlock)
    B.part_cnt[w] = 0;
}

__global__ void __launch_bounds__(kBlock) k_pairs_fill(Broad B, PairCtx P, int2* out, long long cap) {
  __shared__ SlotSpan L;
  const long long e0 = B.espan[0], e1 = B.espan[1];
  {
    const long long wid = ((long long)blockIdx.x * kBlock + threadIdx.x) >> 6;
    const long long nwv = ((long long)gridDim.x * kBlock) >> 6;
    for (long long w = wid; w < B.nSV; w += nwv) vertex_pairs_wave<true>(B, P, (int)w, B.part_off[w], out, cap);
  }
  for (long long S = e0 + (long long)blockIdx.x * kBlock; S < e1; S += (long long)gridDim.x * kBlock) {
    const long long s = S + threadIdx.x;
    const int base = load_span(B, L, S, min(S + (long long)kBlock, e1));
    if (s < e1) {
      long long o = B.part_off[B.nSV + (s - e0)];
      edge_slot_pairs(B, P, L, base, (int)s, [&](int2 pr) {
        if (o < cap) out[o] = pr;
        ++o;
      });
    }
    __syncthreads();
  }
}

// Single-pass emission for the solver's list: the pairs that a block finds are
// gathered in LDS and appended at a position reserved with one atomic (40 ns,
// one after the other over the device), in no particular order; the kind is in the pair:
// (v, f) point-triangle, (e1, ~e2) edge-edge.  counter counts every pair
// found, also those past cap (the caller checks it against cap).
constexpr int kEbuf = 2 * kBlock;   // pairs buffered per block before one counter update

// Corner vertices of pair q of the list and their places among the entries of
// each (in no particular order): the index's counting pass, made where the pair
// is found.
__device__ __forceinline__ void pl_corners(const PairIndex& P, int kind, int a, int b, int (&v)[4]);
__device__ __forceinline__ void pl_enter(const PairIndex& P, long long q, int kind, int a, int b) {
  int v[4], at[4];
  pl_corners(P, kind, a, b, v);
  P.pv[q] = make_int4(v[0], v[1], v[2], kind == 0 ? v[3] : ~v[3]);
#pragma unroll
  for (int i = 0; i < 4; ++i) at[i] = atomicAdd(&P.vcnt[v[i]], 1);
  P.place[q] = make_int4(at[0], at[1], at[2], at[3]);
}

__device__ __forceinline__ int block_excl_scan(int v, int& total, int* sh) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x >> 6;
  int wt;
  const int x = wave_excl_scan(v, wt);
  if (lane == 0) sh[w] = wt;
  __syncthreads();
  int before = 0;
  total = 0;
  for (int i = 0; i < kBlock / kWave; ++i) {
    if (i < w) before += sh[i];
    total += sh[i];
  }
  __syncthreads();
  return before + x;
}

// With an index (I.vcnt) the pairs are entered in it.
__global__ void __launch_bounds__(kBlock) k_pairs_emit(Broad B, PairCtx P, int2* out, long long cap,
                                                      unsigned long long* counter, PairIndex I) {
  __shared__ SlotSpan L;
  __shared__ int2 ebuf[kEbuf];
  __shared__ int ecount;
  __shared__ unsigned long long sbase;
  const long long e0 = B.espan[0], e1 = B.espan[1];
  auto put = [&](unsigned long long q, int2 pr) {
    if ((long long)q >= cap) return;
    out[q] = pr;
    if (I.vcnt) pl_enter(I, q, pr.y < 0 ? 1 : 0, pr.x, pr.y < 0 ? ~pr.y : pr.y);
  };
  // the buffered pairs into the list (the whole block)
  auto flush = [&](int n) {
    if (threadIdx.x == 0) {
      sbase = n ? atomicAdd(counter, (unsigned long long)n) : 0ull;
      ecount = 0;
    }
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += kBlock) put(sbase + j, ebuf[j]);
    __syncthreads();
  };
  if (threadIdx.x == 0) ecount = 0;
  __syncthreads();
  auto emit = [&](int2 pr) {
    const int at = atomicAdd(&ecount, 1);
    if (at < kEbuf) ebuf[at] = pr;
    else put(atomicAdd(counter, 1ull), pr);   // a full buffer: by itself
  };
  // point-triangle: kVertLanes lanes per surface vertex, one per bucket slot
  // (most buckets have 10 to 20)
  {
    constexpr int kVertLanes = 16;
    const int lane = threadIdx.x & (kVertLanes - 1);
    const long long w0 = ((long long)blockIdx.x * kBlock + threadIdx.x) / kVertLanes;
    for (long long w = w0; w < B.nSV; w += (long long)gridDim.x * (kBlock / kVertLanes)) {
      const int v = B.surf[w];
      const V3<double> p = ldx(P.x, v);
      const int3 c = cell_of(p, P.inv, B.shift);
      const unsigned long long key = cell_key(c.x, c.y, c.z);
      const int2 sr = B.range[hash_key(key, B.tsize, false)];
      for (int t = sr.x + lane; t < sr.y; t += kVertLanes) {
        int2 pr;
        if (vertex_slot_pair(B, P, v, p, key, t, pr)) emit(pr);
      }
    }
    __syncthreads();
    const int n = min(ecount, kEbuf);
    __syncthreads();
    if (n > kEbuf / 2) flush(n);
  }
  // edge-edge: a block takes kBlock consecutive edge slots with their buckets
  // in LDS, one slot to a thread
  for (long long S = e0 + (long long)blockIdx.x * kBlock; S < e1; S += (long long)gridDim.x * kBlock) {
    const long long s = S + threadIdx.x;
    const int base = load_span(B, L, S, min(S + (long long)kBlock, e1));
    if (s < e1) {
      if (base >= 0) {
        const LdsRec R{L, base};
        edge_round(B, P, R, (int)s, B.range[hash_key(R.key((int)s), B.tsize, true)], emit);
      } else {
        const GlobalRec R{B};
        edge_round(B, P, R, (int)s, B.range[hash_key(R.key((int)s), B.tsize, true)], emit);
      }
    }
    __syncthreads();
    const int n = min(ecount, kEbuf);
    __syncthreads();
    if (n > kEbuf / 2) flush(n);
  }
  const int n = min(ecount, kEbuf);
  __syncthreads();
  if (n) flush(n);
}

// Flags a grid or list that did not fit (the list is then incomplete) and
// records the list size.
__device__ __forceinline__ void list_check(const Broad& B, const long long* ncand, long long cap, int* err,
                                           long long* n_out) {
  if (B.totals[0] > B.ent_cap || ncand[0] > cap) atomicOr(err, kErrCapacity);
  *n_out = ncand[0];
}
__global__ void k_list_check(Broad B, const long long* ncand, long long cap, int* err, long long* n_out) {
  if (threadIdx.x == 0) list_check(B, ncand, cap, err, n_out);
}

// totals[2] = number of point-triangle pairs = offset of the first edge-edge slot
__global__ void k_pt_total(Broad B) {
  if (threadIdx.x == 0 && blockIdx.x == 0) B.totals[2] = B.part_off[B.nSV];
}

__global__ void __launch_bounds__(kBlock) k_plane_cand(Broad B, const double4* x, Planes P, double r, int2* out,
                                                       long long* n, long long cap) {
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < B.nSV; i += gridDim.x * kBlock) {
    const int v = B.surf[i];
    const V3<double> p = ldx(x, v);
    for (int j = 0; j < P.n; ++j) {
      const double* pl = P.p[j];
      double s;
      {
#pragma clang fp contract(off)
        s = ((pl[0] * p.x + pl[1] * p.y) + pl[2] * p.z) - pl[3];
      }
      if (s <= r) {
        unsigned long long slot = atomicAdd((unsigned long long*)n, 1ull);
        if ((long long)slot < cap) out[slot] = make_int2(v, j);
      }
    }
  }
}

// --------------------------------------------- canonical order of a list
// kind (0 point-triangle, 1 edge-edge) and the two indices of pair q
__device__ __forceinline__ void pl_decode(int2 pr, long long q, long long npt, int& kind, int& a, int& b) {
  if (npt >= 0) {
    kind = q < npt ? 0 : 1;
    a = pr.x;
    b = pr.y;
  } else if (pr.y >= 0) {
    kind = 0;
    a = pr.x;
    b = pr.y;
  } else {
    kind = 1;
    a = pr.x;
    b = ~pr.y;
  }
}
// the four vertices in the order the narrow phase uses them
__device__ __forceinline__ void pl_corners(const PairIndex& P, int kind, int a, int b, int (&v)[4]) {
  if (kind == 0) {
    v[0] = a;
    v[1] = P.tris[3 * b];
    v[2] = P.tris[3 * b + 1];
    v[3] = P.tris[3 * b + 2];
  } else {
    v[0] = P.edges[2 * a];
    v[1] = P.edges[2 * a + 1];
    v[2] = P.edges[2 * b];
    v[3] = P.edges[2 * b + 1];
  }
}

__global__ void __launch_bounds__(kBlock) k_pl_zero(PairIndex P) {
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < P.nV; i += gridDim.x * kBlock) P.vcnt[i] = 0;
}

// corner entries per vertex
__global__ void __launch_bounds__(kBlock) k_pl_count(PairIndex P, const int2* list, const long long* ncand,
                                                     long long cap) {
  const long long n = min(ncand[0], cap), npt = ncand[1];
  for (long long q = blockIdx.x * kBlock + threadIdx.x; q < n; q += (long long)gridDim.x * kBlock) {
    int kind, a, b;
    pl_decode(list[q], q, npt, kind, a, b);
    pl_enter(P, q, kind, a, b);
  }
}

// Content key of pair q: kind, then its two indices.  A vertex belongs to a
// pair at most once, so the keys of one vertex's entries are distinct, and
// their order does not depend on the list order.
__device__ __forceinline__ unsigned long long pair_key(int kind, int a, int b) {
  return ((unsigned long long)kind << 62) | ((unsigned long long)(unsigned)a << 31) | (unsigned long long)(unsigned)b;
}

// entries grouped by vertex (slot ids 4 q + corner and their pairs' keys, in
// no particular order within a vertex) and the entry range of each
// incidence wave; given err, also list_check
__global__ void __launch_bounds__(kBlock) k_pl_corners(PairIndex P, const int2* list, const long long* ncand,
                                                       long long cap, Broad B, int* err, long long* n_out) {
  if (err && blockIdx.x == 0 && threadIdx.x == 0) list_check(B, ncand, cap, err, n_out);
  const long long n = min(ncand[0], cap), npt = ncand[1];
  for (long long q = blockIdx.x * kBlock + threadIdx.x; q < n; q += (long long)gridDim.x * kBlock) {
    int kind, a, b;
    pl_decode(list[q], q, npt, kind, a, b);
    const unsigned long long key = pair_key(kind, a, b);
    const int4 w = P.pv[q], pl = P.place[q];
    const int v[4] = {w.x, w.y, w.z, w.w >= 0 ? w.w : ~w.w}, at[4] = {pl.x, pl.y, pl.z, pl.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int pos = P.coff[v[i]] + at[i];
      P.cent_tmp[pos] = (int)(4 * q + i);
      P.ckey_tmp[pos] = key;
    }
  }
  for (int w = blockIdx.x * kBlock + threadIdx.x; w < P.nWaves; w += gridDim.x * kBlock) {
    const int2 fv = P.wvert[w];
    P.wrange[w] = make_int2(P.coff[fv.x], P.coff[fv.y + 1]);
  }
}

// Each vertex's entries [coff[v], coff[v + 1]) of cent_tmp go to the same
// range of cent in ascending key order: every entry is written at its rank
// (the number of smaller keys of the vertex), which depends on the pairs
// only.  A wave per vertex, an entry per lane, the keys it is compared with
// from the lanes or from LDS; the block together where a vertex has more than
// kRankWave.  (A block per vertex with more than 16 entries left most threads
// idle: 65 us for the 460,000 entries of a packed pile, 20 us now.)
constexpr int kRankWave = 256;
constexpr int kRankLds = 1024;   // keys of a vertex staged in LDS

// the entries first, first + step, ... of a vertex, against its keys kk
__device__ __forceinline__ void rank_entries(const PairIndex& P, int s0, int n, const unsigned long long* kk, int first,
                                             int step) {
  for (int i = first; i < n; i += step) {
    const unsigned long long ki = kk[i];
    int r = 0;
#pragma unroll 8
    for (int j = 0; j < n; ++j) r += kk[j] < ki ? 1 : 0;
    P.cent[s0 + r] = P.cent_tmp[s0 + i];
  }
}

__global__ void __launch_bounds__(kBlock) k_rank(PairIndex P) {
  constexpr int kWaves = kBlock / kWave;
  static_assert(kWaves * kRankWave <= kRankLds, "the waves' keys share the block's LDS");
  __shared__ unsigned long long ks[kRankLds];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  for (int base = blockIdx.x * kWaves; base < P.nV; base += gridDim.x * kWaves) {
    int most = 0;
    for (int w = 0; w < kWaves && base + w < P.nV; ++w) most = max(most, P.coff[base + w + 1] - P.coff[base + w]);
    if (most == 0) continue;   // uniform over the block
    const int v = base + wave, s0 = v < P.nV ? P.coff[v] : 0, n = v < P.nV ? P.coff[v + 1] - s0 : 0;
    if (n > 0 && n <= kWave) {
      unsigned long long k = 0;
      if (lane < n) k = P.ckey_tmp[s0 + lane];
      int r = 0;
      for (int j = 0; j < n; ++j) {
        const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)k, j),
                       hi = (unsigned)__builtin_amdgcn_readlane((int)(k >> 32), j);
        r += (((unsigned long long)hi << 32) | lo) < k ? 1 : 0;
      }
      if (lane < n) P.cent[s0 + r] = P.cent_tmp[s0 + lane];
    } else if (n > kWave && n <= kRankWave) {
      unsigned long long* kk = ks + wave * kRankWave;
      for (int i = lane; i < n; i += kWave) kk[i] = P.ckey_tmp[s0 + i];
      __threadfence_block();
      rank_entries(P, s0, n, kk, lane, kWave);
    }
    if (most <= kRankWave) continue;
    for (int w = 0; w < kWaves && base + w < P.nV; ++w) {
      const int b0 = P.coff[base + w], bn = P.coff[base + w + 1] - b0;
      if (bn <= kRankWave) continue;
      __syncthreads();
      if (bn <= kRankLds)
        for (int i = threadIdx.x; i < bn; i += kBlock) ks[i] = P.ckey_tmp[b0 + i];
      __syncthreads();
      rank_entries(P, b0, bn, bn <= kRankLds ? ks : P.ckey_tmp + b0, threadIdx.x, kBlock);
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kBlock) k_pl_install(const int2* src, long long n, int2* out, long long* ncand,
                                                       long long* n_out) {
  for (long long q = blockIdx.x * kBlock + threadIdx.x; q < n; q += (long long)gridDim.x * kBlock) out[q] = src[q];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ncand[0] = n;
    ncand[1] = -1;
    *n_out = n;
  }
}

}  // namespace

// `entered`: the pairs were entered as they were found (broad_solver_list), and
// err and n_out are to be set.
void pairs_index(const PairIndex& P, const int2* list, const long long* ncand, long long cap, hipStream_t s,
                 bool entered, const Broad* B, int* err, long long* n_out) {
  if (!entered) {
    hipLaunchKernelGGL(k_pl_zero, dim3(P.grid), dim3(kBlock), 0, s, P);
    hipLaunchKernelGGL(k_pl_count, dim3(P.grid), dim3(kBlock), 0, s, P, list, ncand, cap);
  }
  scan_exclusive<int>(P.vcnt, P.nV, P.coff, P.coff + P.nV, P.scan_tmp, s);
  hipLaunchKernelGGL(k_pl_corners, dim3(P.grid), dim3(kBlock), 0, s, P, list, ncand, cap, B ? *B : Broad{}, err, n_out);
  hipLaunchKernelGGL(k_rank, dim3(std::max(1, std::min((P.nV + 3) / 4, 2048))), dim3(kBlock), 0, s, P);
}

__global__ void __launch_bounds__(kBlock) k_copy_positions(double4* dst, const double4* src, int n) {
  for (int v = blockIdx.x * kBlock + threadIdx.x; v < n; v += gridDim.x * kBlock) dst[v] = src[v];
}

void copy_positions(double4* dst, const double4* src, int n, hipStream_t s) {
  const int g = std::min((n + kBlock - 1) / kBlock, 1024);
  hipLaunchKernelGGL(k_copy_positions, dim3(std::max(g, 1)), dim3(kBlock), 0, s, dst, src, n);
}

void pairs_install(const int2* src, long long n, int2* out, long long* ncand, long long* n_out, hipStream_t s) {
  const int g = (int)std::min<long long>(std::max<long long>((n + kBlock - 1) / kBlock, 1), 1024);
  hipLaunchKernelGGL(k_pl_install, dim3(g), dim3(kBlock), 0, s, src, n, out, ncand, n_out);
}

// the grid at positions x
static void build_grid(const Broad& B, const double4* x, double cell, double r, long long* ncand, int* vcnt,
                       double4* xbuild, hipStream_t s) {
  const double inv = 1.0 / cell;
  const int n = B.nF + B.nE, tile = std::min(kBucketsPer * kBlock, B.tsize / 2);
  hipLaunchKernelGGL(k_items, dim3(std::max(1, (n + kItems - 1) / kItems)), dim3(kItemBlock), 0, s, B, x, inv, r, ncand);
  hipLaunchKernelGGL(k_bucket_alloc, dim3(B.tsize / tile), dim3(kBlock), 0, s, B, tile);
  const int nb = std::max(1, std::min((n + kBlock / kItemLanes - 1) / (kBlock / kItemLanes), 2048));
  hipLaunchKernelGGL(k_bucket_fill, dim3(nb), dim3(kBlock), 0, s, B, x, inv, r, vcnt, xbuild);
}

void broad_build_count(const Broad& B, const double4* x, double cell, double r, double filter_d, int filter_obj,
                       hipStream_t s) {
  build_grid(B, x, cell, r, nullptr, nullptr, nullptr, s);
  PairCtx P{x, 1.0 / cell, r, filter_d, filter_obj};
  const int nb = (int)std::min<long long>((B.ent_cap + kBlock - 1) / kBlock, 8192);
  hipLaunchKernelGGL(k_pairs_count, dim3(nb), dim3(kBlock), 0, s, B, P);
  scan_exclusive<long long>(B.part_cnt, B.work_cap, B.part_off, B.totals + 1, B.part_off + B.work_cap, s);
  hipLaunchKernelGGL(k_pt_total, dim3(1), dim3(64), 0, s, B);
}

void broad_fill(const Broad& B, const double4* x, double cell, double r, double filter_d, int filter_obj, int2* out,
                long long cap, hipStream_t s) {
  PairCtx P{x, 1.0 / cell, r, filter_d, filter_obj};
  const int nb = (int)std::min<long long>((B.ent_cap + kBlock - 1) / kBlock, 8192);
  hipLaunchKernelGGL(k_pairs_fill, dim3(nb), dim3(kBlock), 0, s, B, P, out, cap);
}

void broad_solver_list(const Broad& B, const double4* x, double cell, double r, int2* out, long long cap,
                       long long* ncand, int* err, long long* n_out, hipStream_t s, const PairIndex* P,
                       double4* xbuild) {
  build_grid(B, x, cell, r, ncand, P ? P->vcnt : nullptr, xbuild, s);
  PairCtx PC{x, 1.0 / cell, r, r, 0};
  // four blocks fit a compute unit; more would only add updates of the counter
  const int nb = (int)std::min<long long>((B.ent_cap + kBlock - 1) / kBlock, 1024);
  hipLaunchKernelGGL(k_pairs_emit, dim3(nb), dim3(kBlock), 0, s, B, PC, out, cap, (unsigned long long*)ncand,
                     P ? *P : PairIndex{});
  if (P) pairs_index(*P, out, ncand, cap, s, true, &B, err, n_out);
  else hipLaunchKernelGGL(k_list_check, dim3(1), dim3(64), 0, s, B, (const long long*)ncand, cap, err, n_out);
}

void plane_candidates(const Broad& B, const double4* x, const Planes& planes, double r, int2* out, long long* n,
                      long long cap, hipStream_t s) {
  (void)hipMemsetAsync(n, 0, sizeof(long long), s);
  hipLaunchKernelGGL(k_plane_cand, dim3(B.grid), dim3(kBlock), 0, s, B, x, planes, r, out, n, cap);
}

}  // namespace pncg
