// Host-built tables of the persistent iteration kernel (persist.h): each
// block's vertices, tets and incidence lanes by local number, the chunks its
// element terms are formed in, and the layout of its LDS.
#include <algorithm>
#include <cstdlib>
#include <memory>
#include <new>
#include <system_error>
#include <thread>

#include "persist.h"

namespace pncg {

namespace {

// Slice L of n items over the grid's logical blocks (block_slice).
void slice(long long n, int grid, int L, int& b, int& e) {
  const long long per = (n + grid - 1) / grid;
  b = (int)std::min<long long>(L * per, n);
  e = (int)std::min<long long>((L + 1) * per, n);
}

// f(worker, block) for every block, by a few threads where there is enough
// work, each taking consecutive ones, whose counters share cache lines (f must
// not throw); the calling thread alone if none can be started.
template <typename F>
void for_blocks(int blocks, int workers, F&& f) {
  std::vector<std::thread> ts;
  auto part = [&](int w) {
    for (int p = (int)((long long)blocks * w / workers); p < (int)((long long)blocks * (w + 1) / workers); ++p) f(w, p);
  };
  int started = 1;
  try {
    ts.reserve(workers);
    for (; started < workers; ++started) ts.emplace_back(part, started);
  } catch (...) {
  }
  part(0);
  for (int w = started; w < workers; ++w) part(w);
  for (auto& t : ts) t.join();
}

// The lists of all blocks: block p's start at off[p], with room for an upper
// bound of them, until close() moves them together.  (The time goes to first
// touches of pages, so there are neither lists of their own nor copies.)
template <typename T_>
struct Lists {
  std::vector<size_t> off;
  std::vector<int> n;
  std::unique_ptr<T_[]> d;
  explicit Lists(int blocks) : off(blocks + 1, 0), n(blocks, 0) {}
  void room(int p, size_t cap) { off[p + 1] = off[p] + cap; }   // in block order
  void open() { d.reset(new T_[off.back() + 1]); }
  T_* at(int p) { return d.get() + off[p]; }
  int add(int p, const T_& v) {
    d[off[p] + n[p]] = v;
    return n[p]++;
  }
  void close(PersistTable<T_>& out) {
    size_t to = 0;
    for (int p = 0; p < (int)n.size(); ++p) {
      std::copy(at(p), at(p) + n[p], d.get() + to);   // to lower addresses
      to += n[p];
    }
    out.d = std::move(d);
    out.n = to;
  }
};

// Local numbers of a block's vertices or tets by their global ones.  The pages
// that no block of the worker comes to are never touched.
struct Numbers {
  struct Slot {
    int block, local;   // block + 1 that numbered it last, its number there
  };
  std::unique_ptr<Slot, decltype(&std::free)> slot;
  explicit Numbers(size_t n) : slot(static_cast<Slot*>(std::calloc(n, sizeof(Slot))), &std::free) {
    if (!slot) throw std::bad_alloc();
  }
};

}  // namespace

bool persist_build(int nV, int nT, const int* tets, const std::vector<int>& inc, const std::vector<int>& inc_vert,
                   int grid, bool fp64, bool self, int who, PersistTables& T) {
  const int nWaves = (int)(inc.size() / kWave);
  T = PersistTables{};
  PersistArgs P{};
  P.grid = grid;
  P.vb = grid > 256 ? 2 : 1;
  P.blocks = grid / P.vb;
  P.chunks = 1;
  const int blocks = P.blocks;
  const unsigned real = fp64 ? 8 : 4;
  // a share of the mesh that cannot fit even without its neighbours
  if ((size_t)(nV / blocks) * (104 + 12 * real) + (size_t)(nT / blocks) * 12 > kPersistLds) return false;
  // the tables of 4000 tets take about half a millisecond on one core
  const int workers = std::min({blocks, 1 + nT / 4000, 8});
  T.blk.resize(blocks);
  T.lane.resize(inc.size());
  T.run.resize(nV);
  T.wave_last.resize(nWaves);
  T.dtet.resize(nT);
  T.dvert.resize(nV);
  Lists<int> loc_v(blocks), tet_e(blocks);
  Lists<ushort4> tet_l(blocks);
  struct Marks {
    Numbers v, t;
    std::vector<int> entry;     // entry of each local tet
  };
  std::vector<Marks> marks;
  marks.reserve(workers);
  auto add_marks = [&] { marks.push_back(Marks{Numbers(nV), Numbers(nT), std::vector<int>()}); };
  add_marks();
  for (int p = 0; p < blocks; ++p) {
    PersistBlock& B = T.blk[p];
    int b0, e0, b1, e1;
    slice(nWaves, grid, p * P.vb, b0, e0);
    slice(nWaves, grid, p * P.vb + P.vb - 1, b1, e1);
    B.w0 = b0; B.nw = e1 - b0;
    slice(nT, grid, p * P.vb, b0, e0);
    slice(nT, grid, p * P.vb + P.vb - 1, b1, e1);
    B.t0 = b0; B.nt = e1 - b0;
    slice(nV, grid, p * P.vb, b0, e0);
    slice(nV, grid, p * P.vb + P.vb - 1, b1, e1);
    B.v0 = b0; B.nv = e1 - b0;
    const size_t most = std::min<size_t>((size_t)B.nw * kWave + B.nt, nT);
    tet_e.room(p, most);
    tet_l.room(p, most);
    loc_v.room(p, std::min<size_t>(4 * most + (size_t)B.nw * kWave + B.nv, nV));
  }
  loc_v.open();
  tet_e.open();
  tet_l.open();
  auto number = [&](int wk, int p) {
    PersistBlock& B = T.blk[p];
    Numbers::Slot *kv = marks[wk].v.slot.get(), *kt = marks[wk].t.slot.get();
    auto vertex = [&](int v) {
      if (kv[v].block != p + 1) kv[v] = {p + 1, loc_v.add(p, v)};
      return kv[v].local;
    };
    auto tet = [&](int e) {
      if (kt[e].block != p + 1) {
        kt[e] = {p + 1, tet_e.add(p, e)};
        ushort4 c;
        c.x = (unsigned short)vertex(tets[4 * e]);
        c.y = (unsigned short)vertex(tets[4 * e + 1]);
        c.z = (unsigned short)vertex(tets[4 * e + 2]);
        c.w = (unsigned short)vertex(tets[4 * e + 3]);
        tet_l.add(p, c);
      }
      return kt[e].local;
    };
    const size_t i0 = (size_t)B.w0 * kWave, i1 = i0 + (size_t)B.nw * kWave;
    // own vertices: those of the block's incidence waves, consecutive
    for (size_t i = i0; i < i1; ++i)
      if (inc_vert[i] >= 0) vertex(inc_vert[i]);
    B.nown = loc_v.n[p];
    for (size_t i = i0; i < i1; ++i) {
      ushort2 l = make_ushort2(kNone, kLaneVert);
      ulonglong2& w = T.wave_last.d[i / kWave];
      const int bit = (int)(i % kWave), v = inc_vert[i];
      if (bit == 0) w = make_ulonglong2(0, 0);
      if (v >= 0) {
        // a vertex's lanes are consecutive and within one wave
        const bool last = bit == kWave - 1 || inc_vert[i + 1] != v;
        const int lv = vertex(v);
        l.y = (unsigned short)(lv | (last ? kLaneLast : 0));
        if (last) {
          if (!w.x) w.y = (unsigned long long)lv;
          w.x |= 1ull << bit;
        }
      }
      if (inc[i] >= 0) l.x = (unsigned short)(tet(inc[i] >> 2) << 2 | (inc[i] & 3));
      T.lane.d[i] = l;
    }
    for (int e = B.t0; e < B.t0 + B.nt; ++e) T.dtet.d[e] = (unsigned short)tet(e);
    for (int v = B.v0; v < B.v0 + B.nv; ++v) T.dvert[v] = (unsigned short)vertex(v);
    B.nloc = loc_v.n[p];
    B.ntet = tet_e.n[p];
  };
  size_t cap_loc = 0, cap_own = 0, cap_tet = 0, cap_w = 0, cap_dt = 0, cap_dv = 0, nl = 0, nt = 0;
  auto caps = [&](const PersistBlock& B) {
    cap_loc = std::max<size_t>(cap_loc, B.nloc);
    cap_own = std::max<size_t>(cap_own, B.nown);
    cap_tet = std::max<size_t>(cap_tet, B.ntet);
    cap_w = std::max<size_t>(cap_w, B.nw);
    cap_dt = std::max<size_t>(cap_dt, B.nt);
    cap_dv = std::max<size_t>(cap_dv, B.nv);
  };
  // LDS of a block: by tet in `chunks` chunks, or by lane (chunks = 0); the
  // element records in it or not.  True if it fits.
  auto layout = [&](PersistArgs& A, int chunks, int in_lds, int pairs) {
    size_t o = 0;
    auto put = [&](unsigned& f, size_t bytes, size_t align) {
      o = (o + align - 1) / align * align;
      f = (unsigned)o;
      o += bytes;
    };
    // a vertex starts a row run, and each row boundary of a wave at most another
    const size_t cap_seg = cap_own + 3 * cap_w;
    const size_t cw = chunks ? (cap_w + chunks - 1) / chunks : 0;
    PersistLayout& L = A.at;
    put(L.rec, in_lds ? kRec * real * cap_tet : 0, 16);
    put(L.wm, 16 * cap_w, 16);
    put(L.x, 24 * cap_loc, 8);
    put(L.m, 8 * cap_loc, 8);
    put(L.xt, 24 * cap_own, 8);
    put(L.xb, self ? 24 * cap_own : 0, 8);
    put(L.P, 24 * cap_own, 8);
    put(L.res, 6 * real * cw * kWave, 8);
    put(L.tot, 6 * real * (chunks ? cap_seg : cap_own), 8);
    put(L.p, 3 * real * cap_loc, 8);
    put(L.pg, 3 * real * cap_loc, 8);
    put(L.g, 6 * real * cap_own, 8);
    put(L.tl, 8 * cap_tet, 8);
    put(L.te, in_lds ? 0 : 4 * cap_tet, 4);
    put(L.hv, 4 * cap_loc, 4);
    put(L.ce, self ? 8 * cap_own : 0, 4);
    put(L.run, chunks ? 4 * cap_own : 0, 4);
    put(L.seg, chunks ? 4 * cap_seg : 0, 4);
    put(L.lane, chunks ? 0 : 4 * cap_w * kWave, 4);
    put(L.dt, 2 * cap_dt, 2);
    put(L.dv, 2 * cap_dv, 2);
    put(L.fl, cap_loc, 1);
    // what the pair terms keep here if there is room
    A.cap_rp = A.cap_dg = 0;
    if (self && pairs) {
      put(L.rp, 48 * (size_t)kRunPartials, 8);
      put(L.dg, kPairGeom * kWave * (size_t)P.vb, 8);
      A.cap_rp = kRunPartials;
      A.cap_dg = kWave;
    }
    A.elem_lds = in_lds;
    A.lds = o;
    return o <= kPersistLds && cw * kWave < kNone;
  };
  int done = 0;
  // The block with the most vertices alone tells most meshes that are too large.
  {
    int most = 0, at = 0;
    for (int p = 0; p < blocks; ++p) {
      const PersistBlock& B = T.blk[p];
      // (its vertices are consecutive: the first lane's to the last one's that has any)
      size_t i = (size_t)B.w0 * kWave, j = i + (size_t)B.nw * kWave;
      while (i < j && inc_vert[i] < 0) ++i;
      while (i < j && inc_vert[j - 1] < 0) --j;
      const int own = i < j ? inc_vert[j - 1] - inc_vert[i] + 1 : 0;
      if (own > most) most = own, at = p;
    }
    number(0, at);
    caps(T.blk[at]);
    PersistArgs A = P;
    if (!layout(A, who == kForAdjoint ? kMaxChunks : who == 0 ? kStepChunks : 0, 0, 0)) return false;
    done = at;
  }
  while ((int)marks.size() < workers) add_marks();
  for_blocks(blocks, workers, [&](int wk, int p) {
    if (p != done) number(wk, p);
  });
  for (PersistBlock& B : T.blk) {
    B.loc_off = (int)nl;
    B.tet_off = (int)nt;
    nl += B.nloc;
    nt += B.ntet;
    caps(B);
  }
  // 16-bit local numbers; a lane's words also hold the corner (two bits) and the last-lane mark
  if (cap_loc >= kLaneVert || cap_tet >= (kNone >> 2)) return false;
  P.cap_own = (int)cap_own;

  T.form[0] = T.form[1] = P;
  // one pass over the waves before the records in LDS, then as few chunks as fit
  static const int order[][2] = {{1, 1}, {2, 1}, {1, 0}, {2, 0}, {3, 0}, {4, 0}, {kStepChunks, 0}, {kMaxChunks, 0}};
  bool by_tet = false;
  for (const auto& t : order)
    if (!by_tet && (layout(T.form[0], t[0], t[1], 1) || layout(T.form[0], t[0], t[1], 0))) {
      T.form[0].chunks = t[0];
      by_tet = true;
    }
  T.ok[0] = by_tet && T.form[0].chunks <= kStepChunks;
  for (int in_lds = 1; in_lds >= 0 && !T.ok[1]; --in_lds)
    T.ok[1] = layout(T.form[1], 0, in_lds, 1) || layout(T.form[1], 0, in_lds, 0);

  // the chunks' tets
  const int nc = T.form[0].chunks;
  if (by_tet && fp64) {
    size_t o = 0;
    auto put = [&](unsigned& f, size_t bytes, size_t align) {
      o = (o + align - 1) / align * align;
      f = (unsigned)o;
      o += bytes;
    };
    const size_t cap_seg = cap_own + 3 * cap_w, cw = (cap_w + nc - 1) / nc;
    CgLayout& L = T.cg.at;
    put(L.wm, 16 * cap_w, 16);
    put(L.x, 24 * cap_loc, 8);
    put(L.z, 24 * cap_loc, 8);
    put(L.p, 24 * cap_loc, 8);
    put(L.w, 24 * cap_loc, 8);
    put(L.q, 24 * cap_own, 8);
    put(L.diag, 24 * cap_own, 8);
    put(L.lam, 24 * cap_own, 8);
    put(L.m, 8 * cap_own, 8);
    put(L.res, 24 * cw * kWave, 8);
    put(L.tot, 24 * cap_seg, 8);
    put(L.tl, 8 * cap_tet, 8);
    put(L.hv, 4 * cap_loc, 4);
    put(L.seg, 4 * cap_seg, 4);
    put(L.run, 4 * cap_own, 4);
    put(L.fl, cap_own, 1);
    T.cg.lds = o;
    T.cg_ok = o <= kCgLds;
  }
  if (!(who == kForAdjoint ? T.cg_ok : T.ok[who])) return false;
  Lists<PersistEntry> entry(blocks);
  Lists<ushort2> seg(blocks);
  std::vector<int4> chunk((size_t)blocks * (nc + 1), make_int4(0, 0, 0, 0));
  if (T.ok[0] || T.cg_ok) {
    for (int p = 0; p < blocks; ++p) {
      entry.room(p, std::min<size_t>((size_t)T.blk[p].nw * kWave, (size_t)T.blk[p].ntet * nc));
      seg.room(p, T.blk[p].nown + 3 * (size_t)T.blk[p].nw);
    }
    entry.open();
    seg.open();
    for (Marks& m : marks) m.entry.resize(cap_tet);
    for_blocks(blocks, workers, [&](int wk, int p) {
      Marks& K = marks[wk];
      const PersistBlock& B = T.blk[p];
      PersistEntry* en = entry.at(p);
      ushort2* sg = seg.at(p);
      int4* ch = &chunk[(size_t)p * (nc + 1)];
      const int cw = (B.nw + nc - 1) / nc;
      int own = 0, ne = 0, ns = 0;
      std::fill(K.entry.begin(), K.entry.begin() + B.ntet, -1);
      for (int c = 0; c < nc; ++c) {
        const int wb = std::min(c * cw, B.nw), we = std::min(wb + cw, B.nw);
        const size_t i0 = (size_t)(B.w0 + wb) * kWave, i1 = (size_t)(B.w0 + we) * kWave;
        const int e0 = ne;
        ch[c] = make_int4(e0, own, ns, 0);
        for (size_t i = i0; i < i1; ++i) {
          const ushort2 l = T.lane.d[i];
          const int s = (int)(i - i0), lv = l.y & kLaneVert;
          if (lv != kLaneVert) {
            ushort2& run = T.run[loc_v.at(p)[lv]];
            if (lv >= own) {   // the vertex's first lane
              own = lv + 1;
              run = make_ushort2((unsigned short)ns, 0);
            }
            if (l.x != kNone) {
              if (run.y == 0 || s % 16 == 0) {
                sg[ns++] = make_ushort2((unsigned short)s, 0);
                ++run.y;
              } else {
                ++sg[ns - 1].x;
                ++sg[ns - 1].y;
              }
            }
          }
          if (l.x == kNone) continue;
          const int t = l.x >> 2;
          if (K.entry[t] < e0) {
            K.entry[t] = ne;
            en[ne++] = PersistEntry{{kNone, kNone, kNone, kNone}, (unsigned short)t, 0};
          }
          en[K.entry[t]].slot[l.x & 3] = (unsigned short)s;
        }
      }
      ch[nc] = make_int4(ne, own, ns, 0);
      entry.n[p] = ne;
      seg.n[p] = ns;
    });
    int e0 = 0, s0 = 0;
    for (int p = 0; p < blocks; ++p) {
      for (int c = 0; c <= nc; ++c) {
        int4& ch = chunk[(size_t)p * (nc + 1) + c];
        ch.x += e0;
        ch.w = s0;
      }
      e0 += entry.n[p];
      s0 += seg.n[p];
    }
  }
  for (size_t i = 0; i < chunk.size(); ++i)
    if (i % (nc + 1) != (size_t)nc) T.cg.most = std::max(T.cg.most, chunk[i + 1].x - chunk[i].x);
  T.chunk.swap(chunk);
  entry.close(T.entry);
  seg.close(T.seg);
  loc_v.close(T.loc_v);
  T.loc_v.d[T.loc_v.n++] = 0;   // a block without vertices reads its first one
  tet_e.close(T.tet_e);
  tet_l.close(T.tet_l);
  return true;
}

}  // namespace pncg
