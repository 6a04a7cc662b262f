// Row plan of the damage passes: the damage operator's rows by node, for
// workgroups that own a compact run of nodes and keep rings of their
// neighbours (pf_internal.hpp: RowTile, DevRows).  Host code, run once per
// handle.
#include <algorithm>
#include <atomic>
#include <new>
#include <numeric>
#include <thread>

#include "pf_internal.hpp"

namespace pf {

namespace {

// Owned nodes per row tile and the default preconditioner's degree, per
// instance and from the instance alone, so that a batched handle gives each
// instance the tiles, and the bits, of a handle of its own.
//
// A pass of degree k costs k + 1 products on a tile and its shrinking rings,
// and one crossing of the chip for the reductions.  With few tiles per XCD the
// crossing and the memory's latency are most of it, so a high degree and small
// tiles (few serial rows per thread) win although half of a tile's rows are
// then rings; on more nodes the rings' rows cost time of their own.  256 owned
// nodes are one per thread: more of them need registers for a second node's
// vectors.  Measured as degree / owned nodes, us per step of two plates of
// each size:
//   FP64    64x32  8/128 228, 212   6/160 248, 221
//          397x211 8/128 302, 408   6/160 320, 434   6/256 320, 471
//          512x256 8/192 573, 630   6/256 558, 593   5/256 558, 624   6/384 599, 670
//         1024x512 8/192 937, 1042  6/256 752, 865   5/256 778, 889   6/384 779, 921
//   FP32   256x128 8/128 164, 202   6/256 174, 223   4/256 199, 230
//          512x256 8/128 317, 277   6/256 252, 238   4/256 264, 255   6/384 281, 270
//         1024x512 8/128 445, 441   6/256 354, 342   4/256 390, 325   6/384 375, 363
// 8/128 suits a small FP32 plate by itself, but a batch of 16 plates of up to
// 512x256 takes 599 at 6/256 and 660 with 128 owned nodes on its smaller ones,
// and both have to get the same tiles: 6/256 costs the single plate 6 to 10 %.
//
// On a million nodes the set-up pass, which assembles a tile's ring rows too, is
// much of a step with few free nodes, and larger tiles have the fewest.  FP32,
// us per polled step at 6/256 and at 3/704, of an AT2 plate (regular, random
// diagonals) and of AT1 plates whose damage hardly moves:
//   534k nodes 275 / 277, 310 / 314   AT1 119 / 129, 135 / 112
//   702k       333 / 370, 369 / 439       150 / 160, 165 / 148
//   836k       379 / 399, 416 / 477       167 / 146, 155 / 177
//   877k       382 / 410, 431 / 494       163 / 137, 217 / 174
//   1.05M      441 / 453, 509 / 545       181 / 158, 235 / 177   perforated 226 / 187
//   2.1M       865 / 773, 983 / 1034      337 / 302, 405 / 315
// The line at 768k nodes is where the AT1 plates begin to gain (up to 25 %); AT2
// plates up to a million nodes pay 3 to 15 % for it.
//
// Callers that ask for tiles of less than 128 nodes get them, and degree 2:
// the rings of a higher one would outnumber their nodes.
struct RowChoice {
  size_t own;
  int degree;
};
RowChoice row_choice(size_t n, size_t tile_nodes, size_t width) {
  const bool dbl = width == 8;
  if (tile_nodes < 128) return {tile_nodes, 2};
  if (dbl && n <= 100000) return {128, 8};
  if (dbl || n <= 768 * 1024) return {256, 6};
  return {704, 3};
}

constexpr size_t kThreads = 8;
// f(i, t) for i < n, t < kThreads the thread that runs it
template <typename F>
void parallel_for(size_t n, const F& f) {
  const size_t nt = std::min<size_t>({kThreads, std::max<unsigned>(1, std::thread::hardware_concurrency()), n / 16 + 1});
  std::atomic<size_t> next{0};
  std::atomic<bool> out_of_memory{false};
  auto work = [&](size_t t) {
    try {
      for (;;) {
        const size_t b = next.fetch_add(16);
        if (b >= n) return;
        for (size_t i = b; i < std::min(n, b + 16); ++i) f(i, t);
      }
    } catch (const std::bad_alloc&) {
      out_of_memory = true;   // thrown again below, on the caller's thread
    }
  };
  std::vector<std::thread> pool;
  try {
    for (size_t t = 1; t < nt; ++t) pool.emplace_back(work, t);
  } catch (...) {   // no more threads: the ones there are do the work
  }
  work(0);
  for (auto& t : pool) t.join();
  if (out_of_memory) throw std::bad_alloc();
}

// The entries of every node's row, by neighbour (row order), each with the
// element it stands for (c0) and the other element at the pair (c1), as 3 e +
// edge with e the internal element id, or kNone.  An element stands at each of
// its nodes for the neighbour that follows in its counter-clockwise order.
// Rows are in ascending order of c0 (entries without one last).
constexpr uint32_t kNone = 0xffffffffu;
struct Graph {
  std::vector<int64_t> ptr;
  std::vector<int32_t> nbr;
  std::vector<uint32_t> c0, c1;
};

Graph build_graph(const RowMesh& rm, const std::vector<int32_t>& dloc) {
  const size_t n = size_t(rm.n), ne = size_t(rm.ne);
  std::vector<int64_t> start(n + 1, 0);
  for (size_t i = 0; i < 3 * ne; ++i) start[size_t(dloc[rm.tri[i]]) + 1] += 2;
  for (size_t i = 0; i < n; ++i) start[i + 1] += start[i];
  struct Entry { int32_t nbr; uint32_t code; bool own; };
  std::vector<Entry> ent(6 * ne);
  {
    std::vector<int64_t> at(start.begin(), start.end() - 1);
    for (size_t j = 0; j < ne; ++j) {   // ascending internal element id: a fixed order within every pair
      const int32_t* t = rm.tri + 3 * size_t(rm.eorder[j]);
      const int32_t v[3] = {dloc[t[0]], dloc[t[1]], dloc[t[2]]};
      const uint32_t base = 3u * uint32_t(j);
      const uint32_t edge[3] = {0, 2, 1};   // edges 01, 12, 20
      for (int q = 0; q < 3; ++q) {
        ent[size_t(at[v[q]]++)] = {v[(q + 1) % 3], base + edge[q], true};
        ent[size_t(at[v[(q + 1) % 3]]++)] = {v[q], base + edge[q], false};
      }
    }
  }
  struct Slot { int32_t nbr; uint32_t c0, c1; };
  // slots of node i, appended to out
  auto slots = [&](size_t i, std::vector<Slot>& out) {
    Entry* lo = ent.data() + start[i];
    Entry* hi = ent.data() + start[i + 1];
    std::stable_sort(lo, hi, [](const Entry& x, const Entry& y) { return x.nbr < y.nbr; });
    for (Entry* a = lo; a < hi;) {
      Entry* b = a;
      while (b < hi && b->nbr == a->nbr) ++b;
      Entry *o = a, *p = a;   // the next of each kind
      for (;;) {
        while (o < b && !o->own) ++o;
        while (p < b && p->own) ++p;
        if (o == b && p == b) break;
        out.push_back({a->nbr, o < b ? (o++)->code : kNone, p < b ? (p++)->code : kNone});
      }
      a = b;
    }
    std::stable_sort(out.begin(), out.end(), [](const Slot& x, const Slot& y) { return x.c0 < y.c0; });
  };
  const size_t blocks = (n + 1023) / 1024;
  std::vector<std::vector<Slot>> all(blocks);
  std::vector<int32_t> cnt(n, 0);
  parallel_for(blocks, [&](size_t blk, size_t) {
    std::vector<Slot> row;
    all[blk].reserve(1024 * 7);
    for (size_t i = blk * 1024; i < std::min(n, (blk + 1) * 1024); ++i) {
      row.clear();
      slots(i, row);
      cnt[i] = int32_t(row.size());
      all[blk].insert(all[blk].end(), row.begin(), row.end());
    }
  });
  Graph g;
  g.ptr.assign(n + 1, 0);
  for (size_t i = 0; i < n; ++i) g.ptr[i + 1] = g.ptr[i] + cnt[i];
  g.nbr.resize(size_t(g.ptr[n]));
  g.c0.resize(g.nbr.size());
  g.c1.resize(g.nbr.size());
  parallel_for(blocks, [&](size_t blk, size_t) {
    size_t o = size_t(g.ptr[blk * 1024]);
    for (const Slot& q : all[blk]) g.nbr[o] = q.nbr, g.c0[o] = q.c0, g.c1[o] = q.c1, ++o;
  });
  return g;
}

struct HostTile {
  int32_t lo, hi;                  // owned nodes, row order
  int32_t nl[kMaxRing + 1];
  int32_t rings;                   // complete rings
  std::vector<int32_t> ring;       // ring nodes, ring by ring
  std::vector<int32_t> xcount;     // extra pairs of each slice
  std::vector<int32_t> elems;      // internal ids of the elements at its nodes, ring by ring
  int32_t nel[kMaxRing];
};

}  // namespace

bool row_plan_add(RowPlan& rp, const RowMesh& rm, int inst, size_t width, size_t lds_limit) {
  const size_t n = size_t(rm.n);
  const size_t static_lds = 2048;   // the passes' reduction scratch
  const size_t max1 = std::min<size_t>(65535, (lds_limit - static_lds) / 8);            // nodes, one FP64 vector in LDS
  const size_t max2 = std::min<size_t>(kRowMax + kBlock, (lds_limit - static_lds) / (2 * width));  // nodes, two vectors
  const RowChoice choice = row_choice(n, rm.tile_nodes, width);
  const size_t own = choice.own;
  const int ddef = choice.degree, ask = std::max(kAskRing, ddef);
  std::vector<int32_t> dloc(n);
  std::vector<HostTile> tiles;
  Graph g;
  int dmax = 0;
  std::vector<std::vector<int32_t>> scratch(kThreads);   // per thread: the tile's local id of an element, or -1
  // the second plan takes the handle's own tiles, for meshes on which a run of
  // `own` nodes has too many neighbours for the LDS (hubs of thousands of them
  // side by side) and a smaller one has not; what the explicit step's tiles may
  // hold, which pf_mesh_create checks later, always fits here
  for (int plan = 0; plan < 2 && dmax < 1; ++plan) {
    std::vector<std::pair<size_t, size_t>> leaves;
    if (plan == 0) {
      std::vector<int32_t> ids(n);
      std::iota(ids.begin(), ids.end(), 0);
      rcb(ids, 0, n, rm.xy, own, leaves);
      int32_t p = 0;
      for (auto& l : leaves) {
        std::sort(ids.begin() + l.first, ids.begin() + l.second);
        for (size_t i = l.first; i < l.second; ++i) dloc[ids[i]] = p++;
      }
    } else {
      leaves = *rm.leaves;
      for (size_t i = 0; i < n; ++i) dloc[i] = rm.node_int[i];
    }
    g = build_graph(rm, dloc);
    tiles.assign(leaves.size(), HostTile());
    parallel_for(tiles.size(), [&](size_t ti, size_t th) {
      HostTile& t = tiles[ti];
      std::vector<int32_t>& mark = scratch[th];
      if (mark.empty()) mark.assign(size_t(rm.ne), -1);
      t.lo = int32_t(leaves[ti].first);
      t.hi = int32_t(leaves[ti].second);
      t.nl[0] = t.hi - t.lo;
      t.rings = 0;
      // ring k: unseen neighbours of ring k-1 (of the owned nodes for k = 1).  A
      // neighbour of ring k-1 lies in ring k-2, k-1 or k, so those are all to
      // look through
      std::vector<int32_t> prev2, prev, cur;
      for (int k = 1; k <= ask; ++k) {
        cur.clear();
        auto grow = [&](int32_t u) {
          for (int64_t q = g.ptr[u]; q < g.ptr[u + 1]; ++q) {
            const int32_t v = g.nbr[size_t(q)];
            if (v < t.lo || v >= t.hi) cur.push_back(v);
          }
        };
        if (k == 1)
          for (int32_t u = t.lo; u < t.hi; ++u) grow(u);
        else
          for (int32_t u : prev) grow(u);
        std::sort(cur.begin(), cur.end());
        cur.erase(std::unique(cur.begin(), cur.end()), cur.end());
        cur.erase(std::remove_if(cur.begin(), cur.end(),
                                 [&](int32_t v) {
                                   return std::binary_search(prev.begin(), prev.end(), v) ||
                                          std::binary_search(prev2.begin(), prev2.end(), v);
                                 }),
                  cur.end());
        // the elements at the nodes of ring k-1 that are not yet listed
        const size_t e0 = t.elems.size();
        auto list = [&](int32_t u) {
          for (int64_t q = g.ptr[u]; q < g.ptr[u + 1]; ++q)
            if (g.c0[size_t(q)] != kNone && mark[g.c0[size_t(q)] / 3u] < 0) {
              mark[g.c0[size_t(q)] / 3u] = 0;
              t.elems.push_back(int32_t(g.c0[size_t(q)] / 3u));
            }
        };
        if (k == 1)
          for (int32_t u = t.lo; u < t.hi; ++u) list(u);
        else
          for (int32_t u : prev) list(u);
        std::sort(t.elems.begin() + e0, t.elems.end());
        const size_t total = size_t(t.nl[k - 1]) + cur.size();
        // rows are the nodes up to ring k-1; degree 1 keeps one vector in LDS;
        // the set-up pass the start and two values per element; codes have 16 bits
        if (total > (k == 1 ? max1 : max2) || t.nl[k - 1] > kRowMax || t.elems.size() > kCodeElem - 1 ||
            size_t(k == 1 ? total : size_t(t.nl[1])) + 2 * t.elems.size() > max1) {
          for (size_t q = e0; q < t.elems.size(); ++q) mark[size_t(t.elems[q])] = -1;
          t.elems.resize(e0);
          break;
        }
        t.nel[k - 1] = int32_t(t.elems.size());
        t.nl[k] = int32_t(total);
        t.rings = k;
        t.ring.insert(t.ring.end(), cur.begin(), cur.end());
        prev2.swap(prev);
        prev.swap(cur);
      }
      for (int k = t.rings + 1; k <= kMaxRing; ++k) t.nl[k] = t.nl[t.rings];
      for (int32_t e : t.elems) mark[size_t(e)] = -1;
    });
    dmax = ask;
    for (const HostTile& t : tiles) dmax = std::min(dmax, int(t.rings));
  }
  if (dmax < 1) return false;

  // slices and their extra pairs
  auto node_at = [](const HostTile& t, int32_t i) { return i < t.nl[0] ? t.lo + i : t.ring[size_t(i - t.nl[0])]; };
  auto nslices = [&](const HostTile& t) { return (t.nl[dmax - 1] + 63) / 64; };
  parallel_for(tiles.size(), [&](size_t ti, size_t) {
    HostTile& t = tiles[ti];
    t.xcount.assign(size_t(nslices(t)), 0);
    for (int32_t i = 0; i < t.nl[dmax - 1]; ++i) {
      const int32_t u = node_at(t, i);
      const int32_t pairs = int32_t((g.ptr[u + 1] - g.ptr[u] + 1) / 2);
      t.xcount[size_t(i / 64)] = std::max(t.xcount[size_t(i / 64)], pairs - kRowPairs);
    }
  });
  const size_t tile0 = rp.tiles.size();
  size_t slice = rp.xs.size(), halo = rp.halo.size(), xp = rp.xac.size() / 64, el = rp.ete.size();
  for (const HostTile& t : tiles) {
    RowTile r{};
    r.node0 = rm.node_off + t.lo;
    for (int k = 0; k <= kMaxRing; ++k) r.nl[k] = t.nl[std::min(k, dmax)];
    r.halo0 = int32_t(halo);
    r.slice0 = int32_t(slice);
    r.nslice = nslices(t);
    r.inst = inst;
    r.el0 = int64_t(el);
    for (int k = 0; k < kMaxRing; ++k) r.nel[k] = t.nel[std::min(k, dmax - 1)];
    el += size_t(r.nel[dmax - 1]);
    rp.tiles.push_back(r);
    for (int32_t x : t.xcount) {
      rp.xs.push_back(int2{int32_t(xp), x});
      xp += size_t(x);
    }
    slice += size_t(r.nslice);
    halo += size_t(r.nl[dmax] - r.nl[0]);
  }
  rp.halo.resize(halo);
  rp.cmax.resize(slice, 0);
  rp.ac.resize(slice * kRowPairs * 64, 0);
  constexpr uint32_t no2 = kNoCode | (kNoCode << 16);
  rp.code.resize(slice * kRowPairs * 64, uint2{no2, no2});
  rp.xac.resize(xp * 64, 0);
  rp.xcode.resize(xp * 64, uint2{no2, no2});
  rp.ete.resize(el);
  rp.egid.resize(el);
  parallel_for(tiles.size(), [&](size_t ti, size_t th) {
    const HostTile& t = tiles[ti];
    const RowTile& r = rp.tiles[tile0 + ti];
    std::vector<int32_t>& mark = scratch[th];
    if (mark.empty()) mark.assign(size_t(rm.ne), -1);
    for (int32_t q = 0; q < r.nel[dmax - 1]; ++q) {
      const int32_t e = t.elems[size_t(q)];
      rp.ete[size_t(r.el0 + q)] = uint32_t(rm.te_of[e]);
      rp.egid[size_t(r.el0 + q)] = rm.elem_off + e;
      mark[size_t(e)] = q;
    }
    auto code16 = [&](uint32_t c) { return c == kNone ? kNoCode : (1u + uint32_t(mark[c / 3u])) | (c % 3u) << kCodeEdge; };
    const int32_t nhalo = r.nl[dmax] - r.nl[0];
    // ring nodes by position, with their local ids
    std::vector<std::pair<int32_t, int32_t>> loc(static_cast<size_t>(nhalo));
    for (int32_t j = 0; j < nhalo; ++j) {
      rp.halo[size_t(r.halo0 + j)] = rm.node_off + t.ring[size_t(j)];
      loc[size_t(j)] = {t.ring[size_t(j)], r.nl[0] + j};
    }
    std::sort(loc.begin(), loc.end());
    auto local = [&](int32_t u) -> uint32_t {
      if (u >= t.lo && u < t.hi) return uint32_t(u - t.lo);
      return uint32_t(std::lower_bound(loc.begin(), loc.end(), std::make_pair(u, int32_t(0)))->second);
    };
    for (int32_t i = 0; i < r.nl[dmax - 1]; ++i) {
      const int32_t u = node_at(t, i);
      const size_t s = size_t(r.slice0 + i / 64), lane = size_t(i % 64);
      int32_t k = 0;
      for (int64_t q = g.ptr[u]; q < g.ptr[u + 1]; ++q, ++k) {
        const int32_t pair = k / 2;
        const bool base = pair < kRowPairs;
        const size_t at = base ? (s * kRowPairs + size_t(pair)) * 64 + lane
                               : (size_t(rp.xs[s].x) + size_t(pair - kRowPairs)) * 64 + lane;
        uint32_t& ac = base ? rp.ac[at] : rp.xac[at];
        uint2& code = base ? rp.code[at] : rp.xcode[at];
        const uint32_t cc = code16(g.c0[size_t(q)]) | (code16(g.c1[size_t(q)]) << 16);
        const uint32_t l = local(g.nbr[size_t(q)]);
        rp.cmax[s] = std::max(rp.cmax[s], uint16_t(l));
        if (k % 2 == 0) {
          ac |= l;
          code.x = cc;
        } else {
          ac |= l << 16;
          code.y = cc;
        }
      }
    }
    for (int32_t q = 0; q < r.nel[dmax - 1]; ++q) mark[size_t(t.elems[size_t(q)])] = -1;
  });
  for (size_t u = 0; u < n; ++u) {
    rp.pos[size_t(rm.node_off + rm.node_int[u])] = rm.node_off + dloc[u];
    rp.node[size_t(rm.node_off + dloc[u])] = rm.node_off + rm.node_int[u];
  }
  rp.rt0.push_back(int32_t(tile0));
  rp.nrt.push_back(int32_t(tiles.size()));
  rp.dmax.push_back(dmax);
  rp.ddef.push_back(std::min(dmax, ddef));
  return true;
}

// Every lane multiplies the row that it loads, also one past those that its pass
// uses (the sum is then discarded), and such a row's columns lie on any ring: the
// LDS holds whatever they reach.  That costs a few KB at degrees 1 and 2;
// masking the columns in the pass cost registers and 2 % of a gradient.
CgShape cg_shape(const RowPlan& rp, size_t width) {
  CgShape c{};
  c.extra_pairs = !rp.xac.empty();
  // an instance whose tiles hold fewer rings runs with its own largest degree
  auto degree = [&](const RowTile& t, int dg) {
    return dg == 0 ? rp.ddef[size_t(t.inst)] : std::min(dg, rp.dmax[size_t(t.inst)]);
  };
  for (const RowTile& t : rp.tiles) {
    c.max_row_own = std::max(c.max_row_own, t.nl[0]);
    for (int dg = 0; dg <= kAskRing; ++dg) {
      const int de = degree(t, dg);
      c.max_rows[dg] = std::max(c.max_rows[dg], t.nl[de - 1]);
      if (de > 1) c.max_nodes[dg] = std::max(c.max_nodes[dg], t.nl[de]);
      c.max_slds[0][dg] = std::max(c.max_slds[0][dg], t.nl[1] + 2 * (1 + t.nel[de - 1]));
      c.max_slds[1][dg] = std::max(c.max_slds[1][dg], t.nl[1] + 1 + t.nel[de - 1]);
    }
  }
  for (int dg = 0; dg <= kAskRing; ++dg) {
    const int own = cg_own_rows(c, dg) * kWaves, all = cg_rows(c, dg) * kWaves;   // slices
    for (const RowTile& t : rp.tiles) {
      c.max_first[dg] = std::max(c.max_first[dg], t.nl[1]);
      for (int q = 0; q < std::min(t.nslice, all); ++q) {
        const int32_t n = 1 + rp.cmax[size_t(t.slice0 + q)];
        if (q < own) c.max_first[dg] = std::max(c.max_first[dg], n);
        if (degree(t, dg) > 1) c.max_cols[dg] = std::max(c.max_cols[dg], n);
      }
    }
  }
  return c;
}

// The combination in a pass's last workgroup takes one memory round trip per 256
// tiles of the instance, the separate launch about 5 us; in a large batch the
// arrivals of all tiles cost more than one launch.  us per polled step, in the
// pass / by a launch of its own, by row tiles:
//   one plate  FP64  260  212 / 235    516  293 / 317    961  426 / 429   1134  480 / 469   2055  681 / 648
//              FP32  329  145 / 155    516  152 / 161    961  179 / 185   1134  207 / 205   2055  277 / 269
//   batches    FP32  8 x 130   186 / 196   16 x 130   251 / 262   3 x 516   228 / 230
//                    16 uneven plates, 3600 in all   406 / 401   64 uneven plates, 13500   1280 / 1232
// A caller's own tiles of under 128 nodes keep the limit, and the launches per
// round, that they had before the row tiles (519 of 64 nodes: 407 / 443).
bool combine_in_pass(int32_t inst_tiles, int32_t all_tiles, int32_t tile_nodes) {
  return inst_tiles <= (tile_nodes < 128 ? 512 : 1024) && all_tiles <= 3072;
}

int cg_rows(const CgShape& c, int deg) {
  const int rpt = std::max((c.max_rows[deg] + kBlock - 1) / kBlock, (c.max_nodes[deg] + kBlock - 1) / kBlock - 1);
  if (rpt > 4) return 8;
  return c.max_row_own <= kBlock ? std::max(rpt, 1) : std::max(rpt, 3);
}

int cg_own_rows(const CgShape& c, int deg) {
  const int rpt = cg_rows(c, deg);
  return rpt <= 3 && c.max_row_own <= kBlock ? 1 : rpt;
}

size_t cg_lds(const CgShape& c, int deg, int nch, size_t width) {
  if (nch > 0) return size_t(c.max_slds[nch - 1][deg]) * width;
  const size_t half = size_t(cg_rows(c, deg) + 1) * kBlock;
  // a restart's iterate is FP64
  return std::max(size_t(c.max_first[deg]) * sizeof(double),
                  c.max_nodes[deg] > 0 ? (half + std::max(half, size_t(c.max_cols[deg]))) * width : 0);
}

}  // namespace pf
