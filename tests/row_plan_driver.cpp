// Checks the row plan of the damage passes (rows.cpp) on the CPU against the
// meshes it was built from: run by test_row_plan.py.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <numeric>
#include <random>
#include <set>

#include "../paper_2606_23458_amd/csrc/pf_internal.hpp"

using namespace pf;

#define CHECK(c)                                                              \
  do {                                                                        \
    if (!(c)) {                                                               \
      std::printf("FAILED line %d: %s\n", __LINE__, #c);                      \
      std::exit(1);                                                           \
    }                                                                         \
  } while (0)

struct Case {
  const char* name;
  int nx, ny, fan;       // a grid, or `fan` triangles around one node
  bool diag, extra;      // random diagonals; a third triangle at one edge
  size_t tile_nodes;
  int dmax;              // expected
};

int main() {
  const Case cases[] = {{"grid", 64, 32, 0, false, false, 256, 8},       {"diagonals", 397, 211, 0, true, false, 256, 8},
                        {"cell", 1, 1, 0, false, false, 256, 8},         {"strip", 3000, 1, 0, true, false, 256, 8},
                        {"fan12", 0, 0, 12, false, true, 256, 8},        {"fan3000", 0, 0, 3000, false, true, 256, 1},
                        {"small tiles", 120, 60, 0, true, false, 64, 4}, {"large", 700, 400, 0, false, false, 512, 6}};
  std::mt19937 r(1);
  RowPlan rp;
  int off = 0, eoff = 0, teoff = 0, inst = 0;
  for (const Case& c : cases) {
    std::vector<double> xy;
    std::vector<int32_t> tri;
    if (c.fan) {
      xy = {0.0, 0.0};
      for (int i = 0; i < c.fan; ++i) xy.push_back(std::cos(6.283185 * i / c.fan)), xy.push_back(std::sin(6.283185 * i / c.fan));
      for (int i = 0; i < c.fan; ++i) tri.insert(tri.end(), {0, 1 + i, 1 + (i + 1) % c.fan});
    } else {
      for (int j = 0; j <= c.ny; ++j)
        for (int i = 0; i <= c.nx; ++i) xy.push_back(i), xy.push_back(j);
      for (int j = 0; j < c.ny; ++j)
        for (int i = 0; i < c.nx; ++i) {
          const int a = j * (c.nx + 1) + i, b = a + 1, d = a + c.nx + 1, e = d + 1;
          if (c.diag && (r() & 1))
            tri.insert(tri.end(), {a, b, d, b, e, d});
          else
            tri.insert(tri.end(), {a, b, e, a, e, d});
        }
    }
    if (c.extra) tri.insert(tri.end(), {0, 1, 2});
    const int n = int(xy.size() / 2), ne = int(tri.size() / 3);
    std::vector<int32_t> ni(n), eo(ne), te(ne);
    std::iota(ni.begin(), ni.end(), 0);
    std::iota(eo.begin(), eo.end(), 0);
    std::iota(te.begin(), te.end(), teoff);
    std::shuffle(ni.begin(), ni.end(), r);
    std::shuffle(eo.begin(), eo.end(), r);
    std::shuffle(te.begin(), te.end(), r);
    std::vector<std::pair<size_t, size_t>> leaves;
    for (size_t lo = 0; lo < size_t(n); lo += c.tile_nodes) leaves.emplace_back(lo, std::min<size_t>(n, lo + c.tile_nodes));
    rp.pos.resize(size_t(off) + n);
    rp.node.resize(size_t(off) + n);
    RowMesh rm{off, eoff, n, ne, xy.data(), tri.data(), ni.data(), eo.data(), te.data(), &leaves, c.tile_nodes};
    CHECK(row_plan_add(rp, rm, inst, 8, 163840));
    CHECK(rp.dmax[inst] == c.dmax);
    // what every row has to hold: contributions by (node, neighbour), in the mesh's numbering
    std::map<std::pair<int, int>, std::multiset<uint32_t>> want;
    std::vector<int> valence(n, 0), einv(ne);
    for (int j = 0; j < ne; ++j) einv[eo[j]] = j;
    for (int e = 0; e < ne; ++e) {
      const int32_t* t = &tri[3 * e];
      const int a[3] = {0, 0, 1}, b[3] = {1, 2, 2};
      for (int q = 0; q < 3; ++q) {
        want[{t[a[q]], t[b[q]]}].insert(3u * uint32_t(einv[e]) + q);
        want[{t[b[q]], t[a[q]]}].insert(3u * uint32_t(einv[e]) + q);
        valence[t[q]]++;
      }
    }
    std::vector<int> user(n), seen(n, 0);
    for (int u = 0; u < n; ++u) {
      const int p = rp.pos[off + ni[u]];
      CHECK(p >= off && p < off + n && rp.node[p] == off + ni[u]);
      user[p - off] = u;
    }
    const int dm = rp.dmax[inst];
    for (int ti = rp.rt0[inst]; ti < rp.rt0[inst] + rp.nrt[inst]; ++ti) {
      const RowTile& t = rp.tiles[ti];
      auto pos = [&](int i) { return i < t.nl[0] ? t.node0 + i : rp.halo[t.halo0 + i - t.nl[0]]; };
      for (int i = 0; i < t.nl[0]; ++i) seen[t.node0 + i - off]++;
      std::set<int> local;
      for (int i = 0; i < t.nl[dm]; ++i) CHECK(local.insert(pos(i)).second);
      CHECK(t.nslice == (t.nl[dm - 1] + 63) / 64 && t.nl[dm - 1] <= kRowMax);
      for (int i = 0; i < 64 * t.nslice; ++i) {
        const int s = t.slice0 + i / 64, lane = i % 64;
        int ring = 0, last = -1, stands = 0;
        while (ring < dm && i >= t.nl[ring]) ++ring;
        std::map<int, std::multiset<uint32_t>> got;
        auto pair = [&](uint32_t cols, uint2 code) {
          for (int h = 0; h < 2; ++h) {
            const int col = int(h ? cols >> 16 : cols & 0xffffu);
            const uint32_t cc = h ? code.y : code.x;
            CHECK(col < t.nl[std::min(dm, ring + 1)] || cc == (kNoCode | kNoCode << 16));
            CHECK(col < t.nl[dm]);
            for (int u = 0; u < 2; ++u) {
              const uint32_t cd = u ? cc >> 16 : cc & 0xffffu;
              if (cd == kNoCode) continue;
              CHECK(ring < dm);
              const int e = int(cd & kCodeElem) - 1;
              CHECK(e < t.nel[std::min(ring, dm - 1)]);
              const int gid = rp.egid[t.el0 + e] - eoff;
              CHECK(gid >= 0 && gid < ne && int(rp.ete[t.el0 + e]) == te[gid]);
              if (u == 0) {   // the element the entry stands for: ascending along the row
                CHECK(gid > last);
                last = gid, ++stands;
              }
              got[col].insert(3u * uint32_t(gid) + (cd >> kCodeEdge));
            }
          }
        };
        for (int q = 0; q < kRowPairs; ++q) {
          const size_t at = (size_t(s) * kRowPairs + q) * 64 + lane;
          pair(rp.ac[at], rp.code[at]);
        }
        for (int q = 0; q < rp.xs[s].y; ++q) {
          const size_t at = (size_t(rp.xs[s].x) + q) * 64 + lane;
          pair(rp.xac[at], rp.xcode[at]);
        }
        if (i >= t.nl[dm - 1]) continue;   // padding holds nothing
        const int u = user[pos(i) - off];
        CHECK(stands == valence[u]);
        size_t nbrs = 0;
        for (auto it = want.lower_bound({u, -1}); it != want.end() && it->first.first == u; ++it) ++nbrs;
        CHECK(got.size() == nbrs);
        for (const auto& g : got) CHECK((want[{u, user[pos(g.first) - off]}] == g.second));
      }
    }
    for (int s : seen) CHECK(s == 1);
    std::printf("%s ok\n", c.name);
    off += n, eoff += ne, teoff += ne, ++inst;
  }
  return 0;
}
