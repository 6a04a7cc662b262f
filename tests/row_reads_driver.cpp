// Checks on the CPU that every LDS read of the damage passes lies inside the
// bytes that their launch asks for: run by test_row_reads.py.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
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

// A handle of 215 million nodes in plates of 128 owned nodes and degree 8 lists more than 2^31
// elements, too many to build here; its other offsets stay below: at most 5 ring nodes and 5/64
// slices per node, of 3.6e8 nodes.
static_assert(sizeof(RowTile::el0) == 8, "offsets into the element lists need 64 bits");

struct Plate {
  int nx, ny, fan;       // a grid, or `fan` triangles around one node
  bool diag;             // random diagonals
  size_t tile_nodes;
};

static std::mt19937 rng(1);

static void add(RowPlan& rp, const Plate& c, int inst, size_t width) {
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
        if (c.diag && (rng() & 1))
          tri.insert(tri.end(), {a, b, d, b, e, d});
        else
          tri.insert(tri.end(), {a, b, e, a, e, d});
      }
  }
  const int n = int(xy.size() / 2), ne = int(tri.size() / 3), off = int(rp.pos.size());
  std::vector<int32_t> ni(n), eo(ne), te(ne);
  std::iota(ni.begin(), ni.end(), 0);
  std::iota(eo.begin(), eo.end(), 0);
  std::iota(te.begin(), te.end(), 0);
  std::vector<std::pair<size_t, size_t>> leaves;
  for (size_t lo = 0; lo < size_t(n); lo += c.tile_nodes) leaves.emplace_back(lo, std::min<size_t>(n, lo + c.tile_nodes));
  rp.pos.resize(size_t(off) + n);
  rp.node.resize(size_t(off) + n);
  RowMesh rm{off, 0, n, ne, xy.data(), tri.data(), ni.data(), eo.data(), te.data(), &leaves, c.tile_nodes};
  CHECK(row_plan_add(rp, rm, inst, width, 163840));
}

static void check(const RowPlan& rp, size_t width) {
  const CgShape cg = cg_shape(rp, width);
  for (int ask = 0; ask <= kAskRing; ++ask) {
    const int rpt = cg_rows(cg, ask), own = cg_own_rows(cg, ask);
    const long w = long(width), lds = long(cg_lds(cg, ask, 0, width)), half = long((rpt + 1) * kBlock) * w;
    CHECK(lds <= 163840 - 2048 && own * kBlock >= cg.max_row_own && own <= rpt);
    for (const RowTile& t : rp.tiles) {
      const int deg = ask ? std::min(ask, rp.dmax[size_t(t.inst)]) : rp.ddef[size_t(t.inst)];
      CHECK(rpt * kBlock >= t.nl[deg - 1]);
      // the vectors' own nodes, and what a polynomial's steps store
      CHECK(long(t.nl[1]) * 8 <= lds && long(t.nl[deg]) * w <= (deg > 1 ? half : lds));
      if (deg > 1) CHECK(2 * half <= lds && rpt <= kRowMax / kBlock);
      for (int i = 0; i < rpt * kBlock; ++i) {
        // the row that a lane loads (past the last slice: that slice's), and the columns it multiplies by
        const size_t s = size_t(t.slice0) + size_t(std::min(i / 64, t.nslice - 1)), lane = size_t(i % 64);
        auto pair = [&](uint32_t cc) {
          for (uint32_t col : {cc & 0xffffu, cc >> 16}) {
            // rows that a pass uses find their columns among the nodes it holds
            if (i < t.nl[0]) CHECK(int(col) < t.nl[1]);
            if (i < t.nl[deg - 1]) CHECK(int(col) < t.nl[deg]);
            // every row's are read: in a restart and for A z (owned rows per thread), in a step (all)
            if (i < own * kBlock) CHECK(long(col + 1) * 8 <= lds && long(col + 1) * w <= lds);
            if (deg > 1) CHECK(half + long(col + 1) * w <= lds);
          }
        };
        for (int q = 0; q < kRowPairs; ++q) pair(rp.ac[(s * kRowPairs + size_t(q)) * 64 + lane]);
        for (int q = 0; q < rp.xs[s].y; ++q) pair(rp.xac[(size_t(rp.xs[s].x) + size_t(q)) * 64 + lane]);
      }
      // the set-up pass: the start, then the elements' values behind a zero
      for (int nch : {1, 2})
        CHECK(size_t(t.nl[1] + nch % 2 * (1 + t.nel[deg - 1]) + 1 + t.nel[deg - 1]) * width <= cg_lds(cg, ask, nch, width));
    }
  }
}

// Two hubs of 3600 triangles side by side, in one tile of the first plan and too much for it; the
// handle's own tiles of 128 nodes keep them apart, and the second plan takes those.
static void two_hubs() {
  const int n = 3600;
  std::vector<double> xy;
  std::vector<int32_t> tri;
  std::vector<std::set<int>> nbr;
  for (int h = 0; h < 2; ++h) {
    const int hub = int(xy.size() / 2);
    xy.push_back(1e-3 * h), xy.push_back(0.0);
    for (int i = 0; i < n; ++i) {
      const double a = 6.283185307 * i / n;
      xy.push_back((1.0 + h) * std::cos(a)), xy.push_back((1.0 + h) * std::sin(a));
      tri.insert(tri.end(), {hub, hub + 1 + i, hub + 1 + (i + 1) % n});
    }
  }
  const int nn = int(xy.size() / 2), ne = int(tri.size() / 3);
  nbr.resize(size_t(nn));
  for (int e = 0; e < ne; ++e)
    for (int q = 0; q < 6; ++q) nbr[size_t(tri[size_t(3 * e + q / 2)])].insert(tri[size_t(3 * e + (q / 2 + 1 + q % 2) % 3)]);
  std::vector<int32_t> ni(nn), eo(ne), te(ne);
  std::iota(ni.begin(), ni.end(), 0);
  std::iota(eo.begin(), eo.end(), 0);
  std::iota(te.begin(), te.end(), 0);
  std::vector<std::pair<size_t, size_t>> leaves;
  for (size_t lo = 0; lo < size_t(nn); lo += 128) leaves.emplace_back(lo, std::min<size_t>(nn, lo + 128));
  RowPlan rp;
  rp.pos.resize(size_t(nn));
  rp.node.resize(size_t(nn));
  RowMesh rm{0, 0, nn, ne, xy.data(), tri.data(), ni.data(), eo.data(), te.data(), &leaves, 128};
  CHECK(row_plan_add(rp, rm, 0, sizeof(float), 163840));
  CHECK(rp.tiles.size() == leaves.size() && rp.dmax[0] == 1);
  for (size_t k = 0; k < leaves.size(); ++k) {
    const RowTile& t = rp.tiles[k];
    CHECK(t.node0 == int(leaves[k].first) && t.nl[0] == int(leaves[k].second - leaves[k].first));
    for (int i = 0; i < t.nl[0]; ++i) {   // every neighbour once
      const size_t s = size_t(t.slice0 + i / 64), lane = size_t(i % 64);
      std::set<int> got;
      auto pair = [&](uint32_t cc, uint2 code) {
        for (int h = 0; h < 2; ++h) {
          const int col = int(h ? cc >> 16 : cc & 0xffffu);
          if ((h ? code.y : code.x) == (kNoCode | kNoCode << 16)) continue;
          CHECK(got.insert(col < t.nl[0] ? t.node0 + col : rp.halo[size_t(t.halo0 + col - t.nl[0])]).second);
        }
      };
      for (size_t q = 0; q < kRowPairs; ++q) pair(rp.ac[(s * kRowPairs + q) * 64 + lane], rp.code[(s * kRowPairs + q) * 64 + lane]);
      for (int q = 0; q < rp.xs[s].y; ++q)
        pair(rp.xac[(size_t(rp.xs[s].x) + size_t(q)) * 64 + lane], rp.xcode[(size_t(rp.xs[s].x) + size_t(q)) * 64 + lane]);
      CHECK(got == nbr[size_t(t.node0 + i)]);
    }
  }
  check(rp, sizeof(float));
  std::printf("two hubs ok\n");
}

int main() {
  two_hubs();
  const Plate plates[] = {{64, 32, 0, false, 256}, {397, 211, 0, true, 256}, {120, 60, 0, true, 64},
                          {1, 1, 0, false, 256},   {3000, 1, 0, true, 256},  {0, 0, 12, false, 256},
                          {0, 0, 3000, false, 256}, {1448, 724, 0, true, 512}, {700, 300, 0, false, 256}};
  for (size_t width : {sizeof(double), sizeof(float)}) {
    for (const Plate& c : plates) {
      RowPlan rp;
      add(rp, c, 0, width);
      check(rp, width);
      std::printf("plate ok\n");
    }
    // instances of different degrees in one handle: the launch is sized by the largest
    RowPlan rp;
    int inst = 0;
    for (const Plate& c : {plates[0], plates[6], plates[2], plates[3]}) add(rp, c, inst++, width);
    check(rp, width);
    std::printf("batch ok\n");
  }
  return 0;
}
