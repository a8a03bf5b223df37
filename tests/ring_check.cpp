// Host check of the spectral rings and work lists (plan_host.hpp), built and
// run by test_rings.py.  For each decomposition: every slot a box reads holds
// a plane of the same column at the same global z; every plane is transformed
// once; the results of a box lie outside everything another box reads, and
// outside the other boxes' results; and the workspace is no larger than the
// half spectra of all padded boxes.
#include <cstdio>
#include <cstdlib>
#include <set>

#include <hip/hip_runtime.h>

#include "plan_host.hpp"

using namespace psatd;

namespace {

int g_fail = 0;
#define CHECK(c, ...)                       \
  do {                                      \
    if (!(c)) {                             \
      std::fprintf(stderr, __VA_ARGS__);    \
      std::fprintf(stderr, " (%s)\n", #c);  \
      ++g_fail;                             \
      return;                               \
    }                                       \
  } while (0)

struct Box {
  int64_t lo[3], n[3];
  int32_t g[3];
};

void check_places(const char* name, const HostTables& h, const int64_t N[3], const std::vector<BoxD>& box,
                  int64_t elems, bool shared) {
  const WorkLists& w = h.lists;
  const int nsub = h.nsub;
  // what the forward pass leaves at each (field, plane) address: box and z
  std::map<int64_t, PlaneRec> at;
  int64_t planes = 0, nfwd = 0;
  for (const auto& ls : w.xy)
    for (const XyLaunch& l : ls) nfwd += l.nf;
  CHECK(nfwd == (int64_t)w.fwd.size(), "%s: launches cover the planes", name);
  for (const PlaneRec& r : w.fwd) {
    const BoxD& b = box[r.box];
    const int64_t nq = b.pp, used = (int64_t)b.P[1] * b.H;
    for (int f = 0; f < 9; ++f) {
      const int64_t o = b.sb + f * b.sv + ring_slot(b, r.z) * nq;
      CHECK(ring_slot(b, r.z) < b.ring && !at.count(o), "%s: plane written once", name);
      at[o] = r;
    }
    planes += used;
  }
  CHECK((planes < h.slab) == (shared), "%s: sharing", name);
  std::set<int64_t> results;
  for (int s = 0; s < nsub; ++s) {
    const BoxD& b = box[s];
    const int64_t nq = b.pp;
    auto globz = [&](const BoxD& c, int z) { return ((c.lo[2] - c.g[2] + z) % N[2] + N[2]) % N[2]; };
    for (int z = 0; z < b.P[2]; ++z)
      for (int f = 0; f < 9; ++f) {
        const auto it = at.find(b.sb + f * b.sv + ring_slot(b, z) * nq);
        CHECK(it != at.end(), "%s: box %d plane %d has a source", name, s, z);
        const BoxD& c = box[it->second.box];
        CHECK(globz(c, it->second.z) == globz(b, z) && c.lo[0] == b.lo[0] && c.n[0] == b.n[0] &&
                  c.g[0] == b.g[0] && c.lo[1] == b.lo[1] && c.n[1] == b.n[1] && c.g[1] == b.g[1],
              "%s: box %d plane %d is the same plane", name, s, z);
      }
    for (int f = 0; f < 6; ++f)
      for (int i = 0; i < b.n[2]; ++i) {
        const int64_t o = result_plane(b, 0, f, i);
        CHECK(o >= 0 && o + nq <= elems && results.insert(o).second, "%s: result planes distinct", name);
        for (int t = 0; t < nsub; ++t) {
          const BoxD& c = box[t];
          if (t == s) continue;
          for (int z = 0; z < c.P[2]; ++z)
            CHECK(o != c.sb + f * c.sv + ring_slot(c, z) * c.pp,
                  "%s: result of box %d over a plane box %d reads", name, s, t);
        }
      }
    for (int f = 6; f < 9; ++f)  // the held current's spectra outlive the z pass
      for (int z = 0; z < b.P[2]; ++z)
        CHECK(!results.count(b.sb + f * b.sv + ring_slot(b, z) * nq), "%s: J kept", name);
  }
  // every tile of every box once, the guard pieces of each plane those that meet it
  std::set<std::pair<int, int>> tiles;
  for (const ZLaunch& l : w.z[0])
    for (int i = l.u0; i < l.u0 + l.nu; ++i)
      for (int q = w.tiles[i].q0; q < w.tiles[i].q0 + l.PB && q < box[w.tiles[i].box].P[1] * box[w.tiles[i].box].H; ++q)
        CHECK(tiles.insert({w.tiles[i].box, q}).second, "%s: pencil once", name);
  int64_t pencils = 0;
  for (const BoxD& b : box) pencils += (int64_t)b.P[1] * b.H;
  CHECK((int64_t)tiles.size() == pencils, "%s: every pencil", name);
  for (const PlaneRec& r : w.fwd) {
    const BoxD& b = box[r.box];
    int64_t cells = 0;
    for (int i = r.p0; i < r.p1; ++i) {
      CHECK(r.z >= w.pull[i].qz && r.z < w.pull[i].qz + w.pull[i].lz, "%s: piece of the plane", name);
      cells += (int64_t)w.pull[i].ly * w.pull[i].lx;
    }
    const bool inner = r.z >= b.g[2] && r.z < b.g[2] + b.n[2];
    CHECK(cells == (int64_t)b.P[0] * b.P[1] - (inner ? (int64_t)b.n[0] * b.n[1] : 0), "%s: plane covered", name);
  }
}

// Every padded cell in exactly one copy list or alone; the copies of a region are
// the same global cells, in the order of boxes and positions.
void check_sums(const char* name, const HostTables& h, const int64_t N[3]) {
  std::map<int64_t, std::array<int64_t, 3>> cell;  // element -> global cell
  std::map<std::array<int64_t, 3>, std::vector<int64_t>> want;
  for (const BoxD& b : h.box)
    for (int z = 0; z < b.P[2]; ++z)
      for (int y = 0; y < b.P[1]; ++y)
        for (int x = 0; x < b.P[0]; ++x) {
          const int q[3] = {x, y, z};
          std::array<int64_t, 3> G;
          for (int u = 0; u < 3; ++u) G[u] = ((b.lo[u] - b.g[u] + q[u]) % N[u] + N[u]) % N[u];
          const int64_t o = b.foff + ((int64_t)z * b.P[1] + y) * b.P[0] + x;
          cell[o] = G;
          want[G].push_back(o);
        }
  std::set<int64_t> seen;
  for (size_t r = 0; r < h.sumr.size(); ++r) {
    const SumRegion& g = h.sumr[r];
    for (int z = 0; z < h.itemsS[r + 1] - h.itemsS[r]; ++z)
      for (int y = 0; y < g.ly; ++y)
        for (int x = 0; x < g.lx; ++x) {
          std::vector<int64_t> got;
          for (int c = g.c0; c < g.c0 + g.nc; ++c)
            got.push_back(h.sumc[c].off + (int64_t)z * h.sumc[c].sPl + (int64_t)y * h.sumc[c].sP0 + x);
          CHECK(cell.count(got[0]) && want[cell[got[0]]] == got, "%s: copies of a cell", name);
          for (int64_t o : got) CHECK(seen.insert(o).second, "%s: cell in one region", name);
        }
  }
  for (const auto& w : want)
    CHECK(w.second.size() == 1 || seen.count(w.second[0]), "%s: every shared cell summed", name);
  CHECK((int64_t)h.regionOf.size() == h.itemsS.back(), "%s: sum work list", name);
}

void check(const char* name, const int64_t N[3], const std::vector<Box>& bx, bool expect_shared) {
  std::vector<int64_t> lo, n;
  std::vector<int32_t> g;
  for (const Box& b : bx)
    for (int u = 0; u < 3; ++u) {
      lo.push_back(b.lo[u]);
      n.push_back(b.n[u]);
      g.push_back(b.g[u]);
    }
  HostTables h;
  std::string err;
  const double d[3] = {1, 1, 1};
  const int nsub = (int)bx.size();
  CHECK(build_host(h, err, N, d, nsub, lo.data(), n.data(), g.data(), 16, 0.5, 1.0, PSATD_F32_VALU,
                   PSATD_J_REPLICATED) == PSATD_OK, "%s: %s", name, err.c_str());
  for (int share = 0; share < 2; ++share) {
    build_lists(h, share != 0, !h.xyc.empty(), !h.zcls.empty());
    CHECK(h.lists.tight_elems <= 9 * h.slab, "%s: workspace", name);
    check_places(name, h, N, h.lists.tight, h.lists.tight_elems, share && expect_shared);
    check_places(name, h, N, h.lists.box, h.lists.elems, share && expect_shared);
  }
  HostTables dep;
  CHECK(build_host(dep, err, N, d, nsub, lo.data(), n.data(), g.data(), 16, 0.5, 1.0, PSATD_F32_VALU,
                   PSATD_J_DEPOSITED) == PSATD_OK, "%s: %s", name, err.c_str());
  check_sums(name, dep, N);
  std::printf("%s ok\n", name);
}
std::vector<Box> column(std::vector<int64_t> nz, std::vector<int32_t> gz, int nx, int32_t gx) {
  std::vector<Box> out;
  int64_t z = 0;
  for (size_t i = 0; i < nz.size(); ++i) {
    out.push_back({{0, 0, z}, {nx, nx, nz[i]}, {gx, gx, gz[i]}});
    z += nz[i];
  }
  return out;
}

}  // namespace

int main() {
  const int64_t N16[3] = {8, 8, 16};
  check("one box", N16, column({16}, {0}, 8, 2), false);
  check("one box wrapping onto itself", N16, column({16}, {4}, 8, 2), true);
  check("two boxes", N16, column({8, 8}, {2, 2}, 8, 2), true);
  check("guards wider than the neighbour", N16, column({2, 10, 4}, {4, 5, 4}, 8, 2), true);
  check("guards past the whole axis", N16, column({4, 12}, {16, 2}, 8, 2), false);
  // a column of other x guards beside it: each column covers part of the axis only
  std::vector<Box> mixed;
  for (int64_t z = 0; z < 16; z += 4)
    for (int64_t x = 0; x < 8; x += 4)
      mixed.push_back({{x, 0, z}, {4, 8, 4}, {(z / 4 + x / 4) % 3 == 0 ? 2 : 1, 1, (int32_t)(1 + (z == 8))}});
  check("columns with gaps", N16, mixed, true);
  return g_fail ? 1 : 0;
}
