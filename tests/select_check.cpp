// Host check of the launches that the planner chooses by size (plan_host.hpp),
// built and run by test_select.py: on both sides of each limit, and for the
// shapes with which the GPU tests mean to reach a kernel.
#include <cstdio>
#include <cstdlib>

#include <hip/hip_runtime.h>

#include "plan_host.hpp"

using namespace psatd;

namespace {

int g_fail = 0;
#define EXPECT(c, ...)                     \
  do {                                     \
    if (!(c)) {                            \
      std::fprintf(stderr, __VA_ARGS__);   \
      std::fprintf(stderr, " (%s)\n", #c); \
      ++g_fail;                            \
    }                                      \
  } while (0)

// The lists of a grid N in k equal boxes per axis with guards g.
HostTables lists(int prec, std::array<int64_t, 3> N, std::array<int, 3> k = {1, 1, 1},
                 std::array<int32_t, 3> g = {0, 0, 0}, int ntu = 512, bool fuse = false) {
  std::vector<int64_t> lo, n;
  std::vector<int32_t> gu;
  for (int z = 0; z < k[2]; ++z)
    for (int y = 0; y < k[1]; ++y)
      for (int x = 0; x < k[0]; ++x)
        for (int u = 0; u < 3; ++u) {
          const int c = u == 0 ? x : (u == 1 ? y : z);
          lo.push_back(c * (N[u] / k[u]));
          n.push_back(N[u] / k[u]);
          gu.push_back(g[u]);
        }
  HostTables h;
  std::string err;
  const double d[3] = {1, 1, 1};
  if (build_host(h, err, N.data(), d, k[0] * k[1] * k[2], lo.data(), n.data(), gu.data(), 16, 0.5, 1.0, prec,
                 PSATD_J_REPLICATED) != PSATD_OK) {
    std::fprintf(stderr, "%s\n", err.c_str());
    std::exit(1);
  }
  h.ntu = ntu;
  h.fuse_eb = fuse;
  build_lists(h, true, !h.xyc.empty(), !h.zcls.empty());
  return h;
}

bool halves(const HostTables& h) { return h.split && h.lists.xy[0][0].half > 0; }

void check_halves() {
  auto one = [](int64_t x, int64_t y, int64_t z) { return lists(PSATD_F32_VALU, {x, y, z}); };
  // two stages each way: from 0.55 of one round of 256 planes of the 6 fields, 0.67 of more
  EXPECT(!halves(one(256, 256, 22)) && halves(one(256, 256, 24)), "256 x 256, one round");
  EXPECT(halves(one(256, 256, 42)) && !halves(one(256, 256, 44)), "256 x 256, into the second round");
  EXPECT(!halves(one(256, 256, 56)) && halves(one(256, 256, 60)), "256 x 256, two rounds");
  EXPECT(halves(one(256, 256, 256)), "256^3");
  // three stages along x (150 = 5 5 6): from 0.75
  EXPECT(!halves(one(300, 144, 30)) && halves(one(300, 144, 32)), "300 x 144, one round");
  EXPECT(!halves(one(300, 144, 63)) && halves(one(300, 144, 64)), "300 x 144, two rounds");
  for (int z : {1, 2, 4, 16}) EXPECT(!halves(one(192, 256, z)), "%d planes", z);
  EXPECT(halves(lists(PSATD_F32_VALU, {368, 368, 128}, {2, 2, 2}, {8, 8, 8})), "eight boxes");
  // not fused, not FP64, not planes that fit the LDS
  EXPECT(!halves(lists(PSATD_F32_VALU, {256, 256, 64}, {1, 1, 1}, {0, 0, 0}, 512, true)), "fused exchange");
  EXPECT(!halves(lists(PSATD_F64, {256, 256, 64})), "FP64");
  EXPECT(!halves(one(96, 96, 256)), "planes that fit the LDS");
  // test_gpu_halves.py
  EXPECT(halves(lists(PSATD_F32_VALU, {210, 201, 36}, {1, 1, 1}, {3, 12, 2})), "216 x 225");
  EXPECT(halves(lists(PSATD_F32_VALU, {420, 1, 40}, {1, 1, 1}, {0, 87, 1})), "420 x 175, one row");
  EXPECT(halves(one(256, 192, 30)), "256 x 192");
  std::printf("halves ok\n");
}

void check_heat() {
  auto pencils = [](int prec, std::array<int64_t, 3> N, std::array<int, 3> k = {1, 1, 1}) {
    return lists(prec, N, k).lists.heat.PB;
  };
  // as wide as four tiles fit the LDS, while every compute unit has a tile
  EXPECT(pencils(PSATD_F32_VALU, {96, 96, 96}, {1, 1, 1}) == 16, "4704 pencils");
  EXPECT(pencils(PSATD_F32_VALU, {192, 192, 192}, {2, 2, 2}) == 32, "37632 pencils");
  EXPECT(pencils(PSATD_F32_VALU, {64, 64, 64}) == 8 && pencils(PSATD_F64, {64, 64, 64}) == 8, "2112 pencils");
  EXPECT(pencils(PSATD_F64, {48, 48, 48}) == 4, "1200 pencils");
  EXPECT(pencils(PSATD_F32_VALU, {16, 16, 256}) == 4, "144 pencils");
  EXPECT(pencils(PSATD_F64, {192, 192, 192}, {2, 2, 2}) == 16, "FP64, 96 long");
  // 250 and 256 tiles of 32 pencils
  EXPECT(pencils(PSATD_F32_BF16X6, {30, 500, 4}) == 16, "8000 pencils");
  EXPECT(pencils(PSATD_F32_VALU, {30, 512, 8}) == 32, "8192 pencils");
  // test_gpu_heat_tiles.py
  for (int prec : {PSATD_F64, PSATD_F32_VALU, PSATD_F32_BF16X6}) {
    EXPECT(pencils(prec, {16, 14, 96}) == 4, "126 pencils");
    EXPECT(pencils(prec, {60, 70, 12}) == 8, "2170 pencils");
    EXPECT(pencils(prec, {96, 96, 20}) == 16, "4704 pencils, short z");
    EXPECT(lists(prec, {72, 60, 48}, {3, 3, 3}, {8, 8, 8}).lists.heat.PB == 32, "27 boxes");
  }
  std::printf("heat ok\n");
}

const ZLaunch& ztile(const HostTables& h) { return h.lists.z[0][0]; }

void check_held() {
  auto held = [](std::array<int64_t, 3> N, int ntu = 512) {
    const HostTables h = lists(PSATD_F64, N, {1, 1, 1}, {0, 0, 0}, ntu);
    return ztile(h).held ? ztile(h).PB : 0;
  };
  // test_gpu_rings.py
  EXPECT(held({70, 75, 70}) == 8 && held({70, 75, 99}) == 8 && held({70, 75, 100}) == 8, "8 pencils");
  EXPECT(held({48, 45, 147}) == 4 && held({48, 45, 200}) == 4, "4 pencils");
  const HostTables two = lists(PSATD_F64, {64, 64, 160}, {1, 1, 2}, {8, 8, 8});
  EXPECT(ztile(two).held && ztile(two).PB == 8, "two boxes");
  // the other sides: tiles of which two share a compute unit with nine fields, pairs past
  // the threads, one round of tiles, other thread counts and FP32
  EXPECT(!held({70, 75, 56}) && held({70, 75, 70}), "short z");
  EXPECT(!held({70, 75, 105}) && !held({48, 45, 210}), "long z");
  EXPECT(!held({48, 45, 70}) && held({70, 75, 70}) && held({70, 60, 70}), "tiles");  // 141, 338 and 270
  EXPECT(!held({70, 75, 70}, 1024), "1024 threads");
  EXPECT(!ztile(lists(PSATD_F32_VALU, {70, 75, 70})).held, "FP32");
  std::printf("held ok\n");
}

void check_narrow() {
  for (int prec : {PSATD_F64, PSATD_F32_VALU})  // test_gpu_rings.py: 27 boxes of 32^3 padded
    EXPECT(ztile(lists(prec, {72, 72, 72}, {3, 3, 3}, {4, 4, 4})).narrow, "27 boxes");
  auto narrow = [](int prec, std::array<int64_t, 3> N) { return ztile(lists(prec, N)).narrow != 0; };
  // three FP32 tiles or two FP64 ones to a compute unit, and more than one round of them
  EXPECT(narrow(PSATD_F32_VALU, {128, 100, 70}) && !narrow(PSATD_F32_VALU, {128, 100, 75}), "FP32, z");
  EXPECT(narrow(PSATD_F64, {128, 100, 64}) && !narrow(PSATD_F64, {128, 100, 70}), "FP64, z");
  EXPECT(!narrow(PSATD_F32_VALU, {64, 64, 64}) && !narrow(PSATD_F64, {54, 64, 64}), "one round");
  std::printf("narrow ok\n");
}

}  // namespace

int main() {
  check_halves();
  check_heat();
  check_held();
  check_narrow();
  return g_fail ? 1 : 0;
}
