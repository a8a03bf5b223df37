// Host-side planning of the local-FFT PSATD step (no HIP runtime calls):
// validation of the decomposition (Sec. 3.2: boxes tiling the periodic grid,
// guard cells per side), per-box padded extents, FFT radix schedules and their
// twiddle / position tables, modified-wavenumber table layout (Sec. 3.1),
// owner lookup, guard pieces and the work lists of every phase.
#pragma once
#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <map>
#include <string>
#include <tuple>
#include <vector>

#include "psatd.h"
#include "psatd_device.hpp"

namespace psatd {

// ------------------------------------------------------------ host tables
// What the x/y and z passes run on with the current knobs: the boxes with
// their spectral addresses, the plane and tile lists, and the launches of each
// batch (the lists' ranges).
struct WorkLists {
  std::vector<BoxD> box;          // spectral planes at line-aligned, spread pitches
  std::vector<BoxD> tight;        // the same boxes with planes back to back
  std::vector<PullPiece> pull;    // guard pieces per run of padded planes they cover
  std::vector<PlaneRec> fwd, inv;
  std::vector<ZItem> tiles;
  ZLaunch heat{};                 // the heat pass's tiles (unbatched plans), after the field pass's
  std::vector<std::vector<XyLaunch>> xy;  // per batch
  std::vector<std::vector<ZLaunch>> z;
  int64_t elems = 0, tight_elems = 0;  // complex elements of the workspace with either
};

struct HostTables {
  int64_t N[3];
  double d[3];
  int nsub;
  int p;
  double dt, c;
  int prec, jmode;
  std::vector<BoxD> box;
  std::vector<FftPlanD> plans;
  std::vector<long double> twr, twi;  // all twiddle tables, forward sign
  std::vector<int32_t> pos;           // position tables of the plans
  std::vector<KEntry> kent;
  int32_t kmod_len = 0;
  int32_t kmax_len = 0;
  std::vector<int32_t> cut[3];
  int32_t ncut[3];
  std::vector<int32_t> owner;
  std::vector<SumRegion> sumr;    // deposited currents: regions of equal copies, the
  std::vector<SumCopy> sumc;      // copies, and the work list over their z-planes
  std::vector<int32_t> itemsS, regionOf;
  // prefixes over the boxes: planes of 9 fields, z tiles of PB pencils, interior planes
  // of 6 fields; padded and interior planes (the work lists of scatter and gather)
  std::vector<int32_t> itemsF, itemsU, itemsI, itemsP, itemsN;
  WorkLists lists;
  bool split = false;  // x/y pass split into x rows and y columns (large planes)
  std::vector<PushBlk> push;      // fused E,B exchange: guard pieces per source box
  std::vector<int32_t> push_off;  // nsub + 1
  std::vector<FillPiece> fillp;   // guard fill: the pieces with offsets and pitches
  std::vector<int32_t> itemsG;    // guard fill: prefix over pieces of their z extent
  std::vector<int32_t> pieceOf;   // guard fill: item -> piece
  bool fuse_eb = false;           // E,B guards written by the inverse pass
  std::vector<PullPiece> pullp;   // guard regions per destination box, for the forward pass
  std::vector<int32_t> pull_off;  // nsub + 1
  bool pull_eb = false;           // the forward pass reads E,B guard cells from their owners
  int ldsX = 0, ldsY = 0;
  std::vector<Batch> batches;
  int64_t batch_slab = 0;     // complex elements of one spectral field slab of the largest batch
  int32_t batch_boxes = 0;
  int64_t field_elems = 0;
  int64_t slab = 0;
  int ldsF = 0, ldsI = 0, ldsU = 0, PB = 0;
  int maxr = 16;      // largest radix of the x/y schedules (8 or 16; 11 always)
  int maxrz = 16;     // largest radix of the z schedules
  std::vector<char> plan_z;  // per plan: 1 if it is a z schedule
  int spl = 0;        // BF16 terms of the matrix-core first stage (0: VALU form)
  int ntxy = 512;     // threads per work-group of the x/y passes
  int ntu = 512;      // threads per work-group of the z-update
  bool zreg = false;  // the register z pass applies (FP32 VALU form, every padded z length scheduled)
  std::vector<int32_t> boxlds;     // dynamic LDS bytes of one x/y plane of each box
  std::vector<XyClass> xyc;       // x/y launch classes (empty: one launch for every box)
  std::vector<int32_t> itemsXYC;  // their boxes and counts
  std::vector<ZClass> zcls;       // z launch classes (empty: one tile size for every box)
  std::vector<int32_t> itemsZC;   // their boxes and counts
  std::vector<ZGroup> zgroups;    // one per distinct padded z length
  std::vector<int32_t> itemsZR;   // their work lists, nsub + 1 prefix entries each
};

inline bool is_f64(int prec) { return prec == PSATD_F64; }
inline size_t real_size(int prec) { return is_f64(prec) ? 8 : 4; }

// Radix schedules: maxr 16 allows every codelet, maxr 8 the radices up to 8 plus 11.
// Every factorisation of n into exactly `left` radices from R (ordered as in R).
inline void factor_all(int n, int left, const int* R, int nr, std::vector<int>& acc,
                       std::vector<std::vector<int>>& out) {
  if (left == 0) {
    if (n == 1) out.push_back(acc);
    return;
  }
  for (int i = 0; i < nr; ++i) {
    if (n % R[i]) continue;
    acc.push_back(R[i]);
    factor_all(n / R[i], left - 1, R, nr, acc, out);
    acc.pop_back();
  }
}

// Fewest stages; among those the most balanced (largest smallest radix: fewer
// index operations per element in the small-radix stage), then the largest
// first radix.
inline bool factorize(int N, std::vector<int>& out, int maxr = 16) {
  static const int R16[] = {16, 12, 11, 10, 8, 7, 6, 5, 4, 3, 2};
  static const int R8[] = {11, 8, 7, 6, 5, 4, 3, 2};
  const int* R = maxr >= 16 ? R16 : R8;
  const int nr = maxr >= 16 ? 11 : 8;
  out.clear();
  if (N == 1) return true;
  for (int depth = 1; depth <= kMaxStages; ++depth) {
    std::vector<std::vector<int>> all;
    std::vector<int> acc;
    factor_all(N, depth, R, nr, acc, all);
    if (all.empty()) continue;
    const std::vector<int>* best = nullptr;
    int bmin = -1, bfirst = -1;
    for (const auto& f : all) {
      const int mn = *std::min_element(f.begin(), f.end());
      if (mn > bmin || (mn == bmin && f[0] > bfirst)) {
        best = &f;
        bmin = mn;
        bfirst = f[0];
      }
    }
    out = *best;
    return true;
  }
  return false;
}

// Schedule of a transform: with a matrix-core first stage (spl > 0) every
// length divisible by 16 starts with radix 16, the rest as factorize().
inline bool schedule(int N, std::vector<int>& out, int maxr, int spl) {
  if (spl > 0 && N % 16 == 0) {
    std::vector<int> rest;
    if (!factorize(N / 16, rest, maxr) || rest.size() + 1 > (size_t)kMaxStages) return false;
    out.assign(1, 16);
    out.insert(out.end(), rest.begin(), rest.end());
    return true;
  }
  return factorize(N, out, maxr);
}

// Fills the stage fields of a plan of length pl.N from a radix list.
inline void set_stages(FftPlanD& pl, const std::vector<int>& rad) {
  const int N = pl.N;
  pl.nstages = (int)rad.size();
  int prod = 1;
  for (int st = 0; st < kMaxStages; ++st) {
    if (st < pl.nstages) {
      pl.radix[st] = rad[st];
      pl.prod[st] = prod;
      prod *= rad[st];
      pl.stride[st] = N / prod;
    } else {
      pl.radix[st] = 1;
      pl.prod[st] = prod;
      pl.stride[st] = 1;
    }
    pl.rdiv[st] = make_fastdiv((uint32_t)pl.radix[st]);
    pl.sdiv[st] = make_fastdiv((uint32_t)pl.stride[st]);
  }
}

inline bool small_primes_only(int64_t n) {
  for (int p : {2, 3, 5, 7, 11})
    while (n % p == 0) n /= p;
  return n == 1;
}

// Writes the N-entry position table (at pl.pos) and twiddle table (at pl.tw) of
// a plan for its current radix schedule, the twiddles by stage and butterfly, W_N^{j t prod_s} for j < stride_s,
// t = 1..radix_s-1, then ones up to N entries.  Sets pl.twoff.
inline void write_plan_twiddles(HostTables& h, FftPlanD& pl) {
  const int N = pl.N;
  const long double PI = 3.141592653589793238462643383279502884L;
  int o = 0;
  for (int st = 0; st < kMaxStages; ++st) {
    pl.twoff[st] = o;
    if (st >= pl.nstages) continue;
    for (int j = 0; j < pl.stride[st]; ++j)
      for (int t = 1; t < pl.radix[st]; ++t, ++o) {
        const int64_t e = (int64_t)j * t * pl.prod[st];  // < N
        h.twr[pl.tw + o] = cosl(2.0L * PI * e / N);
        h.twi[pl.tw + o] = -sinl(2.0L * PI * e / N);
      }
  }
  for (; o < N; ++o) {  // the stages take N - 1 entries
    h.twr[pl.tw + o] = 1.0L;
    h.twi[pl.tw + o] = 0.0L;
  }
  for (int k = 0; k < N; ++k) h.pos[pl.pos + k] = plan_pos(&pl, k);
}

// Adds (or finds) an FFT plan of length N for the x/y passes or (zp) the z
// pass, which keep schedules of their own (each pass has its largest radix);
// returns its index or -1.
inline int add_plan(HostTables& h, int N, bool zp) {
  for (size_t i = 0; i < h.plans.size(); ++i)
    if (h.plans[i].N == N && (h.plan_z[i] != 0) == zp) return (int)i;
  std::vector<int> rad;
  if (!schedule(N, rad, zp ? h.maxrz : h.maxr, h.spl)) return -1;
  FftPlanD pl{};
  pl.N = N;
  set_stages(pl, rad);
  pl.tw = (int32_t)h.twr.size();
  h.twr.resize(h.twr.size() + N);
  h.twi.resize(h.twi.size() + N);
  pl.pos = (int32_t)h.pos.size();
  h.pos.resize(h.pos.size() + N);
  write_plan_twiddles(h, pl);
  h.plans.push_back(pl);
  h.plan_z.push_back(zp ? 1 : 0);
  return (int)h.plans.size() - 1;
}

// twiddle table W_N^e without a plan (real <-> half spectrum, N = padded x)
inline int add_twiddle(HostTables& h, int N, std::vector<std::pair<int, int>>& cache) {
  for (auto& c : cache)
    if (c.first == N) return c.second;
  const int off = (int)h.twr.size();
  const long double PI = 3.141592653589793238462643383279502884L;
  for (int e = 0; e < N; ++e) {
    h.twr.push_back(cosl(2.0L * PI * e / N));
    h.twi.push_back(-sinl(2.0L * PI * e / N));
  }
  cache.push_back({N, off});
  return off;
}

inline int add_kentry(HostTables& h, int N, double du) {
  for (auto& k : h.kent)
    if (k.N == N && k.du == du) return k.off;
  KEntry k;
  k.N = N;
  k.du = du;
  k.off = h.kmod_len;
  h.kmod_len += N;
  h.kmax_len = std::max(h.kmax_len, N);
  h.kent.push_back(k);
  return k.off;
}

// Groups of consecutive boxes pushed through the FFT/update passes together.
inline void set_batches(HostTables& h, int per) {
  h.batch_boxes = per;
  if (per <= 0 || per > h.nsub) per = h.nsub;
  h.batches.clear();
  h.batch_slab = 0;
  for (int b0 = 0; b0 < h.nsub; b0 += per) {
    const int b1 = std::min(h.nsub, b0 + per);
    Batch b;
    b.b0 = b0;
    b.b1 = b1;
    b.sbias = 9 * h.box[b0].soff;
    const int64_t end = (b1 < h.nsub) ? h.box[b1].soff : h.slab;
    h.batch_slab = std::max(h.batch_slab, end - h.box[b0].soff);
    h.batches.push_back(b);
  }
}

// Work list of the z-update for a tile of PB pencils (9 fields staged in LDS,
// plus the z twiddles).
inline void set_z_tile(HostTables& h, int PB) {
  const int csz = (int)(2 * real_size(h.prec));
  int maxPz = 0;
  h.itemsU.assign(h.nsub + 1, 0);
  for (int s = 0; s < h.nsub; ++s) {
    const BoxD& b = h.box[s];
    h.itemsU[s + 1] = h.itemsU[s] + (int32_t)(((int64_t)b.P[1] * b.H + PB - 1) / PB);
    maxPz = std::max(maxPz, b.P[2]);
  }
  h.PB = PB;
  h.ldsU = maxPz * (9 * PB + 1) * csz + maxPz * 4;  // staged fields, z twiddles, z indices
}

inline bool z_tile_fits(const HostTables& h, int maxPz, int PB) {
  const int csz = (int)(2 * real_size(h.prec));
  return (int64_t)maxPz * (9 * PB + 1) * csz + maxPz * 4 <= kMaxDynLds;
}

// Dynamic LDS of a z tile of PB pencils of padded z length Pz.
inline int64_t z_tile_lds(const HostTables& h, int Pz, int PB) {
  return (int64_t)Pz * (9 * PB + 1) * (int64_t)(2 * real_size(h.prec)) + (int64_t)Pz * 4;
}

// Pencils per z tile of one box on its own.  FP32: the widest of 10, 8 and 6
// pencils of which two tiles fit a compute unit's LDS (the 128-VGPR kernel
// holds two tiles per CU whatever their width, and wider tiles read longer
// runs: 96^3 boxes with 10 instead of 8 pencils, step 2.72 -> 2.69 ms;
// 176^3 boxes with 6 instead of 4, z pass 30.3 -> 26.5 ms), else 4.  FP64: 8
// where one tile fits, else 4.  0 when not even a 4-pencil tile fits.
inline int z_pencils_for(const HostTables& h, int Pz) {
  if (is_f64(h.prec)) {
    if (z_tile_lds(h, Pz, 8) <= kMaxDynLds) return 8;
  } else {
    for (int PB : {10, 8, 6})
      if (2 * z_tile_lds(h, Pz, PB) <= kMaxDynLds) return PB;
  }
  return z_tile_lds(h, Pz, 4) <= kMaxDynLds ? 4 : 0;
}

// Launch classes of the z pass: boxes grouped by their own tile size, each
// class launched with the LDS of its longest padded z, so the short-z boxes
// of an uneven decomposition keep 8-pencil tiles, two per compute unit, next
// to 4-pencil tiles of the long ones.  None when every box takes one size.
inline void build_z_classes(HostTables& h) {
  h.zcls.clear();
  h.itemsZC.clear();
  std::vector<int> pb(h.nsub);
  int used = 0;  // bit PB / 2 per tile size
  for (int s = 0; s < h.nsub; ++s) {
    pb[s] = z_pencils_for(h, h.box[s].P[2]);
    if (!pb[s]) return;
    used |= 1 << (pb[s] / 2);
  }
  if ((used & (used - 1)) == 0) return;  // one size: one launch
  for (int PB : {10, 8, 6, 4}) {
    if (!(used & (1 << (PB / 2)))) continue;
    ZClass k{};
    k.PB = PB;
    k.U = (int32_t)h.itemsZC.size();
    int32_t acc = 0;
    h.itemsZC.push_back(0);
    for (int s = 0; s < h.nsub; ++s) {
      const BoxD& b = h.box[s];
      if (pb[s] == PB) {
        acc += (int32_t)(((int64_t)b.P[1] * b.H + PB - 1) / PB);
        k.lds = std::max<int32_t>(k.lds, (int32_t)z_tile_lds(h, b.P[2], PB));
      }
      h.itemsZC.push_back(acc);
    }
    k.nU = acc;
    h.zcls.push_back(k);
  }
}

// The largest dynamic LDS any z launch of the plan may ask for.
inline int32_t z_lds_max(const HostTables& h) {
  int32_t m = h.ldsU;
  for (const ZClass& k : h.zcls) m = std::max(m, k.lds);
  return m;
}

// Re-derives every FFT schedule with radices up to maxr (twiddle tables
// depend on the length only and are kept).  False if a length has no
// schedule of at most kMaxStages stages.
inline bool set_max_radix(HostTables& h, int maxr, int maxrz) {
  std::vector<FftPlanD> plans = h.plans;
  for (size_t i = 0; i < plans.size(); ++i) {
    std::vector<int> rad;
    if (!schedule(plans[i].N, rad, h.plan_z[i] ? maxrz : maxr, h.spl)) return false;
    set_stages(plans[i], rad);
  }
  for (FftPlanD& pl : plans) write_plan_twiddles(h, pl);  // the layout follows the schedule
  h.plans = plans;
  h.maxr = maxr;
  h.maxrz = maxrz;
  return true;
}

inline int max_padded_z(const HostTables& h) {
  int m = 0;
  for (const BoxD& b : h.box) m = std::max(m, b.P[2]);
  return m;
}

// Runs of padded positions q of box d (global coordinate lo_d - g_d + q mod N)
// that fall on the interior [lo_s, lo_s + n_s) of box s, as (i0, q0, len) with
// i the interior index of s; consecutive q with consecutive i form one run.
struct Run {
  int32_t i0, q0, len;
};
inline void axis_runs(int64_t lo_s, int64_t n_s, int64_t lo_d, int64_t g_d, int64_t P_d, int64_t N,
                      std::vector<Run>& out) {
  out.clear();
  // one run per period: the interior starts at padded position first + k N
  const int64_t first = lo_s - (lo_d - g_d);
  const int64_t back = first + n_s - 1;  // its last cell at k = 0
  int64_t at = first - (back >= 0 ? back / N : -((-back + N - 1) / N)) * N;  // the first run that ends at 0 or after
  for (; at < P_d; at += N) {
    const int64_t q0 = std::max<int64_t>(at, 0), q1 = std::min(at + n_s, P_d);
    out.push_back({(int32_t)(q0 - at), (int32_t)q0, (int32_t)(q1 - q0)});
  }
}

// Guard pieces for the fused E,B exchange (every guard cell of every box in
// exactly one piece; the interior of each box itself excluded).
inline void build_push(HostTables& h) {
  const int nsub = h.nsub;
  h.push.clear();
  h.push_off.assign(nsub + 1, 0);
  std::vector<Run> rz, ry, rx;
  for (int s = 0; s < nsub; ++s) {
    const BoxD& a = h.box[s];
    for (int d = 0; d < nsub; ++d) {
      const BoxD& b = h.box[d];
      axis_runs(a.lo[2], a.n[2], b.lo[2], b.g[2], b.P[2], h.N[2], rz);
      if (rz.empty()) continue;
      axis_runs(a.lo[1], a.n[1], b.lo[1], b.g[1], b.P[1], h.N[1], ry);
      if (ry.empty()) continue;
      axis_runs(a.lo[0], a.n[0], b.lo[0], b.g[0], b.P[0], h.N[0], rx);
      if (rx.empty()) continue;
      for (const Run& z : rz)
        for (const Run& y : ry)
          for (const Run& x : rx) {
            const bool own = d == s && z.q0 == b.g[2] && y.q0 == b.g[1] && x.q0 == b.g[0] &&
                             z.i0 == 0 && y.i0 == 0 && x.i0 == 0;
            if (own) continue;  // the interior itself
            h.push.push_back({s, d, z.i0, z.len, z.q0, y.i0, y.len, y.q0, x.i0, x.len, x.q0});
          }
    }
    h.push_off[s + 1] = (int32_t)h.push.size();
  }
  // the pieces as the guard fill reads them
  const int V = 16 / real_size(h.prec);  // elements per 16-byte access
  h.fillp.clear();
  for (const PushBlk& k : h.push) {
    const BoxD& sb = h.box[k.src];
    const BoxD& db = h.box[k.dst];
    FillPiece f{};
    f.sP0 = sb.P[0];
    f.dP0 = db.P[0];
    f.sPl = sb.P[0] * sb.P[1];
    f.dPl = db.P[0] * db.P[1];
    f.ly = k.ly;
    f.lx = k.lx;
    f.so = sb.foff + ((int64_t)(sb.g[2] + k.z0) * sb.P[1] + (sb.g[1] + k.y0)) * sb.P[0] + sb.g[0] + k.x0;
    f.dof = db.foff + ((int64_t)k.qz * db.P[1] + k.qy) * db.P[0] + k.qx;
    f.vec = (k.lx % V == 0 && f.so % V == 0 && f.dof % V == 0 && f.sP0 % V == 0 && f.dP0 % V == 0 &&
             f.sPl % V == 0 && f.dPl % V == 0);
    h.fillp.push_back(f);
  }
  // the same pieces by destination box, as the forward pass pulls them
  h.pullp.clear();
  h.pull_off.assign(h.nsub + 1, 0);
  for (int d = 0; d < h.nsub; ++d) {
    for (size_t i = 0; i < h.push.size(); ++i) {
      const PushBlk& k = h.push[i];
      if (k.dst != d) continue;
      const BoxD& sb = h.box[k.src];
      PullPiece q{};
      q.so = h.fillp[i].so;
      q.sPl = sb.P[0] * sb.P[1];
      q.sP0 = sb.P[0];
      q.qz = k.qz;
      q.lz = k.lz;
      q.qy = k.qy;
      q.ly = k.ly;
      q.qx = k.qx;
      q.lx = k.lx;
      h.pullp.push_back(q);
    }
    h.pull_off[d + 1] = (int32_t)h.pullp.size();
  }
  // work list of the guard fill: one item per z-plane of every piece
  h.itemsG.assign(h.push.size() + 1, 0);
  for (size_t b = 0; b < h.push.size(); ++b) h.itemsG[b + 1] = h.itemsG[b] + h.push[b].lz;
  h.pieceOf.resize(h.itemsG.back());
  for (size_t b = 0; b < h.push.size(); ++b)
    for (int32_t i = h.itemsG[b]; i < h.itemsG[b + 1]; ++i) h.pieceOf[i] = (int32_t)b;
}

// Threads per x/y work-group for planes of `lds` bytes: the fewest (256, 512
// or 1024) that still keep 16 waves on a compute unit, given how many planes
// fit its LDS.
inline int xy_threads_for(int lds) {
  const int per_cu = lds > 0 ? std::max(1, kMaxDynLds / lds) : 1;
  for (int nt : {256, 512})
    if (per_cu * nt / 64 >= 16) return nt;
  return 1024;
}

// Launch classes of the x/y passes: boxes grouped by their group size, each
// class launched with its own LDS (the largest plane among its boxes), so
// small boxes are not held to one group per compute unit by the largest box
// of an uneven decomposition.  None when every box has the same group size or
// the planes take the split passes.
inline void build_xy_classes(HostTables& h) {
  h.xyc.clear();
  h.itemsXYC.clear();
  if (h.split) return;
  const int sizes[kMaxXyClasses] = {256, 512, 1024};
  std::vector<int> cls(h.nsub);
  int used = 0;
  for (int s = 0; s < h.nsub; ++s) {
    const int nt = xy_threads_for(h.boxlds[s]);
    cls[s] = nt == 256 ? 0 : (nt == 512 ? 1 : 2);
    used |= 1 << cls[s];
  }
  if (used == 1 || used == 2 || used == 4) return;  // one class: one launch
  auto prefix = [&](int c, auto count) {
    const int32_t off = (int32_t)h.itemsXYC.size();
    int32_t acc = 0;
    h.itemsXYC.push_back(0);
    for (int s = 0; s < h.nsub; ++s) {
      if (cls[s] == c) acc += (int32_t)count(h.box[s]);
      h.itemsXYC.push_back(acc);
    }
    return std::make_pair(off, acc);
  };
  for (int c = 0; c < kMaxXyClasses; ++c) {
    if (!(used & (1 << c))) continue;
    XyClass k{};
    k.nt = sizes[c];
    for (int s = 0; s < h.nsub; ++s)
      if (cls[s] == c) k.lds = std::max(k.lds, h.boxlds[s]);
    std::tie(k.F, k.nF) = prefix(c, [](const BoxD& b) { return (int64_t)b.P[2] * 9; });
    std::tie(k.P, k.nP) = prefix(c, [](const BoxD& b) { return (int64_t)b.P[2]; });
    std::tie(k.I, k.nI) = prefix(c, [](const BoxD& b) { return (int64_t)b.n[2] * 6; });
    std::tie(k.N, k.nN) = prefix(c, [](const BoxD& b) { return (int64_t)b.n[2]; });
    h.xyc.push_back(k);
  }
}

// Pencils per work-group of the register z pass for padded z length N (0: no schedule).
inline int zreg_pencils_of(int N) {
#define PSATD_ZREG_P(N_, L_, W_, MINW_) \
  if (N == N_) return zreg_pencils(L_, W_);
  PSATD_ZREG_SHAPES(PSATD_ZREG_P)
#undef PSATD_ZREG_P
  return 0;
}

// Groups of the register z pass: every distinct padded z length must have a
// schedule (else the LDS-staged z pass runs for all boxes).
inline void build_zreg(HostTables& h) {
  h.zreg = false;
  h.zgroups.clear();
  h.itemsZR.clear();
  if (h.prec != PSATD_F32_VALU) return;
  std::vector<int> lens;
  for (const BoxD& b : h.box)
    if (std::find(lens.begin(), lens.end(), b.P[2]) == lens.end()) lens.push_back(b.P[2]);
  if ((int)lens.size() > kMaxZGroups) return;
  for (int N : lens)
    if (!zreg_pencils_of(N)) return;
  for (const BoxD& b : h.box)  // the kernel addresses a box's 9 fields with 32-bit byte offsets
    if (9 * b.svol * 8 >= ((int64_t)1 << 31)) return;
  for (int N : lens) {
    const int P = zreg_pencils_of(N);
    ZGroup g{N, (int32_t)h.itemsZR.size(), 0, 0};
    int32_t acc = 0;
    h.itemsZR.push_back(0);
    for (const BoxD& b : h.box) {
      if (b.P[2] == N) acc += (int32_t)(((int64_t)b.P[1] * b.H + P - 1) / P);
      h.itemsZR.push_back(acc);
    }
    g.n = acc;
    h.zgroups.push_back(g);
  }
  h.zreg = true;
}

// One column of the decomposition: the boxes that share a spectral ring, as
// pairs (box, padded plane) per ring slot (an interior plane where there is
// one), and the slot of each box's padded plane 0.
struct Ring {
  std::vector<int32_t> boxes;
  std::vector<std::pair<int32_t, int32_t>> slot;
};

// Columns: boxes with the same first cell, length and guards along x and y
// have the same padded (x, y) plane at every z where their padded ranges meet.
// The ring lists the distinct z of the column in order, cut where the column
// leaves a gap (so that only a column that covers the whole axis wraps).  A
// column with a box for which zb + P[2] would wrap twice keeps a ring per box,
// as does every box when share is false.
// The x/y passes are bound by issue and memory together, so a plane not
// transformed is time saved in full: 64^3 boxes with 16 guards transform 64 of
// their 96 planes (forward pass 1.11 -> 0.74 ms FP32, 2.31 -> 1.50 ms FP64 on
// 64 boxes), 128^3 with 24 guards 128 of 176 (9.5 -> 6.4 ms on 64 boxes).
inline std::vector<Ring> build_rings(const HostTables& h, std::vector<BoxD>& box, bool share) {
  std::vector<Ring> rings;
  auto alone = [&](int s) {
    Ring r;
    r.boxes.push_back(s);
    for (int z = 0; z < box[s].P[2]; ++z) r.slot.push_back({s, z});
    box[s].ring = box[s].P[2];
    box[s].zb = box[s].slo = box[s].shi = 0;
    rings.push_back(std::move(r));
  };
  if (!share) {
    for (int s = 0; s < h.nsub; ++s) alone(s);
    return rings;
  }
  std::map<std::array<int32_t, 6>, std::vector<int32_t>> columns;
  for (int s = 0; s < h.nsub; ++s) {
    const BoxD& b = box[s];
    columns[{b.lo[1], b.n[1], b.g[1], b.lo[0], b.n[0], b.g[0]}].push_back(s);
  }
  const int64_t N = h.N[2];
  auto globz = [&](const BoxD& b, int z) { return (int)((((int64_t)b.lo[2] - b.g[2] + z) % N + N) % N); };
  for (const auto& col : columns) {
    const std::vector<int32_t>& bs = col.second;
    // per global z: the slot's plane, and how many boxes read it
    std::vector<std::pair<int32_t, int32_t>> at(N, {-1, 0});
    std::vector<int32_t> readers(N, 0);
    for (int s : bs) {
      std::vector<char> seen(N, 0);
      for (int z = 0; z < box[s].P[2]; ++z) {
        const int G = globz(box[s], z);
        const bool inner = z >= box[s].g[2] && z < box[s].g[2] + box[s].n[2];
        if (inner || at[G].first < 0) at[G] = {s, z};
        readers[G] += !seen[G];
        seen[G] = 1;
      }
    }
    int64_t cut = 0;  // the first plane after a gap, if there is one
    while (cut < N && !(at[cut].first >= 0 && at[(cut + N - 1) % N].first < 0)) ++cut;
    // without a gap: slot 0 is the lowest box's first plane, so that one box
    // whose padding wraps the grid starts at slot 0
    if (cut == N) cut = globz(box[bs[0]], 0);
    Ring r;
    r.boxes = bs;
    std::vector<int32_t> slot(N, -1);
    for (int64_t i = 0; i < N; ++i) {
      const int64_t G = (cut + i) % N;
      if (at[G].first < 0) continue;
      slot[G] = (int32_t)r.slot.size();
      r.slot.push_back(at[G]);
    }
    bool once = true;
    for (int s : bs) once = once && slot[globz(box[s], 0)] + box[s].P[2] <= 2 * (int64_t)r.slot.size();
    if (!once) {
      for (int s : bs) alone(s);
      continue;
    }
    for (int s : bs) {
      BoxD& b = box[s];
      b.ring = (int32_t)r.slot.size();
      b.zb = slot[globz(b, 0)];
      // planes other boxes read: they come in from the low end, the high end
      // or, past a box thinner than the guards, from both
      auto shared = [&](int i) { return readers[globz(b, b.g[2] + i)] > 1; };
      int lo = 0, hi = 0;
      while (lo < b.n[2] && shared(lo)) ++lo;
      while (hi < b.n[2] - lo && shared(b.n[2] - 1 - hi)) ++hi;
      b.slo = lo;
      b.shi = hi;
    }
    rings.push_back(std::move(r));
  }
  return rings;
}

// Pencils per heat z tile: the widest of 32, 16 and 8 of which four 256-thread
// tiles (16 waves) fit a compute unit's LDS, else 4; narrower while that leaves
// compute units without a tile.  Four steps with 4, 8, 16, 32 pencils (us), one box,
// FP32: 16 16 256 94, 97, 106, 139; 24 24 128 93, 94, 97, 110; 64^3 114, 112, 110,
// 117; 96^3 187, 163, 163, 171; FP64: 48^3 110, 109, 110, 116; 64^3 150, 128, 128,
// 137; more tiles, 27 boxes of 48^3 padded, FP32: 354, 259, 205, 200.
inline int heat_pencils(const HostTables& h) {
  const int Pz = max_padded_z(h), rb = (int)real_size(h.prec);
  int PB = 32;
  while (PB > 4 && 4 * heat_tile_lds(Pz, PB, rb) > kMaxDynLds) PB /= 2;
  auto tiles = [&] {
    int64_t n = 0;
    for (const BoxD& b : h.box) n += ((int64_t)b.P[1] * b.H + PB - 1) / PB;
    return n;
  };
  while (PB > 4 && tiles() < kComputeUnits) PB /= 2;
  return PB;
}

// Fills h.lists for the current batches and z tile.  share: columns share
// their planes (one batch only); xy_classes / z_classes: one launch per class.
inline void build_lists(HostTables& h, bool share, bool xy_classes, bool z_classes) {
  WorkLists w;
  w.box = h.box;
  const std::vector<Ring> rings = build_rings(h, w.box, share);
  w.tight = w.box;
  // Spectral addresses: the rings' 9 fields, then the shared planes' results.
  // Back to back the planes take at most 9 sum P[2] P[1] H (the results are at
  // most the guard planes saved).  The z pass walks from plane to plane, so a
  // pitch of many 1 KiB steps sends a tile to few memory channels: line-aligned
  // pitches, one line longer where they would be a multiple of 8 lines, took
  // the z pass of one 256^3 box (2064 lines) from 0.62 to 0.40 ms in FP32.
  const int64_t line = 128 / (int64_t)(2 * real_size(h.prec));
  auto spread = [&](int64_t pl) {
    const int64_t lines = (pl + line - 1) / line;
    return (lines % 8 ? lines : lines + 1) * line;
  };
  auto place = [&](std::vector<BoxD>& box, bool pitched) {
    int64_t at = 0;
    for (const Ring& r : rings) {
      const BoxD& b0 = box[r.boxes[0]];
      const int64_t pl = (int64_t)b0.P[1] * b0.H, pp = pitched ? spread(pl) : pl;
      for (int s : r.boxes) {
        box[s].pp = pp;
        box[s].sb = at;
        box[s].sv = pp * (int64_t)r.slot.size();
      }
      at += 9 * pp * (int64_t)r.slot.size();
      for (int s : r.boxes) {
        box[s].xb = at;
        box[s].xv = pp * (box[s].slo + box[s].shi);
        at += 6 * box[s].xv;
      }
    }
    return at;
  };
  w.elems = place(w.box, share);
  w.tight_elems = place(w.tight, false);
  // guard pieces per run of planes with the same ones
  std::vector<std::vector<std::array<int32_t, 2>>> runs(h.nsub);  // per plane [p0, p1)
  for (int s = 0; s < h.nsub; ++s) {
    std::vector<int32_t> prev;
    for (int z = 0; z < h.box[s].P[2]; ++z) {
      std::vector<int32_t> cur;
      for (int i = h.pull_off[s]; i < h.pull_off[s + 1]; ++i)
        if (z >= h.pullp[i].qz && z < h.pullp[i].qz + h.pullp[i].lz) cur.push_back(i);
      if (z == 0 || cur != prev) {
        const int32_t p0 = (int32_t)w.pull.size();
        for (int i : cur) w.pull.push_back(h.pullp[i]);
        runs[s].push_back({p0, (int32_t)w.pull.size()});
        prev = cur;
      } else {
        runs[s].push_back(runs[s].back());
      }
    }
  }
  // The inverse pass in two halves: FP32 planes beyond the LDS of which half fits
  // it and a quarter fits the registers set aside for it.  A plane is one group and
  // fills a compute unit, so the pass takes whole rounds of planes, where the split
  // passes have some 16 short groups for each.  So only where the rounds are full
  // enough on average: 0.67 (in a single round 0.55) if every transform takes two
  // stages, else 0.75 (a lone group exposes the barriers of each stage).  A step in
  // halves against one split, one box of 200^2 to 512 x 96: 1 to 4 planes (0.02 to
  // 0.09 of a round) 1.13 to 1.32; 16 (0.38) 0.99 to 1.11; 48 (two rounds, 0.56) 1.00
  // to 1.09.  Two stages: 24 planes (0.56) 0.95 to 1.01, 0.66 to 0.75 0.90 to 1.01.
  // Three: 0.70 0.94 to 1.04; 0.75 to 0.78 0.90 to 1.04, below 1 on average; 0.82 to
  // 0.98 0.88 to 1.00.
  auto two_stages = [](int N) {
    std::vector<int> r;
    return factorize(N, r, 16) && r.size() <= 2;
  };
  auto halve = [&](const std::vector<char>& in) {
    if (h.prec != PSATD_F32_VALU || h.fuse_eb || h.ldsF <= kMaxDynLds) return 0;
    int half = 0, quarter = 0;
    int64_t groups = 0;  // planes of the 6 fields
    bool two = true;
    for (int s = 0; s < h.nsub; ++s) {
      if (!in[s]) continue;
      const BoxD& b = h.box[s];
      groups += 6 * b.n[2];
      two = two && two_stages(b.P[0] / 2) && two_stages(b.P[1]);
      half = std::max(half, (half_elems(b.P[1], b.ld, b.H) + b.P[0] / 2 + b.P[1] + b.P[0]) * 8 +
                                (b.P[0] / 2 + b.P[1]) * 4);
      quarter = std::max(quarter, (b.P[1] + 1) / 2 * half_cols(b.H));
    }
    const int64_t places = (groups + kComputeUnits - 1) / kComputeUnits * kComputeUnits;
    const int least = !two ? 75 : (places == kComputeUnits ? 55 : 67);
    if (100 * groups < least * places) return 0;
    return half <= kMaxDynLds && quarter <= kHalfHold * kThreadsHalf ? half : 0;
  };
  auto add_planes = [&](const std::vector<char>& in, XyLaunch& l) {
    l.half = halve(in);
    std::vector<PlaneRec> fwd, inv;
    for (const Ring& r : rings) {
      if (!in[r.boxes[0]]) continue;  // the boxes of a ring have the same plane size
      for (const auto& p : r.slot)
        fwd.push_back({p.first, p.second, runs[p.first][p.second][0], runs[p.first][p.second][1]});
    }
    for (int s = 0; s < h.nsub; ++s)
      if (in[s])
        for (int z = 0; z < h.box[s].n[2]; ++z) inv.push_back({s, z, 0, 0});
    // the planes, or (split passes) their blocks of `per` of len(box) rows or columns
    auto put = [&](std::vector<PlaneRec>& to, const std::vector<PlaneRec>& v, int32_t& at, int32_t& count, bool blocks,
                   int per, auto len) {
      at = (int32_t)to.size();
      for (PlaneRec r : v) {
        if (!blocks) to.push_back(r);
        else
          for (r.p0 = 0; r.p0 < len(h.box[r.box]); r.p0 += per) to.push_back(r);
      }
      count = (int32_t)to.size() - at;
    };
    put(w.fwd, fwd, l.f0, l.nf, h.split, kRB, [](const BoxD& b) { return b.P[1]; });
    put(w.inv, inv, l.i0, l.ni, h.split && !l.half, kRB, [](const BoxD& b) { return b.n[1]; });
    if (!h.split) return;
    put(w.fwd, fwd, l.c0, l.nc, true, kCB, [](const BoxD& b) { return b.H; });
    if (!l.half) put(w.inv, inv, l.d0, l.nd, true, kCB, [](const BoxD& b) { return b.H; });
  };
  // tiles of a column side by side at the same pencils, so that the planes
  // its boxes share are read by neighbouring work-groups
  auto add_tiles = [&](const std::vector<char>& in, ZLaunch& l) {
    l.u0 = (int32_t)w.tiles.size();
    for (const Ring& r : rings) {
      const BoxD& b = h.box[r.boxes[0]];
      for (int q = 0; q < b.P[1] * b.H; q += l.PB)
        for (int s : r.boxes)
          if (in[s]) w.tiles.push_back({s, q});
    }
    l.nu = (int32_t)w.tiles.size() - l.u0;
    // Short z: 512-thread tiles are two per compute unit in FP32 and one in FP64
    // (registers) however small they are, and a short tile has no work for all
    // their waves.  256 threads where that puts more tiles on a compute unit (the
    // LDS holds three FP32 or two FP64 ones) and the launch takes more than one
    // round of 512-thread tiles.  Measured, 512 -> 256 threads: 512 boxes of 48^3
    // padded 1.23 -> 0.87 ms FP32, 2.90 -> 1.88 FP64; 216 of 64^3 1.01 -> 0.95,
    // 2.35 -> 1.68; 80^3 (two and one tile) 0.60 -> 0.74, 1.31 -> 1.61 ms, so not
    // there; one round of 68 FP64 tiles of 32-long z 9.8 -> 11.1 us, nor there.
    const bool f64 = is_f64(h.prec);
    l.narrow = kMaxDynLds / l.lds >= (f64 ? 2 : 3) && l.nu > (f64 ? 256 : 512);
  };
  // FP64 tiles of which one fills the LDS: with J's transform in registers two
  // 256-thread tiles share a compute unit, where they fit and every pair +-kz has its
  // thread (8 pencils to padded z 103, 4 to 202).  Measured, nine fields in the LDS ->
  // held: 64 boxes of 96^3 padded 2.07 -> 1.71 ms, 8 of 176^3 2.02 -> 1.57, 16 of
  // 96 96 80 0.51 -> 0.42, 28 of 96 96 144 1.75 -> 1.46, 32 of 96 96 192 2.72 -> 2.16;
  // one box of 264 tiles 34 -> 29 us, 588 54 -> 49.  One round of 512-thread tiles
  // (256) keeps its nine fields.  For 112- and 128-long z, where held tiles have 6 or 4
  // pencils, the full tiles of 8 are faster (0.76 against 0.85 ms, 0.97 against
  // 1.13).  FP32 has no registers left for it: 0.89 -> 1.10 ms.
  auto hold_j = [&](const std::vector<char>& in, ZLaunch& l) {
    if (!is_f64(h.prec) || h.ntu != 512 || l.narrow || (l.PB != 4 && l.PB != 8)) return;
    int Pz = 0;
    for (int s = 0; s < h.nsub; ++s)
      if (in[s]) Pz = std::max(Pz, (int)h.box[s].P[2]);
    const int64_t lds = held_tile_lds(Pz, l.PB, (int)real_size(h.prec));
    if (2 * lds > kMaxDynLds || (Pz / 2 + 1) * l.PB > kHeldPairs * kThreadsHeld || l.nu <= 256) return;
    l.held = 1;
    l.lds = (int32_t)lds;
  };
  for (const Batch& bt : h.batches) {
    w.xy.emplace_back();
    w.z.emplace_back();
    std::vector<char> in(h.nsub, 0);
    if (xy_classes) {
      for (const XyClass& k : h.xyc) {
        const int32_t* F = h.itemsXYC.data() + k.F;
        for (int s = 0; s < h.nsub; ++s) in[s] = F[s + 1] > F[s];
        XyLaunch l{k.nt, k.lds};
        add_planes(in, l);
        w.xy.back().push_back(l);
      }
    } else {
      for (int s = 0; s < h.nsub; ++s) in[s] = s >= bt.b0 && s < bt.b1;
      XyLaunch l{h.ntxy, h.ldsF};
      add_planes(in, l);
      w.xy.back().push_back(l);
    }
    if (z_classes) {
      for (const ZClass& k : h.zcls) {
        const int32_t* U = h.itemsZC.data() + k.U;
        for (int s = 0; s < h.nsub; ++s) in[s] = U[s + 1] > U[s];
        ZLaunch l{k.PB, k.lds};
        add_tiles(in, l);
        hold_j(in, l);
        w.z.back().push_back(l);
      }
    } else {
      for (int s = 0; s < h.nsub; ++s) in[s] = s >= bt.b0 && s < bt.b1;
      ZLaunch l{h.PB, h.ldsU};
      add_tiles(in, l);
      hold_j(in, l);
      w.z.back().push_back(l);
    }
  }
  if (h.batches.size() == 1) {
    std::vector<char> in(h.nsub, 1);
    w.heat.PB = heat_pencils(h);
    w.heat.lds = (int32_t)heat_tile_lds(max_padded_z(h), w.heat.PB, (int)real_size(h.prec));
    add_tiles(in, w.heat);
  }
  h.lists = std::move(w);
}

// Bytes of the spectral workspace that every layout has room for: one batch's half
// spectra of 9 fields, each box's planes its own and back to back.
inline int64_t workspace_bytes(const HostTables& h) {
  return 9 * h.batch_slab * (int64_t)(2 * real_size(h.prec));
}

// Bytes that the fastest layout takes: an unbatched plan's shared planes at pitches of
// their own, which may be more.  A batched plan runs in one batch's planes back to back.
inline int64_t roomy_workspace_bytes(const HostTables& h) {
  return h.batches.size() == 1 ? h.lists.elems * (int64_t)(2 * real_size(h.prec)) : workspace_bytes(h);
}

// Deposited currents: every box interior cut, along each axis, where the set of
// padded copies changes; the regions with more than one copy (boxes ascending,
// then z, y, x positions ascending).
inline void build_sum(HostTables& h) {
  const int V = 16 / (int)real_size(h.prec);  // elements per 16-byte access
  h.sumr.clear();
  h.sumc.clear();
  h.itemsS.assign(1, 0);
  h.regionOf.clear();
  struct Meet {
    int d;
    std::vector<Run> r[3];  // x, y, z
  };
  for (int s = 0; s < h.nsub; ++s) {
    const BoxD& a = h.box[s];
    std::vector<Meet> meets;
    std::vector<int32_t> cut[3];
    for (int u = 0; u < 3; ++u) cut[u] = {0, a.n[u]};
    for (int d = 0; d < h.nsub; ++d) {
      const BoxD& b = h.box[d];
      Meet m;
      m.d = d;
      bool any = true;
      for (int u = 2; u >= 0 && any; --u) {
        axis_runs(a.lo[u], a.n[u], b.lo[u], b.g[u], b.P[u], h.N[u], m.r[u]);
        any = !m.r[u].empty();
      }
      if (!any) continue;
      for (int u = 0; u < 3; ++u)
        for (const Run& r : m.r[u]) {
          cut[u].push_back(r.i0);
          cut[u].push_back(r.i0 + r.len);
        }
      meets.push_back(std::move(m));
    }
    for (int u = 0; u < 3; ++u) {
      std::sort(cut[u].begin(), cut[u].end());
      cut[u].erase(std::unique(cut[u].begin(), cut[u].end()), cut[u].end());
    }
    for (size_t iz = 0; iz + 1 < cut[2].size(); ++iz)
      for (size_t iy = 0; iy + 1 < cut[1].size(); ++iy)
        for (size_t ix = 0; ix + 1 < cut[0].size(); ++ix) {
          const int x0 = cut[0][ix], y0 = cut[1][iy], z0 = cut[2][iz];
          SumRegion g{};
          g.c0 = (int32_t)h.sumc.size();
          g.ly = cut[1][iy + 1] - y0;
          g.lx = cut[0][ix + 1] - x0;
          bool vec = g.lx % V == 0;
          auto covers = [](const Run& r, int i) { return i >= r.i0 && i < r.i0 + r.len; };
          for (const Meet& m : meets) {
            const BoxD& b = h.box[m.d];
            for (const Run& rz : m.r[2]) {
              if (!covers(rz, z0)) continue;
              for (const Run& ry : m.r[1]) {
                if (!covers(ry, y0)) continue;
                for (const Run& rx : m.r[0]) {
                  if (!covers(rx, x0)) continue;
                  SumCopy c;
                  c.sP0 = b.P[0];
                  c.sPl = b.P[0] * b.P[1];
                  c.off = b.foff + ((int64_t)(rz.q0 + z0 - rz.i0) * b.P[1] + (ry.q0 + y0 - ry.i0)) * b.P[0] +
                          (rx.q0 + x0 - rx.i0);
                  vec = vec && c.off % V == 0 && c.sP0 % V == 0 && c.sPl % V == 0;
                  h.sumc.push_back(c);
                }
              }
            }
          }
          g.nc = (int32_t)h.sumc.size() - g.c0;
          if (g.nc < 2) {  // the owner's cells alone
            h.sumc.resize(g.c0);
            continue;
          }
          g.vec = vec;
          h.itemsS.push_back(h.itemsS.back() + cut[2][iz + 1] - z0);
          h.regionOf.resize(h.itemsS.back(), (int32_t)h.sumr.size());
          h.sumr.push_back(g);
        }
  }
}

inline psatd_status build_host(HostTables& h, std::string& err, const int64_t grid_n[3],
                        const double grid_d[3], int32_t nsub, const int64_t* lo, const int64_t* n,
                        const int32_t* guard, int32_t order_p, double dt, double c,
                        int32_t precision, int32_t jmode) {
  auto bad = [&](psatd_status st, const std::string& m) {
    err = m;
    return st;
  };
  if (!grid_n || !grid_d || !lo || !n || !guard) return bad(PSATD_E_INVALID, "null pointer argument");
  if (nsub < 1) return bad(PSATD_E_INVALID, "nsub must be >= 1");
  for (int u = 0; u < 3; ++u) {
    if (grid_n[u] < 1 || grid_n[u] > (1 << 24)) return bad(PSATD_E_INVALID, "grid_n out of range");
    if (!(grid_d[u] > 0.0) || !std::isfinite(grid_d[u])) return bad(PSATD_E_INVALID, "grid_d must be finite and > 0");
  }
  if (order_p < 0 || (order_p % 2) != 0 || order_p == 1)
    return bad(PSATD_E_INVALID, "order_p must be 0 (infinite) or even >= 2");
  if (!(dt != 0.0) || !std::isfinite(dt)) return bad(PSATD_E_INVALID, "dt must be finite and nonzero");
  if (!(c > 0.0) || !std::isfinite(c)) return bad(PSATD_E_INVALID, "c must be finite and > 0");
  if (precision < PSATD_F64 || precision > PSATD_F32_BF16X6) return bad(PSATD_E_INVALID, "unknown precision");
  if (jmode != PSATD_J_REPLICATED && jmode != PSATD_J_DEPOSITED) return bad(PSATD_E_INVALID, "unknown jmode");

  for (int u = 0; u < 3; ++u) {
    h.N[u] = grid_n[u];
    h.d[u] = grid_d[u];
  }
  h.nsub = nsub;
  h.p = order_p;
  h.dt = dt;
  h.c = c;
  h.prec = precision;
  h.jmode = jmode;
  h.spl = precision == PSATD_F32_BF16X3 ? 2 : (precision == PSATD_F32_BF16X6 ? 3 : 0);

  // boxes inside the grid, guards >= 0
  for (int s = 0; s < nsub; ++s)
    for (int u = 0; u < 3; ++u) {
      const int64_t l = lo[3 * s + u], m = n[3 * s + u];
      if (m < 1 || l < 0 || l + m > grid_n[u]) return bad(PSATD_E_INVALID, "box " + std::to_string(s) + " outside the grid");
      if (guard[3 * s + u] < 0) return bad(PSATD_E_INVALID, "negative guard width");
      if (m + 2 * (int64_t)guard[3 * s + u] > (1 << 20)) return bad(PSATD_E_INVALID, "padded length too large");
    }
  // refined cuts and owner table: exact tiling
  for (int u = 0; u < 3; ++u) {
    std::vector<int64_t> pts{0, grid_n[u]};
    for (int s = 0; s < nsub; ++s) {
      pts.push_back(lo[3 * s + u]);
      pts.push_back(lo[3 * s + u] + n[3 * s + u]);
    }
    std::sort(pts.begin(), pts.end());
    pts.erase(std::unique(pts.begin(), pts.end()), pts.end());
    h.ncut[u] = (int32_t)pts.size() - 1;
    h.cut[u].assign(grid_n[u], 0);
    for (int i = 0; i < h.ncut[u]; ++i)
      for (int64_t x = pts[i]; x < pts[i + 1]; ++x) h.cut[u][x] = i;
  }
  const int64_t ncell = (int64_t)h.ncut[0] * h.ncut[1] * h.ncut[2];
  if (ncell > (int64_t)1 << 26) return bad(PSATD_E_UNSUPPORTED, "decomposition too fine");
  h.owner.assign(ncell, -1);
  for (int s = 0; s < nsub; ++s) {
    int c0[3], c1[3];
    for (int u = 0; u < 3; ++u) {
      c0[u] = h.cut[u][lo[3 * s + u]];
      c1[u] = h.cut[u][lo[3 * s + u] + n[3 * s + u] - 1] + 1;
    }
    for (int cz = c0[2]; cz < c1[2]; ++cz)
      for (int cy = c0[1]; cy < c1[1]; ++cy)
        for (int cx = c0[0]; cx < c1[0]; ++cx) {
          int32_t& o = h.owner[((int64_t)cz * h.ncut[1] + cy) * h.ncut[0] + cx];
          if (o != -1) return bad(PSATD_E_INVALID, "boxes " + std::to_string(o) + " and " + std::to_string(s) + " overlap");
          o = s;
        }
  }
  for (int32_t o : h.owner)
    if (o < 0) return bad(PSATD_E_INVALID, "boxes leave part of the grid uncovered");

  // per box: padded extents, FFT plans, tables, offsets
  const bool f64 = is_f64(precision);
  const int csz = (int)(2 * real_size(precision));
  std::vector<std::pair<int, int>> twcache;
  h.box.resize(nsub);
  int64_t foff = 0, soff = 0;
  int maxPz = 0;
  for (int s = 0; s < nsub; ++s) {
    BoxD& b = h.box[s];
    std::memset(&b, 0, sizeof(b));
    for (int u = 0; u < 3; ++u) {
      b.lo[u] = (int32_t)lo[3 * s + u];
      b.n[u] = (int32_t)n[3 * s + u];
      b.g[u] = guard[3 * s + u];
      b.P[u] = b.n[u] + 2 * b.g[u];
      if (!small_primes_only(b.P[u]))
        return bad(PSATD_E_UNSUPPORTED, "padded length " + std::to_string(b.P[u]) + " has a prime factor > 11");
    }
    if (b.P[0] % 2) return bad(PSATD_E_UNSUPPORTED, "padded x length must be even");
    b.H = b.P[0] / 2 + 1;
    b.ld = (b.H % 2) ? b.H : b.H + 1;
    b.planx = add_plan(h, b.P[0] / 2, false);
    b.plany = add_plan(h, b.P[1], false);
    b.planz = add_plan(h, b.P[2], true);
    if (b.planx < 0 || b.plany < 0 || b.planz < 0)
      return bad(PSATD_E_UNSUPPORTED, "no radix schedule of <= 4 stages for a padded length");
    b.twr = add_twiddle(h, b.P[0], twcache);
    b.kx = add_kentry(h, b.P[0], grid_d[0]);
    b.ky = add_kentry(h, b.P[1], grid_d[1]);
    b.kz = add_kentry(h, b.P[2], grid_d[2]);
    // The box starts where its first interior x cell begins a 128-byte line
    // (to within the 16 bytes that keep vector accesses aligned): then the
    // interior rows, and the guard rows pulled from them, are whole lines
    // whenever the row pitch is.  The gap costs under 128 bytes per box.
    {
      const int64_t line = 128 / (int64_t)real_size(precision), vec = 16 / (int64_t)real_size(precision);
      const int64_t t = (line - b.g[0] % line) % line;
      const int64_t want = (t + vec - 1) / vec * vec % line;
      foff += ((want - foff) % line + line) % line;
    }
    b.foff = foff;
    b.soff = soff;
    b.svol = (int64_t)b.H * b.P[1] * b.P[2];
    foff += (int64_t)b.P[0] * b.P[1] * b.P[2];
    soff += (int64_t)b.H * b.P[1] * b.P[2];
    // plane + twiddles of the x plan, the y plan and W_Px + position tables
    h.boxlds.push_back((b.P[1] * b.ld + b.P[0] / 2 + b.P[1] + b.P[0]) * csz + (b.P[0] / 2 + b.P[1]) * 4);
    h.ldsF = std::max<int>(h.ldsF, h.boxlds.back());
    h.ldsI = h.ldsF;
    maxPz = std::max(maxPz, b.P[2]);
  }
  if (h.twr.size() > (size_t)INT32_MAX / 2)
    return bad(PSATD_E_UNSUPPORTED, "tables too large");
  h.field_elems = foff;
  h.slab = soff;
  // planes that do not fit the LDS take the split x-row / y-column passes
  h.split = h.ldsF > kMaxDynLds;
  for (const BoxD& b : h.box) {
    h.ldsX = std::max<int>(h.ldsX, (kRB * b.ld + b.P[0] / 2 + b.P[0]) * csz + (b.P[0] / 2) * 4);
    h.ldsY = std::max<int>(h.ldsY, (b.P[1] * kCB + b.P[1]) * csz + b.P[1] * 4);
  }
  if (h.ldsX > kMaxDynLds || h.ldsY > kMaxDynLds)
    return bad(PSATD_E_UNSUPPORTED, "padded lengths too large for the split x/y passes");
  // z-update tile: PB consecutive (ky, kx) pencils (128-byte rows when possible)
  {
    // Two FP32 tiles per CU, so one tile's loads overlap the other's
    // transforms, each as wide as two still fit (z_pencils_for: 10 pencils for
    // 96-long z, 6 for 176; one 8-pencil tile of 176 would fill a CU alone, and
    // 4 pencils took configuration 5's z pass 35.5 -> 30.4 ms, 6 to 26.5 ms).
    // FP64 keeps 8: its 4-pencil tiles measured slower on 96^3 boxes.
    int PB = 8;
    while (PB > 4 && !z_tile_fits(h, maxPz, PB)) PB /= 2;
    if (!f64 && PB == 8) {
      const int own = z_pencils_for(h, maxPz);
      if (own) PB = own;
    }
    if (!z_tile_fits(h, maxPz, PB))
      return bad(PSATD_E_UNSUPPORTED, "padded z length too large for the z-update kernel");
    h.PB = PB;
  }

  // work lists
  auto prefix = [&](std::vector<int32_t>& v, auto count) {
    v.assign(nsub + 1, 0);
    for (int s = 0; s < nsub; ++s) v[s + 1] = v[s] + (int32_t)count(h.box[s]);
  };
  prefix(h.itemsF, [](const BoxD& b) { return (int64_t)b.P[2] * 9; });
  set_z_tile(h, h.PB);
  prefix(h.itemsI, [](const BoxD& b) { return (int64_t)b.n[2] * 6; });
  prefix(h.itemsP, [](const BoxD& b) { return (int64_t)b.P[2]; });
  prefix(h.itemsN, [](const BoxD& b) { return (int64_t)b.n[2]; });
  build_push(h);
  if (jmode == PSATD_J_DEPOSITED) build_sum(h);
  build_zreg(h);
  set_batches(h, 0);
  // launch-shape defaults (measured on 96^3 and 176^3 boxes): x/y groups of
  // the fewest threads that still keep 16 waves on a CU given how many planes
  // fit its LDS (96^3 FP32: four 40 KB planes x 256 threads; 176^3 FP32: one
  // 127 KB plane x 1024 threads); 512-thread z tiles of 8 pencils; FP64
  // x/y stages of radix <= 8 where a plane fits the LDS (radix 16 measured
  // slower there: 2.41 -> 3.66 ms on 96^3 boxes), radix 16 in the split x/y
  // passes and the z pass (faster: z pass 2.93 -> 2.59 ms on 96^3 boxes,
  // 176^3 steps 221-227 -> 215 ms)
  h.ntu = 512;
  h.ntxy = xy_threads_for(h.ldsF);
  build_xy_classes(h);
  build_z_classes(h);
  if (f64 && !h.split && !set_max_radix(h, 8, 16)) return bad(PSATD_E_UNSUPPORTED, "no radix-8 schedule");
  return PSATD_OK;
}

}  // namespace psatd
