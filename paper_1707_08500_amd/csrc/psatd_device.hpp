// Device data structures and kernel bodies of the local-FFT PSATD step.
//
// Bodies are __host__ __device__ templates taking (work item, thread id,
// thread count, LDS pointer, barrier) so that the same code runs in the
// __global__ wrappers of psatd_kernels.hip.
#pragma once
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "fft_engine.hpp"

namespace psatd {

// Launch shapes (gfx950: 64-wide waves, 160 KiB LDS per compute unit).
constexpr int kThreadsXY = 256;   // x/y plane passes, exchange, scatter/gather
constexpr int kThreadsHalf = 1024;  // inverse x/y pass over planes in two halves
constexpr int kMaxR = 16;         // largest radix codelet (radix 11 is always available)
constexpr int kMaxDynLds = 160 * 1024;
constexpr int kComputeUnits = 256;

// One padded subdomain (Sec. 3.2, Fig. 2a).  Axes (x, y, z).
struct BoxD {
  int32_t lo[3];   // first owned global cell
  int32_t n[3];    // owned cells
  int32_t g[3];    // guard cells per side
  int32_t P[3];    // padded extents n + 2 g
  int32_t H;       // P[0]/2 + 1 (half-spectrum length along x)
  int32_t ld;      // LDS row stride (complex elements) of an (x, y) plane
  int32_t planx;   // FFT plan of length P[0]/2 (packed real rows)
  int32_t plany;   // FFT plan of length P[1]
  int32_t planz;   // FFT plan of length P[2]
  int32_t twr;     // offset of the W_{P[0]}^e table (real <-> half spectrum)
  int32_t kx, ky, kz;  // offsets of the FP64 modified-wavenumber tables
  int32_t ring;    // planes of the box's spectral ring (below)
  int32_t zb;      // ring slot of padded plane 0
  int32_t slo, shi;  // interior planes at the low / high end that other boxes read
  int64_t foff;    // element offset of the box in a field buffer
  int64_t soff;    // sum of the half-spectrum sizes of the boxes before it
  int64_t svol;    // half-spectrum size of one field of the box, P[2] P[1] H (complex)
  int64_t sb, sv;  // spectral ring: offset of field 0, field stride (complex)
  int64_t pp;      // spectral plane pitch (complex), at least P[1] H
  int64_t xb, xv;  // results of the shared planes: offset of field 0, field stride
};

// The spectral workspace holds rings of (ky, kx) planes.  Boxes with the same
// x/y extent and x/y guards (a column of the decomposition) have the same
// padded (x, y) plane wherever their padded z ranges meet: a z-guard plane is
// the neighbour's interior plane, cell for cell.  So a column shares one ring
// of its distinct z-planes, each transformed once along x and y, and the z
// pass of a box reads its P[2] consecutive slots zb, zb + 1, ... (mod ring).
// A ring holds the 9 fields back to back, field f at sb + f sv, [slot][ky][kx]
// each, planes pp elements apart.  The z pass writes the E and B results over the spectra of the box's
// interior planes, except the planes that other boxes of the column still read:
// those results go to the box's own slots after the ring's fields (slo planes
// of the low end, then shi of the high end; 6 fields at xb + f xv).  A box that
// shares with no other is a ring of its own P[2] planes.
template <typename T>
PSATD_HD cx<T>* spec_at(cx<T>* spec, const BoxD& bx, int64_t sbias, int f) {
  return spec + (bx.sb - sbias) + f * bx.sv;
}
template <typename T>
PSATD_HD const cx<T>* spec_at(const cx<T>* spec, const BoxD& bx, int64_t sbias, int f) {
  return spec + (bx.sb - sbias) + f * bx.sv;
}

// Ring slot of padded plane z (zb + z < 2 ring, checked at plan time).
PSATD_HD int ring_slot(const BoxD& bx, int z) {
  const int s = bx.zb + z;
  return s >= bx.ring ? s - bx.ring : s;
}

// Offset of the result of field f at interior plane i (relative to the
// workspace's first element).
PSATD_HD int64_t result_plane(const BoxD& bx, int64_t sbias, int f, int i) {
  const int h = i - (bx.n[2] - bx.shi);
  if (i < bx.slo) return bx.xb - sbias + f * bx.xv + i * bx.pp;
  if (h >= 0) return bx.xb - sbias + f * bx.xv + (bx.slo + h) * bx.pp;
  return bx.sb - sbias + f * bx.sv + ring_slot(bx, bx.g[2] + i) * bx.pp;
}

// One (x, y) plane of the x/y passes' work lists.  Forward: padded plane z of
// the box, with its guard pieces [p0, p1) of the pull list; inverse: interior
// plane z.  Split passes: a block of the plane's rows or columns from p0 on.
struct PlaneRec {
  int32_t box, z, p0, p1;
};

// One z tile: the pencils q0, q0 + 1, ... of a box.
struct ZItem {
  int32_t box, q0;
};

// Launches of the x/y and z passes: ranges of the plane and tile lists with
// their group size or tile width and their dynamic LDS.
struct XyLaunch {
  int32_t nt, lds, f0, nf, i0, ni;  // forward planes [f0, f0 + nf), inverse [i0, i0 + ni)
  int32_t half;                     // LDS of the inverse pass in two halves (0: not taken)
  int32_t c0, nc, d0, nd;           // split passes: forward and inverse column blocks
};
struct ZLaunch {
  int32_t PB, lds, u0, nu;
  int32_t narrow;  // 1: tiles of 256 threads instead of 512
  int32_t held;    // 1: tiles that hold J's transform in registers (body_z_held)
};

// A batch of boxes [b0, b1) for the FFT/update passes and the spectral offset
// of box b0 (the workspace holds the batch only).
struct Batch {
  int32_t b0, b1;
  int64_t sbias;
};

// One rectangular piece of a box interior that is also a guard region of a
// padded box (a neighbour's, or the box's own when its padding wraps the
// grid): interior cells [z0, z0+lz) x [y0, y0+ly) x [x0, x0+lx) of the source
// box are the padded cells starting at (qz, qy, qx) of box dst.  Every guard
// cell of every box lies in exactly one piece of exactly one source box.
struct PushBlk {
  int32_t src, dst;
  int32_t z0, lz, qz;
  int32_t y0, ly, qy;
  int32_t x0, lx, qx;
};

// Register z pass: the padded z lengths with a register schedule, as
// X(N, lanes per transform, waves per work-group, min waves per SIMD).
#define PSATD_ZREG_SHAPES(X) \
  X(96, 2, 4, 2)             \
  X(176, 4, 4, 2)

// A group of boxes sharing one padded z length: its work list is
// itemsZR[off .. off + nsub] (a prefix over all boxes, zero for the others).
struct ZGroup {
  int32_t N, off, n, pad_;
};
constexpr int kMaxZGroups = 8;

// A launch class of the x/y passes: the boxes whose padded planes fit the
// same number of times into a compute unit's LDS, run with their own group
// size and dynamic LDS.  Its counts are prefixes over all boxes (zero for the
// boxes of other classes, which is how its boxes are told) at the given offsets
// of one table: planes of the 9 fields (F), of one field (P), interior planes of
// the 6 outputs (I) and of one output (N), with their totals.
struct XyClass {
  int32_t nt, lds;
  int32_t F, nF, P, nP, I, nI, N, nN;
};
constexpr int kMaxXyClasses = 3;

// A launch class of the z pass: the boxes whose z tile takes the same number
// of pencils (FP32: the widest of 10, 8, 6 of which two tiles fit a compute
// unit's LDS, else 4; FP64: 8 where one tile fits, else 4), launched with the
// LDS of the class's longest padded z.  Its tiles are counted by a prefix over all
// boxes (zero for the others) at offset U of one table.
struct ZClass {
  int32_t PB, lds, U, nU;
};
constexpr int kMaxZClasses = 4;

// Pencils per work-group of the register z pass (9 fields share its lanes).
constexpr int zreg_pencils(int L, int W) { return (64 * W / L) / 9; }

// Work list: item -> box by binary search in a prefix array (size nsub + 1).
PSATD_HD int find_box(const int32_t* prefix, int nsub, int item) {
  int lo = 0, hi = nsub;  // prefix[lo] <= item < prefix[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (prefix[mid] <= item) lo = mid; else hi = mid;
  }
  return lo;
}

PSATD_HD int pmod(int v, int N) {
  int r = v % N;
  return r < 0 ? r + N : r;
}

// Tables shared by all passes.
template <typename T>
struct Tables {
  const BoxD* box;
  int32_t nsub;
  const FftPlanD* plans;
  const cx<T>* tw;        // twiddle tables (forward sign)
  const int32_t* pos;     // position tables (stage-digit order)
  const double* kmod;     // modified wavenumbers (FP64)
};

// Buffer resource over `bytes` bytes at base (raw, untyped; the third word
// selects 32-bit elements on this GPU family).  Accesses at or beyond `bytes`
// read zeros and write nothing.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// One complex FP32 value at byte offset voff + soff (soff wave-uniform).
__device__ __forceinline__ void buf_load(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff, cx<float>* v) {
  const u32x2 w = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)voff, (int)soff, 0);
  __builtin_memcpy(v, &w, sizeof(w));
}

// Copies total elements i -> dst(i, src(i)) with U loads in flight per
// thread (all U loads are issued before the first store).
template <int U, typename V, class Src, class Dst>
PSATD_HD void copy_batched(int total, int tid, int nt, Src src, Dst dst) {
  for (int base = tid; base < total; base += U * nt) {
    V v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = base + u * nt;
      if (i < total) v[u] = src(i);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = base + u * nt;
      if (i < total) dst(i, v[u]);
    }
  }
}

// Two neighbouring values accessed as one vector (aligned to its size, at
// most 16 bytes: the widest single access).
template <typename V>
struct alignas(2 * sizeof(V) < 16 ? 2 * sizeof(V) : 16) Pair {
  V a, b;
};

// Row-major R x C walk shared by a work-group: element i = tid + k nt, with
// its (row, col) advanced incrementally (no per-element division), in
// batches of U whose U loads are all issued before the first store; full
// batches run without bounds checks.  The remainder (fewer than U per
// thread) runs one element at a time, or with TAILB as one more guarded
// batch (fewer round trips to memory, more registers live at once).
// get(i, r, c) -> V, put(i, r, c, v).
template <int U, class V, bool TAILB = false, class Get, class Put>
PSATD_HD void copy_grid(int R, int C, int tid, int nt, Get get, Put put) {
  const int total = R * C;
  const FastDiv dC = make_fastdiv((uint32_t)C);
  int r = (int)fdiv((uint32_t)tid, dC);
  int c = tid - r * C;
  const int dr = (int)fdiv((uint32_t)nt, dC);
  const int dc = nt - dr * C;
  auto advance = [&](int& rr, int& cc) {
    cc += dc;
    rr += dr;
    if (cc >= C) {
      cc -= C;
      ++rr;
    }
  };
  int i = tid;
  for (; i + (U - 1) * nt < total; i += U * nt) {
    V v[U];
    int rs[U], cs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      rs[u] = r;
      cs[u] = c;
      v[u] = get(i + u * nt, r, c);
      advance(r, c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) put(i + u * nt, rs[u], cs[u], v[u]);
  }
  if (!TAILB) {
    for (; i < total; i += nt) {
      put(i, r, c, get(i, r, c));
      advance(r, c);
    }
  } else if (i < total) {  // the last, partial batch, its loads in flight together
    V v[U];
    int rs[U], cs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      rs[u] = r;
      cs[u] = c;
      if (i + u * nt < total) v[u] = get(i + u * nt, r, c);
      advance(r, c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * nt < total) put(i + u * nt, rs[u], cs[u], v[u]);
  }
}

// The same walk over the pairs (e, e+1), e = 2 j, of a row-major R x C grid
// with R C even (a pair may straddle two rows): get(j, r0, c0, r1, c1) -> V,
// put(j, r0, c0, r1, c1, v), with (r1, c1) the position of e + 1.
template <int U, class V, bool TAILB = false, class Get, class Put>
PSATD_HD void copy_grid_pairs(int R, int C, int tid, int nt, Get get, Put put) {
  const int total = (R * C) >> 1;
  const FastDiv dC = make_fastdiv((uint32_t)C);
  int r = (int)fdiv((uint32_t)(2 * tid), dC);
  int c = 2 * tid - r * C;
  const int dr = (int)fdiv((uint32_t)(2 * nt), dC);
  const int dc = 2 * nt - dr * C;
  auto advance = [&](int& rr, int& cc) {
    cc += dc;
    rr += dr;
    if (cc >= C) {
      cc -= C;
      ++rr;
    }
  };
  auto second = [&](int rr, int cc, int& r1, int& c1) {
    const bool wrap = cc + 1 == C;
    r1 = wrap ? rr + 1 : rr;
    c1 = wrap ? 0 : cc + 1;
  };
  int j = tid;
  for (; j + (U - 1) * nt < total; j += U * nt) {
    V v[U];
    int rs[U], cs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      rs[u] = r;
      cs[u] = c;
      int r1, c1;
      second(r, c, r1, c1);
      v[u] = get(j + u * nt, r, c, r1, c1);
      advance(r, c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int r1, c1;
      second(rs[u], cs[u], r1, c1);
      put(j + u * nt, rs[u], cs[u], r1, c1, v[u]);
    }
  }
  if (!TAILB) {
    for (; j < total; j += nt) {
      int r1, c1;
      second(r, c, r1, c1);
      put(j, r, c, r1, c1, get(j, r, c, r1, c1));
      advance(r, c);
    }
  } else if (j < total) {  // the last, partial batch
    V v[U];
    int rs[U], cs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      rs[u] = r;
      cs[u] = c;
      int r1, c1;
      second(r, c, r1, c1);
      if (j + u * nt < total) v[u] = get(j + u * nt, r, c, r1, c1);
      advance(r, c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j + u * nt < total) {
        int r1, c1;
        second(rs[u], cs[u], r1, c1);
        put(j + u * nt, rs[u], cs[u], r1, c1, v[u]);
      }
  }
}

// The same walk over an A x B x C box (C fastest), the remainder always as a
// guarded batch: get(i, a, b, c), put(i, a, b, c, v).
template <int U, class V, class Get, class Put>
PSATD_HD void copy_grid3(int A, int B, int C, int tid, int nt, Get get, Put put) {
  const int total = A * B * C;
  const FastDiv dC = make_fastdiv((uint32_t)C);
  const FastDiv dB = make_fastdiv((uint32_t)B);
  auto split = [&](int v, int& a, int& b, int& c) {
    const int q = (int)fdiv((uint32_t)v, dC);
    c = v - q * C;
    a = (int)fdiv((uint32_t)q, dB);
    b = q - a * B;
  };
  int a, b, c, da, db, dc;
  split(tid, a, b, c);
  split(nt, da, db, dc);
  auto advance = [&](int& aa, int& bb, int& cc) {
    cc += dc;
    bb += db;
    aa += da;
    if (cc >= C) {
      cc -= C;
      ++bb;
    }
    if (bb >= B) {
      bb -= B;
      ++aa;
    }
  };
  int i = tid;
  for (; i + (U - 1) * nt < total; i += U * nt) {
    V v[U];
    int as[U], bs[U], cs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      as[u] = a;
      bs[u] = b;
      cs[u] = c;
      v[u] = get(i + u * nt, a, b, c);
      advance(a, b, c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) put(i + u * nt, as[u], bs[u], cs[u], v[u]);
  }
  if (i < total) {  // the last, partial batch
    V v[U];
    int as[U], bs[U], cs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      as[u] = a;
      bs[u] = b;
      cs[u] = c;
      if (i + u * nt < total) v[u] = get(i + u * nt, a, b, c);
      advance(a, b, c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i + u * nt < total) put(i + u * nt, as[u], bs[u], cs[u], v[u]);
  }
}

// Fused E,B guard exchange: after the inverse pass of interior plane zi (rows
// [ya, yb) of it held by this work-group), write the new values into every
// guard copy of those cells.  val(y, x) returns the new value of interior cell
// (y, x).  The pieces of a source box are visited in a uniform loop; rows of a
// piece are contiguous in the destination.
template <typename T, class Val>
PSATD_HD void push_guards(const PushBlk* blk, int b0, int b1, const BoxD* boxes, T* out, int zi,
                          int ya, int yb, Val val, int tid, int nt) {
  for (int b = b0; b < b1; ++b) {
    const PushBlk k = uniform_load(blk + b);
    if (zi < k.z0 || zi >= k.z0 + k.lz) continue;
    const int y_lo = ya > k.y0 ? ya : k.y0;
    const int y_hi = yb < k.y0 + k.ly ? yb : k.y0 + k.ly;
    if (y_lo >= y_hi) continue;
    const BoxD d = uniform_load(boxes + k.dst);
    T* base = out + d.foff + ((int64_t)(k.qz + zi - k.z0) * d.P[1] + (k.qy + y_lo - k.y0)) * d.P[0] + k.qx;
    const int n = (y_hi - y_lo) * k.lx;
    const FastDiv dl = make_fastdiv((uint32_t)k.lx);
    for (int i = tid; i < n; i += nt) {
      const int r = (int)fdiv((uint32_t)i, dl);
      const int c = i - r * k.lx;
      base[(int64_t)r * d.P[0] + c] = val(y_lo + r, k.x0 + c);
    }
  }
}

// ------------------------------------------------------------------ pass F
// Forward R2C along x and C2C along y of one z-plane of one field of one box.
// Output: half spectrum plane [ky][kx] (kx = 0..H-1) in natural order.
// A guard region of a destination box seen from the box that owns it: the
// padded cells [qz, qz+lz) x [qy, qy+ly) x [qx, qx+lx) of the destination are
// the source's interior cells starting at element `so` (plane 0, row 0,
// column 0) with the source's plane and row pitches.  Every guard cell of a
// box lies in exactly one of its pull pieces.
struct PullPiece {
  int64_t so;
  int32_t sPl, sP0;
  int32_t qz, lz, qy, ly, qx, lx;
};

template <typename T>
struct FwdArgs {
  Tables<T> t;
  const PlaneRec* planes;  // item = field * planes + plane
  FastDiv np;
  const T* in[9];
  cx<T>* spec;             // spectral workspace (see spec_at)
  int64_t sbias;           // spectral offset of the first box held by spec
  // Fields f < npull read their guard cells from the owners (pull pieces of
  // the plane's record) instead of the box's own, possibly stale, guard
  // copies; npull = 0 reads every padded cell in place.
  int32_t npull;
  const PullPiece* pull;
};

// Copies a rectangle of real cells src[r * sP0 + c] (r < ly, c < lx) into the
// LDS plane whose x rows are packed as complex pairs in stage-digit order:
// cell (y0 + r, x0 + c) goes to float 2 posx[(x0 + c) / 2] + (x0 + c) % 2 of
// row y0 + r.  Four cells per access when the rectangle and the source are
// 16-byte aligned, two when 8-byte aligned, else one.
template <typename T>
PSATD_HD void copy_rect_to_plane(const T* src, int sP0, int ly, int lx, int y0, int x0, cx<T>* lds, int ld,
                                 const int32_t* posx, int tid, int nt) {
  T* ldsT = reinterpret_cast<T*>(lds);
  const uintptr_t sa = reinterpret_cast<uintptr_t>(src);
  if (sizeof(T) == 4 && ((x0 | lx | sP0) & 3) == 0 && (sa & 15) == 0) {
    using Q = Pair<Pair<T>>;
    copy_grid<4, Q>(ly, lx >> 2, tid, nt,
                    [&](int, int r, int c4) { return *reinterpret_cast<const Q*>(src + (int64_t)r * sP0 + 4 * c4); },
                    [&](int, int r, int c4, Q v) {
                      cx<T>* row = lds + (y0 + r) * ld;
                      const int h = (x0 >> 1) + 2 * c4;
                      row[posx[h]] = cx<T>{v.a.a, v.a.b};
                      row[posx[h + 1]] = cx<T>{v.b.a, v.b.b};
                    });
  } else if (((x0 | lx | sP0) & 1) == 0 && (sa % sizeof(Pair<T>)) == 0) {
    copy_grid<8, Pair<T>>(ly, lx >> 1, tid, nt,
                          [&](int, int r, int c2) {
                            return *reinterpret_cast<const Pair<T>*>(src + (int64_t)r * sP0 + 2 * c2);
                          },
                          [&](int, int r, int c2, Pair<T> v) {
                            lds[(y0 + r) * ld + posx[(x0 >> 1) + c2]] = cx<T>{v.a, v.b};
                          });
  } else {
    copy_grid<8, T>(ly, lx, tid, nt, [&](int, int r, int c) { return src[(int64_t)r * sP0 + c]; },
                    [&](int, int r, int c, T v) {
                      const int x = x0 + c;
                      ldsT[2 * ((y0 + r) * ld + posx[x >> 1]) + (x & 1)] = v;
                    });
  }
}

// The rows of a padded plane into the LDS.
template <typename T>
PSATD_HD void load_plane(const FwdArgs<T>& a, const PlaneRec& rec, const BoxD& bx, int f, cx<T>* lds,
                         const int32_t* posx, int tid, int nt) {
  const int Px = bx.P[0], Py = bx.P[1], Nh = Px >> 1, ld = bx.ld, z = rec.z;
  if (f < a.npull) {
    // The box's own interior cells, then every guard region of this plane
    // from the box that owns it (Fig. 3 step 3 fused into the next push).
    // The waves share the rectangles (the interior in one row band per wave,
    // the pieces that meet the plane dealt round-robin), each copying its own
    // with its 64 lanes, so their memory round trips overlap.
    const int lane = tid & 63, wave = tid >> 6, nw = nt >> 6;
    const int gx = bx.g[0], gy = bx.g[1], gz = bx.g[2];
    const T* inf = a.in[f];
    int dealt = 0;
    if (z >= gz && z < gz + bx.n[2]) {
      const int ny = bx.n[1];
      const int r0 = (int)(((int64_t)ny * wave) / nw), r1 = (int)(((int64_t)ny * (wave + 1)) / nw);
      if (r1 > r0)
        copy_rect_to_plane<T>(inf + bx.foff + ((int64_t)z * Py + gy + r0) * Px + gx, Px, r1 - r0, bx.n[0], gy + r0,
                              gx, lds, ld, posx, lane, 64);
      dealt = nw;
    }
    for (int b = rec.p0; b < rec.p1; ++b) {
      if (dealt++ % nw != wave) continue;
      const PullPiece k = uniform_load(a.pull + b);
      copy_rect_to_plane<T>(inf + k.so + (int64_t)(z - k.qz) * k.sPl, k.sP0, k.ly, k.lx, k.qy, k.qx, lds, ld, posx,
                            lane, 64);
    }
    return;
  }
  const cx<T>* src = reinterpret_cast<const cx<T>*>(a.in[f] + bx.foff + (int64_t)z * Py * Px);
  if ((Nh & 1) == 0 && (reinterpret_cast<uintptr_t>(src) % sizeof(Pair<cx<T>>)) == 0) {
    // two neighbouring complex values per access (rows of even length)
    const Pair<cx<T>>* src2 = reinterpret_cast<const Pair<cx<T>>*>(src);
    copy_grid<4, Pair<cx<T>>>(Py, Nh >> 1, tid, nt, [&](int i, int, int) { return src2[i]; },
                              [&](int, int y, int x2, Pair<cx<T>> v) {
                                cx<T>* row = lds + y * ld;
                                row[posx[2 * x2]] = v.a;
                                row[posx[2 * x2 + 1]] = v.b;
                              });
  } else {
    copy_grid<8, cx<T>>(Py, Nh, tid, nt, [&](int i, int, int) { return src[i]; },
                        [&](int, int y, int x, cx<T> v) { lds[y * ld + posx[x]] = v; });
  }
}

// LDS: the plane [y][x] with row stride ld, then the twiddles of the x plan
// (Nh), the y plan (Py) and W_Px (real <-> half spectrum).
template <typename T, int MAXR, class Bar, class Eng = FftValu>
PSATD_HD void body_fwd_xy(const FwdArgs<T>& a, int item, int tid, int nt, cx<T>* lds, Bar bar, Eng eng = Eng{}) {
  const int f = (int)fdiv((uint32_t)item, a.np);
  const PlaneRec rec = uniform_load(a.planes + (item - f * (int)a.np.d));
  const BoxD bx = uniform_load(a.t.box + rec.box);
  const int z = rec.z;
  const int Px = bx.P[0], Py = bx.P[1];
  const int Nh = Px >> 1, H = bx.H, ld = bx.ld;
  const PlanRef plx = plan_ref(a.t.plans + bx.planx);
  const PlanRef ply = plan_ref(a.t.plans + bx.plany);
  cx<T>* twx = lds + Py * ld;
  cx<T>* twy = twx + Nh;
  cx<T>* twr = twy + Py;
  int32_t* posx = reinterpret_cast<int32_t*>(twr + Px);
  int32_t* posy = posx + Nh;
  const cx<T>* gtx = a.t.tw + plx->tw;
  const cx<T>* gty = a.t.tw + ply->tw;
  const cx<T>* gtr = a.t.tw + bx.twr;

  // stage-digit positions along x (input of the dit) and y (output of the dif)
  const int32_t* gpx = a.t.pos + plx->pos;
  const int32_t* gpy = a.t.pos + ply->pos;
  for (int i = tid; i < Nh + Py; i += nt) posx[i] = i < Nh ? gpx[i] : gpy[i - Nh];  // posx, posy are contiguous
  bar();
  // packed real rows (x natural) -> LDS rows in stage-digit order along x,
  // together with the three twiddle tables
  for (int i = tid; i < Nh + Py + Px; i += nt)  // twx, twy, twr are contiguous
    twx[i] = i < Nh ? gtx[i] : (i < Nh + Py ? gty[i - Nh] : gtr[i - Nh - Py]);
  load_plane(a, rec, bx, f, lds, posx, tid, nt);
  bar();
  eng.template dit<-1, MAXR>(lds, Py, ld, 1, plx, twx, tid, nt, bar);
  pair_pass_rows<true>(lds, Py, ld, Nh, twr, tid, nt);
  bar();
  eng.template dif<-1, MAXR>(lds, H, 1, ld, ply, twy, tid, nt, bar);
  cx<T>* dst = spec_at(a.spec, bx, a.sbias, f) + ring_slot(bx, z) * bx.pp;
  copy_grid<8, cx<T>>(Py, H, tid, nt, [&](int, int ky, int kx) { return lds[posy[ky] * ld + kx]; },
                      [&](int i, int, int, cx<T> v) { dst[i] = v; });
}

// ------------------------------------------------------------------ pass U
// Along z: forward C2C of 9 fields for a block of PB consecutive (ky, kx)
// pencils, the Eq. PSATD update at every k, backward C2C of the 6 results.
struct UpdConst {
  double c, dt;
};

// sin h and cos h in FP64: Cody-Waite reduction of h by multiples of pi/2
// (the two-term pi/2 leaves r within about 1e-16 of its true value for any
// |h| below 2^30), then the Taylor series of sin and cos on |r| <= pi/4 to
// the r^19 and r^18 terms (truncation below 1e-19), then the quadrant.
PSATD_HD void sincos_cw(double h, double* sh, double* ch) {
  const double two_over_pi = 0.63661977236758134308;
  const double pio2_hi = 1.5707963267948966;      // nearest double to pi/2
  const double pio2_lo = 6.123233995736766036e-17;  // pi/2 - pio2_hi
  const double n = rint(h * two_over_pi);
  const double r = fma(-n, pio2_lo, fma(-n, pio2_hi, h));
  const double r2 = r * r;
  // sin r = r (1 - r^2/3! + r^4/5! - ...), cos r = 1 - r^2/2! + r^4/4! - ...
  double ps = -1.0 / 121645100408832000.0;         // -1/19!
  ps = fma(ps, r2, 1.0 / 355687428096000.0);       // 1/17!
  ps = fma(ps, r2, -1.0 / 1307674368000.0);        // -1/15!
  ps = fma(ps, r2, 1.0 / 6227020800.0);            // 1/13!
  ps = fma(ps, r2, -1.0 / 39916800.0);             // -1/11!
  ps = fma(ps, r2, 1.0 / 362880.0);                // 1/9!
  ps = fma(ps, r2, -1.0 / 5040.0);                 // -1/7!
  ps = fma(ps, r2, 1.0 / 120.0);                   // 1/5!
  ps = fma(ps, r2, -1.0 / 6.0);                    // -1/3!
  const double s = fma(ps * r2, r, r);
  double pc = 1.0 / 6402373705728000.0;            // 1/18!
  pc = fma(pc, r2, -1.0 / 20922789888000.0);       // -1/16!
  pc = fma(pc, r2, 1.0 / 87178291200.0);           // 1/14!
  pc = fma(pc, r2, -1.0 / 479001600.0);            // -1/12!
  pc = fma(pc, r2, 1.0 / 3628800.0);               // 1/10!
  pc = fma(pc, r2, -1.0 / 40320.0);                // -1/8!
  pc = fma(pc, r2, 1.0 / 720.0);                   // 1/6!
  pc = fma(pc, r2, -1.0 / 24.0);                   // -1/4!
  pc = fma(pc, r2, 0.5);
  const double c = fma(-pc, r2, 1.0);
  const int q = (int)((int64_t)n & 3);
  *sh = q == 0 ? s : (q == 1 ? c : (q == 2 ? -s : -c));
  *ch = q == 0 ? c : (q == 1 ? -s : (q == 2 ? -c : s));
}

PSATD_HD float madd(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
PSATD_HD double madd(double a, double b, double c) { return __builtin_fma(a, b, c); }

// The FP64 coefficients of Eqs. PSATD_1 / PSATD_2 at |[k]|^2 = k2 (Sec. 3.1):
// th = c |[k]| dt, C - 1 = -2 sin^2(th/2) (no cancellation), S/(ck),
// X1 = (1 - C)/|[k]|^2 = 2 sin^2(th/2)/|[k]|^2, X2 = (S/(ck) - dt)/|[k]|^2 (by
// its series below th = 0.1, where the difference cancels); the k -> 0
// limits at |[k]| = 0.  rc = 1/c.
struct Coef64 {
  double cm1, sck, x1, x2;
};

PSATD_HD Coef64 psatd_coef(double k2, double c, double rc, double dt) {
#pragma clang fp contract(off)
  Coef64 r;
  const double c2 = c * c;
  if (k2 == 0.0) {
    r.cm1 = 0.0;
    r.sck = dt;
    r.x1 = 0.5 * c2 * dt * dt;
    r.x2 = -c2 * dt * dt * dt / 6.0;
    return r;
  }
  const double rk = rsqrt(k2);
  const double rk2 = rk * rk;
  const double k = k2 * rk;
  const double h = 0.5 * c * dt * k;  // th / 2
  double sh, ch;
  sincos_cw(h, &sh, &ch);
  const double sh2 = sh * sh;
  r.cm1 = -2.0 * sh2;
  r.sck = (2.0 * sh * ch) * rk * rc;
  r.x1 = 2.0 * sh2 * rk2;
  const double t2 = 4.0 * h * h;
  if (t2 < 1e-2) {
    r.x2 = -c2 * dt * dt * dt *
           fma(-t2, fma(-t2, fma(-t2, fma(-t2, 1.0 / 39916800.0, 1.0 / 362880.0), 1.0 / 5040.0), 1.0 / 120.0),
               1.0 / 6.0);
  } else {
    r.x2 = (r.sck - dt) * rk2;
  }
  return r;
}

// Eqs. PSATD_1 / PSATD_2 (general c) at one k-point; coefficients in FP64.
//   E' = C E + i c^2 (S/ck) [k]xB - (S/ck) J + X1 [k]([k].E) + X2 [k]([k].J)
//   B' = C B - i (S/ck) [k]xE + i (X1/c^2) [k]xJ
// with the coefficients of psatd_coef.
//
// INC: return the increments E' - E and B' - B instead (C replaced by
// C - 1 = -2 sin^2(th/2), exact without cancellation).  The FP32 path moves the
// increment through the FFTs: for resolved fields it is far smaller than E,
// so the FFT roundoff, relative to what is transformed, shrinks with it.
// The coefficients of one k-point in the state's type T, evaluated in FP64
// and rounded once: C (or C - 1 for increments), S/(ck), X1, X2, c^2 S/(ck),
// X1/c^2, and the modified wave vector.
template <typename T>
struct UpdCoef {
  T C, S, X1, X2, a1, x1c, kx, ky, kz;
};

template <typename T, bool INC>
PSATD_HD UpdCoef<T> update_coef(double kx, double ky, double kz, double c, double rc, double dt) {
#pragma clang fp contract(off)
  const Coef64 cf = psatd_coef(madd(kz, kz, madd(ky, ky, kx * kx)), c, rc, dt);
  UpdCoef<T> u;
  u.C = (T)(INC ? cf.cm1 : 1.0 + cf.cm1);
  u.S = (T)cf.sck;
  u.X1 = (T)cf.x1;
  u.X2 = (T)cf.x2;
  u.a1 = (T)(c * c * cf.sck);
  u.x1c = (T)(cf.x1 * (rc * rc));
  u.kx = (T)kx;
  u.ky = (T)ky;
  u.kz = (T)kz;
  return u;
}

// The update's multiply-adds in the state's type T (FP64 path: double; FP32
// path: float, where they act on increments).  The factors i leave two real
// problems of the same form, (Re E, Im B, Re J) with SG = +1 and (Im E, Re B,
// Im J) with SG = -1:
//   E' = C E - SG c^2 (S/ck) [k]xB - (S/ck) J + [k] (X1 [k].E + X2 [k].J)
//   B' = C B - SG [k] x ((S/ck) E - (X1/c^2) J)
//
// Its roundings are written out (fma, contraction off), as are those of the
// coefficients: kernels of different shape that share this text then agree in every
// bit, whatever products the compiler finds in common around it.
template <int SG, typename T>
PSATD_HD void update_half(T* e, T* b, const T* j, const UpdCoef<T>& u) {
#pragma clang fp contract(off)
  const T k[3] = {u.kx, u.ky, u.kz};
  const T ak[3] = {SG * u.a1 * u.kx, SG * u.a1 * u.ky, SG * u.a1 * u.kz};
  const T kE = madd(k[2], e[2], madd(k[1], e[1], k[0] * e[0]));
  const T kJ = madd(k[2], j[2], madd(k[1], j[1], k[0] * j[0]));
  const T s = madd(u.X2, kJ, u.X1 * kE);
  T f[3], en[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int p = (a + 1) % 3, q = (a + 2) % 3;
    f[a] = SG * madd(u.S, e[a], -(u.x1c * j[a]));
    en[a] = madd(k[a], s, madd(ak[q], b[p], madd(-ak[p], b[q], madd(-u.S, j[a], u.C * e[a]))));
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int p = (a + 1) % 3, q = (a + 2) % 3;
    b[a] = madd(k[q], f[p], madd(-k[p], f[q], u.C * b[a]));
    e[a] = en[a];
  }
}

template <typename T>
PSATD_HD void update_apply(T* vr, T* vi /* E0 E1 E2 B0 B1 B2 J0 J1 J2 */, const UpdCoef<T>& u) {
  update_half<1>(vr, vi + 3, vr + 6, u);
  update_half<-1>(vi, vr + 3, vi + 6, u);
}

template <typename T>
struct UpdArgs {
  Tables<T> t;
  const ZItem* items;
  cx<T>* spec;
  int64_t sbias;
  UpdConst k;
};

// Writes the 6 results of a tile (LDS [z][f PB + p], rows of W) at the
// interior z-planes only: the inverse pass reads nothing else (the guard planes
// of E and B are rewritten by the exchange).  A full tile whose pencil runs
// start at even offsets moves two neighbouring pencils per access.
template <typename T, int PB, int W>
PSATD_HD void store_results(const BoxD& bx, cx<T>* dst, int64_t sbias, int q0, int np, const cx<T>* lds, int tid,
                            int nt) {
  const cx<T>* res = lds + bx.g[2] * W;
  if (PB % 2 == 0 && np == PB && ((bx.pp | bx.sv | (bx.sb - sbias + q0) | (bx.xb - sbias + q0) | bx.xv) & 1) == 0) {
    copy_grid3<4, Pair<cx<T>>>(6, bx.n[2], PB / 2, tid, nt,
        [&](int, int f, int z, int p2) {
          return *reinterpret_cast<const Pair<cx<T>>*>(res + z * W + f * PB + 2 * p2);
        },
        [&](int, int f, int z, int p2, Pair<cx<T>> v) {
          *reinterpret_cast<Pair<cx<T>>*>(dst + result_plane(bx, sbias, f, z) + 2 * p2) = v;
        });
    return;
  }
  copy_grid3<8, cx<T>>(6, bx.n[2], PB, tid, nt,
                       [&](int, int f, int z, int p) { return res[z * W + f * PB + p]; },
                       [&](int, int f, int z, int p, cx<T> v) {
                         if (p < np) dst[result_plane(bx, sbias, f, z) + p] = v;
                       });
}

// Loads of the first z stage: element z = j + q ms of transform m = f PB + p is
// the plane at ring slot zb + z.  FP32 rings whose 9 fields lie within 4 GiB are
// read by buffer loads: a 32-bit lane offset (field, j, pencil) and a uniform
// offset per q, so that a load costs the vector ALU one select (the one q whose
// lanes fall on both sides of the ring's end takes its whole offset from the
// lane).  The FP64 pass is slower that way (64 boxes of 96^3 padded: 2.14 against
// 2.08 ms; FP32 0.90 against 0.93) and adds its lane offsets itself.
template <typename T, int PB>
struct ZLoad {
  const cx<T>* src;  // field 0, slot 0, first pencil of the tile
  int64_t sv;
  int32_t pp, ring, zb, np;  // np: pencils in the tile
  PSATD_HD ZLoad(const cx<T>* s, const BoxD& bx, int n)
      : src(s), sv(bx.sv), pp((int32_t)bx.pp), ring(bx.ring), zb(bx.zb), np(n) {}
  template <int R>
  PSATD_HD void run(int m, int j, int ms, cx<T>* a) const {
    const int f = m / PB;
    int p = m - f * PB;
    p = p < np ? p : np - 1;  // the idle pencils of a box's last tile repeat its last one
    const int wrap = ring - zb;
#ifdef __HIP_DEVICE_COMPILE__
    if constexpr (sizeof(T) == 4) {
      constexpr uint32_t B = sizeof(cx<T>);
      if (9 * sv * B <= 0xFFFFFFFFll) {
        const int qm = wrap / ms, jm = wrap - qm * ms;
        const uint32_t plane = (uint32_t)pp * B, back = (uint32_t)ring * plane;
        const auto rs = buffer_rsrc(src, (uint32_t)(9 * sv * B));
        const uint32_t lane = ((uint32_t)f * (uint32_t)sv + (uint32_t)p) * B + (uint32_t)j * plane;
        const uint32_t mixed = lane + (uint32_t)(zb + qm * ms) * plane - (j >= jm ? back : 0u);
        uint32_t o = (uint32_t)zb * plane;  // of slot zb + q ms
#pragma unroll
        for (int q = 0; q < R; ++q) {
          const bool mix = q == qm;
          buf_load(rs, mix ? mixed : lane, mix ? 0u : o - (q > qm ? back : 0u), &a[q]);
          o += (uint32_t)ms * plane;
        }
        return;
      }
    }
#endif
    // element offsets within one field's ring fit 32 bits: 2^32 elements of one
    // field, and the state they belong to, are more than the device's memory
    const cx<T>* base = src + (f * sv + p);
    uint32_t o = (uint32_t)(zb + j) * (uint32_t)pp;
    const uint32_t step = (uint32_t)ms * (uint32_t)pp, back = (uint32_t)ring * (uint32_t)pp;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      a[q] = base[j + q * ms >= wrap ? o - back : o];
      o += step;
    }
  }
};

// The 9 fields of a tile's pencils into the LDS as [z][f PB + p]; those past np are
// zeros.  A full tile whose pencil runs start at even offsets moves two neighbouring
// pencils per access.
template <typename T, int PB>
PSATD_HD void stage_tile(const BoxD& bx, const cx<T>* src, int64_t sbias, int q0, int np, cx<T>* lds, int tid,
                         int nt) {
  constexpr int W = 9 * PB;
  const int Pz = bx.P[2];
  const int64_t slab = bx.sv;  // field stride
  if (PB % 2 == 0 && np == PB && ((bx.pp | slab | (bx.sb - sbias + q0)) & 1) == 0) {
    copy_grid3<8, Pair<cx<T>>>(9, Pz, PB / 2, tid, nt,
        [&](int, int f, int z, int p2) {
          return *reinterpret_cast<const Pair<cx<T>>*>(src + f * slab + ring_slot(bx, z) * bx.pp + 2 * p2);
        },
        [&](int, int f, int z, int p2, Pair<cx<T>> v) {
          *reinterpret_cast<Pair<cx<T>>*>(lds + z * W + f * PB + 2 * p2) = v;
        });
    return;
  }
  copy_grid3<8, cx<T>>(9, Pz, PB, tid, nt,
      [&](int, int f, int z, int p) {
        return (p < np) ? src[f * slab + ring_slot(bx, z) * bx.pp + p] : cx<T>{T(0), T(0)};
      },
      [&](int, int f, int z, int p, cx<T> v) { lds[z * W + f * PB + p] = v; });
}

// The z pass.  The 9 fields of PB consecutive (ky, kx) pencils are held in the LDS
// as [z][f PB + p] (W = 9 PB complex per z row), so that all 9 (then the 6 output)
// fields are transformed by one multi-transform pass with a uniform element stride.
// The vector-ALU forms read the ring's planes straight into the butterflies of the
// first z stage; the matrix-core stages take theirs from a staged tile.  The update
// takes the points kz and -kz of a pencil together: they share |[k]| and so the
// FP64 coefficients.  The results go out through the LDS in whole pencil runs:
// stores straight from the last stage's butterflies measured 1.0 -> 1.5 ms (64 boxes
// of 96^3 padded, FP32).  Issue-bound (65 % of the time is VALU busy); with the
// loads and pairs as here 1.03 -> 0.90 ms, FP64 2.32 -> 2.08 ms, 8 boxes of 176^3 in
// FP64 2.44 -> 2.03 ms; the matrix-core forms, with the pairs and what mfma_dft.hpp
// says of its stage, 0.220 -> 0.161 ms on 8 boxes of 96^3.
template <typename T, int PB, bool INC, int MAXR, class Bar, class Eng = FftValu>
PSATD_HD void body_z_update(const UpdArgs<T>& a, int item, int tid, int nt, cx<T>* lds, Bar bar, Eng eng = Eng{}) {
  constexpr bool VALU = std::is_same<Eng, FftValu>::value;
  const ZItem it = uniform_load(a.items + item);
  const BoxD bx = uniform_load(a.t.box + it.box);
  const int Pz = bx.P[2], H = bx.H, nq = bx.P[1] * H, q0 = it.q0;
  const PlanRef plz = plan_ref(a.t.plans + bx.planz);
  constexpr int W = 9 * PB;
  cx<T>* twz = lds + Pz * W;
  int32_t* pos = reinterpret_cast<int32_t*>(twz + Pz);  // slot of each frequency
  const cx<T>* gtz = a.t.tw + plz->tw;
  const int32_t* gpos = a.t.pos + plz->pos;
  for (int i = tid; i < Pz; i += nt) {
    twz[i] = gtz[i];
    pos[i] = gpos[i];
  }
  const int np = (nq - q0) < PB ? (nq - q0) : PB;
  const cx<T>* src = spec_at(a.spec, bx, a.sbias, 0) + q0;
  if constexpr (VALU) {
    bar();
    first_stage_dispatch<-1, MAXR, W, W>(plz, lds, twz, tid, nt, ZLoad<T, PB>{src, bx, np});
    bar();
    fft_dif_inner<-1, MAXR>(lds, W, 1, W, plz, twz, tid, nt, bar);
  } else {
    stage_tile<T, PB>(bx, src, a.sbias, q0, np, lds, tid, nt);
    bar();
    eng.template dif<-1, MAXR>(lds, W, 1, W, plz, twz, tid, nt, bar);
  }

  const double* kxt = a.t.kmod + bx.kx;
  const double* kyt = a.t.kmod + bx.ky;
  const double* kzt = a.t.kmod + bx.kz;
  const FastDiv dH = make_fastdiv((uint32_t)H);
  const double rc = 1.0 / a.k.c;
  for (int i = tid; i < (Pz / 2 + 1) * PB; i += nt) {
    const int kz = (int)((uint32_t)i / (uint32_t)PB);
    const int p = i - kz * PB;
    if (p >= np) continue;
    const int q = q0 + p;
    const int ky = (int)fdiv((uint32_t)q, dH);
    UpdCoef<T> u = update_coef<T, INC>(kxt[q - ky * H], kyt[ky], kzt[kz], a.k.c, rc, a.k.dt);
    // [k](-kz) = -[k](kz), and both entries are 0 at kz = 0 and Nyquist
    for (int k = kz;; k = Pz - kz, u.kz = -u.kz) {
      cx<T>* row = lds + pos[k] * W + p;
      T vr[9], vi[9];
#pragma unroll
      for (int f = 0; f < 9; ++f) {
        const cx<T> v = row[f * PB];
        vr[f] = v.x;
        vi[f] = v.y;
      }
      update_apply<T>(vr, vi, u);
#pragma unroll
      for (int f = 0; f < 6; ++f) row[f * PB] = cx<T>{vr[f], vi[f]};
      if (k != kz || kz == 0 || 2 * kz == Pz) break;
    }
  }
  bar();
  eng.template dit<+1, MAXR>(lds, 6 * PB, 1, W, plz, twz, tid, nt, bar);
  store_results<T, PB, W>(bx, a.spec + q0, a.sbias, q0, np, lds, tid, nt);
}

constexpr int kThreadsHeld = 256;
constexpr int kHeldPairs = 2;  // pairs +-kz per thread

// LDS of a held tile of PB pencils of padded z length Pz.
PSATD_HD int64_t held_tile_lds(int Pz, int PB, int real_bytes) {
  return (int64_t)Pz * ((6 * PB + 1) * 2 * real_bytes + 4);
}

// The same pass with 6 fields of a tile in the LDS: J is transformed first and its
// points are held in registers, each by the thread that updates it, while E and B
// take J's place.  Two tiles then share a compute unit where the nine fields of one
// filled its LDS, so that one tile's loads and barriers overlap the other's
// transforms: 2.07 -> 1.71 ms on 64 boxes of 96^3 padded in FP64, 2.02 -> 1.57 ms on
// 8 of 176^3.  Still issue-bound; 215 VGPRs.
template <typename T, int PB, bool INC, int MAXR, class Bar>
PSATD_HD void body_z_held(const UpdArgs<T>& a, int item, int tid, int nt, cx<T>* lds, Bar bar) {
  const ZItem it = uniform_load(a.items + item);
  const BoxD bx = uniform_load(a.t.box + it.box);
  const int Pz = bx.P[2], H = bx.H, nq = bx.P[1] * H, q0 = it.q0;
  const PlanRef plz = plan_ref(a.t.plans + bx.planz);
  constexpr int W = 6 * PB, WJ = 3 * PB;
  cx<T>* twz = lds + Pz * W;
  int32_t* pos = reinterpret_cast<int32_t*>(twz + Pz);
  const cx<T>* gtz = a.t.tw + plz->tw;
  const int32_t* gpos = a.t.pos + plz->pos;
  for (int i = tid; i < Pz; i += nt) {
    twz[i] = gtz[i];
    pos[i] = gpos[i];
  }
  const int np = (nq - q0) < PB ? (nq - q0) : PB;
  const cx<T>* src = spec_at(a.spec, bx, a.sbias, 0) + q0;
  bar();
  first_stage_dispatch<-1, MAXR, WJ, WJ>(plz, lds, twz, tid, nt, ZLoad<T, PB>{src + 6 * bx.sv, bx, np});
  bar();
  fft_dif_inner<-1, MAXR>(lds, WJ, 1, WJ, plz, twz, tid, nt, bar);
  const int n = (Pz / 2 + 1) * PB;
  cx<T> jh[kHeldPairs][2][3];
#pragma unroll
  for (int h = 0; h < kHeldPairs; ++h) {
    const int i = tid + h * nt;
    if (i < n) {
      const int kz = (int)((uint32_t)i / (uint32_t)PB);
      const int p = i - kz * PB;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const cx<T>* row = lds + pos[s && kz ? Pz - kz : kz] * WJ + p;
#pragma unroll
        for (int f = 0; f < 3; ++f) jh[h][s][f] = row[f * PB];
      }
    }
  }
  bar();
  first_stage_dispatch<-1, MAXR, W, W>(plz, lds, twz, tid, nt, ZLoad<T, PB>{src, bx, np});
  bar();
  fft_dif_inner<-1, MAXR>(lds, W, 1, W, plz, twz, tid, nt, bar);

  const double* kxt = a.t.kmod + bx.kx;
  const double* kyt = a.t.kmod + bx.ky;
  const double* kzt = a.t.kmod + bx.kz;
  const FastDiv dH = make_fastdiv((uint32_t)H);
  const double rc = 1.0 / a.k.c;
#pragma unroll
  for (int h = 0; h < kHeldPairs; ++h) {
    const int i = tid + h * nt;
    const int kz = (int)((uint32_t)i / (uint32_t)PB);
    const int p = i - kz * PB;
    if (i < n && p < np) {
      const int q = q0 + p;
      const int ky = (int)fdiv((uint32_t)q, dH);
      UpdCoef<T> u = update_coef<T, INC>(kxt[q - ky * H], kyt[ky], kzt[kz], a.k.c, rc, a.k.dt);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if (s && (kz == 0 || 2 * kz == Pz)) continue;
        cx<T>* row = lds + pos[s ? Pz - kz : kz] * W + p;
        T vr[9], vi[9];
#pragma unroll
        for (int f = 0; f < 9; ++f) {
          const cx<T> v = f < 6 ? row[f * PB] : jh[h][s][f - 6];
          vr[f] = v.x;
          vi[f] = v.y;
        }
        update_apply<T>(vr, vi, u);
#pragma unroll
        for (int f = 0; f < 6; ++f) row[f * PB] = cx<T>{vr[f], vi[f]};
        u.kz = -u.kz;
      }
    }
  }
  bar();
  fft_dit<+1, MAXR>(lds, 6 * PB, 1, W, plz, twz, tid, nt, bar);
  store_results<T, PB, W>(bx, a.spec + q0, a.sbias, q0, np, lds, tid, nt);
}

// ------------------------------------------------------- heat equation
// Sec. 5 names the diffusion equation among the initial-value problems the
// local-FFT method applies to: du/dt = D lap u, Laplacian symbol -|[k]|^2 with
// the same order-p modified wavenumbers, exact propagator per step.  The x/y
// passes are the field passes with one field; this is its z pass.
template <typename T>
struct HeatArgs {
  Tables<T> t;
  const ZItem* items;
  cx<T>* spec;           // the half spectrum of u
  double D, dt;
};

// LDS of a heat z tile of PB pencils: the staged field, the z twiddles, the
// propagator's z and (kx, ky) factors (FP64) and the positions of the frequencies.
PSATD_HD int64_t heat_tile_lds(int Pz, int PB, int real_bytes) {
  return (int64_t)Pz * (PB + 1) * 2 * real_bytes + (int64_t)(Pz + PB) * 8 + (int64_t)Pz * 4;
}

// PB consecutive (ky, kx) pencils staged as [z][p]: forward z transform,
// multiply by g = exp(-D |[k]|^2 dt) in FP64 (INC: by g - 1, the increment's
// spectrum), inverse z transform.  g is the product of a factor per kz and one
// per (kx, ky), so a tile takes Pz + PB exponentials instead of Pz PB:
// g1 g2, or (g1 - 1) + (g2 - 1) + (g1 - 1)(g2 - 1), whose terms the product
// cannot cancel (both factors are at most 1, or for a negative dt both at least 1).
// One field in LDS leaves room for wide tiles: 32 pencils (256-byte runs) in place of
// the field pass's 10, with the factors and the direct loads, 0.29 -> 0.15 ms on 64
// boxes of 96^3 padded, FP32.
template <typename T, int PB, bool INC, int MAXR, class Bar, class Eng = FftValu>
PSATD_HD void body_z_heat(const HeatArgs<T>& a, int item, int tid, int nt, cx<T>* lds, Bar bar,
                          Eng eng = Eng{}) {
  const ZItem it = uniform_load(a.items + item);
  const BoxD bx = uniform_load(a.t.box + it.box);
  const int Pz = bx.P[2], H = bx.H;
  const int nq = bx.P[1] * H;
  const int q0 = it.q0;
  const int np = (nq - q0) < PB ? (nq - q0) : PB;
  const PlanRef plz = plan_ref(a.t.plans + bx.planz);
  cx<T>* twz = lds + Pz * PB;
  double* gz1 = reinterpret_cast<double*>(twz + Pz);
  double* gxy = gz1 + Pz;
  int32_t* pos = reinterpret_cast<int32_t*>(gxy + PB);
  const cx<T>* gtz = a.t.tw + plz->tw;
  const int32_t* gpos = a.t.pos + plz->pos;
  for (int i = tid; i < Pz; i += nt) {
    twz[i] = gtz[i];
    pos[i] = gpos[i];
  }
  const cx<T>* src = spec_at(a.spec, bx, 0, 0) + q0;
  if constexpr (std::is_same<Eng, FftValu>::value) {
    bar();
    first_stage_dispatch<-1, MAXR, PB, PB>(plz, lds, twz, tid, nt, ZLoad<T, PB>{src, bx, np});
  } else {  // the matrix-core first stage takes its elements from the LDS
    copy_grid<8, cx<T>>(Pz, PB, tid, nt,
                        [&](int, int z, int p) { return src[ring_slot(bx, z) * bx.pp + (p < np ? p : np - 1)]; },
                        [&](int i, int, int, cx<T> v) { lds[i] = v; });
  }
  const double* kxt = a.t.kmod + bx.kx;
  const double* kyt = a.t.kmod + bx.ky;
  const double* kzt = a.t.kmod + bx.kz;
  const FastDiv dH = make_fastdiv((uint32_t)H);
  for (int i = tid; i < Pz + PB; i += nt) {
    double k2;
    if (i < Pz) {
      k2 = kzt[i] * kzt[i];
    } else {
      const int q = q0 + (i - Pz < np ? i - Pz : np - 1);
      const int ky = (int)fdiv((uint32_t)q, dH);
      const double k1 = kxt[q - ky * H];
      k2 = k1 * k1 + kyt[ky] * kyt[ky];
    }
    const double e = -a.D * k2 * a.dt;
    gz1[i] = INC ? expm1(e) : exp(e);
  }
  bar();
  if constexpr (std::is_same<Eng, FftValu>::value)
    fft_dif_inner<-1, MAXR>(lds, PB, 1, PB, plz, twz, tid, nt, bar);
  else
    eng.template dif<-1, MAXR>(lds, PB, 1, PB, plz, twz, tid, nt, bar);
  for (int i = tid; i < Pz * PB; i += nt) {
    const int k = (int)((uint32_t)i / (uint32_t)PB);
    const int p = i - k * PB;
    const double ga = gz1[k], gb = gxy[p];
    const T g = (T)(INC ? fma(ga, gb, ga + gb) : ga * gb);
    cx<T>* v = lds + pos[k] * PB + p;
    *v = cx<T>{v->x * g, v->y * g};
  }
  bar();
  eng.template dit<+1, MAXR>(lds, PB, 1, PB, plz, twz, tid, nt, bar);
  // interior z-planes only (all the inverse pass reads)
  const int gz = bx.g[2];
  cx<T>* dst = a.spec + q0;
  if (np == PB && ((bx.pp | (bx.sb + q0) | (bx.xb + q0)) & 1) == 0) {
    copy_grid<4, Pair<cx<T>>, true>(bx.n[2], PB / 2, tid, nt,
        [&](int, int z, int p2) { return *reinterpret_cast<const Pair<cx<T>>*>(lds + (gz + z) * PB + 2 * p2); },
        [&](int, int z, int p2, Pair<cx<T>> v) {
          *reinterpret_cast<Pair<cx<T>>*>(dst + result_plane(bx, 0, 0, z) + 2 * p2) = v;
        });
    return;
  }
  copy_grid<8, cx<T>, true>(bx.n[2], PB, tid, nt, [&](int, int z, int p) { return lds[(gz + z) * PB + p]; },
                            [&](int, int z, int p, cx<T> v) {
                              if (p < np) dst[result_plane(bx, 0, 0, z) + p] = v;
                            });
}

// ------------------------------------------------------------------ pass I
// Backward C2C along y and C2R along x of one interior z-plane of one of the 6
// output fields; writes the interior cells of the plane, scaled by 1/V.
template <typename T>
struct InvArgs {
  Tables<T> t;
  const PlaneRec* planes;  // interior planes; item = field * planes + plane
  FastDiv np;
  const cx<T>* spec;
  int64_t sbias;
  T* out[6];
  const PushBlk* push;       // fused E,B guard exchange (null: a separate fill pass)
  const int32_t* push_off;   // pieces of box s: [push_off[s], push_off[s+1])
};

// Interior cells gx, gx + 1, ... of ny transformed LDS rows, scaled, to rows of
// dst0 (INC: added).
template <typename T, bool INC>
PSATD_HD void store_rows(T* dst0, int Px, int ny, int nx, int gx, double sc, const cx<T>* lds, int ld,
                         const int32_t* posx, int tid, int nt) {
  if (sizeof(T) == 4 && (gx & 1) == 0 && (nx & 3) == 0 && (Px & 3) == 0 &&
      (reinterpret_cast<uintptr_t>(dst0) % sizeof(Pair<Pair<T>>)) == 0) {
    // FP32: four cells (two complex LDS entries, 16 bytes) per access
    const int hx = gx >> 1;
    using Q = Pair<Pair<T>>;
    copy_grid<4, Q>(ny, nx >> 2, tid, nt,
                    [&](int, int yy, int x4) {
                      const cx<T>* row = lds + yy * ld;
                      const cx<T> v0 = row[posx[hx + 2 * x4]], v1 = row[posx[hx + 2 * x4 + 1]];
                      return Q{{(T)((double)v0.x * sc), (T)((double)v0.y * sc)},
                               {(T)((double)v1.x * sc), (T)((double)v1.y * sc)}};
                    },
                    [&](int, int yy, int x4, Q v) {
                      Q* q = reinterpret_cast<Q*>(dst0 + (int64_t)yy * Px) + x4;
                      if (INC) {  // v is the increment
                        const Q o = *q;
                        v.a.a = o.a.a + v.a.a;
                        v.a.b = o.a.b + v.a.b;
                        v.b.a = o.b.a + v.b.a;
                        v.b.b = o.b.b + v.b.b;
                      }
                      *q = v;
                    });
    return;
  }
  if (((gx | nx) & 1) == 0 && (reinterpret_cast<uintptr_t>(dst0) % sizeof(Pair<T>)) == 0) {
    // cells x, x+1 (x even) are the two halves of one complex LDS entry: one
    // LDS read and one 2-wide access per pair
    const int hx = gx >> 1;
    copy_grid<8, Pair<T>>(ny, nx >> 1, tid, nt,
                          [&](int, int yy, int x2) {
                            const cx<T> v = lds[yy * ld + posx[hx + x2]];
                            return Pair<T>{(T)((double)v.x * sc), (T)((double)v.y * sc)};
                          },
                          [&](int, int yy, int x2, Pair<T> v) {
                            Pair<T>* q = reinterpret_cast<Pair<T>*>(dst0 + (int64_t)yy * Px) + x2;
                            if (INC) {  // v is the increment
                              const Pair<T> o = *q;
                              v.a = o.a + v.a;
                              v.b = o.b + v.b;
                            }
                            *q = v;
                          });
    return;
  }
  copy_grid<8, T>(ny, nx, tid, nt,
                  [&](int, int yy, int xi) {
                    const int x = gx + xi;
                    const cx<T> v = lds[yy * ld + posx[x >> 1]];
                    return (T)((double)((x & 1) ? v.y : v.x) * sc);
                  },
                  [&](int, int yy, int xi, T v) {
                    T* q = dst0 + (int64_t)yy * Px + xi;
                    *q = INC ? *q + v : v;  // INC: v is the increment
                  });
}

// LDS: the plane with row stride ld, then the twiddles of the y plan (Py),
// the x plan (Nh) and W_Px.
template <typename T, bool INC, int MAXR, bool PUSH = false, class Bar, class Eng = FftValu>
PSATD_HD void body_inv_xy(const InvArgs<T>& a, int item, int tid, int nt, cx<T>* lds, Bar bar, Eng eng = Eng{}) {
  const int f = (int)fdiv((uint32_t)item, a.np);
  const PlaneRec rec = uniform_load(a.planes + (item - f * (int)a.np.d));
  const int s = rec.box;
  const BoxD bx = uniform_load(a.t.box + s);
  const int z = bx.g[2] + rec.z;
  const int Px = bx.P[0], Py = bx.P[1], Pz = bx.P[2];
  const int Nh = Px >> 1, H = bx.H, ld = bx.ld;
  const PlanRef plx = plan_ref(a.t.plans + bx.planx);
  const PlanRef ply = plan_ref(a.t.plans + bx.plany);
  cx<T>* twy = lds + Py * ld;
  cx<T>* twx = twy + Py;
  cx<T>* twr = twx + Nh;
  int32_t* posy = reinterpret_cast<int32_t*>(twr + Px);
  int32_t* posx = posy + Py;
  const cx<T>* gty = a.t.tw + ply->tw;
  const cx<T>* gtx = a.t.tw + plx->tw;
  const cx<T>* gtr = a.t.tw + bx.twr;

  // stage-digit positions along y (input of the dit) and x (output of the dif)
  const int32_t* gpx = a.t.pos + plx->pos;
  const int32_t* gpy = a.t.pos + ply->pos;
  for (int i = tid; i < Py + Nh; i += nt) posy[i] = i < Py ? gpy[i] : gpx[i - Py];  // posy, posx are contiguous
  bar();

  // half-spectrum rows (ky natural) -> LDS rows in stage-digit order along y
  const cx<T>* src = a.spec + result_plane(bx, a.sbias, f, rec.z);
  for (int i = tid; i < Py + Nh + Px; i += nt)  // twy, twx, twr are contiguous
    twy[i] = i < Py ? gty[i] : (i < Py + Nh ? gtx[i - Py] : gtr[i - Py - Nh]);
  // FP32: two spectrum entries per access (measured slower in FP64)
  if (sizeof(T) == 4 && ((Py * H) & 1) == 0 && (reinterpret_cast<uintptr_t>(src) % sizeof(Pair<cx<T>>)) == 0) {
    const Pair<cx<T>>* src2 = reinterpret_cast<const Pair<cx<T>>*>(src);
    copy_grid_pairs<4, Pair<cx<T>>, true>(Py, H, tid, nt, [&](int j, int, int, int, int) { return src2[j]; },
        [&](int, int r0, int c0, int r1, int c1, Pair<cx<T>> v) {
          lds[posy[r0] * ld + c0] = v.a;
          lds[posy[r1] * ld + c1] = v.b;
        });
  } else {
    copy_grid<8, cx<T>, true>(Py, H, tid, nt, [&](int i, int, int) { return src[i]; },
                        [&](int, int ky, int kx, cx<T> v) { lds[posy[ky] * ld + kx] = v; });
  }
  bar();
  eng.template dit<+1, MAXR>(lds, H, 1, ld, ply, twy, tid, nt, bar);
  const int ny = bx.n[1], gy = bx.g[1];
  pair_pass_rows<false>(lds + gy * ld, ny, ld, Nh, twr, tid, nt);
  bar();
  eng.template dif<+1, MAXR>(lds + gy * ld, ny, ld, 1, plx, twx, tid, nt, bar);
  // 1/V applied in FP64 and rounded once: an FP32 1/V (not a power of two for
  // most V) would bias every step by the same relative amount.
  const double sc = 1.0 / ((double)Px * (double)Py * (double)Pz);
  const int nx = bx.n[0], gx = bx.g[0];
  T* dst = a.out[f] + bx.foff + (int64_t)z * Py * Px;
  [[maybe_unused]] T* ldsT = reinterpret_cast<T*>(lds);
  constexpr bool push = PUSH;  // the fused E,B exchange (compiled only where used)
  if (!push) {
    store_rows<T, INC>(dst + (int64_t)gy * Px + gx, Px, ny, nx, gx, sc, lds + gy * ld, ld, posx, tid, nt);
    return;
  }
  copy_grid<8, T>(ny, nx, tid, nt,
                  [&](int, int yy, int xi) {
                    const int x = gx + xi;
                    const cx<T> v = lds[(gy + yy) * ld + posx[x >> 1]];
                    return (T)((double)((x & 1) ? v.y : v.x) * sc);
                  },
                  [&](int, int yy, int xi, T v) {
                    const int x = gx + xi;
                    T* q = dst + (gy + yy) * Px + x;
                    const T nv = INC ? *q + v : v;  // INC: v is the increment
                    *q = nv;
                    // the new value back into its own LDS slot for the guard copies
                    if constexpr (push) ldsT[2 * ((gy + yy) * ld + posx[x >> 1]) + (x & 1)] = nv;
                  });
  if constexpr (push) {
    bar();
    push_guards<T>(a.push, uniform_load(a.push_off + s), uniform_load(a.push_off + s + 1), a.t.box, a.out[f], z - bx.g[2], 0, ny,
                   [&](int yi, int xi) {
                     const int x = gx + xi;
                     return ldsT[2 * ((gy + yi) * ld + posx[x >> 1]) + (x & 1)];
                   },
                   tid, nt);
  }
}

// ------------------------------------------------ planes in two halves
// The inverse pass over FP32 planes beyond the LDS of which half fits: the y
// columns are transformed in two halves of ceil(H/2), the interior x rows in two
// halves, with what is not being transformed in registers (the vector registers
// of a compute unit hold three times its LDS).  That saves the passes of their
// own for y and x and the round trip through the workspace between them: one
// 256^3 box 0.55 -> 0.39 ms.  The planes it is taken for are build_lists' choice.
// The forward pass keeps the split passes: 256^2 0.40 -> 0.35 ms in halves, but
// 200^2 to 240 x 216 0.21 -> 0.24 and 0.12 -> 0.15 (a lone group per compute unit
// exposes every stage).  So do FP64 planes (176^2, 8 boxes: inverse 1.19 -> 1.36
// ms), and FP32 planes that fit the LDS once stay whole (176^2 as two 512-thread
// groups per compute unit, 64 boxes: 3.5 -> 4.3 ms).
constexpr int kHalfHold = 10;  // values held per thread and quarter plane

// LDS elements of half a plane: ceil(Py/2) rows, or Py rows of half the columns.
PSATD_HD int half_cols(int H) { return (H + 1) >> 1; }
PSATD_HD int half_ld(int H) { return half_cols(H) | 1; }
PSATD_HD int half_elems(int Py, int ld, int H) {
  const int rows = ((Py + 1) >> 1) * ld, cols = Py * half_ld(H);
  return rows > cols ? rows : cols;
}

// Moves an R x C block between the LDS (rows of pitch ld) and the threads'
// registers, element i = tid + k nt in v[k] (R C <= K nt, checked at plan time).
template <int K, bool SAVE, typename T>
PSATD_HD void hold_block(cx<T>* v, cx<T>* lds, int R, int C, int ld, int tid, int nt) {
  const FastDiv dC = make_fastdiv((uint32_t)C);
  int r = (int)fdiv((uint32_t)tid, dC);
  int c = tid - r * C;
  const int dr = (int)fdiv((uint32_t)nt, dC);
  const int dc = nt - dr * C;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (tid + k * nt < R * C) {
      if (SAVE) v[k] = lds[r * ld + c];
      else lds[r * ld + c] = v[k];
    }
    c += dc;
    r += dr;
    if (c >= C) {
      c -= C;
      ++r;
    }
  }
}

template <typename T, bool INC, int MAXR, class Bar>
PSATD_HD void body_inv_half(const InvArgs<T>& a, int item, int tid, int nt, cx<T>* lds, Bar bar) {
  constexpr int K = kHalfHold;
  const int f = (int)fdiv((uint32_t)item, a.np);
  const PlaneRec rec = uniform_load(a.planes + (item - f * (int)a.np.d));
  const BoxD bx = uniform_load(a.t.box + rec.box);
  const int z = bx.g[2] + rec.z;
  const int Px = bx.P[0], Py = bx.P[1], Pz = bx.P[2];
  const int Nh = Px >> 1, H = bx.H, ld = bx.ld;
  const int ny = bx.n[1], gy = bx.g[1];
  const int Ra = (ny + 1) >> 1, Hl = half_cols(H), Hr = H - Hl, ldc = half_ld(H);
  const PlanRef plx = plan_ref(a.t.plans + bx.planx);
  const PlanRef ply = plan_ref(a.t.plans + bx.plany);
  cx<T>* twy = lds + half_elems(Py, ld, H);
  cx<T>* twx = twy + Py;
  cx<T>* twr = twx + Nh;
  int32_t* posy = reinterpret_cast<int32_t*>(twr + Px);
  int32_t* posx = posy + Py;
  const cx<T>* gty = a.t.tw + ply->tw;
  const cx<T>* gtx = a.t.tw + plx->tw;
  const cx<T>* gtr = a.t.tw + bx.twr;
  const int32_t* gpx = a.t.pos + plx->pos;
  const int32_t* gpy = a.t.pos + ply->pos;
  for (int i = tid; i < Py + Nh; i += nt) posy[i] = i < Py ? gpy[i] : gpx[i - Py];  // posy, posx are contiguous
  for (int i = tid; i < Py + Nh + Px; i += nt)  // twy, twx, twr are contiguous
    twy[i] = i < Py ? gty[i] : (i < Py + Nh ? gtx[i - Py] : gtr[i - Py - Nh]);
  bar();
  const cx<T>* src = a.spec + result_plane(bx, a.sbias, f, rec.z);
  cx<T> al[K], bl[K], br[K];  // interior rows: first half (left columns), second half (left, right)
#pragma unroll 1
  for (int side = 0; side < 2; ++side) {
    const int C = side ? Hr : Hl, c0 = side ? Hl : 0;
    copy_grid<8, cx<T>>(Py, C, tid, nt, [&](int, int ky, int c) { return src[ky * H + c0 + c]; },
                        [&](int, int ky, int c, cx<T> v) { lds[posy[ky] * ldc + c] = v; });
    bar();
    fft_dit<+1, MAXR>(lds, C, 1, ldc, ply, twy, tid, nt, bar);
    if (side) break;
    hold_block<K, true>(al, lds + gy * ldc, Ra, Hl, ldc, tid, nt);
    hold_block<K, true>(bl, lds + (gy + Ra) * ldc, ny - Ra, Hl, ldc, tid, nt);
    bar();
  }
  {
    cx<T> ar[K];
    hold_block<K, true>(ar, lds + gy * ldc, Ra, Hr, ldc, tid, nt);
    hold_block<K, true>(br, lds + (gy + Ra) * ldc, ny - Ra, Hr, ldc, tid, nt);
    bar();
    hold_block<K, false>(al, lds, Ra, Hl, ld, tid, nt);
    hold_block<K, false>(ar, lds + Hl, Ra, Hr, ld, tid, nt);
  }
  const double sc = 1.0 / ((double)Px * (double)Py * (double)Pz);  // in FP64, rounded once (see body_inv_xy)
  const int nx = bx.n[0], gx = bx.g[0];
  T* dst0 = a.out[f] + bx.foff + ((int64_t)z * Py + gy) * Px + gx;
#pragma unroll 1
  for (int part = 0; part < 2; ++part) {
    const int R = part ? ny - Ra : Ra;
    bar();
    pair_pass_rows<false>(lds, R, ld, Nh, twr, tid, nt);
    bar();
    fft_dif<+1, MAXR>(lds, R, ld, 1, plx, twx, tid, nt, bar);
    store_rows<T, INC>(dst0 + (part ? (int64_t)Ra * Px : 0), Px, R, nx, gx, sc, lds, ld, posx, tid, nt);
    if (part) return;
    bar();
    hold_block<K, false>(bl, lds, ny - Ra, Hl, ld, tid, nt);
    hold_block<K, false>(br, lds + Hl, ny - Ra, Hr, ld, tid, nt);
  }
}

// ------------------------------------------------ split x / y passes
// For padded planes larger than the LDS the x/y pass is split: x rows and y
// columns are transformed by separate work items through the workspace
// (natural order in memory between the two).  RB rows / CB columns per item.
constexpr int kRB = 16;
constexpr int kCB = 16;

// Records: p0 is the block's first row or column; item = field * records + record.
template <typename T>
struct SplitArgs {
  Tables<T> t;
  const PlaneRec* planes;
  FastDiv np;
  const T* in[9];      // x forward: field inputs
  T* out[6];           // x inverse: field outputs
  cx<T>* spec;
  const PushBlk* push;       // x inverse: fused E,B guard exchange (or null)
  const int32_t* push_off;
};

// x forward: kRB rows of (box, z, field): packed real rows -> half spectrum rows.
template <typename T, int MAXR, class Bar, class Eng = FftValu>
PSATD_HD void body_x_fwd(const SplitArgs<T>& a, int item, int tid, int nt, cx<T>* lds, Bar bar, Eng eng = Eng{}) {
  const int f = (int)fdiv((uint32_t)item, a.np);
  const PlaneRec rec = uniform_load(a.planes + (item - f * (int)a.np.d));
  const BoxD bx = uniform_load(a.t.box + rec.box);
  const int Px = bx.P[0], Py = bx.P[1];
  const int z = rec.z;
  const int y0 = rec.p0;
  const int ny = (Py - y0) < kRB ? (Py - y0) : kRB;
  const int Nh = Px >> 1, H = bx.H, ld = bx.ld;
  const PlanRef plx = plan_ref(a.t.plans + bx.planx);
  cx<T>* twx = lds + kRB * ld;
  cx<T>* twr = twx + Nh;
  int32_t* posx = reinterpret_cast<int32_t*>(twr + Px);
  for (int i = tid; i < Nh; i += nt) posx[i] = a.t.pos[plx->pos + i];
  bar();
  const cx<T>* src = reinterpret_cast<const cx<T>*>(a.in[f] + bx.foff + ((int64_t)z * Py + y0) * Px);
  const cx<T>* gtx = a.t.tw + plx->tw;
  const cx<T>* gtr = a.t.tw + bx.twr;
  const int nrow = ny * Nh;
  const FastDiv dNh = make_fastdiv((uint32_t)Nh);
  copy_batched<8, cx<T>>(nrow + Nh + Px, tid, nt,
                         [&](int i) {
                           if (i < nrow) return src[i];
                           const int j = i - nrow;
                           return j < Nh ? gtx[j] : gtr[j - Nh];
                         },
                         [&](int i, cx<T> v) {
                           if (i < nrow) {
                             const int y = (int)fdiv((uint32_t)i, dNh);
                             lds[y * ld + posx[i - y * Nh]] = v;
                           } else {
                             twx[i - nrow] = v;  // twx, twr contiguous
                           }
                         });
  bar();
  eng.template dit<-1, MAXR>(lds, ny, ld, 1, plx, twx, tid, nt, bar);
  pair_pass_rows<true>(lds, ny, ld, Nh, twr, tid, nt);
  bar();
  cx<T>* dst = spec_at(a.spec, bx, 0, f) + ring_slot(bx, z) * bx.pp + (int64_t)y0 * H;
  const FastDiv dH = make_fastdiv((uint32_t)H);
  copy_batched<8, cx<T>>(ny * H, tid, nt,
                         [&](int i) {
                           const int y = (int)fdiv((uint32_t)i, dH);
                           return lds[y * ld + (i - y * H)];
                         },
                         [&](int i, cx<T> v) { dst[i] = v; });
}

// y columns: kCB half-spectrum columns of (box, z, field), in place in the
// workspace; DIR -1: forward over all planes and 9 fields; +1: inverse over
// interior planes and the 6 outputs.
template <typename T, int DIR, int MAXR, class Bar, class Eng = FftValu>
PSATD_HD void body_y(const SplitArgs<T>& a, int item, int tid, int nt, cx<T>* lds, Bar bar, Eng eng = Eng{}) {
  const int f = (int)fdiv((uint32_t)item, a.np);
  const PlaneRec rec = uniform_load(a.planes + (item - f * (int)a.np.d));
  const BoxD bx = uniform_load(a.t.box + rec.box);
  const int Py = bx.P[1], H = bx.H;
  const int c0 = rec.p0;
  const int nc = (H - c0) < kCB ? (H - c0) : kCB;
  const PlanRef ply = plan_ref(a.t.plans + bx.plany);
  cx<T>* twy = lds + Py * kCB;
  int32_t* posy = reinterpret_cast<int32_t*>(twy + Py);
  for (int i = tid; i < Py; i += nt) posy[i] = a.t.pos[ply->pos + i];
  bar();
  cx<T>* col = c0 + (DIR < 0 ? spec_at(a.spec, bx, 0, f) + ring_slot(bx, rec.z) * bx.pp
                             : a.spec + result_plane(bx, 0, f, rec.z));
  const cx<T>* gty = a.t.tw + ply->tw;
  const int ntot = Py * kCB;
  copy_batched<8, cx<T>>(ntot + Py, tid, nt,
                         [&](int i) {
                           if (i >= ntot) return gty[i - ntot];
                           const int y = i / kCB, c = i % kCB;
                           return c < nc ? col[(int64_t)y * H + c] : cx<T>{T(0), T(0)};
                         },
                         [&](int i, cx<T> v) {
                           if (i >= ntot) {
                             twy[i - ntot] = v;
                             return;
                           }
                           const int y = i / kCB, c = i % kCB;
                           lds[(DIR < 0 ? y : posy[y]) * kCB + c] = v;
                         });
  bar();
  if (DIR < 0)
    eng.template dif<-1, MAXR>(lds, nc, 1, kCB, ply, twy, tid, nt, bar);
  else
    eng.template dit<+1, MAXR>(lds, nc, 1, kCB, ply, twy, tid, nt, bar);
  copy_batched<8, cx<T>>(ntot, tid, nt,
                         [&](int i) {
                           const int y = i / kCB, c = i % kCB;
                           return lds[(DIR < 0 ? posy[y] : y) * kCB + c];
                         },
                         [&](int i, cx<T> v) {
                           const int y = i / kCB, c = i % kCB;
                           if (c < nc) col[(int64_t)y * H + c] = v;
                         });
}

// x inverse: kRB interior rows of (box, interior z, output field):
// half spectrum rows -> real rows, interior cells written (INC: added).
template <typename T, bool INC, int MAXR, bool PUSH = false, class Bar, class Eng = FftValu>
PSATD_HD void body_x_inv(const SplitArgs<T>& a, int item, int tid, int nt, cx<T>* lds, Bar bar, Eng eng = Eng{}) {
  const int f = (int)fdiv((uint32_t)item, a.np);
  const PlaneRec rec = uniform_load(a.planes + (item - f * (int)a.np.d));
  const int s = rec.box;
  const BoxD bx = uniform_load(a.t.box + s);
  const int Px = bx.P[0], Py = bx.P[1], Pz = bx.P[2];
  const int nyi = bx.n[1];
  const int zz = rec.z;
  const int z = bx.g[2] + zz;
  const int yy0 = rec.p0;
  const int ny = (nyi - yy0) < kRB ? (nyi - yy0) : kRB;
  const int y0 = bx.g[1] + yy0;
  const int Nh = Px >> 1, H = bx.H, ld = bx.ld;
  const PlanRef plx = plan_ref(a.t.plans + bx.planx);
  cx<T>* twx = lds + kRB * ld;
  cx<T>* twr = twx + Nh;
  int32_t* posx = reinterpret_cast<int32_t*>(twr + Px);
  for (int i = tid; i < Nh; i += nt) posx[i] = a.t.pos[plx->pos + i];
  const cx<T>* src = a.spec + result_plane(bx, 0, f, zz) + (int64_t)y0 * H;
  const cx<T>* gtx = a.t.tw + plx->tw;
  const cx<T>* gtr = a.t.tw + bx.twr;
  const int nrow = ny * H;
  const FastDiv dH = make_fastdiv((uint32_t)H);
  copy_batched<8, cx<T>>(nrow + Nh + Px, tid, nt,
                         [&](int i) {
                           if (i < nrow) return src[i];
                           const int j = i - nrow;
                           return j < Nh ? gtx[j] : gtr[j - Nh];
                         },
                         [&](int i, cx<T> v) {
                           if (i < nrow) {
                             const int y = (int)fdiv((uint32_t)i, dH);
                             lds[y * ld + (i - y * H)] = v;
                           } else {
                             twx[i - nrow] = v;
                           }
                         });
  bar();
  pair_pass_rows<false>(lds, ny, ld, Nh, twr, tid, nt);
  bar();
  eng.template dif<+1, MAXR>(lds, ny, ld, 1, plx, twx, tid, nt, bar);
  const double sc = 1.0 / ((double)Px * (double)Py * (double)Pz);
  const int nx = bx.n[0], gx = bx.g[0];
  T* dst = a.out[f] + bx.foff + ((int64_t)z * Py + y0) * Px;
  const FastDiv dnx = make_fastdiv((uint32_t)nx);
  [[maybe_unused]] T* ldsT = reinterpret_cast<T*>(lds);
  constexpr bool push = PUSH;  // the fused E,B exchange (compiled only where used)
  copy_batched<8, T>(ny * nx, tid, nt,
                     [&](int i) {
                       const int y = (int)fdiv((uint32_t)i, dnx);
                       const int x = gx + (i - y * nx);
                       const cx<T> v = lds[y * ld + posx[x >> 1]];
                       return (T)((double)((x & 1) ? v.y : v.x) * sc);
                     },
                     [&](int i, T v) {
                       const int y = (int)fdiv((uint32_t)i, dnx);
                       const int x = gx + (i - y * nx);
                       T* q = dst + y * Px + x;
                       const T nv = INC ? *q + v : v;
                       *q = nv;
                       if constexpr (push) ldsT[2 * (y * ld + posx[x >> 1]) + (x & 1)] = nv;
                     });
  if constexpr (push) {
    bar();
    push_guards<T>(a.push, uniform_load(a.push_off + s), uniform_load(a.push_off + s + 1), a.t.box, a.out[f], zz, yy0, yy0 + ny,
                   [&](int yi, int xi) {
                     const int x = gx + xi;
                     return ldsT[2 * ((yi - yy0) * ld + posx[x >> 1]) + (x & 1)];
                   },
                   tid, nt);
  }
}

// --------------------------------------------------------------- exchange

// A guard piece as the fill reads it: the first cell of its first z-plane in
// the owner's interior and in the destination's guard region, and the
// pitches, worked out on the host (one load per work item instead of a chain
// through the piece and both box descriptors).
struct FillPiece {
  int64_t so, dof;    // first cell (plane 0): owner, destination
  int32_t sPl, dPl;   // plane pitches (elements)
  int32_t sP0, dP0;   // row pitches (elements)
  int32_t ly, lx;     // rows per plane, row length
  int32_t vec, pad_;  // 16-byte accesses: offsets, pitches and lx multiples of 16 bytes
};

template <typename T>
struct FillArgs {
  const FillPiece* piece;   // guard pieces (each guard cell in exactly one)
  const int32_t* items;     // prefix over pieces of lz
  const int32_t* piece_of;  // item -> piece
  int32_t ncomp;
  T* comp[9];
};

// 16 bytes of T, copied as one vector access.
template <typename T>
struct alignas(16) Vec16 {
  T v[16 / sizeof(T)];
};

// Fig. 3 step 3: every guard cell takes the value of the owner of its global
// index (mod N).  One item = one z-plane of one guard piece: ly rows of lx
// cells, contiguous in the owner's interior and in the destination's guard
// region, copied for every component (16-byte accesses when rows and bases
// are 16-byte aligned).
template <typename T>
PSATD_HD void body_fill(const FillArgs<T>& a, int item, int tid, int nt) {
  const int b = uniform_load(a.piece_of + item);
  const FillPiece k = uniform_load(a.piece + b);
  const int zi = item - uniform_load(a.items + b);
  const int sP0 = k.sP0, dP0 = k.dP0;
  const int64_t so = k.so + (int64_t)zi * k.sPl;
  const int64_t dof = k.dof + (int64_t)zi * k.dPl;
  constexpr int V = 16 / (int)sizeof(T);
  const bool vec = k.vec != 0;
  const int W = vec ? V : 1;  // elements per access
  const int lw = k.lx / W;
  const int n = k.ly * lw;
  const FastDiv dn = make_fastdiv((uint32_t)n);
  const FastDiv dl = make_fastdiv((uint32_t)lw);
  auto at = [&](int i, int64_t base, int pitch, int& c) {
    c = (int)fdiv((uint32_t)i, dn);
    const int e = i - c * n;
    const int r = (int)fdiv((uint32_t)e, dl);
    return base + (int64_t)r * pitch + (int64_t)(e - r * lw) * W;
  };
  if (vec) {
    copy_batched<4, Vec16<T>>(n * a.ncomp, tid, nt,
        [&](int i) {
          int c;
          const int64_t o = at(i, so, sP0, c);
          return *reinterpret_cast<const Vec16<T>*>(a.comp[c] + o);
        },
        [&](int i, Vec16<T> v) {
          int c;
          const int64_t o = at(i, dof, dP0, c);
          *reinterpret_cast<Vec16<T>*>(a.comp[c] + o) = v;
        });
  } else {
    copy_batched<8, T>(n * a.ncomp, tid, nt,
        [&](int i) {
          int c;
          const int64_t o = at(i, so, sP0, c);  // sets c before the buffer is chosen
          return a.comp[c][o];
        },
        [&](int i, T v) {
          int c;
          const int64_t o = at(i, dof, dP0, c);
          a.comp[c][o] = v;
        });
  }
}

// Deposited currents: a region of a box interior whose cells have the same
// padded copies (the owner's own cells among them), and where each copy's first
// cell lies.
struct SumCopy {
  int64_t off;        // first cell (plane 0, row 0)
  int32_t sPl, sP0;   // plane and row pitches (elements)
};
struct SumRegion {
  int32_t c0, nc;     // copies [c0, c0 + nc), at least 2
  int32_t ly, lx;     // rows per plane, row length
  int32_t vec;        // 16-byte accesses: offsets, pitches and lx multiples of 16 bytes
};

template <typename T>
struct SumArgs {
  const SumRegion* region;
  const SumCopy* copy;
  const int32_t* items;      // prefix over regions of their z extent
  const int32_t* region_of;  // item -> region
  T* comp[3];
};

// J_tot(X) = sum over every padded copy of X, in fixed order (boxes ascending,
// then z, y, x positions ascending), written back to every copy.  One item =
// one z-plane of one region; no other item touches its cells, so the sum and
// the exchange of the summed currents are one pass, and cells with one copy are
// not touched.  The copies of a cell are found on the host: looked up per cell
// through the boxes, with the exchange as a pass of its own, 64 boxes of 96^3
// padded in FP32 took 0.75 + 0.22 ms, now 0.345 ms (1.3 GB, 3.8 TB/s).
template <typename T, typename V>
PSATD_HD void sum_plane(const SumArgs<T>& a, const SumRegion& r, int zi, int tid, int nt) {
  constexpr int E = sizeof(V) / sizeof(T);
  const int lw = r.lx / E;
  const FastDiv dl = make_fastdiv((uint32_t)lw);
  const SumCopy* cs = a.copy + r.c0;
  for (int i = tid; i < r.ly * lw; i += nt) {
    const int y = (int)fdiv((uint32_t)i, dl);
    const int x = (i - y * lw) * E;
    auto at = [&](int c) {
      const SumCopy k = uniform_load(cs + c);
      return k.off + (int64_t)zi * k.sPl + (int64_t)y * k.sP0 + x;
    };
    T acc[3][E];
    for (int u = 0; u < 3; ++u)
      for (int e = 0; e < E; ++e) acc[u][e] = T(0);
    // four copies' loads in flight
    for (int c0 = 0; c0 < r.nc; c0 += 4) {
      V v[4][3];
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (c0 + c < r.nc) {
          const int64_t o = at(c0 + c);
#pragma unroll
          for (int u = 0; u < 3; ++u) v[c][u] = *reinterpret_cast<const V*>(a.comp[u] + o);
        }
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (c0 + c < r.nc) {
#pragma unroll
          for (int u = 0; u < 3; ++u) {
            const T* t = reinterpret_cast<const T*>(&v[c][u]);
#pragma unroll
            for (int e = 0; e < E; ++e) acc[u][e] += t[e];
          }
        }
    }
    for (int c = 0; c < r.nc; ++c) {
      const int64_t o = at(c);
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        V w;
        T* t = reinterpret_cast<T*>(&w);
#pragma unroll
        for (int e = 0; e < E; ++e) t[e] = acc[u][e];
        *reinterpret_cast<V*>(a.comp[u] + o) = w;
      }
    }
  }
}

template <typename T>
PSATD_HD void body_sum(const SumArgs<T>& a, int item, int tid, int nt) {
  const int b = uniform_load(a.region_of + item);
  const SumRegion r = uniform_load(a.region + b);
  const int zi = item - uniform_load(a.items + b);
  if (r.vec) sum_plane<T, Vec16<T>>(a, r, zi, tid, nt);
  else sum_plane<T, T>(a, r, zi, tid, nt);
}

// ------------------------------------------------------- scatter / gather
template <typename T>
struct ScatterArgs {
  const BoxD* box;
  int32_t nsub;
  const int32_t* items;  // scatter: prefix of P[2]; gather: prefix of n[2]
  int32_t N[3];
  const T* src[3];
  T* dst[3];
};

template <typename T>
PSATD_HD void body_scatter(const ScatterArgs<T>& a, int item, int tid, int nt) {
  const int s = find_box(a.items, a.nsub, item);
  const BoxD& bx = a.box[s];
  const int z = item - a.items[s];
  const int Px = bx.P[0], Py = bx.P[1];
  const int Z = pmod(bx.lo[2] - bx.g[2] + z, a.N[2]);
  for (int i = tid; i < Px * Py; i += nt) {
    const int y = i / Px;
    const int x = i - y * Px;
    const int Y = pmod(bx.lo[1] - bx.g[1] + y, a.N[1]);
    const int X = pmod(bx.lo[0] - bx.g[0] + x, a.N[0]);
    const int64_t gi = ((int64_t)Z * a.N[1] + Y) * a.N[0] + X;
    const int64_t pi = bx.foff + ((int64_t)z * Py + y) * Px + x;
    for (int c = 0; c < 3; ++c) a.dst[c][pi] = a.src[c][gi];
  }
}

template <typename T>
PSATD_HD void body_gather(const ScatterArgs<T>& a, int item, int tid, int nt) {
  const int s = find_box(a.items, a.nsub, item);
  const BoxD& bx = a.box[s];
  const int z = item - a.items[s];
  const int nx = bx.n[0], ny = bx.n[1];
  for (int i = tid; i < nx * ny; i += nt) {
    const int y = i / nx;
    const int x = i - y * nx;
    const int64_t gi = ((int64_t)(bx.lo[2] + z) * a.N[1] + (bx.lo[1] + y)) * a.N[0] + (bx.lo[0] + x);
    const int64_t pi = bx.foff + ((int64_t)(z + bx.g[2]) * bx.P[1] + (y + bx.g[1])) * bx.P[0] + (x + bx.g[0]);
    for (int c = 0; c < 3; ++c) a.dst[c][gi] = a.src[c][pi];
  }
}

// ------------------------------------------------ modified wavenumbers (a1)
// Sec. 3.1: [k](m) = sum_{j=1}^{p/2} w_j sin(j k_m du)/(du/2), k_m = 2 pi m~/(N du),
// w_1 = M/(M+1), w_{j+1} = -w_j j/(j+1) (M-j)/(M+j+1), M = p/2; p = 0: [k] = k_m.
// Even N: the Nyquist entry is exactly 0.
struct KEntry {
  int32_t N;
  int32_t off;
  double du;
};

PSATD_HD double modified_k_entry(int N, double du, int p, int m) {
  if ((N % 2 == 0) && 2 * m == N) return 0.0;
  const int mt = (m <= (N - 1) / 2) ? m : m - N;
  const double PI = 3.14159265358979323846;
  if (p == 0) return 2.0 * PI * (double)mt / ((double)N * du);
  const int M = p / 2;
  double w = (double)M / (double)(M + 1);
  double acc = 0.0;
  for (int j = 1; j <= M; ++j) {
    // sin(2 pi j m~ / N) with the integer argument reduced exactly
    const int64_t e = ((int64_t)j * mt) % N;
    acc += w * sin(2.0 * PI * (double)e / (double)N);
    w = -w * ((double)j / (double)(j + 1)) * ((double)(M - j) / (double)(M + j + 1));
  }
  return acc / (0.5 * du);
}

}  // namespace psatd
