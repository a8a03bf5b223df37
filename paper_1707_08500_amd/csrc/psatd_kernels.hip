// __global__ wrappers and launchers for the phases of the local-FFT PSATD step.
//
// Every phase is ONE launch over a flattened work list spanning all subdomains
// (uneven sizes and guard widths included): a work-group takes items
// blockIdx.x, blockIdx.x + gridDim.x, ... so the same kernel runs either one
// work-group per item or as a persistent grid.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "mfma_dft.hpp"
#include "psatd_launch.hpp"
#include "zreg.hpp"

namespace psatd {

struct BlockBarrier {
  __device__ void operator()() const { __syncthreads(); }
};

extern __shared__ __attribute__((aligned(16))) unsigned char psatd_lds[];

// The matrix-core instruction of the split-BF16 DFT stage.
struct MmaHw {
  __device__ f32x4 operator()(bf16x8 a, bf16x8 b, f32x4 c) const {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// FFT engine by precision form: SPL = 0 VALU radix stages; 2 or 3 BF16 terms
// in a matrix-core first stage.
template <int SPL>
struct EngOf {
  using type = FftMfma<SPL, MmaHw>;
};
template <>
struct EngOf<0> {
  using type = FftValu;
};

// Work-groups are dispatched round-robin over the 8 XCDs; with remap, block
// b of the first 8*floor(G/8) takes item (b % 8) * (G/8) + b / 8 so that
// consecutive items (neighbouring memory) run on one XCD and share its L2.
__device__ __forceinline__ int first_item(int remap) {
  int b = blockIdx.x;
  const int G = gridDim.x;
  if (remap && G >= 8) {
    const int full = G & ~7;
    if (b < full) b = (b & 7) * (full >> 3) + (b >> 3);
  }
  return b;
}

// The thread's index, opaque to the compiler: the persistent loops of the
// kernels below would otherwise hoist what depends on it alone out of the loop
// and hold it in registers through every phase.
__device__ __forceinline__ int fresh_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

template <typename T, int NT, int MAXR, int SPL>
__global__ __launch_bounds__(NT) void k_fwd_xy(FwdArgs<T> a, int nitems, int remap) {
  cx<T>* lds = reinterpret_cast<cx<T>*>(psatd_lds);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_fwd_xy<T, MAXR>(a, it, fresh_tid(), NT, lds, BlockBarrier{}, typename EngOf<SPL>::type{});
    __syncthreads();
  }
}

template <typename T, bool INC, int NT, int MAXR, int SPL, bool PUSH>
__global__ __launch_bounds__(NT) void k_inv_xy(InvArgs<T> a, int nitems, int remap) {
  cx<T>* lds = reinterpret_cast<cx<T>*>(psatd_lds);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_inv_xy<T, INC, MAXR, PUSH>(a, it, fresh_tid(), NT, lds, BlockBarrier{},
                                    typename EngOf<SPL>::type{});
    __syncthreads();
  }
}

// Planes in two halves.
template <typename T, bool INC, int MAXR>
__global__ __launch_bounds__(kThreadsHalf) void k_inv_half(InvArgs<T> a, int nitems, int remap) {
  cx<T>* lds = reinterpret_cast<cx<T>*>(psatd_lds);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_inv_half<T, INC, MAXR>(a, it, fresh_tid(), kThreadsHalf, lds, BlockBarrier{});
    __syncthreads();
  }
}

// FP32: at most 128 VGPRs, so that two 512-thread tiles share a CU (four
// waves per SIMD); FP64 tiles measured slower when held to that budget.
template <typename T, int NT, int PB, bool INC, int MAXR, int SPL>
__global__ __launch_bounds__(NT, sizeof(T) == 4 ? 4 : 1) void k_z_update(UpdArgs<T> a, int nitems,
                                                                          int remap) {
  cx<T>* lds = reinterpret_cast<cx<T>*>(psatd_lds);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_z_update<T, PB, INC, MAXR>(a, it, fresh_tid(), NT, lds, BlockBarrier{}, typename EngOf<SPL>::type{});
    __syncthreads();
  }
}

// J's transform in registers (FP64).
template <typename T, int PB, bool INC, int MAXR>
__global__ __launch_bounds__(kThreadsHeld) void k_z_held(UpdArgs<T> a, int nitems, int remap) {
  cx<T>* lds = reinterpret_cast<cx<T>*>(psatd_lds);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_z_held<T, PB, INC, MAXR>(a, it, fresh_tid(), kThreadsHeld, lds, BlockBarrier{});
    __syncthreads();
  }
}

// Register z pass (FP32 forms, padded z length N).  The VGPR budget keeps
// at least MINW waves per SIMD resident.
template <int N, int L, int W, int MINW>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(MINW)))
void k_z_reg(UpdArgs<float> a, const int32_t* items, int nitems, int remap) {
  __shared__ __attribute__((aligned(16))) unsigned char lds_raw[ZReg<N, L, W>::LDS_BYTES];
  cx<float>* lds = reinterpret_cast<cx<float>*>(lds_raw);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_z_reg<N, L, W>(a, items, it, threadIdx.x, lds);
    __syncthreads();
  }
}

// FP32: at most 128 VGPRs (4 waves per SIMD); the compiler's own choice of 130 left
// three resident: 0.155 -> 0.134 ms on 64 boxes of 96^3 padded.  Budgets for 5 and 6
// waves spill: 0.187 and 0.269 ms.
template <typename T, int PB, bool INC, int MAXR, int SPL>
__global__ __launch_bounds__(kThreadsXY, sizeof(T) == 4 && SPL == 0 ? 4 : 1) void k_z_heat(HeatArgs<T> a, int nitems, int remap) {
  cx<T>* lds = reinterpret_cast<cx<T>*>(psatd_lds);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_z_heat<T, PB, INC, MAXR>(a, it, fresh_tid(), kThreadsXY, lds, BlockBarrier{},
                                  typename EngOf<SPL>::type{});
    __syncthreads();
  }
}

template <typename T, int MAXR, int SPL>
__global__ __launch_bounds__(kThreadsXY) void k_x_fwd(SplitArgs<T> a, int nitems, int remap) {
  cx<T>* lds = reinterpret_cast<cx<T>*>(psatd_lds);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_x_fwd<T, MAXR>(a, it, fresh_tid(), kThreadsXY, lds, BlockBarrier{}, typename EngOf<SPL>::type{});
    __syncthreads();
  }
}

template <typename T, int DIR, int MAXR, int SPL>
__global__ __launch_bounds__(kThreadsXY) void k_y(SplitArgs<T> a, int nitems, int remap) {
  cx<T>* lds = reinterpret_cast<cx<T>*>(psatd_lds);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_y<T, DIR, MAXR>(a, it, fresh_tid(), kThreadsXY, lds, BlockBarrier{}, typename EngOf<SPL>::type{});
    __syncthreads();
  }
}

template <typename T, bool INC, int MAXR, int SPL, bool PUSH>
__global__ __launch_bounds__(kThreadsXY) void k_x_inv(SplitArgs<T> a, int nitems, int remap) {
  cx<T>* lds = reinterpret_cast<cx<T>*>(psatd_lds);
  for (int it = first_item(remap); it < nitems; it += gridDim.x) {
    body_x_inv<T, INC, MAXR, PUSH>(a, it, fresh_tid(), kThreadsXY, lds, BlockBarrier{},
                                   typename EngOf<SPL>::type{});
    __syncthreads();
  }
}

template <typename T>
__global__ __launch_bounds__(kThreadsXY) void k_fill(FillArgs<T> a, int nitems, int remap) {
  for (int item = first_item(remap); item < nitems; item += gridDim.x)
    body_fill(a, item, threadIdx.x, blockDim.x);
}

template <typename T>
__global__ __launch_bounds__(kThreadsXY) void k_sum(SumArgs<T> a, int nitems, int remap) {
  for (int item = first_item(remap); item < nitems; item += gridDim.x)
    body_sum(a, item, threadIdx.x, blockDim.x);
}

template <typename T>
__global__ __launch_bounds__(kThreadsXY) void k_scatter(ScatterArgs<T> a, int nitems) {
  for (int item = blockIdx.x; item < nitems; item += gridDim.x)
    body_scatter(a, item, threadIdx.x, blockDim.x);
}

template <typename T>
__global__ __launch_bounds__(kThreadsXY) void k_gather(ScatterArgs<T> a, int nitems) {
  for (int item = blockIdx.x; item < nitems; item += gridDim.x)
    body_gather(a, item, threadIdx.x, blockDim.x);
}

static __global__ __launch_bounds__(256) void k_modk(const KEntry* ent, int nent, int maxN, int p,
                                              double* kmod) {
  const int e = blockIdx.y;
  if (e >= nent) return;
  const KEntry k = ent[e];
  for (int m = blockIdx.x * blockDim.x + threadIdx.x; m < k.N; m += gridDim.x * blockDim.x)
    kmod[k.off + m] = modified_k_entry(k.N, k.du, p, m);
}

// ------------------------------------------------------------------ helpers
static inline int grid_for(int nitems, int cap) {
  if (nitems <= 0) return 0;
  return (cap > 0 && cap < nitems) ? cap : nitems;
}

template <typename T>
static Tables<T> tables(const DevPlan& p) {
  Tables<T> t;
  t.box = p.box;
  t.nsub = p.nsub;
  t.plans = p.plans;
  t.tw = reinterpret_cast<const cx<T>*>(p.tw);
  t.pos = p.pos;
  t.kmod = p.kmod;
  return t;
}

// The FP32 path transforms increments (INC), the FP64 path the new fields.
template <typename T> struct IncOf { static constexpr bool value = sizeof(T) == 4; };

static hipError_t set_lds(const void* f, int lds) {
  return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
}

template <typename T, int MAXR, int SPL>
hipError_t prepare_t(int ldsF, int ldsI, int ldsU, int ldsX, int ldsY) {
  constexpr bool I = IncOf<T>::value;
  const void* xy[] = {(const void*)k_fwd_xy<T, 256, MAXR, SPL>, (const void*)k_fwd_xy<T, 512, MAXR, SPL>,
                      (const void*)k_fwd_xy<T, 1024, MAXR, SPL>};
  const void* inv[] = {(const void*)k_inv_xy<T, I, 256, MAXR, SPL, false>,
                       (const void*)k_inv_xy<T, I, 512, MAXR, SPL, false>,
                       (const void*)k_inv_xy<T, I, 1024, MAXR, SPL, false>,
                       (const void*)k_inv_xy<T, I, 256, MAXR, SPL, true>,
                       (const void*)k_inv_xy<T, I, 512, MAXR, SPL, true>,
                       (const void*)k_inv_xy<T, I, 1024, MAXR, SPL, true>};
  const void* upd[] = {(const void*)k_z_update<T, 512, 8, I, MAXR, SPL>,
                       (const void*)k_z_update<T, 512, 16, I, MAXR, SPL>,
                       (const void*)k_z_update<T, 1024, 8, I, MAXR, SPL>,
                       (const void*)k_z_update<T, 1024, 16, I, MAXR, SPL>,
                       (const void*)k_z_update<T, 512, 4, I, MAXR, SPL>,
                       (const void*)k_z_update<T, 512, 6, I, MAXR, SPL>,
                       (const void*)k_z_update<T, 512, 10, I, MAXR, SPL>};
  hipError_t e;
  for (const void* f : xy)
    if (ldsF <= kMaxDynLds && (e = set_lds(f, ldsF)) != hipSuccess) return e;
  for (const void* f : inv)
    if (ldsI <= kMaxDynLds && (e = set_lds(f, ldsI)) != hipSuccess) return e;
  for (const void* f : upd)
    if ((e = set_lds(f, ldsU)) != hipSuccess) return e;
  if constexpr (SPL == 0) {
    if constexpr (sizeof(T) == 4) {
      if ((e = set_lds((const void*)k_inv_half<T, I, MAXR>, kMaxDynLds)) != hipSuccess) return e;
    }
    if ((e = set_lds((const void*)k_z_update<T, 256, 8, I, MAXR, SPL>, ldsU)) != hipSuccess) return e;
    if constexpr (sizeof(T) == 8) {
      for (const void* f : {(const void*)k_z_held<T, 4, I, MAXR>, (const void*)k_z_held<T, 8, I, MAXR>})
        if ((e = set_lds(f, kMaxDynLds / 2)) != hipSuccess) return e;
    }
    if ((e = set_lds((const void*)k_z_update<T, 256, 10, I, MAXR, SPL>, ldsU)) != hipSuccess) return e;
  }
  const void* heat[] = {(const void*)k_z_heat<T, 4, I, MAXR, SPL>, (const void*)k_z_heat<T, 8, I, MAXR, SPL>,
                        (const void*)k_z_heat<T, 16, I, MAXR, SPL>, (const void*)k_z_heat<T, 32, I, MAXR, SPL>};
  for (const void* f : heat)
    if ((e = set_lds(f, ldsU)) != hipSuccess) return e;
  if ((e = set_lds((const void*)k_x_fwd<T, MAXR, SPL>, ldsX)) != hipSuccess) return e;
  if ((e = set_lds((const void*)k_x_inv<T, I, MAXR, SPL, false>, ldsX)) != hipSuccess) return e;
  if ((e = set_lds((const void*)k_x_inv<T, I, MAXR, SPL, true>, ldsX)) != hipSuccess) return e;
  if ((e = set_lds((const void*)k_y<T, -1, MAXR, SPL>, ldsY)) != hipSuccess) return e;
  return set_lds((const void*)k_y<T, 1, MAXR, SPL>, ldsY);
}

// ---------------------------------------------------------------- launchers
// MAXR = 8 kernels exist for the VALU form only.  MR: the pass's largest
// radix (p.maxr for the x/y passes, p.maxrz for the z passes).
#define PSATD_MAXR_SWITCH(SPL, MR, CALL8, CALL16) \
  do {                                             \
    if constexpr ((SPL) > 0) {                     \
      CALL16;                                      \
    } else if ((MR) >= 16) {                       \
      CALL16;                                      \
    } else {                                       \
      CALL8;                                       \
    }                                              \
  } while (0)

// One x/y launch with nt threads per group.
template <typename T, int SPL, class Go>
static hipError_t xy_shape(const DevPlan& p, int nt, Go go) {
  if (nt == 1024)
    PSATD_MAXR_SWITCH(SPL, p.maxr, return (go.template run<1024, 8, SPL>()), return (go.template run<1024, 16, SPL>()));
  if (nt == 512)
    PSATD_MAXR_SWITCH(SPL, p.maxr, return (go.template run<512, 8, SPL>()), return (go.template run<512, 16, SPL>()));
  PSATD_MAXR_SWITCH(SPL, p.maxr, return (go.template run<256, 8, SPL>()), return (go.template run<256, 16, SPL>()));
  return hipSuccess;
}

template <typename T>
struct FwdGo {
  const DevPlan& p;
  const FwdArgs<T>& a;
  int g, lds, n;
  hipStream_t st;
  template <int NT, int MAXR, int SPL>
  hipError_t run() const {
    hipLaunchKernelGGL((k_fwd_xy<T, NT, MAXR, SPL>), dim3(g), dim3(NT), lds, st, a, n, p.xcd);
    return hipGetLastError();
  }
};

// The same for planes in two halves (FP32 vector-ALU form).
static hipError_t inv_half(const DevPlan& p, const InvArgs<float>& a, int g, int lds, int n, hipStream_t st) {
  PSATD_MAXR_SWITCH(
      0, p.maxr,
      hipLaunchKernelGGL((k_inv_half<float, true, 8>), dim3(g), dim3(kThreadsHalf), lds, st, a, n, p.xcd),
      hipLaunchKernelGGL((k_inv_half<float, true, 16>), dim3(g), dim3(kThreadsHalf), lds, st, a, n, p.xcd));
  return hipGetLastError();
}

template <typename T, int SPL>
hipError_t fwd_t(const DevPlan& p, const XyLaunch& l, int64_t sbias, void* const* in9, int nf, int npull, void* spec,
                 hipStream_t st) {
  const int n = l.nf * nf;
  const int g = grid_for(n, p.grid_cap[kPhaseFwd]);
  if (!g) return hipSuccess;
  FwdArgs<T> a;
  a.t = tables<T>(p);
  a.planes = p.fwd + l.f0;
  a.np = make_fastdiv((uint32_t)l.nf);
  a.npull = npull;
  a.pull = p.pullp;
  for (int f = 0; f < 9; ++f) a.in[f] = (f < nf) ? reinterpret_cast<const T*>(in9[f]) : nullptr;
  a.spec = reinterpret_cast<cx<T>*>(spec);
  a.sbias = sbias;
  return xy_shape<T, SPL>(p, l.nt, FwdGo<T>{p, a, g, l.lds, n, st});
}

template <typename T, int NT, int PB, int MAXR, int SPL>
static hipError_t upd_launch(const DevPlan& p, const ZLaunch& l, int g, const UpdArgs<T>& a, hipStream_t st) {
  hipLaunchKernelGGL((k_z_update<T, NT, PB, IncOf<T>::value, MAXR, SPL>), dim3(g), dim3(NT), l.lds, st, a, l.nu,
                     p.xcd);
  return hipGetLastError();
}

template <typename T, int PB, int MAXR>
static hipError_t held_launch(const DevPlan& p, const ZLaunch& l, int g, const UpdArgs<T>& a, hipStream_t st) {
  hipLaunchKernelGGL((k_z_held<T, PB, IncOf<T>::value, MAXR>), dim3(g), dim3(kThreadsHeld), l.lds, st, a, l.nu, p.xcd);
  return hipGetLastError();
}

template <typename T, int MAXR, int SPL>
static hipError_t upd_shape(const DevPlan& p, const ZLaunch& l, int g, const UpdArgs<T>& a, hipStream_t st) {
  if constexpr (SPL == 0) {
    if constexpr (sizeof(T) == 8) {
      if (l.held && l.PB == 4) return held_launch<T, 4, MAXR>(p, l, g, a, st);
      if (l.held) return held_launch<T, 8, MAXR>(p, l, g, a, st);
    }
    if (l.narrow && p.ntu == 512 && l.PB == 8) return upd_launch<T, 256, 8, MAXR, SPL>(p, l, g, a, st);
    if (l.narrow && p.ntu == 512 && l.PB == 10) return upd_launch<T, 256, 10, MAXR, SPL>(p, l, g, a, st);
  }
  if (l.PB == 4) return upd_launch<T, 512, 4, MAXR, SPL>(p, l, g, a, st);
  if (l.PB == 6) return upd_launch<T, 512, 6, MAXR, SPL>(p, l, g, a, st);
  if (l.PB == 10) return upd_launch<T, 512, 10, MAXR, SPL>(p, l, g, a, st);
  if (p.ntu == 1024)
    return l.PB == 16 ? upd_launch<T, 1024, 16, MAXR, SPL>(p, l, g, a, st)
                      : upd_launch<T, 1024, 8, MAXR, SPL>(p, l, g, a, st);
  return l.PB == 16 ? upd_launch<T, 512, 16, MAXR, SPL>(p, l, g, a, st)
                    : upd_launch<T, 512, 8, MAXR, SPL>(p, l, g, a, st);
}

template <typename T, int SPL>
hipError_t upd_t(const DevPlan& p, const ZLaunch& l, int64_t sbias, void* spec, hipStream_t st) {
  const int g = grid_for(l.nu, p.grid_cap[kPhaseUpd]);
  if (!g) return hipSuccess;
  UpdArgs<T> a;
  a.t = tables<T>(p);
  a.items = p.tiles + l.u0;
  a.spec = reinterpret_cast<cx<T>*>(spec);
  a.sbias = sbias;
  a.k.c = p.c;
  a.k.dt = p.dt;
  PSATD_MAXR_SWITCH(SPL, p.maxrz, return (upd_shape<T, 8, SPL>(p, l, g, a, st)),
                    return (upd_shape<T, 16, SPL>(p, l, g, a, st)));
  return hipSuccess;
}

template <typename T>
struct InvGo {
  const DevPlan& p;
  const InvArgs<T>& a;
  int g, lds, n;
  hipStream_t st;
  template <int NT, int MAXR, int SPL>
  hipError_t run() const {
    if (a.push_off)
      hipLaunchKernelGGL((k_inv_xy<T, IncOf<T>::value, NT, MAXR, SPL, true>), dim3(g), dim3(NT), lds, st, a, n, p.xcd);
    else
      hipLaunchKernelGGL((k_inv_xy<T, IncOf<T>::value, NT, MAXR, SPL, false>), dim3(g), dim3(NT), lds, st, a, n,
                         p.xcd);
    return hipGetLastError();
  }
};

template <typename T, int SPL>
hipError_t inv_t(const DevPlan& p, const XyLaunch& l, int64_t sbias, const void* spec, void* const* out6, int nf,
                 hipStream_t st) {
  const int n = l.ni * nf;
  const int g = grid_for(n, p.grid_cap[kPhaseInv]);
  if (!g) return hipSuccess;
  InvArgs<T> a;
  a.t = tables<T>(p);
  a.planes = p.inv + l.i0;
  a.np = make_fastdiv((uint32_t)l.ni);
  a.spec = reinterpret_cast<const cx<T>*>(spec);
  a.sbias = sbias;
  for (int f = 0; f < 6; ++f) a.out[f] = f < nf ? reinterpret_cast<T*>(out6[f]) : nullptr;
  const bool fuse = p.fuse && nf == 6;
  a.push = fuse ? p.push : nullptr;
  a.push_off = fuse ? p.push_off : nullptr;
  if constexpr (SPL == 0 && sizeof(T) == 4) {
    if (l.half) return inv_half(p, a, g, l.half, n, st);
  }
  return xy_shape<T, SPL>(p, l.nt, InvGo<T>{p, a, g, l.lds, n, st});
}

template <typename T, int SPL>
hipError_t heat_z_t(const DevPlan& p, const ZLaunch& l, void* spec, double D, double dt, hipStream_t st) {
  const int g = grid_for(l.nu, p.grid_cap[kPhaseUpd]);
  if (!g) return hipSuccess;
  HeatArgs<T> a;
  a.t = tables<T>(p);
  a.items = p.tiles + l.u0;
  a.spec = reinterpret_cast<cx<T>*>(spec);
  a.D = D;
  a.dt = dt;
  constexpr bool I = IncOf<T>::value;
  auto go = [&](auto pbc) -> hipError_t {
    constexpr int PB = decltype(pbc)::value;
    PSATD_MAXR_SWITCH(SPL, p.maxrz,
                      hipLaunchKernelGGL((k_z_heat<T, PB, I, 8, SPL>), dim3(g), dim3(kThreadsXY), l.lds, st, a, l.nu,
                                         p.xcd),
                      hipLaunchKernelGGL((k_z_heat<T, PB, I, 16, SPL>), dim3(g), dim3(kThreadsXY), l.lds, st, a, l.nu,
                                         p.xcd));
    return hipGetLastError();
  };
  if (l.PB == 32) return go(std::integral_constant<int, 32>{});
  if (l.PB == 16) return go(std::integral_constant<int, 16>{});
  if (l.PB == 8) return go(std::integral_constant<int, 8>{});
  return go(std::integral_constant<int, 4>{});
}

template <typename T>
static SplitArgs<T> split_args(const DevPlan& p, const PlaneRec* planes, int np, void* spec) {
  SplitArgs<T> a;
  a.t = tables<T>(p);
  a.planes = planes;
  a.np = make_fastdiv((uint32_t)np);
  for (int f = 0; f < 9; ++f) a.in[f] = nullptr;
  for (int f = 0; f < 6; ++f) a.out[f] = nullptr;
  a.spec = reinterpret_cast<cx<T>*>(spec);
  a.push = p.fuse ? p.push : nullptr;
  a.push_off = p.fuse ? p.push_off : nullptr;
  return a;
}

template <typename T, int SPL>
hipError_t x_fwd_t(const DevPlan& p, const XyLaunch& l, void* const* in9, int nf, void* spec, hipStream_t st) {
  const int n = nf * l.nf;
  const int g = grid_for(n, p.grid_cap[kPhaseFwd]);
  if (!g) return hipSuccess;
  SplitArgs<T> a = split_args<T>(p, p.fwd + l.f0, l.nf, spec);
  for (int f = 0; f < nf; ++f) a.in[f] = reinterpret_cast<const T*>(in9[f]);
  PSATD_MAXR_SWITCH(SPL, p.maxr,
                    hipLaunchKernelGGL((k_x_fwd<T, 8, SPL>), dim3(g), dim3(kThreadsXY), p.ldsX, st, a, n, p.xcd),
                    hipLaunchKernelGGL((k_x_fwd<T, 16, SPL>), dim3(g), dim3(kThreadsXY), p.ldsX, st, a, n, p.xcd));
  return hipGetLastError();
}

template <typename T, int SPL>
hipError_t y_t(const DevPlan& p, const XyLaunch& l, int dir, int nf, void* spec, hipStream_t st) {
  const int np = dir < 0 ? l.nc : l.nd;
  const int n = nf * np;
  const int g = grid_for(n, p.grid_cap[dir < 0 ? kPhaseFwd : kPhaseInv]);
  if (!g) return hipSuccess;
  SplitArgs<T> a = split_args<T>(p, dir < 0 ? p.fwd + l.c0 : p.inv + l.d0, np, spec);
  if (dir < 0)
    PSATD_MAXR_SWITCH(SPL, p.maxr,
                      hipLaunchKernelGGL((k_y<T, -1, 8, SPL>), dim3(g), dim3(kThreadsXY), p.ldsY, st, a, n, p.xcd),
                      hipLaunchKernelGGL((k_y<T, -1, 16, SPL>), dim3(g), dim3(kThreadsXY), p.ldsY, st, a, n, p.xcd));
  else
    PSATD_MAXR_SWITCH(SPL, p.maxr,
                      hipLaunchKernelGGL((k_y<T, 1, 8, SPL>), dim3(g), dim3(kThreadsXY), p.ldsY, st, a, n, p.xcd),
                      hipLaunchKernelGGL((k_y<T, 1, 16, SPL>), dim3(g), dim3(kThreadsXY), p.ldsY, st, a, n, p.xcd));
  return hipGetLastError();
}

template <typename T, int SPL>
hipError_t x_inv_t(const DevPlan& p, const XyLaunch& l, const void* spec, void* const* out6, hipStream_t st) {
  const int n = 6 * l.ni;
  const int g = grid_for(n, p.grid_cap[kPhaseInv]);
  if (!g) return hipSuccess;
  SplitArgs<T> a = split_args<T>(p, p.inv + l.i0, l.ni, const_cast<void*>(spec));
  for (int f = 0; f < 6; ++f) a.out[f] = reinterpret_cast<T*>(out6[f]);
  constexpr bool I = IncOf<T>::value;
  auto go = [&](auto pc) {
    constexpr bool PUSH = decltype(pc)::value;
    PSATD_MAXR_SWITCH(
        SPL, p.maxr,
        hipLaunchKernelGGL((k_x_inv<T, I, 8, SPL, PUSH>), dim3(g), dim3(kThreadsXY), p.ldsX, st, a, n, p.xcd),
        hipLaunchKernelGGL((k_x_inv<T, I, 16, SPL, PUSH>), dim3(g), dim3(kThreadsXY), p.ldsX, st, a, n, p.xcd));
  };
  if (a.push_off) go(std::true_type{});
  else go(std::false_type{});
  return hipGetLastError();
}

#undef PSATD_MAXR_SWITCH

// The kernels of the four precision forms are instantiated by explicit
// instantiation definitions, so that the library can be compiled as one
// translation unit per form in parallel (PSATD_TU 1..4: FP64, FP32, BF16x3,
// BF16x6; 0: the dispatch below) or, without PSATD_TU, as a whole.
#define PSATD_FORM(KIND, T, SPL)                                                                                 \
  KIND template hipError_t fwd_t<T, SPL>(const DevPlan&, const XyLaunch&, int64_t, void* const*, int, int,       \
                                         void*, hipStream_t);                                                    \
  KIND template hipError_t upd_t<T, SPL>(const DevPlan&, const ZLaunch&, int64_t, void*, hipStream_t);           \
  KIND template hipError_t inv_t<T, SPL>(const DevPlan&, const XyLaunch&, int64_t, const void*, void* const*,    \
                                         int, hipStream_t);                                                      \
  KIND template hipError_t heat_z_t<T, SPL>(const DevPlan&, const ZLaunch&, void*, double, double,          \
                                            hipStream_t);                                                        \
  KIND template hipError_t x_fwd_t<T, SPL>(const DevPlan&, const XyLaunch&, void* const*, int, void*,            \
                                           hipStream_t);                                                         \
  KIND template hipError_t y_t<T, SPL>(const DevPlan&, const XyLaunch&, int, int, void*, hipStream_t);           \
  KIND template hipError_t x_inv_t<T, SPL>(const DevPlan&, const XyLaunch&, const void*, void* const*,           \
                                           hipStream_t);                                                         \
  KIND template hipError_t prepare_t<T, 16, SPL>(int, int, int, int, int);
#define PSATD_FORM_VALU(KIND, T) \
  PSATD_FORM(KIND, T, 0)         \
  KIND template hipError_t prepare_t<T, 8, 0>(int, int, int, int, int);

#ifndef PSATD_TU
#define PSATD_TU -1
#endif
#if PSATD_TU == 1 || PSATD_TU < 0
PSATD_FORM_VALU(, double)
#else
PSATD_FORM_VALU(extern, double)
#endif
#if PSATD_TU == 2 || PSATD_TU < 0
PSATD_FORM_VALU(, float)
#else
PSATD_FORM_VALU(extern, float)
#endif
#if PSATD_TU == 3 || PSATD_TU < 0
PSATD_FORM(, float, 2)
#else
PSATD_FORM(extern, float, 2)
#endif
#if PSATD_TU == 4 || PSATD_TU < 0
PSATD_FORM(, float, 3)
#else
PSATD_FORM(extern, float, 3)
#endif

#if PSATD_TU <= 0
#define PSATD_BY_FORM(F, ...)                        \
  do {                                               \
    if (p.f64) return F<double, 0>(__VA_ARGS__);     \
    if (p.spl == 2) return F<float, 2>(__VA_ARGS__); \
    if (p.spl == 3) return F<float, 3>(__VA_ARGS__); \
    return F<float, 0>(__VA_ARGS__);                 \
  } while (0)

hipError_t prepare_kernels(bool f64, int spl, int ldsF, int ldsI, int ldsU, int ldsX, int ldsY) {
  hipError_t e;
  if (f64) {
    if ((e = prepare_t<double, 8, 0>(ldsF, ldsI, ldsU, ldsX, ldsY)) != hipSuccess) return e;
    return prepare_t<double, 16, 0>(ldsF, ldsI, ldsU, ldsX, ldsY);
  }
  if (spl == 2) return prepare_t<float, 16, 2>(ldsF, ldsI, ldsU, ldsX, ldsY);
  if (spl == 3) return prepare_t<float, 16, 3>(ldsF, ldsI, ldsU, ldsX, ldsY);
  if ((e = prepare_t<float, 8, 0>(ldsF, ldsI, ldsU, ldsX, ldsY)) != hipSuccess) return e;
  return prepare_t<float, 16, 0>(ldsF, ldsI, ldsU, ldsX, ldsY);
}

hipError_t launch_fwd(const DevPlan& p, const XyLaunch& l, int64_t sbias, void* const* in9, int nf, int npull,
                      void* spec, hipStream_t st) {
  PSATD_BY_FORM(fwd_t, p, l, sbias, in9, nf, npull, spec, st);
}

hipError_t launch_upd(const DevPlan& p, const ZLaunch& l, int64_t sbias, void* spec, hipStream_t st) {
  PSATD_BY_FORM(upd_t, p, l, sbias, spec, st);
}

hipError_t launch_inv(const DevPlan& p, const XyLaunch& l, int64_t sbias, const void* spec, void* const* out6, int nf,
                      hipStream_t st) {
  PSATD_BY_FORM(inv_t, p, l, sbias, spec, out6, nf, st);
}

hipError_t launch_heat_z(const DevPlan& p, const ZLaunch& l, void* spec, double D, double dt,
                         hipStream_t st) {
  PSATD_BY_FORM(heat_z_t, p, l, spec, D, dt, st);
}

hipError_t launch_x_fwd(const DevPlan& p, const XyLaunch& l, void* const* in9, int nf, void* spec, hipStream_t st) {
  PSATD_BY_FORM(x_fwd_t, p, l, in9, nf, spec, st);
}

hipError_t launch_y(const DevPlan& p, const XyLaunch& l, int dir, int nf, void* spec, hipStream_t st) {
  PSATD_BY_FORM(y_t, p, l, dir, nf, spec, st);
}

hipError_t launch_x_inv(const DevPlan& p, const XyLaunch& l, const void* spec, void* const* out6, hipStream_t st) {
  PSATD_BY_FORM(x_inv_t, p, l, spec, out6, st);
}

template <typename T>
static hipError_t fill_t(const DevPlan& p, void* const* comps, int ncomp, hipStream_t st) {
  FillArgs<T> a;
  a.piece = p.fillp;
  a.items = p.itemsG;
  a.piece_of = p.pieceOf;
  a.ncomp = ncomp;
  for (int c = 0; c < 9; ++c) a.comp[c] = (c < ncomp) ? reinterpret_cast<T*>(comps[c]) : nullptr;
  const int g = grid_for(p.nG, p.grid_cap[kPhaseExchEB]);
  if (!g) return hipSuccess;
  hipLaunchKernelGGL(k_fill<T>, dim3(g), dim3(kThreadsXY), 0, st, a, p.nG, p.xcd);
  return hipGetLastError();
}

hipError_t launch_fill(const DevPlan& p, void* const* comps, int ncomp, hipStream_t st) {
  return p.f64 ? fill_t<double>(p, comps, ncomp, st) : fill_t<float>(p, comps, ncomp, st);
}

template <typename T>
static hipError_t sum_t(const DevPlan& p, void* const* J, hipStream_t st) {
  SumArgs<T> a;
  a.region = p.sumr;
  a.copy = p.sumc;
  a.items = p.itemsS;
  a.region_of = p.regionOf;
  for (int c = 0; c < 3; ++c) a.comp[c] = reinterpret_cast<T*>(J[c]);
  const int g = grid_for(p.nS, p.grid_cap[kPhaseExchJ]);
  if (!g) return hipSuccess;
  hipLaunchKernelGGL(k_sum<T>, dim3(g), dim3(kThreadsXY), 0, st, a, p.nS, p.xcd);
  return hipGetLastError();
}

hipError_t launch_sum(const DevPlan& p, void* const* J, hipStream_t st) {
  return p.f64 ? sum_t<double>(p, J, st) : sum_t<float>(p, J, st);
}

template <int N, int L, int W, int MINW>
static hipError_t zreg_go(const UpdArgs<float>& a, const int32_t* items, int n, int cap, int remap,
                          hipStream_t st) {
  const int g = grid_for(n, cap);
  if (!g) return hipSuccess;
  hipLaunchKernelGGL((k_z_reg<N, L, W, MINW>), dim3(g), dim3(64 * W), 0, st, a, items, n, remap);
  return hipGetLastError();
}

// One launch per group of boxes sharing a padded z length (every box of the
// plan belongs to a group with a register schedule, see zreg_schedule).
hipError_t launch_upd_reg(const DevPlan& p, void* spec, hipStream_t st) {
  UpdArgs<float> a;
  a.t = tables<float>(p);
  a.items = nullptr;
  a.spec = reinterpret_cast<cx<float>*>(spec);
  a.sbias = 0;
  a.k.c = p.c;
  a.k.dt = p.dt;
  const int cap = p.grid_cap[kPhaseUpd];
  for (int i = 0; i < p.nzg; ++i) {
    const ZGroup& zg = p.zg[i];
    const int32_t* items = p.itemsZR + zg.off;
    hipError_t e = hipErrorInvalidValue;
    switch (zg.N) {
#define PSATD_ZREG_CASE(N_, L_, W_, MINW_) \
  case N_: e = zreg_go<N_, L_, W_, MINW_>(a, items, zg.n, cap, p.xcd, st); break;
      PSATD_ZREG_SHAPES(PSATD_ZREG_CASE)
#undef PSATD_ZREG_CASE
      default: break;
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename T>
static hipError_t scat_t(const DevPlan& p, const void* const* src, void* const* dst, bool scatter,
                         hipStream_t st) {
  ScatterArgs<T> a;
  a.box = p.box;
  a.nsub = p.nsub;
  a.items = scatter ? p.itemsP : p.itemsN;
  for (int u = 0; u < 3; ++u) a.N[u] = p.N[u];
  for (int c = 0; c < 3; ++c) {
    a.src[c] = reinterpret_cast<const T*>(src[c]);
    a.dst[c] = reinterpret_cast<T*>(dst[c]);
  }
  const int n = scatter ? p.nP : p.nN;
  if (!n) return hipSuccess;
  if (scatter)
    hipLaunchKernelGGL(k_scatter<T>, dim3(n), dim3(kThreadsXY), 0, st, a, n);
  else
    hipLaunchKernelGGL(k_gather<T>, dim3(n), dim3(kThreadsXY), 0, st, a, n);
  return hipGetLastError();
}

hipError_t launch_scatter(const DevPlan& p, const void* const* glob, void* const* pad, hipStream_t st) {
  return p.f64 ? scat_t<double>(p, glob, pad, true, st) : scat_t<float>(p, glob, pad, true, st);
}

hipError_t launch_gather(const DevPlan& p, const void* const* pad, void* const* glob, hipStream_t st) {
  return p.f64 ? scat_t<double>(p, pad, glob, false, st) : scat_t<float>(p, pad, glob, false, st);
}

hipError_t launch_modk(const KEntry* entries, int nent, int maxN, int order_p, double* kmod,
                       hipStream_t st) {
  if (nent <= 0) return hipSuccess;
  const int bx = (maxN + 255) / 256;
  hipLaunchKernelGGL(k_modk, dim3(bx, nent), dim3(256), 0, st, entries, nent, maxN, order_p, kmod);
  return hipGetLastError();
}

#endif  // PSATD_TU <= 0

}  // namespace psatd
