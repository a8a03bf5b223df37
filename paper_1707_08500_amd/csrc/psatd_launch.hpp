// Device-side view of a plan and the launchers of every phase of the step.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "psatd_device.hpp"

namespace psatd {

enum Phase { kPhaseExchJ = 0, kPhaseFwd = 1, kPhaseUpd = 2, kPhaseInv = 3, kPhaseExchEB = 4, kNumPhases = 5 };

struct DevPlan {
  bool f64;                 // element type: double (true) or float
  int32_t nsub;
  int32_t N[3];
  const BoxD* box;          // with the spectral addresses of the current lists
  const FftPlanD* plans;
  const void* tw;           // cx<double> or cx<float> twiddles
  const int32_t* pos;       // position tables of the FFT plans
  const double* kmod;
  const SumRegion* sumr;    // deposited currents
  const SumCopy* sumc;
  const int32_t* itemsS;
  const int32_t* regionOf;
  int32_t nS;
  const PlaneRec* fwd;      // work lists of the x/y and z passes (see WorkLists)
  const PlaneRec* inv;
  const ZItem* tiles;
  const int32_t* itemsP;    // scatter: P[2]
  const int32_t* itemsN;    // gather: n[2]
  int32_t ldsX, ldsY;
  int32_t split;
  const PushBlk* push;       // guard pieces (guard fill, fused E,B exchange)
  const FillPiece* fillp;    // guard fill: pieces with offsets and pitches
  const int32_t* itemsG;     // guard fill: prefix over pieces of their z extent
  const int32_t* pieceOf;    // guard fill: item -> piece
  int32_t nG;
  const int32_t* push_off;
  int32_t fuse;              // 1: the inverse pass writes the E,B guard copies
  int32_t spl;               // BF16 terms of the matrix-core DFT stage (0: VALU only)
  int32_t nP, nN;
  int32_t zcl;               // 1: one z launch per class of tile size
  int32_t ntu;               // threads per z-update work-group (512 or 1024)
  int32_t ntxy;              // threads per x/y work-group (256, 512 or 1024; 0: per launch class)
  int32_t maxr;              // largest codelet of the x/y schedules (8 or 16)
  int32_t maxrz;             // largest codelet of the z schedules
  int32_t xcd;               // 1: consecutive items on the same XCD (L2 sharing)
  double c, dt;
  int32_t grid_cap[kNumPhases];  // 0: one work-group per item; else persistent grid
  int32_t pull;                  // 1: the forward pass pulls E,B guard cells from their owners
  const PullPiece* pullp;
  int32_t zreg;                  // 1: the z pass runs the register kernels (groups below)
  int32_t nzg;
  ZGroup zg[kMaxZGroups];
  const int32_t* itemsZR;
};

hipError_t launch_fill(const DevPlan& p, void* const* comps, int ncomp, hipStream_t st);
hipError_t launch_sum(const DevPlan& p, void* const* J, hipStream_t st);
// One launch each over a range of the lists.  Forward: the first nf of the 9
// fields (9, 6 when J's spectra are already in the workspace, 1 for heat), of
// which npull read their guard cells from the owners; inverse: nf = 6, or 1.
hipError_t launch_fwd(const DevPlan& p, const XyLaunch& l, int64_t sbias, void* const* in9, int nf, int npull,
                      void* spec, hipStream_t st);
hipError_t launch_upd(const DevPlan& p, const ZLaunch& l, int64_t sbias, void* spec, hipStream_t st);
// the z pass with the z transforms in registers (all boxes, FP32 VALU form)
hipError_t launch_upd_reg(const DevPlan& p, void* spec, hipStream_t st);
hipError_t launch_inv(const DevPlan& p, const XyLaunch& l, int64_t sbias, const void* spec, void* const* out6, int nf,
                      hipStream_t st);
// heat equation (Sec. 5): z pass of one field with the exp(-D |[k]|^2 dt) propagator
hipError_t launch_heat_z(const DevPlan& p, const ZLaunch& l, void* spec, double D, double dt, hipStream_t st);
// split x/y passes (whole plan, no batching)
hipError_t launch_x_fwd(const DevPlan& p, const XyLaunch& l, void* const* in9, int nf, void* spec, hipStream_t st);
hipError_t launch_y(const DevPlan& p, const XyLaunch& l, int dir, int nf, void* spec, hipStream_t st);
hipError_t launch_x_inv(const DevPlan& p, const XyLaunch& l, const void* spec, void* const* out6, hipStream_t st);
hipError_t launch_scatter(const DevPlan& p, const void* const* glob, void* const* pad, hipStream_t st);
hipError_t launch_gather(const DevPlan& p, const void* const* pad, void* const* glob, hipStream_t st);
hipError_t launch_modk(const KEntry* entries, int nent, int maxN, int order_p, double* kmod,
                       hipStream_t st);
hipError_t prepare_kernels(bool f64, int spl, int ldsF, int ldsI, int ldsU, int ldsX, int ldsY);


}  // namespace psatd
