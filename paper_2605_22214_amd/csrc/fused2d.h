// Launch arguments of the fused D2Q9 steps (fused2d.hip).
#pragma once

#include "internal.h"

namespace nflbm {

// One simulation's records before (src) and after (dst) the launch, which
// reads a halo of 2 nsteps nodes around every tile and so never writes what
// it reads.  Tiles are tile_w x tile_h nodes, x fastest.
struct FusedArgs {
  const NFLBM_GLOBAL void* csrc;
  const NFLBM_GLOBAL void* mu_src;
  const NFLBM_GLOBAL void* vel_src;
  const NFLBM_GLOBAL void* frec_src;
  NFLBM_GLOBAL void* cdst;
  NFLBM_GLOBAL void* mu_dst;
  NFLBM_GLOBAL void* vel_dst;
  NFLBM_GLOBAL void* frec_dst;
  NFLBM_GLOBAL int* nanflag;
  int nx, ny;
  int tile_w, tile_h, tiles_x;
  int flags;
};

struct FusedLaunch {
  const FusedArgs* one;       // a single simulation (host), or
  const FusedArgs* batch;     // device [count] with work (member, tile)
  const int2* work;
  const void* params;
  int frecord;                // records of f too; 0: diffusive-only
  int threads;                // workgroup size
  int wlog2;                  // LDS rows of 1 << wlog2 positions
  int blocks;
  int nsteps;
  uint32_t nanmask;           // bit t: step t checks for non-finite values
  size_t lds;
};

// LDS bytes of one position (the fields fused2d.hip lists).
inline size_t fused_position_bytes(int nc, size_t ts, bool frecord) {
  return (3 * size_t(nc - 1) + (frecord ? 10 : 0)) * ts;
}

// One simulation with the concentration-dependent mobility (fused_mob.hip):
// the populations before and after the launch.
struct FusedMobArgs {
  const void* gk_src;
  const void* g0_src;
  void* gk_dst;
  void* g0_dst;
  const void* params;         // DevParams<T>
  const void* mob;            // MobParams<T>
  int* nanflag;
  long long gstride;
  int nx, ny;
  int tile_w, tile_h, tiles_x;
  int flags;
};
// LDS bytes of one position.
inline size_t fused_mob_position_bytes(int nc, size_t ts) { return (2 * size_t(nc) + 3 * size_t(nc - 1)) * ts; }

hipError_t launch_fused_mob_0(int nc, const FusedMobArgs& a, int blocks, int nsteps, uint32_t nanmask, size_t lds,
                              hipStream_t s);
hipError_t launch_fused_mob_1(int nc, const FusedMobArgs& a, int blocks, int nsteps, uint32_t nanmask, size_t lds,
                              hipStream_t s);
hipError_t launch_fused_mob_2(int nc, const FusedMobArgs& a, int blocks, int nsteps, uint32_t nanmask, size_t lds,
                              hipStream_t s);
hipError_t launch_fused2d_0(int nc, const FusedLaunch& f, hipStream_t s);
hipError_t launch_fused2d_1(int nc, const FusedLaunch& f, hipStream_t s);
hipError_t launch_fused2d_2(int nc, const FusedLaunch& f, hipStream_t s);

}  // namespace nflbm
