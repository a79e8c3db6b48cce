// stage_args.hpp -- thread tiles, argument blocks and launchers of the fused
// stage kernels (stage_tile.hpp), shared by the translation units that
// instantiate them and by the host code that picks one.
#pragma once

#include "common.hpp"
#include "kernels.hpp"
#include "mhd_math.hpp"

namespace athmhd {

// Thread tile: BX x BY threads, one per column of a (BX-2) x (BY-2) tile of
// active columns plus a one-column ring.
template <int BX_, int BY_>
struct Tile {
  static constexpr int BX = BX_, BY = BY_, NT = BX_ * BY_, TX = BX_ - 2, TY = BY_ - 2;
};
// Uniform blocks run on one of two tiles (fused_plan picks): 32 x 13 active
// columns in one 8-wave workgroup per CU, which keeps the largest share of
// lanes on active columns (82 %; 80 % at 256^3), or 16 x 12 in a 4-wave
// workgroup, two to a CU (76 %): half the granule, and neither workgroup waits
// at the other's barriers.
using TileU = Tile<34, 15>;
using TileS = Tile<18, 14>;

// Arguments shared by every tile of a stage.
struct StageArgs {
  Gas gas;
  double ct_eps;
  StageCoef cf;          // g0, g1 and (when dt_dev is NULL) beta * dt
  const double* dt_dev;  // optional device copy of dt: bdt = beta * (*dt_dev)
  double beta;
  Floors fl;             // optional primitive floors
  int* bad;              // [0]: threads that met a non-physical cell; floor activations (add_floor_count)
};

struct UniformArgs {
  Geo g;
  StageArgs sa;
  const double* xc;
  const double* xb;
  const double* unc;
  const double* unb;
  double* oc;
  double* ob;
  double* fm;  // NULL, or the face mass-flux output of every block (3 face arrays per block)
  bool domain;  // the tiles cover the domain of a coupled mesh (mesh_domain), not its blocks
  bool lone;    // every workgroup has a CU to itself (FusedPlan)
  int ntx, nty, nseg, kz;
  int64_t total;    // workgroups doing work
  int64_t per_xcd;  // ceil(total / 8)
};

struct BatchArgs {
  const BatchDesc* desc;
  const WorkItem* items;
  int nitems;
  unsigned* queue;  // work counter and workgroups done, both zero at launch and after it
  StageArgs sa;
  const double* xc;
  const double* xb;
  const double* unc;
  const double* unb;
  double* oc;
  double* ob;
  double* fm;  // NULL, or the face mass-flux output, laid out like bface
};

// One stage of uniform blocks / of a batch on thread tile T; one translation
// unit per (T, RECON) holds the kernels.
template <int RECON, class T>
hipError_t launch_uniform(int rs, const UniformArgs& a, hipStream_t s);
// (launch_charac: PLM on characteristic variables, periodic blocks)
template <class T>
hipError_t launch_charac(int rs, const UniformArgs& a, hipStream_t s);
template <class T, int RECON>
hipError_t launch_batch(int rs, const BatchArgs& a, int grid, hipStream_t s, bool mesh);

}  // namespace athmhd
