// kernels_fused.hip -- host side of the fused stage kernels: thread tile and
// x3 segment length of a launch, and the launchers of uniform and batched
// stages.  The kernels (stage_tile.hpp) are compiled in the stage_*.hip units.
#include "stage_args.hpp"

namespace athmhd {

int fused_default_kz(const Geo& g, int nb, int cus) {
  // the longest x3 segment (32 planes down to 4) that still gives the launch
  // at least 2.5 workgroups per CU: longer segments repeat less of the
  // window start-up, more segments fill the chip on small blocks.  64 planes
  // where that still leaves 16 workgroups per CU (512^3: 0.9 % faster with
  // PPM; 256^3, with 2.5 per CU, 12 % slower)
  const int64_t tiles = (int64_t)((g.n1 + TileU::TX - 1) / TileU::TX) * ((g.n2 + TileU::TY - 1) / TileU::TY) * nb;
  if (tiles * ((g.n3 + 63) / 64) >= 16 * (int64_t)cus) return 64 < g.n3 ? 64 : g.n3;
  int kz = 32;
  while (kz > 4 && 2 * tiles * ((g.n3 + kz - 1) / kz) < 5 * (int64_t)cus) kz /= 2;
  return kz < g.n3 ? kz : g.n3;
}

static StageArgs make_stage_args(double gamma, double ct_eps, StageCoef coef, const double* dt_dev, double beta,
                                 Floors fl, int* bad) {
  StageArgs sa;
  sa.fl = fl;
  sa.gas = Gas{gamma, gamma - 1.0, 1.0 / (gamma - 1.0)};
  sa.ct_eps = ct_eps;
  sa.cf = coef;
  sa.dt_dev = dt_dev;
  sa.beta = beta;
  sa.bad = bad;
  return sa;
}

hipError_t launch_stage_fused(const Geo& g, double gamma, int recon, int rs, double ct_eps, const double* xc,
                              const double* xb, const double* unc, const double* unb, double* outc, double* outb,
                              StageCoef coef, const double* dt_dev, double beta, int nb, int kz, Floors fl, int* bad,
                              double* fm, hipStream_t s) {
  UniformArgs fa;
  fa.g = g;
  fa.sa = make_stage_args(gamma, ct_eps, coef, dt_dev, beta, fl, bad);
  fa.xc = xc; fa.xb = xb; fa.unc = unc; fa.unb = unb; fa.oc = outc; fa.ob = outb;
  fa.fm = fm;
  fa.kz = kz;
  fa.ntx = (g.n1 + TileU::TX - 1) / TileU::TX;
  fa.nty = (g.n2 + TileU::TY - 1) / TileU::TY;
  fa.nseg = (g.n3 + fa.kz - 1) / fa.kz;
  fa.total = (int64_t)fa.ntx * fa.nty * fa.nseg * nb;
  fa.per_xcd = (fa.total + 7) / 8;
  if (recon == 0) return launch_uniform<0, TileU>(rs, fa, s);
  if (recon == 1) return launch_uniform<1, TileU>(rs, fa, s);
  return launch_uniform<2, TileU>(rs, fa, s);
}

int batch_tile_count() { return 4; }

void batch_tile_shape(int shape, int* tx, int* ty) {
  static const int t[4][2] = {{16, 12}, {12, 16}, {14, 14}, {16, 8}};
  *tx = t[shape][0];
  *ty = t[shape][1];
}

int batch_tile_threads(int shape) {
  int tx, ty;
  batch_tile_shape(shape, &tx, &ty);
  return (tx + 2) * (ty + 2);
}

__global__ void k_zero_u32(unsigned* p) {
  if (threadIdx.x == 0) *p = 0u;
}

template <class T>
static hipError_t launch_batch_recon(int recon, int rs, const BatchArgs& ba, int grid, hipStream_t s, bool mesh) {
  if (recon == 0) return launch_batch<T, 0>(rs, ba, grid, s, mesh);
  if (recon == 1) return launch_batch<T, 1>(rs, ba, grid, s, mesh);
  return launch_batch<T, 2>(rs, ba, grid, s, mesh);
}

hipError_t launch_stage_batch(int shape, double gamma, int recon, int rs, double ct_eps, const BatchDesc* desc,
                              const WorkItem* items, int nitems, unsigned* queue, const double* xc,
                              const double* xb, const double* unc, const double* unb, double* outc, double* outb,
                              StageCoef coef, const double* dt_dev, double beta, int grid, Floors fl, int* bad,
                              double* fm, hipStream_t s, bool mesh) {
  if (mesh && (fl.on() || fm)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, s, queue);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  BatchArgs ba;
  ba.desc = desc;
  ba.items = items;
  ba.nitems = nitems;
  ba.queue = queue;
  ba.sa = make_stage_args(gamma, ct_eps, coef, dt_dev, beta, fl, bad);
  ba.xc = xc; ba.xb = xb; ba.unc = unc; ba.unb = unb; ba.oc = outc; ba.ob = outb;
  ba.fm = fm;
  switch (shape) {
    case 0: return launch_batch_recon<Tile<18, 14>>(recon, rs, ba, grid, s, mesh);
    case 1: return launch_batch_recon<Tile<14, 18>>(recon, rs, ba, grid, s, mesh);
    case 2: return launch_batch_recon<Tile<16, 16>>(recon, rs, ba, grid, s, mesh);
    default: return launch_batch_recon<Tile<18, 10>>(recon, rs, ba, grid, s, mesh);
  }
}

}  // namespace athmhd
