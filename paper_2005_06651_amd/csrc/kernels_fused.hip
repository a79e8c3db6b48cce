// kernels_fused.hip -- host side of the fused stage kernels: thread tile and
// x3 segment length of a launch, and the launchers of uniform and batched
// stages.  The kernels (stage_tile.hpp) are compiled in the stage_*.hip units.
#include <algorithm>
#include <cmath>

#include "stage_args.hpp"

namespace athmhd {

// Workgroup rounds of a launch, in units of one round of the 34 x 15 tile (one
// workgroup of 8 waves per CU).  Two 18 x 14 workgroups of 4 waves share a CU:
//   * with DC and PLM a full round of them costs as much as one of the larger
//     tile (15.9 and 16.0 us per plane of a VL2 step), with PPM 0.95 of it, and
//     0.9 when rounds follow each other, as their barriers then fall apart
//     (RK3 at 256^3: 53.5 and 47.7 us per plane);
//   * one workgroup alone on each CU takes 0.75 of a round (12 us), with the PPM
//     variant for it (lone) 0.6: 54 us x 0.57 per plane and round in RK3 at 48^3,
//     56^3 and 64^3;
//   * the last, partial round overlaps the one before it: at least half a
//     round, else its share of the CUs (2.75 rounds at 128^3 measured 2.79,
//     1.375 rounds 1.5).
static double rounds_small(int64_t wgs, int cus, int recon, bool lone) {
  const double r = (double)wgs / (2.0 * cus);
  const double full = std::floor(r), f = r - full;
  const double tail = f == 0.0 ? 0.0 : full == 0.0 ? (f <= 0.5 ? (lone ? 0.6 : 0.75) : 1.0) : std::max(0.5, f);
  return (full + tail) * (recon < 2 ? 1.0 : r < 4.0 ? 0.95 : 0.9);
}

// Thread tile and x3 segment length of a launch: the pair with the least
// planes x rounds.  A segment of kz planes costs kz + 2 plane iterations and a
// window start-up; short segments repeat more of them, long ones leave the
// last round of workgroups nearly empty or the chip unfilled.  The same kernels
// with the rule before (34 x 15 only, kz in 4, 8, .. 32 or 64) and now, sustained
// steps of a smooth state without the CFL pass: VL2+PLM at 64^3 91 -> 78 us, 96^3
// 263 -> 178, 192^3 1350 -> 1207; RK3+PPM at 32^3 325 -> 102, 48^3 328 -> 162, 64^3
// 337 -> 283, 200x150x131 with HLLE 2873 -> 2255.  256^3 VL2+PLM stays on 34 x 15
// and 32 planes (2.66 ms; 18 x 14: 2.98); RK3+PPM runs on 18 x 14 (9.9 ms; 34 x 15:
// 10.1).  The lone variant, without and with: 32^3 122 -> 102 us, 48^3 196 -> 162,
// 56^3 268 -> 222.
FusedPlan fused_plan(const Geo& geo, int recon, int nb, int cus, int kz_fixed) {
  FusedPlan best{false, 1, false};
  Geo g = geo;
  if (mesh_domain(geo)) {
    g.n1 *= geo.mesh[0];
    g.n2 *= geo.mesh[1];
    g.n3 *= geo.mesh[2];
    nb = 1;
  }
  double cost = 1e300;
  const int64_t cols_u = (int64_t)((g.n1 + TileU::TX - 1) / TileU::TX) * ((g.n2 + TileU::TY - 1) / TileU::TY) * nb;
  const int64_t cols_s = (int64_t)((g.n1 + TileS::TX - 1) / TileS::TX) * ((g.n2 + TileS::TY - 1) / TileS::TY) * nb;
  const int lo = kz_fixed > 0 ? kz_fixed : 1, hi = kz_fixed > 0 ? kz_fixed : std::min(g.n3, 128);
  for (int kz = lo; kz <= hi; ++kz) {
    const int nseg = (g.n3 + kz - 1) / kz;
    const double planes = std::min(kz, g.n3) + 2.5;
    // the variant for a CU of one's own: PPM of periodic blocks without scalars
    const bool lone = recon == 2 && cols_s * nseg <= cus && geo.mesh[0] == 0 && geo.ns == 0;
    const double u = planes * (double)((cols_u * nseg + cus - 1) / cus);
    const double v = planes * rounds_small(cols_s * nseg, cus, recon, lone);
    if (u < cost) {
      cost = u;
      best = FusedPlan{false, kz, false};
    }
    if (v < cost) {
      cost = v;
      best = FusedPlan{true, kz, lone};
    }
  }
  return best;
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

template <class T>
static hipError_t launch_uniform_recon(int recon, int rs, const UniformArgs& fa, hipStream_t s) {
  if (recon == 0) return launch_uniform<0, T>(rs, fa, s);
  if (recon == 1) return launch_uniform<1, T>(rs, fa, s);
  return launch_uniform<2, T>(rs, fa, s);
}

hipError_t launch_stage_fused(const Geo& g, double gamma, int recon, int rs, double ct_eps, const double* xc,
                              const double* xb, const double* unc, const double* unb, double* outc, double* outb,
                              StageCoef coef, const double* dt_dev, double beta, int nb, FusedPlan plan, Floors fl, int* bad,
                              double* fm, bool charac, hipStream_t s) {
  if (charac && recon > 0 && (recon != 1 || fm || g.mesh[0])) return hipErrorInvalidValue;
  UniformArgs fa;
  fa.g = g;
  fa.sa = make_stage_args(gamma, ct_eps, coef, dt_dev, beta, fl, bad);
  fa.xc = xc; fa.xb = xb; fa.unc = unc; fa.unb = unb; fa.oc = outc; fa.ob = outb;
  fa.fm = fm;
  fa.kz = plan.kz;
  fa.domain = mesh_domain(g);
  fa.lone = plan.lone;
  const int n1 = fa.domain ? g.mesh[0] * g.n1 : g.n1, n2 = fa.domain ? g.mesh[1] * g.n2 : g.n2;
  const int n3 = fa.domain ? g.mesh[2] * g.n3 : g.n3;
  const int TX = plan.small ? TileS::TX : TileU::TX, TY = plan.small ? TileS::TY : TileU::TY;
  fa.ntx = (n1 + TX - 1) / TX;
  fa.nty = (n2 + TY - 1) / TY;
  fa.nseg = (n3 + fa.kz - 1) / fa.kz;
  fa.total = (int64_t)fa.ntx * fa.nty * fa.nseg * (fa.domain ? 1 : nb);
  fa.per_xcd = (fa.total + 7) / 8;
  if (charac && recon == 1) return plan.small ? launch_charac<TileS>(rs, fa, s) : launch_charac<TileU>(rs, fa, s);
  return plan.small ? launch_uniform_recon<TileS>(recon, rs, fa, s) : launch_uniform_recon<TileU>(recon, rs, fa, s);
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
