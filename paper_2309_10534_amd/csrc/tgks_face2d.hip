// tgks_face2d.hip -- launches of the 2-D face kernel (both directions of a
// stage in one launch, all tile shapes), compiled apart from the rest of the library.
#include "tgks_internal.hpp"

using namespace tgks;

// both directions of one stage in one launch
template <int TILE>
static void launch_face2d_xy(tgks_ctx* c, const StageArgs& ax, const StageArgs& ay, int stage, bool fl) {
  constexpr int TN = tile2_tn(TILE), TT = tile2_tt(TILE);
  const int nx = c->g.n[0], ny = c->g.n[1];
  const long long nb = (long long)((nx + 1 + TN - 1) / TN) * ((ny + TT - 1) / TT) +
                       (long long)((ny + 1 + TN - 1) / TN) * ((nx + TT - 1) / TT);
  const dim3 grid((unsigned)nb), block(2 * TN * TT);
#define LXY(kern) hipLaunchKernelGGL(kern, grid, block, 0, c->stream, ax, ay)
  if (stage == 1) {
    if (fl) {
      if (c->ns) LXY((face2d_xy_kernel<1, true, true, TILE>));
      else LXY((face2d_xy_kernel<1, false, true, TILE>));
    } else {
      if (c->ns) LXY((face2d_xy_kernel<1, true, false, TILE>));
      else LXY((face2d_xy_kernel<1, false, false, TILE>));
    }
  } else {
    if (c->ns) LXY((face2d_xy_kernel<2, true, false, TILE>));
    else LXY((face2d_xy_kernel<2, false, false, TILE>));
  }
#undef LXY
}

// characteristic variables, prescribed sides or the fallback: one tile shape
template <bool CH, bool EX>
static void launch_face2d_xy_one(tgks_ctx* c, const StageArgs& ax, const StageArgs& ay, int stage, bool fl) {
  constexpr int TILE = CHAR_TILE2;
  constexpr int TN = tile2_tn(TILE), TT = tile2_tt(TILE);
  const int nx = c->g.n[0], ny = c->g.n[1];
  const long long nb = (long long)((nx + 1 + TN - 1) / TN) * ((ny + TT - 1) / TT) +
                       (long long)((ny + 1 + TN - 1) / TN) * ((nx + TT - 1) / TT);
  const dim3 grid((unsigned)nb), block(2 * TN * TT);
#define LXY(kern) hipLaunchKernelGGL(kern, grid, block, 0, c->stream, ax, ay)
  if (stage == 1) {
    if (fl) {
      if (c->ns) LXY((face2d_xy_kernel<1, true, true, TILE, CH, EX>));
      else LXY((face2d_xy_kernel<1, false, true, TILE, CH, EX>));
    } else {
      if (c->ns) LXY((face2d_xy_kernel<1, true, false, TILE, CH, EX>));
      else LXY((face2d_xy_kernel<1, false, false, TILE, CH, EX>));
    }
  } else {
    if (c->ns) LXY((face2d_xy_kernel<2, true, false, TILE, CH, EX>));
    else LXY((face2d_xy_kernel<2, false, false, TILE, CH, EX>));
  }
#undef LXY
}

int launch_face2d_xy_any(tgks_ctx* c, const StageArgs& ax, const StageArgs& ay, int stage, bool fl) {
  const bool ch = c->p.recon == TGKS_RECON_CHARACTERISTIC, ex = c->ex;
  if (ch || ex) {
    if (ch && ex) launch_face2d_xy_one<true, true>(c, ax, ay, stage, fl);
    else if (ch) launch_face2d_xy_one<true, false>(c, ax, ay, stage, fl);
    else launch_face2d_xy_one<false, true>(c, ax, ay, stage, fl);
    return TGKS_OK;
  }
  switch (c->tile2) {
    case 1:
      launch_face2d_xy<1>(c, ax, ay, stage, fl);
      break;
    case 2:
      launch_face2d_xy<2>(c, ax, ay, stage, fl);
      break;
    default:
      launch_face2d_xy<0>(c, ax, ay, stage, fl);
  }
  return TGKS_OK;
}
