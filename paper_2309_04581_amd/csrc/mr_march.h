// A ray's segment in a field, shared by the march kernels.
#pragma once
#include "mr_mfma.h"
#include "mr_render.h"

namespace mr {

// A ray's segment in the field: origin and direction in the field frame,
// the range [lo, hi] it marches and the sample indices k0 .. k1 that cover it.
struct RaySeg {
  float ox, oy, oz, dx, dy, dz, t_a, lo, hi;
  int k0, k1;
};

__device__ __forceinline__ bool ray_seg(const RayQueue& q, int r, const FieldView& F, const MarchParams& P,
                                        RaySeg& S) {
  S.ox = q.ox[r]; S.oy = q.oy[r]; S.oz = q.oz[r];
  S.dx = q.dx[r]; S.dy = q.dy[r]; S.dz = q.dz[r];
  to_field_frame(F, S.ox, S.oy, S.oz, S.dx, S.dy, S.dz);
  S.t_a = (q.depth[r] & 0xFFFF) == 0 ? P.t_near : 0.0f;
  float box0, box1;
  if (!slab_box(F, S.ox, S.oy, S.oz, S.dx, S.dy, S.dz, box0, box1)) return false;
  S.lo = fmaxf(S.t_a, box0);
  S.hi = fminf(fminf(S.t_a + P.span, q.hit_t[r]), box1);
  if (!(S.hi > S.lo)) return false;
  S.k0 = max(0, (int)floorf((S.lo - S.t_a) / P.delta) - 1);
  S.k1 = min(P.n_samples, (int)ceilf((S.hi - S.t_a) / P.delta) + 1);
  return true;
}

__device__ __forceinline__ void ray_update(const RayQueue& q, int r, float T, float l0, float l1, float l2) {
  const float tr = q.tr[r], tg = q.tg[r], tb = q.tb[r];
  q.lr[r] += tr * l0;
  q.lg[r] += tg * l1;
  q.lb[r] += tb * l2;
  q.tr[r] = tr * T;
  q.tg[r] = tg * T;
  q.tb[r] = tb * T;
}

}  // namespace mr
