// Medium of the light samples toward emitters: the optical depth of the
// render's fields along each sample's shadow segment (Eq. 8-9 without the
// colour), so that the light it carries is attenuated as a bounce that reaches
// the emitter is by its own march.
//
// One wave takes a segment, 16 consecutive grid intervals per tile: the lanes
// gather the features straight into the operands of the density MLP's MFMA
// tiles (FP32 as exact BF16 splits in both MLP precisions: the depth has
// always been FP32).  Per thread inside the shade pass, with the MLP on the
// vector units, this took 31 ms of the 800x800 emitter frame (33 M density
// samples, 47.7 ms per frame); a wave per segment takes 9 ms (25.6 ms per
// frame), bound by the gathers' lines from beyond L2.
#include "mr_levels.h"

using namespace mr;

namespace {

// Grid intervals of one shadow segment in the field: interval k covers
// [k delta, (k + 1) delta] clipped to [lo, hi].
struct LightSeg {
  float ox, oy, oz, dx, dy, dz, lo, hi;
  int64_t k0, k1;   // the intervals k0 .. k1 - 1 cover [lo, hi]
};

__device__ __forceinline__ bool light_seg(const RayQueue& q, int64_t i, const FieldView& F, float delta, LightSeg& S) {
  S.ox = q.ox[i]; S.oy = q.oy[i]; S.oz = q.oz[i];
  S.dx = q.dx[i]; S.dy = q.dy[i]; S.dz = q.dz[i];
  to_field_frame(F, S.ox, S.oy, S.oz, S.dx, S.dy, S.dz);
  float b0, b1;
  if (!slab_box(F, S.ox, S.oy, S.oz, S.dx, S.dy, S.dz, b0, b1)) return false;
  S.lo = fmaxf(0.0f, b0);
  S.hi = fminf(q.hit_t[i], b1);
  if (!(S.hi > S.lo)) return false;
  // the intervals that meet [lo, hi], started one early so that FP32 rounding
  // of k delta cannot skip the first; at most 2^20 per field (a box 2^20 grid
  // intervals across), so the loop is bounded (indices clamped below 2^40)
  const float kf0 = fminf(fmaxf(0.0f, floorf(S.lo / delta) - 1.0f), 1.0995e12f);
  const float kf1 = fminf(ceilf(S.hi / delta) + 1.0f, kf0 + (float)(1 << 20));
  S.k0 = (int64_t)kf0;
  S.k1 = (int64_t)kf1 + 1;
  return true;
}

// The light reaches the ray: in its slot of the next queue, or in the output
// when it has ended.
__device__ __forceinline__ void add_light(const RayQueue& q, const RayQueue& next, int64_t i, float tau,
                                          float* __restrict__ radiance) {
  const float t = expf(-tau);
  const int to = q.rid[i];
  if (to >= 0) {
    next.lr[to] += q.tr[i] * t;
    next.lg[to] += q.tg[i] * t;
    next.lb[to] += q.tb[i] * t;
  } else {
    float* out = radiance + 3 * (int64_t)~to;
    out[0] += q.tr[i] * t;
    out[1] += q.tg[i] * t;
    out[2] += q.tb[i] * t;
  }
}

// A segment that the level-by-level kernel leaves to k_light_march: more
// intervals than a batch holds, or indices that FP32 does not hold exactly.
__device__ __forceinline__ bool light_long(const LightSeg& S) { return S.k1 - S.k0 > kLvSamples || S.k1 > (1 << 24); }

// One hash level at a time (mr_levels.h), long queues only: 9.4 -> 6.7 ms of
// light samples in the 800x800 emitter frame (23.1 -> 20.5 ms per frame).
template <typename TabT>
__global__ __launch_bounds__(kLvThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_light_lv(
    RayQueue q, RayQueue next, const int* __restrict__ count, int* __restrict__ work, FieldView F,
    const TabT* __restrict__ table, float delta, int use_occ,
    float* __restrict__ radiance, double* __restrict__ scratch, int* __restrict__ pace) {
  constexpr int NL = 16;
  using LY = FragLayout<NL, 4, 1, false>;
  __shared__ __align__(16) uint32_t sW[LY::C1];
  __shared__ LvBatch B;
  const int cnt = *count;
  if (cnt < kLvMinRays) return;
  stage_density<NL>(F.mlp, sW);
  const int lane = threadIdx.x & 63, j = lane & 15;
  double* my = scratch + (int64_t)blockIdx.x * kLvSamples * NL;
  LvPace pc(pace);
  const int grab = lv_grab(cnt);
  int cur = 0, end = 0;
  while (true) {
    if (threadIdx.x < 64)
      B.take(work, cnt, grab, cur, end, [&](int i, RaySeg& S) {
        LightSeg L;
        if (q.hit_p[i] != kLightPending || !light_seg(q, i, F, delta, L) || light_long(L)) return false;
        S.ox = L.ox; S.oy = L.oy; S.oz = L.oz;
        S.dx = L.dx; S.dy = L.dy; S.dz = L.dz;
        S.t_a = 0.0f; S.lo = L.lo; S.hi = L.hi;
        S.k0 = (int)L.k0; S.k1 = (int)L.k1;
        return true;
      });
    __syncthreads();
    if (B.n_tiles == 0) break;
    B.encode<NL, TabT>(F, table, pc, use_occ, my,
                       [&](int i, float& px, float& py, float& pz) { return B.place(i, delta, px, py, pz); });
    for (int k = B.next_ray(); k >= 0; k = B.next_ray()) {
      const int t0 = B.tile0[k], nt = (B.k1[k] - B.k0[k] + 15) / 16;
      const float lo = B.lo[k], hi = B.hi[k];
      float tau = 0.0f;
      d4v ahead = lv_load(my, t0, lane);
      for (int t = 0; t < nt; ++t) {
        const uint32_t m = B.mask[t0 + t];
        const bool valid = (m >> j) & 1u;
        float fe[LY::NF];
        lv_features(ahead, valid, fe);
        ahead = lv_load(my, t0 + t + 1, lane);
        if (m == 0) continue;
        const int s = B.k0[k] + 16 * t + j;
        const f4v raw = density_raw<NL, 4, 1, false>(sW, fe, lane);
        // lanes 0..15 hold raw output 0 of their sample
        if (valid && lane < 16)
          tau += softplusf(raw[0] + F.density_offset) * (fminf((float)(s + 1) * delta, hi) - fmaxf((float)s * delta, lo));
      }
      tau = sum16(tau);
      if (lane == 0) add_light(q, next, B.r[k], tau, radiance);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) pc.leave();
}

constexpr int kLightGrab = 16;   // slots a wave takes at a time

template <int NL, typename TabT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_light_march(
    RayQueue q, RayQueue next, const int* __restrict__ count, int* __restrict__ work, FieldView F,
    const TabT* __restrict__ table, float delta, int use_occ, int last, int lv,
    float* __restrict__ radiance) {
  using LY = FragLayout<NL, 4, 1, false>;   // the density layers come first and are the same for every layout
  __shared__ __align__(16) uint32_t sW[LY::C1];
  stage_density<NL>(F.mlp, sW);
  __syncthreads();
  const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15;
  const int cnt = *count, waves = gridDim.x * 4;
  const bool rest = lv && cnt >= kLvMinRays;   // k_light_lv has marched all but the long segments
  int base = -kLightGrab * waves + kLightGrab * (int)(blockIdx.x * 4 + (threadIdx.x >> 6));
  while (true) {
    if (work) {
      if (lane == 0) base = atomicAdd(work, kLightGrab);
      base = __shfl(base, 0, 64);
    } else {
      base += kLightGrab * waves;
    }
    if (base >= cnt) break;
    const int mine = base + lane;
    bool pending = lane < kLightGrab && mine < cnt && q.hit_p[min(mine, cnt - 1)] == kLightPending;
    if (rest && pending) {
      LightSeg S;
      pending = !light_seg(q, mine, F, delta, S) || light_long(S);
    }
    uint64_t todo = __ballot(pending);
    while (todo) {
      const int i = base + __builtin_ctzll(todo);
      todo &= todo - 1;
      LightSeg S;
      float tau = 0.0f;
      if (light_seg(q, i, F, delta, S)) {
        for (int64_t kb = S.k0; kb < S.k1; kb += 16) {
          const int64_t k = kb + j;
          const float a = fmaxf((float)k * delta, S.lo), b = fminf((float)(k + 1) * delta, S.hi);
          bool valid = k < S.k1 && b > a;
          const float tm = 0.5f * (a + b);
          const float px = S.ox + tm * S.dx, py = S.oy + tm * S.dy, pz = S.oz + tm * S.dz;
          if (valid && use_occ) valid = occ_lookup(F, px, py, pz);
          if (__ballot(valid) == 0ull) continue;
          float fe[LY::NF];
          encode_group<NL, TabT>(F, table, px, py, pz, g, fe);
          const f4v raw = density_raw<NL, 4, 1, false>(sW, fe, lane);
          // lanes 0..15 hold raw output 0 of their sample
          if (valid && g == 0) tau += softplusf(raw[0] + F.density_offset) * (b - a);
        }
      }
      tau = sum16(tau);
      if (lane == 0) {
        tau += q.lr[i];
        if (last) add_light(q, next, i, tau, radiance);
        else q.lr[i] = tau;
      }
    }
  }
}

template <int NL, typename TabT>
mr_status launch_light(const mr_field* f, RayQueue q, RayQueue next, const int* count, int* work, float delta, bool occ,
                       bool last, float* radiance, int64_t n, const LvScratch* lv, hipStream_t st) {
  const int use_occ = occ && f->view.occ ? 1 : 0;
  const TabT* tab = reinterpret_cast<const TabT*>(f->table_dev);
  if constexpr (NL == 16)
    if (lv) {
      hipLaunchKernelGGL(k_light_lv<TabT>, dim3(lv_blocks()), dim3(kLvThreads), 0, st, q, next, count, work, f->view, tab,
                         delta, use_occ, radiance, lv->feat, lv->pace);
      MR_HIP(hipGetLastError());
    }
  // its queue head is its own: the counter after k_light_lv's
  if (work && lv) work += kMaxBounces + 2;
  auto* k = k_light_march<NL, TabT>;
  const int blocks = persistent_blocks(reinterpret_cast<const void*>(k), 256, 0, (n + 63) / 64);
  hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, st, q, next, count, work, f->view, tab,
                     delta, use_occ, last ? 1 : 0, lv ? 1 : 0, radiance);
  MR_HIP(hipGetLastError());
  return MR_OK;
}

}  // namespace

namespace mr {

mr_status dispatch_light_march(const mr_field* f, RayQueue q, RayQueue next, const int* count, int* work, float delta,
                               bool use_occupancy, bool last, float* radiance, int64_t n, const LvScratch* lv,
                               hipStream_t st) {
  const bool h = f->view.table_dtype == MR_F16;
  if (f->view.n_levels == 16)
    return h ? launch_light<16, __half>(f, q, next, count, work, delta, use_occupancy, last, radiance, n, lv, st)
             : launch_light<16, float>(f, q, next, count, work, delta, use_occupancy, last, radiance, n, lv, st);
  return h ? launch_light<8, __half>(f, q, next, count, work, delta, use_occupancy, last, radiance, n, nullptr, st)
           : launch_light<8, float>(f, q, next, count, work, delta, use_occupancy, last, radiance, n, nullptr, st);
}

}  // namespace mr
