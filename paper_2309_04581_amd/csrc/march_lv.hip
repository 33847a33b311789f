// Kernels that evaluate incoherent samples one hash level at a time (mr_levels.h):
// the march of bounce rays, and point queries.
#include <mutex>

#include "mr_field_kernels.h"
#include "mr_levels.h"

using namespace mr;

namespace {

// March of bounce rays: the same samples, arithmetic and order as the per-ray
// march (march_mfma.hip), the same bits.  The bounce segments of the 800x800
// mid frame (11.7 M samples) went from 7.65 to 5.56 ms in FP32, from 6.9 to 4.7
// ms with FP16 table and BF16 MLPs (default launch shape; with the shape that the
// search finds for that frame, FP32 6.9 and 5.2).
template <int NL, int SH, int CL, typename TabT, bool BF>
__global__ __launch_bounds__(kLvThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_march_lv(
    RayQueue q, const int* __restrict__ count, int* __restrict__ work, FieldView F, const TabT* __restrict__ table,
    const uint32_t* __restrict__ frags, MarchParams P, double* __restrict__ scratch, int* __restrict__ pace,
    unsigned long long* __restrict__ stats) {
  using LY = FragLayout<NL, SH, CL, BF>;
  __shared__ __align__(16) uint32_t sW[LY::TOTAL];
  __shared__ LvBatch B;
  const int cnt = *count;
  if (cnt < kLvMinRays) return;   // k_march_mfma takes a short queue
  for (int i = threadIdx.x; i < LY::TOTAL; i += kLvThreads) sW[i] = frags[i];
  const int lane = threadIdx.x & 63, j = lane & 15;
  const float delta = P.delta;
  double* my = scratch + (int64_t)blockIdx.x * kLvSamples * NL;
  LvPace pc(pace);
  unsigned long long nsamp = 0;
  const int grab = lv_grab(cnt);
  int cur = 0, end = 0;
  while (true) {
    if (threadIdx.x < 64)
      B.take(work, cnt, grab, cur, end, [&](int r, RaySeg& S) { return ray_seg(q, r, F, P, S); });
    __syncthreads();
    if (B.n_tiles == 0) break;
    B.encode<NL, TabT>(F, table, pc, P.use_occupancy && F.occ, my,
                       [&](int i, float& px, float& py, float& pz) { return B.place(i, delta, px, py, pz); });
    // MLP tiles and compositing, a ray per wave
    for (int k = B.next_ray(); k >= 0; k = B.next_ray()) {
      const int t0 = B.tile0[k], nt = (B.k1[k] - B.k0[k] + 15) / 16;
      const float t_a = B.t_a[k], lo = B.lo[k], hi = B.hi[k];
      // the ray's throughput (lanes 0..2) and radiance (3..5), needed at its end
      float* state = q.tr + (int64_t)min(lane, 5) * (q.tg - q.tr) + B.r[k];
      const float old = *state;
      float u[4][4];
      sh_rows<NL, SH, CL, BF>(sW, B.dx[k], B.dy[k], B.dz[k], lane, u);
      float Tseg = 1.0f, acc0 = 0.0f, acc1 = 0.0f, acc2 = 0.0f;
      d4v ahead = lv_load(my, t0, lane);
      for (int t = 0; t < nt; ++t) {
        const uint32_t m = B.mask[t0 + t];
        const bool valid = (m >> j) & 1u;
        float fe[LY::NF];
        lv_features(ahead, valid, fe);
        ahead = lv_load(my, t0 + t + 1, lane);
        if (m == 0) continue;
        const int s = B.k0[k] + 16 * t + j;
        const float D = fminf(t_a + (float)(s + 1) * delta, hi) - fmaxf(t_a + (float)s * delta, lo);
        float sigma, rgb[3];
        f4v raw;
        mlp_tile<NL, SH, CL, BF>(sW, fe, u, F.density_offset, lane, sigma, rgb, raw);
        const float alpha = valid ? -expm1f(-sigma * D) : 0.0f;
        const float incl = scan16_mul(1.0f - alpha, j);
        float excl = __shfl_up(incl, 1, 16);
        if (j == 0) excl = 1.0f;
        const float w = Tseg * excl * alpha;
        acc0 += w * rgb[0];
        acc1 += w * rgb[1];
        acc2 += w * rgb[2];
        Tseg *= __shfl(incl, 15, 16);
        if (lane == 0) nsamp += __popc(m);
      }
      acc0 = sum16(acc0);
      acc1 = sum16(acc1);
      acc2 = sum16(acc2);
      const float tr = __shfl(old, lane >= 3 ? lane - 3 : lane, 64);
      const float l = lane == 3 ? acc0 : (lane == 4 ? acc1 : acc2);
      if (lane < 6) *state = lane < 3 ? old * Tseg : old + tr * l;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) pc.leave();
  if (stats && lane == 0 && nsamp) atomicAdd(stats + 0, nsamp);
}

// Point queries (3 M random points of a 16-level field, all outputs but features
// and raw: 2.67 ms in k_query_mfma, 1.29 here; FP16 and BF16 2.13 and 1.04).  A
// block takes `batch` consecutive points at a time (a multiple of 64, at most
// kLvSamples, chosen so that the blocks have equal numbers of batches).
template <int NL, int SH, int CL, typename TabT, bool BF>
__global__ __launch_bounds__(kLvThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_query_lv(
    FieldView F, const TabT* __restrict__ table, const uint32_t* __restrict__ frags, int64_t n, int batch,
    const float* __restrict__ x, const float* __restrict__ dirs, float* __restrict__ sigma_out,
    float* __restrict__ rgb_out, float* __restrict__ feat_out, float* __restrict__ raw_out,
    double* __restrict__ scratch, int* __restrict__ pace) {
  using LY = FragLayout<NL, SH, CL, BF>;
  __shared__ __align__(16) uint32_t sW[LY::TOTAL];
  for (int i = threadIdx.x; i < LY::TOTAL; i += kLvThreads) sW[i] = frags[i];
  const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15, wave = threadIdx.x >> 6;
  double* my = scratch + (int64_t)blockIdx.x * kLvSamples * NL;
  LvPace pc(pace);
  for (int64_t base = (int64_t)blockIdx.x * batch; base < n; base += (int64_t)gridDim.x * batch) {
    const int nv = (int)min((int64_t)batch, n - base);
    float xh[kLvPer], yh[kLvPer], zh[kLvPer];
    int dst[kLvPer];
#pragma unroll
    for (int it = 0; it < kLvPer; ++it) {
      const int e = it * kLvThreads + threadIdx.x;
      const int64_t p = base + min(e, nv - 1);
      float px = x[3 * p], py = x[3 * p + 1], pz = x[3 * p + 2], dx = 0.0f, dy = 0.0f, dz = 0.0f;
      to_field_frame(F, px, py, pz, dx, dy, dz);
      to_unit(F, px, py, pz, xh[it], yh[it], zh[it]);
      dst[it] = e < nv ? (e >> 4) * NL * 16 + (e & 15) : -1;
    }
    if (threadIdx.x == 0) pc.my_turn();
    __syncthreads();
    lv_levels<NL, TabT>(F, table, pc, nv, xh, yh, zh, dst, my);
    __syncthreads();
    if (threadIdx.x == 0) pc.encoded();
    d4v ahead = lv_load(my, wave, lane);
    for (int t = wave; t * 16 < nv; t += kLvThreads / 64) {
      const bool valid = t * 16 + j < nv;
      float fe[LY::NF];
      lv_features(ahead, valid, fe);
      ahead = lv_load(my, t + kLvThreads / 64, lane);
      const int64_t p = base + t * 16 + j, pc2 = valid ? p : n - 1;
      float px = 0.0f, py = 0.0f, pz = 0.0f, dx = 0.0f, dy = 0.0f, dz = 1.0f;
      if (dirs) { dx = dirs[3 * pc2]; dy = dirs[3 * pc2 + 1]; dz = dirs[3 * pc2 + 2]; }
      to_field_frame(F, px, py, pz, dx, dy, dz);
      float u[4][4];
      sh_rows<NL, SH, CL, BF>(sW, dx, dy, dz, lane, u);
      float sigma, rgb[3];
      f4v raw;
      mlp_tile<NL, SH, CL, BF>(sW, fe, u, F.density_offset, lane, sigma, rgb, raw);
      if (!valid) continue;
      if (g == 0) {
        sigma_out[p] = sigma;
        if (rgb_out) {
          rgb_out[3 * p] = rgb[0];
          rgb_out[3 * p + 1] = rgb[1];
          rgb_out[3 * p + 2] = rgb[2];
        }
      }
      if (feat_out)
#pragma unroll
        for (int k = 0; k < LY::NF; ++k) feat_out[p * 2 * NL + frag_k(0, LY::NF, 0, g, k)] = fe[k];
      if (raw_out)
#pragma unroll
        for (int v = 0; v < 4; ++v) raw_out[p * 16 + 4 * g + v] = raw[v];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) pc.leave();
}

__global__ void k_zero_pace(int* __restrict__ p) {
  for (int i = threadIdx.x; i <= kLvPaceInts; i += blockDim.x) p[i] = 0;
}

template <int SH, int CL, typename TabT, bool BF>
mr_status launch_lv(const mr_field* f, RayQueue q, const int* count, int* work, const MarchParams& P,
                    const LvScratch& lv, unsigned long long* stats, hipStream_t st) {
  hipLaunchKernelGGL((k_march_lv<16, SH, CL, TabT, BF>), dim3(lv_blocks()), dim3(kLvThreads), 0, st, q, count, work,
                     f->view, reinterpret_cast<const TabT*>(f->table_dev), BF ? f->frag_bf16_dev : f->frag_f32_dev, P,
                     lv.feat, lv.pace, stats);
  MR_HIP(hipGetLastError());
  return MR_OK;
}

template <int SH, int CL, typename TabT, bool BF>
mr_status launch_query_lv(const mr_field* f, int64_t n, const float* x, const float* dirs, float* sigma, float* rgb,
                          float* feat, float* raw, const LvScratch& lv, hipStream_t st) {
  const int64_t grid = lv_blocks(), rounds = (n + grid * kLvSamples - 1) / (grid * kLvSamples);
  const int batch = (int)((n + grid * rounds * 64 - 1) / (grid * rounds * 64)) * 64;
  hipLaunchKernelGGL((k_query_lv<16, SH, CL, TabT, BF>), dim3((unsigned)grid), dim3(kLvThreads), 0, st, f->view,
                     reinterpret_cast<const TabT*>(f->table_dev), BF ? f->frag_bf16_dev : f->frag_f32_dev, n, batch, x,
                     dirs, sigma, rgb, feat, raw, lv.feat, lv.pace);
  MR_HIP(hipGetLastError());
  return MR_OK;
}

// Scratch of calls without a workspace: stream-ordered blocks of a memory pool
// per device, so calls on several streams and threads each have their own and
// a returned block is taken again in stream order.  The pool keeps at most one
// block beyond the calls (its release threshold) and is trimmed when the last
// field is destroyed.
constexpr int kMaxDevices = 64;
std::mutex g_pool_mu;
hipMemPool_t g_pool[kMaxDevices] = {};
int g_fields = 0;

}  // namespace

namespace mr {

int lv_blocks() { return 2 * ((device_cus() + kXcds - 1) / kXcds) * kXcds; }

size_t lv_bytes() {
  return kLvPaceArea + (size_t)lv_blocks() * kLvSamples * (16 * sizeof(double) + sizeof(float));
}

LvScratch lv_scratch(void* area, int launch) {
  char* c = reinterpret_cast<char*>(area);
  LvScratch lv;
  lv.pace = reinterpret_cast<int*>(c) + (size_t)launch * kLvPaceInts;
  lv.feat = reinterpret_cast<double*>(c + kLvPaceArea);
  lv.edge = reinterpret_cast<float*>(lv.feat + (size_t)lv_blocks() * kLvSamples * 16);
  return lv;
}

bool lv_field(const mr_field* f) {
  const auto& v = f->view;
  const size_t level = ((size_t)v.table_mask + 1) * 2 * (v.table_dtype == MR_F16 ? 2 : 4);
  return v.n_levels == 16 && level <= (8u << 20) && level * 16 > (4u << 20);
}

bool lv_lease(hipStream_t st, LvScratch* lv) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  int dev = 0;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone ||
      hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return false;
  }
  hipMemPool_t pool = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_pool_mu);
    if (!g_pool[dev]) {
      hipMemPoolProps props = {};
      props.allocType = hipMemAllocationTypePinned;
      props.location.type = hipMemLocationTypeDevice;
      props.location.id = dev;
      uint64_t keep = lv_bytes();
      if (hipMemPoolCreate(&g_pool[dev], &props) != hipSuccess ||
          hipMemPoolSetAttribute(g_pool[dev], hipMemPoolAttrReleaseThreshold, &keep) != hipSuccess) {
        (void)hipGetLastError();
        return false;
      }
    }
    pool = g_pool[dev];
  }
  void* p = nullptr;
  if (hipMallocFromPoolAsync(&p, lv_bytes(), pool, st) != hipSuccess || !p) {
    (void)hipGetLastError();
    return false;
  }
  *lv = lv_scratch(p, 0);
  hipLaunchKernelGGL(k_zero_pace, dim3(1), dim3(kLvPaceInts), 0, st, lv->pace);
  return true;
}

void lv_return(hipStream_t st, const LvScratch& lv) { (void)hipFreeAsync(lv.pace, st); }

void lv_fields(int change) {
  std::lock_guard<std::mutex> lk(g_pool_mu);
  g_fields += change;
  if (g_fields > 0) return;
  for (hipMemPool_t p : g_pool)
    if (p) (void)hipMemPoolTrimTo(p, 0);
}

#define LV_DISPATCH(fn, ...)                                       \
  do {                                                             \
    const auto& v = f->view;                                       \
    const bool h = v.table_dtype == MR_F16, bf = v.mlp_dtype == MR_BF16; \
    if (v.sh == 16 && v.c_layers == 2) {                           \
      if (bf) return h ? fn<16, 2, __half, true>(__VA_ARGS__) : fn<16, 2, float, true>(__VA_ARGS__);   \
      return h ? fn<16, 2, __half, false>(__VA_ARGS__) : fn<16, 2, float, false>(__VA_ARGS__);         \
    }                                                              \
    if (v.sh == 4 && v.c_layers == 1) {                            \
      if (bf) return h ? fn<4, 1, __half, true>(__VA_ARGS__) : fn<4, 1, float, true>(__VA_ARGS__);     \
      return h ? fn<4, 1, __half, false>(__VA_ARGS__) : fn<4, 1, float, false>(__VA_ARGS__);           \
    }                                                              \
    return fail(MR_ERR_UNSUPPORTED, "field shape not instantiated"); \
  } while (0)

mr_status dispatch_march_lv(const mr_field* f, RayQueue q, const int* count, int* work, const MarchParams& P,
                            const LvScratch& lv, unsigned long long* stats, hipStream_t st) {
  LV_DISPATCH(launch_lv, f, q, count, work, P, lv, stats, st);
}

mr_status query_lv(const mr_field* f, int64_t n, const float* x, const float* dirs, float* sigma, float* rgb,
                   float* feat, float* raw, const LvScratch& lv, hipStream_t st) {
  LV_DISPATCH(launch_query_lv, f, n, x, dirs, sigma, rgb, feat, raw, lv, st);
}

}  // namespace mr
