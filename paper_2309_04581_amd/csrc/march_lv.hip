// March of incoherent segments (bounce rays) one hash level at a time.
//
// A bounce ray's samples share no line of the finer hashed levels, so the
// per-ray march (march_mfma.hip) fetches about 49 lines per sample, 60 % of
// them from beyond L2, and runs at the rate of random lines there (59 G/s).
// One level of a 2^19-entry FP32 table is 4 MiB, what one die's L2 holds.
// Here a block takes a batch of up to kLvSamples samples, evaluates level 0
// of all of them, then level 1, ..., and keeps the features in a scratch area
// of its own; the blocks of a die go from level to level together, so the
// level's lines are fetched into each L2 once per batch of the whole die and
// the gathers hit.  Then the block's waves run the MLP tiles ray by ray as the
// per-ray march does: the same samples, arithmetic and order, the same bits.
//
// Two blocks share a compute unit and take turns: while one gathers, the
// other runs its MLP tiles.  The turns and the levels are kept by counters
// that only pace the blocks: every wait is bounded, and a block whose wait
// runs out stops waiting.
//
// Encoding alone, 16 samples along each of many random rays: 0.62 ns per
// sample per ray, 0.30 in these batches.  The bounce segments of the 800x800
// mid frame (11.7 M samples) went from 7.4 to 5.4 ms in FP32, from 6.9 to
// 4.7 ms with FP16 table and BF16 MLPs.
#include "mr_march.h"

using namespace mr;

namespace {

constexpr int kLvThreads = 512;
constexpr int kLvPer = kLvSamples / kLvThreads;   // samples per thread
constexpr int kLvTiles = kLvSamples / 16;
constexpr int kLvGrab = 64;                       // rays examined together (one wave)

// Pacing of the blocks of one die and turn (blocks i and i + grid / 2 take
// different turns).  Lines of their own: [die][turn] {levels, encodes done}.
struct LvPace {
  int *levels, *done, *other;
  int per, phase, round, turn;
  bool on;
  __device__ __forceinline__ LvPace(int* base) {
    const int half = gridDim.x / 2, die = blockIdx.x % kXcds;
    turn = (int)blockIdx.x >= half ? 1 : 0;
    per = half / kXcds;
    levels = base + ((die * 2 + turn) * 2) * kLvLine;
    done = levels + kLvLine;
    other = base + ((die * 2 + (turn ^ 1)) * 2 + 1) * kLvLine;
    phase = round = 0;
    on = true;
  }
  __device__ __forceinline__ void wait(const int* c, int target, int polls) {
    for (int i = 0; i < polls; ++i) {
      if (__hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= target) return;
      __builtin_amdgcn_s_sleep(1);
    }
    on = false;
  }
  // one thread each; the callers hold the block's other threads at a barrier
  __device__ __forceinline__ void my_turn() {
    if (on) wait(other, per * (round + turn), 2048);
    ++round;
  }
  __device__ __forceinline__ void next_level() {
    ++phase;
    __hip_atomic_fetch_add(levels, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (on) wait(levels, per * phase, 256);
  }
  __device__ __forceinline__ void skip(int n) {   // a batch without samples
    phase += n;
    __hip_atomic_fetch_add(levels, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void encoded() {
    __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void leave() {   // nobody waits for this block again
    __hip_atomic_fetch_add(levels, 1 << 24, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(done, 1 << 24, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
};

// The blocks meet before every second hashed level (meeting before each one
// costs more than it saves: 5.55 against 5.40 ms of bounce marches per mid
// frame); the dense levels together are small.
__device__ __forceinline__ bool paced(const FieldView& F, int l) {
  return !((F.dense_mask >> l) & 1u) && ((l - __popc(F.dense_mask)) & 1) == 0;
}

struct LvRays {   // the batch's rays
  float ox[kLvTiles], oy[kLvTiles], oz[kLvTiles], dx[kLvTiles], dy[kLvTiles], dz[kLvTiles];
  float t_a[kLvTiles], lo[kLvTiles], hi[kLvTiles];
  int r[kLvTiles], k0[kLvTiles], k1[kLvTiles], tile0[kLvTiles];
};

template <int NL, int SH, int CL, typename TabT, bool BF>
__global__ __launch_bounds__(kLvThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_march_lv(
    RayQueue q, const int* __restrict__ count, int* __restrict__ work, FieldView F, const TabT* __restrict__ table,
    const uint32_t* __restrict__ frags, MarchParams P, double* __restrict__ scratch, int* __restrict__ pace,
    unsigned long long* __restrict__ stats) {
  using LY = FragLayout<NL, SH, CL, BF>;
  __shared__ __align__(16) uint32_t sW[LY::TOTAL];
  __shared__ LvRays R;
  __shared__ int sRayOf[kLvTiles];        // tile -> ray of the batch
  __shared__ uint32_t sMask[kLvTiles];    // the tile's valid samples
  __shared__ uint16_t sList[kLvSamples];  // valid samples of the batch, tile * 16 + column
  __shared__ int sTiles, sRays, sValid, sNext;
  const int cnt = *count;
  if (cnt < kLvMinRays) return;   // k_march_mfma takes a short queue
  for (int i = threadIdx.x; i < LY::TOTAL; i += kLvThreads) sW[i] = frags[i];
  const int lane = threadIdx.x & 63, g = lane >> 4, j = lane & 15, wave = threadIdx.x >> 6;
  const bool use_occ = P.use_occupancy && F.occ;
  const float delta = P.delta;
  double* my = scratch + (int64_t)blockIdx.x * kLvSamples * NL;
  LvPace pc(pace);
  unsigned long long nsamp = 0;
  // rays per queue grab: several grabs per block, so that the blocks end together
  const int grab = max(4, min(kLvGrab, cnt / (4 * (int)gridDim.x)));
  int cur = 0, end = 0;   // wave 0: the rays grabbed and not yet batched
  while (true) {
    // --- the batch: wave 0 takes rays while their tiles fit ---
    if (wave == 0) {
      int tiles = 0, rays = 0;
      while (tiles < kLvTiles) {
        if (cur >= end) {
          int v = 0;
          if (lane == 0) v = atomicAdd(work, grab);
          cur = __shfl(v, 0, 64);
          end = min(cur + grab, cnt);
          if (cur >= cnt) break;
        }
        const int r = cur + lane;
        RaySeg S;
        int nt = 0;
        if (r < end && ray_seg(q, r, F, P, S)) nt = max(0, (S.k1 - S.k0 + 15) / 16);
        int sum = nt;   // inclusive over the lanes
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int u = __shfl_up(sum, off, 64);
          if (lane >= off) sum += u;
        }
        const bool fits = tiles + sum <= kLvTiles && r < end;   // a prefix of the lanes (a ray has at most kLvTiles)
        const uint64_t mf = __ballot(fits), ml = __ballot(fits && nt > 0);
        if (fits && nt > 0) {
          const int k = rays + __popcll(ml & ((1ull << lane) - 1ull)), t0 = tiles + sum - nt;
          R.ox[k] = S.ox; R.oy[k] = S.oy; R.oz[k] = S.oz;
          R.dx[k] = S.dx; R.dy[k] = S.dy; R.dz[k] = S.dz;
          R.t_a[k] = S.t_a; R.lo[k] = S.lo; R.hi[k] = S.hi;
          R.r[k] = r; R.k0[k] = S.k0; R.k1[k] = S.k1; R.tile0[k] = t0;
          for (int t = 0; t < nt; ++t) sRayOf[t0 + t] = k;
        }
        const int nf = __popcll(mf);
        if (nf > 0) tiles += __shfl(sum, nf - 1, 64);
        rays += __popcll(ml);
        cur += nf;
        if (cur < end) break;   // the next ray does not fit: full
      }
      if (lane == 0) {
        sTiles = tiles;
        sRays = rays;
        sValid = 0;
        sNext = 0;
      }
    }
    __syncthreads();
    const int tiles = sTiles, rays = sRays;
    if (tiles == 0) break;
    // --- the batch's valid samples ---
    auto place = [&](int i, float& a, float& b, float& px, float& py, float& pz) {
      const int t = i >> 4, k = sRayOf[t], s = R.k0[k] + 16 * (t - R.tile0[k]) + (i & 15);
      const float ta = R.t_a[k];
      a = fmaxf(ta + (float)s * delta, R.lo[k]);
      b = fminf(ta + (float)(s + 1) * delta, R.hi[k]);
      const float tm = 0.5f * (a + b);
      px = R.ox[k] + tm * R.dx[k];
      py = R.oy[k] + tm * R.dy[k];
      pz = R.oz[k] + tm * R.dz[k];
      return s < R.k1[k] && b > a;
    };
    for (int i0 = wave * 64; i0 < tiles * 16; i0 += kLvThreads) {
      const int i = i0 + lane;
      bool valid = i < tiles * 16;
      float a, b, px, py, pz;
      if (valid) valid = place(i, a, b, px, py, pz);
      if (valid && use_occ) valid = occ_lookup(F, px, py, pz);
      const uint64_t m = __ballot(valid);
      if (j == 0 && i < tiles * 16) sMask[i >> 4] = (uint32_t)(m >> (lane & 48)) & 0xFFFFu;
      int base = 0;
      if (lane == 0 && m) base = atomicAdd(&sValid, __popcll(m));
      base = __shfl(base, 0, 64);
      if (valid) sList[base + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)i;
    }
    if (threadIdx.x == 0) pc.my_turn();
    __syncthreads();
    const int nv = sValid;
    // --- the features, level by level ---
    if (nv > 0) {
      float xh[kLvPer], yh[kLvPer], zh[kLvPer];
      int dst[kLvPer];
#pragma unroll
      for (int it = 0; it < kLvPer; ++it) {
        const int e = it * kLvThreads + threadIdx.x, i = sList[min(e, nv - 1)];
        float a, b, px, py, pz;
        place(i, a, b, px, py, pz);
        to_unit(F, px, py, pz, xh[it], yh[it], zh[it]);
        dst[it] = e < nv ? (i >> 4) * NL * 16 + (i & 15) : -1;
      }
#pragma unroll 1
      for (int l = 0; l < NL; ++l) {
        if (paced(F, l)) {
          __syncthreads();
          if (threadIdx.x == 0) pc.next_level();
          __syncthreads();
        }
#pragma unroll
        for (int it = 0; it < kLvPer; ++it)
          if (it * kLvThreads + wave * 64 < nv) {
            const float2 f = encode_level_pair<TabT>(F, table, l, lane, xh[it], yh[it], zh[it]);
            if (dst[it] >= 0) __builtin_nontemporal_store(__builtin_bit_cast(double, f), my + dst[it] + l * 16);
          }
      }
    } else if (threadIdx.x == 0) {
      int waits = 0;
      for (int l = 0; l < NL; ++l) waits += paced(F, l);
      pc.skip(waits);
    }
    __syncthreads();
    if (threadIdx.x == 0) pc.encoded();
    // --- MLP tiles and compositing, a ray per wave ---
    while (true) {
      int k = 0;
      if (lane == 0) k = atomicAdd(&sNext, 1);
      k = __shfl(k, 0, 64);
      if (k >= rays) break;
      const int t0 = R.tile0[k], nt = (R.k1[k] - R.k0[k] + 15) / 16;
      const float t_a = R.t_a[k], lo = R.lo[k], hi = R.hi[k];
      // the ray's throughput (lanes 0..2) and radiance (3..5), needed at its end
      float* state = q.tr + (int64_t)min(lane, 5) * (q.tg - q.tr) + R.r[k];
      const float old = *state;
      float u[4][4];
      sh_rows<NL, SH, CL, BF>(sW, R.dx[k], R.dy[k], R.dz[k], lane, u);
      float Tseg = 1.0f, acc0 = 0.0f, acc1 = 0.0f, acc2 = 0.0f;
      double nx[NL / 4];
#pragma unroll
      for (int ll = 0; ll < NL / 4; ++ll) nx[ll] = __builtin_nontemporal_load(my + ((int64_t)t0 * NL + 4 * ll + g) * 16 + j);
      for (int t = 0; t < nt; ++t) {
        const uint32_t m = sMask[t0 + t];
        double cu[NL / 4];
#pragma unroll
        for (int ll = 0; ll < NL / 4; ++ll) {
          cu[ll] = nx[ll];
          nx[ll] = __builtin_nontemporal_load(my + ((int64_t)min(t0 + t + 1, kLvTiles - 1) * NL + 4 * ll + g) * 16 + j);
        }
        if (m == 0) continue;
        const int s = R.k0[k] + 16 * t + j;
        const bool valid = (m >> j) & 1u;
        const float D = fminf(t_a + (float)(s + 1) * delta, hi) - fmaxf(t_a + (float)s * delta, lo);
        float fe[LY::NF];
#pragma unroll
        for (int ll = 0; ll < NL / 4; ++ll) {
          const float2 f = __builtin_bit_cast(float2, cu[ll]);
          fe[2 * ll] = valid ? f.x : 0.0f;
          fe[2 * ll + 1] = valid ? f.y : 0.0f;
        }
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

template <int SH, int CL, typename TabT, bool BF>
mr_status launch_lv(const mr_field* f, RayQueue q, const int* count, int* work, const MarchParams& P, const LvScratch& lv,
                    unsigned long long* stats, hipStream_t st) {
  hipLaunchKernelGGL((k_march_lv<16, SH, CL, TabT, BF>), dim3(lv_blocks()), dim3(kLvThreads), 0, st, q, count, work,
                     f->view, reinterpret_cast<const TabT*>(f->table_dev), BF ? f->frag_bf16_dev : f->frag_f32_dev, P,
                     lv.feat, lv.pace, stats);
  MR_HIP(hipGetLastError());
  return MR_OK;
}

}  // namespace

namespace mr {

int lv_blocks() { return 2 * ((device_cus() + kXcds - 1) / kXcds) * kXcds; }

size_t lv_bytes() { return kLvPaceArea + (size_t)lv_blocks() * kLvSamples * 16 * sizeof(double); }

bool lv_field(const mr_field* f) {
  const auto& v = f->view;
  const size_t level = ((size_t)v.table_mask + 1) * 2 * (v.table_dtype == MR_F16 ? 2 : 4);
  return v.n_levels == 16 && level <= (8u << 20) && level * 16 > (4u << 20);
}

mr_status dispatch_march_lv(const mr_field* f, RayQueue q, const int* count, int* work, const MarchParams& P,
                            const LvScratch& lv, unsigned long long* stats, hipStream_t st) {
  const auto& v = f->view;
  const bool h = v.table_dtype == MR_F16, bf = v.mlp_dtype == MR_BF16;
#define L(SH, CL)                                                                                    \
  if (v.sh == SH && v.c_layers == CL) {                                                              \
    if (bf) return h ? launch_lv<SH, CL, __half, true>(f, q, count, work, P, lv, stats, st)     \
                     : launch_lv<SH, CL, float, true>(f, q, count, work, P, lv, stats, st);     \
    return h ? launch_lv<SH, CL, __half, false>(f, q, count, work, P, lv, stats, st)            \
             : launch_lv<SH, CL, float, false>(f, q, count, work, P, lv, stats, st);            \
  }
  L(16, 2)
  L(4, 1)
#undef L
  return fail(MR_ERR_UNSUPPORTED, "field shape not instantiated");
}

}  // namespace mr
