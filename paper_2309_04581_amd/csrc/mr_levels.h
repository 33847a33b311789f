// Samples evaluated one hash level at a time, in batches of up to kLvSamples per
// block: what the level-by-level kernels share (march, light samples, proposal
// targets, point queries).
//
// Samples far apart share no line of the finer hashed levels, so a kernel that
// takes all levels of a sample together fetches about 47 lines per sample,
// most of them from beyond L2, and runs at the rate of random lines there (59
// G/s).  One level of a 2^19-entry FP32 table is 4 MiB, what one die's L2
// holds.  So a block takes a batch of samples, evaluates level 0 of all of
// them, then level 1, ..., and keeps the features in a scratch area of its own;
// the blocks of a die go from level to level together, each level's lines are
// fetched into each L2 once per batch of the whole die, and the gathers hit.
// Then the block's waves run the MLP tiles.
//
// Two blocks share a compute unit and take turns: while one gathers, the
// other runs its MLP tiles.  The turns and the levels are kept by counters
// that only pace the blocks: every wait is bounded, and a block whose wait
// runs out stops waiting.
//
// Encoding alone, random points: 0.86 ns per sample all levels together, 0.36
// so; 16 samples along each of many random rays: 0.62 and 0.30.
#pragma once
#include "mr_march.h"

namespace mr {

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

// Level l of the block's samples nv > 0: thread t holds samples t, t + kLvThreads,
// ... (unit-cube points xh yh zh) and stores (feature 0, feature 1) at
// out[dst + 16 l] where dst >= 0; threads past the last sample repeat one.
template <int NL, typename TabT>
__device__ __forceinline__ void lv_levels(const FieldView& F, const TabT* __restrict__ table, LvPace& pc, int nv,
                                          const float (&xh)[kLvPer], const float (&yh)[kLvPer],
                                          const float (&zh)[kLvPer], const int (&dst)[kLvPer],
                                          double* __restrict__ out) {
  const int lane = threadIdx.x & 63, wave0 = threadIdx.x & ~63;
#pragma unroll 1
  for (int l = 0; l < NL; ++l) {
    if (paced(F, l)) {
      __syncthreads();
      if (threadIdx.x == 0) pc.next_level();
      __syncthreads();
    }
#pragma unroll
    for (int it = 0; it < kLvPer; ++it)
      if (it * kLvThreads + wave0 < nv) {
        const float2 f = encode_level_pair<TabT>(F, table, l, lane, xh[it], yh[it], zh[it]);
        if (dst[it] >= 0) __builtin_nontemporal_store(__builtin_bit_cast(double, f), out + dst[it] + l * 16);
      }
  }
}

// Features of one tile as the MLP tiles take them: lane (g, j) holds levels g,
// g + 4, ... of sample j.
typedef double d4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ d4v lv_load(const double* __restrict__ feat, int tile, int lane) {
  const double* p = feat + ((int64_t)min(tile, kLvTiles - 1) * 16 + (lane >> 4)) * 16 + (lane & 15);
  return d4v{__builtin_nontemporal_load(p), __builtin_nontemporal_load(p + 64), __builtin_nontemporal_load(p + 128),
             __builtin_nontemporal_load(p + 192)};
}
// A tile's features, zeros for a sample that was not evaluated.
__device__ __forceinline__ void lv_features(const d4v& f, bool valid, float (&fe)[8]) {
  asm volatile("" ::: "memory");   // the MLP's weights are read from LDS in each tile, not held (they would spill)
  const double v[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
  for (int ll = 0; ll < 4; ++ll) {
    const float2 u = __builtin_bit_cast(float2, v[ll]);
    fe[2 * ll] = valid ? u.x : 0.0f;
    fe[2 * ll + 1] = valid ? u.y : 0.0f;
  }
}

// A batch of rays: their segments and tiles of 16 consecutive samples.
struct LvBatch {
  float ox[kLvTiles], oy[kLvTiles], oz[kLvTiles], dx[kLvTiles], dy[kLvTiles], dz[kLvTiles];
  float t_a[kLvTiles], lo[kLvTiles], hi[kLvTiles];
  int r[kLvTiles], k0[kLvTiles], k1[kLvTiles], tile0[kLvTiles];
  int ray_of[kLvTiles];          // tile -> ray of the batch
  uint32_t mask[kLvTiles];       // the tile's valid samples
  uint16_t list[kLvSamples];     // valid samples, tile * 16 + column
  int n_tiles, n_rays, n_valid, next;

  // Wave 0: takes rays from the queue while their tiles fit.  cur, end: the
  // rays grabbed and not yet batched, kept between batches.  seg(r, S) gives
  // ray r's segment, false if it has none; a ray has at most kLvTiles tiles.
  template <typename Seg>
  __device__ __forceinline__ void take(int* __restrict__ work, int cnt, int grab, int& cur, int& end, Seg seg) {
    const int lane = threadIdx.x & 63;
    int tiles = 0, rays = 0;
    while (tiles < kLvTiles) {
      if (cur >= end) {
        int v = 0;
        if (lane == 0) v = atomicAdd(work, grab);
        cur = __shfl(v, 0, 64);
        end = min(cur + grab, cnt);
        if (cur >= cnt) break;
      }
      const int i = cur + lane;
      RaySeg S;
      int nt = 0;
      if (i < end && seg(i, S)) nt = max(0, (S.k1 - S.k0 + 15) / 16);
      int sum = nt;   // inclusive over the lanes
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(sum, off, 64);
        if (lane >= off) sum += u;
      }
      const bool fits = tiles + sum <= kLvTiles && i < end;   // a prefix of the lanes
      const uint64_t mf = __ballot(fits), ml = __ballot(fits && nt > 0);
      if (fits && nt > 0) {
        const int k = rays + __popcll(ml & ((1ull << lane) - 1ull)), t0 = tiles + sum - nt;
        ox[k] = S.ox; oy[k] = S.oy; oz[k] = S.oz;
        dx[k] = S.dx; dy[k] = S.dy; dz[k] = S.dz;
        t_a[k] = S.t_a; lo[k] = S.lo; hi[k] = S.hi;
        r[k] = i; k0[k] = S.k0; k1[k] = S.k1; tile0[k] = t0;
        for (int t = 0; t < nt; ++t) ray_of[t0 + t] = k;
      }
      const int nf = __popcll(mf);
      if (nf > 0) tiles += __shfl(sum, nf - 1, 64);
      rays += __popcll(ml);
      cur += nf;
      if (cur < end) break;   // the next ray does not fit: full
    }
    if (lane == 0) {
      n_tiles = tiles;
      n_rays = rays;
      n_valid = 0;
      next = 0;
    }
  }

  // Point of the batch's ray k in the middle of [a, b].
  __device__ __forceinline__ void middle(int k, float a, float b, float& px, float& py, float& pz) const {
    const float tm = 0.5f * (a + b);
    px = ox[k] + tm * dx[k];
    py = oy[k] + tm * dy[k];
    pz = oz[k] + tm * dz[k];
  }
  // Sample i (tile * 16 + column) on the uniform grid of spacing delta; false
  // if the ray has no such sample.
  __device__ __forceinline__ bool place(int i, float delta, float& px, float& py, float& pz) const {
    const int t = i >> 4, k = ray_of[t], s = k0[k] + 16 * (t - tile0[k]) + (i & 15);
    const float ta = t_a[k];
    const float a = fmaxf(ta + (float)s * delta, lo[k]), b = fminf(ta + (float)(s + 1) * delta, hi[k]);
    middle(k, a, b, px, py, pz);
    return s < k1[k] && b > a;
  }

  // The whole block: the batch's valid samples and their features.  at(i, px,
  // py, pz) gives sample i's point, false if there is none.
  template <int NL, typename TabT, typename At>
  __device__ __forceinline__ void encode(const FieldView& F, const TabT* __restrict__ table, LvPace& pc, bool use_occ,
                                         double* __restrict__ out, At at) {
    const int lane = threadIdx.x & 63, j = lane & 15, samples = n_tiles * 16;
    for (int i0 = threadIdx.x & ~63; i0 < samples; i0 += kLvThreads) {
      const int i = i0 + lane;
      float px, py, pz;
      bool valid = i < samples && at(i, px, py, pz);
      if (valid && use_occ) valid = occ_lookup(F, px, py, pz);
      const uint64_t m = __ballot(valid);
      if (j == 0 && i < samples) mask[i >> 4] = (uint32_t)(m >> (lane & 48)) & 0xFFFFu;
      int base = 0;
      if (lane == 0 && m) base = atomicAdd(&n_valid, __popcll(m));
      base = __shfl(base, 0, 64);
      if (valid) list[base + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)i;
    }
    if (threadIdx.x == 0) pc.my_turn();
    __syncthreads();
    const int nv = n_valid;
    if (nv > 0) {
      float xh[kLvPer], yh[kLvPer], zh[kLvPer];
      int dst[kLvPer];
#pragma unroll
      for (int it = 0; it < kLvPer; ++it) {
        const int e = it * kLvThreads + threadIdx.x, i = list[min(e, nv - 1)];
        float px, py, pz;
        at(i, px, py, pz);
        to_unit(F, px, py, pz, xh[it], yh[it], zh[it]);
        dst[it] = e < nv ? (i >> 4) * NL * 16 + (i & 15) : -1;
      }
      lv_levels<NL, TabT>(F, table, pc, nv, xh, yh, zh, dst, out);
    } else if (threadIdx.x == 0) {
      int waits = 0;
      for (int l = 0; l < NL; ++l) waits += paced(F, l);
      pc.skip(waits);
    }
    __syncthreads();
    if (threadIdx.x == 0) pc.encoded();
  }

  // The next ray of the batch for this wave, or -1.
  __device__ __forceinline__ int next_ray() {
    int k = 0;
    if ((threadIdx.x & 63) == 0) k = atomicAdd(&next, 1);
    k = __shfl(k, 0, 64);
    return k < n_rays ? k : -1;
  }
};

// Rays per queue grab: several grabs per block, so that the blocks end together.
__device__ __forceinline__ int lv_grab(int cnt) { return max(4, min(kLvGrab, cnt / (4 * (int)gridDim.x))); }

}  // namespace mr
