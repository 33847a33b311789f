// Ray queues and launch parameters of the render path.
#pragma once
#include "mr_common.h"
#include "mr_device.h"

namespace mr {

constexpr int kQueueArrays = 16;       // 4-byte arrays per queue slot
constexpr size_t kHeaderBytes = 4096;  // counters at the start of the workspace
constexpr int kMaxBounces = 60;
constexpr int kMaxCamsPerLaunch = 16;
constexpr int kMaxFields = 8;          // fields marched together by mr_render_fields

// Structure-of-arrays ray queue: one slot per live ray.
struct RayQueue {
  float *ox, *oy, *oz, *dx, *dy, *dz;  // origin, unit direction
  float *tr, *tg, *tb;                 // path throughput T
  float *lr, *lg, *lb;                 // accumulated radiance L
  int* rid;                            // caller's ray index
  int* depth;                          // segment index (= scatter count) | max bounces << 16
  float* hit_t;                        // closest hit distance of the current segment
  int* hit_p;                          // hit primitive (leaf order), -1 = miss
};

struct MarchParams {
  float t_near, span, delta;
  int n_samples;
  int use_occupancy;
  int chunk;          // rays per die chunk of the march queue (0 = one global queue)
  int batch;          // queue positions a wave takes per atomic
  // shadow mask per field sample: each light a mesh hides from the sample
  // multiplies its emitted radiance by shadow_mask
  int shadows;
  float shadow_mask;
  int n_lights;
  float light_pos[kMaxLights][3];
  // producer/consumer packet march: polls each wait takes at most, and the
  // device word that counts the waves whose wait gave up (their packets'
  // rays are then left without this segment's medium)
  int wait_polls;
  int* gave_up;
  int lv;             // queues of kLvMinRays or more are marched level by level
  // blocks of the march kernel that are resident at once: what the splits of
  // short queues are chosen by, whatever grid the caller's launch shape gives
  // (a split rounds differently, and results do not depend on that shape)
  int resident;
};

// Shadow mask of the sample of column j (Sec. 3.1 "Shadow rays"): a lane of
// group 0 sends a ray from the sample's world position to every light, and
// each light a mesh hides multiplies the mask by P.shadow_mask; every lane
// returns its column's mask.  stack: that lane's LDS stack, stride 16.
// This form takes the sample's world position; sample_shadow below takes a
// point in the frame of field F.
__device__ __forceinline__ float sample_shadow_world(const BvhView& B, const MarchParams& P, bool valid, float px,
                                                     float py, float pz, int lane, int* stack) {
  float m = 1.0f;
  if (lane < 16 && valid) {
    for (int li = 0; li < P.n_lights; ++li) {
      const float sx = P.light_pos[li][0] - px, sy = P.light_pos[li][1] - py, sz = P.light_pos[li][2] - pz;
      const float dist = sqrtf(sx * sx + sy * sy + sz * sz);
      const RayPre sr = ray_pre(v3(px, py, pz), v3(sx / dist, sy / dist, sz / dist));
      if (bvh_any(B, sr, dist, stack, 16)) m *= P.shadow_mask;
    }
  }
  return __shfl(m, lane & 15, 64);
}

__device__ __forceinline__ float sample_shadow(const FieldView& F, const BvhView& B, const MarchParams& P,
                                               bool valid, float px, float py, float pz, int lane, int* stack) {
  if (lane < 16 && valid) field_to_world(F, px, py, pz);
  return sample_shadow_world(B, P, valid, px, py, pz, lane, stack);
}

struct ShadeParams {
  int n_lights;
  float lights[kMaxLights][6];
  uint32_t seed;
  int rr_after;
  float t_min;
  int sample_emitters;   // light sampling toward the mesh's emitting triangles
};

// Ray queue depth word: bits 0-15 segment index (= scatter count so far),
// bits 16-23 the ray's bounce limit, bit 24 set when the last scatter was
// diffuse.
constexpr int kDepthAfterDiffuse = 1 << 24;

struct RenderOut {
  float* radiance;
  float* throughput;
  int32_t* bounces;
};

constexpr int kXcds = 8;               // accelerator complex dies; workgroups go round-robin over them

// Counters in the workspace header: live rays, closest-hit and shade queue
// heads and kXcds march queue heads per segment, the march waits that gave up,
// and two light-sample queue heads per segment.
constexpr int kHeaderCounters = (5 + kXcds) * (kMaxBounces + 2) + 1;

// Ray work queue of the persistent march kernels.  chunk == 0: one queue for
// the whole device.  chunk > 0: the rays [0, cnt) are cut into chunks of
// `chunk` rays dealt round-robin to the kXcds dies; the waves of workgroups on
// die x = blockIdx.x % kXcds take the rays of die x's chunks in order
// (neighbouring rays then share that die's L2), then help the other dies.
// A wave takes `batch` queue positions per atomic, when it needs them: taking
// them any earlier widens the window of rays in flight, and the march is
// fastest when neighbouring rays are marched at the same time (they share
// cache lines of the hash table).  ctr: kXcds counters, zero at launch.
struct WorkQueue {
  int* ctr;
  int cnt, chunk, batch, die, tries;
  __device__ __forceinline__ WorkQueue(int* c, int n, int ch, int b)
      : ctr(c), cnt(n), chunk(ch), batch(b > 0 ? b : 1), die(ch > 0 ? (int)(blockIdx.x % kXcds) : 0), tries(0) {}
  __device__ __forceinline__ int map(int i) const {
    if (chunk <= 0) return i;
    const int64_t r = ((int64_t)(i / chunk) * kXcds + die) * chunk + i % chunk;
    return r < cnt ? (int)r : cnt;
  }
  // Start of the wave's next batch in queue positions of `die`, or -1 when
  // every ray has been taken.
  __device__ __forceinline__ int next(int lane) {
    while (true) {
      int v = 0;
      if (lane == 0) v = atomicAdd(ctr + die, batch);
      const int base = __shfl(v, 0, 64);
      if (map(base) < cnt) return base;
      if (chunk <= 0 || ++tries >= kXcds) return -1;
      die = (die + 1) % kXcds;
    }
  }
};

size_t queue_bytes(int64_t cap);
RayQueue queue_at(void* base, int64_t cap);
int device_cus();

// Blocks of a persistent grid of `kernel` (blocks of `threads`): `per_cu`
// per compute unit, or, for per_cu = 0, as many as are resident at once by
// the occupancy calculator (queried once per kernel and size `lds` of its
// dynamic LDS); at least kXcds and at most `cap`.
int persistent_blocks(const void* kernel, int threads, int per_cu, int64_t cap, size_t lds = 0);

// matrix-core march (march_mfma.hip)
// packets: 16 consecutive queue rays per wave in step (else one ray per wave);
// blocks_per_cu: 0 = as many as fit; n: rays in the queue at most
mr_status dispatch_march_mfma(const mr_field* f, RayQueue q, const int* count, int* work, const MarchParams& P,
                              const BvhView& B, bool packets, unsigned long long* stats, int blocks_per_cu, int64_t n,
                              hipStream_t st);

// march of several fields, overlapping or not, over their summed medium
// (march_fields.hip) on the uniform grid; the fields share one layout
// (levels, SH components, colour layers, table and MLP types).  packets: 16
// consecutive queue rays per wave in step (else one ray per wave)
mr_status dispatch_march_fields(const mr_field* const* fields, int n_fields, RayQueue q, const int* count, int* work,
                                const MarchParams& P, const BvhView& B, bool packets, unsigned long long* stats,
                                int blocks_per_cu, int64_t n, hipStream_t st);

// march of incoherent segments level by level (march_lv.hip); it leaves queues
// of fewer than kLvMinRays rays alone.  Its scratch in the workspace: kLvPaceArea
// bytes of pacing counters, kLvPaceInts for each launch and zeroed with the
// header, then the features of the blocks' batches and a value per sample.
constexpr int kLvSamples = 4096;   // samples per batch
// Below this queue length the per-ray march is as fast (mid frames of 128 to
// 800 pixels a side); frames of fewer than kLvMinFrame rays hardly have such
// queues after their first bounce and carry no scratch.
constexpr int kLvMinRays = 8192;
constexpr int64_t kLvMinFrame = 65536;
constexpr int kLvLine = 32;        // words between two counters: a 128-byte line each
constexpr int kLvPaceInts = kXcds * 4 * kLvLine;
constexpr size_t kLvPaceArea = 2 * (size_t)(kMaxBounces + 2) * kLvPaceInts * sizeof(int);
struct LvScratch {
  int* pace;      // this launch's counters
  double* feat;   // (feature 0, feature 1) pairs
  float* edge;    // a value per sample (interval edges of the proposal march)
};
LvScratch lv_scratch(void* area, int launch);   // of the lv_bytes() at area
int lv_blocks();
size_t lv_bytes();
// Point queries go level by level from this many points, whatever order they
// come in: points in order share lines in k_query_mfma too, and gain later or
// not at all.  k_query_mfma / level by level, us, 2^19 entries, random points |
// a regular grid | 64 points along each of many rays:
// FP32      131 072: 119 / 140 | 69 / 111 | 81 / 130    196 608: 175 / 164 | 91 / 128 | 118 / 151
//           524 288: 447 / 308 | 179 / 210 | 309 / 270  3 M: 2574 / 1291 | 639 / 730 | 1767 / 1070
// FP16,     131 072: 96 / 115 | 43 / 93 | 68 / 112      196 608: 140 / 130 | 54 / 100 | 99 / 126
// BF16 MLPs 524 288: 372 / 236 | 99 / 160 | 260 / 216   3 M: 2177 / 1037 | 364 / 554 | 1492 / 870
// The line lies where random points cross (for FP16 tables below 2^19 entries
// that is later: 2^17, 196 608 / 262 144 points, 95 / 107 and 125 / 127).  A
// grid there is no slower than it was when k_query_mfma staged its weights
// before its points (344 / 127 us for 262 144).  With BF16 MLPs of one colour
// layer it would be (57 us against 90 for 166 375, 311 against 511 for 3 M),
// and those fields keep to k_query_mfma.
inline int64_t lv_min_points(const mr_field* f) {
  const auto& v = f->view;
  if (v.mlp_dtype == MR_BF16 && v.c_layers == 1) return INT64_MAX;
  return v.table_dtype == MR_F16 && v.log2_table < 19 ? 262144 : 196608;
}
// Fields whose samples are taken one level at a time: 16 levels, a table larger
// than a die's 4 MiB of L2, and levels of at most 8 MiB.  All levels together /
// level by level, us, FP32 MLPs unless said, 1 M random points | 64 along each of
// many rays | 800x800 mid frames:
//   table   1 MiB, FP32 2^13        303 / 325 | 211 / 293 | 10 124 / 10 808
//           4 MiB, FP32 2^15        319 / 397 | 209 / 322 | 10 279 / 11 344
//           8 MiB, FP32 2^16        488 / 415 | 276 / 331 | 11 372 / 11 802
//           8 MiB, FP16 2^17, BF16  445 / 369 | 255 / 295 |  9 290 /  9 151
//          16 MiB, FP32 2^17        656 / 422 | 344 / 337 | 12 695 / 11 966
//   level   4 MiB, FP32 2^19        858 / 494 | 492 / 388 | 15 034 / 12 915
//           8 MiB, FP32 2^20        913 / 670 | 543 / 500 | 15 655 / 14 139
//           8 MiB, FP16 2^21, BF16  846 / 596 | 509 / 440 | 14 162 / 12 120
//          16 MiB, FP32 2^21        941 / 809 | 566 / 571 | 16 009 / 15 142
//          32 MiB, FP32 2^22        954 / 894 | 574 / 630 | 16 260 / 16 010
// A level twice the L2 still gains, half of its lines are there; from 16 MiB on
// points along rays gain nothing.  At 8 MiB of table random points and light
// samples gain (400x400 emitter frame 7.8 / 7.0 ms) what plain FP32 frames lose.
bool lv_field(const mr_field* f);

// Scratch for a call without a workspace (false under capture or without
// memory: the caller then takes the general path), and its return after the
// call's launches.  The counters of one launch are zeroed, and so is the word
// after them (a queue head).  lv_fields counts the live fields (+1, -1).
bool lv_lease(hipStream_t st, LvScratch* lv);
void lv_return(hipStream_t st, const LvScratch& lv);
void lv_fields(int change);
mr_status query_lv(const mr_field* f, int64_t n, const float* x, const float* dirs, float* sigma, float* rgb,
                   float* feat, float* raw, const LvScratch& lv, hipStream_t st);
mr_status dispatch_march_lv(const mr_field* f, RayQueue q, const int* count, int* work, const MarchParams& P,
                            const LvScratch& lv, unsigned long long* stats, hipStream_t st);

// Medium of the light samples toward emitters (light_march.hip).  The shade
// pass leaves a light sample's record in the slot of the ray it shaded, in the
// queue it has read: origin and direction of the shadow segment, its length in
// hit_t, the light it carries in tr tg tb, the optical depth so far (0) in lr,
// where the light goes in rid (s >= 0: the ray in slot s of the next queue,
// ~i: the finished caller's ray i) and kLightPending in hit_p.  One launch per
// field adds that field's depth; the last one adds the light times the
// transmittance to the ray.  work: a zeroed counter for each of two kernels,
// kMaxBounces + 2 apart, or null for a fixed split; lv: scratch for marching a
// long queue level by level (one field that lv_field accepts), or null.
constexpr int kLightPending = 1;
mr_status dispatch_light_march(const mr_field* f, RayQueue q, RayQueue next, const int* count, int* work, float delta,
                               bool use_occupancy, bool last, float* radiance, int64_t n, const LvScratch* lv,
                               hipStream_t st);

// proposal-sampled march (defined with the proposal kernels)
// packets: 16 consecutive queue rays per wave when n_prop = 32 and n_fine <= 32.
// P.lv: queues of kLvMinRays or more go level by level, with scratch lv
mr_status dispatch_march_proposal(const mr_field* f, const mr_field* prop, RayQueue q, const int* count, int* work,
                                  const MarchParams& P, const BvhView& B, int n_prop, int n_fine, bool packets,
                                  unsigned long long* stats, int blocks_per_cu, int64_t n, const LvScratch& lv,
                                  hipStream_t st);

}  // namespace mr
