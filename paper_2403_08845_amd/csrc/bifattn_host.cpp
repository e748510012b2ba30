// Host side of libbifattn: argument validation, work splitting, workspace
// ownership, launches and the C ABI declared in include/bifattn.h.
#include "bifattn.h"

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <new>
#include <vector>

#include "bifattn_internal.h"

using namespace bifattn;

struct bifattn_plan_s {
  bifattn_dims_t dims{};
  float scale = 0.f;
  int p = 0, M = 0;  // query rows per (sample, group) unit (heads x tokens), rows per group
  int ntok = 1;
  int ctx_mode = kCtxNone;
  int dec_tiles = 1;
  int ctx_keys = 0, S_c = 0, ctx_row_blocks = 1, n_ctx_blocks = 0, n_ctx_small_blocks = 0;
  int ctx_wide = 0;  // many-row path: waves per work-group of its context kernel (8 or 4)
  double many_us = -1.0;  // many_row_split's estimate, where it chose the split
  int dec_keys = 0, S_d = 0, n_dec_blocks = 0;
  int rep_keys = 0, S_r = 0, n_rep_blocks = 0;
  int fused = 1;       // context and decode work-groups in one launch
  int fork = 0;        // many-row path: decode work-groups beside the context ones (in their
                       // launch when fused, else on the side stream)
  // The plan's own stream (non-blocking, default priority): the workspace is
  // allocated and freed in its order (stream-ordered allocator, so that
  // freeing it does not synchronise the device) and, on many-row plans with
  // a large decode part, the decode launch runs on it beside the context
  // kernel.
  hipStream_t side = nullptr;
  bool ws_async = false;  // workspace from hipMallocAsync (else hipMalloc)
  hipEvent_t fork_ev = nullptr, join_ev = nullptr;
  // Recorded on the call's stream after the last launch of every call: what
  // destroy and set_timing wait for (the plan's own work, not the device's).
  hipEvent_t done_ev = nullptr;
  bool done_recorded = false;
  int path = BIFATTN_PATH_BIFURCATED;  // resolved: bifurcated or standard
  int device = 0;
  // workspace
  void* ws = nullptr;
  size_t ws_bytes = 0;
  float* ctx_acc = nullptr;
  float2* ctx_ml = nullptr;
  float* dec_acc = nullptr;
  float2* dec_ml = nullptr;
  int* status = nullptr;
  // timing
  int timed_kernel = -1;
  int timing_cap = 0;
  int timing_n = 0;
  std::vector<hipEvent_t> events;
};

namespace {

// Events that only order the plan's work on its device (the completion
// mark, the side-stream fork and join): no timing, and no system-scope fence
// when recorded (the host reads nothing through them; a recorded system
// fence writes back the L2 and costs ~3 us per call). Each kernel's own
// end-of-dispatch release still publishes its results to the device.
constexpr unsigned kOrderEventFlags = hipEventDisableTiming | hipEventDisableSystemFence;

constexpr int kCUs = 256;  // MI355X compute units; split heuristics aim at whole waves of them

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }
size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Tuning overrides from the environment: a positive integer, else `fallback`.
int env_int(const char* name, int fallback) {
  const char* v = std::getenv(name);
  if (!v || !*v) return fallback;
  char* end = nullptr;
  long x = std::strtol(v, &end, 10);
  return (end && *end == 0 && x > 0 && x < (1 << 30)) ? (int)x : fallback;
}

// A switch from the environment: -1 when unset or not an integer, else its value.
int env_switch(const char* name) {
  const char* v = std::getenv(name);
  if (!v || !*v) return -1;
  char* end = nullptr;
  long x = std::strtol(v, &end, 10);
  return (end && *end == 0 && x >= 0 && x < 16) ? (int)x : -1;
}

bool aligned(const void* ptr, uintptr_t a) { return ((uintptr_t)ptr & (a - 1)) == 0; }

// The plan's workspace lives on the device that was current at its creation:
// a call is accepted only on a stream of that device (the null stream: the
// current device), so that no kernel runs on one GPU against another GPU's
// workspace.
bool on_plan_device(const bifattn_plan_s* P, hipStream_t stream) {
  int dev = -1;
  if (stream) {
    hipDevice_t d = -1;
    if (hipStreamGetDevice(stream, &d) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    dev = d;
  } else if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return dev == P->device;
}

// Keys one decode work-group reads: the whole decode cache up to 1024 keys
// (each work-group writes partials for p rows per wave, so short chunks
// multiply that traffic, and ragged lengths leave short chunks nearly empty),
// halved (never below `least`) only while fewer than half as many work-groups
// as CUs would exist.
int dec_chunk_keys(int64_t units, int64_t rows, int least) {
  int keys = (int)std::min<int64_t>(1024, std::max<int64_t>(128, round_up(rows, 128)));
  while (keys / 2 >= least && units * ceil_div(rows, keys) < kCUs / 2) keys /= 2;
  return keys;
}
// Rounding of the many-row context chunk: its kernel runs 128-key stages when
// its chunks are multiples of 128 keys, so chunks of at least 1024 keys are
// rounded to 128, shorter ones to the 64 keys of its smaller stages.
int ck_step(int64_t m_c, int64_t splits) { return ceil_div(m_c, splits) >= 1024 ? 128 : 64; }

// Waves per work-group and key splits of a launch that holds the 32x32
// context work-groups and the decode work-groups. More splits shorten the
// context work-groups, but each adds a partial of every query row for the
// combine, and context work-groups beyond what the decode ones leave of the
// GPU run behind others. Eight waves (256 rows) halve the reads of a key
// chunk and of its work-groups there is one per CU; four (two per CU, three
// with d = 64: LDS and registers) overlap one's start and end with the
// other's products, which wins on short contexts (b 16, h 16, g 4, 4 tokens,
// m_c 3000: 16.3 us per step, eight 19.1; MQA over 16k: 61.6, eight 56.3).
// The choice is the least of an estimate of the step's time. Its terms are the
// parts of a step, but its constants are a fit of whole steps (1700 random
// layers, 33 to 38400 rows per group, 0.2k to 40k keys, every cache type, at
// about 24 settings each), not times of the parts. The chosen setting is 1.2%
// slower than the best of those on average, 7% at the 95th percentile and 28%
// at worst; the estimate plus 6 us is within 20% of the time of 19 steps in 20.
// With two four-wave work-groups per CU counted for d = 64 too, decode work as
// long for codes as for bf16, and a work-group that shares its CU as fast as
// one alone, it was 2.6% and 42% (h = g = 40, d 64, m_c 12000, b 40: 35.3 us per
// step, now 31.6; g 8, m_c 35226, 54 rows, no decode rows: 44.0, now 36.2).
struct ManySplit {
  int waves = 4;
  int64_t splits = 1;
  double us = 0.0;
};
ManySplit many_row_split(const bifattn_plan_s* P, int64_t rows) {
  const bifattn_dims_t& d = P->dims;
  const bool half = d.d == 64;
  const int S_d = P->S_d;
  const double rows_all = (double)d.g * rows;
  const double codes = d.kv_type == BIFATTN_KV_BF16 ? 1.0 : d.kv_type == BIFATTN_KV_INT4 ? 0.54 : 0.61;
  const double td =
      1.75 + codes * (half ? 0.8 : 1.57) * (double)ceil_div(std::min(P->dec_keys, d.m_d_max), 128);
  const double stream = 2.0 * d.g * kv_row_bytes(d.d, d.kv_type) *
                        ((double)d.m_c + 0.75 * (double)d.b * d.m_d_max) / 5.84e6;
  ManySplit best;
  double least = 0.0;
  for (int waves = 4; waves <= (rows > 128 ? 8 : 4); waves += 4) {
    const int slots = waves == 8 ? kCUs : (half ? 3 : 2) * kCUs;
    const int64_t per_split = (int64_t)d.g * ceil_div(rows, 32 * waves);
    const int64_t dec_wgs = ceil_div((int64_t)d.b * d.g * S_d, waves / kWaves);
    const double start = waves == 8 ? 6.2 : 2.4;
    const double per_key = (waves == 8 ? 0.0182 : 0.0175) * (half ? 0.62 : 1.0);
    const int64_t most = std::max<int64_t>(1, std::min(ceil_div(d.m_c, 128), 2 * slots / per_split));
    for (int64_t S = 1; S <= most; S += 1 + S / 8) {
      const int64_t keys = round_up(ceil_div(d.m_c, S), ck_step(d.m_c, S));
      const int64_t parts = ceil_div(d.m_c, keys);
      const int64_t wgs = per_split * parts;
      // the clock gives way as more than five eighths of the CUs run context
      // work-groups; those that share a CU slow each other
      const int64_t cus = std::min<int64_t>(wgs, kCUs);
      const int64_t per_cu = ceil_div(std::min<int64_t>(wgs, slots), kCUs);
      const double busy = (1.0 + 0.07 * (double)std::max<int64_t>(0, cus - 160) / 96.0) *
                          (1.0 + 0.27 * (double)(per_cu - 1));
      const double tc = start + per_key * (double)keys * busy;
      // whole rounds of context work-groups, then the last ones (if any) with
      // the decode ones beside them
      const int64_t rem = wgs % slots;
      const double tr = rem ? tc : 0.0;
      const double all_slots = (double)ceil_div(dec_wgs, slots - rem) * td;
      const double beside = dec_wgs == 0           ? 0.0
                            : all_slots <= tr + td ? all_slots
                                                   : ((double)rem * tc + (double)dec_wgs * td) / slots + 0.5 * td;
      double t = (double)(wgs / slots) * tc + std::max(tr, beside) + 0.05 * std::min(tr, beside);
      const int64_t loads = ceil_div(parts * d.d, 256) + ceil_div(4 * S_d * d.d, 256);
      t = std::max(t, stream) + 0.15 * t + 2.2 * (double)(ceil_div(loads, 16) - 1) +
          (double)(parts + 4 * S_d) * rows_all * (d.d * 4 + 16) / 2.19e6;
      // of (nearly) equal ones the one with more splits: shorter work-groups
      const bool first = waves == 4 && S == 1;
      if (first || t < least * (waves == best.waves ? 1.005 : 1.0)) {
        least = first ? t : std::min(least, t);
        best.waves = waves;
        best.splits = S;
      }
    }
  }
  best.us = least;
  return best;
}

// Estimated times of a small step (at most 512 units of at most 32 query rows,
// 3200 keys) on either path, us, from a fit to 6000 random layers timed on
// both: within 16% and 20% of the time of 19 in 20.
//   standard: a start (two query tiles 1.3 us more), then the keys, which take
//     longer where two units share a CU and with two query tiles; the rows
//     and the decode caches' bytes;
//   bifurcated, few rows: start and combine, the context and the decode chunk,
//     the partials, the work-groups.
double standard_us(const bifattn_plan_s* P) {
  const bifattn_dims_t& d = P->dims;
  const bool half = d.d == 64, shared = (int64_t)d.b * d.g > kCUs, tiles2 = P->p > 16;
  const double per_key = (half ? (shared ? 5.8 : 3.8) : (shared ? 11.0 : 7.3)) +
                         (tiles2 ? (half ? 1.0 : 2.7) : 0.0);
  return 4.8 + (tiles2 ? 1.3 : 0.0) + per_key * 1e-3 * ((double)d.m_c + d.m_d_max) +
         2.4e-6 * (double)P->M * d.g * d.d +
         0.031e-6 * 2.0 * d.b * d.g * (double)d.m_d_max * kv_row_bytes(d.d, d.kv_type);
}
double bifurcated_us(const bifattn_plan_s* P) {
  const bifattn_dims_t& d = P->dims;
  if (P->ctx_mode == kCtxLarge)
    return 4.5 + 1.17 * (P->many_us >= 0.0 ? P->many_us : many_row_split(P, P->M).us);
  const bool half = d.d == 64;
  return 8.0 + (half ? 4.2e-3 : 7.0e-3) * ((double)d.m_c / P->S_c) +
         (half ? 1.0e-3 : 4.0e-3) * std::min(P->dec_keys, d.m_d_max) +
         1e-6 * (double)(P->S_c + 4 * P->S_d) * P->M * d.g * (d.d * 4 + 16) +
         (half ? 0.3 : 1.1) / (2 * kCUs) * (double)(P->n_ctx_small_blocks + P->n_dec_blocks);
}

// Keys one replicated-ablation work-group reads: `start` by default, halved
// (down to 128) while fewer than two work-groups per CU would exist.
int seq_keys(int64_t units, int64_t rows, int start) {
  int keys = start;
  while (keys > 128 && units * ceil_div(rows, keys) < 2 * kCUs) keys /= 2;
  return keys;
}

// allow_fork: the many-row path may run the decode launch on the plan's own
// stream (off for the allocation-free entry point, which owns no stream).
// coarse: the longest chunks (the allocation-free entry point takes them where
// the partials of the usual ones pass its scratch).
bifattn_status_t plan_splits(bifattn_plan_s* P, bool allow_fork = true, bool coarse = false) {
  const bifattn_dims_t& d = P->dims;
  P->ntok = d.n > 0 ? d.n : 1;
  // The n tokens of a head are consecutive rows of q and out, so a unit's
  // query rows are its p heads times n tokens.
  P->p = d.h / d.g * P->ntok;
  P->M = d.b * P->p;
  P->dec_tiles = P->p <= 16 ? 1 : (P->p <= 32 ? 2 : 4);
  const int64_t M = P->M;
  const int64_t units = (int64_t)d.b * d.g;
  if (d.m_d_max > 0) {
    // Halves under 256 keys (two tiles per wave) don't pay: b 2, h 32, g 8,
    // m_d 200, 12.3 us per step with chunks of 128, 11.3 with one of 256;
    // b 20, h 8, g 4, m_d 300, 32.9 with 192, 30.3 with one chunk.
    P->dec_keys = (int)round_up(
        env_int("BIFATTN_DEC_KEYS", dec_chunk_keys(units, d.m_d_max, coarse ? 128 : 256)), kTileKeys);
    P->S_d = (int)ceil_div(d.m_d_max, P->dec_keys);
  } else {
    P->dec_keys = kTileKeys;
    P->S_d = 0;
  }
  const int64_t quarter = round_up(ceil_div(d.m_c, 4), kWaves * kTileKeys);
  const int64_t long_keys = std::min<int64_t>(2048, std::max<int64_t>(1024, quarter));
  // Few rows: up to two query tiles per wave. (Four, 33 to 64 rows, leave one
  // wave per SIMD: b 16, h 32, g 8, m_c 3001 21.6 us per step against 14.5
  // with the many-row kernel, m_c 20000 34.5 against 29; they stay for units
  // of more than 32 rows, whose decode part needs the same.)
  if (M <= 32 || (M <= 64 && P->dec_tiles == 4)) {
    // Few rows per group: S_c work-groups per group, interleaved over the
    // group's tiles. Where the step fills the GPU, about four of them, each
    // with 1024..2048 keys (2-4 decode work-groups' worth): fewer, longer
    // context work-groups leave fewer partials to merge, too few stop
    // covering the decode part's time. A step that leaves slots idle (two
    // work-groups per CU) is as long as its longest work-group, so it takes
    // chunks of about twice the keys that an even split over the slots would
    // give each, down to 256 (shorter ones cost the combine more than they
    // save). Measured, long chunks against these (us per step, bf16, d = 128):
    // b 5, h 32, g 8, m_c 3001 19.7 -> 13.8; m_c 12000 29.6 -> 19.8; b 20,
    // h 8, g 4, m_c 25000 44.6 -> 30.3; b 16, h = g = 32, m_c 8192, m_d 256
    // 38.0 -> 37.1 (1536 keys; 1024: 40.1). Somewhat more work-groups than CUs
    // are the worst of both: a few CUs hold two (b 2, h 80, g 40, 4 tokens, m_c
    // 10456: 280 of 1536 keys 48.9, 240 of 1792 40.0; b 3, h = g = 40, m_c 8792 41.2,
    // 33.2), so they are cut to one each. Over 260 layers the chunks are 2.5%
    // slower than the best of thirteen, long ones throughout 28%. With four query tiles per wave one
    // work-group fills a CU, and a quarter more than an even share each leaves
    // some free for the decode ones (h 1536, g 32, m_c 3079, m_d 1024: 512 keys
    // 41.0, 1024 34.4, 640 35.9).
    P->ctx_mode = M <= 16 ? kCtxSmall1 : (M <= 32 ? kCtxSmall2 : kCtxSmall4);
    constexpr int step = kWaves * kTileKeys;
    int64_t keys = long_keys;
    if (!coarse) {
      const int64_t all = (int64_t)d.g * d.m_c + units * d.m_d_max;  // keys of every unit
      const int64_t share = M <= 32 ? ceil_div(2 * all, 2 * kCUs) : ceil_div(5 * all, 4 * kCUs);
      const int64_t even = std::max<int64_t>(256, share);
      if (even < keys) {
        int64_t S = ceil_div(d.m_c, even);
        const int64_t whole = kCUs / d.g;  // splits of one work-group per CU, 0 if g alone is more
        if (M <= 32 && d.g * S > kCUs && d.g * S <= kCUs * 7 / 6 && whole > 0 &&
            ceil_div(d.m_c, whole) <= long_keys)
          S = whole;
        keys = round_up(ceil_div(d.m_c, S), step);
      }
    }
    P->ctx_keys = (int)round_up(env_int("BIFATTN_CTX_KEYS", (int)keys), step);
    P->ctx_row_blocks = 1;
  } else {
    // Many rows take the 32x32 MFMA kernel (work-groups of eight or four
    // waves of 32 rows).
    //
    // The context part is bound by the matrix cores and the decode part by
    // HBM, so they run beside each other. The 32x32 kernel's launch holds the
    // decode work-groups after the context ones (units of at most 32 query
    // rows: more need registers that two waves per SIMD don't leave); against
    // a second launch behind it or on a side stream (us per step): MQA, 128
    // samples over 16k, 64.2 -> 53.7-57; 4 draft tokens 89-95 -> 81.6; b 40,
    // h 32, g 8, m_c 3000 31.6 -> 19.5. Otherwise a large decode part (16 MiB
    // or more, its HBM time at ~5 TB/s above half the context's matrix time
    // at ~1 PFLOP/s) goes to the plan's side stream from 128 rows per group;
    // a small one, or one beside fewer rows, follows the context kernel (44
    // layers of 66 to 126 rows and large decode parts take 8% less time so
    // than on the side stream, whose fork and join are about 10 us of their
    // 40 to 100; waves of 16 rows for the context there took 1% more).
    // BIFATTN_FORK=0/1 forces the parts behind or beside each other.
    P->ctx_mode = kCtxLarge;
    const double dec_bytes = 2.0 * d.b * d.g * (double)d.m_d_max * kv_row_bytes(d.d, d.kv_type);
    const double ctx_flops = 4.0 * d.h * P->ntok * d.d * (double)d.b * d.m_c;
    const int fork_env = coarse ? 0 : env_switch("BIFATTN_FORK");
    // Without decode rows there is no second launch for larger units either.
    // The estimate serves them for many rows of d = 64, whose first split may
    // pass the GPU (us per step: b 43, h 2048, g 32, m_c 919 85.4 -> 49.7; b 275,
    // h 40, g 1, m_c 9142 73.0 -> 52.3); filling the GPU is the better rule for
    // fewer rows and d = 128 (b 48, h 160, g 8, 2 tokens, m_c 2072 37.6, 41.8).
    const bool estimated = P->dec_tiles <= 2 || (d.m_d_max == 0 && d.d == 64 && M >= 1024);
    const bool one_launch = !coarse && estimated;
    const bool big_decode = dec_bytes >= 16.0 * (1 << 20) && dec_bytes / 5e12 > 0.5 * ctx_flops / 1e15;
    P->fork = (allow_fork || one_launch) && d.m_d_max > 0 &&
              (fork_env == -1 ? one_launch || (big_decode && M >= 128) : fork_env == 1);
    P->fused = one_launch && P->fork;
    const int wgs = env_int("BIFATTN_CTX_WGS", 0);
    ManySplit split;
    if (one_launch && wgs == 0) {
      split = many_row_split(P, M);
      P->many_us = split.us;
    } else {
      split.waves = M >= 256 ? 8 : 4;
    }
    P->ctx_wide = split.waves;
    P->ctx_row_blocks = (int)ceil_div(M, 32 * P->ctx_wide);
    if (!one_launch || wgs > 0) {
      // With the decode work-groups in a launch of their own: about one
      // work-group per CU for eight-wave work-groups, two for four-wave ones;
      // beside the side stream, one per CU (five eighths of that with eight
      // waves: the decode work-groups take the rest).
      const int target = P->fork ? (P->ctx_wide == 8 ? kCUs * 5 / 8 : kCUs)
                                 : (P->ctx_wide == 8 ? kCUs : 2 * kCUs);
      split.splits = ceil_div(wgs > 0 ? wgs : target, (int64_t)d.g * P->ctx_row_blocks);
    }
    if (coarse && d.d == 64) split.splits = ceil_div(2 * kCUs, d.g * ceil_div(M, 128));
    const int64_t splits = std::max<int64_t>(1, split.splits);
    int64_t ck = round_up(ceil_div(d.m_c, splits), ck_step(d.m_c, splits));
    if (coarse && M <= 64) ck = long_keys;
    P->ctx_keys = (int)round_up(env_int("BIFATTN_CTX_KEYS", (int)ck), 64);
  }
  P->S_c = (int)ceil_div(d.m_c, P->ctx_keys);
  P->n_ctx_blocks = P->ctx_mode == kCtxLarge ? d.g * P->S_c * P->ctx_row_blocks : 0;
  P->n_ctx_small_blocks = P->ctx_mode == kCtxLarge ? 0 : d.g * P->S_c;
  P->n_dec_blocks = (int)(units * P->S_d);
  const int64_t rep_rows = (int64_t)d.m_c + d.m_d_max;
  P->rep_keys = (int)round_up(env_int("BIFATTN_REP_KEYS", seq_keys(units, rep_rows, 1024)),
                              kTileKeys);
  P->S_r = (int)ceil_div(rep_rows, P->rep_keys);
  P->n_rep_blocks = (int)(units * P->S_r);
  // Few-row context and decode work-groups share one launch (the context
  // part then overlaps the decode part's streaming); BIFATTN_LAUNCH=2 splits
  // them into two launches.
  if (P->ctx_mode != kCtxLarge) P->fused = env_int("BIFATTN_LAUNCH", 1) == 1;
  // The workload-based switch: the standard path reads the context once per
  // sample but needs one launch and no partials. It is taken where its estimate
  // is the lower one, while every unit is resident in one round of work-groups
  // (b*g <= 512) and has at most two query tiles; past 3200 keys nothing was
  // measured. Of those 6000 layers the choice is 0.4% slower than the faster
  // path on average (11% at the 99th percentile); a line in keys by head dimension,
  // units per CU and rows per group was 1.6% slower, since the rows of all groups
  // and the decode rows matter as much (us per step, standard against bifurcated: b 64, h 32,
  // g 8, 2164 keys 27.0, 17.3; b 256, h 32, g 2, 2164 keys 27.7, 33.9; b 18, h 32, g 8,
  // 688 + 1024 keys 16.4, 21.6).
  if (d.path == BIFATTN_PATH_AUTO) {
    const bool small = units <= 2 * kCUs && P->p <= 32 && (int64_t)d.m_c + d.m_d_max <= 3200;
    P->path = small && standard_us(P) <= bifurcated_us(P) ? BIFATTN_PATH_STANDARD
                                                          : BIFATTN_PATH_BIFURCATED;
  } else {
    P->path = d.path;
  }
  if ((int64_t)P->n_ctx_blocks + P->n_ctx_small_blocks + P->n_dec_blocks > INT32_MAX / 2 ||
      units * P->S_r > INT32_MAX / 2)
    return BIFATTN_EINVAL;
  return BIFATTN_OK;
}

// Byte offsets of the workspace parts (256-byte aligned) and its size: the
// context partials, the decode partials (sized for the replicated ablation's
// splits too when `replicated`), and the status word.
struct WorkspaceLayout {
  size_t ctx_acc = 0, ctx_ml = 0, dec_acc = 0, dec_ml = 0, status = 0, bytes = 0;
};
WorkspaceLayout workspace_layout(const bifattn_plan_s* P, bool replicated) {
  const bifattn_dims_t& d = P->dims;
  const size_t D = (size_t)d.d;
  const size_t ctx_rows = (size_t)d.g * P->S_c * P->M;
  const int s_dec = replicated && P->S_r > P->S_d ? P->S_r : P->S_d;
  const size_t dec_rows = (size_t)d.b * d.g * (size_t)s_dec * kWaves * P->p;
  WorkspaceLayout L;
  size_t off = 0;
  L.ctx_acc = off;
  off = align256(off + ctx_rows * D * 4);
  L.ctx_ml = off;
  off = align256(off + ctx_rows * 8);
  L.dec_acc = off;
  off = align256(off + dec_rows * D * 4);
  L.dec_ml = off;
  off = align256(off + dec_rows * 8);
  L.status = off;
  L.bytes = align256(off + 4);
  return L;
}

void set_workspace(bifattn_plan_s* P, void* base_ptr, const WorkspaceLayout& L) {
  char* base = static_cast<char*>(base_ptr);
  P->ws = base_ptr;
  P->ws_bytes = L.bytes;
  P->ctx_acc = reinterpret_cast<float*>(base + L.ctx_acc);
  P->ctx_ml = reinterpret_cast<float2*>(base + L.ctx_ml);
  P->dec_acc = reinterpret_cast<float*>(base + L.dec_acc);
  P->dec_ml = reinterpret_cast<float2*>(base + L.dec_ml);
  P->status = reinterpret_cast<int*>(base + L.status);
}

bifattn_status_t check_dims(const bifattn_dims_t* d) {
  if (!d) return BIFATTN_EINVAL;
  if (d->b < 1 || d->h < 1 || d->g < 1 || d->m_c < 1 || d->m_d_max < 0 || d->n < 0)
    return BIFATTN_EINVAL;
  if (d->h % d->g) return BIFATTN_EINVAL;
  if (!(std::isfinite(d->scale))) return BIFATTN_EINVAL;
  if (d->kv_type != BIFATTN_KV_BF16 && d->kv_type != BIFATTN_KV_FP8_E4M3 &&
      d->kv_type != BIFATTN_KV_INT8 && d->kv_type != BIFATTN_KV_INT4)
    return BIFATTN_EINVAL;
  if (d->path != BIFATTN_PATH_AUTO && d->path != BIFATTN_PATH_BIFURCATED &&
      d->path != BIFATTN_PATH_STANDARD)
    return BIFATTN_EINVAL;
  if (d->d != 64 && d->d != 128) return BIFATTN_EUNSUPPORTED;
  const double ntok = d->n > 0 ? d->n : 1;
  if ((double)(d->h / d->g) * ntok > kMaxP) return BIFATTN_EUNSUPPORTED;
  // element counts of the largest tensors must stay far from 2^62
  const double lim = 4.0e18;
  const double dd = d->d;
  if ((double)d->b * d->h * ntok * dd > lim || (double)d->g * d->m_c * dd > lim ||
      (double)d->b * d->g * ((double)d->m_c + d->m_d_max) * dd > lim)
    return BIFATTN_EINVAL;
  if ((double)d->b * d->h * ntok > INT32_MAX / 2 || (double)d->b * d->g > INT32_MAX / 2)
    return BIFATTN_EINVAL;
  // Kernels address one cache (a group's context, a sample's decode rows, or
  // both in the replicated ablation) with 32-bit byte offsets.
  if (((double)d->m_c + d->m_d_max) * kv_row_bytes(d->d, d->kv_type) > INT32_MAX)
    return BIFATTN_EUNSUPPORTED;
  return BIFATTN_OK;
}

// Mark the end of a call's work on its stream.
void mark_done(bifattn_plan_s* P, hipStream_t stream) {
  if (!P->done_ev) return;
  if (hipEventRecord(P->done_ev, stream) == hipSuccess)
    P->done_recorded = true;
  else
    (void)hipGetLastError();
}

// The events of a call's last launch with the completion mark added: the
// launch records the plan's done event itself at the kernel's end (no
// separate marker on the stream), unless it already records a timing stop.
LaunchEvents last_launch(bifattn_plan_s* P, LaunchEvents ev) {
  if (!ev.stop && P->done_ev) {
    ev.stop = P->done_ev;
    P->done_recorded = true;
  }
  return ev;
}

// Wait for the plan's own enqueued work: the last call's end (every earlier
// call of the plan ran on a stream its successor was ordered after, or is
// covered by the caller's one-stream-at-a-time contract) and the side stream.
bool wait_done(bifattn_plan_s* P) {
  bool ok = true;
  if (P->done_recorded && hipEventSynchronize(P->done_ev) != hipSuccess) ok = false;
  if (P->side && hipStreamSynchronize(P->side) != hipSuccess) ok = false;
  return ok;
}

void free_events(bifattn_plan_s* P);

// Free everything the plan owns and the plan itself. The workspace is freed
// in the order of the plan's own stream (a stream-ordered free waits for
// that stream only; hipFree would synchronise the whole device), so the
// caller must have waited for the plan's work first.
bool release_plan(bifattn_plan_s* P) {
  bool ok = true;
  free_events(P);
  if (P->done_ev) (void)hipEventDestroy(P->done_ev);
  if (P->fork_ev) (void)hipEventDestroy(P->fork_ev);
  if (P->join_ev) (void)hipEventDestroy(P->join_ev);
  if (P->ws) {
    if (P->ws_async)
      ok = hipFreeAsync(P->ws, P->side) == hipSuccess && hipStreamSynchronize(P->side) == hipSuccess;
    else
      ok = hipFree(P->ws) == hipSuccess;
  }
  if (P->side) (void)hipStreamDestroy(P->side);
  if (!ok) (void)hipGetLastError();
  delete P;
  return ok;
}

void free_events(bifattn_plan_s* P) {
  for (hipEvent_t e : P->events) (void)hipEventDestroy(e);
  P->events.clear();
  P->timing_cap = P->timing_n = 0;
  P->timed_kernel = -1;
}

// Event pair of one timed section of this call, if that section is being
// timed. With `in_kernel`, the section's launches record the pair
// themselves (the first launch's kernel start, the last launch's kernel
// end: first() / last() / both()), so the time is the kernels' own, as a
// kernel trace shows it; otherwise the pair is recorded on the stream around
// the section.
struct TimedSection {
  bifattn_plan_s* P;
  hipStream_t stream;
  bool on = false;
  bool in_kernel = false;
  TimedSection(bifattn_plan_s* P_, int kernel, hipStream_t s, bool in_kernel_ = false)
      : P(P_), stream(s), in_kernel(in_kernel_) {
    on = P->timed_kernel == kernel && P->timing_n < P->timing_cap;
    if (on && !in_kernel) (void)hipEventRecord(P->events[2 * P->timing_n], stream);
  }
  hipEvent_t ev(int k) const { return on && in_kernel ? P->events[2 * P->timing_n + k] : nullptr; }
  LaunchEvents first() const { return LaunchEvents{ev(0), nullptr}; }
  LaunchEvents last() const { return LaunchEvents{nullptr, ev(1)}; }
  LaunchEvents both() const { return LaunchEvents{ev(0), ev(1)}; }
  // This section's events where they are set, else the other's (sections of
  // one call may share a launch; at most one of them is being timed).
  static LaunchEvents either(const LaunchEvents& a, const LaunchEvents& b) {
    return LaunchEvents{a.start ? a.start : b.start, a.stop ? a.stop : b.stop};
  }
  // For sections that span streams: the pair recorded on the call's stream.
  void record_start() {
    if (on && in_kernel) (void)hipEventRecord(P->events[2 * P->timing_n], stream);
  }
  void record_stop() {
    if (on && in_kernel) (void)hipEventRecord(P->events[2 * P->timing_n + 1], stream);
  }
  void end() {
    if (on) {
      if (!in_kernel) (void)hipEventRecord(P->events[2 * P->timing_n + 1], stream);
      ++P->timing_n;
      on = false;
    }
  }
};

PartialsParams base_params(const bifattn_plan_s* P, const void* q, const int32_t* lens,
                           const float* k_scale) {
  PartialsParams K{};
  K.q = static_cast<const uint16_t*>(q);
  K.lens = lens;
  K.k_scale = k_scale;
  K.ctx_acc = P->ctx_acc;
  K.ctx_ml = P->ctx_ml;
  K.dec_acc = P->dec_acc;
  K.dec_ml = P->dec_ml;
  K.status = P->status;
  K.b = P->dims.b;
  K.h = P->dims.h * P->ntok;
  K.g = P->dims.g;
  K.p = P->p;
  K.M = P->M;
  K.ntok = P->ntok;
  K.m_c = P->dims.m_c;
  K.m_d_max = P->dims.m_d_max;
  // scale * (q . k) = |scale| * ((-q) . k): a negative scale negates q, which
  // is exact in bf16, so the kernels only ever see a positive scale.
  K.scale_log2 = std::fabs(P->scale) * 1.4426950408889634f;
  K.q_sign = P->scale < 0.f ? 0x80008000u : 0u;
  return K;
}

CombineParams combine_params(const bifattn_plan_s* P, const int32_t* lens, const float* k_scale,
                             const float* v_scale, float* out) {
  CombineParams C{};
  C.k_scale = k_scale;
  C.v_scale = v_scale;
  C.ctx_acc = P->ctx_acc;
  C.ctx_ml = P->ctx_ml;
  C.dec_acc = P->dec_acc;
  C.dec_ml = P->dec_ml;
  C.lens = lens;
  C.out = out;
  C.status = P->status;
  C.b = P->dims.b;
  C.h = P->dims.h * P->ntok;
  C.g = P->dims.g;
  C.p = P->p;
  C.M = P->M;
  C.m_d_max = P->dims.m_d_max;
  return C;
}

}  // namespace

extern "C" {

const char* bifattn_status_string(bifattn_status_t s) {
  switch (s) {
    case BIFATTN_OK: return "ok";
    case BIFATTN_EINVAL: return "invalid argument";
    case BIFATTN_EUNSUPPORTED:
      return "unsupported shape (d must be 64 or 128, (h/g)*n at most 64, one sample's cache "
             "rows under 2^31 bytes)";
    case BIFATTN_EALIGN: return "tensor pointer not 16-byte aligned (decode_lens: 4-byte)";
    case BIFATTN_ENOMEM: return "device memory allocation failed";
    case BIFATTN_EHIP: return "HIP runtime error";
    case BIFATTN_ELENS: return "a decode length was outside [0, m_d_max] and was clamped";
    case BIFATTN_ESCALE: return "a key or value scale was not a positive normal float";
    case BIFATTN_ESCRATCH:
      return "the workspace of this problem exceeds the fixed scratch buffer of "
             "bifattn_decode_noalloc (64 MiB)";
  }
  return "unknown status";
}

int32_t bifattn_version(void) { return BIFATTN_VERSION; }

bifattn_status_t bifattn_plan_create(const bifattn_dims_t* dims, bifattn_plan_t* plan) {
  if (!plan) return BIFATTN_EINVAL;
  *plan = nullptr;
  bifattn_status_t st = check_dims(dims);
  if (st != BIFATTN_OK) return st;
  bifattn_plan_s* P = new (std::nothrow) bifattn_plan_s();
  if (!P) return BIFATTN_ENOMEM;
  P->dims = *dims;
  P->scale = dims->scale != 0.f ? dims->scale : 1.0f / std::sqrt((float)dims->d);
  st = plan_splits(P);
  if (st != BIFATTN_OK) {
    delete P;
    return st;
  }
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1 || hipGetDevice(&P->device) != hipSuccess) {
    delete P;
    return BIFATTN_EHIP;
  }
  const WorkspaceLayout L = workspace_layout(P, true);
  const size_t off = L.bytes;
  if (hipStreamCreateWithFlags(&P->side, hipStreamNonBlocking) != hipSuccess) {
    (void)hipGetLastError();
    delete P;
    return BIFATTN_EHIP;
  }
  if (hipMallocAsync(&P->ws, off, P->side) == hipSuccess) {
    P->ws_async = true;
  } else {
    (void)hipGetLastError();
    P->ws = nullptr;
    if (hipMalloc(&P->ws, off) != hipSuccess) {
      (void)hipGetLastError();
      P->ws = nullptr;
      release_plan(P);
      return BIFATTN_ENOMEM;
    }
  }
  set_workspace(P, P->ws, L);
  if (hipMemsetAsync(P->status, 0, 4, P->side) != hipSuccess ||
      hipStreamSynchronize(P->side) != hipSuccess ||
      hipEventCreateWithFlags(&P->done_ev, kOrderEventFlags) != hipSuccess) {
    (void)hipGetLastError();
    release_plan(P);
    return BIFATTN_EHIP;
  }
  if (P->fork && !P->fused) {
    if (hipEventCreateWithFlags(&P->fork_ev, kOrderEventFlags) != hipSuccess ||
        hipEventCreateWithFlags(&P->join_ev, kOrderEventFlags) != hipSuccess) {
      (void)hipGetLastError();
      P->fork = 0;
    }
  }
  *plan = P;
  return BIFATTN_OK;
}

bifattn_status_t bifattn_plan_destroy(bifattn_plan_t P) {
  if (!P) return BIFATTN_OK;
  bifattn_status_t st = BIFATTN_OK;
  if (!wait_done(P)) st = BIFATTN_EHIP;
  if (!release_plan(P)) st = BIFATTN_EHIP;
  return st;
}

bifattn_status_t bifattn_plan_get_info(bifattn_plan_t P, bifattn_plan_info_t* info) {
  if (!P || !info) return BIFATTN_EINVAL;
  info->ctx_keys_per_block = P->ctx_keys;
  info->ctx_splits = P->S_c;
  info->ctx_row_blocks = P->ctx_row_blocks;
  info->ctx_blocks = P->n_ctx_blocks + P->n_ctx_small_blocks;
  info->dec_keys_per_block = P->dec_keys;
  info->dec_splits = P->S_d * kWaves;
  info->dec_blocks = P->n_dec_blocks;
  info->fused = P->fused;
  info->path = P->path;
  info->workspace_bytes = P->ws_bytes;
  info->ctx_kernel = P->ctx_mode != kCtxLarge ? 0 : 2;
  info->side_stream = P->fork && !P->fused;
  return BIFATTN_OK;
}

namespace {

// One decode step of plan P (a created plan, or the allocation-free entry
// point's plan on the stack, whose workspace is the fixed scratch buffer).
bifattn_status_t decode_impl(bifattn_plan_s* P, const void* q, const void* Kc, const void* Vc,
                             const void* Kd, const void* Vd, const int32_t* decode_lens,
                             const float* k_scale, const float* v_scale, float* out,
                             hipStream_t stream) {
  if (!P || !q || !Kc || !Vc || !out || !on_plan_device(P, stream)) return BIFATTN_EINVAL;
  if (!aligned(k_scale, 4) || !aligned(v_scale, 4)) return BIFATTN_EALIGN;
  const bool has_dec = P->dims.m_d_max > 0;
  if (has_dec && (!Kd || !Vd || !decode_lens)) return BIFATTN_EINVAL;
  if (!aligned(q, 16) || !aligned(Kc, 16) || !aligned(Vc, 16) || !aligned(out, 16))
    return BIFATTN_EALIGN;
  if (has_dec && (!aligned(Kd, 16) || !aligned(Vd, 16) || !aligned(decode_lens, 4)))
    return BIFATTN_EALIGN;
  const int kv = P->dims.kv_type;
  PartialsParams K = base_params(P, q, has_dec ? decode_lens : nullptr, k_scale);
  K.Kc = static_cast<const uint8_t*>(Kc);
  K.Vc = static_cast<const uint8_t*>(Vc);
  K.Kd = static_cast<const uint8_t*>(Kd);
  K.Vd = static_cast<const uint8_t*>(Vd);
  K.dec_rows = P->dims.m_d_max;
  K.len_offset = 0;
  K.ctx_keys = P->ctx_keys;
  K.S_c = P->S_c;
  K.ctx_row_blocks = P->ctx_row_blocks;
  K.ctx_wide = P->ctx_wide;
  K.dec_keys = P->dec_keys;
  K.S_d = P->S_d;
  TimedSection whole(P, BIFATTN_KERNEL_CALL, stream);
  TimedSection part(P, BIFATTN_KERNEL_PARTIALS, stream, true);
  TimedSection ctxs(P, BIFATTN_KERNEL_CONTEXT, stream, true);
  TimedSection decs(P, BIFATTN_KERNEL_DECODE, stream, true);
  auto ev = [](const LaunchEvents& a, const LaunchEvents& b) { return TimedSection::either(a, b); };
  hipError_t e = hipSuccess;
  if (P->path == BIFATTN_PATH_STANDARD) {
    K.out = out;
    K.v_scale = v_scale;
    const LaunchEvents lev = part.both();
    e = launch_standard(K, P->dims.d, kv, P->dec_tiles, stream, last_launch(P, lev));
    part.end();
    whole.end();
    if (lev.stop) mark_done(P, stream);
    return e == hipSuccess ? BIFATTN_OK : BIFATTN_EHIP;
  }
  K.n_ctx_blocks = 0;
  K.n_ctx_small_blocks = 0;
  K.n_dec_blocks = 0;
  // Two launches: the first carries the start event and the second the end
  // event, unless there are no decode work-groups (then the first carries both).
  const bool two = P->n_dec_blocks > 0;
  if (P->ctx_mode == kCtxLarge && P->fused && two) {
    // One launch holds the context and the decode work-groups: each section
    // times it.
    K.n_ctx_blocks = P->n_ctx_blocks;
    K.n_dec_blocks = P->n_dec_blocks;
    e = launch_ctx_large(K, P->dims.d, kv, P->dec_tiles, stream,
                         ev(ev(part.both(), ctxs.both()), decs.both()));
  } else if (P->ctx_mode == kCtxLarge && P->fork && two) {
    // The decode work-groups on the side stream, beside the many-row context
    // kernel; the call's stream waits for them before the combine. The timed
    // section is the call's stream from before the fork to after the join.
    PartialsParams Kd = K;
    Kd.n_dec_blocks = P->n_dec_blocks;
    part.record_start();
    if (hipEventRecord(P->fork_ev, stream) != hipSuccess ||
        hipStreamWaitEvent(P->side, P->fork_ev, 0) != hipSuccess)
      return BIFATTN_EHIP;
    e = launch_partials(Kd, P->dims.d, kv, kCtxNone, P->dec_tiles, P->side, decs.both());
    K.n_ctx_blocks = P->n_ctx_blocks;
    if (e == hipSuccess) e = launch_ctx_large(K, P->dims.d, kv, P->dec_tiles, stream, ctxs.both());
    if (e == hipSuccess && (hipEventRecord(P->join_ev, P->side) != hipSuccess ||
                            hipStreamWaitEvent(stream, P->join_ev, 0) != hipSuccess))
      e = hipErrorUnknown;
    part.record_stop();
    K.n_ctx_blocks = 0;
  } else if (P->ctx_mode == kCtxLarge) {
    // The many-row context kernel, then the decode work-groups.
    K.n_ctx_blocks = P->n_ctx_blocks;
    e = launch_ctx_large(K, P->dims.d, kv, P->dec_tiles, stream,
                         ev(two ? part.first() : part.both(), ctxs.both()));
    K.n_ctx_blocks = 0;
    K.n_dec_blocks = P->n_dec_blocks;
    if (e == hipSuccess && two)
      e = launch_partials(K, P->dims.d, kv, kCtxNone, P->dec_tiles, stream,
                          ev(part.last(), decs.both()));
  } else if (P->fused) {
    // One launch holds the context and the decode work-groups: each section
    // times it.
    K.n_ctx_small_blocks = P->n_ctx_small_blocks;
    K.n_dec_blocks = P->n_dec_blocks;
    e = launch_partials(K, P->dims.d, kv, P->ctx_mode, P->dec_tiles, stream,
                        ev(ev(part.both(), ctxs.both()), decs.both()));
  } else {
    K.n_ctx_small_blocks = P->n_ctx_small_blocks;
    e = launch_partials(K, P->dims.d, kv, P->ctx_mode, P->dec_tiles, stream,
                        ev(two ? part.first() : part.both(), ctxs.both()));
    K.n_ctx_small_blocks = 0;
    K.n_dec_blocks = P->n_dec_blocks;
    if (e == hipSuccess && two)
      e = launch_partials(K, P->dims.d, kv, kCtxNone, P->dec_tiles, stream,
                          ev(part.last(), decs.both()));
  }
  part.end();
  ctxs.end();
  decs.end();
  if (e != hipSuccess) {
    mark_done(P, stream);
    return BIFATTN_EHIP;
  }
  TimedSection comb(P, BIFATTN_KERNEL_COMBINE, stream, true);
  CombineParams C = combine_params(P, has_dec ? decode_lens : nullptr, k_scale, v_scale, out);
  C.S_c = P->S_c;
  C.S_d = P->S_d * kWaves;
  const LaunchEvents cev = comb.both();
  e = launch_combine(C, P->dims.d, stream, last_launch(P, cev));
  comb.end();
  whole.end();
  if (cev.stop) mark_done(P, stream);
  return e == hipSuccess ? BIFATTN_OK : BIFATTN_EHIP;
}

}  // namespace

bifattn_status_t bifattn_decode_scaled(bifattn_plan_t P, const void* q, const void* Kc,
                                       const void* Vc, const void* Kd, const void* Vd,
                                       const int32_t* decode_lens, const float* k_scale,
                                       const float* v_scale, float* out, hipStream_t stream) {
  return decode_impl(P, q, Kc, Vc, Kd, Vd, decode_lens, k_scale, v_scale, out, stream);
}

bifattn_status_t bifattn_decode_noalloc(const bifattn_dims_t* dims, const void* q, const void* Kc,
                                        const void* Vc, const void* Kd, const void* Vd,
                                        const int32_t* decode_lens, const float* k_scale,
                                        const float* v_scale, float* out, hipStream_t stream) {
  bifattn_status_t st = check_dims(dims);
  if (st != BIFATTN_OK) return st;
  // A plan on the stack: the same splits as bifattn_plan_create's (the
  // decode launch always on the call's stream), no events, no streams, no
  // device allocation.
  bifattn_plan_s P;
  P.dims = *dims;
  P.scale = dims->scale != 0.f ? dims->scale : 1.0f / std::sqrt((float)dims->d);
  st = plan_splits(&P, false);
  if (st != BIFATTN_OK) return st;
  WorkspaceLayout L = workspace_layout(&P, false);
  if (L.bytes > kScratchBytes) {
    // Longer chunks leave fewer partials.
    bifattn_plan_s Q;
    Q.dims = P.dims;
    Q.scale = P.scale;
    st = plan_splits(&Q, false, true);
    if (st != BIFATTN_OK) return st;
    const WorkspaceLayout Lq = workspace_layout(&Q, false);
    if (Lq.bytes > kScratchBytes) return BIFATTN_ESCRATCH;
    Q.path = P.path;
    P = Q;
    L = Lq;
  }
  if (hipGetDevice(&P.device) != hipSuccess) {
    (void)hipGetLastError();
    return BIFATTN_EHIP;
  }
  void* scratch = nullptr;
  if (scratch_address(P.device, &scratch) != hipSuccess) {
    (void)hipGetLastError();
    return BIFATTN_EHIP;
  }
  set_workspace(&P, scratch, L);
  st = decode_impl(&P, q, Kc, Vc, Kd, Vd, decode_lens, k_scale, v_scale, out, stream);
  P.ws = nullptr;  // the scratch buffer is not the plan's to free
  return st;
}

bifattn_status_t bifattn_decode(bifattn_plan_t P, const void* q, const void* Kc, const void* Vc,
                                const void* Kd, const void* Vd, const int32_t* decode_lens,
                                float* out, hipStream_t stream) {
  return bifattn_decode_scaled(P, q, Kc, Vc, Kd, Vd, decode_lens, nullptr, nullptr, out, stream);
}

bifattn_status_t bifattn_decode_replicated_scaled(bifattn_plan_t P, const void* q, const void* K_,
                                                  const void* V_, const int32_t* decode_lens,
                                                  const float* k_scale, const float* v_scale,
                                                  float* out, hipStream_t stream) {
  if (!P || !q || !K_ || !V_ || !out || !on_plan_device(P, stream)) return BIFATTN_EINVAL;
  if (!aligned(k_scale, 4) || !aligned(v_scale, 4)) return BIFATTN_EALIGN;
  const bool has_dec = P->dims.m_d_max > 0;
  if (has_dec && !decode_lens) return BIFATTN_EINVAL;
  if (!aligned(q, 16) || !aligned(K_, 16) || !aligned(V_, 16) || !aligned(out, 16))
    return BIFATTN_EALIGN;
  if (has_dec && !aligned(decode_lens, 4)) return BIFATTN_EALIGN;
  PartialsParams K = base_params(P, q, has_dec ? decode_lens : nullptr, k_scale);
  K.Kd = static_cast<const uint8_t*>(K_);
  K.Vd = static_cast<const uint8_t*>(V_);
  K.dec_rows = P->dims.m_c + P->dims.m_d_max;
  K.len_offset = P->dims.m_c;
  K.dec_keys = P->rep_keys;
  K.S_d = P->S_r;
  K.S_c = 0;
  K.n_ctx_blocks = 0;
  K.n_ctx_small_blocks = 0;
  K.n_dec_blocks = P->n_rep_blocks;
  TimedSection whole(P, BIFATTN_KERNEL_CALL, stream);
  TimedSection part(P, BIFATTN_KERNEL_PARTIALS, stream, true);
  hipError_t e = launch_partials(K, P->dims.d, P->dims.kv_type, kCtxNone, P->dec_tiles, stream,
                                 part.both());
  part.end();
  if (e != hipSuccess) {
    mark_done(P, stream);
    return BIFATTN_EHIP;
  }
  TimedSection comb(P, BIFATTN_KERNEL_COMBINE, stream, true);
  CombineParams C = combine_params(P, has_dec ? decode_lens : nullptr, k_scale, v_scale, out);
  C.S_c = 0;
  C.S_d = P->S_r * kWaves;
  const LaunchEvents cev = comb.both();
  e = launch_combine(C, P->dims.d, stream, last_launch(P, cev));
  comb.end();
  whole.end();
  if (cev.stop) mark_done(P, stream);
  return e == hipSuccess ? BIFATTN_OK : BIFATTN_EHIP;
}

bifattn_status_t bifattn_decode_replicated(bifattn_plan_t P, const void* q, const void* K_,
                                           const void* V_, const int32_t* decode_lens, float* out,
                                           hipStream_t stream) {
  return bifattn_decode_replicated_scaled(P, q, K_, V_, decode_lens, nullptr, nullptr, out,
                                          stream);
}

bifattn_status_t bifattn_append_kv(bifattn_plan_t P, const void* k_new, const void* v_new,
                                   void* Kd, void* Vd, int32_t* decode_lens, hipStream_t stream) {
  if (!P || !k_new || !v_new || !Kd || !Vd || !decode_lens || P->dims.m_d_max < 1 ||
      !on_plan_device(P, stream))
    return BIFATTN_EINVAL;
  if (!aligned(k_new, 16) || !aligned(v_new, 16) || !aligned(Kd, 16) || !aligned(Vd, 16) ||
      !aligned(decode_lens, 4))
    return BIFATTN_EALIGN;
  AppendParams A{};
  A.k_new = static_cast<const uint8_t*>(k_new);
  A.v_new = static_cast<const uint8_t*>(v_new);
  A.Kd = static_cast<uint8_t*>(Kd);
  A.Vd = static_cast<uint8_t*>(Vd);
  A.lens = decode_lens;
  A.status = P->status;
  A.b = P->dims.b;
  A.g = P->dims.g;
  A.n = P->ntok;
  A.m_d_max = P->dims.m_d_max;
  const hipError_t e = launch_append(A, P->dims.d, P->dims.kv_type, stream,
                                     last_launch(P, LaunchEvents{}));
  return e == hipSuccess ? BIFATTN_OK : BIFATTN_EHIP;
}

bifattn_status_t bifattn_plan_status(bifattn_plan_t P, hipStream_t stream) {
  if (!P) return BIFATTN_EINVAL;
  if (hipStreamSynchronize(stream) != hipSuccess) return BIFATTN_EHIP;
  int flag = 0;
  if (hipMemcpy(&flag, P->status, sizeof flag, hipMemcpyDeviceToHost) != hipSuccess)
    return BIFATTN_EHIP;
  if (flag) {
    if (hipMemset(P->status, 0, sizeof flag) != hipSuccess) return BIFATTN_EHIP;
    return (flag & kStatusScale) ? BIFATTN_ESCALE : BIFATTN_ELENS;
  }
  return BIFATTN_OK;
}

bifattn_status_t bifattn_plan_set_timing(bifattn_plan_t P, bifattn_kernel_t kernel,
                                         int32_t capacity) {
  if (!P || capacity < 0 || (int)kernel < 0 || (int)kernel > BIFATTN_KERNEL_DECODE)
    return BIFATTN_EINVAL;
  if (!wait_done(P)) return BIFATTN_EHIP;  // the events to be freed may still be pending
  free_events(P);
  if (capacity == 0) return BIFATTN_OK;
  P->events.reserve(2 * (size_t)capacity);
  for (int i = 0; i < 2 * capacity; ++i) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) {
      free_events(P);
      return BIFATTN_ENOMEM;
    }
    P->events.push_back(e);
  }
  P->timed_kernel = (int)kernel;
  P->timing_cap = capacity;
  P->timing_n = 0;
  return BIFATTN_OK;
}

bifattn_status_t bifattn_plan_read_timing(bifattn_plan_t P, int32_t* calls, double* total_ms) {
  if (!P || !calls || !total_ms) return BIFATTN_EINVAL;
  double sum = 0.0;
  for (int k = 0; k < P->timing_n; ++k) {
    if (hipEventSynchronize(P->events[2 * k + 1]) != hipSuccess) return BIFATTN_EHIP;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, P->events[2 * k], P->events[2 * k + 1]) != hipSuccess)
      return BIFATTN_EHIP;
    sum += ms;
  }
  *calls = P->timing_n;
  *total_ms = sum;
  P->timing_n = 0;
  return BIFATTN_OK;
}

}  // extern "C"
