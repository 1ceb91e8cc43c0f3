// Threshold search of the cost-based optimizer (Sec. 6.3, step 3) with its
// cost model (Sec. 6.2), on logged per-frame scores: for each candidate
// delta_diff, the detector's errors on the frames that do not fire, the
// c_low / c_high that keep the combined false negative / positive rates below
// FN* / FP*, and the expected cost per frame
//   f_s T_MSE + f_s f_m T_SNN + f_s f_m f_c T_FullNN   (f_s = 1).
//
// One 1024-thread workgroup per candidate.  The paper sorts the fired frames
// by confidence and walks the list; here each threshold is found by exact
// counting over the bit patterns of the fp32 confidences (which order like the
// values for confidences in [0, 1]), 11, 10 and 9 bits at a time:  c_low is
// the smallest confidence v with
//   fn_dd + #{fired, label 1, conf <= v} >= FN* x (frames with the object)
// (1 if none), c_high the largest v with
//   fp_dd + #{fired, label 0, conf >= v} >= FP* x (frames without it)
// (0 if none), raised to c_low.  Frames below c_low are labelled 0, above
// c_high 1, the others defer and get the reference label.  A frame that does
// not fire takes the reference label of the frame it is compared with (frame
// t - delta, or "no object" for a fixed reference image).  Counts are exact;
// the fp64 rates and the cost are evaluated in a fixed operation order with
// contraction off.
#include "nsc_internal.h"

#include <math.h>

namespace nsc {
namespace {

constexpr int kSweepThreads = 1024;
constexpr uint32_t kOneBits = 0x3F800000u;  // 1.0f

struct SweepArgs {
  const double* score;
  const float* conf;
  const uint8_t* truth;
  int64_t n;
  const double* deltas;
  int32_t n_t;
  int32_t ref_mode, delta;
  double fp_target, fn_target, t_mse, t_snn, t_full;
  nsc_sweep_row* rows;
  int32_t* best;
};

// Workgroup sum of two 64-bit counts (every thread gets the totals).
__device__ __forceinline__ void wg_sum2(int64_t& a, int64_t& b, int64_t* red) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();  // the previous use of red is finished
  if (lane == 0) {
    red[2 * wave] = a;
    red[2 * wave + 1] = b;
  }
  __syncthreads();
  a = b = 0;
  for (int w = 0; w < kSweepThreads / 64; ++w) {
    a += red[2 * w];
    b += red[2 * w + 1];
  }
}

__device__ __forceinline__ bool fires(double s, double d) {
  return s == INFINITY || s > d;
}

// Bits of the three counting levels (confidences up to 1.0f have 30 bits).
constexpr int kShift1 = 19, kShift2 = 9;
constexpr int kBins1 = 2048, kBins2 = 1024, kBins3 = 512;
// Frames per thread and step, and the LDS bytes a workgroup may keep of the
// frames' classes (one byte per step and thread).
constexpr int kPer = 4;
constexpr int64_t kClassBytes = 96 * 1024;

// Adds one to h[bin] for every valid lane.  Confidences pile up near 0 and 1,
// so the lanes that share the first valid lane's bin are added by that lane
// at once; the others add on their own.
__device__ __forceinline__ void hist_add(uint32_t* h, int bin, bool valid) {
  const uint64_t m = __ballot(valid);
  if (m == 0) return;
  const int lead = __builtin_ctzll(m);
  const int b0 = __builtin_amdgcn_readlane(bin, lead);
  const uint64_t same = __ballot(valid && bin == b0);
  if ((int)(threadIdx.x & 63) == lead)
    atomicAdd(&h[b0], (uint32_t)__popcll(same));
  else if (valid && bin != b0)
    atomicAdd(&h[bin], 1u);
}

// The first of nb bins, walked up (or, DOWN, from the last bin down), at
// which base plus the bins' running count reaches the budget, and the count
// before it; -1 if none does.  nb <= 2 x kSweepThreads, even.
template <bool DOWN>
__device__ __forceinline__ int find_bin(const uint32_t* h, int nb, int64_t base, double budget,
                                        int64_t* before, int64_t* red) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = 2 * tid, i1 = 2 * tid + 1;
  auto at = [&](int i) -> int64_t { return i < nb ? (int64_t)h[DOWN ? nb - 1 - i : i] : 0; };
  const int64_t c0 = at(i0), c1 = at(i1);
  int64_t x = c0 + c1;  // inclusive scan within the wave
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  __syncthreads();  // the previous use of red is finished
  if (lane == 63) red[wave] = x;
  if (tid == 0) red[kSweepThreads / 64] = -1;
  __syncthreads();
  int64_t pre = x - c0 - c1;
  for (int w = 0; w < wave; ++w) pre += red[w];
  auto reached = [&](int64_t c) { return (double)(base + c) >= budget; };
  const bool p0 = reached(pre + c0), p1 = reached(pre + c0 + c1);
  const bool mine = i0 < nb && p1 && (tid == 0 || !reached(pre));
  if (mine) {
    const int i = p0 ? i0 : i1;
    red[kSweepThreads / 64] = DOWN ? nb - 1 - i : i;
    red[kSweepThreads / 64 + 1] = p0 ? pre : pre + c0;
  }
  __syncthreads();
  *before = red[kSweepThreads / 64 + 1];
  return (int)red[kSweepThreads / 64];
}

// What bounds it: a workgroup reads the whole log through one CU (13 bytes per
// frame at about 64 bytes per clock: 8 us for 100,000 frames), so the log is
// read once: that pass counts the errors, fills the first histogram and keeps
// each frame's class (fired with label 1 / 0) in LDS, and the later passes
// read only the confidences of steps with a fired frame.  100,000 frames, 64
// candidates: 110 us per search against 1,860 for a binary search of up
// to 60 counting passes over the log per candidate.
// VEC: score, conf and truth allow 16-, 16- and 4-byte loads of 4 frames.
template <bool VEC>
__global__ void __launch_bounds__(kSweepThreads) k_sweep(SweepArgs a, int32_t keep) {
#pragma clang fp contract(off)
  __shared__ int64_t red[2 * kSweepThreads / 64];
  __shared__ uint32_t hist[2 * kBins1];  // label 0, then label 1
  extern __shared__ uint8_t cls_lds[];   // keep: [step][thread]
  const int k = blockIdx.x, tid = threadIdx.x;
  const double d = a.deltas[k];
  const int64_t steps = (a.n + kPer * kSweepThreads - 1) / (kPer * kSweepThreads);
  const bool prev = a.ref_mode == NSC_REF_PREV;
  auto frame0 = [&](int64_t s) { return (s * kSweepThreads + tid) * kPer; };
  auto clear = [&]() {
    __syncthreads();  // every reader of the histogram is done
    for (int i = tid; i < 2 * kBins1; i += kSweepThreads) hist[i] = 0;
    __syncthreads();
  };
  auto key_of = [](float c) { return __float_as_uint(c + 0.0f); };  // -0 counts as +0

  // Labels (one byte per frame) and fired flags (bit e) of a step's frames.
  struct Step {
    uint32_t y, fired, in;  // in: bit e set for frames below n
  };
  auto load_step = [&](int64_t s) {
    const int64_t t = frame0(s);
    Step r{0, 0, 0};
    if (VEC && t + kPer <= a.n) {
      const double2 s0 = *reinterpret_cast<const double2*>(a.score + t);
      const double2 s1 = *reinterpret_cast<const double2*>(a.score + t + 2);
      const uint32_t y = *reinterpret_cast<const uint32_t*>(a.truth + t);
      r.fired = (fires(s0.x, d) ? 1u : 0u) | (fires(s0.y, d) ? 2u : 0u) |
                (fires(s1.x, d) ? 4u : 0u) | (fires(s1.y, d) ? 8u : 0u);
      r.y = ((y & 0xFFu) ? 1u : 0u) | ((y & 0xFF00u) ? 2u : 0u) | ((y & 0xFF0000u) ? 4u : 0u) |
            ((y & 0xFF000000u) ? 8u : 0u);
      r.in = 15u;
      return r;
    }
#pragma unroll
    for (int e = 0; e < kPer; ++e)
      if (t + e < a.n) {
        r.in |= 1u << e;
        r.y |= a.truth[t + e] ? 1u << e : 0u;
        r.fired |= fires(a.score[t + e], d) ? 1u << e : 0u;
      }
    return r;
  };
  auto load_conf = [&](int64_t t, uint32_t want, float (&c)[kPer]) {
    if (VEC && t + kPer <= a.n) {
      const float4 v = *reinterpret_cast<const float4*>(a.conf + t);
      c[0] = v.x;
      c[1] = v.y;
      c[2] = v.z;
      c[3] = v.w;
      return;
    }
#pragma unroll
    for (int e = 0; e < kPer; ++e) c[e] = (want >> e) & 1u ? a.conf[t + e] : 0.0f;
  };
  // Fired frames of a step: bits 0-3 with label 1, bits 4-7 with label 0.
  auto class_of = [](const Step& r) { return (r.fired & r.y) | ((r.fired & ~r.y) << 4); };
  auto step_class = [&](int64_t s) -> uint32_t {
    return keep ? cls_lds[s * kSweepThreads + tid] : class_of(load_step(s));
  };

  // frames with the object, fired frames and the detector's errors; the
  // first histogram
  clear();
  int64_t pos = 0, fired = 0, fn_dd = 0, fp_dd = 0;
  for (int64_t s = 0; s < steps; ++s) {
    const int64_t t = frame0(s);
    const Step r = load_step(s);
    uint32_t ref = 0;
    if (prev) {
      if (t >= a.delta && t + kPer <= a.n) {
        uint32_t y;
        __builtin_memcpy(&y, a.truth + (t - a.delta), 4);
        ref = ((y & 0xFFu) ? 1u : 0u) | ((y & 0xFF00u) ? 2u : 0u) |
              ((y & 0xFF0000u) ? 4u : 0u) | ((y & 0xFF000000u) ? 8u : 0u);
      } else {
#pragma unroll
        for (int e = 0; e < kPer; ++e)
          if (t + e >= a.delta && t + e < a.n) ref |= a.truth[t + e - a.delta] ? 1u << e : 0u;
      }
    }
    const uint32_t quiet = r.in & ~r.fired;
    pos += __popc(r.y);
    fired += __popc(r.fired);
    fn_dd += __popc(quiet & r.y & ~ref);
    fp_dd += __popc(quiet & ~r.y & ref);
    if (keep) cls_lds[s * kSweepThreads + tid] = (uint8_t)class_of(r);
    float c[kPer];
    load_conf(t, r.fired, c);
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const uint32_t u = key_of(c[e]);
      const bool ok = ((r.fired >> e) & 1u) && u <= kOneBits;
      hist_add(hist, ok ? (int)(((r.y >> e) & 1u) * kBins1 + (u >> kShift1)) : 0, ok);
    }
  }
  wg_sum2(pos, fired, red);
  wg_sum2(fn_dd, fp_dd, red);  // its barriers also complete the histogram
  const int64_t neg = a.n - pos;
  const double fn_budget = pos ? a.fn_target * (double)pos : INFINITY;
  const double fp_budget = neg ? a.fp_target * (double)neg : INFINITY;
  const bool feasible = (double)fn_dd < fn_budget && (double)fp_dd < fp_budget;

  double c_low = 0.0, c_high = 1.0;
  if (feasible) {  // uniform
    // c_low: the smallest u with fn_dd + #{label 1, bits <= u} >= budget;
    // c_high: the largest u with fp_dd + #{label 0, bits >= u} >= budget;
    // each level narrows both to one bin
    int64_t below = 0, above = 0, part = 0;
    int lo = find_bin<false>(hist + kBins1, kBins1, fn_dd, fn_budget, &part, red);
    below = part;
    int hi = find_bin<true>(hist, kBins1, fp_dd, fp_budget, &part, red);
    above = part;
    c_low = 1.0;
    c_high = 0.0;
    const bool has_lo = lo >= 0, has_hi = hi >= 0;
    if (has_lo || has_hi) {
      // level 2 (bits 18..9), then level 3 (bits 8..0) of the chosen bins
      for (int level = 2; level <= 3; ++level) {
        const int up = level == 2 ? kShift1 : kShift2, down = level == 2 ? kShift2 : 0;
        const int nb = level == 2 ? kBins2 : kBins3;
        clear();
        for (int64_t s = 0; s < steps; ++s) {
          const uint32_t cl = step_class(s);
          if (__ballot(cl != 0) == 0) continue;
          const int64_t t = frame0(s);
          float c[kPer] = {0.f, 0.f, 0.f, 0.f};
          if (cl) load_conf(t, cl | (cl >> 4), c);
#pragma unroll
          for (int e = 0; e < kPer; ++e) {
            const uint32_t u = key_of(c[e]);
            const bool one = (cl >> e) & 1u, zero = (cl >> (4 + e)) & 1u;
            const bool ok = u <= kOneBits && ((one && has_lo && (int)(u >> up) == lo) ||
                                              (zero && has_hi && (int)(u >> up) == hi));
            hist_add(hist, ok ? (one ? kBins1 : 0) + (int)((u >> down) & (uint32_t)(nb - 1)) : 0,
                     ok);
          }
        }
        __syncthreads();
        if (has_lo) {
          const int b = find_bin<false>(hist + kBins1, nb, fn_dd + below, fn_budget, &part, red);
          below += part;
          lo = lo * nb + b;
        }
        if (has_hi) {
          const int b = find_bin<true>(hist, nb, fp_dd + above, fp_budget, &part, red);
          above += part;
          hi = hi * nb + b;
        }
      }
      if (has_lo) c_low = (double)__uint_as_float((uint32_t)lo);
      if (has_hi) c_high = (double)__uint_as_float((uint32_t)hi);
    }
    if (c_high < c_low) c_high = c_low;
  }
  // the decisions these thresholds give
  int64_t fn_cnn = 0, fp_cnn = 0, deferred = 0, unused = 0;
  for (int64_t s = 0; s < steps; ++s) {
    const uint32_t cl = step_class(s);
    if (!cl) continue;
    float c[kPer];
    load_conf(frame0(s), cl | (cl >> 4), c);
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const bool one = (cl >> e) & 1u, zero = (cl >> (4 + e)) & 1u;
      if (!one && !zero) continue;
      const double v = (double)c[e];
      if (v < c_low)
        fn_cnn += one;
      else if (v > c_high)
        fp_cnn += zero;
      else
        ++deferred;
    }
  }
  wg_sum2(fn_cnn, fp_cnn, red);
  wg_sum2(deferred, unused, red);
  if (threadIdx.x == 0) {
    nsc_sweep_row r{};
    r.delta = d;
    r.c_low = c_low;
    r.c_high = c_high;
    r.fired = fired;
    r.deferred = deferred;
    r.fn_dd = fn_dd;
    r.fp_dd = fp_dd;
    r.fn_cnn = fn_cnn;
    r.fp_cnn = fp_cnn;
    r.positives = pos;
    r.negatives = neg;
    r.feasible = feasible ? 1 : 0;
    r.f_m = (double)fired / (double)a.n;
    r.f_c = fired ? (double)deferred / (double)fired : 0.0;
    r.cost = a.t_mse + r.f_m * a.t_snn + (r.f_m * r.f_c) * a.t_full;
    a.rows[k] = r;
  }
}

// The cheapest feasible candidate (the first on ties), or -1.
__global__ void __launch_bounds__(64) k_sweep_best(const nsc_sweep_row* rows, int32_t n_t,
                                                    int32_t* best) {
  int32_t bi = -1;
  double bc = 0.0;
  for (int k = threadIdx.x; k < n_t; k += 64) {
    if (rows[k].feasible && (bi < 0 || rows[k].cost < bc)) {
      bi = k;
      bc = rows[k].cost;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const int32_t oi = __shfl_xor(bi, o, 64);
    const double oc = __shfl_xor(bc, o, 64);
    if (oi >= 0 && (bi < 0 || oc < bc || (oc == bc && oi < bi))) {
      bi = oi;
      bc = oc;
    }
  }
  if (threadIdx.x == 0) *best = bi;
}

}  // namespace
}  // namespace nsc

extern "C" int nsc_threshold_sweep(const nsc_sweep_cfg* cfg, const double* score, const float* conf,
                                   const uint8_t* truth, int64_t n, const double* deltas,
                                   int32_t n_t, nsc_sweep_row* rows, int32_t* best, void* stream) {
  using namespace nsc;
  if (!cfg || !score || !conf || !truth || !deltas || !rows || !best)
    return fail(NSC_E_INVAL, "a pointer argument is NULL");
  if (n < 1 || n > 0x7FFFFFFF) return fail(NSC_E_INVAL, "frame count %lld out of range", (long long)n);
  if (n_t < 1 || n_t > NSC_MAX_SWEEP)
    return fail(NSC_E_INVAL, "%d candidate thresholds outside 1..%d", n_t, NSC_MAX_SWEEP);
  if (cfg->ref_mode != NSC_REF_PREV && cfg->ref_mode != NSC_REF_FIXED)
    return fail(NSC_E_INVAL, "ref_mode %d is neither NSC_REF_PREV nor NSC_REF_FIXED", cfg->ref_mode);
  if (cfg->ref_mode == NSC_REF_PREV && (cfg->delta < 1 || cfg->delta > NSC_MAX_DELTA))
    return fail(NSC_E_INVAL, "delta %d outside 1..%d", cfg->delta, NSC_MAX_DELTA);
  if (!(cfg->fp_target >= 0.0 && cfg->fp_target <= 1.0 && cfg->fn_target >= 0.0 &&
        cfg->fn_target <= 1.0))
    return fail(NSC_E_INVAL, "targets must lie in [0, 1]");
  if (!(cfg->t_mse >= 0.0 && cfg->t_snn >= 0.0 && cfg->t_full >= 0.0 && isfinite(cfg->t_mse) &&
        isfinite(cfg->t_snn) && isfinite(cfg->t_full)))
    return fail(NSC_E_INVAL, "costs must be finite and non-negative");
  SweepArgs a{};
  a.score = score;
  a.conf = conf;
  a.truth = truth;
  a.n = n;
  a.deltas = deltas;
  a.n_t = n_t;
  a.ref_mode = cfg->ref_mode;
  a.delta = cfg->delta;
  a.fp_target = cfg->fp_target;
  a.fn_target = cfg->fn_target;
  a.t_mse = cfg->t_mse;
  a.t_snn = cfg->t_snn;
  a.t_full = cfg->t_full;
  a.rows = rows;
  a.best = best;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the frames' classes stay in LDS when they fit (up to 393,216 frames);
  // longer logs work them out again from the scores in every pass
  const int64_t cls = (n + kPer * kSweepThreads - 1) / (kPer * kSweepThreads) * kSweepThreads;
  const int32_t keep = cls <= kClassBytes ? 1 : 0;
  const size_t lds = keep ? (size_t)cls : 0;
  const bool vec = ((uintptr_t)score & 15) == 0 && ((uintptr_t)conf & 15) == 0 &&
                   ((uintptr_t)truth & 3) == 0;
  if (vec)
    hipLaunchKernelGGL(k_sweep<true>, dim3((unsigned)n_t), dim3(kSweepThreads), lds, st, a, keep);
  else
    hipLaunchKernelGGL(k_sweep<false>, dim3((unsigned)n_t), dim3(kSweepThreads), lds, st, a, keep);
  NSC_CHECK_LAUNCH("k_sweep");
  hipLaunchKernelGGL(k_sweep_best, dim3(1), dim3(64), 0, st, rows, n_t, best);
  NSC_CHECK_LAUNCH("k_sweep_best");
  return NSC_OK;
}
