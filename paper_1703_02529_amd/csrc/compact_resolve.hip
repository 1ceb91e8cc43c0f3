// Stream compaction of fired frames and label resolution (gfx950).
//
// Compaction (frames batched for the GPU model, Sec. 7): tiles of 4096 flags.
// A first kernel counts each tile with wave ballots; one workgroup turns the
// counts into exclusive tile offsets (a single scan, linear in the number of
// tiles) and writes the total; a third kernel scans each tile's four waves'
// counts in LDS and writes the ascending indices at the tile's offset with
// ballot + lane-mask popcounts, so the output order is the frame order.  Up to
// kCompactOne flags one workgroup does all of it (k_compact_one).
//
// Resolution (Sec. 5: a frame on which the earlier-frame detector does not
// fire reuses the compared frame's output): frame u copies frame u - delta,
// so the decision of u is that of the last fired frame of its residue chain
// u, u - delta, u - 2 delta, ...; that is a running max of fired indices per
// residue class.  Frames are viewed as rows of `delta` columns, cut into
// tiles of rows: per-tile last fired index per column, an exclusive max-scan
// across tiles per column, and a per-tile sequential walk down each column.
// Up to kResolveOne frames one workgroup does all of it (resolve_block), the
// launch's other workgroups copying the carried sums.
//
// What bounds these steps is their launches: each takes 4 to 5 us of the
// stream however few bytes it touches.
#include "nsc_internal.h"

#include <mutex>

namespace nsc {
namespace {

constexpr int kTile = 4096;   // flags per compaction tile
constexpr int kTileThreads = 256;

__device__ __forceinline__ uint64_t lanemask_lt(int lane) {
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

__global__ void __launch_bounds__(kTileThreads) k_tile_count(const uint8_t* __restrict__ fire,
                                                             int64_t n,
                                                             int32_t* __restrict__ tile_counts) {
  __shared__ int32_t wsum[kTileThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)wave * (kTile / 4);
  int32_t c = 0;
  for (int s = 0; s < kTile / 4 / 64; ++s) {
    const int64_t u = base + s * 64 + lane;
    const bool f = u < n && fire[u] != 0;
    c += __popcll(__ballot(f));
  }
  if (lane == 0) wsum[wave] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t t = 0;
    for (int w = 0; w < kTileThreads / 64; ++w) t += wsum[w];
    tile_counts[blockIdx.x] = t;
  }
}

// Exclusive scan of the tile counts in place (tile offsets) and the total
// into *count; one workgroup walks the tiles 1024 at a time.
constexpr int kScanThreads = 1024;

__global__ void __launch_bounds__(kScanThreads) k_tile_scan(int32_t* __restrict__ tile_counts,
                                                            int64_t tiles,
                                                            int32_t* __restrict__ count) {
  __shared__ int32_t wsum[kScanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int32_t carry = 0;  // the same in every thread
  for (int64_t b0 = 0; b0 < tiles; b0 += kScanThreads) {
    const int64_t b = b0 + tid;
    const int32_t v = b < tiles ? tile_counts[b] : 0;
    int32_t x = v;  // inclusive scan within the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int32_t before = 0, total = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) {
      before += w < wave ? wsum[w] : 0;
      total += wsum[w];
    }
    if (b < tiles) tile_counts[b] = carry + before + x - v;
    carry += total;
    __syncthreads();  // wsum is rewritten by the next round
  }
  if (tid == 0) *count = carry;
}

__global__ void __launch_bounds__(kTileThreads) k_tile_scatter(const uint8_t* __restrict__ fire,
                                                               int64_t n,
                                                               const int32_t* __restrict__ tile_off,
                                                               int32_t* __restrict__ idx) {
  __shared__ int32_t wcount[kTileThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)wave * (kTile / 4);
  // pass 1: this wave's count
  int32_t c = 0;
  for (int st = 0; st < kTile / 4 / 64; ++st) {
    const int64_t u = base + st * 64 + lane;
    c += __popcll(__ballot(u < n && fire[u] != 0));
  }
  if (lane == 0) wcount[wave] = c;
  __syncthreads();
  int64_t off = tile_off[blockIdx.x];
  for (int w = 0; w < wave; ++w) off += wcount[w];
  // pass 2: write ascending indices
  for (int st = 0; st < kTile / 4 / 64; ++st) {
    const int64_t u = base + st * 64 + lane;
    const bool f = u < n && fire[u] != 0;
    const uint64_t m = __ballot(f);
    if (f) idx[off + __popcll(m & lanemask_lt(lane))] = (int32_t)u;
    off += __popcll(m);
  }
}

// The same by one workgroup: a round takes 16 flags per thread (one 16-byte
// load where the flags are aligned), scans the threads' counts and writes
// their indices; nan_out (nullable) is filled with NaN on the way (n floats).
// 4,095 flags: 5 us against 14.5 in three kernels and 4.9 for the fill;
// 65,536: 8 us against 14.2 and 4.7.
constexpr int64_t kCompactOne = 65536;
constexpr int kOneThreads = 1024;

__global__ void __launch_bounds__(kOneThreads) k_compact_one(const uint8_t* __restrict__ fire,
                                                             int64_t n, int32_t* __restrict__ idx,
                                                             int32_t* __restrict__ count,
                                                             float* __restrict__ nan_out) {
  __shared__ int32_t wsum[2][kOneThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool vec = ((uintptr_t)fire & 15) == 0;
  int32_t carry = 0;  // the same in every thread
  int buf = 0;
  for (int64_t b0 = 0; b0 < n; b0 += 16 * kOneThreads, buf ^= 1) {
    const int64_t u0 = b0 + 16 * tid;
    uint32_t m = 0;  // bit b: flag u0 + b
    if (vec && u0 + 16 <= n) {
      const uint4 v = *reinterpret_cast<const uint4*>(fire + u0);
      const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int b = 0; b < 16; ++b) m |= ((w[b >> 2] >> (8 * (b & 3))) & 0xFFu) ? 1u << b : 0u;
    } else {
#pragma unroll
      for (int b = 0; b < 16; ++b)
        if (u0 + b < n) m |= fire[u0 + b] ? 1u << b : 0u;
    }
    const int32_t c = __popc(m);
    int32_t x = c;  // inclusive scan within the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) wsum[buf][wave] = x;
    __syncthreads();  // the other buffer's readers passed the previous round's barrier
    int32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kOneThreads / 64; ++w) {
      before += w < wave ? wsum[buf][w] : 0;
      total += wsum[buf][w];
    }
    int32_t off = carry + before + x - c;
    for (; m; m &= m - 1) idx[off++] = (int32_t)(u0 + __builtin_ctz(m));
    carry += total;
  }
  if (tid == 0) *count = carry;
  if (nan_out)
    for (int64_t i = tid; i < n; i += kOneThreads) nan_out[i] = __builtin_nanf("");
}

__global__ void k_set_i32(int32_t* p, int32_t v) { *p = v; }

// Survivors of one CNN pass: the slots [off, off + m) of the compacted list
// that exist, i.e. clamp(*count - off, 0, m).
__global__ void k_pass_count(const int32_t* __restrict__ count, int64_t off, int64_t m,
                             int32_t* __restrict__ out) {
  const int64_t left = (int64_t)*count - off;
  *out = (int32_t)(left < 0 ? 0 : left < m ? left : m);
}

// Per-tile last fired local index per residue column (or -1).
__global__ void __launch_bounds__(256) k_resolve_tile_last(const uint8_t* __restrict__ fire,
                                                           int64_t n, int32_t delta,
                                                           int32_t rows_per_tile,
                                                           int32_t* __restrict__ tile_last) {
  __shared__ int32_t last[NSC_MAX_DELTA];
  for (int r = threadIdx.x; r < delta; r += blockDim.x) last[r] = -1;
  __syncthreads();
  const int64_t u0 = (int64_t)blockIdx.x * rows_per_tile * delta;
  const int64_t span = (int64_t)rows_per_tile * delta;
  for (int64_t k = threadIdx.x; k < span; k += blockDim.x) {
    const int64_t u = u0 + k;
    if (u < n && fire[u]) atomicMax(&last[(int)(u % delta)], (int32_t)u);
  }
  __syncthreads();
  for (int r = threadIdx.x; r < delta; r += blockDim.x)
    tile_last[(int64_t)blockIdx.x * delta + r] = last[r];
}

// carry[b][r] = max over tiles b' < b of tile_last[b'][r]; one block per column.
__global__ void __launch_bounds__(1024) k_resolve_carry(const int32_t* __restrict__ tile_last,
                                                        int32_t tiles, int32_t delta,
                                                        int32_t* __restrict__ carry) {
  __shared__ int32_t v[1024];
  const int r = blockIdx.x, b = threadIdx.x;
  v[b] = b < tiles ? tile_last[(int64_t)b * delta + r] : -1;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int32_t x = b >= o ? v[b - o] : -1;
    __syncthreads();
    if (x > v[b]) v[b] = x;
    __syncthreads();
  }
  if (b < tiles) carry[(int64_t)b * delta + r] = b > 0 ? v[b - 1] : -1;
}

// Walks each residue column of a tile and writes label / defer.
__global__ void __launch_bounds__(256) k_resolve_apply(const uint8_t* __restrict__ fire,
                                                       const uint8_t* __restrict__ dec,
                                                       const uint8_t* __restrict__ prev_dec,
                                                       int64_t n, int32_t delta,
                                                       int32_t rows_per_tile,
                                                       const int32_t* __restrict__ carry,
                                                       uint8_t* __restrict__ label,
                                                       uint8_t* __restrict__ defer) {
  for (int r = threadIdx.x; r < delta; r += blockDim.x) {
    int32_t cur = carry[(int64_t)blockIdx.x * delta + r];
    const int64_t row0 = (int64_t)blockIdx.x * rows_per_tile;
    for (int q = 0; q < rows_per_tile; ++q) {
      const int64_t u = (row0 + q) * delta + r;
      if (u >= n) break;
      if (fire[u]) cur = (int32_t)u;
      // no fired frame of this chain in the call: continue the carried state
      const uint8_t d = cur >= 0 ? dec[cur] : (prev_dec ? prev_dec[r] : (uint8_t)0);
      label[u] = d & 1;
      defer[u] = (d >> 1) & 1;
    }
  }
}

// Fixed reference image: a frame that does not fire is labelled "no object".
__global__ void __launch_bounds__(256) k_resolve_fixed(const uint8_t* __restrict__ fire,
                                                       const uint8_t* __restrict__ dec, int64_t n,
                                                       uint8_t* __restrict__ label,
                                                       uint8_t* __restrict__ defer) {
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < n;
       u += (int64_t)gridDim.x * blockDim.x) {
    const uint8_t d = fire[u] ? dec[u] : (uint8_t)0;
    label[u] = d & 1;
    defer[u] = (d >> 1) & 1;
  }
}

// State of the last `delta` frames after a call of n frames.  When n < delta
// the old state is read from `old_*` (a copy), otherwise only from this call.
__global__ void __launch_bounds__(256) k_state_update(const int32_t* __restrict__ sums,
                                                      const uint8_t* __restrict__ label,
                                                      const uint8_t* __restrict__ defer, int64_t n,
                                                      int32_t delta, int64_t cells,
                                                      const int32_t* __restrict__ old_sums,
                                                      const uint8_t* __restrict__ old_dec,
                                                      int32_t* __restrict__ st_sums,
                                                      uint8_t* __restrict__ st_dec) {
  const int64_t total = (int64_t)delta * cells;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = e / cells, c = e - k * cells;
    const int64_t src = n - delta + k;  // local index of the frame kept in slot k
    st_sums[e] = src >= 0 ? sums[src * cells + c] : old_sums[(k + n) * cells + c];
    if (c == 0)
      st_dec[k] = src >= 0 ? (uint8_t)(label[src] | (defer[src] << 1)) : old_dec[k + n];
  }
}

// Label resolution of n frames by one workgroup of kOneThreads threads, and
// the carried decisions of the last delta frames (st_dec, nullable).  Chunks of
// up to kResolveChunk frames (whole rows) go through LDS: per frame one byte,
// 4 | decision if it fired and 0 if not, read and written 16 frames at a time.
// Thread (segment, column) finds the last fired decision of its rows of the
// column, a scan over the segments of each column gives every segment its
// carry, and the thread walks its rows again, leaving each frame's decision.
// prev_dec (nullable, may be st_dec) holds the decisions of the delta frames
// before the call; fire holds 0 or 1.
constexpr int64_t kResolveOne = 65536;
constexpr int kResolveChunk = 65536;

struct ResolveShared {
  uint8_t last[2][kOneThreads];
  uint8_t prev[NSC_MAX_DELTA];
};

// Chunk length of a call (frames; LDS bytes rounded up to 16).
inline int resolve_chunk(int64_t n, int32_t delta) {
  const int most = kResolveChunk / delta * delta;
  return n < most ? (int)n : most;
}

__device__ __forceinline__ void resolve_block(const uint8_t* __restrict__ fire,
                                              const uint8_t* __restrict__ dec,
                                              const uint8_t* prev_dec, int64_t n, int32_t delta,
                                              int chunk, uint8_t* __restrict__ label,
                                              uint8_t* __restrict__ defer, uint8_t* st_dec,
                                              ResolveShared& sh, uint8_t* code) {
  const int tid = threadIdx.x;
  const int segs = kOneThreads / delta;
  const int seg = tid / delta, r = tid - seg * delta;
  if (tid < delta) sh.prev[tid] = prev_dec ? prev_dec[tid] : (uint8_t)0;
  const bool vec = (((uintptr_t)fire | (uintptr_t)dec | (uintptr_t)label | (uintptr_t)defer) & 15) == 0;
  for (int64_t c0 = 0; c0 < n; c0 += chunk) {
    const int cn = (int)(n - c0 < chunk ? n - c0 : chunk);
    const bool v16 = vec && (c0 & 15) == 0;
    auto words = [](const uint4& v, int i) { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; };
    for (int i = 16 * tid; i < cn; i += 16 * kOneThreads) {
      if (v16 && i + 16 <= cn) {
        const uint4 f = *reinterpret_cast<const uint4*>(fire + c0 + i);
        const uint4 d = *reinterpret_cast<const uint4*>(dec + c0 + i);
        uint32_t w[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = (words(d, k) & (words(f, k) * 3u)) | (words(f, k) << 2);
        *reinterpret_cast<uint4*>(code + i) = make_uint4(w[0], w[1], w[2], w[3]);
      } else {
        for (int k = i; k < cn && k < i + 16; ++k)
          code[k] = fire[c0 + k] ? (uint8_t)((dec[c0 + k] & 3) | 4) : (uint8_t)0;
      }
    }
    __syncthreads();  // codes and the previous decisions complete
    // rows per segment, odd so that the segments spread over the LDS banks
    const int rps = (((cn + delta - 1) / delta + segs - 1) / segs) | 1;
    const int u0 = seg < segs ? seg * rps * delta + r : cn;
    const int u1 = min(cn, u0 + rps * delta);
    uint8_t cur = 0;
#pragma unroll 4
    for (int u = u0; u < u1; u += delta) cur = code[u] ? code[u] : cur;
    sh.last[0][tid] = cur;
    __syncthreads();
    int b = 0;
    for (int o = 1; o < segs; o <<= 1, b ^= 1) {
      const uint8_t y = sh.last[b][tid];
      const uint8_t x = seg >= o ? sh.last[b][tid - o * delta] : (uint8_t)0;
      sh.last[b ^ 1][tid] = y ? y : x;
      __syncthreads();
    }
    // no fired frame of this chain so far: the decision before the chunk
    const uint8_t before = seg > 0 && seg < segs ? sh.last[b][tid - delta] : (uint8_t)0;
    uint8_t d = before ? before & 3 : sh.prev[r];
#pragma unroll 4
    for (int u = u0; u < u1; u += delta) {
      d = code[u] ? code[u] & 3 : d;
      code[u] = d;
    }
    __syncthreads();  // decisions complete
    for (int i = 16 * tid; i < cn; i += 16 * kOneThreads) {
      if (v16 && i + 16 <= cn) {
        const uint4 v = *reinterpret_cast<const uint4*>(code + i);
        const uint32_t k1 = 0x01010101u;
        *reinterpret_cast<uint4*>(label + c0 + i) = make_uint4(v.x & k1, v.y & k1, v.z & k1, v.w & k1);
        *reinterpret_cast<uint4*>(defer + c0 + i) =
            make_uint4((v.x >> 1) & k1, (v.y >> 1) & k1, (v.z >> 1) & k1, (v.w >> 1) & k1);
      } else {
        for (int k = i; k < cn && k < i + 16; ++k) {
          label[c0 + k] = code[k] & 1;
          defer[c0 + k] = (code[k] >> 1) & 1;
        }
      }
    }
    if (tid < delta && tid < cn) sh.prev[tid] = code[(cn - 1 - tid) / delta * delta + tid];
    __syncthreads();  // read before the next chunk's codes
  }
  // slot k holds frame n - delta + k, of column (n + k) mod delta (of a call
  // shorter than delta, the columns past n still hold the state before it)
  if (st_dec && tid < delta) st_dec[tid] = sh.prev[(n + tid) % delta] & 3;
}

// Copies count int32 by the workgroups of index wg of nwg.
__device__ __forceinline__ void copy_i32(const int32_t* __restrict__ src, int32_t* __restrict__ dst,
                                         int64_t count, int64_t wg, int64_t nwg) {
  const int64_t i0 = wg * blockDim.x + threadIdx.x, step = nwg * blockDim.x;
  if ((((uintptr_t)src | (uintptr_t)dst) & 15) == 0) {
    for (int64_t i = i0; i < count / 4; i += step)
      reinterpret_cast<int4*>(dst)[i] = reinterpret_cast<const int4*>(src)[i];
    if (i0 < (count & 3)) dst[count / 4 * 4 + i0] = src[count / 4 * 4 + i0];
  } else {
    for (int64_t i = i0; i < count; i += step) dst[i] = src[i];
  }
}

// One launch for a call of up to kResolveOne frames: workgroup 0 resolves the
// labels and keeps the decisions, the others copy `count` sums from src to dst
// (the last delta frames' sums into the state; or, for a call shorter than
// delta, the state's sums that stay into the scratch buffer).  4,095 frames,
// delta 30: 6.3 us against 10 to 19 (a busy stream) in four kernels; 65,536:
// 14 us against 18.6 and, with delta 1, 12.4 against 32.
__global__ void __launch_bounds__(kOneThreads) k_resolve_one(
    const uint8_t* __restrict__ fire, const uint8_t* __restrict__ dec, const uint8_t* prev_dec,
    int64_t n, int32_t delta, uint8_t* __restrict__ label, uint8_t* __restrict__ defer,
    uint8_t* st_dec, int chunk, const int32_t* __restrict__ src, int32_t* __restrict__ dst,
    int64_t count) {
  __shared__ ResolveShared sh;
  extern __shared__ __align__(16) uint8_t code[];
  if (blockIdx.x == 0)
    resolve_block(fire, dec, prev_dec, n, delta, chunk, label, defer, st_dec, sh, code);
  else
    copy_i32(src, dst, count, blockIdx.x - 1, gridDim.x - 1);
}

// The state's sums of a call of n < delta frames: the kept part (from the
// scratch buffer), then the call's sums.
__global__ void __launch_bounds__(256) k_state_short(const int32_t* __restrict__ kept,
                                                     int64_t n_kept,
                                                     const int32_t* __restrict__ sums,
                                                     int64_t n_sums, int32_t* __restrict__ st) {
  copy_i32(kept, st, n_kept, blockIdx.x, gridDim.x);
  copy_i32(sums, st + n_kept, n_sums, blockIdx.x, gridDim.x);
}

// Camera group: workgroup (0, c) resolves camera c's n frames (frames c * n ..
// c * n + n - 1 of the batch).  Earlier-frame cameras take the decision of
// the last fired frame of the chain, else the state slot's; fixed-reference
// cameras label non-firing frames 0.  With `sums` (n >= every delta) the
// workgroups (1 .., c) copy the camera's last delta frames' sums into its
// slot and workgroup (0, c) its decisions; without, k_group_state does.
__global__ void __launch_bounds__(kOneThreads) k_group_resolve(
    const CamDiff* __restrict__ cams, const uint8_t* __restrict__ fire,
    const uint8_t* __restrict__ dec, int64_t n, int64_t t0, unsigned char* state,
    int64_t state_stride, uint8_t* __restrict__ label, uint8_t* __restrict__ defer,
    const int32_t* __restrict__ sums, int64_t cells) {
  __shared__ ResolveShared sh;
  extern __shared__ __align__(16) uint8_t code[];
  const int64_t cam = blockIdx.y;
  const CamDiff cd = cams[cam];
  const int64_t base = cam * n;
  if (cd.ref_mode == NSC_REF_FIXED) {
    if (blockIdx.x > 0) return;
    for (int64_t u = threadIdx.x; u < n; u += blockDim.x) {
      const uint8_t d = fire[base + u] ? dec[base + u] : (uint8_t)0;
      label[base + u] = d & 1;
      defer[base + u] = (d >> 1) & 1;
    }
    return;
  }
  unsigned char* slot = state + cam * state_stride;
  if (blockIdx.x == 0) {
    // slot r holds frame t0 - delta + r (frames t < delta always fire, so
    // t0 = 0 never reads it)
    uint8_t* st_dec = slot + cd.dec_off;
    const int most = kResolveChunk / cd.delta * cd.delta;
    resolve_block(fire + base, dec + base, t0 > 0 ? st_dec : nullptr, n, cd.delta,
                  n < most ? (int)n : most, label + base, defer + base, sums ? st_dec : nullptr, sh,
                  code);
  } else {
    copy_i32(sums + (base + n - cd.delta) * cells, reinterpret_cast<int32_t*>(slot),
             cd.delta * cells, blockIdx.x - 1, gridDim.x - 1);
  }
}

// Camera group state after a call of n frames per camera: every earlier-frame
// camera keeps the sums and decisions of its last delta frames in its slot.
// `old` is a copy of the state before the call, read where n < delta.
__global__ void __launch_bounds__(256) k_group_state(const CamDiff* __restrict__ cams,
                                                     const int32_t* __restrict__ sums,
                                                     const uint8_t* __restrict__ label,
                                                     const uint8_t* __restrict__ defer, int64_t n,
                                                     int64_t cells,
                                                     const unsigned char* __restrict__ old,
                                                     unsigned char* __restrict__ state,
                                                     int64_t state_stride) {
  const int64_t cam = blockIdx.y;
  const CamDiff cd = cams[cam];
  if (cd.ref_mode != NSC_REF_PREV) return;
  const int64_t total = (int64_t)cd.delta * cells;
  int32_t* st_sums = reinterpret_cast<int32_t*>(state + cam * state_stride);
  uint8_t* st_dec = state + cam * state_stride + cd.dec_off;
  const int32_t* o_sums = reinterpret_cast<const int32_t*>(old + cam * state_stride);
  const uint8_t* o_dec = old + cam * state_stride + cd.dec_off;
  const int64_t base = cam * n;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = e / cells, c = e - k * cells;
    const int64_t src = n - cd.delta + k;  // local index of the frame kept in slot k
    st_sums[e] = src >= 0 ? sums[(base + src) * cells + c] : o_sums[(k + n) * cells + c];
    if (c == 0)
      st_dec[k] = src >= 0 ? (uint8_t)(label[base + src] | (defer[base + src] << 1))
                           : o_dec[k + n];
  }
}

// Frame skipping (Sec. 5): each frame takes its checked frame's output.
__global__ void __launch_bounds__(256) k_skip_expand(SkipExpand e) {
  for (int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; u < e.n;
       u += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = e.t0 + u;
    const int64_t k = t / e.s;
    const bool checked = k * e.s == t;  // then k >= k0
    uint8_t l, d;
    if (k >= e.k0) {
      l = e.k_label[k - e.k0];
      d = e.k_defer[k - e.k0];
    } else {
      const uint8_t v = *e.last;
      l = v & 1;
      d = (v >> 1) & 1;
    }
    e.label[u] = l;
    e.defer[u] = d;
    if (e.score) e.score[u] = checked ? e.k_score[k - e.k0] : __builtin_nan("");
    if (e.fire) e.fire[u] = checked ? e.k_fire[k - e.k0] : 0;
    if (e.logit) e.logit[u] = checked ? e.k_logit[k - e.k0] : __builtin_nanf("");
  }
}

__global__ void k_skip_last(const uint8_t* __restrict__ label, const uint8_t* __restrict__ defer,
                            int64_t nc, uint8_t* __restrict__ last) {
  if (threadIdx.x == 0) *last = (uint8_t)(label[nc - 1] | (defer[nc - 1] << 1));
}

__global__ void __launch_bounds__(256) k_copy_u8(const uint8_t* __restrict__ s,
                                                 uint8_t* __restrict__ d, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    d[i] = s[i];
}

__global__ void __launch_bounds__(256) k_fill_nan(float* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = __builtin_nanf("");
}

unsigned grid_for(int64_t n, int per_block) {
  int64_t b = (n + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > kNumCU * 16) b = kNumCU * 16;
  return (unsigned)b;
}

}  // namespace

int64_t compact_tiles(int64_t n) { return (n + kTile - 1) / kTile; }

int launch_compact(const uint8_t* fire, int64_t n, int32_t* idx, int32_t* count,
                   int32_t* tile_counts, hipStream_t stream, float* nan_out) {
  if (n <= 0) {
    hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(1), 0, stream, count, 0);
    NSC_CHECK_LAUNCH("k_set_i32");
    return NSC_OK;
  }
  if (n <= kCompactOne) {
    hipLaunchKernelGGL(k_compact_one, dim3(1), dim3(kOneThreads), 0, stream, fire, n, idx, count,
                       nan_out);
    NSC_CHECK_LAUNCH("k_compact_one");
    return NSC_OK;
  }
  if (nan_out) {
    hipLaunchKernelGGL(k_fill_nan, dim3(grid_for(n, 256)), dim3(256), 0, stream, nan_out, n);
    NSC_CHECK_LAUNCH("k_fill_nan");
  }
  const int64_t tiles = compact_tiles(n);
  hipLaunchKernelGGL(k_tile_count, dim3((unsigned)tiles), dim3(kTileThreads), 0, stream, fire, n,
                     tile_counts);
  NSC_CHECK_LAUNCH("k_tile_count");
  hipLaunchKernelGGL(k_tile_scan, dim3(1), dim3(kScanThreads), 0, stream, tile_counts, tiles,
                     count);
  NSC_CHECK_LAUNCH("k_tile_scan");
  hipLaunchKernelGGL(k_tile_scatter, dim3((unsigned)tiles), dim3(kTileThreads), 0, stream, fire, n,
                     tile_counts, idx);
  NSC_CHECK_LAUNCH("k_tile_scatter");
  return NSC_OK;
}

// Compaction without a caller workspace, for callers that cannot allocate:
// the tile offsets live in this file-scope device array (every GPU holds its
// own copy until the process ends), so at most NSC_NOALLOC_MAX_FLAGS flags
// (kNoAllocTiles tiles) per call.  Every call on one GPU shares the array:
// calls that overlap on a GPU race.  Nothing in it has to start at zero
// (each call writes every tile count it reads).
constexpr int64_t kNoAllocTiles = NSC_NOALLOC_MAX_FLAGS / kTile;
static_assert(NSC_NOALLOC_MAX_FLAGS % kTile == 0, "the flag limit is whole tiles");
static __device__ __align__(256) int32_t scratch[kNoAllocTiles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
int32_t* g_scratch[kMaxDevices] = {};
}  // namespace

// Device address of the current device's copy of `scratch`, looked up once per
// device (the array's name in host code is not a device address).
int noalloc_scratch(int32_t** out) {
  int dev = -1;
  NSC_TRY_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices)
    return fail(NSC_E_HIP, "device %d beyond the %d devices the static scratch tracks", dev,
                kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
      return fail(NSC_E_HIP, "hipGetSymbolAddress of the compaction scratch failed on device %d: %s",
                  dev, hipGetErrorString(e));
    g_scratch[dev] = static_cast<int32_t*>(p);
  }
  *out = g_scratch[dev];
  return NSC_OK;
}

int launch_compact_noalloc(const uint8_t* fire, int64_t n, int32_t* idx, int32_t* count,
                           hipStream_t stream) {
  if (compact_tiles(n) > kNoAllocTiles)
    return fail(NSC_E_WORKSPACE, "%lld flags exceed the static scratch's %lld", (long long)n,
                (long long)NSC_NOALLOC_MAX_FLAGS);
  int32_t* tiles = nullptr;
  if (int rc = noalloc_scratch(&tiles)) return rc;
  return launch_compact(fire, n, idx, count, tiles, stream);
}

ResolvePlan make_resolve_plan(int64_t n, int64_t t0, int32_t delta) {
  ResolvePlan p{};
  p.n = n;
  p.t0 = t0;
  p.delta = delta < 1 ? 1 : delta;
  const int64_t rows = (n + p.delta - 1) / p.delta;
  int64_t rpt = (rows + 1023) / 1024;
  if (rpt < 1) rpt = 1;
  p.rows_per_tile = (int32_t)rpt;
  p.tiles = (int32_t)((rows + rpt - 1) / rpt);
  if (p.tiles < 1) p.tiles = 1;
  return p;
}

namespace {
// State of the last `delta` frames after a call of n frames.
int launch_state_update(const int32_t* sums, const uint8_t* label, const uint8_t* defer, int64_t n,
                        int32_t delta, int64_t cells, const StreamState& st, hipStream_t stream) {
  const int32_t* old_sums = st.sums;
  const uint8_t* old_dec = st.dec;
  if (n < delta) {
    // slots k < delta - n keep frames of the previous state: copy it first
    uint8_t* s = static_cast<uint8_t*>(st.scratch);
    const int64_t sb = (int64_t)delta * cells * 4;
    hipLaunchKernelGGL(k_copy_u8, dim3(grid_for(sb, 256)), dim3(256), 0, stream,
                       reinterpret_cast<const uint8_t*>(st.sums), s, sb);
    NSC_CHECK_LAUNCH("k_copy_u8");
    hipLaunchKernelGGL(k_copy_u8, dim3(1), dim3(256), 0, stream, st.dec, s + sb, (int64_t)delta);
    NSC_CHECK_LAUNCH("k_copy_u8");
    old_sums = reinterpret_cast<const int32_t*>(s);
    old_dec = s + sb;
  }
  hipLaunchKernelGGL(k_state_update, dim3(grid_for((int64_t)delta * cells, 256)), dim3(256), 0,
                     stream, sums, label, defer, n, delta, cells, old_sums, old_dec, st.sums,
                     st.dec);
  NSC_CHECK_LAUNCH("k_state_update");
  return NSC_OK;
}
}  // namespace

int launch_resolve(const ResolvePlan& p, int32_t ref_mode, const uint8_t* fire, const uint8_t* dec,
                   int32_t* tile_last, int32_t* carry, uint8_t* label, uint8_t* defer,
                   const int32_t* sums, int64_t cells, const StreamState& st, hipStream_t stream) {
  if (p.n <= 0) return NSC_OK;
  if (ref_mode == NSC_REF_FIXED) {
    hipLaunchKernelGGL(k_resolve_fixed, dim3(grid_for(p.n, 256)), dim3(256), 0, stream, fire, dec,
                       p.n, label, defer);
    NSC_CHECK_LAUNCH("k_resolve_fixed");
    return NSC_OK;
  }
  const uint8_t* prev_dec = p.t0 > 0 ? st.dec : nullptr;
  if (p.n <= kResolveOne) {
    const bool shrt = p.n < p.delta;  // some of the state's frames stay
    const int64_t kept = shrt ? (p.delta - p.n) * cells : 0;
    const int64_t count = shrt ? kept : p.delta * cells;
    const int32_t* src = shrt ? st.sums + p.n * cells : sums + (p.n - p.delta) * cells;
    int32_t* dst = shrt ? static_cast<int32_t*>(st.scratch) : st.sums;
    hipLaunchKernelGGL(k_resolve_one, dim3(1 + grid_for(count, 4 * kOneThreads)),
                       dim3(kOneThreads), (size_t)align_up(resolve_chunk(p.n, p.delta), 16), stream,
                       fire, dec, prev_dec, p.n, p.delta, label, defer, st.dec,
                       resolve_chunk(p.n, p.delta), src, dst, count);
    NSC_CHECK_LAUNCH("k_resolve_one");
    if (shrt) {
      hipLaunchKernelGGL(k_state_short, dim3(grid_for(p.delta * cells, 1024)), dim3(256), 0,
                         stream, (const int32_t*)dst, kept, sums, p.n * cells, st.sums);
      NSC_CHECK_LAUNCH("k_state_short");
    }
    return NSC_OK;
  }
  hipLaunchKernelGGL(k_resolve_tile_last, dim3(p.tiles), dim3(256), 0, stream, fire, p.n, p.delta,
                     p.rows_per_tile, tile_last);
  NSC_CHECK_LAUNCH("k_resolve_tile_last");
  hipLaunchKernelGGL(k_resolve_carry, dim3(p.delta), dim3(1024), 0, stream, tile_last, p.tiles,
                     p.delta, carry);
  NSC_CHECK_LAUNCH("k_resolve_carry");
  hipLaunchKernelGGL(k_resolve_apply, dim3(p.tiles), dim3(256), 0, stream, fire, dec,
                     prev_dec, p.n, p.delta, p.rows_per_tile, carry, label, defer);
  NSC_CHECK_LAUNCH("k_resolve_apply");
  return launch_state_update(sums, label, defer, p.n, p.delta, cells, st, stream);
}

int launch_group_resolve(const CamDiff* cams, int32_t n_cams, int32_t max_delta,
                         const uint8_t* fire, const uint8_t* dec, const int32_t* sums,
                         int64_t cells, int64_t n, int64_t t0, unsigned char* state,
                         int64_t state_stride, void* scratch, uint8_t* label, uint8_t* defer,
                         hipStream_t stream) {
  if (n <= 0 || n_cams <= 0) return NSC_OK;
  // every camera's state comes from this call alone: one launch
  const bool whole = max_delta > 0 && n >= max_delta;
  unsigned gx = 1;
  if (whole) {
    const unsigned all = grid_for((int64_t)max_delta * cells, 4 * kOneThreads);
    const unsigned per = (unsigned)(kNumCU * 16 / n_cams);  // copying workgroups per camera
    gx += per < 1 ? 1 : (all < per ? all : per);
  }
  const size_t lds = align_up(n < kResolveChunk ? (size_t)n : (size_t)kResolveChunk, 16);
  hipLaunchKernelGGL(k_group_resolve, dim3(gx, (unsigned)n_cams), dim3(kOneThreads), lds, stream,
                     cams, fire, dec, n, t0, state, state_stride, label, defer,
                     whole ? sums : nullptr, cells);
  NSC_CHECK_LAUNCH("k_group_resolve");
  if (whole || max_delta <= 0) return NSC_OK;
  // slots k < delta - n of some camera keep frames of the previous state: copy it first
  unsigned char* cp = static_cast<unsigned char*>(scratch);
  const int64_t bytes = (int64_t)n_cams * state_stride;
  hipLaunchKernelGGL(k_copy_u8, dim3(grid_for(bytes, 256)), dim3(256), 0, stream, state, cp, bytes);
  NSC_CHECK_LAUNCH("k_copy_u8");
  hipLaunchKernelGGL(k_group_state, dim3(grid_for((int64_t)max_delta * cells, 256), (unsigned)n_cams),
                     dim3(256), 0, stream, cams, sums, label, defer, n, cells,
                     (const unsigned char*)cp, state, state_stride);
  NSC_CHECK_LAUNCH("k_group_state");
  return NSC_OK;
}

int launch_pass_count(const int32_t* count, int64_t off, int64_t m, int32_t* out,
                      hipStream_t stream) {
  hipLaunchKernelGGL(k_pass_count, dim3(1), dim3(1), 0, stream, count, off, m, out);
  NSC_CHECK_LAUNCH("k_pass_count");
  return NSC_OK;
}

int launch_set_i32(int32_t* p, int32_t v, hipStream_t stream) {
  hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(1), 0, stream, p, v);
  NSC_CHECK_LAUNCH("k_set_i32");
  return NSC_OK;
}

int launch_skip_expand(const SkipExpand& e, hipStream_t stream) {
  if (e.n <= 0) return NSC_OK;
  hipLaunchKernelGGL(k_skip_expand, dim3(grid_for(e.n, 256)), dim3(256), 0, stream, e);
  NSC_CHECK_LAUNCH("k_skip_expand");
  if (e.nc > 0) {  // after every reader of the previous value
    hipLaunchKernelGGL(k_skip_last, dim3(1), dim3(64), 0, stream, e.k_label, e.k_defer, e.nc,
                       e.last);
    NSC_CHECK_LAUNCH("k_skip_last");
  }
  return NSC_OK;
}

int launch_copy_u8(const uint8_t* src, uint8_t* dst, int64_t n, hipStream_t stream) {
  if (n <= 0) return NSC_OK;
  hipLaunchKernelGGL(k_copy_u8, dim3(grid_for(n, 256)), dim3(256), 0, stream, src, dst, n);
  NSC_CHECK_LAUNCH("k_copy_u8");
  return NSC_OK;
}

}  // namespace nsc
