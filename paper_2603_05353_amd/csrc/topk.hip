// Stage 3 -- Eq. (8): the k context tokens with the largest scores, k = floor(rho N).
//
// The score vector is small (128 KiB at 32K context), so the stage is bound by
// launch latency and dependent steps, not by bandwidth.  Up to 8192 scores run as
// ONE workgroup in ONE launch: the scores are turned into order-preserving
// 32-bit keys, bit-transposed into per-thread bit planes held in registers,
// and the k-th largest key is found by a radix descent of two bits per step
// whose counting is a handful of AND + popcount operations per thread.  There
// are no atomics, so the cost does not depend on how the scores are
// distributed (near-uniform attention puts almost every score into the same
// high-order digits, the worst case for histogram-based selection).
//
// Ties are resolved towards the smaller index and the result is emitted in
// ascending index order by a block-wide prefix sum over (greater, tie) counts.
//
// Up to 131072 scores take two launches of many workgroups (select_bracket_kernel, select_emit_kernel), longer vectors the
// radix select of six short launches.
#include <algorithm>
#include <mutex>

#include "ifkv_device.h"
#include "ifkv_internal.h"

namespace ifkv {

namespace {

// Monotone map float -> uint32: larger float <=> larger key; -0 and +0 coincide.
// Every real (non-NaN) score maps to a key > 0, so key 0 can pad the tail.
__device__ __forceinline__ uint32_t score_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Sum within each row of 16 lanes (data-parallel primitives; every lane of a
// row ends up with the row total).
__device__ __forceinline__ int row16_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
  v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
  v += __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, true);  // row_ror:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, true);  // row_ror:8
  return v;
}
__device__ __forceinline__ int wave64_sum(int v) {
  v = row16_sum(v);
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) +
         __builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
}

// Inclusive prefix sum over the lanes of a wavefront: within the rows of 16, then the rows' last lanes.
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
  int v = static_cast<int>(x);
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2 and 3
  return static_cast<uint32_t>(v);
}
// Largest value of a wavefront.
__device__ __forceinline__ uint32_t wave_largest(uint32_t v) {
  v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0xB1, 0xF, 0xF, true)));
  v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x4E, 0xF, 0xF, true)));
  v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x124, 0xF, 0xF, true)));
  v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), 0x128, 0xF, 0xF, true)));
  auto row = [&](int l) __attribute__((always_inline)) { return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v), l)); };
  return max(max(row(0), row(16)), max(row(32), row(48)));
}

// In-register 32x32 bit-matrix transpose: afterwards word b, bit i == bit b of
// the original word i.
__device__ __forceinline__ void transpose32(uint32_t (&a)[32]) {
  // blocks of 16 and of 8 bits are whole bytes: one byte permute per result
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const uint32_t x = a[k], y = a[k + 16];
    a[k] = __builtin_amdgcn_perm(y, x, 0x05040100u);       // low halves of x, y
    a[k + 16] = __builtin_amdgcn_perm(y, x, 0x07060302u);  // high halves
  }
#pragma unroll
  for (int k = 0; k < 32; k = (k + 9) & ~8) {
    const uint32_t x = a[k], y = a[k + 8];
    a[k] = __builtin_amdgcn_perm(y, x, 0x06020400u);      // even bytes of x, y
    a[k + 8] = __builtin_amdgcn_perm(y, x, 0x07030501u);  // odd bytes
  }
  uint32_t m = 0x0F0F0F0Fu;
#pragma unroll
  for (int j = 4; j != 0; j >>= 1) {
#pragma unroll
    for (int k = 0; k < 32; k = (k + j + 1) & ~j) {
      const uint32_t x = a[k], y = a[k + j];
      a[k] = (x & m) | ((y << j) & ~m);
      a[k + j] = ((x >> j) & m) | (y & ~m);
    }
    m ^= m << (j >> 1);
  }
}

// THREADS x WORDS x 32 keys held in registers as bit planes.
template <int THREADS, int WORDS>
__global__ __launch_bounds__(THREADS) void topk_resident_kernel(const float *__restrict__ scores, int n, int k,
                                                                int32_t *__restrict__ idx_out) {
  constexpr int NW = THREADS / 64;
  // Thread t owns keys 32 t .. 32 t + 31 of a word.  They are loaded with coalesced 16-byte reads (all
  // of a thread's eight requests are issued before anything waits: one memory latency for the whole
  // vector), handed over through LDS (33 words per owner: conflict-free both ways) in one round with
  // one barrier, and transposed into bit planes.
  __shared__ uint32_t stage[THREADS * 33];
  __shared__ uint32_t red[2][16][2];
  __shared__ uint32_t wave_tot[16];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const bool vec_ok = (reinterpret_cast<uintptr_t>(scores) & 15u) == 0;

  uint32_t plane[WORDS][32];
#pragma unroll
  for (int w = 0; w < WORDS; ++w) {
    const int base = w * THREADS * 32;
    float4 f[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int gi = base + (i * THREADS + tid) * 4;
      f[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (vec_ok && gi + 3 < n) {
        f[i] = *reinterpret_cast<const float4 *>(scores + gi);
      } else {
        if (gi < n) f[i].x = scores[gi];
        if (gi + 1 < n) f[i].y = scores[gi + 1];
        if (gi + 2 < n) f[i].z = scores[gi + 2];
        if (gi + 3 < n) f[i].w = scores[gi + 3];
      }
    }
    if (w > 0) __syncthreads();  // the previous word's keys have been taken out of the stage
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = (i * THREADS + tid) * 4;
      const int gi = base + e;
      uint32_t *dst = stage + e + (e >> 5);
      // key 0 pads the tail: every real score maps to a key > 0
      dst[0] = gi < n ? score_key(f[i].x) : 0u;
      dst[1] = gi + 1 < n ? score_key(f[i].y) : 0u;
      dst[2] = gi + 2 < n ? score_key(f[i].z) : 0u;
      dst[3] = gi + 3 < n ? score_key(f[i].w) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 32; ++i) plane[w][i] = stage[tid * 33 + i];
    transpose32(plane[w]);
  }

  // ---- radix descent, two bits per step ------------------------------------
  uint32_t alive[WORDS], greater[WORDS];
#pragma unroll
  for (int w = 0; w < WORDS; ++w) {
    alive[w] = 0xFFFFFFFFu;
    greater[w] = 0u;
  }
  int need = k, left = THREADS * WORDS * 32;  // keys wanted of those alive, keys alive
#pragma unroll
  for (int step = 0; step < 16; ++step) {
    // All that are alive are taken, whatever their remaining bits: with distinct scores that is so after some 20 bits (32768
    // scores spread over a factor of two or more, 15 %: 16.75 -> 13.95 us, 8000: 11.4 -> 8.9; where all lie within some per
    // cent the leading bits are shared and it takes the last steps to tell the scores apart: no gain).  Looked at four times,
    // late, because a check costs a step some 0.1 us (at every step: 15.0, and ties, which never end early, 18.2 -> 20.4 instead
    // of 18.1).
    if (step >= 8 && (step & 1) == 0 && need == left) break;
    const int hi = 31 - 2 * step;
    const int lo = hi - 1;
    int c3 = 0, c2 = 0, c1 = 0;
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
      const uint32_t ah = alive[w] & plane[w][hi];
      const uint32_t pl = plane[w][lo];
      c3 += __popc(ah & pl);
      c2 += __popc(ah & ~pl);
      c1 += __popc(alive[w] & ~plane[w][hi] & pl);
    }
    // per-thread counts <= 32*WORDS, per-wave totals < 2^16: c3 and c2 share a word
    const int w32 = wave64_sum(c3 | (c2 << 16));
    const int w1 = wave64_sum(c1);
    const int p = step & 1;
    if (lane == 0) {
      red[p][wave][0] = static_cast<uint32_t>(w32);
      red[p][wave][1] = static_cast<uint32_t>(w1);
    }
    __syncthreads();
    int t3 = 0, t2 = 0, t1 = 0;
    if (lane < NW) {
      const uint32_t a = red[p][lane][0];
      t3 = static_cast<int>(a & 0xFFFFu);
      t2 = static_cast<int>(a >> 16);
      t1 = static_cast<int>(red[p][lane][1]);
    }
    t3 = __builtin_amdgcn_readlane(row16_sum(t3), 0);
    t2 = __builtin_amdgcn_readlane(row16_sum(t2), 0);
    t1 = __builtin_amdgcn_readlane(row16_sum(t1), 0);

    int digit;
    if (need <= t3) {
      digit = 3;
      left = t3;
    } else if (need <= t3 + t2) {
      digit = 2;
      need -= t3;
      left = t2;
    } else if (need <= t3 + t2 + t1) {
      digit = 1;
      need -= t3 + t2;
      left = t1;
    } else {
      digit = 0;
      need -= t3 + t2 + t1;
      left -= t3 + t2 + t1;
    }
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
      const uint32_t ph = plane[w][hi], pl = plane[w][lo], a = alive[w];
      if (digit == 3) {
        alive[w] = a & ph & pl;
      } else if (digit == 2) {
        greater[w] |= a & ph & pl;
        alive[w] = a & ph & ~pl;
      } else if (digit == 1) {
        greater[w] |= a & ph;
        alive[w] = a & ~ph & pl;
      } else {
        greater[w] |= a & (ph | pl);
        alive[w] = a & ~ph & ~pl;
      }
    }
  }
  // alive = keys equal to the k-th largest; `need` of them (lowest indices) are taken.

  // ---- ordered compaction ----------------------------------------------------
  int carry_g = 0, carry_t = 0;
#pragma unroll
  for (int w = 0; w < WORDS; ++w) {
    const int g = __popc(greater[w]);
    const int t = __popc(alive[w]);
    // greater count in the low half, tie count in the high half; block totals
    // are <= 32768 each, so unsigned sums never carry between the halves
    const uint32_t v = static_cast<uint32_t>(g) | (static_cast<uint32_t>(t) << 16);
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    __syncthreads();  // wave_tot reuse
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t wave_before = 0, block_total = 0;
#pragma unroll
    for (int x = 0; x < NW; ++x) {
      const uint32_t wt = wave_tot[x];
      if (x < wave) wave_before += wt;
      block_total += wt;
    }
    const uint32_t excl = wave_before + incl - v;
    const int g_before = carry_g + static_cast<int>(excl & 0xFFFFu);
    int t_seen = carry_t + static_cast<int>(excl >> 16);
    int pos = g_before + min(t_seen, need);
    const int base_index = (w * THREADS + tid) * 32;
    const uint32_t gm = greater[w];
    uint32_t m = gm | alive[w];
    while (m) {
      const int i = __ffs(m) - 1;
      m &= m - 1;
      bool take = (gm >> i) & 1u;
      if (!take) take = (t_seen++ < need);
      if (take) {
        if (pos < k) idx_out[pos] = base_index + i;  // pos < k always holds; the guard keeps a logic slip in bounds
        ++pos;
      }
    }
    carry_g += static_cast<int>(block_total & 0xFFFFu);
    carry_t += static_cast<int>(block_total >> 16);
  }
}

// ---------------------------------------------------------------------------
// Score vectors of more than kPickMax: radix select over many workgroups.
// The key's 32 bits are resolved in three digits (11 + 11 + 10 bits).  Pass p counts, per digit
// value, the keys that match the prefix found so far (LDS histogram per workgroup, then one global
// atomic add per non-empty bin: integer counts, so the result does not depend on the order).  The next
// kernel starts by locating the digit that holds the k-th largest key in that histogram (every
// workgroup does this small scan for itself, which saves a launch per pass; one of them leaves the
// result for the kernel after it).  After the third digit the threshold key T is exact, and
// the last kernel writes the indices in ascending order, taking ties by ascending index.
//
// Bound by launches and dependent steps: the scores (520 KB at 130K context) sit in the L2s.  Six launches of 2.5 to 5
// us: 300K scores 25 us, 1M 38; 1M 64.4 when one thread scanned the 256 partial sums of each histogram (10 us a scan, and
// every kernel scanned all the histograms before it).
// ---------------------------------------------------------------------------
constexpr int kSelThreads = 256;
constexpr int kSelPer = 8;                        // keys per thread
constexpr int kSelChunk = kSelThreads * kSelPer;  // keys per workgroup of the histogram passes
constexpr int kSelBins = 2048;
constexpr int kWriteThreads = 1024;
constexpr int kWritePer = 4;                            // consecutive keys per thread
constexpr int kWriteChunk = kWriteThreads * kWritePer;  // keys per workgroup of the last two kernels

struct SelectFound {  // digits found by the kernels before: prefix of the threshold key, remaining rank
  uint32_t prefix;
  int need;
};
struct SelectState {  // lives in scratch
  uint32_t hist[3][kSelBins];
  SelectFound found[3];  // found[p]: after p + 1 digits
};
__device__ __forceinline__ int digit_shift(int pass) { return pass == 0 ? 21 : (pass == 1 ? 10 : 0); }
__device__ __forceinline__ uint32_t digit_mask(int pass) { return pass == 2 ? 0x3FFu : 0x7FFu; }

// After `passes` digits: prefix of the threshold key and the remaining rank (1 = the largest of those that match).  The
// last of these digits is located here, in the histogram of the pass before, by all threads of a workgroup of
// THREADS; the ones before it come from the state.  `publish`: this workgroup leaves the result in the state.
// `red` holds THREADS / 64 + 2 words.
template <int THREADS>
__device__ __forceinline__ SelectFound locate(SelectState *__restrict__ st, int passes, int k, bool publish, uint32_t *red) {
  SelectFound f = {0u, k};
  if (passes == 0) return f;
  const int pass = passes - 1;
  if (pass > 0) f = st->found[pass - 1];
  constexpr int PER = kSelBins / THREADS;  // consecutive bins per thread, thread 0 the highest digits
  const uint32_t *hist = st->hist[pass];
  const int top = pass == 2 ? kSelBins / 2 : kSelBins;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  uint32_t c[PER], mine = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int bin = top - 1 - (tid * PER + e);
    c[e] = bin >= 0 ? hist[bin] : 0u;
    mine += c[e];
  }
  const uint32_t incl = wave_scan(mine);
  if (lane == 63) red[wave] = incl;
  __syncthreads();
  uint32_t before = incl - mine;  // keys in digits above this thread's bins
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w)
    if (w < wave) before += red[w];
  const uint32_t need = static_cast<uint32_t>(f.need);
  if (before < need && need <= before + mine) {  // exactly one thread
    uint32_t acc = before;
    int e = 0;
    while (need > acc + c[e]) acc += c[e++];
    red[THREADS / 64] = static_cast<uint32_t>(top - 1 - (tid * PER + e));
    red[THREADS / 64 + 1] = need - acc;
  }
  __syncthreads();
  f.prefix |= red[THREADS / 64] << digit_shift(pass);
  f.need = static_cast<int>(red[THREADS / 64 + 1]);
  if (publish && tid == 0) st->found[pass] = f;
  return f;
}

// Four consecutive scores from index i on (a multiple of 4); zeros past the end.
__device__ __forceinline__ float4 load4(const float *__restrict__ scores, int i, int n, bool vec_ok) {
  if (vec_ok && i + 3 < n) return *reinterpret_cast<const float4 *>(scores + i);
  float4 f = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < n) f.x = scores[i];
  if (i + 1 < n) f.y = scores[i + 1];
  if (i + 2 < n) f.z = scores[i + 2];
  if (i + 3 < n) f.w = scores[i + 3];
  return f;
}

__global__ __launch_bounds__(kSelThreads) void select_hist_kernel(const float *__restrict__ scores, int n, int k,
                                                                  int pass, SelectState *__restrict__ st) {
  __shared__ uint32_t lh[kSelBins];
  __shared__ uint32_t red[kSelThreads / 64 + 2];
  const bool vec_ok = (reinterpret_cast<uintptr_t>(scores) & 15u) == 0;
  const int base = blockIdx.x * kSelChunk + 4 * threadIdx.x;
  float4 f[kSelPer / 4];
#pragma unroll
  for (int u = 0; u < kSelPer / 4; ++u) f[u] = load4(scores, base + u * 4 * kSelThreads, n, vec_ok);
#pragma unroll
  for (int b = 0; b < kSelBins / kSelThreads; ++b) lh[b * kSelThreads + threadIdx.x] = 0u;
  const uint32_t prefix = locate<kSelThreads>(st, pass, k, blockIdx.x == 0, red).prefix;
  const uint32_t hi_mask = pass == 0 ? 0u : (pass == 1 ? 0xFFE00000u : 0xFFFFFC00u);
  const int sh = digit_shift(pass);
  const uint32_t dm = digit_mask(pass);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kSelPer / 4; ++u) {
    const float v[4] = {f[u].x, f[u].y, f[u].z, f[u].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t key = score_key(v[e]), digit = (key >> sh) & dm;
      const bool counts = base + u * 4 * kSelThreads + e < n && (key & hi_mask) == prefix;
      // near-uniform attention puts the high digits of most scores into one bin: one add for the whole wavefront then
      const unsigned long long take = __ballot(counts);
      if (take == 0ull) continue;
      const uint32_t d0 = __builtin_amdgcn_readlane(digit, __builtin_ctzll(take));
      if (__ballot(counts && digit != d0) == 0ull) {
        if ((threadIdx.x & 63) == 0) atomicAdd(&lh[d0], static_cast<uint32_t>(__popcll(take)));
      } else if (counts) {
        atomicAdd(&lh[digit], 1u);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int b = 0; b < kSelBins / kSelThreads; ++b) {
    const uint32_t v = lh[b * kSelThreads + threadIdx.x];
    if (v != 0u) atomicAdd(&st->hist[pass][b * kSelThreads + threadIdx.x], v);
  }
}

// Sums of a packed pair of counts over a workgroup of kWriteThreads; every thread gets them.  `red`: 2 words per wavefront.
__device__ __forceinline__ uint2 block_sum2(uint32_t a, uint32_t b, uint32_t (*red)[2]) {
  a = static_cast<uint32_t>(wave64_sum(static_cast<int>(a)));
  b = static_cast<uint32_t>(wave64_sum(static_cast<int>(b)));
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = a;
    red[threadIdx.x >> 6][1] = b;
  }
  __syncthreads();
  uint2 s = make_uint2(0u, 0u);
#pragma unroll
  for (int w = 0; w < kWriteThreads / 64; ++w) {
    s.x += red[w][0];
    s.y += red[w][1];
  }
  return s;
}

// Per chunk of the write kernel: how many keys are above the threshold and how many equal it.
__global__ __launch_bounds__(kWriteThreads) void select_count_kernel(const float *__restrict__ scores, int n, int k,
                                                                     SelectState *__restrict__ st,
                                                                     uint2 *__restrict__ block_counts) {
  __shared__ uint32_t red[kWriteThreads / 64 + 2];
  __shared__ uint32_t sums[kWriteThreads / 64][2];
  const bool vec_ok = (reinterpret_cast<uintptr_t>(scores) & 15u) == 0;
  const int i = blockIdx.x * kWriteChunk + 4 * threadIdx.x;
  const float4 f = load4(scores, i, n, vec_ok);
  const uint32_t T = locate<kWriteThreads>(st, 3, k, false, red).prefix;
  const float v[4] = {f.x, f.y, f.z, f.w};
  uint32_t g = 0, t = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t key = score_key(v[e]);
    g += i + e < n && key > T;
    t += i + e < n && key == T;
  }
  const uint2 s = block_sum2(g, t, sums);
  if (threadIdx.x == 0) block_counts[blockIdx.x] = s;
}

// Ordered output.  Thread t of workgroup b owns keys [b * kWriteChunk + 4 t, + 4): a contiguous run, so ascending index
// order is (workgroup, thread, element).  (Counting again here what the workgroups before this one take, from the scores,
// instead of in a launch of its own: 15.8 us for this kernel at 130K scores against 8 for the two, the last workgroup
// reads all of them.)
__global__ __launch_bounds__(kWriteThreads) void select_write_kernel(const float *__restrict__ scores, int n, int k,
                                                                     SelectState *__restrict__ st,
                                                                     const uint2 *__restrict__ block_counts,
                                                                     int32_t *__restrict__ idx_out) {
  __shared__ uint32_t red[kWriteThreads / 64 + 2];
  __shared__ uint32_t sums[kWriteThreads / 64][2];
  __shared__ uint32_t wave_tot[kWriteThreads / 64];
  const bool vec_ok = (reinterpret_cast<uintptr_t>(scores) & 15u) == 0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int base = blockIdx.x * kWriteChunk + 4 * tid;
  const float4 f = load4(scores, base, n, vec_ok);
  const SelectFound found = locate<kWriteThreads>(st, 3, k, false, red);
  const uint32_t T = found.prefix;
  uint32_t g_before = 0, t_before = 0;
  for (int b = tid; b < static_cast<int>(blockIdx.x); b += kWriteThreads) {
    const uint2 c = block_counts[b];
    g_before += c.x;
    t_before += c.y;
  }
  const uint2 before = block_sum2(g_before, t_before, sums);
  const float v[4] = {f.x, f.y, f.z, f.w};
  uint32_t gm = 0, tm = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t key = score_key(v[e]);
    gm |= (base + e < n && key > T ? 1u : 0u) << e;
    tm |= (base + e < n && key == T ? 1u : 0u) << e;
  }
  // (greater, tie) counts packed in one word: a workgroup holds 4096 keys, so 16 bits each suffice
  const uint32_t mine = static_cast<uint32_t>(__popc(gm)) | (static_cast<uint32_t>(__popc(tm)) << 16);
  const uint32_t incl = wave_scan(mine);
  if (lane == 63) wave_tot[wave] = incl;
  __syncthreads();
  uint32_t excl = incl - mine;
#pragma unroll
  for (int x = 0; x < kWriteThreads / 64; ++x)
    if (x < wave) excl += wave_tot[x];
  int t_seen = static_cast<int>(before.y + (excl >> 16));
  int pos = static_cast<int>(before.x + (excl & 0xFFFFu)) + min(t_seen, found.need);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    bool take = (gm >> e) & 1u;
    if ((tm >> e) & 1u) take = t_seen++ < found.need;
    if (take) {
      if (pos < k) idx_out[pos] = base + e;  // pos < k always holds; the guard keeps a logic slip in bounds
      ++pos;
    }
  }
}

// ---------------------------------------------------------------------------
// Up to kPickMax scores: two launches.  The first one brackets the threshold key from a sample of the scores, counts the
// keys above the bracket and lists those inside it (some 5 %), per workgroup; the second one finds the threshold among
// the listed keys, every workgroup for itself, and writes its own chunk's indices.  The bracket only decides how many keys
// are listed, never the result: if the threshold lies outside, or the bracket holds many equal or nearly equal keys, the
// second launch reads more keys (all scores, if need be) and takes longer.
//
// Bound by launches and dependent steps: per launch two memory latencies and about seven barriers, and in the second one
// the vector work of every workgroup on all listed keys (32K scores 5.6 + 6.3 us, 130K 6.2 + 7.8).  15 % of n scores that lie within
// some per cent / spread over a factor of two, before -> now (one workgroup up to 32768, the radix select from there on):
// 8193 15.5 / 12.5 -> 10.8 / 11.1 us, 20000 16.1 / 13.6 -> 11.5 / 11.2, 32768 16.9 / 14.2 -> 11.9 / 11.7, 65536 22.9 / 22.6 -> 12.2 / 12.4,
// 130078 23.7 / 23.0 -> 14.3 / 14.0, in repeated calls; a first call on new scores, everything cold, takes 110 to 145 us with the
// host's part, before as now.  Slower than before, of 18 kinds of scores at six sizes: heavy tails (log-normal, deviation 4), 2 % of
// 12000 and 20000 10.5 -> 11.0 and 10.8 -> 11.3, 15 % of 32768 11.5 -> 11.8 (the descent of the one workgroup ends early there); 32768
// ascending or descending scores 14.2 -> 14.5 and 14.0 -> 14.9; 131072 of 64 different values 24.2 -> 24.9.  Below 8193 one workgroup
// takes 9 to 11 us; above kPickMax the
// second launch grows with the number of listed keys, and ties make it slower than the radix select (262144 scores of 64
// values 26 -> 34 us).
// ---------------------------------------------------------------------------
constexpr int kPickThreads = 1024;
constexpr int kPickWaves = kPickThreads / 64;
constexpr int kPickChunk = 4 * kPickThreads;  // scores per workgroup, four consecutive ones per thread
constexpr int kPickBlocks = 32;
constexpr int64_t kPickMax = int64_t(kPickBlocks) * kPickChunk;
constexpr int kPickSample = 4 * kPickThreads;

struct PickHeader {  // lives in scratch, in front of the listed keys (kPickChunk places per workgroup)
  uint32_t lo, hi;              // the bracket
  uint2 counts[kPickBlocks];    // keys above it, keys listed
};

// Counts the keys among x (four per lane, those of a place in `valid`) that lie in lo .. hi into bins of 2^sh: one add where
// all of a wavefront share the bin (near-uniform attention, ties).
__device__ __forceinline__ void add_to_bins(uint32_t *hist, const v4u &x, uint32_t valid, uint32_t lo, uint32_t hi, int sh) {
  uint32_t bin[4];
  bool same = true, counts[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    counts[e] = ((valid >> e) & 1u) != 0u && x[e] - lo <= hi - lo;
    bin[e] = (x[e] - lo) >> sh;
  }
  const unsigned long long take = __ballot(counts[0]);
  const uint32_t b0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(bin[0]), take == 0ull ? 0 : __builtin_ctzll(take)));
#pragma unroll
  for (int e = 0; e < 4; ++e) same &= !counts[e] || bin[e] == b0;
  if (take != 0ull && __all(same)) {
    const int total = __popcll(take) + __popcll(__ballot(counts[1])) + __popcll(__ballot(counts[2])) + __popcll(__ballot(counts[3]));
    if ((threadIdx.x & 63) == 0) atomicAdd(&hist[b0], static_cast<uint32_t>(total));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (counts[e]) atomicAdd(&hist[bin[e]], 1u);
  }
}

// The same for the sample, where one add per lane costs most: of all scores it takes those of the crowded bins as well (many zeros, or a
// few scores far above the rest).  Those that share the bin of the wavefront's first one are counted by one add: 90 % zeros, 2 % selected,
// 32768 scores 14.7 -> 11.9 us, one score far above 32767 near-uniform ones 15.1 -> 14.1, others 0.1 us more.  (In the second launch, whose keys come from the bracket, that is 1 to 3 % of the stage slower.)
__device__ __forceinline__ void add_sample_to_bins(uint32_t *hist, const uint32_t (&x)[4], uint32_t lo, uint32_t hi, int sh) {
  const unsigned long long take = __ballot(x[0] - lo <= hi - lo);
  const uint32_t b0 = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>((x[0] - lo) >> sh), take == 0ull ? 0 : __builtin_ctzll(take)));
  int total = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t bin = (x[e] - lo) >> sh;
    const bool counts = x[e] - lo <= hi - lo, shared = take != 0ull && counts && bin == b0;
    total += __popcll(__ballot(shared));
    if (counts && !shared) atomicAdd(&hist[bin], 1u);
  }
  if (take != 0ull && (threadIdx.x & 63) == 0) atomicAdd(&hist[b0], static_cast<uint32_t>(total));
}

// bins of 2^shift keys, at most kSelBins of them, cover lo .. hi
__device__ __forceinline__ int bin_shift(uint32_t lo, uint32_t hi) {
  return lo == hi ? 0 : max(0, 32 - __builtin_clz(hi - lo) - 11);
}

struct RankBin {
  uint32_t bin, above, in;  // keys in the bins above, keys in it
};
// The bins that hold the keys of N ranks (1 = the largest), by all threads of a workgroup; a rank of 0 or less, or beyond
// the last key, comes back as it went in.  `red`: kPickWaves words.
template <int N>
__device__ __forceinline__ void rank_bins(const uint32_t *hist, const int (&rank)[N], RankBin (&out)[N], uint32_t *red, RankBin *found) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t c0 = hist[kSelBins - 1 - 2 * tid], c1 = hist[kSelBins - 2 - 2 * tid];
  const uint32_t incl = wave_scan(c0 + c1);
  if (lane == 63) red[wave] = incl;
  __syncthreads();
  uint32_t before = incl - c0 - c1;
#pragma unroll
  for (int w = 0; w < kPickWaves; ++w)
    if (w < wave) before += red[w];
#pragma unroll
  for (int x = 0; x < N; ++x) {
    const int r = rank[x] - static_cast<int>(before);
    if (r >= 1 && r <= static_cast<int>(c0 + c1)) {  // at most one thread
      const bool first = r <= static_cast<int>(c0);
      found[x] = {static_cast<uint32_t>(kSelBins - (first ? 1 : 2) - 2 * tid), before + (first ? 0u : c0), first ? c0 : c1};
    }
  }
  __syncthreads();
#pragma unroll
  for (int x = 0; x < N; ++x) out[x] = found[x];
}

__global__ __launch_bounds__(kPickThreads) void select_bracket_kernel(const float *__restrict__ scores, int n, int k,
                                                                      PickHeader *__restrict__ header, uint32_t *__restrict__ listed) {
  __shared__ uint32_t hist[kSelBins];
  __shared__ uint32_t red[kPickWaves], red_lo[kPickWaves], red_hi[kPickWaves], red_out[kPickWaves];
  __shared__ RankBin found[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool vec_ok = (reinterpret_cast<uintptr_t>(scores) & 15u) == 0;
  const int base = blockIdx.x * kPickChunk + 4 * tid;
  const float4 f = load4(scores, base, n, vec_ok);
  hist[tid] = hist[tid + kPickThreads] = 0u;
  uint32_t sample[4], lo = ~0u, hi = 0u;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    // one of every n / kPickSample scores, at a place in its stretch that follows no period (golden ratio)
    const uint32_t x = u * kPickThreads + tid, jitter = x * 2654435769u;
    sample[u] = score_key(scores[(static_cast<uint64_t>(x) << 32 | jitter) * static_cast<uint64_t>(n) / kPickSample >> 32]);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    lo = min(lo, sample[u]);
    hi = max(hi, sample[u]);
  }
  lo = ~wave_largest(~lo);
  hi = wave_largest(hi);
  if (lane == 0) {
    red_lo[wave] = lo;
    red_hi[wave] = hi;
  }
  // Ranks in the sample between which the k-th key lies: its expected rank -+ 4.5 standard deviations of a random sample.
  const float expected = static_cast<float>(k) * kPickSample / n;
  const float margin = 4.5f * sqrtf(fmaxf(expected * (1.f - expected / kPickSample), 0.f)) + 2.f;
  const int r_hi = static_cast<int>(floorf(expected - margin)), r_lo = static_cast<int>(ceilf(expected + margin));
  const uint32_t enough = static_cast<uint32_t>(4.f * margin) + 64u;
  uint32_t above = 0u, inside = kPickSample;  // sample keys above hi, in lo .. hi
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kPickWaves; ++w) {
    lo = min(lo, red_lo[w]);
    hi = max(hi, red_hi[w]);
  }
  // narrowed up to three times: a few keys far away from the rest leave all of these in one bin
  for (int pass = 0; pass < 3 && lo != hi && inside > enough; ++pass) {
    const int sh = bin_shift(lo, hi);
    if (pass > 0) {
      hist[tid] = hist[tid + kPickThreads] = 0u;
      __syncthreads();
    }
    add_sample_to_bins(hist, sample, lo, hi, sh);
    __syncthreads();
    const int rank[2] = {r_hi - static_cast<int>(above), r_lo - static_cast<int>(above)};
    RankBin at[2];
    rank_bins(hist, rank, at, red, found);
    const bool cut_hi = rank[0] >= 1, cut_lo = rank[1] <= static_cast<int>(inside);
    const uint32_t end = cut_lo ? at[1].above + at[1].in : inside, start = cut_hi ? at[0].above : 0u;
    const uint32_t lo_hi = lo + (at[0].bin << sh);  // (sums that could pass 2^32 are not formed)
    if (cut_lo) lo += at[1].bin << sh;
    if (cut_hi) hi = lo_hi + min(hi - lo_hi, (1u << sh) - 1u);
    above += start;
    inside = end - start;
  }
  if (r_hi < 1) hi = ~0u;
  if (r_lo > kPickSample) lo = 0u;
  const float v[4] = {f.x, f.y, f.z, f.w};
  uint32_t key[4], gt = 0u, in = 0u;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    key[e] = score_key(v[e]);
    const bool valid = base + e < n;
    gt += valid && key[e] > hi;
    in |= (valid && key[e] >= lo && key[e] <= hi ? 1u : 0u) << e;
  }
  const uint32_t mine = gt | static_cast<uint32_t>(__popc(in)) << 16;  // a workgroup holds 4096 keys: 16 bits each
  const uint32_t incl = wave_scan(mine);
  if (lane == 63) red_out[wave] = incl;
  __syncthreads();
  uint32_t before = 0u, total = 0u;
#pragma unroll
  for (int w = 0; w < kPickWaves; ++w) {
    if (w < wave) before += red_out[w];
    total += red_out[w];
  }
  uint32_t at = (before + incl - mine) >> 16;
  uint32_t *out = listed + static_cast<int64_t>(blockIdx.x) * kPickChunk;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if ((in >> e) & 1u) out[at++] = key[e];
  if (tid == 0) {
    header->counts[blockIdx.x] = make_uint2(total & 0xFFFFu, total >> 16);
    if (blockIdx.x == 0) {
      header->lo = lo;
      header->hi = hi;
    }
  }
}

// The listed keys are read in segments of 256 (four consecutive ones per lane), dealt out to the wavefronts in turn whatever
// chunk they come from.  A wavefront stages four segments at a time in LDS and loops over them there: the code is small (it
// is fetched anew in every launch), the loads of four segments are in flight together, and where no wavefront has more
// than four, they are read only once.
__global__ __launch_bounds__(kPickThreads) void select_emit_kernel(const float *__restrict__ scores, int n, int k,
                                                                   const PickHeader *__restrict__ header,
                                                                   const uint32_t *__restrict__ listed, int32_t *__restrict__ idx_out) {
  constexpr int kSegment = 256, kStaged = 4;
  constexpr int kFew = 64;  // keys that a wavefront ranks by comparing all pairs
  __shared__ v4u stage[kPickWaves][kStaged][64];
  __shared__ uint32_t hist[kSelBins];
  __shared__ uint32_t red[kPickWaves], few[kFew], few_chunk[kFew], n_few;
  __shared__ RankBin found[1];
  __shared__ uint2 taken[kPickBlocks];  // per chunk: listed keys above the threshold, keys equal to it
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = gridDim.x;
  const bool vec_ok = (reinterpret_cast<uintptr_t>(scores) & 15u) == 0;
  const int base = blockIdx.x * kPickChunk + 4 * tid;
  const uint2 c = lane < nb ? header->counts[lane] : make_uint2(0u, 0u);
  uint32_t lo = header->lo, hi = header->hi;
  // where every chunk lists at most a segment, as a rule, these are the wavefront's segments
  v4u ahead[kStaged];
#pragma unroll
  for (int u = 0; u < kStaged; ++u)
    ahead[u] = *reinterpret_cast<const v4u *>(listed + static_cast<int64_t>(min(wave + u * kPickWaves, nb - 1)) * kPickChunk + 4 * lane);
  const float4 f = load4(scores, base, n, vec_ok);
  if (tid < kPickBlocks) taken[tid] = make_uint2(0u, 0u);
  hist[tid] = hist[tid + kPickThreads] = 0u;
  if (tid == 0) {
    n_few = 0u;
    found[0] = {0u, 0u, 0u};
  }
  __syncthreads();
  const int above = wave64_sum(static_cast<int>(c.x)), inside = wave64_sum(static_cast<int>(c.y));
  int rank = k - above;  // of the threshold among the keys in lo .. hi
  const bool all = rank < 1 || rank > inside;  // it is not among the listed ones: look at the scores themselves
  if (rank < 1) {
    lo = hi + 1u;
    hi = ~0u;
    rank = k;
  } else if (rank > inside) {
    rank -= inside;
    hi = lo - 1u;
    lo = 0u;
  }
  // lane b: keys to look at in chunk b, and in how many segments they and those before them come
  const int keys = all ? max(min(kPickChunk, n - lane * kPickChunk), 0) : static_cast<int>(c.y);
  const int segments = static_cast<int>(wave_scan((keys + kSegment - 1) / kSegment));
  const int n_segments = __builtin_amdgcn_readlane(segments, 63);
  const bool once = n_segments <= kPickWaves * kStaged;
  bool staged = __all(segments == min(lane + 1, nb)) && !all;
  if (staged) {
#pragma unroll
    for (int u = 0; u < kStaged; ++u) stage[wave][u][lane] = ahead[u];
  }
  // f(chunk, keys, which of them count) for this wavefront's segments among the first `end`
  auto visit = [&](int end, auto f) __attribute__((always_inline)) {
    for (int s0 = wave; s0 < end; s0 += kPickWaves * kStaged) {
      if (!(once && staged)) {
        v4u x[kStaged];
#pragma unroll
        for (int u = 0; u < kStaged; ++u) {
          const int s = min(s0 + u * kPickWaves, n_segments - 1), b = __popcll(__ballot(segments <= s));
          const int first = b == 0 ? 0 : __builtin_amdgcn_readlane(segments, b - 1);
          const int i = (s - first) * kSegment + 4 * lane;
          if (!all) {
            x[u] = *reinterpret_cast<const v4u *>(listed + static_cast<int64_t>(b) * kPickChunk + i);  // (past the list: whatever is there, not used)
          } else {
            const float4 y = load4(scores, b * kPickChunk + i, n, vec_ok);
            x[u] = v4u{score_key(y.x), score_key(y.y), score_key(y.z), score_key(y.w)};
          }
        }
#pragma unroll
        for (int u = 0; u < kStaged; ++u) stage[wave][u][lane] = x[u];
        staged = true;
      }
#pragma unroll 1
      for (int u = 0; u < kStaged; ++u) {
        const int s = s0 + u * kPickWaves;
        if (s >= end) break;
        const int b = __popcll(__ballot(segments <= s));
        const int left = __builtin_amdgcn_readlane(keys, b) - (s - (b == 0 ? 0 : __builtin_amdgcn_readlane(segments, b - 1))) * kSegment;
        const v4u x = stage[wave][u][lane];
        f(b, x, (1u << min(max(left - 4 * lane, 0), 4)) - 1u);
      }
    }
  };
  uint32_t T = lo;
  int need = rank;  // keys equal to the threshold that are taken
  const bool one_value = lo == hi && !all;  // every listed key equals the threshold
  bool counted = false;                     // `taken` is complete
  while (lo != hi) {  // at most three times
    const int sh = bin_shift(lo, hi);
    visit(n_segments, [&](int, const v4u &x, uint32_t valid) __attribute__((always_inline)) { add_to_bins(hist, x, valid, lo, hi, sh); });
    __syncthreads();
    const int ranks[1] = {rank};
    RankBin at[1];
    rank_bins(hist, ranks, at, red, found);
    lo += at[0].bin << sh;
    hi = lo + min(hi - lo, (1u << sh) - 1u);
    rank -= static_cast<int>(at[0].above);
    T = lo;
    need = rank;
    if (sh == 0) break;
    if (at[0].in <= kFew) {
      // those in the bin, and how many lie above it in every chunk
      visit(n_segments, [&](int b, const v4u &x, uint32_t valid) __attribute__((always_inline)) {
        int g = 0;
        bool in[4], any = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool is = ((valid >> e) & 1u) != 0u;
          g += __popcll(__ballot(is && x[e] > hi));
          in[e] = is && x[e] - lo <= hi - lo;
          any |= in[e];
        }
        if (lane == 0 && g != 0) atomicAdd(&taken[b].x, static_cast<uint32_t>(g));
        if (any) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (in[e]) {
              const uint32_t p = atomicAdd(&n_few, 1u);
              if (p < kFew) {
                few[p] = x[e];
                few_chunk[p] = static_cast<uint32_t>(b);
              }
            }
        }
      });
      __syncthreads();
      const int m = min(static_cast<int>(n_few), kFew);
      const uint32_t mine = lane < m ? few[lane] : 0u;
      int gt = 0, eq = 0;
#pragma unroll 1
      for (int j = 0; j < m; ++j) {
        const uint32_t x = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mine), j));
        gt += x > mine;
        eq += x == mine;
      }
      const unsigned long long is = __ballot(lane < m && gt < rank && rank <= gt + eq);
      const int l = is == 0ull ? 0 : __builtin_ctzll(is);
      T = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mine), l));
      need = rank - __builtin_amdgcn_readlane(gt, l);
      if (wave == 0 && lane < m) {
        if (mine > T) atomicAdd(&taken[few_chunk[lane]].x, 1u);
        if (mine == T) atomicAdd(&taken[few_chunk[lane]].y, 1u);
      }
      counted = true;
      break;
    }
    hist[tid] = hist[tid + kPickThreads] = 0u;  // (all have read it: rank_bins ends with a barrier)
    __syncthreads();
  }
  // what the chunks before this one take
  if (one_value) {
    if (tid < kPickBlocks) taken[tid].y = c.y;
  } else if (!counted) {
    const int end = blockIdx.x == 0 ? 0 : __builtin_amdgcn_readlane(segments, static_cast<int>(blockIdx.x) - 1);
    visit(end, [&](int b, const v4u &x, uint32_t valid) __attribute__((always_inline)) {
      int g = 0, t = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        g += __popcll(__ballot(((valid >> e) & 1u) != 0u && x[e] > T));
        t += __popcll(__ballot(((valid >> e) & 1u) != 0u && x[e] == T));
      }
      if (lane == 0 && g != 0) atomicAdd(&taken[b].x, static_cast<uint32_t>(g));
      if (lane == 0 && t != 0) atomicAdd(&taken[b].y, static_cast<uint32_t>(t));
    });
  }
  const float v[4] = {f.x, f.y, f.z, f.w};
  uint32_t gm = 0, tm = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t key = score_key(v[e]);
    gm |= (base + e < n && key > T ? 1u : 0u) << e;
    tm |= (base + e < n && key == T ? 1u : 0u) << e;
  }
  // (greater, tie) counts packed in one word: a workgroup holds 4096 keys, so 16 bits each suffice
  const uint32_t mine = static_cast<uint32_t>(__popc(gm)) | (static_cast<uint32_t>(__popc(tm)) << 16);
  const uint32_t incl = wave_scan(mine);
  if (lane == 63) red[wave] = incl;
  __syncthreads();
  const bool is_before = lane < static_cast<int>(blockIdx.x);
  const uint2 tk = is_before ? taken[lane] : make_uint2(0u, 0u);
  const int g_before = wave64_sum(static_cast<int>(tk.x + (is_before && !all ? c.x : 0u)));
  uint32_t excl = incl - mine;
#pragma unroll
  for (int x = 0; x < kPickWaves; ++x)
    if (x < wave) excl += red[x];
  int t_seen = wave64_sum(static_cast<int>(tk.y)) + static_cast<int>(excl >> 16);
  int pos = g_before + static_cast<int>(excl & 0xFFFFu) + min(t_seen, need);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    bool take = (gm >> e) & 1u;
    if ((tm >> e) & 1u) take = t_seen++ < need;
    if (take) {
      if (pos < k) idx_out[pos] = base + e;  // pos < k always holds; the guard keeps a logic slip in bounds
      ++pos;
    }
  }
}

__global__ __launch_bounds__(1024) void select_zero_kernel(SelectState *st) {
  st->hist[blockIdx.x >> 1][(blockIdx.x & 1) * 1024 + threadIdx.x] = 0u;
}

// "Chunk Reordering", Eq. (9), numerator: idx is ascending, so the rows of slot s are the
// index range [lower_bound(bound[s]), lower_bound(bound[s+1])).  One thread per boundary.
__global__ __launch_bounds__(128) void chunk_counts_kernel(const int32_t *__restrict__ idx, int k, SlotBounds b,
                                                           int32_t *__restrict__ counts_out) {
  __shared__ int pos[kRepoMaxChunks + 1];
  const int t = threadIdx.x;
  if (t <= b.n) {
    const int target = b.bound[t];
    int lo = 0, hi = k;  // first position whose index is >= target
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (idx[mid] < target)
        lo = mid + 1;
      else
        hi = mid;
    }
    pos[t] = lo;
  }
  __syncthreads();
  if (t < b.n) counts_out[t] = pos[t + 1] - pos[t];
}

}  // namespace

hipError_t launch_chunk_counts(ifkv_ctx *ctx, const int32_t *idx, int64_t k, const SlotBounds &b,
                               int32_t *counts_out) {
  if (b.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(chunk_counts_kernel, dim3(1), dim3(128), 0, ctx->stream, idx, static_cast<int>(k), b, counts_out);
  return hipGetLastError();
}

namespace {

constexpr size_t kSelStateBytes = (sizeof(SelectState) + 255) & ~static_cast<size_t>(255);

// Device memory of the entry point that allocates nothing: the histograms and the per-workgroup
// counts of the largest score vector it accepts, or the listed keys.  Every GPU the library runs on holds its own copy
// of the array at its own address; in host code the array's name is only a handle for looking that
// address up, never a pointer to pass on.
constexpr int64_t kStaticMaxCtx = int64_t(1) << 22;
constexpr size_t kPickBytes = 1024 + static_cast<size_t>(kPickMax) * sizeof(uint32_t);
static_assert(sizeof(PickHeader) <= 1024, "the listed keys follow");
constexpr size_t kStaticScratchBytes =
    std::max(kSelStateBytes + static_cast<size_t>(kStaticMaxCtx / kWriteChunk) * sizeof(uint2), kPickBytes);
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_static_mutex;
void *g_static_ptr[kMaxDevices] = {};

}  // namespace

int64_t topk_static_max_ctx() { return kStaticMaxCtx; }

// Address of the static scratch on the device that is current; looked up once per device.
hipError_t topk_static_scratch(void **out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_static_mutex);
  if (g_static_ptr[dev] == nullptr) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_static_ptr[dev] = p;
  }
  *out = g_static_ptr[dev];
  return hipSuccess;
}

size_t topk_scratch_bytes(const ifkv_ctx *, int64_t n_ctx) {
  if (n_ctx <= 256 * 32) return 0;
  const size_t blocks = static_cast<size_t>((n_ctx + kWriteChunk - 1) / kWriteChunk);
  return std::max(kSelStateBytes + blocks * sizeof(uint2), kPickBytes);
}

// `work`: device memory of at least topk_scratch_bytes(n_ctx) bytes (may be null when that is 0).  `shared`: other contexts' calls
// may be using it; up to 32768 scores then run in one workgroup, which needs none.  So they do where the indices go into the
// scores' own memory: one workgroup has read all scores before it writes, of several one may be at its scores later.
hipError_t launch_topk(ifkv_ctx *ctx, const float *scores, int64_t n_ctx, int64_t k, int32_t *idx_out, void *work, bool shared) {
  if (k <= 0 || n_ctx <= 0) return hipSuccess;
  const int n = static_cast<int>(n_ctx);
  const int kk = static_cast<int>(k);
  hipStream_t st = ctx->stream;
  const uintptr_t s0 = reinterpret_cast<uintptr_t>(scores), i0 = reinterpret_cast<uintptr_t>(idx_out);
  const bool in_place = i0 < s0 + static_cast<uintptr_t>(n_ctx) * sizeof(float) && s0 < i0 + static_cast<uintptr_t>(k) * sizeof(int32_t);
  if (n <= 256 * 32) {
    hipLaunchKernelGGL((topk_resident_kernel<256, 1>), dim3(1), dim3(256), 0, st, scores, n, kk, idx_out);
  } else if (n <= 1024 * 32 && (shared || in_place)) {
    hipLaunchKernelGGL((topk_resident_kernel<1024, 1>), dim3(1), dim3(1024), 0, st, scores, n, kk, idx_out);
  } else if (n <= kPickMax) {
    if (work == nullptr) return hipErrorInvalidValue;
    PickHeader *header = static_cast<PickHeader *>(work);
    uint32_t *listed = reinterpret_cast<uint32_t *>(static_cast<char *>(work) + 1024);
    const unsigned blocks = static_cast<unsigned>((n + kPickChunk - 1) / kPickChunk);
    hipLaunchKernelGGL(select_bracket_kernel, dim3(blocks), dim3(kPickThreads), 0, st, scores, n, kk, header, listed);
    hipLaunchKernelGGL(select_emit_kernel, dim3(blocks), dim3(kPickThreads), 0, st, scores, n, kk, header, listed, idx_out);
  } else {
    if (work == nullptr) return hipErrorInvalidValue;
    SelectState *state = static_cast<SelectState *>(work);
    uint2 *counts = reinterpret_cast<uint2 *>(static_cast<char *>(work) + kSelStateBytes);
    const unsigned blocks = static_cast<unsigned>((n + kSelChunk - 1) / kSelChunk);
    const unsigned writers = static_cast<unsigned>((n + kWriteChunk - 1) / kWriteChunk);
    hipLaunchKernelGGL(select_zero_kernel, dim3(6), dim3(1024), 0, st, state);
    for (int pass = 0; pass < 3; ++pass)
      hipLaunchKernelGGL(select_hist_kernel, dim3(blocks), dim3(kSelThreads), 0, st, scores, n, kk, pass, state);
    hipLaunchKernelGGL(select_count_kernel, dim3(writers), dim3(kWriteThreads), 0, st, scores, n, kk, state, counts);
    hipLaunchKernelGGL(select_write_kernel, dim3(writers), dim3(kWriteThreads), 0, st, scores, n, kk, state, counts,
                       idx_out);
  }
  return hipGetLastError();
}

}  // namespace ifkv
