// What the matrix kernels of stage 4 share: query columns, the cut along the kv axis, its merge, output.
#pragma once

#include <type_traits>

#include "attention_common.h"
#include "ifkv_device.h"
#include "lds_dma.h"

namespace ifkv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr int kKvTile = 64;         // kv rows per tile
constexpr int kBlockColumns = 128;  // query columns per workgroup: 4 wavefronts x 32
// The running max is only raised (and O, l rescaled) when a new tile exceeds it by more than
// this many powers of two, so probabilities stay <= 2^kSlack: exact in fp32 sums and harmless
// for the bf16 rounding, and the 64-register rescale becomes rare.
constexpr float kSlack = 8.f;
// Reference max of a column that has seen no key yet.  Finite on purpose: differences of two such
// values are 0 (not NaN), a masked logit (-inf) minus it is still -inf, and 2^(kNoMax - m) is 0.
constexpr float kNoMax = -1.0e30f;

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  f32x2 v = {a, b};
  bf16x2 r = __builtin_convertvector(v, bf16x2);  // round-to-nearest-even
  return __builtin_bit_cast(uint32_t, r);
}

// Order in which K rows are fed as MFMA A-rows.  A 32x32 accumulator gives lane
// half hf, register r the A-row 8*(r/4) + 4*hf + r%4; feeding kv row sigma(i) as
// A-row i makes registers 0..7 of a lane hold kv rows 8*hf + 0..7 and registers
// 8..15 hold kv rows 16 + 8*hf + 0..7, i.e. eight consecutive kv rows per
// 16-row contraction step, which is what the B operand of V^T.P^T needs.
// sigma swaps bits 2 and 3 (an involution); K rows are stored in LDS at row
// sigma(j), so A-row i simply reads LDS row i.
__device__ __forceinline__ int sigma(int i) { return (i & ~12) | ((i & 4) << 1) | ((i & 8) >> 1); }

// max of a value with the one held by the lane 32 positions away (the other half of the same
// query column): one lane-half swap in the vector ALU instead of a round trip through LDS.
__device__ __forceinline__ float half_swap_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_swap_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Which of the two wavefronts of a SIMD (one of each workgroup of the CU) issues first where both can.  Between equals the older
// one always does: it then runs through first product, softmax and second product while the younger one waits for the same
// pipe, and where the older one ends early the CU is left with one workgroup (pieces of equal length: half of a launch done
// at 0.75 of its time).  With a priority that rises through the tile the wavefront that is further on finishes its tile
// first, and the two fall out of step: one on the matrix pipe while the other is on the vector pipe.  32/8 heads, spread
// rows: heads of 128, 987 rows over 8654 keys 88.5 -> 82.6 us, 722 over 13305 (28/4) 92.5 -> 85.4, 114 at the end of 43000 85.2
// -> 79.7; heads of 64, 1224 over 8161 82.5 -> 74.7, 4096 over 8K 215 -> 196; fp32, heads of 64, whose products are a third of
// the work: 1 % over 16 calls (0 to 5); of 128, one wavefront per SIMD: nothing.
//   heads of 128: 0 in the first product, 1 in the softmax, 2 in the second product.  Orders that lift neither of the last
// two (1, 0, 1; 1, 0, 0; 2, 0, 1) gain nothing.
//   attn_full_kernel: 0 from the barrier on, 2 from the first probabilities on, by an instruction that is tied to a value: the built-in
// is a fence to the scheduler, and with it, calls of few pieces, one wavefront a SIMD, are 1 to 3 % slower instead of 1 to
// 2 % faster.  (There is such a fence in the other kernel anyway, where the built-in is as good.)
template <int P>
__device__ __forceinline__ void wave_priority() {
  __builtin_amdgcn_s_setprio(P);
}
template <int P, typename X>
__device__ __forceinline__ X wave_priority_with(X x) {
  asm("s_setprio %1" : "+v"(x) : "n"(P));
  return x;
}

// Per-lane query column set-up shared by the kernels.
struct Column {
  int row, hh, p_q, p_wmax, p_wmin;
  bool col_valid, in_range;
  int64_t q_row;  // row * H_q + head: the column's place in q_sel, out (x D) and lse_out
};

// qc: this lane's query column within the block (columns are numbered row-major over (row, head in group)).
__device__ __forceinline__ Column setup_column(const int32_t *__restrict__ row_pos, int n_rows, int n_kv, int row0,
                                               int rows_per_block, int G, int g, int n_q_heads, int qc) {
  Column c;
  const int rr = qc / G;
  c.hh = qc - rr * G;
  c.row = row0 + rr;
  c.col_valid = (rr < rows_per_block) && (c.row < n_rows);
  // Loads are unconditional on a clamped row (then zeroed): no divergent control flow before
  // the main loop, so no memory operation is still pending on a side path when it is entered.
  const int row_c = min(c.row, n_rows - 1);
  const int p_ld = row_pos[row_c];
  c.in_range = c.col_valid && (p_ld >= 0) && (p_ld < n_kv);
  c.p_q = c.in_range ? p_ld : 0;
  c.q_row = static_cast<int64_t>(row_c) * n_q_heads + g * G + c.hh;
  c.p_wmax = wave_max_i(c.p_q);
  c.p_wmin = wave_min_i(c.col_valid ? c.p_q : 0x7FFFFFFF);
  return c;
}

// The query columns of a workgroup of four wavefronts of 32, by direct loads into LDS.  What bounds a piece of a few tiles is
// what comes before its first product, so everything that takes is requested at once -- positions, queries, the first kv
// tile -- before it is known whether the row block reaches that tile.  An operand load of the queries straight into
// registers touches 32 rows with 32 bytes each, four times the address cycles of a contiguous one (2000 for a workgroup's 32);
// so they pass through the second ring stage, which is not filled before the first tile is used, in the layout of a K
// tile's rows.  Every wavefront takes the positions of all 128 columns, so no barrier is needed to know the longest row.  Up
// to the first product 4350 -> 3900 cycles with one workgroup on a CU, 6400 -> 4450 with two (some 400 instructions of
// address arithmetic are what is left).  Calls of 11 to 160 us are 0 to 5 % faster: 234 rows over 5527 keys, 28/4
// heads 32.5 -> 31.0, 418 over 1877, 32/8 heads 24.7 -> 24.0.  Requesting the tile first and leaving the rest as it was made them 2 to 4 %
// slower: the queries then queue behind it.
//   A piece that turns out to have no keys (rows in the front of a long cache) fetches queries and a tile in vain and waits for them before
// it leaves.  That costs a launch of many such pieces nothing that shows: 1 to 1200 rows at the front of 4000 to 65536 keys, start, priorities and
// layout of the partial results together, 0.82 to 1.00 of the time before, but for 8/8 heads of 128, 1 to 64 rows, 1.01 to 1.03 (6.4 -> 6.6 us).
template <int ROW_BYTES>
struct QueryLoads {
  static constexpr int kChunks = ROW_BYTES / 16, kUnitRows = 64 / kChunks, kUnits = 32 / kUnitRows;
  int row0, n_rows, rows_per_block, G, n_q_heads;
  uint32_t magic;  // (column * magic) >> 16 = column / G for fewer than 1024 columns and G <= 32
  __device__ __forceinline__ int row_of(int qc) const { return static_cast<int>((static_cast<uint32_t>(qc) * magic) >> 16); }
  // two load instructions
  __device__ __forceinline__ void request_positions(const int32_t *row_pos, uint32_t lds) const {
    const int lane = threadIdx.x & 63, last = n_rows - 1 - row0;
    const char *base = uniform_pointer(reinterpret_cast<const char *>(row_pos + row0));
    dma4_base(base, 4u * min(row_of(lane), last), lds);
    dma4_base(base, 4u * min(row_of(lane + 64), last), lds + 256u);
  }
  // kUnits load instructions; key(column): XOR of a column's chunk index
  template <typename F>
  __device__ __forceinline__ void request(const char *q_sel, int g, int wave, uint32_t lds, F key) const {
    const int lane = threadIdx.x & 63, last = n_rows - 1 - row0;
    const char *base = uniform_pointer(q_sel + (static_cast<int64_t>(row0) * n_q_heads + g * G) * ROW_BYTES);
#pragma unroll
    for (int x = 0; x < kUnits; ++x) {
      const int c = x * kUnitRows + lane / kChunks, rr = row_of(32 * wave + c), hh = 32 * wave + c - rr * G;
      dma16_base(base, static_cast<uint32_t>(min(rr, last) * n_q_heads + hh) * ROW_BYTES + 16u * ((lane % kChunks) ^ key(c)), lds + x * 1024u);
    }
  }
  // From the positions in LDS: this lane's column (32 wave + lane % 32), the same as setup_column's, and the largest position
  // of the block.
  __device__ __forceinline__ Column column(const int *pos, int g, int wave, int n_kv, int *p_bmax) const {
    const int lane = threadIdx.x & 63, qc = 32 * wave + (lane & 31);
    auto position = [&](int i, int p, bool *valid) __attribute__((always_inline)) {
      const int rr = row_of(i);
      *valid = rr < rows_per_block && row0 + rr < n_rows;
      return *valid && p >= 0 && p < n_kv ? p : -1;
    };
    const int p_lo = pos[lane], p_hi = pos[64 + lane], p_own = pos[qc];
    Column c;
    bool valid;
    const int lo = position(lane, p_lo, &valid), hi = position(lane + 64, p_hi, &valid);
    *p_bmax = max(wave_max_i(max(lo, hi)), 0);
    const int own = position(qc, p_own, &c.col_valid), rr = row_of(qc);
    c.hh = qc - rr * G;
    c.row = row0 + rr;
    c.in_range = own >= 0;
    c.p_q = max(own, 0);
    c.q_row = static_cast<int64_t>(min(c.row, n_rows - 1)) * n_q_heads + g * G + c.hh;
    c.p_wmax = wave_max_i(c.p_q);
    c.p_wmin = wave_min_i(c.col_valid ? c.p_q : 0x7FFFFFFF);
    return c;
  }
};

// Log-sum-exp of a sum l with the reference exponent m (log2 domain): ln 2 (m + e) + ln f for l = f 2^e with f in [0.5, 1),
// so that the only rounding of the result's own size is the last one.
__device__ __forceinline__ float log_sum_exp(float m, float l) {
  constexpr float kLn2 = 0.693147180559945309f, kLn2Rest = static_cast<float>(0.693147180559945309 - static_cast<double>(kLn2));
  int e;
  const float f = frexpf(l, &e);
  return fmaf(static_cast<float>(e), kLn2, fmaf(m, kLn2, fmaf(static_cast<float>(e), kLn2Rest, kLn2 * __log2f(f))));
}

// Normalised output of one query column: out = O / l (bf16 or fp32) and its log-sum-exp.  NDT: 32-column blocks
// of the head; register r of O[dt] is column 32 dt + 8 (r / 4) + 4 hf + r % 4.
template <typename Tag, int NDT>
__device__ __forceinline__ void store_output(const f32x16 (&O)[NDT], float m_ref, float l_tot, const Column &c,
                                             void *__restrict__ out, float *__restrict__ lse_out, int hf) {
  if (!c.col_valid) return;
  const bool ok = c.in_range;  // zeros for a row outside the cache; a sum that is no number has to show
  if (std::is_same<Tag, BF16Tag>::value) {
    const float inv = 1.f / l_tot;
    uint16_t *orow = static_cast<uint16_t *>(out) + c.q_row * (32 * NDT);
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int ri = 0; ri < 4; ++ri) {
        uint2 x;
        x.x = pack_bf16x2(O[dt][4 * ri + 0] * inv, O[dt][4 * ri + 1] * inv);
        x.y = pack_bf16x2(O[dt][4 * ri + 2] * inv, O[dt][4 * ri + 3] * inv);
        *reinterpret_cast<uint2 *>(orow + 32 * dt + 8 * ri + 4 * hf) = ok ? x : make_uint2(0u, 0u);
      }
  } else {
    float *orow = static_cast<float *>(out) + c.q_row * (32 * NDT);
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int ri = 0; ri < 4; ++ri)
        *reinterpret_cast<float4 *>(orow + 32 * dt + 8 * ri + 4 * hf) =
            ok ? make_float4(O[dt][4 * ri + 0] / l_tot, O[dt][4 * ri + 1] / l_tot, O[dt][4 * ri + 2] / l_tot, O[dt][4 * ri + 3] / l_tot)
               : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (lse_out != nullptr && hf == 0) lse_out[c.q_row] = ok ? log_sum_exp(m_ref, l_tot) : 0.f;
}

template <int NWAVES>
__device__ __forceinline__ int block_tiles(int p_wmax, int *s_pmax) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) s_pmax[wave] = p_wmax;
  __syncthreads();
  int p_bmax = 0;
#pragma unroll
  for (int w = 0; w < NWAVES; ++w) p_bmax = max(p_bmax, s_pmax[w]);
  return p_bmax / kKvTile + 1;
}

// ---------------------------------------------------------------------------
// Split over the kv axis.  Row blocks differ in length by two orders of magnitude (a row at
// position p costs p keys), and a launch has only a few blocks per CU, so the longest blocks set
// the finish time.  With `part_tiles` < the tile count of a row block, the block's kv range is
// divided into parts of part_tiles tiles, one workgroup each (blockIdx.z); each part keeps its own
// running (max, sum) and unnormalised O and writes them to scratch, and attn_merge_kernel merges
// the parts of every row that was split.  Row blocks that fit in one part write their output
// directly, as without the split.
// ---------------------------------------------------------------------------
struct SplitPlan {
  int part_tiles;     // kv tiles per part (>= number of tiles of the cache: no split)
  int parts;          // of the longest row block
  int units;          // groups of 32 query columns per row block: 4, or 8 in the wide kernel
  int last_units;     // of the last row block, which may hold fewer rows
  float *partials;    // [row blocks][H_kv][parts][units] results of 32 columns (see PartialSlot)
  int *block_parts;   // [row blocks] parts of each row block (written by part 0; 1: no partial results)
  int exact_only;     // 1: skip the fixed-reference sweep
  int group_size;        // query heads per kv head
  uint32_t group_magic;  // 65536 / (query heads per kv head), rounded up
  // wide kernel, dispatch order of a launch that is not cut, if the rows are spread evenly: how many of the longest blocks come
  // first and how many of the shortest second
  int n_front, n_small;
};

// The partial result of 32 query columns: unnormalised O, then reference max (log2 domain) and sum of each column.  A wavefront
// stores its accumulators as they are, 16 bytes a lane, and the merge reads them the same way: every access is 1 KiB of
// consecutive bytes, and a workgroup's results are one piece of memory, 1 KiB longer than a power of two, so that
// workgroups that store at the same time do not all go to the same memory channel.  As rows of [part][row][head][D] a
// store touched 32 rows with 32 bytes each, and parts that lay nearly a power of two apart could meet in the same
// channels, depending on where the scratch happened to lie (14/2 heads, 296 rows at the end of 1643 keys, seven parts 2 MiB +
// 24 KiB apart: 16 or 24 us, of which the merge 4.4 or 6.7).
// In the last row block only the units that hold rows have slots.
template <int D>
struct PartialSlot {
  static constexpr int kFloats = 32 * D + 64;
  float *o;
  float2 *ml;
  // rb of n_rb row blocks, kv head g of n_g (a cut launch has at most as many slots as the scratch holds, so 32 bits number them)
  __device__ __forceinline__ PartialSlot(const SplitPlan &sp, uint32_t rb, uint32_t n_rb, uint32_t g, uint32_t n_g, uint32_t part, uint32_t unit) {
    const uint32_t units = rb == n_rb - 1 ? sp.last_units : sp.units, parts = sp.parts;
    o = sp.partials + static_cast<uint64_t>(rb * n_g * parts * sp.units + (g * parts + part) * units + unit) * kFloats;
    ml = reinterpret_cast<float2 *>(o + 32 * D);
  }
  // registers 4 ri .. 4 ri + 3 of lane x of 32-column block dt of the head, columns 32 dt + 8 ri + 4 (x / 32) .., are quad
  // 64 (4 dt + ri) + x
  // column d of the head of query column x
  __device__ __forceinline__ float *at(int x, int d) const { return o + ((d >> 3) * 64 + ((d >> 2) & 1) * 32 + x) * 4 + (d & 3); }
};

// The stores write through the L2 (agent scope): what is left dirty there is written at the end of the launch, when nothing else is
// going on, 1 to 2.5 us of a call of 15 to 75 us.  (Stores that also leave the memory-side cache out, non-temporal ones, cost
// the merge more than they gain.)
template <int NDT>
__device__ __forceinline__ void write_partial(const f32x16 (&O)[NDT], float m_run, float l_tot, const Column &c,
                                              const PartialSlot<32 * NDT> &to) {
  if (!c.col_valid) return;
  const int lane = threadIdx.x & 63;
  constexpr int kAgentScope = 16;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(to.o, 0, PartialSlot<32 * NDT>::kFloats * sizeof(float), 0x00027000);
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int ri = 0; ri < 4; ++ri) {
      const v4u x = {__float_as_uint(O[dt][4 * ri + 0]), __float_as_uint(O[dt][4 * ri + 1]), __float_as_uint(O[dt][4 * ri + 2]), __float_as_uint(O[dt][4 * ri + 3])};
      __builtin_amdgcn_raw_buffer_store_b128(x, rsrc, 16 * lane, (4 * dt + ri) * 1024, kAgentScope);
    }
  if (lane < 32) to.ml[lane] = make_float2(m_run, l_tot);
}

// Keys behind a column's own position have probability 0, but 0 x NaN and 0 x infinity are NaN: through the matrix product
// an element of V that is not finite reaches every column of the wavefront, also those that do not see its row (an unwritten
// tail of the cache, for one).  spoilt_columns finds the columns whose result is not finite although their sum is (bit x:
// the column of lanes x and x + 32), unless may_be_right says so, and takes them out of the regular output; rewrite_columns
// computes them again from the keys they see.  Where nothing is wrong that is one multiply-add per register of the result.
template <int NDT, typename F>
__device__ __forceinline__ uint32_t spoilt_columns(const f32x16 (&O)[NDT], float l_tot, Column &c, F may_be_right) {
  float zeros = 0.f;
#pragma unroll
  for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) zeros = fmaf(O[dt][r], 0.f, zeros);
  const uint64_t lanes = __ballot(c.in_range && l_tot > 0.f && l_tot < INFINITY && !(zeros == 0.f));
  uint32_t columns = static_cast<uint32_t>(lanes | lanes >> 32);  // two lanes hold half of a column each
  if (columns != 0 && may_be_right()) columns = 0;
  c.col_valid &= ((columns >> (threadIdx.x & 31)) & 1) == 0;
  return columns;
}

// Whether V rows j0 .. j1-1 (256 bytes of bf16) are finite; the same in every lane.  Where all rows that some column of the
// wavefront does not see are, a result that is not finite comes from rows it does see, and is right (a cache with a NaN in its
// first row would otherwise have every column computed a second time: 4915 rows over 32K keys 758 ms instead of 1.3).  Not
// for probabilities that are a sum of two numbers, which make NaN of a visible infinity.
__device__ __forceinline__ bool finite_rows(const char *__restrict__ v_base, int64_t row_bytes, int j0, int j1) {
  const int lane = threadIdx.x & 63;
  float zeros = 0.f;
  for (int j = j0 + (lane >> 4); j < j1; j += 4) {
    float f[8];
    Elem<BF16Tag>::unpack(*reinterpret_cast<const v4u *>(v_base + j * row_bytes + 16 * (lane & 15)), f);
#pragma unroll
    for (int e = 0; e < 8; ++e) zeros = fmaf(f[e], 0.f, zeros);
  }
  return !__any(!(zeros == 0.f));
}

// What a workgroup's sweep was over.
struct Sweep {
  const void *q_sel;
  const char *k_base, *v_base;
  int64_t row_bytes;
  float scale_log2;
  int t0, t1;  // kv tiles
};

// One column after the other by the whole wavefront: 64 logits at a time, a lane each, then the V rows one by one, D / 64
// columns of the result per lane.  m and l are the sweep's reference exponent and sum of the lane's column.
template <typename Tag, int D>
__device__ __forceinline__ void rewrite_columns(uint32_t columns, const Column &c, float m, float l, const Sweep &sw,
                                                bool split, const PartialSlot<D> &to, void *out, float *lse_out) {
  using E = Elem<Tag>;
  constexpr int C = D / 64, VE = 16 / E::kBytes;
  const int lane = threadIdx.x & 63;
  while (columns != 0) {
    const int x = __builtin_ctz(columns);
    columns &= columns - 1;
    const int j_end = min(sw.t1 * kKvTile, __shfl(c.p_q, x, 64) + 1);
    const float m_x = __shfl(m, x, 64), l_x = __shfl(l, x, 64);
    const int64_t q_row = __shfl(c.q_row, x, 64);
    const v4u *q = reinterpret_cast<const v4u *>(static_cast<const char *>(sw.q_sel) + q_row * D * E::kBytes);
    float acc[C];
#pragma unroll
    for (int e = 0; e < C; ++e) acc[e] = 0.f;
    for (int j0 = sw.t0 * kKvTile; j0 < j_end; j0 += 64) {
      const v4u *k = reinterpret_cast<const v4u *>(sw.k_base + min(j0 + lane, j_end - 1) * sw.row_bytes);
      float dot = 0.f;
#pragma unroll 2
      for (int i = 0; i < D / VE; ++i) {
        float a[VE], b[VE];
        E::unpack(q[i], a);
        E::unpack(k[i], b);
#pragma unroll
        for (int e = 0; e < VE; ++e) dot = fmaf(a[e], b[e], dot);
      }
      const float prob = __builtin_amdgcn_exp2f(fmaf(dot, sw.scale_log2, -m_x));
      const int n = min(64, j_end - j0);
      for (int jj = 0; jj < n; ++jj) {
        const float w = __shfl(prob, jj, 64);
        const char *v = sw.v_base + (j0 + jj) * sw.row_bytes;
#pragma unroll
        for (int e = 0; e < C; ++e) acc[e] = fmaf(w, E::load1(v, C * lane + e), acc[e]);
      }
    }
#pragma unroll
    for (int e = 0; e < C; ++e) {
      if (split)
        *to.at(x, C * lane + e) = acc[e];
      else
        E::store1(out, q_row * D + C * lane + e, acc[e] / l_x);
    }
    if (lane == 0) {
      if (split)
        to.ml[x] = make_float2(m_x, l_x);
      else if (lse_out != nullptr)
        lse_out[q_row] = log_sum_exp(m_x, l_x);
    }
  }
}

// The merge of the parts of a row block: O = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s.  A wavefront takes four query columns,
// 16 lanes each, D / 64 quads of the head per lane: a load is 16 pieces of 64 bytes, a store whole lines of the result.  A lane
// knows reference and sum of its own column and needs no other lane.  Bound: latency -- the partial results come from memory,
// other workgroups wrote them in the previous launch -- so up to eight parts are requested at once.  MANY: the parts are dealt
// out to the four wavefronts of a workgroup, which add up through LDS; with more than 16 parts, and with more than eight where there
// are so few columns that one round of latency counts and not the number of workgroups (32/8 heads, 16 parts: 128 rows 7.5 us
// one way, 12.1 the other; 40/8 heads, 11 parts, 4 rows, the whole call 13.8 and 12.5).
//   With this layout, stores that write through the L2 and this merge, against [part][row][head][D] and a (row, head) pair per
// wavefront, attention and merge together: 32/8 heads of 128, 178 rows over 4850 keys 25.5 -> 24.5 us, 128 at the end of 32K 76 ->
// 72.6 (70 to 82 from box to box), 987 over 8654 83 -> 79.4; 28/4, 722 over 13305 87 -> 82; heads of 64, 1224 over 8161 74 -> 70.5; 14/2, 600 over 6000 26 -> 23.
// A whole 32-column slot per workgroup, every load 1 KiB of consecutive bytes, was 0.5 to 1.2 us slower: its stores are 16-byte
// pieces of 32 rows.
constexpr int kMergeBatch = 8, kMergeMany = 16, kMergeFewColumns = 2048;

// What a part holds counts as nothing where its weight is 0, whatever it is (an infinite value with a weight that vanishes), and so
// does what was added up before; a weight that is no number shows.
__device__ __forceinline__ float weighted(float x, float weight) { return (weight == 0.f ? 0.f : x) * weight; }

// Adds parts s0, s0 + STEP, .. (BATCH of them, those below n_parts) of a lane's column to (m_max, l, acc).
template <int D, int BATCH, int STEP>
__device__ __forceinline__ void merge_parts(const SplitPlan &sp, int rb, int n_g, int g, int unit, int col, int n_parts, int s0, float &m_max,
                                            float &l, float (&acc)[D / 64][4]) {
  constexpr int V = D / 64;
  const int quad = (threadIdx.x & 63) >> 2;
  float2 ml[BATCH];
  float4 o[BATCH][V];
#pragma unroll
  for (int u = 0; u < BATCH; ++u) {
    const PartialSlot<D> from(sp, rb, gridDim.z, g, n_g, min(s0 + u * STEP, n_parts - 1), unit);  // past the last part: a valid slot, of weight 0
    ml[u] = from.ml[col];
#pragma unroll
    for (int v = 0; v < V; ++v) o[u][v] = reinterpret_cast<const float4 *>(from.o)[(16 * v + quad) * 32 + col];
  }
  float m_new = m_max;
  // A part whose sum is exactly 0 holds no key that this column sees, and may hold anything else: it takes no part.  (Any other
  // sum does, also one that is no number.)
#pragma unroll
  for (int u = 0; u < BATCH; ++u) {
    if (s0 + u * STEP >= n_parts || ml[u].y == 0.f) ml[u] = make_float2(-INFINITY, 0.f);
    m_new = fmaxf(m_new, ml[u].x);
  }
  const float keep = m_max == m_new ? 1.f : __builtin_amdgcn_exp2f(m_max - m_new);  // 0 for the first parts that hold anything
  l *= keep;
#pragma unroll
  for (int v = 0; v < V; ++v)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[v][e] = weighted(acc[v][e], keep);
  m_max = m_new;
#pragma unroll
  for (int u = 0; u < BATCH; ++u) {
    const float weight = ml[u].y == 0.f ? 0.f : __builtin_amdgcn_exp2f(ml[u].x - m_max);
    l += ml[u].y * weight;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      acc[v][0] += weighted(o[u][v].x, weight);
      acc[v][1] += weighted(o[u][v].y, weight);
      acc[v][2] += weighted(o[u][v].z, weight);
      acc[v][3] += weighted(o[u][v].w, weight);
    }
  }
}

template <typename Tag, int D, bool MANY>
__global__ __launch_bounds__(256) void attn_merge_kernel(SplitPlan sp, const int32_t *__restrict__ row_pos, int n_rows, int n_kv,
                                                         int n_q_heads, int n_kv_heads, int rows_per_block, void *__restrict__ out,
                                                         float *__restrict__ lse_out) {
  constexpr int V = D / 64;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int four = MANY ? blockIdx.x : 4 * blockIdx.x + wave, unit = four >> 3, g = blockIdx.y, rb = blockIdx.z;
  const int qc = 4 * four + (lane & 3), col = qc & 31, rr = static_cast<int>((static_cast<uint32_t>(qc) * sp.group_magic) >> 16);
  const int row = rb * rows_per_block + rr;
  const bool valid = rr < rows_per_block && row < n_rows;
  if (!__any(valid)) return;  // (MANY: the same for all wavefronts)
  const int n_parts = sp.block_parts[rb], pos = row_pos[min(row, n_rows - 1)];
  if (n_parts <= 1) return;  // written directly by the attention kernel
  float m_max = -INFINITY, l = 0.f, acc[V][4] = {};
  if constexpr (MANY) {
    if (n_parts <= 16)
      merge_parts<D, 4, 4>(sp, rb, n_kv_heads, g, unit, col, n_parts, wave, m_max, l, acc);
    else
      for (int s0 = wave; s0 < n_parts; s0 += 4 * kMergeBatch) merge_parts<D, kMergeBatch, 4>(sp, rb, n_kv_heads, g, unit, col, n_parts, s0, m_max, l, acc);
    __shared__ float4 o_lds[4][V][64];
    __shared__ float2 ml_lds[4][64];
#pragma unroll
    for (int v = 0; v < V; ++v) o_lds[wave][v][lane] = make_float4(acc[v][0], acc[v][1], acc[v][2], acc[v][3]);
    ml_lds[wave][lane] = make_float2(m_max, l);
    __syncthreads();
    if (wave != 0) return;
    float2 ml[4];
#pragma unroll
    for (int w = 1; w < 4; ++w) ml[w] = ml_lds[w][lane];
    const float m_own = m_max;
#pragma unroll
    for (int w = 1; w < 4; ++w) m_max = fmaxf(m_max, ml[w].x);
    const float keep = l == 0.f ? 0.f : __builtin_amdgcn_exp2f(m_own - m_max);
    l *= keep;
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[v][e] = weighted(acc[v][e], keep);
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float weight = ml[w].y == 0.f ? 0.f : __builtin_amdgcn_exp2f(ml[w].x - m_max);
      l += ml[w].y * weight;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const float4 o = o_lds[w][v][lane];
        acc[v][0] += weighted(o.x, weight);
        acc[v][1] += weighted(o.y, weight);
        acc[v][2] += weighted(o.z, weight);
        acc[v][3] += weighted(o.w, weight);
      }
    }
  } else if (n_parts <= 2) {
    merge_parts<D, 2, 1>(sp, rb, n_kv_heads, g, unit, col, n_parts, 0, m_max, l, acc);
  } else if (n_parts <= 4) {
    merge_parts<D, 4, 1>(sp, rb, n_kv_heads, g, unit, col, n_parts, 0, m_max, l, acc);
  } else {
    for (int s0 = 0; s0 < n_parts; s0 += kMergeBatch) merge_parts<D, kMergeBatch, 1>(sp, rb, n_kv_heads, g, unit, col, n_parts, s0, m_max, l, acc);
  }
  if (!valid) return;
  const bool ok = pos >= 0 && pos < n_kv;
  const int64_t q_row = static_cast<int64_t>(row) * n_q_heads + g * sp.group_size + qc - rr * sp.group_size;
  const float inv = 1.f / l;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int64_t at = q_row * D + 64 * v + 4 * (lane >> 2);
    if (std::is_same<Tag, BF16Tag>::value) {
      const uint2 x = make_uint2(pack_bf16x2(acc[v][0] * inv, acc[v][1] * inv), pack_bf16x2(acc[v][2] * inv, acc[v][3] * inv));
      *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(out) + at) = ok ? x : make_uint2(0u, 0u);
    } else {
      *reinterpret_cast<float4 *>(static_cast<float *>(out) + at) =
          ok ? make_float4(acc[v][0] / l, acc[v][1] / l, acc[v][2] / l, acc[v][3] / l) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  if (lse_out != nullptr && lane < 4) lse_out[q_row] = ok ? log_sum_exp(m_max, l) : 0.f;
}

template <typename Tag, int D>
void launch_merge(ifkv_ctx *ctx, const SplitPlan &sp, const int32_t *row_pos, int64_t n_rows, int64_t n_kv, int rows_per_block,
                  void *out, float *lse_out) {
  const auto &d = ctx->desc;
  const bool many = sp.parts > kMergeMany || (sp.parts > kMergeBatch && n_rows * d.n_q_heads <= kMergeFewColumns);
  const dim3 grid(many ? 8 * sp.units : 2 * sp.units, d.n_kv_heads, static_cast<unsigned>((n_rows + rows_per_block - 1) / rows_per_block));
  auto *kernel = many ? attn_merge_kernel<Tag, D, true> : attn_merge_kernel<Tag, D, false>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, ctx->stream, sp, row_pos, static_cast<int>(n_rows), static_cast<int>(n_kv),
                     d.n_q_heads, d.n_kv_heads, rows_per_block, out, lse_out);
}

// The choice of the cut (host), defined in attention_mfma.hip.
struct SplitChoice {
  int parts, part_tiles;
};
SplitChoice choose_split(const ifkv_ctx *ctx, int64_t n_rows, int64_t n_kv, size_t scratch_bytes);
// lays the partial results of a cut launch out in the context's scratch; false if they do not fit
bool place_partials(const ifkv_ctx *ctx, int64_t n_rows, const SplitChoice &sc, SplitPlan *sp);

// attention_full.hip: launch of one row range for bf16 heads of 64 and fp32
hipError_t launch_attention_full_range(ifkv_ctx *ctx, const void *q_sel, const int32_t *row_pos, int64_t n_rows,
                                       const void *k_cache, const void *v_cache, int64_t n_kv, void *out, float *lse_out);

}  // namespace ifkv
