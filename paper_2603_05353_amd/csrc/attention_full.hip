// Stage 4 on the matrix units with more than bf16 probabilities -- "KV Recomputation": bf16 layers with heads of 64 and
// fp32 layers.  The shape of the work is that of attention_mfma.hip (128 query columns per workgroup, kv tiles of
// 64 rows through a ring of two LDS stages, transposed products, online softmax); what differs is the precision:
//   bf16: the logits are bf16 products summed in fp32; a probability enters the second product as the sum of two
//         bf16 numbers (its rounding and the rounding of the remainder: 16 bits of mantissa, relative error
//         at most 2^-17), so that product takes two MFMAs per operand of V.  The rounding of the result outweighs this: against
//         64 bits the error of the result is that of the ALU kernel with fp32 probabilities to one part in 10^6 (200 to
//         8161 keys), and 0.25 % of its elements are the other neighbour.
//   fp32: an operand is the sum of three bf16 numbers, which hold its 24 bits (rounding, rounding of the remainder, what is left),
//         and a product the sum of six of their nine (the scheme of Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
//         Intelligence Datatype For Higher-Precision Computations", 2019); the three left out are at most 2^-24 of it, 2^-27.5 in the
//         root mean square.  The leading product has a sum
//         of its own, so the other five add roundings of their own small size only: against 64 bits the error of the result
//         is 0.4 to 0.7 of that with 32x32x2 fp32 MFMAs, whose chains of roundings are eight times as long (relative to the norm of
//         the result; 8/8 heads of 64 over 1024 keys 1.9e-7 -> 1.2e-7, 32/8 over 8192 4.0e-7 -> 2.2e-7; heads of 128, 1600 keys
//         3.3e-7 -> 1.4e-7, 8192 5.2e-7 -> 2.3e-7).  Of Q once, of K and V by every wavefront on its way from LDS, of the
//         probabilities as they are formed.  Where that cannot be had -- an infinity, a number whose rounding to bf16 is one,
//         elements out of proportion to each other by 2^46 and more (kQueryLeast and what follows) -- the workgroup repeats its sweep
//         on fp32 MFMAs, whose accumulator layout is the operand layout of the second product too (kv rows 8 a + b and
//         8 a + 4 + b).  Such a call takes 1.4 to 2.3 times as long (8/8 heads of 64, 153 rows over 1024 keys 14.4 -> 19.9 us, 32/8, 819
//         over 8192 keys 207 -> 469, of 128 416 -> 965); heads filled up with zeros, whose results of exactly 0 are looked at, up to 2 us more.
//
// Bound: fp32 by matrix and vector pipe alike (a tile of 64 rows is 96 MFMAs of 32 cycles per wavefront at d = 64, 192 at 128, and some
// 600 and 1200 instructions for the parts, 220 for the softmax; 8192 and 16384 cycles with fp32 MFMAs).  Before -> now: 32/8 heads, 819
// rows over 8192 keys, heads of 64 268 -> 201 us, of 128 600 -> 445; 1600 keys, 320 rows, 128 86 -> 70; 16/4 of 64, 180 over 1500 25.4
// -> 21.5; 8/8 of 64, 153 over 1024, parts of one tile, 13.9 -> 13.9.  Of these, knowing that no element is out of proportion takes 1 to
// 2 % with heads of 64 and up to 1 % with 128: what is hardly ever run stands out of line, and the look at V is spread over the second
// product (in one piece after the first one 1 % more; with everything in line calls of few tiles 2.5 % more).  The remainders by shift and
// subtraction, four instructions for two numbers instead of two dot products: 8 % slower with heads of 128.  fp32 MFMAs for parts of one tile: no better, and
// both kinds live at once cost registers (all fp32 calls 4 to 9 % slower).  bf16 by the vector pipe (160 instructions per tile for the
// softmax and the split of the probabilities against 24 MFMAs of 32 cycles).
#include <algorithm>

#include "attention_tile.h"
#include "lds_dma.h"

namespace ifkv {

namespace {

template <typename Tag_, int D_>
struct Tile {
  using Tag = Tag_;
  static constexpr int D = D_;
  static constexpr bool kBf16 = std::is_same<Tag, BF16Tag>::value;
  static constexpr int kRowBytes = D * Elem<Tag>::kBytes;  // 128, 256 or 512
  static constexpr int kChunks = kRowBytes / 16;
  static constexpr int kSteps = kChunks / 2;               // contraction steps of the first product: 16 bytes per lane half
  static constexpr int NDT = D / 32;                       // 32-column blocks of the output
  static constexpr int kStage = kKvTile * kRowBytes;       // one K or V tile
  static constexpr int kUnitRows = 64 / kChunks;           // rows per 1 KiB load instruction
  static constexpr int kUnits = kStage / 1024 / 4;         // load instructions per wavefront, tile and matrix
  static constexpr int kWavesPerSimd = kRowBytes > 256 ? 1 : 2;  // 128 KiB of LDS per workgroup at 512-byte rows
};

// LDS row i of a K tile holds kv row k_row(i): see sigma for bf16.
template <typename T>
__device__ __forceinline__ int k_row(int i) {
  return T::kBf16 ? sigma(i) : i;
}
// XOR of the 16-byte chunk index with which LDS row i is stored.  K: 16 rows of one chunk cover all banks (two
// 128-byte rows share a line).  V: the rows a lane half reads together (four consecutive ones in bf16, rows 4 apart in
// fp32) cover all banks.
template <typename T>
__device__ __forceinline__ int k_key(int i) {
  return T::kChunks == 8 ? (i >> 1) & 7 : i & 15;
}
template <typename T>
__device__ __forceinline__ int v_key(int i) {
  return T::kBf16 ? 4 * ((i >> 1) & 1) : 8 * ((i >> 2) & 1);
}

// What a lane fetches for each of its load instructions, as byte offsets from the tile's first row.
template <typename T>
struct TileLoads {
  uint32_t k_off[T::kUnits], v_off[T::kUnits];
  __device__ __forceinline__ TileLoads(uint32_t row_bytes, int lane, int wave) {
#pragma unroll
    for (int x = 0; x < T::kUnits; ++x) {
      const int i = (wave * T::kUnits + x) * T::kUnitRows + lane / T::kChunks, pos = lane % T::kChunks;
      k_off[x] = k_row<T>(i) * row_bytes + 16u * (pos ^ k_key<T>(i));
      v_off[x] = i * row_bytes + 16u * (pos ^ v_key<T>(i));
    }
  }
  // requests kv tile `tile` into the stages at byte addresses k_stage, v_stage
  __device__ __forceinline__ void issue(const char *k_base, const char *v_base, int64_t row_bytes, int tile, int n_kv,
                                        uint32_t k_stage, uint32_t v_stage, int lane, int wave) const {
    const uint32_t unit0 = static_cast<uint32_t>(wave * T::kUnits) * 1024u;
    const int j0 = tile * kKvTile;
    if (j0 + kKvTile <= n_kv || (j0 >= n_kv && n_kv >= kKvTile)) {
      const int64_t at = (j0 < n_kv ? j0 : 0) * row_bytes;  // look-ahead past the end: any valid tile, it is never read
      const char *kb = uniform_pointer(k_base + at), *vb = uniform_pointer(v_base + at);
#pragma unroll
      for (int x = 0; x < T::kUnits; ++x) {
        dma16_base(kb, k_off[x], k_stage + unit0 + x * 1024u);
        dma16_base(vb, v_off[x], v_stage + unit0 + x * 1024u);
      }
    } else {  // the tile that straddles the end of the cache: rows past the end are clamped (and masked later)
      asm volatile("" : "+v"(lane));  // its addresses are formed here and do not take up registers during the other tiles
#pragma unroll
      for (int x = 0; x < T::kUnits; ++x) {
        const int i = (wave * T::kUnits + x) * T::kUnitRows + lane / T::kChunks, pos = lane % T::kChunks;
        dma16(k_base + min(j0 + k_row<T>(i), n_kv - 1) * row_bytes + 16 * (pos ^ k_key<T>(i)), k_stage + unit0 + x * 1024u);
        dma16(v_base + min(j0 + i, n_kv - 1) * row_bytes + 16 * (pos ^ v_key<T>(i)), v_stage + unit0 + x * 1024u);
      }
    }
  }
};

// kv row, within its 32-row block, of accumulator register r: see sigma for bf16.
template <typename T>
__device__ __forceinline__ constexpr int reg_row(int r) {
  return T::kBf16 ? 16 * (r >> 3) + (r & 7) : 8 * (r >> 2) + (r & 3);
}
template <typename T>
__device__ __forceinline__ int half_row(int hf) {
  return T::kBf16 ? 8 * hf : 4 * hf;
}

// x minus one element of a pair of bf16 (which one: the place of -1 in `minus`)
__device__ __forceinline__ float minus_part(uint32_t pair, uint32_t minus, float x) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, minus), x, false);
}

// Eight fp32 numbers as sums of three bf16 each: the rounding, the rounding of the remainder, and what is left, which 8 bits hold.
// An infinity, and what rounds to one, becomes NaN.
struct Parts {
  v4u p[3];
};
__device__ __forceinline__ Parts split3(float (&x)[8], uint32_t minus_lo, uint32_t minus_hi) {
  Parts out;
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const uint32_t pair = pack_bf16x2(x[2 * e], x[2 * e + 1]);
      out.p[i][e] = pair;
      if (i == 2) break;
      x[2 * e] = minus_part(pair, minus_lo, x[2 * e]);
      x[2 * e + 1] = minus_part(pair, minus_hi, x[2 * e + 1]);
    }
  return out;
}
__device__ __forceinline__ Parts split_chunks(const v4u &a, const v4u &b, uint32_t minus_lo, uint32_t minus_hi) {
  float x[8];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[e] = __uint_as_float(a[e]);
    x[4 + e] = __uint_as_float(b[e]);
  }
  return split3(x, minus_lo, minus_hi);
}
// hi + lo += a . b over 16 steps of the contraction: the leading product apart from the five smaller ones
__device__ __forceinline__ void multiply_parts(const Parts &a, const Parts &b, f32x16 &hi, f32x16 &lo) {
  auto mul = [&](int i, int j, f32x16 &c) __attribute__((always_inline)) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a.p[i]), __builtin_bit_cast(bf16x8, b.p[j]), c, 0, 0, 0);
  };
  mul(0, 2, lo);
  mul(2, 0, lo);
  mul(1, 1, lo);
  mul(0, 1, lo);
  mul(1, 0, lo);
  mul(0, 0, hi);
}

// What three bf16 numbers do not hold.  Their smallest step is 2^-133 (denormal ones count in MFMAs and dot products), so an
// element below 2^-110 is known to 2^-134 only.  That is nothing where it stands beside ordinary ones, unless the other
// operand or the rest of the sum is far out of proportion to them.  So the sweep is repeated on fp32 MFMAs where
//   a query element is not zero and below 2^-110 (whatever the keys), or above 2^64 (2^-134 of a key element is less than 2^-69 then);
//   a value is 2^30 or more: what up to 2^31 keys lose of their weights changes a result by less than 2^-73 times the sum l of its weights
//   (rows of the last tile behind the last position hold anything: where a look at whole tiles finds one, those in front are looked at);
//   a result is less than 2^-46 l (so that 2^-73 l, and the 2^-134 l lost of the values, are below its 27th bit), or exactly 0 though
//   its column of V is not.
constexpr float kQueryLeast = 0x1p-110f, kQueryMost = 0x1p64f, kValueMost = 0x1p30f, kResultLeast = 0x1p-46f;

// Magnitudes so that zero is the largest: 2 |x| - 1 as a whole number.
__device__ __forceinline__ uint32_t zero_last(float x) { return 2u * __float_as_uint(x) - 1u; }
constexpr uint32_t kZero = 0xFFFFFFFFu;

__device__ __forceinline__ float max_magnitude(float m, float a, float b) {
  asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
  return m;
}
__device__ __forceinline__ float min_magnitude(float m, float a, float b) {
  asm("v_min3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
  return m;
}

// The largest magnitudes of V, four columns of the head per lane: 4 (lane % kChunks) ...  Every wavefront looks at the quarter
// of a tile's rows that it has loaded, so a tile costs it kUnits LDS reads and 2 kUnits instructions.
template <typename T>
struct ValueRange {
  float most[4];
  __device__ __forceinline__ void clear() { most[0] = most[1] = most[2] = most[3] = 0.f; }
  // load instructions x0 .. x1 - 1 of a tile
  __device__ __forceinline__ void add(const unsigned char *vs, int lane, int wave, int x0, int x1) {
    // kUnits rows of 1 KiB: chunk c of row i lies at c ^ v_key(i), whose bit 3 changes every four rows
    const unsigned char *at[2] = {vs + wave * T::kUnits * 1024 + 16 * lane, vs + wave * T::kUnits * 1024 + 16 * (lane ^ 8)};
#pragma unroll
    for (int x = x0; x < x1; x += 2) {
      v4u v[2];
#pragma unroll
      for (int y = 0; y < 2; ++y) v[y] = *reinterpret_cast<const v4u *>(at[(x + y) * T::kUnitRows / 4 & 1] + (x + y) * 1024);
#pragma unroll
      for (int e = 0; e < 4; ++e) most[e] = max_magnitude(most[e], __uint_as_float(v[0][e]), __uint_as_float(v[1][e]));
    }
  }
  __device__ __forceinline__ bool beyond() const { return !(fmaxf(fmaxf(most[0], most[1]), fmaxf(most[2], most[3])) < kValueMost); }
  // What `beyond` says of a share of rows j0 .. j1 - 1, from memory: the last tile may hold rows that nobody sees, with anything in them.
  static __device__ __forceinline__ bool beyond_among(const char *__restrict__ v_base, int64_t row_bytes, int j0, int j1, int lane, int wave) {
    float m = 0.f;
    for (int j = j0 + wave * T::kUnitRows + lane / T::kChunks; j < j1; j += 4 * T::kUnitRows) {
      const v4u v = *reinterpret_cast<const v4u *>(v_base + j * row_bytes + 16 * (lane % T::kChunks));
      m = max_magnitude(max_magnitude(m, __uint_as_float(v[0]), __uint_as_float(v[1])), __uint_as_float(v[2]), __uint_as_float(v[3]));
    }
    return !(m < kValueMost);
  }
  // To be called by all wavefronts of a workgroup that no longer uses `lds`: whether some column of V is not zero where `zeros` says
  // that a result is.  Bit 16 dt + r of a lane: column 32 dt + 8 (r / 4) + 4 (lane / 32) + r % 4 of the head, so chunk c of four columns is
  // nibble c / 2 of lane half c % 2.
  __device__ __forceinline__ bool nonzero_at(const uint32_t (&zeros)[2], unsigned char *lds, int lane, int wave) const {
    uint64_t *all = reinterpret_cast<uint64_t *>(lds);  // [4 columns of a chunk][4 wavefronts]: the lanes that saw a non-zero element
#pragma unroll
    for (int e = 0; e < 4; ++e) all[4 * e + wave] = __ballot(most[e] != 0.f);
    __syncthreads();
    const int chunk = lane % T::kChunks;
    uint32_t found = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint64_t lanes = all[4 * e] | all[4 * e + 1] | all[4 * e + 2] | all[4 * e + 3];
#pragma unroll
      for (int o = 32; o >= T::kChunks; o /= 2) lanes |= lanes >> o;
      found |= static_cast<uint32_t>(lanes >> chunk & 1) << e;
    }
    // the zeros of a lane half, nibbles 0 .. 7 and 8 .. 15
    uint32_t half[2][2];
#pragma unroll
    for (int w = 0; w < (T::NDT + 1) / 2; ++w) wave_or_halves(zeros[w], half[w][0], half[w][1]);
    const int w = T::NDT > 2 ? chunk >> 4 : 0;
    const uint32_t z = chunk & 1 ? (w != 0 ? half[T::NDT > 2][1] : half[0][1]) : (w != 0 ? half[T::NDT > 2][0] : half[0][0]);
    return (z >> (4 * (chunk >> 1 & 7)) & found) != 0;
  }
};

template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(T::kWavesPerSimd, T::kWavesPerSimd))) void attn_full_kernel(
    const char *__restrict__ q_sel, const int32_t *__restrict__ row_pos, int n_rows, const char *__restrict__ k_cache,
    const char *__restrict__ v_cache, int n_kv, void *__restrict__ out, float *__restrict__ lse_out, int n_q_heads,
    int n_kv_heads, float scale_log2, int rows_per_block, int64_t token_bytes, int64_t head_bytes, SplitPlan sp) {
  using Tag = typename T::Tag;
  constexpr int NDT = T::NDT, STEPS = T::kSteps;
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds[2][T::kStage];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds[2][T::kStage];
  __shared__ int pos_lds[4][kBlockColumns];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, hf = lane >> 5;
  const int G = sp.group_size;
  const int g = blockIdx.x;
  const int rb = gridDim.y - 1 - blockIdx.y;  // longest prefixes are dispatched first
  const int part = blockIdx.z;
  // this workgroup's share of the kv axis: tiles t0 .. t1-1 (the whole range unless the block is split)
  const int t0 = part * sp.part_tiles;
  const char *k_base = k_cache + g * head_bytes, *v_base = v_cache + g * head_bytes;
  const TileLoads<T> loads(static_cast<uint32_t>(token_bytes), lane, wave);
  const uint32_t k_addr = __builtin_amdgcn_readfirstlane(lds_address(&k_lds[0][0]));
  const uint32_t v_addr = __builtin_amdgcn_readfirstlane(lds_address(&v_lds[0][0]));
  const QueryLoads<T::kRowBytes> queries = {rb * rows_per_block, n_rows, rows_per_block, G, n_q_heads, sp.group_magic};
  unsigned char *q_lds = (wave < 2 ? k_lds[1] : v_lds[1]) + (wave & 1) * 32 * T::kRowBytes;
  queries.request_positions(row_pos, __builtin_amdgcn_readfirstlane(lds_address(pos_lds[wave])));
  queries.request(q_sel, g, wave, __builtin_amdgcn_readfirstlane(lds_address(q_lds)), [](int i) __attribute__((always_inline)) { return k_key<T>(i); });
  loads.issue(k_base, v_base, token_bytes, t0, n_kv, k_addr, v_addr, lane, wave);
  wait_vmem<QueryLoads<T::kRowBytes>::kUnits + 2 * T::kUnits>();  // the positions have landed
  int p_bmax;
  Column c = queries.column(pos_lds[wave], g, wave, n_kv, &p_bmax);
  const int n_tiles = p_bmax / kKvTile + 1;
  const int t1 = min(n_tiles, t0 + sp.part_tiles);
  if (t0 >= n_tiles) {  // nothing left for this part (uniform over the workgroup)
    wait_vmem<0>();     // before the LDS is given back
    return;
  }
  if (part == 0 && g == 0 && threadIdx.x == 0 && sp.block_parts != nullptr)
    sp.block_parts[rb] = (n_tiles + sp.part_tiles - 1) / sp.part_tiles;
  const int my_tiles = min(t1, c.p_wmax / kKvTile + 1);

  // K operand reads: row `col` of a 32-row block, chunk 2 s + hf of step s (steps 8 .. 15 repeat 256 bytes on)
  constexpr int kOffsets = STEPS < 8 ? STEPS : 8;
  int k_off[kOffsets];
#pragma unroll
  for (int s = 0; s < kOffsets; ++s) k_off[s] = col * T::kRowBytes + 16 * ((2 * s + hf) ^ k_key<T>(col));
  wait_vmem<2 * T::kUnits>();  // the wavefront's own queries have landed
  v4u qf[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    qf[s] = *reinterpret_cast<const v4u *>(q_lds + k_off[s & 7] + 256 * (s >> 3));
    if (!c.col_valid) qf[s] = v4u{0u, 0u, 0u, 0u};
  }
  // bf16 pairs (-1, 0) and (0, -1), kept out of the instruction's constant field, whose meaning for a pair of bf16 is
  // not that of the first element
  uint32_t minus_lo = 0x0000BF80u, minus_hi = 0xBF800000u;
  asm volatile("" : "+s"(minus_lo), "+s"(minus_hi));
  Parts qp[T::kBf16 ? 1 : STEPS / 2];
  uint32_t q_beyond = 0;
  if constexpr (!T::kBf16) {
    float q_most = 0.f, q_least = kQueryMost;
#pragma unroll
    for (int s = 0; s < STEPS; ++s)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        const float a = __uint_as_float(qf[s][e]), b = __uint_as_float(qf[s][e + 1]);
        q_most = max_magnitude(q_most, a, b);
        q_least = min_magnitude(q_least, a, b);
      }
    q_beyond = q_most <= kQueryMost ? 0u : 1u;
    if (__builtin_expect(__any(c.col_valid && q_least < kQueryLeast), 0)) {  // zeros do not count, but are rare
#pragma unroll
      for (int s = 0; s < STEPS; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e) q_beyond |= zero_last(__uint_as_float(qf[s][e])) < zero_last(kQueryLeast) ? 1u : 0u;
    }
    asm volatile("" : "+v"(q_beyond));  // formed here, not where it is used after the sweep
#pragma unroll
    for (int s = 0; s < STEPS; s += 2) qp[s / 2] = split_chunks(qf[s], qf[s + 1], minus_lo, minus_hi);
  }
  // V operand reads.  bf16: transpose reads; in every group of 16 lanes, lane j supplies row j / 4, d columns
  // 4 (j % 4)..+3 and receives the four rows of d column j; group covers d columns 16 (group & 1)..+15, rows + 8 hf.
  // fp32: d column `col` of the row, rows 4 hf + ...
  int v_off[2];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt) {
    if (T::kBf16) {
      const int j = lane & 15, r = j >> 2, low = 2 * ((lane >> 4) & 1) + ((j & 3) >> 1);
      v_off[dt] = (8 * hf + r) * T::kRowBytes + 16 * ((4 * dt + low) ^ v_key<T>(r)) + 8 * (j & 1);
    } else {
      v_off[dt] = 4 * hf * T::kRowBytes + 16 * ((8 * dt + (col >> 2)) ^ (8 * hf)) + 4 * (col & 3);
    }
  }

  // fp32: two sums, which are added at the end.  The leading products and the others; in the repeated sweep each half of a tile has
  // its own, because with one sum over all keys, and one per logit with heads of 64, the error against 64 bits was larger than the
  // ALU kernel's (4-to-1 to 8-to-1 grouped heads of 64, 8161 keys: one sum 5.3e-7, two 3.7e-7, ALU kernel 3.7e-7).
  constexpr int kTurns = T::kBf16 ? 1 : 2;
  f32x16 O[kTurns][NDT];
  float m_run, l_run;
  ValueRange<T> values;  // (fp32)
  auto tile_step = [&](auto exact_tag, int i, int st) __attribute__((always_inline)) {
    constexpr bool kExact = decltype(exact_tag)::value, kParts = !T::kBf16 && !kExact;
    wait_vmem<0>();   // this wavefront's share of tile i has landed
    __syncthreads();  // everyone's share is visible, and everyone is done with tile i-1
    wave_priority<0>();
    loads.issue(k_base, v_base, token_bytes, i + 1, n_kv, k_addr + (st ^ 1) * T::kStage, v_addr + (st ^ 1) * T::kStage, lane, wave);
    const unsigned char *ks = k_lds[st], *vs = v_lds[st];
    if (i >= my_tiles) {  // this wavefront's rows end before the tile (it still stages and syncs, and looks at its share of V)
      if constexpr (kParts) values.add(vs, lane, wave, 0, T::kUnits);
      return;
    }
    // S^T = K_tile . Q^T; fp32 with fp32 operands and heads of 64 in two sums of half the steps each: shorter chains of roundings
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    constexpr int kSums = T::kBf16 || (kExact && T::D == 128) ? 1 : 2;
    f32x16 S[2], H[kSums][2];
    if constexpr (kParts) {
#pragma unroll
      for (int t = 0; t < 2; ++t) H[0][t] = H[1][t] = zero;
#pragma unroll
      for (int s = 0; s < STEPS; s += 2)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          v4u k[2];
#pragma unroll
          for (int x = 0; x < 2; ++x) k[x] = *reinterpret_cast<const v4u *>(ks + k_off[(s + x) & 7] + 256 * (s >> 3) + t * 32 * T::kRowBytes);
          multiply_parts(split_chunks(k[0], k[1], minus_lo, minus_hi), qp[s / 2], H[0][t], H[1][t]);
        }
    } else {
#pragma unroll
      for (int s = 0; s < STEPS; ++s)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const v4u k = *reinterpret_cast<const v4u *>(ks + k_off[s & 7] + 256 * (s >> 3) + t * 32 * T::kRowBytes);
          f32x16 &sum = H[s * kSums / STEPS][t];
          if (s % (STEPS / kSums) == 0) sum = zero;
          if (T::kBf16) {
            sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k), __builtin_bit_cast(bf16x8, qf[s]), sum, 0, 0, 0);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              sum = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(k[e]), __uint_as_float(qf[s][e]), sum, 0, 0, 0);
          }
        }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) S[t] = kSums == 1 ? H[0][t] : H[0][t] + H[kSums - 1][t];
    // bf16: all operands of the second product are requested here, so that they arrive under the softmax
    bf16x8 vf[T::kBf16 ? 4 : 1][NDT];
    if constexpr (T::kBf16) {
      typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          const unsigned char *p = vs + v_off[dt & 1] + 16 * u * T::kRowBytes;
          const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
          const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * T::kRowBytes));
          vf[u][dt] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
        }
    }
    // the fixed reference of the fast sweep: register 0 of the lower lane half is the sweep's first key
    if (T::kBf16 && !kExact && i == t0) m_run = __shfl(S[0][0], col, 64) * scale_log2;
    // causal mask, only on tiles that reach past the wavefront's smallest position
    const int j0 = i * kKvTile;
    if (j0 + kKvTile - 1 > c.p_wmin) {
      const int base = j0 + half_row<T>(hf) - c.p_q;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (base + 32 * t + reg_row<T>(r) > 0) S[t][r] = -INFINITY;
    }
    if (kExact || !T::kBf16) {  // running max, raised (and O, l rescaled) only when the tile exceeds it by more than 2^kSlack
      float mx = S[0][0];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, S[t][r]);
      mx = half_swap_max(mx);
      const float m_new = fmaxf(m_run, mx * scale_log2);
      if (__any(m_new > m_run + kSlack)) {
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);  // 0 when m_run is still kNoMax, 1 when neither moved
        l_run *= alpha;
#pragma unroll
        for (int x = 0; x < kTurns; ++x)
#pragma unroll
          for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) O[x][dt][r] *= alpha;
        m_run = m_new;
      }
    }
    float psum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        S[t][r] = __builtin_amdgcn_exp2f(fmaf(S[t][r], scale_log2, -m_run));
        psum[r & 3] += S[t][r];
      }
    l_run += (psum[0] + psum[1]) + (psum[2] + psum[3]);
    // O^T += V_tile^T . P^T
    if constexpr (T::kBf16) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {  // kv rows 16 u + 8 hf + 0..7 of this lane's query column
        v4u hi, lo;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a = S[u >> 1][8 * (u & 1) + 2 * e], b = S[u >> 1][8 * (u & 1) + 2 * e + 1];
          hi[e] = pack_bf16x2(a, b);
          if (u == 0 && e == 3) hi[e] = wave_priority_with<2>(hi[e]);
          // the remainders a - hi, b - hi (exact): one dot product of two bf16 pairs each
          lo[e] = pack_bf16x2(minus_part(hi[e], minus_lo, a), minus_part(hi[e], minus_hi, b));
        }
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
          O[0][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u][dt], __builtin_bit_cast(bf16x8, lo), O[0][dt], 0, 0, 0);
          O[0][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u][dt], __builtin_bit_cast(bf16x8, hi), O[0][dt], 0, 0, 0);
        }
      }
    } else if constexpr (kParts) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = S[u >> 1][8 * (u & 1) + e];
        Parts pr = split3(x, minus_lo, minus_hi);
        if (2 * u < T::kUnits) values.add(vs, lane, wave, 2 * u, 2 * u + 2);
        if (u == 0) pr.p[0][0] = wave_priority_with<2>(pr.p[0][0]);
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            x[e] = *reinterpret_cast<const float *>(vs + v_off[dt & 1] + 256 * (dt >> 1) + (32 * (u >> 1) + reg_row<T>(8 * (u & 1) + e)) * T::kRowBytes);
          multiply_parts(split3(x, minus_lo, minus_hi), pr, O[0][dt], O[1][dt]);
        }
      }
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int dt = 0; dt < NDT; ++dt) {
            const float v = *reinterpret_cast<const float *>(vs + v_off[dt & 1] + 256 * (dt >> 1) + (32 * t + reg_row<T>(r)) * T::kRowBytes);
            if (t == 0 && r == 0 && dt == 0) S[t][r] = wave_priority_with<2>(S[t][r]);
            O[t][dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(v, S[t][r], O[t][dt], 0, 0, 0);
          }
    }
  };
  // The softmax needs SOME reference exponent per query column that keeps the exponentials inside the fp32 range, not
  // the column maximum: the first sweep keeps the logit of its first key (no maximum, no lane exchange, no
  // rescaling).  A column whose sum leaves [0, 2^60] makes the workgroup repeat the sweep with a running maximum.
  // fp32 layers keep the running maximum throughout, and repeat the sweep where the parts of their operands are not enough (or on
  // request): a sum that is no number, or elements out of proportion to each other (see kQueryLeast).
  auto sweep = [&](auto exact_tag, bool requested) __attribute__((always_inline)) {
#pragma unroll
    for (int x = 0; x < kTurns; ++x)
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[x][dt][r] = 0.f;
    m_run = kNoMax;
    l_run = 0.f;
    if constexpr (!T::kBf16) values.clear();
    if (!requested) loads.issue(k_base, v_base, token_bytes, t0, n_kv, k_addr, v_addr, lane, wave);
    if constexpr (!T::kBf16) {  // (the code of one stage instead of both)
#pragma unroll 1
      for (int i = t0; i < t1; ++i) tile_step(exact_tag, i, (i - t0) & 1);
    } else {
      for (int i = t0; i < t1; i += 2) {
        tile_step(exact_tag, i, 0);
        if (i + 1 < t1) tile_step(exact_tag, i + 1, 1);
      }
    }
    wait_vmem<0>();  // drain the look-ahead loads before the LDS is filled again or released
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
      if (kTurns == 2) O[0][dt] += O[kTurns - 1][dt];
  };
  const bool fast = sp.exact_only == 0;
  bool redo = !fast;
  if (fast) {
    sweep(std::false_type{}, true);
    bool again = !(l_run <= 0x1p60f), zero = false, large = false;  // also true for NaN
    if constexpr (!T::kBf16) {
      const float least_l = c.in_range ? kResultLeast * half_swap_sum(l_run) : 0.f;  // (0: nothing to be asked)
      float least = INFINITY;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; r += 2) least = min_magnitude(least, O[0][dt][r], O[0][dt][r + 1]);
      again |= q_beyond != 0;
      large = values.beyond();
      if (__builtin_expect(__any(least < least_l), 0)) {
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float x = O[0][dt][r];
            zero |= x == 0.f && least_l > 0.f;
            again |= zero_last(x) < zero_last(least_l) && least_l > 0.f;
          }
      }
    }
    redo = __syncthreads_or(again || zero || large ? 1 : 0) != 0;  // uniform over the workgroup
    if constexpr (!T::kBf16) {
      if (__builtin_expect(redo, 0)) {
        if (__syncthreads_or(large ? 1 : 0) != 0) large = values.beyond_among(v_base, token_bytes, t0 * kKvTile, min(t1 * kKvTile, p_bmax + 1), lane, wave);
        // a result of exactly 0 is right if its column of V is zero (a head filled up with zeros, for one)
        uint32_t zeros[2] = {0, 0};
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) zeros[dt / 2] |= zero && O[0][dt][r] == 0.f ? 1u << (16 * (dt & 1) + r) : 0u;
        redo = __syncthreads_or(values.nonzero_at(zeros, k_lds[0], lane, wave) || again || large ? 1 : 0) != 0;
      }
    }
  }
  if (__builtin_expect(redo, 0)) {
    if constexpr (!T::kBf16) {
      int64_t q_at = c.q_row * T::kRowBytes + 16 * hf;
      asm volatile("" : "+v"(q_at));  // nothing of this is formed before the first sweep
#pragma unroll
      for (int s = 0; s < STEPS; ++s) {
        qf[s] = v4u{0u, 0u, 0u, 0u};
        if (c.col_valid) qf[s] = *reinterpret_cast<const v4u *>(q_sel + q_at + 32 * s);
      }
    }
    sweep(std::true_type{}, !fast);
  }
  const bool split = n_tiles > sp.part_tiles;
  const float l_tot = half_swap_sum(l_run);
  const uint32_t spoilt = spoilt_columns(O[0], l_tot, c, [] { return false; });
  const PartialSlot<T::D> slot(sp, rb, gridDim.y, g, n_kv_heads, part, wave);
  if (split)
    write_partial(O[0], m_run, l_tot, c, slot);
  else
    store_output<Tag>(O[0], m_run, l_tot, c, out, lse_out, hf);
  rewrite_columns<Tag, T::D>(spoilt, c, m_run, l_tot, Sweep{q_sel, k_base, v_base, token_bytes, scale_log2, t0, t1}, split, slot, out, lse_out);
}

template <typename Tag, int D>
hipError_t run(ifkv_ctx *ctx, const void *q_sel, const int32_t *row_pos, int64_t n_rows, const void *k_cache,
               const void *v_cache, int64_t n_kv, void *out, float *lse_out) {
  using T = Tile<Tag, D>;
  const auto &d = ctx->desc;
  const int rpb = kBlockColumns / (d.n_q_heads / d.n_kv_heads);
  const unsigned n_rb = static_cast<unsigned>((n_rows + rpb - 1) / rpb);
  const SplitChoice sc = choose_split(ctx, n_rows, n_kv, ctx->scratch_bytes);
  SplitPlan sp;
  if (!place_partials(ctx, n_rows, sc, &sp)) return hipErrorInvalidValue;
  const float scale_log2 = static_cast<float>(ctx->sm_scale * 1.4426950408889634);
  if (!T::kBf16 && scale_log2 > 0x1p20f) sp.exact_only = 1;  // see kQueryMost: of logits that are not made larger than that
  const int64_t e = Elem<Tag>::kBytes;
  hipLaunchKernelGGL((attn_full_kernel<T>), dim3(d.n_kv_heads, n_rb, sc.parts), dim3(256), 0, ctx->stream,
                     static_cast<const char *>(q_sel), row_pos, static_cast<int>(n_rows), static_cast<const char *>(k_cache),
                     static_cast<const char *>(v_cache), static_cast<int>(n_kv), out, lse_out, d.n_q_heads, d.n_kv_heads,
                     scale_log2, rpb, ctx->token_stride * e, ctx->head_stride * e, sp);
  if (sc.parts > 1) launch_merge<Tag, D>(ctx, sp, row_pos, n_rows, n_kv, rpb, out, lse_out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attention_full_range(ifkv_ctx *ctx, const void *q_sel, const int32_t *row_pos, int64_t n_rows,
                                       const void *k_cache, const void *v_cache, int64_t n_kv, void *out, float *lse_out) {
  if (ctx->desc.dtype == IFKV_BF16) return run<BF16Tag, 64>(ctx, q_sel, row_pos, n_rows, k_cache, v_cache, n_kv, out, lse_out);
  if (ctx->desc.head_dim == 128) return run<F32Tag, 128>(ctx, q_sel, row_pos, n_rows, k_cache, v_cache, n_kv, out, lse_out);
  return run<F32Tag, 64>(ctx, q_sel, row_pos, n_rows, k_cache, v_cache, n_kv, out, lse_out);
}

}  // namespace ifkv
