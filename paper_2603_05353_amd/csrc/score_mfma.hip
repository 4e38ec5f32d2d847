// Stage 2 on the matrix units -- Eq. (7): s_j = sum_i A_ij.
//
// Per kv head the work is a [M*G x d] x [d x N] product (all prompt rows of the G query heads that share
// the kv head against every context key) whose softmax is taken along N and then summed along M*G.  At
// M*G = 512 and d = 128 that is ~500 flop per byte of K: the stage is bound by the matrix and
// transcendental units, not by HBM, and A cannot be stored (four times the size of K), so it takes two
// sweeps over the keys:
//   pass A (score_stats_mfma):  S^T = K.Q^T, a lane owns one query row -> (reference exponent, sum) per lane
//           with no cross-lane traffic; one partial result per (key slice, query row).
//   pass B (score_colsum_mfma): S = Q.K^T, a lane owns one key -> sum over query rows of exp2(S*c - m_q) / Z_q,
//           in-lane.  (1 / Z_q enters as the factor of a multiply-add: folded into the exponent as log2 Z_q it would
//           cost nothing less and its rounding, 5e-7 at 16 K keys, would show in every score of the row.)
//
// Layout of one block.  The query rows stay in REGISTERS for the whole block (32 * QB rows per wavefront as
// MFMA operands); the keys stream through a ring of NS LDS stages filled by direct global -> LDS loads NS-1
// tiles ahead and are read by all wavefronts.  WQ wavefronts split the query rows, WK split the 32-key
// subtiles of a tile.  So a block starts as soon as its query rows and ONE tile of keys have arrived, and
// one LDS operand read feeds QB products.  With the query rows in LDS and every wavefront streaming keys of
// its own into registers, 256 KB per compute unit had to arrive before anything could start: 7.5 us of pass A
// and 11 us of pass B.  Both passes together, 32/8 heads of 128 in bf16, before -> now:
//   512 context keys, 128 prompt rows  28.3 -> 15.6 us     8K keys, 64 rows    27.3 -> 20.9 us
//   32K keys, 128 prompt rows          84.6 -> 75 us       128K keys, 128 rows  284 -> 263 us
// What is left at 32K: 64 us of loop, 1024 MFMAs per SIMD and pass at 31 ns each -- 32 cycles of matrix pipe and
// about as many of vector pipe (six instructions per MFMA: scale-subtract, exponential at half rate, add, for two
// logits), which two wavefronts per SIMD overlap to two thirds, at a shader clock that the power limit holds
// between 1.7 and 2.3 GHz -- and 11 us of launches, query rows, merges and the final sums.
//
// Element types.  Everything moves in 16-byte chunks: a contraction step is one chunk per lane and operand, one
// 32x32x16 bf16 MFMA or four 32x32x2 fp32 MFMAs (full fp32 products and sums).
#include <algorithm>
#include <type_traits>

#include "ifkv_device.h"
#include "lds_dma.h"
#include "score_common.h"

namespace ifkv {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr double kLog2e = 1.4426950408889634;

struct ScoreGeom {
  int n_ctx, m_prompt, n_q_heads, n_kv_heads;
  int n_qchunks;       // query-row chunks per kv head
  int q_chunk_rows;    // rows per chunk (at most Shape::kRows); the last chunk may hold fewer
  int kv_per_block;    // context keys per slice (whole tiles)
  int n_slices;        // context slices
  int n_partials;      // slices of pass A: the context's and, if the prompt's own keys take part, one more for them
  float scale_log2;
  int64_t token_bytes, head_bytes;  // layout of k_global
};

// D elements of type Tag per row; QB 32-row query blocks per wavefront, WQ x WK wavefronts, NS LDS stages.
template <typename Tag_, int D_, int QB_, int WQ_, int WK_, int NS_>
struct Shape {
  using Tag = Tag_;
  static constexpr int D = D_, QB = QB_, WQ = WQ_, WK = WK_, NS = NS_;
  static constexpr int kRowBytes = D * Elem<Tag>::kBytes;
  static constexpr int kChunks = kRowBytes / 16;         // 8, 16 or 32
  static constexpr int kSteps = kChunks / 2;             // contraction steps: the two lane halves take a chunk each
  static constexpr int KT = WK == 1 ? 2 : 1;             // 32-key subtiles per wavefront and tile
  static constexpr int TK = 32 * KT * WK;                // keys per tile
  static constexpr int kWaves = WQ * WK;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kRows = 32 * QB * WQ;             // query rows per block
  static constexpr int kStage = TK * kRowBytes;          // bytes of one LDS stage
  static constexpr int kUnitRows = 64 / kChunks;         // key rows per 1 KiB load instruction
  static constexpr int kUnits = kStage / 1024 / kWaves;  // load instructions per wavefront and tile
  static constexpr int kSlots = KT * QB;                 // 32x32 products per wavefront and tile
  // Query rows reach their operand registers through LDS, 32 rows x at most 256 bytes per wavefront and piece.  The
  // pieces lie where the last ring stage (not filled before the first tile is used) begins.
  static constexpr int kPieceBytes = kRowBytes < 256 ? kRowBytes : 256;
  static constexpr int kPieces = kRowBytes / kPieceBytes;  // per query block
  static constexpr int kPiece = 32 * kPieceBytes;
  static constexpr int kRing = NS * kStage;
  static constexpr int kPieceBase = (NS - 1) * kStage;
  static constexpr int kLds = kPieceBase + kWaves * kPiece > kRing ? kPieceBase + kWaves * kPiece : kRing;
  static constexpr int kMinWavesPerSimd = kThreads == 512 || kLds <= 72 * 1024 ? 2 : 1;  // two blocks of 256 threads share the LDS
  static_assert(kUnits >= 1 && (NS - 2) * kUnits <= 15, "wait counter");
  static_assert(kRows <= kThreads, "one query row per thread");
};

// Key rows sit in LDS at row * kRowBytes with their chunks XOR-permuted, so that 16 consecutive rows of one
// chunk index cover all banks (rows of 128 bytes: two rows share a 256-byte line).
template <int CHUNKS>
__device__ __forceinline__ int chunk_key(int row) {
  return CHUNKS == 8 ? (row >> 1) & 7 : row & 15;
}

__device__ __forceinline__ f32x16 mma(BF16Tag, const v4u &a, const v4u &b, const f32x16 &c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// contraction index of product i: element i of the lower lane half's chunk and element i of the upper one's
__device__ __forceinline__ f32x16 mma(F32Tag, const v4u &a, const v4u &b, f32x16 c) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[i]), __uint_as_float(b[i]), c, 0, 0, 0);
  return c;
}

// Where a block's keys come from: rows 0 .. n_keys-1 of one kv head.
struct KeySource {
  const char *base;
  int64_t row_bytes;
  int n_keys;
};

// What a lane fetches for each of its load instructions, as byte offsets from the tile's first key: fixed for the
// whole kernel, so a tile that lies inside the cache costs scalar arithmetic and kUnits loads, no vector instruction.
template <typename S>
struct TileLoads {
  uint32_t off[S::kUnits];
  int row[S::kUnits];
  __device__ __forceinline__ TileLoads(const KeySource &src, int lane, int wave) {
    const int r = lane / S::kChunks, pos = lane % S::kChunks;
#pragma unroll
    for (int x = 0; x < S::kUnits; ++x) {
      row[x] = (wave * S::kUnits + x) * S::kUnitRows + r;  // LDS row
      off[x] = static_cast<uint32_t>(row[x]) * static_cast<uint32_t>(src.row_bytes) +
               16u * (pos ^ chunk_key<S::kChunks>(row[x]));
    }
  }
  // requests the tile that starts at key j0 into the LDS stage at byte address `stage`
  __device__ __forceinline__ void issue(const KeySource &src, int j0, uint32_t stage, int wave) const {
    const uint32_t unit0 = stage + static_cast<uint32_t>(wave * S::kUnits) * 1024u;
    if (j0 + S::TK <= src.n_keys || (j0 >= src.n_keys && src.n_keys >= S::TK)) {
      const char *base = uniform_pointer(src.base + (j0 < src.n_keys ? j0 : 0) * src.row_bytes);  // past the end: any tile, it is never used
#pragma unroll
      for (int x = 0; x < S::kUnits; ++x) dma16_base(base, off[x], unit0 + x * 1024u);
    } else {
      // the one tile that straddles the end: rows past the last key are clamped to it (their products are masked or
      // never stored)
#pragma unroll
      for (int x = 0; x < S::kUnits; ++x) {
        const int j = min(j0 + row[x], src.n_keys - 1);
        dma16(src.base + j * src.row_bytes + (off[x] - static_cast<uint32_t>(row[x]) * static_cast<uint32_t>(src.row_bytes)),
              unit0 + x * 1024u);
      }
    }
  }
};

// This lane's operand reads of its wavefront's first 32-key subtile of a tile: key `lane & 31`, chunk 2 s + lane / 32 of step s.  Steps 8 .. 15
// of 512-byte rows repeat the offsets of steps 0 .. 7, 256 bytes on.
template <typename S>
struct KeyReads {
  int off[S::kSteps < 8 ? S::kSteps : 8];
  __device__ __forceinline__ KeyReads(int lane, int wk) {
    const int row = lane & 31, hf = lane >> 5;
#pragma unroll
    for (int s = 0; s < (S::kSteps < 8 ? S::kSteps : 8); ++s)
      off[s] = (wk * S::KT * 32 + row) * S::kRowBytes + 16 * ((2 * s + hf) ^ chunk_key<S::kChunks>(row));
  }
  __device__ __forceinline__ v4u read(const unsigned char *subtile, int s) const {
    return *reinterpret_cast<const v4u *>(subtile + off[s & 7] + 256 * (s >> 3));
  }
};

// Query rows of a wavefront as MFMA operands: lane (row, hf) holds chunks 2 s + hf of row qb * 32 + row.  Rows are
// numbered (prompt row, head in group); rows past the chunk's real ones repeat its last one (their results are
// never used).  Straight from global memory an operand load touches 32 rows with 32 bytes each, four times the
// cycles of a contiguous one (4 us of either pass at 512 rows per compute unit); so the rows go through the
// wavefront's own piece of LDS, filled by contiguous direct loads.  `after_first` is called when the first piece has
// been requested; it requests the first NS - 1 key tiles, which the first piece does not wait for (both passes, 1024 keys
// 13.4 -> 13.0 us, 3000 16.6 -> 16.3).
template <typename S, typename F>
__device__ __forceinline__ void load_queries(v4u (&qf)[S::QB][S::kSteps], unsigned char *lds,
                                             const char *__restrict__ q_prompt, const ScoreGeom &gm, int g, int qc,
                                             int q_rows, int wq, F after_first) {
  constexpr int kChunks = S::kPieceBytes / 16, kSteps = kChunks / 2, kUnitRows = 64 / kChunks, kUnits = 32 / kUnitRows;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = lane & 31, hf = lane >> 5;
  const int G = gm.n_q_heads / gm.n_kv_heads;
  unsigned char *piece = lds + S::kPieceBase + wave * S::kPiece;
  const uint32_t piece_addr = __builtin_amdgcn_readfirstlane(lds_address(piece));
  const char *head = uniform_pointer(q_prompt + static_cast<int64_t>(g) * G * S::kRowBytes);
  const uint32_t row_bytes = static_cast<uint32_t>(gm.n_q_heads) * S::kRowBytes;
  const int dr = kUnitRows / G, dh = kUnitRows - dr * G;  // consecutive load instructions are kUnitRows rows apart
  const int last = q_rows - 1, r_last = (qc * gm.q_chunk_rows + last) / G;
  const uint32_t off_last = r_last * row_bytes + (qc * gm.q_chunk_rows + last - r_last * G) * S::kRowBytes;
#pragma unroll
  for (int qb = 0; qb < S::QB; ++qb)
#pragma unroll
    for (int h = 0; h < S::kPieces; ++h) {
      if (qb + h > 0) wait_lds_reads();  // of the previous piece
      int ql = (wq * S::QB + qb) * 32 + lane / kChunks;
      int r = (qc * gm.q_chunk_rows + ql) / G, hh = qc * gm.q_chunk_rows + ql - r * G;
#pragma unroll
      for (int x = 0; x < kUnits; ++x) {
        const uint32_t off = ql <= last ? r * row_bytes + hh * S::kRowBytes : off_last;
        dma16_base(head, off + h * 256 + 16 * ((lane % kChunks) ^ chunk_key<kChunks>(x * kUnitRows + lane / kChunks)),
                   piece_addr + x * 1024u);
        ql += kUnitRows;
        r += dr;
        hh += dh;
        if (hh >= G) {
          hh -= G;
          ++r;
        }
      }
      if (qb + h == 0) {
        after_first();
        wait_vmem<std::min((S::NS - 1) * S::kUnits, 15)>();  // the key tiles may still be on their way
      } else {
        wait_vmem<0>();
      }
#pragma unroll
      for (int s = 0; s < kSteps; ++s)
        qf[qb][h * kSteps + s] =
            *reinterpret_cast<const v4u *>(piece + row * S::kPieceBytes + 16 * ((2 * s + hf) ^ chunk_key<kChunks>(row)));
    }
}

// Which (slice, kv head, query chunk) a block serves.  Blocks are dealt out to the XCDs in turn; every XCD gets a
// contiguous range of the numbering (kv head, slice, query chunk), so that the blocks that stage the same keys, and
// those that use the same query rows, share an L2.  (In plain order the three query chunks of a 28/4-head layer
// landed on different XCDs, and the keys crossed the fabric three times.)
struct BlockPlace {
  int kb, g, qc;
  __device__ __forceinline__ BlockPlace(int id, int total, int n_slices, int n_qchunks) {
    constexpr int kXcds = 8;
    const int per = total / kXcds, extra = total - per * kXcds, xcd = id % kXcds;
    const int v = xcd * per + min(xcd, extra) + id / kXcds;
    const int w = v / n_qchunks;
    // (divisions run in the vector unit; the results are the same in every lane)
    qc = __builtin_amdgcn_readfirstlane(v - w * n_qchunks);
    g = __builtin_amdgcn_readfirstlane(w / n_slices);
    kb = __builtin_amdgcn_readfirstlane(w) - g * n_slices;
  }
};

// ---------------------------------------------------------------------------
// pass A
// ---------------------------------------------------------------------------
// The sums only need SOME reference exponent per row that keeps them inside the fp32 range, not the row
// maximum: the fast sweep takes the logit of the first key a lane sees for the row (always the logit of a
// real key, because the key loads are clamped) and keeps it, which saves the maximum over every tile and the
// rescaling.  Sums that leave [0, 2^60] (a logit more than 60 above the reference: attention far more peaked
// than anything a model produces) make the block repeat its sweep with a running maximum.
//
// The prompt's own keys (slice n_slices) are one more slice whose keys each row sees causally: prompt row r takes
// part in keys 0 .. r.  A lane's keys ascend, so a lane whose first key is masked sees none.
template <typename S>
__global__ __launch_bounds__(S::kThreads) __attribute__((amdgpu_waves_per_eu(S::kMinWavesPerSimd, 2))) void score_stats_mfma(
    const char *__restrict__ k_global, const char *__restrict__ k_prompt, const char *__restrict__ q_prompt,
    ScoreGeom gm, float2 *__restrict__ partial) {
  using Tag = typename S::Tag;
  constexpr int QB = S::QB, KT = S::KT, NS = S::NS, STEPS = S::kSteps;
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds[S::kLds];
  const BlockPlace at(blockIdx.x, gridDim.x, gm.n_partials, gm.n_qchunks);
  const int kb = at.kb, g = at.g, qc = at.qc;
  const int G = gm.n_q_heads / gm.n_kv_heads;
  const int q_rows = min(gm.q_chunk_rows, gm.m_prompt * G - qc * gm.q_chunk_rows);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wq = S::WK == 1 ? wave : wave % S::WQ, wk = S::WK == 1 ? 0 : wave / S::WQ;
  const int row = lane & 31, hf = lane >> 5;
  const float c = gm.scale_log2;

  const bool own_keys = kb == gm.n_slices;  // the prompt's keys: packed, causal
  KeySource src;
  src.base = own_keys ? k_prompt + static_cast<int64_t>(g) * S::kRowBytes : k_global + g * gm.head_bytes;
  src.row_bytes = own_keys ? static_cast<int64_t>(gm.n_kv_heads) * S::kRowBytes : gm.token_bytes;
  src.n_keys = own_keys ? gm.m_prompt : gm.n_ctx;
  const int j_begin = own_keys ? 0 : kb * gm.kv_per_block;
  const int j_end = own_keys ? gm.m_prompt : min(gm.n_ctx, j_begin + gm.kv_per_block);
  const int n_tiles = (j_end - j_begin + S::TK - 1) / S::TK;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(k_lds));

  const TileLoads<S> loads(src, lane, wave);
  auto first_tiles = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NS - 1; ++t) loads.issue(src, j_begin + t * S::TK, lds0 + t * S::kStage, wave);
  };
  v4u qf[QB][STEPS];
  load_queries<S>(qf, k_lds, q_prompt, gm, g, qc, q_rows, wq, first_tiles);
  int limit[QB];  // keys below this index count for the lane's row
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
    limit[qb] = own_keys ? (qc * gm.q_chunk_rows + min((wq * QB + qb) * 32 + row, q_rows - 1)) / G + 1 : j_end;
  const bool active = wq * QB * 32 < q_rows;  // otherwise the wavefront only stages keys
  const KeyReads<S> kr(lane, wk);

  float m[QB], z[QB];
  // register r of a product: key 8 (r/4) + 4 hf + r%4 of the subtile, query row `row` of the block
  v4u kf[STEPS];
  // One slot: the MFMAs of a new product N (query block qn against the subtile in kf) in slices, each preceded
  // by a share of the vector work on the finished product C (query block qo, keys from jc): the matrix pipe works
  // underneath the vector instructions.  The empty asm statements and the fences keep the shares in their
  // slices.  `refill`: the subtile whose operands replace kf as its steps are used up.
  auto slot = [&](auto tail_tag, auto exact_tag, auto product_tag, auto vector_first_tag, f32x16 &N, int qn, f32x16 &C,
                  int qo, int jc, bool first, const unsigned char *refill) __attribute__((always_inline)) {
    constexpr bool kExact = decltype(exact_tag)::value;
    constexpr bool kProduct = decltype(product_tag)::value;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    // The pending product of a tile's first slot is long finished, its operands are not there yet: vector work
    // first.  In the other slots the first MFMA covers the end of the product that the vector work waits for.
    constexpr bool kVectorFirst = decltype(vector_first_tag)::value;
    auto product = [&](int s) __attribute__((always_inline)) {
      if (kProduct) {
        N = mma(Tag{}, kf[s], qf[qn][s], s == 0 ? zero : N);
        if (refill != nullptr) kf[s] = kr.read(refill, s);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if (!kVectorFirst) product(0);
    const float first_logit = C[0];  // before the mask
    if (decltype(tail_tag)::value) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (jc + 8 * (r >> 2) + 4 * hf + (r & 3) >= limit[qo]) C[r] = -INFINITY;
    }
    float m_use = m[qo], m_new = 0.f, acc = 0.f;
    if (kExact) {
      float mx = C[0];
#pragma unroll
      for (int r = 1; r < 16; ++r) mx = fmaxf(mx, C[r]);
      m_new = fmaxf(m[qo], mx * c);
      m_use = fmaxf(m_new, -1e30f);  // a lane that has seen no valid key yet stays at (-inf, 0)
    } else if (first) {
      m_use = first_logit * c;
    }
    asm volatile("" : "+v"(m_use));
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (!kVectorFirst && s > 0) product(s);
#pragma unroll
      for (int r = 16 * s / STEPS; r < 16 * (s + 1) / STEPS; ++r) acc += __builtin_amdgcn_exp2f(fmaf(C[r], c, -m_use));
      asm volatile("" : "+v"(acc));
      if (kVectorFirst) product(s);
    }
    if (kExact) {
      z[qo] = z[qo] * __builtin_amdgcn_exp2f(m[qo] - m_use) + acc;
      m[qo] = m_new;
    } else {
      z[qo] += acc;
      m[qo] = m_use;
    }
  };
  // Products of a tile in the order (subtile, query block); the last one of a tile is absorbed by the first slot
  // of the next tile.
  f32x16 X, P;  // the two products in flight; P is the pending one between tiles
  auto tile = [&](auto tail_tag, auto exact_tag, int i, const unsigned char *stage) __attribute__((always_inline)) {
    const int j0 = j_begin + i * S::TK + wk * KT * 32;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) kf[s] = kr.read(stage, s);
#pragma unroll
    for (int u = 0; u < S::kSlots; ++u) {
      const int t = u / QB, qb = u % QB;
      const int qo = u == 0 ? QB - 1 : (u - 1) % QB;
      const int jc = u == 0 ? j0 - S::TK + 32 * (KT - 1) : j0 + 32 * ((u - 1) / QB);
      const bool first = u == 0 ? (KT == 1 && i == 1) : ((u - 1) / QB == 0 && i == 0);
      const unsigned char *refill = (qb == QB - 1 && t + 1 < KT) ? stage + (t + 1) * 32 * S::kRowBytes : nullptr;
      if (u == 0)
        slot(tail_tag, exact_tag, std::true_type{}, std::true_type{}, X, qb, P, qo, jc, first, refill);
      else if (u % 2 == 0)
        slot(tail_tag, exact_tag, std::true_type{}, std::false_type{}, X, qb, P, qo, jc, first, refill);
      else
        slot(tail_tag, exact_tag, std::true_type{}, std::false_type{}, P, qb, X, qo, jc, first, refill);
    }
    if (S::kSlots % 2 == 1) P = X;
  };
  auto sweep = [&](auto exact_tag, bool primed) __attribute__((always_inline)) {
    constexpr bool kExact = decltype(exact_tag)::value;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      m[qb] = kExact ? -INFINITY : 0.f;
      z[qb] = 0.f;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) P[r] = -INFINITY;  // nothing pending: adds zeros
    if (!primed) first_tiles();
    // One copy of the tile's code: unrolled over the ring, so that the stage folds into the LDS reads' offsets, the loop itself is
    // no faster and a block of a few tiles waits for instructions (28/4 heads, 30 rows, 5000 keys 17.6 -> 16.8 us for both passes;
    // pass B, unrolled: no difference).
    auto arrive = [&](int i, int st) __attribute__((always_inline)) {
      wait_vmem<(NS - 2) * S::kUnits>();  // tile i has landed when only the younger ones are outstanding
      __syncthreads();                    // everyone's share is visible, and everyone is done with tile i - 1
      loads.issue(src, j_begin + (i + NS - 1) * S::TK, lds0 + (st == 0 ? NS - 1 : st - 1) * S::kStage, wave);
    };
    const bool masked = kExact || own_keys;
    const int n_plain = masked ? 0 : (j_end - j_begin) / S::TK;  // whole tiles, every key counts
    int i = 0, st = 0;
    if (!kExact) {
#pragma unroll 1
      for (; i < n_plain; ++i) {
        arrive(i, st);
        if (active) tile(std::false_type{}, exact_tag, i, k_lds + st * S::kStage);
        st = st + 1 == NS ? 0 : st + 1;
      }
    }
#pragma unroll 1
    for (; i < n_tiles; ++i) {
      arrive(i, st);
      if (active) tile(std::true_type{}, exact_tag, i, k_lds + st * S::kStage);
      st = st + 1 == NS ? 0 : st + 1;
    }
    if (active)
      slot(std::true_type{}, exact_tag, std::false_type{}, std::true_type{}, X, 0, P, QB - 1,
           j_begin + (n_tiles - 1) * S::TK + wk * KT * 32 + 32 * (KT - 1),
           KT == 1 && n_tiles == 1, nullptr);
    wait_vmem<0>();  // drain the look-ahead loads before the LDS is reused or released
  };
  sweep(std::false_type{}, true);
  {
    bool out_of_range = false;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) out_of_range |= !(z[qb] <= 0x1p60f);  // also true for NaN
    if (__syncthreads_or(out_of_range ? 1 : 0)) sweep(std::true_type{}, false);  // uniform over the block
  }
  // Prompt keys whose sum is no number (a NaN, an infinite logit) leave the row without a normaliser: a reference
  // exponent of infinity, which wins every merge, makes each of the row's terms 0 in pass B, so that it adds nothing.
  auto result = [&](float mm, float zz) __attribute__((always_inline)) {
    return own_keys && isnan(zz) ? make_float2(INFINITY, 1.f) : make_float2(mm, zz);
  };
  // Merge the two lane halves (same query row, disjoint keys), then the wavefronts that split the keys.
  float2 *dst = partial + ((static_cast<int64_t>(kb) * gm.n_kv_heads + g) * gm.n_qchunks + qc) * S::kRows;
  float2 *w_stats = reinterpret_cast<float2 *>(k_lds);  // [WK][kRows]
  if (S::WK > 1) __syncthreads();                              // nobody still reads keys
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    // a lane that saw no valid key, or whose terms all vanished against its reference, takes no part
    const float mq = z[qb] > 0.f ? m[qb] : -INFINITY;
    const float mo = __shfl_xor(mq, 32, 64);
    const float zo = __shfl_xor(z[qb], 32, 64);
    const float mm = fmaxf(mq, mo);
    const float mu = fmaxf(mm, -1e30f);
    const float zz = z[qb] * __builtin_amdgcn_exp2f(mq - mu) + zo * __builtin_amdgcn_exp2f(mo - mu);
    const int ql = (wq * QB + qb) * 32 + row;
    if (hf == 0 && active) (S::WK > 1 ? w_stats[wk * S::kRows + ql] : dst[ql]) = S::WK > 1 ? make_float2(mm, zz) : result(mm, zz);
  }
  if (S::WK > 1) {
    __syncthreads();
    if (threadIdx.x < q_rows) {
      float mm = -INFINITY, zz = 0.f;
#pragma unroll
      for (int w = 0; w < S::WK; ++w) {
        const float2 p = w_stats[w * S::kRows + threadIdx.x];
        const float mn = fmaxf(mm, p.x);
        const float mu = fmaxf(mn, -1e30f);
        zz = zz * __builtin_amdgcn_exp2f(mm - mu) + p.y * __builtin_amdgcn_exp2f(p.x - mu);
        mm = mn;
      }
      dst[threadIdx.x] = result(mm, zz);
    }
  }
}

// ---------------------------------------------------------------------------
// pass B
// ---------------------------------------------------------------------------
// Every block merges the per-slice partials of its own query rows first, while its first key tiles are on their
// way.  The per-(kv head, query chunk) column sums go to `colpart`; the block that is the last of a key range to
// finish (counted in `arrived`, which reads zero between launches) adds them up in a fixed order and writes
// the scores.
struct ColsumIo {
  const float2 *partial;
  float *colpart;
  int *arrived;     // [key ranges]
  float *scores;
  float inv_heads;
  int accumulate;
};

// The column sums travel between blocks that sit on different XCDs, whose L2s are not coherent with
// each other: they are written and read with device-scope relaxed atomics (write-through stores,
// loads that do not hit a stale line) instead of cache-wide write-backs and invalidations.
__device__ __forceinline__ void store_coherent(float *p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_coherent(const float *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kMergeBatch = 16;      // partials of a row that are loaded together
constexpr int kSegment = 2048;       // context keys whose sums a block keeps in LDS before it writes them out

template <typename S>
__global__ __launch_bounds__(S::kThreads) __attribute__((amdgpu_waves_per_eu(S::kMinWavesPerSimd, 2))) void score_colsum_mfma(
    const char *__restrict__ k_global, const char *__restrict__ q_prompt, ScoreGeom gm, ColsumIo io) {
  using Tag = typename S::Tag;
  constexpr int QB = S::QB, KT = S::KT, NS = S::NS, STEPS = S::kSteps, WQ = S::WQ;
  constexpr int kPerRow = S::kThreads / S::kRows;  // threads that share a row's partials
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds[S::kLds];
  __shared__ __attribute__((aligned(16))) float m_lds[S::kRows], w_lds[S::kRows];
  __shared__ float2 merge_lds[kPerRow > 1 ? S::kThreads : 1];
  __shared__ float exchange[3][WQ][S::TK];  // column sums of the wavefronts: even tiles, odd tiles, a segment's last tile
  __shared__ float sums[kSegment];
  __shared__ int s_last;
  const BlockPlace at(blockIdx.x, gridDim.x, gm.n_slices, gm.n_qchunks);
  const int kb = at.kb, g = at.g, qc = at.qc;
  const int y = g * gm.n_qchunks + qc;  // which of the column sums' parts this block forms
  const int n_parts = gm.n_kv_heads * gm.n_qchunks;
  const int G = gm.n_q_heads / gm.n_kv_heads;
  const int q_rows = min(gm.q_chunk_rows, gm.m_prompt * G - qc * gm.q_chunk_rows);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wq = S::WK == 1 ? wave : wave % WQ, wk = S::WK == 1 ? 0 : wave / WQ;
  const int row = lane & 31, hf = lane >> 5;
  const float c = gm.scale_log2;
  const int kv_begin = kb * gm.kv_per_block;
  const int kv_end = min(gm.n_ctx, kv_begin + gm.kv_per_block);
  const KeySource src = {k_global + g * gm.head_bytes, gm.token_bytes, gm.n_ctx};
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(k_lds));

  // requests first: partials (other blocks wrote them in the previous launch: they come from memory), query rows, keys
  const int my_row = threadIdx.x % S::kRows, my_part = threadIdx.x / S::kRows;
  const float2 *prow = io.partial + static_cast<int64_t>(y) * S::kRows + min(my_row, q_rows - 1);
  const uint32_t slice_stride = static_cast<uint32_t>(n_parts) * S::kRows;  // (the launch checks the extent of the array)
  auto load_partials = [&](float2 (&p)[kMergeBatch], int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kMergeBatch; ++u) p[u] = prow[static_cast<uint32_t>(min(s0 + u * kPerRow, gm.n_slices - 1)) * slice_stride];
  };
  float2 part[kMergeBatch], own = make_float2(-INFINITY, 0.f);
  load_partials(part, my_part);
  // the prompt's own keys come on top of the slices: as one more among them, the 33rd at 8K keys, they would cost another
  // batch and its latency (64 prompt rows 22.6 -> 22.0 us for both passes)
  if (gm.n_partials > gm.n_slices && my_part == 0) own = prow[static_cast<uint32_t>(gm.n_slices) * slice_stride];
  const TileLoads<S> loads(src, lane, wave);
  v4u qf[QB][STEPS];
  load_queries<S>(qf, k_lds, q_prompt, gm, g, qc, q_rows, wq, [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NS - 1; ++t) loads.issue(src, kv_begin + t * S::TK, lds0 + t * S::kStage, wave);
  });
  {
    float m = own.y > 0.f ? own.x : -INFINITY, z = own.y > 0.f ? own.y : 0.f;
    for (int s0 = my_part; s0 < gm.n_slices; s0 += kMergeBatch * kPerRow) {
      if (s0 != my_part) load_partials(part, s0);
      float mn = m;
#pragma unroll
      for (int u = 0; u < kMergeBatch; ++u)
        if (s0 + u * kPerRow < gm.n_slices && part[u].y > 0.f) mn = fmaxf(mn, part[u].x);
      if (mn > -INFINITY) {
        float acc = z * __builtin_amdgcn_exp2f(fminf(m - mn, 0.f));  // (1 where both are infinite)
#pragma unroll
        for (int u = 0; u < kMergeBatch; ++u) {
          const float w = s0 + u * kPerRow < gm.n_slices && part[u].y > 0.f ? part[u].y : 0.f;
          acc += w * __builtin_amdgcn_exp2f(fminf(part[u].x - mn, 0.f));
        }
        z = acc;
        m = mn;
      }
    }
    if (kPerRow > 1) {
      merge_lds[threadIdx.x] = make_float2(m, z);
      __syncthreads();
      if (my_part == 0) {
#pragma unroll
        for (int w = 1; w < kPerRow; ++w) {
          const float2 p = merge_lds[w * S::kRows + my_row];
          const float mn = fmaxf(m, p.x);
          const float mu = fmaxf(mn, -1e30f);
          z = z * __builtin_amdgcn_exp2f(m - mu) + p.y * __builtin_amdgcn_exp2f(p.x - mu);
          m = mn;
        }
      }
    }
    if (my_part == 0) {
      const bool counts = my_row < q_rows && z > 0.f;
      m_lds[my_row] = counts ? m : INFINITY;  // padded rows add exp2(-inf) = 0
      w_lds[my_row] = counts ? 1.f / z : 0.f;
    }
  }
  __syncthreads();
  // register r of a product: query row 8 (r/4) + 4 hf + r%4 of the block, key `row` of the subtile
  f32x4 mq[QB][4], wgt[QB][4];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb)
#pragma unroll
    for (int ri = 0; ri < 4; ++ri) {
      mq[qb][ri] = *reinterpret_cast<const f32x4 *>(&m_lds[(wq * QB + qb) * 32 + 8 * ri + 4 * hf]);
      wgt[qb][ri] = *reinterpret_cast<const f32x4 *>(&w_lds[(wq * QB + qb) * 32 + 8 * ri + 4 * hf]);
    }
  const int n_wq = (q_rows + QB * 32 - 1) / (QB * 32);  // wavefronts along the rows that hold any
  const bool active = wq < n_wq;
  const KeyReads<S> kr(lane, wk);
  wait_vmem<0>();

  float *const dst = io.colpart + static_cast<int64_t>(y) * gm.n_ctx;
  v4u kf[STEPS];
  float col[KT];
  f32x16 X, P;
  // One slot, as in pass A: the MFMAs of a new product in slices, each preceded by a share of the exponentials of
  // the finished one.
  auto slot = [&](auto product_tag, auto vector_first_tag, f32x16 &N, int qn, const f32x16 &C, int qo, float &sum,
                  const unsigned char *refill) __attribute__((always_inline)) {
    constexpr bool kProduct = decltype(product_tag)::value, kVectorFirst = decltype(vector_first_tag)::value;
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto product = [&](int s) __attribute__((always_inline)) {
      if (kProduct) {
        N = mma(Tag{}, qf[qn][s], kf[s], s == 0 ? zero : N);
        if (refill != nullptr) kf[s] = kr.read(refill, s);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      if (!kVectorFirst) product(s);
#pragma unroll
      for (int r = 16 * s / STEPS; r < 16 * (s + 1) / STEPS; ++r)
        sum = fmaf(__builtin_amdgcn_exp2f(fmaf(C[r], c, -mq[qo][r >> 2][r & 3])), wgt[qo][r >> 2][r & 3], sum);
      asm volatile("" : "+v"(sum));
      if (kVectorFirst) product(s);
    }
  };
  // the finished sums of a tile, both lane halves added, to this wavefront's row of the exchange buffer
  auto publish = [&](int buffer) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      const float v = col[t] + __shfl_xor(col[t], 32, 64);
      if (hf == 0) exchange[buffer][wq][(wk * KT + t) * 32 + row] = v;
      col[t] = 0.f;
    }
  };
  auto collect = [&](int i, int buffer) __attribute__((always_inline)) {
    if (threadIdx.x < S::TK) {
      float v = 0.f;
      for (int w = 0; w < n_wq; ++w) v += exchange[buffer][w][threadIdx.x];
      sums[i * S::TK + threadIdx.x] = v;
    }
  };
  // The products of a tile in the order (subtile, query block); the last one is absorbed by the first slot of
  // the next tile, after which the tile's sums are published; they are collected after the barrier after that.  The last tile of a
  // segment has no next one: its sums are published without a barrier between them and the collection of the tile two before,
  // which other wavefronts may still be at, so they have a buffer of their own.
  auto tile = [&](int i, const unsigned char *stage) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < STEPS; ++s) kf[s] = kr.read(stage, s);
#pragma unroll
    for (int u = 0; u < S::kSlots; ++u) {
      const int t = u / QB, qb = u % QB;
      const int qo = u == 0 ? QB - 1 : (u - 1) % QB;
      const int to = u == 0 ? KT - 1 : (u - 1) / QB;
      const unsigned char *refill = (qb == QB - 1 && t + 1 < KT) ? stage + (t + 1) * 32 * S::kRowBytes : nullptr;
      if (u == 0)
        slot(std::true_type{}, std::true_type{}, X, qb, P, qo, col[to], refill);
      else if (u % 2 == 0)
        slot(std::true_type{}, std::false_type{}, X, qb, P, qo, col[to], refill);
      else
        slot(std::true_type{}, std::false_type{}, P, qb, X, qo, col[to], refill);
      if (u == 0 && i > 0) publish((i - 1) & 1);
    }
    if (S::kSlots % 2 == 1) P = X;
  };
  for (int seg = kv_begin; seg < kv_end; seg += kSegment) {
    const int seg_end = min(kv_end, seg + kSegment);
    const int n_tiles = (seg_end - seg + S::TK - 1) / S::TK;
    if (seg != kv_begin) {
#pragma unroll
      for (int t = 0; t < NS - 1; ++t) loads.issue(src, seg + t * S::TK, lds0 + t * S::kStage, wave);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) P[r] = -INFINITY;  // nothing pending: adds zeros
#pragma unroll
    for (int t = 0; t < KT; ++t) col[t] = 0.f;
    auto step = [&](int i, int st) __attribute__((always_inline)) {
      wait_vmem<(NS - 2) * S::kUnits>();
      __syncthreads();
      loads.issue(src, seg + (i + NS - 1) * S::TK, lds0 + (st == 0 ? NS - 1 : st - 1) * S::kStage, wave);
      if (i >= 2) collect(i - 2, i & 1);
      if (active) tile(i, k_lds + st * S::kStage);
    };
    for (int i0 = 0; i0 < n_tiles; i0 += NS) {
#pragma unroll
      for (int st = 0; st < NS; ++st)
        if (i0 + st < n_tiles) step(i0 + st, st);
    }
    if (active) {
      slot(std::false_type{}, std::true_type{}, X, 0, P, QB - 1, col[KT - 1], nullptr);
      publish(2);
    }
    wait_vmem<0>();  // drain the look-ahead loads before the stages are filled again or released
    __syncthreads();
    if (n_tiles >= 2) collect(n_tiles - 2, n_tiles & 1);
    collect(n_tiles - 1, 2);
    __syncthreads();
    for (int j = seg + threadIdx.x; j < seg_end; j += S::kThreads) store_coherent(&dst[j], sums[j - seg]);
  }
  // This block's column sums have reached memory when its stores have completed; the block that
  // completes the count of its key range adds up all partials of the range.
  wait_vmem<0>();
  __syncthreads();
  if (threadIdx.x == 0) {
    const int done = __hip_atomic_fetch_add(&io.arrived[kb], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    s_last = done == n_parts ? 1 : 0;
    if (done == n_parts) __hip_atomic_store(&io.arrived[kb], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (s_last != 0) {
    constexpr int kBatch = 16;  // partial sums requested together
    for (int j = kv_begin + threadIdx.x; j < kv_end; j += S::kThreads) {
      float sum = 0.f;
      for (int p0 = 0; p0 < n_parts; p0 += kBatch) {
        float v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
          v[u] = load_coherent(&io.colpart[static_cast<int64_t>(min(p0 + u, n_parts - 1)) * gm.n_ctx + j]);
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
          if (p0 + u < n_parts) sum += v[u];
      }
      sum *= io.inv_heads;
      io.scores[j] = io.accumulate ? io.scores[j] + sum : sum;
    }
  }
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
template <typename S>
hipError_t run(ifkv_ctx *ctx, ScoreGeom gm, const char *k_global, const char *q_prompt, const char *k_prompt,
               int accumulate, float *scores) {
  const auto &d = ctx->desc;
  const int rows = gm.m_prompt * (gm.n_q_heads / gm.n_kv_heads);
  gm.n_qchunks = (rows + S::kRows - 1) / S::kRows;
  gm.q_chunk_rows = std::min(S::kRows, ((rows + gm.n_qchunks - 1) / gm.n_qchunks + 31) / 32 * 32);
  const int per_slice = d.n_kv_heads * gm.n_qchunks;
  // One round of blocks at two wavefronts per SIMD; a block owns whole tiles.  Blocks of four wavefronts: with fewer
  // than four tiles per block, half as many blocks (one wavefront per SIMD) are better, because a block's query rows,
  // partial results and column sums cost as much as two or three tiles (8K context, 256 query rows per kv head: 20.9
  // against 24.8 us for both passes with 64 slices of two tiles; at 16K, four tiles, 30.8 against 31.6).
  int slices = std::min(kScoreMaxKeyRanges, std::max(1, 256 * 8 / S::kWaves / per_slice));
  if (S::kWaves == 4 && gm.n_ctx < slices * S::TK * 4) slices = std::max(1, slices / 2);
  const int max_slices = (gm.n_ctx + S::TK - 1) / S::TK;
  slices = std::min(slices, max_slices);
  int per = (gm.n_ctx + slices - 1) / slices;
  per = (per + S::TK - 1) / S::TK * S::TK;
  slices = (gm.n_ctx + per - 1) / per;
  gm.kv_per_block = per;
  gm.n_slices = slices;
  gm.n_partials = slices + (k_prompt != nullptr ? 1 : 0);

  const ScoreScratch sc = score_scratch_layout(ctx, gm.n_ctx, gm.m_prompt);
  char *base = static_cast<char *>(ctx->scratch);
  float2 *partial = reinterpret_cast<float2 *>(base + sc.partial_off);
  // host-side bounds: the partial results must fit what was allocated
  if (ctx->score_arrived == nullptr || gm.n_qchunks > kMaxQChunks || slices > kScoreMaxKeyRanges ||
      static_cast<size_t>(gm.n_partials) * per_slice * S::kRows * sizeof(float2) > sc.colpart_off - sc.partial_off)
    return hipErrorInvalidValue;
  ColsumIo io;
  io.partial = partial;
  io.colpart = reinterpret_cast<float *>(base + sc.colpart_off);
  io.arrived = ctx->score_arrived;
  io.scores = scores;
  io.inv_heads = 1.0f / d.n_q_heads;
  io.accumulate = accumulate;
  hipLaunchKernelGGL((score_stats_mfma<S>), dim3(gm.n_partials * per_slice), dim3(S::kThreads), 0, ctx->stream, k_global,
                     k_prompt, q_prompt, gm, partial);
  hipLaunchKernelGGL((score_colsum_mfma<S>), dim3(slices * per_slice), dim3(S::kThreads), 0, ctx->stream, k_global, q_prompt,
                     gm, io);
  return hipGetLastError();
}

// Query rows of a kv head go to blocks of 32, 128, 256 or 512 rows (at most kMaxQChunks of them).  The larger the
// block, the fewer times its keys are staged; the smaller, the fewer rows are padding.
template <typename Tag, int D>
hipError_t run_sized(ifkv_ctx *ctx, const ScoreGeom &gm, const char *k, const char *q, const char *kp, int accumulate,
                     float *scores) {
  constexpr int QB = D * Elem<Tag>::kBytes > 256 ? 1 : 2;  // 512-byte rows: one query block fills the operand registers
  constexpr int NS = D * Elem<Tag>::kBytes > 256 ? 2 : 3;
  const int rows = gm.m_prompt * (gm.n_q_heads / gm.n_kv_heads);
  auto padded = [&](int size) {
    const int n = (rows + size - 1) / size;
    return n <= kMaxQChunks ? n * size : 1 << 28;
  };
  if (rows <= 32) return run<Shape<Tag, D, 1, 1, 4, 2>>(ctx, gm, k, q, kp, accumulate, scores);
  const int big = padded(QB * 256), mid = padded(QB * 128), small = padded(QB * 64);
  if (small + small / 12 < mid && small + small / 12 < big)
    return run<Shape<Tag, D, QB, 2, 2, NS>>(ctx, gm, k, q, kp, accumulate, scores);
  if (mid < big) return run<Shape<Tag, D, QB, 4, 1, NS>>(ctx, gm, k, q, kp, accumulate, scores);
  return run<Shape<Tag, D, QB, 8, 1, NS>>(ctx, gm, k, q, kp, accumulate, scores);
}

}  // namespace

bool score_mfma_supported(const ifkv_ctx *ctx, int m_prompt) {
  const auto &d = ctx->desc;
  const int64_t rows = static_cast<int64_t>(m_prompt) * (d.n_q_heads / d.n_kv_heads);
  const int64_t e = static_cast<int64_t>(dtype_size(d.dtype));
  const int largest = d.dtype == IFKV_F32 && d.head_dim == 128 ? 256 : 512;  // query rows of the largest block
  return m_prompt > 0 && rows <= static_cast<int64_t>(kMaxQChunks) * largest &&
         ctx->token_stride * e <= int64_t(1) << 25 && static_cast<int64_t>(m_prompt) * d.n_q_heads * d.head_dim * e < int64_t(1) << 32;  // 32-bit offsets
}

hipError_t launch_score_mfma(ifkv_ctx *ctx, const void *k_global, int64_t n_ctx, const void *q_prompt, int m_prompt,
                             const void *k_prompt, int accumulate, float *scores) {
  const auto &d = ctx->desc;
  const int64_t e = static_cast<int64_t>(dtype_size(d.dtype));
  ScoreGeom gm = {};
  gm.n_ctx = static_cast<int>(n_ctx);
  gm.m_prompt = m_prompt;
  gm.n_q_heads = d.n_q_heads;
  gm.n_kv_heads = d.n_kv_heads;
  gm.scale_log2 = static_cast<float>(ctx->sm_scale * kLog2e);  // rounded once
  gm.token_bytes = ctx->token_stride * e;
  gm.head_bytes = ctx->head_stride * e;
  const char *k = static_cast<const char *>(k_global), *q = static_cast<const char *>(q_prompt),
             *kp = static_cast<const char *>(k_prompt);
  if (d.dtype == IFKV_BF16)
    return d.head_dim == 128 ? run_sized<BF16Tag, 128>(ctx, gm, k, q, kp, accumulate, scores)
                             : run_sized<BF16Tag, 64>(ctx, gm, k, q, kp, accumulate, scores);
  return d.head_dim == 128 ? run_sized<F32Tag, 128>(ctx, gm, k, q, kp, accumulate, scores)
                           : run_sized<F32Tag, 64>(ctx, gm, k, q, kp, accumulate, scores);
}

}  // namespace ifkv
