// Stage 4, bf16 MFMA kernels -- "KV Recomputation": each selected row attends
// causally to cache rows 0..p_r of the concatenated sequence.
//
// Shape of the problem: few, scattered query rows (k = rho N of them) against a
// long, dense K/V prefix.  The kernel therefore packs the G query heads that
// share a kv head together with a block of consecutive selected rows into one
// "row block" of 128 query columns, so that every K/V tile fetched from HBM/L2
// is used by all of them, and walks the kv axis in tiles of 64 rows with an
// online softmax (flash-attention style).  Rows are sorted by position, so only
// the last one or two kv tiles of a wavefront need the causal mask.
//
// Two kernels: attn_mfma_kernel (128 query columns per workgroup, two workgroups per CU) and, for large launches,
// attn_wide_kernel (256 columns, one per CU), described there.  wide_jobs says which serves a launch.
//
// Per wavefront (32 query columns), per kv tile, with 32x32x16 bf16 MFMAs:
//   S^T [64 kv x 32 q]  = K_tile . Q^T         (A = K rows from LDS, B = Q in registers)
//   P^T = exp2(S^T * c - m)                     (fp32, per-lane statistics: a lane owns one query column)
//   O^T [128 d x 32 q] += V_tile^T . P^T       (A = V^T from LDS, B = P^T straight from the S^T registers)
// Computing the transposed products keeps each query column in one lane (two
// lanes, one per half-wave), so a column's statistics need at most one
// cross-lane exchange per tile, and the S^T accumulator layout is exactly the
// B-operand layout of the second product once the K rows are fed in a fixed
// permuted order (sigma below): no LDS round trip for P.  The reference
// exponent m is, in the first sweep, the logit of the sweep's first key (kept
// for the whole sweep: no maximum, no exchange, no rescaling); a second sweep
// with a running maximum follows where the first is not accepted (see the kernel).
// Staging uses the gfx950 direct global->LDS loads (16 bytes per lane, no registers, no VALU) and
// keeps NS tiles in an LDS ring.  K rows land in sigma order with their 16-byte chunks XOR-swizzled
// by the row index, so the A-operand reads (32 rows, one chunk) hit distinct banks.  V lands
// row-major, swizzled by the row within each group of four rows, and the A operand of the second
// product -- which needs eight kv values of one d column per lane, the strided axis -- is read
// with the LDS transpose loads (ds_read_b64_tr_b16), two per operand.
//
// Work distribution.  One workgroup per (kv head, row block), dispatched longest row block first,
// so that the short ones fill the end of the launch; all workgroups of a head start at tile 0 and
// walk the kv axis together, which lets the L2 serve most tile fetches (0.8 GB reach the fabric per
// launch at 32K context; cutting the blocks' tiles into equal contiguous shares per workgroup
// instead, which balances the launch perfectly on paper, sends 6.8 GB through the fabric and is
// slower).  Launches with fewer row blocks than the chip has workgroup slots are cut along the kv
// axis: each part leaves its unnormalised O, reference max and sum in scratch and
// attn_merge_kernel merges them.
#include <algorithm>
#include <type_traits>

#include "attention_tile.h"
#include "lds_dma.h"

namespace ifkv {

namespace {

constexpr int D = 128;        // head_dim served by these kernels
constexpr int TK = kKvTile;   // kv rows per tile
constexpr int TILE_ELEMS = TK * D;  // one K or V tile in LDS: 64 rows x 256 B, no padding (swizzled instead)
// Everything one wavefront carries through the kv loop.
struct WaveState {
  f32x16 O[4];   // O^T accumulator, 128 d x 32 q
  float m_run;   // reference max of the scaled logits (log2 domain); may lag the true max by <= kSlack
  float l_run;   // this lane's share of the running sum
};

// Per-lane LDS read offsets (in elements) that do not change from tile to tile.
struct ReadOffsets {
  int k[8];  // K A-operand, contraction step s: row (lane & 31), chunk (2 s + hf) ^ (row & 15)
  int v[4];  // V transpose read, d tile dt (see pv_tile)
};

__device__ __forceinline__ ReadOffsets make_read_offsets(int lane) {
  ReadOffsets o;
  const int col = lane & 31, hf = lane >> 5;
#pragma unroll
  for (int s = 0; s < 8; ++s) o.k[s] = col * D + (((2 * s + hf) ^ (col & 15)) << 3);
  // transpose read: in every group of 16 lanes, lane j supplies row j / 4, d columns 4 (j % 4)..+3
  // (8 bytes) and receives the four rows of d column j.  Group g covers d columns 16 (g & 1)..+15
  // of the 32-column d tile; hf = g / 2 selects kv rows +8.
  const int g = lane >> 4, j = lane & 15;
  const int r = j >> 2;
  const int low = 2 * (g & 1) + ((j & 3) >> 1);  // 16-byte chunk within the d tile's four chunks
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
    o.v[dt] = (2 * hf) * 512 + ((16 * r + ((4 * dt + low) ^ (4 * r))) << 3) + 4 * (j & 1);
  return o;
}

// S^T = K_tile . Q^T for one 64-row tile held in LDS stage `k_stage`.  An MFMA takes 32 cycles, an
// LDS read returns after a few hundred when eight wavefronts share the LDS, so the A operands are
// requested four contraction steps (eight reads) ahead of their use; the fences keep the
// compiler from sinking the reads back next to their consumers.
__device__ __forceinline__ void qk_tile(f32x16 (&S)[2], const uint16_t *k_stage, const bf16x8 (&qf)[8],
                                        const ReadOffsets &ro) {
  v4u ka[8], kb[8];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    ka[s] = *reinterpret_cast<const v4u *>(&k_stage[ro.k[s]]);
    kb[s] = *reinterpret_cast<const v4u *>(&k_stage[ro.k[s] + 32 * D]);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    S[0][r] = 0.f;
    S[1][r] = 0.f;
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    S[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ka[s]), qf[s], S[0], 0, 0, 0);
    S[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kb[s]), qf[s], S[1], 0, 0, 0);
    if (s + 4 < 8) {
      ka[s + 4] = *reinterpret_cast<const v4u *>(&k_stage[ro.k[s + 4]]);
      kb[s + 4] = *reinterpret_cast<const v4u *>(&k_stage[ro.k[s + 4] + 32 * D]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Causal mask (only on tiles that reach past the wavefront's smallest position) and, in the exact
// variant, the row max with the lazy update of the reference max and the rescale of O and l it
// implies.  The fast variant keeps the reference it was given (see the kernel): nothing but the mask.
// Register r of S[t] is kv row j0 + 32 t + 16 (r / 8) + 8 hf + r % 8.
template <bool EXACT>
__device__ __forceinline__ void row_stats(f32x16 (&S)[2], WaveState &w, int j0, int p_q, int p_wmin, int hf,
                                          float scale_log2) {
  if (j0 + TK - 1 > p_wmin) {
    const int base = j0 + 8 * hf - p_q;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (base + 32 * t + 16 * (r >> 3) + (r & 7) > 0) S[t][r] = -INFINITY;
  }
  if (!EXACT) return;
  float mx = S[0][0];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, S[t][r]);
  mx = half_swap_max(mx);
  const float m_new = fmaxf(w.m_run, mx * scale_log2);
  if (__any(m_new > w.m_run + kSlack)) {
    const float alpha = __builtin_amdgcn_exp2f(w.m_run - m_new);  // 0 when m_run is still kNoMax, 1 when neither moved
    w.l_run *= alpha;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) w.O[dt][r] *= alpha;
    w.m_run = m_new;
  }
}

// P^T of one tile, rounded to bf16 and packed as the four B operands of the second product.
struct PTile {
  v4u step[4];  // contraction step u: kv rows 16 u + 8 hf + 0..7 of this lane's query column
};

// P^T = exp2(S^T c - m) and l += sum P (fp32, before rounding).
__device__ __forceinline__ void exp_tile(f32x16 (&S)[2], WaveState &w, PTile &P, float scale_log2) {
  float psum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      S[t][r] = __builtin_amdgcn_exp2f(fmaf(S[t][r], scale_log2, -w.m_run));
      psum[r & 3] += S[t][r];
    }
  w.l_run += (psum[0] + psum[1]) + (psum[2] + psum[3]);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int t = u >> 1, r0 = 8 * (u & 1);
    P.step[u][0] = pack_bf16x2(S[t][r0 + 0], S[t][r0 + 1]);
    P.step[u][1] = pack_bf16x2(S[t][r0 + 2], S[t][r0 + 3]);
    P.step[u][2] = pack_bf16x2(S[t][r0 + 4], S[t][r0 + 5]);
    P.step[u][3] = pack_bf16x2(S[t][r0 + 6], S[t][r0 + 7]);
  }
}

// O^T += V_tile^T . P^T.  The A operand of contraction step u, d tile dt is lane (d = 32 dt + lane % 32)
// x kv rows 16 u + 8 hf + 0..7: two transpose reads of four rows each from the row-major V tile.
// The sixteen operands are numbered x = 4 u + dt and requested four ahead; the first four are
// requested by pv_preload, which the caller places before the exponentials (they do not depend on
// them), so that they arrive while the vector ALU is busy.
struct VFrags {
  s16x4 lo[4], hi[4];
};
__device__ __forceinline__ void v_read(s16x4 &lo, s16x4 &hi, const uint16_t *v_stage, const ReadOffsets &ro, int x) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const uint16_t *p = v_stage + ro.v[x & 3] + (4 * (x >> 2)) * 512;  // 4-row groups 4 u + 2 hf (+1)
  lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
  hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 512));
}
__device__ __forceinline__ void pv_preload(VFrags &f, const uint16_t *v_stage, const ReadOffsets &ro) {
#pragma unroll
  for (int x = 0; x < 4; ++x) v_read(f.lo[x], f.hi[x], v_stage, ro, x);
}
__device__ __forceinline__ void pv_tile(const PTile &P, VFrags &f, WaveState &w, const uint16_t *v_stage,
                                        const ReadOffsets &ro) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int x = 0; x < 16; ++x) {
    const int u = x >> 2, dt = x & 3;
    const s16x8 a = __builtin_shufflevector(f.lo[x & 3], f.hi[x & 3], 0, 1, 2, 3, 4, 5, 6, 7);
    w.O[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                      __builtin_bit_cast(bf16x8, P.step[u]), w.O[dt], 0, 0, 0);
    if (x + 4 < 16) v_read(f.lo[x & 3], f.hi[x & 3], v_stage, ro, x + 4);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Direct global->LDS staging of one kv tile.  A load instruction moves 64 x 16 bytes: lane L's
// 16 bytes land at the instruction's LDS base + 16 L, whatever global address the lane names, so
// a "unit" of 1 KiB = four 256-byte tile rows is filled per instruction and the lanes choose which
// chunk goes where.  K unit q: LDS rows 4q..4q+3 hold kv rows sigma(4q..4q+3); position c of a row
// holds chunk c ^ (row & 15).  V unit q: kv rows 4q..4q+3; position c of row r holds chunk c ^ 4r.
template <int NWAVES>
struct Dma {
  static constexpr int UPW = 16 / NWAVES;   // units per wavefront and matrix (2 or 4)
  static constexpr int PER_TILE = 2 * UPW;  // load instructions a wavefront issues per tile
};

// What a lane fetches for each of its units, as byte offsets from the tile's first row: fixed for
// the whole kernel, so a tile that lies fully inside the cache costs one scalar base update and
// PER_TILE load instructions, no vector arithmetic.
template <int NWAVES>
struct DmaPlan {
  uint32_t k_off[Dma<NWAVES>::UPW];
  uint32_t v_off[Dma<NWAVES>::UPW];
};

template <int NWAVES>
__device__ __forceinline__ DmaPlan<NWAVES> make_dma_plan(int64_t kv_row_elems) {
  DmaPlan<NWAVES> pl;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane >> 4, cpos = lane & 15;
  const uint32_t row_bytes = static_cast<uint32_t>(kv_row_elems) * 2u;
#pragma unroll
  for (int x = 0; x < Dma<NWAVES>::UPW; ++x) {
    const int i = 4 * (wave * Dma<NWAVES>::UPW + x) + r;  // LDS row
    pl.k_off[x] = sigma(i) * row_bytes + 16u * (cpos ^ (i & 15));
    pl.v_off[x] = i * row_bytes + 16u * (cpos ^ (4 * r));
  }
  return pl;
}

// k_stage / v_stage: wavefront-uniform LDS byte addresses of the stage to fill (plain integers, so
// the per-instruction LDS base is scalar arithmetic and costs no vector instruction)
template <int NWAVES>
__device__ __forceinline__ void issue_tile_dma(const DmaPlan<NWAVES> &pl, uint32_t k_stage, uint32_t v_stage,
                                               const uint16_t *k_base, const uint16_t *v_base, int64_t kv_row_elems,
                                               int tile, int n_kv) {
  const uint32_t unit0 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * Dma<NWAVES>::UPW;
  int j0 = tile * TK;
  const bool partial = (j0 < n_kv && j0 + TK > n_kv) || n_kv < TK;
  if (!partial) {
    if (j0 >= n_kv) j0 = 0;  // look-ahead past the end: fetch any valid tile, it is never read
    const uint16_t *kb = k_base + j0 * kv_row_elems;
    const uint16_t *vb = v_base + j0 * kv_row_elems;
#pragma unroll
    for (int x = 0; x < Dma<NWAVES>::UPW; ++x) {
      dma16_base(kb, pl.k_off[x], k_stage + (unit0 + x) * 1024u);
      dma16_base(vb, pl.v_off[x], v_stage + (unit0 + x) * 1024u);
    }
  } else {
    // the one tile that straddles the end of the cache: rows past the end are clamped (and masked later)
    const int lane = threadIdx.x & 63;
    const int r = lane >> 4, cpos = lane & 15;
#pragma unroll
    for (int x = 0; x < Dma<NWAVES>::UPW; ++x) {
      const uint32_t unit = unit0 + x;
      const int i = 4 * unit + r;
      const int jk = min(j0 + sigma(i), n_kv - 1);
      const int jv = min(j0 + i, n_kv - 1);
      dma16(k_base + jk * kv_row_elems + 8 * (cpos ^ (i & 15)), k_stage + unit * 1024u);
      dma16(v_base + jv * kv_row_elems + 8 * (cpos ^ (4 * r)), v_stage + unit * 1024u);
    }
  }
}

__device__ __forceinline__ void load_q_frags(bf16x8 (&qf)[8], const uint16_t *__restrict__ q_sel, const Column &c,
                                             int hf) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    v4u x = *reinterpret_cast<const v4u *>(q_sel + c.q_row * D + 16 * s + 8 * hf);
    if (!c.col_valid) x = v4u{0u, 0u, 0u, 0u};
    qf[s] = __builtin_bit_cast(bf16x8, x);
  }
}

// ---------------------------------------------------------------------------
// NWAVES wavefronts, ring of NS LDS stages filled by direct global->LDS loads NS-1 tiles ahead.
// ---------------------------------------------------------------------------
template <int NWAVES, int NS>
__global__ __launch_bounds__(NWAVES * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_mfma_kernel(
    const uint16_t *__restrict__ q_sel, const int32_t *__restrict__ row_pos, int n_rows,
    const uint16_t *__restrict__ k_cache, const uint16_t *__restrict__ v_cache, int n_kv,
    uint16_t *__restrict__ out, float *__restrict__ lse_out, int n_q_heads, int n_kv_heads, float scale_log2,
    int rows_per_block, CacheLayout lay, SplitPlan sp) {
  __shared__ __attribute__((aligned(1024))) uint16_t k_lds[NS][TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) uint16_t v_lds[NS][TILE_ELEMS];
  __shared__ int pos_lds[NWAVES][kBlockColumns];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hf = lane >> 5;
  const int G = sp.group_size;
  const int g = blockIdx.x;
  const int rb = gridDim.y - 1 - blockIdx.y;  // longest prefixes are dispatched first
  const int part = blockIdx.z;
  // this workgroup's share of the kv axis: tiles t0 .. t1-1 (the whole range unless the block is split)
  const int t0 = part * sp.part_tiles;
  const int64_t kv_row_elems = lay.token_stride;
  const uint16_t *k_base = k_cache + g * lay.head_stride;
  const uint16_t *v_base = v_cache + g * lay.head_stride;
  const auto plan = make_dma_plan<NWAVES>(kv_row_elems);
  const uint32_t k_lds_addr = __builtin_amdgcn_readfirstlane(lds_address(&k_lds[0][0]));
  const uint32_t v_lds_addr = __builtin_amdgcn_readfirstlane(lds_address(&v_lds[0][0]));
  constexpr uint32_t kStageBytes = TILE_ELEMS * 2;
  // Tiles t0 .. t0+NS-2 are requested up front; iteration i requests tile i + NS - 1 (rows past the
  // end are clamped, the data is never used), so exactly NS-1 tiles are in flight at every wait.
  auto request_first = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < NS - 1; ++t)
      issue_tile_dma<NWAVES>(plan, k_lds_addr + t * kStageBytes, v_lds_addr + t * kStageBytes, k_base, v_base,
                             kv_row_elems, t0 + t, n_kv);
  };
  static_assert(NWAVES == 4, "columns of a row block, queries in the last ring stage");
  const QueryLoads<2 * D> queries = {rb * rows_per_block, n_rows, rows_per_block, G, n_q_heads, sp.group_magic};
  uint16_t *q_lds = (wave < 2 ? k_lds[NS - 1] : v_lds[NS - 1]) + (wave & 1) * 32 * D;
  queries.request_positions(row_pos, __builtin_amdgcn_readfirstlane(lds_address(pos_lds[wave])));
  queries.request(reinterpret_cast<const char *>(q_sel), g, wave, __builtin_amdgcn_readfirstlane(lds_address(q_lds)),
                  [](int i) __attribute__((always_inline)) { return i & 15; });
  request_first();
  wait_vmem<QueryLoads<2 * D>::kUnits + (NS - 1) * Dma<NWAVES>::PER_TILE>();  // the positions have landed
  int p_bmax;
  Column c = queries.column(pos_lds[wave], g, wave, n_kv, &p_bmax);
  const int n_tiles = p_bmax / TK + 1;
  const int t1 = min(n_tiles, t0 + sp.part_tiles);
  if (t0 >= n_tiles) {  // nothing left for this part (uniform over the workgroup)
    wait_vmem<0>();     // before the LDS is given back
    return;
  }
  const bool split = n_tiles > sp.part_tiles;
  if (part == 0 && g == 0 && threadIdx.x == 0 && sp.block_parts != nullptr)
    sp.block_parts[rb] = (n_tiles + sp.part_tiles - 1) / sp.part_tiles;
  const ReadOffsets ro = make_read_offsets(lane);
  wait_vmem<(NS - 1) * Dma<NWAVES>::PER_TILE>();  // the wavefront's own queries have landed
  bf16x8 qf[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    v4u x = *reinterpret_cast<const v4u *>(&q_lds[ro.k[s]]);
    if (!c.col_valid) x = v4u{0u, 0u, 0u, 0u};
    qf[s] = __builtin_bit_cast(bf16x8, x);
  }

  WaveState w;
  const int my_tiles = min(t1, c.p_wmax / TK + 1);
  // The sweep over this workgroup's kv tiles, in two variants.  The softmax only needs SOME reference
  // exponent per query column that keeps exp2(logit - reference) inside the fp32 / bf16 range, not the
  // column maximum.  The fast variant takes the logit of the first key of the sweep (key t0 * 64: the
  // reference of both lane halves of a column, which feed one product) and keeps it: no maximum over
  // the tile, no lane-half exchange, no rescaling of O, ever (2.3 % of the launch at 32K context).
  // It is accepted when every column's sum stays below 4096 x the keys of the sweep, i.e. when no key
  // outweighs the first one by more than that: flat and moderately peaked attention.  Otherwise --
  // sharply peaked columns, where the running maximum makes the dominant probability exactly 1 and
  // thereby free of rounding error, and sums on their way out of the fp32 range -- the whole
  // workgroup repeats the sweep in the exact variant, which tracks the running maximum (lazily: O is
  // rescaled only when a tile exceeds the reference by more than 2^8).
  auto sweep = [&](auto exact_tag, bool requested) __attribute__((always_inline)) {
    constexpr bool kExact = decltype(exact_tag)::value;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) w.O[dt][r] = 0.f;
    w.m_run = kNoMax;
    w.l_run = 0.f;

    if (!requested) request_first();

    // One tile.  `st` is a compile-time constant at every call (the loop below is unrolled over the
    // ring), so the LDS stage base folds into the immediate offset of every LDS read and the reads
    // cost no address arithmetic.
    auto tile_step = [&](int i, int st) __attribute__((always_inline)) {
      // this wavefront's share of tile i has landed when at most the NS-2 younger tiles are outstanding
      // (loads complete in order; the query loads issued before them are therefore complete too)
      __builtin_amdgcn_s_waitcnt(0x0F70 | ((NS - 2) * Dma<NWAVES>::PER_TILE));
      __syncthreads();  // everyone's share is visible, and everyone is done with tile i-1
      {
        const int wr = (st == 0) ? NS - 1 : st - 1;  // the stage tile i-1 occupied
        issue_tile_dma<NWAVES>(plan, k_lds_addr + wr * kStageBytes, v_lds_addr + wr * kStageBytes, k_base, v_base,
                               kv_row_elems, i + NS - 1, n_kv);
      }
      if (i < my_tiles) {  // otherwise this wavefront's rows end before the tile (it still stages and syncs)
        f32x16 S[2];
        qk_tile(S, k_lds[st], qf, ro);
        wave_priority<1>();
        VFrags vf;
        pv_preload(vf, v_lds[st], ro);
        if (!kExact && i == t0) {
          // register 0 of the lower lane half is key t0 * 64 (before the mask: a real key's logit even
          // for a column that does not see it); the upper half takes it from its partner lane
          w.m_run = __shfl(S[0][0], lane & 31, 64) * scale_log2;
        }
        row_stats<kExact>(S, w, i * TK, c.p_q, c.p_wmin, hf, scale_log2);
        PTile P;
        exp_tile(S, w, P, scale_log2);
        wave_priority<2>();
        pv_tile(P, vf, w, v_lds[st], ro);
        wave_priority<0>();
      }
    };
    for (int i0 = t0; i0 < t1; i0 += NS) {
#pragma unroll
      for (int st = 0; st < NS; ++st)
        if (i0 + st < t1) tile_step(i0 + st, st);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // drain the look-ahead loads before the LDS is reused or released
  };
  bool redo = sp.exact_only != 0;
  if (!redo) {
    sweep(std::false_type{}, true);
    const float limit = 4096.f * TK * static_cast<float>(t1 - t0);
    redo = __syncthreads_or(!(w.l_run <= limit) ? 1 : 0) != 0;  // also true for NaN; uniform over the workgroup
    // every wavefront has passed that barrier, so nobody still reads the LDS ring
  }
  if (redo) sweep(std::true_type{}, sp.exact_only != 0);
  const float l_tot = w.l_run + __shfl_xor(w.l_run, 32, 64);
  const uint32_t spoilt = spoilt_columns(w.O, l_tot, c, [&] {
    return finite_rows(reinterpret_cast<const char *>(v_base), 2 * kv_row_elems, max(c.p_wmin + 1, t0 * TK), min(my_tiles * TK, n_kv));
  });
  const PartialSlot<D> slot(sp, rb, gridDim.y, g, n_kv_heads, part, wave);
  if (split)
    write_partial(w.O, w.m_run, l_tot, c, slot);
  else
    store_output<BF16Tag>(w.O, w.m_run, l_tot, c, out, lse_out, hf);
  const Sweep sw = {q_sel, reinterpret_cast<const char *>(k_base), reinterpret_cast<const char *>(v_base), 2 * kv_row_elems, scale_log2, t0, t1};
  rewrite_columns<BF16Tag, D>(spoilt, c, w.m_run, l_tot, sw, split, slot, out, lse_out);
}

// ---------------------------------------------------------------------------
// The wide variant: 64 query columns per wavefront (two 32-column blocks A and B), 256 per workgroup, one wavefront per
// SIMD.  Every operand read of K and V feeds two MFMAs and every kv tile brought into LDS serves twice the columns, so
// the bytes that move per product are half of those of attn_mfma_kernel -- under the power limit, which holds the clock
// of this stage between 1.8 and 2.0 GHz on real data, that is what its time goes down with.  With no second
// wavefront to fill the gaps, the overlap of matrix and vector work is laid out by hand: in iteration i the MFMAs of
// the first product of tile i + 1 are interleaved with the softmax of tile i (each MFMA is followed by the vector work
// of two logits), then the second product of tile i runs with the operand reads of what follows.
//
// Bound: instruction issue, under the power limit.  An iteration (64 columns x 64 keys: 64 MFMAs, 32 pairs of logits per
// lane) is 2950 cycles against 2048 of the matrix pipe alone (3050 by the counters, start and end of a block included; matrix
// and vector unit work together in 0.37 of the matrix unit's time, 0.23 in attn_mfma_kernel).  attn_mfma_kernel -> this one: 32K context, 4915 rows of a 32/8-head
// layer 1.20 -> 1.11 ms (1193 TFLOP/s; 1.04 to 1.16 ms from box to box); 20K, 3072 rows, 28/4 heads 0.460 -> 0.424; 130K, 13007 rows 12.6 ->
// 11.3 ms (1224 TFLOP/s; a library product of 8192^3 reaches 1265).  Not better: the loop unrolled four times (spills), short
// remainders merged into the last whole part.
// ---------------------------------------------------------------------------
constexpr int kWideColumns = 256;

// The first product's MFMA with its accumulator in vector registers and the query operand in accumulation registers.
// The compiler gives a kernel that uses more than 256 registers accumulation registers for ALL its MFMA results, and
// the vector unit can only reach those through copies (64 per tile); the second product's accumulators, which no vector
// instruction touches, are welcome there.  What the compiler then does not see are the wait states between such an
// MFMA and a vector instruction that reads its result (at most 19): see settle.
__device__ __forceinline__ void mfma_first(f32x16 &acc, bf16x8 k, bf16x8 q) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(k), "a"(q));
}
__device__ __forceinline__ void mfma_next(f32x16 &acc, bf16x8 k, bf16x8 q) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(k), "a"(q));
}
// the same where the compiler may have moved an operand just before: two wait states first
__device__ __forceinline__ void mfma_after_moves(f32x16 &acc, bf16x8 k, bf16x8 q) {
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(k), "a"(q));
}
// 32 wait states before the accumulator may be read
__device__ __forceinline__ void settle(f32x16 &acc) { asm volatile("s_nop 15\n\ts_nop 15" : "+v"(acc)); }

constexpr int kWideStages = 4;

// How many of a tile's 32 pairs of logits have gone through the softmax before MFMA `slot` of an iteration (slots 0 .. 31:
// first product of the next tile, 32 .. 63: second product of this one).  An MFMA keeps the matrix pipe for 32
// cycles, 8 of them of issue; a pair takes 38 cycles of vector pipe; so two pairs per three to four slots fit
// underneath.  The second product needs pairs 0 .. 8 u + 7 from slot 32 + 8 u on.
__device__ __forceinline__ constexpr int wide_pairs(int slot) {
  return slot <= 32 ? (slot * 18 + 31) / 32 : (slot >= 56 ? 32 : 18 + ((slot - 32) * 14 + 23) / 24);
}
static_assert(wide_pairs(32) >= 16 && wide_pairs(48) >= 24 && wide_pairs(56) >= 32, "probabilities ready in time");

// The row block (counted from the longest) at place y of a launch that is not cut: the `n_small` shortest ones follow the `n_front`
// longest ones (see set_order).  Any order is right.
__device__ __forceinline__ int whole_order(int y, int n_rb, int n_front, int n_small) {
  return y < n_front ? y : (y < n_front + n_small ? n_rb - n_small + (y - n_front) : y - n_small);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void attn_wide_kernel(
    const uint16_t *__restrict__ q_sel, const int32_t *__restrict__ row_pos, int n_rows,
    const uint16_t *__restrict__ k_cache, const uint16_t *__restrict__ v_cache, int n_kv,
    uint16_t *__restrict__ out, float *__restrict__ lse_out, int n_q_heads, int n_kv_heads, float scale_log2,
    int rows_per_block, CacheLayout lay, SplitPlan sp) {
  constexpr int NS = kWideStages;
  __shared__ __attribute__((aligned(1024))) uint16_t k_lds[NS][TILE_ELEMS];
  __shared__ __attribute__((aligned(1024))) uint16_t v_lds[NS][TILE_ELEMS];
  __shared__ int s_pmax[4];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, hf = lane >> 5;
  const int G = n_q_heads / n_kv_heads;
  const int g = blockIdx.x;
  const bool few = gridDim.z > 1 && gridDim.x * gridDim.y <= 256;  // see part_tiles
  const bool ordered = gridDim.z == 1 && sp.n_small > 0;
  int p_sample = 0;  // the positions of 64 rows
  if (few || ordered) p_sample = row_pos[max(static_cast<int>(static_cast<int64_t>(lane + 1) * n_rows / 64) - 1, 0)];
  const int t_sample = (p_sample >= 0 && p_sample < n_kv ? p_sample : 0) / TK + 1;
  int place = blockIdx.y;  // longest prefixes are dispatched first
  if (ordered) {
    // Another order only where the rows are spread evenly, each 64th of them within a twentieth of the longest block of its place: up to
    // there it gains 2 to 6 %.  Rows that are denser towards the end lose from twice that distance on (density growing with the
    // position, 616 jobs over 32K 1559 -> 1694 us, 714 1736 -> 1865; rows at the END of 16/2 heads 2040 -> 2135).  Blocks of 40 tiles or less
    // end before it matters (64/8 heads, rows 0 to 2499 116 -> 121; 70 tiles 167 -> 156).
    const float longest = static_cast<float>(__builtin_amdgcn_readlane(t_sample, 63));
    if (longest >= 64.f && __all(fabsf(64.f * static_cast<float>(t_sample) - static_cast<float>(lane + 1) * longest) <= 3.2f * longest))
      place = whole_order(place, gridDim.y, sp.n_front, sp.n_small);
  }
  const int rb = gridDim.y - 1 - place;
  const Column cA = setup_column(row_pos, n_rows, n_kv, rb * rows_per_block, rows_per_block, G, g, n_q_heads, wave * 64 + col);
  const Column cB = setup_column(row_pos, n_rows, n_kv, rb * rows_per_block, rows_per_block, G, g, n_q_heads, wave * 64 + 32 + col);
  bf16x8 qf[2][8];
  load_q_frags(qf[0], q_sel, cA, hf);
  load_q_frags(qf[1], q_sel, cB, hf);
  const int p_wmax = max(cA.p_wmax, cB.p_wmax), p_wmin = min(cA.p_wmin, cB.p_wmin);
  const int n_tiles = block_tiles<4>(p_wmax, s_pmax);
  // The length of the parts is for rows spread over the cache, whose blocks average half the tiles of the longest.  Where they
  // are about as long as it (the rows of a long prompt at the end of the cache) and there is at most one per CU, cutting them
  // gains nothing: no block is cut if the even share is 0.7 of the longest block or more (32/8 heads, 1661 and 2048 rows at the end of 8K
  // 208 -> 191 and 234 -> 216 us, of 32K 749 -> 726 and 856 -> 838; 16/2 heads, 4096 rows of 8K 255 -> 205).  The positions are
  // requested at the very start: then launches of spread rows take as long as without this.
  int part_tiles = sp.part_tiles;
  if (few) {
    const int total = __builtin_amdgcn_readfirstlane(wave_sum_i(t_sample)), longest = __builtin_amdgcn_readlane(t_sample, 63);
    if (static_cast<int64_t>(gridDim.x * gridDim.y) * total >= int64_t(64) * 179 * longest) part_tiles = 0x40000000;
  }
  // Parts: z = 0, 1, .. are the whole ones, the last z is the remainder of the row block (all of it, if it is shorter than a
  // part).  So the dispatch order is all pieces of full length first, the shorter ones last, where they fill the end
  // of the launch.
  const int whole = gridDim.z == 1 ? 0 : n_tiles / part_tiles;  // (one z: the launch is not cut)
  const int part = blockIdx.z + 1 == gridDim.z ? whole : blockIdx.z;
  // nothing left for this part (uniform over the workgroup; by number: a length that stands for "not cut" times z leaves the range)
  if (part > whole || (part == whole && (blockIdx.z + 1 < gridDim.z || whole * part_tiles >= n_tiles))) return;
  const int t0 = part * part_tiles;
  const int t1 = min(n_tiles, t0 + part_tiles);
  const bool split = n_tiles > part_tiles;
  if (part == 0 && g == 0 && threadIdx.x == 0 && sp.block_parts != nullptr)
    sp.block_parts[rb] = split ? (n_tiles + part_tiles - 1) / part_tiles : 1;
  const int my_tiles = min(t1, p_wmax / TK + 1);
  const ReadOffsets ro = make_read_offsets(lane);

  const int64_t kv_row_elems = lay.token_stride;
  const uint16_t *k_base = k_cache + g * lay.head_stride;
  const uint16_t *v_base = v_cache + g * lay.head_stride;
  const auto plan = make_dma_plan<4>(kv_row_elems);
  const uint32_t k_addr = __builtin_amdgcn_readfirstlane(lds_address(&k_lds[0][0]));
  const uint32_t v_addr = __builtin_amdgcn_readfirstlane(lds_address(&v_lds[0][0]));
  constexpr uint32_t kStageBytes = TILE_ELEMS * 2;

  f32x16 O[2][4];
  float m_run[2], l_run[2];
  auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
#pragma unroll
      for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) O[q][dt][r] = 0.f;
      m_run[q] = kNoMax;
      l_run[q] = 0.f;
    }
  };
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // A tile is staged from row min(64 tile, n_kv - 64) on: the one that straddles the end of the cache is moved back into
  // it, and the keys it then shares with the tile before are masked like those behind the row's own position.
  auto first_row = [&](int tile) __attribute__((always_inline)) { return min(tile * TK, n_kv - TK); };
  auto mask = [&](f32x16 (&S)[2], int tile, int p_q) __attribute__((always_inline)) {
    // keys tile * 64 .. p_q count: o - first below their number, as unsigned numbers
    const int first = tile * TK - first_row(tile) - 8 * hf;
    const uint32_t count = static_cast<uint32_t>(max(p_q - tile * TK + 1, 0));
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (static_cast<uint32_t>(32 * t + 16 * (r >> 3) + (r & 7) - first) >= count) S[t][r] = -INFINITY;
        if (r % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // (else all comparisons come first, and their masks fill the scalar registers)
      }
  };
  // one load instruction (of four) of a tile's K or V rows
  auto load_part = [&](const uint16_t *src, const uint32_t (&off)[4], uint32_t stage, int x) __attribute__((always_inline)) {
    dma16_base(src, off[x], stage + (wave * 4 + x) * 1024u);
  };
  auto tile_base = [&](const uint16_t *base, int tile) __attribute__((always_inline)) {
    return reinterpret_cast<const uint16_t *>(uniform_pointer(reinterpret_cast<const char *>(base + first_row(tile) * kv_row_elems)));
  };
  // K operand x = 2 s + t of contraction step s, 32-row block t; V operand x = 4 u + dt
  auto k_read = [&](const uint16_t *stage, int x) __attribute__((always_inline)) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const v4u *>(&stage[ro.k[x >> 1] + (x & 1) * 32 * D]));
  };

  // ---- first sweep: fixed reference exponent (see attn_mfma_kernel), software-pipelined -------------------------
  auto fast_sweep = [&]() __attribute__((always_inline)) {
    clear();
    // Iteration i uses K of tile i + 1 and V of tile i.  At its top, K up to tile i + 2 and V up to tile i + 1 have
    // landed everywhere (so the first K operands of the next iteration can be read before its barrier), and
    // what is requested there are K of tile i + 4 and V of tile i + 3.
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        load_part(tile_base(k_base, t0 + t), plan.k_off, k_addr + t * kStageBytes, x);
        if (t < 3) load_part(tile_base(v_base, t0 + t), plan.v_off, v_addr + t * kStageBytes, x);
      }
    bf16x8 k_first[8];  // key 0 of the cache, chunk 2 s + hf: the reference of parts that do not start with it
    if (t0 != 0) {
#pragma unroll
      for (int s = 0; s < 8; ++s) k_first[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const v4u *>(k_base + 16 * s + 8 * hf));
    }
    wait_vmem<0>();
    __syncthreads();
    f32x16 E[2][2], F[2][2];  // logits [column block][32-row block] of the even and the odd tiles
    constexpr int kAhead = 6;
    bf16x8 kf[kAhead];
    if (t0 < my_tiles) {
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int t = 0; t < 2; ++t) E[q][t] = zero;
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const bf16x8 k = k_read(k_lds[0], x);
#pragma unroll
        for (int q = 0; q < 2; ++q)
          mfma_after_moves(E[q][x & 1], k, qf[q][x >> 1]);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int t = 0; t < 2; ++t) settle(E[q][t]);
      // The reference of a column is the logit of key 0 of the cache in EVERY part, so that a probability is rounded to the
      // same bf16 number whether and wherever the launch is cut.  (Every row sees key 0; what vanishes against it in a
      // part is as small against the whole sum.)
      if (t0 == 0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) m_run[q] = __shfl(E[q][0][0], col, 64) * scale_log2;
      } else {  // the product of 32 copies of that key, in the order in which the first tile's is formed: bit for bit the same
#pragma unroll
        for (int q = 0; q < 2; ++q) F[q][0] = zero;
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
          for (int q = 0; q < 2; ++q) mfma_after_moves(F[q][0], k_first[s], qf[q][s]);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          settle(F[q][0]);
          m_run[q] = F[q][0][0] * scale_log2;
        }
      }
#pragma unroll
      for (int x = 0; x < kAhead; ++x) kf[x] = k_read(k_lds[1], x);
    }
    // S: logits of tile i, N: of tile i + 1
    auto iteration = [&](int i, f32x16 (&S)[2][2], f32x16 (&N)[2][2]) __attribute__((always_inline)) {
      // in flight from the iteration before: K of tile i + 3, V of tile i + 2
      wait_vmem<8>();
      __syncthreads();  // everyone is done with K of tile i, V of tile i - 1
      // K of tile i + 4 and V of tile i + 3 are requested one load at a time between the MFMAs (all of them here would
      // hold the four wavefronts up for 500 cycles: 32 loads at 16 cycles).
      const uint32_t st = static_cast<uint32_t>(i - t0) % NS;
      const uint16_t *k_src = tile_base(k_base, i + 4), *v_src = tile_base(v_base, i + 3);
      const uint32_t k_stage = k_addr + st * kStageBytes, v_stage = v_addr + ((st + 3) % NS) * kStageBytes;
      const uint16_t *ks = k_lds[(st + 1) % NS], *kn = k_lds[(st + 2) % NS], *vs = v_lds[st];
      if (i * TK + TK - 1 > p_wmin) {
        mask(S[0], i, cA.p_q);
        mask(S[1], i, cB.p_q);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)  // the query operands stay in accumulation registers
        asm volatile("" : "+a"(qf[q][0]), "+a"(qf[q][1]), "+a"(qf[q][2]), "+a"(qf[q][3]), "+a"(qf[q][4]), "+a"(qf[q][5]), "+a"(qf[q][6]), "+a"(qf[q][7]));
      PTile P[2];
      float psum[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
      // The vector work of two logits, in the order in which the second product needs them: contraction step y / 8, column
      // block y / 4 % 2, word y % 4.
      auto softmax_pair = [&](int y) __attribute__((always_inline)) {
        const int u = y >> 3, q = (y >> 2) & 1, w = y & 3, t = u >> 1, r = 8 * (u & 1) + 2 * w;
        const float a = __builtin_amdgcn_exp2f(fmaf(S[q][t][r], scale_log2, -m_run[q]));
        const float b = __builtin_amdgcn_exp2f(fmaf(S[q][t][r + 1], scale_log2, -m_run[q]));
        psum[q][0] += a;
        psum[q][1] += b;
        P[q].step[u][w] = pack_bf16x2(a, b);
        asm volatile("" : "+v"(psum[q][0]), "+v"(psum[q][1]));  // the sums are formed here, not collected for later
      };
      VFrags vf;
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const bf16x8 k = kf[x % kAhead];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int slot = 2 * x + q;
          if (x < 2)
            mfma_first(N[q][x & 1], k, qf[q][x >> 1]);
          else
            mfma_next(N[q][x & 1], k, qf[q][x >> 1]);
          if (q == 1) {
            if (x + kAhead < 16) kf[x % kAhead] = k_read(ks, x + kAhead);
            if (x >= 12) v_read(vf.lo[x - 12], vf.hi[x - 12], vs, ro, x - 12);
          }
          if (slot % 8 == 4) load_part(k_src, plan.k_off, k_stage, slot / 8);
#pragma unroll
          for (int y = wide_pairs(slot); y < wide_pairs(slot + 1); ++y) softmax_pair(y);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int x = 0; x < 16; ++x) {
        const int u = x >> 2, dt = x & 3;
        const s16x8 a = __builtin_shufflevector(vf.lo[x & 3], vf.hi[x & 3], 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int slot = 32 + 2 * x + q;
          O[q][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, P[q].step[u]), O[q][dt], 0, 0, 0);
          if (q == 1) {
            if (x + 4 < 16) v_read(vf.lo[x & 3], vf.hi[x & 3], vs, ro, x + 4);
            if (x >= 16 - kAhead) kf[x - (16 - kAhead)] = k_read(kn, x - (16 - kAhead));
          }
          if (slot % 8 == 4) load_part(v_src, plan.v_off, v_stage, slot / 8 - 4);
#pragma unroll
          for (int y = wide_pairs(slot); y < wide_pairs(slot + 1); ++y) softmax_pair(y);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) l_run[q] += psum[q][0] + psum[q][1];
    };
    int i = t0;
    for (; i + 1 < my_tiles; i += 2) {
      iteration(i, E, F);
      iteration(i + 1, F, E);
    }
    if (i < my_tiles) iteration(i++, E, F);
    for (; i < t1; ++i) {  // this wavefront's rows end before the tile: it still stages and syncs
      wait_vmem<8>();
      __syncthreads();
      const uint32_t st = static_cast<uint32_t>(i - t0) % NS;
      const uint16_t *k_src = tile_base(k_base, i + 4), *v_src = tile_base(v_base, i + 3);
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        load_part(k_src, plan.k_off, k_addr + st * kStageBytes, x);
        load_part(v_src, plan.v_off, v_addr + ((st + 3) % NS) * kStageBytes, x);
      }
    }
    wait_vmem<0>();  // drain the look-ahead loads before the LDS is reused or released
  };
  uint32_t spoilt[2];
  auto finish = [&](const f32x16 (&o)[4], int q, Column c) __attribute__((always_inline)) {
    l_run[q] += __shfl_xor(l_run[q], 32, 64);
    spoilt[q] = spoilt_columns(o, l_run[q], c, [&]() __attribute__((always_inline)) {
      return finite_rows(reinterpret_cast<const char *>(v_base), 2 * kv_row_elems, max(c.p_wmin + 1, t0 * TK), min(my_tiles * TK, n_kv));
    });
    if (split)
      write_partial(o, m_run[q], l_run[q], c, PartialSlot<D>(sp, rb, gridDim.y, g, n_kv_heads, part, 2 * wave + q));
    else
      store_output<BF16Tag>(o, m_run[q], l_run[q], c, out, lse_out, hf);
  };
  bool done = false;
  if (sp.exact_only == 0) {
    fast_sweep();
    const float limit = 4096.f * TK * static_cast<float>(t1 - t0);
    if (__syncthreads_or(!(l_run[0] <= limit) || !(l_run[1] <= limit) ? 1 : 0) == 0) {  // NaN counts as out of range
      finish(O[0], 0, cA);
      finish(O[1], 1, cB);
      done = true;
    }
  }
  // ---- second sweep: running maximum, one column block after the other (a sweep each: registers, not time, count) ----
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (done) break;
    const Column &c = q == 0 ? cA : cB;
    WaveState w;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) w.O[dt] = zero;
    w.m_run = kNoMax;
    w.l_run = 0.f;
    issue_tile_dma<4>(plan, k_addr, v_addr, k_base, v_base, kv_row_elems, t0, n_kv);
    for (int i = t0; i < t1; ++i) {
      const int st = (i - t0) & 1;
      wait_vmem<0>();
      __syncthreads();
      issue_tile_dma<4>(plan, k_addr + (st ^ 1) * kStageBytes, v_addr + (st ^ 1) * kStageBytes, k_base, v_base, kv_row_elems, i + 1, n_kv);
      if (i >= my_tiles) continue;
      f32x16 S[2];
#pragma unroll
      for (int x = 0; x < 16; ++x)
        S[x & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_read(k_lds[st], x), qf[q][x >> 1], x < 2 ? zero : S[x & 1], 0, 0, 0);
      row_stats<true>(S, w, i * TK, c.p_q, c.p_wmin, hf, scale_log2);
      PTile P;
      exp_tile(S, w, P, scale_log2);
      VFrags vf;
      pv_preload(vf, v_lds[st], ro);
      pv_tile(P, vf, w, v_lds[st], ro);
    }
    wait_vmem<0>();
    __syncthreads();
    m_run[q] = w.m_run;
    l_run[q] = w.l_run;
    finish(w.O, q, c);
  }
  const Sweep sw = {q_sel, reinterpret_cast<const char *>(k_base), reinterpret_cast<const char *>(v_base), 2 * kv_row_elems, scale_log2, t0, t1};
#pragma unroll 1
  for (int q = 0; q < 2; ++q) {
    const uint32_t columns = q == 0 ? spoilt[0] : spoilt[1];
    if (columns == 0) continue;
    const Column c = setup_column(row_pos, n_rows, n_kv, rb * rows_per_block, rows_per_block, G, g, n_q_heads, wave * 64 + 32 * q + col);
    rewrite_columns<BF16Tag, D>(columns, c, q == 0 ? m_run[0] : m_run[1], q == 0 ? l_run[0] : l_run[1], sw, split,
                                PartialSlot<D>(sp, rb, gridDim.y, g, n_kv_heads, part, 2 * wave + q), out, lse_out);
  }
}

}  // namespace

bool attention_mfma_supported(const ifkv_ctx *ctx) {
  return ctx->desc.n_q_heads / ctx->desc.n_kv_heads <= 32;
}

namespace {

constexpr int kSlots = 512;       // workgroups the chip holds at a time (256 CUs, two each; one of fp32 with heads of 128)
constexpr int kMaxParts = 8;      // parts of a launch that fills the slots (the scratch is sized for this)
constexpr int kMaxPartsFew = 64;  // launches with a handful of row blocks: as many parts as slots stay free

// bf16 heads of 128 run the kernels of this file, everything else attn_full_kernel (attention_full.hip)
bool narrow_probabilities(const ifkv_ctx *ctx) { return ctx->desc.dtype == IFKV_BF16 && ctx->desc.head_dim == D; }

// Shortest part worth its partial results and its share of the merge: 8 tiles, and 4 where even parts of 8 leave
// more than three quarters of the slots empty (32/8 heads of 128, 32 -> 8 -> 4 tiles: 16 rows against 4000 keys 39 -> 16 ->
// 13 us, 64 against 2000 37 -> 18 -> 15, 128 against 4000 43 -> 22 -> 27, 300 spread over 2000 37 -> 23 -> 25).
// Launches that nearly fill the slots gain less than the merge costs (64/8 heads, 700 rows over 3000 keys, 352 jobs: 60
// us with parts of 32, 64 with 26).  A tile of the fp32 kernel is 3072 or 6144 cycles of matrix pipe and as many of vector
// instructions, as much as four tiles of the bf16 kernels or more.
int min_part_tiles(const ifkv_ctx *ctx, int64_t jobs, int n_kv_tiles) {
  if (ctx->desc.dtype != IFKV_BF16) return 1;
  if (jobs >= 350) return 32;
  return jobs * (n_kv_tiles / 8) <= kSlots / 4 ? 4 : 8;
}

size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// groups of 32 query columns of the last row block of `columns` columns, and of all of them per kv head
int last_units(const ifkv_ctx *ctx, int64_t n_rows, int columns) {
  const int G = ctx->desc.n_q_heads / ctx->desc.n_kv_heads, rpb = columns / G;
  return n_rows > 0 ? static_cast<int>(((n_rows - 1) % rpb + 1) * G + 31) / 32 : 0;
}
int64_t all_units(const ifkv_ctx *ctx, int64_t n_rows, int columns) {
  const int rpb = columns / (ctx->desc.n_q_heads / ctx->desc.n_kv_heads);
  return n_rows > 0 ? (n_rows - 1) / rpb * (columns / 32) + last_units(ctx, n_rows, columns) : 0;
}

// bytes of partial results for a launch of n_rows rows cut into `parts`, whichever kernel of the layer serves it
size_t partial_bytes(const ifkv_ctx *ctx, int64_t n_rows, int parts) {
  int64_t units = all_units(ctx, n_rows, kBlockColumns);
  if (narrow_probabilities(ctx)) units = std::max(units, all_units(ctx, n_rows, kWideColumns));
  const size_t slot = ctx->desc.head_dim == D ? PartialSlot<D>::kFloats : PartialSlot<64>::kFloats;
  return align256(static_cast<size_t>(units) * ctx->desc.n_kv_heads * static_cast<size_t>(parts) * slot * sizeof(float)) +
         align256(static_cast<size_t>(n_rows) * sizeof(int));
}

// Workgroups of the wide kernel for a launch (256 query columns each, one per CU), 0 where the narrow one serves it.
// The wide one is faster per tile, but half as many jobs, twice as long, spread worse: it wins from about 0.8 jobs per CU
// on, from 128 kv tiles on and, between one and 1.6 jobs per CU, where what is left over for the second round
// costs most, from 256 tiles on.  32/8 heads, rows spread over the context, narrow -> wide:
//   32K keys: 1277 rows (160 jobs) 377 -> 456 us, 1661 (208) 442 -> 411, 2429 (304) 673 -> 605, 3197 (400) 824 -> 773,
//             4915 (616) 1200 -> 1107;  130K keys, 13007 rows: 12604 -> 11306
//   8K keys:  1661 (208) 128 -> 130, 2749 (344) 188 -> 195, 3581 (448) 245 -> 219;  4K keys, 2048 (256): 86 -> 93
// Narrow over wide, geometric means over six head shapes (each with its cut): spread rows, 128 to 160 jobs 0.79 .. 0.89, 160 to 199
// 0.92 .. 1.00, 200 to 256 1.09 (128 tiles) .. 1.21 (1024), 288 to 415 0.93 (128), 0.95 (219), 1.05 (320), 1.09 (1024), more 1.03 ..
// 1.13; rows at the END of the context, whose row blocks are all of the full length, 200 to 256 jobs 0.95 (128 tiles, before such
// blocks were left whole) .. 1.14, 288 to 415 1.00 (128) .. 1.12, more 1.06 .. 1.15.
// Below 200 jobs such rows lose what spread ones gain (32K keys, 1228 rows: 637 -> 682), and 128 rows spread over 32K keys,
// most of whose tiles need the mask, take 114 us instead of 67.  What the rule cannot see is that all rows lie at the front of a
// much longer cache: 2429 rows at the front of 16K take 76 us, 61 on the narrow kernel.
// The last rows of a long cache (a prompt) alone would gain from a wide piece per CU (32/8 heads, 32K keys, 128 rows 84.0 -> 79.9),
// but the host sees neither where the rows lie nor what they attend to: with a logit far above the reference the wide
// kernel repeats its sweep once per column block (154 -> 189), and rows in the front half leave half of its pieces empty (52 -> 66;
// 256 rows 84 -> 121).
int64_t wide_jobs(const ifkv_ctx *ctx, int64_t n_rows, int64_t n_kv) {
  const auto &d = ctx->desc;
  if (!narrow_probabilities(ctx) || n_kv < TK || ctx->tune.attn_wide == 2) return 0;
  const int rpb = kWideColumns / (d.n_q_heads / d.n_kv_heads);
  const int64_t jobs = (n_rows + rpb - 1) / rpb * d.n_kv_heads;
  if (ctx->tune.attn_wide == 1) return jobs;
  const int64_t n_tiles = (n_kv + TK - 1) / TK;
  if (jobs < 200 || n_tiles < 128) return 0;
  return jobs < 288 || jobs >= 416 || n_tiles >= 256 ? jobs : 0;
}

}  // namespace

// Whether and where the kv axis is cut.  A row block at position p costs p keys, so a launch is bound either by its
// total work (tiles per slot, if the jobs spread evenly) or by its longest row block alone.  With rows spread uniformly
// over the context a job averages half the tiles of the cache; when the longest job is clearly longer than the even
// share per slot, the kv axis is cut into parts of about that share: row blocks shorter than one part are not
// affected (they write their output directly), only the long ones run as several workgroups whose partial
// results are merged by attn_merge_kernel.
//   Narrow kernel and the layer types of attention_full.hip: even share of 512 slots (two of these workgroups per CU; the one
// that holds a CU alone, fp32 with heads of 128, is better off with that share too: of 256 slots it is 1 % slower over the
// sizes below, up to 40 % with 280 jobs), parts of 1.25 to 1.6 times the share, by how the whole parts and the remainders of that
// many row blocks fill the slots.
// 32/8 heads, rows spread over the context, parts of 1.15 times the share -> these: heads of 128, 8K keys, 160 jobs 71 ->
// 63 us, 224 95 -> 81, 312 117 -> 108, 400 131 -> 122, 496 145 -> 141; heads of 64, 8K keys, 312 jobs 93 -> 88.  Not cut, 312
// jobs take 135 us.  Six head shapes, 1 to 4096 rows over 2.5K to 130K keys, against 1.15 times the share and parts of 32 tiles
// or more: spread rows 11 % faster at 100 to 200 jobs, 5 % at 350, even from there on; rows at the END of the context, whose
// blocks are all long, within 3 % from 100 jobs on (single shapes lose up to 16 %: 64/8 heads, 256 rows at the end of 8K 84 -> 91).
//   Only launches with no more jobs than slots are cut: with more, every slot is busy for most of the
// launch anyway and the partial writes plus the merge cost more than the shorter tail gains (684 jobs:
// 0.469 -> 0.479 ms; 1232 jobs: 1.28 -> 1.37 ms).  A part spans at least min_part_tiles tiles and there are at most
// 8 parts -- with so few row blocks that 8 parts each would leave slots empty (a few dozen rows against a long
// context), up to 64, as long as jobs x parts stays within the slots, which also keeps the partial results
// within the scratch.
//   fp32, up to 16 jobs: jobs x parts within 256 instead: the matrix pipe is what bounds these kernels, one workgroup per CU
// fills it, and a second round of pieces costs as much as the first.  32/8 heads of 128, 64 rows: 2000 keys 42.0 -> 33.7 us, 4000
// 61.3 -> 53.1, 1200 (60 rows) 37.1 -> 32.0; heads of 64, 1600 keys 23.0 -> 20.9; over 500 to 8161 keys and four head shapes up to
// 25 % faster, slower where the finer pieces of spread rows would have fitted one round too (14/2 heads, 100 rows over 1600 keys
// 28.8 -> 32.6).  With more jobs it depends on how the pieces fall (28 jobs over 1200 keys: 33 -> 40 us, 32 jobs 53 -> 40).
//   bf16 heads of 128, one row block: every piece reads keys and values of its own, one workgroup per CU draws all the bandwidth
// there is, and more of them only add partial results: parts as for 256 pieces, up to 32 tiles.  Rows at the end of the cache
// (a decoding step, the last prompt rows), 512 pieces -> these: 32/8 heads, one row over 20K keys 25.6 -> 23.0 us, 32K 33.7 -> 30.7,
// 64K 54.1 -> 50.1, 16 rows over 32K 37.2 -> 31.7; 16/16 heads, 128 rows over 32K 66.1 -> 62.7.  Few rows in the middle of the cache
// have shorter pieces: 16 rows spread over 32K 37.6 -> 34.6, a single one 18.9 -> 25.6.
//   Wide kernel (256 at a time): parts of 1.25 times the even share, down to 32 tiles, as long as that is shorter than the
// longest row block (32K context, 208 jobs: 427 us; 1.1 and 1.45 times: 499 and 452; not cut: 462.  20K context, 304
// jobs of a 28/4-head layer: 404; 1.1, 1.45, not cut: 420, 420, 450).  Blocks that are all long are not cut after all: see
// part_tiles in the kernel.  What is not a whole part goes out as the row blocks come, the longest block first.  By length instead,
// rows spread over 20000 keys: 32/8 heads, 220 jobs 278 -> 291, 320 jobs 396 -> 406, 344 jobs of 28/4 heads 426 -> 436; only rows that are
// denser towards the end gain (304 jobs over 32K 925 -> 792).  Parts of at most 0.86 of the cache (352 to 410 jobs): rows at the END up
// to 9 % faster, spread rows of 400 jobs over 32K 770 -> 802, of 16/16 heads over 40000 keys 938 -> 1008.
//   The tuning knobs override all this; a cut whose partial results would not fit the scratch is not made.
SplitChoice choose_split(const ifkv_ctx *ctx, int64_t n_rows, int64_t n_kv, size_t scratch_bytes) {
  const auto &d = ctx->desc;
  const int G = d.n_q_heads / d.n_kv_heads;
  const int rpb = kBlockColumns / G;
  const int64_t n_rb = (n_rows + rpb - 1) / rpb, jobs = n_rb * d.n_kv_heads, wide = wide_jobs(ctx, n_rows, n_kv);
  const int n_kv_tiles = static_cast<int>((n_kv + TK - 1) / TK);
  int part_tiles = n_kv_tiles;
  if (ctx->tune.attn_part_tiles > 0) {
    part_tiles = ctx->tune.attn_part_tiles;
  } else if (ctx->tune.attn_split_parts > 0) {
    part_tiles = (n_kv_tiles + ctx->tune.attn_split_parts - 1) / ctx->tune.attn_split_parts;
  } else if (wide > 0) {
    const double even_share = static_cast<double>(wide) * (0.5 * n_kv_tiles) / (kSlots / 2);
    part_tiles = std::max(32, static_cast<int>(1.25 * even_share + 0.5));
  } else {
    const double even_share = static_cast<double>(jobs) * (0.5 * n_kv_tiles) / kSlots;
    const double longer = jobs < 200 ? 1.35 : jobs < 350 ? 1.25 : jobs < 450 ? 1.6 : 1.4;
    if (jobs > 0 && jobs <= kSlots && even_share < 0.9 * n_kv_tiles) part_tiles = static_cast<int>(longer * even_share + 0.5);
    part_tiles = std::max(part_tiles, min_part_tiles(ctx, jobs, n_kv_tiles));
    int max_parts = kMaxParts;
    const int pieces = d.dtype != IFKV_BF16 && jobs <= 16 ? 256 : kSlots;
    if (jobs > 0 && jobs * kMaxParts < pieces) max_parts = static_cast<int>(std::min<int64_t>(kMaxPartsFew, pieces / jobs));
    if (part_tiles * max_parts < n_kv_tiles) part_tiles = (n_kv_tiles + max_parts - 1) / max_parts;
    if (narrow_probabilities(ctx) && n_rb == 1)
      part_tiles = std::max(part_tiles, std::min(32, static_cast<int>((n_kv_tiles * jobs + 255) / 256)));
    // fewer parts if their results do not fit (fp32, 8192 keys, 819 rows of a 32/8-head layer: 1034 us not cut, 557 cut)
    for (int parts = (n_kv_tiles + part_tiles - 1) / part_tiles; parts > 1 && partial_bytes(ctx, n_rows, parts) > scratch_bytes; --parts)
      part_tiles = (n_kv_tiles + parts - 2) / (parts - 1);
  }
  if (part_tiles < 1) part_tiles = 1;
  if (part_tiles > n_kv_tiles) part_tiles = n_kv_tiles > 0 ? n_kv_tiles : 1;
  SplitChoice c;
  c.part_tiles = part_tiles;
  c.parts = (n_kv_tiles + part_tiles - 1) / part_tiles;
  if (c.parts < 1) c.parts = 1;
  // host-side bounds: the grid's z extent, and the partial results must fit what was allocated
  if (c.parts > 65534 || (c.parts > 1 && partial_bytes(ctx, n_rows, c.parts) > scratch_bytes)) {
    c.parts = 1;
    c.part_tiles = n_kv_tiles > 0 ? n_kv_tiles : 1;
  }
  return c;
}

bool place_partials(const ifkv_ctx *ctx, int64_t n_rows, const SplitChoice &sc, SplitPlan *sp) {
  sp->part_tiles = sc.part_tiles;
  sp->partials = nullptr;
  sp->block_parts = nullptr;
  sp->parts = sc.parts;
  sp->units = kBlockColumns / 32;
  sp->last_units = last_units(ctx, n_rows, kBlockColumns);
  sp->exact_only = ctx->tune.attn_exact_sweep;
  const uint32_t G = static_cast<uint32_t>(ctx->desc.n_q_heads / ctx->desc.n_kv_heads);
  sp->group_magic = (65536u + G - 1) / G;
  sp->group_size = static_cast<int>(G);
  sp->n_front = sp->n_small = 0;
  if (sc.parts == 1) return true;
  if (ctx->scratch == nullptr || partial_bytes(ctx, n_rows, sc.parts) > ctx->scratch_bytes) return false;
  char *base = static_cast<char *>(ctx->scratch);
  sp->partials = reinterpret_cast<float *>(base);
  sp->block_parts = reinterpret_cast<int *>(base + partial_bytes(ctx, n_rows, sc.parts) - align256(static_cast<size_t>(n_rows) * sizeof(int)));
  return true;
}

// Scratch for the partial results, fixed for a layer shape: the largest launch the library cuts by
// itself (as many row blocks as the chip has workgroup slots, 8 parts).  A call has at most one row per cache row,
// which bounds it for short contexts, and the layer types of attention_full.hip, whose contexts are
// short, are held to 64 MiB (a cut that does not fit is not made).
size_t attention_mfma_scratch_bytes(const ifkv_ctx *ctx) {
  const auto &d = ctx->desc;
  const int G = d.n_q_heads / d.n_kv_heads;
  const int64_t rows = static_cast<int64_t>((kSlots + d.n_kv_heads - 1) / d.n_kv_heads) * (kBlockColumns / G);
  if (narrow_probabilities(ctx)) return partial_bytes(ctx, rows, kMaxParts);
  return std::min(partial_bytes(ctx, std::min<int64_t>(rows, d.max_ctx), kMaxPartsFew), size_t(64) << 20);
}

namespace {

// One launch covers at most 65535 row blocks (the y extent of a grid); more rows than that are
// served by several launches over consecutive row ranges (rows are independent).  Launches of one
// stream run one after the other, so they share the scratch.
constexpr int64_t kMaxRowBlocks = 65535;

// Dispatch order of the wide kernel's row blocks in a launch that is not cut, by the lengths that rows spread evenly over the cache
// give them.  Longest first, 2 + f rounds of blocks, f between 0 and 1: two rounds pair long with short and end together, and the f
// rounds of the shortest come on top.  With these behind the longest 1 - 0.7 f rounds, the compute units that take them are early by as
// much as the rest of the launch can use.  Rows spread over 32K keys, longest first -> this: 32/8 heads, 576 jobs 1112 -> 1056 us,
// 616 1189 -> 1130, 664 1268 -> 1207, 704 1338 -> 1276; 28/4, 16/16, 16/2, 40/8 and 64/8 heads 2 to 7 %, 16K and 50000 keys 3 to 6 %.
// Nothing to gain at two rounds and from three on.
void set_order(const ifkv_ctx *ctx, int n_rb, SplitPlan *sp) {
  const int hkv = ctx->desc.n_kv_heads, round = kSlots / 2 / hkv, step = std::max(1, 32 / hkv);  // 8 dies of 4 engines are filled in turn
  const double f = static_cast<double>(n_rb) / round - 2.0;
  if (f < 0.08 || f > 0.9 || round < 8) return;
  sp->n_front = std::min(round - step, static_cast<int>(round * (1.0 - 0.7 * f) / step + 0.75) * step);
  sp->n_small = static_cast<int>(round * (f + 0.125));
}

hipError_t launch_attention_range(ifkv_ctx *ctx, const void *q_sel, const int32_t *row_pos, int64_t n_rows,
                                  const void *k_cache, const void *v_cache, int64_t n_kv, void *out, float *lse_out) {
  if (!narrow_probabilities(ctx))
    return launch_attention_full_range(ctx, q_sel, row_pos, n_rows, k_cache, v_cache, n_kv, out, lse_out);
  const auto &d = ctx->desc;
  const float scale_log2 = ctx->sm_scale * 1.4426950408889634f;
  int rpb = kBlockColumns / (d.n_q_heads / d.n_kv_heads);
  const unsigned n_rb = static_cast<unsigned>((n_rows + rpb - 1) / rpb);
  const SplitChoice sc = choose_split(ctx, n_rows, n_kv, ctx->scratch_bytes);
  SplitPlan sp;
  if (!place_partials(ctx, n_rows, sc, &sp)) return hipErrorInvalidValue;
  dim3 grid(d.n_kv_heads, n_rb, sc.parts);
  const int64_t n_kv_tiles = (n_kv + TK - 1) / TK;
  if (wide_jobs(ctx, n_rows, n_kv) > 0) {
    rpb = kWideColumns / (d.n_q_heads / d.n_kv_heads);
    sp.units = kWideColumns / 32;
    sp.last_units = last_units(ctx, n_rows, kWideColumns);
    grid.y = static_cast<unsigned>((n_rows + rpb - 1) / rpb);
    if (sc.parts > 1) grid.z = static_cast<unsigned>(n_kv_tiles / sc.part_tiles + 1);
    if (sc.parts == 1) set_order(ctx, static_cast<int>(grid.y), &sp);
    hipLaunchKernelGGL(attn_wide_kernel, grid, dim3(256), 0, ctx->stream, static_cast<const uint16_t *>(q_sel), row_pos,
                       static_cast<int>(n_rows), static_cast<const uint16_t *>(k_cache), static_cast<const uint16_t *>(v_cache),
                       static_cast<int>(n_kv), static_cast<uint16_t *>(out), lse_out, d.n_q_heads, d.n_kv_heads, scale_log2,
                       rpb, cache_layout(ctx), sp);
  } else {
    hipLaunchKernelGGL((attn_mfma_kernel<4, 2>), grid, dim3(256), 0, ctx->stream, static_cast<const uint16_t *>(q_sel), row_pos,
                       static_cast<int>(n_rows), static_cast<const uint16_t *>(k_cache), static_cast<const uint16_t *>(v_cache),
                       static_cast<int>(n_kv), static_cast<uint16_t *>(out), lse_out, d.n_q_heads, d.n_kv_heads, scale_log2, rpb,
                       cache_layout(ctx), sp);
  }
  if (sc.parts > 1) launch_merge<BF16Tag, D>(ctx, sp, row_pos, n_rows, n_kv, rpb, out, lse_out);
  return hipGetLastError();
}

}  // namespace

namespace {
int64_t rows_per_launch_of(const ifkv_ctx *ctx) {
  const int G = ctx->desc.n_q_heads / ctx->desc.n_kv_heads;
  int64_t max_rb = kMaxRowBlocks;
  if (ctx->tune.attn_max_row_blocks > 0 && ctx->tune.attn_max_row_blocks < max_rb) max_rb = ctx->tune.attn_max_row_blocks;
  return max_rb * (128 / G);
}
}  // namespace

// What launch_attention_mfma would do for n_rows rows against n_kv keys with a scratch of
// scratch_bytes: the launches, the largest number of kv parts and the smallest part length among
// them, and the most bytes of partial results any of them keeps.  Host arithmetic only.
void attention_mfma_plan(const ifkv_ctx *ctx, int64_t n_rows, int64_t n_kv, size_t scratch_bytes, int64_t out[4]) {
  const int64_t rows_per_launch = rows_per_launch_of(ctx);
  out[0] = out[3] = 0;
  out[1] = 1;
  out[2] = (n_kv + TK - 1) / TK;
  for (int64_t r0 = 0; r0 < n_rows; r0 += rows_per_launch) {
    const int64_t nr = n_rows - r0 < rows_per_launch ? n_rows - r0 : rows_per_launch;
    const SplitChoice sc = choose_split(ctx, nr, n_kv, scratch_bytes);
    ++out[0];
    if (sc.parts > out[1]) out[1] = sc.parts;
    if (sc.part_tiles < out[2]) out[2] = sc.part_tiles;
    if (sc.parts > 1) out[3] = std::max<int64_t>(out[3], static_cast<int64_t>(partial_bytes(ctx, nr, sc.parts)));
  }
}

hipError_t launch_attention_mfma(ifkv_ctx *ctx, const void *q_sel, const int32_t *row_pos, int64_t n_rows,
                                 const void *k_cache, const void *v_cache, int64_t n_kv, void *out,
                                 float *lse_out) {
  const auto &d = ctx->desc;
  const int64_t rows_per_launch = rows_per_launch_of(ctx);
  const int64_t row_bytes = static_cast<int64_t>(d.n_q_heads) * d.head_dim * dtype_size(d.dtype);
  for (int64_t r0 = 0; r0 < n_rows; r0 += rows_per_launch) {
    const int64_t nr = n_rows - r0 < rows_per_launch ? n_rows - r0 : rows_per_launch;
    hipError_t e = launch_attention_range(ctx, static_cast<const char *>(q_sel) + r0 * row_bytes, row_pos + r0, nr, k_cache,
                                          v_cache, n_kv, static_cast<char *>(out) + r0 * row_bytes,
                                          lse_out != nullptr ? lse_out + r0 * d.n_q_heads : nullptr);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace ifkv
