// basp_attn_fwd.hip -- causal GQA attention forward for the rank's heads.
//
// Computes the scaled dot-product attention of Sec. II-A of the paper over
// the full sequence, masked causally (key j visible to query i iff j <= i),
// for each local query head h with local kv head h / n_rep:
//   O_i = sum_j softmax_j(scale * q_i . k_j) v_j,   LSE_i = log sum_j exp(.)
// The S x S score matrix is never stored: keys are visited in tiles with a
// running row maximum and row sum (online softmax), a re-association that
// changes only rounding.
//
// gfx950 mapping
//   * workgroup = 8 waves = 256 query rows of one (sequence, head), one
//     workgroup per CU (two waves per SIMD); wave w owns rows q0 + 32w .. +31,
//     one row per lane pair (l, l+32).
//   * scores are formed transposed, S^T = K Q^T, with
//     v_mfma_f32_32x32x16_bf16: K (A operand) from LDS, Q (B operand) kept
//     in registers for the whole loop.  The 32x32 accumulator then gives each
//     lane one query row and 16 keys, so the softmax statistics are lane-local
//     up to one exchange with the partner lane l^32.
//   * O^T = V^T P^T: P goes from the score accumulator straight into the B
//     operand (bf16, round to nearest even).  V^T (A operand) is read from the
//     row-major V tile with ds_read_b64_tr_b16, two 4-key reads per operand,
//     in exactly the key order the accumulator holds P in.
//   * K/V tiles of 64 keys are copied HBM -> LDS by buffer loads that write
//     LDS directly (no register staging; rows past S arrive as zeros) into a
//     ring of four stages.  Tiles are stored row-major with an XOR swizzle
//     that is conflict-free for both read patterns.  Each wave waits only for
//     its own copies of the tile it needs next, passes a fence-free barrier,
//     and then issues the copies of the tile three ahead into the stage every
//     wave has just finished with, so two later tiles stay in flight.
//   * tiles left of the diagonal band are software-pipelined inside each
//     wave: the score products of tile t+1 are issued between the
//     exponentials of tile t, and the row sum of t (and, on short sequences,
//     the row maxima of t+1) between the P V products of t, one product per
//     slot with its operand read two slots ahead.  Every stretch of a wave's
//     instruction stream thus mixes matrix and vector work.
//   * LDS holds the K tiles of the four ring stages, then their V tiles, and
//     the pipelined loop is unrolled over the four stages: every operand
//     address is a lane's fixed offset plus an instruction immediate, with
//     no per-tile address arithmetic.
//   * the exponent reference of a row starts as its first tile's maximum and
//     follows only when it has been outgrown, so that O is rescaled on few
//     tiles: by 8 (in log2 units) where the maxima are formed, before the
//     exponentials; in the pipelined loop of long sequences, which sees it in
//     the row sums, once a lane's sum of a tile has passed 2^16, after that
//     tile's products.  P above 1 is as exact in bf16 and in the fp32 sums as
//     P <= 1.
//   * tiles strictly below the workgroup's diagonal band run a loop without
//     any masking code; band tiles are masked, and a wave skips band tiles
//     past its last row.  The grid is one-dimensional, heaviest query tiles
//     first, heads fastest, so heads sharing a kv head run side by side.
//   * in the diagonal band a wave raises its issue priority over the score
//     products, so the two waves of a SIMD drift apart: one's softmax
//     overlaps the other's MFMAs.
//   * small shares run 128- or 64-row workgroups whose waves share the keys of
//     a tile (P = 2 below, and attn_fwd_split_kernel).
//   * tensors are read and written through row views: the local
//     head-sharded tensors, or (SH) the G sequence shards of the exchange in
//     place, whose row counts are multiples of 256 so that a workgroup's
//     rows and a key tile each lie in one shard; K/V tiles then take the
//     buffer of their own rows.
#include <math.h>

#include <type_traits>

#include "basp_device.hpp"
#include "basp_internal.hpp"

namespace basp {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = 8;
constexpr int kBN = 64;           // keys per wave and tile
constexpr float kRescaleSlack = 8.f;  // log2 headroom before the reference max moves
// A lane's sum of a tile's P past which the pipelined loop moves the reference:
// low enough for the row sums of many tiles, high enough to be rare.
constexpr float kFollowSum = 65536.f;
// Instruction classes of __builtin_amdgcn_sched_group_barrier.
constexpr int kSchedValu = 0x002;
constexpr int kSchedMfma = 0x008;
constexpr int kSchedDsRead = 0x100;

// P = 1: the 8 waves are 8 row groups of 32 query rows, which share every tile
// of 64 keys.  P = 2 (small shares): 4 row groups, and two waves of a row group
// take the two halves of a tile of 128 keys, each with its own online softmax,
// merged once through LDS.
template <int D, int PARTS>
struct FwdCfg {
  static constexpr int P = PARTS;
  static constexpr int DC = HeadDim<D>::DC;  // computed width of O
  static constexpr int LW = HeadDim<D>::LW;  // LDS row layout
  static constexpr int R = kWaves / P;            // row groups
  static constexpr int BM = 32 * R;               // query rows per workgroup
  static constexpr int BT = kBN * P;              // keys per tile
  static constexpr int STAGES = P == 1 ? 4 : 2;
  static constexpr int PD = 2;                    // P = 1: tiles in flight behind the one being read
  static constexpr int TILE_BYTES = BT * LW * 2;
  static constexpr int STAGE_BYTES = 2 * TILE_BYTES;  // K, V
  static constexpr int NS = D / 16;                   // 16-deep steps over the head dim
  static constexpr int NE = DC / 32;                  // 32-wide head-dim subtiles of O
  static constexpr int CPR = LW / 8;                  // 16-byte chunk slots per LDS row
  static constexpr int DMA_PER_WAVE = BT * CPR / kThreads;  // 1 KB loads per wave per tensor
  // A part's slot of the merge area: NE*4 register groups of O (1 KB each: 64
  // lanes x 16 B), then the reference and the row sum (256 B each).
  static constexpr int PART_BYTES = NE * 4 * 1024 + 512;
  static_assert((P - 1) * R * PART_BYTES <= STAGES * STAGE_BYTES, "the merge area fits the ring");
};

// The key parts of a row group brought together at the end (every copy landed,
// nothing left to read in the ring): parts 1 .. C::P-1 put their reference, row
// sum (of both lanes of a row) and O in LDS, part 0 merges them in order into
// its own.  True in part 0.
template <class C>
__device__ __forceinline__ bool merge_parts(unsigned char *smem, int rg, int part, int lane,
                                            float &m_ref, float &l_tot, f32x16 (&oacc)[C::NE]) {
  auto area = [&](int p) __attribute__((always_inline)) {
    return smem + ((p - 1) * C::R + rg) * C::PART_BYTES;
  };
  constexpr int kScalars = C::NE * 4 * 1024;
  barrier_no_fence();
  if (part > 0) {
    unsigned char *a = area(part);
#pragma unroll
    for (int n = 0; n < C::NE; ++n)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<f32x4 *>(a + (n * 4 + g) * 1024 + 16 * lane) =
            f32x4{oacc[n][4 * g], oacc[n][4 * g + 1], oacc[n][4 * g + 2], oacc[n][4 * g + 3]};
    *reinterpret_cast<float *>(a + kScalars + 4 * lane) = m_ref;
    *reinterpret_cast<float *>(a + kScalars + 256 + 4 * lane) = l_tot;
  }
  __syncthreads();
  if (part > 0) return false;
  float m_all = m_ref, pm[C::P], wt[C::P];
  pm[0] = m_ref;
#pragma unroll
  for (int p = 1; p < C::P; ++p) {
    pm[p] = *reinterpret_cast<const float *>(area(p) + kScalars + 4 * lane);
    m_all = fmaxf(m_all, pm[p]);
  }
#pragma unroll
  for (int p = 0; p < C::P; ++p) wt[p] = pm[p] == -INFINITY ? 0.f : fast_exp2(pm[p] - m_all);
  m_ref = m_all;
  l_tot *= wt[0];
#pragma unroll
  for (int n = 0; n < C::NE; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[n][r] *= wt[0];
#pragma unroll
  for (int p = 1; p < C::P; ++p) {
    l_tot = fmaf(wt[p], *reinterpret_cast<const float *>(area(p) + kScalars + 256 + 4 * lane),
                 l_tot);
#pragma unroll
    for (int n = 0; n < C::NE; ++n)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 z =
            *reinterpret_cast<const f32x4 *>(area(p) + (n * 4 + g) * 1024 + 16 * lane);
#pragma unroll
        for (int y = 0; y < 4; ++y) oacc[n][4 * g + y] = fmaf(wt[p], z[y], oacc[n][4 * g + y]);
      }
  }
  return true;
}

template <int D, bool SH, int P, bool FOLLOW>
__global__ __launch_bounds__(kThreads, 1) void attn_fwd_kernel(
    const RowView qv, const RowView kv, const RowView vv, const RowView ov,
    float *__restrict__ lse, int S, int Hl, int n_rep, int heads_total, int qtiles,
    float c /* scale * log2(e) */) {
  using C = FwdCfg<D, P>;
  constexpr int kStages = C::STAGES, kPD = C::PD;
  using T = LdsTile<C::LW>;
  // LDS: the K tiles of the kStages ring stages, then their V tiles, so that
  // a stage's K and V tiles sit at the same offset from two fixed bases.
  __shared__ __attribute__((aligned(16))) unsigned char smem[kStages * C::STAGE_BYTES];
  constexpr int kVRegion = kStages * C::TILE_BYTES;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, held in an SGPR
  const int l32 = lane & 31, hh = lane >> 5;

  const int L = blockIdx.x;
  const int qt = qtiles - 1 - L / heads_total;
  const int hb = L % heads_total;
  const int beta = hb / Hl, h = hb % Hl, kvh = h / n_rep;
  const int q0 = qt * C::BM;
  const int rg = w % C::R, part = w / C::R;  // row group, key part
  const int wrow0 = q0 + 32 * rg;
  const int row = wrow0 + l32;

  const uint32_t q_row_bytes = qv.row_elems * 2, kv_row_bytes = kv.row_elems * 2;
  uint32_t q_left, kv_left;
  // Q of rows q0 .. (rows past the buffer's end read as zeros)
  const rsrc_t rq =
      make_rsrc(view_row<SH, const uint16_t>(qv, beta, q0, h, D, q_left), q_left * q_row_bytes);
  // Local K/V: one resource per head for every tile.  Sharded: one per shard.
  u32x4 rk = {}, rv = {};
  if constexpr (!SH) {
    rk = make_rsrc_words(view_row<false, const uint16_t>(kv, beta, 0, kvh, D, kv_left),
                         kv_left * kv_row_bytes);
    rv = make_rsrc_words(view_row<false, const uint16_t>(vv, beta, 0, kvh, D, kv_left),
                         kv_left * kv_row_bytes);
  }
  const uint32_t smem_lds = lds_addr_of(smem);

  // Q fragments (B operand of S^T = K Q^T): row `row`, e = 16s + 8hh .. +7.
  bf16x8 qf[C::NS];
#pragma unroll
  for (int s = 0; s < C::NS; ++s)
    qf[s] = as_bf16x8(buf_load16(rq, (uint32_t)(row - q0) * q_row_bytes + (2 * s + hh) * 16));
  // Retire the Q loads before any tile copy is in flight: the compiler does
  // not count the copies, and a wait for Q inside the tile loop would also
  // drain the prefetched tiles.
  wait_vmcnt<0>();

  const int kv_end = min(S, q0 + C::BM);
  const int nt = (kv_end + C::BT - 1) / C::BT;

  uint32_t g_off[C::DMA_PER_WAVE];
#pragma unroll
  for (int i = 0; i < C::DMA_PER_WAVE; ++i)
    g_off[i] = dma_src_off<C::LW, D>((w * C::DMA_PER_WAVE + i) * 64 + lane, kv_row_bytes);
  // Sharded: tiles are loaded in order, so the resources move to the next
  // shard only when the tiles of the current one are used up.
  uint32_t sh_tiles = 0, sh_base = 0;
  auto load_tile = [&](int t) {  // issue; lands asynchronously in stage t % kStages
    const uint32_t ks = smem_lds + (t % kStages) * C::TILE_BYTES;
    uint32_t base = (uint32_t)(t * kBN) * kv_row_bytes;
    if constexpr (SH) {
      if (sh_tiles == 0) {  // wave-uniform; tile t is the first of its shard
        uint32_t left;
        rk = make_rsrc_words(view_row<true, const uint16_t>(kv, beta, t * kBN, kvh, D, left),
                             left * kv_row_bytes);
        rv = make_rsrc_words(view_row<true, const uint16_t>(vv, beta, t * kBN, kvh, D, left),
                             left * kv_row_bytes);
        sh_tiles = left / kBN;
        sh_base = 0;
      }
      base = sh_base;
      sh_base += kBN * kv_row_bytes;
      --sh_tiles;
    }
#pragma unroll
    for (int i = 0; i < C::DMA_PER_WAVE; ++i) {
      const uint32_t lds_off = ks + (w * C::DMA_PER_WAVE + i) * 1024;
      buf_load16_lds_async(rk, base + g_off[i], lds_off);
      buf_load16_lds_async(rv, base + g_off[i], lds_off + kVRegion);
    }
  };
  // K or V of one tile.  P = 2: tile t's scores are formed one iteration before
  // its P V, so K runs one tile ahead of V and two stages of each are enough.
  auto load_one = [&](int t, const RowView &view, u32x4 r, uint32_t region)
                      __attribute__((always_inline)) {
    uint32_t base = (uint32_t)(t * C::BT) * kv_row_bytes;
    if constexpr (SH) {  // the tile's shard (shard rows are a multiple of 256)
      uint32_t left;
      r = make_rsrc_words(view_row<true, const uint16_t>(view, beta, t * C::BT, kvh, D, left),
                          left * kv_row_bytes);
      base = 0;
    }
    const uint32_t ks = smem_lds + (t % kStages) * C::TILE_BYTES + region;
#pragma unroll
    for (int i = 0; i < C::DMA_PER_WAVE; ++i)
      buf_load16_lds_async(r, base + g_off[i], ks + (w * C::DMA_PER_WAVE + i) * 1024);
  };
  auto load_k = [&](int t) __attribute__((always_inline)) { load_one(t, kv, rk, 0); };
  auto load_v = [&](int t) __attribute__((always_inline)) { load_one(t, vv, rv, kVRegion); };
  // Wait until this wave's loads of tile t landed, with `ahead` later tiles
  // (2 * DMA_PER_WAVE loads each) still in flight.
  auto wait_tile = [&](int ahead) {
    if (ahead >= 2) wait_vmcnt<4 * C::DMA_PER_WAVE>();
    else if (ahead == 1) wait_vmcnt<2 * C::DMA_PER_WAVE>();
    else wait_vmcnt<0>();
  };

  // LDS offsets of this lane's operand reads (fixed across tiles).
  // A of S^T: K row 32m + l32, chunk 2s + hh.  The swizzle depends on the
  // row modulo 16 only, so row 32 + r sits 32 rows further on.
  const int part_off = part * kBN * T::ROW_BYTES;  // first row of the wave's keys
  int k_off[C::NS];
#pragma unroll
  for (int s = 0; s < C::NS; ++s) {
    k_off[s] = T::off(l32, 2 * s + hh) + part_off;
    asm volatile("" : "+v"(k_off[s]));  // keep in a register, do not recompute per tile
  }
  // A of O^T: V^T rows e = 32n + l32, keys 16*s2 + 4hh + {0..3} and + 8.
  // Transposed A operand: rows 16*s2 + 4hh (+8), columns 32n + 16*((lane/16)&1);
  // row block s2 sits 16*s2 rows further on (same swizzle).
  int v_off[C::NE][2];
#pragma unroll
  for (int n = 0; n < C::NE; ++n)
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      v_off[n][x] =
          kVRegion + part_off +
          tr_piece_off<C::LW>(4 * hh + 8 * x, 32 * n + 16 * ((lane >> 4) & 1), lane);
      asm volatile("" : "+v"(v_off[n][x]));
    }

  f32x16 oacc[C::NE];
#pragma unroll
  for (int n = 0; n < C::NE; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[n][r] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;

  if constexpr (P == 1) {
    for (int t = 0; t <= kPD && t < nt; ++t) load_tile(t);
  } else {
    load_k(0);
    load_v(0);
    if (nt > 1) load_k(1);
  }

  // One tile: scores, softmax update, P V.  MASK only for tiles that can
  // hold keys past some row of the workgroup (the diagonal band).
  auto tile = [&](int t, auto mask_tag) {
    constexpr bool MASK = decltype(mask_tag)::value;
    const int j0 = t * C::BT + kBN * part;
    const unsigned char *Ks = smem + (t % kStages) * C::TILE_BYTES;
    const unsigned char *Vs = Ks;  // v_off holds the V region's base

    wave_priority<1>();  // the score products run ahead of the partner wave's softmax
    f32x16 sacc[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const bf16x8 a = *reinterpret_cast<const bf16x8 *>(Ks + k_off[0] + m * 32 * T::ROW_BYTES);
      sacc[m] = mfma32x32x16(a, qf[0], f32x16{});
    }
#pragma unroll
    for (int s = 1; s < C::NS; ++s)
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(Ks + k_off[s] + m * 32 * T::ROW_BYTES);
        sacc[m] = mfma32x32x16(a, qf[s], sacc[m]);
      }
    // Schedule: LDS reads run one k-step ahead of the MFMAs.
    __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 4, 0);
#pragma unroll
    for (int i = 0; i < C::NS - 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(kSchedMfma, 2, 0);
      __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(kSchedMfma, 4, 0);
    wave_priority<0>();

    // sacc[m][r] = S^T[key j0 + 32m + 8(r/4) + 4hh + r%4][query row]
    if constexpr (MASK) {
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int j = j0 + 32 * m + 8 * (r >> 2) + 4 * hh + (r & 3);
          if (j > row) sacc[m][r] = -INFINITY;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[m][r]);
    mx = pair_max(mx) * c;
    // Move the reference only when the row maximum outgrew it by the slack
    // (always on a row's first tile, where m_ref is -inf).
    const bool grow = mx > m_ref + kRescaleSlack;
    if (__builtin_amdgcn_ballot_w64(grow)) {  // wave-uniform, rare after the first tiles
      asm volatile("" ::: "memory");  // keep this a real branch (no if-conversion)
      const float m_new = grow ? mx : m_ref;
      // P = 2: a row of which this part has seen no key yet keeps its -inf
      const float alpha = P == 1 || grow ? fast_exp2(m_ref - m_new) : 1.f;
      m_ref = m_new;
      l_run *= alpha;
#pragma unroll
      for (int n = 0; n < C::NE; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[n][r] *= alpha;
    }
    const float m_use = P > 1 && m_ref == -INFINITY ? 0.f : m_ref;  // no key yet: P = 0
    float psum = 0.f;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = fast_exp2(fmaf(sacc[m][r], c, -m_use));
        sacc[m][r] = p;
        psum += p;
      }
    l_run += psum;

    bf16x8 pf[kBN / 16];
#pragma unroll
    for (int s2 = 0; s2 < kBN / 16; ++s2) {
      const int m = s2 >> 1, b8 = (s2 & 1) * 8;
      u32x4 t4 = {pack_bf16x2(sacc[m][b8 + 0], sacc[m][b8 + 1]),
                  pack_bf16x2(sacc[m][b8 + 2], sacc[m][b8 + 3]),
                  pack_bf16x2(sacc[m][b8 + 4], sacc[m][b8 + 5]),
                  pack_bf16x2(sacc[m][b8 + 6], sacc[m][b8 + 7])};
      pf[s2] = as_bf16x8(t4);
    }
#pragma unroll
    for (int n = 0; n < C::NE; ++n)
#pragma unroll
      for (int s2 = 0; s2 < kBN / 16; ++s2) {
        const bf16x8 a = tr_operand(Vs, v_off[n][0] + s2 * 16 * T::ROW_BYTES,
                                    v_off[n][1] + s2 * 16 * T::ROW_BYTES);
        oacc[n] = mfma32x32x16(a, pf[s2], oacc[n]);
      }
    // Schedule: transposed reads run two operands ahead of the MFMAs.
    __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 4, 0);
#pragma unroll
    for (int i = 0; i < C::NE * (kBN / 16) - 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(kSchedMfma, 2, 0);
  };
  // Ring discipline: tiles 0 .. kPD are issued up front, then iteration t
  // (of either loop below) issues tile t + kPD + 1 into the stage of tile
  // t - 1, after a barrier that every wave passes only once it has finished
  // with tile t - 1.  Before the barrier a wave waits for its own copies of
  // the tile it is about to read, with `ahead` later tiles left in flight.
  // P = 2: iteration t of the pipelined loop reads K of tile t+1 and V of tile
  // t, which its own wait (for every copy) made visible, and issues K of tile
  // t+2 and V of tile t+1 into the stages of K of t and V of t-1, which every
  // wave has finished with.  The one masked tile is the last: nothing is
  // issued past it.
  auto make_visible = [&](int ahead, int issue) __attribute__((always_inline)) {
    if constexpr (P == 1) {
      wait_tile(ahead);
      barrier_no_fence();
      if (issue < nt) load_tile(issue);
    } else {
      wait_vmcnt<0>();
      barrier_no_fence();
      const int t = issue - kPD - 1;
      if (t + 2 < nt) load_k(t + 2);
      if (t + 1 < nt) load_v(t + 1);
    }
  };

  // Tiles before t_mask need no mask.  They run software-pipelined: while
  // the softmax of tile t (exponentials, conversions) is computed, the score
  // products of tile t+1 are issued, and while P V of tile t runs, its row sum
  // is formed, so that every stretch of the wave's instruction stream mixes
  // matrix and vector work.
  const int t_mask = min(nt, q0 / C::BT);
  auto scores = [&](int t, f32x16 (&sc)[2]) __attribute__((always_inline)) {
    const unsigned char *Ks = smem + (t % kStages) * C::TILE_BYTES;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const bf16x8 a = *reinterpret_cast<const bf16x8 *>(Ks + k_off[0] + m * 32 * T::ROW_BYTES);
      sc[m] = mfma32x32x16(a, qf[0], f32x16{});
    }
#pragma unroll
    for (int s2 = 1; s2 < C::NS; ++s2)
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(Ks + k_off[s2] + m * 32 * T::ROW_BYTES);
        sc[m] = mfma32x32x16(a, qf[s2], sc[m]);
      }
  };
  auto row_max = [&](const f32x16 (&sc)[2]) __attribute__((always_inline)) {
    float mx = -INFINITY;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[m][r]);
    return pair_max(mx) * c;
  };
  auto move_reference = [&](float mx) __attribute__((always_inline)) {
    const bool grow = mx > m_ref + kRescaleSlack;
    if (__builtin_amdgcn_ballot_w64(grow)) {  // wave-uniform, rare after the first tiles
      asm volatile("" ::: "memory");
      const float m_new = grow ? mx : m_ref;
      const float alpha = fast_exp2(m_ref - m_new);
      m_ref = m_new;
      l_run *= alpha;
#pragma unroll
      for (int n = 0; n < C::NE; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[n][r] *= alpha;
    }
  };
  auto exps = [&](f32x16 (&sc)[2], bf16x8 (&pf)[kBN / 16]) __attribute__((always_inline)) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[m][r] = fast_exp2(fmaf(sc[m][r], c, -m_ref));
#pragma unroll
    for (int s2 = 0; s2 < kBN / 16; ++s2) {
      const int m = s2 >> 1, b8 = (s2 & 1) * 8;
      pf[s2] = as_bf16x8(u32x4{pack_bf16x2(sc[m][b8 + 0], sc[m][b8 + 1]),
                               pack_bf16x2(sc[m][b8 + 2], sc[m][b8 + 3]),
                               pack_bf16x2(sc[m][b8 + 4], sc[m][b8 + 5]),
                               pack_bf16x2(sc[m][b8 + 6], sc[m][b8 + 7])});
    }
  };
  auto row_sum = [&](const f32x16 (&sc)[2]) __attribute__((always_inline)) {
    float psum = 0.f;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) psum += sc[m][r];
    return psum;
  };
  auto pv = [&](int t, const bf16x8 (&pf)[kBN / 16]) __attribute__((always_inline)) {
    const unsigned char *Vs = smem + (t % kStages) * C::TILE_BYTES;
#pragma unroll
    for (int n = 0; n < C::NE; ++n)
#pragma unroll
      for (int s2 = 0; s2 < kBN / 16; ++s2) {
        const bf16x8 a = tr_operand(Vs, v_off[n][0] + s2 * 16 * T::ROW_BYTES,
                                    v_off[n][1] + s2 * 16 * T::ROW_BYTES);
        oacc[n] = mfma32x32x16(a, pf[s2], oacc[n]);
      }
  };
  // With FOLLOW the pipelined loop forms no row maxima: the row sums, needed
  // anyway, say when the reference has been outgrown, and it then follows them
  // (half a row's sum is at least its maximum), 18 vector instructions less per
  // tile for a check of the workgroup's rows at the end (follows_sums).
  // In the tile that outgrows it P can come near the end of fp32's range, up to
  // 128 powers of two above the reference, so what was summed is scaled by
  // 2^(-up/2) twice: 2^-up itself can lie below fp32's normal range, where the
  // exp unit gives 0.  Where P passed the range, O or the row sum is no finite
  // number from then on, and the rows are done over (below).
  auto follow = [&](float psum) __attribute__((always_inline)) {
    if (__builtin_amdgcn_ballot_w64(!(psum <= kFollowSum))) {  // wave-uniform, rare
      asm volatile("" ::: "memory");
      const float up = fast_log2(fmaxf(pair_max(psum), 1.f));
      const float half = fast_exp2(-0.5f * up);
      m_ref += up;
      l_run = l_run * half * half;
#pragma unroll
      for (int n = 0; n < C::NE; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[n][r] = oacc[n][r] * half * half;
    }
  };
  // Iteration t of the pipelined loop, tile t+1 unmasked: `cur` holds the
  // scores of tile t (reference already moved for them); the scores of tile
  // t+1 go to `nxt`.  Each block is a sequence of slots of one product each,
  // fenced by scheduling barriers: the slot's share of the vector work, and
  // the operand read for the product kPf slots later.
  constexpr int kPf = 2;
  auto pipelined = [&](int t, auto stage_tag, f32x16 (&cur)[2], f32x16 (&nxt)[2])
                       __attribute__((always_inline)) {
    constexpr int ST = decltype(stage_tag)::value;  // t % kStages
    make_visible(min(1, nt - 2 - t), t + kPD + 1);  // tile t+1 readable, t+2 in flight
    asm volatile("" : "+v"(m_ref));  // keep the exponent arguments here
    bf16x8 pf[kBN / 16];
    // Block X: scores of tile t+1 (16 products), exponentials of tile t, at
    // raised issue priority: of the two waves of a SIMD, the one in this
    // block keeps the matrix unit while the other is in block Y.
    wave_priority<1>();
    {
      constexpr int NG = 2 * C::NS;
      const unsigned char *Ks = smem + ((ST + 1) % kStages) * C::TILE_BYTES;
      bf16x8 op[NG];
      auto read = [&](int g) __attribute__((always_inline)) {
        op[g] = *reinterpret_cast<const bf16x8 *>(Ks + k_off[g / 2] + (g % 2) * 32 * T::ROW_BYTES);
      };
#pragma unroll
      for (int g = 0; g < kPf; ++g) read(g);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g + kPf < NG) read(g + kPf);
        const int m = g % 2, s2 = g / 2;
        nxt[m] = mfma32x32x16(op[g], qf[s2], s2 == 0 ? f32x16{} : nxt[m]);
        // 32 exponentials over the 16 slots; each full group of 8 converted
#pragma unroll
        for (int e = 32 * g / NG; e < 32 * (g + 1) / NG; ++e) {
          const int mm = e / 16, r = e % 16;
          cur[mm][r] = fast_exp2(fmaf(cur[mm][r], c, -m_ref));
          if (r % 8 == 7) {
            const int b8 = r - 7;
            pf[2 * mm + b8 / 8] = as_bf16x8(u32x4{pack_bf16x2(cur[mm][b8 + 0], cur[mm][b8 + 1]),
                                                  pack_bf16x2(cur[mm][b8 + 2], cur[mm][b8 + 3]),
                                                  pack_bf16x2(cur[mm][b8 + 4], cur[mm][b8 + 5]),
                                                  pack_bf16x2(cur[mm][b8 + 6], cur[mm][b8 + 7])});
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    wave_priority<0>();
    // Block Y: P V of tile t (16 products), row sum of t, (no FOLLOW) row
    // maxima of t+1.
    float psum = 0.f, mx = -INFINITY;
    {
      constexpr int NG = C::NE * (kBN / 16);
      const unsigned char *Vs = smem + ST * C::TILE_BYTES;
      bf16x8 op[NG];
      auto read = [&](int g) __attribute__((always_inline)) {
        const int n = g / (kBN / 16), s2 = g % (kBN / 16);
        op[g] = tr_operand(Vs, v_off[n][0] + s2 * 16 * T::ROW_BYTES,
                           v_off[n][1] + s2 * 16 * T::ROW_BYTES);
      };
#pragma unroll
      for (int g = 0; g < kPf; ++g) read(g);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g + kPf < NG) read(g + kPf);
        const int n = g / (kBN / 16), s2 = g % (kBN / 16);
        oacc[n] = mfma32x32x16(op[g], pf[s2], oacc[n]);
#pragma unroll
        for (int e = 32 * g / NG; e < 32 * (g + 1) / NG; ++e) psum += cur[e / 16][e % 16];
        if constexpr (!FOLLOW) {
#pragma unroll
          for (int e = 32 * g / NG; e < 32 * (g + 1) / NG; ++e)
            mx = fmaxf(mx, nxt[e / 16][e % 16]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    l_run += psum;
    // After P V of tile t, before the exponentials of t+1.
    if constexpr (FOLLOW) follow(psum);
    else move_reference(pair_max(mx) * c);
  };
  // The last unmasked tile t: no scores to start.
  auto pipelined_last = [&](int t, f32x16 (&cur)[2]) __attribute__((always_inline)) {
    make_visible(min(1, nt - 2 - t), t + kPD + 1);  // tile t+1 (the first masked one)
    asm volatile("" : "+v"(m_ref));
    bf16x8 pf[kBN / 16];
    exps(cur, pf);
    __builtin_amdgcn_sched_barrier(0);
    pv(t, pf);
    const float psum = row_sum(cur);
    l_run += psum;
    __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 4, 0);
#pragma unroll
    for (int i = 0; i < C::NE * (kBN / 16) - 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 2, 0);
      __builtin_amdgcn_sched_group_barrier(kSchedValu, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(kSchedMfma, 2, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (FOLLOW) follow(psum);
  };
  if (t_mask > 0) {
    f32x16 sa[2], sb[2];
    if constexpr (P == 1) {
      make_visible(min(kPD, nt - 1), nt);  // tile 0; tile kPD + 1 is issued by iteration 0
    } else {
      wait_vmcnt<0>();  // K of tile 0 (and every other copy)
      barrier_no_fence();
    }
    scores(0, sa);
    move_reference(row_max(sa));
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    int t = 0;
    if constexpr (P == 1) {
      using I2 = std::integral_constant<int, 2>;
      using I3 = std::integral_constant<int, 3>;
      static_assert(P > 1 || kStages == 4, "the unrolled loop assumes four ring stages");
      for (; t + 4 < t_mask; t += 4) {  // t % 4 == 0: every stage offset a constant
        pipelined(t, I0{}, sa, sb);
        pipelined(t + 1, I1{}, sb, sa);
        pipelined(t + 2, I2{}, sa, sb);
        pipelined(t + 3, I3{}, sb, sa);
      }
      // 1 to 4 unmasked tiles left, the last of them without scores to start
      if (t + 1 < t_mask) {
        pipelined(t, I0{}, sa, sb);
        if (t + 2 < t_mask) {
          pipelined(t + 1, I1{}, sb, sa);
          if (t + 3 < t_mask) {
            pipelined(t + 2, I2{}, sa, sb);
            pipelined_last(t + 3, sb);
          } else {
            pipelined_last(t + 2, sa);
          }
        } else {
          pipelined_last(t + 1, sb);
        }
      } else {
        pipelined_last(t, sa);
      }
    } else {
      for (; t + 2 < t_mask; t += 2) {  // t % 2 == 0
        pipelined(t, I0{}, sa, sb);
        pipelined(t + 1, I1{}, sb, sa);
      }
      if (t + 1 < t_mask) {
        pipelined(t, I0{}, sa, sb);
        pipelined_last(t + 1, sb);
      } else {
        pipelined_last(t, sa);
      }
    }
  }
  for (int t = t_mask; t < nt; ++t) {  // the diagonal band, masked
    make_visible(min(kPD, nt - 1 - t), t + kPD + 1);
    if (t * C::BT + kBN * part <= wrow0 + 31) tile(t, std::true_type{});  // wave-uniform
  }

  // A sum that is no finite number, in any row of the workgroup: P overflowed,
  // or the inputs hold such numbers.  All rows are done over, tile by tile with
  // the row maxima, so that P <= 2^8.
  if (FOLLOW && t_mask > 0) {
    float z = 0.f * l_run;
#pragma unroll
    for (int n = 0; n < C::NE; ++n)
#pragma unroll
      for (int r = 0; r < 16; ++r) z = fmaf(0.f, oacc[n][r], z);
    if (__syncthreads_or(!(z == 0.f))) {
      m_ref = -INFINITY;
      l_run = 0.f;
#pragma unroll
      for (int n = 0; n < C::NE; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[n][r] = 0.f;
      for (int t = 0; t < nt; ++t) {
        barrier_no_fence();  // every wave is done with the stage
        load_one(t, kv, rk, 0);
        load_one(t, vv, rv, kVRegion);
        wait_vmcnt<0>();
        barrier_no_fence();
        if (t * C::BT + kBN * part <= wrow0 + 31) tile(t, std::true_type{});  // wave-uniform
      }
    }
  }

  // oacc[n][r] = O^T[e = 32n + 8(r/4) + 4hh + r%4][query row] (unnormalised)
  float l_tot = pair_sum(l_run);
  if constexpr (P > 1) {
    if (!merge_parts<C>(smem, rg, part, lane, m_ref, l_tot, oacc)) return;
  }
  if (row < S) {
    const float inv = 1.f / l_tot;
    uint32_t o_left;
    uint16_t *ob = view_row<SH, uint16_t>(ov, beta, q0, h, D, o_left) +
                   (size_t)(row - q0) * ov.row_elems;
#pragma unroll
    for (int n = 0; n < C::NE; ++n)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (32 * n + 8 * g >= D) continue;  // padding columns
        u32x2 val = {pack_bf16x2(oacc[n][4 * g] * inv, oacc[n][4 * g + 1] * inv),
                     pack_bf16x2(oacc[n][4 * g + 2] * inv, oacc[n][4 * g + 3] * inv)};
        *reinterpret_cast<u32x2 *>(ob + 32 * n + 8 * g + 4 * hh) = val;
      }
    if (hh == 0)
      lse[((size_t)beta * Hl + h) * S + row] = (m_ref + fast_log2(l_tot)) * 0.69314718055994531f;
  }
}

// ---------------------------------------------------------------- split form
// The forward of the smallest shares (and of small ones at d = 64): the 8
// waves are R row groups of 32 query rows times P = 8 / R key parts, and part p
// takes keys 32p .. 32p+31 of each tile of 32 P keys.  A workgroup is
// then 32 R rows, with the same two waves per SIMD and the same products per
// tile, for a half or a quarter of the rows and of the key loop's length.
// Each wave runs its own online softmax over its keys, merged at the end.  A
// wave's tile is not software-pipelined: it is 32 keys, and the loop is short.
template <int D, int RG>
struct SplitCfg {
  static constexpr int R = RG;
  static constexpr int DC = HeadDim<D>::DC;
  static constexpr int LW = HeadDim<D>::LW;
  static constexpr int P = kWaves / R;
  static constexpr int BM = 32 * R;  // query rows per workgroup
  static constexpr int BN = 32 * P;  // keys per tile
  static constexpr int TILE_BYTES = BN * LW * 2;
  // 128 KB of ring, but for 64-wide rows with R = 4: 64 KB, two workgroups a CU.
  static constexpr int STAGES = 2 * TILE_BYTES > 32768 ? 2 : 4;
  static constexpr int LDS_BYTES = STAGES * 2 * TILE_BYTES;
  static constexpr int NS = D / 16;
  static constexpr int NE = DC / 32;
  static constexpr int CPR = LW / 8;
  static constexpr int DMA_PER_WAVE = BN * CPR / kThreads;
  static constexpr int PART_BYTES = NE * 4 * 1024 + 512;
  static_assert((P - 1) * R * PART_BYTES <= LDS_BYTES, "the merge area fits the ring");
};

template <int D, bool SH, int R>
__global__ __launch_bounds__(kThreads, 1) void attn_fwd_split_kernel(
    const RowView qv, const RowView kv, const RowView vv, const RowView ov,
    float *__restrict__ lse, int S, int Hl, int n_rep, int heads_total, int qtiles,
    float c /* scale * log2(e) */) {
  using C = SplitCfg<D, R>;
  using T = LdsTile<C::LW>;
  // LDS: the K tiles of the ring stages, then their V tiles.
  __shared__ __attribute__((aligned(16))) unsigned char smem[C::LDS_BYTES];
  constexpr int kSt = C::STAGES, kVRegion = kSt * C::TILE_BYTES;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hh = lane >> 5;
  const int rg = w % R, part = w / R;  // row group, key part

  const int L = blockIdx.x;
  const int qt = qtiles - 1 - L / heads_total;
  const int hb = L % heads_total;
  const int beta = hb / Hl, h = hb % Hl, kvh = h / n_rep;
  const int q0 = qt * C::BM;
  const int wrow0 = q0 + 32 * rg;
  const int row = wrow0 + l32;

  const uint32_t q_row_bytes = qv.row_elems * 2, kv_row_bytes = kv.row_elems * 2;
  uint32_t q_left, kv_left;
  const rsrc_t rq =
      make_rsrc(view_row<SH, const uint16_t>(qv, beta, q0, h, D, q_left), q_left * q_row_bytes);
  u32x4 rk = {}, rv = {};  // local: one resource per head; sharded: one per shard
  if constexpr (!SH) {
    rk = make_rsrc_words(view_row<false, const uint16_t>(kv, beta, 0, kvh, D, kv_left),
                         kv_left * kv_row_bytes);
    rv = make_rsrc_words(view_row<false, const uint16_t>(vv, beta, 0, kvh, D, kv_left),
                         kv_left * kv_row_bytes);
  }
  const uint32_t smem_lds = lds_addr_of(smem);

  const int kv_end = min(S, q0 + C::BM);
  const int nt = (kv_end + C::BN - 1) / C::BN;
  uint32_t g_off[C::DMA_PER_WAVE];
#pragma unroll
  for (int i = 0; i < C::DMA_PER_WAVE; ++i)
    g_off[i] = dma_src_off<C::LW, D>((w * C::DMA_PER_WAVE + i) * 64 + lane, kv_row_bytes);

  bf16x8 qf[C::NS];
#pragma unroll
  for (int s = 0; s < C::NS; ++s)
    qf[s] = as_bf16x8(buf_load16(rq, (uint32_t)(row - q0) * q_row_bytes + (2 * s + hh) * 16));
  wait_vmcnt<0>();  // retire the tracked loads before untracked copies start

  uint32_t sh_tiles = 0, sh_base = 0;
  auto load_tile = [&](int t) __attribute__((always_inline)) {
    const uint32_t ks = smem_lds + (t % kSt) * C::TILE_BYTES;
    uint32_t base = (uint32_t)(t * C::BN) * kv_row_bytes;
    if constexpr (SH) {
      if (sh_tiles == 0) {  // wave-uniform; tile t is the first of its shard
        uint32_t left;
        rk = make_rsrc_words(view_row<true, const uint16_t>(kv, beta, t * C::BN, kvh, D, left),
                             left * kv_row_bytes);
        rv = make_rsrc_words(view_row<true, const uint16_t>(vv, beta, t * C::BN, kvh, D, left),
                             left * kv_row_bytes);
        sh_tiles = left / C::BN;
        sh_base = 0;
      }
      base = sh_base;
      sh_base += C::BN * kv_row_bytes;
      --sh_tiles;
    }
#pragma unroll
    for (int i = 0; i < C::DMA_PER_WAVE; ++i) {
      const uint32_t lds_off = ks + (w * C::DMA_PER_WAVE + i) * 1024;
      buf_load16_lds_async(rk, base + g_off[i], lds_off);
      buf_load16_lds_async(rv, base + g_off[i], lds_off + kVRegion);
    }
  };
  // Tiles 0 .. kSt-2 are issued up front; iteration t waits for its own copies
  // of tile t, passes the barrier and issues tile t + kSt-1 into the stage of
  // tile t-1, which every wave has finished with.
  auto begin_tile = [&](int t) __attribute__((always_inline)) {
    if constexpr (kSt == 4) {
      const int ahead = min(2, nt - 1 - t);
      if (ahead >= 2) wait_vmcnt<4 * C::DMA_PER_WAVE>();
      else if (ahead == 1) wait_vmcnt<2 * C::DMA_PER_WAVE>();
      else wait_vmcnt<0>();
    } else {
      wait_vmcnt<0>();
    }
    barrier_no_fence();
    if (t + kSt - 1 < nt) load_tile(t + kSt - 1);
  };
#pragma unroll
  for (int t = 0; t < kSt - 1; ++t)
    if (t < nt) load_tile(t);

  // This lane's operand reads: K row l32 and V^T rows of the wave's part.
  const int part_off = part * 32 * T::ROW_BYTES;
  int k_off[C::NS], v_off[C::NE][2];
#pragma unroll
  for (int s = 0; s < C::NS; ++s) {
    k_off[s] = T::off(l32, 2 * s + hh) + part_off;
    asm volatile("" : "+v"(k_off[s]));
  }
#pragma unroll
  for (int n = 0; n < C::NE; ++n)
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      v_off[n][x] = kVRegion + part_off +
                    tr_piece_off<C::LW>(4 * hh + 8 * x, 32 * n + 16 * ((lane >> 4) & 1), lane);
      asm volatile("" : "+v"(v_off[n][x]));
    }

  f32x16 oacc[C::NE];
#pragma unroll
  for (int n = 0; n < C::NE; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[n][r] = 0.f;
  float m_ref = -INFINITY, l_run = 0.f;  // -inf: no key of this part reached the row yet

  auto tile = [&](int t, int st, auto mask_tag) __attribute__((always_inline)) {
    constexpr bool MASK = decltype(mask_tag)::value;
    const int j0 = t * C::BN + 32 * part;
    if (MASK && j0 > wrow0 + 31) return;  // wave-uniform: every key past every row
    const unsigned char *Ks = smem + st * C::TILE_BYTES;
    wave_priority<1>();
    f32x16 sacc;
#pragma unroll
    for (int s = 0; s < C::NS; ++s) {
      const bf16x8 a = *reinterpret_cast<const bf16x8 *>(Ks + k_off[s]);
      sacc = mfma32x32x16(a, qf[s], s == 0 ? f32x16{} : sacc);
    }
    wave_priority<0>();
    // sacc[r] = S^T[key j0 + 8(r/4) + 4hh + r%4][query row]
    if constexpr (MASK) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (j0 + 8 * (r >> 2) + 4 * hh + (r & 3) > row) sacc[r] = -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[r]);
    mx = pair_max(mx) * c;
    const bool grow = mx > m_ref + kRescaleSlack;
    if (__builtin_amdgcn_ballot_w64(grow)) {  // wave-uniform, rare after the first tiles
      asm volatile("" ::: "memory");
      const float alpha = grow ? fast_exp2(m_ref - mx) : 1.f;
      m_ref = grow ? mx : m_ref;
      l_run *= alpha;
#pragma unroll
      for (int n = 0; n < C::NE; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[n][r] *= alpha;
    }
    // A row no key of the part has reached: every score is -inf, P = 0.
    const float m_use = m_ref == -INFINITY ? 0.f : m_ref;
    float psum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sacc[r] = fast_exp2(fmaf(sacc[r], c, -m_use));
      psum += sacc[r];
    }
    l_run += psum;
    bf16x8 pf[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      const int b8 = 8 * s2;
      pf[s2] = as_bf16x8(u32x4{pack_bf16x2(sacc[b8 + 0], sacc[b8 + 1]),
                               pack_bf16x2(sacc[b8 + 2], sacc[b8 + 3]),
                               pack_bf16x2(sacc[b8 + 4], sacc[b8 + 5]),
                               pack_bf16x2(sacc[b8 + 6], sacc[b8 + 7])});
    }
#pragma unroll
    for (int n = 0; n < C::NE; ++n)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        const bf16x8 a = tr_operand(Ks, v_off[n][0] + s2 * 16 * T::ROW_BYTES,
                                    v_off[n][1] + s2 * 16 * T::ROW_BYTES);
        oacc[n] = mfma32x32x16(a, pf[s2], oacc[n]);
      }
    __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 4, 0);
#pragma unroll
    for (int i = 0; i < 2 * C::NE - 2; ++i) {
      __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(kSchedMfma, 2, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  const int t_mask = min(nt, q0 / C::BN);  // tiles before t_mask need no mask
  int t = 0;
  for (; t + kSt <= t_mask; t += kSt) {  // t % kSt == 0: constant stage offsets
#pragma unroll
    for (int u = 0; u < kSt; ++u) {
      begin_tile(t + u);
      tile(t + u, u, std::false_type{});
    }
  }
  for (; t < t_mask; ++t) {
    begin_tile(t);
    tile(t, t % kSt, std::false_type{});
  }
  for (; t < nt; ++t) {
    begin_tile(t);
    tile(t, t % kSt, std::true_type{});
  }

  float l_tot = pair_sum(l_run);
  if (!merge_parts<C>(smem, rg, part, lane, m_ref, l_tot, oacc) || row >= S) return;
  const float inv = 1.f / l_tot;
  uint32_t o_left;
  uint16_t *ob = view_row<SH, uint16_t>(ov, beta, q0, h, D, o_left) +
                 (size_t)(row - q0) * ov.row_elems;
#pragma unroll
  for (int n = 0; n < C::NE; ++n)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (32 * n + 8 * g >= D) continue;  // padding columns
      *reinterpret_cast<u32x2 *>(ob + 32 * n + 8 * g + 4 * hh) =
          u32x2{pack_bf16x2(oacc[n][4 * g] * inv, oacc[n][4 * g + 1] * inv),
                pack_bf16x2(oacc[n][4 * g + 2] * inv, oacc[n][4 * g + 3] * inv)};
    }
  if (hh == 0)
    lse[((size_t)beta * Hl + h) * S + row] = (m_ref + fast_log2(l_tot)) * 0.69314718055994531f;
}

// Row groups of a workgroup: 8 (attn_fwd_kernel, P = 1), 4 (P = 2; at d = 64
// the split kernel) or 2 (the split kernel).  256-row workgroups, causal and so
// of very different lengths, leave CUs idle on small shares; wider workgroups
// have the higher rate: a K or V tile feeds more products.  The lines are where
// the two meet, in two measures.
// Long sequences: up to W = b * Hl * S query rows.  Forward, us on MI355X for 8 |
// 4 | 2: d = 128: W = 16K 45 | - | 22; 31K 146 | 93 | 76; 37K 339 | 221 | 216; 40K
// 370 | 243 | 248; 56K 280 | 197 | 241; 75K 108 | 105 | 122; 87K 149 | 150 | 175;
// 183K 932 | 954 | 1165.  d = 96: 81K 103 | 98 | 118; 108K 373 | 392 | 478.  d = 64,
// where VALU work bounds both and two workgroups of 128 rows fit a CU: 35K 127 |
// 87 | 68; 43K 31 | 24 | 28; 76K 190 | 160 | 184; 107K 216 | 216 | 266; 115K 135 |
// 141 | 185; 172K 274 | 261 | 358.
// Short ones (many heads of them): a workgroup is mostly its start and end, so
// what counts is how often the CUs are filled.  One filling (256 workgroups) up to
// S = 512 and, as the tiles' lengths part, 3/16 to 1/4 workgroup more per row of S
// past it, or, for 128 rows, two fillings where 256 rows take two as well.  d = 128,
// 8 | 4 | 2, heads x S: 48 x 256 13 | 12 | 9.4, 92 x 256 13 | 13 | 16, 140 x 256 14 |
// 19 | 25; 32 x 512 18 | 15 | 11, 38 x 512 19 | 16 | 17, 78 x 512 20 | 24 | 30; 22 x 1024
// 28 | 22 | 20, 31 x 1024 29 | 25 | 28, 62 x 1024 35 | 39 | 58; 16 x 2048 47 | 33 | 31, 18
// x 2048 48 | 35 | 43; 140 x 257 26 | 23 | 24.  Up to 128 rows all have one workgroup
// per head and 8 is best (376 x 64 10.4 | 14 | 15), at d = 64 4 (7.5 | 7.0 | 9.8),
// which there takes the whole range but one filling against two of S <= 256 (188 x
// 129 7.3 | 8.3 | 13.8).
int row_groups(const AttnShape &s) {
  const long long heads = (long long)s.b * s.Hl, rows = heads * s.S;
  const long long b2 = heads * ((s.S + 63) / 64), b4 = heads * ((s.S + 127) / 128),
                  b8 = heads * ((s.S + 255) / 256);
  if (s.S <= 128) return s.d == 64 ? 4 : 8;
  const long long past = s.S > 512 ? s.S - 512 : 0;
  if (rows <= 38400 && b2 <= 256 + past * (s.d == 64 ? 4 : 3) / 16) return 2;
  if (s.d == 64) return rows <= 106496 && !(s.S <= 256 && b8 <= 256 && b4 > 256) ? 4 : 8;
  const bool few = b4 <= 256 + past * (s.d == 128 ? 3 : 4) / 16 || (b8 > 256 && b4 <= 512);
  return rows <= 81920 && few ? 4 : 8;
}

// Whether the pipelined loop follows the row sums or forms the row maxima: a
// few percent less time per tile against a check of O and the sums at the end of
// the workgroup, where 256-row workgroups of d = 128 also lose to registers kept
// in scratch around the loop.  Forward, us, maxima | sums, 240K rows in sequences
// of S, 8 heads on 2: d = 128: S = 1024 100 | 108; 3000 187 | 195; 6000 340 | 341;
// 8192 370 | 367; 32K 1783 | 1743.  d = 96: 1024 88 | 91; 4096 190.5 | 190.5; 6000 282 |
// 278; 32K 1477 | 1428.  d = 80: 4096 180 | 182; 6000 268 | 265; 32K 1375 | 1327.  d =
// 64: 2048 87.3 | 89.6; 3000 120.1 | 120.3; 4096 144 | 142; 32K 1118 | 1055.  128 rows:
// d = 128: 2048 43.3 | 44.1; 4096 60.8 | 59.4; d = 96: 2048 34.6 | 35.2; 4096 50.3 | 48.8.
bool follows_sums(const AttnShape &s, int R) {
  return s.S > (R == 4 || s.d == 64 ? 3072 : s.d == 128 ? 6144 : 4608);
}

}  // namespace

hipError_t launch_attn_fwd(const RowView &q, const RowView &k, const RowView &v,
                           const RowView &o, float *lse, const AttnShape &s, bool sharded,
                           hipStream_t stream) {
  const int R = row_groups(s);
  const bool follow = follows_sums(s, R);
  const int qtiles = (s.S + 32 * R - 1) / (32 * R);
  const int heads_total = s.b * s.Hl;
  const long long blocks = (long long)qtiles * heads_total;
  if (blocks == 0) return hipSuccess;
  const float c = s.scale * 1.4426950408889634f;
  const int n_rep = s.Hl / s.Hkl;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(kThreads), 0, stream, q, k, v, o, lse,
                       s.S, s.Hl, n_rep, heads_total, qtiles, c);
  };
  auto by_groups = [&](auto dim, auto sh) {
    constexpr int D = decltype(dim)::value;
    constexpr bool SH = decltype(sh)::value;
    switch (R) {
      case 2: go(attn_fwd_split_kernel<D, SH, 2>); break;
      case 4:
        if constexpr (D == 64) go(attn_fwd_split_kernel<D, SH, 4>);
        else go(follow ? attn_fwd_kernel<D, SH, 2, true> : attn_fwd_kernel<D, SH, 2, false>);
        break;
      default:
        go(follow ? attn_fwd_kernel<D, SH, 1, true> : attn_fwd_kernel<D, SH, 1, false>);
        break;
    }
  };
  auto by_dim = [&](auto sh) {
    switch (s.d) {
      case 64: by_groups(std::integral_constant<int, 64>{}, sh); break;
      case 80: by_groups(std::integral_constant<int, 80>{}, sh); break;
      case 96: by_groups(std::integral_constant<int, 96>{}, sh); break;
      default: by_groups(std::integral_constant<int, 128>{}, sh); break;
    }
  };
  if (sharded)
    by_dim(std::true_type{});
  else
    by_dim(std::false_type{});
  return hipGetLastError();
}

}  // namespace basp
