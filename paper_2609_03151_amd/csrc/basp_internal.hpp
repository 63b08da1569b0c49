// basp_internal.hpp -- host-side launch interfaces between the C ABI layer
// (basp_api.cpp) and the kernel translation units.  Shapes arrive here
// already validated.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/basp.h"

namespace basp {

// n / d for 32-bit n and a divisor d fixed per launch, by multiplication
// (Granlund and Montgomery, "Division by invariant integers using
// multiplication", 1994: the round-up multiplier with the fix-up add).
struct FastDiv {
  uint32_t m, s1, s2;
  static FastDiv make(uint32_t d) {
    uint32_t l = 0;
    while (l < 32 && (1ull << l) < d) ++l;  // ceil(log2 d)
    FastDiv f;
    f.m = (uint32_t)((((1ull << 32) * ((1ull << l) - d)) / d + 1) & 0xFFFFFFFFull);
    f.s1 = l < 1 ? l : 1;
    f.s2 = l > 1 ? l - 1 : 0;
    return f;
  }
  // High half of m*n written as a 64-bit product, which the device compiler
  // turns into one multiply-high; callable on the host for checking.
  __host__ __device__ __forceinline__ uint32_t div(uint32_t n) const {
    const uint32_t t1 = (uint32_t)(((uint64_t)m * n) >> 32);
    return (t1 + ((n - t1) >> s1)) >> s2;
  }
};

// Work schedule of the key-stationary backward pass (dV and dK).  A key
// tile is kKvKeys keys; the rows it needs, [k0, S), are cut at multiples of
// the chunk (T key tiles long; bwd_chunks picks it), and a unit is one (key
// tile kt, row chunk ch) pair, for all query heads of the kv head or one part
// of them, that writes its own partial sum.  Per
// (sequence, kv head) there are kv_units(n, T) units for n row chunks: first
// the units that start at their chunk's first row ("full"), chunk by chunk
// (chunk ch has tiles 0 .. ch*T of them); then the diagonal units (key tile
// inside its first chunk but not at its start), longest first (exactly so
// when S fills whole chunks; a partial last chunk's are shorter).  Units
// whose tile lies past S, or whose rows are empty, do nothing.  Longer chunks
// mean fewer partial sums to write and add, shorter ones more, smaller units
// to balance.  kv_chunk_rows is the chunk of a share that fills the GPU with
// units of all query heads: a quarter of the sequence, between 2048 and 8192
// rows, measured best.  Past S = 128K the cap grows with S so that there are
// at most 16 chunks: the partial sums take (chunks x S) rows of workspace,
// which would otherwise grow with S squared.  Host-callable for checking.
constexpr int kKvKeys = 128;
constexpr int kKvMaxChunks = 16;
constexpr int kBwdCus = 256;  // compute units the backward's units are spread over

__host__ __device__ inline int kv_chunk_rows(int S) {
  int rows = (S / 4) / kKvKeys * kKvKeys;
  if (rows < 2048) rows = 2048;
  int cap = ((S + kKvMaxChunks - 1) / kKvMaxChunks + kKvKeys - 1) / kKvKeys * kKvKeys;
  if (cap < 8192) cap = 8192;
  if (rows > cap) rows = cap;
  return rows;
}
__host__ __device__ inline int kv_units(int nchunks, int T) {
  return T * nchunks * (nchunks - 1) / 2 + nchunks + nchunks * (T - 1);
}
__host__ __device__ inline void kv_unit(int u, int nchunks, int T, int &kt, int &ch) {
  ch = 0;
  while (ch < nchunks && u >= ch * T + 1) {  // full units of chunk ch
    u -= ch * T + 1;
    ++ch;
  }
  if (ch < nchunks) {
    kt = u;
  } else {  // diagonal units, j-th key tile of its chunk
    ch = u % nchunks;
    kt = ch * T + u / nchunks + 1;
  }
}
// Row steps of `step_rows` at the start of a unit's rows r_lo.. that overlap
// some key of its tile [k0, k0 + kKvKeys) in a wave's 32-key block: the
// masked steps, at most ceil((k0 + kKvKeys - 1 - r_lo) / step_rows).  Every
// later step starts at or after k0 + kKvKeys - 1.
__host__ __device__ inline int kv_masked_steps(int k0, int r_lo, int steps, int step_rows) {
  const int dm = k0 + kKvKeys - 1 - r_lo;
  if (dm <= 0) return 0;
  const int n = (dm + step_rows - 1) / step_rows;
  return n < steps ? n : steps;
}

// How the attention kernels find one tensor of the share.  Row r (a token
// of the full sequence) of sequence beta lies in buffer p[r / rows], at row
// r % rows of that buffer; a row holds row_elems elements, among them the
// rank's heads from head0 on, d elements each:
//   p[r / rows] + ((beta * rows + r % rows) * row_elems + (head0 + h) * d + e)
// A head-sharded local tensor [b, S, nl, d] is the one-buffer case
// (rows = S, row_elems = nl*d, head0 = 0).  The G sequence shards
// [b, S/G, n, d] of the exchange are G buffers (rows = S/G, row_elems = n*d,
// head0 = rank*n/G), so the kernels read and write them in place.  The
// view travels as a kernel argument: 64 buffers keep the largest argument
// list (the key-stationary pass, six views) near 3.3 KB.
constexpr int kMaxViewBuffers = 64;

struct RowView {
  const void *p[kMaxViewBuffers];
  FastDiv by_rows;  // division by `rows`
  uint32_t rows, row_elems, head0;
};

RowView local_view(const void *p, int S, int nl, int d);
RowView shard_view(const void *const *shards, int G, int S, int n, int d, int rank);

// Element pointer of row r of (beta, head h) in view v, and in `left` the
// rows of that buffer from r on.  SH = false: v is known to be one buffer
// (no division).  r must be wave-uniform for the pointer to stay scalar.
template <bool SH, typename T>
__device__ __forceinline__ T *view_row(const RowView &v, int beta, uint32_t r, int h, int d,
                                       uint32_t &left) {
  uint32_t j = 0, t = r;
  if constexpr (SH) {
    j = v.by_rows.div(r);
    t = r - j * v.rows;
  }
  left = v.rows - t;
  return static_cast<T *>(const_cast<void *>(v.p[j])) +
         (((size_t)beta * v.rows + t) * v.row_elems + (size_t)(v.head0 + h) * d);
}

// Every permutation of the library is a batch of strided row copies: G*b
// blocks (member j, sequence beta) of Sg rows, each row a contiguous run of
// row_bytes.  Row t of block (j, beta) goes from
//   src_tab[j] + beta*src_beta + j*src_j + t*src_row + src_off
// to the same expression on the dst side (all in bytes).  A side that is a
// single buffer repeats its pointer in all G table entries.
//
// Two fp32 variants reduce instead of copying (gradients of a kv head that
// several members share): kAddDst adds the source row into the destination
// row; kSumSrc writes the in-order sum of `reps` source rows spaced src_rep
// bytes apart (the first taken as is, each next one added).
enum class PermMode { kCopy, kAddDst, kSumSrc };

struct PermShape {
  int b, G, Sg;
  uint64_t row_bytes;
  uint64_t src_beta, src_j, src_row, src_off;
  uint64_t dst_beta, dst_j, dst_row, dst_off;
  int vec_bytes;  // 16, 8, 4 or 2: widest access every row start allows
  PermMode mode;  // kCopy unless set; the other two need fp32 rows
  int reps;       // kSumSrc: source rows per destination row
  uint64_t src_rep;
};

hipError_t launch_permute(const void *const *src_tab, void *const *dst_tab, const PermShape &s,
                          hipStream_t stream);

// One permutation with its pointer tables, ready to launch.
struct PermCall {
  PermShape s;
  const void *src[BASP_MAX_GROUP];
  void *dst[BASP_MAX_GROUP];
};

// Up to three permutations in one launch when each has at most
// kMaxBatchBuffers members and all take the same vector width (at least 4
// bytes); otherwise one launch each.  Results are those of launch_permute.
constexpr int kMaxBatchBuffers = 16;
hipError_t launch_permute_batch(const PermCall *calls, int n, hipStream_t stream);

// The owner's send-side split of an fp32 tensor with the conversion to bf16
// fused (round to nearest even): like a kCopy PermShape, but every offset and
// the row length count elements (4 bytes read, 2 written), and vec_elems (4
// or 1) elements move together.
struct CastShape {
  int b, G, Sg;
  uint64_t row_elems;
  uint64_t src_beta, src_j, src_row, src_off;
  uint64_t dst_beta, dst_j, dst_row, dst_off;
  int vec_elems;
};

hipError_t launch_cast_bf16(const float *const *src_tab, uint16_t *const *dst_tab,
                            const CastShape &s, hipStream_t stream);

struct AttnShape {
  int b, S, Hl, Hkl, d;  // local heads
  float scale;
  size_t workspace_bytes = (size_t)-1;  // what the backward's cut has to fit
};

// `sharded`: the views may span several buffers (sequence shards whose row
// count is a multiple of 256, so no workgroup tile straddles two of them).
hipError_t launch_attn_fwd(const RowView &q, const RowView &k, const RowView &v,
                           const RowView &o, float *lse, const AttnShape &s, bool sharded,
                           hipStream_t stream);

// Workspace of the backward: the planes LSE * log2(e) and -D, each
// [b][Hl][Sp] fp32 with Sp = S rounded up to 64 (padding rows zero), then,
// when the key pass has more than one partial sum per key, the dV and dK
// partial sums [slot][b][S][Hkl][d] (fp32), slot = chunk * splits + part.
// Host-callable.
struct BwdChunks {
  int rows;    // rows per chunk (a multiple of kKvKeys)
  int T;       // key tiles per chunk
  int n;       // row chunks
  int units;   // (key tile, row chunk) pairs per (sequence, kv head)
  int splits;  // parts the query heads of a kv head are cut into; units each
  size_t part_offset_floats;
};

__host__ __device__ inline int bwd_plane_rows(int S) { return (S + 63) / 64 * 64; }

inline size_t bwd_workspace_floats(const AttnShape &s, const BwdChunks &ck) {
  size_t floats = ck.part_offset_floats;
  if (ck.n * ck.splits > 1) floats += 2 * (size_t)ck.n * ck.splits * s.b * s.Hkl * s.S * s.d;
  return floats;
}

inline BwdChunks bwd_chunks_of(const AttnShape &s, int rows, int splits) {
  BwdChunks ck;
  ck.rows = rows;
  ck.T = rows / kKvKeys;
  ck.n = (s.S + rows - 1) / rows;
  if (ck.n < 1) ck.n = 1;
  ck.units = kv_units(ck.n, ck.T);
  ck.splits = splits;
  const size_t ld_floats = 2 * (size_t)s.b * s.Hl * bwd_plane_rows(s.S);
  ck.part_offset_floats = (ld_floats + 63) & ~(size_t)63;  // 256-byte aligned
  return ck;
}

// How the key pass is cut.  A workgroup's step is 64 rows of one query head
// (1.3 to 1.7 us); the pass has `mean` of them per CU.  A unit much longer
// than that leaves the other CUs idle while it runs (a kv head of 4 query
// heads at S = 2048 is 128 steps per key tile for 8.5 per CU); a unit much
// shorter pays its start, its 128 KB of partial sums and their reduction
// (together about 4 steps) too often.  The dQ pass, in the same launch, fills
// the CUs beside the units, so a unit is about 2 `mean` steps, at least 8, from
// a mean of 128 on 256 steps and from 512 on `mean` / 2.  Measured on MI355X,
// backward, unit lengths in steps: 8 heads on 2 kv heads of 128, S = 4096 (mean
// 33): 64 steps 128 to 139 us, 32 steps 133 to 142, 16 steps 145, uncut 318; 2 heads on 1, S =
// 8192 (33): 131, 140, -, 308; 4 on 1 of 64, S = 4096 (16): 32 steps 48, 16 steps
// 53, 64 steps 57; 8 on 2, S = 16K (520): 256 steps 1536, 512 steps 1576.
// Up to a mean of 256 rows are cut first, down to 256, then query heads: the
// fewest partial sums.  Past it whole chunks of the longest size
// kv_chunk_rows allows are cut by query heads (S = 16K of 64: 8192 rows of two
// heads 872 us, 4096 of four 885).  Chunks are of equal length: a short last one
// is as many units as a long one (two sequences of 8564 rows, 7 heads on 1 of
// 128, as 8192 + 372 rows of one head 970 us, as equal chunks of two heads 854).
// The partial sums may take what one part per chunk of kv_chunk_rows takes, or
// the static buffer of basp_attn_bwd_noalloc if that is more, and no more than
// the workspace at hand holds; where they would not fit, units take more query
// heads, then longer chunks, at last that cut.  A caller's buffer may be sized
// for another, even a longer sequence, whose own cut needs less (8 heads on 2 of
// 128: 61.6 MB at S = 3000, 33.8 MB at 4096).
inline BwdChunks bwd_chunks(const AttnShape &s) {
  const BwdChunks whole = bwd_chunks_of(s, kv_chunk_rows(s.S), 1);
  if (s.S < 1 || s.Hkl < 1) return whole;
  const int n_rep = s.Hl / s.Hkl;
  const long long ktiles = (s.S + kKvKeys - 1) / kKvKeys;
  const long long mean = (long long)s.b * s.Hl * ktiles * (ktiles + 1) / kBwdCus;
  const long long steps = mean < 4 ? 8 : mean <= 128 ? 2 * mean : mean <= 512 ? 256 : mean / 2;
  const long long cap = kv_chunk_rows(s.S) > 8192 ? kv_chunk_rows(s.S) : 8192;
  auto equal_rows = [&](long long longest) {
    const int n = (int)((s.S + longest - 1) / longest);
    return ((s.S + n - 1) / n + kKvKeys - 1) / kKvKeys * kKvKeys;
  };
  const long long want = steps * 64;  // rows of one head in a unit
  int rows, heads;
  if (mean <= 256) {
    long long r = (want / n_rep + kKvKeys / 2) / kKvKeys * kKvKeys;
    r = r < 256 ? 256 : r > cap ? cap : r;
    rows = equal_rows(r);
    heads = (int)(want / rows < n_rep ? want / rows : n_rep);
  } else {
    rows = equal_rows(cap);
    heads = (int)((want + rows / 2) / rows < n_rep ? (want + rows / 2) / rows : n_rep);
  }
  if (heads < 1) heads = 1;
  const BwdChunks best = bwd_chunks_of(s, rows, (n_rep + heads - 1) / heads);
  auto fit = [&](size_t limit) {  // the cut in `limit` floats
    BwdChunks ck = best;
    if (bwd_workspace_floats(s, ck) <= limit) return ck;
    const size_t slot = 2 * (size_t)s.b * s.Hkl * s.S * s.d;
    const size_t slots = limit > ck.part_offset_floats ? (limit - ck.part_offset_floats) / slot : 0;
    const size_t splits = slots / ck.n;  // below ck.splits
    if (splits < 1) {
      if (slots <= (size_t)whole.n) return whole;
      return bwd_chunks_of(s, equal_rows((s.S + (long long)slots - 1) / (long long)slots), 1);
    }
    const int h = (int)((n_rep + splits - 1) / splits);
    ck.splits = (n_rep + h - 1) / h;
    return ck;
  };
  const size_t whole_floats = bwd_workspace_floats(s, whole);
  const size_t most = whole_floats > BASP_NOALLOC_SCRATCH_BYTES / sizeof(float)
                          ? whole_floats : BASP_NOALLOC_SCRATCH_BYTES / sizeof(float);
  const BwdChunks ck = fit(most);
  const size_t given = s.workspace_bytes / sizeof(float);
  return bwd_workspace_floats(s, ck) <= given ? ck : fit(given);
}

// Row groups of 32 query rows among the 8 waves of a dQ workgroup (R = 8, 4
// or 2; its 8 / R waves per row group share the keys).  Fewer rows per
// workgroup are more workgroups with shorter key loops, for 2-3% (R = 4) to
// 7-10% (R = 2) more time per product once the GPU is full: each K and V tile
// feeds fewer products.  In W = b * Hl * S query rows the lines are where the
// two sides cross (backward, us, MI355X, 110 shares of 2^8.5 to 2^15.5 rows):
// W = 14K 8: 77, 4: 56, 2: 56; 17K one head 145, 94, 88; 21K 59, 55, 62; 31K
// one head 938, 745, 793; 34K 98, 97, 115; 41K 158, 161, 178; 51K 233, 240,
// 256.
inline int dq_row_groups(const AttnShape &s) {
  const long long rows = (long long)s.b * s.Hl * s.S;
  return rows <= 18432 ? 2 : rows <= 36864 ? 4 : 8;
}

// Whether the key pass's units go before the dQ tiles in the launch: the longer
// kind first.  A dQ tile's longest loop, S / 64 tiles of 64 keys x 32 R rows x 3
// products, is 3 R S / 1024 key-pass steps of 64 rows x 128 keys x 4 products.
// (8 heads on 2 kv heads of 128, S = 4096, R = 4: units of 64 steps against 48
// first 128 us, last 135; of 32 steps 147 and 134; 8 on 8, S = 8K, 128 steps
// against 192: 466 and 413.)
inline bool bwd_keys_first(const AttnShape &s, const BwdChunks &ck) {
  const int n_rep = s.Hl / s.Hkl;
  const long long unit = (long long)(ck.rows / 64) * ((n_rep + ck.splits - 1) / ck.splits);
  return unit * 1024 > 3LL * dq_row_groups(s) * s.S;
}

// Workgroups of the two passes.  They go in one launch where its threads are a
// 32-bit count, as a launch's have to be; past that (more than 2^23 - 1 heads and
// kv heads of sequences of up to 256 rows, say) in one launch each.
constexpr int kBwdThreads = 512;
inline long long bwd_dq_blocks(const AttnShape &s) {
  const int rows = 32 * dq_row_groups(s);
  return (long long)((s.S + rows - 1) / rows) * s.b * s.Hl;
}
inline long long bwd_kv_blocks(const AttnShape &s, const BwdChunks &ck) {
  return (long long)ck.units * ck.splits * s.b * s.Hkl;
}
inline bool bwd_one_launch(const AttnShape &s, const BwdChunks &ck) {
  return (bwd_dq_blocks(s) + bwd_kv_blocks(s, ck)) * kBwdThreads <= 0xFFFFFFFFll;
}

// The least workspace the backward runs in: the whole-chunk cut's.
inline size_t attn_bwd_least_workspace_bytes(const AttnShape &s) {
  return bwd_workspace_floats(s, bwd_chunks_of(s, kv_chunk_rows(s.S), 1)) * sizeof(float);
}

// What the cut takes when the workspace does not limit it; never less than the
// least (the whole-chunk cut can take more than the one in use), so
// basp_attn_bwd_noalloc takes what that cut lets it take.
inline size_t attn_bwd_workspace_bytes(AttnShape s) {
  s.workspace_bytes = (size_t)-1;
  const size_t cut = bwd_workspace_floats(s, bwd_chunks(s)) * sizeof(float);
  const size_t least = attn_bwd_least_workspace_bytes(s);
  return cut > least ? cut : least;
}

// Device address of the static scratch buffer of basp_attn_bwd_noalloc
// (BASP_NOALLOC_SCRATCH_BYTES) on the device of `stream` (the current device
// for the null stream), looked up once per device.  Allocates nothing.
hipError_t noalloc_scratch(hipStream_t stream, void **ptr);

// q, k, v and d_o must be one-buffer (local) views, also when `sharded`
// (then only o and the gradients are shard views).
hipError_t launch_attn_bwd(const RowView &q, const RowView &k, const RowView &v,
                           const RowView &o, const float *lse, const RowView &d_o,
                           const RowView &dq, const RowView &dk, const RowView &dv,
                           void *workspace, const AttnShape &s, bool sharded,
                           hipStream_t stream);

}  // namespace basp
