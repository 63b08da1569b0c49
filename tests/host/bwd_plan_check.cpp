// Host check of the cut of the backward's key pass (bwd_chunks in
// basp_internal.hpp), over every combination of many sequence lengths, head
// counts, batch sizes and head dims:
//  * chunks are whole key tiles and cover the sequence; no chunk is empty;
//  * the query-head parts of a kv head are all non-empty and cover the heads;
//  * the workspace holds the planes and every partial sum, is no smaller than
//    one part per row chunk of kv_chunk_rows takes (so the static buffer's
//    limit admits the same shapes), and no larger than both that and the
//    static buffer;
//  * the schedule of the chosen chunks reaches every (key tile, chunk) pair
//    that has rows exactly once;
//  * in a workspace of any size from the least (one part per row chunk of
//    kv_chunk_rows) up, the cut fits, and is the unlimited one from the size
//    the query reports on;
//  * the shapes of the GPU tests are cut the way those tests mean to run;
//  * no launch of the two passes has more than 2^32 - 1 threads, and both go in
//    one where that allows it.
// Prints the number of shapes checked; exits 1 at the first failure.
#include <stdio.h>

#include <algorithm>
#include <set>
#include <utility>
#include <vector>

#include "../../paper_2609_03151_amd/csrc/basp_internal.hpp"

using namespace basp;

static int fail(const char *what, const AttnShape &s) {
  printf("FAIL %s: b=%d S=%d Hl=%d Hkl=%d d=%d\n", what, s.b, s.S, s.Hl, s.Hkl, s.d);
  return 1;
}

// The cut in a workspace of `bytes`: whole chunks and parts that fit it.
static const char *limited(AttnShape s, size_t bytes, const BwdChunks &best, size_t need) {
  s.workspace_bytes = bytes;
  const BwdChunks ck = bwd_chunks(s);
  const int n_rep = s.Hl / s.Hkl;
  if (ck.rows < kKvKeys || ck.T * kKvKeys != ck.rows || (long long)ck.n * ck.rows < s.S ||
      (long long)(ck.n - 1) * ck.rows >= s.S || ck.n > kKvMaxChunks)
    return "chunks in a small workspace";
  if (ck.splits < 1 || ck.splits > n_rep) return "parts in a small workspace";
  for (int p = 0; p < ck.splits; ++p)
    if (p * n_rep / ck.splits >= (p + 1) * n_rep / ck.splits) return "empty part in a small one";
  if (bwd_workspace_floats(s, ck) * sizeof(float) > bytes) return "cut larger than its workspace";
  if (bytes >= need && (ck.rows != best.rows || ck.splits != best.splits))
    return "another cut in a full workspace";
  return nullptr;
}

// Shares at the limit of a launch: many short sequences (b up to 65535).
static const char *launches(const AttnShape &s) {
  const BwdChunks ck = bwd_chunks(s);
  const long long dq = bwd_dq_blocks(s), kv = bwd_kv_blocks(s, ck), most = 0xFFFFFFFFll / kBwdThreads;
  if (dq < 1 || kv < 1 || dq > most || kv > most) return "a pass past a launch's limit";
  return bwd_one_launch(s, ck) == (dq + kv <= most) ? nullptr : "launches";
}

// Local shapes of the GPU tests whose cases stand for a cut: row chunks, parts.
struct Meant {
  int b, S, Hl, Hkl, d, n, splits;
};
const Meant kMeant[] = {
    // without a workspace argument; in place; moving references
    {1, 4096, 4, 1, 128, 8, 1}, {2, 1000, 2, 2, 64, 2, 1}, {3, 320, 2, 2, 64, 1, 1},
    {1, 1024, 2, 1, 128, 4, 1}, {2, 4096, 4, 2, 64, 2, 1}, {2, 4096, 4, 4, 64, 1, 1},
    {2, 8192, 1, 1, 128, 2, 1}, {1, 2048, 2, 1, 128, 8, 1}, {2, 4096, 2, 1, 64, 4, 1},
    {16, 2048, 1, 1, 64, 1, 1},
    // small shapes against the oracle; the long sequence at the cap of 16 chunks
    {1, 2500, 2, 1, 128, 10, 1}, {1, 4096, 4, 2, 64, 4, 1}, {1, 2500, 2, 1, 80, 10, 1},
    {2, 2112, 4, 2, 128, 4, 2}, {1, 4160, 7, 1, 64, 9, 1}, {1, 131200, 1, 1, 64, 16, 1},
    // cuts of small shares
    {1, 1024, 8, 1, 128, 4, 4}, {1, 1100, 7, 1, 96, 5, 4}, {2, 2048, 4, 1, 128, 8, 1},
    {1, 3000, 7, 1, 128, 12, 1}, {3, 769, 6, 2, 80, 4, 2}, {1, 2113, 3, 3, 64, 5, 1},
    {1, 6000, 10, 2, 64, 3, 1}, {1, 8192, 8, 2, 64, 2, 1}, {1, 8192, 8, 8, 64, 1, 1},
    {2, 9000, 10, 2, 128, 2, 2}, {1, 11008, 20, 1, 64, 2, 7},
};

int main() {
  for (const Meant &m : kMeant) {
    const AttnShape s{m.b, m.S, m.Hl, m.Hkl, m.d, 1.f};
    const BwdChunks ck = bwd_chunks(s);
    if (ck.n != m.n || ck.splits != m.splits) return fail("another cut than its test means", s);
  }
  for (int S : {1, 64, 128, 200, 256})
    for (int b : {60000, 65535})
      for (int Hl : {1, 64, 65, 100, 128}) {
        if (S > 64 && Hl > 64) continue;  // bwd_pre's own limit
        const AttnShape s{b, S, Hl, Hl, 64, 1.f};
        if (const char *what = launches(s)) return fail(what, s);
      }
  {  // each pass alone within a launch's limit, both together not
    const AttnShape s{65535, 1, 65, 65, 64, 1.f};
    if (bwd_one_launch(s, bwd_chunks(s))) return fail("one launch too large", s);
    const AttnShape t{65535, 1, 64, 64, 64, 1.f};
    if (!bwd_one_launch(t, bwd_chunks(t))) return fail("one launch would do", t);
  }
  std::vector<int> lengths = {1,    64,   127,  128,  129,  255,  256,  500,   512,   1000,  1024,
                              1500, 2047, 2048, 2049, 3000, 4096, 5000, 8191,  8192,  8193,  12345,
                              16384, 20000, 32768, 65536, 100000, 131072, 131200, 262144, 524289};
  int checked = 0;
  for (int S : lengths)
    for (int b : {1, 2, 3, 16})
      for (int Hkl : {1, 2, 4, 8})
        for (int n_rep : {1, 2, 3, 4, 7, 8, 64})
          for (int d : {64, 80, 128}) {
            const AttnShape s{b, S, Hkl * n_rep, Hkl, d, 1.f};
            const BwdChunks ck = bwd_chunks(s);
            if (ck.rows < kKvKeys || ck.rows % kKvKeys || ck.T * kKvKeys != ck.rows)
              return fail("chunk rows", s);
            if ((long long)ck.n * ck.rows < S || (long long)(ck.n - 1) * ck.rows >= S)
              return fail("chunk count", s);
            if (ck.n > kKvMaxChunks) return fail("more row chunks than the cap", s);
            if (ck.splits < 1 || ck.splits > n_rep) return fail("parts", s);
            for (int p = 0; p < ck.splits; ++p)
              if (p * n_rep / ck.splits >= (p + 1) * n_rep / ck.splits)
                return fail("empty part", s);
            const size_t planes = 2 * (size_t)b * s.Hl * ((S + 63) / 64 * 64) * 4;
            const size_t sum = (size_t)b * S * Hkl * d * 4;
            const size_t parts = (size_t)ck.n * ck.splits;
            const size_t need = attn_bwd_workspace_bytes(s);
            const size_t use = planes + (parts > 1 ? 2 * parts * sum : 0);
            const size_t n0 = (S + kv_chunk_rows(S) - 1) / kv_chunk_rows(S);
            const size_t whole = planes + (n0 > 1 ? 2 * n0 * sum : 0);
            if (need < use || need < whole) return fail("workspace too small", s);
            if (need > std::max(whole, (size_t)BASP_NOALLOC_SCRATCH_BYTES) + 256)
              return fail("workspace too large", s);
            if (attn_bwd_least_workspace_bytes(s) < whole ||
                attn_bwd_least_workspace_bytes(s) > whole + 256)
              return fail("least workspace", s);
            const size_t least = attn_bwd_least_workspace_bytes(s);
            for (size_t bytes : {least, least + 1, least + 2 * sum, (least + need) / 2,
                                 least + (need - least) / 4 * 3, need - 1, need, 2 * need})
              if (const char *what = bytes < least ? nullptr : limited(s, bytes, ck, need))
                return fail(what, s);
            if (b == 1 && d == 64) {
              const int ktiles = (S + kKvKeys - 1) / kKvKeys;
              std::set<std::pair<int, int>> seen;
              for (int u = 0; u < ck.units; ++u) {
                int kt, ch;
                kv_unit(u, ck.n, ck.T, kt, ch);
                if (kt < ktiles && std::max(kt * kKvKeys, ch * ck.rows) < std::min(S, (ch + 1) * ck.rows) &&
                    !seen.insert({kt, ch}).second)
                  return fail("pair twice", s);
              }
              for (int kt = 0; kt < ktiles; ++kt)
                for (int ch = 0; ch < ck.n; ++ch)
                  if (std::max(kt * kKvKeys, ch * ck.rows) < std::min(S, (ch + 1) * ck.rows) &&
                      !seen.count({kt, ch}))
                    return fail("pair missing", s);
            }
            ++checked;
          }
  printf("bwd plan ok %d\n", checked);
  return 0;
}
