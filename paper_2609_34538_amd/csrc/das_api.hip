// Host side of the DAS attention library: argument validation, split
// planning, workspace sizing and kernel dispatch behind the C ABI of das.h.
//
// Every check runs before the first HIP call, so a rejected request has
// enqueued nothing and the checks can be exercised without a GPU.

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>

#include "das_internal.h"

namespace das {
namespace {

constexpr size_t kAlign = 256;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

int elem_bytes(int dtype) { return dtype == DAS_F32 ? 4 : 2; }

bool aligned(const void *ptr, size_t a) { return reinterpret_cast<uintptr_t>(ptr) % a == 0; }

das_status check_cache(const das_cache *c) {
  if (!c) return DAS_ERR_NULL;
  if (!c->k_pool || !c->v_pool) return DAS_ERR_NULL;
  if (!aligned(c->k_pool, 16) || !aligned(c->v_pool, 16)) return DAS_ERR_ALIGN;
  if (c->dtype != DAS_F32 && c->dtype != DAS_BF16) return DAS_ERR_DTYPE;
  if (c->num_depths < 1 || c->num_depths > DAS_MAX_DEPTH) return DAS_ERR_SHAPE;
  if (c->num_layers < 1 || c->num_kv_heads < 1 || c->num_pages < 1) return DAS_ERR_SHAPE;
  if (c->num_kv_heads > 65535) return DAS_ERR_SHAPE;
  if (c->num_k_planes < 1 || c->num_v_planes < 1) return DAS_ERR_SHAPE;
  if (c->head_dim != 64 && c->head_dim != 96 && c->head_dim != 128) return DAS_ERR_SHAPE;
  for (int r = 1; r <= c->num_depths; ++r) {
    if (c->k_plane[r] < -1 || c->k_plane[r] >= c->num_k_planes) return DAS_ERR_SHAPE;
    if (c->v_plane[r] < -1 || c->v_plane[r] >= c->num_v_planes) return DAS_ERR_SHAPE;
  }
  return DAS_OK;
}

das_status check_batch(const das_batch *b) {
  if (!b) return DAS_ERR_NULL;
  if (!b->prefix_len || !b->block_table) return DAS_ERR_NULL;
  if (!aligned(b->prefix_len, 4) || !aligned(b->block_table, 4) || !aligned(b->dev_error, 4))
    return DAS_ERR_ALIGN;
  if (b->batch < 1 || b->batch > 65535 || b->max_pages_per_seq < 1) return DAS_ERR_SHAPE;
  // positions (pages x 64) and table offsets (B x pages) stay within int32
  if (b->max_pages_per_seq > (1 << 24) ||
      static_cast<long long>(b->batch) * b->max_pages_per_seq > 0x7fffffffLL)
    return DAS_ERR_SHAPE;
  return DAS_OK;
}

// Which kernel family (and schedule) runs a request. The balanced schedule
// serves batches with many (sequence, KV head) units: every resident wave
// streams an equal share of all tiles, so unequal prefix lengths leave no
// idle slots. With few units for the chip's workers (at most 8 workers per
// unit) each worker holds a short run behind its dependent start-up round
// trips and leaves one piece per unit it shares, and the split grid's
// chunks, dealt out by the hardware dispatcher, are faster; a single
// sequence has nothing to balance and keeps the split grid too.
bool balanced_pays(const das_cache *c, const das_batch *b, int rows) {
  return 8LL * b->batch * c->num_kv_heads >
         static_cast<long long>(kNumCUs) *
             balanced_workers_per_cu(rows, c->head_dim, elem_bytes(c->dtype));
}

// fp32 requests run on the matrix cores too (full fp32 products). Narrow
// blocks over few tiles take the vector-ALU plan, and in its place the
// workgroup-per-chunk kernel (plan_chunks): the split grid's single waves
// stream a 16-token tile at a time there (55 heads x 331 tokens x 1 row: split
// grid 48.6, vector ALU 45.2, chunks 40.6 us for four calls).
int choose_path(const das_cache *c, const das_batch *b, int rows, const das_attn_options *o) {
  const int want = o ? o->path : DAS_PATH_AUTO;
  if (want != DAS_PATH_AUTO) return want;
  const long long units = static_cast<long long>(b->batch) * c->num_kv_heads;
  if (c->dtype == DAS_F32 && rows <= 16 && units * b->max_pages_per_seq <= 2048)
    return DAS_PATH_VALU;
  if (b->batch >= 2 && b->batch <= kBalancedMaxBatch && rows <= balanced_max_rows(c->head_dim) &&
      !(o && o->pages_per_split != 0) && balanced_pays(c, b, rows))
    return DAS_PATH_BALANCED;
  return DAS_PATH_MFMA;
}

struct Plan {
  int path;
  int chunk_tiles;      // > 0: one workgroup per chunk of so many tiles
  int rows;             // w * G query rows per (sequence, kv head)
  int pages_per_split;
  int nsplit;
  int nsplit_ml;        // nsplit rounded up to a multiple of 4
  int n_workers;        // balanced schedule: workers launched
  int piece_cap;        // balanced schedule: pieces the workspace holds
  int piece_stride;     // matrix-core kernels: bytes of one piece record
  size_t ws_o_bytes, ws_ml_bytes, ws_rec_bytes, total;
};

// Prefix pages of one sequence are cut into splits of pages_per_split pages;
// each (split, KV head, row tile) is one chunk of work, one workgroup. The
// default aims for about 512 chunks (two single-wave workgroups per compute
// unit of a 256-CU part; 2048 row tiles where they share a workgroup): with
// `units` = sequences x KV heads x row tiles, each (sequence, KV head) gets
// max(2, the largest power of two <= 512 / units) splits, and a split holds
// between 2 and 32 pages. (Single-sequence call 16.2 / 15.8 / 15.4 / 16.0 /
// 17.0 / 19.8 us at 2 / 3 / 4 / 5 / 6 / 8 pages, the default 4; four such
// sequences 39.7 against 40.5 with a target of 1024.)
das_status plan_path(const das_cache *c, const das_batch *b, int w, const das_attn_options *o,
                     int path, Plan *plan) {
  const int es = elem_bytes(c->dtype);
  plan->path = path;
  if (plan->path == DAS_PATH_BALANCED) {
    if (b->batch > kBalancedMaxBatch || plan->rows > balanced_max_rows(c->head_dim))
      return DAS_ERR_UNSUPPORTED;
    // workers: one per resident single-wave workgroup of the chip; pieces:
    // at most units + workers - 1 (index unit + worker)
    plan->n_workers = kNumCUs * balanced_workers_per_cu(plan->rows, c->head_dim, es);
    plan->piece_cap = b->batch * c->num_kv_heads + plan->n_workers;
    plan->pages_per_split = 0;
    plan->nsplit = 0;
    plan->nsplit_ml = 0;
    // a piece record: the rows' outputs, then 16 bytes per row
    plan->piece_stride = static_cast<int>(piece_record_bytes(plan->rows, c->head_dim, es));
    const size_t pieces = static_cast<size_t>(plan->piece_cap);
    plan->ws_o_bytes = pieces * plan->piece_stride;
    plan->ws_ml_bytes = 0;
    plan->ws_rec_bytes =
        align_up(static_cast<size_t>(b->batch) * c->num_kv_heads * 2 * sizeof(int32_t));
    plan->total = plan->ws_o_bytes + plan->ws_rec_bytes;
    // merge grid: (sequence, KV head) x 64 threads along x
    if (static_cast<long long>(b->batch) * c->num_kv_heads * 64 > 0xffffffffLL)
      return DAS_ERR_SHAPE;
    return DAS_OK;
  }
  plan->n_workers = 0;
  plan->piece_cap = 0;
  plan->piece_stride = 0;
  plan->ws_rec_bytes = 0;
  const int maxp = b->max_pages_per_seq;
  int pps = o ? o->pages_per_split : 0;
  int even_pps = 0;  // > pps: fewer splits, of equal length
  if (pps == 0) {
    const long tile_rows = plan->path == DAS_PATH_MFMA ? (plan->rows <= 16 ? 16 : 32)
                                                      : valu_tile_rows(plan->rows);
    const long units = static_cast<long>(b->batch) * c->num_kv_heads *
                       ((plan->rows + tile_rows - 1) / tile_rows);
    // about two chunks per CU: longer chunks amortise their first round
    // trip and leave fewer partials to merge. Matrix-core blocks of more than
    // 32 rows run their row tiles as the waves of one workgroup (two per CU):
    // they take four times the row-tile chunks. On the vector-ALU path a
    // split may be one page.
    const bool mfma = plan->path == DAS_PATH_MFMA;
    const long target = mfma && plan->rows > 32 ? 2048 : 512;
    long splits = 2;
    while (splits * 2 * units <= target) splits *= 2;
    long want = maxp / splits;
    const long least = mfma && es == 2 ? 2 : 1;
    if (want < least) want = least;
    if (want > 32) want = 32;
    pps = static_cast<int>(want);
    // Row tiles that share a workgroup: the division above rounds down and so
    // adds one short split or more to the planned ones. The prefix and the block
    // are cut into `splits` even ones instead, with the longer splits,
    // - for two row tiles of bf16 where they are more than three workgroups per
    //   CU, which then get three or four each (even ones three, or less and
    //   alike): 96 heads x 12000 tokens x 64 rows, dh 64, 9 -> 8 splits 68.7 ->
    //   59.9 us; 55 heads x 4000, dh 96, 22 -> 16 splits 30.8 -> 25.3; but 40
    //   heads x 8000 x 48 rows, dh 64, 19 splits 23.9 against 25.6 with 16. 776
    //   shapes of 24-256 units x 1000-16000 tokens 1.03-1.06x, at worst 0.95;
    // - for four waves, and for fp32, which a short split costs less than a
    //   longer one, where those past the first round of workgroups (two of four
    //   waves per CU, four of two) hold more than half a split's pages and the
    //   even ones' rounds take no more pages in turn (a twentieth aside): 8 heads x
    //   30000 tokens x 128 rows, dh 128, 68 -> 59 splits 51.5 -> 39.8 us; 18 x 55
    //   heads x 152-319 x 232 rows, dh 64, 3 -> 2 splits 114 -> 94; but not 4 x 8
    //   x 16384 x 128 rows, whose 17th split is one page (66.1 against 67.2), and
    //   not 40 heads x 8000 x 72 rows (three row tiles: 640 even workgroups are two
    //   rounds), dh 96, 43.1 against 46.1; fp32 96 heads x 8000 x 64 rows, dh 96, 218
    //   against 229.
    // The workspace stays sized for the former count.
    if (mfma && plan->rows > 32 && pps < 32) {
      const long nw = mfma_waves(plan->rows), n_rt = (plan->rows + 31) / 32;
      const long wgs = units / n_rt * ((n_rt + nw - 1) / nw);  // of one split
      const long round = (nw == 4 ? 2 : 4) * kNumCUs;
      const int even = static_cast<int>((maxp + splits) / splits);
      const bool uneven = nw == 2 && es == 2 && splits_of(maxp, pps) * wgs > 3 * kNumCUs;
      // pages that the rounds of workgroups take one after the other
      auto pages = [&](int p) { return (splits_of(maxp, p) * wgs + round - 1) / round * p; };
      if (uneven || (2 * (maxp + 1 - round / wgs * pps) > pps &&
                     20 * pages(even) <= 21 * pages(pps)))
        even_pps = even;
    }
  }
  // at most maxp + 1 pages: one split then holds any sequence and its block
  if (pps > maxp + 1) pps = maxp + 1;
  if (plan->path == DAS_PATH_MFMA && pps > kMaxPagesPerSplit) pps = kMaxPagesPerSplit;
  plan->pages_per_split = pps;
  plan->nsplit = splits_of(maxp, pps);
  // Every grid dimension of the launches stays within what HIP accepts:
  // at most 2^32 - 1 work-items (workgroups x threads) per dimension.
  const long long kMaxItems = 0xffffffffLL;
  const long long units = static_cast<long long>(b->batch) * c->num_kv_heads;
  if (plan->path == DAS_PATH_MFMA) {
    const long long nq = mfma_tiles_per_wave(plan->rows), nw = mfma_waves(plan->rows);
    const long long n_rt = (plan->rows + 16 * nq - 1) / (16 * nq);
    const long long chunks = units * plan->nsplit * ((n_rt + nw - 1) / nw);
    if (chunks * 64 * nw > kMaxItems) return DAS_ERR_SHAPE;
  } else {
    const long long n_rt = (plan->rows + valu_tile_rows(plan->rows) - 1) /
                           valu_tile_rows(plan->rows);
    // grid (splits, KV heads, sequences x row tiles) of 256-thread workgroups
    if (static_cast<long long>(plan->nsplit) * 256 > kMaxItems ||
        static_cast<long long>(b->batch) * n_rt > 65535)
      return DAS_ERR_SHAPE;
  }
  if (units * 64 > kMaxItems) return DAS_ERR_SHAPE;  // the merge: (sequence, KV head) x 64
  plan->nsplit_ml = (plan->nsplit + 3) & ~3;
  if (plan->path == DAS_PATH_MFMA) {
    // one piece record per (sequence, KV head, split)
    plan->piece_stride = static_cast<int>(piece_record_bytes(plan->rows, c->head_dim, es));
    plan->ws_o_bytes = static_cast<size_t>(units) * plan->nsplit * plan->piece_stride;
    plan->ws_ml_bytes = 0;
    plan->total = plan->ws_o_bytes;
    if (even_pps > pps && even_pps <= 32) {
      plan->pages_per_split = even_pps;
      plan->nsplit = splits_of(maxp, even_pps);
    }
    return DAS_OK;
  }
  const size_t per_split_rows =
      static_cast<size_t>(b->batch) * c->num_kv_heads * plan->nsplit * plan->rows;
  plan->ws_o_bytes = align_up(per_split_rows * c->head_dim * sizeof(float));
  plan->ws_ml_bytes = align_up(static_cast<size_t>(b->batch) * c->num_kv_heads * plan->rows *
                               plan->nsplit_ml * sizeof(float));
  plan->total = plan->ws_o_bytes + 2 * plan->ws_ml_bytes;
  return DAS_OK;
}

// The workgroup-per-chunk kernel in place of the plan's own kernels: the units
// (sequence, KV head, row tile of the matrix-core kernels) of a call, of
// `tiles` tiles at most, are cut into ns chunks of kChunkWaves * k tiles, k per
// wave. Chosen where it measured faster than the plan it replaces (uniform and
// ragged batches of 1-48 sequences, 4-2000 units, 24-30000 tokens, both types,
// every head dim, 1-512 rows):
// - one chunk per unit needs no merge (3.9 us and the record traffic), but a
//   CU takes no more than about 38 GB/s from a large pool in memory (50 of a
//   batch's table width, which its lengths do not fill), so long units need
//   several; with k > 1 a wave waits for every tile in turn (1 us and its
//   arithmetic; 0.5 us where the call is under 1 MB, which a loop reads from the
//   L2: 4 fp32 heads x 256 tokens x 4 rows, dh 64, called eagerly 6.6 us with one
//   chunk of five tiles per wave, 7.5 with five chunks and the merge's launch). The
//   estimate below, in us per call and without the launch, weighs these, the
//   whole stream (8.5 TB/s of the table's width: memory gives 6.3, a batch's
//   lengths average less than its table, and between plans that are all bound by
//   it the others decide) and the dispatch of many workgroups. Its constants are
//   fitted to every cut of 3186 calls (8-256 units x 160-16000 tokens, every head
//   dim, 8 and 32 rows, one sequence and four ragged ones, pages spread over 48 GB
//   and cached): the cut it takes is 1.3-1.4 % off the best one on average, and
//   against the split grid in its first form 0.92 at worst (46 calls below 0.97).
//   Single short sequence (55 heads, 331 tokens): 8.9 -> 6.8 us; 4 x 55 heads x
//   512-2048: 33.5 -> 19.4.
// - against the balanced schedule, which does not care how unequal the lengths
//   are: units of up to 1.6 MB (4 x 55 heads x 512-4096 tokens 53.5 -> 47 us,
//   but 1024-8192 tokens 51 against 61), and, when they do not all fit at once,
//   up to 450 MB in all, less what the last round leaves idle (8 x 55 x
//   512-2048 40 -> 37 us, 16 x 55 x 512-4096 131 against 141); the same while
//   the split grid's units fill one to two rounds (48 x 8 heads x 500-4096, dh
//   128, 32 rows 94 against 111). fp32 blocks of two row tiles are bound by
//   the matrix cores and gain from two waves per SIMD: 16 x 55 heads x 512-4096
//   x 32 rows 355 -> 328 us.
// - against the split grid, blocks of one row tile: otherwise always, but for
//   several chunks where that grid fills the chip (below): 80 heads x 4000, dh 64,
//   26.0 -> 20.8 us; 512 units x 1024-8192, dh 128, 20 rows, 239 -> 200; fp32 512
//   units x 512-4096, dh 128, 32 rows 498 -> 261. Blocks of several row tiles read
//   each tile once per row tile, from the L2 as long as they keep pace (18 tiles
//   per wave; 55 heads x 9000 tokens, 36 per wave, 52 against 65 us): at most one
//   workgroup per CU where a unit has several chunks, and, in bf16, only where
//   the estimate beats the shared ring's: 16 x 8 heads x 1000 tokens x 52 rows, dh
//   128, 28.6 -> 17.9 us, x 512-8192 tokens 61 against 97; 4 x 8 heads x 300
//   tokens x 100 rows 12.7 -> 9.8, x 2500 20-25 us either way. fp32 always: 1.15
//   to 1.19 times the shared ring's rate on average over 813 shapes, though not at
//   every one (24 heads x 6000 tokens x 128 rows, dh 64, 87 against 65 us).
// - in place of the vector-ALU kernel (narrow fp32 blocks over few tiles):
//   always.
void plan_chunks(const das_cache *c, const das_batch *b, int w, size_t ws_bytes, Plan *plan) {
  const int es = elem_bytes(c->dtype), tt = 64 / es, nq = mfma_tiles_per_wave(plan->rows);
  const long long seq_heads = static_cast<long long>(b->batch) * c->num_kv_heads;
  const long long all_tiles =
      static_cast<long long>(kPage / tt) * b->max_pages_per_seq + (w + tt - 1) / tt;
  if (seq_heads > 65536 || all_tiles > 65536) return;
  const int n_rt = (plan->rows + 16 * nq - 1) / (16 * nq);
  const int units = static_cast<int>(seq_heads) * n_rt, tiles = static_cast<int>(all_tiles);
  const float tile_bytes = 128.f * c->head_dim;  // keys and values, 64 * dh each
  const int whole_k = (tiles + kChunkWaves - 1) / kChunkWaves;  // tiles of a wave, one chunk per unit
  const int rounds = (units + kNumCUs - 1) / kNumCUs;
  const bool f32_wide = es == 4 && nq == 2;
  if (plan->path == DAS_PATH_BALANCED && tiles * tile_bytes > 1.6e6f &&
      !(f32_wide && units >= 2 * kNumCUs))
    return;
  if (units > kNumCUs && !f32_wide && (plan->path != DAS_PATH_MFMA || units < 2 * kNumCUs) &&
      tiles * tile_bytes * rounds * kNumCUs > 450e6f)
    return;

  const float t_mem = kChunkWaves * tile_bytes / (b->batch == 1 || es == 4 ? 38e3f : 50e3f);
  const float t_cmp = nq * c->head_dim * (es == 4 ? 16.f / 2400.f : 0.002f);
  const float t_hbm = static_cast<float>(seq_heads) * tiles * tile_bytes / 8.5e6f;
  const float t_wg = nq == 2 ? 0.0115f : 0.0065f;
  const float t_tile = seq_heads * tiles * tile_bytes < 1e6f ? 0.5f : 1.f;
  const size_t stride = piece_record_bytes(plan->rows, c->head_dim, es);
  auto time = [&](int k, int ns) {
    const int m = (units * ns + kNumCUs - 1) / kNumCUs;
    float t = k * (t_tile + t_cmp);
    if (m * k * t_cmp > t) t = m * k * t_cmp;
    if (m * k * t_mem > t) t = m * k * t_mem;
    if (n_rt > 1) t *= 1.1f;
    if (t_hbm > t) t = t_hbm;
    if (units * ns * t_wg > t) t = units * ns * t_wg;
    if (ns > 1) t += 3.9f + 0.012f * ns + static_cast<float>(stride * ns * seq_heads) / 0.88e6f;
    return t;
  };
  // bf16 requests keep the workspace they always asked for; fp32 ones may take
  // more where it is there, up to the allocation-free entry point's scratch
  size_t room = plan->total;
  if (es == 4) room = std::max(room, std::min<size_t>(ws_bytes, DAS_NOALLOC_SCRATCH_BYTES));
  int best_k = 0, best_ns = 0;
  float best = 0.f;
  if (whole_k * kChunkWaves <= kChunkMaxTiles) best = time(best_k = whole_k, best_ns = 1);
  const int most = (n_rt > 1 ? 1 : 2) * kNumCUs / units;  // chunks of a unit
  if (most > 1) {
    for (int k = (whole_k + most - 1) / most; k < whole_k && k * kChunkWaves <= kChunkMaxTiles; ++k) {
      const int ns = (tiles + kChunkWaves * k - 1) / (kChunkWaves * k);
      if (stride * ns * seq_heads <= room) {
        const float t = time(k, ns);
        if (!best_k || t < best) best = t, best_k = k, best_ns = ns;
        if (units * ns <= kNumCUs) break;  // fewer chunks only take longer
      }
    }
  }
  if (!best_k) return;
  // Tables of one page, two row tiles, more units than two per CU: the split grid
  // needs no merge either, and one wave for the three tiles at most: dh 128, 31
  // rows, 440 units 12.1 / 10.6, 880 17.1 / 20.1, 1760 31.4 / 34.7, 3520 53.5 /
  // 60.7 us (split / chunk).
  if (plan->path == DAS_PATH_MFMA && es == 2 && n_rt == 1 && nq == 2 && plan->nsplit == 1 &&
      units > 2 * kNumCUs)
    return;
  // Several chunks of several tiles per wave, 16 units and more: only where the
  // split grid's power of two of splits leaves over 30 % of its 512 waves idle.
  // Elsewhere the two are within a few percent in calls on their own (55 heads x
  // 2048 tokens from memory 13.6 split, 13.8 chunks; 64 x 2000 14.9, 14.4), but a
  // step that commits to many planes is slower with chunks: their key loads
  // displace the written lines from the last-level cache, where the split grid's
  // are non-temporal. Four layers of draft, verifier and the commit to 32 + 32
  // planes, dh 96, split / chunks: 16 units x 2048 80 / 86 us, 24 x 4096 107 / 121,
  // 55 x 2048 121 / 141, 128 x 2048 195 / 228; 8 x 2048 74 / 67, 8 x 8192 101 /
  // 100. Idle waves: 40 units x 4096, dh 64, 143 / 131, dh 96 154 / 160; the same
  // in four sequences with a commit to 6 planes 148 / 125.
  if (plan->path == DAS_PATH_MFMA && es == 2 && n_rt == 1 && best_ns > 1 && best_k > 1 &&
      units >= 16) {
    int splits = 2;
    while (splits * 2 * units <= 512) splits *= 2;
    if (10 * splits * units > 7 * 512) return;
  }
  if (plan->path == DAS_PATH_MFMA && es == 2 && n_rt > 1) {
    // the shared ring: launch, merge and the stream at 4.2 or 3 TB/s (the
    // lengths of a batch vary; chunks of a unit suffer less from that)
    const float slope = b->batch == 1 ? 2.04f : best_ns > 1 ? 1.6f : 1.23f;
    if (best_k > 18 ||
        best > (n_rt == 2 ? 6.f + slope * t_hbm : 9.5f + 1.38f * slope * t_hbm))
      return;
  }
  plan->chunk_tiles = kChunkWaves * best_k;
  plan->nsplit = best_ns;
  plan->piece_stride = static_cast<int>(stride);
  if (best_ns > 1) plan->total = std::max<size_t>(plan->total, stride * best_ns * seq_heads);
}

// The plan of a request. `ws_bytes`: the workspace it has, SIZE_MAX when its
// size is asked for.
das_status make_plan(const das_cache *c, const das_batch *b, int hq, int w,
                     const das_attn_options *o, size_t ws_bytes, Plan *plan) {
  if (hq < 1 || hq % c->num_kv_heads != 0) return DAS_ERR_SHAPE;
  const int group = hq / c->num_kv_heads;
  if (group > 8) return DAS_ERR_UNSUPPORTED;
  if (w < 1 || w > DAS_MAX_BLOCK) return DAS_ERR_SHAPE;
  if (o && (o->pages_per_split < 0 || o->path < DAS_PATH_AUTO || o->path > DAS_PATH_BALANCED))
    return DAS_ERR_SHAPE;
  if (o && (o->path == DAS_PATH_MFMA || o->path == DAS_PATH_BALANCED) && c->dtype != DAS_BF16)
    return DAS_ERR_UNSUPPORTED;
  plan->rows = w * group;
  plan->chunk_tiles = 0;
  const int path = choose_path(c, b, plan->rows, o);
  // where the caller leaves the kernel and its cut to the library; a call that
  // names a path runs that path's kernel
  const bool may_chunk = !o || (o->path == DAS_PATH_AUTO && o->pages_per_split == 0);
  if (c->dtype != DAS_F32 || path == DAS_PATH_VALU) {
    const das_status st = plan_path(c, b, w, o, path, plan);
    if (st == DAS_OK && may_chunk) plan_chunks(c, b, w, ws_bytes, plan);
    return st;
  }
  // fp32 on the matrix cores: the vector-ALU kernel's bounds on the shapes
  // hold for both, and a request whose partials do not fit the workspace it
  // has, or pass the allocation-free entry point's scratch, where those of
  // the vector-ALU plan (other splits) fit keeps that plan.
  Plan matrix;
  matrix.rows = plan->rows;
  matrix.chunk_tiles = 0;
  const das_status st = plan_path(c, b, w, o, DAS_PATH_VALU, plan);
  if (st != DAS_OK || plan_path(c, b, w, o, path, &matrix) != DAS_OK) return st;
  const bool misses_scratch = matrix.total > DAS_NOALLOC_SCRATCH_BYTES &&
                              plan->total <= DAS_NOALLOC_SCRATCH_BYTES;
  const bool misses_ws = matrix.total > ws_bytes && plan->total <= ws_bytes;
  if (!misses_scratch && !misses_ws) *plan = matrix;
  if (may_chunk) plan_chunks(c, b, w, ws_bytes, plan);
  return DAS_OK;
}

// Validates an attention request and fills every launch parameter except the
// workspace pointers. No HIP call.
das_status prepare_attn(const das_cache *c, const das_batch *b, int layer, int kappa, int nu,
                        int hq, int w, const void *q, const void *kb, const void *vb,
                        void *out, float *lse, const das_attn_options *o, size_t ws_bytes,
                        AttnParams *pp, Plan *plan) {
  das_status st = check_cache(c);
  if (st != DAS_OK) return st;
  st = check_batch(b);
  if (st != DAS_OK) return st;
  if (!q || !kb || !vb || !out) return DAS_ERR_NULL;
  if (!aligned(q, 16) || !aligned(kb, 16) || !aligned(vb, 16) || !aligned(out, 16) ||
      !aligned(lse, 4))
    return DAS_ERR_ALIGN;
  if (layer < 0 || layer >= c->num_layers) return DAS_ERR_SHAPE;
  if (kappa < 1 || kappa > c->num_depths || nu < 1 || nu > c->num_depths) return DAS_ERR_DEPTH;
  const int kplane = c->k_plane[kappa];
  const int vplane = c->v_plane[nu];
  if (kplane < 0 || vplane < 0) return DAS_ERR_DEPTH;
  st = make_plan(c, b, hq, w, o, ws_bytes, plan);
  if (st != DAS_OK) return st;

  const int dh = c->head_dim;
  const size_t eb = static_cast<size_t>(elem_bytes(c->dtype));
  const size_t layer_elems = static_cast<size_t>(c->num_kv_heads) * c->num_pages * kPage * dh;
  AttnParams &p = *pp;
  p.k_layer = static_cast<const char *>(c->k_pool) +
              (static_cast<size_t>(kplane) * c->num_layers + layer) * layer_elems * eb;
  p.v_layer = static_cast<const char *>(c->v_pool) +
              (static_cast<size_t>(vplane) * c->num_layers + layer) * layer_elems * eb;
  p.q = q;
  p.kb = kb;
  p.vb = vb;
  p.out = out;
  p.lse = lse;
  p.prefix_len = b->prefix_len;
  p.block_table = b->block_table;
  p.dev_error = b->dev_error;
  p.ws_o = p.ws_m = p.ws_l = nullptr;
  p.ws_rec = nullptr;
  p.batch = b->batch;
  p.hq = hq;
  p.hkv = c->num_kv_heads;
  p.group = hq / c->num_kv_heads;
  p.w = w;
  p.rows = plan->rows;
  p.num_pages = c->num_pages;
  p.max_pages = b->max_pages_per_seq;
  p.pages_per_split = plan->pages_per_split;
  p.nsplit = plan->nsplit;
  p.chunk_tiles = plan->chunk_tiles;
  p.nsplit_ml = plan->nsplit_ml;
  p.n_workers = plan->n_workers;
  p.piece_cap = plan->piece_cap;
  p.piece_stride = plan->piece_stride;
  // log2(e) / sqrt(dh): logits are kept in base-2 units so exp2 can be used.
  const double log2e = 1.4426950408889634074;
  p.scale_log2 = static_cast<float>(log2e / __builtin_sqrt(static_cast<double>(dh)));
  return DAS_OK;
}

// Enqueues a prepared request with its workspace (plan.total bytes at ws,
// 256-byte aligned): the attention kernel, then the split merge when a
// sequence can span several splits.
das_status launch_attn(AttnParams p, const Plan &plan, int dtype, int dh, void *ws,
                       hipStream_t stream) {
  char *wsb = static_cast<char *>(ws);
  p.ws_o = reinterpret_cast<float *>(wsb);
  p.ws_m = reinterpret_cast<float *>(wsb + plan.ws_o_bytes);
  p.ws_l = reinterpret_cast<float *>(wsb + plan.ws_o_bytes + plan.ws_ml_bytes);
  p.ws_rec = reinterpret_cast<int32_t *>(wsb + plan.ws_o_bytes + 2 * plan.ws_ml_bytes);
  if (plan.path == DAS_PATH_BALANCED && !plan.chunk_tiles)
    return launch_attn_balanced(p, dtype, dh, stream) == hipSuccess ? DAS_OK : DAS_ERR_HIP;
  const bool valu = plan.path == DAS_PATH_VALU && !plan.chunk_tiles;
  const hipError_t e = plan.chunk_tiles ? launch_attn_chunk(p, dtype, dh, stream)
                       : valu           ? launch_attn_valu(p, dtype, dh, stream)
                                        : launch_attn_mfma(p, dtype, dh, stream);
  if (e != hipSuccess) return DAS_ERR_HIP;
  // one split per sequence: the attention kernel wrote every output itself
  if (plan.nsplit > 1 && (valu ? launch_attn_combine(p, dtype, dh, 1, stream)
                               : launch_attn_combine_records(p, dtype, dh, stream)) != hipSuccess)
    return DAS_ERR_HIP;
  return DAS_OK;
}

das_status attn_common(const das_cache *c, const das_batch *b, int layer, int kappa, int nu,
                       int hq, int w, const void *q, const void *kb, const void *vb, void *out,
                       float *lse, void *ws, size_t ws_bytes, const das_attn_options *o,
                       hipStream_t stream) {
  AttnParams p;
  Plan plan;
  const das_status st = prepare_attn(c, b, layer, kappa, nu, hq, w, q, kb, vb, out, lse, o,
                                     ws_bytes, &p, &plan);
  if (st != DAS_OK) return st;
  if (!ws || ws_bytes < plan.total) return DAS_ERR_WORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) % kAlign != 0) return DAS_ERR_WORKSPACE;
  return launch_attn(p, plan, c->dtype, c->head_dim, ws, stream);
}

// ---------------------------------------------------------------------------
// Library-owned scratch of the allocation-free attention entry point: one
// copy per GPU, part of the code object (the loader places it when the
// library's code is loaded on a device, and it lives until the process ends).
// Host code never passes `scratch` itself to a kernel (in host code the name
// stands for a host-side shadow, not a device address): the device address of
// each GPU's copy is looked up once per device with hipGetSymbolAddress, with
// that device current, and kept in scratch_ptr[].
// ---------------------------------------------------------------------------
constexpr int kMaxDevices = 64;
__device__ __attribute__((aligned(256))) uint8_t scratch[DAS_NOALLOC_SCRATCH_BYTES];
void *scratch_ptr[kMaxDevices];
std::mutex scratch_mutex;

// Device address of the current device's scratch copy, or nullptr.
void *scratch_of_current_device(das_status *st) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) {
    *st = DAS_ERR_HIP;
    return nullptr;
  }
  if (dev >= kMaxDevices) {
    *st = DAS_ERR_UNSUPPORTED;
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_ptr[dev]) {
    void *ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      *st = DAS_ERR_HIP;
      return nullptr;
    }
    scratch_ptr[dev] = ptr;
  }
  return scratch_ptr[dev];
}

}  // namespace
}  // namespace das

using namespace das;

extern "C" {

size_t das_attn_workspace_bytes_ex(const das_cache *cache, const das_batch *batch,
                                   int32_t num_q_heads, int32_t block_len,
                                   const das_attn_options *opts) {
  if (check_cache(cache) != DAS_OK || check_batch(batch) != DAS_OK) return 0;
  Plan plan;
  if (make_plan(cache, batch, num_q_heads, block_len, opts, SIZE_MAX, &plan) != DAS_OK) return 0;
  return plan.total;
}

size_t das_attn_workspace_bytes(const das_cache *cache, const das_batch *batch,
                                int32_t num_q_heads, int32_t block_len) {
  return das_attn_workspace_bytes_ex(cache, batch, num_q_heads, block_len, nullptr);
}

das_status das_attn_policy(const das_cache *cache, const das_batch *batch, int32_t layer,
                           int32_t kappa, int32_t nu, int32_t num_q_heads, int32_t block_len,
                           const void *q, const void *k_blk, const void *v_blk, void *out,
                           float *lse, void *workspace, size_t workspace_bytes,
                           const das_attn_options *opts, hipStream_t stream) {
  return attn_common(cache, batch, layer, kappa, nu, num_q_heads, block_len, q, k_blk, v_blk,
                     out, lse, workspace, workspace_bytes, opts, stream);
}

das_status das_attn_policy_noalloc(const das_cache *cache, const das_batch *batch,
                                   int32_t layer, int32_t kappa, int32_t nu,
                                   int32_t num_q_heads, int32_t block_len, const void *q,
                                   const void *k_blk, const void *v_blk, void *out, float *lse,
                                   const das_attn_options *opts, hipStream_t stream) {
  AttnParams p;
  Plan plan;
  das_status st = prepare_attn(cache, batch, layer, kappa, nu, num_q_heads, block_len, q,
                               k_blk, v_blk, out, lse, opts, DAS_NOALLOC_SCRATCH_BYTES, &p,
                               &plan);
  if (st != DAS_OK) return st;
  if (plan.total > DAS_NOALLOC_SCRATCH_BYTES) return DAS_ERR_WORKSPACE;
  // the stream must belong to the current device, whose scratch copy is used
  if (stream) {
    int cur = -1, sdev = -1;
    if (hipGetDevice(&cur) != hipSuccess || hipStreamGetDevice(stream, &sdev) != hipSuccess)
      return DAS_ERR_HIP;
    if (sdev != cur) return DAS_ERR_UNSUPPORTED;
  }
  void *ws = scratch_of_current_device(&st);
  if (!ws) return st;
  return launch_attn(p, plan, cache->dtype, cache->head_dim, ws, stream);
}

das_status das_attn_draft_maturev(const das_cache *cache, const das_batch *batch,
                                  int32_t layer, int32_t draft_depth, int32_t num_q_heads,
                                  int32_t block_len, const void *q, const void *k_blk,
                                  const void *v_blk, void *out, float *lse, void *workspace,
                                  size_t workspace_bytes, hipStream_t stream) {
  if (!cache) return DAS_ERR_NULL;
  // Mature-V: keys at the draft depth, values at the full depth R.
  return attn_common(cache, batch, layer, draft_depth, cache->num_depths, num_q_heads,
                     block_len, q, k_blk, v_blk, out, lse, workspace, workspace_bytes,
                     nullptr, stream);
}

das_status das_attn_verify(const das_cache *cache, const das_batch *batch, int32_t layer,
                           int32_t depth, int32_t num_q_heads, int32_t block_len,
                           const void *q, const void *k_blk, const void *v_blk, void *out,
                           float *lse, void *workspace, size_t workspace_bytes,
                           hipStream_t stream) {
  // Aligned read: keys and values at the same depth.
  return attn_common(cache, batch, layer, depth, depth, num_q_heads, block_len, q, k_blk,
                     v_blk, out, lse, workspace, workspace_bytes, nullptr, stream);
}

das_status das_kv_append(const das_cache *cache, const das_batch *batch, const void *k_new,
                         const void *v_new, int32_t w_max, const int32_t *num_new,
                         int32_t *len_out, hipStream_t stream) {
  das_status st = check_cache(cache);
  if (st != DAS_OK) return st;
  st = check_batch(batch);
  if (st != DAS_OK) return st;
  if (!k_new || !v_new || !num_new) return DAS_ERR_NULL;
  if (!aligned(k_new, 16) || !aligned(v_new, 16) || !aligned(num_new, 4) ||
      !aligned(len_out, 4))
    return DAS_ERR_ALIGN;
  if (w_max < 1 || w_max > DAS_MAX_BLOCK) return DAS_ERR_SHAPE;
  // The commit's grid: one wave per (plane, layer, KV head), four per
  // 256-thread workgroup, keys and values in separate workgroups; at most
  // 2^32 - 1 work-items along x.
  const long long per_plane = static_cast<long long>(cache->num_layers) * cache->num_kv_heads;
  const long long blocks = (cache->num_k_planes * per_plane + 3) / 4 +
                           (cache->num_v_planes * per_plane + 3) / 4;
  if (blocks * 256 > 0xffffffffLL) return DAS_ERR_SHAPE;
  if (len_out && static_cast<const void *>(len_out) ==
                     static_cast<const void *>(batch->prefix_len))
    return DAS_ERR_SHAPE;
  AppendParams p;
  p.k_new = k_new;
  p.v_new = v_new;
  p.k_pool = cache->k_pool;
  p.v_pool = cache->v_pool;
  p.prefix_len = batch->prefix_len;
  p.block_table = batch->block_table;
  p.num_new = num_new;
  p.len_out = len_out;
  p.dev_error = batch->dev_error;
  p.batch = batch->batch;
  p.n_k_planes = cache->num_k_planes;
  p.n_v_planes = cache->num_v_planes;
  p.layers = cache->num_layers;
  p.hkv = cache->num_kv_heads;
  p.num_pages = cache->num_pages;
  p.max_pages = batch->max_pages_per_seq;
  p.w_max = w_max;
  if (launch_kv_append(p, cache->dtype, cache->head_dim, stream) != hipSuccess)
    return DAS_ERR_HIP;
  return DAS_OK;
}

das_status das_greedy_accept(int32_t batch, int32_t block_len, const int32_t *proposals,
                             const int32_t *target_pred, const int32_t *tested,
                             int32_t *accepted, int32_t *num_keep, int32_t *emitted,
                             int32_t *num_emitted, uint32_t *dev_error, hipStream_t stream) {
  if (!proposals || !target_pred || !accepted || !num_keep) return DAS_ERR_NULL;
  if (batch < 1 || block_len < 1 || block_len > DAS_MAX_BLOCK) return DAS_ERR_SHAPE;
  if (!aligned(proposals, 4) || !aligned(target_pred, 4) || !aligned(tested, 4) ||
      !aligned(accepted, 4) || !aligned(num_keep, 4) || !aligned(emitted, 4) ||
      !aligned(num_emitted, 4) || !aligned(dev_error, 4))
    return DAS_ERR_ALIGN;
  AcceptParams p;
  p.proposals = proposals;
  p.target_pred = target_pred;
  p.tested = tested;
  p.accepted = accepted;
  p.num_keep = num_keep;
  p.emitted = emitted;
  p.num_emitted = num_emitted;
  p.dev_error = dev_error;
  p.batch = batch;
  p.w = block_len;
  if (launch_greedy_accept(p, stream) != hipSuccess) return DAS_ERR_HIP;
  return DAS_OK;
}

const char *das_status_string(das_status status) {
  switch (status) {
    case DAS_OK: return "ok";
    case DAS_ERR_NULL: return "a required pointer is NULL";
    case DAS_ERR_SHAPE: return "a size is out of range or inconsistent";
    case DAS_ERR_DEPTH: return "depth outside 1..R or not stored in the cache";
    case DAS_ERR_DTYPE: return "unknown element type";
    case DAS_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case DAS_ERR_HIP: return "a HIP kernel launch failed";
    case DAS_ERR_UNSUPPORTED: return "request not supported by this build";
    case DAS_ERR_ALIGN: return "a device array is not aligned as required";
  }
  return "unknown status";
}

int32_t das_version(void) { return 100; }

}  // extern "C"
