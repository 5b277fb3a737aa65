// Commit of verified block K/V into the depth-indexed paged cache
// (Sec. 3.4: full-depth K/V of accepted, materialised inputs are retained;
// App. B.1: draft-side K/V never enter the cache).
//
// One wave per (plane, layer, KV head) of one sequence, four independent waves
// per workgroup, all keys or all values. The wave reads the sequence's length,
// count and the (at most two) page ids its n new positions fall in once, then
//  - keys: copies the n token rows with 16-byte vectors (rows of head_dim
//    are contiguous in both the source and the token-major page);
//  - values: stages token rows in LDS, two 8-position groups of the
//    token-grouped page ([8][dh][8]) per pass and every row at its position's
//    place in them; then, one group after the other, each lane takes a head dim
//    and writes its run of new positions with the widest aligned stores that
//    fit (a full group is one 16-byte store for bf16). The run of a group is
//    the same in every lane, so the choice of stores is a scalar branch, and no
//    group is written in two pieces.
// Commits of few tokens are bound by the dispatch of the waves and their three
// dependent round trips, and by partial lines where they begin or end inside a
// group: 8 tokens that fill their groups 9.2 us, 7 tokens from position 187, in
// two groups, 12.6 (32 + 32 planes x 4 layers x 55 heads, one buffer, graph
// replays). Wide ones are bound by memory. Against staging 16 tokens from the first new
// position with workgroup barriers and per-lane runs: 32 + 32 planes x 4 layers
// x 55 heads x 1, 7, 30 and 64 tokens 10.6, 14.8, 45.4, 80.6 -> 9.6, 14.7,
// 41.8, 70.5 us (265 MB, 3.8 TB/s). Measured and not kept: two or four units
// per wave (17 and 22 us at 7 tokens), two head dims per lane (16 us: twice the
// partial lines per store).
// Pure copies: results are bit-exact.

#include "das_internal.h"

namespace das {
namespace {

constexpr int kWaves = 4;
constexpr int kRows = 16;  // value rows staged per pass: two groups

struct alignas(16) Vec16 {
  uint32_t x, y, z, w;
};

// Elements [lo, hi) of an 8-element row (16-byte aligned for bf16, 32 for
// fp32) from the row's words (two bf16 per word, one fp32), in aligned pieces
// of at most 16 bytes.
template <typename T, int NW>
__device__ __forceinline__ void store_run(T *row, const uint32_t (&v)[NW], int lo, int hi) {
  static_assert(NW * 4 == 8 * static_cast<int>(sizeof(T)), "eight elements");
  auto inside = [&](int a, int b) { return lo <= a && b <= hi; };
  uint32_t *words = reinterpret_cast<uint32_t *>(row);
  if constexpr (sizeof(T) == 2) {
    if (inside(0, 8)) {
      *reinterpret_cast<Vec16 *>(words) = Vec16{v[0], v[1], v[2], v[3]};
      return;
    }
  }
#pragma unroll
  for (int q = 0; q < 8; q += 4) {
    constexpr int HW = NW / 2;  // words of four elements
    const int w0 = q / 4 * HW;
    if (inside(q, q + 4)) {  // 8 bytes (bf16) or 16 bytes (fp32)
      if constexpr (sizeof(T) == 2)
        *reinterpret_cast<uint2 *>(words + w0) = make_uint2(v[w0], v[w0 + 1]);
      else
        *reinterpret_cast<Vec16 *>(words + w0) = Vec16{v[w0], v[w0 + 1], v[w0 + 2], v[w0 + 3]};
      continue;
    }
#pragma unroll
    for (int e = q; e < q + 4; ++e) {
      if constexpr (sizeof(T) == 2) {
        if (e % 2 == 0 && inside(e, e + 2)) {
          words[e / 2] = v[e / 2];
          continue;
        }
        if (e % 2 == 1 && inside(e - 1, e + 1)) continue;
        if (inside(e, e + 1)) row[e] = static_cast<T>(v[e / 2] >> (16 * (e % 2)));
      } else {
        if (inside(e, e + 1)) words[e] = v[e];
      }
    }
  }
}

template <typename T, int DH>
__global__ __launch_bounds__(64 * kWaves) void kv_append_kernel(AppendParams p) {
  constexpr int VEC = 16 / sizeof(T);  // elements per 16-byte vector
  constexpr int NV = DH / VEC;         // vectors per token row
  __shared__ __attribute__((aligned(16))) T stage[kWaves][kRows * DH];

  const int b = blockIdx.y;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int per_plane = p.layers * p.hkv;
  const int k_units = p.n_k_planes * per_plane, v_units = p.n_v_planes * per_plane;
  const int k_blocks = (k_units + kWaves - 1) / kWaves;
  const bool is_v = static_cast<int>(blockIdx.x) >= k_blocks;
  const int rel = (is_v ? blockIdx.x - k_blocks : blockIdx.x) * kWaves + wave;

  const int S = p.prefix_len[b];
  const int n = p.num_new[b];
  const bool bad = S < 0 || n < 0 || n > p.w_max ||
                   static_cast<long>(S) + n > static_cast<long>(p.max_pages) * kPage;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (bad) report_error(p.dev_error, DAS_DEVERR_COMMIT);
    if (p.len_out) p.len_out[b] = bad ? S : S + n;
  }
  // uniform over the wave; no workgroup barrier below
  if (bad || n == 0 || rel >= (is_v ? v_units : k_units)) return;

  // n <= 64 new positions span at most two pages
  const int32_t *table = p.block_table + static_cast<size_t>(b) * p.max_pages;
  const int first_page = S / kPage;
  const int pg0 = table[first_page];
  const int pg1 = table[(S + n - 1) / kPage];
  const bool ok0 = pg0 >= 0 && pg0 < p.num_pages;
  const bool ok1 = pg1 >= 0 && pg1 < p.num_pages;
  if (blockIdx.x == 0 && threadIdx.x == 0 && (!ok0 || !ok1))
    report_error(p.dev_error, DAS_DEVERR_PAGE);

  const int plane = rel / per_plane;
  const int layer = (rel / p.hkv) % p.layers;
  const int h = rel % p.hkv;
  // source [plane][layer][B][w_max][Hkv][DH]; token t's row at src + t * hkv * DH
  const size_t src_off =
      ((((static_cast<size_t>(plane) * p.layers + layer) * p.batch + b) * p.w_max) * p.hkv + h) *
      DH;
  const size_t src_stride = static_cast<size_t>(p.hkv) * DH;
  // destination pages of this (plane, layer, head): [P][64 * DH]
  const size_t dst_head =
      ((static_cast<size_t>(plane) * p.layers + layer) * p.hkv + h) * p.num_pages * kPage * DH;

  if (!is_v) {
    const T *src = static_cast<const T *>(p.k_new) + src_off;
    T *dst = static_cast<T *>(p.k_pool) + dst_head;
    const int total = n * NV;
    // vector v: token v / NV, columns (v % NV) * VEC ..
    auto load = [&](int v) {
      Vec16 r = {0, 0, 0, 0};
      if (v < total) r = *reinterpret_cast<const Vec16 *>(src + (v / NV) * src_stride + (v % NV) * VEC);
      return r;
    };
    auto store = [&](int v, const Vec16 &r) {
      if (v >= total) return;
      const int t = v / NV, c = (v % NV) * VEC;
      const int pos = S + t;
      const bool second = pos / kPage != first_page;
      if (second ? ok1 : ok0) {
        const size_t page = second ? pg1 : pg0;
        *reinterpret_cast<Vec16 *>(dst + (page * kPage + pos % kPage) * DH + c) = r;
      }
    };
    for (int v0 = lane; v0 < total; v0 += 4 * 64) {
      const Vec16 r0 = load(v0), r1 = load(v0 + 64), r2 = load(v0 + 128), r3 = load(v0 + 192);
      store(v0, r0);
      store(v0 + 64, r1);
      store(v0 + 128, r2);
      store(v0 + 192, r3);
    }
    return;
  }

  const T *src = static_cast<const T *>(p.v_new) + src_off;
  T *dst = static_cast<T *>(p.v_pool) + dst_head;
  T *st = stage[wave];  // row r: position gbase + r
  for (int gbase = S & ~7; gbase < S + n; gbase += kRows) {
    const int r0 = max(S - gbase, 0), r1 = min(S + n - gbase, kRows);
    for (int v = lane; v < (r1 - r0) * NV; v += 64) {
      const int r = r0 + v / NV, c = (v % NV) * VEC;
      *reinterpret_cast<Vec16 *>(st + r * DH + c) =
          *reinterpret_cast<const Vec16 *>(src + (gbase + r - S) * src_stride + c);
    }
    // the wave's own LDS writes are read by its other lanes
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int g = 0; g < kRows; g += 8) {
      const int lo = max(r0 - g, 0), hi = min(r1 - g, 8), gp = gbase + g;
      const bool second = gp / kPage != first_page;  // 8 | 64: a group lies in one page
      if (lo >= hi || !(second ? ok1 : ok0)) continue;  // uniform
      T *rows = dst + static_cast<size_t>(second ? pg1 : pg0) * kPage * DH + gp % kPage * DH;
      for (int c = lane; c < DH; c += 64) {
        T e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) e[j] = st[(g + j) * DH + c];
        uint32_t w[2 * sizeof(T)];
        if constexpr (sizeof(T) == 2) {
#pragma unroll
          for (int k = 0; k < 4; ++k)
            w[k] = static_cast<uint32_t>(e[2 * k]) | (static_cast<uint32_t>(e[2 * k + 1]) << 16);
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) w[j] = __float_as_uint(e[j]);
        }
        store_run<T>(rows + c * 8, w, lo, hi);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

template <typename T, int DH>
hipError_t launch_typed(const AppendParams &p, hipStream_t s) {
  const int per_plane = p.layers * p.hkv;
  const int blocks = (p.n_k_planes * per_plane + kWaves - 1) / kWaves +
                     (p.n_v_planes * per_plane + kWaves - 1) / kWaves;
  dim3 grid(blocks, p.batch);
  return launch_kernel(kv_append_kernel<T, DH>, grid, dim3(64 * kWaves), s, p);
}

}  // namespace

hipError_t launch_kv_append(const AppendParams &p, int dtype, int dh, hipStream_t s) {
  if (dtype == DAS_F32) {
    if (dh == 64) return launch_typed<float, 64>(p, s);
    if (dh == 96) return launch_typed<float, 96>(p, s);
    return launch_typed<float, 128>(p, s);
  }
  if (dh == 64) return launch_typed<bf16_t, 64>(p, s);
  if (dh == 96) return launch_typed<bf16_t, 96>(p, s);
  return launch_typed<bf16_t, 128>(p, s);
}

}  // namespace das
