// Matrix-core attention with one workgroup per chunk of a unit (Eq. (2)-(3)),
// for calls whose units hold few tiles.
//
// A unit is one (sequence, KV head, row tile of 16 * NQ query rows); its tiles,
// the draft block's first, then the prefix's, are cut into chunks of
// chunk_tiles. The four waves of a workgroup take a chunk's tiles in turn, each
// with its own running maximum, sum and output, and merge through LDS. Where
// one chunk holds every unit the call is a single launch: no records in
// memory, no merge kernel and no kernel boundary, which are about 4 us of a
// short call's 9; otherwise a chunk leaves one record, a quarter of what four
// single-wave workgroups would.
//
// Nothing in the loop is shared between waves: keys and values go straight
// from memory into the MFMA operand registers (a lane's 16 bytes of a fragment
// are contiguous in either page layout). The next tile's keys are loaded when
// the logits have consumed the current ones, its values after the P.V product,
// so a wave keeps about one tile in flight. That is enough: a CU takes about
// 50 GB/s from memory however many waves ask (55 CUs: 36 GB/s each with two
// waves, 51-54 with 4, 8 or 12), and eight waves per workgroup measured no
// faster. Bound by that rate where few units are long, by the memory's where
// they fill the chip, by the round trips (length, first tile, output) where
// they are short. Measured against the kernels it replaces: 55 heads x 331
// tokens 8.9 -> 6.8 us; 4 x 55 heads x 512-2048 tokens, 16 rows, 33.5 -> 19.4
// us (5.6 TB/s); 32 x 8 heads x 500-4096, dh 128, 32 rows 76 -> 61 us; 8 heads
// x 30011 tokens 37.6 -> 24 us; fp32 4 x 55 heads x 512-2048 83 -> 45 us.
//
// The first round trip of a wave fetches the prefix length, the Q fragments,
// the draft block's tile (whose addresses need neither the length nor the page
// table) and the page ids of its tiles, lane i holding the i-th tile's: at
// most 64 tiles per wave, to which the host limits a chunk.

#include "mfma_tile.h"

namespace das {
namespace {

// 16 bytes per lane of a tile.
template <int POLICY>
__device__ __forceinline__ u32x4 load_frag(__amdgpu_buffer_rsrc_t r, uint32_t voff, int soff) {
  return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, POLICY));
}

template <typename T, int DH, int NQ>
__global__ __launch_bounds__(64 * kChunkWaves) __attribute__((amdgpu_waves_per_eu(2)))
void attn_chunk_kernel(AttnParams p, int n_rt) {
  using G = Geo<T, DH, NQ, 1>;
  constexpr int ES = G::ES, KS = G::KS, DT = G::DT, TT = G::TT, TPP = G::TPP, QK = G::QK;
  constexpr int NW = kChunkWaves;
  constexpr int RS = DH + 4;  // row stride of the merge area (floats)
  // the merge area of one row tile; before that, wave u's part holds the raw
  // values of draft-block tile u ([TT][DH], 64 * DH bytes)
  __shared__ __attribute__((aligned(16))) float part[NW][16 * RS];
  // every wave's row maxima, sums and largest output magnitudes
  __shared__ float sm[NW][16 * NQ], sl[NW][16 * NQ], sa[NW][16 * NQ];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ln = lane & 15;
  const int lg = lane >> 4;
  // workgroup number -> (chunk of a unit, row tile): the row tiles of a chunk
  // are numbered 8 apart, so they start together on one XCD (workgroups are
  // dealt to the 8 XCDs in turn) and share its L2 for the tiles they all read;
  // every unit's first chunk comes before any second one
  int grp = blockIdx.x, rt = 0;
  if (n_rt > 1) {
    const int span = 8 * n_rt, run = grp / span, full = p.batch * p.hkv * p.nsplit / 8;
    const int in = grp % span;
    if (run < full) {
      grp = 8 * run + in % 8;
      rt = in / 8;
    } else {
      grp = 8 * full + in / n_rt;
      rt = in % n_rt;
    }
  }
  const int unit = grp % (p.batch * p.hkv), chunk = grp / (p.batch * p.hkv);
  const int b = unit / p.hkv, kvh = unit % p.hkv;
  const int row0 = rt * (16 * NQ);
  const int nb = (p.w + TT - 1) / TT;  // draft-block tiles, at most 4 <= NW
  const int g0 = chunk * p.chunk_tiles + wave;  // this wave's first tile of the unit

  const int s_raw = p.prefix_len[b];
  // lane i: page id of this wave's i-th tile, tile g0 + NW * i of the unit
  const int my_page = (g0 + NW * lane - nb) / TPP;
  int page_id = 0;
  if (g0 + NW * lane >= nb && my_page < p.max_pages)
    page_id = p.block_table[static_cast<size_t>(b) * p.max_pages + my_page];
  u32x4 qf[NQ][QK];
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    // rows past the last are clamped; their outputs are never written
    const int row = min(row0 + qt * 16 + ln, p.rows - 1);
    const int i = row / p.group, g = row % p.group;
    const T *qrow = static_cast<const T *>(p.q) +
                    ((static_cast<size_t>(b) * p.w + i) * p.hq + kvh * p.group + g) * DH;
#pragma unroll
    for (int ks = 0; ks < QK; ++ks)
      qf[qt][ks] = *reinterpret_cast<const u32x4 *>(qrow + (64 * ks + 16 * lg) / ES);
  }
  u32x4 kf[2 * KS], vf[DT];
  const bool has_block = g0 < nb;  // chunk 0 only
  if (has_block) {
    const size_t tok_bytes = static_cast<size_t>(p.hkv) * DH * ES;
    const size_t base = (static_cast<size_t>(b) * p.w * p.hkv + kvh) * DH * ES;
    const char *kblk = static_cast<const char *>(p.kb) + base;
    const char *vblk = static_cast<const char *>(p.vb) + base;
    uint8_t *raw = reinterpret_cast<uint8_t *>(part[wave]);
#pragma unroll
    for (int f = 0; f < DT; ++f) {
      const int o = f * kFragBytes + 16 * lane;  // byte in the [TT][DH] rows
      const int tok = min(TT * wave + o / (ES * DH), p.w - 1);
      dma16(vblk + tok * tok_bytes + o % (ES * DH), raw + f * kFragBytes);
    }
#pragma unroll
    for (int f = 0; f < 2 * KS; ++f) {
      const int tok = min(TT * wave + G::key_token(ln, f), p.w - 1);
      kf[f] = *reinterpret_cast<const u32x4 *>(kblk + tok * tok_bytes + G::key_col(f, lg));
    }
  }
  wait_vmcnt<0>();

  bool bad;
  const int S = clamp_prefix(s_raw, p.max_pages, &bad);
  if (bad && kvh == 0 && rt == 0 && chunk == 0 && threadIdx.x == 0)
    report_error(p.dev_error, DAS_DEVERR_PREFIX);
  const int ntile = nb + (S + TT - 1) / TT;
  const int nsb = (ntile + p.chunk_tiles - 1) / p.chunk_tiles;  // chunks of this unit
  if (chunk >= nsb) return;
  const int g_end = min(ntile, (chunk + 1) * p.chunk_tiles);
  const int n = g_end > g0 ? (g_end - g0 + NW - 1) / NW : 0;  // this wave's tiles
  // Out-of-range page ids are reported and read as page 0 (their tiles are
  // masked out).
  const bool page_ok = page_id >= 0 && page_id < p.num_pages;
  const uint64_t ok_mask = __builtin_amdgcn_ballot_w64(page_ok);
  if (!page_ok && lane < n) report_error(p.dev_error, DAS_DEVERR_PAGE);
  if (!page_ok) page_id = 0;

  const size_t head_off = static_cast<size_t>(kvh) * p.num_pages * kPage * DH * ES;
  const char *kl = static_cast<const char *>(p.k_layer) + head_off;
  const char *vl = static_cast<const char *>(p.v_layer) + head_off;
  const uint32_t lane_k = G::key_lane(ln, lg);
  const uint32_t lane_v = G::val_lane(ln, lg);
  // keys / values of this wave's i-th tile
  auto tile_off = [&](int i) {
    const int page = __builtin_amdgcn_readlane(page_id, i);
    const int u = (g0 + NW * i - nb) % TPP;
    return static_cast<size_t>(page) * kPage * DH * ES + 64 * DH * u;
  };
  auto load_keys = [&](int i) {
    const auto r = buffer_of(kl + tile_off(i), 64 * DH);
#pragma unroll
    for (int f = 0; f < 2 * KS; ++f) kf[f] = load_frag<kCached>(r, lane_k, G::key_frag(f));
  };
  auto load_values = [&](int i) {
    const auto r = buffer_of(vl + tile_off(i), 64 * DH);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vf[dt] = load_frag<kNonTemporal>(r, lane_v, G::val_frag(dt));
  };

  State<DH, NQ> st;
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    st.m[qt] = kNegInf;
    st.l[qt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) st.o[qt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  int cap[NQ];
  const int i0 = has_block ? 1 : 0;
  if (has_block) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) cap[qt] = (row0 + qt * 16 + ln) / p.group - TT * wave;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      vf[dt] = gather_block_values<T, DH>(reinterpret_cast<const uint8_t *>(part[wave]), dt, ln, lg);
    compute_tile<T, DH, NQ, true>(st, kf, vf, qf, cap, p.w - TT * wave, false, p.scale_log2, lg,
                                  [&](int stage) {
                                    if (stage == 1 && n > 1) load_keys(1);
                                  });
    if (n > 1) load_values(1);
  } else if (n > 0) {
    load_keys(0);
    load_values(0);
  }
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) cap[qt] = 0x7fffffff;
  for (int i = i0; i < n; ++i) {
    const bool more = i + 1 < n;
    const int limit = (ok_mask >> i) & 1 ? min(TT, S - TT * (g0 + NW * i - nb)) : 0;
    const bool full = limit >= TT;
    if (!full) {
      // invisible tokens enter P.V with probability 0; their values are
      // zeroed so that whatever the page holds there (NaN, Inf) adds nothing
      const u32x4 keep = value_mask<T>(limit, lg);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) vf[dt] &= keep;
    }
    compute_tile<T, DH, NQ, true>(st, kf, vf, qf, cap, limit, full, p.scale_log2, lg,
                                  [&](int stage) {
                                    if (stage == 1 && more) load_keys(i + 1);
                                  });
    if (more) load_values(i + 1);
  }

  // Merge of the waves' results: every row's maxima and sums first, then, one
  // 16-row tile at a time, the outputs scaled to the common maximum.
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    st.l[qt] = group_sum(st.l[qt]);
    float amax = 0.f;
    if (ES == 2 && nsb > 1) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 4; ++v) amax = fmaxf(amax, fabsf(st.o[qt][dt][v]));
      amax = group_max(amax);
    }
    if (lg == 0) {
      sm[wave][16 * qt + ln] = st.m[qt];
      sl[wave][16 * qt + ln] = st.l[qt];
      sa[wave][16 * qt + ln] = amax;
    }
  }
  uint8_t *rec = reinterpret_cast<uint8_t *>(p.ws_o) +
                 (static_cast<size_t>(unit) * p.nsplit + chunk) * p.piece_stride;
  __syncthreads();  // also: every block tile's raw values have been read
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    if (row0 + 16 * qt >= p.rows) break;  // uniform
    float mx = kNegInf;
#pragma unroll
    for (int k = 0; k < NW; ++k) mx = fmaxf(mx, sm[k][16 * qt + ln]);
    // no visible position in the whole chunk (an unreadable page): every
    // output is 0 already
    const float ref = mx == kNegInf ? 0.f : mx;
    const float sc = __builtin_amdgcn_exp2f(st.m[qt] - ref);
    if (qt > 0) __syncthreads();  // the previous row tile has been summed
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      *reinterpret_cast<f32x4 *>(&part[wave][ln * RS + 16 * dt + 4 * lg]) = st.o[qt][dt] * sc;
    __syncthreads();
    constexpr int CG = DH / 4;
    for (int item = threadIdx.x; item < 16 * CG; item += 64 * NW) {
      const int r = item / CG, c = 4 * (item % CG);
      const int row = row0 + 16 * qt + r;
      if (row >= p.rows) break;  // items are in row order
      float m2 = kNegInf;
#pragma unroll
      for (int k = 0; k < NW; ++k) m2 = fmaxf(m2, sm[k][16 * qt + r]);
      const float ref2 = m2 == kNegInf ? 0.f : m2;
      float den = 0.f, bound = 0.f;
      f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const float sck = __builtin_amdgcn_exp2f(sm[k][16 * qt + r] - ref2);
        den += sck * sl[k][16 * qt + r];
        bound += sck * sa[k][16 * qt + r];
        o += *reinterpret_cast<const f32x4 *>(&part[k][r * RS + c]);
      }
      if (nsb > 1) {
        write_piece_item<T, DH>(rec, p.rows, row, c, o, m2, den, bound);
        continue;
      }
      const int i = row / p.group, h = kvh * p.group + row % p.group;
      store_out4(static_cast<T *>(p.out) + ((static_cast<size_t>(b) * p.w + i) * p.hq + h) * DH + c,
                 o * (1.f / den));
      if (p.lse && c == 0)
        p.lse[(static_cast<size_t>(b) * p.hq + h) * p.w + i] =
            (m2 + log2f(den)) * 0.69314718055994530942f;
    }
  }
}

template <typename T, int DH>
hipError_t launch_dh(const AttnParams &p, hipStream_t s) {
  const int nq = p.rows <= 16 ? 1 : 2, n_rt = (p.rows + 16 * nq - 1) / (16 * nq);
  const dim3 grid(static_cast<unsigned>(p.batch) * p.hkv * p.nsplit * n_rt), block(64 * kChunkWaves);
  if (nq == 1) return launch_kernel(attn_chunk_kernel<T, DH, 1>, grid, block, s, p, n_rt);
  return launch_kernel(attn_chunk_kernel<T, DH, 2>, grid, block, s, p, n_rt);
}

template <typename T>
hipError_t launch_typed(const AttnParams &p, int dh, hipStream_t s) {
  if (dh == 64) return launch_dh<T, 64>(p, s);
  if (dh == 96) return launch_dh<T, 96>(p, s);
  return launch_dh<T, 128>(p, s);
}

}  // namespace

hipError_t launch_attn_chunk(const AttnParams &p, int dtype, int dh, hipStream_t s) {
  return dtype == DAS_F32 ? launch_typed<float>(p, dh, s) : launch_typed<bf16_t>(p, dh, s);
}

}  // namespace das
