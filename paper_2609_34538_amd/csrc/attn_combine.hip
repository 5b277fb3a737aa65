// Merge of the per-split partial results into the attention output.
//
// Each split s of a (sequence, KV head) left, per query row, an unnormalised
// output O_s, its running maximum m_s (base-2 logit units) and its running
// sum l_s. With M = max_s m_s the joint softmax of Eq. (2) over all splits is
//   O = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s,
// and the natural-log normaliser is (M + log2 sum_s 2^(m_s - M) l_s) * ln 2.
// Split 0 always holds the block's diagonal, so M is finite.

#include "mfma_tile.h"

namespace das {
namespace {

constexpr int kRowsPerBlock = 8;
constexpr int kColsPerBlock = 32;
constexpr int kEager = 24;  // splits whose partials are loaded before the count is known

// One single-wave workgroup per (sequence, KV head, 8 rows, 32 columns); one
// thread per (row, 4 consecutive columns). A row's per-split maxima and sums
// are contiguous, so they arrive as 16-byte vectors; the partials of the first
// 24 splits the workspace holds are loaded together with the prefix length,
// so a merge of up to 24 splits costs one memory round trip. Values of splits
// past the sequence's count are discarded by selection, never used in
// arithmetic.
template <typename T, int DH>
__global__ __launch_bounds__(64) void attn_combine_kernel(AttnParams p, int skip_single) {
  const int unit = blockIdx.x;  // b * hkv + kvh
  const int b = unit / p.hkv;
  const int kvh = unit % p.hkv;
  const int row = blockIdx.y * kRowsPerBlock + threadIdx.x / 8;
  const int c = blockIdx.z * kColsPerBlock + 4 * (threadIdx.x % 8);
  const bool live = row < p.rows && c < DH;
  const int r0 = live ? row : 0, c0 = live ? c : 0;
  const size_t obase = (static_cast<size_t>(unit) * p.nsplit) * p.rows + r0;  // split 0's row
  const size_t mbase = (static_cast<size_t>(unit) * p.rows + r0) * p.nsplit_ml;

  const int s_raw = p.prefix_len[b];
  float mv[kEager], lv[kEager];
  float4 ov[kEager];
#pragma unroll
  for (int k4 = 0; k4 < kEager / 4; ++k4) {
    // the row's nsplit_ml (a multiple of 4) slots; split slots past the
    // plan's count are not loaded (a uniform branch), those past the
    // sequence's count are discarded below
    if (4 * k4 < p.nsplit_ml) {
      const float4 m4 = *reinterpret_cast<const float4 *>(p.ws_m + mbase + 4 * k4);
      const float4 l4 = *reinterpret_cast<const float4 *>(p.ws_l + mbase + 4 * k4);
      mv[4 * k4] = m4.x, mv[4 * k4 + 1] = m4.y, mv[4 * k4 + 2] = m4.z, mv[4 * k4 + 3] = m4.w;
      lv[4 * k4] = l4.x, lv[4 * k4 + 1] = l4.y, lv[4 * k4 + 2] = l4.z, lv[4 * k4 + 3] = l4.w;
    }
  }
#pragma unroll
  for (int k = 0; k < kEager; ++k) {
    if (k < p.nsplit)
      ov[k] = *reinterpret_cast<const float4 *>(p.ws_o + (obase + static_cast<size_t>(k) * p.rows) * DH + c0);
  }
  // keep every load above ahead of the first use of its result (one round trip)
  __builtin_amdgcn_sched_barrier(0);
  bool bad;
  const int S = clamp_prefix(s_raw, p.max_pages, &bad);
  const int npages = (S + kPage - 1) / kPage;
  const int ns = splits_of(npages, p.pages_per_split);
  // a single split was written by the attention kernel. The merge below runs
  // regardless and only the stores are skipped, so that the partials' loads
  // are not deferred behind the prefix length.
  const bool write = live && !(ns == 1 && skip_single);

  float mx = -__builtin_huge_valf();
#pragma unroll
  for (int k = 0; k < kEager; ++k) mx = k < ns ? fmaxf(mx, mv[k]) : mx;
  float den = 0.f, n0 = 0.f, n1 = 0.f, n2 = 0.f, n3 = 0.f;
#pragma unroll
  for (int k = 0; k < kEager; ++k) {
    if (k < ns) {
      const float sc = exp2f(mv[k] - mx);
      den += sc * lv[k];
      n0 += sc * ov[k].x;
      n1 += sc * ov[k].y;
      n2 += sc * ov[k].z;
      n3 += sc * ov[k].w;
    }
  }
  // splits beyond the first kEager, merged in the same online form
  for (int s0 = kEager; s0 < ns && live; ++s0) {
    const float m = p.ws_m[mbase + s0], l = p.ws_l[mbase + s0];
    const float4 o = *reinterpret_cast<const float4 *>(p.ws_o + (obase + static_cast<size_t>(s0) * p.rows) * DH + c);
    const float nm = fmaxf(mx, m);
    const float a = exp2f(mx - nm), sc = exp2f(m - nm);
    den = den * a + sc * l;
    n0 = n0 * a + sc * o.x;
    n1 = n1 * a + sc * o.y;
    n2 = n2 * a + sc * o.z;
    n3 = n3 * a + sc * o.w;
    mx = nm;
  }
  if (!write) return;
  const int i = row / p.group, g = row % p.group;
  const int h = kvh * p.group + g;
  T *out = static_cast<T *>(p.out) + ((static_cast<size_t>(b) * p.w + i) * p.hq + h) * DH + c;
  const float inv = 1.f / den;
  out[0] = from_f32<T>(n0 * inv);
  out[1] = from_f32<T>(n1 * inv);
  out[2] = from_f32<T>(n2 * inv);
  out[3] = from_f32<T>(n3 * inv);
  if (p.lse && c == 0)
    p.lse[(static_cast<size_t>(b) * p.hq + h) * p.w + i] = (mx + log2f(den)) * 0.69314718055994530942f;
}

// The same merge over the piece records of the matrix-core kernels (one per
// (sequence, KV head, split or chunk)): a row's {m, l, q} of a record arrive
// as one 16-byte vector and its outputs as four values (fp16 or fp32)
// scaled by q. The SG waves of a workgroup take every SG-th record, the first
// kEagerRec of each loaded together with the prefix length, so up to
// SG * kEagerRec records cost one memory round trip; further ones arrive in
// batches of as many. Four waves where a plan has more than kEagerRec records
// (measured with 34 records of 16 rows, dh 128, 8 units: 11.7 us with one wave
// and 24 records at once, the rest one by one).
constexpr int kEagerRec = 8;

template <typename T, int DH, int SG>
__global__ __launch_bounds__(64 * SG) void attn_combine_records_kernel(AttnParams p) {
  const int unit = blockIdx.x;  // b * hkv + kvh
  const int b = unit / p.hkv;
  const int kvh = unit % p.hkv;
  const int lane = threadIdx.x & 63;
  const int wave = SG == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = blockIdx.y * kRowsPerBlock + lane / 8;
  const int c = blockIdx.z * kColsPerBlock + 4 * (lane % 8);
  const bool live = row < p.rows && c < DH;
  const int r0 = live ? row : 0, c0 = live ? c : 0;
  const size_t stride = static_cast<size_t>(p.piece_stride);
  typedef typename RecVec<T>::type Ov;
  const uint8_t *rec0 = reinterpret_cast<const uint8_t *>(p.ws_o) +
                        static_cast<size_t>(unit) * p.nsplit * stride;
  const uint8_t *orow = rec0 + (r0 * DH + c0) * rec_elem_bytes(sizeof(T));
  const uint8_t *mrow = rec0 + static_cast<size_t>(p.rows) * DH * rec_elem_bytes(sizeof(T)) + r0 * 16;

  const int s_raw = p.prefix_len[b];
  f32x4 meta[kEagerRec];
  Ov ov[kEagerRec];
  auto load = [&](int first, int count) {
#pragma unroll
    for (int k = 0; k < kEagerRec; ++k) {
      const int rec = first + SG * k;
      if (rec < count) {  // uniform
        meta[k] = *reinterpret_cast<const f32x4 *>(mrow + rec * stride);
        ov[k] = *reinterpret_cast<const Ov *>(orow + rec * stride);
      }
    }
  };
  load(wave, p.nsplit);  // slots of the plan; past the sequence's count: unused
  // keep every load above ahead of the first use of its result (one round trip)
  __builtin_amdgcn_sched_barrier(0);
  bool bad;
  const int S = clamp_prefix(s_raw, p.max_pages, &bad);
  const int npages = (S + kPage - 1) / kPage;
  constexpr int TT = 64 / sizeof(T);  // tokens per tile
  const int ntile = (S + TT - 1) / TT + (p.w + TT - 1) / TT;
  const int ns = p.chunk_tiles ? (ntile + p.chunk_tiles - 1) / p.chunk_tiles
                               : splits_of(npages, p.pages_per_split);
  if (SG > 1 && ns == 1) return;  // written by the attention kernel; uniform

  // record k: maximum meta[0], sum meta[1], unnormalised output = stored * meta[2]
  float mx = -__builtin_huge_valf(), den = 0.f;
  f32x4 n = {0.f, 0.f, 0.f, 0.f};
  // one wave takes the records of a plan of at most kEagerRec in one pass
  for (int first = wave; SG == 1 ? first == 0 : first < ns; first += SG * kEagerRec) {
    if (SG > 1 && first != wave) load(first, ns);
    float nm = mx;
#pragma unroll
    for (int k = 0; k < kEagerRec; ++k) nm = first + SG * k < ns ? fmaxf(nm, meta[k][0]) : nm;
    // no visible position so far: every weight is 0
    const float ref = nm == -__builtin_huge_valf() ? 0.f : nm;
    const float a = __builtin_amdgcn_exp2f(mx - ref);
    den *= a;
    n *= a;
#pragma unroll
    for (int k = 0; k < kEagerRec; ++k) {
      if (first + SG * k < ns) {
        const float sc = __builtin_amdgcn_exp2f(meta[k][0] - ref);
        const float wgt = sc * meta[k][2];
        den += sc * meta[k][1];
#pragma unroll
        for (int v = 0; v < 4; ++v) n[v] += wgt * static_cast<float>(ov[k][v]);
      }
    }
    mx = nm;
  }
  if constexpr (SG > 1) {
    __shared__ __attribute__((aligned(16))) f32x4 sn[SG][64];
    __shared__ float smx[SG][64], sden[SG][64];
    sn[wave][lane] = n;
    smx[wave][lane] = mx;
    sden[wave][lane] = den;
    __syncthreads();
    if (wave > 0) return;
#pragma unroll
    for (int k = 1; k < SG; ++k) mx = fmaxf(mx, smx[k][lane]);
    den = 0.f;
    n = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < SG; ++k) {
      const float sc = __builtin_amdgcn_exp2f(smx[k][lane] - mx);
      den += sc * sden[k][lane];
      n += sn[k][lane] * sc;
    }
  }
  if (!live || ns == 1) return;
  const int i = row / p.group, g = row % p.group;
  const int h = kvh * p.group + g;
  store_out4(static_cast<T *>(p.out) + ((static_cast<size_t>(b) * p.w + i) * p.hq + h) * DH + c,
             n * (1.f / den));
  if (p.lse && c == 0)
    p.lse[(static_cast<size_t>(b) * p.hq + h) * p.w + i] = (mx + log2f(den)) * 0.69314718055994530942f;
}

template <typename T, int DH>
hipError_t launch_typed(const AttnParams &p, int skip_single, hipStream_t s) {
  dim3 grid(p.batch * p.hkv, (p.rows + kRowsPerBlock - 1) / kRowsPerBlock,
            (DH + kColsPerBlock - 1) / kColsPerBlock);
  return launch_kernel(attn_combine_kernel<T, DH>, grid, dim3(64), s, p, skip_single);
}

template <typename T, int DH>
hipError_t launch_records(const AttnParams &p, hipStream_t s) {
  dim3 grid(p.batch * p.hkv, (p.rows + kRowsPerBlock - 1) / kRowsPerBlock,
            (DH + kColsPerBlock - 1) / kColsPerBlock);
  if (p.nsplit <= kEagerRec)
    return launch_kernel(attn_combine_records_kernel<T, DH, 1>, grid, dim3(64), s, p);
  return launch_kernel(attn_combine_records_kernel<T, DH, 4>, grid, dim3(256), s, p);
}

template <typename T>
hipError_t launch_records_dh(const AttnParams &p, int dh, hipStream_t s) {
  if (dh == 64) return launch_records<T, 64>(p, s);
  if (dh == 96) return launch_records<T, 96>(p, s);
  return launch_records<T, 128>(p, s);
}

}  // namespace

hipError_t launch_attn_combine_records(const AttnParams &p, int dtype, int dh, hipStream_t s) {
  return dtype == DAS_F32 ? launch_records_dh<float>(p, dh, s)
                          : launch_records_dh<bf16_t>(p, dh, s);
}

hipError_t launch_attn_combine(const AttnParams &p, int dtype, int dh, int skip_single,
                               hipStream_t s) {
  if (dtype == DAS_F32) {
    if (dh == 64) return launch_typed<float, 64>(p, skip_single, s);
    if (dh == 96) return launch_typed<float, 96>(p, skip_single, s);
    return launch_typed<float, 128>(p, skip_single, s);
  }
  if (dh == 64) return launch_typed<bf16_t, 64>(p, skip_single, s);
  if (dh == 96) return launch_typed<bf16_t, 96>(p, skip_single, s);
  return launch_typed<bf16_t, 128>(p, skip_single, s);
}

}  // namespace das
