// Device building blocks shared by the matrix-core attention kernels:
// direct-to-LDS fragment loads, memory-counter waits, the bf16 MFMA, the
// 4-lane row reductions, and one 32-token tile through both products and
// the online softmax (Eq. (2)-(3)).
//
// MFMA 16x16x32 bf16 lane layout (lane l, n = l % 16, g = l / 16):
//   A[m][k]: lane holds m = n, k = 8g..8g+7   B[k][n]: k = 8g..8g+7, n
//   C[m][n]: lane holds m = 4g..4g+3, n
// Both products take the key / value tile as the A operand:
//   S^T (tokens x rows) = K_tile (tokens x dh) . Q^T (dh x rows)
//   O^T (dh x rows)    += V^T_tile (dh x tokens) . P^T (tokens x rows)
// so a lane's 8 probabilities of one query row (after exp2 and bf16
// rounding) are directly the B operand of the P.V product.
//
// fp32 caches run the same schedules on v_mfma_f32_16x16x4_f32 (full fp32
// products and sums) over 16-token tiles, which have the bytes and the
// fragment count of a 32-token bf16 tile. Lane layout: A[m][k]: m = n, k = g;
// B[k][n]: k = g, n; C as above. Reduction slots may be numbered freely as
// long as both operands agree, so each 16-byte load serves four steps: step
// 4 j + i of S^T reduces over dims 16 j + 4 g + i, step i of O^T over tokens
// 4 g + i, which are a lane's own four logits, so the probabilities are the B
// operand as they stand. Bound by memory up to 32 rows (dh / 2 MFMAs of 32
// cycles per 16 rows and tile), by the matrix cores above. Against the
// vector-ALU kernel: 16 sequences x 55 heads x 512-4096 tokens, dh 96, 16 rows
// 554 -> 265 us (2.9 -> 5.9 TB/s); 4 x 8 heads x 4096, dh 128, 128 rows 788 ->
// 97 us; error against 64 bits 7.8e-7 -> 7.2e-7.
#pragma once

#include "das_internal.h"

namespace das {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

constexpr float kNegInf = -__builtin_huge_valf();
constexpr int kFragBytes = 64 * 16;  // one 16-byte fragment per lane

// 16 bytes per lane, global -> LDS at lds + 16 * lane (lds wave-uniform).
__device__ __forceinline__ void dma16(const void *src, uint8_t *lds) {
  __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void *)(src),
                                   (__attribute__((address_space(3))) void *)(lds), 16, 0, 0);
}

// Raw buffer resource over `bytes` bytes at `base` (stride 0; word 3 = the
// gfx9 raw-buffer format). Out-of-range lanes read zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void *base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00020000);
}

// Cache policy of the prefix loads (aux operand of the buffer loads). Values
// are non-temporal everywhere: prefix K/V are streamed once per call, and
// letting them displace the L2 like reused data cost 5-10 % of the rate on
// batched calls. A value fragment covers whole 128-byte lines; a key fragment
// covers half of each line it touches, and a non-temporal line is gone from the
// L1 when the fragment with its other half asks for it. Kernels that load key
// fragments straight into registers therefore use the default policy for them
// (a bare stream of this pattern: 51 against 38 GB/s per CU on 55 CUs, 42
// against 34 on 128, the same 27 on all 256); those that stage tiles in LDS
// load whole lines, non-temporally (default policy: 16 sequences x 55 heads
// 136 against 131 us).
constexpr int kCached = 0, kNonTemporal = 2;

// 16 bytes per lane from resource r at byte voff (per lane) + soff (uniform)
// -> LDS at lds + 16 * lane. The uniform part travels in an SGPR, so a
// fragment costs no vector address arithmetic.
template <int POLICY>
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, uint32_t voff, int soff,
                                      uint8_t *lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(lds),
                                           16, voff, soff, 0, POLICY);
}

// s_waitcnt vmcnt(n), other counters untouched (gfx9 encoding).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// Wait until at most `tiles` tiles of NF loads each are outstanding. Other
// loads or stores issued later only make the wait stricter.
template <int NF>
__device__ __forceinline__ void wait_tiles(int tiles) {
  if (tiles <= 0) wait_vmcnt<0>();
  else if (tiles == 1) wait_vmcnt<NF>();
  else if (tiles == 2) wait_vmcnt<(2 * NF < 64 ? 2 * NF : 0)>();
  else wait_vmcnt<(3 * NF < 64 ? 3 * NF : 0)>();
}

__device__ __forceinline__ f32x4 mfma16x16x4(uint32_t a, uint32_t b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a), __uint_as_float(b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma16x16x32(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Reductions over the 4 lanes n, n + 16, n + 32, n + 48 (the rows of the C
// fragment that hold one query row): gfx950's permlane swaps exchange 16-lane
// rows (xor 16) and 32-lane halves (xor 32) between two registers in one
// VALU op, so with both operands = x the pair {x[l], x[l ^ 16]} (or
// {x[l], x[l ^ 32]}) lands in every lane; max and + are commutative, so the
// lanes of a group agree bit for bit.
__device__ __forceinline__ float group_max(float x) {
  const unsigned u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const unsigned v = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float group_sum(float x) {
  const unsigned u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const unsigned v = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

typedef _Float16 h16x4 __attribute__((ext_vector_type(4)));

// Four outputs of a piece record as stored.
template <typename T> struct RecVec;
template <> struct RecVec<bf16_t> { typedef h16x4 type; };
template <> struct RecVec<float> { typedef f32x4 type; };

// One query row of a piece record (piece_record_bytes); the merge takes the
// row's unnormalised output as the stored values times q.
// bf16 caches: the row's normalised output O / l in fp16, scaled by 2^-e so
// that its largest magnitude lies in [2^14, 2^15) (full fp16 precision for the
// row whatever the value scale, half the bytes of fp32 partials), and
// {m, l, q = l 2^e, 0}. fp32 caches: the unnormalised output in fp32 and
// {m, l, q = 1, 0}. m = -inf and l = 0 when no position was visible (weight 0
// in the merge). Lane (n, g) holds head dims 16 dt + 4 g .. + 3 of the row;
// the 4 lanes of a row call this together (the row maximum is a 4-lane
// reduction).
template <typename T, int DH>
__device__ __forceinline__ void write_piece_row(uint8_t *rec, int rows, int row, int lg,
                                                const f32x4 (&o)[DH / 16], float m, float l) {
  float q = 1.f;
  if constexpr (sizeof(T) == 4) {
    float *orow = reinterpret_cast<float *>(rec) + row * DH;
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) *reinterpret_cast<f32x4 *>(orow + 16 * dt + 4 * lg) = o[dt];
  } else {
    const float inv = l > 0.f ? 1.f / l : 0.f;
    float amax = 0.f;
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt)
#pragma unroll
      for (int v = 0; v < 4; ++v) amax = fmaxf(amax, fabsf(o[dt][v]));
    amax = group_max(amax) * inv;
    const int e = (amax > 0.f && amax < __builtin_huge_valf()) ? __builtin_amdgcn_frexp_expf(amax) - 15 : 0;
    const float sc = __builtin_amdgcn_ldexpf(inv, -e);
    _Float16 *orow = reinterpret_cast<_Float16 *>(rec) + row * DH;
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) {
      const h16x4 hv = {static_cast<_Float16>(o[dt][0] * sc), static_cast<_Float16>(o[dt][1] * sc),
                        static_cast<_Float16>(o[dt][2] * sc), static_cast<_Float16>(o[dt][3] * sc)};
      *reinterpret_cast<h16x4 *>(orow + 16 * dt + 4 * lg) = hv;
    }
    q = __builtin_amdgcn_ldexpf(l, e);
  }
  if (lg == 0) {
    const f32x4 meta = {m, l, q, 0.f};
    *reinterpret_cast<f32x4 *>(rec + static_cast<size_t>(rows) * DH * rec_elem_bytes(sizeof(T)) +
                               row * 16) = meta;
  }
}

// Four outputs (columns c .. c + 3) of a row of a piece record, from a thread
// that holds only these: `bound` is a bound of the row's |O|, the same in
// every thread of the row, in place of its maximum (a few powers of two too
// large at most, and fp16 keeps full precision for 2^29 below).
template <typename T, int DH>
__device__ __forceinline__ void write_piece_item(uint8_t *rec, int rows, int row, int c,
                                                 const f32x4 &o, float m, float l, float bound) {
  float q = 1.f;
  const size_t at = static_cast<size_t>(row) * DH + c;
  if constexpr (sizeof(T) == 4) {
    *reinterpret_cast<f32x4 *>(rec + at * 4) = o;
  } else {
    const float inv = l > 0.f ? 1.f / l : 0.f;
    bound *= inv;
    const int e = (bound > 0.f && bound < __builtin_huge_valf()) ? __builtin_amdgcn_frexp_expf(bound) - 15 : 0;
    const float sc = __builtin_amdgcn_ldexpf(inv, -e);
    *reinterpret_cast<h16x4 *>(rec + at * 2) =
        h16x4{static_cast<_Float16>(o[0] * sc), static_cast<_Float16>(o[1] * sc),
              static_cast<_Float16>(o[2] * sc), static_cast<_Float16>(o[3] * sc)};
    q = __builtin_amdgcn_ldexpf(l, e);
  }
  if (c == 0)
    *reinterpret_cast<f32x4 *>(rec + static_cast<size_t>(rows) * DH * rec_elem_bytes(sizeof(T)) +
                               row * 16) = f32x4{m, l, q, 0.f};
}

// Four consecutive outputs of a row in the cache's type.
__device__ __forceinline__ void store_out4(bf16_t *dst, const f32x4 &o) {
  u32x2 packed;
  packed[0] = static_cast<uint32_t>(f32_to_bf16(o[0])) |
              (static_cast<uint32_t>(f32_to_bf16(o[1])) << 16);
  packed[1] = static_cast<uint32_t>(f32_to_bf16(o[2])) |
              (static_cast<uint32_t>(f32_to_bf16(o[3])) << 16);
  *reinterpret_cast<u32x2 *>(dst) = packed;
}
__device__ __forceinline__ void store_out4(float *dst, const f32x4 &o) {
  *reinterpret_cast<f32x4 *>(dst) = o;
}

// Geometry of a tile of T elements: TT tokens, so that its keys and its
// values are 64 * DH bytes each whatever the type. LINES: how a kernel that
// stages tiles in LDS holds the keys there (see key_swizzle).
template <typename T, int DH, int NQ, int NB_, bool LINES = true>
struct Geo {
  static constexpr int ES = sizeof(T);
  static constexpr int E = 4 / ES;         // 16-token S^T tiles per tile
  static constexpr int TT = 16 * E;        // tokens per tile
  static constexpr int TPP = kPage / TT;   // tiles per page
  static constexpr int KS = DH / 32;       // key fragments per issue part
  static constexpr int QK = DH * ES / 64;  // Q fragments of a 16-row tile
  static constexpr int DT = DH / 16;       // head-dim tiles of P V (value fragments)
  static constexpr int NF = 2 * KS + DT;   // fragments (loads) per tile
  static constexpr int SLOT = NF * kFragBytes;
  static constexpr int NB = NB_;           // ring depth
  static constexpr int LDS = NB * SLOT;

  // Per-lane byte offset of a key fragment's lane inside a tile's key rows
  // ([TT][DH]), and the uniform part of fragment f. bf16: token slot
  // 8(n/4) + n%4 (+ 4 for the second S^T tile), dims 32 ks + 8 g .. + 7;
  // fp32: token n, dims 16 f + 4 g .. + 3.
  static __device__ __forceinline__ int key_token(int ln, int f) {
    return ES == 2 ? 8 * (ln >> 2) + (ln & 3) + 4 * (f / KS) : ln;
  }
  static __device__ __forceinline__ uint32_t key_lane(int ln, int lg) {
    return (ES == 2 ? 8 * (ln >> 2) + (ln & 3) : ln) * DH * ES + 16 * lg;
  }
  static __device__ __forceinline__ constexpr int key_frag(int f) {
    return ES == 2 ? (4 * (f / KS) * DH + 32 * (f % KS)) * 2 : 64 * f;
  }
  // byte in its token's row at which a lane's piece of key fragment f starts
  static __device__ __forceinline__ int key_col(int f, int lg) {
    return (ES == 2 ? 64 * (f % KS) : 64 * f) + 16 * lg;
  }
  // Keys in LDS, LINES: the direct-to-LDS loads of a tile's keys read its rows
  // as they lie in memory, whole lines per instruction, so the slot holds the
  // rows in order; to spread the lanes that read a fragment (16 rows, 4
  // neighbouring 16-byte pieces) over the banks, the pieces of a row change
  // places inside its 64, 128 or 256 bytes by an exclusive or with
  // key_swizzle(row). Otherwise a load fetches a fragment, which the slot holds
  // lane by lane; it asks for half of each line at a time, 38 against 54 GB/s
  // per CU on 55 CUs, 24.8 against 26.0 on 256 with four waves each.
  static constexpr int CPR = DH * ES / 16;  // 16-byte pieces of a row
  static __device__ __forceinline__ int key_swizzle(int row) {
    if (ES == 2) {
      if (DH == 96) return (row >> 3) & 3;
      return (DH == 64 ? (row >> 1) & 1 : row & 3) * 4 + ((row >> 3) & 3);
    }
    return (DH == 96 ? (row >> 1) & 1 : row & 3) * 4 + ((row >> 2) & 3);
  }
  // row of the tile and byte in that row that lane `lane` of key load f fetches
  static __device__ __forceinline__ int key_load_row(int lane, int f) {
    return LINES ? (64 * f + lane) / CPR : key_token(lane & 15, f);
  }
  static __device__ __forceinline__ int key_load_col(int lane, int f) {
    return LINES ? (((64 * f + lane) % CPR) ^ key_swizzle(key_load_row(lane, f))) * 16
                 : key_col(f, lane >> 4);
  }
  // byte in the tile's keys: key_load(lane, f % LP) of the first LP loads
  // carries every lane-dependent part, (.. ^ key_load_xor(f)) + key_load_off(f)
  // is load f's
  static constexpr int LP = LINES && DH == 96 ? 3 : 1;
  static __device__ __forceinline__ uint32_t key_load(int lane, int f) {
    return key_load_row(lane, f) * (DH * ES) + key_load_col(lane, f);
  }
  static __device__ __forceinline__ constexpr int key_load_xor(int f) {
    if (!LINES) return 0;
    if (DH == 96) return 16 * 2 * (f / 3);
    if (DH == 64) return 16 * f;
    return 16 * (ES == 4 ? 8 * (f & 1) + (f >> 1) : f >> 1);
  }
  static __device__ __forceinline__ constexpr int key_load_off(int f) {
    return LINES ? (f - f % LP) * 1024 : key_frag(f);
  }
  // byte of the slot at which a lane reads its piece of fragment f:
  // key_read(lane, key_read_set(f)) + key_read_off(f)
  static constexpr int KJ = !LINES ? 1 : DH == 96 ? (ES == 2 ? 1 : 2) : (ES == 2 && DH == 64 ? 2 : 4);
  static __device__ __forceinline__ uint32_t key_read(int lane, int set) {
    if (!LINES) return 16 * lane;
    const int row = key_token(lane & 15, 0);
    return (row * CPR + ((4 * set + (lane >> 4)) ^ key_swizzle(row))) * 16;
  }
  static constexpr int key_read_set(int f) { return (ES == 2 ? f % KS : f) % KJ; }
  static constexpr int key_read_off(int f) {
    if (!LINES) return f * kFragBytes;
    return ES == 2 ? (f / KS) * 64 * CPR + (f % KS - f % KS % KJ) * 64 : (f - f % KJ) * 64;
  }

  // The same for the values of the tile in the token-grouped page: bf16:
  // token group g, head dim n; fp32: group g / 2, dim n, tokens 4 (g % 2) ..
  static __device__ __forceinline__ uint32_t val_lane(int ln, int lg) {
    return ES == 2 ? (lg * DH + ln) * 16 : ((lg >> 1) * DH + ln) * 32 + (lg & 1) * 16;
  }
  static __device__ __forceinline__ int val_frag(int dt) { return 128 * ES * dt; }
};

// V^T fragment dt of a draft-block tile, whose values are token-major
// [TT][DH] in LDS: the lane's consecutive tokens of head dim 16 dt + n.
template <typename T, int DH>
__device__ __forceinline__ u32x4 gather_block_values(const uint8_t *raw, int dt, int ln, int lg) {
  if constexpr (sizeof(T) == 2) {
    const uint16_t *r = reinterpret_cast<const uint16_t *>(raw);
    u16x8 v8;
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) v8[jj] = r[(8 * lg + jj) * DH + 16 * dt + ln];
    return __builtin_bit_cast(u32x4, v8);
  } else {
    const uint32_t *r = reinterpret_cast<const uint32_t *>(raw);
    u32x4 v4;
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) v4[jj] = r[(4 * lg + jj) * DH + 16 * dt + ln];
    return v4;
  }
}

// Mask of a lane's value fragment that keeps the tile's first `limit` tokens
// (bf16: the lane holds tokens 8 g .. + 7, two per word; fp32: 4 g .. + 3).
template <typename T>
__device__ __forceinline__ u32x4 value_mask(int limit, int lg) {
  u32x4 keep;
  if constexpr (sizeof(T) == 2) {
    const int nv = min(max(limit - 8 * lg, 0), 8);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      keep[k] = (2 * k < nv ? 0xffffu : 0u) | (2 * k + 1 < nv ? 0xffff0000u : 0u);
  } else {
#pragma unroll
    for (int k = 0; k < 4; ++k) keep[k] = 4 * lg + k < limit ? 0xffffffffu : 0u;
  }
  return keep;
}

template <int DH, int NQ>
struct State {
  float m[NQ], l[NQ];
  f32x4 o[NQ][DH / 16];
};

// One tile through both products and the online softmax. Token t of the tile
// is visible when t < limit and t <= cap[qt]; a full tile (every token
// visible) skips the mask.
// `hook(k)` runs between the stages (k = 0 before the logits, 1 before the
// softmax, 2 before P.V) so that the caller can spread work over the tile.
// LANE_SUM: st.l holds this lane's share of its row's sum (alpha is the same
// in a row's 4 lanes), which the caller reduces over the 4 lanes when it
// writes the row; otherwise st.l holds the row's sum after every tile.
// fp32 logits run in two accumulation chains, which halves a chain's roundings.
// Error against 64 bits of one chain / two: 2 x 8 heads x 350-700 tokens x 28
// rows, dh 96, 4.2e-7 / 2.7e-7; 8 heads x 4000 x 32 rows, dh 128, 6.0e-7 / 5.0e-7,
// with keys times 3 1.35e-6 / 7.9e-7 (the vector-ALU kernel: 6.3e-7, 1.21e-6).
template <typename T, int DH, int NQ, bool LANE_SUM = false, typename Hook>
__device__ __forceinline__ void compute_tile(State<DH, NQ> &st, const u32x4 (&kf)[DH / 16],
                                             const u32x4 (&vf)[DH / 16],
                                             const u32x4 (&qf)[NQ][Geo<T, DH, NQ, 1>::QK],
                                             const int (&cap)[NQ], int limit, bool full,
                                             float scale, int lg, Hook &&hook) {
  constexpr int E = Geo<T, DH, NQ, 1>::E;
  constexpr int QK = Geo<T, DH, NQ, 1>::QK;
  u16x8 pf[NQ];     // bf16: the probabilities as the B operand of P.V
  f32x4 pw[NQ];     // fp32
  float alpha[NQ];
  bool moved[NQ];
  f32x4 sacc[NQ][E];
  hook(0);
  // reduction step outermost: the accumulators are independent, so no MFMA
  // waits for the one before it. The two chains of fp32 keep that true with one
  // row tile at a time, which is what the registers take at head dim 128.
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int QG = F32 && DH == 128 ? 1 : NQ;  // row tiles side by side
  f32x4 odd[NQ];                                 // the second chains
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    odd[qt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int e = 0; e < E; ++e) sacc[qt][e] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int q0 = 0; q0 < NQ; q0 += QG) {
#pragma unroll
    for (int ks = 0; ks < QK; ++ks) {
      if constexpr (!F32) {
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
          for (int e = 0; e < E; ++e)
            sacc[qt][e] = mfma16x16x32(kf[e * QK + ks], qf[qt][ks], sacc[qt][e]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int qt = q0; qt < q0 + QG; ++qt) {
            f32x4 &acc = i & 1 ? odd[qt] : sacc[qt][0];
            acc = mfma16x16x4(kf[ks][i], qf[qt][ks][i], acc);
          }
      }
    }
    if constexpr (QG < NQ) sacc[q0][0] += odd[q0];
  }
  hook(1);
  if constexpr (F32 && QG == NQ) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) sacc[qt][0] += odd[qt];
  }
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    // raw logits; masked ones are -inf. scale > 0, so the maximum of the
    // scaled logits is the scaled maximum.
    float x[E][4];
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
      for (int v = 0; v < 4; ++v) x[e][v] = sacc[qt][e][v];
    if (!full) {  // uniform: a full tile skips the mask
#pragma unroll
      for (int e = 0; e < E; ++e) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int t = 4 * E * lg + 4 * e + v;
          x[e][v] = ((t < limit) & (t <= cap[qt])) ? x[e][v] : kNegInf;
        }
      }
    }
    float mx = kNegInf;
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
      for (int v = 0; v < 4; ++v) mx = fmaxf(mx, x[e][v]);
    // Running maximum (base-2 units): the row's largest probability is
    // exactly 1 and those near it fall just below, where bf16 rounds finest.
    mx = group_max(mx) * scale;
    const float mnew = fmaxf(st.m[qt], mx);
    const float neg = mnew == kNegInf ? 0.f : -mnew;  // nothing visible yet: every p is 0
    alpha[qt] = __builtin_amdgcn_exp2f(st.m[qt] + neg);
    moved[qt] = alpha[qt] != 1.f;
    float psum = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(x[e][v], scale, neg));
        psum += pv;
        if constexpr (sizeof(T) == 2)
          pf[qt][4 * e + v] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(pv));
        else
          pw[qt][v] = pv;
      }
    }
    if (!LANE_SUM) psum = group_sum(psum);
    st.l[qt] = st.l[qt] * alpha[qt] + psum;
    st.m[qt] = mnew;
  }
  hook(2);
  // rescale a row tile's accumulators only when the maximum of one of its
  // rows moved (a lane's accumulators of row tile qt all belong to one row)
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    if (__builtin_amdgcn_ballot_w64(moved[qt]) != 0) {
#pragma unroll
      for (int dt = 0; dt < DH / 16; ++dt) st.o[qt][dt] *= alpha[qt];
    }
  }
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int dt = 0; dt < DH / 16; ++dt) {
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt)
        st.o[qt][dt] = mfma16x16x32(vf[dt], __builtin_bit_cast(u32x4, pf[qt]), st.o[qt][dt]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int dt = 0; dt < DH / 16; ++dt)
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt)
          st.o[qt][dt] = mfma16x16x4(vf[dt][i], __float_as_uint(pw[qt][i]), st.o[qt][dt]);
  }
}

}  // namespace
}  // namespace das
