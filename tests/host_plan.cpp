// The library's host dispatcher as a CPU library: das_api.hip compiled by the
// host compiler, with the kernel launchers replaced by functions that note
// which kernel a call would run and how it cuts the work. A call through the C
// ABI with any non-null pointers then leaves its plan in last_plan().
#include <hip/hip_runtime.h>
#include <string.h>

// the device helpers of das_internal.h name these; nothing here calls them
inline unsigned __float_as_uint(float f) { unsigned u; memcpy(&u, &f, 4); return u; }
inline float __uint_as_float(unsigned u) { float f; memcpy(&f, &u, 4); return f; }
inline unsigned atomicOr(unsigned *p, unsigned v) { const unsigned o = *p; *p |= v; return o; }

#define HIP_SYMBOL(x) static_cast<const void *>(x)
#include "das_api.hip"

namespace {
enum { kNone, kValu, kSplit, kBalanced, kChunk };
struct LastPlan {
  int32_t kernel, merge, pages_per_split, nsplit, chunk_tiles, n_workers;
} last;

hipError_t note(int kernel, const das::AttnParams &p) {
  last = {kernel, 0, p.pages_per_split, p.nsplit, p.chunk_tiles, p.n_workers};
  return hipSuccess;
}
hipError_t note_merge() {
  last.merge = 1;
  return hipSuccess;
}
}  // namespace

namespace das {
hipError_t launch_attn_valu(const AttnParams &p, int, int, hipStream_t) { return note(kValu, p); }
hipError_t launch_attn_mfma(const AttnParams &p, int, int, hipStream_t) { return note(kSplit, p); }
hipError_t launch_attn_balanced(const AttnParams &p, int, int, hipStream_t) { return note(kBalanced, p); }
hipError_t launch_attn_chunk(const AttnParams &p, int, int, hipStream_t) { return note(kChunk, p); }
hipError_t launch_attn_combine(const AttnParams &, int, int, int, hipStream_t) { return note_merge(); }
hipError_t launch_attn_combine_records(const AttnParams &, int, int, hipStream_t) { return note_merge(); }
hipError_t launch_kv_append(const AppendParams &, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_greedy_accept(const AcceptParams &, hipStream_t) { return hipSuccess; }
}  // namespace das

extern "C" {
void last_plan(LastPlan *out) {
  *out = last;
  last = {};
}
hipError_t hipGetDevice(int *dev) { *dev = 0; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *dev) { *dev = 0; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **ptr, const void *) {
  static char there[256];
  *ptr = there;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipErrorUnknown; }
}
