// Internal helpers shared by the HIP sources of the C2R library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <initializer_list>

#include "../../include/c2r.h"

#define C2R_WAVE 64
#define C2R_MAX_E 64
#define C2R_CANON_CHUNK 256

namespace c2r {

// An error that the caller's own earlier HIP work left behind in this thread must not be blamed
// on this library's launches: every entry point reads (and thereby clears) it before it
// launches anything, and launch_status() then reports only what its own launches raised.
static inline void drop_stale_error() { (void)hipGetLastError(); }

static inline int launch_status() {
    return hipGetLastError() == hipSuccess ? C2R_OK : C2R_ERR_LAUNCH;
}

static inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

static inline size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Memory that a launch reads or writes (no bytes, or a null pointer: none).
struct MemRange {
    const void *p;
    size_t bytes;
};
static inline bool apart(const MemRange &a, const MemRange &b) {
    const uintptr_t pa = reinterpret_cast<uintptr_t>(a.p), pb = reinterpret_cast<uintptr_t>(b.p);
    return !pa || !pb || !a.bytes || !b.bytes || pa + a.bytes <= pb || pb + b.bytes <= pa;
}
// Whether nothing that is written meets anything else.  Stages that are enqueued one after the other may hand memory on (one scratch for
// all of them, a result in the place of an input that is done with); workgroups of ONE launch that does their work run in no order, so
// it is taken only where this holds.
static inline bool all_apart(std::initializer_list<MemRange> written, std::initializer_list<MemRange> read) {
    for (const MemRange *w = written.begin(); w != written.end(); ++w) {
        for (const MemRange *v = w + 1; v != written.end(); ++v)
            if (!apart(*w, *v)) return false;
        for (const MemRange &r : read)
            if (!apart(*w, r)) return false;
    }
    return true;
}

// bf16 <-> fp32 on raw bits. Storage is uint16_t; conversion to fp32 is exact.
__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// fp32 -> bf16, round to nearest even, NaN stays NaN: the hardware conversion
// (v_cvt_pk_bf16_f32), one instruction for two values and no branch on NaN.
typedef __bf16 c2r_bf16x2 __attribute__((ext_vector_type(2)));
typedef float c2r_f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const c2r_f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, c2r_bf16x2));
}

__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) { return pack_bf16x2(f, 0.0f) & 0xffffu; }

// permute.hip: the argument checks of c2r_permute, and its row scatter alone.
int permute_check(const void *x, c2r_dtype dt, const int32_t *topk_idx, int64_t T, int d, int E, int K,
                  const int32_t *local_slot, int E_local, int32_t *counts, int32_t *offsets, int32_t *perm,
                  int32_t *inv_perm, void *x_perm, void *ws, size_t ws_bytes);
int permute_rows(const void *x, c2r_dtype dt, int64_t T, int d, int K, const int32_t *inv_perm, void *x_perm,
                 hipStream_t st);
// route.hip.  later: not null only where route_may_finish_later; then the chunk results are all that is enqueued, and the next launch has
// to do the rest (route_few.h).
struct FewRoute;
constexpr int FEW_TOKENS = 16, FEW_ASSIGNMENTS = 32;
bool route_may_finish_later(int64_t T, int d, int E, int K);
int route_and_permute(const void *x, c2r_dtype dt, const float *Wg, const float *bias, int64_t T, int d, int E, int K,
                      const int32_t *collab_idx, int Tc, int32_t *topk_idx, float *gates, void *ws_route,
                      size_t ws_route_bytes, const int32_t *local_slot, int E_local, int32_t *counts, int32_t *offsets,
                      int32_t *perm, int32_t *inv_perm, void *x_perm, void *ws_permute, size_t ws_permute_bytes,
                      FewRoute *later, void *stream);

__device__ __forceinline__ int lane_id() { return threadIdx.x & (C2R_WAVE - 1); }

// Inclusive prefix sum over the 64 lanes of a wave with data-parallel-primitive moves (no
// LDS round trips): shifts by 1, 2, 4, 8 inside each row of 16 lanes, then the row totals
// are passed on with the two row broadcasts.  Every lane must be active.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
#endif
    return v;
}

// The largest of the 64 lanes' values, in every lane, without LDS round trips.  Every lane must be active.
__device__ __forceinline__ int wave_max(int v) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int LOWEST = (int)0x80000000;
    v = max(v, __builtin_amdgcn_update_dpp(LOWEST, v, 0x111, 0xf, 0xf, false));  // row_shr:1, 2, 4, 8
    v = max(v, __builtin_amdgcn_update_dpp(LOWEST, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(LOWEST, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(LOWEST, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(LOWEST, v, 0x142, 0xa, 0xf, false));  // row_bcast:15 into rows 1, 3
    v = max(v, __builtin_amdgcn_update_dpp(LOWEST, v, 0x143, 0xc, 0xf, false));  // row_bcast:31 into rows 2, 3
    v = __builtin_amdgcn_readlane(v, 63);
#endif
    return v;
}

}  // namespace c2r
