// Internal helpers shared by the HIP translation units of libeagletv.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "eagletv.h"

namespace etv {

extern thread_local int32_t g_last_hip_error;

inline int32_t check_launch() {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        g_last_hip_error = (int32_t)e;
        return ETV_ERR_HIP;
    }
    return ETV_OK;
}

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// fp32 -> bf16, round to nearest even (inputs are finite or inf; NaN is kept quiet)
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ int clampi(int x, int lo, int hi) { return x < lo ? lo : (x > hi ? hi : x); }

// x / d and x % d for any 32-bit x, with inv = floor(2^32 / d) or floor((2^32 - 1) / d), which differ where d is a power of two: the
// estimate is at most one too small.  (A smaller inv is not enough: d = 3, inv = 0x55555554, x = 0xffffffff is two too small.  The
// compiler's general division is some forty dependent instructions, each 3.5 ns of a lone wavefront's start-up.)
__device__ __forceinline__ uint32_t fast_div(uint32_t x, uint32_t d, uint32_t inv, uint32_t &rem) {
    uint32_t q = __umulhi(x, inv);
    rem = x - q * d;
    if (rem >= d) {
        q++;
        rem -= d;
    }
    return q;
}

static uint32_t fast_div_inv(int d) { return d == 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (uint32_t)d); }

// Inclusive sums / maxima (of values that are not negative) over the lanes before and with each, by lane moves of the vector unit:
// six dependent instructions, where a shuffle through LDS costs some 100 cycles a step.
template <int CTRL, int ROWS>
__device__ __forceinline__ int lane_move(int v) { return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false); }
template <class F>
__device__ __forceinline__ int wave_scan(int v, F f) {
    v = f(v, lane_move<0x111, 0xf>(v));  // the neighbours 1, 2, 4, 8 lanes down within the 16 of a row
    v = f(v, lane_move<0x112, 0xf>(v));
    v = f(v, lane_move<0x114, 0xf>(v));
    v = f(v, lane_move<0x118, 0xf>(v));
    v = f(v, lane_move<0x142, 0xa>(v));  // the last lane of row 0 / 2 to row 1 / 3
    return f(v, lane_move<0x143, 0xc>(v));  // lane 31 to rows 2 and 3
}
__device__ __forceinline__ int wave_scan_sum(int v) { return wave_scan(v, [](int a, int b) { return a + b; }); }
__device__ __forceinline__ int wave_scan_max(int v) { return wave_scan(v, [](int a, int b) { return max(a, b); }); }

// The best over the wavefront, f(x, x) being x (a maximum, a minimum): lanes whose neighbour is outside a row combine with themselves.
template <class T, class F>
__device__ __forceinline__ T wave_best(T v, F f) {
    static_assert(sizeof(T) == 4, "one register");
#define ETV_STEP(ctrl, rows) \
    v = f(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, v), __builtin_bit_cast(int, v), ctrl, rows, 0xf, false)))
    ETV_STEP(0x111, 0xf);
    ETV_STEP(0x112, 0xf);
    ETV_STEP(0x114, 0xf);
    ETV_STEP(0x118, 0xf);
    ETV_STEP(0x142, 0xa);
    ETV_STEP(0x143, 0xc);
#undef ETV_STEP
    return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

}  // namespace etv
