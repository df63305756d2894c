// Shared device/host helpers for the gfx950 kernels (wave64, MFMA 16x16x32 bf16).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "specvlm.h"

namespace specvlm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;
constexpr int kNumXcd = 8;          // MI355X: 8 accelerator dies, each with its own L2
constexpr int kNumCu = 256;

// D = A(16x32 bf16) * B(32x16 bf16) + C.  Per lane (r = lane % 16, c = lane / 16):
//   A holds row r,    contraction indices 8c..8c+7
//   B holds column r, contraction indices 8c..8c+7
//   C/D hold column r, rows 4c..4c+3
__device__ __forceinline__ floatx4 mfma16(bf16x8 a, bf16x8 b, floatx4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Another lane's value by DPP, inside the lane's row of 16 (0xB1: lane ^ 1, 0x4E: lane ^ 2, 0x141: lane ^ 7, 0x124 and 0x128: 4 and 8
// lanes on, around the row; 0x00, 0x55, 0xAA, 0xFF: lane 0 to 3 of the four): a VALU move, where a shuffle goes through LDS.
template <int CTRL> __device__ __forceinline__ float row_move(float x)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, true));
}

// Workgroups are dealt to the XCDs round-robin by linear id.  Map the hardware
// id to a logical id so that consecutive logical ids share an XCD (and its L2).
// `padded` is the launch size, a multiple of kNumXcd; ids >= the real count exit.
__device__ __forceinline__ int xcd_logical_id(int hw_id, int padded)
{
    const int per_xcd = padded / kNumXcd;
    return (hw_id % kNumXcd) * per_xcd + hw_id / kNumXcd;
}

// Division by a launch's own divisor d, with inv = reciprocal(d) from the host: exact for every x >= 0.  (The compiler's
// sequence for a divisor that it does not know is a chain of about 25 instructions, and the kernels here that take a few
// microseconds had four to six of them in front of their first load.)
struct QuotRem { int q, r; };
__host__ __device__ __forceinline__ QuotRem divide(int x, int d, uint32_t inv)
{
    // inv <= 2^32 / d < inv + 1 (or inv = 2^32 - 1 for d = 1): the estimate is the quotient or one less
    const int q = (int)(((uint64_t)(uint32_t)x * inv) >> 32), r = x - q * d;
    return r >= d ? QuotRem{q + 1, r - d} : QuotRem{q, r};
}
// Share k of n_help equal ones of a request's rows, with inv = reciprocal(n_help).  Empty where the request has nothing to
// compute (no queries, or fewer keys than queries), whatever its offsets say: divide() is exact from 0 on only.
struct RowRange { int first, n; };
__host__ __device__ __forceinline__ RowRange helper_rows(int n_queries, int n_keys, int k, int n_help, uint32_t inv)
{
    if (n_queries <= 0 || n_keys < n_queries) return {0, 0};
    const int per = divide(n_keys + n_help - 1, n_help, inv).q, first = k * per;
    const int n = (n_keys < first + per ? n_keys : first + per) - first;
    return {first, n > 0 ? n : 0};
}
inline uint32_t reciprocal(int d) { return d > 1 ? (uint32_t)((1ull << 32) / (uint32_t)d) : 0xffffffffu; }

inline int round_up(int x, int m) { return (x + m - 1) / m * m; }
inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

inline int launch_status()
{
    return hipGetLastError() == hipSuccess ? SPECVLM_OK : SPECVLM_ELAUNCH;
}

constexpr int kMaxDevices = 64;         // per-device host state (kernel attributes, scratch addresses)

// Lets a kernel be launched with `bytes` of dynamic LDS, more than the 64 KB that need no leave.  The attribute belongs to
// the kernel as loaded on one device: it is raised once per device, before the call's first launch.
template <auto* KERNEL>
inline int allow_lds(int bytes)
{
    static std::atomic<bool> raised[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return SPECVLM_ELAUNCH;
    if (raised[dev].load(std::memory_order_acquire)) return SPECVLM_OK;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess)
        return SPECVLM_ELAUNCH;
    raised[dev].store(true, std::memory_order_release);
    return SPECVLM_OK;
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

}  // namespace specvlm
