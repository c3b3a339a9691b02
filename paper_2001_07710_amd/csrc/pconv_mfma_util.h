// Device helpers shared by the matrix-core kernels of libpconv (pconv_mfma.hip, pconv_small.hip, pconv_backward.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

namespace pconv {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

constexpr uint32_t kInvalid = 0x80000000u;

// Division by a divisor fixed for the launch (Granlund and Montgomery's round-up method, exact for 32-bit dividends).
struct FastDiv {
    unsigned m, s1, s2;
};
inline FastDiv make_fastdiv(unsigned d) {
    unsigned l = 0;
    while ((1ull << l) < d) ++l;
    FastDiv f;
    f.m = (unsigned)((((1ull << l) - d) << 32) / d + 1);
    f.s1 = l < 1 ? l : 1;
    f.s2 = l > 0 ? l - 1 : 0;
    return f;
}
__device__ __forceinline__ unsigned fastdiv(unsigned x, const FastDiv& f) {
    const unsigned t = __umulhi(x, f.m);
    return (t + ((x - t) >> f.s1)) >> f.s2;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}

// More than 64 KiB of dynamic LDS has to be asked for once per kernel and device (one static object per kernel).
struct LdsAllowance {
    std::atomic<unsigned long long> devices{0};
    hipError_t ask(const void* kern) {
        int dev = 0;
        if (hipError_t e = hipGetDevice(&dev)) return e;
        const unsigned long long bit = 1ull << (dev & 63);
        if (dev < 64 && (devices.load(std::memory_order_relaxed) & bit)) return hipSuccess;
        const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e == hipSuccess && dev < 64) devices.fetch_or(bit, std::memory_order_relaxed);
        return e;
    }
};

template <int LW>
struct Piece;   // LW pixels of one channel, as loaded
template <>
struct Piece<8> {
    uint4v v;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
        v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0);
    }
    __device__ __forceinline__ unsigned dword(int i) const { return i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w; }
};
template <>
struct Piece<4> {
    uint2v v;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
        v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0);
    }
    __device__ __forceinline__ unsigned dword(int i) const { return i ? v.y : v.x; }
};
template <>
struct Piece<2> {
    unsigned v;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
        v = __builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0);
    }
    __device__ __forceinline__ unsigned dword(int) const { return v; }
};
template <>
struct Piece<1> {
    unsigned v;
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
        v = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, (int)voff, (int)soff, 0);
    }
    __device__ __forceinline__ unsigned dword(int) const { return v; }
};

// pixel `px` (0: low halves, 1: high halves) of two channels' dwords -> one dword {channel a, channel b}
__device__ __forceinline__ unsigned interleave(unsigned a, unsigned b, int px) {
    return px ? __builtin_amdgcn_perm(b, a, 0x07060302u) : __builtin_amdgcn_perm(b, a, 0x05040100u);
}

}  // namespace
}  // namespace pconv
