// mfma_util.h -- element-type traits of the 16 x 16 x 4 MFMA instructions
// used by the small-block and dense kernels (FP64 and FP32 block data).
#pragma once

#include <hip/hip_runtime.h>

namespace bsmm {

typedef double v4d_t __attribute__((ext_vector_type(4)));
typedef double v2d_t __attribute__((ext_vector_type(2)));
typedef float v2f_t __attribute__((ext_vector_type(2)));
typedef float v4f_t __attribute__((ext_vector_type(4)));

// Buffer of `bytes` bytes at p (both the same on every lane).
typedef __amdgpu_buffer_rsrc_t BufferRsrc;
__device__ __forceinline__ BufferRsrc buffer_at(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);  // raw, 32-bit data
}
// An offset past the end of any buffer of less than 2 GB, all 16 bytes from it too
// (an offset near 2^32 would wrap to the buffer's first bytes).
constexpr uint32_t kPastBuffer = 1u << 31;

// Both instructions take lane l's operands at row (or column) l % 16 and
// k = l / 16 of the step and return four results per lane.
template <class T> struct Mfma;
template <> struct Mfma<double> {
    typedef v4d_t acc_t;
    static __device__ __forceinline__ acc_t zero() { return (v4d_t){0.0, 0.0, 0.0, 0.0}; }
    static __device__ __forceinline__ acc_t step(double a, double b, acc_t c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // Result element e of lane l: row 4 e + l / 16, column l % 16.
    static __device__ __forceinline__ int row(int e, int lk) { return 4 * e + lk; }
    // One value, and two consecutive ones (16 bytes at 8-byte alignment:
    // dword alignment is all the vector loads need), at a byte offset of a
    // buffer; dwords past the buffer's end read as zero (and are not stored).
    static __device__ __forceinline__ double load(BufferRsrc r, uint32_t off) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        double x;
        __builtin_memcpy(&x, &v, sizeof x);
        return x;
    }
    static __device__ __forceinline__ void load2(BufferRsrc r, uint32_t off, double &x, double &y) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
        v2d_t d;
        __builtin_memcpy(&d, &v, sizeof d);
        x = d[0];
        y = d[1];
    }
    static __device__ __forceinline__ void store(BufferRsrc r, uint32_t off, double x) {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        u32x2 v;
        __builtin_memcpy(&v, &x, sizeof v);
        __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, 0);
    }
};
template <> struct Mfma<float> {
    typedef v4f_t acc_t;
    static __device__ __forceinline__ acc_t zero() { return (v4f_t){0.0f, 0.0f, 0.0f, 0.0f}; }
    static __device__ __forceinline__ acc_t step(float a, float b, acc_t c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    // Result element e of lane l: row 4 (l / 16) + e, column l % 16.
    static __device__ __forceinline__ int row(int e, int lk) { return 4 * lk + e; }
    static __device__ __forceinline__ float load(BufferRsrc r, uint32_t off) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
        float x;
        __builtin_memcpy(&x, &v, sizeof x);
        return x;
    }
    static __device__ __forceinline__ void load2(BufferRsrc r, uint32_t off, float &x, float &y) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
        v2f_t d;
        __builtin_memcpy(&d, &v, sizeof d);
        x = d[0];
        y = d[1];
    }
    static __device__ __forceinline__ void store(BufferRsrc r, uint32_t off, float x) {
        unsigned int v;
        __builtin_memcpy(&v, &x, sizeof v);
        __builtin_amdgcn_raw_buffer_store_b32(v, r, off, 0, 0);
    }
};

}  // namespace bsmm
