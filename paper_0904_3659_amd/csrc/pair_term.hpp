// Device form of one term of Eq. (gravity) (Sec. I), shared by the
// row-gather kernels and the masked (diagonal) tiles of the pair-once kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace nbody {

// s[k] = s[k]^(-1/2) (v_rsq_f32) for K independent values, the wave's issue
// priority raised over them.  v_rsq_f32 takes the SIMD for 8 cycles, alone;
// other float32 operations of two waves issue together, 2.1 cycles each, as
// long as the two waves stay in step.  At equal priority a wave's rsq lets
// the others run on while it waits, the pair falls out of step and every
// operation takes 4 cycles: the 19-operation pair term of four rows measured
// 62 cycles per row without the priority (79 with the four rsq apart), 47
// with it.  One raise per group of rows costs least.  The closing s_setprio
// is also the wait state that the use of a transcendental's result needs.
template <int K>
__device__ __forceinline__ void rsq_group(float (&s)[K])
{
    static_assert(K >= 1 && K <= 8, "rows per lane");
    if constexpr (K > 4) {
        float lo[4], hi[K - 4];
#pragma unroll
        for (int k = 0; k < K; ++k) (k < 4 ? lo[k & 3] : hi[k & 3]) = s[k];
        rsq_group<4>(lo);
        rsq_group<K - 4>(hi);
#pragma unroll
        for (int k = 0; k < K; ++k) s[k] = k < 4 ? lo[k & 3] : hi[k & 3];
    } else if constexpr (K == 1) {
        __asm__ volatile("s_setprio 1\n\tv_rsq_f32 %0, %0\n\ts_setprio 0" : "+v"(s[0]));
    } else if constexpr (K == 2) {
        __asm__ volatile("s_setprio 1\n\tv_rsq_f32 %0, %0\n\tv_rsq_f32 %1, %1\n\ts_setprio 0"
                         : "+v"(s[0]), "+v"(s[1]));
    } else if constexpr (K == 3) {
        __asm__ volatile("s_setprio 1\n\tv_rsq_f32 %0, %0\n\tv_rsq_f32 %1, %1\n\t"
                         "v_rsq_f32 %2, %2\n\ts_setprio 0"
                         : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]));
    } else {
        __asm__ volatile("s_setprio 1\n\tv_rsq_f32 %0, %0\n\tv_rsq_f32 %1, %1\n\t"
                         "v_rsq_f32 %2, %2\n\tv_rsq_f32 %3, %3\n\ts_setprio 0"
                         : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]), "+v"(s[3]));
    }
}

// Holds a value that is the same in every lane in a vector register: an
// operation with a scalar-register operand does not issue beside another
// wave's (4.4 cycles instead of 2.2).
__device__ __forceinline__ void in_vgpr(float &v) { __asm__("" : "+v"(v)); }

// A raw buffer of `bytes` bytes at p (word 3: 32-bit data format), for loads
// that give zero past its end.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_buffer(const float *p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, (int)bytes, 0x00027000);
}

// (x_j, y_j, z_j, m_j), or zeros where j is past the end of the buffers.
__device__ __forceinline__ float4 buffer_xm(__amdgpu_buffer_rsrc_t bx, __amdgpu_buffer_rsrc_t bm,
                                            unsigned j)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b96(bx, (int)(12u * j), 0, 0);
    const auto w = __builtin_amdgcn_raw_buffer_load_b32(bm, (int)(4u * j), 0, 0);
    return make_float4(__builtin_bit_cast(float, (unsigned)v[0]),
                       __builtin_bit_cast(float, (unsigned)v[1]),
                       __builtin_bit_cast(float, (unsigned)v[2]),
                       __builtin_bit_cast(float, (unsigned)w));
}

// One term of Eq. (gravity): particle i at (xi, yi, zi) against
// q = (x_j, y_j, z_j, m_j); adds m_j d r^3 to (ax, ay, az) and m_j r to pp,
// with d = x_i - x_j and r = (|d|^2 + eps2)^(-1/2).  13 VALU operations plus
// one hardware reciprocal square root (v_rsq_f32).
__device__ __forceinline__ void pair_term(float xi, float yi, float zi, float4 q, float eps2,
                                          float &ax, float &ay, float &az, float &pp)
{
    const float dx = xi - q.x;
    const float dy = yi - q.y;
    const float dz = zi - q.z;
    float s = __builtin_fmaf(dx, dx, eps2);
    s = __builtin_fmaf(dy, dy, s);
    s = __builtin_fmaf(dz, dz, s);
    const float r = __builtin_amdgcn_rsqf(s);
    const float mr = q.w * r;
    const float r2 = r * r;
    const float mr3 = mr * r2;
    pp += mr;
    ax = __builtin_fmaf(mr3, dx, ax);
    ay = __builtin_fmaf(mr3, dy, ay);
    az = __builtin_fmaf(mr3, dz, az);
}

// The same term with the pair removed when `skip` holds (j == i, or a
// padded slot): r is forced to 0 so every product vanishes exactly, also
// for eps2 == 0 where the self distance would give an infinite r.
__device__ __forceinline__ void pair_term_masked(float xi, float yi, float zi, float4 q,
                                                 float eps2, bool skip, float &ax, float &ay,
                                                 float &az, float &pp)
{
    const float dx = xi - q.x;
    const float dy = yi - q.y;
    const float dz = zi - q.z;
    float s = __builtin_fmaf(dx, dx, eps2);
    s = __builtin_fmaf(dy, dy, s);
    s = __builtin_fmaf(dz, dz, s);
    const float r = skip ? 0.0f : __builtin_amdgcn_rsqf(s);
    const float mr = q.w * r;
    const float r2 = r * r;
    const float mr3 = mr * r2;
    pp += mr;
    ax = __builtin_fmaf(mr3, dx, ax);
    ay = __builtin_fmaf(mr3, dy, ay);
    az = __builtin_fmaf(mr3, dz, az);
}

}  // namespace nbody
