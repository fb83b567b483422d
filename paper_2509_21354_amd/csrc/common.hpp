// Shared device helpers of the kvev kernels (gfx950 only, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/kvev.h"

namespace kvev {

typedef uint16_t bf16_t;   // raw bfloat16 bits

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

constexpr int kWave = 64;

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float((uint32_t)v << 16); }

typedef __bf16 bf16x2_hw_t __attribute__((ext_vector_type(2)));
typedef float f32x2_hw_t __attribute__((ext_vector_type(2)));

// two fp32 -> packed bf16 bits (lo in bits 0..15), round to nearest even, in
// one v_cvt_pk_bf16_f32 (gfx950 converts in hardware; NaN stays NaN).
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    f32x2_hw_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_hw_t));
}

// fp32 -> bf16 bits, round to nearest even.
__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(pack_bf16x2(f, 0.f) & 0xFFFFu); }

template <typename T> struct Storage;
template <> struct Storage<float> {
    static __device__ __forceinline__ float load(const float *p) { return *p; }
    static __device__ __forceinline__ void store(float *p, float v) { *p = v; }
};
template <> struct Storage<bf16_t> {
    static __device__ __forceinline__ float load(const bf16_t *p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void store(bf16_t *p, float v) { *p = f32_to_bf16(v); }
};

// N consecutive elements of storage type T -> fp32 registers, with the widest
// loads the alignment allows (the caller guarantees N*sizeof(T)-byte alignment
// up to 16 bytes).
template <typename T, int N> struct VecLoad;
template <> struct VecLoad<float, 4> {
    static __device__ __forceinline__ void run(const float *p, float (&o)[4])
    {
        float4 v = *reinterpret_cast<const float4 *>(p);
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    }
};
template <> struct VecLoad<float, 8> {
    static __device__ __forceinline__ void run(const float *p, float (&o)[8])
    {
        float4 a = reinterpret_cast<const float4 *>(p)[0];
        float4 b = reinterpret_cast<const float4 *>(p)[1];
        o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w;
        o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
    }
};
template <> struct VecLoad<bf16_t, 4> {
    static __device__ __forceinline__ void run(const bf16_t *p, float (&o)[4])
    {
        uint2 v = *reinterpret_cast<const uint2 *>(p);
        o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xFFFF0000u);
        o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xFFFF0000u);
    }
};
template <> struct VecLoad<bf16_t, 8> {
    static __device__ __forceinline__ void run(const bf16_t *p, float (&o)[8])
    {
        uint4 v = *reinterpret_cast<const uint4 *>(p);
        o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xFFFF0000u);
        o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xFFFF0000u);
        o[4] = __uint_as_float(v.z << 16); o[5] = __uint_as_float(v.z & 0xFFFF0000u);
        o[6] = __uint_as_float(v.w << 16); o[7] = __uint_as_float(v.w & 0xFFFF0000u);
    }
};

// N consecutive elements kept in their raw register form (a 16-byte load is 4
// registers, not 8) until they are used.
// load_stream: the same load with the non-temporal hint, for cache rows that are read once per launch.  A plain
// streaming kernel reads 7.3 TB/s with the hint against 6.4 TB/s without on this chip.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
template <typename T, int N> struct Raw;
template <> struct Raw<bf16_t, 8> {
    uint4 v;
    __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const uint4 *>(p); }
    __device__ __forceinline__ void load_stream(const bf16_t *p)
    {
        const u32x4_t r = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
        v = make_uint4(r[0], r[1], r[2], r[3]);
    }
    __device__ __forceinline__ void get(float (&o)[8]) const
    {
        o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xFFFF0000u);
        o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xFFFF0000u);
        o[4] = __uint_as_float(v.z << 16); o[5] = __uint_as_float(v.z & 0xFFFF0000u);
        o[6] = __uint_as_float(v.w << 16); o[7] = __uint_as_float(v.w & 0xFFFF0000u);
    }
};
template <> struct Raw<bf16_t, 4> {
    uint2 v;
    __device__ __forceinline__ void load(const bf16_t *p) { v = *reinterpret_cast<const uint2 *>(p); }
    __device__ __forceinline__ void load_stream(const bf16_t *p)
    {
        const u32x2_t r = __builtin_nontemporal_load(reinterpret_cast<const u32x2_t *>(p));
        v = make_uint2(r[0], r[1]);
    }
    __device__ __forceinline__ void get(float (&o)[4]) const
    {
        o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xFFFF0000u);
        o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xFFFF0000u);
    }
};
template <> struct Raw<float, 4> {
    float4 v;
    __device__ __forceinline__ void load(const float *p) { v = *reinterpret_cast<const float4 *>(p); }
    __device__ __forceinline__ void load_stream(const float *p)
    {
        const u32x4_t r = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
        v = make_float4(__uint_as_float(r[0]), __uint_as_float(r[1]), __uint_as_float(r[2]), __uint_as_float(r[3]));
    }
    __device__ __forceinline__ void get(float (&o)[4]) const { o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w; }
};
template <> struct Raw<float, 8> {
    float4 a, b;
    __device__ __forceinline__ void load(const float *p)
    {
        a = reinterpret_cast<const float4 *>(p)[0];
        b = reinterpret_cast<const float4 *>(p)[1];
    }
    __device__ __forceinline__ void load_stream(const float *p)
    {
        const u32x4_t r0 = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p));
        const u32x4_t r1 = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p) + 1);
        a = make_float4(__uint_as_float(r0[0]), __uint_as_float(r0[1]), __uint_as_float(r0[2]), __uint_as_float(r0[3]));
        b = make_float4(__uint_as_float(r1[0]), __uint_as_float(r1[1]), __uint_as_float(r1[2]), __uint_as_float(r1[3]));
    }
    __device__ __forceinline__ void get(float (&o)[8]) const
    {
        o[0] = a.x; o[1] = a.y; o[2] = a.z; o[3] = a.w; o[4] = b.x; o[5] = b.y; o[6] = b.z; o[7] = b.w;
    }
};

// 16-byte load through a buffer descriptor: address = descriptor base (SGPRs) +
// voff (one VGPR, shared by every load of the lane) + soff (SGPR or constant),
// with the constant part of voff folded into the instruction's immediate.  Keeps
// per-load 64-bit addresses out of the vector registers; a load past the
// descriptor's size returns zeros instead of faulting.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x00027000);
}
template <typename V> __device__ __forceinline__ V buffer_load16(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, uint32_t soff)
{
    const u32x4_t raw = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)voff, (int)soff, 0);
    return __builtin_bit_cast(V, raw);
}
// The same with the non-temporal hint: for data read once, so that it does not push re-used lines out of L2.
template <typename V> __device__ __forceinline__ V buffer_load16_nt(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, uint32_t soff)
{
    const u32x4_t raw = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)voff, (int)soff, 2);
    return __builtin_bit_cast(V, raw);
}

// The data registers of a 16-byte store are still being read when the next instruction issues: overwritten there, the
// first or last word stored is now and then the new value (0.3 to 2 % of the stores of a busy chip).  Measured on gfx950:
// stores of 12 or 16 bytes need one instruction in between when a buffer store takes its offset from a scalar register, two
// otherwise; 8 bytes and LDS writes need none.  The compiler puts none and one.  Called right behind the store, this keeps
// the registers until they are free.
__device__ __forceinline__ void hold_store_data(u32x4_t v) { asm volatile("s_nop 1" : : "v"(v) : "memory"); }

typedef __attribute__((address_space(3))) unsigned char lds_byte_t;
typedef __attribute__((address_space(4))) const int32_t const_int_t;

typedef short v4i16_t __attribute__((ext_vector_type(4)));
typedef v4i16_t __attribute__((address_space(3))) lds_v4i16_t;

// 64 lanes' 16 bytes at src straight into LDS at lds + 16 lane.  Not through the builtin: the compiler then waits for every
// copy in flight before each transposing LDS load, also of another slot; the kernel's own waits say what a load needs.
template <bool STREAM> __device__ __forceinline__ void copy_to_lds(const void *src, uint32_t lds)
{
    if (STREAM) asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" : : "{m0}"(lds), "v"(src) : "memory");
    else asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "{m0}"(lds), "v"(src) : "memory");
}
// What slots past the last row of a tile are filled with: their softmax weight is 0, and 0 times an infinite value is NaN.
static __device__ __align__(256) const unsigned char kZeroRow[256] = {};
template <int N> __device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
__device__ __forceinline__ float max3(float x, float y, float z) { return fmaxf(fmaxf(x, y), z); }

template <class F, int... Is>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): a loop whose index is a constant expression
template <int N, class F> __device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// sum over the 16 lanes of a lane group (lanes that share lane/16)
__device__ __forceinline__ float group16_sum(float v)
{
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 8);
    return v;
}

__device__ __forceinline__ float sigmoidf_(float x) { return 1.0f / (1.0f + __expf(-x)); }

template <int CTRL> __device__ __forceinline__ float dpp_move(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kRowShl4 = 0x104, kRowShr4 = 0x114, kRowRor4 = 0x124, kRowRor8 = 0x128;

// Exchanges between the four rows of 16 lanes of a wave, on the vector unit (v_permlane16_swap, v_permlane32_swap; a
// shuffle goes through LDS).  swap16: rows 1, 3 of a against rows 0, 2 of b; swap32: the upper half of a against the
// lower half of b.
__device__ __forceinline__ void swap16(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap32(float &a, float &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]); b = __uint_as_float(r[1]);
}
// over the four lanes that share lane % 16
__device__ __forceinline__ float rows_sum(float v)
{
    float w = v;
    swap16(v, w);
    v += w; w = v;
    swap32(v, w);
    return v + w;
}
__device__ __forceinline__ float rows_max(float v)
{
    float w = v;
    swap16(v, w);
    v = fmaxf(v, w); w = v;
    swap32(v, w);
    return fmaxf(v, w);
}
// N values over the four rows at once (op: sum or maximum): afterwards lane row r holds, in v[i], i < N / 4, the result of
// value rows_value(i, r): an exchange halves the values that a lane still carries.
template <int N, class F> __device__ __forceinline__ void rows_fold(float (&v)[N], F op)
{
    static_assert(N % 4 == 0, "two halvings");
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
        swap16(v[2 * i], v[2 * i + 1]);
        v[i] = op(v[2 * i], v[2 * i + 1]);
    }
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
        swap32(v[2 * i], v[2 * i + 1]);
        v[i] = op(v[2 * i], v[2 * i + 1]);
    }
}
__device__ __forceinline__ int rows_value(int i, int row) { return 4 * i + 2 * (row >> 1) + (row & 1); }

// The sums over 16 lanes of four values at once: lane q (mod 4) receives the sum of v[value_of_lane(q)].
// (every exchange halves the values a lane still carries: 4 -> 2 -> 1, then the four quads are added: those eight lanes
// apart first, in fold8 and fold16 too, so that a sum has the same bits whichever of them takes it)
__device__ __forceinline__ int value_of_lane(int lane) { return ((lane & 1) << 1) | ((lane >> 1) & 1); }
__device__ __forceinline__ float fold4(const float (&v)[4], int lane)
{
    const bool b0 = lane & 1, b1 = lane & 2;
    const float r0 = (b0 ? v[2] : v[0]) + dpp_move<kQuadXor1>(b0 ? v[0] : v[2]);
    const float r1 = (b0 ? v[3] : v[1]) + dpp_move<kQuadXor1>(b0 ? v[1] : v[3]);
    float q = (b1 ? r1 : r0) + dpp_move<kQuadXor2>(b1 ? r0 : r1);
    q += dpp_move<kRowRor8>(q);
    q += dpp_move<kRowRor4>(q);
    return q;
}

// The same for 16 values, v[m][gate]: lane 4 m + q receives the sum over the 16 lanes of v[m][value_of_lane(q)].
__device__ __forceinline__ float fold16(const float (&v)[4][4], int lane)
{
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4, b3 = lane & 8;
    float q[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const float r0 = (b0 ? v[m][2] : v[m][0]) + dpp_move<kQuadXor1>(b0 ? v[m][0] : v[m][2]);
        const float r1 = (b0 ? v[m][3] : v[m][1]) + dpp_move<kQuadXor1>(b0 ? v[m][1] : v[m][3]);
        q[m] = (b1 ? r1 : r0) + dpp_move<kQuadXor2>(b1 ? r0 : r1);
    }
    const float p0 = (b3 ? q[2] : q[0]) + dpp_move<kRowRor8>(b3 ? q[0] : q[2]);
    const float p1 = (b3 ? q[3] : q[1]) + dpp_move<kRowRor8>(b3 ? q[1] : q[3]);
    const float away = b2 ? p0 : p1;        // what the lane four further on (b2: four back) is short of
    const float fwd = dpp_move<kRowShl4>(away), back = dpp_move<kRowShr4>(away);
    return (b2 ? p1 : p0) + (b2 ? back : fwd);
}

// The same for 8 values, v[m][value]: lane 8 m + q (mod 4 in q) receives the sum over the 16 lanes of v[m][value_of_lane(q)].
__device__ __forceinline__ float fold8(const float (&v)[2][4], int lane)
{
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4, b3 = lane & 8;
    float q[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const float r0 = (b0 ? v[m][2] : v[m][0]) + dpp_move<kQuadXor1>(b0 ? v[m][0] : v[m][2]);
        const float r1 = (b0 ? v[m][3] : v[m][1]) + dpp_move<kQuadXor1>(b0 ? v[m][1] : v[m][3]);
        q[m] = (b1 ? r1 : r0) + dpp_move<kQuadXor2>(b1 ? r0 : r1);
    }
    const float p = (b3 ? q[1] : q[0]) + dpp_move<kRowRor8>(b3 ? q[0] : q[1]);
    const float fwd = dpp_move<kRowShl4>(p), back = dpp_move<kRowShr4>(p);
    return p + (b2 ? back : fwd);
}

// four consecutive elements of a weight row from element k on, zeros at and past n.  VEC: the row allows one load.
template <typename T, bool VEC> __device__ __forceinline__ void load4(const T *row, int k, int n, float (&o)[4])
{
    if (VEC) {
        if (k < n) VecLoad<T, 4>::run(row + k, o);
        else o[0] = o[1] = o[2] = o[3] = 0.f;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = k + e < n ? Storage<T>::load(row + k + e) : 0.f;
    }
}

// exact (erf) GELU in fp32
__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

}  // namespace kvev
