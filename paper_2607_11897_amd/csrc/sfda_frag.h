// Complex 16 x 16 matrix operands of the factored kernels, on both kinds of matrix instruction,
// and the loads and stores they share.
#pragma once

#include "sfda_chunk_common.h"

namespace sfda {
namespace fac {

typedef uint32_t u32;
typedef u32 u32x2 __attribute__((ext_vector_type(2)));
typedef u32 u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// LDS written and read by one wave: its LDS instructions run in order, so only the compiler has
// to keep the order
__device__ __forceinline__ void wave_order() { asm volatile("" ::: "memory"); }

// two floats -> (lo, hi) bf16 pair, round to nearest even
__device__ __forceinline__ u32 pack_bf16(float lo, float hi) {
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(u32, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf_lo(u32 w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(u32 w) { return __uint_as_float(w & 0xFFFF0000u); }

// wave-uniform size kept in a scalar register (a size in a vector register turns every access
// into a loop over the wave's descriptors)
__device__ __forceinline__ rsrc_t rsrc(const void* base, int bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, __builtin_amdgcn_readfirstlane(bytes),
                                             0x00020000);
}
__device__ __forceinline__ u32x4 ld128(rsrc_t r, u32 off) { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0); }

// ------------------------------------------------------------------ complex matrix operands
// A complex 16 x 16 result is two accumulator tiles (real and imaginary part; lane (c, g) holds
// rows 4g + r of column c).  A fragment holds 4 consecutive K entries of one row (left operand)
// or of one column (right operand) as (re, im) pairs; a right operand enters one product per
// output part, as (Re, -Im) and as (Im, Re).
struct CAcc { f32x4 re, im; };
__device__ __forceinline__ void czero(CAcc& z) { z.re = zero4(); z.im = zero4(); }

template <int P> struct Frag;
template <> struct Frag<PREC_BF16> { u32x4 w; };
template <> struct Frag<PREC_F32> { float2 x[4]; };
template <int P> struct Right;
template <> struct Right<PREC_BF16> { u32x4 re, im; };
template <> struct Right<PREC_F32> { float re[4], im[4], nim[4]; };

template <int P> __device__ __forceinline__ Frag<P> frag4(const float2 (&x)[4]) {
    Frag<P> f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if constexpr (P == PREC_BF16) f.w[r] = pack_bf16(x[r].x, x[r].y);
        else f.x[r] = x[r];
    }
    return f;
}
// s = -1 negates
template <int P> __device__ __forceinline__ Frag<P> frag_acc(const CAcc& z, float s = 1.f) {
    float2 x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = make_float2(s * z.re[r], s * z.im[r]);
    return frag4<P>(x);
}
// what the rounding of x to a fragment leaves over
__device__ __forceinline__ float2 rest(float2 x) {
    const uint32_t w = pack_bf16(x.x, x.y);
    return make_float2(x.x - bf_lo(w), x.y - bf_hi(w));
}
template <int P> __device__ __forceinline__ float2 frag_get(const Frag<P>& f, int r) {
    if constexpr (P == PREC_BF16) return make_float2(bf_lo(f.w[r]), bf_hi(f.w[r]));
    else return f.x[r];
}
template <int P> __device__ __forceinline__ Right<P> right(const Frag<P>& f) {
    Right<P> b;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if constexpr (P == PREC_BF16) {
            b.re[r] = f.w[r] ^ 0x80000000u;
            b.im[r] = __builtin_amdgcn_alignbit(f.w[r], f.w[r], 16);
        } else {
            b.re[r] = f.x[r].x;
            b.im[r] = f.x[r].y;
            b.nim[r] = -f.x[r].y;
        }
    }
    return b;
}
// right operand from a split accumulator
template <int P> __device__ __forceinline__ Right<P> right_acc(const CAcc& y) {
    Right<P> b;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if constexpr (P == PREC_BF16) {
            b.re[r] = pack_bf16(y.re[r], -y.im[r]);
            b.im[r] = pack_bf16(y.im[r], y.re[r]);
        } else {
            b.re[r] = y.re[r];
            b.im[r] = y.im[r];
            b.nim[r] = -y.im[r];
        }
    }
    return b;
}
// z += X Y over 16 complex K indices
template <int P> __device__ __forceinline__ void cmma(CAcc& z, const Frag<P>& a, const Right<P>& b) {
    if constexpr (P == PREC_BF16) {
        z.re = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.w), __builtin_bit_cast(bf16x8, b.re), z.re, 0, 0, 0);
        z.im = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.w), __builtin_bit_cast(bf16x8, b.im), z.im, 0, 0, 0);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            z.re = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[r].x, b.re[r], z.re, 0, 0, 0);
            z.im = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[r].x, b.im[r], z.im, 0, 0, 0);
            z.re = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[r].y, b.nim[r], z.re, 0, 0, 0);
            z.im = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x[r].y, b.re[r], z.im, 0, 0, 0);
        }
    }
}
// a lane's entries of a fragment in the records' order
template <int P> __device__ __forceinline__ void put_frag(char* f, int lane, const Frag<P>& x) {
    if constexpr (P == PREC_BF16) {
        *reinterpret_cast<u32x4*>(f + lane * 16) = x.w;
    } else {
        *reinterpret_cast<float4*>(f + lane * 16) = make_float4(x.x[0].x, x.x[0].y, x.x[1].x, x.x[1].y);
        *reinterpret_cast<float4*>(f + 1024 + lane * 16) = make_float4(x.x[2].x, x.x[2].y, x.x[3].x, x.x[3].y);
    }
}

template <typename TOUT> __device__ __forceinline__ void st_real(rsrc_t r, u32 off, int s, float x) {
    if constexpr (sizeof(TOUT) == 4) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, off, s, 0);
    else __builtin_amdgcn_raw_buffer_store_b16(static_cast<uint16_t>(pack_bf16(x, 0.f)), r, off, s, 0);
}
template <typename TV> __device__ __forceinline__ float2 ld_cplx(rsrc_t r, u32 off, int s = 0) {
    if constexpr (sizeof(TV) == 4) {
        return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, s, 0));
    } else {
        const u32 w = __builtin_amdgcn_raw_buffer_load_b32(r, off, s, 0);
        return make_float2(bf_lo(w), bf_hi(w));
    }
}

__device__ __forceinline__ f32x4 ldv4(rsrc_t r, u32 off, int s = 0) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, s, 0));
}
__device__ __forceinline__ float2 ldv2(rsrc_t r, u32 off, int s = 0) {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, s, 0));
}
// LDS-poison debug build: a kernel's whole exchange area at entry (every thread of the workgroup), and
// this lane's slot of a parity once the barrier behind its last read is passed, so that a read of what
// is not written yet, or of what another block left, gives NaN
template <typename T> __device__ __forceinline__ void poison_area(T& area, int nthr) {
#ifdef SFDA_LDS_POISON
    lds_poison(&area, sizeof(area), threadIdx.x, nthr);
    __syncthreads();
#endif
}
template <typename T> __device__ __forceinline__ void poison_slot(T& slot) {
#ifdef SFDA_LDS_POISON
    static_assert(sizeof(T) % 4 == 0, "whole words");
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) reinterpret_cast<u32*>(&slot)[i] = 0xFFFFFFFFu;
#endif
}

// keeps the loads before it in this order for every block, so that the wait counts stay exact
#define LOAD_ORDER() __builtin_amdgcn_sched_barrier(0)

}  // namespace fac
}  // namespace sfda
