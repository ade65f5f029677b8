// Device helpers shared by the bf16 GEMM translation units: vector types, bf16 conversions, scalar loads.
#pragma once

#include "moe_internal.h"

namespace moe355 {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
// Types for reading operand fragments out of LDS.  The compiler orders an LDS read that carries type-based
// alias information after EVERY direct-to-LDS load in flight (s_waitcnt vmcnt(0) in front of the read), which
// drains the load pipeline once per K tile; reads through vector types and may_alias types carry none, and
// the explicit vmcnt before each stage barrier is what orders them.
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef uint32_t __attribute__((may_alias)) u32_lds;
typedef uint16_t __attribute__((may_alias)) u16_lds;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void glb_void;

// What direct-to-LDS loads take for the 16-byte chunks of the last K tile that lie past K: either operand is then zero there, whatever
// the other holds.  (By address and not with a mask behind the LDS read: the K loop stays as it is.)
__device__ __align__(16) static const uint16_t chunk_of_zeros[8] = {0, 0, 0, 0, 0, 0, 0, 0};

// One 32-bit word at an address that is the same for every lane of the wave, through the scalar data path
// (read only).  The compiler issues such loads as vector loads here (it cannot prove that the kernel's own
// stores leave the tile map alone), and a vector load's result can only be waited for together with every
// vector load issued before it -- at a tile switch that drains the whole operand pipeline.  The scalar path
// has its own counter.  The words read were written by an earlier kernel.
__device__ __forceinline__ int32_t uniform_load(const int32_t *ptr)
{
    int32_t v;
    asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=s"(v) : "s"(ptr) : "memory");
    return v;
}
// two independent words with one wait
__device__ __forceinline__ void uniform_load2(const int32_t *pa, const int32_t *pb, int32_t &a, int32_t &b)
{
    asm volatile("s_load_dword %0, %2, 0x0\n\ts_load_dword %1, %3, 0x0\n\ts_waitcnt lgkmcnt(0)"
                 : "=&s"(a), "=&s"(b)
                 : "s"(pa), "s"(pb)
                 : "memory");
}

// The K tile that a tile of an expert's begins with where its K loop goes round K.  Weight rows of a multiple of 4 KB have the same
// K tile in the same few memory channels, and the blocks, which walk K in step, ask those all at once (a bare read of 256 rows a
// block, from 0 / from different places: rows of 4 KB 4.9 / 6.3 TB/s, 8 KB 4.7 / 6.3, 16 KB 6.0 / 6.3).  By the expert (Fibonacci
// hashing: neighbours lie far apart) over the whole of K, and a K tile further with every column tile, so that column tiles find
// their common rows in the L2 still (col: less than KT).  An expert's row tiles, which share its weights, agree.
// e4m3 weights come in blocks of 1 KB along K, and the 16-row groups of blocks are 16 K bytes apart: the same, four channels at a time.
static constexpr int kTurnedK = 2048, kTurnedK8 = 1024;  // rows of a multiple of so many bf16, e4m3 weights
__device__ __forceinline__ int turned_k(int expert, int col, int KT)
{
    const uint32_t by_expert = ((uint32_t)expert * 2654435761u >> 16) * (uint32_t)KT >> 16;
    const int k = (int)by_expert + col;
    return k >= KT ? k - KT : k;
}

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ uint32_t to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
// two fp32 -> packed bf16, round to nearest even (one v_cvt_pk_bf16_f32)
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    const bf16x2 b = __builtin_convertvector(v, bf16x2);
    return *reinterpret_cast<const uint32_t *>(&b);
}

// max(x, 0) on two packed bf16: a bf16 is negative exactly when its bit pattern is negative as a 16-bit integer,
// so one packed integer max replaces two fp32 compares (and the canonicalisation the compiler puts in front of
// them); rounding is monotonic and keeps zero, so ReLU after the conversion equals ReLU before it.
typedef __attribute__((ext_vector_type(2))) short i16x2;
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t packed)
{
    const i16x2 zero = {0, 0};
    const i16x2 r = __builtin_elementwise_max(*reinterpret_cast<const i16x2 *>(&packed), zero);
    return *reinterpret_cast<const uint32_t *>(&r);
}

}  // namespace moe355
