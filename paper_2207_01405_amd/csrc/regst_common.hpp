// Pieces shared by the Dense kernels built on LDS-direct loads (gemm_rs.hip, gemm_ks.hip, gemm_tl.hip, gemm_st.hip,
// token_block.hip): those loads, scalar pointers, the median of three, the token order of the MFMA "A" operand.
#pragma once
#include <type_traits>
#include <utility>

#include "ivit_kernels.hpp"

namespace ivit {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

namespace regst {

enum Epilogue { EPI_PLAIN = 0, EPI_RESIDUAL = 1, EPI_GELU = 2 };
constexpr int NXCD = 8;
constexpr int OP = 48;                       // pitch (bytes) of a channel row of the output staging tile: 32 tokens + padding
constexpr int WCK = 384;                     // bytes of K per weight chunk of the prologue
constexpr int WPITCH = WCK + 16;             // its row pitch in LDS
constexpr int WWI = 4 * 32 * (WPITCH / 16) / 64;    // load instructions (64 lanes x 16 bytes) per chunk: [4 wavefronts][32 channels][WPITCH]

// f(0), .. f(N - 1), each with its number as a type
template <int N, class F> __device__ __forceinline__ void static_for(F&& f) {
    [&]<int... I>(std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>()), ...); }(std::make_integer_sequence<int, N>());
}

__device__ __forceinline__ uint32_t lds_offset(const int8_t* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) int8_t*)p;
}
__device__ __forceinline__ const int8_t* uniform_ptr(const int8_t* p) {          // a pointer every lane agrees on -> scalar registers
    const uint64_t v = (uint64_t)p;
    // (the builtin returns a signed int: each half goes through uint32_t so that nothing is sign-extended into the other)
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    return (const int8_t*)(((uint64_t)hi << 32) | (uint64_t)lo);
}

// 16 bytes per lane from global memory straight into LDS: lane l's piece, read at base + off, lands at lds + 16 l
// (base and lds are the same for all lanes).  Written as asm statements so that the compiler does not make every
// later LDS read wait for all such loads; the waits are placed by hand (s_waitcnt vmcnt) where the data is first read.
__device__ __forceinline__ void dma16(const int8_t* base, uint32_t off, uint32_t lds_wave_base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 : : "s"(__builtin_amdgcn_readfirstlane(lds_wave_base)), "v"(off), "s"(base) : "memory", "m0");
}
// ... 4 bytes per lane
__device__ __forceinline__ void dma4(const void* base, uint32_t off, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 : : "s"(__builtin_amdgcn_readfirstlane(dst)), "v"(off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void wait_vm0() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ int32_t med3(int32_t v, int32_t lo, int32_t hi) {
    int32_t m;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(m) : "v"(v), "v"(lo), "v"(hi));
    return m;
}

// Residual layers: the first term floor((acc b + h) / 2^c), h = bias b + rounding addend, is the high word of one 64-bit
// multiply-add by the factor b 2^(32-c).  It takes every dyadic_fits32 pair, b <= 2^c: the factor and the sum it multiplies are
// unsigned.  To that end the products of such a layer are added to kSumStart = 2^30 (the bits of 2.0, which a matrix instruction
// has at hand) and not to 0: |acc| <= 2^14 K <= 2^30, so u = acc + 2^30 is not negative; the addend takes 2^30 times the factor away
// again.  A form with 24-bit multiplies, which has to keep the sum's nine bits above the fraction, ends at c = 23, and layers
// with long rows need c = 24 (ViT-B's second MLP layer, 50432 rows: 150 us with the general 64-bit form, 131.6 with a multiply-add
// by b, an addition and a shift; forwards against that one: DeiT-S batch 128 1230 -> 1214 us, ViT-B batch 256 5580 -> 5548).
// With a signed factor, which leaves pairs of b >= 2^(c-1) to the general form, two blocks of DeiT-S with such pairs, batch
// 128, took 260 us instead of 181.  The addend is one 64-bit register pair that the compiler cannot look into: it would add the two
// halves one after the other.
constexpr uint32_t kSumStart = 0x40000000u;
struct Residual64 { uint32_t b; uint64_t h; };
__device__ __forceinline__ bool residual64_of(Residual64& q, int32_t b, int32_t c, int32_t bias, int32_t rnd) {
    const int up = 32 - (c & 31);
    const uint32_t one = 1u << (c & 31);
    const int64_t h = (int64_t)bias * b + ((int64_t)b * -(int32_t)kSumStart + (int64_t)((uint32_t)rnd << ((c - 1) & 31)));
    // b = 2^c, a factor of 2^32: u 2^32 + h' has the high word of u (2^32 - 1) + (h' | 2^32 - 1), u being below 2^32
    const uint32_t whole = (uint32_t)b == one ? 0xffffffffu : 0u;
    q.b = ((uint32_t)b << (up & 31)) | whole;
    q.h = (uint64_t)h << up | whole;
    asm volatile("" : "+v"(q.h));
    return (c >= 1) & (c <= 31) & (b >= 1) & ((uint32_t)b <= one);       // dyadic_fits32, without branches
}
__device__ __forceinline__ int32_t residual64_first(int32_t u, const Residual64& q) { return (int32_t)(((uint64_t)(uint32_t)u * q.b + q.h) >> 32); }
// acc + bias from sums that exceed acc by `start`, for the general form
__device__ __forceinline__ int32_t sum_of(int32_t u, int32_t bias, uint32_t start) { return (int32_t)((uint32_t)u + ((uint32_t)bias - start)); }
__device__ __forceinline__ v16i sums_from(uint32_t start) {
    v16i v;
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = (int)start;
    return v;
}
// The residual term round(b_r r / 2^c_r) takes one 24-bit multiply-add under these conditions.
__device__ __forceinline__ bool residual_term_24(Dyadic d) { return d.b >= 1 && d.b < (1 << 23) && d.c >= 1 && d.c <= 30; }

// Token of the tile that sits in row i of the MFMA "A" operand.  Accumulator register e = 4 q + r of lane group g is
// row 8 q + 4 g + r of the product; with this assignment it is token 16 g + e: a lane holds 16 consecutive tokens.
__device__ __forceinline__ int token_of_row(int i) { return 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3); }

}  // namespace regst
}  // namespace ivit
