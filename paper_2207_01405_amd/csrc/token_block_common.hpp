// What the two forms of the token-wise part of a block share (token_block.hip, token_stream.hip): the table of constants that
// a launch reads, the requantisation constants in it and the swizzle of token tiles in LDS.
#pragma once
#include "regst_common.hpp"

namespace ivit {
namespace tokblk {

using namespace regst;

template <int I> using ic = std::integral_constant<int, I>;

// Offsets in the table of one launch: LN2 (gamma, beta), LN1 or the final LN, then 16 bytes per channel of proj, fc2, fc1, qkv.
__host__ __device__ constexpr int TB_LN1(int C) { return 8 * C; }
__host__ __device__ constexpr int TB_PROJ(int C) { return 16 * C; }
__host__ __device__ constexpr int TB_FC2(int C) { return 32 * C; }
__host__ __device__ constexpr int TB_FC1(int C) { return 48 * C; }
__host__ __device__ constexpr int TB_QKV(int C, int F) { return 48 * C + 16 * F; }
__host__ __device__ constexpr int TB_BYTES(int C, int F) { return TB_QKV(C, F) + 48 * C; }

// XOR applied to the piece number of row r of a tile of P 16-byte pieces per row, G16 = gcd(P, 16), so that the same piece of
// 16 consecutive rows meets every bank group once.
__host__ __device__ constexpr int gcd16(int p) { return (p & 15) == 0 ? 16 : (p & 7) == 0 ? 8 : (p & 3) == 0 ? 4 : (p & 1) == 0 ? 2 : 1; }
template <int G16> __device__ __forceinline__ int swz(int r) { return (r / (16 / G16)) & (G16 - 1); }

// Requantisation constants of a channel, 16 bytes in the tables that table_kernel prepares.
//   Rq     24-bit form (derivation in gemm_rs.hip); lo > hi: the channel needs the general form
//   Rq64   residual layers: b and h of Residual64 (regst_common.hpp), the first term at most 2^30; b = 0: the channel needs
//          the general form.  Bytes 4 .. 7 of the entry are unused.
struct Rq { int32_t lo, hi, mb, ad; };
using Rq64 = Residual64;

// median of three as the pattern the compiler turns into one v_med3_i32
__device__ __forceinline__ int32_t med3c(int32_t v, int32_t lo, int32_t hi) { return max(min(v, lo), min(max(v, lo), hi)); }
template <class T> __device__ __forceinline__ void pin(T& v) { asm volatile("" : "+v"(v)); }      // keeps a value's computation in its place

__device__ __forceinline__ Rq as_rq(const v4i& v) { return Rq{v[0], v[1], v[2], v[3]}; }
__device__ __forceinline__ Rq64 as_rq64(const v4i& v) {
    Rq64 q{(uint32_t)v[0], ((uint64_t)(uint32_t)v[3] << 32) | (uint32_t)v[2]};
    pin(q.h);
    return q;
}

// The residual pair of a layer; ok: its term takes the 24-bit multiply-add
struct ResRq { int32_t b, c, h; bool ok; };
__device__ __forceinline__ ResRq make_res(Dyadic d) { return ResRq{d.b, d.c, 1 << ((d.c - 1) & 31), residual_term_24(d)}; }

// one result, 24-bit form: in the top byte
__device__ __forceinline__ uint32_t out_top(int32_t a, const Rq& q) { return (uint32_t)(__mul24(med3c(a, q.lo, q.hi), q.mb) + q.ad); }
// one result of a residual layer: one 64-bit multiply-add, the residual term, the sum limited (it fits
// 32 bits: at most 2^30 from channels with a 32-bit form, see table_kernel, and 2^29 from the residual)
__device__ __forceinline__ uint32_t out_res(int32_t a, const Rq64& q, const ResRq& rr, int32_t res) {
    return (uint32_t)clamp8(residual64_first(a, q) + ((__mul24(res, rr.b) + rr.h) >> rr.c));
}
// the low (or top) bytes of four results as a word
template <bool LOW> __device__ __forceinline__ int pack4(const uint32_t (&o)[4]) {
    const uint32_t p01 = __builtin_amdgcn_perm(o[1], o[0], LOW ? 0x0c0c0400u : 0x0c0c0703u);
    const uint32_t p23 = __builtin_amdgcn_perm(o[3], o[2], LOW ? 0x04000c0cu : 0x07030c0cu);
    return (int)(p01 | p23);
}

}  // namespace tokblk
}  // namespace ivit
