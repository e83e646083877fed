// Fused integer multi-head attention for gfx950 (I-ViT, arXiv 2207.01405: Eq. 3-4 with the dyadic
// pipeline of Sec. 3.2 and Shiftmax of Sec. 3.3 / Algorithm 1):
//   A = requant(Q K^T) [+ relative-position bias];  P = Shiftmax(rows of A);  O = requant(P V).
//
// One workgroup (4 wavefronts) handles one (image-or-window, head) at a time: K and V live in LDS, both
// row by row as they come from memory, and each wavefront takes 16 query tokens at a time.  Scores are produced by
// v_mfma_i32_16x16x64_i8 (d = 64) or 16x16x32 (d = 32) in the orientation keys x queries, so that a lane
// holds, for ONE query, four keys of every 16-key tile: the whole score row of a query sits in the
// registers of four lanes.  Max and sum need an in-lane pass plus two cross-lane steps; ShiftExp is a
// table lookup on Delta = max - value (at most 510); the packed int8 probabilities are already laid out as
// the MFMA "B" operand (contraction index = key) of O^T = V^T P^T, so scores and probabilities never
// leave registers.  The "A" operand of that product, V^T, is read from the rows of V with the transposing
// LDS read of gfx950 (ds_read_b64_tr_b8): the lanes of a 16-lane block name eight key rows each for the even and
// the odd lanes, so the key order the register layout asks for and the choice of features are a matter of which
// addresses the lanes name, and V needs no rearranging when it is written.  One exchange between neighbouring
// lane blocks then gives every lane d/4 consecutive features of its query: one 16-byte (d = 64) store.
//
// The kernel is bound by the vector ALU (five integer operations and a table read per score element in the 24-bit form, about a
// dozen in the general one, against 2 d multiply-accumulates on the matrix core), so the per-element path is kept minimal:
// debug taps, the bias and the 64-bit requantisation are compiled in only when asked for (template flags), and masking
// of padded keys is done only for key tiles that are not completely valid.  Many 7 x 7 windows have a form of their own below.
#include <algorithm>
#include <type_traits>

#include "attention_form.hpp"
#include "ivit_kernels.hpp"

namespace ivit {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int ATT_WAVES = 4, ATT_THREADS = 64 * ATT_WAVES;   // wavefronts per workgroup

typedef int v2i_att __attribute__((ext_vector_type(2)));

// Constants of the 24-bit requantisation of one per-tensor dyadic pair (no bias): the accumulator is limited to
// [lo, hi], the first values that give -127 / +127, after which (v b + 2^(c-1)) 2^(24-c) fits 32 bits with the int8
// result in its top byte.  Valid for c <= 24, b < 2^(c-1) and bounds inside 24 bits (narrow_of() decides).
struct Narrow { int32_t lo, hi, mb, ad; };

// Constants of the 24-bit IntDiv (intdiv24_up): the scale of the table's entries, 2^(M+up) as a float and modulo 2^32, and the scaled
// sum of a row in which one key has all of it.  Formed here, for every row, from `up`, which stands in the place of k_out in the
// kernels' arguments (k_out is M - 23 in that form): more arguments part the loads of the others, which a workgroup with one item
// waits for (100 images x 8 heads of 81 tokens with a bias 11.1 -> 11.8 us with four), and the constants kept take scalar registers
// that the forms with a bias do not have.
struct Div24 { int32_t up; float num; uint32_t num32; int32_t alone; };
__device__ __forceinline__ Div24 div24_of(ShiftParams sm) {
    int up = sm.k_out;
    asm volatile("" : "+s"(up));
    const int bits = sm.m_bits + up;
    return Div24{up, __uint_as_float((uint32_t)(127 + bits) << 23), (uint32_t)((uint64_t)1 << bits), sm.i0 << (sm.n_shift + up)};
}

// FAST: 0 general 64-bit requantisation, 1 pairs that fit 32 bits, 2 the 24-bit form above (and the 24-bit IntDiv).
template <int FAST>
__device__ __forceinline__ int32_t requant8(int32_t v, Dyadic d, Narrow n, int32_t rnd) {
    if (FAST == 2) {
        // The median of three as the one instruction, by hand because the compiler cannot know lo <= hi.  The compiler
        // does not see what an asm statement reads and puts no wait states between it and the producer of v: v must
        // have been written long before (here: MFMA results of a whole tile sweep), never by the instruction just
        // before (a dot product feeding this directly was seen to read a stale register).
        int32_t m;
        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(m) : "v"(v), "v"(n.lo), "v"(n.hi));
        return (__mul24(m, n.mb) + n.ad) >> 24;
    }
    return FAST ? clamp8(rnd_shift_fit32(v, d.b, d.c, rnd)) : requant64(v, d.b, d.c, rnd);
}

// Four values at once: the four medians first, then the four multiply-adds, so that no instruction reads the result of
// the asm statement right before it (the compiler, not knowing what the statement is, would put a wait state there).
template <int FAST>
__device__ __forceinline__ void requant8x4(int32_t (&v)[4], Dyadic d, Narrow n, int32_t rnd) {
    if (FAST == 2) {
        int32_t m[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) asm("v_med3_i32 %0, %1, %2, %3" : "=v"(m[r]) : "v"(v[r]), "v"(n.lo), "v"(n.hi));
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = (__mul24(m[r], n.mb) + n.ad) >> 24;
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = requant8<FAST>(v[r], d, n, rnd);
    }
}

// ---- pieces of the 24-bit form.  A result T has its int8 value in the top byte; sub-dword selects (SDWA) read and write bytes in
// the instruction that needs them.  The asm statements read ordinary vector results and loads only (see requant8).
__device__ __forceinline__ int32_t med3_i32(int32_t v, int32_t lo, int32_t hi) {
    int32_t m;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(m) : "v"(v), "v"(lo), "v"(hi));
    return m;
}
__device__ __forceinline__ int32_t narrow_top(int32_t v, Narrow n) { return __mul24(med3_i32(v, n.lo, n.hi), n.mb) + n.ad; }
// a - 2 v for a v of 24 bits (written out: the compiler cannot know that a score has no more)
__device__ __forceinline__ uint32_t minus_twice(int32_t a, int32_t v) {
    uint32_t r;
    asm("v_mad_i32_i24 %0, %1, -2, %2" : "=v"(r) : "v"(v), "v"(a));
    return r;
}
// twice the top byte: the byte offset of a 16-bit table entry
__device__ __forceinline__ uint32_t twice_top(uint32_t d) {
    uint32_t r;
    asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "v"(1), "v"(d));
    return r;
}
// top byte of t plus byte R of w, both signed
template <int R> __device__ __forceinline__ int32_t top_plus_byte(int32_t t, uint32_t w) {
    int32_t r;
    if constexpr (R == 0) asm("v_add_u32_sdwa %0, sext(%1), sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:BYTE_0" : "=v"(r) : "v"(t), "v"(w));
    if constexpr (R == 1) asm("v_add_u32_sdwa %0, sext(%1), sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:BYTE_1" : "=v"(r) : "v"(t), "v"(w));
    if constexpr (R == 2) asm("v_add_u32_sdwa %0, sext(%1), sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:BYTE_2" : "=v"(r) : "v"(t), "v"(w));
    if constexpr (R == 3) asm("v_add_u32_sdwa %0, sext(%1), sext(%2) dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:BYTE_3 src1_sel:BYTE_3" : "=v"(r) : "v"(t), "v"(w));
    return r;
}
// Four words of probabilities: byte r of word i is (f e[i][r]) >> 32, f and e below 2^24.  Every product is written into its byte;
// writes to one register stand four instructions apart (a byte write may not be followed directly by a reader of that register).
__device__ __forceinline__ void div_pack4(uint32_t (&w)[4], uint32_t f, const int32_t (&e0)[4], const int32_t (&e1)[4], const int32_t (&e2)[4], const int32_t (&e3)[4]) {
#define IVIT_DP(D, E, B, U) "v_mul_hi_u32_u24_sdwa %" #D ", %4, %" #E " dst_sel:BYTE_" #B " dst_unused:" U " src0_sel:DWORD src1_sel:DWORD\n\t"
    asm(IVIT_DP(0, 5, 0, "UNUSED_PAD") IVIT_DP(1, 9, 0, "UNUSED_PAD") IVIT_DP(2, 13, 0, "UNUSED_PAD") IVIT_DP(3, 17, 0, "UNUSED_PAD")
        IVIT_DP(0, 6, 1, "UNUSED_PRESERVE") IVIT_DP(1, 10, 1, "UNUSED_PRESERVE") IVIT_DP(2, 14, 1, "UNUSED_PRESERVE") IVIT_DP(3, 18, 1, "UNUSED_PRESERVE")
        IVIT_DP(0, 7, 2, "UNUSED_PRESERVE") IVIT_DP(1, 11, 2, "UNUSED_PRESERVE") IVIT_DP(2, 15, 2, "UNUSED_PRESERVE") IVIT_DP(3, 19, 2, "UNUSED_PRESERVE")
        IVIT_DP(0, 8, 3, "UNUSED_PRESERVE") IVIT_DP(1, 12, 3, "UNUSED_PRESERVE") IVIT_DP(2, 16, 3, "UNUSED_PRESERVE") IVIT_DP(3, 20, 3, "UNUSED_PRESERVE") "s_nop 0"
        : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
        : "v"(f), "v"(e0[0]), "v"(e0[1]), "v"(e0[2]), "v"(e0[3]), "v"(e1[0]), "v"(e1[1]), "v"(e1[2]), "v"(e1[3]),
          "v"(e2[0]), "v"(e2[1]), "v"(e2[2]), "v"(e2[3]), "v"(e3[0]), "v"(e3[1]), "v"(e3[2]), "v"(e3[3]));
#undef IVIT_DP
}
// ... one word
__device__ __forceinline__ uint32_t div_pack(uint32_t f, const int32_t (&e)[4]) {
    uint32_t w;
#define IVIT_DP(E, B, U) "v_mul_hi_u32_u24_sdwa %0, %1, %" #E " dst_sel:BYTE_" #B " dst_unused:" U " src0_sel:DWORD src1_sel:DWORD\n\ts_nop 0\n\t"
    asm(IVIT_DP(2, 0, "UNUSED_PAD") IVIT_DP(3, 1, "UNUSED_PRESERVE") IVIT_DP(4, 2, "UNUSED_PRESERVE") IVIT_DP(5, 3, "UNUSED_PRESERVE")
        : "=&v"(w) : "v"(f), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]));
#undef IVIT_DP
    return w;
}

// The rows of a 24-bit form with a relative-position bias and / or the shifted-window mask, up to the row maximum.  A masked key
// gets mask_add.  Returns the maximum; masked: whether anything in the tile's rows is masked.  nfull: key tiles whose keys all exist;
// left: keys from this lane's first one on.
template <bool MASK, int NKT>
__device__ __forceinline__ int32_t biased_scores(int32_t (&sc)[NKT][4], const uint32_t (&bw)[NKT], const uint32_t (&mw)[NKT], Narrow nqk, int32_t mask_add,
                                                 int nfull, int left, bool& masked) {
    uint32_t any = 0;
    int32_t mx = INT32_MIN;
#pragma unroll
    for (int t = 0; t < NKT; ++t) {
        int32_t tp[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) tp[r] = narrow_top(sc[t][r], nqk);
        sc[t][0] = top_plus_byte<0>(tp[0], bw[t]); sc[t][1] = top_plus_byte<1>(tp[1], bw[t]);
        sc[t][2] = top_plus_byte<2>(tp[2], bw[t]); sc[t][3] = top_plus_byte<3>(tp[3], bw[t]);
        any |= mw[t];
        __builtin_amdgcn_sched_barrier(0);
    }
    // (most windows of a shifted grid have nothing masked)
    masked = false;
    if (MASK) {
        masked = __builtin_amdgcn_ballot_w64(any != 0) != 0;
        if (masked) {
#pragma unroll
            for (int t = 0; t < NKT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) if ((mw[t] >> (8 * r)) & 0xffu) sc[t][r] += mask_add;
        }
    }
#pragma unroll
    for (int t = 0; t < NKT; ++t) {
        if (t < nfull) {
            mx = max(mx, max(max(sc[t][0], sc[t][1]), max(sc[t][2], sc[t][3])));
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) if (16 * t + r < left) mx = max(mx, sc[t][r]);
        }
    }
    return rows_allreduce(mx, [](int32_t a, int32_t b) { return max(a, b); });
}

// ShiftExp of the scores by table (16-bit entries); returns the row sum.  !BIAS: the score's product is subtracted from `base`.
// CLAMP: a delta may lie beyond the table, whose last entry stands for it.
template <bool BIAS, bool CLAMP, int NKT>
__device__ __forceinline__ int32_t look_up(int32_t (&sc)[NKT][4], const uint16_t* lut, int n_lut, int32_t mx, uint32_t base, Narrow nqk, int nfull, int left) {
    const char* lut_b = reinterpret_cast<const char*>(lut);
    const int32_t mx2 = 2 * mx;
    int32_t sum = 0;
#pragma unroll
    for (int t = 0; t < NKT; ++t) {
        uint32_t at[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (!BIAS) {
                at[r] = twice_top(base + (uint32_t)__mul24(med3_i32(sc[t][r], nqk.lo, nqk.hi), -nqk.mb));
            } else {
                at[r] = minus_twice(mx2, sc[t][r]);
                if constexpr (CLAMP) at[r] = min(at[r], 2u * (uint32_t)(n_lut - 1));
            }
        }
        if (t < nfull) {
#pragma unroll
            for (int r = 0; r < 4; ++r) sc[t][r] = (int32_t)*reinterpret_cast<const uint16_t*>(lut_b + at[r]);
        } else {                                   // (an absent key may stand above the maximum)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool there = 16 * t + r < left;
                const int32_t e = (int32_t)*reinterpret_cast<const uint16_t*>(lut_b + (there ? at[r] : 0u));
                sc[t][r] = there ? e : 0;
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) sum += sc[t][r];
        if (t & 1) __builtin_amdgcn_sched_barrier(0);
    }
    return rows_allreduce(sum, [](int32_t a, int32_t b) { return a + b; });
}

// IntDiv of the 24-bit form (intdiv24_up): entries and their sum come scaled by 2^up, this is inv 2^(8-up), and the quotient is
// the upper word of its product with an entry.  2^(k_out-1), which a byte may not become, is the quotient only where one key has
// the whole sum, ShiftExp(0); taking one from inv there gives 2^(k_out-1) - 1 and leaves every other row
// alone.  The reciprocal floor(2^M / sum) = floor(2^(M+up) / scaled), below 2^24, from a single-precision quotient with one
// correction (a power of two times the reciprocal is exact but for the reciprocal's own last bit): to one, which the remainder repairs.
__device__ __forceinline__ uint32_t div_factor(int32_t scaled, Div24 d) {
    const float s = (float)(uint32_t)scaled, r = __builtin_amdgcn_rcpf(s), q = d.num * r;
    uint32_t inv = (uint32_t)__builtin_fmaf(__builtin_fmaf(-q, s, d.num), r, q);
    const int32_t rem = (int32_t)(d.num32 - inv * (uint32_t)scaled);
    inv += (rem >= scaled);
    inv -= (rem < 0);
    inv -= scaled == d.alone;
    return inv << (8 - d.up);
}

// The lane's four output tiles requantised (24-bit form) to one word each
template <int ND> __device__ __forceinline__ void narrow_words(uint32_t (&ow)[ND], const v4i (&oacc)[ND], Narrow npv) {
#pragma unroll
    for (int n = 0; n < ND; ++n) {
        uint32_t ov[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) ov[r] = (uint32_t)narrow_top(oacc[n][r], npv);
        ow[n] = __builtin_amdgcn_perm(ov[1], ov[0], 0x0c0c0703u) | __builtin_amdgcn_perm(ov[3], ov[2], 0x07030c0cu);
    }
}

// FAST: both dyadic pairs are rescales by at most 1 with c <= 31 (32-bit requantisation) and the row sum always
// exceeds 2^(k_out-1), so that IntDiv is one multiply-high by the pre-shifted reciprocal.
// TFIX: 0, or the token count known at compile time (49, the 7 x 7 windows; 197, the 14 x 14 patches with a class token):
// every test of a key or query against T then folds, and the absent keys of the last key tile cost nothing.
template <int D, int NKT, bool TAPS, bool BIAS, bool MASK, int FAST, int TFIX = 0>
__global__ __launch_bounds__(ATT_THREADS, 3) void attention_kernel(const int8_t* __restrict__ qkv,
                                                        const int8_t* __restrict__ rel_bias,
                                                        const int8_t* __restrict__ mask, FastDiv n_mask,
                                                        const int32_t* __restrict__ tok_index, FastDiv n_win,
                                                        int8_t* __restrict__ o, int n_items, FastDiv split_d, int T_arg, int C, FastDiv H,
                                                        Dyadic qk, ShiftParams sm, Dyadic pv, Narrow nqk, Narrow npv, int rnd,
                                                        int8_t* __restrict__ tap_s, int8_t* __restrict__ tap_p) {
    const int T = TFIX ? TFIX : T_arg, split = (int)split_d.d;
    constexpr int KROW = D + 16;                  // K row pitch (bytes)
    constexpr int NKC = (NKT + 3) / 4;            // 64-key chunks of the P V contraction
    constexpr int VP = D == 64 ? 72 : 40;         // V row pitch (bytes): the transposing reads below meet no bank twice
    constexpr int ND = D / 16;                    // 16-feature tiles of the output
    constexpr int DCH = D / 16;                   // 16-byte chunks per K / V row
    constexpr bool ONE = TFIX && TFIX <= 16 * ATT_WAVES;      // no wavefront has a second query tile
    __shared__ __align__(16) int8_t Ks[NKT * 16 * KROW];
    __shared__ __align__(16) int8_t Vs[NKC * 64 * VP];
    // table of ShiftExp(-delta): int8 scores give delta <= 254; with a bias and the mask the exact range is wider,
    // and beyond the table the value is 0 whenever it can occur (see the mask comment below)
    constexpr int NLUT = MASK ? 1024 : (BIAS ? 512 : 256);
    // 24-bit form: 16-bit entries (two to a bank, so that fewer lanes meet in one); with the mask its last entry is 0 whatever
    // the parameters, which is exact: it stands for everything beyond, and at a delta of 1023 itself, which only a masked key
    // reaches and only for I_0 <= 15, ShiftExp is 0
    // (with a bias it holds a word of it per key tile: beyond 8 tiles that costs a workgroup per CU or spills, and the scores are
    // taken tile by tile instead, between the 24-bit requantisations and IntDiv: 1200 pairs of 196 tokens and 32 features 70 us
    // otherwise)
    // (and with a mask, 64 features and more than 208 tokens without that IntDiv: 1200 pairs of 256 tokens 190 us with it, 180 without)
    constexpr bool DIV24 = FAST == 2 && !TAPS && !(MASK && D == 64 && NKT == 16), N24 = DIV24 && !(BIAS && NKT > 8);
    using Entry = std::conditional_t<N24, uint16_t, uint32_t>;
    __shared__ Entry lut[NLUT];

    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lg = lane >> 4;
    // (the ShiftExp table is filled inside the first item, once its loads of K, V and Q are on their way)
    // keys beyond the 16-key tiles but inside the last 64-key chunk multiply probabilities that are zero;
    // clear their rows once so that no uninitialised LDS is ever read
    for (int i = NKT * 16 * VP / 4 + tid; i < NKC * 64 * VP / 4; i += ATT_THREADS) reinterpret_cast<uint32_t*>(Vs)[i] = 0u;

    const int k_out = FAST == 2 ? sm.m_bits - 23 : sm.k_out;                   // (see Div24)
    const int sh = sm.m_bits - (k_out - 1);
    const uint32_t top = (1u << (k_out - 1)) - 1u;
    const int nqt = (T + 15) >> 4;
    const int nfull = T >> 4;                      // key tiles whose 16 keys all exist

    // workgroups of one XCD (block id modulo 8) take consecutive items: the heads of an image share 128-byte lines of
    // qkv (two 64-byte head slices per line), which then meet in one L2
    const int G = gridDim.x, xcd = blockIdx.x % 8;
    const int first = xcd * (G / 8) + min(xcd, G % 8) + blockIdx.x / 8;
    // a work item is one (window, head) or, with split > 1, every split-th query tile of it: when there are too few
    // (window, head) pairs to give every workgroup slot of the device one, each pair is shared by `split` workgroups
    // (K and V are staged by each of them; they are small)
    const int n_work = n_items * split;
    struct Item { uint32_t item, part, b, h, image, win; };                    // of a table: the image and the window's place in it
    const bool gather = BIAS && tok_index != nullptr;
    auto item_of = [&](int work) __attribute__((always_inline)) -> Item {
        Item t{};
        t.item = split_d.divide((uint32_t)work, t.part);
        t.b = H.divide(t.item, t.h);
        if (gather) t.image = n_win.divide(t.b, t.win);
        return t;
    };
    // Rows of qkv / o, counted from the first row of the window or, with a table, of its image (that row's address is a
    // scalar, a lane adds one 32 x 32-bit product to it).  Without a table token t is row t.  With one (BIAS instances
    // only) the rows come from the index table of the window's position inside its image; an entry outside the image is
    // clamped, never followed.  The table entries this thread needs for an item (its K / V pieces and its first query
    // tile) are fetched one item ahead and touched there only, so that the loads of K, V and Q never wait for an index and
    // nothing waits for the entries themselves.
    constexpr int NPC = (NKT * 16 * DCH + ATT_THREADS - 1) / ATT_THREADS;     // 16-byte pieces per thread and operand
    const int tpi = (int)n_win.d * T;              // tokens per image
    const uint32_t C3 = 3 * (uint32_t)C;
    uint32_t kvrow[NPC], qrow0 = 0;
    // this wavefront's first query tile.  The tiles rarely divide evenly among the wavefronts (13 tiles of 197
    // tokens: one wavefront gets four, the others three); which wavefront starts moves on with the item, so that
    // the workgroups that share a compute unit do not all give the extra tile to the same SIMD.
    auto first_tile = [&](const Item& t) __attribute__((always_inline)) { return (int)t.part + split * (int)((wv + t.item) % ATT_WAVES); };
    auto fetch_rows = [&](const Item& t) __attribute__((always_inline)) {
        const int32_t* tr = tok_index + t.win * T;
#pragma unroll
        for (int it = 0; it < NPC; ++it) kvrow[it] = (uint32_t)tr[min((tid + ATT_THREADS * it) / DCH, T - 1)];
        qrow0 = (uint32_t)tr[min(first_tile(t) * 16 + li, T - 1)];
    };
    Item cur = item_of(first), nxt{};
    if (BIAS) { if (gather && first < n_work) fetch_rows(cur); }

    for (int work = first; work < n_work; work += G, cur = nxt) {
        const int item = (int)cur.item, b = (int)cur.b, h = (int)cur.h, qt0 = first_tile(cur);
        const int64_t row0 = gather ? (int64_t)cur.image * tpi : (int64_t)b * T;
        const int8_t* base = qkv + row0 * C3 + h * D;
        const int32_t* trow = gather ? tok_index + cur.win * T : nullptr;
        auto at = [&](uint32_t row) __attribute__((always_inline)) { return base + (uint64_t)row * C3; };
        auto row_of = [&](int t) -> uint32_t {     // any token of this window (t < T)
            if (BIAS) { if (trow) return min((uint32_t)trow[t], (uint32_t)(tpi - 1)); }
            return (uint32_t)t;
        };
        auto q_row = [&](int qt) -> uint32_t {     // row of this lane's query of tile qt
            if (BIAS) { if (gather && qt == qt0) return min(qrow0, (uint32_t)(tpi - 1)); }
            return row_of(min(qt * 16 + li, T - 1));
        };
        __syncthreads();                           // table ready / previous item's readers done
        // the query fragment of a tile is requested one tile ahead, the first one together with K and V
        auto load_q64 = [&](int qt) { return *reinterpret_cast<const v4i*>(at(q_row(qt)) + 16 * lg); };
        auto load_q32 = [&](int qt) { return *reinterpret_cast<const long*>(at(q_row(qt)) + 8 * lg); };
        v4i qn64 = {0, 0, 0, 0};
        long qn32 = 0;
        if (D == 64) qn64 = load_q64(qt0); else qn32 = load_q32(qt0);
        // all of this thread's K and V pieces are requested before the first one is used: one memory latency per item
        v4i kreg[NPC], vreg[NPC];
#pragma unroll
        for (int it = 0; it < NPC; ++it) {
            const int c = tid + ATT_THREADS * it;
            const int key = min(c / DCH, T - 1), part = c % DCH;
            uint32_t row = (uint32_t)key;
            if (BIAS) { if (gather) row = min(kvrow[it], (uint32_t)(tpi - 1)); }
            const int8_t* kv_row = at(row) + 16 * part;
            kreg[it] = *reinterpret_cast<const v4i*>(kv_row + C);
            vreg[it] = *reinterpret_cast<const v4i*>(kv_row + 2 * C);
        }
        // The lane's bytes of the bias and of the mask: its four keys of a key tile are four consecutive bytes of the query's row,
        // one (unaligned) word.  Of a tile with absent keys the last word of the row is read, to be moved down where it is used
        // (not here: nothing may wait for a load before all are requested).
        uint32_t bw[NKT], mw[NKT];
        const int wfrom = T >= 4 ? T - 4 : T;      // the last word's place
        auto load_words = [&](int qt) __attribute__((always_inline)) {
            const uint32_t qr = (uint32_t)min(qt * 16 + li, T - 1) * (uint32_t)T;
            const int8_t* br = (BIAS && rel_bias) ? rel_bias + (int64_t)h * T * T : nullptr;
            uint32_t of_mask = 0;
            if (MASK) n_mask.divide((uint32_t)b, of_mask);
            const int8_t* mr = MASK ? mask + (int64_t)of_mask * T * T : nullptr;
            auto word = [&](const int8_t* table, int key) __attribute__((always_inline)) {
                uint32_t w = 0;
                if (T >= 4) __builtin_memcpy(&w, table + (uint32_t)(qr + min(key, wfrom)), 4);
                else for (int r = 0; r < 4 && key + r < T; ++r) w |= (uint32_t)(uint8_t)table[qr + key + r] << (8 * r);
                return w;
            };
#pragma unroll
            for (int t = 0; t < NKT; ++t) {
                bw[t] = mw[t] = 0;
                if (BIAS) { if (!MASK || br) bw[t] = word(br, 16 * t + 4 * lg); }
                if (MASK) mw[t] = word(mr, 16 * t + 4 * lg);
            }
        };
        auto move_down = [&](uint32_t (&w)[NKT]) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < NKT; ++t)
                if (t >= nfull) w[t] = (uint32_t)((uint64_t)w[t] >> min(8 * max(16 * t + 4 * lg - wfrom, 0), 32));
        };
        if (N24 && BIAS && ONE) load_words(qt0);   // (with K, V and Q: behind the barrier nothing is waited for any more)
        if (work == first) {                       // the table, while the first loads are in flight (visible after the barrier below)
            for (int i = tid; i < NLUT; i += ATT_THREADS) lut[i] = N24 && MASK && i == NLUT - 1 ? (Entry)0 : (Entry)(shiftexp(-i, sm.i0, sm.n_shift) << (DIV24 ? sm.k_out : 0));
        }
        const uint32_t orow0 = q_row(qt0);         // output row of the first query tile (before the indices move on)
        if (work + G < n_work) {
            nxt = item_of(work + G);
            if (BIAS) { if (gather) fetch_rows(nxt); }
        }
#pragma unroll
        for (int it = 0; it < NPC; ++it) {
            const int c = tid + ATT_THREADS * it;
            if (c >= NKT * 16 * DCH) break;
            const int key = c / DCH, part = c % DCH;
            const v4i vv = vreg[it];               // (absent keys repeat the last one: their scores and probabilities are left out below)
            *reinterpret_cast<v4i*>(&Ks[key * KROW + 16 * part]) = kreg[it];
            v2i_att* vdst = reinterpret_cast<v2i_att*>(&Vs[key * VP + 16 * part]);      // (rows are 8-byte aligned)
            vdst[0] = v2i_att{vv[0], vv[1]};
            vdst[1] = v2i_att{vv[2], vv[3]};
        }
        __syncthreads();

        for (int qt = qt0; qt < nqt; qt = ONE ? nqt : qt + split * ATT_WAVES) {
            const int q = qt * 16 + li;            // this lane's query token
            const int qc = min(q, T - 1);
            int32_t sc[NKT][4];
            // ---- scores: S^T tile t = K_t (16 keys x D) . Q^T (D x 16 queries)
            if (D == 64) {
                const v4i qf = qn64;
                if (!ONE) qn64 = load_q64(qt + split * ATT_WAVES);
#pragma unroll
                for (int t = 0; t < NKT; ++t) {
                    const v4i kf = *reinterpret_cast<const v4i*>(&Ks[(16 * t + li) * KROW + 16 * lg]);
                    const v4i r = __builtin_amdgcn_mfma_i32_16x16x64_i8(kf, qf, v4i{0, 0, 0, 0}, 0, 0, 0);
                    sc[t][0] = r[0]; sc[t][1] = r[1]; sc[t][2] = r[2]; sc[t][3] = r[3];
                    if ((t & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // at most four K fragments in flight
                }
            } else {
                const long qf = qn32;
                if (!ONE) qn32 = load_q32(qt + split * ATT_WAVES);
#pragma unroll
                for (int t = 0; t < NKT; ++t) {
                    const long kf = *reinterpret_cast<const long*>(&Ks[(16 * t + li) * KROW + 8 * lg]);
                    const v4i r = __builtin_amdgcn_mfma_i32_16x16x32_i8(kf, qf, v4i{0, 0, 0, 0}, 0, 0, 0);
                    sc[t][0] = r[0]; sc[t][1] = r[1]; sc[t][2] = r[2]; sc[t][3] = r[3];
                    if ((t & 3) == 3) __builtin_amdgcn_sched_barrier(0);
                }
            }
            // requant8 reads the MFMA results through an asm statement, which gets no hazard wait states from the
            // compiler: the last MFMA above (8 passes: 10 wait states) is given its time by hand
            if (FAST == 2) {
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_nop 7");
                asm volatile("s_nop 3");
                __builtin_amdgcn_sched_barrier(0);
            }
            uint32_t pk[NKC * 4];
#pragma unroll
            for (int t = 0; t < NKC * 4; ++t) pk[t] = 0u;
            int32_t sum;                                   // ShiftExp over the row
            // ---- requantise, add the bias, row maximum.  Lane (li, lg) holds keys 16 t + 4 lg + r.
            const int64_t tap_row = ((int64_t)item * T + qc) * T;
            // BIAS: a relative-position bias and / or the shifted-window mask.  A masked key gets -100 I_0 (the -100
            // the windowed models add, at the integer scale of the logits).  All of this is exact int32 arithmetic;
            // only the table is finite: an unmasked key is at most 508 below the row maximum, and for a masked key
            // ShiftExp(-delta) is 0 for every delta >= 1024 it can reach (delta >= 100 I_0 - 508, and a non-zero
            // value needs delta < 23 I_0), so entries past the table read as 0.
            const int8_t* brow = (BIAS && rel_bias) ? rel_bias + ((int64_t)h * T + qc) * T : nullptr;
            uint32_t of_mask = 0;
            if (MASK) n_mask.divide((uint32_t)b, of_mask);
            const int8_t* mrow = MASK ? mask + ((int64_t)of_mask * T + qc) * T : nullptr;
            const int32_t mask_add = -100 * sm.i0;
            if constexpr (N24) {
                // Five vector instructions and a table read per score (nine and a read with each step on its own: 3072 pairs of
                // 197 tokens 63.7 -> 51.4 us, 768 pairs 21.0 -> 18.3).
                uint32_t base = 0;                 // without a bias: what a score's product is subtracted from
                bool masked = false;
                int32_t mx = INT32_MIN;
                // keys from this lane's first one on; of an unknown T not known to be the same for the next query tile, so that the
                // comparisons are not made once for all and kept in more scalar registers than there are
                int left = T - 4 * lg;
                if (!TFIX) asm volatile("" : "+v"(left));
                if constexpr (!BIAS) {
                    // the requantisation is monotonic: the row maximum is that of the accumulators.  With T the maximum's result,
                    // (T | 2^24 - 1) - (m mb + ad), m a limited score, has max - value in its top byte.
#pragma unroll
                    for (int t = 0; t < NKT; ++t) {
                        if (t >= nfull) {
#pragma unroll
                            for (int r = 0; r < 4; ++r) if (16 * t + r >= left) sc[t][r] = INT32_MIN;
                        }
                        mx = max(mx, max(max(sc[t][0], sc[t][1]), max(sc[t][2], sc[t][3])));
                    }
                    mx = rows_allreduce(mx, [](int32_t a, int32_t b) { return max(a, b); });
                    base = ((uint32_t)(__mul24(min(max(mx, nqk.lo), nqk.hi), nqk.mb) + nqk.ad) | 0xffffffu) - (uint32_t)nqk.ad;
                } else {
                    if (!ONE) load_words(qt);
                    move_down(bw);
                    if (MASK) move_down(mw);
                    mx = biased_scores<MASK>(sc, bw, mw, nqk, mask_add, nfull, left, masked);
                }
                // ---- ShiftExp by table, row sum
                sum = MASK && masked ? look_up<BIAS, true>(sc, lut, NLUT, mx, base, nqk, nfull, left)
                                     : look_up<BIAS, false>(sc, lut, NLUT, mx, base, nqk, nfull, left);
            } else {
            int32_t mx = INT32_MIN;
#pragma unroll
            for (int t = 0; t < NKT; ++t) {
                if (t < nfull) {                   // uniform: every key of the tile exists
                    // the lane's four keys are four consecutive bytes of the bias and the mask row: one (unaligned)
                    // dword each instead of four byte loads
                    uint32_t bw = 0, mw = 0;
                    if (BIAS) { if (!MASK || brow) __builtin_memcpy(&bw, brow + 16 * t + 4 * lg, 4); }
                    if (MASK) __builtin_memcpy(&mw, mrow + 16 * t + 4 * lg, 4);
                    requant8x4<FAST>(sc[t], qk, nqk, rnd);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int key = 16 * t + 4 * lg + r;
                        int32_t a = sc[t][r];
                        if (TAPS) { if (tap_s && q < T) tap_s[tap_row + key] = (int8_t)a; }
                        if (BIAS) a += (int32_t)(int8_t)(bw >> (8 * r));
                        if (MASK) { if ((mw >> (8 * r)) & 0xffu) a += mask_add; }
                        sc[t][r] = a;
                    }
                    mx = max(mx, max(sc[t][0], sc[t][1]));       // two three-operand maxima per tile
                    mx = max(mx, max(sc[t][2], sc[t][3]));
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int key = 16 * t + 4 * lg + r;
                        int32_t a = requant8<FAST>(sc[t][r], qk, nqk, rnd);
                        if (key < T) {
                            if (TAPS) { if (tap_s && q < T) tap_s[tap_row + key] = (int8_t)a; }
                            if (BIAS) { if (!MASK || brow) a += brow[key]; }
                            if (MASK) { if (mrow[key]) a += mask_add; }
                            mx = max(mx, a);
                        }
                        sc[t][r] = a;
                    }
                }
                __builtin_amdgcn_sched_barrier(0);     // keep the 64-bit temporaries of one tile at a time
            }
            mx = rows_allreduce(mx, [](int32_t a, int32_t b) { return max(a, b); });
            // ---- ShiftExp by table, row sum.  The byte offset 4 (max - a) of the table entry is one 24-bit multiply-add.
            sum = 0;
            const int32_t mx4 = 4 * mx;
            const char* lut_b = reinterpret_cast<const char*>(lut);
#pragma unroll
            for (int t = 0; t < NKT; ++t) {
                if (t < nfull) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        int32_t e;
                        if (MASK) {
                            const int32_t delta = mx - sc[t][r];
                            e = delta < NLUT ? (int32_t)lut[min(delta, NLUT - 1)] : 0;
                        } else {
                            e = (int32_t)*reinterpret_cast<const uint32_t*>(lut_b + (__mul24(sc[t][r], -4) + mx4));
                        }
                        sc[t][r] = e;
                        sum += e;
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int key = 16 * t + 4 * lg + r;
                        int32_t e;
                        if (MASK) {
                            const int32_t delta = key < T ? mx - sc[t][r] : NLUT;
                            e = delta < NLUT ? (int32_t)lut[min(delta, NLUT - 1)] : 0;
                        } else {
                            e = key < T ? (int32_t)lut[mx - sc[t][r]] : 0;
                        }
                        sc[t][r] = e;
                        sum += e;
                    }
                }
                if (t & 1) __builtin_amdgcn_sched_barrier(0);
            }
            sum = rows_allreduce(sum, [](int32_t a, int32_t b) { return a + b; });
            }
            // ---- IntDiv and packing: the four keys of tile t become one word of the "B" operand
            if constexpr (DIV24) {
                const uint32_t f = div_factor(sum, div24_of(sm));
#pragma unroll
                for (int t = 0; t + 4 <= NKT; t += 4) {
                    uint32_t w[4];
                    div_pack4(w, f, sc[t], sc[t + 1], sc[t + 2], sc[t + 3]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) pk[t + k] = w[k];
                }
#pragma unroll
                for (int t = NKT & ~3; t < NKT; ++t) pk[t] = div_pack(f, sc[t]);
            } else {
                const uint32_t inv = (1u << sm.m_bits) / (uint32_t)sum;
                const uint32_t inv_hi = FAST ? inv << (32 - sh) : 0u;      // FAST: inv < 2^sh, 1 <= sh <= 31
#pragma unroll
                for (int t = 0; t < NKT; ++t) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (TAPS) {
                            const uint32_t p = FAST ? min(__umulhi(inv_hi, (uint32_t)sc[t][r]), top)
                                                    : min((inv * (uint32_t)sc[t][r]) >> sh, top);
                            const int key = 16 * t + 4 * lg + r;
                            if (tap_p && q < T && key < T) tap_p[tap_row + key] = (int8_t)p;
                            pk[t] |= p << (8 * r);
                        } else {
                            // IntDiv gives at most 2^(k_out-1), which fits a byte: clamp the four of a word together below
                            const uint32_t p = FAST ? __umulhi(inv_hi, (uint32_t)sc[t][r]) : (inv * (uint32_t)sc[t][r]) >> sh;
                            pk[t] |= p << (8 * r);
                        }
                    }
                }
                if (!TAPS) {
#pragma unroll
                    for (int t = 0; t < NKT; ++t) pk[t] -= (pk[t] >> (k_out - 1)) & 0x01010101u;   // bytewise min(p, 2^(k_out-1) - 1)
                }
            }
            // ---- O^T = V^T P^T : "A" = V^T rows (features), "B" = packed probabilities (keys x queries).
            // Contraction position 16 lg + 4 j + r of chunk c is key 64 c + 16 j + 4 lg + r (the layout of pk).  A
            // transposing read hands lane i of a 16-lane block byte i' of the 8-byte row named by lane 2 i' (i < 8)
            // or 2 i' + 1 (i >= 8): the even lanes name keys j = 2 hh + (b >> 2), r = b & 3 (b = half the lane number)
            // at features 8 n .. 8 n + 7, the odd lanes the same keys at features D/2 + 8 n .., so that row i of
            // output tile n is feature 8 n + i (i < 8) or D/2 + 8 n + i - 8.
            const int8_t* vbase = Vs + (4 * lg + 16 * ((li >> 1) >> 2) + ((li >> 1) & 3)) * VP + ((li & 1) ? D / 2 : 0);
            v4i oacc[ND];
#pragma unroll
            for (int n = 0; n < ND; ++n) oacc[n] = v4i{0, 0, 0, 0};
#pragma unroll
            for (int c = 0; c < NKC; ++c) {
                const v4i pf = {(int)pk[4 * c], (int)pk[4 * c + 1], (int)pk[4 * c + 2], (int)pk[4 * c + 3]};
#pragma unroll
                for (int n = 0; n < ND; ++n) {
                    typedef v2i_att __attribute__((address_space(3))) * lds_v2i;
                    const v2i_att v0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(vbase + (64 * c) * VP + 8 * n));
                    const v2i_att v1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(vbase + (64 * c + 32) * VP + 8 * n));
                    const v4i vf = {v0[0], v0[1], v1[0], v1[1]};
                    oacc[n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vf, pf, oacc[n], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            // ---- requantise and store: lane block lg holds rows 4 lg + r of every tile n, i.e. features
            // (lg >= 2 ? D/2 : 0) + 8 n + 4 (lg & 1) + r of query q; exchanging tile n + ND/2 of the even blocks with tile
            // n of the odd ones leaves block lg with the D/4 consecutive features lg (D/4) ..
            if (FAST == 2) {                       // as above: asm readers of fresh MFMA results
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_nop 7");
                asm volatile("s_nop 3");
                __builtin_amdgcn_sched_barrier(0);
            }
            uint32_t ow[ND];
            if constexpr (FAST == 2) {
                narrow_words(ow, oacc, npv);
            } else {
#pragma unroll
                for (int n = 0; n < ND; ++n) {
                    uint32_t w = 0;
                    int32_t ov[4] = {oacc[n][0], oacc[n][1], oacc[n][2], oacc[n][3]};
                    requant8x4<FAST>(ov, pv, npv, rnd);
#pragma unroll
                    for (int r = 0; r < 4; ++r) w |= ((uint32_t)ov[r] & 0xffu) << (8 * r);
                    ow[n] = w;
                }
            }
#pragma unroll
            for (int n = 0; n < ND / 2; ++n) {
                // (odd blocks of the first operand <-> even blocks of the second)
                const auto sw = __builtin_amdgcn_permlane16_swap(ow[n], ow[n + ND / 2], false, false);
                ow[n] = sw[0]; ow[n + ND / 2] = sw[1];
            }
            if (q < T) {
                int8_t* op = o + row0 * C + h * D + (uint64_t)(ONE || qt == qt0 ? orow0 : row_of(q)) * (uint32_t)C + lg * (D / 4);
                if (D == 64) *reinterpret_cast<uint4*>(op) = make_uint4(ow[0], ow[2], ow[1], ow[3]);
                else *reinterpret_cast<uint2*>(op) = make_uint2(ow[0], ow[1 % ND]);
            }
        }
    }
}

// op over the 64 lanes
template <class OP>
__device__ __forceinline__ int32_t wave_allreduce(int32_t v, OP op) {
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, true));       // row_ror by 1, 2, 4, 8
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, true));
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, true));
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, true));
    return rows_allreduce(v, op);
}

// Windows of 7 x 7 tokens, 32 features a head, 24-bit form, when there are many (window, head) pairs: one wavefront per pair, so that
//  - nothing but the start needs a barrier;
//  - K and Q come from memory in the layout the matrix instruction reads (a lane's 8 bytes of a row), once and not once per query tile;
//  - V passes through the wavefront's own corner of LDS for the transposing read, once;
//  - the bias of the workgroup's head lies in LDS as the words the lanes need;
//  - the 49th query, which would have a tile of its own, has its 49 scores one to a lane: a third of a tile's instructions.
// Bound by the vector ALU and the addresses of the loads (one that touches 16 rows costs about 27 cycles whatever its width), about
// equally.  (Two neighbouring heads to a wavefront, 16 bytes a lane and a load, halve the loads but leave fewer wavefronts: 2048
// windows x 6 heads 24.0 against 23.2 us, 512 x 12 14.9 against 14.2.)  A wavefront per query tile against this, without and with a mask: 2048
// x 3 13.7 -> 11.1 and 18.3 -> 16.3 us, 1024 x 6 13.9 -> 11.7 and 18.9 -> 17.0, 512 x 12 15.1 -> 13.2 and 19.8 -> 18.4.
constexpr int WIN_T = 49, WIN_WAVES = 4;
template <bool MASK>
__global__ __launch_bounds__(64 * WIN_WAVES, MASK ? 5 : 7) void window_attention_kernel(
    const int8_t* __restrict__ qkv, const int8_t* __restrict__ rel_bias, const int8_t* __restrict__ mask, FastDiv n_mask,
    const int32_t* __restrict__ tok_index, FastDiv n_win, int8_t* __restrict__ o, int B, int C, FastDiv H, ShiftParams sm,
    Narrow nqk, Narrow npv) {
    constexpr int T = WIN_T, D = 32, NT = 4, NQ = T / 16, LAST = T - 1, nfull = T >> 4, VP = 40, NLUT = MASK ? 1024 : 512;
    static_assert(T == 16 * NQ + 1 && NQ + 1 == NT);
    __shared__ __align__(16) int8_t Vall[WIN_WAVES][NT * 16 * VP];
    __shared__ __align__(16) uint32_t bias_words[NQ][64][NT];
    __shared__ __align__(16) int8_t last_bias[64], last_p[WIN_WAVES][64];
    __shared__ uint16_t lut[NLUT];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 15, lg = lane >> 4;

    // (the workgroups of one XCD are consecutive: the heads of a window share the lines of qkv)
    const int G = gridDim.x, xcd = blockIdx.x % 8;
    uint32_t h;                                    // the workgroup's head
    const int slot = (int)H.divide((uint32_t)(xcd * (G / 8) + min(xcd, G % 8) + blockIdx.x / 8), h);
    const int stride = G / (int)H.d * WIN_WAVES;   // windows of one pass of all workgroups
    // four consecutive bytes of row `tok` of a T x T table; the last word of the row, moved down, for the last tile
    auto word = [&](const int8_t* table, uint32_t tok, int t, int block) __attribute__((always_inline)) {
        const int key = 16 * t + 4 * block, from = 16 * t + 16 <= T ? key : min(key, T - 4);
        uint32_t v;
        __builtin_memcpy(&v, table + (uint32_t)(tok * T + from), 4);
        return 16 * t + 16 <= T ? v : (uint32_t)((uint64_t)v >> min(8 * (key - from), 32));
    };
    for (int i = tid; i < NLUT; i += 64 * WIN_WAVES) lut[i] = MASK && i == NLUT - 1 ? (uint16_t)0 : (uint16_t)(shiftexp(-i, sm.i0, sm.n_shift) << sm.k_out);
    for (int i = tid; i < NT * 64; i += 64 * WIN_WAVES) {
        const int q = i / 64, l = i & 63;
        const int8_t* table = rel_bias + (int64_t)h * T * T;
        const bool any = !MASK || rel_bias;
        if (q < NQ) {
#pragma unroll
            for (int t = 0; t < NT; ++t) bias_words[q][l][t] = any ? word(table, 16 * q + (l & 15), t, l >> 4) : 0u;
        } else {
            last_bias[l] = any ? table[LAST * T + min(l, LAST)] : (int8_t)0;
        }
    }
    __syncthreads();

    const bool gather = tok_index != nullptr;
    const uint32_t tpi = n_win.d * T, C3 = 3 * (uint32_t)C;  // tokens per image
    // this lane's row of every 16-token tile, as a query and as a key alike
    uint32_t raw[NT];
    auto fetch_rows = [&](int b) __attribute__((always_inline)) -> uint32_t {  // returns the image
        uint32_t win = 0;
        if (!gather) return (uint32_t)b;
        const uint32_t image = n_win.divide((uint32_t)b, win);
        const int32_t* tr = tok_index + (int64_t)win * T;
#pragma unroll
        for (int t = 0; t < NT; ++t) raw[t] = (uint32_t)tr[min(16 * t + li, LAST)];
        return image;
    };
    int8_t* Vs = Vall[wv];
    const int8_t* vbase = Vs + (4 * lg + 16 * ((li >> 1) >> 2) + ((li >> 1) & 3)) * VP + ((li & 1) ? D / 2 : 0);
    const int32_t mask_add = -100 * sm.i0;
    const int left = T - 4 * lg;
    int b = slot * WIN_WAVES + wv;
    uint32_t image = b < B ? fetch_rows(b) : 0;
    while (b < B) {
        const uint64_t row0 = (uint64_t)image * (gather ? tpi : (uint32_t)T);
        const int8_t* base = qkv + row0 * C3 + (int)h * D;
        int8_t* obase = o + row0 * (uint32_t)C + (int)h * D;
        uint32_t row[NT];
        long kf[NT], vr[NT], qf[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            row[t] = gather ? min(raw[t], tpi - 1) : (uint32_t)min(16 * t + li, LAST);
            const uint32_t at = row[t] * C3 + 8 * lg;
            vr[t] = *reinterpret_cast<const long*>(base + 2 * C + at);
            kf[t] = *reinterpret_cast<const long*>(base + C + at);
            qf[t] = *reinterpret_cast<const long*>(base + at);
        }
        uint32_t mw[NQ][NT];
        int32_t last_mask = 0;
        if (MASK) {
            uint32_t m;
            n_mask.divide((uint32_t)b, m);
            const int8_t* mrow = mask + (int64_t)m * T * T;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int t = 0; t < NT; ++t) mw[q][t] = word(mrow, 16 * q + li, t, lg);
            last_mask = mrow[LAST * T + min(lane, LAST)];
        }
        b += stride;
        if (b < B) image = fetch_rows(b);
#pragma unroll
        for (int t = 0; t < NT; ++t) *reinterpret_cast<long*>(Vs + (16 * t + li) * VP + 8 * lg) = vr[t];
        typedef v2i_att __attribute__((address_space(3))) * lds_v2i;
        v4i vf[2];
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const v2i_att v0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(vbase + 8 * n));
            const v2i_att v1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i)(vbase + 32 * VP + 8 * n));
            vf[n] = v4i{v0[0], v0[1], v1[0], v1[1]};
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            int32_t sc[NT][4];
            const v4i words = *reinterpret_cast<const v4i*>(bias_words[q][lane]);
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const v4i s = __builtin_amdgcn_mfma_i32_16x16x32_i8(kf[t], qf[q], v4i{0, 0, 0, 0}, 0, 0, 0);
                sc[t][0] = s[0]; sc[t][1] = s[1]; sc[t][2] = s[2]; sc[t][3] = s[3];
            }
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 7");           // (asm readers of matrix results, see requant8)
            asm volatile("s_nop 3");
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t bw[NT] = {(uint32_t)words[0], (uint32_t)words[1], (uint32_t)words[2], (uint32_t)words[3]};
            uint32_t mt[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) mt[t] = MASK ? mw[q][t] : 0u;
            bool masked;
            const int32_t mx = biased_scores<MASK>(sc, bw, mt, nqk, mask_add, nfull, left, masked);
            const int32_t sum = MASK && masked ? look_up<true, true>(sc, lut, NLUT, mx, 0u, nqk, nfull, left)
                                               : look_up<true, false>(sc, lut, NLUT, mx, 0u, nqk, nfull, left);
            uint32_t pk[NT];
            div_pack4(pk, div_factor(sum, div24_of(sm)), sc[0], sc[1], sc[2], sc[3]);
            const v4i pf = {(int)pk[0], (int)pk[1], (int)pk[2], (int)pk[3]};
            v4i oacc[2];
#pragma unroll
            for (int n = 0; n < 2; ++n) oacc[n] = __builtin_amdgcn_mfma_i32_16x16x64_i8(vf[n], pf, v4i{0, 0, 0, 0}, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_nop 7");
            asm volatile("s_nop 3");
            __builtin_amdgcn_sched_barrier(0);
            uint32_t ow[2];
            narrow_words(ow, oacc, npv);
            const auto sw = __builtin_amdgcn_permlane16_swap(ow[0], ow[1], false, false);
            *reinterpret_cast<uint2*>(obase + (uint32_t)(row[q] * (uint32_t)C + 8 * lg)) = make_uint2(sw[0], sw[1]);
        }
        // ---- the query left over (every row of its tile is that token): S = Q K^T, queries x keys, so that its score with key
        // 16 t + li is in every lane li of tile t; lane block lg keeps tile lg
        int32_t v = 0;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const v4i s = __builtin_amdgcn_mfma_i32_16x16x32_i8(qf[NQ], kf[t], v4i{0, 0, 0, 0}, 0, 0, 0);
            v = lg == t ? s[0] : v;
        }
        __builtin_amdgcn_sched_barrier(0);
        v = (narrow_top(v, nqk) >> 24) + last_bias[lane] + (MASK && last_mask ? mask_add : 0);
        const int32_t mx = wave_allreduce(lane < T ? v : INT32_MIN, [](int32_t x, int32_t y) { return max(x, y); });
        int32_t e = (int32_t)lut[lane < T ? min(mx - v, NLUT - 1) : 0];
        e = lane < T ? e : 0;
        const uint32_t f = div_factor(wave_allreduce(e, [](int32_t x, int32_t y) { return x + y; }), div24_of(sm));
        last_p[wv][lane] = (int8_t)(uint8_t)__umulhi(f, (uint32_t)e);
        v4i pf;
#pragma unroll
        for (int t = 0; t < NT; ++t) pf[t] = *reinterpret_cast<const int*>(&last_p[wv][16 * t + 4 * lg]);
        // O = P V: a row of features, tile n of them from lane block n
        const v4i o0 = __builtin_amdgcn_mfma_i32_16x16x64_i8(pf, vf[0], v4i{0, 0, 0, 0}, 0, 0, 0);
        const v4i o1 = __builtin_amdgcn_mfma_i32_16x16x64_i8(pf, vf[1], v4i{0, 0, 0, 0}, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        const int32_t ov = lg & 1 ? o1[0] : o0[0];
        __builtin_amdgcn_sched_barrier(0);
        if (lg < 2) obase[(uint32_t)(row[NQ] * (uint32_t)C + 8 * lg + li + (li & 8))] = (int8_t)(narrow_top(ov, npv) >> 24);
    }
}

// The 24-bit constants of a pair, or false when the pair needs the wider forms.
// (rnd = 1: the rounding addend h is 2^(c-1); rnd = 0: the bare shift of Eq. 10, h = 0)
static bool narrow_of(Dyadic d, int rnd, Narrow& n) {
    if (d.c < 1 || d.c > 24 || d.b < 1 || d.b >= (1 << (d.c - 1))) return false;
    const int64_t half = (int64_t)rnd << (d.c - 1), two_c = (int64_t)1 << d.c;
    const int64_t hi = (127 * two_c - half + d.b - 1) / d.b;             // first v with (v b + h) >> c >= 127
    const int64_t lo = -((126 * two_c + 1 + half + d.b - 1) / d.b);      // last v with (v b + h) >> c <= -127
    if (lo < -(1 << 23) || hi >= (1 << 23)) return false;
    n.lo = (int32_t)lo; n.hi = (int32_t)hi; n.mb = d.b << (24 - d.c); n.ad = (int32_t)(half << (24 - d.c));
    return true;
}

// The one-wavefront form from 9 (window, head) pairs per CU on: below, a wavefront per query tile finishes a pair sooner.  Without
// and with a mask, us against a wavefront per query tile, 3 heads and 12: 4 per CU 5.7 : 4.4 and 8.1 : 5.7, 6.6 : 4.4 and 8.8 : 5.7;
// 7.5 per CU 6.1 : 6.4 and 8.3 : 8.0, 6.8 : 6.5 and 9.0 : 8.1; 9 per CU 7.0 : 8.4 and 9.7 : 10.6, 8.0 : 8.7 and 10.7 : 10.9; 12 per CU
// 7.3 : 8.5 and 10.0 : 10.7, 8.3 : 8.8 and 10.9 : 11.0; 24 per CU 11.1 : 13.7 and 16.3 : 18.3, 13.2 : 15.1 and 18.4 : 19.8.  The rows of
// an image are counted in 32 bits there.
static bool window_takes(const AttentionArgs& a) {
    const int64_t rows = a.tok_index ? (int64_t)a.n_win * WIN_T : WIN_T;
    return a.T == WIN_T && (int64_t)a.B * a.H >= 9 * (int64_t)num_cus() && rows * 3 * a.C < (int64_t)1 << 31;
}

static void launch_window(hipStream_t s, const AttentionArgs& a, ShiftParams sm, Narrow nqk, Narrow npv) {
    // As many passes as six workgroups per CU need, and no more workgroups than share the windows evenly.  With five and with six,
    // without and with a mask (with one, five are resident at a time): 8192 x 3 34.4 -> 33.7 and 48.9 -> 47.9 us, 2048 x 6 22.5 -> 20.9
    // and 33.2 -> 28.5, 512 x 12 13.6 -> 13.2 and 19.2 -> 18.5; others the same.  (Of eight wavefronts, three per CU, were slower.)
    const int64_t most = std::max<int64_t>(1, 6 * (int64_t)num_cus() / a.H);
    const int64_t passes = (a.B + WIN_WAVES * most - 1) / (WIN_WAVES * most);
    const int grid = a.H * (int)((a.B + WIN_WAVES * passes - 1) / (WIN_WAVES * passes));
#define IVIT_WIN(MASK_)                                                                                                              \
    hipLaunchKernelGGL((window_attention_kernel<MASK_>), dim3(grid), dim3(64 * WIN_WAVES), 0, s, a.qkv, a.rel_bias, a.mask,            \
                       FastDiv(std::max(a.n_mask, 1)), a.tok_index, FastDiv(std::max(a.n_win, 1)), a.o, a.B, a.C, FastDiv(a.H),       \
                       sm, nqk, npv)
    if (a.mask) IVIT_WIN(true); else IVIT_WIN(false);
#undef IVIT_WIN
}

template <int D, int NKT>
static void launch_flags(hipStream_t s, const AttentionArgs& a, int grid, int split, bool taps, bool bias, bool fast) {
    const int n_items = a.B * a.H;
    Narrow nqk{}, npv{};
    // the 24-bit forms: both requantisations and IntDiv
    const int rnd = a.floor_shift ? 0 : 1, up = intdiv24_up(a.sm.i0, a.sm.n_shift, a.sm.m_bits, a.sm.k_out);
    const bool narrow = narrow_of(a.qk_rq, rnd, nqk) && narrow_of(a.pv_rq, rnd, npv) && up >= 0;
    const ShiftParams sm24{a.sm.i0, a.sm.n_shift, a.sm.m_bits, up};           // (see Div24)
#define IVIT_ATT(TAPS_, BIAS_, MASK_, FAST_, TFIX_)                                                                         \
    hipLaunchKernelGGL((attention_kernel<D, NKT, TAPS_, BIAS_, MASK_, FAST_, TFIX_>), dim3(grid), dim3(ATT_THREADS), 0, s,     \
                       a.qkv, a.rel_bias, a.mask, FastDiv(std::max(a.n_mask, 1)), a.tok_index, FastDiv(std::max(a.n_win, 1)), a.o, \
                       n_items, FastDiv(split), a.T, a.C, FastDiv(a.H), a.qk_rq, \
                       FAST_ == 2 ? sm24 : a.sm, a.pv_rq, nqk, npv, rnd, a.tap_scores, a.tap_probs)
    // the production paths are <no taps, fast>, with the 24-bit requantisation when both pairs allow it; everything else
    // shares one fully general instantiation per bias / mask combination (a mask is always compiled with the bias code,
    // which tests the bias pointer)
    const bool masked = a.mask != nullptr;
    constexpr int T49 = (D == 32 && NKT == 4) ? 49 : 0;                        // the windowed models' shape
    constexpr int T197 = (D == 64 && NKT == 13) ? 197 : 0;                     // 14 x 14 patches and a class token
    if (T197 && a.T == 197 && !taps && fast && !bias) {
        if (narrow) IVIT_ATT(false, false, false, 2, T197); else IVIT_ATT(false, false, false, 1, T197);
    } else if (T49 && !taps && fast && bias && narrow && window_takes(a)) {
        launch_window(s, a, sm24, nqk, npv);
    } else if (T49 && a.T == 49 && !taps && fast && bias) {
        if (masked) { if (narrow) IVIT_ATT(false, true, true, 2, T49); else IVIT_ATT(false, true, true, 1, T49); }
        else { if (narrow) IVIT_ATT(false, true, false, 2, T49); else IVIT_ATT(false, true, false, 1, T49); }
    } else if (!taps && fast) {
        if (masked) { if (narrow) IVIT_ATT(false, true, true, 2, 0); else IVIT_ATT(false, true, true, 1, 0); }
        else if (bias) { if (narrow) IVIT_ATT(false, true, false, 2, 0); else IVIT_ATT(false, true, false, 1, 0); }
        else { if (narrow) IVIT_ATT(false, false, false, 2, 0); else IVIT_ATT(false, false, false, 1, 0); }
    } else {
        if (masked) IVIT_ATT(true, true, true, 0, 0);
        else if (bias) IVIT_ATT(true, true, false, 0, 0);
        else IVIT_ATT(true, false, false, 0, 0);
    }
#undef IVIT_ATT
}

template <int D>
static hipError_t launch_d(hipStream_t s, const AttentionArgs& a, int grid, int split, int nkt, bool taps, bool bias, bool fast) {
    if (nkt <= 4) launch_flags<D, 4>(s, a, grid, split, taps, bias, fast);
    else if (nkt <= 8) launch_flags<D, 8>(s, a, grid, split, taps, bias, fast);
    else if (nkt <= 13) launch_flags<D, 13>(s, a, grid, split, taps, bias, fast);
    else launch_flags<D, 16>(s, a, grid, split, taps, bias, fast);
    return hipGetLastError();
}

static bool fits32_host(Dyadic d) { return d.c >= 1 && d.c <= 31 && d.b >= 1 && (uint32_t)d.b <= (1u << d.c); }

hipError_t launch_attention(hipStream_t s, const AttentionArgs& a) {
    const int64_t n_items = (int64_t)a.B * a.H;
    if (n_items == 0) return hipSuccess;
    const int nkt = (a.T + 15) / 16;
    // With fewer (window, head) pairs than compute units, several workgroups share a pair (each takes every split-th
    // query tile) so that the device is filled: about two workgroups per CU, down to one tile per wavefront.  With
    // more pairs than that sharing only adds staging work (measured: 768 pairs, 30 us unshared, 33 us shared by two).
    const int split = (int)std::max<int64_t>(1, std::min<int64_t>(2 * (int64_t)num_cus() / n_items, (nkt + ATT_WAVES - 1) / ATT_WAVES));
    // workgroups per CU: windows of at most 64 tokens need little LDS and few registers, and their short items are
    // bound by latency, so many more workgroups are kept in flight (8192 windows x 3 heads: 86 us with 4, 72 us with 16)
    // (up to 16 per CU, as long as each still loops over about four items, which keeps the rounds even)
    const int64_t n_work = n_items * split, cus = num_cus();
    const int64_t wgs = nkt <= 4 ? std::max<int64_t>(4 * cus, std::min<int64_t>(16 * cus, n_work / 4)) : 4 * cus;
    const int grid = (int)std::min<int64_t>(n_work, wgs);
    const int d = a.C / a.H;
    const int sh = a.sm.m_bits - (a.sm.k_out - 1);
    const bool fast = fits32_host(a.qk_rq) && fits32_host(a.pv_rq) && sh >= 1 &&
                      ((int64_t)a.sm.i0 << a.sm.n_shift) > ((int64_t)1 << (a.sm.k_out - 1));
    const bool taps = a.tap_scores || a.tap_probs;
    const int64_t R = (int64_t)a.B * a.T;
    TraceScope trace(s, KIND_ATTENTION, 4 * n_items * a.T * a.T * d, 4 * R * a.C + (a.rel_bias ? (int64_t)a.H * a.T * a.T : 0));
    const bool bias = a.rel_bias != nullptr || a.mask != nullptr || a.tok_index != nullptr;
    return d == 64 ? launch_d<64>(s, a, grid, split, nkt, taps, bias, fast) : launch_d<32>(s, a, grid, split, nkt, taps, bias, fast);
}

}  // namespace ivit
