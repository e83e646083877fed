// Everything of an encoder block that acts on single tokens, as one kernel (I-ViT, arXiv 2207.01405, Eq. 1-2 and 5 with
// the dyadic pipeline of Sec. 3.2, ShiftGELU of Sec. 3.4 and I-LayerNorm of Sec. 3.5):
//   xhat = Dense(o; proj) + x;  v = LN2(xhat);  y = Dense(ShiftGELU(Dense(v; fc1)); fc2) + xhat;
//   then, for the block that follows, u = LN1'(y) and qkv' = Dense(u)   (or a final LN, or nothing).
// Between two attentions a block is one launch instead of six, and v, the hidden layer and u stay on the chip.  xhat does
// too until it has been normalised; its LDS then goes to the hidden layer, so it is written out once (to the workspace,
// from where the L2 has it) and comes back as the residual of the last layer, during that layer's last products.
//
// A workgroup of four or eight wavefronts (one or two per SIMD) takes M tokens through all layers.  Weights stream through two LDS
// buffers in sets (128 to 192 rows of proj / fc1 / qkv, or 128 bytes of every row of fc2), each requested while its
// predecessor is multiplied; every compute unit reads the same sets at about the same time, from its L2.  Activations
// stand: those of proj, fc1 and qkv in registers as the "A" operand for all k-steps, the hidden layer in chunks of 128
// channels in LDS, fc2's accumulators (M tokens x C channels) in registers through the whole MLP.  A lane holds one
// channel and 16 tokens of a product, so requantisation constants are registers; results turn into token rows through
// wavefront-private LDS with the transposing LDS read.  The LayerNorms work on the token tile in LDS.
//
// What bounds it is the rate at which a wavefront issues instructions (one per 4.5 to 5.5 cycles; a second wavefront on the SIMD
// runs beside it at the same rate: a step of one product, 12 vector, 2 LDS and 4 scalar instructions takes 160 cycles with one
// wavefront and 164 with two).  So the results of a channel tile are requantised between the products of the next one, spread
// evenly, loads are three instructions, and where the tokens of a workgroup divide among eight wavefronts there are eight, which
// leaves 128 registers beside 128 accumulation registers to each: forwards of 197 tokens, four wavefronts against eight, one model again
// and again (three models in turn), DeiT-S batch 64 687 -> 650 us (688 -> 650) and batch 128 1013 -> 946 (1024 -> 970), DeiT-T batch 128
// 615 -> 538 (614 -> 538) and batch 256 1004 -> 845 (1019 -> 863).  Nothing may be spilled: with 29 registers in scratch memory DeiT-S
// batch 128 took 5 % longer (6 %), as stores and reloads wait for the weights in flight and go through HBM (91 -> 108 MB a launch).
#include "token_block_common.hpp"
#include <algorithm>
#include <type_traits>
#include <utility>

namespace ivit {

namespace {

using namespace tokblk;

constexpr int FC = 128;                          // hidden channels per chunk of the MLP

// M = 32 MT tokens, NW wavefronts
template <int C, int MT, int NW>
struct TbLayout {
    static constexpr int KS = C / 32, P = C / 16;                  // k-steps and 16-byte pieces of a row of C bytes
    static constexpr int M = 32 * MT;                              // tokens of a workgroup
    static constexpr int WNG = C / 96, WMG = NW / WNG, TT = MT / WMG;     // wavefront grid of proj / fc2 / qkv, token tiles of a wavefront
    static constexpr int WM1 = WNG != 4 ? WMG : NW == 8 ? MT : MT < 2 ? MT : 2, WN1 = NW / WM1;      // ... of fc1
    static constexpr int T1 = MT / WM1, N1 = 4 / WN1;
    static constexpr int PT = WNG == 4 ? 1 : 3;                    // channel tiles of a wavefront per weight set of proj / qkv
    static constexpr int RS = PT * WNG * 32;                       // weight rows of such a set
    static constexpr int NPROJ = C / RS, NQKV = 3 * C / RS;
    static constexpr int G16 = gcd16(P);
    static constexpr int SETR = RS * C, SET1 = FC * C;             // bytes of a set of proj / qkv, of fc1 and fc2
    static constexpr int SETW = SETR > SET1 ? SETR : SET1;
    static constexpr int CW = (RS > FC ? RS + 63 : FC + 63) / 64;  // wavefronts that fetch the constants of a set's rows, 64 each
    static constexpr int SETB = SETW + 1024 * CW;                  // weights, then those constants
    static constexpr int HP = M + 16, HB = FC * HP;                // hidden chunk [channel][token]
    static constexpr int LUT = 0, SET = 256;                       // the ShiftGELU table lies at address 0: an index is its address
    static constexpr int ACT = SET + 2 * SETB;                     // token tile [row][C], or the two hidden chunks
    static constexpr int ACTB = M * C > 2 * HB ? M * C : 2 * HB;
    static constexpr int LN = ACT + ACTB;                          // gamma, beta
    static constexpr int STG = LN + (8 * C + 1023) / 1024 * 1024, STGB = 32 * 32;      // staging tile of a wavefront: [32 channels][32 tokens]
    static constexpr int SINK = STG + NW * STGB;                   // 256 bytes that nobody reads
    static constexpr int TOTAL = SINK + 256;
    static_assert(C % 96 == 0 && NW % WNG == 0 && MT % WMG == 0 && TT >= 1 && MT % WM1 == 0 && 4 % WN1 == 0, "shape");
    static_assert(C % RS == 0 && SETW >= M * C && (NPROJ == 1 || NPROJ == 3) && NQKV % 2 == 1, "sets");
    static_assert(TOTAL <= 160 * 1024, "LDS");
};

// The constants of up to MAXJ layers: one thread per channel, one row of workgroups per layer.  Prepared by a launch of
// its own because the two divisions per channel, done by every workgroup for every channel, cost the block kernel more
// than requantising the results (C = 384, 25216 rows: 10 of 60 thousand cycles of its MLP).
constexpr int MAXJ = 6 * kTableLaunches;
struct TableJob { const int32_t* b; const int32_t* c; const int32_t* bias; int32_t* dst; int n; int kind; };      // kind 0 Rq, 1 Rq64, 2 LayerNorm (b gamma, c beta, bias unused)
struct TableJobs { TableJob j[MAXJ]; int arg[MAXJ]; };      // arg: kind 1 the layer's K, kind 2 the rounding addend

__global__ __launch_bounds__(256) void table_kernel(TableJobs J) {
    const TableJob t = J.j[blockIdx.y];
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= t.n) return;
    if (t.kind == 2) {                                              // gamma, then beta + 2^(c-1)
        t.dst[i] = t.b[i];
        t.dst[t.n + i] = (int32_t)((uint32_t)t.c[i] + (uint32_t)J.arg[blockIdx.y]);
        return;
    }
    const int32_t b = t.b[i], c = t.c[i], bias = t.bias ? t.bias[i] : 0;
    v4i e;
    if (t.kind == 1) {
        Residual64 q;
        residual64_of(q, b, c, bias, 1);
        // |acc| <= 2^14 K.  A term of up to 2^30 is asked for here, once per channel, so that its sum with the residual's needs
        // no saturating addition there (the longer instruction costs 0.6 % of a forward: DeiT-S batch 128 1216 -> 1223 us)
        const int64_t sum = (bias < 0 ? -(int64_t)bias : (int64_t)bias) + ((int64_t)J.arg[blockIdx.y] << 14);
        const bool fits = dyadic_fits32(b, c) && sum * b < (int64_t)1 << (30 + c);
        e = v4i{fits ? (int32_t)q.b : 0, 0, (int32_t)(uint32_t)q.h, (int32_t)(q.h >> 32)};
    } else {
        e = v4i{1, 0, 0, 0};
        if (c >= 1 && c <= 24 && b >= 1 && b < (1 << ((c - 1) & 31))) {
            const int64_t half = (int64_t)1 << (c - 1), two_c = (int64_t)1 << c;
            const int64_t Lp = (int64_t)((uint32_t)(127 * two_c - half + b - 1) / (uint32_t)b);
            const int64_t Ln = -(int64_t)((uint32_t)(126 * two_c + 1 + half + b - 1) / (uint32_t)b);
            const int64_t l = Ln - bias, h = Lp - bias;
            if (l >= -(1 << 23) && h < (1 << 23))
                e = v4i{(int32_t)l, (int32_t)h, b << (24 - c), (int32_t)(uint32_t)((uint64_t)((int64_t)bias * b + half) << (24 - c))};
        }
    }
    *reinterpret_cast<v4i*>(t.dst + 4 * i) = e;
}

// v_mfma_i32_32x32x32_i8 with the register file of the accumulators (ACCA) and of the first operand (AA) chosen: the
// kernel needs both files filled, and what vector instructions read must not sit in the accumulation registers.  The
// compiler sees no matrix instruction here, so its results are read by others only after three more of them (or settle()).
template <bool ACCA, bool AA> __device__ __forceinline__ void mfma(v16i& acc, const v4i& a, const v4i& b) {
    if constexpr (ACCA && AA) asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+a"(acc) : "a"(a), "v"(b));
    else if constexpr (ACCA) asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
    else if constexpr (AA) asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(acc) : "a"(a), "v"(b));
    else asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
// ... on a zero accumulator, or (RES) on one of kSumStart
template <bool AA, bool RES = false> __device__ __forceinline__ void mfma_first(v16i& acc, const v4i& a, const v4i& b) {
    static_assert(kSumStart == 0x40000000u, "2.0 below");
    if constexpr (AA && RES) asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, 2.0" : "=&v"(acc) : "a"(a), "v"(b));
    else if constexpr (AA) asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, 0" : "=&v"(acc) : "a"(a), "v"(b));
    else asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
}

// The product that piece i of n goes with when they are spread over the products from .. to - 1.
constexpr int spread_slot(int i, int n, int from, int to) {
    for (int m = from; m < to; ++m)
        if (i < (m - from + 1) * n / (to - from)) return m;
    return to;
}

template <int C, int MT, int NW>
__global__ __launch_bounds__(64 * NW) void token_block_kernel(TokenBlockArgs P) {
    using LY = TbLayout<C, MT, NW>;
    constexpr int KS = LY::KS, PP = LY::P, M = LY::M, TT = LY::TT, T1 = LY::T1, N1 = LY::N1, PT = LY::PT, RS = LY::RS;
    constexpr int WNG = LY::WNG, WN1 = LY::WN1, G16 = LY::G16, SETW = LY::SETW, HP = LY::HP;
    constexpr int NX = G16 / 2 > 0 ? G16 / 2 : 1;
    constexpr int LPR = PP / 3;                                    // lanes of a row in the LayerNorm passes, three pieces each
    constexpr int RD = KS == 12 && NW == 4 ? 4 : 3;                           // ring of weight fragments: requested RD - 1 k-steps ahead
    static_assert((KS % RD) == 0 || ((PT * KS) % RD == 0 && (N1 * KS) % RD == 0), "the ring must align with a set");

    extern __shared__ __align__(1024) int8_t lds[];
    int8_t* act = lds + LY::ACT;
    const int tid = threadIdx.x, lane = tid & 63, lj = lane & 31, lg = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wv % WNG, wm = wv / WNG, wn1 = wv % WN1, wm1 = wv / WN1;
    int8_t* stg = lds + LY::STG + wv * LY::STGB;
    const int64_t m0 = (int64_t)blockIdx.x * M;
    const int rows = __builtin_amdgcn_readfirstlane((int)min64(P.R - m0, M));
    const int F = P.F, NC = F / FC;
    const uint32_t lds0 = lds_offset(lds);
    const bool front = P.o != nullptr;
    auto set_at = [&](int b) __attribute__((always_inline)) -> int8_t* { return lds + LY::SET + b * LY::SETB; };

    auto sync = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto sync_lds = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    // With eight wavefronts what a phase derives from the lane it derives anew, from a copy that the compiler cannot trace to the lane: kept from
    // one phase to the next these addresses are 20 of the 128 registers that a wavefront has beside its accumulation registers.  Where the MLP's
    // accumulators, activations and first results leave no register for the lane either it is counted anew, and so it is for what comes
    // again with every set, channel tile or token tile (counted anew everywhere DeiT-T batch 256 takes 1.5 % longer).
    constexpr bool TIGHT = 4 * KS * T1 + 16 * (3 * TT + N1 * T1) > 160;
    auto fresh_lane = [&]() __attribute__((always_inline)) -> int {
        int l;
        if constexpr (TIGHT) {
            asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
            __builtin_assume(l >= 0 && l < 64);
        } else {
            l = lane;
            if constexpr (NW == 8) pin(l);
        }
        return l;
    };
    auto lane_again = [&]() __attribute__((always_inline)) -> int { if constexpr (TIGHT) return fresh_lane(); else return lane; };
    auto settle = []() __attribute__((always_inline)) {             // the matrix instructions issued so far have written their results
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- loads into LDS.  A set of rows (proj, fc1, qkv) is contiguous in memory, a set of fc2 is 128 bytes of every row,
    // a token tile has its rows permuted (LDS row i holds token 32 (i / 32) + token_of_row(i % 32)).  Load instruction
    // n = NW i + wavefront covers 16-byte slots 64 n .. 64 n + 63; what differs from piece i to i + 3 is a constant step.
    uint32_t vr[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int s = 64 * (NW * i + wv) + lane, r = s / PP, p = s % PP;
        vr[i] = (uint32_t)(r * C + 16 * (p ^ swz<G16>(r)));
    }
    uint32_t v2 = 0;                                                // (of fc2, from the MLP on)
    auto buffer = [](const int8_t* p, uint32_t bytes) __attribute__((always_inline)) -> v4i {
        const uint64_t a = (uint64_t)uniform_ptr(p);
        return v4i{(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)bytes, 0x00020000};
    };
    struct Load { v4i rsrc; uint32_t so, d1, d3, v[3], dst; const int8_t* cst; };      // offset so far, its steps, per-lane offsets; constants
    auto set_dst = [&](int b) __attribute__((always_inline)) -> uint32_t {
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + LY::SET + b * LY::SETB + wv * 1024));
    };
    auto load_rows = [&](const int8_t* w, const int8_t* cst, int row0, int b) __attribute__((always_inline)) -> Load {
        return Load{buffer(w + row0 * C, 0x7fffffffu), 0u - 3072u * NW, 0, 3072 * NW, {vr[0], vr[1], vr[2]}, set_dst(b), uniform_ptr(cst + row0 * 16)};
    };
    auto load_f2 = [&](int chunk, int b) __attribute__((always_inline)) -> Load {
        return Load{buffer(P.fc2.w + chunk * FC, 0x7fffffffu), 0u - 8u * NW * (uint32_t)F, 8u * NW * (uint32_t)F, 8u * NW * (uint32_t)F, {v2, v2, v2}, set_dst(b),
                    uniform_ptr(P.fc2.w)};
    };
    // piece i of a set of `bytes`; the last piece brings the constants of the set's rows (64 rows a wavefront, the last ones repeat
    // each other; a set of fc2 has none and fetches some bytes that nobody reads instead, so that nothing branches here)
    auto load_piece = [&](Load& l, auto i_c, auto bytes_c) __attribute__((always_inline)) {
        constexpr int i = decltype(i_c)::value, NI = decltype(bytes_c)::value / 1024, NP = (NI + NW - 1) / NW, nr = decltype(bytes_c)::value / C;
        if constexpr (i < NP) {
            // (the addition between the write of m0 and the load is the wait state that pair needs)
            if (NW * i + NW - 1 < NI || NW * i + wv < NI)
                asm volatile("s_add_u32 m0, %1, %5\n\ts_add_u32 %0, %0, %2\n\tbuffer_load_dwordx4 %3, %4, %0 offen lds"
                             : "+s"(l.so) : "s"(l.dst), "s"(i % 3 == 0 ? l.d3 : l.d1), "v"(l.v[i % 3]), "s"(l.rsrc), "i"(i * NW * 1024) : "memory", "m0", "scc");
        } else {
            const int w = min(wv, LY::CW - 1);
            dma16(l.cst, (uint32_t)(16 * min(64 * w + lane_again(), nr - 1)), l.dst + SETW - 1024 * (wv - w));
        }
    };
    auto load_range = [&](Load& l, auto lo_c, auto hi_c, auto bytes_c) __attribute__((always_inline)) {
        static_for<decltype(hi_c)::value - decltype(lo_c)::value>([&](auto i) __attribute__((always_inline)) {
            load_piece(l, ic<decltype(lo_c)::value + decltype(i)::value>(), bytes_c);
        });
    };
    using BR = ic<LY::SETR>; using B1 = ic<LY::SET1>;
    constexpr int NPR = (LY::SETR / 1024 + NW - 1) / NW + 1, NP1 = (LY::SET1 / 1024 + NW - 1) / NW + 1;      // pieces of a set
    // a token tile: rows past the matrix read as zero (the buffer ends there)
    constexpr int NPA = (M * PP / 64 + NW - 1) / NW;
    struct Tile { v4i rsrc; uint32_t dst, v[3]; };
    auto act_piece = [&](const Tile& l, auto i_c) __attribute__((always_inline)) {
        constexpr int i = decltype(i_c)::value, NI = M * PP / 64;
        if (NW * i + NW - 1 < NI || NW * i + wv < NI)
            asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                         : : "s"(l.dst), "v"(l.v[i % 3] + (i / 3) * 3072 * NW), "s"(l.rsrc), "i"(i * NW * 1024) : "memory", "m0", "scc");
    };
    auto act_tile = [&](const int8_t* src, int off) __attribute__((always_inline)) -> Tile {
        Tile l{buffer(src + m0 * C, (uint32_t)(rows * C)), (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + off + wv * 1024)), {}};
        const int ll = lane_again();
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int s = 64 * (NW * i + wv) + ll, r = s / PP, p = s % PP;
            l.v[i] = (uint32_t)(((r & ~31) + token_of_row(r & 31)) * C + 16 * (p ^ swz<G16>(r)));
        }
        return l;
    };
    auto load_act = [&](const int8_t* src, int off) __attribute__((always_inline)) {
        const Tile l = act_tile(src, off);
        static_for<NPA>([&](auto i) __attribute__((always_inline)) { act_piece(l, i); });
    };
    auto load_ln = [&](const int8_t* src) __attribute__((always_inline)) {       // gamma, beta: 8 C bytes, one after the other
        const int at = 1024 * wv + 16 * lane_again();
        if (1024 * wv < 8 * C) dma16(uniform_ptr(src), (uint32_t)min(at, 8 * C - 16), lds0 + LY::LN + wv * 1024);
    };
    // ---- the launch's weights and constants into this XCD's L2, every 128-byte line by one lane of one of its first round of
    // workgroups.  A forward's weights are larger than an L2, so they are not there from the launch before, and a set is
    // requested only about a set's products ahead.
    // (Requested where the next wait for loads is a set's products or a LayerNorm away.)
    // Without and with it, three models in turn (one model again and again): DeiT-S batch 64 666 -> 650 us (666 -> 650), batch 128 1096 -> 970
    // (929 -> 946), DeiT-T batch 256 911 -> 863 (852 -> 845), Swin-T batch 128 1514 -> 1438 (1513 -> 1438); requested all at once at
    // the start, where the first barrier waits for it, DeiT-T batch 128 544 instead of 522.
    // Not for what four wavefronts take at widths 96 and 192, where all of it is 0.1 to 0.5 MB: blocks of width 96 were 1 to 3 % slower with it,
    // whether it had anything to do or not (four blocks of 392 rows 77.5 -> 79.5 us, of 50176 144.8 -> 148.4).
    constexpr bool WARM = NW == 8 || C == 384;
    const uint32_t warm_n = min(max(gridDim.x / 8, 1u), 32u), warm_i = blockIdx.x / 8;
    auto warm = [&](const int8_t* p, uint32_t bytes) __attribute__((always_inline)) {
        if (WARM && warm_n >= 4 && warm_i < warm_n)
            for (uint32_t at = (warm_i * 64 * NW + 64 * wv + fresh_lane()) * 128; at < bytes; at += warm_n * 64 * NW * 128)
                dma4(uniform_ptr(p), at, lds0 + LY::SINK);
    };
    // ---- fragments.  Lane (lj, lg) of k-step ks: piece 2 ks + lg of row lj of a tile.
    int xr[NX];                                                     // tiles of rows of C bytes
#pragma unroll
    for (int i = 0; i < NX; ++i) xr[i] = lj * C + 16 * ((2 * i + lg) ^ swz<G16>(lj));
    auto frag = [&](const int8_t* tile, int ks) __attribute__((always_inline)) -> v4i {
        return *reinterpret_cast<const v4i*>(tile + xr[ks % NX] + 16 * G16 * (ks / NX));
    };
    int x2[4] = {};                                                 // tiles of rows of 128 bytes

    // ---- residual and staging addresses (see gemm_rs.hip for the transposing reads)
    // Byte offsets in a token tile's 32 rows, of the first channel tile of this wavefront (the next one lies 32 WNG bytes on: the
    // swizzle does not reach beyond the pieces of WNG tiles).
    int dj, d_o, lb;                                                // destination side of a transposing read: token 8 lb + dj
    int res_p;                                                      // + 16 h rows: the token of result 8 h + jb, A rows in permuted order
    int res_i;                                                      // + 4 h rows: ... A rows in natural order
    int out_at;                                                     // row of token 8 lb + dj
    static_assert(G16 == 2 * WNG, "pieces that the swizzle permutes");
    // (8-byte unit u of row r of the staging tile lies at u ^ ((r / 4) % 4), so that no bank is met twice)
    int stg_src, stg_src8, stg_dst, stg_x, stg_g;
    auto row_addresses = [&]() __attribute__((always_inline)) {
        const int l = fresh_lane(), g = l >> 5;
        const int jb = (l & 15) >> 1, jo = l & 1;                   // source side
        dj = l & 7; d_o = (l >> 3) & 1; lb = l >> 4;
        auto at = [&](int r, int piece) __attribute__((always_inline)) { return r * C + 16 * ((2 * wn + piece) ^ swz<G16>(r)); };
        res_p = at(8 * (jb >> 2) + 4 * g + (jb & 3), lb & 1) + 8 * jo;
        res_i = at(16 * (jb >> 2) + 8 * g + (jb & 3), lb & 1) + 8 * jo;
        out_at = at(16 * (lb & 1) + 8 * (dj >> 2) + 4 * (lb >> 1) + (dj & 3), d_o);
        stg_src = (16 * jo + jb) * 32 + 8 * (lb ^ (jb >> 2));
        stg_src8 = (16 * jo + jb + 8) * 32 + 8 * (lb ^ (jb >> 2) ^ 2);
        stg_dst = (l & 31) * 32;
        stg_x = (l >> 2) & 3;
        stg_g = g;
    };
    auto res_read = [&](const int8_t* tile, int g, auto perm_c, v2i (&rw)[2]) __attribute__((always_inline)) {      // channel tile g WNG + wn
        constexpr bool perm = decltype(perm_c)::value;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // (4 rows on, the swizzle differs by G16 / 4)
            const int8_t* a = tile + (perm ? res_p + 16 * h * C : (res_i ^ (h * (G16 / 4) * 16)) + 4 * h * C) + 32 * WNG * g;
            rw[h] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3)))*)(a));
        }
    };
    auto stg_put = [&](const v4i& w, auto perm_c) __attribute__((always_inline)) {
        constexpr bool perm = decltype(perm_c)::value;
        if (perm) {
            v2i* d = reinterpret_cast<v2i*>(stg + stg_dst);
            d[(2 * stg_g) ^ stg_x] = v2i{w[0], w[1]}; d[(2 * stg_g + 1) ^ stg_x] = v2i{w[2], w[3]};
        } else {
            int* d = reinterpret_cast<int*>(stg + stg_dst + 4 * stg_g);
#pragma unroll
            for (int u = 0; u < 4; ++u) d[2 * (u ^ stg_x)] = w[u];
        }
    };
    auto stg_get = [&]() __attribute__((always_inline)) -> v4i {
        const v2i a = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3)))*)(stg + stg_src));
        const v2i b = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3)))*)(stg + stg_src8));
        return v4i{a[0], a[1], b[0], b[1]};
    };
    auto act_put = [&](int tt, int g, const v4i& w) __attribute__((always_inline)) {      // results of (token tile, channel tile g WNG + wn) into the token tile
        *reinterpret_cast<v4i*>(act + 32 * tt * C + out_at + 32 * WNG * g) = w;
    };

    // a lane's 16 results of a tile in 64-bit arithmetic, channel ch of W; results in the low byte
    auto unit_slow = [&](const v16i& a, const DenseW& W, int ch, bool gelu) __attribute__((always_inline)) -> v4i {
        const int32_t b = W.rq_b[ch], c = W.rq_c[ch], bias = W.bias ? W.bias[ch] : 0;
        v4i w;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t o[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                o[r] = (uint32_t)clamp8_64(rnd_shift64(a[4 * d + r] + bias, b, c));
                if (gelu) o[r] = (uint32_t)(uint8_t)lds[LY::LUT + (o[r] & 0xffu)];
            }
            w[d] = pack4<true>(o);
        }
        return w;
    };
    // ... of a residual layer; the residual rows come from global memory
    auto unit_slow_res = [&](const v16i& a, const DenseW& W, const ResRq& rr, const int8_t* res, int tt, int ct, auto perm_c) __attribute__((always_inline)) -> v4i {
        constexpr bool perm = decltype(perm_c)::value;
        const int l = lane_again(), lg = l >> 5, ch = 32 * ct + (l & 31);
        const int32_t b = W.rq_b[ch], c = W.rq_c[ch], bias = W.bias ? W.bias[ch] : 0;
        v4i w;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t o[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int tok = min(32 * tt + (perm ? 16 * lg + 4 * d : 8 * d + 4 * lg) + r, rows - 1);
                o[r] = (uint32_t)clamp8_64(rnd_shift64(sum_of(a[4 * d + r], bias, kSumStart), b, c) + rnd_shift64(res[(m0 + tok) * C + ch], rr.b, rr.c));
            }
            w[d] = pack4<true>(o);
        }
        return w;
    };

    // ---- I-LayerNorm of the token tile, in place; `st`: the rows before normalisation also go to global memory, `dst`:
    // the normalised ones do
    auto layernorm = [&](int f_bits, int c_shift, int8_t* st, int8_t* dst) __attribute__((always_inline)) {
        constexpr int RPP = 64 / LPR, RW = M / NW;                   // rows per pass, rows of a wavefront
        const __amdgpu_buffer_rsrc_t sb = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(uniform_ptr(st + m0 * C)), 0, st ? rows * C : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t db = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(uniform_ptr(dst + m0 * C)), 0, dst ? rows * C : 0, 0x00020000);
        constexpr int NPASS = RW / RPP;
        static_assert(RW % RPP == 0 && NPASS <= LPR, "rows of a wavefront");
        v4i v[NPASS][3];
        int32_t sm[NPASS], sq[NPASS];
        const int ll = fresh_lane(), q = ll % LPR, rl = ll / LPR;
        const int i0 = wv * RW + rl;                                // row of pass k: i0 + k RPP
#pragma unroll
        for (int k = 0; k < NPASS; ++k) {
            const int i = i0 + k * RPP;
#pragma unroll
            for (int j = 0; j < 3; ++j) v[k][j] = *reinterpret_cast<const v4i*>(act + i * C + 16 * ((q + LPR * j) ^ swz<G16>(i)));
        }
#pragma unroll
        for (int k = 0; k < NPASS; ++k) {
            const int i = i0 + k * RPP, tok = (i & ~31) + token_of_row(i & 31);
            int32_t s = 0, ss = 0;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                if (st) __builtin_amdgcn_raw_buffer_store_b128(v[k][j], sb, tok * C + 16 * (q + LPR * j), 0, 0);
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    s = __builtin_amdgcn_sdot4(v[k][j][d], 0x01010101, s, false);
                    ss = __builtin_amdgcn_sdot4(v[k][j][d], v[k][j][d], ss, false);
                }
            }
            s += dpp_i32<0xB1>(s); ss += dpp_i32<0xB1>(ss);
            if (LPR >= 4) { s += dpp_i32<0x4E>(s); ss += dpp_i32<0x4E>(ss); }
            if (LPR >= 8) { s += dpp_i32<0x141>(s); ss += dpp_i32<0x141>(ss); }
            sm[k] = s; sq[k] = ss;
        }
        // the scalar chain of a row once: lane q of a row's lanes takes pass q
        int32_t s = sm[0], ss = sq[0];
#pragma unroll
        for (int k = 1; k < NPASS; ++k) { s = q == k ? sm[k] : s; ss = q == k ? sq[k] : ss; }
        const LnStat own = ln_stat(s, ss, C, f_bits);
        LnStat row[NPASS];
#pragma unroll
        for (int k = 0; k < NPASS; ++k) {
            const int from = 4 * ((ll & ~(LPR - 1)) + k);
            row[k] = LnStat{__builtin_amdgcn_ds_bpermute(from, own.mean), __builtin_amdgcn_ds_bpermute(from, own.f)};
        }
        // (gamma and beta of one piece at a time: all three would be 96 registers)
        const int32_t* gt = reinterpret_cast<const int32_t*>(lds + LY::LN);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            v4i g[4], b[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                g[e] = *reinterpret_cast<const v4i*>(gt + 16 * (q + LPR * j) + 4 * e);
                b[e] = *reinterpret_cast<const v4i*>(gt + C + 16 * (q + LPR * j) + 4 * e);
            }
#pragma unroll
            for (int k = 0; k < NPASS; ++k) {
                const int i = i0 + k * RPP, tok = (i & ~31) + token_of_row(i & 31);
                v4i w;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    uint32_t o[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int32_t xe = (int32_t)(int8_t)((uint32_t)v[k][j][d] >> (8 * r));
                        o[r] = (uint32_t)ln_value(xe, row[k], g[d][r], b[d][r], c_shift);
                    }
                    w[d] = pack4<true>(o);
                }
                if (dst) __builtin_amdgcn_raw_buffer_store_b128(w, db, tok * C + 16 * (q + LPR * j), 0, 0);
                *reinterpret_cast<v4i*>(act + i * C + 16 * ((q + LPR * j) ^ swz<G16>(i))) = w;
            }
        }
    };

    // ---- products.  A stream of channel tiles of C bytes a row: tile p at w0 + p stride, its k-steps one after the other,
    // NT products a step: mm(p, t, ks) issues one, aux(m) is the work that goes with product m.  The first RD - 1 fragments
    // are in the ring already.  TAIL: before the last RD - 1 steps, when every fragment of the set is in registers, tail()
    // meets the other wavefronts, after which the next set is there and this one's memory is free; next(k) then requests
    // the first fragments of the next set between the remaining products.
    v4i bf[RD];
    auto stream = [&](auto nb_c, auto nt_c, const int8_t* w0, auto stride_c, auto tail_c, auto mm, auto aux, auto tail, auto next) __attribute__((always_inline)) {
        constexpr int NB = decltype(nb_c)::value, NT = decltype(nt_c)::value, stride = decltype(stride_c)::value, NS = NB * KS;
        static_for<NS>([&](auto q_c) __attribute__((always_inline)) {
            constexpr int q = decltype(q_c)::value, qn = q + RD - 1;
            if constexpr (decltype(tail_c)::value && q == NS - RD + 1) tail();
            if constexpr (qn < NS) bf[qn % RD] = frag(w0 + (qn / KS) * stride, qn % KS);
            else if constexpr (decltype(tail_c)::value) next(ic<qn - NS>());
            static_for<NT>([&](auto t_c) __attribute__((always_inline)) {
                mm(ic<q / KS>(), t_c, ic<q % KS>(), bf[q % RD]);
                aux(ic<q * NT + decltype(t_c)::value>());
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    auto first_frags = [&](const int8_t* w0) __attribute__((always_inline)) {
        static_for<RD - 1>([&](auto k) __attribute__((always_inline)) { bf[k] = frag(w0, k); });
    };
    // `n` pieces of work (numbered from lo) spread over the products from .. to - 1
    auto spread = [&](auto lo_c, auto n_c, auto from_c, auto to_c, auto m_c, auto f) __attribute__((always_inline)) {
        constexpr int n = decltype(n_c)::value, from = decltype(from_c)::value, to = decltype(to_c)::value, m = decltype(m_c)::value, w = to - from;
        static_assert(w > 0, "somewhere to go");
        if constexpr (m >= from && m < to) {
            constexpr int lo = (m - from) * n / w, hi = (m - from + 1) * n / w;
            static_for<hi - lo>([&](auto i) __attribute__((always_inline)) { f(ic<decltype(lo_c)::value + lo + decltype(i)::value>()); });
        }
    };

    v4i ar[TT][KS];                                                 // this wavefront's activations in proj and qkv
    auto load_ar = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) ar[t][ks] = frag(act + 32 * (wm * TT + t) * C, ks);
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(ar[t][ks]));
    };

    // ---- proj and qkv: tile g of a wavefront goes to accumulators g % 2 and is requantised while tile g + 1 is multiplied
    constexpr int NMT = KS * TT, NOT = TT * 16;                     // products and results of a lane per tile
    constexpr int EF = NMT > 3 ? 3 : NMT - 1;                       // first product after which the previous tile's results can be read
    v16i pa[2][TT];
    uint32_t eo[4];
    v4i ew = {}, es = {};
    v2i rw[2] = {}, rwn[2] = {};
    bool fast = false;
    auto cst_at = [&](int b, int row) __attribute__((always_inline)) -> v4i {      // of this lane's row of 32
        return *reinterpret_cast<const v4i*>(set_at(b) + SETW + 16 * (row + (lane_again() & 31)));
    };
    const int8_t* const tab = P.table;

    if (front) {
        Load L0 = load_rows(P.proj.w, tab + TB_PROJ(C), 0, 0), L1 = LY::NPROJ > 1 ? load_rows(P.proj.w, tab + TB_PROJ(C), RS, 1) : load_rows(P.fc1.w, tab + TB_FC1(C), 0, 1);
        load_act(P.o, LY::ACT);
        load_ln(tab);
        load_range(L0, ic<0>(), ic<NPR>(), BR());
        if constexpr (LY::NPROJ > 1) load_range(L1, ic<0>(), ic<NPR>(), BR()); else load_range(L1, ic<0>(), ic<NP1>(), B1());
        lds[LY::LUT + (tid & 255)] = (int8_t)requant64(shiftgelu_raw((int32_t)(int8_t)tid, P.gelu_p), P.gelu_rq.b, P.gelu_rq.c);
        const ResRq rr1 = make_res(P.res1);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(LY::NPROJ > 1 && LY::SETR % (1024 * NW) == 0 ? NPR : 0) : "memory");
        load_ar();
        first_frags(set_at(0) + wn * 32 * C);
        sync_lds();
        load_act(P.x, LY::ACT);
        row_addresses();
        // ---- proj.  Sets 0 .. NPROJ - 1, then fc1's first two, alternate between the two buffers.
        Rq64 pq = {};
        v4i pqn = {};
        auto ct_of = [&](int g) __attribute__((always_inline)) -> int { return g * WNG + wn; };        // channel tile of tile g
        auto proj_res = [&](int g, int t) __attribute__((always_inline)) { res_read(act + 32 * (wm * TT + t) * C, g, std::true_type(), rwn); };
        auto proj_out = [&](int g, auto par_c, auto i_c) __attribute__((always_inline)) {      // piece i of tile g: 16 TT results, then its last rows
            constexpr int i = decltype(i_c)::value, t = i / 16, e = i % 16, par = decltype(par_c)::value;
            if constexpr (i == NOT) { es = stg_get(); return; }
            else if constexpr (i == NOT + 1) { act_put(wm * TT + TT - 1, g, es); return; }
            else {
                if constexpr (e == 0) { rw[0] = rwn[0]; rw[1] = rwn[1]; }
                eo[e & 3] = out_res(pa[par][t][e], pq, rr1, (int32_t)(int8_t)((uint32_t)rw[e >> 3][(e >> 2) & 1] >> (8 * (e & 3))));
                if constexpr ((e & 3) == 3) { int w = pack4<true>(eo); pin(w); ew[e >> 2] = w; }
                if constexpr (e == 8 && t + 1 < TT) proj_res(g, t + 1);
                if constexpr (e == 3 && t > 0) es = stg_get();
                if constexpr (e == 11 && t > 0) act_put(wm * TT + t - 1, g, es);
                if constexpr (e == 15) stg_put(ew, std::true_type());
            }
        };
        auto proj_slow = [&](int g, auto par_c) __attribute__((always_inline)) {
            if (fast) return;
            static_for<TT>([&](auto t_c) __attribute__((always_inline)) {
                constexpr int t = decltype(t_c)::value;
                stg_put(unit_slow_res(pa[decltype(par_c)::value][t], P.proj, rr1, P.x, wm * TT + t, ct_of(g), std::true_type()), std::true_type());
                act_put(wm * TT + t, g, stg_get());
            });
        };
        static_for<LY::NPROJ>([&](auto s_c) __attribute__((always_inline)) {
            constexpr int s = decltype(s_c)::value, b = s & 1;
            constexpr bool last = s + 1 == LY::NPROJ;
            Load L = s >= 1 ? (last ? load_rows(P.fc1.w, tab + TB_FC1(C), 0, b ^ 1) : load_rows(P.proj.w, tab + TB_PROJ(C), (s + 1) * RS, b ^ 1)) : Load{};
            stream(ic<PT>(), ic<TT>(), set_at(b) + wn * 32 * C, ic<WNG * 32 * C>(), std::bool_constant<!last>(),
                [&](auto p_c, auto t_c, auto ks_c, const v4i& f) __attribute__((always_inline)) {
                    constexpr int par = (s * PT + decltype(p_c)::value) & 1, t = decltype(t_c)::value, ks = decltype(ks_c)::value;
                    if constexpr (ks == 0) mfma_first<true, true>(pa[par][t], ar[t][ks], f); else mfma<false, true>(pa[par][t], ar[t][ks], f);
                },
                [&](auto m_c) __attribute__((always_inline)) {
                    constexpr int m = decltype(m_c)::value, p = m / NMT, mt = m % NMT, g = s * PT + p;
                    if constexpr (s >= 1) spread(ic<0>(), ic<NPR>(), ic<0>(), ic<PT * NMT * 3 / 4>(), m_c, [&](auto i) __attribute__((always_inline)) { load_piece(L, i, BR()); });
                    if constexpr (LY::NPROJ == 1 && g == 1 && mt == 0) sync();       // the residual rows are there
                    if constexpr (mt == 0 && (LY::NPROJ == 1 ? g == 1 : p == 0)) {
                        if constexpr (LY::NPROJ == 1 || s == 0) warm(P.fc1.w, F * C);
                        if constexpr (LY::NPROJ == 1 || s == 1) warm(P.fc2.w, F * C);
                        if constexpr (s + 1 == LY::NPROJ) {
                            warm(P.table, TB_BYTES(C, F));
                            if (P.next == 2) warm(P.qkv_w.w, 3 * C * C);
                        }
                    }
                    if constexpr (g > 0) {
                        if constexpr (mt == 0) proj_res(g - 1, 0);
                        spread(ic<0>(), ic<NOT + 2>(), ic<EF>(), ic<NMT>(), ic<mt>(), [&](auto i) __attribute__((always_inline)) { proj_out(g - 1, ic<(g - 1) & 1>(), i); });
                        if constexpr (mt == NMT - 1) proj_slow(g - 1, ic<(g - 1) & 1>());
                    }
                    if constexpr (mt == 0) pqn = cst_at(b, (p * WNG + wn) * 32);
                    if constexpr (mt == NMT - 1) { pq = as_rq64(pqn); fast = __builtin_amdgcn_ballot_w64(pq.b != 0 && rr1.ok) == ~0ull; }
                },
                [&]() __attribute__((always_inline)) { sync(); },
                [&](auto k) __attribute__((always_inline)) { bf[k] = frag(set_at(b ^ 1) + wn * 32 * C, k); });
        });
        {
            constexpr int g = LY::NPROJ * PT - 1;
            proj_res(g, 0);
            settle();
            static_for<NOT + 2>([&](auto i) __attribute__((always_inline)) { proj_out(g, ic<g & 1>(), i); });
            proj_slow(g, ic<g & 1>());
        }
        sync_lds();
        // ---- LN2
        Load L = load_rows(P.fc1.w, tab + TB_FC1(C), FC, 0);
        load_range(L, ic<0>(), ic<NP1>(), B1());
        layernorm(P.ln2_f, P.ln2_c, P.xhat, nullptr);
        sync();
        if (P.next) load_ln(tab + TB_LN1(C));
        // ---- MLP.  Sets: F1(0), F1(1), F2(0), F1(2), F2(1), ..., F1(NC - 1), F2(NC - 2), F2(NC - 1), the rows of xhat; F1(0) is in
        // buffer 1, from then on F1 sets are in buffer 0, F2 sets in buffer 1 (the last one, having no F1 set after its
        // predecessor, in buffer 0).  Results of fc1: channel tile n is requantised while tile n + 1 is multiplied, the last
        // one during the next F2.
        constexpr int NM1 = KS * T1, NO1 = T1 * 16, NM2 = 12 * TT, LAG = NW == 8 ? 4 : 8;     // results between a table read and its use
        constexpr int EF1 = NM1 > 3 ? 3 : NM1 - 1;
        constexpr int TP = NP1 / 3;                                 // pieces of a set requested before the end of the set before its predecessor
        constexpr auto vv_acc = [](int t, int ks) constexpr { return 3 * TT * 16 + 4 * (t * KS + ks + 1) <= 1024 / NW; };      // fits beside fc2's accumulators (half of the registers)
        v4i vv[T1][KS];
        static_for<T1>([&](auto t) __attribute__((always_inline)) {
            static_for<KS>([&](auto ks) __attribute__((always_inline)) {
                vv[t][ks] = frag(act + 32 * (wm1 * T1 + decltype(t)::value) * C, ks);
            });
        });
#pragma unroll
        for (int t = 0; t < T1; ++t)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                if (vv_acc(t, ks)) asm volatile("" : "+a"(vv[t][ks]));
        v16i acc[3][TT], ha[N1][T1];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int t = 0; t < TT; ++t) { acc[j][t] = sums_from(kSumStart); asm volatile("" : "+a"(acc[j][t])); }
        const int8_t* f1w0 = set_at(0) + wn1 * N1 * 32 * C;
        const int8_t* f1w1 = set_at(1) + wn1 * N1 * 32 * C;
        first_frags(f1w1);
        sync_lds();
        Rq hq[N1];
        bool hfast = false;
        uint32_t gl[LAG + 4];
        const int hl = fresh_lane();
        int8_t* const h_out = act + (wn1 * N1 * 32 + (hl & 31)) * HP + 32 * wm1 * T1 + 16 * (hl >> 5);
        auto h_at = [&](int hbuf, int u) __attribute__((always_inline)) -> int8_t* {
            return h_out + hbuf * LY::HB + (u / T1) * 32 * HP + 32 * (u % T1);
        };
        // piece i of a channel tile's results, or of the last ones' packing; u0: first unit (tile of 32 x 32) of the channel tile
        auto gelu_out = [&](int hbuf, auto u0_c, auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value, j = i - LAG, u0 = decltype(u0_c)::value;
            if constexpr (j >= 0 && (j & 3) == 3) {
                const uint32_t o[4] = {gl[(j - 3) % (LAG + 4)], gl[(j - 2) % (LAG + 4)], gl[(j - 1) % (LAG + 4)], gl[j % (LAG + 4)]};
                int w = pack4<true>(o);
                pin(w);
                ew[(j >> 2) & 3] = w;
                if constexpr ((j & 15) == 15) *reinterpret_cast<v4i*>(h_at(hbuf, u0 + j / 16)) = ew;
            }
            if constexpr (i < NO1) {
                constexpr int u = u0 + i / 16;
                const uint32_t at = out_top(ha[u / T1][u % T1][i % 16], hq[u / T1]) >> 24;
                gl[i % (LAG + 4)] = *reinterpret_cast<const __attribute__((address_space(3))) uint8_t*>(at);
            }
        };
        auto gelu_slow = [&](int hbuf, int chunk) __attribute__((always_inline)) {
            if (hfast) return;
            static_for<N1 * T1>([&](auto u_c) __attribute__((always_inline)) {
                constexpr int u = decltype(u_c)::value;
                *reinterpret_cast<v4i*>(h_at(hbuf, u)) = unit_slow(ha[u / T1][u % T1], P.fc1, chunk * FC + (wn1 * N1 + u / T1) * 32 + (lane_again() & 31), true);
            });
        };
        const int r2 = 8 * wv + (hl >> 3);
        v2 = (uint32_t)(r2 * F + 16 * ((hl & 7) ^ swz<8>(r2)));
#pragma unroll
        for (int i = 0; i < 4; ++i) x2[i] = (hl & 31) * FC + 16 * ((2 * i + (hl >> 5)) ^ swz<8>(hl & 31));
        const int8_t* h0 = act + (16 * (hl >> 5) + ((hl & 15) >> 1)) * HP + 32 * wm * TT + (hl & 16) + 8 * (hl & 1);
        constexpr int RB = TIGHT ? 3 : 4;                           // ring of weight fragments of fc2: requested RB - 1 steps ahead
        v4i af[2][TT], b2[RB];
        auto read_a = [&](int hbuf, auto kk_c) __attribute__((always_inline)) {
            constexpr int kk = decltype(kk_c)::value;
#pragma unroll
            for (int t = 0; t < TT; ++t) {
                const int8_t* p = h0 + hbuf * LY::HB + 32 * kk * HP + 32 * t;
                const v2i a = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3)))*)(p));
                const v2i c = __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3)))*)(p + 8 * HP));
                af[kk & 1][t] = v4i{a[0], a[1], c[0], c[1]};
            }
        };
        auto read_b = [&](int b, auto st_c) __attribute__((always_inline)) {
            constexpr int st = decltype(st_c)::value;
            b2[st % RB] = *reinterpret_cast<const v4i*>(set_at(b) + wn * 32 * FC + (st % 3) * WNG * 32 * FC + x2[st / 3]);
        };
        auto f2_first = [&](int b, int hbuf, auto k_c) __attribute__((always_inline)) {      // piece k of RD - 1 of an F2's first fragments
            constexpr int k = decltype(k_c)::value;
            if constexpr (k == 0) read_a(hbuf, ic<0>());
            read_b(b, k_c);
            if constexpr (k == RD - 2 && RB > RD) read_b(b, ic<RD - 1>());
        };
        // body(m): the loads and whatever else goes with product m; after(): loads to start once this set's memory is free
        auto f1 = [&](const int8_t* w0, int b, int hbuf, auto body, auto after, auto next) __attribute__((always_inline)) {
            v4i hc[N1];
            stream(ic<N1>(), ic<T1>(), w0, ic<32 * C>(), std::true_type(),
                [&](auto n_c, auto t_c, auto ks_c, const v4i& f) __attribute__((always_inline)) {
                    constexpr int n = decltype(n_c)::value, t = decltype(t_c)::value, ks = decltype(ks_c)::value;
                    if constexpr (ks == 0) mfma_first<vv_acc(t, ks)>(ha[n][t], vv[t][ks], f); else mfma<false, vv_acc(t, ks)>(ha[n][t], vv[t][ks], f);
                },
                [&](auto m_c) __attribute__((always_inline)) {
                    constexpr int m = decltype(m_c)::value, n = m / NM1, mt = m % NM1;
                    body(m_c);
                    if constexpr (m == 0) {
#pragma unroll
                        for (int k = 0; k < N1; ++k) hc[k] = cst_at(b, (wn1 * N1 + k) * 32);
                    }
                    if constexpr (m == NM1 - 1) {
                        bool ok = true;
#pragma unroll
                        for (int k = 0; k < N1; ++k) { hq[k] = as_rq(hc[k]); ok = ok && hq[k].lo <= hq[k].hi; }
                        hfast = __builtin_amdgcn_ballot_w64(ok) == ~0ull;
                    }
                    if constexpr (n == 0) { }
                    else spread(ic<0>(), ic<NO1 + LAG>(), ic<EF1>(), ic<NM1>(), ic<mt>(), [&](auto i) __attribute__((always_inline)) { gelu_out(hbuf, ic<(n - 1) * T1>(), i); });
                },
                [&]() __attribute__((always_inline)) { sync(); after(); }, next);
        };
        auto f2 = [&](int b, int hbuf, auto tail_c, auto body, auto after, auto next) __attribute__((always_inline)) {
            static_for<12>([&](auto st_c) __attribute__((always_inline)) {
                constexpr int st = decltype(st_c)::value, kk = st / 3, j = st % 3;
                if constexpr (decltype(tail_c)::value && st == 10) { sync(); after(); }
                if constexpr (st + RB - 1 < 12) read_b(b, ic<st + RB - 1>());
                if constexpr (j == 1 && kk < 3) read_a(hbuf, ic<kk + 1>());
                if constexpr (decltype(tail_c)::value && st >= 10) {
                    next(ic<2 * (st - 10)>());
                    next(ic<2 * (st - 10) + 1>());
                }
                static_for<TT>([&](auto t_c) __attribute__((always_inline)) {
                    constexpr int t = decltype(t_c)::value;
                    mfma<true, false>(acc[j][t], af[kk & 1][t], b2[st % RB]);
                    body(ic<st * TT + t>());
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
        };
        auto none = [](auto...) __attribute__((always_inline)) {};
        constexpr int EF2 = NM2 > 6 ? 3 : 2;
        auto rest = [&](auto m_c, auto nm_c) __attribute__((always_inline)) {       // the rest of the set being loaded
            spread(ic<TP>(), ic<NP1 - TP>(), ic<0>(), ic<(decltype(nm_c)::value * 6) / 10>(), m_c, [&](auto i) __attribute__((always_inline)) { load_piece(L, i, B1()); });
        };
        auto start = [&](const Load& l) __attribute__((always_inline)) { L = l; load_range(L, ic<0>(), ic<TP>(), B1()); };
        auto next_f1 = [&](auto k) __attribute__((always_inline)) { if constexpr (decltype(k)::value < RD - 1) bf[k] = frag(f1w0, k); };

        f1(f1w1, 1, 0, none, [&]() __attribute__((always_inline)) { start(load_f2(0, 1)); }, next_f1);
        settle();
        static_for<NO1 + LAG>([&](auto i) __attribute__((always_inline)) { gelu_out(0, ic<(N1 - 1) * T1>(), i); });
        gelu_slow(0, 0);
        auto f1_loop = [&](int i) __attribute__((always_inline)) {      // F1(i), then F2(i - 1)
            f1(f1w0, 0, i & 1, [&](auto m) __attribute__((always_inline)) { rest(m, ic<N1 * NM1>()); },
               [&]() __attribute__((always_inline)) {
                   const bool more = i + 1 < NC;
                   const Load a = load_rows(P.fc1.w, tab + TB_FC1(C), (more ? i + 1 : 0) * FC, 0), c = load_f2(i, 0);
                   Load l = a;
                   if (!more) l = c;
                   start(l);
               },
               [&](auto k) __attribute__((always_inline)) { f2_first(1, (i - 1) & 1, k); });
        };
        auto f2_epi = [&](int i, auto m_c) __attribute__((always_inline)) {        // the last results of F1(i + 1), during F2(i)
            spread(ic<0>(), ic<NO1 + LAG>(), ic<EF2>(), ic<NM2>(), m_c, [&](auto k) __attribute__((always_inline)) { gelu_out((i + 1) & 1, ic<(N1 - 1) * T1>(), k); });
        };
        f1_loop(1);
#pragma unroll 1
        for (int i = 0; i + 2 < NC; ++i) {
            f2(1, i & 1, std::true_type(), [&](auto m) __attribute__((always_inline)) { rest(m, ic<NM2>()); f2_epi(i, m); },
               [&]() __attribute__((always_inline)) { start(load_f2(i + 1, 1)); }, next_f1);
            gelu_slow((i + 1) & 1, i + 1);
            f1_loop(i + 2);
        }
        f2(1, NC & 1, std::true_type(), [&](auto m) __attribute__((always_inline)) { rest(m, ic<NM2>()); f2_epi(NC - 2, m); }, none,
           [&](auto k) __attribute__((always_inline)) { if constexpr (decltype(k)::value == 0) { static_for<RD - 1>([&](auto kk) __attribute__((always_inline)) { (void)kk; }); } });
        gelu_slow((NC - 1) & 1, NC - 1);
        sync_lds();                                                 // the last hidden chunk is complete
        static_for<RD - 1>([&](auto k) __attribute__((always_inline)) { f2_first(0, (NC - 1) & 1, k); });
        // constants of fc2 for the epilogue, requested before the loads that follow
        v4i fb[3];
#pragma unroll
        for (int j = 0; j < 3; ++j) fb[j] = *reinterpret_cast<const v4i*>(tab + TB_FC2(C) + 16 * (32 * (j * WNG + wn) + (lane_again() & 31)));
        {
            const Tile l = act_tile(P.xhat, LY::SET + LY::SETB);
            f2(0, (NC - 1) & 1, std::false_type(), [&](auto m) __attribute__((always_inline)) {
                spread(ic<0>(), ic<NPA>(), ic<0>(), ic<(NM2 / 2 > 0 ? NM2 / 2 : 1)>(), m, [&](auto i) __attribute__((always_inline)) { act_piece(l, i); });
            }, none, none);
        }
        const ResRq rr2 = make_res(P.res2);
        Rq64 fq[3];
        bool ok2 = rr2.ok;
#pragma unroll
        for (int j = 0; j < 3; ++j) { fq[j] = as_rq64(fb[j]); ok2 = ok2 && fq[j].b != 0; }
        const bool fast2 = __builtin_amdgcn_ballot_w64(ok2) == ~0ull;
        sync();                                                     // the rows of xhat are there; the hidden chunks are done with
        if (P.next == 2) { L = load_rows(P.qkv_w.w, tab + TB_QKV(C, F), 0, 0); load_range(L, ic<0>(), ic<NPR>(), BR()); }
        settle();
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int t = 0; t < TT; ++t) asm volatile("" : "+a"(acc[j][t]));      // (not to be copied out before)
        auto f2_res = [&](int u) __attribute__((always_inline)) {
            res_read(set_at(1) + 32 * (wm * TT + u % TT) * C, u / TT, std::false_type(), rwn);
        };
        auto f2_put = [&](int u, const v4i& w) __attribute__((always_inline)) { act_put(wm * TT + u % TT, u / TT, w); };
        row_addresses();
        f2_res(0);
        static_for<3 * TT>([&](auto u_c) __attribute__((always_inline)) {
            constexpr int u = decltype(u_c)::value;
            rw[0] = rwn[0]; rw[1] = rwn[1];
            if constexpr (u + 1 < 3 * TT) f2_res(u + 1);
            if constexpr (u > 0) es = stg_get();
            static_for<16>([&](auto e_c) __attribute__((always_inline)) {
                constexpr int e = decltype(e_c)::value;
                eo[e & 3] = out_res(acc[u / TT][u % TT][e], fq[u / TT], rr2, (int32_t)(int8_t)((uint32_t)rw[e >> 3][(e >> 2) & 1] >> (8 * (e & 3))));
                if constexpr ((e & 3) == 3) ew[e >> 2] = pack4<true>(eo);
            });
            if constexpr (u > 0) f2_put(u - 1, es);
            stg_put(ew, std::false_type());
        });
        es = stg_get(); f2_put(3 * TT - 1, es);
        if (!fast2)
            static_for<3 * TT>([&](auto u_c) __attribute__((always_inline)) {
                constexpr int u = decltype(u_c)::value;
                stg_put(unit_slow_res(acc[u / TT][u % TT], P.fc2, rr2, P.xhat, wm * TT + u % TT, (u / TT) * WNG + wn, std::false_type()), std::false_type());
                f2_put(u, stg_get());
            });
        sync_lds();
    } else {
        Load L = load_rows(P.qkv_w.w, tab + TB_QKV(C, F), 0, 0);
        load_act(P.x, LY::ACT);
        load_ln(tab + TB_LN1(C));
        load_range(L, ic<0>(), ic<NPR>(), BR());
        sync();
        warm(P.qkv_w.w, 3 * C * C);
        warm(P.table, TB_BYTES(C, F));
    }
    if (!P.next) {                                                  // only the block's output leaves
        constexpr int NI = M * PP / 64;
        const __amdgpu_buffer_rsrc_t yb = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(uniform_ptr(P.y + m0 * C)), 0, rows * C, 0x00020000);
        const int l = lane_again();
#pragma unroll
        for (int i = 0; i < (NI + NW - 1) / NW; ++i) {
            const int s = 64 * (NW * i + wv) + l, r = s / PP, p = s % PP;
            if (s < M * PP) __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const v4i*>(act + r * C + 16 * (p ^ swz<G16>(r))), yb,
                                                                  ((r & ~31) + token_of_row(r & 31)) * C + 16 * p, 0, 0);
        }
        return;
    }
    if (P.next == 2) { Load L1 = load_rows(P.qkv_w.w, tab + TB_QKV(C, F), RS, 1); load_range(L1, ic<0>(), ic<NPR>(), BR()); }
    layernorm(P.ln1_f, P.ln1_c, front ? P.y : nullptr, P.next == 1 ? P.out : nullptr);
    if (P.next == 1) return;
    sync();
    load_ar();
    first_frags(set_at(0) + wn * 32 * C);
    // ---- qkv of the next block: set s in buffer s % 2; its loads start when set s - 2 has been read
    const int N3 = 3 * C;
    // rows of qkv from this workgroup's first one on, as a buffer that ends with the matrix
    const uint64_t q_base = (uint64_t)uniform_ptr(P.out + m0 * N3);
    row_addresses();
    uint32_t q_off[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) q_off[t] = (uint32_t)((32 * (wm * TT + t) + 8 * lb + dj) * N3 + 16 * d_o);
    constexpr int TPR = NPR / 3;
    Load L = {};
    Rq rq = {};
    v4i rqn = {};
    // Stores that follow the last piece of a set's loads and come before its tail: the wait for the loads leaves them out.
    constexpr int QL = PT * NMT * 4 / 10 > 0 ? PT * NMT * 4 / 10 : 1;      // the loads of the next set go with the first QL products
    constexpr auto stores_after_loads = []() constexpr {
        const int from = spread_slot(NPR - TPR - 1, NPR - TPR, 0, QL), to = (PT * KS - RD + 1) * TT;
        int n = 0;
        for (int p = 0; p < PT; ++p)
            for (int t = 0; t < TT; ++t) {
                const int at = p * NMT + spread_slot(t + 1 < TT ? 16 * (t + 1) + 11 : NOT + 1, NOT + 2, EF, NMT);
                n += at > from && at < to;
            }
        return n;
    };
    constexpr int NSA = stores_after_loads();
    auto qkv_put = [&](int g, int t, const v4i& w, bool real) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t ob = __builtin_amdgcn_make_buffer_rsrc((int8_t*)q_base, 0, real ? rows * N3 : 0, 0x00020000);
        // (The offset all in a vector register: behind a 16-byte store with a scalar offset the compiler leaves out the wait state
        // before the next write of its data registers, and with a second wavefront on the SIMD some lanes then stored the new value.)
        __builtin_amdgcn_raw_buffer_store_b128(w, ob, (int)q_off[t] + (g * WNG + wn) * 32, 0, 0);
    };
    auto qkv_out = [&](int g, auto par_c, auto i_c) __attribute__((always_inline)) {
        constexpr int i = decltype(i_c)::value, t = i / 16, e = i % 16, par = decltype(par_c)::value;
        if constexpr (i == NOT) es = stg_get();
        else if constexpr (i == NOT + 1) qkv_put(g, TT - 1, es, fast);
        else {
            eo[e & 3] = out_top(pa[par][t][e], rq);
            if constexpr ((e & 3) == 3) { int w = pack4<false>(eo); pin(w); ew[e >> 2] = w; }
            if constexpr (e == 3 && t > 0) es = stg_get();
            if constexpr (e == 11 && t > 0) qkv_put(g, t - 1, es, fast);
            if constexpr (e == 15) stg_put(ew, std::true_type());
        }
    };
    auto qkv_slow = [&](int g, auto par_c) __attribute__((always_inline)) {
        if (fast) return;
        static_for<TT>([&](auto t_c) __attribute__((always_inline)) {
            stg_put(unit_slow(pa[decltype(par_c)::value][decltype(t_c)::value], P.qkv_w, (g * WNG + wn) * 32 + (lane_again() & 31), false), std::true_type());
            qkv_put(g, decltype(t_c)::value, stg_get(), true);
        });
    };
    // set s (b: its buffer, the parity of its first tile); FIRST: no results wait yet and its successor is being loaded already
    auto qkv_set = [&](int s, auto b_c, auto first_c, auto last_c) __attribute__((always_inline)) {
        constexpr int b = decltype(b_c)::value;
        constexpr bool first = decltype(first_c)::value, last = decltype(last_c)::value;
        stream(ic<PT>(), ic<TT>(), set_at(b) + wn * 32 * C, ic<WNG * 32 * C>(), std::bool_constant<!last>(),
            [&](auto p_c, auto t_c, auto ks_c, const v4i& f) __attribute__((always_inline)) {
                constexpr int par = (b + decltype(p_c)::value) & 1, t = decltype(t_c)::value, ks = decltype(ks_c)::value;
                if constexpr (ks == 0) mfma_first<true>(pa[par][t], ar[t][ks], f); else mfma<false, true>(pa[par][t], ar[t][ks], f);
            },
            [&](auto m_c) __attribute__((always_inline)) {
                constexpr int m = decltype(m_c)::value, p = m / NMT, mt = m % NMT, par = (b + p + 1) & 1;
                if constexpr (!first && !last) spread(ic<TPR>(), ic<NPR - TPR>(), ic<0>(), ic<QL>(), m_c, [&](auto i) __attribute__((always_inline)) { load_piece(L, i, BR()); });
                if constexpr (p > 0 || !first) {
                    spread(ic<0>(), ic<NOT + 2>(), ic<EF>(), ic<NMT>(), ic<mt>(), [&](auto i) __attribute__((always_inline)) { qkv_out(s * PT + p - 1, ic<par>(), i); });
                    if constexpr (mt == NMT - 1) qkv_slow(s * PT + p - 1, ic<par>());
                }
                if constexpr (mt == 0) rqn = cst_at(b, (p * WNG + wn) * 32);
                if constexpr (mt == NMT - 1) { rq = as_rq(rqn); fast = __builtin_amdgcn_ballot_w64(rq.lo <= rq.hi) == ~0ull; }
            },
            [&]() __attribute__((always_inline)) {
                // (the first set's successor was requested before it, with nothing in between)
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(first ? 0 : NSA) : "memory");
                if (s + 2 < LY::NQKV) { L = load_rows(P.qkv_w.w, tab + TB_QKV(C, F), (s + 2) * RS, b); load_range(L, ic<0>(), ic<TPR>(), BR()); }
            },
            [&](auto k) __attribute__((always_inline)) { bf[k] = frag(set_at(b ^ 1) + wn * 32 * C, k); });
    };
    qkv_set(0, ic<0>(), std::true_type(), std::false_type());
#pragma unroll 1
    for (int s = 1; s + 2 < LY::NQKV; s += 2) {
        qkv_set(s, ic<1>(), std::false_type(), std::false_type());
        qkv_set(s + 1, ic<0>(), std::false_type(), std::false_type());
    }
    qkv_set(LY::NQKV - 2, ic<1>(), std::false_type(), std::false_type());
    qkv_set(LY::NQKV - 1, ic<0>(), std::false_type(), std::true_type());
    settle();
    static_for<NOT + 2>([&](auto i) __attribute__((always_inline)) { qkv_out(LY::NQKV * PT - 1, ic<(PT + 1) & 1>(), i); });
    qkv_slow(LY::NQKV * PT - 1, ic<(PT + 1) & 1>());
}

template <int C, int MT, int NW>
hipError_t launch_tb(hipStream_t s, const TokenBlockArgs& a) {
    using LY = TbLayout<C, MT, NW>;
    const int64_t grid = (a.R + LY::M - 1) / LY::M;
    hipLaunchKernelGGL((token_block_kernel<C, MT, NW>), dim3((unsigned)grid), dim3(64 * NW), LY::TOTAL, s, a);
    return hipGetLastError();
}

}  // namespace

bool token_block_takes(int C, int F, int64_t R, int n_blocks) {
    // C = 384: with few tiles a CU spends its time on fetching the layers' 1.7 MB of weights through one workgroup; the
    // separate kernels spread each layer over the chip.  Whole forwards, fused against separate, F = 4 C (token_stream.hip): DeiT-S
    // batch 4 378 against 350 us, 6 (1182 rows) 368 against 372, 8 (1576) 367 against 382, 16 382 against 452, 25 413 against 542.
    // The constants' launch and the two ends of a stack cost the same however few blocks it has, so short ones need more rows: time fused /
    // separate, one block 1576 rows 1.13, 2364 1.06, 2758 0.99; two 1576 1.05, 1970 1.02, 2364 1.00; three 1576 1.03, 1970 0.99; four
    // 1576 1.015, 1970 0.98; six 1379 1.01, 1576 1.00; eight 1379 1.00.
    // Other F: DeiT-S's sizes in the form with shared sets, batch 24 (4728 rows) 570 against 556, 32 (6304) 591 against 661.
    // What is left beyond full rounds of tiles is cheap in the form for few rows: batch 168 (33096 rows, 328 of them beyond) 1481
    // against 1567 us with separate kernels, 184 (36248) 1567 against 1731.
    // A workgroup walks the F / 128 chunks of the MLP one after the other, where a separate layer spreads them over the chip,
    // so a long MLP needs rows.  us a block, fused against separate: up to F = 4 C + 128 any number of rows (C = 96, F = 384,
    // 197 rows 24.2 against 24.4, F = 512 25.3 against 27.1; C = 192, F = 768 25.4 against 26.1, F = 896 28.3 against 30.1);
    // beyond, C = 96: F = 1536, 3152 rows 37.9 against 36.4, 4728 38.1 against 39.8; F = 8192, 12608 rows 121 against 94,
    // 16548 120 against 121, 23640 129 against 159; C = 192: F = 1536, 2364 rows 36.4 against 35.1, 3152 36.7 against 38.7;
    // F = 3072, 4728 rows 56 against 53, 6304 57 against 58; F = 8192, 197 rows 102 against 43, 12608 117 against 113; F = 16384,
    // 12608 rows 186 against 166, 16548 244 against 267; C = 384: F = 3072, 5122 rows 66 against 55, 6304 68 against 62, 9456 83
    // against 86; F = 8192, 9850 rows 143 against 135; F = 16384, 16548 rows 333 against 290, 19700 337 against 338.
    if (F > 4 * C + FC) {
        const int64_t need = (C == 96 ? 3 : 2) * (int64_t)F;
        if (R < (C == 384 ? need : std::min(need, 64 * (int64_t)num_cus()))) return false;
    }
    if (C == 384 && R < (F == 4 * C ? 1300 + (n_blocks < 8 ? 1400 / n_blocks : 0) : 5120)) return false;
    // A little more than one full round of workgroups at a longer MLP: the rest is a launch of its own (launch_token_block) that walks the whole
    // MLP for a few rows in the form with shared sets, which is the longer the larger F is.  Three blocks of 197 tokens, rows beyond the round:
    // time fused / separate on two boxes: F = 3072 722 1.13 and 1.05, 1510 1.07 and 0.99, 3480 1.03 and 0.96; F = 2048 722 1.07 and 0.97, 1510 1.03
    // and 0.94; F = 1664 131 1.03, 722 1.01, 1510 0.98; F = 256 to 1280 131 to 5056 0.88 to 0.99; F = 8192 3480 1.10.
    // One block: F = 1536 131 rows 1.02, 722 1.01, 1116 1.01, 1904 0.99; F = 512 1.02, 1.01, 1.00, 1.00; two blocks 0.92 to 0.98.
    const int64_t round = 128 * (int64_t)num_cus(), beyond = F > 4 * C ? std::min(round / 9, 2 * (int64_t)(F - 4 * C)) : n_blocks == 1 ? round / 32 : 0;
    if (C == 384 && R > round && R - round < beyond) return false;
    return (C == 96 || C == 192 || C == 384) && F >= 2 * FC && F % FC == 0 && R >= 1 && R < (1 << 30) && (int64_t)F * C < (1 << 30);
}

size_t token_block_table_bytes(int C, int F) { return (size_t)TB_BYTES(C, F); }

hipError_t launch_token_tables(hipStream_t s, const TokenBlockArgs* a, int n) {
    TableJobs J;
    int nj = 0, most = 0;
    int64_t bytes = 0;
    auto job = [&](const int32_t* b, const int32_t* c, const int32_t* bias, const int8_t* dst, int off, int cnt, int kind, int arg) {
        J.j[nj] = TableJob{b, c, bias, reinterpret_cast<int32_t*>(const_cast<int8_t*>(dst) + off), cnt, kind};
        J.arg[nj] = arg;
        ++nj; most = std::max(most, cnt);
        bytes += cnt * (kind == 2 ? 16LL : bias ? 28LL : 24LL);
    };
    for (int i = 0; i < n; ++i) {
        const TokenBlockArgs& t = a[i];
        if (t.o) {
            job(t.ln2_g, t.ln2_b, nullptr, t.table, 0, t.C, 2, 1 << (t.ln2_c - 1));
            job(t.proj.rq_b, t.proj.rq_c, t.proj.bias, t.table, TB_PROJ(t.C), t.C, 1, t.C);
            job(t.fc2.rq_b, t.fc2.rq_c, t.fc2.bias, t.table, TB_FC2(t.C), t.C, 1, t.F);
            job(t.fc1.rq_b, t.fc1.rq_c, t.fc1.bias, t.table, TB_FC1(t.C), t.F, 0, 0);
        }
        if (t.next) job(t.ln1_g, t.ln1_b, nullptr, t.table, TB_LN1(t.C), t.C, 2, 1 << (t.ln1_c - 1));
        if (t.next == 2) job(t.qkv_w.rq_b, t.qkv_w.rq_c, t.qkv_w.bias, t.table, TB_QKV(t.C, t.F), 3 * t.C, 0, 0);
    }
    if (nj == 0) return hipSuccess;
    TraceScope trace(s, KIND_TOKEN_TABLES, 0, bytes);
    hipLaunchKernelGGL(table_kernel, dim3((unsigned)((most + 255) / 256), (unsigned)nj), dim3(256), 0, s, J);
    return hipGetLastError();
}

hipError_t launch_token_block(hipStream_t s, const TokenBlockArgs& a) {
    const int64_t cus = num_cus(), r = a.R;
    const int64_t per_row = (a.o ? (int64_t)a.C * a.C + 2LL * a.C * a.F : 0) + (a.next == 2 ? 3LL * a.C * a.C : 0);
    const int64_t row_bytes = (int64_t)a.C * ((a.o ? 3 : 1) + (a.next == 2 ? 3 : a.next == 1 ? 1 : 0));
    auto tile = [&](const TokenBlockArgs& t) -> hipError_t {
        TraceScope trace(s, KIND_TOKEN_BLOCK, 2 * t.R * per_row, per_row + t.R * row_bytes);
        // (us a launch, form with shared sets against the one for few rows: C = 384, 5122 rows 34.3 against 27.9, 8077 rows 38.0
        // against 32.8; C = 192, forwards of DeiT-T, batch 8 298 against 202, 40 330 against 237, 64 376 against 349, 83 396 against 366)
        if (token_stream_takes(t.C, t.F, t.R)) return launch_token_stream(s, t);
        if (t.C == 384) {
            if (t.R <= 32 * cus) return launch_tb<384, 1, 4>(s, t);
            if (t.R <= 64 * cus) return launch_tb<384, 2, 8>(s, t);
            return launch_tb<384, 4, 8>(s, t);
        }
        if (t.C == 192) return t.R <= 64 * cus ? launch_tb<192, 2, 4>(s, t) : launch_tb<192, 4, 8>(s, t);
        return launch_tb<96, 4, 4>(s, t);
    };
    // One workgroup fits a CU (C = 192, 384), so the last round of 128-row tiles takes as long as a full one however few rows
    // it has: what is left beyond full rounds goes to a launch with tiles of its own size (forwards: DeiT-S batch 192 2220 ->
    // 1930 us, batch 224 2250 -> 2060 us, DeiT-T batch 200 1042 -> 993 us, Swin-T batch 180 2796 -> 2586 us).
    const int64_t rest = r % (128 * cus);
    if (a.C == 96 || r < 128 * cus || rest == 0 || rest > 64 * cus) return tile(a);
    TokenBlockArgs t = a;
    t.R = r - rest;
    if (hipError_t e = tile(t)) return e;
    t.R = rest;
    auto skip = [&](auto& p, int64_t width) { if (p) p += (r - rest) * width; };
    skip(t.o, a.C); skip(t.x, a.C); skip(t.xhat, a.C); skip(t.y, a.C); skip(t.out, a.next == 2 ? 3 * a.C : a.C);
    return tile(t);
}

}  // namespace ivit
