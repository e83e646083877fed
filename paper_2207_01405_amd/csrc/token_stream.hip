// Everything of an encoder block that acts on single tokens, as one kernel (I-ViT, arXiv 2207.01405, Eq. 1-2 and 5 with the
// dyadic pipeline of Sec. 3.2, ShiftGELU of Sec. 3.4 and I-LayerNorm of Sec. 3.5), for few rows: what token_block.hip
// computes, with 32 or 64 tokens to a workgroup and F = 4 C.
//
// With so few tokens nothing that a compute unit fetches of a layer's weights is used twice, so weights need not be shared:
// wavefront w of the C / 32 takes channel tiles w, w + C / 32, ... of every layer and streams their rows through a ring in LDS
// that no other wavefront reads, two units of 3 to 6 KB, in an order that does not depend on the data.  No barrier stands in
// that stream, and it runs ahead across layers: the next layer's first units are requested before this layer's results are
// ready.  Barriers (seven) stand only where token rows change hands.  The whole hidden layer lies in LDS, and a wavefront's
// tile of xhat stays in its registers for the residual of the last layer.
//
// What bounds it at C = 384 is half the stream of weights and half what stands between its parts.  Of 50 to 52 thousand cycles of a
// workgroup (49 to 253 of them; read from the cycle counter in a copy) proj takes 3.0, the first MLP layer 11.2 to 13.0, the second 5.4 to 7.2
// and qkv 6.9, that is 460 cycles per 48 KB of weights in the second MLP layer, which has one epilogue, and 770 to 1080 in the others.  The first
// tiles and units take 5 to 6 to arrive, the two LayerNorms with their barriers 6.3, the results of the second MLP layer with theirs 6.0, and
// the barriers behind proj and the first MLP layer, where the slowest wavefront is waited for, 4.7.
// token_block.hip's buffers of 48 KB, one set in flight that first waits for a latency, took 34 us for 161 workgroups, this 28.
#include "token_block_common.hpp"

namespace ivit {
namespace {

using namespace tokblk;

template <int C, int TT> struct TsLayout {
    static constexpr int KS = C / 32, PP = C / 16, NW = KS, M = 32 * TT, F = 4 * C;
    static constexpr int G16 = gcd16(PP);
    static constexpr int KU = KS == 12 ? 4 : KS, UB = 32 * KU;      // k-steps of a unit of weights: 32 rows x UB bytes
    static constexpr int PU = 2 * KU, GU = gcd16(PU), UBYTES = 32 * UB, UL = UBYTES / 1024;
    static constexpr int PER = PU == 8 ? 2 : 3, PROWS = 64 * PER / PU;      // load instructions after which lanes repeat, their rows
    static constexpr int UT = KS / KU, FU = F / UB;                 // units of a channel tile, of K = F
    static constexpr int LPR = 2 * PP / 3, RPP = 64 / LPR, LNW = M / RPP;  // LayerNorm: lanes of a row, rows of a wavefront, wavefronts
    static constexpr int HP = M;                                    // hidden layer [channel][token]
    static constexpr int LUT = 0, RING = 256, ACT = RING + NW * 2 * UBYTES;      // (an index into the ShiftGELU table is its address)
    static constexpr int HID = ACT + M * C, X = HID, STG = HID + M * C;      // x, then xhat, and the staging tiles lie where the hidden layer will
    static constexpr int LN = HID + F * HP, SINK = LN + (8 * C + 1023) / 1024 * 1024, TOTAL = SINK + 256;
    static_assert(UL % PER == 0 && PROWS % 16 == 0 && KS % KU == 0 && F % UB == 0 && M % RPP == 0, "shape");
    static_assert(STG + NW * 1024 <= LN && TOTAL <= 160 * 1024, "LDS");
};

template <int C, int TT, bool FRONT>
__global__ __launch_bounds__(2 * C) void token_stream_kernel(TokenBlockArgs P) {
    using LY = TsLayout<C, TT>;
    constexpr int KS = LY::KS, PP = LY::PP, NW = LY::NW, M = LY::M, F = LY::F, G16 = LY::G16, KU = LY::KU, UB = LY::UB, UT = LY::UT, FU = LY::FU;
    constexpr int NX = G16 / 2 > 0 ? G16 / 2 : 1, NXU = LY::GU / 2 > 0 ? LY::GU / 2 : 1, HP = LY::HP;

    extern __shared__ __align__(1024) int8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane & 31, lg = lane >> 5, lb = lane >> 4;
    int8_t* const act = lds + LY::ACT;
    int8_t* const stg = lds + LY::STG + wv * 1024;
    const int64_t m0 = (int64_t)blockIdx.x * M;
    const int rows = __builtin_amdgcn_readfirstlane((int)min64(P.R - m0, M));
    const uint32_t lds0 = lds_offset(lds);
    const int8_t* const tab = P.table;

    auto sync_lds = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    auto buffer = [](const int8_t* p, uint32_t bytes) __attribute__((always_inline)) -> v4i {
        const uint64_t a = (uint64_t)uniform_ptr(p);
        return v4i{(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)bytes, 0x00020000};
    };
    auto uniform = [](uint32_t v) __attribute__((always_inline)) -> uint32_t { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
    // 16 bytes per lane from a buffer into LDS at lds + AT (the wait state is the one that such a load needs after m0 was written)
    auto load_lds = [](auto at_c, const v4i& buf, uint32_t off, uint32_t more, uint32_t dst) __attribute__((always_inline)) {
        asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     : : "s"(dst), "v"(off), "s"(buf), "s"(more), "i"(decltype(at_c)::value) : "memory", "m0", "scc");
    };

    // ---- token tiles: rows past the matrix read as zero (the buffer ends there).  LDS row i holds token
    // 32 (i / 32) + token_of_row(i % 32), its pieces permuted.
    auto load_tile = [&](const int8_t* src, int at) __attribute__((always_inline)) {
        constexpr int NI = M * PP / 64;
        const v4i r = buffer(src + m0 * C, (uint32_t)(rows * C));
        const uint32_t dst = uniform(lds0 + at + wv * 1024);
        static_for<(NI + NW - 1) / NW>([&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value;
            const int s = 64 * (NW * i + wv) + lane, row = s / PP, p = s % PP;
            const uint32_t v = (uint32_t)(((row & ~31) + token_of_row(row & 31)) * C + 16 * (p ^ swz<G16>(row)));
            if (NW * i + NW - 1 < NI || NW * i + wv < NI) load_lds(ic<i * NW * 1024>(), r, v, 0, dst);
        });
    };
    auto load_ln = [&](const int8_t* src) __attribute__((always_inline)) {       // gamma, beta: 8 C bytes, one after the other
        if (1024 * wv < 8 * C) dma16(uniform_ptr(src), (uint32_t)min(1024 * wv + 16 * lane, 8 * C - 16), lds0 + LY::LN + wv * 1024);
    };

    // ---- the wavefront's weights: units in the order of their use, unit u in half u % 2 of its ring.  A load instruction covers
    // 64 16-byte slots of [32 rows][PU pieces]; a row's pieces are permuted.
    constexpr int U1 = UT, U2 = 5 * UT, U3 = U2 + FU, NU = U3 + 3 * UT, FIRST = FRONT ? 0 : U3;      // first units of fc1, fc2, qkv
    uint32_t vc[LY::PER], vf[LY::PER];
#pragma unroll
    for (int i = 0; i < LY::PER; ++i) {
        const int s = 64 * i + lane, r = s / LY::PU, p = 16 * ((s % LY::PU) ^ swz<LY::GU>(r));
        vc[i] = (uint32_t)(r * C + p);
        vf[i] = (uint32_t)(r * F + p);
    }
    const uint32_t ring = uniform(lds0 + LY::RING + wv * 2 * LY::UBYTES);
    const v4i w_proj = buffer(P.proj.w + wv * 32 * C, 0x7fffffffu), w_fc1 = buffer(P.fc1.w + wv * 32 * C, 0x7fffffffu);
    const v4i w_fc2 = buffer(P.fc2.w + wv * 32 * F, 0x7fffffffu);
    const v4i w_qkv = buffer(P.qkv_w.w + wv * 32 * C, P.next == 2 ? 0x7fffffffu : 0u);      // (no layer: the loads read nothing)
    auto issue = [&](auto u_c) __attribute__((always_inline)) {
        constexpr int u = decltype(u_c)::value;
        if constexpr (u < NU) {
            constexpr bool f2 = u >= U2 && u < U3;
            constexpr int v = u < U1 ? u : u < U2 ? u - U1 : f2 ? u - U2 : u - U3, tile = f2 ? 0 : v / UT, col = f2 ? v : v % UT;
            static_for<LY::UL>([&](auto n_c) __attribute__((always_inline)) {
                constexpr int n = decltype(n_c)::value;
                constexpr uint32_t more = (uint32_t)(col * UB + tile * NW * 32 * C + (n / LY::PER) * LY::PROWS * (f2 ? F : C));
                load_lds(ic<(u & 1) * LY::UBYTES + n * 1024>(), u < U1 ? w_proj : u < U2 ? w_fc1 : f2 ? w_fc2 : w_qkv,
                         f2 ? vf[n % LY::PER] : vc[n % LY::PER], uniform(more), ring);
            });
        }
    };
    int bx[NXU];
#pragma unroll
    for (int i = 0; i < NXU; ++i) bx[i] = LY::RING + wv * 2 * LY::UBYTES + lj * UB + 16 * ((2 * i + lg) ^ swz<LY::GU>(lj));
    // unit u: its loads have arrived when at most those of unit u + 1 are outstanding (whatever else was requested since makes
    // the wait longer, not shorter); once its fragments are in registers its place takes unit u + 2
    auto unit = [&](auto u_c, auto use) __attribute__((always_inline)) {
        constexpr int u = decltype(u_c)::value;
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"(u + 1 < NU ? LY::UL : 0) : "memory");
        v4i f[KU];
#pragma unroll
        for (int k = 0; k < KU; ++k) f[k] = *reinterpret_cast<const v4i*>(lds + bx[k % NXU] + 16 * LY::GU * (k / NXU) + (u & 1) * LY::UBYTES);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int k = 0; k < KU; ++k) pin(f[k]);                     // (all of them read before the first is used)
        issue(ic<u + 2>());
        use(f);
    };

    // ---- the launch's weights and constants into this XCD's L2 (see token_block.hip): lines by wavefronts from `w0` on.  Not with
    // fewer than four workgroups on an XCD: DeiT-S batch 2 497 us with it, 386 without, batch 4 389 and 378.
    constexpr int WARM0 = LY::LNW < NW ? LY::LNW : 0;
    const uint32_t warm_n = min(max(gridDim.x / 8, 1u), 32u), warm_i = blockIdx.x / 8;
    auto warm = [&](const int8_t* p, uint32_t bytes, int w0) __attribute__((always_inline)) {
        if (warm_n >= 4 && warm_i < warm_n && wv >= w0)
            for (uint32_t at = ((warm_i * (NW - w0) + (wv - w0)) * 64 + lane) * 128; at < bytes; at += warm_n * (NW - w0) * 64 * 128)
                dma4(uniform_ptr(p), at, lds0 + LY::SINK);
    };

    // ---- residual and staging addresses (as in token_block.hip)
    const int jb = (lane & 15) >> 1, jo = lane & 1, dj = lane & 7, d_o = (lane >> 3) & 1;
    const int res_row = 8 * (jb >> 2) + 4 * lg + (jb & 3);          // + 16 h: row of the token of result 8 h + jb
    const int out_row = 16 * (lb & 1) + 8 * (dj >> 2) + 4 * (lb >> 1) + (dj & 3);      // row of token 8 lb + dj
    const int out_xor = swz<G16>(out_row), stg_x = (lj >> 2) & 3;
    const int stg_src = (16 * jo + jb) * 32 + 8 * (lb ^ (jb >> 2)), stg_src8 = (16 * jo + jb + 8) * 32 + 8 * (lb ^ (jb >> 2) ^ 2);
    auto tr8 = [](const int8_t* p) __attribute__((always_inline)) -> v2i {
        return __builtin_amdgcn_ds_read_tr8_b64_v2i32((v2i __attribute__((address_space(3)))*)(p));
    };
    // a channel tile's 32 x 32 results, lane (lj, lg) holding channel lj, turned into token rows.  Tokens of a lane: PERM 16 lg + e,
    // else 8 (e / 4) + 4 lg + e % 4.
    auto turn = [&](const v4i& w, auto perm_c) __attribute__((always_inline)) -> v4i {
        if constexpr (decltype(perm_c)::value) {
            v2i* d = reinterpret_cast<v2i*>(stg + lj * 32);
            d[(2 * lg) ^ stg_x] = v2i{w[0], w[1]}; d[(2 * lg + 1) ^ stg_x] = v2i{w[2], w[3]};
        } else {
            int* d = reinterpret_cast<int*>(stg + lj * 32 + 4 * lg);
#pragma unroll
            for (int u = 0; u < 4; ++u) d[2 * (u ^ stg_x)] = w[u];
        }
        const v2i a = tr8(stg + stg_src), b = tr8(stg + stg_src8);
        return v4i{a[0], a[1], b[0], b[1]};
    };
    auto put_rows = [&](int8_t* tile, int t, int ct, const v4i& w) __attribute__((always_inline)) {
        *reinterpret_cast<v4i*>(tile + (32 * t + out_row) * C + 16 * ((2 * ct + d_o) ^ out_xor)) = w;
    };

    // ---- a lane's 16 results of a tile in 64-bit arithmetic, channel ch of W; res: the residual's bytes, in the results' order
    auto slow = [&](const v16i& a, const DenseW& W, int ch, auto kind_c, Dyadic rr, const v4i& res) __attribute__((always_inline)) -> v4i {
        constexpr int kind = decltype(kind_c)::value;
        const int32_t b = W.rq_b[ch], c = W.rq_c[ch], bias = W.bias ? W.bias[ch] : 0;
        v4i w;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t o[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int64_t v = rnd_shift64(kind == EPI_RESIDUAL ? sum_of(a[4 * d + r], bias, kSumStart) : a[4 * d + r] + bias, b, c);
                if (kind == EPI_RESIDUAL) v += rnd_shift64((int32_t)(int8_t)((uint32_t)res[d] >> (8 * r)), rr.b, rr.c);
                o[r] = (uint32_t)clamp8_64(v);
                if (kind == EPI_GELU) o[r] = (uint32_t)(uint8_t)lds[LY::LUT + (o[r] & 0xffu)];
            }
            w[d] = pack4<true>(o);
        }
        return w;
    };
    auto residual_words = [&](const v16i& a, const v4i& cst, const DenseW& W, int ch, Dyadic rd, const ResRq& rr, const v4i& res) __attribute__((always_inline)) -> v4i {
        const Rq64 q = as_rq64(cst);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(q.b != 0 && rr.ok) != ~0ull, 0)) return slow(a, W, ch, ic<EPI_RESIDUAL>(), rd, res);
        v4i w;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            uint32_t o[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = out_res(a[4 * d + r], q, rr, (int32_t)(int8_t)((uint32_t)res[d] >> (8 * r)));
            w[d] = pack4<true>(o);
        }
        return w;
    };

    // ---- I-LayerNorm of the tile at `src`, to `dst`: LNW wavefronts' worth of rows, LPR lanes a row, three half pieces each.  `raw`: the rows
    // before normalisation also go to global memory, `out`: the normalised ones do
    auto layernorm_rows = [&](int w0, const int8_t* src, int8_t* dst, int f_bits, int c_shift, int8_t* raw, int8_t* out) __attribute__((always_inline)) {
        constexpr int LPR = LY::LPR;
        const int q = lane % LPR, i = w0 * LY::RPP + lane / LPR, tok = (i & ~31) + token_of_row(i & 31);
        const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(uniform_ptr(raw + m0 * C)), 0, raw ? rows * C : 0, 0x00020000);
        const __amdgpu_buffer_rsrc_t ob = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(uniform_ptr(out + m0 * C)), 0, out ? rows * C : 0, 0x00020000);
        // lane q of a row has its 8-byte pieces q, q + LPR, q + 2 LPR
        auto at = [&](int j) __attribute__((always_inline)) { return i * C + 16 * (((q + LPR * j) >> 1) ^ swz<G16>(i)) + 8 * (q & 1); };
        v2i v[3];
        int32_t s = 0, ss = 0;
#pragma unroll
        for (int j = 0; j < 3; ++j) v[j] = *reinterpret_cast<const v2i*>(src + at(j));
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if (raw) __builtin_amdgcn_raw_buffer_store_b64(v[j], rb, tok * C + 8 * (q + LPR * j), 0, 0);
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                s = __builtin_amdgcn_sdot4(v[j][d], 0x01010101, s, false);
                ss = __builtin_amdgcn_sdot4(v[j][d], v[j][d], ss, false);
            }
        }
        s += dpp_i32<0xB1>(s); ss += dpp_i32<0xB1>(ss);
        if (LPR >= 4) { s += dpp_i32<0x4E>(s); ss += dpp_i32<0x4E>(ss); }
        if (LPR >= 8) { s += dpp_i32<0x141>(s); ss += dpp_i32<0x141>(ss); }
        if (LPR >= 16) { s += dpp_i32<0x140>(s); ss += dpp_i32<0x140>(ss); }
        const LnStat st = ln_stat(s, ss, C, f_bits);
        const int32_t* gt = reinterpret_cast<const int32_t*>(lds + LY::LN);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            v2i w;
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const v4i g = *reinterpret_cast<const v4i*>(gt + 8 * (q + LPR * j) + 4 * d);
                const v4i b = *reinterpret_cast<const v4i*>(gt + C + 8 * (q + LPR * j) + 4 * d);
                uint32_t o[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) o[r] = (uint32_t)ln_value((int32_t)(int8_t)((uint32_t)v[j][d] >> (8 * r)), st, g[r], b[r], c_shift);
                w[d] = pack4<true>(o);
            }
            if (out) __builtin_amdgcn_raw_buffer_store_b64(w, ob, tok * C + 8 * (q + LPR * j), 0, 0);
            *reinterpret_cast<v2i*>(dst + at(j)) = w;
        }
    };

    auto layernorm = [&](const int8_t* src, int8_t* dst, int f_bits, int c_shift, int8_t* raw, int8_t* out) __attribute__((always_inline)) {
#pragma unroll 1
        for (int w = wv; w < LY::LNW; w += NW) layernorm_rows(w, src, dst, f_bits, c_shift, raw, out);
    };

    // ---- products of a channel tile, K = C: units u .. u + UT - 1 with the activations in registers
    v4i ar[TT][KS];
    auto load_ar = [&]() __attribute__((always_inline)) {
        int xr[NX];
#pragma unroll
        for (int i = 0; i < NX; ++i) xr[i] = lj * C + 16 * ((2 * i + lg) ^ swz<G16>(lj));
#pragma unroll
        for (int t = 0; t < TT; ++t)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) ar[t][ks] = *reinterpret_cast<const v4i*>(act + 32 * t * C + xr[ks % NX] + 16 * G16 * (ks / NX));
    };
    auto products = [&](auto u_c, v16i (&acc)[TT]) __attribute__((always_inline)) {
        static_for<UT>([&](auto col_c) __attribute__((always_inline)) {
            constexpr int col = decltype(col_c)::value;
            unit(ic<decltype(u_c)::value + col>(), [&](const v4i (&f)[KU]) __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k < KU; ++k)
#pragma unroll
                    for (int t = 0; t < TT; ++t) acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(ar[t][col * KU + k], f[k], acc[t], 0, 0, 0);
            });
        });
    };
    auto constants = [&](int at, int ct) __attribute__((always_inline)) -> v4i { return *reinterpret_cast<const v4i*>(tab + at + 16 * (32 * ct + lj)); };

    if constexpr (FRONT) {
        warm(P.fc1.w, F * C, 0);
        warm(tab, TB_BYTES(C, F), 0);
        load_tile(P.o, LY::ACT);
        load_tile(P.x, LY::X);
        load_ln(tab);
        v4i cp = constants(TB_PROJ(C), wv);
        issue(ic<0>()); issue(ic<1>());
        if (wv < 4) lds[LY::LUT + tid] = (int8_t)requant64(shiftgelu_raw((int32_t)(int8_t)tid, P.gelu_p), P.gelu_rq.b, P.gelu_rq.c);
        pin(cp);
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");      // (one latency, whatever was requested)
        load_ar();
        // ---- proj, xhat in the place of x
        const ResRq rr1 = make_res(P.res1), rr2 = make_res(P.res2);
        v16i acc[TT];
        v4i xh[TT];
#pragma unroll
        for (int t = 0; t < TT; ++t) acc[t] = sums_from(kSumStart);
        products(ic<0>(), acc);
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            const int8_t* tile = lds + LY::X + 32 * t * C;
            v2i rw[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int r = res_row + 16 * h;
                rw[h] = tr8(tile + r * C + 16 * ((2 * wv + (lb & 1)) ^ swz<G16>(r)) + 8 * jo);
            }
            xh[t] = residual_words(acc[t], cp, P.proj, 32 * wv + lj, P.res1, rr1, v4i{rw[0][0], rw[0][1], rw[1][0], rw[1][1]});
            put_rows(lds + LY::X, t, wv, turn(xh[t], std::true_type()));
        }
        v4i c1[4], c2 = constants(TB_FC2(C), wv);
#pragma unroll
        for (int j = 0; j < 4; ++j) c1[j] = constants(TB_FC1(C), j * NW + wv);
        sync_lds();
        // ---- LN2; the wavefronts that have no part in it request the rest of the launch's weights into L2
        layernorm(lds + LY::X, act, P.ln2_f, P.ln2_c, nullptr, nullptr);
        pin(c2);
#pragma unroll
        for (int j = 0; j < 4; ++j) pin(c1[j]);
        warm(P.fc2.w, F * C, WARM0);
        if (P.next == 2) warm(P.qkv_w.w, 3 * C * C, WARM0);
        sync_lds();
        if (P.next) load_ln(tab + TB_LN1(C));
        load_ar();
        // ---- fc1, ShiftGELU: the hidden layer, [channel][token]
        static_for<4>([&](auto j_c) __attribute__((always_inline)) {
            constexpr int j = decltype(j_c)::value;
#pragma unroll
            for (int t = 0; t < TT; ++t) acc[t] = v16i{};
            products(ic<U1 + j * UT>(), acc);
            const Rq q = as_rq(c1[j]);
            const int ch = 32 * (j * NW + wv) + lj;
            const bool fast = __builtin_amdgcn_ballot_w64(q.lo <= q.hi) == ~0ull;
#pragma unroll
            for (int t = 0; t < TT; ++t) {
                v4i w;
                if (__builtin_expect(fast, 1)) {
                    uint32_t o[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const uint32_t at = out_top(acc[t][e], q) >> 24;
                        o[e] = *reinterpret_cast<const __attribute__((address_space(3))) uint8_t*>(at);
                    }
#pragma unroll
                    for (int d = 0; d < 4; ++d) { const uint32_t o4[4] = {o[4 * d], o[4 * d + 1], o[4 * d + 2], o[4 * d + 3]}; w[d] = pack4<true>(o4); }
                } else {
                    w = slow(acc[t], P.fc1, ch, ic<EPI_GELU>(), Dyadic{}, v4i{});
                }
                *reinterpret_cast<v4i*>(lds + LY::HID + ch * HP + 32 * t + 16 * lg) = w;
            }
        });
        sync_lds();
        // ---- fc2
#pragma unroll
        for (int t = 0; t < TT; ++t) acc[t] = sums_from(kSumStart);
        const int8_t* const h0 = lds + LY::HID + (16 * lg + jb) * HP + 16 * (lb & 1) + 8 * jo;
        static_for<FU>([&](auto v_c) __attribute__((always_inline)) {
            constexpr int v = decltype(v_c)::value;
            v4i af[KU][TT];
#pragma unroll
            for (int k = 0; k < KU; ++k)
#pragma unroll
                for (int t = 0; t < TT; ++t) {
                    const int8_t* p = h0 + 32 * (v * KU + k) * HP + 32 * t;
                    const v2i a = tr8(p), b = tr8(p + 8 * HP);
                    af[k][t] = v4i{a[0], a[1], b[0], b[1]};
                }
            unit(ic<U2 + v>(), [&](const v4i (&f)[KU]) __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k < KU; ++k)
#pragma unroll
                    for (int t = 0; t < TT; ++t) acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[k][t], f[k], acc[t], 0, 0, 0);
            });
        });
        sync_lds();                                                 // (the staging tiles lie where the hidden layer was)
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            // xhat from a lane's tokens 16 lg + e to 8 (e / 4) + 4 lg + e % 4: words 1 and 3 of the lower half change places with
            // words 0 and 2 of the upper one
            const auto s0 = __builtin_amdgcn_permlane32_swap((uint32_t)xh[t][0], (uint32_t)xh[t][1], false, false);
            const auto s1 = __builtin_amdgcn_permlane32_swap((uint32_t)xh[t][2], (uint32_t)xh[t][3], false, false);
            const v4i w = residual_words(acc[t], c2, P.fc2, 32 * wv + lj, P.res2, rr2, v4i{(int)s0[0], (int)s1[0], (int)s0[1], (int)s1[1]});
            put_rows(act, t, wv, turn(w, std::false_type()));
        }
        sync_lds();
    } else {
        load_tile(P.x, LY::ACT);
        load_ln(tab + TB_LN1(C));
        issue(ic<FIRST>()); issue(ic<FIRST + 1>());
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(2 * LY::UL) : "memory");
        warm(P.qkv_w.w, 3 * C * C, WARM0);
        warm(tab, TB_BYTES(C, F), WARM0);
    }
    if (!P.next) {                                                  // only the block's output leaves
        constexpr int NI = M * PP / 64;
        const __amdgpu_buffer_rsrc_t yb = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(uniform_ptr(P.y + m0 * C)), 0, rows * C, 0x00020000);
#pragma unroll
        for (int i = 0; i < (NI + NW - 1) / NW; ++i) {
            const int s = 64 * (NW * i + wv) + lane, r = s / PP, p = s % PP;
            if (s < M * PP) __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const v4i*>(act + r * C + 16 * (p ^ swz<G16>(r))), yb,
                                                                  ((r & ~31) + token_of_row(r & 31)) * C + 16 * p, 0, 0);
        }
        wait_vm0();
        return;
    }
    v4i c3[3] = {};
    if (P.next == 2) {
#pragma unroll
        for (int j = 0; j < 3; ++j) c3[j] = constants(TB_QKV(C, F), j * NW + wv);
    }
    layernorm(act, act, P.ln1_f, P.ln1_c, FRONT ? P.y : nullptr, P.next == 1 ? P.out : nullptr);
    if (P.next == 1) { wait_vm0(); return; }
#pragma unroll
    for (int j = 0; j < 3; ++j) pin(c3[j]);
    sync_lds();
    load_ar();
    // ---- qkv of the next block
    const int N3 = 3 * C;
    const __amdgpu_buffer_rsrc_t qb = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(uniform_ptr(P.out + m0 * N3)), 0, rows * N3, 0x00020000);
    static_for<3>([&](auto j_c) __attribute__((always_inline)) {
        constexpr int j = decltype(j_c)::value;
        v16i acc[TT];
#pragma unroll
        for (int t = 0; t < TT; ++t) acc[t] = v16i{};
        products(ic<U3 + j * UT>(), acc);
        const Rq q = as_rq(c3[j]);
        const int ct = j * NW + wv;
        const bool fast = __builtin_amdgcn_ballot_w64(q.lo <= q.hi) == ~0ull;
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            v4i w;
            if (__builtin_expect(fast, 1)) {
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const uint32_t o[4] = {out_top(acc[t][4 * d], q), out_top(acc[t][4 * d + 1], q), out_top(acc[t][4 * d + 2], q), out_top(acc[t][4 * d + 3], q)};
                    w[d] = pack4<false>(o);
                }
            } else {
                w = slow(acc[t], P.qkv_w, 32 * ct + lj, ic<EPI_PLAIN>(), Dyadic{}, v4i{});
            }
            __builtin_amdgcn_raw_buffer_store_b128(turn(w, std::true_type()), qb, (32 * t + 8 * lb + dj) * N3 + 32 * ct + 16 * d_o, 0, 0);
        }
    });
}

template <int C, int TT>
hipError_t launch_ts(hipStream_t s, const TokenBlockArgs& a) {
    using LY = TsLayout<C, TT>;
    const dim3 g((unsigned)((a.R + LY::M - 1) / LY::M)), b(64 * LY::NW);
    if (a.o) hipLaunchKernelGGL((token_stream_kernel<C, TT, true>), g, b, LY::TOTAL, s, a);
    else hipLaunchKernelGGL((token_stream_kernel<C, TT, false>), g, b, LY::TOTAL, s, a);
    return hipGetLastError();
}

}  // namespace

// One round of workgroups: 32 tokens a CU at width 384, where the weights' rings and the hidden layer of 64 do not fit the LDS, and
// 64 at width 192.  A second round costs as much as the first (both sides at launch_token_block).  Two workgroups of 32 tokens on
// a CU, with units of 3 KB, are no faster than one of 64: DeiT-T batch 64 349 us either way, batch 83 391 against 366.
bool token_stream_takes(int C, int F, int64_t R) {
    if (F != 4 * C) return false;
    return (C == 384 && R <= 32 * (int64_t)num_cus()) || (C == 192 && R <= 64 * (int64_t)num_cus());
}

hipError_t launch_token_stream(hipStream_t s, const TokenBlockArgs& a) {
    if (a.C == 384) return launch_ts<384, 1>(s, a);
    return a.R <= 32 * (int64_t)num_cus() ? launch_ts<192, 1>(s, a) : launch_ts<192, 2>(s, a);
}

}  // namespace ivit
