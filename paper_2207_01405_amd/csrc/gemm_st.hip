// int8 x int8 -> int32 Dense / MatMul on the gfx950 matrix cores with the dyadic requantisation of I-ViT (arXiv
// 2207.01405, Sec. 3.2, Eq. 7-10) fused into the epilogue, optionally with the residual add of Eq. 1-2 or with ShiftGELU
// (Sec. 3.4, Algorithm 2) and its rescale: the form for any K % 16 == 0, any N and any number of rows.
//
// A workgroup of GM x GN wavefronts (2 x 2 or eight) computes one tile of 32 MT GM tokens x 32 NT GN channels.  Both operands stream
// through S LDS stages of 128 bytes of K, filled by LDS-direct loads S - 1 stages ahead (no register pass, one barrier
// per stage); 16-byte pieces of a row are permuted by an XOR with bits of the row number, which costs the loads nothing
// and spreads the fragment reads over the banks.  Several workgroups share a compute unit, so one's prologue and
// epilogue run under another's multiplies.  The weights are the MFMA "A" operand and the loads put the channel rows in
// such an order that a lane ends up with 16 NT consecutive channels of one token: results leave as 16-byte stores at
// whatever alignment the row has.
#include <type_traits>

#include "dense_form.hpp"
#include "linear_rows.hpp"
#include "regst_common.hpp"

namespace ivit {
namespace {

using namespace regst;

constexpr int BK = 128;                       // bytes of K per stage

struct StParams {
    const int8_t* x; const int8_t* w; const int32_t* bias; const int32_t* rq_b; const int32_t* rq_c;
    const int8_t* residual; Dyadic res_rq; ShiftParams gelu_p; Dyadic gelu_rq;
    int8_t* y; int64_t M; int N; int K; FastDiv inner; uint32_t tiles, per_xcd; int m_fast;      // inner: tiles in the dimension that runs fastest
    int64_t ldx;                              // bytes between rows of x
    int rnd;                                  // 1: round to nearest, 0: floor (every requantisation of the epilogue)
    const int32_t* ln_g; const int32_t* ln_b; int ln_f, ln_c;   // XS > 0: I-LayerNorm of the rows of x
};

typedef int v4i_w __attribute__((ext_vector_type(4), aligned(4)));     // 16 bytes at any address of words
typedef int v4i_any __attribute__((ext_vector_type(4), aligned(1)));   // 16 bytes at any address

// 16 bytes per lane from a buffer into LDS at lds + AT (the wait state is the one that such a load needs after m0 was written)
template <int AT> __device__ __forceinline__ void load_lds(const v4i& buf, uint32_t off, uint32_t more, uint32_t lds) {
    asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 : : "s"(lds), "v"(off), "s"(buf), "s"(more), "i"(AT) : "memory", "m0", "scc");
}

// every load but the newest N of this wavefront has arrived, its LDS reads have returned, and so for all wavefronts
template <int N> __device__ __forceinline__ void arrive() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}

// XS > 0: the rows of x are normalised first (I-LayerNorm, Sec. 3.5, Eq. 19-20).  The token rows of the tile, all of K
// (K <= 128 XS), are fetched at once and stay in LDS, where they are normalised in place; only the weights stream.  Every
// workgroup of a row of tiles repeats that work, so the four wavefronts stand side by side: 32 tokens x 128 channels.
template <int MT, int NT, int XS, int GM = 2, int GN = 2> struct StTile {
    static constexpr int WGM = XS > 0 ? 1 : GM, WGN = XS > 0 ? 4 : GN, W = WGM * WGN, TM = 32 * MT * WGM, TN = 32 * NT * WGN;
    static_assert(TM % (8 * W) == 0 && TN % (8 * W) == 0 && W % 2 == 0, "a load instruction of all wavefronts fills rows of one operand");
};

template <int EPI, int MT, int NT, int S, int XS, int GM, int GN>
__global__ __launch_bounds__((64 * StTile<MT, NT, XS, GM, GN>::W), 2) void gemm_st_kernel(StParams P) {
    using TL = StTile<MT, NT, XS, GM, GN>;
    constexpr int W = TL::W, TM = TL::TM, TN = TL::TN, XI = XS > 0 ? TM / 32 : TM / (8 * W), WI = TN / (8 * W);
    constexpr int DPX = XS > 0 ? 0 : XI, DPW = DPX + WI;           // load instructions of a wavefront and streamed stage: of x, in all
    constexpr int XB = XS * TM * BK, WR = XS > 0 ? 0 : TM, STG = (WR + TN) * BK;    // resident bytes of x; rows of x in a streamed stage
    __shared__ __align__(16) int8_t lds[XB + S * STG];
    __shared__ __align__(16) int32_t qb_s[TN], qc_s[TN], bias_s[TN];
    __shared__ __align__(16) v4i cst[TN];     // a channel's factor, 0, and the two words of its addend (Residual64 of regst_common.hpp)
    __shared__ int8_t gelu_lut[256];          // of the results -128 .. 127

    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 31, lg = lane >> 5, wm = wv / TL::WGN, wn = wv % TL::WGN;

    // each XCD takes a contiguous range of tiles; the operand with fewer rows runs fastest, so that the other one is read by
    // few XCDs
    const uint32_t tile = (blockIdx.x % NXCD) * P.per_xcd + blockIdx.x / NXCD;
    if (tile >= P.tiles) return;
    uint32_t in;
    const uint32_t out = P.inner.divide(tile, in);
    const int64_t m0 = (int64_t)(P.m_fast ? in : out) * TM;
    const int n0 = (int)(P.m_fast ? out : in) * TN;
    const int K = P.K, N = P.N;
    const int rows = (int)min64(P.M - m0, TM);

    // this lane's outputs: tokens row0 + 32 tt, channels n_l + 16 ct .. + 15
    const int row0 = wm * 32 * MT + li, cl = wn * 32 * NT + 16 * NT * lg, n_l = n0 + cl;
    v4i res[MT][NT] = {};
    if (EPI == EPI_RESIDUAL) {                // requested first: the wait for the first stage covers them
#pragma unroll
        for (int tt = 0; tt < MT; ++tt)
#pragma unroll
            for (int ct = 0; ct < NT; ++ct)
                if (row0 + 32 * tt < rows && n_l + 16 * ct + 16 <= N)
                    res[tt][ct] = *reinterpret_cast<const v4i_any*>(P.residual + (m0 + row0 + 32 * tt) * N + n_l + 16 * ct);
    }

    // the channels' constants, 64 channels a wavefront
    if (wv < TN / 64) {
        const uint32_t off = 4u * min(n0 + 64 * wv + lane, N - 1);
        auto fetch = [&](const int32_t* src, int32_t* dst) __attribute__((always_inline)) {
            dma4(uniform_ptr(reinterpret_cast<const int8_t*>(src)), off, lds_offset(reinterpret_cast<const int8_t*>(dst + 64 * wv)));
        };
        fetch(P.rq_b, qb_s); fetch(P.rq_c, qc_s);
        if (P.bias) fetch(P.bias, bias_s); else bias_s[64 * wv + lane] = 0;
    }

    // I-LayerNorm: a thread normalises piece n_p of rows n_r, n_r + n_rows, ...; its 16 channels' parameters are requested now
    const int pieces = K >> 4, n_rows = 256 / max(pieces, 4), n_r = tid / pieces, n_p = tid - n_r * pieces;
    v4i g[4] = {}, bt[4] = {};
    if (XS > 0 && n_r < n_rows) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            g[e] = *reinterpret_cast<const v4i_w*>(P.ln_g + 16 * n_p + 4 * e);
            bt[e] = *reinterpret_cast<const v4i_w*>(P.ln_b + 16 * n_p + 4 * e);
        }
    }

    // (32-bit offsets from the tile's first row: linear_rows_per_launch sees to it that they are enough)
    // Load instruction i of a wavefront fills LDS rows 8 W i + r, r = 8 wavefront + lane / 8, eight lanes a row; the lane
    // lands in physical piece lane % 8 and fetches piece (lane % 8) ^ ((r / 2) % 8).  Rows past the last token or channel
    // repeat it (never stored), pieces past the end of a row its last piece (never multiplied, see below).
    const int ld_r = 8 * wv + (lane >> 3), ld_col = 16 * ((lane & 7) ^ ((ld_r >> 1) & 7));
    const int8_t* xg = uniform_ptr(P.x + m0 * P.ldx);
    const int8_t* wg = uniform_ptr(P.w + (int64_t)n0 * K);
    uint32_t off[XI + WI];
#pragma unroll
    for (int i = 0; i < XI + WI; ++i) {
        if (i < XI) {
            off[i] = (uint32_t)min(8 * W * i + ld_r, rows - 1) * (uint32_t)P.ldx + ld_col;
        } else {
            // row 8 q + 4 g + r of MFMA tile ct holds channel 16 NT g + 16 ct + 4 q + r of the wavefront's 32 NT: that is
            // accumulator register 4 q + r of lane group g
            const int R = 8 * W * (i - XI) + ld_r, ct = (R >> 5) % NT, rr = R & 31;
            const int ch = (R / (32 * NT)) * 32 * NT + 16 * NT * ((rr >> 2) & 1) + 16 * ct + 4 * (rr >> 3) + (rr & 3);
            off[i] = (uint32_t)min(ch, N - 1 - n0) * (uint32_t)K + ld_col;
        }
    }
    auto buffer = [](const int8_t* p) __attribute__((always_inline)) {
        const uint64_t a = (uint64_t)p;
        return v4i{(int)(uint32_t)a, (int)(uint32_t)(a >> 32), (int)kTileBytes, 0x00020000};
    };
    const int stages = (K + BK - 1) / BK, k_last = K - (stages - 1) * BK;      // bytes of K in the last stage: 16 .. 128
    const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_offset(lds) + XB + wv * 1024));
    if (XS > 0) {
#pragma unroll 1
        for (int s = 0; s < stages; ++s) {
            const uint32_t end = s == stages - 1 ? (uint32_t)max(ld_col - (k_last - 16), 0) : 0u;
#pragma unroll
            for (int i = 0; i < XI; ++i) dma16(xg + s * BK, off[i] - end, lds0 - XB + s * TM * BK + i * 4096);
        }
    }
    // A stage's loads: stage `is` goes to buffer is % S, known where the loads stand.  A lane whose piece lies past the end of
    // the rows moves back to the last one (the last stage only).  One scalar offset serves both operands.
    const int back = max(ld_col - (k_last - 16), 0), moves = k_last < BK ? stages - 1 : -1;
    const v4i x_buf = buffer(xg), w_buf = buffer(wg);
    int is = 0;
    uint32_t k_off = 0;
    auto issue_one = [&](auto i_c, auto buf_c) __attribute__((always_inline)) {
        constexpr int i = decltype(i_c)::value;
        load_lds<decltype(buf_c)::value * STG + i * W * 1024>(i < DPX ? x_buf : w_buf, off[XI - DPX + i], k_off, lds0);
    };
    auto issue_begin = [&]() __attribute__((always_inline)) {
        if (is == moves) {
#pragma unroll
            for (int i = XI - DPX; i < XI + WI; ++i) off[i] -= back;
        }
    };
    auto issue_done = [&]() __attribute__((always_inline)) { ++is; k_off += BK; };
    static_for<S - 1>([&](auto buf) __attribute__((always_inline)) {
        if (decltype(buf)::value < stages) {
            issue_begin();
            static_for<DPW>([&](auto i) __attribute__((always_inline)) { issue_one(i, buf); });
            issue_done();
        }
    });
    if (EPI == EPI_GELU && tid < 256) {
        const int32_t I = (int32_t)(int8_t)tid;
        gelu_lut[(uint8_t)(I + 128)] = (int8_t)requant64(shiftgelu_raw(I, P.gelu_p), P.gelu_rq.b, P.gelu_rq.c, P.rnd);
    }
    // a result is the high word of one 64-bit multiply-add, whatever the epilogue; with ShiftGELU it comes as 0 .. 255.  The epilogue
    // of 16 results is 104 vector instructions with a residual (217 when every result needed its own shift and residual product).
    if (wv < TN / 64) {
        if (stages >= S - 1) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"((S - 1) * DPW) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        const int ch = 64 * wv + lane;
        const int32_t b = qb_s[ch], c = qc_s[ch], bias = bias_s[ch];
        Residual64 q;
        bool ok = residual64_of(q, b, c, bias, P.rnd);
        // (the 128 must not carry a result out of int32: it is at most 2^30 for b < 2^(c-1), and |acc| at most 2^30)
        if (EPI == EPI_GELU) ok &= (b < (1 << ((c - 1) & 31))) | ((uint32_t)bias + 0x3fffff00u < 0x7ffffe00u);
        cst[ch] = v4i{ok ? (int32_t)q.b : 0, 0, (int32_t)(uint32_t)q.h, (int32_t)((uint32_t)(q.h >> 32) + (EPI == EPI_GELU ? 128u : 0u))};
    }

    if constexpr (XS > 0) {
        __shared__ int2 stat[TM];                          // (mean, f) of a row
        if (stages >= S - 1) arrive<(S - 1) * DPW>(); else arrive<0>();
        auto at = [&](int row, int p) __attribute__((always_inline)) {      // piece p of a row
            return reinterpret_cast<v4i*>(lds + (p >> 3) * TM * BK + row * BK + 16 * ((p & 7) ^ ((row >> 1) & 7)));
        };
        constexpr int TPR = 256 / TM;                      // threads that add up a row
        static_assert(TPR == 8, "lanes of a row");
        const int row = tid / TPR;
        int32_t sm = 0, sq = 0;
        for (int p = tid % TPR; p < pieces; p += TPR) {
            const v4i v = *at(row, p);
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                sm = __builtin_amdgcn_sdot4(v[d], 0x01010101, sm, false);
                sq = __builtin_amdgcn_sdot4(v[d], v[d], sq, false);
            }
        }
        sm += dpp_i32<0xB1>(sm); sq += dpp_i32<0xB1>(sq);
        sm += dpp_i32<0x4E>(sm); sq += dpp_i32<0x4E>(sq);
        sm += dpp_i32<0x141>(sm); sq += dpp_i32<0x141>(sq);
        const LnStat st = ln_stat(sm, sq, K, P.ln_f);
        if (tid % TPR == 0) stat[row] = make_int2(st.mean, st.f);
        __syncthreads();
        if (n_r < n_rows) {
            const int32_t half = 1 << (P.ln_c - 1);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int r = 0; r < 4; ++r) bt[e][r] = (int32_t)((uint32_t)bt[e][r] + (uint32_t)half);
#pragma unroll 1
            for (int i = n_r; i < TM; i += n_rows) {
                const int2 mf = stat[i];
                const LnStat st{mf.x, mf.y};
                const v4i v = *at(i, n_p);
                v4i w;
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    uint32_t o[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int32_t xe = (int32_t)(int8_t)((uint32_t)v[d] >> (8 * r));
                        o[r] = (uint32_t)ln_value(xe, st, g[d][r], bt[d][r], P.ln_c);
                    }
                    w[d] = (int)(__builtin_amdgcn_perm(o[1], o[0], 0x0c0c0400u) | __builtin_amdgcn_perm(o[3], o[2], 0x04000c0cu));
                }
                *at(i, n_p) = w;
            }
        }
        // (the barrier of the first stage is the one that makes the normalised rows everybody's)
    }

    v16i acc[NT][MT];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
        for (int tt = 0; tt < MT; ++tt) acc[ct][tt] = sums_from(kSumStart);
    constexpr int KS = BK / 32, AHEAD = MT * NT == 1 ? KS : 2;      // fragments are read AHEAD k-steps before their use
    int fx[KS], fw[KS];                                   // where this lane's fragments of k-step kk lie (buffer 0)
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
        const int col = 16 * ((2 * kk + lg) ^ ((li >> 1) & 7));
        fx[kk] = (XS > 0 ? 0 : XB) + row0 * BK + col;
        fw[kk] = XB + (WR + wn * 32 * NT + li) * BK + col;
    }
    struct Frag { v4i a[NT], b[MT]; };
    auto read_frag = [&](Frag& f, int kk, int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) f.a[ct] = *reinterpret_cast<const v4i*>(lds + fw[kk] + buf * STG + ct * 32 * BK);
#pragma unroll
        for (int tt = 0; tt < MT; ++tt) f.b[tt] = *reinterpret_cast<const v4i*>(lds + fx[kk] + (XS > 0 ? 0 : buf * STG) + tt * 32 * BK);
    };
    auto multiply = [&](const Frag& f) __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct)
#pragma unroll
            for (int tt = 0; tt < MT; ++tt) acc[ct][tt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.a[ct], f.b[tt], acc[ct][tt], 0, 0, 0);
    };
    // Stage s: its loads have arrived when at most those of the later stages requested so far (S - 2, fewer at the end)
    // are outstanding; behind the barrier nobody reads stage s - 1 any more and its buffer takes stage s + S - 1.  Those
    // loads go out behind the first fragment reads.  The loop is written out for the S buffers, so that addresses are constants
    // and a stage of a 64 x 64 tile is 48 instructions instead of 70 (1576 x 2304 x 768 6.6 -> 6.0 us, 197 x 384 x 1536 5.4 -> 5.2).
    // What bounds it then is the LDS: a 64 x 64 stage writes 16 KB and reads 32 KB, 384 cycles at 128 bytes a cycle, for 128
    // cycles of products; the loads would come at 64 bytes a cycle and CU.
    auto wait_stage = [&](int left) __attribute__((always_inline)) {      // left: stages after this one
        if (S == 2 || left == 0) arrive<0>();
        else if (S == 3 || left == 1) arrive<DPW>();
        else if (S == 4 || left == 2) arrive<2 * DPW>();
        else arrive<3 * DPW>();
    };
    int s = 0;
    const int full = k_last == BK ? stages : stages - 1;  // a last stage of less than 128 bytes comes after the loop
    auto body = [&](auto buf_c) __attribute__((always_inline)) {
        constexpr int buf = decltype(buf_c)::value;
        wait_stage(stages - 1 - s);
        Frag f[AHEAD];
        static_for<AHEAD - 1>([&](auto kk) __attribute__((always_inline)) { read_frag(f[decltype(kk)::value], decltype(kk)::value, buf); });
        if (is < stages) {
            issue_begin();
            static_for<DPW>([&](auto i) __attribute__((always_inline)) { issue_one(i, std::integral_constant<int, (buf + S - 1) % S>()); });
            issue_done();
        }
        static_for<KS>([&](auto kk_c) __attribute__((always_inline)) {
            constexpr int kk = decltype(kk_c)::value;
            if constexpr (kk + AHEAD - 1 < KS) read_frag(f[(kk + AHEAD - 1) % AHEAD], kk + AHEAD - 1, buf);
            multiply(f[kk % AHEAD]);
        });
        if (XS > 0) {
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) fx[kk] += TM * BK;
        }
        ++s;
    };
#pragma unroll 1
    while (s < full)
        static_for<S>([&](auto buf) __attribute__((always_inline)) { if (s < full) body(buf); });
    if (full < stages) {                                  // what is left of K; of its last 32 bytes maybe the first half only
        arrive<0>();
        const int buf = s % S;
        static_for<KS>([&](auto kk_c) __attribute__((always_inline)) {
            constexpr int kk = decltype(kk_c)::value;
            if (32 * kk >= k_last) return;
            Frag f;
            read_frag(f, kk, buf);
            if (32 * kk + 16 >= k_last && lg) {
#pragma unroll
                for (int ct = 0; ct < NT; ++ct) f.a[ct] = v4i{0, 0, 0, 0};
            }
            multiply(f);
        });
    }
    static_assert(S >= 2 && S <= 5 && (S - 1) * DPW + 2 <= 63, "wait counts");

    // ---- epilogue
    bool fits = EPI != EPI_RESIDUAL || residual_term_24(P.res_rq);
#pragma unroll
    for (int t = 0; t < NT; ++t) fits = fits && cst[32 * (wn * NT + t) + li][0] != 0;
    const bool fast = __builtin_amdgcn_ballot_w64(fits) == ~0ull;
    const int32_t rb = P.res_rq.b, rc = P.res_rq.c, rh = P.rnd << ((P.res_rq.c - 1) & 31);
    auto finish = [&](auto fastc) __attribute__((always_inline)) {
        constexpr bool FAST = decltype(fastc)::value;
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int n = n_l + 16 * ct;
            v4i out[MT];
#pragma unroll
            for (int d = 0; d < 4; ++d) {                 // 4 channels per packed output word
                const int ch = cl + 16 * ct + 4 * d;
                Residual64 q[4];
                v4i qb, qc, bi;
                if (FAST) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const v4i e = cst[ch + r];
                        q[r] = Residual64{(uint32_t)e[0], ((uint64_t)(uint32_t)e[3] << 32) | (uint32_t)e[2]};
                        asm volatile("" : "+v"(q[r].h));  // (see regst_common.hpp)
                    }
                } else {
                    qb = *reinterpret_cast<const v4i*>(&qb_s[ch]);
                    qc = *reinterpret_cast<const v4i*>(&qc_s[ch]);
                    bi = *reinterpret_cast<const v4i*>(&bias_s[ch]);
                }
#pragma unroll
                for (int tt = 0; tt < MT; ++tt) {
                    uint32_t o[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int32_t a32 = acc[ct][tt][4 * d + r];
                        int32_t rv = 0;
                        if (EPI == EPI_RESIDUAL) {
                            if (n + 16 <= N) rv = (int32_t)(int8_t)((uint32_t)res[tt][ct][d] >> (8 * r));
                            else if (n + 4 * d + r < N && row0 + 32 * tt < rows) rv = P.residual[(m0 + row0 + 32 * tt) * N + n + 4 * d + r];
                        }
                        int32_t v;
                        if (FAST) {
                            v = residual64_first(a32, q[r]);
                            if (EPI == EPI_RESIDUAL) v = clamp8_sum(v, (__mul24(rv, rb) + rh) >> rc);
                            else if (EPI == EPI_GELU) v = min(max(v, 1), 255);
                            else v = clamp8(v);
                        } else {
                            int64_t r64 = rnd_shift64(sum_of(a32, bi[r], kSumStart), qb[r], qc[r], P.rnd);
                            if (EPI == EPI_RESIDUAL) r64 += rnd_shift64(rv, P.res_rq.b, P.res_rq.c, P.rnd);
                            v = clamp8_64(r64) + (EPI == EPI_GELU ? 128 : 0);
                        }
                        if (EPI == EPI_GELU) v = gelu_lut[v];
                        o[r] = (uint32_t)v;
                    }
                    // low bytes of o[0..3] -> one word
                    out[tt][d] = (int)(__builtin_amdgcn_perm(o[1], o[0], 0x0c0c0400u) | __builtin_amdgcn_perm(o[3], o[2], 0x04000c0cu));
                }
                __builtin_amdgcn_sched_barrier(0);        // keep the register footprint of the epilogue small
            }
#pragma unroll
            for (int tt = 0; tt < MT; ++tt) {
                if (row0 + 32 * tt >= rows || n >= N) continue;
                int8_t* yp = P.y + (m0 + row0 + 32 * tt) * N + n;
                if (n + 16 <= N) {
                    *reinterpret_cast<v4i_any*>(yp) = out[tt];
                } else {
#pragma unroll
                    for (int e = 0; e < 15; ++e)
                        if (n + e < N) yp[e] = (int8_t)((uint32_t)out[tt][e >> 2] >> (8 * (e & 3)));
                }
            }
        }
    };
    if (fast) finish(std::true_type()); else finish(std::false_type());
}

constexpr int64_t kBigRows = 256;              // rows of the tallest tile of all, taken, as that of 192, only where its offsets fit

template <int MT, int NT, int S, int XS, int GM = 2, int GN = 2>
hipError_t launch_tile(hipStream_t s, const LinearArgs& a) {
    StParams P;
    P.x = a.x; P.w = a.w; P.bias = a.bias; P.rq_b = a.rq_b; P.rq_c = a.rq_c;
    P.residual = a.residual; P.res_rq = a.res_rq; P.gelu_p = a.gelu_p; P.gelu_rq = a.gelu_rq;
    P.y = a.y; P.M = a.M; P.N = a.N; P.K = a.K; P.ldx = a.ldx ? a.ldx : a.K; P.rnd = a.floor_shift ? 0 : 1;
    P.ln_g = a.ln_g; P.ln_b = a.ln_b; P.ln_f = a.ln_f; P.ln_c = a.ln_c;
    using TL = StTile<MT, NT, XS, GM, GN>;
    constexpr int TM = TL::TM, TN = TL::TN;
    constexpr bool BIG = MT * NT == 8;         // (no registers for a residual: 300 bytes a lane would be spilled)
    static_assert(TM <= (BIG ? kBigRows : MT == 3 ? 192 : kTileRows), "row offsets");
    const int64_t tm = (a.M + TM - 1) / TM, tn = (a.N + TN - 1) / TN, grid = (tm * tn + NXCD - 1) / NXCD * NXCD;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    P.m_fast = a.M < a.N;
    P.inner = FastDiv((uint32_t)(P.m_fast ? tm : tn));
    P.tiles = (uint32_t)(tm * tn); P.per_xcd = (uint32_t)(grid / NXCD);
    const dim3 g((unsigned)grid), b(64 * TL::W);
    if constexpr (XS == 0 && !BIG) {
        if (a.residual) {
            hipLaunchKernelGGL((gemm_st_kernel<EPI_RESIDUAL, MT, NT, S, XS, GM, GN>), g, b, 0, s, P);
            return hipGetLastError();
        }
    }
    if (a.gelu) hipLaunchKernelGGL((gemm_st_kernel<EPI_GELU, MT, NT, S, XS, GM, GN>), g, b, 0, s, P);
    else hipLaunchKernelGGL((gemm_st_kernel<EPI_PLAIN, MT, NT, S, XS, GM, GN>), g, b, 0, s, P);
    return hipGetLastError();
}

}  // namespace

// Up to two of these tiles per CU the repeated normalisation takes less than the launch it saves, beyond that more (fewer rows than
// that take the form inside gemm_kq.hip).  Forwards with it, without it and with it up to four tiles per CU: DeiT-S batch 2 266, 276 and
// 267 us, batch 4 331, 338 and 327, batch 8 372, 374 and 409, Swin-S batch 2 627, 644 and 628, batch 4 721, 736 and 721, batch 8 801,
// 795 and 856.  Rows of 768 bytes have lost by it since the separate layers became faster: ViT-B batch 1 340, 336 and 340, batch 2
// 450, 419 and 450, batch 4 464, 460 and 537.  (With 64 x 64 tiles, twice the rows to normalise, it was slower: batch 1 of DeiT-S by
// 9 %, of ViT-B by 13 %.)
bool linear_ln_takes(const LinearArgs& a) {
    if (!a.residual && a.K <= 768 && linear_kq_takes(a)) return true;
    using TL = StTile<1, 1, 6>;
    return !a.residual && (a.K & 15) == 0 && a.K >= 64 && a.K <= 768 &&
           ((a.M + TL::TM - 1) / TL::TM) * ((a.N + TL::TN - 1) / TL::TN) <= 2 * num_cus();
}

// 256 x 256 tiles, eight wavefronts of 128 x 64, one workgroup a CU, against 128 x 128 tiles, two workgroups of four wavefronts a CU: six
// fragments from LDS for eight products instead of four for four, and half the loads.  A round of the larger ones is twice the
// work of a round of the smaller, so what decides is how many rounds either takes; up to 6 : 5 against them the larger ones win, from
// 4 : 3 on they lose.  us, 128 x 128 and 256 x 256, rounds in units of the smaller: 10 : 10 40000 x 2000 x 896 108 and 93, 8000 x 2000 x
// 640 15.8 and 15.0, 12000 x 1040 x 400 14.3 and 12.3; 13 : 14 50000 x 2056 x 560 113 and 100; 7 : 8 50000 x 1000 x 1200 97 and 96; 5 : 6 20000 x
// 2000 x 2000 121 and 100, 12000 x 3000 x 2800 with ShiftGELU 146 and 123, 40000 x 1024 x 448 34.2 and 32.9; 3 : 4 12000 x 2000 x
// 448 23.1 and 24.0, 40000 x 512 x 576 21.5 and 24.2.  Not for one stage (30000 x 1000 x 96 19.8 and 21.2).
static bool big_tiles(const LinearArgs& a) {
    if (a.residual || a.K <= BK || (kBigRows - 1) * (a.ldx ? a.ldx : (int64_t)a.K) + a.K > (int64_t)kTileBytes) return false;
    const int64_t cus = num_cus();
    auto rounds = [&](int64_t t, int64_t per_cu) { return (((a.M + t - 1) / t) * ((a.N + t - 1) / t) + per_cu * cus - 1) / (per_cu * cus); };
    return 10 * rounds(kBigRows, 1) <= 6 * rounds(128, 2);
}

bool linear_st_one_round(const LinearArgs& a) {
    return !a.ln_g && one_round_of_192(a.M, a.N, a.K, a.residual, num_cus()) && 191 * (a.ldx ? a.ldx : (int64_t)a.K) + a.K <= (int64_t)kTileBytes;
}

hipError_t launch_linear_st(hipStream_t s, const LinearArgs& a) {
    if (a.ln_g) return a.K <= 384 ? launch_tile<1, 1, 3, 3>(s, a) : launch_tile<1, 1, 3, 6>(s, a);
    // The tile grows with the number of 64 x 64 tiles: larger ones load less per multiply, smaller ones leave no CU idle and
    // have shorter chains.  Measured with 256 CUs (times with 64 x 64, 128 x 64 and 128 x 128): 1576 x 768 x 3072 (300 tiles)
    // 10.1, 14.8 and 18.0 us; 3137 x 768 x 768 (600) 6.7, 7.2 and 9.0; 1576 x 2304 x 768 (900) 7.7, 5.9 and 7.1;
    // 6000 x 1000 x 768 (1504) 10.2, 9.4 and 9.6; 25216 x 1000 x 768 (6304) 37, 31 and 31; with longer rows the largest
    // tile pays earlier: 6000 x 768 x 3072 (1128) 24.8, 33.3 and 23.4 (but 3137 x 1000 x 3072 (800) 19.3, 17.7 and 20.8).
    // Stages: two workgroups of 128 x 128 share a CU with two stages, one with four: 6000 x 1000 x 768 9.6 against 14.6 us;
    // 64 x 64 with three stages against four (three workgroups per CU against two): 10.2 against 12.4 us.
    if (a.kernel == LINEAR_MANY_ROWS) return launch_tile<2, 2, 2, 0>(s, a);
    const int64_t tiles = ((a.M + 63) / 64) * ((a.N + 63) / 64), cus = num_cus();
    // Rows of 768 bytes and more: where some tile gives every CU at most one workgroup, the smallest such tile, with the stages that
    // fit and eight wavefronts for the larger ones (a SIMD issues twice as much from two).  Inputs in turn, us, the rule below against
    // this one: 64 x 64 with four stages for three 394 x 768 x 3072 9.4 and 8.2, 788 x 384 x 1536 6.4 and 6.0, 788 x 768 x 768 5.1
    // and 5.0 (six stages 5.2; 1568 x 384 x 384 3.9 and 4.0); 128 x 64 1576 x 768 x 3072 12.0 and 10.9, 2364 x 768 x 3072 13.3 and
    // 11.3, 788 x 2304 x 768 5.5 and 5.3 (1568 x 1152 x 384 4.35 and 4.42); 128 x 128 1576 x 2304 x 768 7.9 and 7.0, 4000 x 768 x
    // 3072 18.5 and 15.5 (1568 x 1536 x 384 5.3 and 5.7).  Beyond one workgroup a CU they lose: 3152 x 768 x 3072 with 128 x 64 19.3
    // against 16.4, 1576 x 3072 x 768 with 128 x 128 12.1 against 9.1.
    if (a.K >= 768) {
        const int64_t tm = (a.M + 127) / 128, tn = (a.N + 63) / 64;
        if (tiles <= cus) return launch_tile<1, 1, 4, 0>(s, a);
        if (tm * tn <= cus) return launch_tile<1, 1, 4, 0, 4, 2>(s, a);
        if (one_round_of_128(a.M, a.N, a.K, a.residual, cus)) return launch_tile<2, 1, 3, 0, 2, 4>(s, a);
        if (linear_st_one_round(a)) return launch_tile<3, 1, 3, 0, 2, 4>(s, a);
    }
    if (2 * tiles <= 5 * cus) return launch_tile<1, 1, 3, 0>(s, a);
    if (tiles * (a.K > 1024 ? 2 : 1) <= 6 * cus) return launch_tile<2, 1, 2, 0>(s, a);
    if (big_tiles(a)) return launch_tile<4, 2, 2, 0, 2, 4>(s, a);
    return launch_tile<2, 2, 2, 0>(s, a);
}

}  // namespace ivit
