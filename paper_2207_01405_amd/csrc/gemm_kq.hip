// int8 x int8 -> int32 Dense with the dyadic requantisation of I-ViT (arXiv 2207.01405, Sec. 3.2, Eq. 7-10) for few rows,
// optionally with the residual add of Eq. 1-2, with ShiftGELU (Sec. 3.4, Algorithm 2) and with the I-LayerNorm (Sec. 3.5,
// Eq. 19-20) of the token rows in front: the form in which nothing is waited for twice.
//
// A workgroup of four wavefronts computes one tile of 32 tokens x 32 channels; the wavefronts split K.  Each requests its
// part of both operands at once, into LDS that no other wavefront reads (so no barrier stands between the loads and the
// products), multiplies, and leaves its partial sums in LDS; behind the one barrier each wavefront adds up a quarter of the
// tile and finishes it, four channels a lane.  Rows longer than 768 bytes go through a ring of two or three such parts.
// With an I-LayerNorm the wavefronts exchange the row sums of their parts first; the operand is then normalised in the
// registers it is multiplied from.
//
// What bounds it is the chain of latencies of a launch with one or two workgroups per CU; a kernel that only stores takes
// 2.3 us in the same loop.  Against 64 x 64 tiles whose wavefronts meet at every 128 bytes of K and finish 16 results a lane:
// 197 x 384 x 384 with a residual 3.9 -> 2.9 us, 197 x 384 x 1536 5.4 -> 3.5, 197 x 768 x 3072 7.7 -> 4.4 (launches of a graph); forwards:
// DeiT-S batch 1 357 -> 292 us.
#include "linear_rows.hpp"
#include "regst_common.hpp"

namespace ivit {
namespace {

using namespace regst;

struct KqParams {
    const int8_t* x; const int8_t* w; int64_t ldx; int M, N, K, rounds;
    FastDiv inner; uint32_t tiles, per_xcd; int m_fast;              // tiles in the dimension that runs fastest: rows or channels
    const int32_t* bias; const int32_t* rq_b; const int32_t* rq_c;
    const int8_t* residual; Dyadic res_rq; ShiftParams gelu_p; Dyadic gelu_rq;
    int8_t* y; int rnd;                                              // rnd 1: round to nearest, 0: floor
    const int32_t* ln_g; const int32_t* ln_b; int ln_f, ln_c;
};

typedef int v4i_w __attribute__((ext_vector_type(4), aligned(4)));
typedef int int_any __attribute__((aligned(1)));

constexpr int TILE = 32;

// Q k-steps of 32 bytes a wavefront and part, NB parts in LDS
template <int Q, int NB> struct KqLayout {
    static constexpr int P = 2 * Q, PB = 2 * TILE * 32 * Q;          // 16-byte pieces of a row of a part; bytes of a part (both operands)
    static constexpr int G16 = (P & 15) == 0 ? 16 : (P & 7) == 0 ? 8 : (P & 3) == 0 ? 4 : 2;      // gcd(P, 16)
    static constexpr int WREG = NB * PB > 4096 ? NB * PB : 4096;     // of a wavefront; the partial sums take its first 4 KB
    static constexpr int LUT = 4 * WREG, STAT = LUT + 256, PAR = STAT + 1024;      // I-LayerNorm: row sums of the parts, gamma and beta
};

template <int EPI, int Q, int NB, bool LN>
__global__ __launch_bounds__(256) void gemm_kq_kernel(KqParams P) {
    using LY = KqLayout<Q, NB>;
    extern __shared__ __align__(1024) int8_t lds[];
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane & 31, lg = lane >> 5;

    // each XCD takes a contiguous range of tiles; the operand with fewer rows runs fastest, the other one is then read by
    // as few XCDs as possible
    const uint32_t tile = (blockIdx.x % NXCD) * P.per_xcd + blockIdx.x / NXCD;
    if (tile >= P.tiles) return;
    uint32_t in;
    const uint32_t out = P.inner.divide(tile, in);
    const int m0 = (int)(P.m_fast ? in : out) * TILE, n0 = (int)(P.m_fast ? out : in) * TILE;
    const int rows = min(P.M - m0, TILE), cols = min(P.N - n0, TILE), pieces = P.K >> 4;

    // ---- the loads of a part: load instruction i covers 16-byte slots 64 i .. 64 i + 63 of [32 rows][2 Q pieces]; slot p of
    // a row holds its piece p ^ swz(row).  Rows and pieces that do not exist repeat the last one.
    auto swz = [](int r) __attribute__((always_inline)) { return (r / (16 / LY::G16)) & (LY::G16 - 1); };
    const int8_t* const xg = uniform_ptr(P.x + (int64_t)m0 * P.ldx);
    const int8_t* const wg = uniform_ptr(P.w + (int64_t)n0 * P.K);
    const uint32_t lds_w = lds_offset(lds) + wv * LY::WREG;
    uint32_t xo[Q], wo[Q];
    int pl[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int s = 64 * i + lane, r = s / LY::P;
        pl[i] = (s % LY::P) ^ swz(r);
        xo[i] = (uint32_t)min(r, rows - 1) * (uint32_t)P.ldx;
        wo[i] = (uint32_t)min(r, cols - 1) * (uint32_t)P.K;
    }
    // first piece of this wavefront's part of round rd
    auto first_piece = [&](int rd) __attribute__((always_inline)) { return (4 * rd + wv) * LY::P; };
    auto issue = [&](int rd, int buf) __attribute__((always_inline)) {
        const int p0 = first_piece(rd);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const uint32_t at = 16u * (uint32_t)min(p0 + pl[i], pieces - 1);
            dma16(xg, xo[i] + at, lds_w + buf * LY::PB + i * 1024);
            dma16(wg, wo[i] + at, lds_w + buf * LY::PB + LY::PB / 2 + i * 1024);
        }
    };

    // ---- what the lane finishes: token lj, channels n .. n + 3.  Requested first: the wait for the first part covers them.
    const int nl = 8 * wv + 4 * lg, n = n0 + nl;
    const int64_t at_y = (int64_t)(m0 + min(lj, rows - 1)) * P.N + n;
    const bool whole = nl + 4 <= cols;
    auto load4 = [&](const int32_t* p) __attribute__((always_inline)) {
        v4i v;
        if (whole) v = *reinterpret_cast<const v4i_w*>(p + n);
        else for (int e = 0; e < 4; ++e) v[e] = p[min(n + e, P.N - 1)];
        return v;
    };
    const v4i qb = load4(P.rq_b), qc = load4(P.rq_c);
    v4i bi = {0, 0, 0, 0};
    if (P.bias) bi = load4(P.bias);
    uint32_t res = 0;
    if (EPI == EPI_RESIDUAL) {
        if (whole) res = *reinterpret_cast<const int_any*>(P.residual + at_y);
        else for (int e = 0; e < 4; ++e) if (nl + e < cols) res |= (uint32_t)(uint8_t)P.residual[at_y + e] << (8 * e);
    }
    if constexpr (LN) {                                              // gamma and beta, 64 channels a load
        const uint32_t par = lds_offset(lds) + LY::PAR;
        for (int c = 64 * wv; c < P.K; c += 256) {
            const uint32_t off = 4u * (uint32_t)min(c + lane, P.K - 1);
            dma4(P.ln_g, off, par + 4 * c);
            dma4(P.ln_b, off, par + 4 * (Q * 128) + 4 * c);
        }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) issue(b, b);
    if (EPI == EPI_GELU) {
        const int32_t I = (int32_t)(int8_t)tid;
        lds[LY::LUT + tid] = (int8_t)requant64(shiftgelu_raw(I, P.gelu_p), P.gelu_rq.b, P.gelu_rq.c, P.rnd);
    }

    const int xr = lj * 32 * Q, sw = swz(lj);
    auto frag = [&](const int8_t* t, int ks) __attribute__((always_inline)) { return *reinterpret_cast<const v4i*>(t + xr + 16 * ((2 * ks + lg) ^ sw)); };
    const int8_t* const mine = lds + wv * LY::WREG;
    v16i acc = {};
    if constexpr (LN) {
        v4i xf[Q];
        wait_vm0();
        // the sums of this part of a row, two lanes a row
        int32_t sm = 0, sq = 0;
        const int p0 = first_piece(0);
#pragma unroll
        for (int ks = 0; ks < Q; ++ks) {
            xf[ks] = frag(mine, ks);
            if (p0 + 2 * ks + lg >= pieces) xf[ks] = v4i{0, 0, 0, 0};
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                sm = __builtin_amdgcn_sdot4(xf[ks][d], 0x01010101, sm, false);
                sq = __builtin_amdgcn_sdot4(xf[ks][d], xf[ks][d], sq, false);
            }
        }
        const auto s2 = __builtin_amdgcn_permlane32_swap((uint32_t)sm, (uint32_t)sm, false, false);
        const auto q2 = __builtin_amdgcn_permlane32_swap((uint32_t)sq, (uint32_t)sq, false, false);
        int2* const stat = reinterpret_cast<int2*>(lds + LY::STAT);
        if (lg == 0) stat[32 * wv + lj] = make_int2((int)(s2[0] + s2[1]), (int)(q2[0] + q2[1]));
        __syncthreads();                                             // (gamma and beta too: every wavefront has waited for its loads)
        sm = sq = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) { const int2 t = stat[32 * k + lj]; sm += t.x; sq += t.y; }
        const LnStat st = ln_stat(sm, sq, P.K, P.ln_f);
        const int32_t half = 1 << (P.ln_c - 1);
        const int32_t* const g = reinterpret_cast<const int32_t*>(lds + LY::PAR);
        const int32_t* const b = g + Q * 128;
#pragma unroll
        for (int ks = 0; ks < Q; ++ks) {
            const int c = 16 * min(p0 + 2 * ks + lg, pieces - 1);
            v4i wf = frag(mine + LY::PB / 2, ks);
            if (p0 + 2 * ks + lg >= pieces) wf = v4i{0, 0, 0, 0};
            v4i xn;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const v4i gv = *reinterpret_cast<const v4i*>(g + c + 4 * d), bv = *reinterpret_cast<const v4i*>(b + c + 4 * d);
                uint32_t o[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t xe = (int32_t)(int8_t)((uint32_t)xf[ks][d] >> (8 * r));
                    o[r] = (uint32_t)ln_value(xe, st, gv[r], (int32_t)((uint32_t)bv[r] + (uint32_t)half), P.ln_c);
                }
                xn[d] = (int)(__builtin_amdgcn_perm(o[1], o[0], 0x0c0c0400u) | __builtin_amdgcn_perm(o[3], o[2], 0x04000c0cu));
            }
            acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf, xn, acc, 0, 0, 0);
        }
    } else {
        auto multiply = [&](int rd, int buf) __attribute__((always_inline)) {
            const int8_t* t = mine + buf * LY::PB;
            const int p0 = first_piece(rd);
            v4i xf[Q], wf[Q];
#pragma unroll
            for (int ks = 0; ks < Q; ++ks) { wf[ks] = frag(t + LY::PB / 2, ks); xf[ks] = frag(t, ks); }
            if (p0 + LY::P > pieces) {                               // past the end of the rows: nothing to add
#pragma unroll
                for (int ks = 0; ks < Q; ++ks) if (p0 + 2 * ks + lg >= pieces) wf[ks] = v4i{0, 0, 0, 0};
            }
#pragma unroll
            for (int ks = 0; ks < Q; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[ks], xf[ks], acc, 0, 0, 0);
        };
        if constexpr (NB == 1) {
            wait_vm0();
            multiply(0, 0);
        } else {
            int buf = 0;
            // (the part NB ahead is requested when this one's fragments have been read, NB - 1 are then on their way)
#pragma unroll 1
            for (int rd = 0; rd + NB < P.rounds; ++rd) {
                asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NB - 1) * 2 * Q) : "memory");
                multiply(rd, buf);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                issue(rd + NB, buf);
                buf = buf + 1 == NB ? 0 : buf + 1;
            }
            static_for<NB>([&](auto k) __attribute__((always_inline)) {
                constexpr int K_ = decltype(k)::value;
                asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NB - 1 - K_) * 2 * Q) : "memory");
                multiply(P.rounds - NB + K_, buf);
                buf = buf + 1 == NB ? 0 : buf + 1;
            });
        }
    }

    // ---- partial sums: register 4 q + r of lane group g is channel 8 q + 4 g + r; wavefront q finishes registers 4 q .. + 3
    v4i* const part = reinterpret_cast<v4i*>(lds);
#pragma unroll
    for (int q = 0; q < 4; ++q) part[wv * (LY::WREG / 16) + 64 * q + lane] = v4i{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    v4i a = bi;
#pragma unroll
    for (int k = 0; k < 4; ++k) a += part[k * (LY::WREG / 16) + 64 * wv + lane];

    bool fits = EPI != EPI_RESIDUAL || dyadic_fits32(P.res_rq.b, P.res_rq.c);
#pragma unroll
    for (int e = 0; e < 4; ++e) fits = fits && dyadic_fits32(qb[e], qc[e]);
    uint32_t o[4];
    if (__builtin_amdgcn_ballot_w64(fits) == ~0ull) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int32_t v = rnd_shift_fit32(a[e], qb[e], qc[e], P.rnd);
            o[e] = (uint32_t)(EPI == EPI_RESIDUAL ? clamp8_sum(v, rnd_shift_fit32((int32_t)(int8_t)(res >> (8 * e)), P.res_rq.b, P.res_rq.c, P.rnd)) : clamp8(v));
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int64_t r64 = rnd_shift64(a[e], qb[e], qc[e], P.rnd);
            if (EPI == EPI_RESIDUAL) r64 += rnd_shift64((int32_t)(int8_t)(res >> (8 * e)), P.res_rq.b, P.res_rq.c, P.rnd);
            o[e] = (uint32_t)clamp8_64(r64);
        }
    }
    if (EPI == EPI_GELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (uint32_t)(uint8_t)lds[LY::LUT + (o[e] & 0xffu)];
    }
    if (lj >= rows) return;
    int8_t* const yp = P.y + at_y;
    if (whole) {
        *reinterpret_cast<int_any*>(yp) = (int)(__builtin_amdgcn_perm(o[1], o[0], 0x0c0c0400u) | __builtin_amdgcn_perm(o[3], o[2], 0x04000c0cu));
    } else {
#pragma unroll
        for (int e = 0; e < 3; ++e) if (nl + e < cols) yp[e] = (int8_t)o[e];
    }
}

template <int EPI, int Q, int NB, bool LN>
hipError_t launch(hipStream_t s, const KqParams& P) {
    using LY = KqLayout<Q, NB>;
    const size_t bytes = LN ? LY::PAR + 2 * 4 * (size_t)(Q * 128) : LY::STAT;
    static_assert(LY::PAR + 2 * 4 * Q * 128 <= 160 * 1024, "LDS");
    hipLaunchKernelGGL((gemm_kq_kernel<EPI, Q, NB, LN>), dim3(P.per_xcd * NXCD), dim3(256), bytes, s, P);
    return hipGetLastError();
}

template <int EPI, bool LN>
hipError_t launch_k(hipStream_t s, KqParams& P) {
    const int steps = (P.K + 31) / 32, q = (steps + 3) / 4;
    P.rounds = 1;
    switch (q) {
        case 1: return launch<EPI, 1, 1, LN>(s, P);
        case 2: return launch<EPI, 2, 1, LN>(s, P);
        case 3: return launch<EPI, 3, 1, LN>(s, P);
        case 4: return launch<EPI, 4, 1, LN>(s, P);
        case 5: return launch<EPI, 5, 1, LN>(s, P);
        case 6: return launch<EPI, 6, 1, LN>(s, P);
    }
    if constexpr (!LN) {
        P.rounds = (steps + 23) / 24;
        return P.rounds == 2 ? launch<EPI, 6, 2, false>(s, P) : launch<EPI, 6, 3, false>(s, P);
    }
    return hipErrorInvalidValue;
}

}  // namespace

// Up to two tiles per CU; one where the rows are so long that a workgroup's operands fill a CU's LDS.  Beyond that the larger
// tiles of gemm_st.hip, which move half the bytes per product, are faster.  us with this kernel against those (rows x N,
// tiles in brackets, 256 CUs, launches of a graph): K = 384 with a residual 197 x 384 (84) 2.9 against 3.9, 1568 x 384 (588) 3.8
// against 4.0, 3737 x 384 (1404) 5.5 against 4.6; without 512 x 1024 (512) 3.3 against 3.4, 788 x 1152 (900) 4.0 against 3.6; K = 768
// 197 x 2304 (504) 3.8 against 4.0, 394 x 1280 (520) 4.2 against 4.0, 392 x 3072 (1248) 6.6 against 4.7; K = 1536 197 x 384 (84) 3.5
// against 5.4, 500 x 512 (256) 3.8 against 5.5, 788 x 384 (300) 5.7 against 5.5; K = 3072 197 x 768 (168) 4.4 against 7.7, 320 x 768
// (240) 4.6 against 7.7, 788 x 768 (600) 10.4 against 7.9.
bool linear_kq_takes(const LinearArgs& a) {
    if ((a.K & 15) || a.M < 1 || a.M > (1 << 24) || (a.ln_g && (a.residual || a.K > 768))) return false;
    return ((a.M + TILE - 1) / TILE) * ((a.N + TILE - 1) / TILE) <= (a.K > 768 ? 1 : 2) * num_cus();
}

hipError_t launch_linear_kq(hipStream_t s, const LinearArgs& a) {
    KqParams P{};
    P.x = a.x; P.w = a.w; P.ldx = a.ldx ? a.ldx : a.K; P.M = (int)a.M; P.N = a.N; P.K = a.K;
    const uint32_t tm = (uint32_t)((a.M + TILE - 1) / TILE), tn = (uint32_t)((a.N + TILE - 1) / TILE);
    P.m_fast = a.M < a.N;
    P.inner = FastDiv(P.m_fast ? tm : tn);
    P.tiles = tm * tn;
    P.per_xcd = (P.tiles + NXCD - 1) / NXCD;
    P.bias = a.bias; P.rq_b = a.rq_b; P.rq_c = a.rq_c;
    P.residual = a.residual; P.res_rq = a.res_rq; P.gelu_p = a.gelu_p; P.gelu_rq = a.gelu_rq;
    P.y = a.y; P.rnd = a.floor_shift ? 0 : 1;
    P.ln_g = a.ln_g; P.ln_b = a.ln_b; P.ln_f = a.ln_f; P.ln_c = a.ln_c;
    if (a.residual) return launch_k<EPI_RESIDUAL, false>(s, P);
    if (a.gelu) return a.ln_g ? launch_k<EPI_GELU, true>(s, P) : launch_k<EPI_GELU, false>(s, P);
    return a.ln_g ? launch_k<EPI_PLAIN, true>(s, P) : launch_k<EPI_PLAIN, false>(s, P);
}

}  // namespace ivit
