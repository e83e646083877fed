// Host-side launchers of the gfx950 kernels (internal to libivit.so; the public surface is include/ivit.h).
// Each launcher assumes arguments already validated by the C-ABI layer and returns a hipError_t.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ivit_device.hpp"

namespace ivit {

hipError_t launch_ilayernorm(hipStream_t s, const int8_t* x, const int32_t* gamma_q, const int32_t* beta_q,
                             int8_t* y, int64_t rows, int C, int f_bits, int c_shift);

// The I-LayerNorm of patch merging (rows of 4 C bytes, see launch_patch_merge_gather), reading the tokens where they lie.
bool merge_ilayernorm_takes(const int8_t* x, const int32_t* gamma_q, const int32_t* beta_q, const int8_t* y, int B, int g, int C);
hipError_t launch_merge_ilayernorm(hipStream_t s, const int8_t* x, const int32_t* gamma_q, const int32_t* beta_q, int8_t* y, int B, int g,
                                   int C, int f_bits, int c_shift);

hipError_t launch_shiftmax(hipStream_t s, const int8_t* x, const int8_t* bias, int H, int T, int8_t* y,
                           int64_t rows, int cols, int ld, ShiftParams p);

hipError_t launch_shiftgelu(hipStream_t s, const int8_t* x, int8_t* y8, int16_t* y16, int64_t n,
                            ShiftParams p, Dyadic out_rq);

hipError_t launch_shiftgelu_rowmax(hipStream_t s, const int8_t* x, int8_t* y, int64_t rows, int cols, ShiftParams p,
                                   Dyadic rq);

struct LinearArgs {
    const int8_t* x; const int8_t* w; const int32_t* bias; const int32_t* rq_b; const int32_t* rq_c;
    const int8_t* residual; Dyadic res_rq;
    bool gelu; ShiftParams gelu_p; Dyadic gelu_rq;
    int8_t* y; int64_t M; int N; int K;
    int64_t ldx;                         // bytes between rows of x; 0 means K (dense rows)
    int kernel;                          // 0: chosen from the shape; otherwise one of LinearKernel, forced (tests, measurements)
    int floor_shift;                     // 0: requantisations round to nearest (Eq. 8 through Eq. 10); 1: bare shift of Eq. 10 (floor)
    // an I-LayerNorm over the rows of x first (K = its C; only where linear_ln_takes says so); nullptr: none
    const int32_t* ln_g; const int32_t* ln_b; int ln_f, ln_c;
};
enum LinearKernel { LINEAR_AUTO = 0, LINEAR_MANY_ROWS = 1, LINEAR_REG_STATIONARY = 2, LINEAR_BIG_TILES = 3 };
hipError_t launch_linear(hipStream_t s, const LinearArgs& a);
// Register-stationary kernel (gemm_rs.hip): whether it takes this shape at all, and its launch.
bool linear_rs_takes(const LinearArgs& a);
hipError_t launch_linear_rs(hipStream_t s, const LinearArgs& a);
// The same with K = 1536 split over pairs of wavefronts (gemm_ks.hip).
bool linear_ks_takes(const LinearArgs& a);
hipError_t launch_linear_ks(hipStream_t s, const LinearArgs& a);
// Long rows, both operands streamed through LDS in 256 x 128 tiles (gemm_tl.hip).
bool linear_tl_takes(const LinearArgs& a);
hipError_t launch_linear_tl(hipStream_t s, const LinearArgs& a);
// Few rows, K split over the wavefronts of a workgroup (gemm_kq.hip).
bool linear_kq_takes(const LinearArgs& a);
hipError_t launch_linear_kq(hipStream_t s, const LinearArgs& a);
// Any shape, both operands streamed through LDS in small tiles (gemm_st.hip).
hipError_t launch_linear_st(hipStream_t s, const LinearArgs& a);
bool linear_st_one_round(const LinearArgs& a);    // long rows and a tile for every CU at most: before the kernels for many rows
bool linear_ln_takes(const LinearArgs& a);

// The token-wise part of an encoder block in one kernel (token_block.hip).
struct DenseW { const int8_t* w; const int32_t* bias; const int32_t* rq_b; const int32_t* rq_c; };
struct TokenBlockArgs {
    const int8_t* o;                     // attention output [R, C]; nullptr: only the LN and the QKV layer below, on x
    const int8_t* x;                     // block input [R, C]
    int8_t* xhat; int8_t* y;             // scratch [R, C], written and read back by the launch; block output [R, C]
    int8_t* out;                         // next == 1: LN output [R, C]; next == 2: qkv of the next block [R, 3 C]
    int64_t R; int C, F;
    int next;                            // what follows the block: 0 nothing, 1 an I-LayerNorm, 2 the next block's I-LayerNorm and QKV layer
    const int32_t* ln2_g; const int32_t* ln2_b; int ln2_f, ln2_c;
    const int32_t* ln1_g; const int32_t* ln1_b; int ln1_f, ln1_c;
    DenseW proj, fc1, fc2, qkv_w;
    Dyadic res1, res2; ShiftParams gelu_p; Dyadic gelu_rq;
    const int8_t* table;                 // token_block_table_bytes of constants, filled by launch_token_tables before the launch; 16-byte aligned
};
size_t token_block_table_bytes(int C, int F);
constexpr int kTableLaunches = 15;       // launches whose constants one table launch prepares
hipError_t launch_token_tables(hipStream_t s, const TokenBlockArgs* a, int n);      // n <= kTableLaunches
bool token_block_takes(int C, int F, int64_t R, int n_blocks);
hipError_t launch_token_block(hipStream_t s, const TokenBlockArgs& a);
bool token_stream_takes(int C, int F, int64_t R);       // the form of launch_token_block for few rows (token_stream.hip)
hipError_t launch_token_stream(hipStream_t s, const TokenBlockArgs& a);

hipError_t launch_embed_tokens(hipStream_t s, const int8_t* patch_tok, const int8_t* cls, const int8_t* pos, Dyadic tok_rq,
                               Dyadic pos_rq, int8_t* tokens, int B, int P, int C);

hipError_t launch_patch_merge_gather(hipStream_t s, const int8_t* x, int8_t* y, int B, int g, int C);
hipError_t launch_mean_pool(hipStream_t s, const int8_t* x, int8_t* y, int B, int T, int C, Dyadic rq);

struct AttentionArgs {
    const int8_t* qkv; const int8_t* rel_bias; int8_t* o;
    const int8_t* mask; int n_mask;      // shifted-window mask [n_mask, T, T] or nullptr
    const int32_t* tok_index; int n_win; // rows of the tokens of the n_win windows of an image [n_win, T], or nullptr
    int B, T, C, H;
    Dyadic qk_rq; ShiftParams sm; Dyadic pv_rq;
    int8_t* tap_scores; int8_t* tap_probs;
    int floor_shift;                     // as LinearArgs::floor_shift, for both requantisations (scores, output)
};
hipError_t launch_attention(hipStream_t s, const AttentionArgs& a);

// Number of compute units of the current device (cached); used to size persistent grids.
int num_cus();

// Kinds of launches reported by the trace (ivit_trace_end); values are part of the C ABI.
enum LaunchKind { KIND_ILAYERNORM = 1, KIND_GEMM = 2, KIND_GEMM_RESIDUAL = 3, KIND_GEMM_GELU = 4,
                  KIND_ATTENTION = 5, KIND_SHIFTMAX = 6, KIND_SHIFTGELU = 7, KIND_EMBED = 8, KIND_PATCH_MERGE = 9, KIND_MEAN_POOL = 10,
                  KIND_TOKEN_BLOCK = 11, KIND_TOKEN_TABLES = 12 };

// Brackets one kernel launch with two HIP events on its stream while a trace is active; otherwise a no-op.
// ops = algorithmic integer operations (2 per int8 multiply-accumulate), bytes = algorithmic HBM bytes.
class TraceScope {
public:
    TraceScope(hipStream_t s, int kind, int64_t ops, int64_t bytes);
    ~TraceScope();
    TraceScope(const TraceScope&) = delete;
    TraceScope& operator=(const TraceScope&) = delete;
private:
    hipStream_t stream_;
    int slot_;
};

}  // namespace ivit
