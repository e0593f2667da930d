// Host-side declarations of the kernel launchers behind the C ABI (one translation unit each).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace rnn {

// ---------------------------------------------------------------------------------------
// float32 matrix product:  C[M,N] = (beta ? C : 0) + op(A) op(B) + bias_n[col]
//   a_t == false : A stored [M,K] (lda >= K)      a_t == true : A stored [K,M] (lda >= M)
//   b_t == false : B stored [K,N] (ldb >= N)      b_t == true : B stored [N,K] (ldb >= K)
// splitk_ws must hold gemm_splitk_floats(M,N,K) floats (0 => not needed).
struct GemmArgs {
    const float* A;
    const float* B;
    float* C;
    int M, N, K;
    int lda, ldb, ldc;
    bool a_t, b_t;
    const float* bias_n;  // nullable, length N
    int beta;             // 0 overwrite, 1 accumulate
    float* splitk_ws;     // nullable when gemm_splitk_floats == 0
    int prof_id;          // kernel id under which the profiler books this product (prof.hpp)
    // nullable: [M][gemm_stat_parts()][2] receives, per row and per column part of the final
    // result, (max, sum of exp relative to that max); written only when gemm_fuses_stats()
    float* row_stats;
    int parts = 3;        // bf16 numbers a float32 operand is split into: 3 keeps all of it, 2 its first 16 bits
};
size_t gemm_splitk_floats(int M, int N, int K, int parts = 3);
int gemm_stat_parts(int M, int N, int K, int parts = 3);
bool gemm_fuses_stats(int M, int N, int K, int parts = 3);
hipError_t launch_gemm(const GemmArgs& g, hipStream_t s);

// C[m,n] = (beta ? C : 0) + sum over splits of part[s][m][n] + bias_n[n], fixed order
hipError_t launch_splitk_reduce(const float* part, float* C, const float* bias_n, int M, int N, int ldc,
                                int splits, int beta, hipStream_t s);

// ---------------------------------------------------------------------------------------
// Recurrence (forward and reverse-time loops)
struct RecFwdArgs {
    const float* Wh;   // [H,H]
    const float* Wx;   // token input: [NV,H]; unused for dense input
    const float* b;    // [H]
    const int32_t* x;  // token ids [T,B] or NULL
    const float* U;    // dense input: precomputed Wx x_t + b, [T,B,H]; NULL for token input
    const float* h0;   // nullable [B,H]
    float* hist;       // [T+1,B,H], or a 2-slot ring [2,B,H] when ring != 0
    float* h_last;     // nullable [B,H]
    int H, T, B, act, ring;
};
struct RecBwdArgs {
    const float* Wh;      // [H,H]
    const float* WhT;     // [H,H] transposed copy (reference and step-wise kernels)
    const float* G;       // [T,B,H] output-layer contribution to d loss / d h_t
    const float* h_all;   // [T+1,B,H]
    const float* dh_last; // nullable [B,H]
    float* Delta;         // [T,B,H] receives d loss / d a_t
    float* dh0;           // nullable [B,H]
    int H, T, B, act;
    float* splitk_ws;     // split-K scratch for the dh0 product (stepwise path)
};
// Resident-weight persistent loops (recurrence.hip).  One struct serves both directions.
struct RecResArgs {
    const float* Wh;
    int H, T, B, act;
    int P, R, L, ldw, w_floats;  // filled from the plan by the launcher
    int nq4, hpad;               // float4 per lane of a row, zero-padded row/vector length
    int32_t* flags;              // exchange boxes in the workspace (P > 1): [2][B][H] 64-bit words, 8-byte aligned
    int32_t* status;             // device status word: set to 1 when a bounded wait expires
    int spin_limit;              // <= 0: default
    int xcd_pack;                // set by the launcher: workgroup p of a sequence is blockIdx.x / 8 (see the kernel)
    int poll_sleep;              // role-split loop: pauses of 64 clocks between a workgroup's own stores and its first poll
    // forward
    const float* Wx; const float* b; const int32_t* x; const float* U; const float* h0;
    float* hist; float* h_last; int ring;
    // reverse
    const float* G; const float* h_all; const float* dh_last; float* Delta; float* dh0;
    // fused weight gradients of a short single sequence (reverse, P == 1, B == 1)
    int fuse_post; float* dWh; float* db; float* dWx; int beta;
    // Short single sequence (fuse_post): G is produced by the other workgroups of the launch
    // (gpart non-NULL marks this mode; otherwise G is given)
    const float* gpart; int gstrips; float* Gw;
    const unsigned long long* g_box; uint32_t epoch;   // G arrives as tagged words [T][H]; the fused
                                                       // launch fills epoch from the tag word
};
struct RecResPlan { int P, R, L, ldw, w_floats, nq4, hpad; size_t smem; };
// strips: column strips of the short-sequence output layer (fuse_post only, else 0)
bool rec_resident_plan(int H, int B, int T, bool bwd, bool fuse_post, int strips, RecResPlan* out);
hipError_t launch_rec_resident(RecResArgs a, const RecResPlan& pl, bool bwd, hipStream_t s);
// The same loop for sequences whose matrix needs several compute units, with the wavefronts of a
// workgroup split into computing and polling ones (recurrence_grid.hip).  Serves what the resident
// plan gives more than one workgroup, as long as the slice fits the registers of four wavefronts.
struct RecGridPlan { int P, R, OPW, hpad; size_t smem; };
bool rec_grid_plan(int H, int B, RecGridPlan* out);
hipError_t launch_rec_grid(RecResArgs a, const RecGridPlan& pl, bool bwd, hipStream_t s);
struct SkinnyArgs;
// reverse loop with fused weight gradients (workgroup 0) and the output layer's backward strips
// (one workgroup per strip) in one launch; a must have fuse_post set
hipError_t launch_rec_bwd_with_strips(RecResArgs a, const RecResPlan& pl, const SkinnyArgs& k, hipStream_t s);

// Batched recurrence run as one fused GEMM launch per time step (recurrence_step.hip); serves
// the shapes the resident-weight kernels do not cover (batch > 4).
hipError_t run_rec_fwd_stepwise(const RecFwdArgs& a, hipStream_t s);
hipError_t run_rec_bwd_stepwise(const RecBwdArgs& a, hipStream_t s);

// Persistent batched loop with register-resident weights (recurrence_mfma.hip), H <= 256.
struct RecMfmaArgs {
    const float* Wh;
    int H, T, B, act;
    // forward
    const float* U;       // [T,B,H] input term including the bias (always materialised)
    const float* h0;      // nullable
    float* hist;          // [T+1,B,H] or 2-slot ring
    float* h_last;        // nullable
    int ring;
    // reverse
    const float* G; const float* h_all; const float* dh_last; float* Delta; float* dh0;
};
bool rec_batch_mfma_supported(int H, int B);
hipError_t launch_gather_input(const int32_t* x, const float* Wx, const float* b, float* U, int N,
                               int H, hipStream_t s);
hipError_t launch_rec_batch_mfma(const RecMfmaArgs& a, bool bwd, hipStream_t s);

// Persistent batched loop for 192 < H <= 1024 (recurrence_xcd.hip): one to four batch groups per XCD, the state
// handed over through that XCD's L2.  Needs the full history.
struct RecXcdArgs {
    const float* Wh;
    int H, T, B, act;
    // forward
    const int32_t* x;     // token ids [T,B] with Wx [NV,H] and b [H], or NULL with
    const float* Wx; const float* b;
    const float* U;       // [T,B,H] input term including the bias
    const float* h0;      // nullable
    float* hist;          // [T+1,B,H]
    float* h_last;        // nullable
    // reverse
    const float* G; const float* h_all; const float* dh_last; float* Delta; float* dh0;
    int32_t* counters;    // 40 words of workspace (cleared by the launcher)
    float* ring;          // rec_xcd_ring_bytes of workspace, 16-byte aligned (filled by the launcher)
    int32_t* status;      // device status word: set to 1 when a bounded wait expires
    int spin_limit;       // <= 0: default
    bool cleared;         // ring and counters are as rec_xcd_fills wants them
    int slots, patience;  // workgroups of a group; 10 ns they wait for each other to come (filled in by the launcher)
    int absent;           // workgroups a group waits for beyond those it has (filled in by the launcher: 0 but in tests)
};
bool rec_xcd_supported(int H, int B, int T, bool tokens);          // shape only (host)
// ... also in a captured call (whose launch is cooperative), where rec_batch_mfma_supported sizes are concerned
bool rec_xcd_pays_captured(int H, int T);
int rec_xcd_workgroups(int H, int B);
size_t rec_xcd_ring_bytes(int H, int B);
bool rec_xcd_ready(int H, int B, int act, bool bwd);             // and the current device can hold the grid at once
// groups of the launch that left these counters that one workgroup computed by itself
constexpr int REC_XCD_COUNTERS = 40;
int rec_xcd_groups_alone(const int32_t* counters);
// in launches of the calling thread: microseconds to wait for a group (< 0: the rule), workgroups that never come
void rec_xcd_test_roll_call(int microseconds, int absent);
// what the ring and the counters have to hold before a launch, for a kernel that sets it on the side
void rec_xcd_fills(const RecXcdArgs& a, struct FillJob* ring, struct FillJob* counters);
hipError_t launch_rec_xcd(const RecXcdArgs& a, bool bwd, hipStream_t s);

// Launch of a kernel whose workgroups wait for each other: it takes turns with others of its kind on the device (gang.hip).
// finishes_with_any: it ends with right results whatever part of its workgroups runs at once, and need not be cooperative
hipError_t launch_gang(const void* fn, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s, bool finishes_with_any = false);
// before a launch of `fn` with that much dynamic LDS on the current device (lds_limit.hip)
hipError_t allow_lds(const void* fn, size_t bytes);
hipError_t launch_zero_words(int32_t* p, int n, hipStream_t s);
// polls a bounded wait between workgroups makes before it gives up (host state, rnn_set_wait_limit)
int wait_limit();
hipError_t launch_transpose(const float* src, float* dst, int rows, int cols, hipStream_t s);
hipError_t launch_rec_fwd_reference(const RecFwdArgs& a, hipStream_t s);
hipError_t launch_rec_bwd_reference(const RecBwdArgs& a, hipStream_t s);

// ---------------------------------------------------------------------------------------
// Output layer element-wise / row-wise kernels
hipError_t launch_ce_row_stats(const float* Z, const int32_t* y, float* lse, float* rowloss,
                               int N, int O, hipStream_t s);
// the same from the statistics the logits product left: stats [N][parts][2]
hipError_t launch_ce_merge_stats(const float* stats, int parts, const float* Z, const int32_t* y,
                                 float* lse, float* rowloss, int N, int O, hipStream_t s);
// squared-error partial sums over the flat [N*O] arrays: *n_partial (<= N) floats in `partial`
hipError_t launch_mse_partial(const float* Z, const float* Y, float* partial, int N, int O,
                              int* n_partial, hipStream_t s);
hipError_t launch_loss_reduce(const float* rowloss, int N, double scale, float* loss, hipStream_t s);
// A grid of n workgroups and a few more, for kernels that have one per row and take `workgroup()` (common.hpp) for its number: a
// dimension of a grid holds 2^32 threads at most, and what is beyond is left out without an error
inline dim3 grid_of(size_t n) {
    const size_t x = n < (1u << 20) ? n : (1u << 20);
    return dim3((unsigned)x, (unsigned)((n + x - 1) / x));
}
// n words of p to be set to v by a kernel that has other work (n == 0: none)
struct FillJob { int32_t* p; size_t n; int32_t v; };
// second stage of a column sum: 256 threads per group of columns
struct ColsumJob { const float* part; float* out; int chunks, C, beta, txs, groups; };
ColsumJob colsum_job(const float* part, float* out, int chunks, int C, int beta);
// Z -> dZ in place, plus per-row-chunk column sums into part[chunks][O]; the fills ride along
int colsum_chunks(int N);
hipError_t launch_dz(float* Z, const float* lse, const int32_t* y, const float* Y, float* part,
                     int N, int O, int loss_kind, FillJob ring, FillJob counters, hipStream_t s);
hipError_t launch_colsum_partial(const float* M, float* part, int N, int C, FillJob zero, hipStream_t s);
hipError_t launch_colsum_finish(const float* part, float* out, int chunks, int C, int beta,
                                hipStream_t s);

// ---------------------------------------------------------------------------------------
// Output layer of a short single sequence (skinny.hip): column-strip kernels, N <= 32 rows
struct SkinnyArgs {
    const float* Hs;      // [N,H] rows h_t
    const float* V;       // [H,O]
    const float* c;       // [O]
    const int32_t* y;     // [N]
    float* Z;             // [N,O] logits (workspace)
    unsigned long long* stat_box;  // tagged words: [N][strips][2] strip max / sum exp, then [N] target logits
    unsigned long long* g_box;     // tagged words: [N][H] G, from the backward strips to the reverse loop
    uint32_t epoch;       // tag of this launch's words (never 0): filled in by the kernel from *epoch_word
    uint32_t* epoch_word; // device word: tag of the last launch on these boxes (see next_tag)
    int spin_limit;       // polls a bounded wait makes before it gives up
    int32_t* status;      // device status word: set to 1 when a bounded wait expires
    float* loss;          // device scalar written by the merging workgroup (logits kernel)
    float* lse;           // [N]
    float* dV; float* dc; // gradients
    float* gpart;         // [strips][N][H]
    float* dWx_zero;      // token-gradient matrix to zero fill, or NULL
    const int32_t* xids;  // [N] input token ids (rows of dWx the reverse loop's workgroup writes itself)
    float* vy;            // [N][H] column y_n of V per row (workspace)
    int H, O, N, NV, beta;
};
int skinny_strips(int O);
bool skinny_supported(int N, int H, int O);
size_t skinny_stat_box_bytes(int N, int O);
hipError_t launch_skinny_logits(const SkinnyArgs& a, hipStream_t s);   // logits, statistics and loss

// ---------------------------------------------------------------------------------------
// Small kernels of the Gauss-Newton-vector product (gauss_newton.hip)
hipError_t launch_reverse_rows(const float* src, float* dst, int T, int row, hipStream_t s);   // dst[t] = src[T-1-t]
// Crev[t] = C[T-1-t] (+ M[x[T-1-t]]), hrev[t] = Hs[T-1-t], WhT = Wh^T; the fills ride along
hipError_t launch_gn_prepare(const int32_t* x, const float* M, const float* C, const float* Hs, const float* Wh, float* Crev,
                             float* hrev, float* WhT, int T, int B, int H, FillJob ring, FillJob counters, hipStream_t s);
hipError_t launch_fill_zero(float* p, size_t n, hipStream_t s);
hipError_t launch_scale(float* p, size_t n, float alpha, hipStream_t s);
// RZ_n <- (p * RZ_n - p (p . RZ_n)) * scale, p = softmax(Z_n)
hipError_t launch_gn_softmax_metric(const float* Z, float* RZ, int N, int O, float scale, hipStream_t s);

// ---------------------------------------------------------------------------------------
// Token-keyed gradient of the input matrix and id validation
size_t dwx_scratch_floats(int N, int H);
size_t dwx_table_ints(int N, int NV);
hipError_t launch_dwx_tokens(const int32_t* x, const float* Delta, float* dWx, int N, int NV, int H, int beta, hipStream_t s);
// The grouped form: scratch holds dwx_scratch_floats(N, H) floats, slot_table dwx_table_ints(N, NV) zeros; the second stage of two
// column sums is done on the side.
hipError_t launch_dwx_tokens_grouped(const int32_t* x, const float* Delta, float* dWx, int N, int NV, int H, int beta,
                                     float* scratch, int32_t* slot_table, const ColsumJob& a, const ColsumJob& b, hipStream_t s);
hipError_t launch_check_tokens(const int32_t* ids, int64_t n, int32_t limit, int32_t* bad,
                               hipStream_t s);

}  // namespace rnn
