// Training step of a feed-forward classifier (the paper's neural-network training benchmark:
// 10-class classification of a 784-dimensional input by logistic regression, one hidden layer
// of 500 units or three of 1000, stochastic gradient descent on batches of 1, 10 or 60):
//
//     a_l = act(W_l a_{l-1} + b_l),  z = W_L a_{L-1} + b_L,  loss = mean(logsumexp(z) - z[y]),
//     W_l <- W_l - lr dloss/dW_l,  b_l <- b_l - lr dloss/db_l      after every batch.
//
// At these sizes a step moves a few megabytes of weights and computes almost nothing, so what it
// costs is launches and memory round trips.  With at most one hidden layer all batches of a call share
// one launch (mlp_one_kernel below).  Otherwise a step is 2 L launches (L hidden
// layers, at most 16 classes and 1024 units: L forward, one with the output layer, the loss and the first two backward
// products, L - 2 backward, and ONE update of all layers, which also adds up the batch's loss; with more classes or units
// the output layer, the loss and the backward products are launches of their own), each
// built like the batched recurrence's step kernel to pay one round trip: a workgroup owns a
// 16 x 16 tile of the result, its 16 wavefronts split the contraction in slices of 64 and request
// their whole share of both operands at once, straight into the lane registers
// v_mfma_f32_16x16x4_f32 reads them from; the partial tiles meet in LDS once and the epilogue is
// fused (bias + activation forward, activation derivative backward).  The update kernel forms
// dW = dZ^T a in matrix-core tiles over the batch and applies it in place together with the
// bias update, so weight gradients never exist in memory; all layers share that launch, which
// is why every dZ_l is kept until the backward chain has ended.  No atomics: results are
// run-to-run identical.
#include "../../include/rnn.h"

#include "common.hpp"
#include "internal.hpp"
#include "prof.hpp"

#include <math.h>

namespace rnn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int MW = 16, MNT = MW * kWave, MKC = 64;

template <bool VEC>
__device__ __forceinline__ float4 ld_k4(const float* __restrict__ row, int k, int klim) {
    if (VEC && k + 3 < klim) return *reinterpret_cast<const float4*>(row + k);
    float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
    if (k + 0 < klim) t.x = row[k + 0];
    if (k + 1 < klim) t.y = row[k + 1];
    if (k + 2 < klim) t.z = row[k + 2];
    if (k + 3 < klim) t.w = row[k + 3];
    return t;
}

template <int ACT>
__device__ __forceinline__ float apply_act(float a) {
    return ACT == 0 ? sigmoidf_fast(a) : (ACT == 1 ? tanhf_fast(a) : a);
}

// Tile of a workgroup, gx column tiles by ceil(M / 16) row tiles.  Workgroups go round the eight dies, each with an L2 of its own,
// so the row tiles of a column tile, which read the same 16 rows or columns of the weights, follow one another on
// one die.  Column tiles are rounded up to whole rounds; a workgroup with none leaves at once.
__device__ __forceinline__ bool tile_of(int gx, int M, int& x, int& y) {
    const int gy = (M + 15) / 16, die = blockIdx.x % 8, i = blockIdx.x / 8;
    y = i % gy;
    x = i / gy * 8 + die;
    return x < gx;
}
int tiles_of(int gx, int M) { return (gx + 7) / 8 * 8 * ((M + 15) / 16); }

// C[M,N] = act(A[M,K] W[N,K]^T + bias[N]);  ACT 0 sigmoid, 1 tanh, 2 none.
// tiles_of(ceil(N/16), M) workgroups, 1024 threads.  Lane (r = lane % 16, g = lane / 16) of a wavefront
// holds k = k0 + 16 s + 4 g + e of row r of A and of row r of W: the same permuted walk of K for both.
// CE (output layer with N <= 16, ACT 2): the tile holds whole rows of logits, so the epilogue goes on
// to the loss: C receives dZ = (softmax - onehot(y)) / M instead of the logits and losspart[row tile]
// the sum of the workgroup's row losses lse - z[y] (rows in order).
template <int ACT, bool VEC, bool CE = false>
__global__ __launch_bounds__(MNT) void mlp_fwd_kernel(const float* __restrict__ A, const float* __restrict__ W,
                                                      const float* __restrict__ bias, float* __restrict__ C,
                                                      int M, int N, int K, const int32_t* __restrict__ y,
                                                      float* __restrict__ losspart) {
    __shared__ float red[MW][4][kWave];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int g = lane / 16, nn = lane % 16;
    int tx, ty;
    if (!tile_of((N + 15) / 16, M, tx, ty)) return;
    const int n0 = tx * 16, m0 = ty * 16;
    const int col = n0 + nn;
    const float bv = (wave < 4 && col < N) ? bias[col] : 0.f;   // requested before the product
    const bool a_ok = m0 + nn < M, b_ok = col < N;
    const float* arow = A + (size_t)min(m0 + nn, M - 1) * K;
    const float* brow = W + (size_t)min(col, N - 1) * K;
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    const int nchunks = (K + MKC - 1) / MKC;
    for (int kc = wave; kc < nchunks; kc += MW) {
        const int k0 = kc * MKC + 4 * g;
        float4 a[4], b[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            a[s] = a_ok ? ld_k4<VEC>(arow, k0 + 16 * s, K) : make_float4(0.f, 0.f, 0.f, 0.f);
            b[s] = b_ok ? ld_k4<VEC>(brow, k0 + 16 * s, K) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s].x, b[s].x, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s].y, b[s].y, acc1, 0, 0, 0);
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s].z, b[s].z, acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s].w, b[s].w, acc1, 0, 0, 0);
        }
    }
    // result layout of the 16x16 tile: lane -> column nn; register i -> row 4 g + i
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][i][lane] = acc0[i] + acc1[i];
    __syncthreads();
    if constexpr (!CE) {
        if (wave >= 4) return;
        const int row = m0 + 4 * g + wave;
        if (row >= M || col >= N) return;
        float v = bv;
#pragma unroll
        for (int w = 0; w < MW; ++w) v += red[w][wave][lane];
        C[(size_t)row * N + col] = apply_act<ACT>(v);
    } else {
        __shared__ float rowloss[16];
        if (wave < 4) {
            // the 16 lanes of a quarter-wave hold the 16 columns of row 4 g + wave
            const int row = m0 + 4 * g + wave;
            const bool ok = row < M && col < N;
            float v = bv;
#pragma unroll
            for (int w = 0; w < MW; ++w) v += red[w][wave][lane];
            const int yy = row < M ? y[row] : -1;
            const float m = max16(ok ? v : -INFINITY);
            const float se = sum16(ok ? __expf(v - m) : 0.f);
            const float lse = m + __logf(se);
            const float zy = sum16((ok && col == yy) ? v : 0.f);
            if (ok) C[(size_t)row * N + col] = (__expf(v - lse) - (col == yy ? 1.f : 0.f)) * (1.0f / (float)M);
            if (nn == 0) rowloss[4 * g + wave] = row < M ? lse - zy : 0.f;
        }
        __syncthreads();
        if (tid == 0) {
            float sum = 0.f;
            for (int r = 0; r < 16; ++r) sum += rowloss[r];
            losspart[ty] = sum;
        }
    }
}

// dZprev[M,Kin] = (dZ[M,Nout] W[Nout,Kin]) * act'(Aprev[M,Kin]): the contraction runs over the rows
// of W, so W is the n-contiguous operand (one value per request, 16 lanes = 64 contiguous bytes).
// tiles_of(ceil(Kin/16), M) workgroups, 1024 threads.
template <int ACT, bool VEC>
__global__ __launch_bounds__(MNT) void mlp_bwd_data_kernel(const float* __restrict__ dZ, const float* __restrict__ W,
                                                           const float* __restrict__ Aprev, float* __restrict__ dZprev,
                                                           int M, int Nout, int Kin) {
    __shared__ float red[MW][4][kWave];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int g = lane / 16, nn = lane % 16;
    int tx, ty;
    if (!tile_of((Kin + 15) / 16, M, tx, ty)) return;
    const int n0 = tx * 16, m0 = ty * 16;
    const int col = n0 + nn;
    float hv = 0.f;
    if (wave < 4 && col < Kin && m0 + 4 * g + wave < M) hv = Aprev[(size_t)(m0 + 4 * g + wave) * Kin + col];
    const bool a_ok = m0 + nn < M, b_ok = col < Kin;
    const float* arow = dZ + (size_t)min(m0 + nn, M - 1) * Nout;
    const float* bcol = W + min(col, Kin - 1);
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    const int nchunks = (Nout + MKC - 1) / MKC;
    for (int kc = wave; kc < nchunks; kc += MW) {
        const int k0 = kc * MKC + 4 * g;
        float a[16], b[16];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const float4 av = a_ok ? ld_k4<VEC>(arow, k0 + 16 * s, Nout) : make_float4(0.f, 0.f, 0.f, 0.f);
            a[4 * s] = av.x; a[4 * s + 1] = av.y; a[4 * s + 2] = av.z; a[4 * s + 3] = av.w;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = k0 + 16 * s + e;
                b[4 * s + e] = (b_ok && k < Nout) ? bcol[(size_t)k * Kin] : 0.f;
            }
        }
#pragma unroll
        for (int q = 0; q < 16; q += 2) {
            acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q], b[q], acc0, 0, 0, 0);
            acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q + 1], b[q + 1], acc1, 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][i][lane] = acc0[i] + acc1[i];
    __syncthreads();
    if (wave >= 4) return;
    const int row = m0 + 4 * g + wave;
    if (row >= M || col >= Kin) return;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < MW; ++w) v += red[w][wave][lane];
    dZprev[(size_t)row * Kin + col] = v * (ACT == 0 ? act_grad<0>(hv) : act_grad<1>(hv));
}

// The output layer, the loss and the first two backward products in one launch, for at most 16 classes and at most 1024
// units in front of them:
//     z = Ah Wo^T + bo,  dZo = (softmax(z) - onehot(y)) / M,  dZh = (dZo Wo) * act'(Ah),  dZprev = (dZh Wl) * act'(Aprev).
// What bounds it is round trips, so a workgroup forms its 16 rows of logits and of dZo again (a product of 16 x 16 x Kh) rather than
// wait for another launch: all operands are requested at once.  Every wavefront holds 64 of the Kh units.  dZh never passes
// through LDS: Wo^T dZo^T leaves the matrix cores as lane -> row of the batch, register -> four consecutive units, which is
// what a lane supplies to the product with Wl, and the lane has act'(Ah) of the same elements from the first product.
// (784-1000-1000-1000-10, batch 60: three launches of 5.4, 3.7 and 6.7 us with two gaps between them; this one 11.5 us.  The whole
// batch 54.1 -> 50.4 us, and 47.8 with the tiles of a column on one die.)
// tiles_of(ceil(Kp/16), M) workgroups, 1024 threads; those of the first column tile store dZo, dZh and the losses.
template <int ACT, bool VEC>
__global__ __launch_bounds__(MNT) void mlp_out_bwd_kernel(const float* __restrict__ Ah, const float* __restrict__ Wo,
                                                          const float* __restrict__ bo, const int32_t* __restrict__ y,
                                                          const float* __restrict__ Wl, const float* __restrict__ Aprev,
                                                          float* __restrict__ dZo, float* __restrict__ dZh,
                                                          float* __restrict__ dZprev, float* __restrict__ losspart, int M, int O,
                                                          int Kh, int Kp) {
    __shared__ __attribute__((aligned(16))) float red[MW][4][kWave];
    __shared__ float dz[16][17], rowloss[16];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int g = lane / 16, nn = lane % 16;
    int tx, ty;
    if (!tile_of((Kp + 15) / 16, M, tx, ty)) return;
    const int n0 = tx * 16, m0 = ty * 16;
    const int col = n0 + nn, row_e = m0 + 4 * g + wave;         // row_e: of the epilogues (wavefronts 0 to 3)
    const bool keeps = tx == 0;
    const int k0 = MKC * wave + 4 * g;                          // this lane's units: k0 + 16 s + e
    const bool a_ok = m0 + nn < M;
    const float* arow = Ah + (size_t)min(m0 + nn, M - 1) * Kh;
    const float* orow = Wo + (size_t)min(nn, O - 1) * Kh;
    const float* bcol = Wl + min(col, Kp - 1);
    float4 a[4], wo[4];
    float wt[4][4], b[16];
    float bv = 0.f, hv = 0.f;
    int yy = -1;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        a[s] = a_ok ? ld_k4<VEC>(arow, k0 + 16 * s, Kh) : make_float4(0.f, 0.f, 0.f, 0.f);
        wo[s] = nn < O ? ld_k4<VEC>(orow, k0 + 16 * s, Kh) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (wave < 4) {
        if (nn < O) bv = bo[nn];
        if (row_e < M) {
            yy = y[row_e];
            if (col < Kp) hv = Aprev[(size_t)row_e * Kp + col];
        }
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int k = k0 + 16 * (q / 4) + q % 4;
        b[q] = col < Kp && k < Kh ? bcol[(size_t)k * Kp] : 0.f;
    }

    // logits and dZo of the workgroup's 16 rows
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s].x, wo[s].x, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s].y, wo[s].y, acc1, 0, 0, 0);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s].z, wo[s].z, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s].w, wo[s].w, acc1, 0, 0, 0);
    }
    // this wavefront's columns of Wo turned through its part of LDS: wt[s][j] = Wo[4 j + g][64 wave + 16 s + nn]
    float* mine = &red[wave][0][0];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        *reinterpret_cast<float4*>(mine + 16 * nn + 4 * g) = wo[s];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int j = 0; j < 4; ++j) wt[s][j] = mine[16 * (4 * j + g) + nn];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][i][lane] = acc0[i] + acc1[i];
    lds_barrier();
    if (wave < 4) {
        // the 16 lanes of a quarter-wave hold the classes of row 4 g + wave
        const bool ok = row_e < M && nn < O;
        float v = bv;
#pragma unroll
        for (int w = 0; w < MW; ++w) v += red[w][wave][lane];
        const float m = max16(ok ? v : -INFINITY);
        const float se = sum16(ok ? __expf(v - m) : 0.f);
        const float lse = m + __logf(se);
        const float zy = sum16((ok && nn == yy) ? v : 0.f);
        const float d = ok ? (__expf(v - lse) - (nn == yy ? 1.f : 0.f)) * (1.0f / (float)M) : 0.f;
        dz[4 * g + wave][nn] = d;
        if (nn == 0) rowloss[4 * g + wave] = row_e < M ? lse - zy : 0.f;
        if (keeps && ok) dZo[(size_t)row_e * O + nn] = d;
    }
    lds_barrier();
    if (keeps && tid == 0) {
        float sum = 0.f;
        for (int r = 0; r < 16; ++r) sum += rowloss[r];
        losspart[ty] = sum;
    }

    // dZh in the layout of the next product's operand, and that product
    float dzv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) dzv[j] = dz[nn][4 * j + g];
    acc0 = acc1 = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) d = __builtin_amdgcn_mfma_f32_16x16x4f32(wt[s][j], dzv[j], d, 0, 0, 0);
        const float4 h = a[s];
        d[0] *= act_grad<ACT>(h.x); d[1] *= act_grad<ACT>(h.y); d[2] *= act_grad<ACT>(h.z); d[3] *= act_grad<ACT>(h.w);
        if (keeps && a_ok) store4u(dZh + (size_t)(m0 + nn) * Kh + k0 + 16 * s, make_float4(d[0], d[1], d[2], d[3]), Kh - k0 - 16 * s);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(d[0], b[4 * s], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(d[1], b[4 * s + 1], acc1, 0, 0, 0);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(d[2], b[4 * s + 2], acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(d[3], b[4 * s + 3], acc1, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][i][lane] = acc0[i] + acc1[i];   // (the logits' partial sums were read before the last barrier)
    lds_barrier();
    if (wave >= 4 || row_e >= M || col >= Kp) return;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < MW; ++w) v += red[w][wave][lane];
    dZprev[(size_t)row_e * Kp + col] = v * act_grad<ACT>(hv);
}

// W[n,k] -= lr sum_m dZ[m,n] Aprev[m,k];  b[n] -= lr sum_m dZ[m,n].
// A wavefront owns 16 rows of W by 64 columns (four 16x16 tiles sharing the dZ operand) and walks
// the batch four rows per matrix instruction; per layer (ceil(Kin/256), ceil(Nout/16)) workgroups of 256 threads.
// The columns of the four tiles are interleaved, tile t holding columns k0 + 4 r + t, so that a lane's
// share of a row of W or of the inputs is one 16-byte piece: 36 requests and 4 stores per lane instead of
// 96 and 16, which is what bounded it (784-1000-1000-1000-10, batch 60: 12.4 -> 10.8 us;
// batch 16, where the weights' own traffic is most of it: 7.7 -> 7.6).
// MB > 0: the batch has at most 16 MB rows and every operand (and the tile of W itself) is
// requested before the first product, one memory round trip for the whole update; MB = 0: any batch.
struct UpdateLayers {
    const float* dZ[RNN_MLP_MAX_LAYERS];      // [M, Nout]
    const float* Aprev[RNN_MLP_MAX_LAYERS];   // [M, Kin]
    float* W[RNN_MLP_MAX_LAYERS];
    float* b[RNN_MLP_MAX_LAYERS];
    int Nout[RNN_MLP_MAX_LAYERS], Kin[RNN_MLP_MAX_LAYERS];
    int gx[RNN_MLP_MAX_LAYERS];               // workgroups along Kin
    int first[RNN_MLP_MAX_LAYERS + 1];        // first workgroup of the layer in the flat grid
    int layers;
    const float* losspart;                    // per 16-row group of the batch: sum of its row losses
    int nparts;                               // 0: the loss was written by its own kernel
    float* loss;
};

// One launch updates every layer: the flat grid is the layers' (ceil(Kin/256) x ceil(Nout/16)) grids
// one after another (all dZ_l are kept until the backward chain has ended).
template <int MB>
__global__ __launch_bounds__(256) void mlp_update_kernel(const UpdateLayers ul, int M, float lr) {
    int l = 0;
    while (l + 1 < ul.layers && (int)blockIdx.x >= ul.first[l + 1]) ++l;
    const int local = blockIdx.x - ul.first[l];
    const int bx = local % ul.gx[l], by = local / ul.gx[l];
    const float* __restrict__ dZ = ul.dZ[l];
    const float* __restrict__ Aprev = ul.Aprev[l];
    float* __restrict__ W = ul.W[l];
    float* __restrict__ b = ul.b[l];
    const int Nout = ul.Nout[l], Kin = ul.Kin[l];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int q = lane / 16, r = lane % 16;
    const int n0 = by * 16;
    const int k0 = (bx * 4 + wave) * 64;
    if (blockIdx.x == 0 && tid == 64 && ul.nparts > 0) {   // the batch's mean loss, groups in order
        float sum = 0.f;
        for (int g = 0; g < ul.nparts; ++g) sum += ul.losspart[g];
        *ul.loss = sum / (float)M;
    }
    if (bx == 0 && wave == 0) {
        // bias: lane (q, r) sums the rows m = q, q + 4, ... of column n0 + r; the four partial sums
        // of a column meet through lane exchanges in a fixed order
        float s = 0.f;
        if (n0 + r < Nout)
            for (int m = q; m < M; m += 4) s += dZ[(size_t)m * Nout + n0 + r];
        s += __shfl_xor(s, 16, kWave);
        s += __shfl_xor(s, 32, kWave);
        if (q == 0 && n0 + r < Nout) b[n0 + r] -= lr * s;
    }
    if (k0 >= Kin) return;
    const bool n_ok = n0 + r < Nout;
    const int ncol = min(n0 + r, Nout - 1);
    f32x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // tile layout: lane -> column r (k = k0 + 4 r + t); register i -> row 4 q + i (n index)
    const int k = k0 + 4 * r, left = Kin - k;          // left <= 0: this lane has no columns
    float4 wv[4];
    if (MB > 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = n0 + 4 * q + i;
            wv[i] = piece(W + (size_t)n * Kin + k, n < Nout ? left : 0);
        }
    }
    constexpr int UB = MB > 0 ? MB : 1;
    const int mend = MB > 0 ? 16 * MB : M;
    for (int mb = 0; mb < mend; mb += 16 * UB) {
        float a[UB][4];
        float4 x[UB][4];
#pragma unroll
        for (int v = 0; v < UB; ++v)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int m = mb + 16 * v + 4 * u + q;
                const bool m_ok = m < M;
                const int mm = min(m, M - 1);
                a[v][u] = (m_ok && n_ok) ? dZ[(size_t)mm * Nout + ncol] : 0.f;
                x[v][u] = piece(Aprev + (size_t)mm * Kin + k, m_ok ? left : 0);
            }
#pragma unroll
        for (int v = 0; v < UB; ++v)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][u], x[v][u].x, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][u], x[v][u].y, acc[1], 0, 0, 0);
                acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][u], x[v][u].z, acc[2], 0, 0, 0);
                acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[v][u], x[v][u].w, acc[3], 0, 0, 0);
            }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int n = n0 + 4 * q + i;
        float* dst = W + (size_t)n * Kin + k;
        const int l = n < Nout ? left : 0;
        float4 v = MB > 0 ? wv[i] : piece(dst, l);
        v.x -= lr * acc[0][i]; v.y -= lr * acc[1][i]; v.z -= lr * acc[2][i]; v.w -= lr * acc[3][i];
        store4u(dst, v, l);
    }
}

// One workgroup of 16 wavefronts: per row log-sum-exp, the row's loss, dZ = (softmax - onehot) / M
// in place over the logits, and the batch's mean loss (rows summed in order).  M <= 1024.
__global__ __launch_bounds__(1024) void mlp_ce_kernel(float* __restrict__ Z, const int32_t* __restrict__ y,
                                                      float* __restrict__ loss, int M, int O) {
    __shared__ float rowloss[1024];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const float inv = 1.0f / (float)M;
    for (int row = wave; row < M; row += 16) {
        float* z = Z + (size_t)row * O;
        const int yy = y[row];
        float m = -INFINITY;
        for (int k = lane; k < O; k += kWave) m = fmaxf(m, z[k]);
        m = max64(m);
        float s = 0.f;
        for (int k = lane; k < O; k += kWave) s += __expf(z[k] - m);
        s = sum64(s);
        const float lse = m + __logf(s);
        if (lane == 0) rowloss[row] = lse - z[yy];
        for (int k = lane; k < O; k += kWave) {
            float d = __expf(z[k] - lse);
            if (k == yy) d -= 1.f;
            z[k] = d * inv;
        }
    }
    __syncthreads();
    if (wave == 0) {   // fixed order: lane l adds rows l, l + 64, ...; then the lanes in a fixed tree
        float s = 0.f;
        for (int r = lane; r < M; r += kWave) s += rowloss[r];
        s = sum64(s);
        if (lane == 0) *loss = s * inv;
    }
}

// ---- all batches of a call in one launch: at most one hidden layer ------------------------------------
//
// What bounds the launches above at these sizes is the launches themselves (4 us each, 4 per batch with
// one hidden layer).  Here the model stays in registers from batch to batch: workgroup p owns hidden units
// 16p .. 16p+15 with their rows of W_1 (or, without a hidden layer, one workgroup owns the classes), its
// eight wavefronts the blocks of 16 inputs w, w + 8, ...  A lane's registers hold W[n = lane % 16]
// [k = 4 (lane / 16) + e] of a block, which is the operand v_mfma_f32_16x16x4_f32 wants for the forward
// product (walking k in that order) and also the layout in which it leaves dW^T = X^T dZ: the update
// is a subtraction in place.  Of W_2 a workgroup keeps its 16 columns.  The only thing workgroups
// exchange per batch is logits: every workgroup publishes its share of them and either (few
// words: P * batch * classes <= ONE_HOP) everyone adds up all shares and forms the same softmax, or the
// rows are dealt to the workgroups, which add them up and publish dZ.  Words carry the batch's number
// as their tag (tagged_store).  The shares alternate between two boxes: a workgroup can write share i+2
// only when it has everyone's share i+1, which they publish after they have read share i.  Sums run in
// a fixed order.
//
// Per batch, launches -> this (calls of 200 batches, inputs in the caches): 784-500-10 single examples 17.1 -> 4.9 us,
// 10 rows 18.0 -> 8.1, 60 rows 22.3 -> 17.5; 784-10 single examples 9.1 -> 1.7 us, 10 rows 9.4 -> 3.4, 60 rows
// 13.5 -> 11.9.  With the inputs coming from memory (calls of 400 batches): 60 rows of 784-500-10 22.9 -> 18.0, of 784-10
// 14.5 -> 14.1.
constexpr int OT = 512, OW = OT / kWave, ONE_HOP = 2048, ONE_BATCHES = 1024;
constexpr int ONE_SPINS = 1 << 26;   // a bound, not a time-out: the launch is cooperative

struct MlpOneArgs {
    const float* X; const int32_t* y;
    float *W1, *b1, *W2, *b2;        // no hidden layer: W1, b1 are the output layer's
    float* losses;                   // nullable
    unsigned long long *zbox, *dbox; // [2][P][B * O] shares of the logits; [B][O + 1] dZ and row losses
    int B, K, H, O, P, act, rows_per, n_batches;   // rows_per: rows a workgroup adds up (B: one hop)
    float lr;
};

// K is covered by 8 * KB blocks of 16 inputs, the batch by TILES tiles of 16 rows.  TILES = 0: one example,
// multiplied on the vector units (a matrix instruction would compute 16 rows for it).
template <bool HID, int KB, int TILES>
__global__ __launch_bounds__(OT, 2) void mlp_one_kernel(const MlpOneArgs a) {
    constexpr bool SINGLE = TILES == 0;
    constexpr int MT = SINGLE ? 1 : TILES, MR = SINGLE ? 1 : 16 * MT;
    __shared__ float red[OW][4 * MT][kWave];
    __shared__ float a_s[MR][17], dz_s[MR][17], d1_s[MR][17], w2_s[16][17], b1_s[16], b2_s[16], rowloss[64];
    __shared__ float zp[ONE_HOP];
    __shared__ int s_fail;
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int g = lane / 16, nn = lane % 16;
    const int B = a.B, K = a.K, O = a.O, P = a.P, wg = blockIdx.x;
    const int N1 = HID ? a.H : O, n0 = wg * 16, n1 = min(n0 + nn, N1 - 1);
    const bool n_on = n0 + nn < N1;

    float w[KB][4];
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 16 * (wave + OW * b) + 4 * g + e;
            const float v = a.W1[(size_t)n1 * K + min(k, K - 1)];
            w[b][e] = n_on && k < K ? v : 0.f;
        }
    if (tid < 16) {
        b1_s[tid] = n0 + tid < N1 ? a.b1[n0 + tid] : 0.f;
        b2_s[tid] = HID && tid < O ? a.b2[tid] : 0.f;
    }
    if (HID && tid < 256) {
        const int c = tid / 16, n = tid % 16;
        w2_s[c][n] = c < O && n0 + n < a.H ? a.W2[(size_t)c * a.H + n0 + n] : 0.f;
    }
    if (tid == 0) s_fail = 0;

    // The batch as the forward product reads it: row m = 16 mt + nn, inputs 4 g .. 4 g + 3 of each block;
    // as the update reads it: row m = 4 u + g, input nn of each block.  Buffer requests: one lane offset per
    // row for all blocks, the block in the scalar base.  What does not exist reads as zero, by the request's
    // bound: rows past the batch, blocks past the end of a row and, in the forward product, the pieces past
    // it (an infinite input of the next row must not meet the zero weights there).  The update's requests
    // may read into the next row: those columns of W are set to zero after it.
    // With two tiles of rows those past the batch repeat its last one in the forward product (nothing takes
    // their results) and whole blocks are asked for without the check of their pieces: 784-126-10, 21 rows 9.44 ->
    // 9.21 us per batch, 784-10 6.25 -> 5.65; with one tile that costs 3 % and with four 5.
    constexpr unsigned NONE = 0x80000000u;
    float4 xa[MT][KB];
    unsigned row_a[MT], row_t[4 * MT];   // bytes
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int m = 16 * mt + nn;
        row_a[mt] = SINGLE ? 16u * g : m < B || MT == 2 ? (unsigned)(min(m, B - 1) * K + 4 * g) * 4u : NONE;
    }
#pragma unroll
    for (int u = 0; u < 4 * MT; ++u) row_t[u] = 4 * u + g < B ? (unsigned)((4 * u + g) * K + nn) * 4u : NONE;
    auto window = [&](int batch, int b) {
        const int k = 16 * (wave + OW * b);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.X + (size_t)batch * B * K + min(k, K)), 0, k < K ? (B * K - k) * 4 : 0, 0x00020000);
    };
    auto load_rows = [&](int batch) {
        if (MT == 2 && K % 16 == 0) {
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                const auto x = window(batch, b);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    xa[mt][b] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(x, row_a[mt], 0, 0));
            }
            return;
        }
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            const auto x = window(batch, b);
            const bool in = SINGLE || 16 * (wave + OW * b) + 4 * g < K;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
                xa[mt][b] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(x, in ? row_a[mt] : NONE, 0, 0));
        }
    };
    auto load_t = [&](int batch, int b, float (&v)[4 * MT]) {
        const auto x = window(batch, b);
#pragma unroll
        for (int u = 0; u < 4 * MT; ++u) v[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(x, row_t[u], 0, 0));
    };
    // which words this thread writes and waits for: the same for every batch
    const int r0 = HID ? (a.rows_per == B ? 0 : min(wg * a.rows_per, B)) : 0;
    const int r1 = HID ? min(r0 + a.rows_per, B) : B, per = (r1 - r0) * O;
    int zm[2], zc[2], zat[4], dm[4], dc[4];   // -1: no such word
    if (HID) {
#pragma unroll
        for (int u = 0; u < 2; ++u) { const int v = tid + OT * u; zm[u] = v < B * O ? v / O : -1; zc[u] = v % O; }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = tid + OT * u;
            zat[u] = v < per * P ? (v / per) * B * O + r0 * O + v % per : -1;
            dm[u] = v < B * (O + 1) ? v / (O + 1) : -1;
            dc[u] = v % (O + 1);
        }
    }
    auto await = [&](const unsigned long long* box, const long long (&at)[4], unsigned tag, unsigned long long (&word)[4]) {
        if (!wait4(box, at, tag, ONE_SPINS, word)) s_fail = 1;
    };
    load_rows(0);
    __syncthreads();

    for (int i = 0; i < a.n_batches; ++i) {
        const unsigned tag = (unsigned)i + 1u;
        // ---- forward product of this workgroup's 16 units ------------------------------------------
        float4 xc[SINGLE ? KB : 1];    // the single example, for the update
        if constexpr (SINGLE) {
            float sum[2] = {0.f, 0.f};
#pragma unroll
            for (int b = 0; b < KB; ++b) {
                const float4 v = xc[b] = xa[0][b];
                sum[b & 1] = fmaf(v.x, w[b][0], sum[b & 1]); sum[b & 1] = fmaf(v.y, w[b][1], sum[b & 1]);
                sum[b & 1] = fmaf(v.z, w[b][2], sum[b & 1]); sum[b & 1] = fmaf(v.w, w[b][3], sum[b & 1]);
            }
            const float all = swap32_sum(swap16_sum(sum[0] + sum[1]));
            if (g == 0) red[wave][0][nn] = all;
        } else {
            f32x4 acc[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const float4 v = xa[mt][b];
                        acc[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w, w[b][e], acc[mt], 0, 0, 0);
                    }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int e = 0; e < 4; ++e) red[wave][4 * mt + e][lane] = acc[mt][e];
        }
        // The update's operands: all of them now, where there are few, else block by block later; and
        // the next batch's rows.  Both arrive while the workgroups exchange their shares.
        constexpr bool EARLY = MT == 1;
        float xt[EARLY ? KB : 2][4 * MT];
        if (!SINGLE)
#pragma unroll
            for (int b = 0; b < (EARLY ? KB : 1); ++b) load_t(i, b, xt[b]);
        if (MT < 4) load_rows(min(i + 1, a.n_batches - 1));   // (four tiles: no registers for both; see the end)
        lds_barrier();
        for (int v = tid; v < MR * 16; v += OT) {
            const int q = v / kWave, l = v % kWave, m = 16 * (q / 4) + 4 * (l / 16) + q % 4, n = l % 16;
            float sum = b1_s[n];
#pragma unroll
            for (int ww = 0; ww < OW; ++ww) sum += red[ww][q][l];
            const bool on = m < B && n0 + n < N1;
            if (HID) sum = a.act == RNN_ACT_SIGMOID ? sigmoidf_fast(sum) : tanhf_fast(sum);
            a_s[m][n] = on ? sum : 0.f;
        }
        lds_barrier();
        // ---- logits of rows [r0, r1), shares of all workgroups added in order ------------------------
        if (HID) {
            unsigned long long* zb = a.zbox + (size_t)(i & 1) * P * B * O;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (zm[u] < 0) continue;
                float sum = 0.f;
#pragma unroll
                for (int n = 0; n < 16; ++n) sum = fmaf(a_s[zm[u]][n], w2_s[zc[u]][n], sum);
                tagged_store(zb + (size_t)wg * B * O + tid + OT * u, tag, sum);
            }
            if (zat[0] >= 0) {
                unsigned long long word[4];
                await(zb, {zat[0], zat[1], zat[2], zat[3]}, tag, word);
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (zat[u] >= 0) zp[tid + OT * u] = tagged_value(word[u]);
            }
            lds_barrier();
        }
        // ---- softmax, loss and dZ of those rows: 16 lanes per row -------------------------------------
        const int32_t* yb = a.y + (size_t)i * B;
        for (int r = r0 + 4 * wave + g; r < r0 + ((r1 - r0 + 3) / 4) * 4; r += 4 * OW) {
            const bool ok = r < r1 && nn < O;
            float z = 0.f;
            if (HID) {
                z = b2_s[nn];
                if (ok) {
                    const float* q = zp + (r - r0) * O + nn;
#pragma unroll 8
                    for (int p = 0; p < P; ++p) z += q[p * per];
                }
            } else if (ok) {
                z = a_s[r][nn];
            }
            const int yy = r < r1 ? yb[r] : -1;
            const float mx = max16(ok ? z : -INFINITY);
            const float lse = mx + __logf(sum16(ok ? __expf(z - mx) : 0.f));
            const float loss = lse - sum16(ok && nn == yy ? z : 0.f);
            const float d = ok ? (__expf(z - lse) - (nn == yy ? 1.f : 0.f)) * (1.0f / (float)B) : 0.f;
            if (HID && a.rows_per != B) {
                if (ok) tagged_store(a.dbox + (size_t)r * (O + 1) + nn, tag, d);
                if (r < r1 && nn == 0) tagged_store(a.dbox + (size_t)r * (O + 1) + O, tag, loss);
            } else if (r < r1) {
                dz_s[r][nn] = d;
                if (nn == 0) rowloss[r] = loss;
            }
        }
        if (HID && a.rows_per != B) {
            unsigned long long word[4];
            if (dm[0] >= 0) {
                long long at[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) at[u] = dm[u] < 0 ? -1 : tid + OT * u;
                await(a.dbox, at, tag, word);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (dm[u] < 0) continue;
                    if (dc[u] < O) dz_s[dm[u]][dc[u]] = tagged_value(word[u]);
                    else rowloss[dm[u]] = tagged_value(word[u]);
                }
            }
        }
        // columns and rows that do not exist: zero (the products below run over whole tiles)
        for (int v = tid; v < MR * 16; v += OT)
            if (v / 16 >= B || v % 16 >= O) dz_s[v / 16][v % 16] = 0.f;
        lds_barrier();
        if (s_fail) {                // cannot happen while the workgroups are co-resident
            if (wg == 0 && tid == 0 && a.losses)
                for (int j = i; j < a.n_batches; ++j) a.losses[j] = __uint_as_float(0x7fc00000u);
            return;
        }
        if (wg == 0 && wave == 0 && a.losses) {
            const float sum = sum64(lane < B ? rowloss[lane] : 0.f);
            if (lane == 0) a.losses[i] = sum / (float)B;
        }
        // ---- dZ of the hidden units -------------------------------------------------------------------
        if (HID) {
            for (int v = tid; v < MR * 16; v += OT) {
                const int m = v / 16, n = v % 16;
                float sum = 0.f;
#pragma unroll
                for (int c = 0; c < 16; ++c) sum = fmaf(dz_s[m][c], w2_s[c][n], sum);
                const float h = a_s[m][n];
                d1_s[m][n] = m < B && n0 + n < N1 ? sum * (a.act == RNN_ACT_SIGMOID ? act_grad<0>(h) : act_grad<1>(h)) : 0.f;
            }
            lds_barrier();
        }
        const float(*d1)[17] = HID ? d1_s : dz_s;
        // ---- updates ----------------------------------------------------------------------------------
#pragma unroll
        for (int b = 0; b < KB; ++b) {
            f32x4 dw = {0.f, 0.f, 0.f, 0.f};
            if constexpr (SINGLE) {
                const float d = d1[0][nn];
                dw = (f32x4){xc[b].x * d, xc[b].y * d, xc[b].z * d, xc[b].w * d};
            } else {
                if (!EARLY && b + 1 < KB) load_t(i, b + 1, xt[(b + 1) & 1]);
                if (!EARLY) __builtin_amdgcn_sched_barrier(0);       // one block ahead and no more
#pragma unroll
                for (int u = 0; u < 4 * MT; ++u)
                    dw = __builtin_amdgcn_mfma_f32_16x16x4f32(xt[EARLY ? b : b & 1][u], d1[4 * u + g][nn], dw, 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) w[b][e] -= a.lr * dw[e];
            if (16 * (wave + OW * b) + 16 > K)                   // the ragged last block: K % 4 == 0
#pragma unroll
                for (int e = 0; e < 4; ++e) w[b][e] = 16 * (wave + OW * b) + 4 * g < K ? w[b][e] : 0.f;
        }
        if (wave == OW - 1 || (HID && wave >= OW - 3)) {
            if (wave == OW - 1) {            // b_1 (no hidden layer: b)
                float sum = 0.f;
                for (int m = g; m < MR; m += 4) sum += d1[m][nn];
                sum = swap32_sum(swap16_sum(sum));
                if (g == 0) b1_s[nn] -= a.lr * sum;
            } else if (wave == OW - 2) {     // b_2: the same in every workgroup
                float sum = 0.f;
                for (int m = g; m < MR; m += 4) sum += dz_s[m][nn];
                sum = swap32_sum(swap16_sum(sum));
                if (g == 0) b2_s[nn] -= a.lr * sum;
            } else {                         // W_2's columns: rows 4 g + e, column nn
                f32x4 dw = {0.f, 0.f, 0.f, 0.f};
                if constexpr (SINGLE) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) dw[e] = dz_s[0][4 * g + e] * a_s[0][nn];
                } else {
#pragma unroll
                    for (int u = 0; u < 4 * MT; ++u) dw = __builtin_amdgcn_mfma_f32_16x16x4f32(dz_s[4 * u + g][nn], a_s[4 * u + g][nn], dw, 0, 0, 0);
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) w2_s[4 * g + e][nn] -= a.lr * dw[e];
            }
        }
        if (MT == 4) load_rows(min(i + 1, a.n_batches - 1));
        lds_barrier();
    }
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 16 * (wave + OW * b) + 4 * g + e;
            if (n_on && k < K) a.W1[(size_t)n1 * K + k] = w[b][e];
        }
    if (tid < 16) {
        if (n0 + tid < N1) a.b1[n0 + tid] = b1_s[tid];
        if (HID && wg == 0 && tid < O) a.b2[tid] = b2_s[tid];
    }
    if (HID && tid < 256) {
        const int c = tid / 16, n = tid % 16;
        if (c < O && n0 + n < a.H) a.W2[(size_t)c * a.H + n0 + n] = w2_s[c][n];
    }
}

// Shapes the one-launch kernel holds: rows of whole 16-byte pieces, 7 blocks of 16 inputs per wavefront (the form of
// four row tiles with a hidden layer takes all 256 registers and 48 bytes of scratch with 7), 64 rows, 16 classes, and no more
// hidden units than 64 workgroups own (beyond that polling the shares costs what launches do).  Without a hidden layer
// one workgroup does all the work, which still gains at the largest batch: 64 rows of 784 inputs 13.9 -> 12.0 us, from
// memory 14.8 -> 14.5; of 896 inputs 14.8 -> 13.9, from memory 15.3 -> 15.4.
bool mlp_one_supported(const rnn_mlp_dims* d) {
    return d->n_hidden <= 1 && d->out_dim <= 16 && d->batch <= 64 && d->in_dim % 4 == 0 && d->in_dim <= 896 && (d->n_hidden == 0 || d->hidden <= 1024);
}
int mlp_one_wgs(const rnn_mlp_dims* d) { return d->n_hidden ? (d->hidden + 15) / 16 : 1; }

template <bool HID>
const void* mlp_one_pick(int K, int B) {
#define RNN_ONE(KB) (B == 1 ? (const void*)mlp_one_kernel<HID, KB, 0> : B <= 16 ? (const void*)mlp_one_kernel<HID, KB, 1> : B <= 32 ? (const void*)mlp_one_kernel<HID, KB, 2> : (const void*)mlp_one_kernel<HID, KB, 4>)
    return K <= 256 ? RNN_ONE(2) : RNN_ONE(7);
#undef RNN_ONE
}

struct Widths { int w[RNN_MLP_MAX_LAYERS + 2]; int layers; };

bool mlp_dims_ok(const rnn_mlp_dims* d) {
    if (!d) return false;
    if (d->in_dim <= 0 || d->out_dim <= 0 || d->batch <= 0 || d->n_hidden < 0) return false;
    if (d->n_hidden + 1 > RNN_MLP_MAX_LAYERS) return false;
    if (d->n_hidden > 0 && d->hidden <= 0) return false;
    if (d->act != RNN_ACT_SIGMOID && d->act != RNN_ACT_TANH) return false;
    if (d->flags & ~RNN_FLAG_SYNC) return false;
    if (d->in_dim > (1 << 20) || d->hidden > (1 << 20) || d->out_dim > (1 << 20)) return false;
    return true;
}

Widths widths_of(const rnn_mlp_dims* d) {
    Widths w;
    w.layers = d->n_hidden + 1;
    w.w[0] = d->in_dim;
    for (int l = 1; l <= d->n_hidden; ++l) w.w[l] = d->hidden;
    w.w[w.layers] = d->out_dim;
    return w;
}

inline size_t up256(size_t v) { return (v + 255) / 256 * 256; }

// workspace: activations of the hidden layers, logits / dZ of the output layer, two dZ buffers of
// the hidden width
struct MlpPlan { size_t act[RNN_MLP_MAX_LAYERS + 1], Z, dz[RNN_MLP_MAX_LAYERS], losspart, zbox, dbox, total; };

MlpPlan mlp_plan(const rnn_mlp_dims* d) {
    const Widths w = widths_of(d);
    MlpPlan p{};
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += up256(bytes); return o; };
    for (int l = 1; l < w.layers; ++l) p.act[l] = take((size_t)d->batch * w.w[l] * 4);
    p.Z = take((size_t)d->batch * d->out_dim * 4);
    // dZ of layer l's outputs, l < layers - 1 (the last layer's is Z itself, in place)
    for (int l = 0; l + 1 < w.layers; ++l) p.dz[l] = take((size_t)d->batch * w.w[l + 1] * 4);
    p.losspart = take((size_t)((d->batch + 15) / 16 + 1) * 4);   // + one word that takes the loss when the caller wants none
    const bool boxes = d->n_hidden == 1 && mlp_one_supported(d);
    p.zbox = take(boxes ? (size_t)2 * mlp_one_wgs(d) * d->batch * d->out_dim * 8 : 0);
    p.dbox = take(boxes ? (size_t)d->batch * (d->out_dim + 1) * 8 : 0);
    p.total = off;
    return p;
}

bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

hipError_t launch_fwd(int act, const float* A, const float* W, const float* b, float* C, int M, int N, int K,
                      hipStream_t s) {
    dim3 grid(tiles_of((N + 15) / 16, M));
    const bool vec = K % 4 == 0 && al16(A) && al16(W);
    ProfileScope ps(K_MLP_FWD, s);
#define RNN_MLP_FWD(ACT)                                                                              \
    do {                                                                                              \
        if (vec) hipLaunchKernelGGL((mlp_fwd_kernel<ACT, true>), grid, dim3(MNT), 0, s, A, W, b, C, M, N, K, nullptr, nullptr);  \
        else hipLaunchKernelGGL((mlp_fwd_kernel<ACT, false>), grid, dim3(MNT), 0, s, A, W, b, C, M, N, K, nullptr, nullptr);     \
    } while (0)
    if (act == 0) RNN_MLP_FWD(0); else if (act == 1) RNN_MLP_FWD(1); else RNN_MLP_FWD(2);
#undef RNN_MLP_FWD
    return hipGetLastError();
}

// output layer of at most 16 classes with the loss in its epilogue
hipError_t launch_fwd_ce(const float* A, const float* W, const float* b, float* dZ, int M, int N, int K,
                         const int32_t* y, float* losspart, hipStream_t s) {
    dim3 grid(tiles_of(1, M));
    const bool vec = K % 4 == 0 && al16(A) && al16(W);
    ProfileScope ps(K_MLP_FWD, s);
    if (vec) hipLaunchKernelGGL((mlp_fwd_kernel<2, true, true>), grid, dim3(MNT), 0, s, A, W, b, dZ, M, N, K, y, losspart);
    else hipLaunchKernelGGL((mlp_fwd_kernel<2, false, true>), grid, dim3(MNT), 0, s, A, W, b, dZ, M, N, K, y, losspart);
    return hipGetLastError();
}

// Are the workgroups of the one-launch kernel co-resident on the current device?
bool mlp_one_ready(const void* fn, int wgs) {
    int dev = 0, per_cu = 0, cus = 0;
    return hipGetDevice(&dev) == hipSuccess &&
           hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, OT, 0) == hipSuccess &&
           hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && per_cu * cus >= wgs;
}

hipError_t run_mlp_one(const rnn_mlp_dims* d, const rnn_mlp_params* p, const float* X, const int32_t* y, int64_t n_batches,
                       float lr, float* losses, char* ws, const MlpPlan& pl, const void* fn, hipStream_t s) {
    MlpOneArgs a{};
    const bool hid = d->n_hidden == 1;
    a.W1 = p->W[0]; a.b1 = p->b[0]; a.W2 = hid ? p->W[1] : nullptr; a.b2 = hid ? p->b[1] : nullptr;
    a.zbox = reinterpret_cast<unsigned long long*>(ws + pl.zbox);
    a.dbox = reinterpret_cast<unsigned long long*>(ws + pl.dbox);
    a.B = d->batch; a.K = d->in_dim; a.H = d->hidden; a.O = d->out_dim; a.P = mlp_one_wgs(d); a.act = d->act; a.lr = lr;
    a.rows_per = !hid || a.P * a.B * a.O <= ONE_HOP ? a.B : (a.B + a.P - 1) / a.P;
    for (int64_t i = 0; i < n_batches; i += ONE_BATCHES) {
        a.X = X + (size_t)i * a.B * a.K;
        a.y = y + (size_t)i * a.B;
        a.losses = losses ? losses + i : nullptr;
        a.n_batches = (int)(n_batches - i < ONE_BATCHES ? n_batches - i : ONE_BATCHES);
        hipError_t e = hipSuccess;
        if (hid) {   // cleared words are "not written yet"
            ProfileScope ps(K_MISC, s);
            e = launch_zero_words(reinterpret_cast<int32_t*>(ws + pl.zbox), (int)((pl.total - pl.zbox) / 4), s);
            if (e != hipSuccess) return e;
        }
        ProfileScope ps(K_MLP_ONE, s);
        void* args[] = {&a};
        e = hid ? launch_gang(fn, dim3(a.P), dim3(OT), args, 0, s) : hipLaunchKernel(fn, dim3(1), dim3(OT), args, 0, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace
}  // namespace rnn

extern "C" {

int rnn_mlp_workspace_bytes(const rnn_mlp_dims* dims, size_t* bytes) {
    if (!rnn::mlp_dims_ok(dims) || !bytes) return RNN_EINVAL;
    *bytes = rnn::mlp_plan(dims).total;
    return RNN_OK;
}

int rnn_mlp_train(const rnn_mlp_dims* dims, const rnn_mlp_params* params, const float* X, const int32_t* y,
                  int64_t n_batches, float lr, float* losses, void* workspace, size_t workspace_bytes,
                  void* hip_stream) {
    using namespace rnn;
    if (!mlp_dims_ok(dims) || !params || !X || !y || n_batches < 0) return RNN_EINVAL;
    if (dims->batch > 1024) return RNN_EUNSUPPORTED;
    const Widths w = widths_of(dims);
    for (int l = 0; l < w.layers; ++l)
        if (!params->W[l] || !params->b[l] || !al16(params->W[l]) || !al16(params->b[l])) return RNN_EINVAL;
    if ((reinterpret_cast<uintptr_t>(X) & 15u) || (reinterpret_cast<uintptr_t>(y) & 3u) ||
        (reinterpret_cast<uintptr_t>(losses) & 3u))
        return RNN_EINVAL;
    const MlpPlan pl = mlp_plan(dims);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 15u) || workspace_bytes < pl.total)
        return RNN_EWORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    char* ws = static_cast<char*>(workspace);
    const int B = dims->batch, L = w.layers;
    if (n_batches > 0 && mlp_one_supported(dims)) {
        const void* fn = dims->n_hidden ? mlp_one_pick<true>(dims->in_dim, B) : mlp_one_pick<false>(dims->in_dim, B);
        if (!dims->n_hidden || mlp_one_ready(fn, mlp_one_wgs(dims))) {
            if (run_mlp_one(dims, params, X, y, n_batches, lr, losses, ws, pl, fn, s) != hipSuccess) return RNN_EHIP;
            if (dims->flags & RNN_FLAG_SYNC)
                if (hipStreamSynchronize(s) != hipSuccess) return RNN_EHIP;
            return RNN_OK;
        }
    }
    float* Z = reinterpret_cast<float*>(ws + pl.Z);
    // the one update launch of a batch: every layer's grid, one after another
    // at most 16 classes: the output layer's tile holds whole rows, its epilogue forms the loss and
    // dZ, and the update launch adds up the batch's loss
    const bool fused_ce = dims->out_dim <= 16;
    float* losspart = reinterpret_cast<float*>(ws + pl.losspart);
    float* scratch_loss = losspart + (B + 15) / 16;   // when the caller wants no losses
    const bool fused_out = fused_ce && dims->n_hidden >= 2 && dims->hidden <= MW * MKC;   // output layer, loss and two backward products
    UpdateLayers ul{};
    ul.layers = L;
    ul.losspart = losspart;
    ul.nparts = fused_ce ? (B + 15) / 16 : 0;
    int total_wgs = 0;
    for (int l = 0; l < L; ++l) {
        ul.dZ[l] = l + 1 < L ? reinterpret_cast<const float*>(ws + pl.dz[l]) : Z;
        ul.W[l] = params->W[l];
        ul.b[l] = params->b[l];
        ul.Nout[l] = w.w[l + 1];
        ul.Kin[l] = w.w[l];
        ul.gx[l] = (w.w[l] + 255) / 256;
        ul.first[l] = total_wgs;
        total_wgs += ul.gx[l] * ((w.w[l + 1] + 15) / 16);
    }
    ul.first[L] = total_wgs;
    for (int64_t i = 0; i < n_batches; ++i) {
        const float* x_in = X + (size_t)i * B * dims->in_dim;
        const float* a_prev = x_in;
        // forward
        float* loss_out = losses ? losses + i : scratch_loss;
        for (int l = 0; l < (fused_out ? L - 1 : L); ++l) {
            float* out = l + 1 < L ? reinterpret_cast<float*>(ws + pl.act[l + 1]) : Z;
            hipError_t e;
            if (l + 1 == L && fused_ce)
                e = launch_fwd_ce(a_prev, params->W[l], params->b[l], Z, B, w.w[l + 1], w.w[l], y + (size_t)i * B,
                                  losspart, s);
            else
                e = launch_fwd(l + 1 < L ? dims->act : 2, a_prev, params->W[l], params->b[l], out, B, w.w[l + 1],
                               w.w[l], s);
            if (e != hipSuccess) return RNN_EHIP;
            a_prev = out;
        }
        if (!fused_ce) {
            ProfileScope ps(K_MLP_CE, s);
            hipLaunchKernelGGL(mlp_ce_kernel, dim3(1), dim3(1024), 0, s, Z, y + (size_t)i * B, loss_out, B,
                               dims->out_dim);
            if (hipGetLastError() != hipSuccess) return RNN_EHIP;
        }
        // backward: dZ_{l-1} from dZ_l and the weights as they were in the forward pass, layer by
        // layer; every dZ_l is kept, and one launch then updates all W_l and b_l in place
        const float* dz = Z;
        if (fused_out) {
            const int H = dims->hidden;
            float* dz_prev = reinterpret_cast<float*>(ws + pl.dz[L - 3]);
            dim3 grid(tiles_of((H + 15) / 16, B));
            ProfileScope ps(K_MLP_BWD, s);
#define RNN_MLP_OUT(ACT, VEC)                                                                                       \
    hipLaunchKernelGGL((mlp_out_bwd_kernel<ACT, VEC>), grid, dim3(MNT), 0, s, a_prev, params->W[L - 1], params->b[L - 1], \
                       y + (size_t)i * B, params->W[L - 2], reinterpret_cast<const float*>(ws + pl.act[L - 2]), Z,  \
                       reinterpret_cast<float*>(ws + pl.dz[L - 2]), dz_prev, losspart, B, w.w[L], H, H)
            if (dims->act == 0) { if (H % 4 == 0) RNN_MLP_OUT(0, true); else RNN_MLP_OUT(0, false); }
            else { if (H % 4 == 0) RNN_MLP_OUT(1, true); else RNN_MLP_OUT(1, false); }
#undef RNN_MLP_OUT
            if (hipGetLastError() != hipSuccess) return RNN_EHIP;
            dz = dz_prev;
        }
        for (int l = fused_out ? L - 3 : L - 1; l > 0; --l) {
            const float* a_in = reinterpret_cast<const float*>(ws + pl.act[l]);
            float* dz_prev = reinterpret_cast<float*>(ws + pl.dz[l - 1]);
            dim3 grid(tiles_of((w.w[l] + 15) / 16, B));
            ProfileScope ps(K_MLP_BWD, s);
            const bool vec = w.w[l + 1] % 4 == 0;   // dZ rows stay 16-byte aligned (workspace regions are)
#define RNN_MLP_BWD(ACT, VEC)                                                                              \
    hipLaunchKernelGGL((mlp_bwd_data_kernel<ACT, VEC>), grid, dim3(MNT), 0, s, dz, params->W[l], a_in, dz_prev, \
                       B, w.w[l + 1], w.w[l])
            if (dims->act == 0) { if (vec) RNN_MLP_BWD(0, true); else RNN_MLP_BWD(0, false); }
            else { if (vec) RNN_MLP_BWD(1, true); else RNN_MLP_BWD(1, false); }
#undef RNN_MLP_BWD
            if (hipGetLastError() != hipSuccess) return RNN_EHIP;
            dz = dz_prev;
        }
        {
            for (int l = 0; l < L; ++l)
                ul.Aprev[l] = l > 0 ? reinterpret_cast<const float*>(ws + pl.act[l]) : x_in;
            ul.loss = loss_out;
            ProfileScope ps(K_MLP_UPDATE, s);
#define RNN_MLP_UPD(MB) hipLaunchKernelGGL(mlp_update_kernel<MB>, dim3(total_wgs), dim3(256), 0, s, ul, B, lr)
            if (B <= 16) RNN_MLP_UPD(1); else if (B <= 32) RNN_MLP_UPD(2); else if (B <= 64) RNN_MLP_UPD(4);
            else RNN_MLP_UPD(0);
#undef RNN_MLP_UPD
            if (hipGetLastError() != hipSuccess) return RNN_EHIP;
        }
    }
    if (dims->flags & RNN_FLAG_SYNC)
        if (hipStreamSynchronize(s) != hipSuccess) return RNN_EHIP;
    return RNN_OK;
}

}  // extern "C"
