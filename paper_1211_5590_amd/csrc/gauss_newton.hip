// Small kernels of the Gauss-Newton-vector product (the paper's section on the R-operator):
// everything heavy in that product is one of the path's existing matrix products or time loops;
// what is left is re-ordering rows in time, adding gathered rows, and applying the Hessian of the
// loss with respect to the outputs to the rows of R z.
#include "common.hpp"
#include "internal.hpp"
#include "prof.hpp"

namespace rnn {
namespace {

// dst row t = src row T-1-t, rows of `row` floats
__global__ __launch_bounds__(256) void reverse_rows_kernel(const float* __restrict__ src, float* __restrict__ dst,
                                                           int T, int row) {
    const int t = blockIdx.y;
    const float* s = src + (size_t)(T - 1 - t) * row;
    float* d = dst + (size_t)t * row;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < row; i += gridDim.x * blockDim.x) d[i] = s[i];
}

// What the R-operator's sweep needs before its loop, in one launch of 256 threads per workgroup: the first workgroups turn rows
// of C (with the row of M that its token picks) and of Hs round in time, 2^txs threads a row, the next transpose a 32 x 32 tile of Wh
// each, and all fill a share of the loop's exchange words.  (Four launches before, 3 us each.  With a workgroup for every row
// however narrow, 524288 rows of 64 took 324 us, the four launches 273; now 168.)
struct GnPrepare {
    const int32_t* x; const float* M;          // x NULL: no gathered rows
    const float *C, *Hs, *Wh;
    float *Crev, *hrev, *WhT;
    int T, B, H, txs;
    FillJob ring, counters;
};
__host__ __device__ inline int gn_row_workgroups(int N, int txs) { return (int)(((size_t)N + (256 >> txs) - 1) >> (8 - txs)); }
__global__ __launch_bounds__(256) void gn_prepare_kernel(GnPrepare a) {
    const int H = a.H, N = a.T * a.B, tid = threadIdx.x;
    fill_share(a.ring.p, a.ring.n, a.ring.v, workgroup(), workgroups(), 256);
    fill_share(a.counters.p, a.counters.n, a.counters.v, workgroup(), workgroups(), 256);
    const int wg = (int)workgroup(), row_wgs = gn_row_workgroups(N, a.txs);
    if (wg < row_wgs) {
        if (((size_t)wg << (8 - a.txs)) + (tid >> a.txs) >= (size_t)N) return;
        const int n = (wg << (8 - a.txs)) + (tid >> a.txs), t = n / a.B, src = (a.T - 1 - t) * a.B + n % a.B;
        const float* row = a.x ? a.M + (size_t)a.x[src] * H : nullptr;
        const size_t from = (size_t)src * H, to = (size_t)n * H;
        for (int j = tid & ((1 << a.txs) - 1); j < H; j += 1 << a.txs) {
            const float c = a.C[from + j];
            a.Crev[to + j] = row ? c + row[j] : c;
            a.hrev[to + j] = a.Hs[from + j];
        }
        return;
    }
    __shared__ float tile[32][33];
    // (past the last tile: r0 >= H, nothing to move)
    const int side = (H + 31) / 32, b = wg - row_wgs, r0 = b / side * 32, c0 = b % side * 32, tx = tid % 32, ty = tid / 32;
    for (int i = ty; i < 32; i += 8)
        if (r0 + i < H && c0 + tx < H) tile[i][tx] = a.Wh[(size_t)(r0 + i) * H + c0 + tx];
    __syncthreads();
    for (int i = ty; i < 32; i += 8)
        if (c0 + i < H && r0 + tx < H) a.WhT[(size_t)(c0 + i) * H + r0 + tx] = tile[tx][i];
}

__global__ __launch_bounds__(256) void fill_zero_kernel(float* p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0.f;
}

__global__ __launch_bounds__(256) void scale_kernel(float* p, size_t n, float alpha) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] *= alpha;
}

// RZ_n <- (p * RZ_n - p (p . RZ_n)) * scale with p = softmax(Z_n), the product of the cross-entropy's Hessian with respect to the
// logits and RZ_n; R rows per workgroup: one, or one per wavefront.
// What bounds it is the memory it reads and writes, so both rows stay in registers between the three passes over them: P pieces
// of four per thread, all requested at once, at 4-byte alignment (a row starts anywhere).  Rows of more than 16384 classes
// are read again, a piece at a time.  (800 rows of 10000, one float at a time and every pass from memory: 41.8 us; now 12.5.)
// A wavefront holds rows of up to 1024 classes, and then needs no barrier: four pieces a lane.  (Rows with a workgroup and with a
// wavefront each, us: 524288 of 16 classes 939 and 129, 131072 of 300, 512, 800 and 1000 classes 256 and 74, 238 and 128, 316
// and 219, 338 and 292; 800 rows 6 to 8 either way.)
constexpr int GN_T = 512;                              // threads
template <int P, int R>
__global__ __launch_bounds__(GN_T) void gn_softmax_metric_kernel(const float* __restrict__ Z, float* __restrict__ RZ,
                                                                 int N, int O, float scale) {
    constexpr int TR = GN_T / R, NW = TR / kWave;      // threads and wavefronts of a row
    static_assert(R == 1 || NW == 1, "rows share no barrier");
    const size_t n = R == 1 ? workgroup() : workgroup() * R + __builtin_amdgcn_readfirstlane(threadIdx.x / TR);
    if (n >= (size_t)N) return;
    __shared__ float red[3][NW];
    const size_t base = n * O;
    const int tid = R == 1 ? threadIdx.x : threadIdx.x % TR, lane = tid & 63, wave = tid >> 6;
    const float* z = Z + base;
    float* rz = RZ + base;
    constexpr bool KEPT = P > 0;
    float4 e[KEPT ? P : 1], r[KEPT ? P : 1];
    const int steps = KEPT ? P : (O + 4 * TR - 1) / (4 * TR);
    auto at = [&](int u) { return 4 * (u * TR + tid); };
    auto logits = [&](int u) {                         // what does not exist takes no part: exp(-inf) = 0
        const int k = at(u), left = O - k;
        float4 v = piece(z + k, left);
        if (left < 4) {
            if (left < 1) v.x = -INFINITY;
            if (left < 2) v.y = -INFINITY;
            if (left < 3) v.z = -INFINITY;
            v.w = -INFINITY;
        }
        return v;
    };
    float m = -INFINITY;
#pragma unroll
    for (int u = 0; u < P; ++u) { e[u] = logits(u); r[u] = piece(rz + at(u), O - at(u)); }
    if constexpr (KEPT) {
#pragma unroll
        for (int u = 0; u < P; ++u) m = fmaxf(m, fmaxf(fmaxf(e[u].x, e[u].y), fmaxf(e[u].z, e[u].w)));
    } else {
        for (int u = 0; u < steps; ++u) { const float4 v = logits(u); m = fmaxf(m, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w))); }
    }
    m = max64(m);
    if constexpr (R == 1) {
        if (lane == 0) red[0][wave] = m;
        __syncthreads();
        m = red[0][0];
#pragma unroll
        for (int w = 1; w < NW; ++w) m = fmaxf(m, red[0][w]);
    }
    float s = 0.f, dot = 0.f;
    auto take = [&](float4& v, const float4& q) {      // v <- exp(v - m)
        v.x = exp_exact(v.x - m); v.y = exp_exact(v.y - m); v.z = exp_exact(v.z - m); v.w = exp_exact(v.w - m);
        s += (v.x + v.y) + (v.z + v.w);
        dot = fmaf(v.x, q.x, dot); dot = fmaf(v.y, q.y, dot); dot = fmaf(v.z, q.z, dot); dot = fmaf(v.w, q.w, dot);
    };
    if constexpr (KEPT) {
#pragma unroll
        for (int u = 0; u < P; ++u) take(e[u], r[u]);
    } else {
        for (int u = 0; u < steps; ++u) { float4 v = logits(u); take(v, piece(rz + at(u), O - at(u))); }
    }
    s = sum64(s);
    dot = sum64(dot);
    if constexpr (R == 1) {
        if (lane == 0) { red[1][wave] = s; red[2][wave] = dot; }
        __syncthreads();
        s = dot = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) { s += red[1][w]; dot += red[2][w]; }
    }
    const float inv = 1.0f / s;
    const float pdot = dot * inv;                      // p . RZ
    auto out = [&](int u, const float4& v, const float4& q) {
        const float4 o = make_float4(v.x * inv * (q.x - pdot) * scale, v.y * inv * (q.y - pdot) * scale,
                                     v.z * inv * (q.z - pdot) * scale, v.w * inv * (q.w - pdot) * scale);
        store4u(rz + at(u), o, O - at(u));
    };
    if constexpr (KEPT) {
#pragma unroll
        for (int u = 0; u < P; ++u) out(u, e[u], r[u]);
    } else {
        for (int u = 0; u < steps; ++u) {
            float4 v = logits(u);
            v.x = exp_exact(v.x - m); v.y = exp_exact(v.y - m); v.z = exp_exact(v.z - m); v.w = exp_exact(v.w - m);
            out(u, v, piece(rz + at(u), O - at(u)));
        }
    }
}

int blocks_for(size_t n) {
    const size_t b = (n + 255) / 256;
    return (int)(b < 1 ? 1 : (b > 4096 ? 4096 : b));
}

}  // namespace

hipError_t launch_reverse_rows(const float* src, float* dst, int T, int row, hipStream_t s) {
    ProfileScope ps(K_MISC, s);
    hipLaunchKernelGGL(reverse_rows_kernel, dim3(blocks_for((size_t)row), T), dim3(256), 0, s, src, dst, T, row);
    return hipGetLastError();
}
hipError_t launch_gn_prepare(const int32_t* x, const float* M, const float* C, const float* Hs, const float* Wh, float* Crev,
                             float* hrev, float* WhT, int T, int B, int H, FillJob ring, FillJob counters, hipStream_t s) {
    const int side = (H + 31) / 32;
    int txs = 0;
    while (txs < 8 && (1 << txs) < H) ++txs;
    const GnPrepare a = {x, M, C, Hs, Wh, Crev, hrev, WhT, T, B, H, txs, ring, counters};
    ProfileScope ps(K_MISC, s);
    hipLaunchKernelGGL(gn_prepare_kernel, grid_of((size_t)gn_row_workgroups(T * B, txs) + (size_t)side * side), dim3(256), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_fill_zero(float* p, size_t n, hipStream_t s) {
    ProfileScope ps(K_MISC, s);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks_for(n)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}
hipError_t launch_scale(float* p, size_t n, float alpha, hipStream_t s) {
    ProfileScope ps(K_GN_METRIC, s);
    hipLaunchKernelGGL(scale_kernel, dim3(blocks_for(n)), dim3(256), 0, s, p, n, alpha);
    return hipGetLastError();
}
hipError_t launch_gn_softmax_metric(const float* Z, float* RZ, int N, int O, float scale, hipStream_t s) {
    ProfileScope ps(K_GN_METRIC, s);
#define RNN_GN(P, R) hipLaunchKernelGGL((gn_softmax_metric_kernel<P, R>), grid_of(((size_t)N + R - 1) / R), dim3(GN_T), 0, s, Z, RZ, N, O, scale)
    constexpr int ROWS = GN_T / kWave;
    const int pieces = (O - 1) / (4 * GN_T) + 1;       // of a thread, where a row has a workgroup
    if (O <= 4 * kWave) RNN_GN(1, ROWS);
    else if (O <= 8 * kWave) RNN_GN(2, ROWS);
    else if (O <= 16 * kWave) RNN_GN(4, ROWS);
    else if (pieces <= 1) RNN_GN(1, 1);
    else if (pieces <= 3) RNN_GN(3, 1);
    else if (pieces <= 5) RNN_GN(5, 1);
    else if (pieces <= 8) RNN_GN(8, 1);
    else RNN_GN(0, 1);
#undef RNN_GN
    return hipGetLastError();
}

}  // namespace rnn
