// Gradient of the token-indexed input matrix, dWx[v,:] = sum over the rows n with x_n = v of
// Delta[n,:], without floating-point atomics: results are run-to-run identical however skewed
// (Zipf) the ids are, and the same pass writes the zero rows of tokens that do not occur.
//
// Grouped form (the normal one): the id list is cut into ranges of CL ids.  A workgroup per
// range and slice of columns sorts its (id, position) pairs in LDS (keys are unique), which groups equal ids
// with ascending positions, and sums the Delta rows of every group in that order into a compact
// partial row; a table [token][range] records which partial row, if any, belongs to a token
// (or, for a token that occurs once in the range, which row of Delta).
// A second kernel, one wavefront per vocabulary row, adds the token's partial rows in ascending
// range order.  Delta is read once and every sum has a fixed order.
//
// Scan form (a short id list): every wavefront owns one
// vocabulary row and scans the whole id list for its token.
#include "colsum_dev.hpp"
#include "common.hpp"
#include "internal.hpp"
#include "prof.hpp"

namespace rnn {
namespace {

constexpr int kQ = 16;                      // columns per lane per pass
constexpr int kColsPerPass = kQ * kWave;    // 1024: one pass for H <= 1024, many loads in flight

// Sum of the Delta rows whose id equals v among ids [n_begin, n_end), ascending n; 16 columns
// per lane starting at c0.  Returns whether any row matched.
__device__ __forceinline__ bool scan_token(const int32_t* __restrict__ x,
                                           const float* __restrict__ Delta, int v, int n_begin,
                                           int n_end, int H, int c0, int lane, float (&acc)[kQ]) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) acc[q] = 0.f;
    bool seen = false;
    for (int n0 = n_begin; n0 < n_end; n0 += kWave) {
        const int n = n0 + lane;
        const bool hit = n < n_end && x[n] == v;
        unsigned long long mask = __ballot(hit);
        while (mask) {
            const int src = __ffsll((long long)mask) - 1;
            mask &= mask - 1;
            seen = true;
            const float* row = Delta + (size_t)(n0 + src) * H;
#pragma unroll
            for (int q = 0; q < kQ; ++q) {
                const int col = c0 + q * kWave + lane;
                if (col < H) acc[q] += row[col];
            }
        }
    }
    return seen;
}

// Whole id list per wavefront (short lists).
__global__ __launch_bounds__(256) void dwx_tokens_kernel(const int32_t* __restrict__ x,
                                                         const float* __restrict__ Delta,
                                                         float* __restrict__ dWx, int N, int NV,
                                                         int H, int beta) {
    const int lane = threadIdx.x % kWave;
    const long long task = (long long)workgroup() * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (task >= NV) return;
    const int v = (int)task;
    for (int c0 = 0; c0 < H; c0 += kColsPerPass) {
        float acc[kQ];
        const bool seen = scan_token(x, Delta, v, 0, N, H, c0, lane, acc);
        if (beta && !seen) continue;  // accumulate mode leaves untouched rows alone
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int col = c0 + q * kWave + lane;
            if (col < H) {
                float* dst = dWx + (size_t)v * H + col;
                *dst = beta ? *dst + acc[q] : acc[q];
            }
        }
    }
}

// four columns of a row from c on; SHORT: all of a row of fewer than four columns
template <bool SHORT>
__device__ __forceinline__ float4 columns(const float* __restrict__ row, int c, int H) {
    if (!SHORT) return load4u(row + c);
    return make_float4(row[0], H > 1 ? row[1] : 0.f, H > 2 ? row[2] : 0.f, 0.f);
}

constexpr int kGroupThreads = 512;
constexpr int kRowsInFlight = 8;

// One range of CL ids by one slice of 4 LANES columns per workgroup: sort, group, sum.  part: compact partial rows
// [range*CL + group][H]; slot[token][range] = group + 1, or -(n + 1) for a single occurrence at
// row n, where the token occurs in the range (the table is zeroed before this kernel).  Further rows of
// workgroups finish column sums.
// With few ranges (700 ids: 3) what bounds it is the chain sort - group - sum of the longest group: so every slice of 64 columns
// sorts its range again rather than wait for another, and 16 lanes have a group, 32 groups at a time.  (One workgroup
// per range, all columns, bitonic sort: 14.9 us for 100 rows of 500, 25.4 for 800 of 500, 34.3 for 2310 of 650, 57.0 for 16384 of
// 1024; in slices 8.3, 13.5, 12.9 and 25.4.  Sixteen rows in flight: 7.8, 13.0, 12.1 and 29.7.)
// With many it is the memory it moves, a wavefront has a group, 256 columns at a time, and there are fewer slices that sort the same.
template <int CL, int LANES, bool SHORT>
__global__ __launch_bounds__(kGroupThreads) void dwx_group_kernel(const int32_t* __restrict__ x,
                                                                  const float* __restrict__ Delta,
                                                                  float* __restrict__ part,
                                                                  int32_t* __restrict__ slot,
                                                                  int N, int NV, int H, int slices, ColsumJob sum_a,
                                                                  ColsumJob sum_b) {
    if ((int)blockIdx.y >= slices) {         // column sums to be finished on the side, two groups per workgroup at a time
        __shared__ float red[kGroupThreads];
        static_assert(kGroupThreads == 512, "two groups of 256 threads");
        const int half = threadIdx.x / 256, groups = sum_a.groups + sum_b.groups, step = 2 * (gridDim.y - slices) * gridDim.x;
        for (int g0 = 2 * ((blockIdx.y - slices) * gridDim.x + blockIdx.x); g0 < groups; g0 += step) {
            const int g = g0 + half;
            const bool first = g < sum_a.groups;
            colsum_finish(first ? sum_a : sum_b, first ? g : g - sum_a.groups, threadIdx.x % 256, red + 256 * half);
            if (g0 + step < groups) __syncthreads();     // `red` is taken again
        }
        return;
    }
    __shared__ __attribute__((aligned(16))) unsigned long long key[CL];   // (id << 32) | position in the range; padding = ~0
    __shared__ int seg_start[CL + 1];
    __shared__ int s_heads[kGroupThreads / kWave];
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int base = blockIdx.x * CL;
    const int nvalid = min(CL, N - base);
    if constexpr (CL <= 256) {
        // an id's place is the number of ids before it: 32 looks per thread and two barriers.  (512 ids are 128 looks, more than the 45
        // stages of the other form take: 100000 ids of 64 columns 77 and 71 us for both launches, of 512 columns 112 and 104)
        __shared__ __attribute__((aligned(16))) int ids[CL];
        constexpr int TPK = kGroupThreads / CL, SPAN = CL / TPK;      // threads per id, ids each of them looks at
        const int i = tid / TPK, q = tid % TPK;
        if (tid < CL) ids[tid] = tid < nvalid ? x[base + tid] : 0x7fffffff;   // padding: behind every id
        __syncthreads();
        const int mine = ids[i];
        int place = 0;
        for (int j = q * SPAN; j < (q + 1) * SPAN; j += 4) {
            const int4 o = *reinterpret_cast<const int4*>(ids + j);
            place += (o.x < mine || (o.x == mine && j < i)) + (o.y < mine || (o.y == mine && j + 1 < i)) +
                     (o.z < mine || (o.z == mine && j + 2 < i)) + (o.w < mine || (o.w == mine && j + 3 < i));
        }
#pragma unroll
        for (int t = 1; t < TPK; t <<= 1) place += __shfl_xor(place, t, kWave);
        if (q == 0) key[place] = i < nvalid ? ((unsigned long long)(unsigned)mine << 32) | (unsigned)i : ~0ull;
        __syncthreads();
    } else {
        for (int i = tid; i < CL; i += kGroupThreads)
            key[i] = i < nvalid ? ((unsigned long long)(unsigned)x[base + i] << 32) | (unsigned)i : ~0ull;
        __syncthreads();
        for (int k = 2; k <= CL; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int i = tid; i < CL; i += kGroupThreads) {
                    const int partner = i ^ j;
                    if (partner > i) {
                        const unsigned long long a = key[i], b = key[partner];
                        const bool up = (i & k) == 0;
                        if ((a > b) == up) { key[i] = b; key[partner] = a; }
                    }
                }
                __syncthreads();
            }
    }
    // group heads -> group numbers (prefix sum over CL flags: lanes, then wavefronts)
    constexpr int PER = (CL + kGroupThreads - 1) / kGroupThreads;
    int heads = 0;
    for (int u = 0; u < PER; ++u) {
        const int i = tid * PER + u;
        heads += (i < nvalid && (i == 0 || (key[i] >> 32) != (key[i - 1] >> 32))) ? 1 : 0;
    }
    int upto = heads;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int v = __shfl_up(upto, off, kWave);
        if (lane >= off) upto += v;
    }
    if (lane == kWave - 1) s_heads[wave] = upto;
    __syncthreads();
    int g = upto - heads, ngroups = 0;       // groups before this thread's elements, groups of the range
#pragma unroll
    for (int w = 0; w < kGroupThreads / kWave; ++w) {
        if (w < wave) g += s_heads[w];
        ngroups += s_heads[w];
    }
    for (int u = 0; u < PER; ++u) {
        const int i = tid * PER + u;
        if (i < nvalid && (i == 0 || (key[i] >> 32) != (key[i - 1] >> 32))) seg_start[g++] = i;
    }
    if (tid == 0) seg_start[ngroups] = nvalid;
    __syncthreads();
    // LANES lanes per group: rows added in ascending position, four columns per lane (at 4-byte alignment; the lane of a
    // ragged end reads the row's last four), eight rows in flight.
    // A token that occurs once in the range needs no partial row: the table points at its
    // Delta row instead (negative entry).
    const int ranges = gridDim.x;
    const bool notes = blockIdx.y == 0 && tid % LANES == 0;      // enters the group in the table
    const int c0 = 4 * (blockIdx.y * LANES + tid % LANES), c = max(min(c0, H - 4), 0);
    for (int grp = tid / LANES; grp < ngroups; grp += kGroupThreads / LANES) {
        const int i0 = seg_start[grp], i1 = seg_start[grp + 1];
        const int v = (int)(key[i0] >> 32);
        const bool once = i1 - i0 == 1;
        if (notes) slot[(size_t)v * ranges + blockIdx.x] = once ? -(base + (int)(unsigned)key[i0] + 1) : grp + 1;
        if (once || c0 >= H) continue;
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int i = i0; i < i1; i += kRowsInFlight) {
            float4 r[kRowsInFlight];
#pragma unroll
            for (int u = 0; u < kRowsInFlight; ++u)
                r[u] = columns<SHORT>(Delta + (size_t)(base + (int)(unsigned)key[min(i + u, i1 - 1)]) * H, c, H);
#pragma unroll
            for (int u = 0; u < kRowsInFlight; ++u)
                if (i + u < i1) { acc.x += r[u].x; acc.y += r[u].y; acc.z += r[u].z; acc.w += r[u].w; }
        }
        store4u(part + ((size_t)base + grp) * H + c0, shifted(acc, c0 - c), H - c0);
    }
}

// dWx[v] = sum over the ranges (ascending) of the token's partial rows; zero row if none.
// One wavefront per (token, chunk of 256 columns), four columns per lane as in dwx_group_kernel; eight
// rows in flight, added in range order.
template <bool SHORT>
__global__ __launch_bounds__(256) void dwx_gather_kernel(const float* __restrict__ part,
                                                         const int32_t* __restrict__ slot,
                                                         const float* __restrict__ Delta,
                                                         float* __restrict__ dWx, int NV, int H,
                                                         int ranges, int CL, int beta, int col_chunks) {
    const int lane = threadIdx.x % kWave;
    const long long task = (long long)workgroup() * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (task >= (long long)NV * col_chunks) return;
    const int v = (int)(task / col_chunks), chunk = (int)(task % col_chunks);
    const int c0 = chunk * 4 * kWave + 4 * lane, c = max(min(c0, H - 4), 0);
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    bool any = false;
    for (int r0 = 0; r0 < ranges; r0 += kWave) {     // 64 table entries per look
        const int r = r0 + lane;
        const int sl = r < ranges ? slot[(size_t)v * ranges + r] : 0;
        unsigned long long mask = __ballot(sl != 0);
        any = any || mask != 0;
        while (mask) {
            const float* rows[kRowsInFlight];
            int cnt = 0;
#pragma unroll
            for (int u = 0; u < kRowsInFlight; ++u) {
                rows[u] = Delta;                       // placeholder, not added
                if (mask) {
                    const int src = __ffsll((long long)mask) - 1;
                    mask &= mask - 1;
                    const int e = __shfl(sl, src, kWave);
                    rows[u] = e > 0 ? part + ((size_t)(r0 + src) * CL + (e - 1)) * H
                                    : Delta + (size_t)(-e - 1) * H;
                    cnt = u + 1;
                }
            }
            float4 t[kRowsInFlight];
#pragma unroll
            for (int u = 0; u < kRowsInFlight; ++u) t[u] = columns<SHORT>(rows[u], c, H);
#pragma unroll
            for (int u = 0; u < kRowsInFlight; ++u)
                if (u < cnt) { acc.x += t[u].x; acc.y += t[u].y; acc.z += t[u].z; acc.w += t[u].w; }
        }
    }
    if ((beta && !any) || c0 >= H) return;         // accumulate mode leaves untouched rows alone
    float* dst = dWx + (size_t)v * H;
    if (beta) { const float4 o = columns<SHORT>(dst, c, H); acc.x += o.x; acc.y += o.y; acc.z += o.z; acc.w += o.w; }
    store4u(dst + c0, shifted(acc, c0 - c), H - c0);
}

__global__ __launch_bounds__(256) void zero_i32_kernel(int32_t* p) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0;
}

__global__ __launch_bounds__(256) void check_tokens_kernel(const int32_t* __restrict__ ids,
                                                           int64_t n, int32_t limit,
                                                           int32_t* __restrict__ bad) {
    int cnt = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = ids[i];
        cnt += (v < 0 || v >= limit) ? 1 : 0;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, kWave);
    if (threadIdx.x % kWave == 0 && cnt) atomicAdd(bad, cnt);  // integer: order-independent
}

}  // namespace

// ids per range of the grouped form: 256 while that gives at most 256 ranges, then larger
int dwx_range_len(int N) {
    int cl = 256;
    while (cl < 4096 && (N + cl - 1) / cl > 256) cl *= 2;
    return cl;
}
int dwx_ranges(int N) { const int cl = dwx_range_len(N); return (N + cl - 1) / cl; }
size_t dwx_scratch_floats(int N, int H) { return (size_t)dwx_ranges(N) * dwx_range_len(N) * H; }
size_t dwx_table_ints(int N, int NV) { return (size_t)dwx_ranges(N) * NV; }

hipError_t launch_dwx_tokens_grouped(const int32_t* x, const float* Delta, float* dWx, int N, int NV, int H, int beta,
                                     float* scratch, int32_t* slot_table, const ColsumJob& a, const ColsumJob& b, hipStream_t s) {
    const int cl = dwx_range_len(N), ranges = dwx_ranges(N);
    // A wavefront for a group, and 256 columns for a workgroup, where that leaves enough workgroups for the chip's 256 compute units and
    // three quarters of the lanes have columns.  (us of both launches, 64 columns and 256, 10000 tokens by Zipf's law: 2000 ids,
    // H = 1024: 29 and 32; 16384 ids, H = 512: 39 and 40, H = 1024: 46 and 44; 65536 ids, H = 256, 512, 1024: 82 and 78, 108 and 94, 153
    // and 124; 140000 ids, H = 256: 97 and 107; 1048576 ids, H = 100, 256, 512, 1024: 335 and 366, 643 and 469, 1200 and 751, 1904 and 1306.)
    const bool wide = H > 192 && ranges * ((H + 255) / 256) >= 192;
    const int cols = wide ? 256 : 64, slices = (H + cols - 1) / cols;
    // further rows of workgroups for the column sums, as many as a grid's second dimension is sure to hold
    const int side = min(((a.groups + b.groups + 1) / 2 + ranges - 1) / ranges, 32768);
    {
        ProfileScope ps(K_DWX_TOKENS, s);
        const dim3 grid(ranges, slices + side);
#define RNN_GROUP_OF(CL, LANES, SHORT)                                                                                         \
    hipLaunchKernelGGL((dwx_group_kernel<CL, LANES, SHORT>), grid, dim3(kGroupThreads), 0, s, x, Delta, scratch, slot_table, N, NV, H, \
                       slices, a, b)
#define RNN_GROUP(CL)                                   \
    do {                                                \
        if (wide) RNN_GROUP_OF(CL, 64, false);          \
        else if (H >= 4) RNN_GROUP_OF(CL, 16, false);   \
        else RNN_GROUP_OF(CL, 16, true);                \
    } while (0)
        switch (cl) {
            case 256: RNN_GROUP(256); break;
            case 512: RNN_GROUP(512); break;
            case 1024: RNN_GROUP(1024); break;
            case 2048: RNN_GROUP(2048); break;
            default: RNN_GROUP(4096); break;
        }
#undef RNN_GROUP
#undef RNN_GROUP_OF
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    ProfileScope ps(K_DWX_TOKENS, s);
    const int rows_per_block = 256 / kWave, col_chunks = (H + 4 * kWave - 1) / (4 * kWave);
    const long long tasks = (long long)NV * col_chunks;
    const dim3 gb = grid_of((size_t)((tasks + rows_per_block - 1) / rows_per_block));
    if (H >= 4) hipLaunchKernelGGL(dwx_gather_kernel<false>, gb, dim3(256), 0, s, scratch, slot_table, Delta, dWx,
                                   NV, H, ranges, cl, beta, col_chunks);
    else hipLaunchKernelGGL(dwx_gather_kernel<true>, gb, dim3(256), 0, s, scratch, slot_table, Delta, dWx,
                            NV, H, ranges, cl, beta, col_chunks);
    return hipGetLastError();
}

hipError_t launch_dwx_tokens(const int32_t* x, const float* Delta, float* dWx, int N, int NV, int H, int beta, hipStream_t s) {
    const int rows_per_block = 256 / kWave;
    const dim3 blocks = grid_of(((size_t)NV + rows_per_block - 1) / rows_per_block);
    ProfileScope ps(K_DWX_TOKENS, s);
    hipLaunchKernelGGL(dwx_tokens_kernel, blocks, dim3(256), 0, s, x, Delta, dWx, N, NV, H, beta);
    return hipGetLastError();
}

hipError_t launch_check_tokens(const int32_t* ids, int64_t n, int32_t limit, int32_t* bad,
                               hipStream_t s) {
    ProfileScope ps(K_CHECK_TOKENS, s);
    hipLaunchKernelGGL(zero_i32_kernel, dim3(1), dim3(64), 0, s, bad);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int blocks = (int)((n + 255) / 256);
    if (blocks > 1024) blocks = 1024;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(check_tokens_kernel, dim3(blocks), dim3(256), 0, s, ids, n, limit, bad);
    return hipGetLastError();
}

}  // namespace rnn
