// Second stage of a column sum, for a launch of its own and for workgroups that ride on another kernel's.
#pragma once
#include "common.hpp"
#include "internal.hpp"

namespace rnn {

// Group `group` of a job: out[col] = (beta ? out[col] : 0) + sum over chunks of part[chunk][col] for 2^txs columns, the chunks spread
// over the row lanes.  t: thread 0 .. 255 of the group, red: 256 floats.  All threads of the workgroup call it.
__device__ __forceinline__ void colsum_finish(const ColsumJob& j, int group, int t, float* red) {
    constexpr int U = 8;
    const int tx = 1 << j.txs, ty = 256 >> j.txs, cx = t & (tx - 1), ry = t >> j.txs;
    const int col = group * tx + cx;
    const bool on = group < j.groups && col < j.C;
    float cs = 0.f;
    if (on) {
        for (int k0 = ry; k0 < j.chunks; k0 += ty * U) {
            float m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) m[u] = j.part[(size_t)min(k0 + u * ty, j.chunks - 1) * j.C + col];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + u * ty < j.chunks) cs += m[u];
        }
    }
    red[t] = cs;
    __syncthreads();
    if (ry == 0 && on) {
        float s = 0.f;
        for (int r = 0; r < ty; ++r) s += red[r * tx + cx];
        j.out[col] = j.beta ? j.out[col] + s : s;
    }
}

}  // namespace rnn
