// Persistent batched time loop for hidden sizes whose matrix needs many compute units (256 < hidden <= 1024, batch up to 64), or
// that take longer on one (193 to 256 units, batch up to 128, sequences that are not short): ONE launch for all steps instead of one launch per step.
//
// The paper's Scan keeps the loop inside one graph node so that nothing per step happens outside
// compiled code (properties 4 and 5) and keeps every state (property 1); the per-step kernel
// boundary of recurrence_step.hip costs more than the step's arithmetic.  Here the chip's layout
// does the work instead: batch rows are independent, so the batch is cut into up to 32 groups of up to 4
// rows, groups x, x + 8, x + 16 and x + 24 on XCD x, and the 32 compute units of an XCD share its one group's recurrence, or
// have 16, 10 or 8 for each of its two, three or four groups' (batch above 32, 64 and 96).  Every workgroup holds 16, 32 or 64 output columns of the matrix (all K) in
// registers for the whole launch, as few as cover H, and produces, per step, its tile of the new state on the
// matrix cores; the eight wavefronts split K and meet in LDS.  Groups never talk to each other.
//
// Matrix instruction: v_mfma_f32_4x4x1, 16 blocks of 4 rows by 4 columns.  With 64 columns per workgroup the state is broadcast
// over all 16 blocks (cbsz = 4): lane l supplies the matrix value M[k][c0 + l] of one k per instruction and the state
// value of row l % 4 for the 16 k of its block l / 4, and receives rows 0..3 at column c0 + l.  With 32 or 16 columns the
// lanes are two or four parts that each have all columns and a part of the k (cbsz = 3 or 2: the state is broadcast
// within a part), so a step takes half or a quarter of the instructions, and a lane a half or a quarter of the registers.
// The parts are added up after the wavefronts' tiles have met.  The
// 16-byte piece of the state a lane fetches from memory (row l % 4, four consecutive k) is exactly
// what it feeds the instruction, so the state goes from the cache into the operand registers
// without passing LDS.  A wavefront's share of K is an eighth of H in whole blocks of 16 (32 to 128),
// and the instructions of blocks past it are left out.
//
// Inside a group the new state travels through the L2 cache its compute units share, with no flags,
// no fences and no kernel boundaries, in a ring of four states kept beside the history:
//   * every word of a free slot holds a bit pattern arithmetic never produces (an all-ones NaN; a value
//     that came in as one is published as another NaN); every wavefront fetches the K slice its own
//     product needs and repeats until no such word is left.  Every 4-byte value validates itself, so
//     no ordering between the stores of a step is needed;
//   * a state is laid out as [k / 4][row][k % 4], the order of a wavefront's lanes: its fetch is one
//     contiguous stretch.  (From rows as the history holds them, each quad of lanes would touch four
//     cache lines: the exchange alone took 2050 clocks that way, 1350 this way);
//   * the stores are workgroup-scope: they stop at the XCD's L2, where the group's readers look.  Device
//     scope sends them on to memory first: 2600 to 3900 clocks for the exchange, by how early the
//     readers look.  The looks are device-scope loads, which pass the first-level cache;
//   * who publishes state s + 1 turns its share of state s - 1 back into a free slot (everybody has read
//     that: state s is complete) and waits for that store with its next look at the ring, that is before
//     it publishes state s + 2.  The slot is published again as state s + 3, which nobody looks for
//     without having seen all of state s + 2: no look can find the words of the state before.
// The operands of the epilogues come from memory, and their requests cost more than they take: a compute unit's requests return in
// the order they were made, so a look at the ring waits for an operand of a later step that was requested before it, and a
// wavefront's look also for its own stores.  So operands are requested eight steps at a time, and one look in eight waits; and up to 32
// columns a ninth wavefront, the carrier, does it and stores the new states' rows, through LDS, so that the wavefronts of the
// product make no request but to the ring.  (us a step, forward and reverse; 256 units, batch 128, 2047 steps, whose arrays are
// beyond the last-level cache: requests a step ahead by the epilogue's lanes 0.95 and 1.03, by the carrier four steps ahead but every step
// 0.96 and 1.09 - 0.78 and 0.88 when they are made to hit the cache -, two at a time 0.88 and 0.94, four 0.79 and 0.86, eight 0.76 and
// 0.80; 500 units, batch 1: 0.91 and 0.91 -> 0.84 and 0.83; 513 units, batch 19: 1.20 and 1.16 -> 1.11 and 1.10.)
// Token input takes its rows of Wx in the loop, as the other operands, instead of a gather launch that writes them
// out for all steps and is read back (256 steps of 64 rows at H = 1024: 27 us).
// A hidden size that is no multiple of 4 has the rest of a row's last piece published as zeros.
// A workgroup takes its group from the XCD it finds itself on and its column slice from a per-XCD
// counter, so all workgroups of a group share one L2 by construction whenever the 256 workgroups are
// co-resident (checked before the launch).  That is all the exchange asks for: its looks pass the first-level cache, so it does not
// matter to it whether two workgroups of a group share a compute unit, which the LDS they take rules out.  (Two on each would have half
// the columns, and twice as many parts of K to add up: other sums in the last bits.)  The launch is not cooperative but takes turns with
// others of its kind (gang.hip).  Where other work keeps a part of a group off the chip for longer than the loop would
// take on one workgroup, one of those that did come runs it by itself and the others leave, so the launch ends with the same
// results, bit for bit, whatever else the GPU does (run_alone below).
// Every wait is bounded, the one for the group by time, and an expired wait for a state sets the status word: the wavefront that gave
// up sets s_abort, and the workgroup's others leave at their next look at it, the carrier up to 16 steps later.  Each passes at
// most one barrier per step and then ends, and a barrier does not wait for wavefronts that have ended.
//
// Measured (a forward loop of 256 steps, batch 64, H = 1024): 600 us with the state read from the history and
// device-scope stores, 455 now (1000 words; 512 right behind the large products of 10000 words, which
// leave the chip at a lower clock); 100 steps at H = 513, batch 33: 207 -> 148, at H = 512, batch 64:
// 158 -> 101.  A step at H = 1024, batch 64 takes about 3700 clocks: 2050 for the matrix instructions of the
// two wavefronts of a SIMD at the rate of float32, 550 from the last of them to the store, the rest for the
// store and the look.  With fewer columns the instructions are less of it (100 steps, us of a forward loop with 64, 32, 16
// columns before the carrier, and now with the fewest): H = 500, batch 1: 134, 113, 110, 91; H = 513, batch 19: 165, 136, 117; H = 1024,
// batch 32: 200, 154, 146; H = 400, batch 40: 137, 117, 99; H = 300, batch 20: 122, 110, 109, 88.
#include "common.hpp"
#include "internal.hpp"
#include "prof.hpp"

#include <math.h>

#include <mutex>
#include <type_traits>
#include <utility>

namespace rnn {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NW = 8;              // wavefronts of the product
constexpr int CHUNK = 8;           // steps whose operands the carrier requests at a time
constexpr int OWN_CHUNK = 4;       // the same of the epilogue's lanes where there is no carrier
// up to 32 columns a ninth wavefront fetches the operands and stores the rows; with 64 the registers do not suffice
__host__ __device__ constexpr bool has_carrier(int cwd) { return cwd <= 32; }
__host__ __device__ constexpr int threads_of(int cwd) { return 64 * (NW + (has_carrier(cwd) ? 1 : 0)); }
constexpr int RB = 4;              // batch rows per group
constexpr int NXCD = 8;            // XCDs: the layout this loop is built on
constexpr int WG_PER_XCD = 32;     // compute units per XCD = workgroups per XCD
constexpr int NGRP = 32;           // groups at most: x, x + 8, x + 16 and x + 24 on XCD x
constexpr int H_MAX = 1024;
static_assert(REC_XCD_COUNTERS == NXCD + NGRP, "a slice counter per XCD, a roll per group");
constexpr int RSLOTS = 4;          // states the exchange ring holds
constexpr unsigned kSentinel = 0xFFFFFFFFu;
constexpr int ROLL_CLOSED = 1 << 16;
// what a workgroup does in its group: not known yet, its own columns, nothing, everything
constexpr int PART_OPEN = 0, PART_ONE = 1, PART_NONE = 2, PART_ALL = 3;

#ifdef RNN_REC_TRACE
__device__ long long g_xcd_trace[4 * 8];
#define XT_DECL long long xt_prev = clock64(); long long xt_acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}
#define XTM(k) do { const long long xt_n = clock64(); xt_acc[k] += xt_n - xt_prev; xt_prev = xt_n; } while (0)
#define XT_COUNT(k, n) do { xt_acc[k] += (n); } while (0)
#define XT_FLUSH(bwd) do { if (grp == 0 && slot == 0 && (tid == 0 || tid == 256)) \
        for (int k_ = 0; k_ < 8; ++k_) g_xcd_trace[((bwd ? 2 : 0) + (tid == 0 ? 0 : 1)) * 8 + k_] = xt_acc[k_]; } while (0)
#else
#define XT_DECL
#define XTM(k)
#define XT_COUNT(k, n)
#define XT_FLUSH(bwd)
#endif

// leaves the first-level cache and stays in the XCD's L2, where every reader of the word looks for it (a
// device-scope store would go on to memory first: see above)
__device__ __forceinline__ void ring_store(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ bool fresh(float4 v) {
    return __float_as_uint(v.x) != kSentinel && __float_as_uint(v.y) != kSentinel &&
           __float_as_uint(v.z) != kSentinel && __float_as_uint(v.w) != kSentinel;
}

// the four values of one state piece against the matrix: every 64 / S lanes have the state of block AB of their own 16 / S
// (abid), k = 4 AB + e of their share of the piece; w: from the weights of block FIRST on
template <int S, int FIRST, int... AB>
__device__ __forceinline__ void mfma_blocks(const float4 st, const float* __restrict__ w, f32x4 (&acc)[4],
                                            std::integer_sequence<int, AB...>) {
    constexpr int CB = S == 1 ? 4 : S == 2 ? 3 : 2;
    ((acc[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(st.x, w[4 * AB + 0], acc[0], CB, FIRST + AB, 0),
      acc[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(st.y, w[4 * AB + 1], acc[1], CB, FIRST + AB, 0),
      acc[2] = __builtin_amdgcn_mfma_f32_4x4x1f32(st.z, w[4 * AB + 2], acc[2], CB, FIRST + AB, 0),
      acc[3] = __builtin_amdgcn_mfma_f32_4x4x1f32(st.w, w[4 * AB + 3], acc[3], CB, FIRST + AB, 0)),
     ...);
}

// words of one state in the exchange ring: 8 KW columns of the batch's groups of RB rows, as [k / 4][row][k % 4]
// inside a group, the order in which a wavefront's lanes want them
__host__ __device__ inline int ring_state(int B, int kw) { return (B + RB - 1) / RB * RB * 8 * kw; }

// Partial tile of a wavefront's K slice: element i = row i at column c0 + lane % CWD, of the lane's part of K.
// w[64 / S * q + j] = M[k][c0 + lane % CWD], k = kb + 64 q + nq / S * (lane / CWD) + j with nq the k of piece q.
template <int KW, int S>
__device__ __forceinline__ f32x4 slice_product(const float4 (&st)[(KW + 63) / 64], const float (&w)[KW / S]) {
    constexpr int N0 = KW < 64 ? KW : 64, N1 = KW - N0;
    f32x4 acc[4] = {};
    mfma_blocks<S, 0>(st[0], w, acc, std::make_integer_sequence<int, N0 / S / 4>{});
    if constexpr (N1 > 0) mfma_blocks<S, 0>(st[1], w + 64 / S, acc, std::make_integer_sequence<int, N1 / S / 4>{});
    return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}
// The wavefronts' partial sums of an element (pp: the first one's, of this lane's part of K), then those of the S parts.  All
// lanes of the wavefront call it.
template <int S>
__device__ __forceinline__ float tile_sum(const float* pp) {
    float v[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) v[w] = pp[w * RB * 64];
    float sum = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    if constexpr (S == 4) sum = swap16_sum(sum);
    if constexpr (S >= 2) sum = swap32_sum(sum);
    return sum;
}

// slice_product's part of one piece of NBLK blocks, from block FIRST on, with the weights M[k0 + ..][col] fetched here, four blocks
// at a time (more would not fit the registers beside what the kernel holds)
template <bool BWD, int S, int NBLK, int FIRST = 0>
__device__ __forceinline__ void fetched_product(const float* __restrict__ Wh, int H, int k0, int col, const float4 st, f32x4 (&acc)[4]) {
    if constexpr (FIRST < NBLK) {
        constexpr int M = NBLK - FIRST < 4 ? NBLK - FIRST : 4;
        float w[4 * M];
        asm volatile("" : "+s"(H));      // the offsets are formed here each time, not kept for all blocks
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const int k = k0 + 4 * (FIRST + m), left = col < H ? H - k : 0;
            if (BWD) {
#pragma unroll
                for (int e = 0; e < 4; ++e) w[4 * m + e] = e < left ? Wh[(k + e) * H + col] : 0.f;
            } else {
                const float4 p = piece(Wh + col * H + k, left);
                w[4 * m] = p.x; w[4 * m + 1] = p.y; w[4 * m + 2] = p.z; w[4 * m + 3] = p.w;
            }
        }
        mfma_blocks<S, FIRST>(st, w, acc, std::make_integer_sequence<int, M>{});
        __builtin_amdgcn_sched_barrier(0);
        fetched_product<BWD, S, NBLK, FIRST + M>(Wh, H, k0, col, st, acc);
    }
}

// floats of LDS that run_alone takes: two sets of partial tiles and two states
template <int KW>
constexpr int alone_floats() { return 2 * NW * RB * 64 + 2 * RB * (8 * KW + 4); }

// The whole recurrence of one group on one workgroup's wavefronts of the product, for a group of which not all workgroups came.  The
// columns of each workgroup in turn, the matrix read from the caches every step: the same products in the same order, so the results
// are those of the group, bit for bit.
template <int ACT, bool BWD, int KW, int CWD>
__device__ __forceinline__ void run_alone(const RecXcdArgs& a, int b0, int nrows, float* sm) {
    constexpr int NQ = (KW + 63) / 64, S = 64 / CWD, N0 = KW < 64 ? KW : 64, N1 = KW - N0;
    constexpr int XT = NW * kWave, PITCH = 8 * KW + 4;
    const int H = a.H, T = a.T, tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int kb = KW * wave, part_k = lane / CWD, part_c = lane % CWD, ri = lane % 4, block = (lane / 4) % (16 / S);
    const int ej = lane % (64 / S), ep = lane / (64 / S), em = (ej >> 2) & 3, et = CWD / 4 * (wave & 3) + 4 * (ej >> 4) + (ej & 3);
    const size_t bh = (size_t)a.B * H;
    float *part = sm, *cur = sm + 2 * NW * RB * 64, *nxt = cur + RB * PITCH;
    __syncthreads();
    for (int e = tid; e < RB * PITCH; e += XT) {
        const int r = e / PITCH, c = e - r * PITCH;
        float v = 0.f;
        if (r < nrows && c < H) {
            const size_t off = (size_t)(b0 + r) * H + c;
            if (!BWD) {
                v = a.h0 ? a.h0[off] : 0.f;
                a.hist[off] = v;
            } else {
                const size_t i = (size_t)(T - 1) * bh + off;
                v = (a.G[i] + (a.dh_last ? a.dh_last[off] : 0.f)) * act_grad<ACT>(a.h_all[(size_t)T * bh + off]);
                a.Delta[i] = v;
            }
        }
        cur[e] = v;
        nxt[e] = 0.f;
    }
    __syncthreads();
    const int nsteps = BWD ? T - 1 : T;
#pragma unroll 1
    for (int s = 0; s < nsteps + (BWD && a.dh0 ? 1 : 0); ++s) {
        float4 st[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int nq = q ? N1 : N0, k = kb + 64 * q + nq / S * part_k + 4 * block;
            st[q] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (4 * block < nq / S) st[q] = *reinterpret_cast<const float4*>(cur + ri * PITCH + k);
        }
#pragma unroll 1
        for (int c0 = 0, par = 0; c0 < H; c0 += CWD, par ^= 1) {
            const int col = c0 + part_c, ec = c0 + et;
            f32x4 acc[4] = {};
            fetched_product<BWD, S, N0 / S / 4>(a.Wh, H, kb + N0 / S * part_k, col, st[0], acc);
            if constexpr (N1 > 0) fetched_product<BWD, S, N1 / S / 4>(a.Wh, H, kb + 64 + N1 / S * part_k, col, st[1], acc);
            float* tiles = part + par * NW * RB * 64;
            *reinterpret_cast<f32x4*>(tiles + wave * RB * 64 + RB * lane) = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            __syncthreads();                             // (the set written next was read in front of this)
            if (wave >= 4) continue;
            const float sum = tile_sum<S>(tiles + RB * (CWD * ep + et) + em);
            if (ep != 0 || em >= nrows || ec >= H) continue;
            const size_t off = (size_t)(b0 + em) * H + ec;
            if (s == nsteps) {                           // reverse: the gradient of the initial state
                a.dh0[off] = sum;
                continue;
            }
            float v;
            if (BWD) {
                const size_t i = (size_t)(T - 2 - s) * bh + off;
                v = (sum + a.G[i]) * act_grad<ACT>(a.h_all[i + bh]);
            } else {
                const size_t n = (size_t)s * a.B + b0 + em;
                v = activate<ACT>(sum + (a.x ? a.Wx[(size_t)a.x[n] * H + ec] + a.b[ec] : a.U[n * H + ec]));
            }
            if (__float_as_uint(v) == kSentinel) v = __uint_as_float(0x7FC00000u);   // as the group publishes it
            if (BWD) {
                a.Delta[(size_t)(T - 2 - s) * bh + off] = v;
            } else {
                a.hist[(size_t)(s + 1) * bh + off] = v;
                if (a.h_last && s == nsteps - 1) a.h_last[off] = v;
            }
            nxt[em * PITCH + ec] = v;
        }
        __syncthreads();
        float* t = cur; cur = nxt; nxt = t;
    }
}

// KW = k per wavefront (8 KW >= H), CWD = output columns per workgroup
template <int ACT, bool BWD, int KW, int CWD>
__global__ __launch_bounds__(threads_of(CWD)) void rec_xcd_kernel(RecXcdArgs a) {
    constexpr bool CARRY = has_carrier(CWD);
    constexpr int NQ = (KW + 63) / 64;     // 16-byte state pieces per lane and step
    constexpr int S = 64 / CWD;            // k per instruction, in as many parts of a wavefront's lanes
    constexpr int N0 = KW < 64 ? KW : 64, N1 = KW - N0;   // k of the two pieces
    extern __shared__ __attribute__((aligned(16))) float smem[];
    __shared__ int s_abort, s_grp, s_slot, s_part;
    __shared__ int s_stored;                   // steps whose first row this workgroup has stored
    // what the carrier hands to the epilogues and takes from them, by step parity: input term or G, slope, new state
    __shared__ float s_in[2][CARRY ? RB * CWD : 1], s_slope[2][CARRY && BWD ? RB * CWD : 1], s_out[2][CARRY ? RB * CWD : 1];
    float* part = smem;                    // [2][NW][S][CWD][RB] partial tiles, by step parity

    const int H = a.H, B = a.B, T = a.T;
    const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int ri = lane % 4;
    const size_t bh = (size_t)B * H;

    // ---- which group and which column slice: by the XCD this workgroup runs on ------------------
    if (tid == 0) {
        unsigned id;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(id));
        const int xcc = (int)(id & 0xf);
        const int n = xcc < NXCD ? atomicAdd(a.counters + xcc, 1) : WG_PER_XCD;
        s_grp = n < WG_PER_XCD ? xcc + NXCD * (n / a.slots) : NGRP;
        s_slot = n % a.slots;
        s_abort = 0;
        s_stored = 0;
    }
    __syncthreads();
    const int grp = s_grp, slot = s_slot;
    const int b0 = grp * RB, c0 = slot * CWD;
    if (grp >= NGRP) {                           // not the layout this kernel is built on
        if (tid == 0) atomicExch(a.status, 1);
        return;
    }
    if (b0 >= B || c0 >= H) return;              // nothing to do here, and nobody waits for this workgroup
    const int nrows = min(RB, B - b0);

    // ---- the group's roll: how many of its workgroups have come; ROLL_CLOSED once one of them has stopped waiting for the rest.
    //      It is complete or closed for good: nobody closes a complete one, and who comes to a closed one leaves -------------
    const int whole = (H + CWD - 1) / CWD + a.absent;
    int* roll = a.counters + NXCD + grp;
    long long came = 0;
    auto settle = [&]() {                        // thread 0: what this workgroup does
        for (;;) {
            int w = __hip_atomic_load(roll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (w == whole) return PART_ONE;
            if (w & ROLL_CLOSED) return PART_NONE;
            if (wall_clock64() - came > a.patience) {
                if (__hip_atomic_compare_exchange_strong(roll, &w, w | ROLL_CLOSED, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT))
                    return PART_ALL;
                continue;                        // somebody came, or closed it, at this moment
            }
            __builtin_amdgcn_s_sleep(8);
        }
    };
    if (tid == 0) {
        came = wall_clock64();
        const int before = atomicAdd(roll, 1);
        s_part = before & ROLL_CLOSED ? PART_NONE : PART_OPEN;
    }

    // ---- resident weights, laid out as slice_product takes them: M = Wh^T (forward) or Wh (reverse); zero outside the matrix ----
    const int nsteps = BWD ? T - 1 : T;

    // ---- the carrier (wavefront NW) ---------------------------------------------------------------
    // In the interval before barrier s it puts the operands of step s in place, whose epilogue follows that barrier, and stores the
    // state of step s - 2, whose epilogue was before the barrier before.
    if constexpr (CARRY) if (wave == NW) {
        constexpr int NL = RB * CWD / kWave;
        size_t off[NL];
        int place[NL], cc[NL], cb[NL];
        bool on[NL];
        float bias[NL], x0[2 * CHUNK][NL], x1[2 * CHUNK][NL];
        int id[CHUNK][NL];
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int e = lane + kWave * i, row = e / CWD, col = e % CWD;
            cb[i] = min(b0 + row, B - 1);
            cc[i] = min(c0 + col, H - 1);
            off[i] = (size_t)cb[i] * H + cc[i];
            place[i] = 16 * (col / 4) + 4 * row + col % 4;
            on[i] = row < nrows && c0 + col < H;
            bias[i] = !BWD && a.x ? a.b[cc[i]] : 0.f;
        }
        auto carry = [&](auto tokens_c) __attribute__((always_inline)) {
            constexpr bool TOK = decltype(tokens_c)::value;
            // (requests past the last step repeat it)
            auto want_id = [&](int s, int (&v)[NL]) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < NL; ++i)
                    if (TOK) v[i] = a.x[(size_t)min(s, nsteps - 1) * B + cb[i]];
            };
            auto want = [&](int s, const int (&v)[NL], float (&p)[NL], float (&q)[NL]) __attribute__((always_inline)) {
                const int sc = min(s, nsteps - 1);
                const size_t base = (size_t)(BWD ? T - 2 - sc : sc) * bh;
#pragma unroll
                for (int i = 0; i < NL; ++i) {
                    p[i] = TOK ? a.Wx[(size_t)v[i] * H + cc[i]] : BWD ? a.G[base + off[i]] : a.U[base + off[i]];
                    if (BWD) q[i] = a.h_all[base + bh + off[i]];
                }
            };
            auto keep = [&](int s) __attribute__((always_inline)) {
                float* dst = BWD ? a.Delta + (ptrdiff_t)(T - 2 - s) * (ptrdiff_t)bh : a.hist + (ptrdiff_t)(s + 1) * (ptrdiff_t)bh;
#pragma unroll
                for (int i = 0; i < NL; ++i) {
                    const float v = s_out[s & 1][place[i]];
                    if (on[i] && s >= 0) dst[off[i]] = v;
                }
            };
            // one interval; the step's parity and its slot of the operands are those of u
            auto interval = [&](int u, int s) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < NL; ++i) {
                    s_in[u & 1][place[i]] = TOK ? x0[u][i] + bias[i] : x0[u][i];
                    if (BWD) s_slope[u & 1][place[i]] = act_grad<ACT>(x1[u][i]);
                }
                if (u % CHUNK == 0) {        // the next chunk, and the tokens of the one after it
                    const int v = CHUNK - u;
#pragma unroll
                    for (int c = 0; c < CHUNK; ++c) want(s + CHUNK + c, id[c], x0[v + c], x1[v + c]);
#pragma unroll
                    for (int c = 0; c < CHUNK; ++c) want_id(s + 2 * CHUNK + c, id[c]);
                }
                keep(s - 2);
                lds_barrier();
            };
            if (nsteps > 0) {
#pragma unroll
                for (int c = 0; c < CHUNK; ++c) want_id(c, id[c]);
#pragma unroll
                for (int c = 0; c < CHUNK; ++c) want(c, id[c], x0[c], x1[c]);
#pragma unroll
                for (int c = 0; c < CHUNK; ++c) want_id(CHUNK + c, id[c]);
            }
            __syncthreads();                                         // (the matrix is in registers, and the group's roll is settled)
            if (s_part != PART_ONE) return;
            // (no branch inside the loop: the compiler then counts the requests in flight and waits for the oldest only)
            int s0 = 0;
            for (; s0 + 2 * CHUNK <= nsteps && !s_abort; s0 += 2 * CHUNK) {
#pragma unroll
                for (int u = 0; u < 2 * CHUNK; ++u) interval(u, s0 + u);
            }
#pragma unroll
            for (int u = 0; u < 2 * CHUNK - 1; ++u)
                if (s0 + u < nsteps && !s_abort) interval(u, s0 + u);
            keep(nsteps - 2);
            __syncthreads();
            if (s_abort) return;
            keep(nsteps - 1);
            if (BWD && a.dh0) __syncthreads();
        };
        if (!BWD && a.x) carry(std::true_type{});
        else carry(std::false_type{});
        return;
    }

    const int kb = KW * wave;
    const int part_k = lane / CWD, part_c = lane % CWD;   // this lane's part of every piece's k, and its column
    float wreg[KW / S];
    if (BWD) {
        // M[k][col] = Wh[k][col]: a lane's values lie along a column of Wh.  Fetched as 16-byte pieces
        // along the rows into a wavefront-private LDS tile [64 k][CWD columns], 64 k at a time, from which
        // every lane takes its column.
        float* stg = smem + wave * 64 * 65;
        constexpr int RP = 256 / CWD;             // rows per request
        const int r4 = lane / (CWD / 4), c4 = 4 * (lane % (CWD / 4));
        auto stage = [&](auto piece_c) __attribute__((always_inline)) {
            constexpr int q = decltype(piece_c)::value, nq = q ? N1 : N0, NV = 64 / RP;
            float4 v[NV];
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int k = kb + 64 * q + r4 + RP * i, cc = c0 + c4;
                v[i] = piece(a.Wh + (size_t)k * H + cc, k < H ? H - cc : 0);
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) *reinterpret_cast<float4*>(stg + (r4 + RP * i) * CWD + c4) = v[i];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the tile is this wavefront's own
#pragma unroll
            for (int j = 0; j < nq / S; ++j) wreg[64 / S * q + j] = stg[(nq / S * part_k + j) * CWD + part_c];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        };
        stage(std::integral_constant<int, 0>{});
        if constexpr (NQ > 1) stage(std::integral_constant<int, 1>{});
    } else {
        // M[k][col] = Wh[col][k]: a lane's values lie along a row of Wh.  Fetched as 16-byte pieces
        // along the rows (a request covers four rows of 256 bytes) and turned through a
        // wavefront-private LDS tile [CWD columns][64 k], 64 k at a time.
        constexpr int PITCH = 65;                 // odd: the transposed reads fall into distinct banks
        float* stg = smem + wave * 64 * PITCH;
        const int r4 = lane >> 4, k4 = 4 * (lane & 15);
        auto stage = [&](auto piece_c) __attribute__((always_inline)) {
            constexpr int q = decltype(piece_c)::value, nq = q ? N1 : N0, NV = CWD / 4;
            float4 v[NV];
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int row = c0 + r4 + 4 * i, k = kb + 64 * q + k4;
                v[i] = piece(a.Wh + (size_t)row * H + k, row < H ? H - k : 0);
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                float* d = stg + (r4 + 4 * i) * PITCH + k4;
                d[0] = v[i].x; d[1] = v[i].y; d[2] = v[i].z; d[3] = v[i].w;
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the tile is this wavefront's own
#pragma unroll
            for (int j = 0; j < nq / S; ++j) wreg[64 / S * q + j] = stg[part_c * PITCH + nq / S * part_k + j];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        };
        stage(std::integral_constant<int, 0>{});
        if constexpr (NQ > 1) stage(std::integral_constant<int, 1>{});
    }

    // by now the others have come, or something else holds their compute units
    if (tid == 0 && s_part == PART_OPEN) s_part = settle();
    __syncthreads();
    const int mine = s_part;
    if (mine != PART_ONE) {
        if (mine == PART_ALL) run_alone<ACT, BWD, KW, CWD>(a, b0, nrows, smem);
        return;
    }

    // ---- the state pieces of this lane: row ri, four columns from p_k on; pieces outside the matrix (rows past
    //      the batch, columns past H) or another wavefront's stay zero.  The 16 / S blocks of a part of the lanes hold the part's
    //      k in order; a piece of fewer than 64 k leaves the last blocks of every part unused ------------
    const int block = (lane / 4) % (16 / S);
    int p_k[NQ], p_off[NQ], p_shift[NQ];
    bool p_on[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int nq = q ? N1 : N0, k = kb + 64 * q + nq / S * part_k + 4 * block;
        p_k[q] = k;
        p_on[q] = ri < nrows && k < H && 4 * block < nq / S;
        p_off[q] = p_on[q] ? (b0 + ri) * H + min(k, H - 4) : b0 * H;   // clamped duplicates outside the matrix
        p_shift[q] = p_on[q] ? max(k - (H - 4), 0) : 0;
    }
    // the same pieces in the exchange ring: one contiguous stretch per wavefront and q (per part of it, where nq < 64)
    const int rstate = ring_state(B, KW);
    int r_off[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) r_off[q] = p_on[q] ? b0 * 8 * KW + p_k[q] * RB + 4 * ri : b0 * 8 * KW + kb * RB;
    float4 st[NQ];                         // the state of the coming step
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p_on[q]) {
            if (!BWD) {
                if (a.h0) v = piece(a.h0 + p_off[q], 4);
            } else {
                const float4 g = piece(a.G + (size_t)(T - 1) * bh + p_off[q], 4);
                const float4 h = piece(a.h_all + (size_t)T * bh + p_off[q], 4);
                float4 c = make_float4(0.f, 0.f, 0.f, 0.f);
                if (a.dh_last) c = piece(a.dh_last + p_off[q], 4);
                v.x = (g.x + c.x) * act_grad<ACT>(h.x); v.y = (g.y + c.y) * act_grad<ACT>(h.y);
                v.z = (g.z + c.z) * act_grad<ACT>(h.z); v.w = (g.w + c.w) * act_grad<ACT>(h.w);
            }
            v = shifted(v, p_shift[q]);
        }
        st[q] = v;
    }

    // ---- epilogue lanes (wavefronts 0..3): CWD / 4 columns of the tile per wavefront, in the ring's order, so
    //      that a wavefront's share of the new state leaves as one stretch of 4 CWD bytes.  The S parts of an element
    //      are summed by lanes 64 / S apart; the first of them stores the element ------------------------
    const int ej = lane % (64 / S), ep = lane / (64 / S);
    const int em = (ej >> 2) & 3, et = CWD / 4 * (wave & 3) + 4 * (ej >> 4) + (ej & 3), ec = c0 + et;
    const bool e_on = wave < 4 && ep == 0 && em < nrows && ec < H;
    // the columns that fill the ragged last piece of a row are published as zeros
    const bool e_pub = wave < 4 && ep == 0 && em < nrows && ec < (H + 3) / 4 * 4;
    const size_t e_off = (size_t)min(b0 + em, B - 1) * H + min(ec, H - 1);
    const int e_ring = b0 * 8 * KW + c0 * RB + 64 / S * (wave & 3) + ej;
    if (e_on) {    // slot 0 of the history (forward) / Delta[T-1] (reverse): the owner of a column stores it
        if (!BWD) {
            a.hist[e_off] = a.h0 ? a.h0[e_off] : 0.f;
        } else {
            const size_t e = (size_t)(T - 1) * bh + e_off;
            const float c = a.dh_last ? a.dh_last[e_off] : 0.f;
            a.Delta[e] = (a.G[e] + c) * act_grad<ACT>(a.h_all[(size_t)T * bh + e_off]);
        }
    }
    const int e_at = 64 / S * (wave & 3) + ej;     // this lane's element in the tiles of the carrier
    // Without a carrier: the operands of OWN_CHUNK steps are requested together, a chunk ahead (clamped: always valid), and kept in
    // places of LDS of the lane's own.  Token input takes the rows of Wx itself; their numbers are requested another chunk ahead.
    float* own = smem + 2 * NW * RB * 64 + tid;        // [OWN_CHUNK][2][256]
    const float bias = !CARRY && !BWD && a.x && wave < 4 ? a.b[min(ec, H - 1)] : 0.f;
    const int eb = min(b0 + em, B - 1);
    int id[OWN_CHUNK];
    float n0[OWN_CHUNK], n1[OWN_CHUNK];
    auto step_of = [&](int s) { return max(min(s, nsteps - 1), 0); };
    auto load_ids = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < OWN_CHUNK; ++c) id[c] = !BWD && a.x ? a.x[(size_t)step_of(s + c) * B + eb] : 0;
    };
    auto load_chunk = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < OWN_CHUNK; ++c) {
            const int sc = step_of(s + c);
            const size_t base = (size_t)(BWD ? max(T - 2 - sc, 0) : sc) * bh;
            n1[c] = 0.f;
            if (BWD) {
                n0[c] = a.G[base + e_off];
                n1[c] = a.h_all[base + bh + e_off];
            } else {
                n0[c] = a.x ? a.Wx[(size_t)id[c] * H + min(ec, H - 1)] : a.U[base + e_off];
            }
        }
    };
    if (!CARRY && wave < 4) {
        load_ids(0);
        load_chunk(0);
        load_ids(OWN_CHUNK);
    }

    XT_DECL;
    auto product = [&]() __attribute__((always_inline)) { return slice_product<KW, S>(st, wreg); };
    auto park_partial = [&](int par, const f32x4 p4) __attribute__((always_inline)) {
        *reinterpret_cast<f32x4*>(part + (par * 8 + wave) * RB * 64 + RB * lane) = p4;
    };
    auto element_sum = [&](int par) __attribute__((always_inline)) {   // epilogue lanes
        return tile_sum<S>(part + par * NW * RB * 64 + RB * (CWD * ep + et) + em);
    };
    // The lane's pieces of the state at `src` in the ring, waiting until no "not written yet" word is left.
    auto collect = [&](const float* src) __attribute__((always_inline)) {
        float4 v[NQ];
        unsigned need = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) need |= p_on[q] ? 1u << q : 0u;
        const unsigned wanted = need;
        for (int spins = 0; need != 0; ++spins) {
            XT_COUNT(6, 1);
            if (spins > a.spin_limit) { s_abort = 1; break; }
            if (spins > 0) __builtin_amdgcn_s_sleep(2);
            if constexpr (NQ == 2)
                asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %3, off sc1\n\ts_waitcnt vmcnt(0)"
                             : "=&v"(v[0]), "=&v"(v[1]) : "v"(src + r_off[0]), "v"(src + r_off[1]) : "memory");
            else
                asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(v[0]) : "v"(src + r_off[0]) : "memory");
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (fresh(v[q])) need &= ~(1u << q);
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            st[q] = (wanted & (1u << q)) ? v[q] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };

    float last_v = 0.f;
    // One workgroup barrier per step (the partial tiles are complete); the partial buffers alternate by
    // step parity, and no wavefront can be more than one step ahead of the epilogue of its own
    // workgroup, because every later tile of the group needs that epilogue's output.
    auto step = [&](int s, auto slot_c, bool fetch_next) __attribute__((always_inline)) {
        constexpr int SLOT = decltype(slot_c)::value;   // s & 1: partial buffer and operand slot
        XTM(0);
        if (!CARRY && wave < 4 && s % OWN_CHUNK == 0) {
#pragma unroll
            for (int c = 0; c < OWN_CHUNK; ++c) {
                own[512 * c] = BWD ? n0[c] : n0[c] + bias;
                if (BWD) own[512 * c + 256] = act_grad<ACT>(n1[c]);
            }
            load_chunk(s + OWN_CHUNK);
            load_ids(s + 2 * OWN_CHUNK);
        }
        park_partial(SLOT, product());
        XTM(1);
        lds_barrier();
        XTM(2);
        const int t = BWD ? T - 2 - s : s;
        float* dst = BWD ? a.Delta + (size_t)t * bh : a.hist + (size_t)(s + 1) * bh;
        float* box = a.ring + (size_t)((s + 1) % RSLOTS) * rstate;
        if (wave < 4) {
            const float in = CARRY ? s_in[SLOT][e_at] : own[512 * (s % OWN_CHUNK)];
            const float slope = !BWD ? 0.f : CARRY ? s_slope[SLOT][e_at] : own[512 * (s % OWN_CHUNK) + 256];
            const float sum = element_sum(SLOT);
            float v = BWD ? (sum + in) * slope : activate<ACT>(sum + in);
            if (__float_as_uint(v) == kSentinel) v = __uint_as_float(0x7FC00000u);   // a NaN that came in as all ones
            if (e_pub) ring_store(box + e_ring, e_on ? v : 0.f);
            if (tid == 0) s_stored = s + 1;
            if (CARRY) {
                if (ep == 0) s_out[SLOT][e_at] = v;
            } else if (e_on) {
                dst[e_off] = v;
            }
            if (e_pub) ring_store(a.ring + (size_t)((s + 3) % RSLOTS) * rstate + e_ring, __uint_as_float(kSentinel));
            last_v = v;
        }
        XTM(3);
        if (fetch_next) {
            // The other workgroups are in step with this one.  The wavefronts that have just stored a row
            // look at once; the others look when the first row is on its way (a look that comes long
            // before its data costs a second, slower one).
            if (wave >= 4)
                for (int spins = 0; spins < (1 << 16) && lds_peek(&s_stored) != s + 1; ++spins) __builtin_amdgcn_s_sleep(1);
            XTM(4);
            collect(box);
        }
        XTM(5);
    };

    const bool final_state = BWD && a.dh0 != nullptr;   // delta_0 is needed once more, for dh0
    int s2 = 0;
    bool left = false;
    for (; s2 + 1 < nsteps; s2 += 2) {
        step(s2, std::integral_constant<int, 0>{}, true);
        step(s2 + 1, std::integral_constant<int, 1>{}, s2 + 2 < nsteps || final_state);
        if (s_abort) { left = true; break; }
    }
    if (!left && s2 < nsteps) step(s2, std::integral_constant<int, 0>{}, final_state);
    XT_FLUSH(BWD);
    __syncthreads();
    if (left || s_abort) {
        if (tid == 0) atomicExch(a.status, 1);
        return;
    }
    if (!BWD) {
        if (a.h_last && e_on) a.h_last[e_off] = last_v;     // T >= 1: the last step's value
        return;
    }
    if (a.dh0) {   // dh0 = delta_0 Wh: one more product, no epilogue
        park_partial(0, product());
        __syncthreads();
        if (wave < 4) {
            const float sum = element_sum(0);
            if (e_on) a.dh0[e_off] = sum;
        }
    }
}

// the exchange ring starts as sentinels (n4 pieces of 16 bytes), the slice counters and the rolls at zero
__global__ __launch_bounds__(256) void xcd_clear_kernel(float* __restrict__ ring, int n4, int32_t* __restrict__ counters) {
    const float s = __uint_as_float(kSentinel);
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n4) reinterpret_cast<float4*>(ring)[i] = make_float4(s, s, s, s);
    if (i < REC_XCD_COUNTERS) counters[i] = 0;
}

// k per wavefront: an eighth of H in whole blocks of 16
int xcd_kw(int H) { return H <= 256 ? 32 : (H + 127) / 128 * 16; }

// Workgroups of a group and their columns.  Up to 32 rows are one group per XCD, which then has all 32 compute units; the
// fewer columns a workgroup has the fewer matrix instructions a step takes (measured: see the top).
int xcd_slots(int B) { return WG_PER_XCD / ((B + NXCD * RB - 1) / (NXCD * RB)); }
int xcd_columns(int H, int B) {
    const int per = (H + xcd_slots(B) - 1) / xcd_slots(B);
    return per <= 16 ? 16 : per <= 32 ? 32 : 64;
}

template <int ACT, bool BWD>
const void* pick_xcd_kernel(int kw, int cwd) {
#define RNN_XCD(KW, CWD) if (kw == KW && cwd == CWD) return (const void*)rec_xcd_kernel<ACT, BWD, KW, CWD>
    RNN_XCD(32, 16); RNN_XCD(48, 16); RNN_XCD(64, 16); RNN_XCD(32, 32); RNN_XCD(48, 32); RNN_XCD(64, 32); RNN_XCD(80, 32);
    RNN_XCD(96, 32); RNN_XCD(112, 32); RNN_XCD(128, 32); RNN_XCD(80, 64); RNN_XCD(96, 64); RNN_XCD(112, 64); RNN_XCD(128, 64);
#undef RNN_XCD
    return nullptr;
}

// partial tiles of a step; the forward kernel first stages its matrix slice there.  (More than half of a compute unit's)
constexpr size_t xcd_lds_bytes() { return (size_t)8 * 64 * 65 * 4; }
static_assert(alone_floats<H_MAX / 8>() * sizeof(float) <= xcd_lds_bytes(), "run_alone's tiles and states");

// of the calling thread (rec_xcd_test_roll_call)
thread_local int t_roll_us = -1, t_roll_absent = 0;

}  // namespace

int rec_xcd_groups_alone(const int32_t* counters) {
    int n = 0;
    for (int g = 0; g < NGRP; ++g) n += (counters[NXCD + g] & ROLL_CLOSED) != 0;
    return n;
}
void rec_xcd_test_roll_call(int microseconds, int absent) {
    t_roll_us = microseconds < 0 ? -1 : microseconds < 1000000 ? microseconds : 1000000;
    t_roll_absent = absent != 0;
}

// Shapes the one-launch loop serves.  Above 256 units it takes 10 us (H = 300) to 18 (H = 1024, batch 64) for the ring's clearing and
// every workgroup's part of the matrix, and then 0.8 to 1.8 us per step, a launch per step (batch above 4) up to 5.5 and the loops that
// give every sequence its own workgroups (batch 1 to 4) 1.7.  Forward, loss and backward with 1000 words, the other loop
// and this one, us: 100 steps, H = 641, 800 and 1024, batch 1: 420 and 307, 428 and 320, 435 and 339, batch 2: 463 and 326, 442 and
// 339, 459 and 358; batch 1, H = 500, 10 and 15 steps: 145 and 85, 160 and 94; batch 3, H = 700, 15 steps: 221 and 113; batch 5, H = 300,
// 4 and 9 steps: 97 and 76, 138 and 88; batch 16, H = 500: 102 and 79, 160 and 105; batch 64, H = 1024: 146 and 127, 243 and 177.  The
// lines below are where this loop began to win when it was a cooperative launch with 64 columns a workgroup; by these figures
// there is no such line from 4 steps on.
// 193 to 256 units fit one workgroup per 4 rows (recurrence_mfma.hip), whose step is bound by its matrix instructions: 0.97 us
// at H = 256 and 0.90 at H = 200, here 0.73 to 0.82 (4096 steps, batch 128: 0.78 and 0.81); up to
// 192 units 0.63 there, here 0.73 to 0.77.  35 steps of tokens, H = 200, batch 20, with the gathered input term there and the ring's
// clearing here: 46 and 38 us there, 36 and 35 here; dense input has no rows to gather.  What it costs: there a loop has a compute unit per 4
// rows and those of several streams run side by side, here they take turns (1000 steps of H = 256, batch 128 on one, two and four
// streams: 1034, 1082 and 1216 us there, 812, 1685 and 3388 here).
bool rec_xcd_supported(int H, int B, int T, bool tokens) {
    if (H <= 192 || H > H_MAX || B < 1 || B > (H <= 256 ? 128 : 64)) return false;
    if (H <= 256) return T >= (tokens && B > 4 ? 33 : 64);
    return B > 4 ? T >= 10 : T >= 16 && (B > 2 || H <= 640);
}

// A captured loop is a cooperative launch (gang.hip), and the loop of one workgroup per 4 rows is plain in any case: up to 256 units a
// captured call takes that one until the steps make up for the launch.  How much that is depends on what the program has launched
// before: 26 us a loop, or 235 if it has replayed two graphs without a cooperative launch in them first.  Three captured calls, that loop and
// this one: 128 steps of 193 units, 1 row: 317 us and 305 or 711; of 256 units, 20 dense rows: 355 and 338 or 880; 2048 steps, 20 rows, 193
// units: 3931 and, in the slower state, 3775, of 256 units 4249 and 3703.
bool rec_xcd_pays_captured(int H, int T) { return H > 256 || T >= 2048; }

// compute units the loop of these sizes keeps busy
int rec_xcd_workgroups(int H, int B) {
    const int c = xcd_columns(H, B);
    return (B + RB - 1) / RB * ((H + c - 1) / c);
}

size_t rec_xcd_ring_bytes(int H, int B) { return (size_t)RSLOTS * ring_state(B, xcd_kw(H)) * 4; }

template <bool BWD>
const void* xcd_kernel_for(int H, int B, int act) {
    const int kw = xcd_kw(H), cwd = xcd_columns(H, B);
    return act == 0 ? pick_xcd_kernel<0, BWD>(kw, cwd) : pick_xcd_kernel<1, BWD>(kw, cwd);
}

// Can all 256 workgroups be resident at once on the current device (one per compute unit)?  Asked
// once per kernel and device; also raises the kernel's LDS limit.
bool rec_xcd_ready(int H, int B, int act, bool bwd) {
    const void* fn = bwd ? xcd_kernel_for<true>(H, B, act) : xcd_kernel_for<false>(H, B, act);
    const size_t lds = xcd_lds_bytes();
    struct Seen { const void* fn; int dev; bool ok; };
    static Seen seen[512];
    static int n_seen = 0;
    static std::mutex mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    std::lock_guard<std::mutex> lock(mu);
    for (int i = 0; i < n_seen; ++i)
        if (seen[i].fn == fn && seen[i].dev == dev) return seen[i].ok;
    int per_cu = 0, cus = 0;
    const bool ok = allow_lds(fn, lds) == hipSuccess &&
                    hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads_of(xcd_columns(H, B)), lds) == hipSuccess &&
                    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
                    per_cu >= 1 && cus == NXCD * WG_PER_XCD;
    if (n_seen < 512) seen[n_seen++] = Seen{fn, dev, ok};
    return ok;
}

void rec_xcd_fills(const RecXcdArgs& a, FillJob* ring, FillJob* counters) {
    *ring = {reinterpret_cast<int32_t*>(a.ring), (size_t)RSLOTS * ring_state(a.B, xcd_kw(a.H)), (int32_t)kSentinel};
    *counters = {a.counters, (size_t)REC_XCD_COUNTERS, 0};
}

hipError_t launch_rec_xcd(const RecXcdArgs& a, bool bwd, hipStream_t s) {
    if (a.H > H_MAX || a.B < 1 || a.B > NGRP * RB || (a.H + 63) / 64 > xcd_slots(a.B)) return hipErrorInvalidValue;
    if (!rec_xcd_ready(a.H, a.B, a.act, bwd)) return hipErrorNotSupported;
    const void* fn = bwd ? xcd_kernel_for<true>(a.H, a.B, a.act) : xcd_kernel_for<false>(a.H, a.B, a.act);
    const size_t lds = xcd_lds_bytes();

    if (!a.cleared) {
        ProfileScope ps(K_MISC, s);
        const int n4 = RSLOTS * ring_state(a.B, xcd_kw(a.H)) / 4;
        hipLaunchKernelGGL(xcd_clear_kernel, dim3((n4 + 255) / 256), dim3(256), 0, s, a.ring, n4, a.counters);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    ProfileScope ps(bwd ? K_REC_BWD : K_REC_FWD, s);
    RecXcdArgs args = a;
    if (args.spin_limit <= 0) args.spin_limit = wait_limit();
    args.slots = xcd_slots(a.B);
    // As long as one workgroup would take by itself: waiting costs at most as much again.  A quarter of a second at most: a replayed
    // graph may have brought a loop here beside another that waits for about a second and then gives up.  (100 steps at H = 200, 300, 500, 700 and
    // 1024, by batch and direction: 0.9 to 1.3, 1.2 to 2.1, 2.9 to 4.0, 4.5 to 6.0 and 12 to 16 ms)
    const double alone_us = a.T * (5.0 + 125.0 * a.H / H_MAX * a.H / H_MAX);
    args.patience = (int)(100.0 * (t_roll_us >= 0 ? t_roll_us : fmin(fmax(alone_us, 200.0), 2.5e5)));
    args.absent = t_roll_absent;
    void* kargs[] = {&args};
    return launch_gang(fn, dim3(NXCD * WG_PER_XCD), dim3(threads_of(xcd_columns(a.H, a.B))), kargs, lds, s, true);
}

}  // namespace rnn

#ifdef RNN_REC_TRACE
extern "C" int rnn_xcd_trace(long long* host_out, int n) {
    return hipMemcpyFromSymbol(host_out, HIP_SYMBOL(rnn::g_xcd_trace), (size_t)n * 8) == hipSuccess ? 0 : -4;
}
#endif
