// Attention of one query head over a list of selected keys, for a block of
// 1024 threads or, over short lists, fewer (Eqs. approx_weight, approx_output):
//   o = sum_{i in list} softmax_i(scale <k_i, q>) v_i,  float16 in, float32 math.
// Shared by the stand-alone attention kernel and the fused top-k + attention
// kernel, so both produce the same bits.
//
// 64 key slots of 16 lanes: lane l16 owns dims [8 l16, 8 l16 + 8), so a K or
// V row is one 256-byte contiguous read by 16 lanes.  Slot s takes list
// entries s, s + 64, ...; every lane keeps 8 K and 8 V row segments in flight.
// Each slot keeps an online-softmax state (running max, sum, 8 accumulators
// per lane).  At the end the 4 slots of a wave merge by two butterfly steps
// across its rows of 16 lanes (partners lane ^ 16, then lane ^ 32), and the 16
// wave states merge through LDS, 8 threads per dimension.
//
// A block of 512 (256) threads plays the same 64 slots, 2 (4) per group of 16 lanes with 4 (2)
// rows in flight each, over lists of at most 256 (128) rows, which is one round: every sum
// is taken over the same values in the same order, so the result has the same bits.  Short
// lists then cost a quarter of the waves, and several blocks share a CU.
//
// Rows come from one of two caches: a list entry with kWinRow set names row
// (entry - kWinRow) of the window cache (Kw, Vw, win_capacity: Sink and Local /
// Update Buffer kept on the GPU), any other entry >= 0 a row of the main cache
// (K, V, kv_capacity: the retrieval rows, in HBM or in host memory).  Entries
// past their cache's capacity, and negative entries (-1 padding), are skipped.
//
// A caller that already holds some rows in LDS passes prow (LDS rows of 32
// uint4: K then V) and lists such a row as entry -2 - (LDS row); it is read from
// LDS, the same bytes in the same order, so the result does not depend on which
// rows were held.  Without prow every negative entry is skipped.
#pragma once

#include <hip/hip_fp16.h>

#include "internal.hpp"

namespace pariskv {

constexpr int kAtThreads = 1024;
constexpr int kAtGroups = kAtThreads / 16;  // key slots of a block
constexpr int kAtWaves = kAtThreads / 64;   // slot states left after the merge of 4 slots
constexpr int kAtUnroll = 8;                // K/V rows in flight per lane
// Longest list a block of TH threads takes (one round of its rows in flight).
template <int TH>
constexpr int kAtRows = TH == kAtThreads ? kMaxAttendRows : kAtGroups * kAtUnroll * TH / kAtThreads;

// LDS the row needs beyond the key list: running max, sum and accumulators per wave.
struct AttendScratch {
    float m[kAtWaves];
    float l[kAtWaves];
    float acc[kAtWaves][kD];
};

__device__ __forceinline__ void unpack8_half(const uint4 v, float* f) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        f[2 * h] = __half2float(__ushort_as_half((unsigned short)(w[h] & 0xffffu)));
        f[2 * h + 1] = __half2float(__ushort_as_half((unsigned short)(w[h] >> 16)));
    }
}

// Any value: a row segment that is not loaded is never used, and setting it would cost
// 4 instructions a row.
__device__ __forceinline__ uint4 unset_uint4() {
    uint4 v;
    asm volatile("" : "=v"(v.x), "=v"(v.y), "=v"(v.z), "=v"(v.w));
    return v;
}

// Sum of x over the 16 lanes of each row of the wave, in every lane, through
// DPP adds (no LDS): partners lane ^ 1 and lane ^ 2 (quad_perm), then the
// mirrored lane in the half row and in the row.  After the quad steps the lanes
// of a quad hold equal values, so the mirror partners add the same values as
// partners lane ^ 4 and lane ^ 8 would: the xor butterfly's result, bit for bit.
__device__ __forceinline__ float sum16(float x) { return row_sum_f32(x); }

// The 16 bytes of the head's float16 query that thread `tid` uses: dims
// [8 (tid & 15), 8 (tid & 15) + 8).  Callers load it first, so its latency
// overlaps their own work.
__device__ __forceinline__ uint4 attend_query_part(const __half* q_row) {
    return reinterpret_cast<const uint4*>(q_row)[threadIdx.x & 15];
}

// qv: this thread's query part (attend_query_part); K, V: the KV head's rows
// [kv_capacity][D]; Kw, Vw: its window-cache rows [win_capacity][D] (entries
// with kWinRow); list: k <= kAtRows<TH> entries in LDS (already synchronised); out: D floats.
// Every thread of the block must call it; it ends with the block synchronised.
template <int TH = kAtThreads>
__device__ __forceinline__ void attend_row(uint4 qv, const __half* __restrict__ K,
                                           const __half* __restrict__ V, int64_t kv_capacity,
                                           const __half* __restrict__ Kw, const __half* __restrict__ Vw,
                                           int64_t win_capacity, const int32_t* list, int32_t k,
                                           float scale, float* __restrict__ out, AttendScratch& sm,
                                           const uint4* prow = nullptr) {
    constexpr int kSlots = kAtThreads / TH;       // slots a group of 16 lanes plays
    constexpr int kRows = kAtUnroll / kSlots;     // rows in flight per slot
    constexpr int kGroups = kAtGroups / kSlots;   // groups of 16 lanes in the block
    constexpr int kWaves = TH / 64;
    const int tid = threadIdx.x;
    const int grp16 = tid >> 4;  // key slots grp16, grp16 + kGroups, ...
    const int l16 = tid & 15;

    float qf[8];
    unpack8_half(qv, qf);
#pragma unroll
    for (int d = 0; d < 8; ++d) qf[d] *= scale;

    float m[kSlots], lsum[kSlots], acc[kSlots][8];
#pragma unroll
    for (int v = 0; v < kSlots; ++v) {
        m[v] = -__builtin_huge_valf();
        lsum[v] = 0.f;
#pragma unroll
        for (int d = 0; d < 8; ++d) acc[v][d] = 0.f;
    }

    // Capacities fit 30 bits; without a window cache the entries need no test for it.
    const uint32_t kv_rows = (uint32_t)kv_capacity, win_rows = (uint32_t)win_capacity;
    const uint4* Kl = reinterpret_cast<const uint4*>(K) + l16;
    const uint4* Vl = reinterpret_cast<const uint4*>(V) + l16;
    for (int base = 0; base < k; base += kAtGroups * kRows) {
        int32_t key[kAtUnroll];  // row u of slot v at v kRows + u
        uint4 kc[kAtUnroll], vc[kAtUnroll];
        // Every list entry read before the first is used.
#pragma unroll
        for (int i = 0; i < kAtUnroll; ++i)
            key[i] = list[min(base + grp16 + kGroups * (i / kRows) + kAtGroups * (i % kRows), k - 1)];
#pragma unroll
        for (int i = 0; i < kAtUnroll; ++i) {
            if (base + grp16 + kGroups * (i / kRows) + kAtGroups * (i % kRows) >= k) key[i] = -1;
            uint32_t rowi = (uint32_t)key[i], cap = kv_rows;  // a negative entry is past every capacity
            const uint4 *kb = Kl, *vb = Vl;
            if (win_rows) {
                const bool win = key[i] >= kWinRow;
                rowi = win ? (uint32_t)(key[i] - kWinRow) : rowi;
                cap = win ? win_rows : cap;
                kb = win ? reinterpret_cast<const uint4*>(Kw) + l16 : kb;
                vb = win ? reinterpret_cast<const uint4*>(Vw) + l16 : vb;
            }
            const bool in = rowi < cap;
            if (!in && (prow == nullptr || key[i] >= 0)) key[i] = -1;  // else held (<= -2) or -1
            kc[i] = unset_uint4();
            vc[i] = unset_uint4();
            if (in) {
                const int64_t off = (int64_t)rowi * (kD / 8);
                kc[i] = kb[off];
                vc[i] = vb[off];
            }
        }
        float dot[kAtUnroll];
#pragma unroll
        for (int i = 0; i < kAtUnroll; ++i) {
            if (prow != nullptr && key[i] <= -2) {
                kc[i] = prow[32 * (-2 - key[i]) + l16];
                vc[i] = prow[32 * (-2 - key[i]) + 16 + l16];
            }
            float kf[8];
            unpack8_half(kc[i], kf);
            float d0 = 0.f;
#pragma unroll
            for (int d = 0; d < 8; ++d) d0 += qf[d] * kf[d];
            dot[i] = d0;
        }
#pragma unroll
        for (int i = 0; i < kAtUnroll; ++i) dot[i] = sum16(dot[i]);
#pragma unroll
        for (int v = 0; v < kSlots; ++v) {
            float mn = m[v];
#pragma unroll
            for (int u = 0; u < kRows; ++u)
                if (key[v * kRows + u] != -1) mn = fmaxf(mn, dot[v * kRows + u]);
            if (mn > -__builtin_huge_valf()) {
                const float corr = __expf(m[v] - mn);
                lsum[v] *= corr;
#pragma unroll
                for (int d = 0; d < 8; ++d) acc[v][d] *= corr;
#pragma unroll
                for (int u = 0; u < kRows; ++u) {
                    const int i = v * kRows + u;
                    if (key[i] != -1) {
                        const float p = __expf(dot[i] - mn);
                        float vf[8];
                        unpack8_half(vc[i], vf);
                        lsum[v] += p;
#pragma unroll
                        for (int d = 0; d < 8; ++d) acc[v][d] += p * vf[d];
                    }
                }
                m[v] = mn;
            }
        }
    }

    // The 4 slots in the rows of 16 lanes of a wave (holding the same dims) into one.
    const int lane = tid & 63;
    const int wave = tid >> 6;
#pragma unroll
    for (int v = 0; v < kSlots; ++v) {
#pragma unroll
        for (int step = 16; step <= 32; step <<= 1) {
            const float mp = __uint_as_float(lane_xor(__float_as_uint(m[v]), step, lane));
            const float lp = __uint_as_float(lane_xor(__float_as_uint(lsum[v]), step, lane));
            float ap[8];
#pragma unroll
            for (int d = 0; d < 8; ++d) ap[d] = __uint_as_float(lane_xor(__float_as_uint(acc[v][d]), step, lane));
            const float mn = fmaxf(m[v], mp);
            if (mn > -__builtin_huge_valf()) {
                const float c0 = __expf(m[v] - mn), c1 = __expf(mp - mn);
                lsum[v] = lsum[v] * c0 + lp * c1;
#pragma unroll
                for (int d = 0; d < 8; ++d) acc[v][d] = acc[v][d] * c0 + ap[d] * c1;
            }
            m[v] = mn;
        }
        if (lane < 16) {
            const int st = wave + kWaves * v;  // slots 4 st .. 4 st + 3
            if (l16 == 0) {
                sm.m[st] = m[v];
                sm.l[st] = lsum[v];
            }
#pragma unroll
            for (int d = 0; d < 8; ++d) sm.acc[st][8 * l16 + d] = acc[v][d];
        }
    }
    __syncthreads();
    {
        // Every thread: dim d of 2 of the 16 states, then a sum over the 8 threads
        // of the dim (lanes 8 d' + part) by lane exchanges.  An empty state (m = -inf,
        // l = 0, acc = 0) is scaled by exp(-inf) = 0, so it needs no test.
        static_assert(kAtThreads == 8 * kD && kAtWaves == 16, "8 threads per dim, 2 states each");
        float M = -__builtin_huge_valf();
#pragma unroll
        for (int j = 0; j < kAtWaves; ++j) M = fmaxf(M, sm.m[j]);
        const int part = tid & 7;
#pragma unroll
        for (int v = 0; v < kSlots; ++v) {
            const int d = (tid >> 3) + TH / 8 * v;
            float L = 0.f, O = 0.f;
            if (M > -__builtin_huge_valf()) {
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    const int j = 2 * part + r;
                    const float c = __expf(sm.m[j] - M);
                    L += sm.l[j] * c;
                    O += sm.acc[j][d] * c;
                }
            }
#pragma unroll
            for (int x = 1; x < 8; x <<= 1) {
                L += __uint_as_float(lane_xor(__float_as_uint(L), x, lane));
                O += __uint_as_float(lane_xor(__float_as_uint(O), x, lane));
            }
            if (part == 0) out[d] = L > 0.f ? O / L : 0.f;
        }
    }
    __syncthreads();
}

}  // namespace pariskv
