// Stage II of the decode-time retrieval: RSQ-IP reranking of the candidates
// and the final top-k (Sec. "Retrieval" (2); Appendix "RSQ-IP Reranking from
// 4-Bit Key Summaries", Eqs. rsqip_raw and rsqip_raw_weighted; Alg. 1 Stage II).
//
// With z = H(s q) (so ||q|| q_tilde_b = z_b / sqrt(D)) and the stored
// W_b = sqrt(D) w_b, the estimator of <k_i, q> is
//     s_hat_i = ||q|| sum_b w_b <v_b, q_tilde_b> = sum_b W_b <v_b, z_b / D>,
// where v_b has coordinates sign * a[t] decoded from the 4-bit codes.  The
// query side z/D arrives as float from the query kernel.
//
// compact_rerank_kernel: one block per (query head, 4096-key chunk).  Large
// grids take blocks of 128 threads (32 keys per thread), so that 16 blocks
// share a CU and their selection phases hide under each other's gathers; a
// grid that fits the chip in one round of 256-thread blocks takes those (16
// keys per thread), which halves each block's serial work, and a smaller one
// 512-thread blocks.  It selects the chunk's candidates
// (all S > theta, then S == theta in ascending key order while the row's quota
// lasts), which occupy consecutive positions of the row's candidate list,
// writes them (and keeps them in LDS as 16-bit offsets in the chunk), and
// scores them at once: 8 lanes
// per candidate, lane l reads the 16-byte chunk l of the 128-byte record
// (codes of subspaces 2l, 2l+1 and their W), so one candidate is one fully
// used 128-byte line and a wave reads 8 lines per load instruction.  Lane l
// keeps the 16 query coordinates of its two subspaces in registers; the
// signed level table (16 floats) lives in LDS.
//
// topk_reg_kernel (blocks of 256, 512 or 1024 threads, at most 8 candidates per thread) and
// topk_lds_kernel (more): one block per list; the k-th largest estimate is found exactly on
// order-preserving uint32 keys, ties at it taken in candidate order, then an
// ordered compaction lists the winners in ascending key index (candidate order)
// without a sort.  The keys are held in registers (staged in LDS by the second
// kernel), binned linearly in value over [min, max] (the float bit patterns
// crowd into a few exponent prefixes), and the boundary bin is ranked by brute force when it holds
// at most 64 keys, else by radix passes of 9 to 11 bits restricted to it.  A list
// is one query head's candidates (C <= 32768), or, in two passes, first every
// 4096-candidate slice of a head and then the concatenated winners of its slices
// (more than 32768 candidates, or more than 8192 for few heads).  With the
// attention fused (topk_reg_kernel), keys in bins above the boundary bin win
// whatever the rest of the selection finds, so once that bin is known each wave
// requests the K/V rows of up to 12 of them; those gathers run while the
// selection finishes, the rows wait in LDS, and the attention reads them there.

#include "attend_row.hpp"
#include "internal.hpp"

namespace pariskv {

namespace {

// One 4096-key chunk per block: 128 threads for large grids, 256 for grids of at
// most kRrWideGrid blocks (8 such blocks per CU on 256 CUs: one round), 512 up to
// kRrWidestGrid blocks (2 per CU: each block's serial selection counts; 256 blocks of 32K-key
// rows 7.6 -> 6.4 us, 8 blocks 8.9 -> 6.2, 512 blocks 8.8 -> 8.4, but 1024 blocks 11.5 -> 12.0).
constexpr int64_t kRrWidestGrid = 512;
static_assert(kTopkPart >= PARISKV_MAX_TOPK, "a top-k slice holds at least k candidates");
static_assert(PARISKV_MAX_CAND / kTopkPart * PARISKV_MAX_TOPK <= 1024 * 32, "the slices' winners fit one block");
constexpr int kRrUnroll = 4;  // records in flight per lane
constexpr int64_t kManyRows = 256;  // top-k blocks past one per CU

// Order-preserving uint32 key of a float (larger float, larger key; finite floats
// map above 0) and back.
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_float(uint32_t k) {
    const uint32_t u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
    return __uint_as_float(u);
}

// What a block of the folded rerank derives for its row and chunk.
struct RowSelect {
    uint32_t theta, quota, base_g, base_e;
};

template <int TH>
struct FoldScratch {
    uint32_t part[TH / 64][4][64];  // per wave: row totals (v = lane, 64 + lane), totals before the chunk
    uint32_t sum[2][TH / 64][2];    // the search's, per pass and wave: counts before the chunk, from it on
};

// The selection threshold of row `row` and the chunk's bases, as the threshold kernel leaves
// them (there one block per row does it for all chunks), for rows of at most kFoldChunks
// chunks: see fold_threshold.  Every thread of the block calls it.  It costs the rerank 1 to
// 2 us (a chunk histogram read and one more barrier, where the plain form waits for the
// threshold's words) and saves a launch of 4.
template <int TH>
__device__ __forceinline__ RowSelect row_select(const RetrieveArgs& a, int64_t row, int64_t chunk,
                                                FoldScratch<TH>& sm) {
    constexpr int kWaves = TH / 64;
    constexpr int kPer = kFoldChunks / kWaves;  // chunk histograms per wave
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t* sfx = a.chunk_sfx + row * a.n_chunks * kSfx;
    int32_t* t = a.thresh + row * kThreshRow;
    const uint32_t fl = (uint32_t)t[4];  // the floor the scan used
    const int nc = (int)a.n_chunks, ck = (int)chunk;
    // Every load is issued (clamped into the row) before the first wait.
    uint32_t xl[kPer], xh[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int c = min(wave + kWaves * u, nc - 1);
        xl[u] = sfx[c * kSfx + lane];
        xh[u] = sfx[c * kSfx + 64 + min(lane, kSfx - 65)];
    }
    uint32_t tl = 0, thi = 0, bl = 0, bh = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int c = wave + kWaves * u;
        const uint32_t l = c < nc ? xl[u] : 0u, h = c < nc && lane < kSfx - 64 ? xh[u] : 0u;
        tl += l;
        thi += h;
        bl += c < ck ? l : 0u;
        bh += c < ck ? h : 0u;
    }
    sm.part[wave][0][lane] = tl;
    sm.part[wave][1][lane] = thi;
    sm.part[wave][2][lane] = bl;
    sm.part[wave][3][lane] = bh;
    __syncthreads();
    tl = thi = bl = bh = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        tl += sm.part[w][0][lane];
        thi += sm.part[w][1][lane];
        bl += sm.part[w][2][lane];
        bh += sm.part[w][3][lane];
    }
    const uint32_t C = (uint32_t)a.c_eff;
    // The counts are exact for v = 0 and v >= the floor: with #{S >= floor} >= C (or floor 1)
    // theta is found among them, otherwise the scores below it are counted too.
    const uint32_t at_floor = fl < 64 ? __shfl(tl, (int)fl, 64) : __shfl(thi, (int)fl - 64, 64);
    const bool recount = fl > 1u && at_floor < C;
    auto pick = [](uint32_t lo, uint32_t hi, int v) {
        return v < 64 ? (uint32_t)__builtin_amdgcn_readlane((int)lo, v) : (uint32_t)__builtin_amdgcn_readlane((int)hi, v - 64);
    };
    RowSelect r;
    uint32_t gt;
    if (!recount) {
        int theta;
        theta_of(tl, thi, C, lane, &theta, &gt);
        theta = __builtin_amdgcn_readfirstlane(theta);
        r.theta = (uint32_t)theta;
        r.base_g = pick(bl, bh, theta + 1);
        r.base_e = pick(bl, bh, theta) - r.base_g;
    } else {
        // theta is the one v of [lo, hi] with count(v) >= C > count(v + 1).  Every pass over the row's
        // scores counts two neighbours, from the floor downwards (theta mostly lies 1 or 2 below it),
        // from the third pass on halving.  Every block of the row does it, so it has to cost little:
        // scores are at most 96, so adding 128 - v to each byte carries into none and sets its top bit
        // iff S >= v (as in the compaction), 3 instructions for 4 keys and level and no atomics.
        // Keys of 16 modes, C = n / 8 (most heads), with the threshold kernel / a histogram of the row
        // per block / this: 128 rows x 45679 keys 67.6 / 104 / 61.9 us a call, 64 x 128K 89.6 / 302 /
        // 77.9, 384 x 64K 183 / 430 / 169.
        static_assert(kFoldChunks * kChunk / kWaves <= 0xffff, "a wave's counts in 16 bits");
        const uint8_t* srow = a.score8 + row * a.n_pad;
        const int n = (int)a.n, whole = n & ~15, split = ck * kChunk;
        int lo = 0, hi = (int)fl - 1;
        gt = at_floor;  // count(hi + 1), in the row and before the chunk
        r.base_g = pick(bl, bh, (int)fl);
        for (int pass = 0;; ++pass) {
            const int m = pass < 2 ? max(lo, hi - 1) : (lo + hi) >> 1;
            const uint32_t k0 = (uint32_t)(128 - m) * 0x01010101u, k1 = k0 - 0x01010101u;  // S >= m, S >= m + 1
            // #{S >= m + 1} + 2^16 #{S >= m} of this thread's 16-key words of [from, to).
            auto count = [&](int from, int to) -> uint32_t {
                uint32_t c0 = 0, c1 = 0;
#pragma unroll 4
                for (int i = from + 16 * tid; i < to; i += 16 * TH) {
                    const uint4 w = *reinterpret_cast<const uint4*>(srow + i);
                    const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        c0 += (uint32_t)__popc((ww[q] + k0) & 0x80808080u);
                        c1 += (uint32_t)__popc((ww[q] + k1) & 0x80808080u);
                    }
                }
                return c0 << 16 | c1;
            };
            uint32_t before = count(0, split), after = count(split, whole);
            if (tid < n - whole) {  // the row's last keys, one each
                const int v = srow[whole + tid];
                after += (v >= m ? 0x10000u : 0u) + (v > m ? 1u : 0u);
            }
            before = wave_incl_sum(before);
            after = wave_incl_sum(after);
            if (lane == 63) {
                sm.sum[pass & 1][wave][0] = before;
                sm.sum[pass & 1][wave][1] = after;
            }
            __syncthreads();
            uint32_t b0 = 0, b1 = 0, g0 = 0, g1 = 0;  // count(m), count(m + 1): before the chunk, in the row
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t x = sm.sum[pass & 1][w][0], y = sm.sum[pass & 1][w][1];
                b0 += x >> 16;
                b1 += x & 0xffffu;
                g0 += (x >> 16) + (y >> 16);
                g1 += (x & 0xffffu) + (y & 0xffffu);
            }
            b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b0);
            b1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)b1);
            g0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)g0);
            g1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)g1);
            if (g1 >= C) {
                lo = m + 1;
                if (lo < hi) continue;
                r.theta = (uint32_t)hi;
                r.base_e = b1 - r.base_g;
                break;
            }
            if (g0 >= C) {
                r.theta = (uint32_t)m;
                gt = g1;
                r.base_g = b1;
                r.base_e = b0 - b1;
                break;
            }
            hi = m - 1;
            gt = g0;
            r.base_g = b0;
        }
    }
    r.quota = C - gt;
    if (tid == 0) {
        int32_t* cb = a.chunk_base + (row * a.n_chunks + chunk) * 2;
        cb[0] = (int32_t)r.base_g;
        cb[1] = (int32_t)r.base_e;
        if (chunk == 0) {  // t[4] stays the scan's: the other blocks read it
            t[0] = (int32_t)r.theta;
            t[1] = (int32_t)gt;
            t[2] = (int32_t)r.quota;
            t[3] = (int32_t)C;
            t[5] = recount ? 1 : 0;
            t[6] = t[7] = 0;
        }
    }
    return r;
}

// Compaction of one chunk's candidates (Stage I selection) fused with their
// RSQ-IP rerank (Stage II).  The selected keys of a chunk hold consecutive
// positions [P0, P0 + m) of the row's ascending candidate list, so the block
// writes them to `cand`, keeps them in LDS and scores them right away.
template <int kRrThreads, bool kFold>
__global__ __launch_bounds__(kRrThreads, 8) void compact_rerank_kernel(RetrieveArgs a) {
    constexpr int kKpt = kChunk / kRrThreads;   // keys per thread
    constexpr int kRrSlots = kRrThreads / 8;    // candidates reranked per block iteration
    constexpr int kWords = kKpt / 4;            // score words per thread
    static_assert(kKpt >= 8 && kKpt <= 32, "pairs of score words, one 32-bit mask");
    __shared__ float s_tab[16];
    __shared__ uint32_t s_wsum[kRrThreads / 64];
    // The selected keys as offsets in the chunk (2 bytes each, so 16 blocks fit a CU).
    __shared__ uint16_t s_list[kChunk];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int64_t chunk = blockIdx.x;
    const int64_t row = blockIdx.y;  // seq * hq + head
    const int seq = (int)(row / a.hq);
    const int hq = (int)(row % a.hq);
    const int64_t grp = (int64_t)seq * a.hkv + hq / a.g;

    // Everything this block reads up front.
    uint32_t theta = 0, quota = 0, base_g = 0, base_e = 0;
    if constexpr (!kFold) {
        const int32_t* th = a.thresh + row * kThreshRow;
        const int32_t* cb = a.chunk_base + (row * a.n_chunks + chunk) * 2;
        theta = (uint32_t)th[0];
        quota = (uint32_t)th[2];
        base_g = (uint32_t)cb[0];
        base_e = (uint32_t)cb[1];
    }
    // This thread's kKpt keys; score rows are padded to a multiple of 64 bytes, so a
    // load that starts before n stays inside the row.
    const int64_t i0 = chunk * kChunk + kKpt * tid;
    uint32_t ww[kWords];
    {
        const uint8_t* sp = a.score8 + row * a.n_pad + i0;
        if constexpr (kWords >= 4) {
#pragma unroll
            for (int u = 0; u < kWords / 4; ++u) {
                uint4 t = make_uint4(0, 0, 0, 0);
                if (i0 + 16 * u < a.n) t = reinterpret_cast<const uint4*>(sp)[u];
                ww[4 * u] = t.x;
                ww[4 * u + 1] = t.y;
                ww[4 * u + 2] = t.z;
                ww[4 * u + 3] = t.w;
            }
        } else {
            uint2 t = make_uint2(0, 0);
            if (i0 < a.n) t = *reinterpret_cast<const uint2*>(sp);
            ww[0] = t.x;
            ww[1] = t.y;
        }
    }
    const int l = tid & 7;
    float z[16];
    {
        const float4* zp = reinterpret_cast<const float4*>(a.zq + row * kD + 16 * l);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float4 t = zp[v];
            z[4 * v] = t.x; z[4 * v + 1] = t.y; z[4 * v + 2] = t.z; z[4 * v + 3] = t.w;
        }
    }
    if (tid < 16) s_tab[tid] = (tid & 8) ? -a.qc.a32[tid & 7] : a.qc.a32[tid & 7];

    if constexpr (kFold) {
        __shared__ FoldScratch<kRrThreads> s_fold;
        const RowSelect r = row_select<kRrThreads>(a, row, chunk, s_fold);
        theta = r.theta;
        quota = r.quota;
        base_g = r.base_g;
        base_e = r.base_e;
    }

    // ---- compaction: all S > theta, and S == theta while the row's quota lasts.
    // Four keys a word: scores are at most 96, so adding 127 - theta (128 - theta) to every byte
    // carries into none and sets its top bit iff S > theta (S >= theta); a byte dot product
    // gathers the top bits of two words: 30 instructions for 16 keys where testing each key
    // took 160, which is what the selection was bound by (rerank of 128 rows x 45K keys 15.2 ->
    // 14.1 us, 448 x 7001 16.9 -> 15.6, 128 x 100K 24.0 -> 22.3).  Bytes past n may hold
    // anything: a carry only reaches later bytes, which are past n too.
    uint32_t gmask = 0, emask = 0;
    {
        static_assert(kMaxScore <= 127, "7-bit scores");
        const uint32_t gt = (127u - theta) * 0x01010101u, ge = (128u - theta) * 0x01010101u;
#pragma unroll
        for (int v = 0; v < kWords; v += 2) {
            uint32_t g = __builtin_amdgcn_udot4((ww[v] + gt) & 0x80808080u, 0x08040201u, 0u, false);
            uint32_t e = __builtin_amdgcn_udot4((ww[v] + ge) & 0x80808080u, 0x08040201u, 0u, false);
            g = __builtin_amdgcn_udot4((ww[v + 1] + gt) & 0x80808080u, 0x80402010u, g, false);
            e = __builtin_amdgcn_udot4((ww[v + 1] + ge) & 0x80808080u, 0x80402010u, e, false);
            gmask |= (g >> 7) << (4 * v);
            emask |= (e >> 7) << (4 * v);
        }
        const int64_t left = a.n - i0;  // this thread's keys inside the row
        const uint32_t in = left >= kKpt ? 0xffffffffu : left > 0 ? (1u << (int)left) - 1u : 0u;
        gmask &= in;
        emask &= in & ~gmask;
    }
    // Packed (gt, eq) counts: each at most 4096 per chunk, 16 bits each.
    const uint32_t mine = (uint32_t)__popc(gmask) | ((uint32_t)__popc(emask) << 16);
    const uint32_t incl = wave_incl_sum(mine);
    if (lane == 63) s_wsum[wave] = incl;
    __syncthreads();
    uint32_t pre = incl - mine, tot = 0;
#pragma unroll
    for (int w = 0; w < kRrThreads / 64; ++w) {
        const uint32_t x = s_wsum[w];
        if (w < wave) pre += x;
        tot += x;
    }
    const uint32_t P0 = base_g + min(base_e, quota);
    const uint32_t m = (tot & 0xffffu) + (min(base_e + (tot >> 16), quota) - min(base_e, quota));
    const uint32_t eb = base_e + (pre >> 16);  // S == theta keys before this thread's keys
    // Ties are taken while the quota lasts: all of this thread's, none, or (one thread of the
    // row) the first `rest`.
    const uint32_t rest = quota > eb ? quota - eb : 0u;
    emask = rest ? emask : 0u;
    while ((uint32_t)__popc(emask) > rest) emask &= ~(0x80000000u >> __clz((int)emask));
    // The taken keys (about 1 in 16) in ascending order, at consecutive places.
    uint32_t p = (pre & 0xffffu) + min(eb, quota) - min(base_e, quota);
    for (uint32_t sel = gmask | emask; sel; sel &= sel - 1u) s_list[p++] = (uint16_t)(kKpt * tid + __builtin_ctz(sel));
    __syncthreads();

    // ---- RSQ-IP: 8 lanes per candidate, lane l reads record chunk l (subspaces 2l, 2l+1).
    const int slot = tid >> 3;
    // The chunk's part of the candidate list, in whole lines (a store per key inside the
    // selection loop, or beside each estimate, took 0.5 to 2 us longer over 2M candidates).
    int32_t* cand = a.cand + row * a.n_cand + P0;
    for (uint32_t i = tid; i < m; i += kRrThreads) cand[i] = (int32_t)chunk * kChunk + s_list[i];
    float* out = a.cand_score + row * a.n_cand + P0;
    const uint4* rec = reinterpret_cast<const uint4*>(a.rec + grp * a.capacity * kRec);
    const uint32_t two = 2u;
    const char* tab = reinterpret_cast<const char*>(s_tab);
    auto entry = [&](uint32_t byte_off) { return *reinterpret_cast<const float*>(tab + byte_off); };
#pragma unroll 1
    for (uint32_t it = 0; it < m; it += kRrSlots * kRrUnroll) {
        uint4 rc[kRrUnroll];
#pragma unroll
        for (int u = 0; u < kRrUnroll; ++u) {
            // Past the end, re-read the last candidate; its result is not stored.
            const uint32_t ci = min(it + u * kRrSlots + slot, m - 1u);
            rc[u] = rec[((uint64_t)chunk * kChunk + s_list[ci]) * (kRec / 16) + l];
        }
#pragma unroll
        for (int u = 0; u < kRrUnroll; ++u) {
            // Code of coordinate 2k in the low nibble of byte k, of 2k+1 in the high
            // nibble: one mask per word, then one byte-select shift per lookup.
            const uint32_t e0 = rc[u].x & 0x0f0f0f0fu, o0 = rc[u].x & 0xf0f0f0f0u;
            const uint32_t e1 = rc[u].y & 0x0f0f0f0fu, o1 = rc[u].y & 0xf0f0f0f0u;
            float d0 = 0.f, d1 = 0.f;
            d0 += entry(byte_shl2<0>(e0, two)) * z[0];
            d0 += entry(byte_shr2<0>(o0, two)) * z[1];
            d0 += entry(byte_shl2<1>(e0, two)) * z[2];
            d0 += entry(byte_shr2<1>(o0, two)) * z[3];
            d0 += entry(byte_shl2<2>(e0, two)) * z[4];
            d0 += entry(byte_shr2<2>(o0, two)) * z[5];
            d0 += entry(byte_shl2<3>(e0, two)) * z[6];
            d0 += entry(byte_shr2<3>(o0, two)) * z[7];
            d1 += entry(byte_shl2<0>(e1, two)) * z[8];
            d1 += entry(byte_shr2<0>(o1, two)) * z[9];
            d1 += entry(byte_shl2<1>(e1, two)) * z[10];
            d1 += entry(byte_shr2<1>(o1, two)) * z[11];
            d1 += entry(byte_shl2<2>(e1, two)) * z[12];
            d1 += entry(byte_shr2<2>(o1, two)) * z[13];
            d1 += entry(byte_shl2<3>(e1, two)) * z[14];
            d1 += entry(byte_shr2<3>(o1, two)) * z[15];
            float part = __uint_as_float(rc[u].z) * d0 + __uint_as_float(rc[u].w) * d1;
            part += __uint_as_float(lane_xor(__float_as_uint(part), 1, lane));
            part += __uint_as_float(lane_xor(__float_as_uint(part), 2, lane));
            part += __uint_as_float(lane_xor(__float_as_uint(part), 4, lane));
            // + 0.0f turns -0 into +0, so equal estimates compare equal in the top-k keys.
            const uint32_t ci = it + u * kRrSlots + slot;
            if (l == 0 && ci < m) out[ci] = part + 0.0f;
        }
    }
}

// ---------------------------------------------------------------- top-k


// Shared by both top-k kernels, run by one whole wave: the digit holding the
// need-th largest element of a histogram of NB bins.  Lane L owns bins
// NB-1-L*PER .. NB-PER-L*PER (descending); a scan of the lane totals finds the
// lane whose bins hold the crossing, then PER lanes take its bins from the
// largest down and a second scan finds the bin.  Writes s_digit and s_need (the
// rank inside that bin).  Needs 1 <= need <= the histogram's total.
template <int NB>
__device__ __forceinline__ void find_digit(const uint32_t* hist, uint32_t need, int lane, uint32_t* s_digit,
                                           uint32_t* s_need) {
    constexpr int PER = NB / 64;
    static_assert(PER >= 1 && PER <= 64, "bins per lane");
    const uint32_t* h = hist + NB - PER * (lane + 1);  // this lane's bins, ascending
    uint32_t tot = 0;
#pragma unroll 8
    for (int r = 0; r < PER; ++r) tot += h[r];
    const uint32_t above = wave_incl_sum(tot) - tot;  // elements with a larger digit
    const int L = (int)__builtin_ctzll(__ballot(above < need && above + tot >= need));
    const uint32_t above_L = __shfl(above, L, 64);
    const int bin = NB - PER * (L + 1) + (PER - 1 - lane);  // lane r < PER: L's bins, largest first
    const uint32_t c = lane < PER ? hist[bin] : 0u;
    const uint32_t ci = wave_incl_sum(c);
    if (lane == (int)__builtin_ctzll(__ballot(lane < PER && above_L + ci >= need))) {
        *s_digit = (uint32_t)bin;
        *s_need = need - (above_L + ci - c);
    }
}

// Top-k for C <= TH * EPT held in LDS (more than 8 candidates per thread).  Scores and candidate indices are staged
// with coalesced 16-byte loads; each thread then owns EPT consecutive candidates.
// Exact radix select with 11-bit digits taken from the top of the occupied
// [min, max] key range, then an ordered compaction (ascending key index).
template <int TH, int EPT, bool kAttend>
__global__ __launch_bounds__(TH) void topk_lds_kernel(RetrieveArgs a) {
    constexpr int kWaves = TH / 64;
    constexpr int kCap = TH * EPT;
    constexpr int kNB = 2048;
    // Up to 16 keys per thread the candidate indices are staged in LDS too (the
    // winners then read them without a global round trip); beyond that they are
    // read back from global memory for the k winners only.
    constexpr bool kStageIdx = EPT <= 16;
    // One LDS area: region A = staged keys (+ indices), region B = two histograms.
    // With kAttend the winners list reuses B once the histograms are done, and
    // the attention's per-slot state reuses A once the winners are out.
    constexpr size_t kA0 = (size_t)kCap * 4 * (kStageIdx ? 2 : 1);
    constexpr size_t kA = kAttend && kA0 < sizeof(AttendScratch) ? sizeof(AttendScratch) : kA0;
    constexpr size_t kBytes = kA + 2 * kNB * 4;
    static_assert(!kAttend || 2 * kNB * 4 >= kMaxAttendRows * 4, "the attention list fits in region B");
    __shared__ __align__(16) unsigned char s_raw[kBytes];
    uint32_t* s_key = reinterpret_cast<uint32_t*>(s_raw);
    int32_t* s_idx = reinterpret_cast<int32_t*>(s_raw + (size_t)kCap * 4);
    uint32_t (*s_hist)[kNB] = reinterpret_cast<uint32_t (*)[kNB]>(s_raw + kA);
    int32_t* s_win = reinterpret_cast<int32_t*>(s_raw + kA);
    __shared__ uint32_t s_w[kWaves];
    __shared__ uint32_t s_mm[2][kWaves];
    __shared__ uint32_t s_digit, s_need, s_nsmall;
    __shared__ uint32_t s_small[64];
    // With kAttend the winners' estimates wait here until the attention is done.
    __shared__ float s_wsc[kAttend ? PARISKV_MAX_TOPK : 1];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // This block's list: part blk % tk_parts of row blk / tk_parts (see RetrieveArgs).
    const int64_t blk = blockIdx.x;
    const int64_t row = blk / a.tk_parts;
    const int64_t off = (blk % a.tk_parts) * (int64_t)a.tk_part_len;
    const int C = (int)min((int64_t)a.tk_part_len, a.tk_c - off);
    const int kk = min(a.top_k, C);
    const float* sc = a.tk_score + row * a.tk_stride + off;
    const int32_t* cand = a.tk_idx + row * a.tk_stride + off;
    if (tid == 0) s_nsmall = 0;

    // With kAttend, this thread's part of the query, requested first.
    const uint4 qv = kAttend ? attend_query_part(static_cast<const __half*>(a.q) + row * kD)
                             : make_uint4(0, 0, 0, 0);

    // Staging of the estimates as order-preserving keys (and of the candidate
    // indices): every load of the thread is issued before the first LDS store, and
    // the smallest and largest valid keys are reduced on the way.  The arrays start
    // 256-byte aligned, so 16-byte loads are taken when the row stride and the part's
    // offset are multiples of 4 (the list then starts 16-byte aligned); slots past
    // the list re-read the row's last 16 bytes and are masked.
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    if (((a.tk_stride | off) & 3) == 0) {
        constexpr int kIt = kCap / 4 / TH;
        const int nq = (int)((a.tk_stride - off) >> 2);
        float4 f[kIt];
        int4 ix[kIt];
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int p4 = min(tid + it * TH, nq - 1);
            f[it] = reinterpret_cast<const float4*>(sc)[p4];
            if (kStageIdx) ix[it] = reinterpret_cast<const int4*>(cand)[p4];
        }
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int p = 4 * (tid + it * TH);
            const float fq[4] = {f[it].x, f[it].y, f[it].z, f[it].w};
            uint32_t k4[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                k4[q] = p + q < C ? order_key(fq[q]) : 0u;  // valid keys are all > 0
                if (k4[q] != 0u) { kmin = min(kmin, k4[q]); kmax = max(kmax, k4[q]); }
            }
            reinterpret_cast<uint4*>(s_key)[tid + it * TH] = make_uint4(k4[0], k4[1], k4[2], k4[3]);
            if (kStageIdx)
                reinterpret_cast<int4*>(s_idx)[tid + it * TH] =
                    make_int4(p < C ? ix[it].x : -1, p + 1 < C ? ix[it].y : -1, p + 2 < C ? ix[it].z : -1,
                              p + 3 < C ? ix[it].w : -1);
        }
    } else {
        for (int p = tid; p < kCap; p += TH) {
            const uint32_t k1 = p < C ? order_key(sc[p]) : 0u;
            if (k1 != 0u) { kmin = min(kmin, k1); kmax = max(kmax, k1); }
            s_key[p] = k1;
            if (kStageIdx) s_idx[p] = p < C ? cand[p] : -1;
        }
    }
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if (lane == 0) { s_mm[0][wave] = kmin; s_mm[1][wave] = kmax; }
    for (int i = tid; i < 2 * kNB; i += TH) (&s_hist[0][0])[i] = 0;
    __syncthreads();

    // Each thread then owns EPT consecutive candidates.
    uint32_t key[EPT];
#pragma unroll
    for (int e4 = 0; e4 < EPT / 4; ++e4) {
        const uint4 kv = reinterpret_cast<const uint4*>(s_key)[tid * (EPT / 4) + e4];
        key[4 * e4] = kv.x; key[4 * e4 + 1] = kv.y; key[4 * e4 + 2] = kv.z; key[4 * e4 + 3] = kv.w;
    }
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        kmin = min(kmin, s_mm[0][w]);
        kmax = max(kmax, s_mm[1][w]);
    }

    // Pass 0: 2048 bins linear in the score over [min, max].  The float bit
    // patterns of the scores are concentrated in few sign/exponent prefixes, so
    // value-linear bins spread the counts (and the atomics) far better.  The bin
    // index is a non-decreasing function of the score, so the keys of a higher
    // bin are all larger.
    const float fmin = key_float(kmin), fmax = key_float(kmax);
    const float frange = fmax - fmin;
    float inv = frange > 0.0f ? (float)kNB / frange : 0.0f;
    if (!(inv < 1e30f)) inv = 0.0f;  // a range that under- or overflows: one bin
    auto bin_of = [&](uint32_t k) -> uint32_t {
        return (uint32_t)fminf((float)(kNB - 1), (key_float(k) - fmin) * inv);
    };
#pragma unroll
    for (int e = 0; e < EPT; ++e)
        if (key[e] != 0u) atomicAdd(&s_hist[0][bin_of(key[e])], 1u);
    __syncthreads();
    if (wave == 0) find_digit<kNB>(s_hist[0], (uint32_t)kk, lane, &s_digit, &s_need);
    __syncthreads();
    const uint32_t bsel = s_digit;       // bin holding the kk-th largest key
    uint32_t need = s_need;              // its rank (from the top) inside that bin
    const uint32_t in_bin = s_hist[0][bsel];
    uint32_t T, quota;
    if (in_bin <= 64) {
        // Few keys in the bin: gather them and rank them by brute force in one wave.
#pragma unroll
        for (int e = 0; e < EPT; ++e)
            if (key[e] != 0u && bin_of(key[e]) == bsel) s_small[atomicAdd(&s_nsmall, 1u)] = key[e];
        __syncthreads();
        if (wave == 0) {
            const uint32_t kl = lane < (int)in_bin ? s_small[lane] : 0u;
            uint32_t gt = 0, eq = 0;
            for (uint32_t j = 0; j < in_bin; ++j) {
                const uint32_t kj = s_small[j];
                gt += kj > kl ? 1u : 0u;
                eq += kj == kl ? 1u : 0u;
            }
            const bool hit = lane < (int)in_bin && gt < need && need <= gt + eq;
            const uint64_t hits = __ballot(hit);
            if (hit && lane == __builtin_ctzll(hits)) {
                s_digit = kl;
                s_need = need - gt;
            }
        }
        __syncthreads();
        T = s_digit;
        quota = s_need;
    } else {
        // Exact radix select on the full key restricted to the bin: 11, 11, 10 bits.
        uint32_t prefix = 0, mask = 0;
        int shift = 21;
#pragma unroll 1
        for (int pass = 1; pass <= 3; ++pass) {
            uint32_t* hist = s_hist[pass & 1];
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                if (key[e] != 0u && (key[e] & mask) == prefix && bin_of(key[e]) == bsel)
                    atomicAdd(&hist[(key[e] >> shift) & (kNB - 1)], 1u);
            __syncthreads();
            if (wave == 0) find_digit<kNB>(hist, need, lane, &s_digit, &s_need);
            // The other buffer was read in the previous pass; clear it for the next one.
            for (int i = tid; i < kNB; i += TH) s_hist[(pass + 1) & 1][i] = 0;
            __syncthreads();
            prefix |= s_digit << shift;
            mask |= (uint32_t)(kNB - 1) << shift;
            need = s_need;
            shift = shift >= 11 ? shift - 11 : 0;
        }
        T = prefix;     // the kk-th largest key value
        quota = need;   // how many keys equal to T are taken (lowest indices)
    }

    // Ordered compaction: an element's output slot is (#keys > T before it) +
    // min(#keys == T before it, quota), which lists the winners by ascending index.
    uint32_t ng = 0, ne = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        ng += (key[e] > T) ? 1u : 0u;
        ne += (key[e] == T && key[e] != 0u) ? 1u : 0u;
    }
    const uint32_t mine = ng | (ne << 16);
    // This thread's candidate indices, read before they are needed.
    int32_t widx[EPT];
    if (kStageIdx) {
#pragma unroll
        for (int e4 = 0; e4 < EPT / 4; ++e4) {
            const int4 v4 = reinterpret_cast<const int4*>(s_idx)[tid * (EPT / 4) + e4];
            widx[4 * e4] = v4.x; widx[4 * e4 + 1] = v4.y; widx[4 * e4 + 2] = v4.z; widx[4 * e4 + 3] = v4.w;
        }
    }
    const uint32_t incl = wave_incl_sum(mine);
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    uint32_t pre = incl - mine;
#pragma unroll
    for (int w = 0; w < kWaves; ++w)
        if (w < wave) pre += s_w[w];
    uint32_t gb = pre & 0xffffu, eb = pre >> 16;
    int32_t* oi = a.tk_out_idx + blk * a.top_k;
    float* os = a.tk_out_score ? a.tk_out_score + blk * a.top_k : nullptr;
    // With kAttend the attention list in region B is Sink rows, then Local +
    // Update Buffer rows (nd in all), then the winners at their cache rows
    // (retr_begin + key; the host checked they stay below dense_begin), and the
    // outputs are written after the attention, so that its first loads do not
    // wait behind these stores.
    const int nd = kAttend ? (int)a.win.dense_rows() : 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        uint32_t p = 0xffffffffu;
        if (key[e] > T) {
            p = gb + min(eb, quota);
            ++gb;
        } else if (key[e] == T && key[e] != 0u) {
            if (eb < quota) p = gb + eb;
            ++eb;
        }
        if (p < (uint32_t)kk) {
            const int32_t win = kStageIdx ? widx[e] : cand[tid * EPT + e];
            if (kAttend) {
                s_win[nd + p] = (int32_t)(a.win.retr_begin + win);
                s_wsc[p] = key_float(key[e]);
            } else {
                oi[p] = win;
                if (os) os[p] = key_float(key[e]);
            }
        }
    }
    if (!kAttend) {
        for (int r = kk + tid; r < a.top_k; r += TH) {
            oi[r] = -1;
            if (os) os[r] = -__builtin_huge_valf();
        }
    }
    if (kAttend) {
        // Attention over the dense rows and the kk winners (Eqs. approx_weight,
        // approx_output), from LDS.  Region B is free once the compaction runs.
        for (int r = tid; r < nd; r += TH) s_win[r] = a.win.dense_entry(r);
        __syncthreads();
        const int seq = (int)(row / a.hq);
        const int h = (int)(row % a.hq);
        const int64_t kvrow0 = ((int64_t)seq * a.hkv + h / a.g) * a.kv_capacity;
        const bool wc = a.win.win_capacity > 0;
        const int64_t wrow0 = wc ? ((int64_t)seq * a.hkv + h / a.g) * a.win.win_capacity : kvrow0;
        attend_row(qv, static_cast<const __half*>(a.K) + kvrow0 * kD,
                   static_cast<const __half*>(a.V) + kvrow0 * kD, a.kv_capacity,
                   static_cast<const __half*>(wc ? a.Kw : a.K) + wrow0 * kD,
                   static_cast<const __half*>(wc ? a.Vw : a.V) + wrow0 * kD, a.win.win_capacity,
                   s_win, nd + kk, a.scale,
                   a.attn_out + row * kD, *reinterpret_cast<AttendScratch*>(s_raw));
        // The winners in ascending key index, then the padding.
        for (int r = tid; r < a.top_k; r += TH) {
            const bool w = r < kk;
            oi[r] = w ? (int32_t)((int64_t)s_win[nd + r] - a.win.retr_begin) : -1;
            if (os) os[r] = w ? s_wsc[r] : -__builtin_huge_valf();
        }
    }
}

// Top-k for C <= TH * EPT <= 8192 candidates, held in registers: thread t owns the 4-candidate
// groups at positions 4 (t + j TH) .. 4 (t + j TH) + 3 for j < EPT / 4, read with
// coalesced 16-byte loads.  Exact selection on order-preserving uint32 keys: one
// histogram pass with 2 TH bins linear in the estimate over [min, max], then the
// boundary bin ranked by brute force (at most 64 keys) or by radix passes of log2(2 TH)
// bits restricted to it; ties at the k-th key taken in candidate order.  An ordered
// compaction (a block scan per group of positions) then lists the winners in
// ascending key index without a sort.
template <int TH, int EPT, bool kAttend>
__global__ __launch_bounds__(TH) void topk_reg_kernel(RetrieveArgs a) {
    constexpr int kWaves = TH / 64;
    constexpr int kIt = EPT / 4;   // 4-candidate groups per thread
    constexpr int kNB = 2 * TH;    // bins of the histogram
    constexpr int kDigit = TH == 1024 ? 11 : TH == 512 ? 10 : 9;  // log2 kNB
    static_assert(kNB == 1 << kDigit, "digit width");
    // LDS: region A = the attention's per-slot state (kAttend), region B = two
    // histograms, whose place the attention list takes once they are done.
    constexpr size_t kA = kAttend ? sizeof(AttendScratch) : 0;
    constexpr size_t kBytes = kA + 2 * kNB * 4;
    static_assert(!kAttend || 2 * kNB >= kAtRows<TH>, "the attention list fits in region B");
    static_assert(EPT % 4 == 0 && EPT <= 8, "whole 4-candidate groups, few enough to stay in registers");
    __shared__ __align__(16) unsigned char s_raw[kBytes];
    uint32_t (*s_hist)[kNB] = reinterpret_cast<uint32_t (*)[kNB]>(s_raw + kA);
    int32_t* s_win = reinterpret_cast<int32_t*>(s_raw + kA);
    __shared__ uint32_t s_w[kIt][kWaves];
    __shared__ uint32_t s_mm[2][kWaves];
    __shared__ uint32_t s_digit, s_need, s_nsmall;
    __shared__ uint32_t s_small[64];
    // With kAttend the winners' estimates wait here until the attention is done.
    __shared__ float s_wsc[kAttend ? (kAtRows<TH> < PARISKV_MAX_TOPK ? kAtRows<TH> : PARISKV_MAX_TOPK) : 1];
    __shared__ int32_t s_dump[kAttend ? TH : 1];  // a word per thread for non-winners' stores
    // With kAttend: K/V rows of up to kPf sure winners per wave, requested as soon as
    // the boundary bin is known (see below), and their cache rows.
    constexpr int kPf = 12;
    __shared__ uint4 s_prow[kAttend ? kWaves * kPf * 32 : 1];
    __shared__ __align__(16) int32_t s_pfrow[kAttend ? kWaves : 1][kPf];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // This block's list: part blk % tk_parts of row blk / tk_parts (see RetrieveArgs).
    const int64_t blk = blockIdx.x;
    const int64_t row = blk / a.tk_parts;
    const int64_t off = (blk % a.tk_parts) * (int64_t)a.tk_part_len;
    const int C = (int)min((int64_t)a.tk_part_len, a.tk_c - off);
    const int kk = min(a.top_k, C);
    const float* sc = a.tk_score + row * a.tk_stride + off;
    const int32_t* cand = a.tk_idx + row * a.tk_stride + off;
    if (tid == 0) s_nsmall = 0;

    uint32_t kmin = 0xffffffffu, kmax = 0u;

    // The estimates as keys (0 past the list; valid keys are all > 0) and the
    // candidate indices.  The arrays start 256-byte aligned, so 16-byte loads are
    // taken when the row stride and the part's offset are multiples of 4 (the list
    // then starts 16-byte aligned); groups past the list re-read the row's last 16
    // bytes and are masked.  Otherwise every candidate is read on its own.
    uint32_t key[EPT];
    int32_t widx[EPT];
    if (((a.tk_stride | off) & 3) == 0) {
        const int nq = (int)((a.tk_stride - off) >> 2);
        float4 f[kIt];
        int4 ix[kIt];
#pragma unroll
        for (int it = 0; it < kIt; ++it)
            f[it] = reinterpret_cast<const float4*>(sc)[min(tid + it * TH, nq - 1)];
#pragma unroll
        for (int it = 0; it < kIt; ++it)
            ix[it] = reinterpret_cast<const int4*>(cand)[min(tid + it * TH, nq - 1)];
        // The estimates are needed first (the indices only after the digit search):
        // an empty asm that reads them keeps each 16-byte load whole and makes the
        // one wait here cover just them.
#pragma unroll
        for (int it = 0; it < kIt; ++it) asm volatile("" ::"v"(f[it].x), "v"(f[it].y), "v"(f[it].z), "v"(f[it].w));
#pragma unroll
        for (int it = 0; it < kIt; ++it) {
            const int p = 4 * (tid + it * TH);
            key[4 * it] = p < C ? order_key(f[it].x) : 0u;
            key[4 * it + 1] = p + 1 < C ? order_key(f[it].y) : 0u;
            key[4 * it + 2] = p + 2 < C ? order_key(f[it].z) : 0u;
            key[4 * it + 3] = p + 3 < C ? order_key(f[it].w) : 0u;
            widx[4 * it] = ix[it].x;
            widx[4 * it + 1] = ix[it].y;
            widx[4 * it + 2] = ix[it].z;
            widx[4 * it + 3] = ix[it].w;
        }
    } else {
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int p = 4 * (tid + (e >> 2) * TH) + (e & 3);
            key[e] = p < C ? order_key(sc[p]) : 0u;
            widx[e] = p < C ? cand[p] : -1;
        }
    }
    // With kAttend, this thread's part of the query (needed only by the attention).
    const uint4 qv = kAttend ? attend_query_part(static_cast<const __half*>(a.q) + row * kD)
                             : make_uint4(0, 0, 0, 0);
    for (int i = tid; i < 2 * kNB; i += TH) (&s_hist[0][0])[i] = 0;
#pragma unroll
    for (int e = 0; e < EPT; ++e)
        if (key[e] != 0u) { kmin = min(kmin, key[e]); kmax = max(kmax, key[e]); }
    kmin = wave_min_u32(kmin);
    kmax = wave_max_u32(kmax);
    if (lane == 0) { s_mm[0][wave] = kmin; s_mm[1][wave] = kmax; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        kmin = min(kmin, s_mm[0][w]);
        kmax = max(kmax, s_mm[1][w]);
    }

    // Pass 0: kNB bins linear in the score over [min, max].  The float bit
    // patterns of the scores are concentrated in few sign/exponent prefixes, so
    // value-linear bins spread the counts (and the atomics) far better.  The bin
    // index is a non-decreasing function of the score, so the keys of a higher
    // bin are all larger.
    const float fmin = key_float(kmin), fmax = key_float(kmax);
    const float frange = fmax - fmin;
    float inv = frange > 0.0f ? (float)kNB / frange : 0.0f;
    if (!(inv < 1e30f)) inv = 0.0f;  // a range that under- or overflows: one bin
    auto bin_of = [&](uint32_t k) -> uint32_t {
        return (uint32_t)fminf((float)(kNB - 1), (key_float(k) - fmin) * inv);
    };
#pragma unroll
    for (int e = 0; e < EPT; ++e)
        if (key[e] != 0u) atomicAdd(&s_hist[0][bin_of(key[e])], 1u);
    __syncthreads();
    if (wave == 0) find_digit<kNB>(s_hist[0], (uint32_t)kk, lane, &s_digit, &s_need);
    __syncthreads();
    const uint32_t bsel = s_digit;       // bin holding the kk-th largest key
    uint32_t need = s_need;              // its rank (from the top) inside that bin
    const uint32_t in_bin = s_hist[0][bsel];
    const int32_t retr0 = (int32_t)a.win.retr_begin;  // below kv_capacity <= 2^30 - 1 (host-checked)
    // KV group of the row: row = seq hq + h with hq = hkv g, so seq hkv + h / g = row / g.
    const int64_t kvrow0 = kAttend ? (int64_t)((int)row / a.g) * a.kv_capacity : 0;

    // With kAttend: a key in a bin above bsel wins whatever the rest of the selection
    // finds.  Each lane offers the first such key among its first kPfKeys, and each
    // wave requests the K/V rows of the first kPf lanes that offer one into registers
    // now, so that these gathers overlap the rest of the selection (a barrier does not
    // wait for them); they go to LDS just before the attention, which reads them from
    // there (listed as -2 - LDS row).  The bin test is the bin's own arithmetic: the
    // bin is the truncated (f - fmin) inv, so bin > bsel iff that product >= bsel + 1.
    constexpr int kPfKeys = EPT < 4 ? EPT : 4;
    static_assert(kPf == 12, "six row loads per lane, in named registers");
    uint4 pf0 = make_uint4(0, 0, 0, 0), pf1 = pf0, pf2 = pf0, pf3 = pf0, pf4 = pf0, pf5 = pf0;
    int npf = 0, pf_e = -1, pf_slot = 0;  // this lane's held key (index e, or -1) and its LDS row
    if (kAttend) {
        const float edge = (float)(bsel + 1);
        const uint32_t cap = (uint32_t)a.kv_capacity;
        int e1 = -1;
        int32_t r1 = 0;
#pragma unroll
        for (int e = kPfKeys - 1; e >= 0; --e) {
            const int32_t rowi = retr0 + widx[e];
            const bool sure = key[e] != 0u && (key_float(key[e]) - fmin) * inv >= edge && (uint32_t)rowi < cap;
            e1 = sure ? e : e1;
            r1 = sure ? rowi : r1;
        }
        const uint64_t m = __ballot(e1 >= 0);
        const int pos = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        npf = min(kPf, (int)__popcll(m));
        if (e1 >= 0 && pos < kPf) {
            s_pfrow[wave][kPf / 2 * (pos & 1) + (pos >> 1)] = r1;
            pf_e = e1;
            pf_slot = wave * kPf + pos;
        }
        // The wave reads back its own LDS words (in order, no barrier needed).  Load u:
        // lanes 0-31 take row 2u (K in lanes 0-15, V in 16-31), lanes 32-63 row 2u + 1;
        // row w sits at word kPf/2 (w % 2) + w / 2, so a lane's ids are consecutive.
        // Loads 0 and 1 go out now, 2 and 3 before the compaction scan, 4 and 5 before
        // the winner list is built (more at once stalled the waves at issue).  The
        // loads are unconditional: a missing row reads the group's row 0 (there is
        // one, kv_capacity >= 1 is checked on the host) and is not used; branches
        // around them made the compiler wait for their data early.
        const uint4* kv = reinterpret_cast<const uint4*>(static_cast<const __half*>((lane & 16) ? a.V : a.K) +
                                                         kvrow0 * kD) + (lane & 15);
        const int hi = lane >> 5;
        const int32_t* idp = &s_pfrow[wave][kPf / 2 * hi];
        pf0 = kv[(int64_t)(hi < npf ? idp[0] : 0) * (kD / 8)];
        pf1 = kv[(int64_t)(2 + hi < npf ? idp[1] : 0) * (kD / 8)];
    }
    uint32_t T, quota;
    if (in_bin <= 64) {
        // Few keys in the bin: gather them, then every wave ranks them by brute force
        // (the same result in each, so no second barrier hands it out).
#pragma unroll
        for (int e = 0; e < EPT; ++e)
            if (key[e] != 0u && bin_of(key[e]) == bsel) s_small[atomicAdd(&s_nsmall, 1u)] = key[e];
        __syncthreads();
        const uint32_t kl = lane < (int)in_bin ? s_small[lane] : 0u;
        uint32_t gt = 0, eq = 0;
        for (uint32_t j = 0; j < in_bin; ++j) {
            const uint32_t kj = s_small[j];
            gt += kj > kl ? 1u : 0u;
            eq += kj == kl ? 1u : 0u;
        }
        const bool hit = lane < (int)in_bin && gt < need && need <= gt + eq;
        const int first = (int)__builtin_ctzll(__ballot(hit));  // some key of the bin has rank need
        T = (uint32_t)__builtin_amdgcn_readlane((int)kl, first);
        quota = need - (uint32_t)__builtin_amdgcn_readlane((int)gt, first);
    } else {
        // Exact radix select on the full key restricted to the bin: kDigit bits a pass (the
        // last one repeats bits that are already fixed).
        uint32_t prefix = 0, mask = 0;
        int shift = 32 - kDigit;
#pragma unroll 1
        for (int pass = 1; pass <= (32 + kDigit - 1) / kDigit; ++pass) {
            uint32_t* hist = s_hist[pass & 1];
#pragma unroll
            for (int e = 0; e < EPT; ++e)
                if (key[e] != 0u && (key[e] & mask) == prefix && bin_of(key[e]) == bsel)
                    atomicAdd(&hist[(key[e] >> shift) & (kNB - 1)], 1u);
            __syncthreads();
            if (wave == 0) find_digit<kNB>(hist, need, lane, &s_digit, &s_need);
            // The other buffer was read in the previous pass; clear it for the next one.
            for (int i = tid; i < kNB; i += TH) s_hist[(pass + 1) & 1][i] = 0;
            __syncthreads();
            prefix |= s_digit << shift;
            mask |= (uint32_t)(kNB - 1) << shift;
            need = s_need;
            shift = shift >= kDigit ? shift - kDigit : 0;
        }
        T = prefix;     // the kk-th largest key value
        quota = need;   // how many keys equal to T are taken (lowest indices)
    }

    if constexpr (kAttend) {
        // Prefetch loads 2 and 3 (see above).
        const uint4* kv = reinterpret_cast<const uint4*>(static_cast<const __half*>((lane & 16) ? a.V : a.K) +
                                                         kvrow0 * kD) + (lane & 15);
        const int hi = lane >> 5;
        const int2 t = *reinterpret_cast<const int2*>(&s_pfrow[wave][kPf / 2 * hi + 2]);
        pf2 = kv[(int64_t)(4 + hi < npf ? t.x : 0) * (kD / 8)];
        pf3 = kv[(int64_t)(6 + hi < npf ? t.y : 0) * (kD / 8)];
    }
    // Ordered compaction: an element's output slot is (#keys > T before it) +
    // min(#keys == T before it, quota), which lists the winners by ascending index.
    // Positions run group by group (j), thread by thread inside a group, so the
    // counts before an element are the earlier groups' totals plus a block scan of
    // this group (counts > T in the low 16 bits, == T in the high 16).
    uint32_t pre[kIt];
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        uint32_t mine = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t k1 = key[4 * it + q];
            mine += (k1 > T) ? 1u : (k1 == T && k1 != 0u) ? 0x10000u : 0u;
        }
        const uint32_t incl = wave_incl_sum(mine);
        if (lane == 63) s_w[it][wave] = incl;
        pre[it] = incl - mine;
    }
    __syncthreads();
    // The waves' totals of each group: lane w < kWaves takes wave w's, one wave scan, and
    // the prefix before this wave read from lane wave - 1 (the group total from the last).
    static_assert(kWaves <= 64, "one lane per wave in the scan of the wave totals");
    uint32_t before_groups = 0;
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        const uint32_t x = lane < kWaves ? s_w[it][lane] : 0u;
        const uint32_t ix = wave_incl_sum(x);
        const int wv = __builtin_amdgcn_readfirstlane(wave);
        const uint32_t earlier = wv > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)ix, wv - 1) : 0u;
        const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)ix, kWaves - 1);
        pre[it] += before_groups + earlier;
        before_groups += tot;
    }
    int32_t* oi = a.tk_out_idx + blk * a.top_k;
    float* os = a.tk_out_score ? a.tk_out_score + blk * a.top_k : nullptr;
    // With kAttend the attention list in region B is Sink rows, then Local +
    // Update Buffer rows (nd in all), then the winners at their cache rows
    // (retr_begin + key; the host checked they stay below dense_begin), and the
    // outputs are written after the attention, so that its first loads do not
    // wait behind these stores.
    const int nd = kAttend ? (int)a.win.dense_rows() : 0;
    if constexpr (kAttend) {
        // Prefetch loads 4 and 5 (see above).
        const uint4* kv = reinterpret_cast<const uint4*>(static_cast<const __half*>((lane & 16) ? a.V : a.K) +
                                                         kvrow0 * kD) + (lane & 15);
        const int hi = lane >> 5;
        const int2 t = *reinterpret_cast<const int2*>(&s_pfrow[wave][kPf / 2 * hi + 4]);
        pf4 = kv[(int64_t)(8 + hi < npf ? t.x : 0) * (kD / 8)];
        pf5 = kv[(int64_t)(10 + hi < npf ? t.y : 0) * (kD / 8)];
    }
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
        uint32_t gb = pre[it] & 0xffffu, eb = pre[it] >> 16;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = 4 * it + q;
            const bool gt = key[e] > T;
            const bool eq = key[e] == T && key[e] != 0u;
            const uint32_t p = gt ? gb + min(eb, quota) : (eq && eb < quota) ? gb + eb : 0xffffffffu;
            gb += gt ? 1u : 0u;
            eb += eq ? 1u : 0u;
            if (kAttend) {
                // Branch-free: a key that does not win writes this thread's own dump word.
                const bool w = p < (uint32_t)kk;
                int32_t* dw = w ? &s_win[nd + p] : &s_dump[tid];
                float* ds = w ? &s_wsc[p] : reinterpret_cast<float*>(&s_dump[tid]);
                *dw = e == pf_e ? -2 - pf_slot : retr0 + widx[e];
                *ds = key_float(key[e]);
            } else if (p < (uint32_t)kk) {
                oi[p] = widx[e];
                if (os) os[p] = key_float(key[e]);
            }
        }
    }
    if (!kAttend) {
        for (int r = kk + tid; r < a.top_k; r += TH) {
            oi[r] = -1;
            if (os) os[r] = -__builtin_huge_valf();
        }
    }
    if (kAttend) {
        // Attention over the dense rows and the kk winners (Eqs. approx_weight,
        // approx_output), from LDS.  Region B is free once the compaction runs.
        for (int r = tid; r < nd; r += TH) s_win[r] = a.win.dense_entry(r);
        {
            uint4* dst = s_prow + 32 * (wave * kPf + (lane >> 5)) + (lane & 31);
            const int hi = lane >> 5;
            // Unconditional: rows past npf are never listed, and a store on every
            // path keeps the compiler's view of the loads settled from here on.
            dst[0] = pf0;
            dst[2 * 32] = pf1;
            dst[4 * 32] = pf2;
            dst[6 * 32] = pf3;
            dst[8 * 32] = pf4;
            dst[10 * 32] = pf5;
        }
        __syncthreads();
        const bool wc = a.win.win_capacity > 0;
        const int64_t wrow0 = wc ? (int64_t)((int)row / a.g) * a.win.win_capacity : kvrow0;
        attend_row<TH>(qv, static_cast<const __half*>(a.K) + kvrow0 * kD,
                   static_cast<const __half*>(a.V) + kvrow0 * kD, a.kv_capacity,
                   static_cast<const __half*>(wc ? a.Kw : a.K) + wrow0 * kD,
                   static_cast<const __half*>(wc ? a.Vw : a.V) + wrow0 * kD, a.win.win_capacity,
                   s_win, nd + kk, a.scale,
                   a.attn_out + row * kD, *reinterpret_cast<AttendScratch*>(s_raw), s_prow);
        // The winners in ascending key index (a held row's from its prefetch record),
        // then the padding.
        for (int r = tid; r < a.top_k; r += TH) {
            const bool w = r < kk;
            int32_t v = w ? s_win[nd + r] : 0;
            if (v <= -2) {
                const int slot = -2 - v, pos = slot % kPf;
                v = s_pfrow[slot / kPf][kPf / 2 * (pos & 1) + (pos >> 1)];
            }
            oi[r] = w ? (int32_t)((int64_t)v - a.win.retr_begin) : -1;
            if (os) os[r] = w ? s_wsc[r] : -__builtin_huge_valf();
        }
    }
}

__global__ void pad_outputs_kernel(int32_t* out_idx, float* out_score, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) {
        out_idx[i] = -1;
        if (out_score) out_score[i] = -__builtin_huge_valf();
    }
}

}  // namespace

hipError_t launch_compact_rerank(const RetrieveArgs& a, hipStream_t s) {
    const ProfEvents pe = prof_begin("compact_rerank");
    const dim3 grid((unsigned)a.n_chunks, (unsigned)(a.batch * a.hq));
    const int64_t blocks = (int64_t)grid.x * grid.y;
#define PARISKV_RERANK(TH, FOLD) \
    hipExtLaunchKernelGGL((compact_rerank_kernel<TH, FOLD>), grid, dim3(TH), 0, s, pe.start, pe.stop, 0, a)
    const bool fold = fold_threshold(a);
    if (blocks <= kRrWidestGrid)
        fold ? PARISKV_RERANK(512, true) : PARISKV_RERANK(512, false);
    else if (fold)
        PARISKV_RERANK(256, true);
    else if (blocks <= kRrWideGrid)
        PARISKV_RERANK(256, false);
    else
        PARISKV_RERANK(128, false);
#undef PARISKV_RERANK
    return hipGetLastError();
}

hipError_t launch_topk(const RetrieveArgs& a0, hipStream_t s, bool attend, bool* fused) {
    RetrieveArgs a = a0;
    a.tk_score = a.cand_score;
    a.tk_idx = a.cand;
    a.tk_stride = a.n_cand;
    a.tk_c = a.c_eff;
    a.tk_parts = 1;
    a.tk_part_len = (int32_t)a.c_eff;
    a.tk_out_idx = a.out_idx;
    a.tk_out_score = a.out_score;
    const int64_t rows = (int64_t)a.batch * a.hq;
    if (a.topk_parts > 1) {
        // First pass: the k best of every 4096-candidate slice, in ascending key
        // index.  Every winner of the row is among its slice's k best (fewer than k
        // keys of its slice precede it), so the final pass over the slices' winners,
        // concatenated in slice order, selects the same keys in the same order.
        RetrieveArgs p = a;
        p.tk_parts = a.topk_parts;
        p.tk_part_len = kTopkPart;
        p.tk_out_idx = a.surv_idx;
        p.tk_out_score = a.surv_score;
        const ProfEvents pp = prof_begin("topk_part");
        hipExtLaunchKernelGGL((topk_reg_kernel<1024, 4, false>), dim3((unsigned)(rows * a.topk_parts)), dim3(1024),
                              0, s, pp.start, pp.stop, 0, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        a.tk_score = a.surv_score;
        a.tk_idx = a.surv_idx;
        a.tk_stride = (int64_t)a.topk_parts * a.top_k;
        // only the last slice can hold fewer than k candidates (kTopkPart >= k)
        const int64_t last = a.c_eff - (int64_t)(a.topk_parts - 1) * kTopkPart;
        a.tk_c = (int64_t)(a.topk_parts - 1) * a.top_k + (last < a.top_k ? last : a.top_k);
        a.tk_part_len = (int32_t)a.tk_c;
    }
    const dim3 grid((unsigned)rows);
    const int64_t C = a.tk_c;
    if (fused) *fused = attend;
    const ProfEvents pe = prof_begin(attend ? "topk_attend" : "topk");
#define PARISKV_TOPK_REG(TH, EPT)                                                                    \
    (attend ? hipExtLaunchKernelGGL((topk_reg_kernel<TH, EPT, true>), grid, dim3(TH), 0, s,           \
                                    pe.start, pe.stop, 0, a)                                          \
            : hipExtLaunchKernelGGL((topk_reg_kernel<TH, EPT, false>), grid, dim3(TH), 0, s,          \
                                    pe.start, pe.stop, 0, a))
#define PARISKV_TOPK_LDS(EPT)                                                                        \
    (attend ? hipExtLaunchKernelGGL((topk_lds_kernel<1024, EPT, true>), grid, dim3(1024), 0, s,       \
                                    pe.start, pe.stop, 0, a)                                          \
            : hipExtLaunchKernelGGL((topk_lds_kernel<1024, EPT, false>), grid, dim3(1024), 0, s,      \
                                    pe.start, pe.stop, 0, a))
    // The smallest block that holds the candidates in registers and the attended list in one
    // round, at 4 candidates per thread: fewer waves at every barrier, and 2 to 4 blocks a CU
    // where there are more rows than CUs (448 rows, C = 876, k = 100: 19.8 -> 11.1 us; 8 rows,
    // C = 512, k = 64: 9.9 -> 9.1).  8 per thread instead of twice the threads pays only with
    // more rows than CUs (512 rows, C = 2048, k = 256: 23.7 -> 17.3 us; 128 rows, C = 2855,
    // k = 256: 12.1 -> 12.7).
    const int64_t list = attend ? a.win.dense_rows() + a.top_k : 0;  // rows attended
    const int64_t per = rows > kManyRows ? 8 : 4;
    if (C <= 256 * 4 && list <= kAtRows<256>)
        PARISKV_TOPK_REG(256, 4);
    else if (C <= 256 * per && list <= kAtRows<256>)
        PARISKV_TOPK_REG(256, 8);
    else if (C <= 512 * 4 && list <= kAtRows<512>)
        PARISKV_TOPK_REG(512, 4);
    else if (C <= 512 * per && list <= kAtRows<512>)
        PARISKV_TOPK_REG(512, 8);
    else if (C <= 1024 * 4)
        PARISKV_TOPK_REG(1024, 4);
    else if (C <= 1024 * 8)
        PARISKV_TOPK_REG(1024, 8);
    else if (C <= 1024 * 16)
        PARISKV_TOPK_LDS(16);
    else
        PARISKV_TOPK_LDS(32);  // C <= 32768: at most 16 slices x 2048 winners after a first pass
#undef PARISKV_TOPK_LDS
#undef PARISKV_TOPK_REG
    return hipGetLastError();
}

hipError_t launch_pad_outputs(const RetrieveArgs& a, hipStream_t s) {
    const int64_t count = (int64_t)a.batch * a.hq * a.top_k;
    const ProfEvents pe = prof_begin("pad_outputs");
    hipExtLaunchKernelGGL(pad_outputs_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, pe.start, pe.stop, 0,
                       a.out_idx, a.out_score, count);
    return hipGetLastError();
}

}  // namespace pariskv
