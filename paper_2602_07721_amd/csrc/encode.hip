// Key summarisation kernel: centroid ids, 4-bit direction codes, weights W
// and cluster counts (Sec. "Prefill Phase" steps (1)-(3), Eqs. dir_assign,
// rsqip_sign_mag_code, alpha_def, scaling_factor; Alg. 1 encode loop).
//
// Arithmetic (bit-exact by construction):
//   y = H (s (.) k) in float64.  float16 inputs are integer multiples of 2^-24
//   below 2^16, so every partial sum of at most 128 of them is an integer
//   multiple of 2^-24 below 2^47 and is exact in float64 in any order.  y is
//   sqrt(D) ||k|| times the rotated, normalised key, a positive factor that
//   every decision below is invariant to.
//   id bit j    = [y_j < 0]                      (argmax over {+-1/sqrt m}^m),
//                 stored as id_slot(id); counts are kept by the id itself
//   Y_j         = fl(y_j * y_j)
//   S_b         = ((Y0+Y1)+(Y2+Y3))+((Y4+Y5)+(Y6+Y7))
//   t_j         = #{t : Y_j >= fl(tau_t^2 * S_b)}   (|u_j| >= tau_t), 0 if S_b = 0
//   A_b         = same tree over fl(a[t_j] * |y_j|) (= sqrt(S_b) alpha_b)
//   W_b         = float(fl(S_b / A_b))              (= sqrt(D) w_b), 0 if S_b = 0
// Every float64 operation is an explicit round-to-nearest multiply or add
// (no contraction), so the results do not depend on the compiler.
//
// Transform.  H (s (.) k) is a 128 x 128 matrix of +-1 times the keys: 32 inputs at a time
// on matrix instructions (16x16x32, float16 in, float32 sums), the four sums of a coordinate
// combined in float64.  The products are made exact by splitting every key coordinate
// x = hi + lo: lo = x less its rounding to a multiple of 2^-6 when |x| < 8, else 0.  So
// |lo| <= 2^-7 in units of 2^-24, and 32 of them sum below 2^24 units; |x| < 4096 gives hi in
// units of 2^-7 and a sum of at most 2^24 of them.  Every partial sum of either part is then
// exact in float32 in any order, and so are hi + lo and the rest in float64.  lo is carried
// as 2^11 lo, a normal float16 number.  A tile of 16 keys whose sums of squares may come from
// a coordinate of 4096 or more (or are not finite) is done again with those coordinates as a third
// operand: multiples of 4 below 2^16, whose sums are exact too.
//
// Mapping: a wave takes 16 keys; lane 16 g + r holds coordinates [32 g, 32 g + 32) of
// key r, i.e. subspaces 4g..4g+3, before and after the transform.  Coordinate 8 s +
// 2 j + e (s < 16, j < 4, e < 2): a matrix step multiplies the 32 inputs of one j,
// which lie in the 4 loaded uint4 as component j of each, so no data moves before
// the product; output tile T holds (s, e) rows chosen so that lane group g gets
// subspaces 4g + 2T, 4g + 2T + 1, and the 4 steps of a coordinate meet in one lane.
//
// Bins.  t_j compares Y_j with at most one of the 7 products tau_t^2 S_b: u = |y_j| /
// sqrt(S_b) in float32 (error below 2^-20) falls in one of 64 buckets of [0, 1]; the
// bucket's entry names the bins surely passed and the one threshold that is not decided,
// which is then compared in float64 as defined above.  Buckets are far narrower than
// the gaps between thresholds (0.08 at least).
//
// What bounds it: vector issue.  A 16-key tile is about 830 vector instructions and 16
// matrix instructions (1665 vector ones with the transform as float64 butterflies and 7
// compares per coordinate); the vector unit is busy 3/4 of the time with 3 waves per SIMD.
// Measured: 8 x 131072 keys 238 -> 134 us, 24 x 10007 keys 177 -> 38 us, most of
// the second from blocks sized to fill the chip (launch_encode).  Two waves per SIMD, with
// the matrix operands held in registers, took 14% longer; summing all 128 inputs on the matrix
// unit (64 instructions, no float64 stages) 2% longer.  With a coordinate of 5000 in every tile
// 238 -> 172 us, in 1 of 6 tiles 168 (340 and 172 when such a tile went through the
// butterflies, a function of their own, after the matrix path).
//
// Each lane counts its 4 ids in an LDS histogram per block, added to global memory
// once per block; records go through LDS so that a wave stores whole lines.

#include <hip/hip_fp16.h>

#include "internal.hpp"

// The decision path is specified operation by operation; never fuse.
#pragma clang fp contract(off)

namespace pariskv {

namespace {

constexpr int kThreads = 256;
constexpr int kTile = 16;                           // keys per wave and iteration
constexpr int kWaves = kThreads / 64;
constexpr int kKeysPerIter = kWaves * kTile;
constexpr int kBuckets = 64;                        // of u in [0, 1]; u may round up past 1: more entries
constexpr int kBucketLut = 2 * kBuckets;            // (a power of two, so that a mask bounds the index)
constexpr int kFrags = 8;                           // matrix operands: 2 tiles x 4 steps
constexpr int kStageRow = kRec + 16;                // bytes per staged record (padded against bank conflicts)

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f16x2 as_f16x2(uint32_t w) { return __builtin_bit_cast(f16x2, w); }
__device__ __forceinline__ uint32_t as_u32(f16x2 h) { return __builtin_bit_cast(uint32_t, h); }

__device__ __forceinline__ uint32_t pk_clamp8(uint32_t w) {
    uint32_t r;
    asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(w), "v"(0x48004800u));
    asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(r), "v"(0xC800C800u));
    return r;
}

// Two coordinates as (hi, 2^11 lo), see the transform above.
__device__ __forceinline__ void split_pair(uint32_t w, uint32_t* hi, uint32_t* lo) {
    const f16x2 x = as_f16x2(w), xc = as_f16x2(pk_clamp8(w));
    const f16x2 magic = as_f16x2(0x4E004E00u);   // 24: the sum with |xc| <= 8 rounds to multiples of 2^-6
    const f16x2 t = xc + magic;
    // -2^11 (t - 24), then 2^11 (xc - (t - 24)); each exact
    const f16x2 nr = __builtin_elementwise_fma(t, as_f16x2(0xE800E800u), as_f16x2(0x7A007A00u));
    const f16x2 l = __builtin_elementwise_fma(xc, as_f16x2(0x68006800u), nr);
    *lo = as_u32(l);
    *hi = as_u32(__builtin_elementwise_fma(l, as_f16x2(0x90009000u), x));  // x - lo
}

__device__ __forceinline__ f16x8 frag(const uint32_t (&w)[4]) {
    return __builtin_bit_cast(f16x8, make_uint4(w[0], w[1], w[2], w[3]));
}

// All ones in the halves of w whose float16 is 4096 or more in size, an infinity or NaN.
__device__ __forceinline__ uint32_t large_halves(uint32_t w) {
    // 0x7fff - 0x6bff more sets the top bit of such a half, and carries into none.
    const uint32_t top = ((w & 0x7fff7fffu) + 0x14001400u) & 0x80008000u;
    return top | (top - (top >> 15));
}

// The four matrix steps' sums of one (s, e) combined by two butterfly stages: y[0], y[2], y[4], y[6].
__device__ __forceinline__ void combine(const double (&v)[4], double* y) {
    const double t0 = __dadd_rn(v[0], v[1]), t1 = __dsub_rn(v[0], v[1]);
    const double t2 = __dadd_rn(v[2], v[3]), t3 = __dsub_rn(v[2], v[3]);
    y[0] = __dadd_rn(t0, t2);
    y[2] = __dadd_rn(t1, t3);
    y[4] = __dsub_rn(t0, t2);
    y[6] = __dsub_rn(t1, t3);
}

__device__ __forceinline__ double tree8_sum(const double* v) {
    double s01 = __dadd_rn(v[0], v[1]);
    double s23 = __dadd_rn(v[2], v[3]);
    double s45 = __dadd_rn(v[4], v[5]);
    double s67 = __dadd_rn(v[6], v[7]);
    return __dadd_rn(__dadd_rn(s01, s23), __dadd_rn(s45, s67));
}

// id_slot of the 4 bytes of a word.
__device__ __forceinline__ uint32_t id_slot4(uint32_t w) {
    const uint32_t b5 = (w >> 5) & 0x01010101u, b6 = (w >> 6) & 0x01010101u, b7 = (w >> 7) & 0x01010101u;
    return w ^ (b5 | b5 << 1 | b5 << 2) ^ (b6 | b6 << 3 | b6 << 4) ^ (b7 << 1 | b7 << 2 | b7 << 3);
}

// Both float16 of a word as float64.
__device__ __forceinline__ void widen(uint32_t w, double* lo, double* hi) {
    *lo = (double)__half2float(__ushort_as_half((unsigned short)(w & 0xffffu)));
    *hi = (double)__half2float(__ushort_as_half((unsigned short)(w >> 16)));
}

// Per bucket of u: the next threshold (tau^2) and the bins surely passed, both 8 bytes apart
// so that one address serves the two reads.
struct Buckets {
    double next[kBucketLut];
    uint32_t passed[kBucketLut][2];
};

// One subspace's summary: id (bit j = [y_j < 0]), code word, weight.
struct Summary {
    uint32_t id, code;
    float w;
};

// Without the alpha-correction the weight is ||y_b|| = sqrt(S_b).
template <bool kAlpha>
__device__ __forceinline__ float weight(double S, double A) {
    const float w = kAlpha ? (float)(S / A) : (float)__dsqrt_rn(S);
    return S > 0.0 ? w : 0.0f;
}

// Any y: 7 compares per coordinate.
template <bool kAlpha>
__device__ __forceinline__ Summary summarise_any(const double* y, double S, const double* tau2, const double* s_a) {
    double TS[7], P[8];
#pragma unroll
    for (int t = 0; t < 7; ++t) TS[t] = __dmul_rn(tau2[t], S);
    const bool nz = S > 0.0;
    Summary r{0u, 0u, 0.0f};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const double Y = __dmul_rn(y[j], y[j]);
        const uint32_t neg = y[j] < 0.0 ? 1u : 0u;
        uint32_t t = 0;
#pragma unroll
        for (int u = 0; u < 7; ++u) t += (Y >= TS[u]) ? 1u : 0u;
        t = nz ? t : 0u;
        P[j] = __dmul_rn(s_a[t], fabs(y[j]));
        r.id |= neg << j;
        r.code |= (neg << 3 | t) << (4 * j);
    }
    r.w = weight<kAlpha>(S, tree8_sum(P));
    return r;
}

// Finite y, none of them -0: one compare per coordinate, chosen by its bucket.
template <bool kAlpha>
__device__ __forceinline__ Summary summarise(const double* y, const double* Y, double S, const Buckets& s_bk, const double* s_a) {
    // |u| kBuckets <= kBuckets (1 + 2^-20); S = 0 gives NaN, whose masked bits are bucket 0.
    const float rs = (float)kBuckets * __builtin_amdgcn_rsqf((float)S);
    double P[8];
    uint32_t code = 0;
#pragma unroll
    for (int j = 7; j >= 0; --j) {
        // u kBuckets + 2^20 leaves the bucket in bits 3..9 of the sum (rounded to eighths), which is
        // its byte offset in the 8-byte entries: one mask instead of a conversion and a shift.
        const uint32_t at = __float_as_uint(__fmaf_rn(fabsf((float)y[j]), rs, 0x1p20f)) & (8u * (kBucketLut - 1));
        const uint32_t t = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(s_bk.passed) + at) +
                           (Y[j] >= __dmul_rn(*reinterpret_cast<const double*>(reinterpret_cast<const char*>(s_bk.next) + at), S) ? 1u : 0u);
        P[j] = __dmul_rn(s_a[t], fabs(y[j]));
        code = __builtin_amdgcn_alignbit(code, (uint32_t)__double2hiint(y[j]), 31);  // code << 1 | sign
        code = code << 3 | t;
    }
    code = S > 0.0 ? code : 0u;
    Summary r;
    r.code = code;
    // The sign bits 3, 7, .. 31 of the code word, gathered into a byte.
    const uint32_t sg = code & 0x88888888u;
    r.id = (__builtin_amdgcn_udot8(sg, 0x00008421u, 0u, false) >> 3) |
           (__builtin_amdgcn_udot8(sg, 0x84210000u, 0u, false) << 1);
    r.w = weight<kAlpha>(S, tree8_sum(P));
    return r;
}

// Sum of squares of the lane's 32 coordinates.  Rounding never takes it below the largest of them:
// below 2^24 no coordinate is 4096 or more, an infinity or NaN.
__device__ __forceinline__ float squares(const uint4 (&v)[4]) {
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint32_t w[4] = {v[c].x, v[c].y, v[c].z, v[c].w};
#pragma unroll
        for (int h = 0; h < 4; ++h) s = __builtin_amdgcn_fdot2(as_f16x2(w[h]), as_f16x2(w[h]), s, false);
    }
    return s;
}

// The 64 bytes of coordinates [32 (lane / 16), +32) of key base + lane % 16 (zeros past the end).
__device__ __forceinline__ void load_part(const __half* src, int64_t base, int64_t k_end, int lane, uint4 (&v)[4]) {
    const int64_t i = base + (lane & 15);
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = make_uint4(0, 0, 0, 0);
    if (i < k_end) {
        const uint4* p = reinterpret_cast<const uint4*>(src + i * kD + 32 * (lane >> 4));
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = p[c];
    }
}

template <bool kLdsCounts, bool kRotate, bool kAlpha>
__global__ __launch_bounds__(kThreads, 3) void encode_kernel(
    const __half* __restrict__ keys, int64_t n_src, int64_t src_stride, int64_t keys_per_block, int64_t row0,
    int64_t capacity, uint8_t* __restrict__ ids, uint8_t* __restrict__ rec,
    uint32_t* __restrict__ counts, SignBits sb, QuantConsts qc) {
    __shared__ double s_a[8], s_tau2[7];
    __shared__ Buckets s_bk;
    __shared__ uint4 s_frag[kRotate ? kFrags : 1][64];
    __shared__ __align__(16) uint8_t s_stage[kWaves][kTile * kStageRow];
    __shared__ uint32_t s_cnt[kLdsCounts ? kB * kCentroids : 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, r16 = lane & 15;
    const int64_t grp = blockIdx.y;
    const int64_t k_begin = (int64_t)blockIdx.x * keys_per_block;
    const int64_t k_end = min(k_begin + keys_per_block, n_src);

    const __half* src = keys + grp * src_stride * kD;
    uint4 raw[4];
    load_part(src, k_begin + wave * kTile, k_end, lane, raw);

    const uint32_t smask = g == 0 ? sb.w[0] : g == 1 ? sb.w[1] : g == 2 ? sb.w[2] : sb.w[3];
    // Matrix operands, one uint4 per lane: output (s, e) of tile T in row r16, inputs
    // 8 (4g + c) + 2 j + e', the rotation's signs folded in.
    if (kRotate) {
        for (int f = wave; f < kFrags; f += kWaves) {
            const int T = f >> 2, j = f & 3;
            const int so = 4 * (r16 >> 2) + 2 * T + ((r16 >> 1) & 1);
            uint32_t w[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint32_t b = smask >> (8 * c + 2 * j);
                w[c] = (0x3C003C00u | (b & 1u) << 15 | (b & 2u) << 30) ^
                       (__popc(so & (4 * g + c)) & 1 ? 0x80008000u : 0u) ^ (r16 & 1 ? 0x80000000u : 0u);
            }
            s_frag[f][lane] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    if (tid < 8) s_a[tid] = qc.a[tid];
    if (tid < 7) s_tau2[tid] = qc.tau2[tid];
    for (int i = tid; i < kBucketLut; i += kThreads) {
        // Bins surely passed by every u that may fall in bucket i (rounding may lift it by 1/16
        // of a bucket), and the next threshold.
        const double lo = fmax(0.0, ((double)i - 0.07) / kBuckets);
        uint32_t c = 0;
        double next = __builtin_huge_val();
#pragma unroll
        for (int t = 6; t >= 0; --t) {
            const bool passed = qc.tau2[t] <= lo * lo;
            c += passed ? 1u : 0u;
            next = passed ? next : qc.tau2[t];
        }
        s_bk.next[i] = next;
        s_bk.passed[i][0] = c;
    }
    if (kLdsCounts) {
        for (int i = tid; i < kB * kCentroids; i += kThreads) s_cnt[i] = 0;
    }
    __syncthreads();

    // The tile's records and ids out, and its counts.
    auto emit = [&](const Summary (&sm)[4], int64_t base, bool count) {
        uint8_t* stage = s_stage[wave];
        uint4* st = reinterpret_cast<uint4*>(stage + r16 * kStageRow + 32 * g);
        st[0] = make_uint4(sm[0].code, sm[1].code, __float_as_uint(sm[0].w), __float_as_uint(sm[1].w));
        st[1] = make_uint4(sm[2].code, sm[3].code, __float_as_uint(sm[2].w), __float_as_uint(sm[3].w));
        const int64_t row = grp * capacity + row0 + base;
        if (base + r16 < k_end) {
            *reinterpret_cast<uint32_t*>(ids + (row + r16) * kB + 4 * g) =
                id_slot4(sm[0].id | sm[1].id << 8 | sm[2].id << 16 | sm[3].id << 24);
            if (count) {
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    const int at = (4 * g + b) * kCentroids + (int)sm[b].id;
                    if (kLdsCounts)
                        atomicAdd(&s_cnt[at], 1u);
                    else
                        atomicAdd(&counts[grp * (kB * kCentroids) + at], 1u);
                }
            }
        }
        // The wave's own staged rows (LDS operations of a wave complete in order).
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int k = 8 * p + (lane >> 3);
            const uint4 v = *reinterpret_cast<const uint4*>(stage + k * kStageRow + 16 * (lane & 7));
            if (base + k < k_end) *reinterpret_cast<uint4*>(rec + (row + k) * kRec + 16 * (lane & 7)) = v;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    // Tiles with large coordinates, left to the second loop: bit t, the wave's t-th.  Where the first
    // and the middle one have keys that the first loop may leave (a norm of 3000 or so), all are: large
    // keys then pay for one transform.  A test before it for every tile took 4% of ordinary keys' time.
    uint32_t later = 0;
    const int64_t begin = k_begin + wave * kTile;
    if (kRotate && __any(!(squares(raw) < 0x1p22f))) {
        const int tiles = (int)((max(k_end - begin, (int64_t)0) + kKeysPerIter - 1) / kKeysPerIter);
        uint4 mid[4];
        load_part(src, begin + (int64_t)(tiles / 2) * kKeysPerIter, k_end, lane, mid);
        if (__any(!(squares(mid) < 0x1p22f))) later = 0xffffffffu >> (32 - tiles);
    }
    uint32_t bit = 1;
    for (int64_t base = later ? k_end : begin; base < k_end; base += kKeysPerIter, bit <<= 1) {
        uint4 cur[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) cur[c] = raw[c];
        load_part(src, base + kKeysPerIter, k_end, lane, raw);  // the next tile's keys arrive under this one's work

        Summary sm[4];
        bool large = false;
        if (kRotate) {
            double total = 0.0;  // sum of squares of this lane's y
            uint32_t hi[4][4], lo[4][4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                split_pair(cur[c].x, &hi[0][c], &lo[0][c]);
                split_pair(cur[c].y, &hi[1][c], &lo[1][c]);
                split_pair(cur[c].z, &hi[2][c], &lo[2][c]);
                split_pair(cur[c].w, &hi[3][c], &lo[3][c]);
            }
            // Read for every tile: 32 registers less than holding them, which is another wave per SIMD.
            int at = lane;
            asm volatile("" : "+v"(at));
#pragma unroll
            for (int T = 0; T < 2; ++T) {
                f32x4 ah[4], al[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const f16x8 m = __builtin_bit_cast(f16x8, s_frag[4 * T + j][at]);
                    ah[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(m, frag(hi[j]), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    al[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(m, frag(lo[j]), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                }
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    double y[8], Y[8];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        double v[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            v[j] = __fma_rn((double)al[j][2 * q + e], 0x1p-11, (double)ah[j][2 * q + e]);
                        combine(v, y + e);
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) Y[j] = __dmul_rn(y[j], y[j]);
                    const double S = tree8_sum(Y);
                    total += S;
                    sm[2 * T + q] = summarise<kAlpha>(y, Y, S, s_bk, s_a);
                }
                __builtin_amdgcn_sched_barrier(0);  // the halves of a tile share registers
            }
            // A coordinate of 4096 makes the key's squares sum to 2^31 over its 4 lanes, 2^29 in one of
            // them, less a relative 2^-13 for its inexact sums.
            large = __any(!(total < 0x1.FFp28));
            later |= large ? bit : 0u;
        } else {
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const uint32_t w[4] = {cur[b].x, cur[b].y, cur[b].z, cur[b].w};
                double y[8], Y[8];
#pragma unroll
                for (int h = 0; h < 4; ++h) widen(w[h], &y[2 * h], &y[2 * h + 1]);
#pragma unroll
                for (int j = 0; j < 8; ++j) Y[j] = __dmul_rn(y[j], y[j]);
                sm[b] = summarise_any<kAlpha>(y, tree8_sum(Y), s_tau2, s_a);
            }
        }

        emit(sm, base, !large);  // a tile left to the second loop is written over there
    }

    // The tiles with large coordinates, in a loop of its own so that the two share the registers.
    if (kRotate) {
#pragma unroll 1
        for (; later; later &= later - 1) {
            const int64_t base = begin + (int64_t)__builtin_ctz(later) * kKeysPerIter;
            uint4 cur[4];
            load_part(src, base, k_end, lane, cur);
            const bool finite = !__any(!(squares(cur) < __builtin_huge_valf()));
            Summary sm[4];
            int at_lane = lane;
            asm volatile("" : "+v"(at_lane));
#pragma unroll
            for (int T = 0; T < 2; ++T) {
                f32x4 ah[4], al[4], at[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t hi[4], lo[4], top[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const uint32_t w = j == 0 ? cur[c].x : j == 1 ? cur[c].y : j == 2 ? cur[c].z : cur[c].w;
                        const uint32_t mask = large_halves(w);
                        split_pair(w & ~mask, &hi[c], &lo[c]);
                        top[c] = w & mask;
                    }
                    const f16x8 m = __builtin_bit_cast(f16x8, s_frag[4 * T + j][at_lane]);
                    ah[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(m, frag(hi), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    al[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(m, frag(lo), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    at[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(m, frag(top), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                }
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    double y[8], Y[8];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        double v[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const double low = __fma_rn((double)al[j][2 * q + e], 0x1p-11, (double)ah[j][2 * q + e]);
                            v[j] = __dadd_rn(low, (double)at[j][2 * q + e]);
                        }
                        combine(v, y + e);
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) Y[j] = __dmul_rn(y[j], y[j]);
                    const double S = tree8_sum(Y);
                    if (finite)
                        sm[2 * T + q] = summarise<kAlpha>(y, Y, S, s_bk, s_a);
                    else
                        sm[2 * T + q] = summarise_any<kAlpha>(y, S, s_tau2, s_a);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            emit(sm, base, true);
        }
    }

    if (kLdsCounts) {
        __syncthreads();
        for (int i = tid; i < kB * kCentroids; i += kThreads) {
            const uint32_t v = s_cnt[i];
            if (v) atomicAdd(&counts[grp * (kB * kCentroids) + i], v);
        }
    }
}

// Blocks that run at once (3 per CU by registers).  Keys are dealt evenly over the fewest
// whole rounds of that many blocks with at most 2048 keys each, so that no round is partly
// empty; 64 keys are one step of a block.
constexpr int64_t kFillBlocks = 768;
constexpr int64_t kMaxKeysPerBlock = 2048;
static_assert(kMaxKeysPerBlock <= 32 * kKeysPerIter, "a bit per tile of a wave");
// Calls of at most one tile per group count straight into global memory.  Scattered global
// atomics run at about 22 per ns over the chip (64 groups x 600 keys: 28 us with them, 18 us
// through LDS); for one tile the LDS histogram costs more to clear and flush than it saves.
constexpr int64_t kDirectCountKeys = 16;
constexpr int64_t kBulkKeys = 1024;  // calls of fewer keys per group are profiled as appends

__global__ void zero_u32_kernel(uint32_t* p, int64_t count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

}  // namespace

hipError_t launch_zero_u32(uint32_t* p, int64_t count, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const int64_t blocks = (count + 255) / 256;
    const ProfEvents pe = prof_begin("zero_counts");
    hipExtLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, pe.start, pe.stop, 0, p, count);
    return hipGetLastError();
}

hipError_t launch_encode(const void* keys, int64_t n_src, int64_t src_stride, int64_t groups,
                         int64_t row0, int64_t capacity, uint8_t* ids, uint8_t* rec,
                         uint32_t* counts, const SignBits& sb, const QuantConsts& qc, uint32_t flags,
                         hipStream_t s) {
    if (n_src <= 0 || groups <= 0) return hipSuccess;
    const __half* k = static_cast<const __half*>(keys);
    const bool rotate = !(flags & kFlagNoRotation), alpha = !(flags & kFlagNoAlpha);
    const int64_t total = n_src * groups;
    const int64_t fill = kFillBlocks * ((total + kFillBlocks * kMaxKeysPerBlock - 1) / (kFillBlocks * kMaxKeysPerBlock));
    int64_t per = (total + fill - 1) / fill;
    per = (per + kKeysPerIter - 1) / kKeysPerIter * kKeysPerIter;
    const bool lds = n_src > kDirectCountKeys;
    const dim3 grid((unsigned)((n_src + per - 1) / per), (unsigned)groups);
    const dim3 block(kThreads);
    // The profiler's names: by the size of the call, however it counts.
    const ProfEvents pe = prof_begin(n_src >= kBulkKeys ? "encode" : "append");
#define PARISKV_ENCODE(LDS, ROT, ALPHA)                                                                   \
    hipExtLaunchKernelGGL((encode_kernel<LDS, ROT, ALPHA>), grid, block, 0, s, pe.start, pe.stop, 0, k, n_src,   \
                          src_stride, per, row0, capacity, ids, rec, counts, sb, qc)
#define PARISKV_ENCODE_FLAGS(LDS)                                       \
    (rotate ? (alpha ? PARISKV_ENCODE(LDS, true, true) : PARISKV_ENCODE(LDS, true, false)) \
            : (alpha ? PARISKV_ENCODE(LDS, false, true) : PARISKV_ENCODE(LDS, false, false)))
    if (lds)
        PARISKV_ENCODE_FLAGS(true);
    else
        PARISKV_ENCODE_FLAGS(false);
#undef PARISKV_ENCODE_FLAGS
#undef PARISKV_ENCODE
    return hipGetLastError();
}

}  // namespace pariskv
