// Key quantization for gfx950 (Sec. 3.1; App. A; App. C depths): each bf16 key vector of 128 dims
// becomes b-bit codes on the scale s = M/Lv (M = max |k_i|, Lv = (2^b - 1)/2, nearest level c - Lv,
// ties to the upper level), the absmax M, and an int8 residual r = rint(254 Lv k / M) - 254 c + 254 Lv.
// b = 2 is App. A's codebook {-1.5, -0.5, 0.5, 1.5} with the residual rint(381 k / M) - 254 c + 381.
//
// Exactness. With F = 254 Lv and Q = F k / M, the code is c = i + 2^(b-1), i = floor(Q / 254), and
// the residual rint(Q) - 254 i - 127. For 2^-100 < M < 2^16:
//  * F / M is held as hi + lo (lo from the exact remainder of the division), so q = fma(k, hi, k lo)
//    is Q rounded to fp32: where Q itself is an fp32 value (every tie of the rounding, every bin edge
//    254 i) q == Q exactly.
//  * 254 j * fl(1/254) rounds to j exactly for every bin edge, and a Q that is no edge lies at least
//    2^-17 Q from every edge (|(2^b - 1) k - 2 M j| is a multiple of the smaller ulp), so
//    floor(q * fl(1/254)) is the exact floor. The product has to keep the sign of a k far below M: the
//    smallest, 2^-133 (2^b - 1) / M, stays above the 2^-150 that would round to 0 while M < 2^17.
//  * a Q that is no tie lies at least 2^-18 Q (b = 2) or 2^-20 Q (b = 4) from every half-integer, so
//    rint(q), half to even, is the exact rounding. For b = 8 that distance is 2^-24 Q, so q can land
//    on a half-integer that Q only comes near: there the exact remainder F k - q M decides.
// Other tokens (M outside that range, infinities or NaN among the dims) are redone in fp64, where
// nothing overflows and a quotient that is not a tie lies at least 2^-24 Q from every half-integer
// while the division moves it by at most 2^-53 Q.
//
// Bound: HBM (2D bytes read, 16b + 2 + D written per token), as long as the arithmetic stays near a
// dozen VALU instructions per element. At 8 x 131072 tokens, b = 2 (438 MB) a call takes 80 us,
// 5.5 TB/s, about what a device copy reaches; with three edge comparisons, integer packing and an fp64
// redo of every near-tie (a quarter percent of N(0, 1) keys are exactly +- M / 2, a tie, so most waves
// took it) it took 138 us. One-wave workgroups: 80 us; four waves: 84 us.
//
// Mapping: one wave per 64-token block; lane l = n + 16 g holds token n's 16-dim slices 16 g (both
// 64-dim halves) of each 16-token tile, which is the slice that the storage layouts of ffd.h give to
// lane l: codes and residuals are assembled in the lane and leave as 16-byte stores, 1 KiB contiguous
// over the wave, and the absmax takes two lane swaps per tile.
#include "ffd_device.h"
#include "ffd_kernels.h"

namespace ffd {

namespace {

typedef unsigned short v2u16 __attribute__((ext_vector_type(2)));

// A token's absmax and 254 Lv / M as hi + lo (zero for M = 0).
struct TokenScale {
    float m, hi, lo;
    bool special;       // M outside (2^-100, 2^16), infinities or NaN: the fp64 path
};

// One 16-dim slice: its code words (those of lane l in ffd.h) and residual bytes.
template <int BITS>
struct QuantSlice {
    uint32_t code[BITS / 2];
    uint32_t res[4];
};

__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(v2u16, a), __builtin_bit_cast(v2u16, b)));
}

// Largest |k| bit patterns of the slice, even and odd dims in the two halves.
__device__ __forceinline__ uint32_t slice_absmax(const uint4 (&raw)[2]) {
    uint32_t m = raw[0].x & 0x7fff7fffu;
    const uint32_t w[7] = {raw[0].y, raw[0].z, raw[0].w, raw[1].x, raw[1].y, raw[1].z, raw[1].w};
#pragma unroll
    for (int i = 0; i < 7; ++i) m = pk_max_u16(m, w[i] & 0x7fff7fffu);
    return m;
}

// The token's constants from the largest bit pattern of all its dims (bf16 magnitudes order as
// integers, NaN above infinity).
template <int BITS>
__device__ __forceinline__ TokenScale token_scale(uint32_t absmax2) {
    const uint32_t bits = max(absmax2 & 0xffffu, absmax2 >> 16);
    constexpr float kFull = 127.f * ((1 << BITS) - 1);      // 254 Lv
    TokenScale s;
    s.m = bf16_to_f32((uint16_t)bits);
    s.special = !(s.m < 0x1p16f && s.m > 0x1p-100f) && bits != 0;
    const float r = 1.f / s.m, hi = kFull / s.m;
    s.hi = bits == 0 ? 0.f : hi;
    s.lo = bits == 0 ? 0.f : fmaf(-hi, s.m, kFull) * r;
    return s;
}

// Byte I of a word from a float in [0, 255], rounded half to even by the conversion.
template <int I>
__device__ __forceinline__ uint32_t put_u8(float x, uint32_t word) {
    return __builtin_amdgcn_cvt_pk_u8_f32(x, I, word);
}

template <int BITS>
__device__ __forceinline__ void unpack_slice(const uint4 (&raw)[2], float (&x)[16]) {
    const uint32_t w[8] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w, raw[1].x, raw[1].y, raw[1].z, raw[1].w};
#pragma unroll
    for (int i = 0; i < 8; ++i) { x[2 * i] = bf16_lo(w[i]); x[2 * i + 1] = bf16_hi(w[i]); }
}

// Word and bit position of dim e's code in a slice's code words.
template <int BITS> __device__ constexpr int code_word(int e) { return (e >> 2) / (8 / BITS); }
template <int BITS> __device__ constexpr int code_shift(int e) { return 8 * (e & 3) + BITS * ((e >> 2) % (8 / BITS)); }

// The fp64 path; m is the absmax over the dims that are not NaN (0: no dim but zeros and NaN, residual 0).
template <int BITS>
__device__ __forceinline__ QuantSlice<BITS> quantize_slice_f64(uint4 raw0, uint4 raw1, float m) {
#pragma clang fp contract(off)
    constexpr int kLevels = 1 << BITS;
    constexpr double kTwoLv = kLevels - 1, kFull = 127.0 * (kLevels - 1);
    const uint4 raw[2] = {raw0, raw1};
    float x[16];
    unpack_slice<BITS>(raw, x);
    QuantSlice<BITS> qs = {};
    const double md = m, two_md = 2.0 * md;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const double xv = x[e], u = kTwoLv * xv;
        double i = floor(u / two_md);
        if ((i + 1.0) * two_md <= u) i += 1.0;
        if (i * two_md > u) i -= 1.0;
        const int c = min(max((int)i + kLevels / 2, 0), kLevels - 1);
        const int r = m == 0.f ? 0 : (int)rint((kFull * xv) / md) - 254 * c + (int)kFull;
        qs.code[code_word<BITS>(e)] |= (uint32_t)(BITS == 8 ? (c - 128) & 0xff : c) << code_shift<BITS>(e);
        qs.res[e >> 2] |= (uint32_t)(r & 0xff) << (8 * (e & 3));
    }
    return qs;
}

template <int BITS>
__device__ __forceinline__ QuantSlice<BITS> quantize_slice(const uint4 (&raw)[2], const TokenScale& s) {
#pragma clang fp contract(off)          // the rounding arguments above name every fused product
    constexpr float kFull = 127.f * ((1 << BITS) - 1);
    float x[16], t[16], fi[16];
    unpack_slice<BITS>(raw, x);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        const float q = fmaf(x[e], s.hi, x[e] * s.lo);
        fi[e] = floorf(q * (1.f / 254.f));
        if constexpr (BITS == 8) {
            float n = rintf(q);
            const float d = q - n, rem = fmaf(-q, s.m, kFull * x[e]);   // exact: |d| = 1/2 has q in 16 bits
            n += fabsf(d) == 0.5f && d * rem > 0.f ? 2.f * d : 0.f;
            t[e] = fmaf(-254.f, fi[e], n);
        } else {
            t[e] = fmaf(-254.f, fi[e], q);                              // exact difference in [0, 254]
        }
    }
    QuantSlice<BITS> qs;
    const uint32_t any = s.m != 0.f ? 0xffffffffu : 0u;                 // M = 0: residual 0
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        uint32_t r = put_u8<0>(t[4 * w], 0u);
        r = put_u8<1>(t[4 * w + 1], r);
        r = put_u8<2>(t[4 * w + 2], r);
        r = put_u8<3>(t[4 * w + 3], r);
        // bytes rint(Q) - 254 i in [0, 254] to rint(Q) - 254 i - 127: + 1 without a carry, - 128
        qs.res[w] = ((r + 0x01010101u) ^ 0x80808080u) & any;
    }
    // the codes of one byte as a float sum of i * 2^(bit), biased by 2^(b-1) per code, at most 255
    constexpr int kPer = 8 / BITS;
    constexpr float kBias = (1 << (BITS - 1)) * (255.f / ((1 << BITS) - 1));
#pragma unroll
    for (int w = 0; w < BITS / 2; ++w) {
        float a[4] = {kBias, kBias, kBias, kBias};
#pragma unroll
        for (int k = 0; k < kPer; ++k)
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = fmaf(fi[4 * (w * kPer + k) + i], (float)(1 << (BITS * k)), a[i]);
        uint32_t c = put_u8<0>(a[0], 0u);
        c = put_u8<1>(a[1], c);
        c = put_u8<2>(a[2], c);
        c = put_u8<3>(a[3], c);
        qs.code[w] = BITS == 8 ? c ^ 0x80808080u : c;
    }
    return qs;
}

__device__ __forceinline__ uint16_t bf16_bits(float m) { return (uint16_t)(__float_as_uint(m) >> 16); }

// Store the slice of 64-dim half cc, group g, of token n16 of tile t4 of a (b, kvh)'s block blk.
template <int BITS>
__device__ __forceinline__ void store_slice(const QuantSlice<BITS>& qs, float m, size_t blk, int t4, int n16, int cc,
                                            int g, uint32_t* codes, uint16_t* absmax, int8_t* resid) {
    const int w = (2 * t4 + cc) * (BITS / 2), l = n16 + 16 * g;
    uint32_t* dst = codes + blk * (64 * 4 * BITS) + (w >> 2) * 256 + l * 4 + (w & 3);
    if constexpr (BITS == 2) dst[0] = qs.code[0];
    else if constexpr (BITS == 4) *reinterpret_cast<uint2*>(dst) = make_uint2(qs.code[0], qs.code[1]);
    else *reinterpret_cast<uint4*>(dst) = make_uint4(qs.code[0], qs.code[1], qs.code[2], qs.code[3]);
    reinterpret_cast<uint4*>(resid)[blk * 512 + t4 * 128 + cc * 64 + l] =
        make_uint4(qs.res[0], qs.res[1], qs.res[2], qs.res[3]);
    if (cc == 0 && g == 0) absmax[blk * 64 + n16 * 4 + t4] = bf16_bits(m);
}

// max over the four lanes n, n + 16, n + 32, n + 48 (one token's slices), every lane receiving it
__device__ __forceinline__ uint32_t token_max4(uint32_t m) {
    const auto a = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    m = pk_max_u16(a[0], a[1]);
    const auto b = __builtin_amdgcn_permlane16_swap(m, m, false, false);
    return pk_max_u16(b[0], b[1]);
}

// max of |x| over the dims of a slice that are not NaN
__device__ __forceinline__ float slice_fmax(uint4 raw0, uint4 raw1) {
    const uint4 raw[2] = {raw0, raw1};
    float x[16], m = 0.f;
    unpack_slice<2>(raw, x);
#pragma unroll
    for (int e = 0; e < 16; ++e) m = fmaxf(m, fabsf(x[e]));
    return m;
}

}  // namespace

// Workgroup x, one wave, covers block t_begin / 64 + x of one (b, kvh); only tokens in [t_begin,
// t_end) are stored. The four tiles' loads are issued first.
template <int BITS>
__global__ __launch_bounds__(kQuantThreads) void quantize_keys_kernel(QuantArgs a) {
    const int lane = threadIdx.x, g = lane >> 4, n = lane & 15;
    const int j = (a.t_begin >> 6) + blockIdx.x;
    const size_t bh = (size_t)blockIdx.z * a.Hkv + blockIdx.y;
    const bool whole = 64 * j >= a.t_begin && 64 * j + 64 <= a.t_end;       // uniform in the wave
    const uint4* kp = reinterpret_cast<const uint4*>(a.k) + bh * a.Lcap * (kD / 8) + 2 * g;
    uint4 raw[4][2][2];
    bool in[4];
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4) {
        const int t = 64 * j + 16 * t4 + n;
        in[t4] = t >= a.t_begin && t < a.t_end;
        // a token outside the range reads one inside it (no branch around the loads) and stores nothing
        const uint4* tok = kp + (size_t)min(max(t, a.t_begin), a.t_end - 1) * (kD / 8);
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
#pragma unroll
            for (int h = 0; h < 2; ++h) raw[t4][cc][h] = tok[8 * cc + h];
    }
    const size_t blk = bh * (size_t)(a.Lcap / 64) + j;
    uint4* cdst = reinterpret_cast<uint4*>(a.codes) + blk * (64 * BITS) + lane;
    uint4* rdst = reinterpret_cast<uint4*>(a.resid) + blk * 512 + lane;
    uint16_t* mdst = a.absmax + blk * 64 + n * 4;
    uint32_t m4[4], w2[4];                          // absmaxes of the lane's tokens; b = 2: words of two tiles
    int special = 0;                                // tiles in which the lane's token needs the fp64 path
#pragma unroll
    for (int t4 = 0; t4 < 4; ++t4) {
        const TokenScale s = token_scale<BITS>(token_max4(pk_max_u16(slice_absmax(raw[t4][0]), slice_absmax(raw[t4][1]))));
        QuantSlice<BITS> qs[2];
#pragma unroll
        for (int cc = 0; cc < 2; ++cc) qs[cc] = quantize_slice<BITS>(raw[t4][cc], s);
        special |= (int)s.special << t4;
        m4[t4] = bf16_bits(s.m);
        if (whole || in[t4]) {
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                const QuantSlice<BITS>& v = qs[cc];
                rdst[t4 * 128 + cc * 64] = make_uint4(v.res[0], v.res[1], v.res[2], v.res[3]);
                if constexpr (BITS == 8) cdst[(2 * t4 + cc) * 64] = make_uint4(v.code[0], v.code[1], v.code[2], v.code[3]);
            }
            if constexpr (BITS == 4) cdst[t4 * 64] = make_uint4(qs[0].code[0], qs[0].code[1], qs[1].code[0], qs[1].code[1]);
        }
        if constexpr (BITS == 2) {
            w2[2 * (t4 & 1)] = qs[0].code[0];
            w2[2 * (t4 & 1) + 1] = qs[1].code[0];
            if (whole) {
                if (t4 & 1) cdst[(t4 >> 1) * 64] = make_uint4(w2[0], w2[1], w2[2], w2[3]);
            } else if (in[t4]) {
                reinterpret_cast<uint2*>(cdst + (t4 >> 1) * 64)[t4 & 1] = make_uint2(qs[0].code[0], qs[1].code[0]);
            }
        }
    }
    if (g == 0) {
        if (whole) {
            *reinterpret_cast<uint2*>(mdst) = make_uint2(m4[0] | (m4[1] << 16), m4[2] | (m4[3] << 16));
        } else {
#pragma unroll
            for (int t4 = 0; t4 < 4; ++t4)
                if (in[t4]) mdst[t4] = (uint16_t)m4[t4];
        }
    }
    if (special == 0) return;
#pragma unroll 1
    for (int t4 = 0; t4 < 4; ++t4) {                // rare: these tokens again, over what was stored
        const int t = 64 * j + 16 * t4 + n;
        if (!(special >> t4 & 1) || t < a.t_begin || t >= a.t_end) continue;      // a token's four lanes together
        const uint4* tok = kp + (size_t)t * (kD / 8);
        float m = fmaxf(slice_fmax(tok[0], tok[1]), slice_fmax(tok[8], tok[9]));
        m = fmaxf(m, __shfl_xor(m, 16));
        m = fmaxf(m, __shfl_xor(m, 32));
#pragma unroll 1
        for (int cc = 0; cc < 2; ++cc)
            store_slice<BITS>(quantize_slice_f64<BITS>(tok[8 * cc], tok[8 * cc + 1], m), m, blk, t4, n, cc, g, a.codes,
                              a.absmax, a.resid);
    }
}

// Decode-step append: workgroup b writes the new token of every KV head of sequence b at position
// L = seq_lens[b] (bf16 K/V rows when the caches are given, and its quantized key), then sets
// seq_lens[b] = L + 1. 8 lanes per KV head, one 16-dim slice each; a sequence already at capacity is
// left unchanged.
template <int BITS>
__global__ __launch_bounds__(kThreads) void append_kv_kernel(AppendArgs a) {
    const int tid = threadIdx.x, s8 = tid & 7, cc = s8 >> 2, g = s8 & 3;
    const int b = blockIdx.x;
    const int L = a.seq_lens[b];
    const bool room = L >= 0 && L < a.Lcap;
    for (int kvh = tid >> 3; kvh < a.Hkv; kvh += kThreads / 8) {
        const size_t bh = (size_t)b * a.Hkv + kvh;
        const uint4* kp = reinterpret_cast<const uint4*>(a.k_new + bh * kD) + 2 * s8;
        const uint4* vp = reinterpret_cast<const uint4*>(a.v_new + bh * kD) + 2 * s8;
        const uint4 raw[2] = {kp[0], kp[1]};
        const uint4 v0 = vp[0], v1 = vp[1];
        uint32_t m2 = slice_absmax(raw);            // then over the head's eight lanes
        m2 = pk_max_u16(m2, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m2, kDppXor1, 0xf, 0xf, false));
        m2 = pk_max_u16(m2, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m2, kDppXor2, 0xf, 0xf, false));
        m2 = pk_max_u16(m2, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m2, kDppHalfMirror, 0xf, 0xf, false));
        const TokenScale s = token_scale<BITS>(m2);
        if (room) {
            const size_t row = (bh * a.Lcap + L) * (kD / 8) + 2 * s8;
            if (a.k_cache) {
                reinterpret_cast<uint4*>(a.k_cache)[row] = raw[0];
                reinterpret_cast<uint4*>(a.k_cache)[row + 1] = raw[1];
            }
            if (a.v_cache) {
                reinterpret_cast<uint4*>(a.v_cache)[row] = v0;
                reinterpret_cast<uint4*>(a.v_cache)[row + 1] = v1;
            }
            const int n16 = L & 15, t4 = (L >> 4) & 3;
            const size_t blk = bh * (size_t)(a.Lcap / 64) + (L >> 6);
            if (s.special) {                        // the head's eight lanes together
                float m = slice_fmax(raw[0], raw[1]);
                m = fmaxf(m, __shfl_xor(m, 1));
                m = fmaxf(m, __shfl_xor(m, 2));
                m = fmaxf(m, __shfl_xor(m, 4));
                store_slice<BITS>(quantize_slice_f64<BITS>(raw[0], raw[1], m), m, blk, t4, n16, cc, g, a.codes, a.absmax,
                                  a.resid);
            } else {
                store_slice<BITS>(quantize_slice<BITS>(raw, s), s.m, blk, t4, n16, cc, g, a.codes, a.absmax, a.resid);
            }
        }
    }
    __syncthreads();                    // every thread has read L before it moves
    if (tid == 0 && room) a.seq_lens[b] = L + 1;
}

template __global__ void quantize_keys_kernel<2>(QuantArgs);
template __global__ void quantize_keys_kernel<4>(QuantArgs);
template __global__ void quantize_keys_kernel<8>(QuantArgs);
template __global__ void append_kv_kernel<2>(AppendArgs);
template __global__ void append_kv_kernel<4>(AppendArgs);
template __global__ void append_kv_kernel<8>(AppendArgs);

}  // namespace ffd
