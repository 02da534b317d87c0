// Log-sum-exp merge of split partials (the flash-decoding reduction, Sec. 2): for each (sequence,
// query head), M* = max_s m_s, l* = sum_s e^{m_s - M*} l_s, out = sum_s e^{m_s - M*} acc_s / l*,
// lse = M* + ln l*. Splits that kept nothing carry m = -inf and are skipped (their l and acc may hold
// anything); a head with no split gets out = 0 and lse = -inf.
//
// Partial rows of head bh = b * Hq + h: i * G + bh % G for i = first .. last, (first, last) = table[bh / G]
// (last < first: none), or, without a table, the S rows from S * (bh / G) on.
//
// Bound: latency (a table load, the rows, two reductions, the store), and with very many heads the number
// of waves. One workgroup of NW waves per head and quarter of its dims, so that few heads still spread over
// the CUs; thread (r, d4) takes rows r, r + 8 NW, ... of dims 4 d4 .. 4 d4 + 3, all of a batch's rows
// requested at once (16 NW rows, or 64 NW where there are more), their common maximum first and then one
// rescaling per row. Against one workgroup per head that folded the rows one after the other: 4 heads of
// 256 rows 6.4 -> 3.9 us (NW = 4), the step at 1 x 256K 25.7 -> 23.9 us;
// 1024, 2048 and 4096 heads of 2 to 4 rows 5.2, 9.3 and 16.0 -> 4.0, 5.0 and 8.0 us (NW = 1; 6.3, 10.8 and
// 18.8 us with four waves).
#include "ffd_device.h"
#include "ffd_kernels.h"

namespace ffd {

namespace {

constexpr int kSliceDims = kD / kMergeSlices;  // 8 lanes of 4 dims

struct State {
    float m, l;
    float a[4];
};

__device__ __forceinline__ float rescale(float m, float M) { return m == -INFINITY ? 0.f : __expf(m - M); }

// Folds rows s0 + LANES u (u < U) below count into st; the row index is clamped, so that the loads are
// unconditional.
template <int U, int LANES>
__device__ __forceinline__ void fold_rows(State& st, const float* __restrict__ part_m, const float* __restrict__ part_l,
                                          const float* __restrict__ part_acc, size_t row0, size_t stride, int count,
                                          int s0) {
    float m[U], l[U];
    float4 a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int s = s0 + u * LANES;
        const size_t row = row0 + (size_t)min(s, count - 1) * stride;
        m[u] = part_m[row];
        l[u] = part_l[row];
        a[u] = *reinterpret_cast<const float4*>(part_acc + row * kD);
        if (s >= count) m[u] = -INFINITY;
    }
    float M = st.m;
#pragma unroll
    for (int u = 0; u < U; ++u) M = fmaxf(M, m[u]);
    const float c = rescale(st.m, M);
    st.m = M;
    st.l *= c;
#pragma unroll
    for (int e = 0; e < 4; ++e) st.a[e] *= c;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float w = rescale(m[u], M);
        const bool any = m[u] != -INFINITY;         // else l and a may be NaN
        st.l = fmaf(w, any ? l[u] : 0.f, st.l);
        st.a[0] = fmaf(w, any ? a[u].x : 0.f, st.a[0]);
        st.a[1] = fmaf(w, any ? a[u].y : 0.f, st.a[1]);
        st.a[2] = fmaf(w, any ? a[u].z : 0.f, st.a[2]);
        st.a[3] = fmaf(w, any ? a[u].w : 0.f, st.a[3]);
    }
}

// max and sum over the lanes that differ in bits 3, 4 and 5 (the rows of a wave)
__device__ __forceinline__ float rows_max(float x) {
    x = fmaxf(x, dpp_f<kDppRor8>(x));
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum(float x) {
    x += dpp_f<kDppRor8>(x);
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

}  // namespace

// Grid (B * Hq, kMergeSlices).
template <int NW>
__global__ __launch_bounds__(64 * NW) void lse_merge_kernel(const float* __restrict__ part_m,
                                                             const float* __restrict__ part_l,
                                                             const float* __restrict__ part_acc, int S,
                                                             const int2* __restrict__ table, int G,
                                                             uint16_t* __restrict__ out, float* __restrict__ lse) {
    constexpr int kRowLanes = 8 * NW;               // rows in parallel
    alignas(16) __shared__ float part[NW][8][8];    // each wave's state per d4
    const int tid = threadIdx.x, d4 = tid & 7, r = tid >> 3, wave = tid >> 6, lane = tid & 63;
    const size_t x = blockIdx.x / G;                        // blockIdx.x = b * Hq + h
    size_t first = x * S;
    if (table) {
        const int2 fl = table[x];
        first = fl.x;
        S = fl.y - fl.x + 1;
    }
    const size_t row0 = first * G + blockIdx.x % G;
    const float* acc = part_acc + blockIdx.y * kSliceDims + 4 * d4;
    State st{-INFINITY, 0.f, {0.f, 0.f, 0.f, 0.f}};
    if (S > 2 * kRowLanes) {                                // uniform
        for (int s0 = 0; s0 < S; s0 += 8 * kRowLanes) fold_rows<8, kRowLanes>(st, part_m, part_l, acc, row0, G, S, s0 + r);
    } else if (S > 0) {
        fold_rows<2, kRowLanes>(st, part_m, part_l, acc, row0, G, S, r);
    }
    const float M = rows_max(st.m);
    const float c = rescale(st.m, M);
    const float l = rows_sum(st.l * c);
    float a[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] = rows_sum(st.a[e] * c);
    if (lane < 8) {
        *reinterpret_cast<float4*>(&part[wave][d4][0]) = make_float4(a[0], a[1], a[2], a[3]);
        *reinterpret_cast<float2*>(&part[wave][d4][4]) = make_float2(M, l);
    }
    if constexpr (NW > 1) __syncthreads();
    else wave_lds_fence();
    if (tid >= 8) return;
    float Mw[NW], Mx = -INFINITY, lx = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        Mw[w] = part[w][d4][4];
        Mx = fmaxf(Mx, Mw[w]);
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float cw = rescale(Mw[w], Mx);
        const float4 aw = *reinterpret_cast<const float4*>(&part[w][d4][0]);
        lx = fmaf(cw, part[w][d4][5], lx);
        o.x = fmaf(cw, aw.x, o.x);
        o.y = fmaf(cw, aw.y, o.y);
        o.z = fmaf(cw, aw.z, o.z);
        o.w = fmaf(cw, aw.w, o.w);
    }
    const bool any = Mx != -INFINITY;
    const float inv = any ? 1.f / lx : 0.f;
    uint2 packed;
    packed.x = (uint32_t)f32_to_bf16(o.x * inv) | ((uint32_t)f32_to_bf16(o.y * inv) << 16);
    packed.y = (uint32_t)f32_to_bf16(o.z * inv) | ((uint32_t)f32_to_bf16(o.w * inv) << 16);
    *reinterpret_cast<uint2*>(out + (size_t)blockIdx.x * kD + blockIdx.y * kSliceDims + 4 * d4) = packed;
    if (lse && blockIdx.y == 0 && d4 == 0) lse[blockIdx.x] = any ? Mx + logf(lx) : -INFINITY;
}

template __global__ void lse_merge_kernel<1>(const float*, const float*, const float*, int, const int2*, int, uint16_t*, float*);
template __global__ void lse_merge_kernel<4>(const float*, const float*, const float*, int, const int2*, int, uint16_t*, float*);

}  // namespace ffd
