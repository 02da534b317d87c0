// FFD decode attention for gfx950: b-bit thumbnail scan (b = 2, 4, 8; App. C) + top-delta
// selection, then refinement + online softmax over the kept blocks.
//
// Method (Alg. 1; Eq. 1-4): for each query head h of a KV group,
//   s_hat[t] = alpha * q . k^quant_t                      (thumbnail scan)
//   m~       = max of s_hat over the first n_sink and last n_local tokens      (pseudo-max, Eq. 3)
//   keep j   iff max_{t in block j} s_hat[t] >= m~ - delta                       (top-delta, Eq. 1)
//   z[t]     = s_hat[t] + alpha * q . k^res_t   for t in kept blocks            (scan reuse, Eq. 4)
//   out      = softmax(z) . V over kept tokens, split into partial states merged by LSE.
//
// Arithmetic. The group's queries are the A operand of v_mfma_i32_16x16x64_i8: each query is held in
// fixed point Q = rint(q * 2^(22-E)) (|q| < 2^E), split into three signed 8-bit limbs, one MFMA row
// per (head, limb). The B operand is either a 16-token tile's codes as bytes (2- and 4-bit codes
// expanded by two VALU ops per 4 codes, 8-bit codes stored as the signed bytes c - 128) or its stored
// int8 residual, so both dot products are exact integer sums, combined and rounded once to fp32:
//   sum_d Q_d (2 c_d - (2^b - 1)) = T  (exact: int32 for b = 2, int64 otherwise),
//                                   s_hat = T * M_t * alpha 2^(E-23) / Lv,   Lv = (2^b - 1) / 2
//   sum_d Q_d r_d                 = R  (three int32 limbs), z = s_hat + R * M_t * alpha 2^(E-22) / (254 Lv)
// Output register i of lane (g, n) is row 4g + i, column n: head g's limbs for token n, so each
// 16-lane row group owns one head and a tile's maximum is a 16-lane DPP reduction.
//
// Two ways to run a step, chosen by the host (FFD_KERNELS_*):
//  * ffd_decode_kernel, the fused kernel (short and mid contexts: at most 64 blocks per
//    workgroup): S1 workgroups per (sequence, KV head) each scan an interleaved share of the group's
//    blocks (j = s + S1 i), decide them, and refine and attend their own kept blocks; one partial
//    state per head (or, with S1 = 1, the outputs themselves).
//  * the split kernels, where the kept blocks are too many for their owners to refine in time:
//    - ffd_scan_kernel streams the codes and absmaxes of every block once (the dominant, perfectly
//      regular stream; one 8-wave workgroup per CU whose waves take blocks from an LDS counter),
//      keeps each block's per-head maximum score in LDS and, once its stream and the pseudo-max are
//      done, takes the keep decision per (head, block): the kept blocks, with their per-head keep
//      bits, form its workgroup's kept list (in block order) in the workspace, plus the list's
//      length;
//    - ffd_refine_kernel lays the kept blocks of all groups on one line and gives each 8-wave
//      workgroup an equal share of it (every workgroup computes the same line from the scan's
//      records, so no cross-workgroup synchronisation is needed), wave w taking 16-token tile w % 4
//      of every other block, with several tiles' residual and value loads in flight; it writes one
//      partial (m, l, acc) per head of every group in its share, and lse_merge_kernel combines the
//      partials of each head through a small per-group table.
// Both recompute the scan scores s_hat of each kept tile from its codes (Eq. 4's reuse term: the
// same integer MFMA and fp32 operations as the scan, so the same values; storing them would cost
// as many bytes, written then read).
#include <type_traits>

#include "ffd_device.h"
#include "ffd_kernels.h"

namespace ffd {

namespace {

#ifndef FFD_SCAN_RING
#define FFD_SCAN_RING 4
#endif
#ifndef FFD_REFINE_RING
#define FFD_REFINE_RING 2
#endif
constexpr int kRing2 = FFD_SCAN_RING;         // 2-bit scan loads in flight per wave (blocks)
constexpr int kRefineRing = FFD_REFINE_RING;  // refinement tiles in flight per wave (fused: RING)

__device__ __forceinline__ int limb_of(int Q, int which) {
    const int l0 = ((Q + 128) & 255) - 128;
    const int q1 = (Q - l0) >> 8;
    const int l1 = ((q1 + 128) & 255) - 128;
    const int l2 = (q1 - l1) >> 8;
    return which == 0 ? l0 : (which == 1 ? l1 : l2);
}

// The 16 codes of one (tile, 64-dim chunk) group of a lane, from its b/2 words, as the MFMA B
// operand: byte i of dword k is dim 4k + i of the lane's 16-dim slice.
template <int BITS>
__device__ __forceinline__ v4i expand_codes(const uint32_t* w) {
    v4i r;
    if constexpr (BITS == 2) {
        r.x = (int)(w[0] & 0x03030303u);
        r.y = (int)((w[0] >> 2) & 0x03030303u);
        r.z = (int)((w[0] >> 4) & 0x03030303u);
        r.w = (int)((w[0] >> 6) & 0x03030303u);
    } else if constexpr (BITS == 4) {
        r.x = (int)(w[0] & 0x0f0f0f0fu);
        r.y = (int)((w[0] >> 4) & 0x0f0f0f0fu);
        r.z = (int)(w[1] & 0x0f0f0f0fu);
        r.w = (int)((w[1] >> 4) & 0x0f0f0f0fu);
    } else {
        r.x = (int)w[0]; r.y = (int)w[1]; r.z = (int)w[2]; r.w = (int)w[3];
    }
    return r;
}

template <int NT>
struct HeadConsts {
    v4i A[NT][2];      // MFMA A operand per head tile and 64-dim chunk
    int sumq[NT];      // sum_d Q_d of head 4t + g
    float kap[NT];     // alpha * 2^(E-23) / Lv
    float kap2[NT];    // alpha * 2^(E-22) / (254 Lv)
    bool live[NT];     // head 4t + g exists
};

template <int NT>
struct QueryLds {
    alignas(16) int8_t limbs[4][4 * NT][kD];     // [limb][head][dim]; limb 3 is zero
    int sumq[4 * NT];
    float kap[4 * NT];
    float kap2[4 * NT];
};

// Wave w < 4 NT: this lane's dword (dims 2*lane, 2*lane + 1) of head min(w, G - 1) of the group whose
// first query row is row0.
template <int NT>
__device__ __forceinline__ uint32_t load_query_word(const uint16_t* __restrict__ q, size_t row0, int G, int wave, int lane) {
    return reinterpret_cast<const uint32_t*>(q + (row0 + min(wave, G - 1)) * kD)[lane];
}

// Queries -> fixed-point limbs in LDS and this lane's per-head constants, by the workgroup's eight
// waves. Head h (wave h): E with max|q| < 2^E, Q = rint(q 2^(22-E)) split into three signed bytes
// stored as limbs[limb][h][d]; the fourth limb row and heads past G are zero. lv is the thumbnail's
// outer level Lv. One workgroup barrier, before the constants are read; the caller sees to it that no
// wave still reads those of an earlier group.
template <int NT>
__device__ __forceinline__ void build_query_consts(QueryLds<NT>& sm, uint32_t qw, int G, float scale, float lv, int wave,
                                                   int lane, HeadConsts<NT>& hc) {
    const int g = lane >> 4, n = lane & 15;
    if (wave < 4 * NT) {
        const bool live = wave < G;
        const float x0 = live ? bf16_lo(qw) : 0.f, x1 = live ? bf16_hi(qw) : 0.f;     // dims 2*lane, 2*lane + 1
        const float mx = wave_max_dpp(fmaxf(fabsf(x0), fabsf(x1)));
        int E = 0;
        (void)frexpf(mx, &E);                       // mx < 2^E (mx == 0 -> E = 0)
        const int Q0 = (int)rintf(ldexpf(x0, 22 - E));
        const int Q1 = (int)rintf(ldexpf(x1, 22 - E));
#pragma unroll
        for (int li = 0; li < 3; ++li) {
            const uint32_t pair = ((uint32_t)limb_of(Q0, li) & 0xffu) | (((uint32_t)limb_of(Q1, li) & 0xffu) << 8);
            reinterpret_cast<uint16_t*>(&sm.limbs[li][wave][0])[lane] = (uint16_t)pair;
        }
        reinterpret_cast<uint16_t*>(&sm.limbs[3][wave][0])[lane] = 0;
        const int sum = wave_sum_dpp(Q0 + Q1);
        if (lane == 0) {
            sm.sumq[wave] = sum;
            sm.kap[wave] = ldexpf(scale / lv, E - 23);
            sm.kap2[wave] = ldexpf(scale / (254.f * lv), E - 22);
        }
    }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        // A operand: row m = n is (head 4t + n/4, limb n%4); its 16 bytes are dims 64cc + 16g + e.
        const int hrow = 4 * t + (n >> 2), limb = n & 3;
#pragma unroll
        for (int cc = 0; cc < 2; ++cc)
            hc.A[t][cc] = *reinterpret_cast<const v4i*>(&sm.limbs[limb][hrow][64 * cc + 16 * g]);
        const int hh = 4 * t + g;      // this lane's output head
        hc.live[t] = hh < G;
        hc.sumq[t] = hc.live[t] ? sm.sumq[hh] : 0;
        hc.kap[t] = hc.live[t] ? sm.kap[hh] : 0.f;
        hc.kap2[t] = hc.live[t] ? sm.kap2[hh] : 0.f;
    }
}

// One lane's share of a block's thumbnail: its 4b code words (both 64-dim halves of its token in
// each of the four tiles; w[i] = words 4i .. 4i + 3, each load 1 KiB contiguous over the wave) and
// the absmax of its four tokens.
template <int BITS>
struct BlockScan {
    uint4 w[BITS];
    uint2 mm;
};

template <int BITS>
__device__ __forceinline__ BlockScan<BITS> load_block_scan(const uint32_t* __restrict__ codes_bh,
                                                           const uint16_t* __restrict__ absmax_bh, int j,
                                                           int lane) {
    const uint4* cp = reinterpret_cast<const uint4*>(codes_bh) + (size_t)j * 64 * BITS + lane;
    BlockScan<BITS> r;
#pragma unroll
    for (int i = 0; i < BITS; ++i) r.w[i] = cp[64 * i];               // words 4i .. 4i + 3
    r.mm = *reinterpret_cast<const uint2*>(absmax_bh + (size_t)j * 64 + (lane & 15) * 4);
    return r;
}

// The same loads through buffer resources whose ranges end at a workgroup's last block: a block
// index at or past that end reads zeros without touching memory (the hardware range check of a raw
// buffer), so a wave may request blocks that turn out not to exist.
constexpr int kRawBufferWord3 = 0x00020000;    // gfx9 raw buffer: 32-bit data format, no swizzle
template <int BITS>
__device__ __forceinline__ BlockScan<BITS> load_block_scan_rsrc(__amdgpu_buffer_rsrc_t rc, __amdgpu_buffer_rsrc_t ra,
                                                                int j, int lane) {
    BlockScan<BITS> r;
    const uint32_t base = (uint32_t)j * (1024u * BITS) + (uint32_t)lane * 16u;
#pragma unroll
    for (int i = 0; i < BITS; ++i) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(rc, (int)(base + 1024u * i), 0, 0);
        r.w[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
    const auto m = __builtin_amdgcn_raw_buffer_load_b64(ra, (int)((uint32_t)j * 128u + (uint32_t)(lane & 15) * 8u), 0, 0);
    r.mm = make_uint2(m[0], m[1]);
    return r;
}

// Thumbnail scores of one 16-token tile for this lane's head(s) and token n: tw holds the lane's b
// words of the tile (64-dim chunk 0, then chunk 1), M the token's absmax; -inf for a token past L.
template <int NT, int BITS>
__device__ __forceinline__ void tile_scores(const uint32_t* tw, float M, bool valid, const HeadConsts<NT>& hc,
                                            float (&sc)[NT]) {
    const v4i b0 = expand_codes<BITS>(tw);
    const v4i b1 = expand_codes<BITS>(tw + BITS / 2);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        v4i acc = {0, 0, 0, 0};
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(hc.A[t][0], b0, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(hc.A[t][1], b1, acc, 0, 0, 0);
        float Tf;
        if constexpr (BITS == 2) {
            // |sum_d Q_d (2 c_d - 3)| <= 3 * 128 * 2^22 < 2^31: exact modulo 2^32
            const uint32_t s = (uint32_t)acc.x + ((uint32_t)acc.y << 8) + ((uint32_t)acc.z << 16);
            Tf = (float)(int)(2u * s - 3u * (uint32_t)hc.sumq[t]);
        } else {
            const long long s = (long long)acc.x + ((long long)acc.y << 8) + ((long long)acc.z << 16);
            // 8-bit codes are the bytes c - 128, and 2c - 255 = 2 (c - 128) + 1
            const long long T = BITS == 8 ? 2 * s + hc.sumq[t]
                                          : 2 * s - (long long)((1 << BITS) - 1) * hc.sumq[t];
            Tf = (float)T;
        }
        sc[t] = valid ? Tf * (M * hc.kap[t]) : -INFINITY;
    }
}

// Thumbnail scores of block j for this lane's head(s) and tokens 64j + 16*T4 + n; -inf past L.
// Lane words of tile T4 are words T4*b .. T4*b + b - 1 (the storage layout of ffd.h).
template <int NT, int BITS>
__device__ __forceinline__ void block_scores(const BlockScan<BITS>& ld, int j, int lane, int L,
                                             const HeadConsts<NT>& hc, float (&sc)[NT][4]) {
    const int n = lane & 15;
    const float M[4] = {bf16_lo(ld.mm.x), bf16_hi(ld.mm.x), bf16_lo(ld.mm.y), bf16_hi(ld.mm.y)};
    uint32_t words[4 * BITS];
#pragma unroll
    for (int i = 0; i < BITS; ++i) {
        words[4 * i] = ld.w[i].x; words[4 * i + 1] = ld.w[i].y;
        words[4 * i + 2] = ld.w[i].z; words[4 * i + 3] = ld.w[i].w;
    }
#pragma unroll
    for (int T4 = 0; T4 < 4; ++T4) {
        float st[NT];
        tile_scores<NT, BITS>(&words[T4 * BITS], M[T4], 64 * j + 16 * T4 + n < L, hc, st);
#pragma unroll
        for (int t = 0; t < NT; ++t) sc[t][T4] = st[t];
    }
}

// The scan's workgroups of one KV head, the slots, and the sequences. A sequence of n blocks gets S =
// max(1, ceil(n / T)) slots, T the smallest number of blocks per slot for which all sequences fit, so
// that a ragged batch's workgroups end together: with as many slots for every sequence the longest one
// sets the end (16 sequences of 8K to 128K tokens, 8 slots each: scan 79 us, now 73). Every wave computes
// the same for itself, lane b holding sequence b; the divisions go through reciprocals because this
// chain precedes every load of the kernel. Batches of more than kBalanceMaxSeqs keep S1 slots per
// sequence. Slots past the last one used have b = -1.
struct Slot {
    int b, kvh;         // sequence, KV head
    int s, S;           // the slot's number among the sequence's S slots
    int base;           // slots of the sequences before it
    int L;              // sequence length, clamped to the capacity
};

// floor(n / d) and ceil(n / d) for 0 <= n < 2^24, quotients below 2^20; r = 1 / d to an ulp or two
__device__ __forceinline__ int floor_div(int n, int d, float r) {
    int q = (int)((float)n * r);                    // off by at most one
    q -= q * d > n ? 1 : 0;
    q += (q + 1) * d <= n ? 1 : 0;
    return q;
}
__device__ __forceinline__ int ceil_div(int n, int d, float r) { return floor_div(n + d - 1, d, r); }

// The workgroup's (sequence, KV head, slot): with the KV heads first, (kvh, at) are its grid position and at
// is the slot; in order (IN_ORDER), at numbers the workgroups by sequence, KV head and slot. Slots that are not
// used come last either way, so that a CU is not given two workgroups while another gets an empty one (5
// ragged sequences, 64 of 70 slots used: scan 25.4 us, with unused ones in between 34.8).
//
// T is chosen for the fewest rounds of `round` slots (which fill the CUs) that hold the sequences in shares of
// kFfdMaxScanBlocks, up to the grid's slots (>= B * ceil(capacity blocks / kFfdMaxScanBlocks)): a second round
// that is begun is then filled with smaller shares (5 sequences of 112K to 150K, 8 KV heads: scan 42.5 us with
// 42 slots of up to 256 blocks, 38.0 with 50 of up to 210).
template <bool IN_ORDER>
__device__ __forceinline__ Slot slot_of(const int32_t* __restrict__ seq_lens, int B, int Hkv, int S1, int round,
                                        int grid_slots, int Lcap, int kvh, int at, int lane) {
    if (B == 1 || S1 == 1 || B > kBalanceMaxSeqs) { // uniform
        int b = B == 1 ? 0 : (S1 == 1 ? at : at / S1), s = at - b * S1;
        if constexpr (IN_ORDER) {
            const int x = at / S1;
            b = x / Hkv;
            kvh = x - b * Hkv;
            s = at - x * S1;
        }
        return Slot{b, kvh, s, S1, b * S1, min(max(seq_lens[b], 0), Lcap)};
    }
    const int L = lane < B ? min(max(seq_lens[lane], 0), Lcap) : 0;
    const int n = (L + kBlock - 1) / kBlock;
    const int N = wave_sum_dpp(n), longest = (int)wave_max_dpp((float)n);
    int slots = grid_slots;
    if (grid_slots > round) {                       // uniform
        const int full = (int)((uint32_t)(n + kFfdMaxScanBlocks - 1) / kFfdMaxScanBlocks);
        const int least = wave_sum_dpp(lane < B ? max(full, 1) : 0);
        slots = min(grid_slots, round * ceil_div(least, round, __builtin_amdgcn_rcpf((float)round)));
    }
    // T lies between N / slots and what gives every sequence the same number of slots; candidates
    // lo + i step, one per lane, from coarse to fine
    const int each = floor_div(slots, B, __builtin_amdgcn_rcpf((float)B));
    int hi = min(max(ceil_div(longest, each, __builtin_amdgcn_rcpf((float)each)), 1), kFfdMaxScanBlocks);
    int lo = max(ceil_div(N, slots, __builtin_amdgcn_rcpf((float)slots)),
                 (longest + kFfdMaxScanSplits - 1) / kFfdMaxScanSplits);
    lo = min(max(lo, 1), hi);
    while (lo < hi) {
        const int step = (hi - lo + 63) >> 6, T = min(lo + lane * step, hi);
        const float rT = __builtin_amdgcn_rcpf((float)T);
        int need = 0;
        for (int b = 0; b < B; ++b) need += max(ceil_div(__builtin_amdgcn_readlane(n, b), T, rT), 1);
        const uint64_t fits = __ballot(need <= slots);      // monotonic in the lane; hi fits
        const int first = fits ? (int)__builtin_ctzll(fits) : 64;
        hi = min(lo + first * step, hi);
        lo = first > 0 ? min(lo + (first - 1) * step + 1, hi) : hi;
    }
    const int S = lane < B ? max(ceil_div(n, hi, __builtin_amdgcn_rcpf((float)hi)), 1) : 0;
    const int incl = wave_inclusive_scan(S);
    const int per_slot = IN_ORDER ? Hkv : 1;
    const uint64_t after = __ballot(incl * per_slot > at);
    if (after == 0) return Slot{-1, 0, 0, 1, 0, 0};
    const int b = (int)__builtin_ctzll(after);
    const int Sb = __builtin_amdgcn_readlane(S, b), base = __builtin_amdgcn_readlane(incl, b) - Sb;
    at -= base * per_slot;
    if constexpr (IN_ORDER) {
        kvh = floor_div(at, Sb, __builtin_amdgcn_rcpf((float)Sb));
        at -= kvh * Sb;
    }
    return Slot{b, kvh, at, Sb, base, __builtin_amdgcn_readlane(L, b)};
}

template <int NT>
struct ScanLds {
    QueryLds<NT> qs;
    alignas(16) float pm[kScanWaves][4 * NT];             // each wave's window maxima per head
    alignas(16) float sig[kFfdMaxScanBlocks][4 * NT];     // block maxima of the thumbnail scores per head
    int nkept[kScanWaves];                    // kept blocks per wave
    int next;                                 // next block to hand out
};

// ---- refinement helpers ---------------------------------------------------------------------

// One wave's loads for one 16-token tile of a kept block: int8 residual, its lane's value dwords,
// the token's absmax and the lane's RBITS code words of the tile, from which the scan scores are
// recomputed.
template <int NT, int RBITS>
struct RefineTile {
    v4i r0, r1;
    VTile vt;
    uint32_t cw[RBITS];
    uint32_t m;       // absmax bf16 bits in the low half
};

// An address every lane holds alike, moved to scalar registers: a buffer resource built from it is
// then one scalar value (the compiler cannot always see that the block number and the wave index
// are uniform, and otherwise loops over the lanes' distinct resources).
template <typename T>
__device__ __forceinline__ void* uniform_ptr(const T* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<void*>(((uint64_t)hi << 32) | lo);
}

// All five loads go through buffer resources based at the tile (the block number is wave-uniform):
// the per-lane offsets are 32-bit and shared, the per-row ones immediates, which saves the 64-bit
// address arithmetic of every row (about a tenth of the tile's instructions). The value resource
// ends at the sequence end, so value rows past it read zeros (their probability is zero).
template <int NT, int RBITS>
__device__ __forceinline__ RefineTile<NT, RBITS> load_refine_tile(const int8_t* __restrict__ resid_bh,
                                                                  const uint16_t* __restrict__ v_bh,
                                                                  const uint32_t* __restrict__ codes_bh,
                                                                  const uint16_t* __restrict__ absmax_bh,
                                                                  int j, int T4, int lane, int L) {
    RefineTile<NT, RBITS> r;
    const int tile = 4 * j + T4;
    const uint32_t lo16 = (uint32_t)lane * 16u;
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
        uniform_ptr(resid_bh + (size_t)tile * 2048), (short)0, 2048, kRawBufferWord3);
    r.r0 = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rr, (int)lo16, 0, 0);
    r.r1 = (v4i)__builtin_amdgcn_raw_buffer_load_b128(rr, (int)(lo16 + 1024u), 0, 0);
    const int vrows = __builtin_amdgcn_readfirstlane(min(max(L - 16 * tile, 0), 16));
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
        uniform_ptr(v_bh + (size_t)tile * (16 * kD)), (short)0, vrows * (2 * kD), kRawBufferWord3);
#pragma unroll
    for (int t = 0; t < 16; ++t) r.vt.v[t] = __builtin_amdgcn_raw_buffer_load_b32(rv, lane * 4 + t * (2 * kD), 0, 0);
    // tile T4 is the lane's words T4*b .. T4*b + b - 1 of block j; word w at [w / 4][lane][w % 4]
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        uniform_ptr(codes_bh + (size_t)j * (256 * RBITS)), (short)0, 1024 * RBITS, kRawBufferWord3);
    if constexpr (RBITS == 2) {
        const auto w = __builtin_amdgcn_raw_buffer_load_b64(rc, (int)(lo16 + (T4 >> 1) * 1024u + (T4 & 1) * 8u), 0, 0);
        r.cw[0] = w[0]; r.cw[1] = w[1];
    } else {
#pragma unroll
        for (int i = 0; i < RBITS / 4; ++i) {
            const auto w = __builtin_amdgcn_raw_buffer_load_b128(rc, (int)(lo16 + (T4 * (RBITS / 4) + i) * 1024u), 0, 0);
            r.cw[4 * i] = w[0]; r.cw[4 * i + 1] = w[1]; r.cw[4 * i + 2] = w[2]; r.cw[4 * i + 3] = w[3];
        }
    }
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        uniform_ptr(absmax_bh + (size_t)j * 64), (short)0, 128, kRawBufferWord3);
    r.m = __builtin_amdgcn_raw_buffer_load_b16(ra, ((lane & 15) * 4 + T4) * 2, 0, 0);
    return r;
}

template <int NT>
struct RefineLds {
    QueryLds<NT> qs;
    int4 rec[kRefineRecords + 1];        // the scan's records, .x their prefix on the line
    int unit[2];                         // the next unit, by turns
    int4 list[kRefineChunk];             // staged kept blocks: j | keep bits << 24, group, sequence length
    TileP<NT> tp[kRefineWaves];
    EpilogueLds<NT, kRefineWaves> epi;
};

}  // namespace

// ================================================================================================
// Scan: b-bit thumbnail scan and pseudo-max, then the keep decisions; the kept list (or, for the
// top-k rule, every block's scores) to the workspace.
// Grid (Hkv, slots) of kScanWaves-wave workgroups, or slots * Hkv in one dimension where scan_in_order; slot s
// of the S given to a sequence (slot_of) scans blocks [s * bps, (s + 1) * bps) of one (sequence, KV head),
// bps = ceil(nblk / S) <= kFfdMaxScanBlocks;
// its waves take the blocks one at a time from an LDS counter and keep kRing blocks in flight each.
// ================================================================================================
// Blocks in flight per wave, fewer for the wider thumbnails (whose blocks are 2x and 4x larger).
template <int BITS> constexpr int scan_ring() { return BITS == 2 ? kRing2 : 2; }

// Adds the residual term of Eq. 4 to the thumbnail scores sc of block j (the refined logits of its
// tokens, computed exactly as the refinement kernel computes them).
template <int NT>
__device__ __forceinline__ void add_residual_term(const int8_t* __restrict__ resid_bh, uint2 mm, int j,
                                                  int lane, const HeadConsts<NT>& hc, float (&sc)[NT][4]) {
    const float M[4] = {bf16_lo(mm.x), bf16_hi(mm.x), bf16_lo(mm.y), bf16_hi(mm.y)};
    v4i r[4][2];
#pragma unroll
    for (int T4 = 0; T4 < 4; ++T4) {
        const v4i* rp = reinterpret_cast<const v4i*>(resid_bh) + (size_t)(4 * j + T4) * 128 + lane;
        r[T4][0] = rp[0];
        r[T4][1] = rp[64];
    }
#pragma unroll
    for (int T4 = 0; T4 < 4; ++T4) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            v4i acc = {0, 0, 0, 0};
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(hc.A[t][0], r[T4][0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(hc.A[t][1], r[T4][1], acc, 0, 0, 0);
            const float R = fmaf(65536.f, (float)acc.z, fmaf(256.f, (float)acc.y, (float)acc.x));
            const float sct = sc[t][T4];
            sc[t][T4] = sct == -INFINITY ? -INFINITY : fmaf(R, M[T4] * hc.kap2[t], sct);
        }
    }
}

// Workgroups per CU the registers must allow: two, so that a grid slightly larger than the CU count
// (S1 rounded up) runs in one wave of workgroups; the 8-bit blocks need more registers.
template <int BITS> constexpr int scan_occupancy() { return BITS == 8 ? 1 : 2; }

template <int NT, int BITS, int MODE>
__global__ __launch_bounds__(kScanThreads, scan_occupancy<BITS>()) void ffd_scan_kernel(ScanArgs a) {
    constexpr bool kTopK = MODE == kSelTopK;
    constexpr int kRing = scan_ring<BITS>();
    __shared__ ScanLds<NT> sm;
    constexpr bool kInOrder = scan_in_order(BITS);
    const int at = kInOrder ? (int)blockIdx.x : (int)(blockIdx.y + kSlotGridY * blockIdx.z);
    if (!kInOrder && at >= a.grid_slots) return;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int g = lane >> 4, n = lane & 15;
    const Slot sl = slot_of<kInOrder>(a.seq_lens, a.B, a.Hkv, a.S1, a.round_slots, a.grid_slots, a.Lcap, blockIdx.x, at,
                                      lane);
    const int b = sl.b, kvh = sl.kvh, s = sl.s, S = sl.S, L = sl.L;
    // records in (group, split) order; a slot that is not used holds no block and begins no group
    const size_t rec = kInOrder ? (size_t)at : b < 0 ? (size_t)at * a.Hkv + blockIdx.x
                                                     : (size_t)sl.base * a.Hkv + (size_t)kvh * S + s;
    if (b < 0) {                                    // uniform
        if constexpr (!kTopK) {
            if (tid == 0) a.info[rec] = make_int4(0, 0, 0, 1 | (1 << kInfoSplitBits));
        }
        return;
    }
    const int G = a.G, hq0 = kvh * G;
    const size_t bh = (size_t)b * a.Hkv + kvh;
    const int nblk = (L + kBlock - 1) / kBlock;
    const int nblk_cap = a.Lcap / kBlock;
    const int bps = (nblk + S - 1) / S;
    const int jb = min(s * bps, nblk), je = min(jb + bps, nblk);
    // this workgroup's record for the refinement, and the group's entry of the merge table (no rows
    // until the refinement meets a kept block)
    auto write_record = [&](int kept) {
        if (tid == 0) a.info[rec] = make_int4(kept, L, (int)bh, s | (S << kInfoSplitBits));
        if (tid == 0 && s == 0) a.table[bh] = make_int2(0, -1);
        if (tid == 0 && s == 0 && bh == 0) *a.ticket = 0;
    };
    if (jb >= je && (kTopK || !a.mask)) {       // nothing to scan (short sequence), nothing to clear
        if constexpr (!kTopK) {
            write_record(0);
            if (a.m_tilde && s == 0 && tid < G) a.m_tilde[(size_t)b * a.Hq + hq0 + tid] = -INFINITY;   // L = 0
        }
        return;
    }

    const uint32_t* codes_bh = a.codes + bh * (size_t)a.Lcap * (4 * BITS);
    const uint16_t* absmax_bh = a.absmax + bh * (size_t)a.Lcap;

    // The stream reads through buffer resources whose ranges end at block je, so a request for a
    // block >= je reads zeros without touching memory (the hardware range check of a raw buffer):
    // every load is issued unconditionally, and uniform control flow lets the compiler wait for
    // exactly the load it needs instead of draining every load in flight (which a conditional load
    // made it do). Offsets and sizes are unsigned 32-bit: at most 2^18 blocks of 8 KiB.
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(codes_bh), (short)0, (int)((uint32_t)je * (1024u * BITS)), kRawBufferWord3);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(absmax_bh), (short)0, (int)((uint32_t)je * 128u), kRawBufferWord3);
    // Work distribution: wave w starts with blocks jb + kRing w + r (r < kRing), then takes the next
    // block from an LDS counter each time it scores one, so the waves of a CU finish together however
    // its memory requests are served (a CU serves its oldest waves first: with fixed shares, the
    // workgroups of one CU ended up to 12 us apart at 4 x 128K).
    int js[kRing];                                  // block held by each ring slot (>= je: none)
#pragma unroll
    for (int r = 0; r < kRing; ++r) js[r] = jb + kRing * wave + r;

    // Order of requests: queries, the window blocks of the first pseudo-max pass (clamped to valid
    // blocks), the first ring round. Each wave scores its window blocks on its own before its first
    // block (the refined logits: after the stream, with the window blocks' residual tiles) and only
    // writes their maxima to LDS; every keep decision waits for the end of the stream, where the
    // pseudo-max is known, so no wave waits on another before or during its stream (a
    // workgroup-wide window pass before the stream held every wave until the slowest one's window
    // blocks had arrived behind the whole chip's first round: 6 us at the median, 20 us at worst at
    // 4 x 128K). Until then a block costs G floats of LDS.
    const uint32_t qw = load_query_word<NT>(a.q, (size_t)b * a.Hq + hq0, G, wave, lane);
    const int jlast = max(nblk, 1) - 1;
    const int sink_end = min(a.n_sink, L);
    const int loc_beg = max(0, L - a.n_local);
    const int sink_blk_end = (sink_end + kBlock - 1) / kBlock;
    const int loc_blk_beg = max(loc_beg / kBlock, sink_blk_end);
    const int npm = sink_blk_end + max(nblk - loc_blk_beg, 0);
    auto pm_block = [&](int idx) { return idx < sink_blk_end ? idx : loc_blk_beg + (idx - sink_blk_end); };
    auto win_block = [&](int idx) { return min(pm_block(min(idx, max(npm, 1) - 1)), jlast); };
    constexpr bool kEarlyWindows = MODE == kSelThumbnailPM;
    BlockScan<BITS> win;                            // wave w's window block of the current pass
    auto load_window = [&](int base) { win = load_block_scan<BITS>(codes_bh, absmax_bh, win_block(base + wave), lane); };
    if constexpr (kEarlyWindows) load_window(0);
    BlockScan<BITS> ring[kRing];
#pragma unroll
    for (int i = 0; i < kRing; ++i) ring[i] = load_block_scan_rsrc<BITS>(rc, ra, min(js[i], je), lane);
    if (tid == 0) sm.next = jb + kScanWaves * kRing;   // visible after the barriers below
    if constexpr (MODE == kSelRefinedPM) load_window(0);

    HeadConsts<NT> hc;
    build_query_consts<NT>(sm.qs, qw, G, a.scale, thumb_top_level(BITS), wave, lane, hc);

    // ---- scan (Alg. 1): block maxima sigma per head, and the pseudo-max's window maxima -------
    float pm[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) pm[t] = -INFINITY;
    auto window_max = [&](const float (&sc)[NT][4], int j) {     // over the window tokens of block j
#pragma unroll
        for (int T4 = 0; T4 < 4; ++T4) {
            const int tok = 64 * j + 16 * T4 + n;
            const bool in_win = tok < L && (tok < sink_end || tok >= loc_beg);
#pragma unroll
            for (int t = 0; t < NT; ++t) pm[t] = fmaxf(pm[t], in_win ? sc[t][T4] : -INFINITY);
        }
    };
    auto window_pass = [&](int base) {              // wave w: window block base + w
        const int idx = base + wave;
        if (idx >= npm) return;                     // wave-uniform
        const int j = pm_block(idx);
        float sc[NT][4];
        block_scores<NT, BITS>(win, j, lane, L, hc, sc);
        if constexpr (MODE == kSelRefinedPM)
            add_residual_term<NT>(a.resid + bh * (size_t)a.Lcap * kD, win.mm, j, lane, hc, sc);
        window_max(sc, j);
    };
    auto consume = [&](const BlockScan<BITS>& blk, int j) {
        float sc[NT][4];
        block_scores<NT, BITS>(blk, j, lane, L, hc, sc);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            // + 0 turns a -0 score (a zero key) into +0, so that equal scores compare equal
            const float sig = row16_max(fmaxf(fmaxf(sc[t][0], sc[t][1]), fmaxf(sc[t][2], sc[t][3]))) + 0.f;
            if constexpr (kTopK) {
                if (n == 0 && hc.live[t]) a.sigma[(bh * (size_t)nblk_cap + j) * G + 4 * t + g] = sig;
            } else {
                if (n == 0) sm.sig[j - jb][4 * t + g] = sig;
            }
        }
    };
    if constexpr (kEarlyWindows) window_pass(0);     // its block arrives ahead of the first round
    // Each slot in turn: take the next block number (its LDS round trip hides behind the scoring),
    // score the slot's block if it has one, refill the slot. The loop ends once a whole round has
    // taken no block below je: every slot then holds none, and its last loads read no memory.
    for (bool more = true; more;) {                 // wave-uniform
        more = false;
#pragma unroll
        for (int r = 0; r < kRing; ++r) {
            int jn = 0;
            if (lane == 0) jn = atomicAdd(&sm.next, 1);
            jn = __builtin_amdgcn_readfirstlane(jn);
            if (js[r] < je) consume(ring[r], js[r]);
            ring[r] = load_block_scan_rsrc<BITS>(rc, ra, min(jn, je), lane);
            js[r] = jn;
            more |= jn < je;
        }
    }

    if constexpr (kTopK) return;                // the top-k rule compares block scores with each other

    // ---- pseudo-max over the sink and local windows (Eq. 3): the first pass unless done during
    // the stream, further passes (wide windows) loaded now -------------------------------------
    if constexpr (!kEarlyWindows) window_pass(0);
    for (int base = kScanWaves; base < npm; base += kScanWaves) {
        load_window(base);
        window_pass(base);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        pm[t] = row16_max(pm[t]);
        if (n == 0) sm.pm[wave][4 * t + g] = pm[t];
    }
    __syncthreads();

    // ---- decide (Eq. 1) per (head, block): keep iff sigma >= m~ - delta; the workgroup's kept
    // list in block order, its length and the optional mask -----------------------------------
    float thr[4 * NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float4 m = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
#pragma unroll
        for (int w = 0; w < kScanWaves; ++w) {
            const float4 p = reinterpret_cast<const float4*>(sm.pm[w])[t];
            m.x = fmaxf(m.x, p.x); m.y = fmaxf(m.y, p.y); m.z = fmaxf(m.z, p.z); m.w = fmaxf(m.w, p.w);
        }
        thr[4 * t] = m.x - a.delta;                     // -inf when both windows are empty
        thr[4 * t + 1] = m.y - a.delta;
        thr[4 * t + 2] = m.z - a.delta;
        thr[4 * t + 3] = m.w - a.delta;
    }
    if (a.m_tilde && s == 0 && tid < G) {
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < kScanWaves; ++w) m = fmaxf(m, sm.pm[w][tid]);
        a.m_tilde[(size_t)b * a.Hq + hq0 + tid] = m;
    }
    // lane i of wave w decides block jb + 64 w + i (bps <= kFfdMaxScanBlocks <= 64 kScanWaves)
    static_assert(kFfdMaxScanBlocks <= 64 * kScanWaves, "one decision per lane");
    uint32_t bits = 0;
    const int jl = jb + 64 * wave + lane;
    if (jl < je) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float4 sg = reinterpret_cast<const float4*>(sm.sig[jl - jb])[t];
            bits |= ((uint32_t)(sg.x >= thr[4 * t]) | (uint32_t)(sg.y >= thr[4 * t + 1]) << 1 |
                     (uint32_t)(sg.z >= thr[4 * t + 2]) << 2 | (uint32_t)(sg.w >= thr[4 * t + 3]) << 3) << (4 * t);
        }
        bits &= (1u << G) - 1u;                         // heads past G are never kept
        if (a.mask)
            for (int h = 0; h < G; ++h) a.mask[((size_t)b * a.Hq + hq0 + h) * nblk_cap + jl] = (bits >> h) & 1u;
    }
    const uint64_t kept = __ballot(bits != 0);
    const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
    if (lane == 0) sm.nkept[wave] = __popcll(kept);
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kScanWaves; ++w) {
        const int c = sm.nkept[w];
        before += w < wave ? c : 0;
        total += c;
    }
    if (bits != 0) a.lists[bh * (size_t)nblk_cap + jb + before + below] = (uint32_t)jl | (bits << 24);
    write_record(total);

    // Mask entries past the end of the sequence are zero (spread over the scan workgroups).
    if (a.mask) {
        for (int j = nblk + s * kScanThreads + tid; j < nblk_cap; j += S * kScanThreads)
            for (int h = 0; h < G; ++h) a.mask[((size_t)b * a.Hq + hq0 + h) * nblk_cap + j] = 0;
    }
}

// ================================================================================================
// Fused top-delta decode: one workgroup per (sequence, KV head, split s) of kScanWaves waves, the splits given to
// the sequences by their lengths (slot_of). Workgroup s of the S1 of a (sequence, KV head) owns the blocks j = s +
// S1 i (i < cnt) of its group, an interleaved share, so the kept blocks of a group (windows, planted clusters)
// spread evenly over its S1 workgroups. It
//  1. streams the thumbnail codes of its blocks (waves take block numbers i from an LDS counter,
//     kRing blocks in flight each) and keeps each block's per-head maximum score in LDS, while each
//     wave also scores its share of the pseudo-max window blocks (Alg. 1; Eq. 3);
//  2. decides per (head, block): keep iff sigma >= m~ - delta (Eq. 1), the kept blocks (with their
//     keep bits) forming a list in LDS, in block order;
//  3. refines and attends its own kept blocks (Eq. 4; online softmax and PV): wave w takes tile
//     w % 4 of the kept entries w / 4, w / 4 + 2, ..., with RING tiles in flight; the
//     thumbnail term of each kept tile is recomputed from its codes with the same integer MFMA and
//     fp32 operations as in step 1, so it equals the value the decision used;
//  4. combines the eight waves' states into one partial state per head, or,
//     when it is the group's only workgroup (S1 == 1), writes the bf16 output and lse itself.
// No workgroup waits for another: each needs only its own blocks, the window blocks (re-read by
// every workgroup of the group, L2-resident) and the query.
// ================================================================================================
template <int NT>
struct FusedLds {
    QueryLds<NT> qs;
    alignas(16) float pm[kScanWaves][4 * NT];             // each wave's window maxima per head
    alignas(16) float sig[kFfdMaxScanBlocks][4 * NT];     // block maxima per head, by share index i
    uint32_t list[kFfdMaxScanBlocks];                     // kept blocks j | keep bits << 24
    int nkept[kScanWaves];
    int next;                                             // next share index to hand out
    TileP<NT> tp[kScanWaves];
    EpilogueLds<NT, kScanWaves> epi;
};

// RING refinement tiles in flight per wave. With one, a workgroup of eight heads (NT = 2; 2- and 4-bit codes) needs
// 117 to 124 registers a lane, so that two fit a CU (four waves per SIMD); with two, 147 to 150, and one does. Up to
// four heads two workgroups fit with two tiles (120 to 122 registers; 8-bit codes, 134, are held to 128: 16 x 8K, 512
// workgroups, 37.3 -> 32.3 us).
template <int NT, int BITS, int MODE, int RING>
__global__ __launch_bounds__(kScanThreads, RING == 1 || (NT == 1 && BITS == 8) ? 4 : 1) void ffd_decode_kernel(FusedArgs a) {
    static_assert(MODE == kSelThumbnailPM || MODE == kSelRefinedPM, "top-delta modes only");
    constexpr int kRing = scan_ring<BITS>();
    __shared__ FusedLds<NT> sm;
    // KV heads first, turned by one with every 64 workgroups and so that workgroups i and i + 256, which share a CU,
    // are of heads far apart: workgroups go to the XCDs in turn, so with eight heads unturned each XCD would hold one
    // head, and a head that keeps most of its blocks would end late on the 32 CUs it has (one such head: 1 x 64K
    // 34.3 us, turned 23.5, in (sequence, KV head, slot) order 21.6 to 23.5; 4 x 32K 58.4, 35.2, 43.0). Eight
    // neighbouring slots of a head still share an XCD's L2 for its window blocks: with even heads the order makes
    // 16 x 8K 20.7 us, unturned 20.8, in (sequence, KV head, slot) order 22.9.
    const int t = blockIdx.y + kSlotGridY * blockIdx.z, i = t * a.Hkv;
    int kvh = (int)blockIdx.x + (int)(((unsigned)i / 64 + (unsigned)a.turn * ((unsigned)i / 256)) % (unsigned)a.Hkv);
    kvh -= kvh >= a.Hkv ? a.Hkv : 0;
    if (t >= a.grid_slots) return;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int g = lane >> 4, n = lane & 15;
    const Slot sl = slot_of<false>(a.seq_lens, a.B, a.Hkv, a.S1, a.round_slots, a.grid_slots, a.Lcap, kvh, t, lane);
    if (sl.b < 0) return;                           // uniform: a slot no sequence needs
    const int b = sl.b, s = sl.s, S1 = sl.S, L = sl.L;
    const int G = a.G, hq0 = kvh * G;
    const size_t row = (size_t)sl.base * a.Hkv + (size_t)kvh * S1 + s;       // partials, in rows of G heads
    const size_t bh = (size_t)b * a.Hkv + kvh;
    const size_t hrow0 = (size_t)b * a.Hq + hq0;             // [B, Hq] row of the group's head 0
    const int nblk = (L + kBlock - 1) / kBlock;
    const int nblk_cap = a.Lcap / kBlock;
    const int cnt = nblk > s ? (nblk - 1 - s) / S1 + 1 : 0;  // blocks of this workgroup
    uint16_t* out_h = a.out ? a.out + hrow0 * kD : nullptr;
    float* lse_h = a.out && a.lse ? a.lse + hrow0 : nullptr;

    if (a.table && s == 0 && tid == 0) a.table[bh] = make_int2((int)row, (int)row + S1 - 1);
    // Mask entries past the end of the sequence are zero (spread over the group's workgroups).
    if (a.mask) {
        for (int j = nblk + s * kScanThreads + tid; j < nblk_cap; j += S1 * kScanThreads)
            for (int h = 0; h < G; ++h) a.mask[(hrow0 + h) * nblk_cap + j] = 0;
    }
    if (cnt == 0) {                                 // uniform: nothing to scan
        if (out_h) {                                // an empty sequence: out = 0, lse = -inf
            for (int idx = tid; idx < G * kD; idx += kScanThreads) out_h[idx] = 0;
            if (lse_h && tid < G) lse_h[tid] = -INFINITY;
        } else if (tid < G) {
            a.part_m[row * G + tid] = -INFINITY;     // an empty partial state
        }
        if (a.m_tilde && s == 0 && tid < G) a.m_tilde[hrow0 + tid] = -INFINITY;   // L = 0
        return;
    }

    const uint32_t* codes_bh = a.codes + bh * (size_t)a.Lcap * (4 * BITS);
    const uint16_t* absmax_bh = a.absmax + bh * (size_t)a.Lcap;

    // The stream reads through buffer resources whose ranges end after this workgroup's last block
    // s + S1 (cnt - 1): a request for an index i >= cnt (block s + S1 i beyond it) reads zeros
    // without touching memory, so every load is issued unconditionally (uniform control flow keeps
    // the compiler's in-order vmcnt accounting exact). Offsets are unsigned 32-bit: at most 2^18 + S1
    // blocks of 8 KiB.
    const uint32_t jend = (uint32_t)(s + S1 * (cnt - 1)) + 1u;
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(codes_bh), (short)0, (int)(jend * (1024u * BITS)), kRawBufferWord3);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(absmax_bh), (short)0, (int)(jend * 128u), kRawBufferWord3);
    auto block_of = [&](int i) { return s + S1 * min(i, cnt); };     // i >= cnt: past the range
    int is[kRing];                                  // share index held by each ring slot (>= cnt: none)
#pragma unroll
    for (int r = 0; r < kRing; ++r) is[r] = kRing * wave + r;

    // Requests: queries, the first window blocks, the first ring round.
    const uint32_t qw = load_query_word<NT>(a.q, (size_t)b * a.Hq + hq0, G, wave, lane);
    const int jlast = nblk - 1;
    const int sink_end = min(a.n_sink, L);
    const int loc_beg = max(0, L - a.n_local);
    const int sink_blk_end = (sink_end + kBlock - 1) / kBlock;
    const int loc_blk_beg = max(loc_beg / kBlock, sink_blk_end);
    const int npm = sink_blk_end + max(nblk - loc_blk_beg, 0);
    auto pm_block = [&](int idx) { return idx < sink_blk_end ? idx : loc_blk_beg + (idx - sink_blk_end); };
    auto win_block = [&](int idx) { return min(pm_block(min(idx, max(npm, 1) - 1)), jlast); };
    constexpr bool kEarlyWindows = MODE == kSelThumbnailPM;
    BlockScan<BITS> win;
    auto load_window = [&](int base) { win = load_block_scan<BITS>(codes_bh, absmax_bh, win_block(base + wave), lane); };
    if constexpr (kEarlyWindows) load_window(0);
    BlockScan<BITS> ring[kRing];
#pragma unroll
    for (int r = 0; r < kRing; ++r) ring[r] = load_block_scan_rsrc<BITS>(rc, ra, block_of(is[r]), lane);
    if (tid == 0) sm.next = kScanWaves * kRing;
    if constexpr (MODE == kSelRefinedPM) load_window(0);

    HeadConsts<NT> hc;
    build_query_consts<NT>(sm.qs, qw, G, a.scale, thumb_top_level(BITS), wave, lane, hc);

    // ---- scan (Alg. 1): block maxima per head, and the window maxima of the pseudo-max ---------
    float pm[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) pm[t] = -INFINITY;
    auto window_pass = [&](int base) {
        const int idx = base + wave;
        if (idx >= npm) return;                     // wave-uniform
        const int j = pm_block(idx);
        float sc[NT][4];
        block_scores<NT, BITS>(win, j, lane, L, hc, sc);
        if constexpr (MODE == kSelRefinedPM)
            add_residual_term<NT>(a.resid + bh * (size_t)a.Lcap * kD, win.mm, j, lane, hc, sc);
#pragma unroll
        for (int T4 = 0; T4 < 4; ++T4) {
            const int tok = 64 * j + 16 * T4 + n;
            const bool in_win = tok < L && (tok < sink_end || tok >= loc_beg);
#pragma unroll
            for (int t = 0; t < NT; ++t) pm[t] = fmaxf(pm[t], in_win ? sc[t][T4] : -INFINITY);
        }
    };
    auto consume = [&](const BlockScan<BITS>& blk, int i) {
        float sc[NT][4];
        block_scores<NT, BITS>(blk, s + S1 * i, lane, L, hc, sc);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float sig = row16_max(fmaxf(fmaxf(sc[t][0], sc[t][1]), fmaxf(sc[t][2], sc[t][3])));
            if (n == 0) sm.sig[i][4 * t + g] = sig;
        }
    };
    if constexpr (kEarlyWindows) window_pass(0);
    for (bool more = true; more;) {                 // wave-uniform
        more = false;
#pragma unroll
        for (int r = 0; r < kRing; ++r) {
            int in = 0;
            if (lane == 0) in = atomicAdd(&sm.next, 1);
            in = __builtin_amdgcn_readfirstlane(in);
            if (is[r] < cnt) consume(ring[r], is[r]);
            ring[r] = load_block_scan_rsrc<BITS>(rc, ra, block_of(in), lane);
            is[r] = in;
            more |= in < cnt;
        }
    }
    if constexpr (!kEarlyWindows) window_pass(0);
    for (int base = kScanWaves; base < npm; base += kScanWaves) {
        load_window(base);
        window_pass(base);
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        pm[t] = row16_max(pm[t]);
        if (n == 0) sm.pm[wave][4 * t + g] = pm[t];
    }
    __syncthreads();

    // ---- decide (Eq. 1): keep iff sigma >= m~ - delta; the kept list in LDS, in block order ----
    float thr[4 * NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        float4 m = make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
#pragma unroll
        for (int w = 0; w < kScanWaves; ++w) {
            const float4 p = reinterpret_cast<const float4*>(sm.pm[w])[t];
            m.x = fmaxf(m.x, p.x); m.y = fmaxf(m.y, p.y); m.z = fmaxf(m.z, p.z); m.w = fmaxf(m.w, p.w);
        }
        thr[4 * t] = m.x - a.delta;                 // -inf when both windows are empty
        thr[4 * t + 1] = m.y - a.delta;
        thr[4 * t + 2] = m.z - a.delta;
        thr[4 * t + 3] = m.w - a.delta;
    }
    if (a.m_tilde && s == 0 && tid < G) {
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < kScanWaves; ++w) m = fmaxf(m, sm.pm[w][tid]);
        a.m_tilde[hrow0 + tid] = m;
    }
    // lane l of wave w decides share index 64 w + l (cnt <= kFfdMaxScanBlocks <= 64 kScanWaves)
    static_assert(kFfdMaxScanBlocks <= 64 * kScanWaves, "one decision per lane");
    uint32_t bits = 0;
    const int il = 64 * wave + lane;
    const int jl = s + S1 * il;
    if (il < cnt) {
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const float4 sg = reinterpret_cast<const float4*>(sm.sig[il])[t];
            bits |= ((uint32_t)(sg.x >= thr[4 * t]) | (uint32_t)(sg.y >= thr[4 * t + 1]) << 1 |
                     (uint32_t)(sg.z >= thr[4 * t + 2]) << 2 | (uint32_t)(sg.w >= thr[4 * t + 3]) << 3) << (4 * t);
        }
        bits &= (1u << G) - 1u;                     // heads past G are never kept
        if (a.mask)
            for (int h = 0; h < G; ++h) a.mask[(hrow0 + h) * nblk_cap + jl] = (bits >> h) & 1u;
    }
    const uint64_t kept = __ballot(bits != 0);
    const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(kept >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)kept, 0u));
    if (lane == 0) sm.nkept[wave] = __popcll(kept);
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kScanWaves; ++w) {
        const int c = sm.nkept[w];
        before += w < wave ? c : 0;
        total += c;
    }
    if (bits != 0) sm.list[before + below] = (uint32_t)jl | (bits << 24);
    __syncthreads();

    // ---- refine (Eq. 4) and attend the kept blocks: wave w, tile T4 = w % 4, entries w / 4 + 2k --
    const int T4 = wave & 3, par = wave >> 2;
    const int mine = total > par ? (total - par + 1) / 2 : 0;
    const int8_t* resid_bh = a.resid + bh * (size_t)a.Lcap * kD;
    const uint16_t* v_bh = a.v + bh * (size_t)a.Lcap * kD;
    PvAcc<NT> pv;
    pv.zero();
    float m_run[NT], l_part[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) { m_run[t] = -INFINITY; l_part[t] = 0.f; }
    TileP<NT>& tp = sm.tp[wave];
    auto entry = [&](int k) { return sm.list[par + 2 * min(k, mine - 1)]; };
    auto attend = [&](const RefineTile<NT, BITS>& rt, int j, uint32_t kb) {
        float z[NT];
        bool keep[NT];
        const float Mt = bf16_to_f32((uint16_t)rt.m);
        float shat[NT];                             // Eq. 4's first term: the scan scores, recomputed
        tile_scores<NT, BITS>(rt.cw, Mt, 64 * j + 16 * T4 + n < L, hc, shat);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            v4i acc = {0, 0, 0, 0};
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(hc.A[t][0], rt.r0, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(hc.A[t][1], rt.r1, acc, 0, 0, 0);
            const float R = fmaf(65536.f, (float)acc.z, fmaf(256.f, (float)acc.y, (float)acc.x));
            const float sct = shat[t];
            z[t] = sct == -INFINITY ? -INFINITY : fmaf(R, Mt * hc.kap2[t], sct);
            keep[t] = (kb >> (4 * t + g)) & 1u;
        }
        softmax_tile<NT>(z, keep, m_run, l_part, tp, g, n);
        wave_lds_fence();
        pv_tile<NT>(pv, tp, rt.vt);
        wave_lds_fence();
    };
    if (mine > 0) {                                 // wave-uniform
        RefineTile<NT, BITS> rr[RING];
#pragma unroll
        for (int r = 0; r < RING; ++r)
            rr[r] = load_refine_tile<NT, BITS>(resid_bh, v_bh, codes_bh, absmax_bh,
                                               (int)(entry(r) & 0xffffffu), T4, lane, L);
        for (int k0 = 0; k0 < mine; k0 += RING) {
#pragma unroll
            for (int r = 0; r < RING; ++r) {
                const int k = k0 + r;
                if (k < mine) {
                    const uint32_t e = entry(k);
                    attend(rr[r], (int)(e & 0xffffffu), e >> 24);
                }
                // the last round's refills re-read the wave's last tile (clamped): still cached
                rr[r] = load_refine_tile<NT, BITS>(resid_bh, v_bh, codes_bh, absmax_bh,
                                                   (int)(entry(k + RING) & 0xffffffu), T4, lane, L);
            }
        }
    }

    write_partials<NT, kScanWaves>(sm.epi, pv, m_run, l_part, wave, lane, G, row * G, 1,
                                   a.part_m, a.part_l, a.part_acc, out_h, lse_h);
}

// ================================================================================================
// Refinement: Eq. 4 on the kept blocks, online softmax and PV, one partial state per workgroup and
// KV group it meets. The kept blocks of all groups, in (group, block) order, form one line on which
// every group is preceded by kGroupCost positions that hold no block (the price of beginning a group:
// its query constants and one more partial state); workgroup w of W takes the positions
// [w T / W, (w + 1) T / W) of the T in all, so shares are equal whatever the groups hold and cross
// group boundaries where they must. Its partial of group x goes to row w + x: along the line w + x
// grows with every change of w or x, so no two partials share a row and a group's rows are consecutive.
// Bound: HBM (the gather of the kept blocks arrives at 5.2 to 5.8 TB/s). A whole number of workgroups
// per group, and one fixed share each, took 397 us where half of 16 sequences of 8K to 128K tokens is
// kept (2.1 GB; the step 477 us); equal shares and units from a counter take 372 us (446 us). At 4 x
// 128K, 6 % kept, the step went from 58.5 to 56.9 us.
// ================================================================================================
// Exclusive prefix, on the line, of the scan's records in front of the refinement when there are more
// than a workgroup keeps in LDS: one workgroup; info[i].x becomes the prefix of record i, info[0].x
// (whose prefix is 0) the line's length.
__global__ __launch_bounds__(kOffsetThreads) void ffd_offsets_kernel(int4* info, int nent) {
    __shared__ int wsum[2][kOffsetThreads / 64];
    int run = 0, half = 0;
    for (int i0 = 0; i0 < nent; i0 += kOffsetThreads) {
        const int i = i0 + (int)threadIdx.x;
        int cost = 0;
        if (i < nent) {
            const int4 e = info[i];
            cost = e.x + ((e.w & kInfoSplitMask) == 0 ? kGroupCost : 0);
        }
        int tot = 0;
        const int before = wg_exclusive_scan<kOffsetThreads / 64>(cost, wsum[half], &tot);
        half ^= 1;
        if (i > 0 && i < nent) info[i].x = run + before;
        run += tot;
    }
    if (threadIdx.x == 0) info[0].x = run;
}

template <int NT, int RBITS>
__global__ __launch_bounds__(kRefineThreads, 1) void ffd_refine_kernel(RefineArgs a) {
    __shared__ RefineLds<NT> sm;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int g = lane >> 4, n = lane & 15;
    constexpr int kPar = kRefineWaves / 4;          // waves per tile index
    const int T4 = wave & 3, par = wave >> 2;       // tile T4 of the staged entries par, par + kPar, ...
    const int G = a.G, nent = a.nent;
    const int nblk_cap = a.Lcap / kBlock;

    // ---- the line: records and their prefix. Every wave loads all records (64 neighbouring ones at a time:
    // with a run of 16 records per lane, so that each request met 64 cache lines, 400 records cost 1.1 us more:
    // 6 x 128K, 8 KV heads, 27.1 -> 26.1 us; up to 256 records, four per lane, the same) and writes them to LDS
    // with their prefix: identical values, so each wave reads back its own writes and no workgroup barrier is
    // needed.
    const bool cached = nent <= kRefineRecords;
    int T = 0;
    auto load_records = [&](auto per) {
        constexpr int kPer = decltype(per)::value;
        int4 e[kPer];
        int cost[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) e[k] = 64 * k + lane < nent ? a.info[64 * k + lane] : make_int4(0, 0, 0, 1);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            cost[k] = e[k].x + ((e[k].w & kInfoSplitMask) == 0 ? kGroupCost : 0);
            e[k].x = wave_inclusive_scan(cost[k]);
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int sum = __builtin_amdgcn_readlane(e[k].x, 63);
            e[k].x += T - cost[k];
            if (64 * k + lane < nent) sm.rec[64 * k + lane] = e[k];
            T += sum;
        }
        if (lane == 0) sm.rec[nent].x = T;
        wave_lds_fence();
    };
    if (nent <= 64 * 4) load_records(std::integral_constant<int, 4>{});
    else if (nent <= 64 * 8) load_records(std::integral_constant<int, 8>{});
    else if (cached) load_records(std::integral_constant<int, kRefineRecords / 64>{});
    else T = __builtin_amdgcn_readfirstlane(a.info[0].x);
    auto prefix = [&](int i) { return cached ? sm.rec[i].x : (i == 0 ? 0 : (i == nent ? T : a.info[i].x)); };
    // U units on the line, usually one of equal length per workgroup (fewer where the line is shorter
    // than that). Long shares are worked as units from a counter: the chip's memory serves its XCDs at
    // rates that differ by up to a fifth (workgroups of equal shares of 310 blocks ended between 324 and
    // 411 us), and a fixed share ends with the slowest; but only where there is room for two units per workgroup
    // (kUnitBlocks). The first W units, one per workgroup, then cover
    // kFirstShare of the line, and the rest shrinks linearly to a ninth of its first length, so that the
    // workgroups end together. Which workgroup takes a unit does not enter the results.
    if (T == 0) return;                             // uniform
    const int U1 = min(a.W, T);
    const bool queue = T / a.W >= 2 * kUnitBlocks && a.max_units >= 2 * a.W;
    const int U = queue ? min(a.max_units, T / kUnitBlocks) : U1;
    const double T1 = queue ? floor((double)T * kFirstShare) : (double)T;
    // first position of unit u <= U; every unit has at least one (queued ones: 0.2 (1 - kFirstShare)
    // kUnitBlocks = 1.7 or more). Products stay below 2^52, so that whole results are exact.
    auto first_of = [&](int u) {
        if (u <= U1) return (int)floor((double)u * T1 / (double)U1);
        const double v = (double)(u - U1) / (double)(U - U1);
        return u >= U ? T : (int)(T1 + floor(((double)T - T1) * v * (1.8 - 0.8 * v)));
    };
    int unit = blockIdx.x;
    uint32_t qw = 0;
    int qx = -1;                                    // the group whose queries qw holds
    auto load_query = [&](int x) {
        qw = load_query_word<NT>(a.q, (size_t)x * G, G, wave, lane);
        qx = x;
    };

    // Stage the blocks at positions [c0, c1), at most kRefineChunk, in LDS (by every wave, as above);
    // returns their number. The lanes that meet a group's first and last block write the group's first
    // and last row into the table.
    // Requests the queries of the first position's group on the way (usually the first block's).
    auto stage = [&](int c0, int c1, bool want_query) {
        int m = 0;
        for (int q0 = c0; q0 < c1; q0 += 4 * 64) {
            int4 st[4];
            bool real[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int pos = q0 + 64 * k + lane;
                real[k] = false;
                st[k] = make_int4(0, 0, 0, 0);
                if (q0 + 64 * k < c1 && pos < c1) {
                    int lo = 0, hi = nent;              // the largest record with prefix <= pos
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        if (prefix(mid) <= pos) lo = mid; else hi = mid;
                    }
                    const int4 r = cached ? sm.rec[lo] : a.info[lo];
                    const int L = r.y, x = r.z, s = r.w & kInfoSplitMask, S = r.w >> kInfoSplitBits;
                    if (want_query && k == 0 && q0 == c0) load_query(__builtin_amdgcn_readfirstlane(x));
                    const int at = pos - prefix(lo) - (s == 0 ? kGroupCost : 0);
                    real[k] = at >= 0;
                    if (real[k]) {
                        const int nblk = (L + kBlock - 1) / kBlock;
                        st[k] = make_int4((int)a.lists[(size_t)x * nblk_cap + s * ((nblk + S - 1) / S) + at], x, L, 0);
                        if (wave == 0 && pos == prefix(lo - s) + kGroupCost) a.table[x].x = unit + x;
                        if (wave == 0 && pos == prefix(lo - s + S) - 1) a.table[x].y = unit + x;
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint64_t b = __ballot(real[k]);
                if (real[k])
                    sm.list[m + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = st[k];
                m += __popcll(b);
            }
        }
        wave_lds_fence();
        return m;
    };

    HeadConsts<NT> hc;
    PvAcc<NT> pv;
    float m_run[NT], l_part[NT];
    TileP<NT>& tp = sm.tp[wave];
    auto begin_group = [&] {                        // of the group whose queries qw holds; a barrier inside
        build_query_consts<NT>(sm.qs, qw, G, a.scale, a.top_level, wave, lane, hc);
        pv.zero();
#pragma unroll
        for (int t = 0; t < NT; ++t) { m_run[t] = -INFINITY; l_part[t] = 0.f; }
    };
    auto end_group = [&](int x) {                   // the barrier inside separates the groups' use of sm.qs
        write_partials<NT, kRefineWaves>(sm.epi, pv, m_run, l_part, wave, lane, G, (size_t)(unit + x) * G, 1, a.part_m,
                                         a.part_l, a.part_acc);
    };

    // refine (Eq. 4) and attend tile T4 of one kept block (j | keep bits << 24) of a sequence of length L
    auto attend = [&](const RefineTile<NT, RBITS>& rt, uint32_t entry, int L) {
        const int j = (int)(entry & 0xffffffu);
        const uint32_t bits = entry >> 24;
        float z[NT];
        bool keep[NT];
        const float Mt = bf16_to_f32((uint16_t)rt.m);
        float shat[NT];                             // Eq. 4's first term: the scan scores, recomputed
        tile_scores<NT, RBITS>(rt.cw, Mt, 64 * j + 16 * T4 + n < L, hc, shat);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            v4i acc = {0, 0, 0, 0};
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(hc.A[t][0], rt.r0, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(hc.A[t][1], rt.r1, acc, 0, 0, 0);
            const float R = fmaf(65536.f, (float)acc.z, fmaf(256.f, (float)acc.y, (float)acc.x));
            const float sct = shat[t];
            z[t] = sct == -INFINITY ? -INFINITY : fmaf(R, Mt * hc.kap2[t], sct);
            keep[t] = (bits >> (4 * t + g)) & 1u;
        }
        softmax_tile<NT>(z, keep, m_run, l_part, tp, g, n);
        wave_lds_fence();
        pv_tile<NT>(pv, tp, rt.vt);
        wave_lds_fence();
    };

    bool written = false;                           // partials were written: their LDS may still be read
    for (int turn = 0; unit < U; turn ^= 1) {
        int ticket = 0;
        if (queue && tid == 0) ticket = atomicAdd(a.ticket, 1);        // arrives while the unit is worked on
        const int pl = first_of(unit + (lane & 1));
        const int p0 = __builtin_amdgcn_readlane(pl, 0), p1 = __builtin_amdgcn_readlane(pl, 1);
        int cur = -1;                               // the group being attended
        for (int c0 = p0; c0 < p1; c0 += kRefineChunk) {
            if (c0 > p0) __syncthreads();           // every wave is done with the staged entries
            const int m = __builtin_amdgcn_readfirstlane(stage(c0, min(c0 + kRefineChunk, p1), cur < 0));
            if (m == 0) continue;                   // uniform in the workgroup
            auto group_at = [&](int e) { return __builtin_amdgcn_readfirstlane(sm.list[e].y); };
            auto group_end = [&](int e) {           // first entry after e of another group, or m
                const int x = group_at(e);
                for (; e < m; e += 64) {
                    const uint64_t other = __ballot(e + lane < m && sm.list[min(e + lane, m - 1)].y != x);
                    if (other) return e + (int)__builtin_ctzll(other);
                }
                return m;
            };
            // this wave's tiles of the staged entries par, par + kPar, ..., kRefineRing of them in flight; the
            // refill of the last round re-reads the wave's last tile (clamped): it is still cached, and a
            // conditional refill would cost more registers than it saves
            const int last = m - 1 - ((m - 1 - par) & (kPar - 1));     // the wave's last entry; -1: it has none
            RefineTile<NT, RBITS> ring[kRefineRing];
            uint32_t word[kRefineRing];
            int rL[kRefineRing];
            auto refill = [&](int r, int e) {
                const int4 ent = sm.list[max(min(e, last), 0)];
                word[r] = __builtin_amdgcn_readfirstlane((uint32_t)ent.x);
                const size_t bh = (size_t)__builtin_amdgcn_readfirstlane(ent.y);
                rL[r] = __builtin_amdgcn_readfirstlane(ent.z);
                ring[r] = load_refine_tile<NT, RBITS>(a.resid + bh * a.Lcap * kD, a.v + bh * a.Lcap * kD,
                                                      a.codes + bh * a.Lcap * (4 * RBITS), a.absmax + bh * a.Lcap,
                                                      (int)(word[r] & 0xffffffu), T4, lane, rL[r]);
            };
            // a group's queries are requested ahead: the first one's before the tiles (its constants are
            // built while they are in flight), the next one's when its predecessor begins
            if (group_at(0) != cur && group_at(0) != qx) load_query(group_at(0));
#pragma unroll
            for (int r = 0; r < kRefineRing; ++r) refill(r, par + kPar * r);
            int next = 0;                           // first staged entry of the next group
            if (cur < 0 || group_at(0) == cur) {
                if (cur < 0) {
                    cur = group_at(0);
                    begin_group();
                }
                next = group_end(0);
                if (next < m) load_query(group_at(next));
            }
            for (int e0 = 0; e0 < m; e0 += kPar * kRefineRing) {       // uniform in the workgroup
                const int e1 = min(e0 + kPar * kRefineRing, m);
                for (int sb = e0;;) {               // the round's entries, group by group
#pragma unroll
                    for (int r = 0; r < kRefineRing; ++r) {
                        const int e = e0 + kPar * r + par;
                        if (e >= sb && e < min(next, e1)) {
                            attend(ring[r], word[r], rL[r]);
                            refill(r, e + kPar * kRefineRing);
                        }
                    }
                    if (next >= e1) break;
                    if (written) __syncthreads();
                    end_group(cur);
                    written = true;
                    cur = group_at(next);
                    begin_group();
                    sb = next;
                    next = group_end(next);
                    if (next < m) load_query(group_at(next));
                }
            }
        }
        if (cur >= 0) {
            if (written) __syncthreads();
            end_group(cur);
            written = true;
        }
        if (!queue) break;
        if (tid == 0) sm.unit[turn] = (int)gridDim.x + ticket;
        __syncthreads();                            // also: every wave is done with the staged entries
        unit = __builtin_amdgcn_readfirstlane(sm.unit[turn]);
    }
}

template __global__ void ffd_scan_kernel<1, 2, kSelThumbnailPM>(ScanArgs);
template __global__ void ffd_scan_kernel<2, 2, kSelThumbnailPM>(ScanArgs);
template __global__ void ffd_scan_kernel<1, 4, kSelThumbnailPM>(ScanArgs);
template __global__ void ffd_scan_kernel<2, 4, kSelThumbnailPM>(ScanArgs);
template __global__ void ffd_scan_kernel<1, 8, kSelThumbnailPM>(ScanArgs);
template __global__ void ffd_scan_kernel<2, 8, kSelThumbnailPM>(ScanArgs);
template __global__ void ffd_scan_kernel<1, 2, kSelRefinedPM>(ScanArgs);
template __global__ void ffd_scan_kernel<2, 2, kSelRefinedPM>(ScanArgs);
template __global__ void ffd_scan_kernel<1, 4, kSelRefinedPM>(ScanArgs);
template __global__ void ffd_scan_kernel<2, 4, kSelRefinedPM>(ScanArgs);
template __global__ void ffd_scan_kernel<1, 8, kSelRefinedPM>(ScanArgs);
template __global__ void ffd_scan_kernel<2, 8, kSelRefinedPM>(ScanArgs);
template __global__ void ffd_scan_kernel<1, 2, kSelTopK>(ScanArgs);
template __global__ void ffd_scan_kernel<2, 2, kSelTopK>(ScanArgs);
template __global__ void ffd_scan_kernel<1, 4, kSelTopK>(ScanArgs);
template __global__ void ffd_scan_kernel<2, 4, kSelTopK>(ScanArgs);
template __global__ void ffd_scan_kernel<1, 8, kSelTopK>(ScanArgs);
template __global__ void ffd_scan_kernel<2, 8, kSelTopK>(ScanArgs);
template __global__ void ffd_decode_kernel<1, 2, kSelThumbnailPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 2, kSelThumbnailPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 2, kSelThumbnailPM, 1>(FusedArgs);
template __global__ void ffd_decode_kernel<1, 4, kSelThumbnailPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 4, kSelThumbnailPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 4, kSelThumbnailPM, 1>(FusedArgs);
template __global__ void ffd_decode_kernel<1, 8, kSelThumbnailPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 8, kSelThumbnailPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<1, 2, kSelRefinedPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 2, kSelRefinedPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 2, kSelRefinedPM, 1>(FusedArgs);
template __global__ void ffd_decode_kernel<1, 4, kSelRefinedPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 4, kSelRefinedPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 4, kSelRefinedPM, 1>(FusedArgs);
template __global__ void ffd_decode_kernel<1, 8, kSelRefinedPM, 2>(FusedArgs);
template __global__ void ffd_decode_kernel<2, 8, kSelRefinedPM, 2>(FusedArgs);
template __global__ void ffd_refine_kernel<1, 2>(RefineArgs);
template __global__ void ffd_refine_kernel<2, 2>(RefineArgs);
template __global__ void ffd_refine_kernel<1, 4>(RefineArgs);
template __global__ void ffd_refine_kernel<2, 4>(RefineArgs);
template __global__ void ffd_refine_kernel<1, 8>(RefineArgs);
template __global__ void ffd_refine_kernel<2, 8>(RefineArgs);

}  // namespace ffd
