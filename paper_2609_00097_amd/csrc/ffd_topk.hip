// Fixed-budget (top-k) block selection: the rule the paper sets top-delta against (Sec. 1, Fig. 1 (a);
// the selection-rule overhead comparison of Table 3). Per query head, the k blocks with the largest
// block scores sigma (the maxima of the thumbnail scores over a block's valid tokens, as top-delta
// uses them) are kept; equal scores are taken in block order. Unlike top-delta, whose decision is a
// comparison with a per-head constant made while the scan streams, this needs every block score of
// the head first: the scan kernel writes them, and this kernel, one workgroup per (sequence, KV
// head), holds the group's scores in registers (as the order-preserving integer image of the fp32
// score; each wave holds whole 64-block runs of one head) and finds each head's k-th largest score by
// narrowing an interval of keys that holds it: a histogram of 512 equal bins in LDS, first over the
// head's range of scores, shows the bin where the count from the top reaches k; up to 64 keys in it are
// ranked against each other, of more (outliers that stretch the range, ties) the least and the largest key
// are the next interval, whose bins are equal in the integer image. It then marks the blocks above and
// equal to the k-th score in LDS bitmaps, goes through the blocks in order, keeps those above the
// threshold and the first ones equal to it, and writes the group's kept list (block | keep bits << 24, the
// union over the group's heads) and its length in the scan's format, so the refinement kernel runs unchanged.
//
// Bound: one workgroup per group works alone on its CU; each round is a chain of LDS atomics, a prefix and
// a few barriers. Scan and selection of 32 groups of 2048 blocks x 4 heads, k = 67: 40.0 us (45.4 with a radix
// select of four 8-bit digits in the histogram's place); with one block's scores 300 times the others' 48.4
// (48.6; 58.0 where the digits followed a crowded bin of the range), with exact ties throughout 42.8 (48.7; 59.3).
#include <climits>

#include "ffd_device.h"
#include "ffd_kernels.h"

namespace ffd {

namespace {

constexpr int kSelThreads = kTopkSelectThreads;      // 16 waves: 4 per SIMD hide each other's latency
constexpr int kSelWaves = kSelThreads / 64;
constexpr int kSlots = 8;                            // keys held per thread
constexpr int kTileKeys = kSlots * kSelThreads;      // (block, head) keys per tile
constexpr int kBinBits = 9;
constexpr int kBins = 1 << kBinBits;                 // bins per histogram
constexpr int kMaxCand = 64;                         // keys of one bin that are ranked by a wave
constexpr int kCrowded = 16;                         // lanes of a wave in one bin from which on it adds them up

// Order-preserving image of a float: larger float, larger key. The scan writes +0 for a zero score.
__device__ __forceinline__ uint32_t order_key(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_value(uint32_t key) {
    return __uint_as_float((key & 0x80000000u) ? key & 0x7fffffffu : ~key);
}

// Whether many active lanes of the wave share the first one's bin. Atomics of many lanes on one address go one
// after the other, so such waves add their counts up first.
__device__ __forceinline__ bool crowded(int bin, bool active) {
    const uint64_t act = __ballot(active);                              // wave-uniform
    const int b0 = __builtin_amdgcn_readlane(bin, act ? __builtin_ctzll(act) : 0);
    return __popcll(__ballot(active && bin == b0)) > kCrowded;
}

// hist[bin] += 1 for every active lane of a crowded wave: the bins of the first active lane and of the first one
// of another bin are counted by one leader lane each (adding the bin's population in the wave); the remaining
// lanes add one each.
__device__ __forceinline__ void hist_add(int* hist, int bin, bool active, int lane) {
    const uint64_t act = __ballot(active);
    const int l0 = act ? __builtin_ctzll(act) : 0;
    const int b0 = __builtin_amdgcn_readlane(bin, l0);
    const uint64_t s0 = __ballot(active && bin == b0);
    const uint64_t rest = act & ~s0;
    const int l1 = rest ? __builtin_ctzll(rest) : 0;
    const int b1 = __builtin_amdgcn_readlane(bin, l1);                  // != b0 when rest != 0
    const uint64_t s1 = __ballot(active && bin == b1) & rest;
    const bool lead0 = act != 0 && lane == l0;
    const bool lead1 = rest != 0 && lane == l1;
    const bool other = active && bin != b0 && bin != b1;
    const int at = lead0 ? b0 : (lead1 ? b1 : bin);
    const int val = lead0 ? (int)__popcll(s0) : (lead1 ? (int)__popcll(s1) : 1);
    if (lead0 || lead1 || other) atomicAdd(&hist[at], val);
}

// Which keys a thread holds. A tile is TB = kTileKeys / G blocks of every head. Register slot i of
// wave w (lane l) holds head w mod G at block 64 * (i * WPH + w / G) + l of the tile: each head's
// 64-block runs are spread over WPH = 16 / G waves.
template <int G>
struct Slots {
    static constexpr int TB = kTileKeys / G;
    static constexpr int WPH = kSelWaves / G;
    static constexpr int RUNS = TB / 64;             // 64-block runs per head per tile
    __device__ static int head(int wave) { return wave % G; }
    __device__ static int run(int wave, int i) { return i * WPH + wave / G; }
};

template <int G>
struct TopkLds {
    int hist[G][kBins];
    uint64_t gtmap[G][Slots<G>::RUNS];    // per head and 64-block run: blocks above the threshold
    uint64_t eqmap[G][Slots<G>::RUNS];    // ... and equal to it
    uint32_t lo[G], hi[G];                // the least and largest key of the interval that holds the k-th largest
    int rem[G];                           // the k-th largest key is the interval's rem-th largest
    int bin[G], inbin[G], ncand[G];       // its bin, keys in the bin, candidates written
    int found[G];                         // lo is the k-th largest key; rem keys equal to it (INT_MAX: all) are taken
    uint32_t next_lo[G], next_hi[G];      // the bin's least and largest key
    uint32_t cand[G][kMaxCand];
    int wsum[2][kSelWaves];
};

// This thread's keys of tile ti (blocks [ti * TB, ti * TB + nb)); slots past nb are not valid.
template <int G>
__device__ __forceinline__ void load_keys(uint32_t (&key)[kSlots], const float* __restrict__ sig, int ti,
                                          int nb, int wave, int lane) {
    using S = Slots<G>;
    float v[kSlots];
#pragma unroll
    for (int i = 0; i < kSlots; ++i) {
        const int jj = 64 * S::run(wave, i) + lane;
        v[i] = jj < nb ? sig[((size_t)ti * S::TB + jj) * G + S::head(wave)] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < kSlots; ++i) key[i] = order_key(v[i]);
}

}  // namespace

// Grid (B * Hkv), kSelThreads threads; G query heads per KV head.
template <int G>
__global__ __launch_bounds__(kSelThreads) void ffd_topk_select_kernel(TopkArgs a) {
    using S = Slots<G>;
    constexpr int TB = S::TB;
    constexpr int BPT = TB / kSelThreads;            // blocks per thread in the keep pass (<= 8)
    __shared__ TopkLds<G> sm;
    const int x = blockIdx.x;
    const int b = x / a.Hkv, kvh = x % a.Hkv;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int L = min(max(a.seq_lens[b], 0), a.Lcap);
    const int nblk = (L + kBlock - 1) / kBlock;
    const int nblk_cap = a.Lcap / kBlock;
    const int keff = min(a.k, nblk);
    const int ntiles = (nblk + TB - 1) / TB;
    const float* sig = a.sigma + (size_t)x * nblk_cap * G;
    uint32_t key[kSlots];
    int loaded = -1;                                 // tile now in key[]
    auto use_tile = [&](int ti) {
        if (ti != loaded) load_keys<G>(key, sig, ti, min(TB, nblk - ti * TB), wave, lane);
        loaded = ti;
    };
    auto valid = [&](int ti, int i) { return 64 * S::run(wave, i) + lane < nblk - ti * TB; };

    // ---- the k-th largest key of each head ---------------------------------------------------
    if (tid < G) {
        sm.lo[tid] = sm.next_lo[tid] = 0xffffffffu;
        sm.hi[tid] = sm.next_hi[tid] = 0u;
        sm.rem[tid] = keff;
        sm.ncand[tid] = 0;
        sm.found[tid] = 0;
    }
    for (int i = tid; i < G * kBins; i += kSelThreads) (&sm.hist[0][0])[i] = 0;
    __syncthreads();
    const int hw = S::head(wave);                    // this wave's head (wave h < G: head h)
    const bool select = keff < nblk;                 // else every block is kept
    // The least and largest of the wave's keys that `of` selects, into lo and hi of its head.
    auto extremes = [&](uint32_t* lo, uint32_t* hi, auto of) {
        uint32_t klo = 0xffffffffu, khi = 0u;
        for (int ti = 0; ti < ntiles; ++ti) {
            use_tile(ti);
#pragma unroll
            for (int i = 0; i < kSlots; ++i)
                if (valid(ti, i) && of(key[i])) {
                    klo = min(klo, key[i]);
                    khi = max(khi, key[i]);
                }
        }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            klo = min(klo, (uint32_t)__shfl_xor((int)klo, o));
            khi = max(khi, (uint32_t)__shfl_xor((int)khi, o));
        }
        if (lane == 0) {
            atomicMin(&lo[hw], klo);
            atomicMax(&hi[hw], khi);
        }
    };
    if (select) {                                    // uniform
        extremes(sm.lo, sm.hi, [](uint32_t) { return true; });
        __syncthreads();
        for (bool first = true;; first = false) {
            // The interval's bins: (score - least) * 512 / range in the first round, which grows with the score
            // (each step is monotonic in fp32), where range and scores are finite (the extremes show them);
            // else equal steps of the key, of which the interval after it holds one: every round takes 9 bits
            // off the interval's length, and a bin of one key is never narrowed, so five rounds are the most.
            const uint32_t klo = sm.lo[hw], khi = sm.hi[hw];
            const float least = key_value(klo), range = key_value(khi) - least;
            const float per = (float)kBins / range;
            const bool by_score =
                first && __builtin_isfinite(least) && __builtin_isfinite(range) && __builtin_isfinite(per);
            const int shift = max(32 - kBinBits - __clz((int)(khi - klo)), 0);
            auto bin_of = [&](uint32_t k) {
                return by_score ? min(max((int)((key_value(k) - least) * per), 0), kBins - 1) : (int)((k - klo) >> shift);
            };
            auto inside = [&](uint32_t k) { return k >= klo && k <= khi; };
            const bool live = !sm.found[hw];         // uniform in the wave
            for (int ti = 0; ti < ntiles && live; ++ti) {
                use_tile(ti);
                const bool in0 = valid(ti, 0) && inside(key[0]);
                const bool adding_up = crowded(in0 ? bin_of(key[0]) : 0, in0);
#pragma unroll
                for (int i = 0; i < kSlots; ++i) {
                    const bool in = valid(ti, i) && inside(key[i]);
                    const int at = in ? bin_of(key[i]) : 0;
                    if (adding_up) hist_add(sm.hist[hw], at, in, lane);  // uniform in the wave
                    else if (in) atomicAdd(&sm.hist[hw][at], 1);
                }
            }
            __syncthreads();
            if (wave < G && live) {                  // wave h: head h; lane l holds bins 8 l .. 8 l + 7
                constexpr int kPer = kBins / 64;
                int c[kPer], tot = 0;
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    c[i] = sm.hist[wave][kPer * lane + i];
                    tot += c[i];
                }
                const int incl = wave_inclusive_scan(tot), rem = sm.rem[wave];
                int above = __builtin_amdgcn_readlane(incl, 63) - incl;      // keys in the bins of higher lanes
#pragma unroll
                for (int i = kPer - 1; i >= 0; --i) {
                    if (above < rem && above + c[i] >= rem) {
                        sm.bin[wave] = kPer * lane + i;
                        sm.inbin[wave] = c[i];
                        sm.rem[wave] = rem - above;
                    }
                    above += c[i];
                }
            }
            __syncthreads();
            bool again = false;                      // uniform: some head's bin is to be narrowed
#pragma unroll
            for (int h = 0; h < G; ++h) again = again || (!sm.found[h] && sm.inbin[h] > kMaxCand);
            const int bin = sm.bin[hw];
            if (live && sm.inbin[hw] <= kMaxCand) {
                for (int ti = 0; ti < ntiles; ++ti) {
                    use_tile(ti);
#pragma unroll
                    for (int i = 0; i < kSlots; ++i)
                        if (valid(ti, i) && inside(key[i]) && bin_of(key[i]) == bin)
                            sm.cand[hw][atomicAdd(&sm.ncand[hw], 1)] = key[i];
                }
            } else if (live) {
                extremes(sm.next_lo, sm.next_hi, [&](uint32_t k) { return inside(k) && bin_of(k) == bin; });
            }
            if (again)
                for (int i = tid; i < G * kBins; i += kSelThreads) (&sm.hist[0][0])[i] = 0;
            __syncthreads();
            if (wave < G && live) {
                const int nc = sm.inbin[wave], r = sm.rem[wave];
                if (nc <= kMaxCand) {                // the bin's r-th largest key is sought
                    const uint32_t mine = lane < nc ? sm.cand[wave][lane] : 0u;
                    int larger = 0, equal = 0;
                    for (int i = 0; i < nc; ++i) {
                        const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)mine, i);
                        larger += other > mine ? 1 : 0;
                        equal += other == mine ? 1 : 0;
                    }
                    if (lane < nc && larger < r && larger + equal >= r) {    // equal keys write the same
                        sm.lo[wave] = mine;
                        sm.rem[wave] = larger + equal == r ? INT_MAX : r - larger;
                    }
                    if (lane == 0) sm.found[wave] = 1;
                } else if (lane == 0) {
                    const uint32_t lo = sm.next_lo[wave], hi = sm.next_hi[wave];
                    sm.lo[wave] = lo;
                    sm.hi[wave] = hi;
                    sm.found[wave] = lo == hi;       // all of the bin's keys are equal
                    if (lo == hi && r == nc) sm.rem[wave] = INT_MAX;
                    sm.next_lo[wave] = 0xffffffffu;
                    sm.next_hi[wave] = 0u;
                }
            }
            __syncthreads();
            bool all_found = true;
#pragma unroll
            for (int h = 0; h < G; ++h) all_found = all_found && sm.found[h];
            if (all_found) break;                    // uniform: read after the barrier
        }
    }

    // ---- keep: key > threshold, or key == threshold among the first `need` equal ones ----------
    // keep-all: threshold 0 with no limit on equal keys takes every key
    const uint32_t thr_w = select ? sm.lo[hw] : 0u;
    int need[G], eq_run[G];                          // uniform: kept in scalar registers
    bool take_equal = true;                          // every head takes all of its equal keys
#pragma unroll
    for (int h = 0; h < G; ++h) {
        need[h] = __builtin_amdgcn_readfirstlane(select ? sm.rem[h] : INT_MAX);
        eq_run[h] = 0;
        take_equal = take_equal && need[h] == INT_MAX;
    }
    uint32_t* list_x = a.lists + (size_t)x * nblk_cap;
    uint8_t* mask_x = a.mask ? a.mask + ((size_t)b * a.Hq + (size_t)kvh * G) * nblk_cap : nullptr;
    int list_run = 0, half = 0;
    auto scan = [&](int v, int* tot) {
        const int e = wg_exclusive_scan<kSelWaves>(v, sm.wsum[half], tot);
        half ^= 1;
        return e;
    };
    for (int ti = 0; ti < ntiles; ++ti) {
        use_tile(ti);
#pragma unroll
        for (int i = 0; i < kSlots; ++i) {
            const bool ok = valid(ti, i);
            const uint64_t gb = __ballot(ok && key[i] > thr_w), eb = __ballot(ok && key[i] == thr_w);
            if (lane == 0) {
                sm.gtmap[hw][S::run(wave, i)] = gb;
                sm.eqmap[hw][S::run(wave, i)] = eb;
            }
        }
        __syncthreads();
        const int jt0 = ti * TB, nb = min(TB, nblk - jt0);
        const int jj0 = BPT * tid;                      // this thread's blocks jt0 + jj0 + i, i < BPT
        const uint32_t low = (1u << BPT) - 1u;
        uint32_t eqm[G], gtm[G];
#pragma unroll
        for (int h = 0; h < G; ++h) {
            gtm[h] = (uint32_t)(sm.gtmap[h][jj0 / 64] >> (jj0 % 64)) & low;
            eqm[h] = (uint32_t)(sm.eqmap[h][jj0 / 64] >> (jj0 % 64)) & low;
        }
        // equal keys of each head before this thread's blocks (two heads per scan in 16-bit fields:
        // a tile holds at most 8192 blocks)
        int eq_before[G];
#pragma unroll
        for (int h = 0; h < G; ++h) eq_before[h] = 0;
        if (!take_equal) {                              // uniform
#pragma unroll
            for (int h = 0; h < G; h += 2) {
                const int hi = h + 1 < G ? __popc(eqm[h + 1]) : 0;
                int tot = 0;
                const int e = scan(__popc(eqm[h]) | (hi << 16), &tot);
                tot = __builtin_amdgcn_readfirstlane(tot);
                eq_before[h] = eq_run[h] + (e & 0xffff);
                eq_run[h] += tot & 0xffff;
                if (h + 1 < G) {
                    eq_before[h + 1] = eq_run[h + 1] + (e >> 16);
                    eq_run[h + 1] += tot >> 16;
                }
            }
        }
        uint32_t take[G], any = 0u;
#pragma unroll
        for (int h = 0; h < G; ++h) {
            take[h] = gtm[h] | (take_equal ? eqm[h] : 0u);
            uint32_t e = take_equal ? 0u : eqm[h];
            int rank = eq_before[h];
            while (e != 0u && rank < need[h]) {         // the first `need` equal keys, in block order
                const uint32_t lowbit = e & (0u - e);
                take[h] |= lowbit;
                e ^= lowbit;
                ++rank;
            }
            any |= take[h];
        }
        int tot = 0;
        int pos = list_run + scan(__popc(any), &tot);
        list_run += __builtin_amdgcn_readfirstlane(tot);
#pragma unroll
        for (int i = 0; i < BPT; ++i) {
            const int j = jt0 + jj0 + i;
            if (jj0 + i < nb) {
                uint32_t bits = 0u;
#pragma unroll
                for (int h = 0; h < G; ++h) bits |= ((take[h] >> i) & 1u) << h;
                if (bits) list_x[pos++] = (uint32_t)j | (bits << 24);
                if (mask_x) {
#pragma unroll
                    for (int h = 0; h < G; ++h) mask_x[(size_t)h * nblk_cap + j] = (uint8_t)((bits >> h) & 1u);
                }
            }
        }
        __syncthreads();                                // the maps are rewritten for the next tile
    }
    if (tid == 0) {
        a.info[x] = make_int4(list_run, L, x, 1 << kInfoSplitBits);
        a.table[x] = make_int2(0, -1);
        if (x == 0) *a.ticket = 0;
    }
    if (mask_x) {
        for (int j = nblk + tid; j < nblk_cap; j += kSelThreads)
#pragma unroll
            for (int h = 0; h < G; ++h) mask_x[(size_t)h * nblk_cap + j] = 0;
    }
}

template __global__ void ffd_topk_select_kernel<1>(TopkArgs);
template __global__ void ffd_topk_select_kernel<2>(TopkArgs);
template __global__ void ffd_topk_select_kernel<4>(TopkArgs);
template __global__ void ffd_topk_select_kernel<8>(TopkArgs);

}  // namespace ffd
