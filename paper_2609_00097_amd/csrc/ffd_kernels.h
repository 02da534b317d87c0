// Kernel argument blocks and declarations of the library's HIP kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ffd {

// Refinement: line positions whose blocks are staged in LDS at a time, and scan records kept in LDS
// (more go through ffd_offsets_kernel).
constexpr int kRefineChunk = 256;
constexpr int kRefineRecords = 1024;
constexpr int kOffsetThreads = 1024;
// Line positions that a group's beginning counts for, in blocks: at 4 x 128K, 15 blocks per workgroup,
// a step takes 59.0 us with 0, 57.8 with 2, 56.8 with 5 and 6, 57.1 with 8, 57.4 with 12. Over 27 other shapes
// (1 to 64 sequences, 7 to 60 blocks per workgroup) the refinement's times with 2, 3, 4 and 6 lie within 2 % of
// each other, 3 or 6 being the best; with 12 and 20 they are up to 5 and 15 % longer.
constexpr int kGroupCost = 6;
// Units where workgroups take several: blocks per unit on average, at least, and the share of all blocks
// in the workgroups' first units. Ragged batch of 16, 310 blocks per workgroup, 897 units: 446 us per
// step; first share 0.7: 448, 0.9: 448; at least 96 blocks per unit: 450. Taken from two units per workgroup
// on, by the blocks and by the rows that the workspace has for partials (units + groups - 1): with fewer, those
// after the first are too long to even out what the first ones differ by. 16 x 64K, half of the sequences
// without structure, rows for 385 units on 256 CUs: 434 us a step with them, 367 with equal shares; 8 x 64K,
// 449: 207 and 188; 6 x 128K, 465: 317 and 285.
constexpr int kUnitBlocks = 48;
constexpr double kFirstShare = 0.82;
// A record int4 describes one kept list: (kept blocks, sequence length, KV group, split | splits <<
// kInfoSplitBits); the list of split s of S starts at the group's block s * ceil(blocks / S).
constexpr int kInfoSplitBits = 11;
constexpr int kInfoSplitMask = (1 << kInfoSplitBits) - 1;
// Most blocks one scan workgroup covers (its kept list is staged in LDS), most scan workgroups per
// (sequence, KV head).
constexpr int kFfdMaxScanBlocks = 256;
// Whether the scan's workgroups are numbered by sequence, KV head and slot (neighbours read neighbouring
// ranges) and not with the KV heads first (neighbours read the same range of each head). Steps over six
// caches in turn, in order / KV heads first: 4 bits, 4 x 128K, 8 KV heads, where the heads' codes are 8
// MiB apart, 71.8 / 74.5 us, 2 x 256K 70.5 / 71.7, 1 x 512K 69.3 / 69.8, but 4 x 98K 59.5 / 58.8 and 8 x 64K
// 73.0 / 71.5; 2 bits 49.7 / 49.4, 48.6 / 49.4, 48.1 / 48.1, 43.7 / 42.9, 50.8 / 51.0; 8 bits 117.2 / 113.9,
// 114.1 / 117.7, 113.4 / 113.6, 93.4 / 92.6, 116.8 / 115.3. So in order for 4 bits, for its worst case.
__host__ __device__ constexpr bool scan_in_order(int bits) { return bits == 4; }
constexpr int kSlotGridY = 32768;              // slots along the grid's y (then z)
constexpr int kBalanceMaxSeqs = 64;            // largest batch whose scan slots follow the lengths
constexpr int kScanWaves = 8;                  // waves per scan workgroup (one workgroup per CU)
constexpr int kScanThreads = 64 * kScanWaves;
// Waves per refinement workgroup (one workgroup per CU): 8 (two per SIMD) overlap one wave's waits
// with the other's work, which pays on long shares (the ragged 16-sequence batch, where half of the
// blocks are kept: 430 us of refinement against 503 us with 4 waves) and costs nothing at 4 x 128K.
constexpr int kRefineWaves = 8;
constexpr int kRefineThreads = 64 * kRefineWaves;
constexpr int kFfdMaxScanSplits = 1024;        // below 2^kInfoSplitBits

// Thumbnail depth b (App. C: 2+8, 4+8, 8+8): 2^b levels c - Lv, Lv = (2^b - 1) / 2; a token's codes
// take 4b words.
__host__ __device__ constexpr float thumb_top_level(int bits) { return ((1 << bits) - 1) * 0.5f; }

struct ScanArgs {
    const uint16_t* q;          // bf16 [B, Hq, 128]
    const uint32_t* codes;      // [B, Hkv, Lcap/64, 64, 4b] (b = the kernel's thumbnail depth)
    const uint16_t* absmax;     // bf16 [B, Hkv, Lcap/64, 16, 4]
    const int8_t* resid;        // [B, Hkv, Lcap/16, 2, 64, 16]: read for the refined pseudo-max only
    const int32_t* seq_lens;    // [B]
    uint32_t* lists;            // [B*Hkv, Lcap/64]: kept blocks j | keep bits << 24, per scan split
    int4* info;                 // [grid_slots * Hkv]: one record per kept list, in (group, split) order
    int2* table;                // [B*Hkv]: set to (0, -1)
    int* ticket;                // the refinement's unit counter: set to 0
    float* sigma;               // top-k selection: block scores [B*Hkv, Lcap/64, G]
    uint8_t* mask;              // [B, Hq, Lcap/64] or null
    float* m_tilde;             // [B, Hq] or null: the pseudo-max of each head
    int B, Hq, Hkv, Lcap, G, S1, round_slots, grid_slots;    // S1 per sequence, or by the lengths (slot_of)
    float delta, scale;
    int n_sink, n_local;
};

struct RefineArgs {
    const uint16_t* q;          // bf16 [B, Hq, 128]
    const uint32_t* codes;      // thumbnail codes, from which the scan scores are recomputed
    const uint16_t* absmax;     // bf16 [B, Hkv, Lcap/64, 16, 4]
    const int8_t* resid;        // [B, Hkv, Lcap/16, 2, 64, 16]
    const uint16_t* v;          // bf16 [B, Hkv, Lcap, 128]
    const uint32_t* lists;      // written by ffd_scan_kernel or ffd_topk_select_kernel
    const int4* info;           // their records, in (group, split) order
    int2* table;                // [B*Hkv]: (first row, last row) of each KV group, rows in units of G heads
    int* ticket;                // units taken from the counter
    float* part_m;              // [(max_units + B*Hkv - 1) * G]
    float* part_l;
    float* part_acc;            // [(max_units + B*Hkv - 1) * G, 128]
    int Lcap, G, W, max_units, nent;       // W workgroups, as many units or up to max_units of them
    float scale;
    float top_level;            // Lv of the thumbnail depth: the residual step is M / (254 Lv)
};

// The fused top-delta decode kernel: scan, pseudo-max, decisions, refinement and attention in one
// workgroup per (sequence, KV head, split), on an interleaved share of the group's blocks.
struct FusedArgs {
    const uint16_t* q;          // bf16 [B, Hq, 128]
    const uint32_t* codes;      // [B, Hkv, Lcap/64, 64, 4b]
    const uint16_t* absmax;     // bf16 [B, Hkv, Lcap/64, 16, 4]
    const int8_t* resid;        // [B, Hkv, Lcap/16, 2, 64, 16]
    const uint16_t* v;          // bf16 [B, Hkv, Lcap, 128]
    const int32_t* seq_lens;    // [B]
    uint8_t* mask;              // [B, Hq, Lcap/64] or null
    float* m_tilde;             // [B, Hq] or null: the pseudo-max of each head
    float* part_m;              // [B * S1 * Hkv, G] partial states (S1 > 1)
    float* part_l;
    float* part_acc;            // [B * S1 * Hkv, G, 128]
    int2* table;                // [B*Hkv]: (first, last) row of each group, or null: S1 rows per group
    uint16_t* out;              // bf16 [B, Hq, 128], written by the kernel itself when S1 == 1, else null
    float* lse;                 // [B, Hq] or null (S1 == 1 only)
    int turn;                   // KV heads turned with every 256 workgroups, beside one with every 64
    int B, Hq, Hkv, Lcap, G, S1, round_slots, grid_slots;    // S1 per sequence, or by the lengths (slot_of)
    float delta, scale;
    int n_sink, n_local;
};

// Fixed-budget (top-k) selection over the block scores the scan kernel wrote; its output takes the
// place of the scan's kept lists and records (each group's whole list as one split).
struct TopkArgs {
    const float* sigma;         // [B*Hkv, Lcap/64, G]
    const int32_t* seq_lens;    // [B]
    uint32_t* lists;            // [B*Hkv, Lcap/64]: kept blocks j | keep bits << 24, in block order
    int4* info;                 // [B*Hkv]: the group's record (one split)
    int2* table;                // [B*Hkv]: set to (0, -1)
    int* ticket;                // the refinement's unit counter: set to 0
    uint8_t* mask;              // [B, Hq, Lcap/64] or null
    int Hq, Hkv, Lcap, k;
};

// Dense decode. Balanced mode (table != null, B <= kDenseBalanceMaxSeqs): a 1-D grid of
// (S + 1) * B * Hkv workgroups; sequence b (n_b blocks) gets W_b = ceil(n_b * min(W, N) / N)
// workgroups per KV head (W = S * B * Hkv, N = Hkv * sum n_b; 1 for an empty sequence), numbered in
// (sequence, KV head) order, each taking an equal run of the sequence's blocks and writing its
// partial rows at its own index (table[b * Hkv + kvh] = first and last workgroup). Otherwise a grid
// (S, Hkv, B) of equal runs per sequence with rows [B, Hq, S].
constexpr int kDenseBalanceMaxSeqs = 256;
struct DenseArgs {
    const uint16_t* q;          // bf16 [B, Hq, 128]
    const uint16_t* k;          // bf16 [B, Hkv, Lcap, 128]
    const uint16_t* v;          // bf16 [B, Hkv, Lcap, 128]
    const int32_t* seq_lens;
    float* part_m;
    float* part_l;
    float* part_acc;
    int2* table;                // balanced mode: [B * Hkv] (first, last workgroup); else null
    int B, Hq, Hkv, Lcap, G, S;
    float scale;
};

struct QuantArgs {
    const uint16_t* k;          // bf16 [B, Hkv, Lcap, 128]
    uint32_t* codes;
    uint16_t* absmax;
    int8_t* resid;
    int Hkv, Lcap, t_begin, t_end;
};

constexpr int kQuantThreads = 64;              // one wave, one 64-token block per quantizer workgroup

struct AppendArgs {
    const uint16_t* k_new;      // bf16 [B, Hkv, 128]
    const uint16_t* v_new;      // bf16 [B, Hkv, 128]
    uint16_t* k_cache;          // bf16 [B, Hkv, Lcap, 128] or null
    uint16_t* v_cache;          // bf16 [B, Hkv, Lcap, 128] or null
    uint32_t* codes;
    uint16_t* absmax;
    int8_t* resid;
    int32_t* seq_lens;          // [B], read and advanced
    int Hkv, Lcap;
};

// What the scan kernel does after scoring a block:
//  kSelThumbnailPM  top-delta against the pseudo-max of the window tokens' thumbnail scores (Alg. 1);
//  kSelRefinedPM    top-delta against the pseudo-max of their refined logits (Eq. 3's reading);
//  kSelTopK         no decision: the block scores go to the workspace for ffd_topk_select_kernel.
// The first two write the kept lists and records; no mode stores the scan scores.
enum ScanMode { kSelThumbnailPM = 0, kSelRefinedPM = 1, kSelTopK = 2 };
template <int NT, int BITS, int MODE> __global__ void ffd_scan_kernel(ScanArgs a);
// MODE kSelThumbnailPM or kSelRefinedPM; the scan scores of the kept tiles are recomputed from the
// codes the kernel has just streamed (bit for bit the values the decisions used).
template <int NT, int BITS, int MODE, int RING> __global__ void ffd_decode_kernel(FusedArgs a);
// The scan scores of the kept tiles (Eq. 4's first term) are recomputed from the RBITS-bit codes with
// the scan kernel's own integer MFMA and fp32 operations, so they equal the scan's bit for bit.
template <int NT, int RBITS> __global__ void ffd_refine_kernel(RefineArgs a);
__global__ void ffd_offsets_kernel(int4* info, int nent);
template <int G> __global__ void ffd_topk_select_kernel(TopkArgs a);
constexpr int kTopkSelectThreads = 1024;
template <int NT> __global__ void dense_decode_kernel(DenseArgs a);
template <int BITS> __global__ void quantize_keys_kernel(QuantArgs a);
template <int BITS> __global__ void append_kv_kernel(AppendArgs a);
constexpr int kMergeSlices = 4;                // workgroups per head of the merge, 32 dims each
// NW waves per workgroup: 4, or 1 from kMergeOneWaveHeads heads on (their waves fill the chip alone).
constexpr int kMergeOneWaveHeads = 256;
template <int NW>
__global__ void lse_merge_kernel(const float* __restrict__ part_m, const float* __restrict__ part_l,
                                 const float* __restrict__ part_acc, int S, const int2* __restrict__ table, int G,
                                 uint16_t* __restrict__ out, float* __restrict__ lse);

}  // namespace ffd
