// What the matrix-core attention kernels share: vector types, conversions, the LDS reads and waits
// written as asm, and the reciprocal divisions of their work-item decode.
#pragma once

#include "common.hpp"

namespace ddt {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

constexpr float kLog2e = 1.4426950408889634f;

__host__ __device__ __forceinline__ uint32_t magic_of(uint64_t d, uint64_t x_max)
{
    return (d >= 2 && x_max * d < 0x100000000ull) ? (uint32_t)((0x100000000ull + d - 1) / d) : 0u;
}
__host__ __device__ __forceinline__ int div_by(int x, int d, uint32_t magic)
{
    return magic != 0u ? (int)(((uint64_t)(uint32_t)x * magic) >> 32) : (d == 1 ? x : x / d);
}

constexpr int kHD = 128;  // head dim of attn_mfma_kernel
constexpr int kKT = 64;   // its keys per tile
constexpr int kSK = 32;   // attn_wave_kernel: keys per sub-tile

// ---- how a call is cut into workgroups, and the layout of its scratch (attn_plan.hip) ----
struct AttnSeqPlan {
    int32_t splits;       // key ranges of a row group (attn_wave_kernel) or of a whole row tile
    int32_t tail_splits;  // of a tail block (attn_mfma_kernel, uneven form)
    int32_t ranges;       // partial results of a row: the larger of the two; 1: none, the output is direct
    int32_t first_slot;   // the first of its partial results
};
struct AttnPlan {
    double cost;          // estimated time (us)
    // partial results: `slots` times the T * Hq rows of a sequence
    long long slots;
    size_t part_off, lse_off, bytes;
    bool wide;            // they are fp32 rows, otherwise fp16 relative to their row's largest magnitude
    AttnSeqPlan seq[DDTREE_MAX_BATCH];
    long long items;      // workgroups with work
    // attn_wave_kernel (row_blocks > 0): `groups` row groups of rows_per_group <= 32 * row_blocks rows
    int row_blocks, groups, rows_per_group;
    // attn_mfma_kernel: the query rows of one (sequence, kv head) pair, in blocks of 32.  Even form: dealt
    // as evenly as possible to n_tiles row tiles of at most 8 blocks, tile i holds blk_base +
    // (i < blk_extra).  Uneven form: n_tiles tiles of 8 blocks and blk_extra tail blocks on their own.
    int n_tiles, blk_base, blk_extra;
    bool uneven;
};
bool attn_mfma_shape(int dtype, int D, int Hkv);
bool attn_rows_fit(int T, int Hq, int Hkv);  // the query rows of a KV head are counted in 32 bits
// scratch: bytes at hand.
AttnPlan attn_plan(int batch, int T, int Hq, int Hkv, int D, const int32_t *kv_len, size_t scratch);
bool attn_lacks_scratch(int batch, int T, int Hq, int Hkv, int D, const int32_t *kv_len, size_t scratch);

// ---- attn_wave_kernel ----
struct AttnWaveSeq {
    int32_t seq, kv_start, kv_len, first_unit;  // sequences longest first; their first (key range, kv head)
    int32_t splits, first_slot, ranges;
    uint32_t splits_magic;               // reciprocal of splits
};
struct AttnWaveArgs {
    const uint16_t *q, *k_cache, *v_cache, *k_tree, *v_tree;
    const uint64_t *mask;
    uint16_t *out;
    void *part;
    float2 *lse;
    int32_t T, Hq, Hkv;
    int32_t batch, items, run;           // work items; consecutive ones that an XCD takes at a time
    int32_t groups, rows_per_group;
    int32_t group_size;                  // G = Hq / Hkv
    uint32_t g_magic, groups_magic, hkv_magic, run_magic;  // reciprocals of G, groups, Hkv, run
    int32_t per_seq;                     // (key range, kv head) pairs of every sequence, 0 where they differ
    uint32_t per_seq_magic;
    int32_t grid;
    float scale_log2e;
    AttnWaveSeq seq[DDTREE_MAX_BATCH];   // (behind what every workgroup reads first)
};
bool attn_wave_args(AttnWaveArgs &args, const AttnPlan &p, const int32_t *kv_start, const int32_t *kv_len, int batch,
                    int T, int Hq, int Hkv);
bool attn_wave_launch(const AttnWaveArgs &args, int D, int row_blocks, bool wide, hipStream_t st);

struct AttnWaveItem {
    int seq, hk, grp, split, splits, ranges, first_slot, kv_start, kv_len;
    int r0, r1;                  // query rows (node, head of the group)
    int n_cache, t_begin, t_end; // cache sub-tiles; the sub-tiles of the key range
};
// What workgroup `b` works on; false: nothing.
__host__ __device__ __forceinline__ bool attn_wave_item(const AttnWaveArgs &args, int b, AttnWaveItem &w)
{
    // Workgroups are dealt to the 8 XCDs in turn; an XCD takes `run` consecutive work items at a time.
    // (A single sequence's entry is requested with everything else, not behind the search: 61 nodes x 3001 keys, launch to
    // launch with the merge, whose first range is a scalar argument now too, 14.85 -> 14.15 us.)
    const AttnWaveSeq first = args.seq[0];
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" ::"s"(first.kv_start), "s"(first.kv_len), "s"(first.splits), "s"(first.splits_magic), "s"(first.first_slot),
                 "s"(first.ranges));
#endif
    const int j = b >> 3, k = div_by(j, args.run, args.run_magic);
    const int wid = (k * 8 + (b & 7)) * args.run + (j - k * args.run);
    if (wid >= args.items) return false;
    const int unit = div_by(wid, args.groups, args.groups_magic);
    w.grp = wid - unit * args.groups;
    AttnWaveSeq e = first;
    if (args.batch > 1) {
        int pos = 0;  // the last sequence whose first unit is not behind this one
        if (args.per_seq > 0) {
            pos = div_by(unit, args.per_seq, args.per_seq_magic);
        } else {
#pragma unroll
            for (int s = 32; s >= 1; s >>= 1)
                if (pos + s < args.batch && args.seq[pos + s].first_unit <= unit) pos += s;
        }
        e = args.seq[pos];
    }
    const int local = unit - e.first_unit;
    w.split = div_by(local, args.Hkv, args.hkv_magic);
    w.hk = local - w.split * args.Hkv;
    w.seq = e.seq, w.kv_start = e.kv_start, w.kv_len = e.kv_len;
    w.splits = e.splits, w.first_slot = e.first_slot, w.ranges = e.ranges;
    w.r0 = w.grp * args.rows_per_group;
    w.r1 = w.r0 + args.rows_per_group;
    if (w.r1 > args.T * args.group_size) w.r1 = args.T * args.group_size;
    const int last_node = div_by(w.r1 - 1, args.group_size, args.g_magic);
    w.n_cache = (int)(((unsigned)w.kv_len + kSK - 1) / (unsigned)kSK);
    const int nt = w.n_cache + last_node / kSK + 1;
    w.t_begin = div_by(nt * w.split, w.splits, e.splits_magic);
    w.t_end = div_by(nt * (w.split + 1), w.splits, e.splits_magic);
    return true;
}

// ---- attn_mfma_kernel ----
struct AttnMainSeq {
    int32_t seq, kv_start, kv_len;       // sequences longest first
    int32_t first_item, first_tail;      // their first work item among the whole tiles', among the tail blocks'
    int32_t splits, tail_splits, first_slot, ranges;
    // reciprocals of the work items per kv head (whole tiles', tail blocks'), of splits and of tail_splits
    uint32_t head_magic, tail_head_magic, splits_magic, tail_magic;
};
struct AttnMainArgs {
    // XCD x executes the whole tiles' work items xcd_start[x] .. xcd_start[x + 1] - 1, then the tail
    // blocks' tail_start[x] .. tail_start[x + 1] - 1
    int32_t xcd_start[9], tail_start[9];
    int32_t batch, n_tiles, blk_base, blk_extra, uneven;
    int32_t group_size;                  // G = Hq / Hkv
    uint32_t g_magic, tiles_magic, extra_magic;  // reciprocals of G, n_tiles and blk_extra
    // work items of every sequence, whole tiles' and tail blocks', 0 where they differ (the search for the sequence
    // is a chain of six loads: 0.7 us of 14 for 16 sequences of 36 nodes x 127 keys)
    int32_t per_seq, tail_per_seq;
    uint32_t per_seq_magic, tail_per_seq_magic;
    int32_t grid;
    AttnMainSeq seq[DDTREE_MAX_BATCH];
};
bool attn_main_args(AttnMainArgs &args, const AttnPlan &p, const int32_t *kv_start, const int32_t *kv_len, int batch,
                    int T, int Hq, int Hkv);

struct AttnMainItem {
    int seq, hk, split, splits, ranges, first_slot, kv_start, kv_len;
    bool tail;                    // a tail block: sub-tiles of kSK keys, otherwise tiles of kKT
    int m0, m_end;                // query rows
    int n_cache, t_begin, t_end;  // (sub-)tiles of the cache; those of the key range
};
// What workgroup `b` works on; false: nothing.  Work items of either kind: sequence by sequence, kv head by
// kv head, key range by key range, row tile (tail block) fastest.
__host__ __device__ __forceinline__ bool attn_main_item(const AttnMainArgs &args, int b, int T, AttnMainItem &w)
{
    // (a single sequence's entry is requested with everything else, not behind the search)
    const AttnMainSeq first = args.seq[0];
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" ::"s"(first.kv_start), "s"(first.kv_len), "s"(first.splits), "s"(first.head_magic), "s"(first.splits_magic),
                 "s"(first.tail_splits), "s"(first.tail_head_magic), "s"(first.tail_magic), "s"(first.ranges), "s"(first.first_slot));
#endif
    const int x = b & 7, n_main = args.xcd_start[x + 1] - args.xcd_start[x];
    int wid = b >> 3;
    w.tail = wid >= n_main;
    wid += w.tail ? args.tail_start[x] - n_main : args.xcd_start[x];
    if (w.tail && wid >= args.tail_start[x + 1]) return false;
    AttnMainSeq e = first;
    if (args.batch > 1) {
        int pos = 0;
        const int per_seq = w.tail ? args.tail_per_seq : args.per_seq;
        if (per_seq > 0) {
            pos = div_by(wid, per_seq, w.tail ? args.tail_per_seq_magic : args.per_seq_magic);
        } else {
#pragma unroll
            for (int s = 32; s >= 1; s >>= 1)
                if (pos + s < args.batch && (w.tail ? args.seq[pos + s].first_tail : args.seq[pos + s].first_item) <= wid) pos += s;
        }
        e = args.seq[pos];
    }
    const int local = wid - (w.tail ? e.first_tail : e.first_item);
    const int tiles = w.tail ? args.blk_extra : args.n_tiles;
    const int per_head = tiles * (w.tail ? e.tail_splits : e.splits);
    w.hk = div_by(local, per_head, w.tail ? e.tail_head_magic : e.head_magic);
    const int wg = local - w.hk * per_head;
    w.split = div_by(wg, tiles, w.tail ? args.extra_magic : args.tiles_magic);
    const int tile = wg - w.split * tiles;
    w.splits = w.tail ? e.tail_splits : e.splits;
    w.seq = e.seq, w.kv_start = e.kv_start, w.kv_len = e.kv_len, w.ranges = e.ranges, w.first_slot = e.first_slot;
    const int M = T * args.group_size;
    const int extra = args.uneven ? 0 : args.blk_extra;
    const int first_blk = w.tail ? args.n_tiles * 8 + tile : tile * args.blk_base + (tile < extra ? tile : extra);
    const int n_blk = w.tail ? 1 : args.blk_base + (tile < extra ? 1 : 0);
    w.m0 = first_blk * 32;
    w.m_end = (first_blk + n_blk) * 32 < M ? (first_blk + n_blk) * 32 : M;
    const int last_node = div_by(w.m_end - 1, args.group_size, args.g_magic);
    const int keys = w.tail ? kSK : kKT;
    w.n_cache = (int)(((unsigned)w.kv_len + keys - 1) / (unsigned)keys);
    const int nt = w.n_cache + last_node / keys + 1;
    // key ranges rounded up, so that a surplus tile goes to the early ranges: the last range holds
    // the tree tiles, which carry the mask work on top
    // (nt * splits < 2^30 wherever a key range is cut: 32-bit arithmetic is exact)
    const uint32_t magic = w.tail ? e.tail_magic : e.splits_magic;
    w.t_begin = div_by(nt * w.split + w.splits - 1, w.splits, magic);
    w.t_end = div_by(nt * (w.split + 1) + w.splits - 1, w.splits, magic);
    return true;
}

#if defined(__HIPCC__)
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
// two floats -> packed bf16 pair (round to nearest even), one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t f2bf_pair(float lo, float hi)
{
    const floatx2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// two floats -> packed fp16 pair (round to nearest even)
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t f2h_pair(float lo, float hi)
{
    const f16x2 h = {(_Float16)lo, (_Float16)hi};
    return __builtin_bit_cast(uint32_t, h);
}

// Compile-time loop: f(IC<B>{}), ..., f(IC<E-1>{}); the index is a constant expression inside f,
// as the immediate operands of the asm helpers below require.
template <int N>
struct IC {
    static constexpr int value = N;
};
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (B < E) {
        f(IC<B>{});
        static_for<B + 1, E>(f);
    }
}

// Reads of the K/V tiles are written as asm.  The tiles are filled by LDS-DMA
// (global_load_lds); the compiler cannot tell which stage a given LDS read touches and would
// wait for every outstanding tile load before each read, serialising prefetch and compute.  With
// asm reads the waits are placed by hand: s_waitcnt vmcnt(0) + barrier once per tile for the
// DMA, lds_wait_*() below for the reads (LDS reads return in order, so "at most N outstanding"
// identifies exactly which of them have landed).
// The destination of a read is tied to its previous value ("+v"): the read lands in the register
// of the operand it replaces and cannot be scheduled above the matrix instruction that still
// reads that operand.
template <int OFF>
__device__ __forceinline__ void lds_rd128(u32x4 &v, uint32_t addr)
{
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "+v"(v) : "v"(addr), "n"(OFF) : "memory");
}
// LDS transpose read (ds_read_b64_tr_b16).  Within each group of 16 lanes, lane 4*j + r points
// at four consecutive 16-bit elements; afterwards lane i of the group holds, for j = 0..3, element
// i % 4 of what lane 4*j + i / 4 pointed at.  With lane 4*j + r pointing at V[key_j][d0 + 4*r ..],
// lane i receives V[key_0..3][d0 + i]: a column of the row-major V tile, which is what the A
// operand (V^T) of the second product needs.
template <int OFF>
__device__ __forceinline__ void lds_rdtr(u32x2 &v, uint32_t addr)
{
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "+v"(v) : "v"(addr), "n"(OFF) : "memory");
}
template <int N>
__device__ __forceinline__ void vm_wait()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

#endif

}  // namespace ddt
