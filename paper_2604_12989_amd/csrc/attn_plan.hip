// How a call of the attention is cut into workgroups: which of the two matrix-core kernels, how many
// key ranges each sequence's rows are cut into, the launch tables the kernels decode, and the host-side
// self-check that holds this arithmetic against plain division and exact coverage.  Host code only.
#include <algorithm>
#include <vector>

#include "attn_common.hpp"

namespace ddt {

// Shapes of the matrix-core kernels.  (The bound on the KV heads keeps the pitch between cache
// rows below 2^24 bytes, which the kernels' 24-bit address multiplies rely on.)
bool attn_mfma_shape(int dtype, int D, int Hkv)
{
    return dtype == DDTREE_DTYPE_BF16 && (D == kHD || D == 64) && Hkv <= 32768;
}

// Whether the partial results of a call are fp32 rows.  They are, except where few workgroups share long caches:
// there, row tiles of the same height walked uncut leave compute units idle or a last round nearly empty, the key
// ranges have to be cut for any speed at all, and fp16 relative to the row's largest magnitude (2^-11, the
// result's own rounding is 2^-9) halves the bytes of many partials (a merge of 7 x 257 x 32 rows: 5.3 us).  A call
// that does not have to be cut loses no bits where it is cut all the same.  Heads of 64: always fp32.
static bool wide_partials(int batch, int T, int Hq, int Hkv, int D, long long sum_L)
{
    if (D != kHD) return true;
    const long long tiles = (sum_L / batch + T) / kKT;
    const long long items = (long long)batch * Hkv * (((long long)T * (Hq / Hkv) + 255) / 256), rounds = (items + 255) / 256;
    for (long long s = 2; s <= 32 && s * 4 <= tiles; ++s)
        if ((double)((items * s + 255) / 256) * (1.0 + 0.02 * (double)(s - 1)) < (double)(s * rounds)) return false;
    return true;
}

// Scratch of `slots` partial results: their rows, then (log2-sum-exp, scale) per row.
static void plan_scratch(AttnPlan &p, int T, int Hq, int D, bool wide, long long slots)
{
    p.slots = slots;
    p.wide = wide;
    p.part_off = p.lse_off = p.bytes = 0;
    if (slots == 0) return;
    const size_t rows = (size_t)slots * T * Hq;
    p.lse_off = align_up(rows * D * (wide ? 4 : 2), 256);
    p.bytes = align_up(p.lse_off + rows * 8, 256);
}

// Partial results that `bytes` of scratch have room for: the most that plan_scratch lays out in them.
static long long slot_room(int T, int Hq, int D, bool wide, size_t bytes)
{
    const long long slots = (long long)(bytes / ((size_t)T * Hq * (D * (wide ? 4 : 2) + 8)));
    AttnPlan p{};
    plan_scratch(p, T, Hq, D, wide, slots);
    return p.bytes <= bytes ? slots : slots - 1;  // (each array is padded to 256 bytes)
}

static inline int up(int a, int b) { return (int)(((unsigned)a + (unsigned)b - 1u) / (unsigned)b); }  // (lengths reach 2^31 - 1)

bool attn_rows_fit(int T, int Hq, int Hkv) { return (long long)T * (Hq / Hkv) <= 0x7FFFFF00ll; }

// Partial results a plan may leave: what about two rounds of workgroups on 256 compute units make.
static long long wave_slot_cap(int batch, int T, int Hq, int Hkv, int row_blocks)
{
    const long long M = (long long)T * (Hq / Hkv);
    return std::max<long long>(batch, 512 / (Hkv * ((M + 32 * row_blocks - 1) / (32 * row_blocks))));
}
static long long main_slot_cap(int batch, int T, int Hq, int Hkv)
{
    const long long M = (long long)T * (Hq / Hkv);
    return batch + 640 / (Hkv * ((M + 255) / 256));
}

static long long slot_cap(int batch, int T, int Hq, int Hkv, int D)
{
    const long long wave = std::max(wave_slot_cap(batch, T, Hq, Hkv, 1), wave_slot_cap(batch, T, Hq, Hkv, 2));
    return D == kHD ? std::max(wave, main_slot_cap(batch, T, Hq, Hkv)) : wave;
}

// Time (us) of the merge of `slots` partial results: a launch, and reading them.  (Measured, fp16: 4.0 us for
// 3 x 65 x 32 rows of 128, 4.7 for 7 x 257 x 32, 22 for 32 x 129 x 64.)
static double merge_us(long long slots, int T, int Hq, int D, bool wide) { return 4.0 + (double)slots * T * Hq * D * (wide ? 4 : 2) / 6.0e6; }

// Workgroups of a few sizes, longest first: `count` of `cost` us each.
struct Sized {
    double cost;
    long long count;
};
// Their time on 256 compute units, one at a time on each: k times the k-th round's longest, and, where others run
// beside them (`beside`) or their sizes differ, no less than what all of them make together and a third of the longest.
static double rounds_us(const Sized *w, int n, bool beside, double tail)
{
    long long items = 0;
    double sum = 0.0, t = 0.0;
    for (int i = 0; i < n; ++i) {
        for (long long k = (items + 255) / 256; k * 256 < items + w[i].count; ++k) t = std::max(t, (double)(k + 1) * w[i].cost);
        items += w[i].count;
        sum += w[i].cost * w[i].count;
    }
    return items <= 256 || (n == 1 && !beside) ? t : std::max(t, sum / 256 + tail * w[0].cost);
}

// The lengths of a call as the plans see them: sequences longest first, those of the same number of cache
// sub-tiles counted together.  (A plan is made for every call, in its host time: one sort, one entry for each
// different length, and searches that end where neither fewer keys a range nor another partial result
// can pay any more.  Host time of a plan before and now: 257 nodes x 8192 keys 3.0 -> 1.5, four ragged sequences of 101 nodes
// 4.6 -> 2.2, 16 of 129 10.5 -> 2.3, 64 of 257 36 -> 4.0 us.)
struct Lens {
    int n = 0;
    int32_t sub[DDTREE_MAX_BATCH], count[DDTREE_MAX_BATCH];
    int32_t order[DDTREE_MAX_BATCH];
};
static Lens lens_of(const int32_t *kv_len, int batch)
{
    Lens l;
    uint64_t key[DDTREE_MAX_BATCH];
    for (int i = 0; i < batch; ++i) key[i] = (uint64_t)(0x7FFFFFFF - kv_len[i]) << 32 | (uint32_t)i;
    std::sort(key, key + batch);
    for (int i = 0; i < batch; ++i) {
        l.order[i] = (int32_t)(uint32_t)key[i];
        const int sub = up(kv_len[l.order[i]], kSK);
        if (l.n > 0 && l.sub[l.n - 1] == sub) {
            ++l.count[l.n - 1];
        } else {
            l.sub[l.n] = sub;
            l.count[l.n++] = 1;
        }
    }
    return l;
}

// x / d rounded up for many x: a multiplication by ceil(2^64 / d), exact for 32-bit operands.
struct DivUp {
    unsigned d;
    uint64_t m;
    explicit DivUp(int by) : d((unsigned)by), m(~0ull / (unsigned)by + 1) {}
    int operator()(int x) const
    {
        const unsigned y = (unsigned)x + d - 1u;
        return d == 1u ? (int)y : (int)(uint64_t)((unsigned __int128)y * m >> 64);
    }
};

// attn_wave_kernel: every sequence's key range in pieces of about the same length, so that the pieces
// of a ragged batch end together.
static AttnPlan plan_wave(int batch, int T, int Hq, int Hkv, int D, const int32_t *kv_len, const Lens &lens, int row_blocks, bool wide,
                          long long room)
{
    AttnPlan p{};
    const int M = T * (Hq / Hkv);
    p.row_blocks = row_blocks;
    p.groups = up(M, 32 * row_blocks);
    p.rows_per_group = up(M, p.groups);
    const long long cap = std::min(room, wave_slot_cap(batch, T, Hq, Hkv, row_blocks));
    const int tree = up(T, kSK);
    long long sub_tiles = 0;
    for (int i = 0; i < lens.n; ++i) sub_tiles += (long long)(lens.sub[i] + tree) * lens.count[i];
    const int nt_max = lens.sub[0] + tree;
    Sized sized[DDTREE_MAX_BATCH];
    // Measured (us): a workgroup's fixed cost (launch, first requests, combining the waves' results), a
    // step of its eight waves (32 keys each), the rates at which the L2s and HBM serve all of them.
    // A step whose keys no L2 holds waits for HBM, in one workgroup's row group at least (48 workgroups of one row
    // group over 85 MB: 2.7 us; 192 to 512 of four over 79 to 363 MB: 2.3 to 2.5, of ten and more 1.3 to 1.8).
    const double far = D == 64 ? 0.0 : std::min(1.0, std::max(0.0, ((double)sub_tiles * Hkv * (kSK * 4.0 * D) * 1e-6 - 24.0) / 48.0)) *
                                           (p.groups <= 6 ? 1.0 : p.groups <= 9 ? 0.7 : 0.3);
    const double fix = 7.0, step = D == 64 ? (row_blocks == 1 ? 0.62 : 1.17) : 1.2 + 1.2 * far;
    const double masked = D == 64 ? 0.0 : 0.19;  // more for each sub-tile of a large tree (997 nodes over 230 keys: 2.7 us a step)
    const double l2_us = (double)sub_tiles * Hkv * p.groups * (kSK * 4.0 * D) / 20.0e6;
    const double hbm_us = (double)sub_tiles * Hkv * (kSK * 4.0 * D) / 4.0e6;
    const double least = 5.0 + std::max(l2_us, hbm_us);
    int best_c = nt_max;
    p.cost = 1e30;
    for (int s = 1; s <= 64 && (s == 1 || (s * 4 <= nt_max && (long long)s * nt_max < (1ll << 30))); ++s) {
        const int c = up(nt_max, s);
        const DivUp by_c(c);
        long long slots = 0;
        for (int i = 0; i < lens.n; ++i) {
            const int nt = lens.sub[i] + tree, si = by_c(nt);
            slots += (long long)si * lens.count[i];
            const int range = si == 1 ? nt : up(nt, si);
            sized[i] = Sized{fix + step * up(range, 8) + masked * std::max(0, std::min(tree, range) - 8),
                             (long long)lens.count[i] * si * Hkv * p.groups};
        }
        const double merge = s > 1 ? merge_us(slots, T, Hq, D, wide) : 0.0;
        if (s > 1 && (slots > cap || least + merge >= p.cost)) break;  // (partial results only grow in number)
        const double cost = std::max(rounds_us(sized, lens.n, false, 0.0), least) + merge;
        if (cost < p.cost) p.cost = cost, best_c = c;
    }
    int first = 0;
    bool cut = false;
    const DivUp by_c(best_c);
    for (int i = 0; i < batch; ++i) {
        const int si = by_c(up(kv_len[i], kSK) + tree);
        p.seq[i] = AttnSeqPlan{si, 0, si, first};
        first += si;
        cut = cut || si > 1;
    }
    p.items = (long long)first * Hkv * p.groups;
    plan_scratch(p, T, Hq, D, wide, cut ? first : 0);
    return p;
}

// attn_mfma_kernel.  Even form: row tiles of the same height.  Uneven form, where the blocks of 32 rows are
// a few more than whole tiles of 8 (T = 257 with four heads per KV head: 33 blocks): whole tiles, and each
// block left as a work item of its own with key ranges of its own (attn_wave_rows).
static AttnPlan plan_main(int batch, int T, int Hq, int Hkv, const int32_t *kv_len, const Lens &lens, bool wide, long long room)
{
    const int nblk = up(T * (Hq / Hkv), 32), full = nblk / 8, rem = nblk % 8;
    const int tree = up(T, kKT), tree_sub = up(T, kSK);
    static_assert(kKT == 2 * kSK, "key tiles from sub-tiles");
    const int nt_max = up(lens.sub[0], 2) + tree;
    const int sub_max = lens.sub[0] + tree_sub;
    Sized sized[DDTREE_MAX_BATCH];
    long long key_tiles = 0;
    for (int i = 0; i < lens.n; ++i) key_tiles += (long long)(up(lens.sub[i], 2) + tree) * lens.count[i];
    const double hbm_us = (double)key_tiles * Hkv * (kKT * 4.0 * kHD) / 5.8e6;
    // Measured (us): a workgroup's fixed cost and a key tile (below three quarters of the compute units at work,
    // and with all of them, where the chip lowers its clock: 1.92 over 131 key tiles); for a tail block, and a
    // step of eight sub-tiles beside them (1.2 alone, keys from the L2).  With 513 nodes x 32768 keys, four key
    // ranges and the tail blocks in a second round (the sum of times says 246 us) took 340 where three and
    // everything in one round take 307: the few workgroups of that second round wait for HBM.
    // Workgroups of fewer blocks (few rows over long caches) spend less on a tile: of one or two 0.9, of three or four
    // 1.05 and with all compute units at work 1.15, of five or six 1.45 and 1.55; up to four, less on the rest too.
    const double tail_fix = 7.0, tail_step = 2.4;
    const long long cap = std::min(room, main_slot_cap(batch, T, Hq, Hkv));
    AttnPlan best{};
    best.cost = 1e30;
    int best_c = nt_max, best_ct = 0;
    int si[DDTREE_MAX_BATCH], range[DDTREE_MAX_BATCH];
    for (int uneven = 0; uneven < 2; ++uneven) {
        if (uneven && !(full >= 1 && rem >= 1 && rem <= 4)) break;
        const int tiles = uneven ? full : up(nblk, 8), blocks = uneven ? 8 : up(nblk, tiles);
        const double tile_few = blocks <= 2 ? 0.95 : blocks <= 4 ? 1.05 : blocks <= 6 ? 1.45 : 1.52;
        const double tile_all = blocks <= 2 ? 0.95 : blocks <= 4 ? 1.15 : blocks <= 6 ? 1.55 : 1.9;
        const double fix = blocks <= 4 ? 9.0 : 11.0;
        bool more = true;
        for (int s = 1, c_before = 0; more && s <= 32 && (s == 1 || s * 2 <= nt_max); ++s) {
            const int c = up(nt_max, s);
            if (c == c_before) continue;
            c_before = c;
            const DivUp by_c(c);
            long long items = 0, main_slots = 0;
            for (int i = 0; i < lens.n; ++i) {
                si[i] = by_c(up(lens.sub[i], 2) + tree);
                items += sized[i].count = (long long)tiles * si[i] * Hkv * lens.count[i];
                main_slots += (long long)si[i] * lens.count[i];
            }
            // (with shorter key ranges both kinds leave more partial results: what is too many, or too many to pay, stays so)
            const double least = fix + hbm_us;
            if (s > 1 && (main_slots > cap || least + merge_us(main_slots, T, Hq, kHD, wide) >= best.cost)) break;
            // compute units at work while the longest range is walked, on average (those of short sequences end early)
            int longest = 1;
            double walked = 0.0;
            for (int i = 0; i < lens.n; ++i) {
                const int nt = up(lens.sub[i], 2) + tree;
                range[i] = si[i] == 1 ? nt : up(nt, si[i]);
                longest = std::max(longest, range[i]);
                walked += (double)range[i] * sized[i].count;
            }
            const double tile = tile_few + (tile_all - tile_few) * std::min(1.0, std::max(0.0, (walked / longest - 192) / 64.0));
            double main_sum = 0.0;
            for (int i = 0; i < lens.n; ++i) {
                sized[i].cost = fix + tile * range[i];
                main_sum += sized[i].cost * sized[i].count;
            }
            const double main_work = rounds_us(sized, lens.n, uneven != 0, 0.5);
            if (s > 1 && std::max(main_work, least) + merge_us(main_slots, T, Hq, kHD, wide) >= best.cost) continue;
            // ranges of a tail block: those that take as long as a whole tile's, and more of them in turn
            const int t0 = uneven ? std::min(32, std::max(1, (int)(tail_step * up(sub_max, 8) / (fix - tail_fix + tile_few * c)))) : 0;
            for (int t = t0; t <= std::min(8 * t0, 32); t *= 2) {
                if (t > 1 && (long long)t * sub_max >= (1ll << 30)) break;
                const int ct = uneven ? up(sub_max, t) : 0;
                long long tails = 0, slots = main_slots;
                double sum = main_sum, tail_longest = 0.0;
                if (uneven) {
                    const DivUp by_ct(ct);
                    for (int i = 0; i < lens.n; ++i) {
                        const int sub = lens.sub[i] + tree_sub, ti = by_ct(sub);
                        const double each = tail_fix + tail_step * up(ti == 1 ? sub : up(sub, ti), 8);
                        const long long n = (long long)rem * ti * Hkv * lens.count[i];
                        sum += each * n;
                        tail_longest = std::max(tail_longest, each);
                        tails += n;
                        slots += (long long)std::max(0, ti - si[i]) * lens.count[i];
                    }
                }
                const bool cut = s > 1 || t > 1;
                const double merge = cut ? merge_us(slots, T, Hq, kHD, wide) : 0.0;
                if (cut && (slots > cap || least + merge >= best.cost)) {
                    more = t > t0;
                    break;
                }
                // the whole tiles' items as if alone; the tail blocks' beside them, or where they end
                double work = main_work;
                if (items + tails <= 256)
                    work = std::max(work, tail_longest);
                else if (items <= 256)
                    work += tails > 0 ? std::max(1.5 * tail_longest * up((int)tails, 256), 1.2 * hbm_us) : 0.0;  // (they read the keys again)
                else
                    work = std::max(work, sum / 256 + 0.5 * tail_longest);
                const double cost = std::max(work, least) + merge;
                if (cost < best.cost) {
                    best.cost = cost;
                    best.uneven = uneven != 0;
                    best_c = c, best_ct = ct;
                    best.items = items + tails;
                }
                if (!uneven) break;
            }
        }
    }
    best.n_tiles = best.uneven ? full : up(nblk, 8);
    best.blk_base = best.uneven ? 8 : nblk / best.n_tiles;
    best.blk_extra = best.uneven ? rem : nblk % best.n_tiles;
    int first = 0;
    bool cut = false;
    const DivUp by_c(best_c), by_ct(std::max(1, best_ct));
    for (int i = 0; i < batch; ++i) {
        const int cuts = by_c(up(kv_len[i], kKT) + tree);
        const int ti = best.uneven ? by_ct(up(kv_len[i], kSK) + tree_sub) : 0;
        best.seq[i] = AttnSeqPlan{cuts, ti, std::max(cuts, ti), first};
        first += best.seq[i].ranges;
        cut = cut || best.seq[i].ranges > 1;
    }
    plan_scratch(best, T, Hq, kHD, wide, cut ? first : 0);
    return best;
}

// The cheaper of the two by the estimates above.  Both measured where they meet (32 query and 8 KV heads
// of 128, one sequence; waves of their own / shared tiles, us): 129 nodes x 4096 keys 26.8 / 26.9,
// 401 x 600 21.8 / 25.7, 257 x 8192 102 / 51, 17 x 8192 17.5 / 20.7; 16 sequences of 10 nodes over up to 26246 keys, 16 and
// 4 heads, 145 / 103, four of 19 over up to 8468 31 / 36.  Heads of 64: 32-row groups against 64-row
// groups at 257 x 4096 36.9 / 28.5 (two rounds of workgroups against one), at 65 x 2047 11.5 / 13.0.
AttnPlan attn_plan(int batch, int T, int Hq, int Hkv, int D, const int32_t *kv_len, size_t scratch)
{
    long long sum_L = 0;
    for (int i = 0; i < batch; ++i) sum_L += kv_len[i];
    const bool wide = wide_partials(batch, T, Hq, Hkv, D, sum_L);
    const long long room = slot_room(T, Hq, D, wide, scratch);
    const Lens lens = lens_of(kv_len, batch);
    const AttnPlan w = plan_wave(batch, T, Hq, Hkv, D, kv_len, lens, 1, wide, room);
    const AttnPlan m = D == kHD ? plan_main(batch, T, Hq, Hkv, kv_len, lens, wide, room)
                                : plan_wave(batch, T, Hq, Hkv, D, kv_len, lens, 2, wide, room);
    return w.cost <= m.cost ? w : m;
}

// A long key range that few workgroups share is not walked uncut because a workspace is missing: such a call
// is refused, unless its plan takes no scratch in any case.
bool attn_lacks_scratch(int batch, int T, int Hq, int Hkv, int D, const int32_t *kv_len, size_t scratch)
{
    const long long tiles = (long long)batch * Hkv * (((long long)T * (Hq / Hkv) + 255) / 256);
    if (D != kHD || tiles > 128) return false;
    long long sum_L = 0;
    for (int i = 0; i < batch; ++i) sum_L += kv_len[i];
    if ((sum_L / batch + T) / kKT < 8 || slot_room(T, Hq, D, false, scratch) >= 2LL * batch) return false;
    return attn_plan(batch, T, Hq, Hkv, D, kv_len, SIZE_MAX).bytes > scratch;
}

size_t attn_scratch_upper(int batch, int T, int Hq, int Hkv, int D)
{
    if (!attn_mfma_shape(DDTREE_DTYPE_BF16, D, Hkv)) return 0;
    const long long slots = slot_cap(batch, T, Hq, Hkv, D);
    const long long tiles = (long long)batch * Hkv * (((long long)T * (Hq / Hkv) + 255) / 256);
    // (fp32 partials of at most 128 row tiles: fewer than eight key tiles a sequence, no range shorter than two)
    AttnPlan narrow{}, wide{};
    plan_scratch(narrow, T, Hq, D, false, slots);
    plan_scratch(wide, T, Hq, D, true, D == kHD && tiles <= 128 ? std::min(slots, 6LL * batch) : slots);
    return std::max(D == kHD ? narrow.bytes : 0, wide.bytes);
}

// The lengths of the sequences are not known here: no key range is shorter than two key tiles, and a
// single sequence takes what the plan for its length takes.
size_t attn_scratch_bytes(int batch, int T, int Hq, int Hkv, int D, int dtype, long long sum_L)
{
    if (!attn_mfma_shape(dtype, D, Hkv) || !attn_rows_fit(T, Hq, Hkv)) return 0;
    if (batch == 1 && sum_L <= 0x7FFFFFFF) {
        const int32_t len = (int32_t)sum_L;
        return attn_plan(1, T, Hq, Hkv, D, &len, SIZE_MAX).bytes;
    }
    const long long slots = std::min(slot_cap(batch, T, Hq, Hkv, D), batch + (sum_L + (T + 128LL) * batch) / (2 * kKT));
    AttnPlan p{};
    plan_scratch(p, T, Hq, D, wide_partials(batch, T, Hq, Hkv, D, sum_L), slots);
    return p.bytes;
}

static bool same_of_all(const AttnPlan &p, int batch, int32_t AttnSeqPlan::*of)
{
    for (int i = 1; i < batch; ++i)
        if (p.seq[i].*of != p.seq[0].*of) return false;
    return true;
}

// False if the launch would exceed 2^28 work items.
bool attn_wave_args(AttnWaveArgs &args, const AttnPlan &p, const int32_t *kv_start, const int32_t *kv_len, int batch,
                    int T, int Hq, int Hkv)
{
    if (p.items > (1ll << 28)) return false;
    const int G = Hq / Hkv;
    args.T = T, args.Hq = Hq, args.Hkv = Hkv, args.batch = batch;
    args.items = (int32_t)p.items;
    args.groups = p.groups;
    args.rows_per_group = p.rows_per_group;
    args.group_size = G;
    // One round: an eighth of the items per XCD, consecutive ones, which read the same keys.  More: the row
    // groups of one key range go to one XCD, the key ranges to the XCDs in turn, so that each has its
    // share of the long sequences.
    args.run = p.items <= 256 ? (int32_t)((p.items + 7) / 8) : p.groups;
    const int per_pass = 8 * args.run;
    args.grid = (int32_t)((p.items + per_pass - 1) / per_pass * per_pass);
    args.g_magic = magic_of((uint64_t)G, (uint64_t)T * G);
    args.groups_magic = magic_of((uint64_t)p.groups, (uint64_t)p.items);
    args.hkv_magic = magic_of((uint64_t)Hkv, (uint64_t)p.items);
    args.run_magic = magic_of((uint64_t)args.run, (uint64_t)args.grid);
    const Lens lens = lens_of(kv_len, batch);
    const int32_t *const order = lens.order;
    int unit = 0;
    for (int i = 0; i < batch; ++i) {
        const int s = order[i];
        args.seq[i] = AttnWaveSeq{s, kv_start[s], kv_len[s], unit, p.seq[s].splits, p.seq[s].first_slot, p.seq[s].ranges,
                                  magic_of((uint64_t)p.seq[s].splits, (uint64_t)(up(kv_len[s], kSK) + up(T, kSK)) * p.seq[s].splits)};
        unit += p.seq[s].splits * Hkv;
    }
    args.per_seq = batch > 1 && same_of_all(p, batch, &AttnSeqPlan::splits) ? p.seq[0].splits * Hkv : 0;
    args.per_seq_magic = magic_of((uint64_t)args.per_seq, (uint64_t)unit);
    return true;
}

// False if the launch would exceed 2^28 work items, or if the tables do not hold exactly the plan's items.
bool attn_main_args(AttnMainArgs &args, const AttnPlan &p, const int32_t *kv_start, const int32_t *kv_len, int batch,
                    int T, int Hq, int Hkv)
{
    const int G = Hq / Hkv, tails = p.uneven ? p.blk_extra : 0;
    args.batch = batch, args.n_tiles = p.n_tiles, args.blk_base = p.blk_base, args.blk_extra = p.blk_extra;
    args.uneven = p.uneven ? 1 : 0;
    args.group_size = G;
    args.g_magic = magic_of((uint64_t)G, (uint64_t)T * G);
    const Lens lens = lens_of(kv_len, batch);
    int32_t order[DDTREE_MAX_BATCH];
    // In one round, where the XCDs take equal numbers of items, each gets long and short sequences alike: the 8 k-th
    // longest are dealt to the XCDs in turn, forth and back.
    if (p.items <= 256 && batch >= 16)
        for (int x = 0, n = 0; x < 8; ++x)
            for (int i = 0; i < batch; i += 8) {
                const int from = i + ((i & 8) ? 7 - x : x);
                if (from < batch) order[n++] = lens.order[from];
            }
    else
        std::copy(lens.order, lens.order + batch, order);
    long long total = 0, tail_total = 0, per_head_max = 1;
    for (int i = 0; i < batch; ++i) {
        const int s = order[i];
        const AttnSeqPlan &q = p.seq[s];
        const long long per_head = (long long)p.n_tiles * q.splits, per_tail = (long long)tails * q.tail_splits;
        const uint64_t nt = (uint64_t)(up(kv_len[s], kKT) + up(T, kKT)), sub = (uint64_t)up(kv_len[s], kSK) + up(T, kSK);
        args.seq[i] = AttnMainSeq{s, kv_start[s], kv_len[s], (int32_t)total, (int32_t)tail_total,
                                  q.splits, q.tail_splits, q.first_slot, q.ranges,
                                  magic_of((uint64_t)per_head, (uint64_t)per_head * Hkv),
                                  per_tail ? magic_of((uint64_t)per_tail, (uint64_t)per_tail * Hkv) : 0u,
                                  magic_of((uint64_t)q.splits, nt * q.splits + q.splits),
                                  per_tail ? magic_of((uint64_t)q.tail_splits, sub * q.tail_splits + q.tail_splits) : 0u};
        total += per_head * Hkv;
        tail_total += per_tail * Hkv;
        if (total + tail_total > (1ll << 28)) return false;
        per_head_max = std::max(per_head_max, std::max(per_head, per_tail));
    }
    args.per_seq = batch > 1 && same_of_all(p, batch, &AttnSeqPlan::splits) ? (int32_t)(total / batch) : 0;
    args.tail_per_seq = batch > 1 && same_of_all(p, batch, &AttnSeqPlan::tail_splits) ? (int32_t)(tail_total / batch) : 0;
    args.per_seq_magic = magic_of((uint64_t)args.per_seq, (uint64_t)total);
    args.tail_per_seq_magic = magic_of((uint64_t)args.tail_per_seq, (uint64_t)tail_total);
    args.tiles_magic = magic_of((uint64_t)p.n_tiles, (uint64_t)per_head_max);
    args.extra_magic = tails ? magic_of((uint64_t)tails, (uint64_t)per_head_max) : 0u;
    // Consecutive work items run on the same XCD: the row tiles that read the same K and V rows share an
    // L2, and those rows leave HBM once.  In one round each XCD has an eighth of the items, at most one
    // per compute unit; otherwise an eighth of the work.
    // The tail blocks' items: to compute units without a whole tile's where there are enough of those,
    // otherwise an eighth of their work to each XCD.
    args.xcd_start[0] = args.tail_start[0] = 0;
    auto by_work = [&](int32_t *start, bool tail, long long all) {
        // in key tiles (sub-tiles): those to visit, and seven for a workgroup's fixed cost
        const int rows = tail ? tails : p.n_tiles, keys = tail ? kSK : kKT;
        auto pieces = [&](int i) { return (long long)rows * (tail ? p.seq[order[i]].tail_splits : p.seq[order[i]].splits) * Hkv; };
        auto cost = [&](int i) { return (double)(up(kv_len[order[i]], keys) + up(T, keys)) * rows * Hkv + 7.0 * pieces(i); };
        double work = 0.0, done = 0.0;
        for (int i = 0; i < batch; ++i) work += cost(i);
        int x = 1;
        for (int i = 0; i < batch; ++i) {
            const double each = cost(i) / pieces(i);
            for (; x < 8 && work * x / 8 < done + cost(i); ++x)
                start[x] = (tail ? args.seq[i].first_tail : args.seq[i].first_item) +
                           (int32_t)std::min<long long>(pieces(i), (long long)((work * x / 8 - done) / each + 0.5));
            done += cost(i);
        }
        for (; x <= 8; ++x) start[x] = (int32_t)all;
        start[8] = (int32_t)all;
        for (x = 0; x < 8; ++x) start[x + 1] = std::max(start[x + 1], start[x]);
    };
    if (total <= 256) {
        const int run = (int)((total + 7) / 8);
        for (int x = 1; x <= 8; ++x) args.xcd_start[x] = (int32_t)std::min<long long>(total, (long long)run * x);
    } else {
        by_work(args.xcd_start, false, total);
    }
    if (tail_total == 0) {
        for (int x = 1; x <= 8; ++x) args.tail_start[x] = 0;
    } else if (total + tail_total > 256) {
        by_work(args.tail_start, true, tail_total);
    } else {
        for (int x = 0; x < 8; ++x) {  // (at most 32 whole tiles' items on each XCD here)
            int idle_behind = 0;  // compute units without an item on the XCDs that follow
            for (int y = x + 1; y < 8; ++y) idle_behind += 32 - (args.xcd_start[y + 1] - args.xcd_start[y]);
            const long long left = tail_total - args.tail_start[x];
            const long long take = std::min<long long>(std::max((tail_total + 7) / 8, left - idle_behind), 32 - (args.xcd_start[x + 1] - args.xcd_start[x]));
            args.tail_start[x + 1] = (int32_t)(args.tail_start[x] + std::min(left, take));
        }
    }
    // every work item has a workgroup, or the call is refused: nothing else would notice a missing one
    bool whole = total + tail_total == p.items && args.xcd_start[8] == total && args.tail_start[8] == tail_total;
    for (int x = 0; x < 8; ++x) whole = whole && args.xcd_start[x + 1] >= args.xcd_start[x] && args.tail_start[x + 1] >= args.tail_start[x];
    if (!whole) return false;
    int run_max = 0;
    for (int x = 0; x < 8; ++x)
        run_max = std::max(run_max, args.xcd_start[x + 1] - args.xcd_start[x] + args.tail_start[x + 1] - args.tail_start[x]);
    args.grid = run_max * 8;
    return true;
}

// ------------------------------------------------------------------------------------------
// Host-side self-check (no GPU involved): for a list of shapes, and for a seeded sweep over batches, head
// layouts, cache lengths and scratch at hand, the plan and the launch tables of both kernels are built as for a
// launch, every workgroup index of the grid is decoded the way the kernel decodes it, and the work items
// are held against what the decomposition promises: every (sequence, KV head, query row) meets every key
// tile exactly once, in consecutive key ranges, and each of its key ranges has a partial result of its own
// within the scratch.
// Returns 0, or 100 * (index of the failing shape + 1) + the number of the failed check, the shapes of the sweep
// counted from kSweepBase on.
// ------------------------------------------------------------------------------------------
namespace {
struct Shape {
    int batch, T, Hq, Hkv, D;
    std::vector<int32_t> len;
};
struct Item {
    int seq, hk, r0, r1, t0, t1, split, ranges, slot, keys_per_tile, nt;
};
constexpr int kSweepBase = 10000, kSweepShapes = 600;
}  // namespace

static int check_items(const Shape &sh, const AttnPlan &p, std::vector<Item> &items, long long expected)
{
    const int G = sh.Hq / sh.Hkv, M = sh.T * G;
    if ((long long)items.size() != expected) return 4;
    for (const Item &w : items) {
        if (w.seq < 0 || w.seq >= sh.batch || w.hk < 0 || w.hk >= sh.Hkv || w.r0 < 0 || w.r0 >= w.r1 || w.r1 > M) return 5;
        if (w.t0 < 0 || w.t0 > w.t1 || w.t1 > w.nt || w.split < 0 || w.split >= w.ranges) return 6;
        if (w.ranges > 1 && (w.slot < 0 || w.slot >= p.slots)) return 7;
        // the last row's own tree key is among the tiles
        if (w.nt < (sh.len[w.seq] + w.keys_per_tile - 1) / w.keys_per_tile + (w.r1 - 1) / G / w.keys_per_tile + 1) return 10;
    }
    // head by head: the row blocks follow each other from 0 to M, the key ranges of a block from 0 to nt
    std::sort(items.begin(), items.end(), [](const Item &a, const Item &b) {
        return a.seq != b.seq ? a.seq < b.seq : a.hk != b.hk ? a.hk < b.hk : a.r0 != b.r0 ? a.r0 < b.r0 : a.split < b.split;
    });
    size_t at = 0;
    for (int head = 0; head < sh.batch * sh.Hkv; ++head)
        for (int row = 0; row < M;) {
            const Item *first = at < items.size() ? &items[at] : nullptr;
            if (!first || first->seq != head / sh.Hkv || first->hk != head % sh.Hkv || first->r0 != row) return 8;
            int next = 0, split = 0;
            for (; at < items.size() && items[at].seq == first->seq && items[at].hk == first->hk && items[at].r0 == row; ++at, ++split) {
                if (items[at].split != split || items[at].t0 != next || items[at].r1 != first->r1) return 8;
                next = items[at].t1;
            }
            if (next != first->nt) return 9;
            row = first->r1;
        }
    if (at != items.size()) return 9;
    // the slots of two sequences do not overlap
    for (int a = 0; a < sh.batch; ++a)
        for (int b = 0; b < sh.batch; ++b)
            if (a != b && p.slots > 0 && p.seq[a].first_slot < p.seq[b].first_slot + p.seq[b].ranges &&
                p.seq[b].first_slot < p.seq[a].first_slot + p.seq[a].ranges)
                return 11;
    return 0;
}

// kind 0, 1: attn_wave_kernel with 32 and 64 rows; 2: attn_mfma_kernel
static int check_plan(const Shape &sh, int kind, long long room)
{
    std::vector<int32_t> kv_start(sh.batch);
    int32_t sum = 0;
    for (int i = 0; i < sh.batch; ++i) {
        kv_start[i] = sum;
        sum += sh.len[i];
    }
    // the scratch that the library says a call uses is enough for the plan that unlimited scratch gives
    {
        const AttnPlan free = attn_plan(sh.batch, sh.T, sh.Hq, sh.Hkv, sh.D, sh.len.data(), SIZE_MAX);
        const size_t said = attn_scratch_bytes(sh.batch, sh.T, sh.Hq, sh.Hkv, sh.D, DDTREE_DTYPE_BF16, sum);
        if (free.bytes > said || (sh.batch == 1 && free.bytes != said)) return 12;
        const AttnPlan again = attn_plan(sh.batch, sh.T, sh.Hq, sh.Hkv, sh.D, sh.len.data(), said);
        if (again.bytes != free.bytes || again.items != free.items || again.cost != free.cost) return 13;
        if (attn_lacks_scratch(sh.batch, sh.T, sh.Hq, sh.Hkv, sh.D, sh.len.data(), said)) return 14;
    }
    const bool wide = wide_partials(sh.batch, sh.T, sh.Hq, sh.Hkv, sh.D, sum);
    const Lens lens = lens_of(sh.len.data(), sh.batch);
    const AttnPlan p = kind == 2 ? plan_main(sh.batch, sh.T, sh.Hq, sh.Hkv, sh.len.data(), lens, wide, room)
                                 : plan_wave(sh.batch, sh.T, sh.Hq, sh.Hkv, sh.D, sh.len.data(), lens, kind + 1, wide, room);
    if (p.slots > room || p.bytes > attn_scratch_upper(sh.batch, sh.T, sh.Hq, sh.Hkv, sh.D)) return 1;
    std::vector<Item> items;
    if (kind == 2) {
        AttnMainArgs args;
        if (!attn_main_args(args, p, kv_start.data(), sh.len.data(), sh.batch, sh.T, sh.Hq, sh.Hkv)) return 2;
        if (p.items <= 256 && args.grid > 256) return 3;  // one round stays one
        for (int b = 0; b < args.grid; ++b) {
            AttnMainItem w;
            if (!attn_main_item(args, b, sh.T, w)) continue;
            if (w.kv_start != kv_start[w.seq] || w.kv_len != sh.len[w.seq] || w.splits > w.ranges) return 3;
            const int keys = w.tail ? kSK : kKT;
            if (w.tail && w.m_end - w.m0 > 32) return 3;
            items.push_back({w.seq, w.hk, w.m0, w.m_end, w.t_begin, w.t_end, w.split, w.ranges, w.first_slot + w.split, keys,
                             w.n_cache + (w.m_end - 1) / (sh.Hq / sh.Hkv) / keys + 1});
        }
    } else {
        AttnWaveArgs args;
        if (!attn_wave_args(args, p, kv_start.data(), sh.len.data(), sh.batch, sh.T, sh.Hq, sh.Hkv)) return 2;
        for (int b = 0; b < args.grid; ++b) {
            AttnWaveItem w;
            if (!attn_wave_item(args, b, w)) continue;
            if (w.kv_start != kv_start[w.seq] || w.kv_len != sh.len[w.seq] || w.splits != w.ranges) return 3;
            items.push_back({w.seq, w.hk, w.r0, w.r1, w.t_begin, w.t_end, w.split, w.ranges, w.first_slot + w.split, kSK,
                             w.n_cache + (w.r1 - 1) / (sh.Hq / sh.Hkv) / kSK + 1});
        }
    }
    return check_items(sh, p, items, p.items);
}

int attn_selftest_host()
{
    static const Shape shapes[] = {
        {1, 257, 32, 8, 128, {8192}},        {1, 513, 32, 8, 128, {32768}},       {1, 65, 32, 8, 128, {2048}},
        {4, 129, 64, 8, 128, {1533, 7527, 4000, 1024}},                           {1, 1025, 8, 2, 128, {1500}},
        {3, 33, 16, 2, 128, {130, 0, 517}},  {1, 17, 4, 1, 128, {128}},           {2, 40, 12, 1, 128, {1000, 3}},
        {1, 2, 1, 1, 128, {0}},              {4, 1024, 8, 8, 128, {100, 0, 64, 7}}, {1, 75, 16, 4, 128, {3000}},
        {1, 300, 6, 2, 128, {9000}},         {2, 273, 32, 8, 128, {5000, 4999}},  {1, 1025, 128, 1, 128, {200000}},
        {1, 65, 16, 4, 64, {2047}},          {3, 257, 32, 8, 64, {4096, 31, 33}}, {1, 2, 1, 1, 64, {0}},
        {4, 101, 24, 8, 128, {37, 3001, 900, 1700}}, {4, 1025, 40, 8, 128, {5000, 300, 9000, 700}},
        // row tiles of the same height in more than one round of workgroups
        {16, 161, 32, 8, 128, std::vector<int32_t>(16, 4096)}, {8, 289, 32, 8, 128, std::vector<int32_t>(8, 1024)},
        {4, 545, 32, 8, 128, std::vector<int32_t>(4, 4096)},   {2, 545, 32, 8, 128, {16384, 16384}},
        {1, 321, 112, 16, 128, {5000}},                        {64, 41, 32, 8, 128, std::vector<int32_t>(64, 4096)},
    };
    // exhaustive check of the reciprocal division itself on small divisors
    for (uint32_t d = 2; d <= 64; ++d) {
        const uint64_t x_max = 0xFFFFFFFFull / d;
        const uint32_t m = magic_of(d, x_max);
        if (m == 0u) return 1;
        for (uint64_t x = 0; x <= x_max; x += (x < 70000 ? 1 : 9973))
            if (div_by((int)(x & 0x7FFFFFFF), (int)d, m) != (int)((x & 0x7FFFFFFF) / d)) return 2;
        if (magic_of(d, x_max + 1) != 0u && (x_max + 1) * d >= 0x100000000ull) return 3;
    }
    int si = 0;
    for (const Shape &sh : shapes) {
        ++si;
        for (int kind = 0; kind < 3; ++kind)
            for (long long room : {1ll << 40, 0ll}) {  // with scratch and without
                if ((kind == 1 && sh.D != 64) || (kind == 2 && sh.D != kHD)) continue;
                if (const int rc = check_plan(sh, kind, room)) return 100 * si + rc;
            }
    }
    uint64_t seed = 1;
    auto below = [&seed](uint64_t n) {  // splitmix64
        uint64_t z = (seed += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return (int)((z ^ (z >> 31)) % n);
    };
    for (si = kSweepBase; si < kSweepBase + kSweepShapes; ++si) {
        Shape sh;
        sh.batch = below(3) == 0 ? 1 : 1 + below(below(2) ? 8 : DDTREE_MAX_BATCH);
        sh.T = 1 + below(below(2) ? 300 : DDTREE_MAX_N + 1);
        sh.Hkv = 1 + below(16);
        sh.Hq = sh.Hkv * (1 + below(below(2) ? 4 : 16));
        sh.D = below(4) == 0 ? 64 : kHD;
        const int longest = 1 << below(17), ragged = below(2);
        for (int i = 0; i < sh.batch; ++i) sh.len.push_back(ragged ? below(longest + 1) : longest);
        const long long room = below(3) == 0 ? below(4 * sh.batch) : 1ll << 40;
        for (int kind = 0; kind < 3; ++kind) {
            if ((kind == 1 && sh.D != 64) || (kind == 2 && sh.D != kHD)) continue;
            if (const int rc = check_plan(sh, kind, room)) return 100 * si + rc;
        }
    }
    return 0;
}

}  // namespace ddt
