// Per-position log-softmax and exact top-K over the vocabulary (paper Section 4.3: the
// ordering q_i^(1) >= q_i^(2) >= ... of each position's distribution; Lemma 1: K ranks suffice).
//
// Two kernels.
//   chunk kernel   one workgroup per (row, vocabulary chunk): reads the chunk once, into registers, and
//                  leaves its maximum, its sum of exponentials (fp64), the maxima of its groups of
//                  adjacent threads, and its "hot" elements, about twice as many as it is likely to
//                  contribute to the row's top K.  It orders nothing.
//   finish kernel  one workgroup per row: the K-th largest of the row's group maxima is a lower bound on
//                  the row's K-th largest element (the maxima are K distinct elements) and a tight
//                  one, about 1.1 K elements reach it.  Those are all hot unless a chunk's hot bound
//                  turns out to lie above it: that chunk is read again.  They are ranked exactly (key
//                  descending, token id ascending) and written with their log-probabilities.
// A row of one chunk is finished by its chunk workgroup; rows whose candidates do not fit on chip (heavy
// ties, fewer maxima than ranks) take a radix select over the row.
//
// Every candidate is the 64-bit composite (key << 32) | ~token_id, so all composites of a row
// are distinct and "larger composite" is exactly "larger logit, or equal logit and smaller id".
//
// What bounds it: latencies (two launches, two first touches of memory), and in the chunk kernel the fp64
// exponentials; at 256 rows the chunk kernel reads 3.4 TB/s, four workgroups of 512 threads on a compute
// unit each waiting for memory or computing.  Before, every chunk ranked its exact top K (three barriers
// and per-slot code worth 3.2 us) for a merge that looked at a sixteenth of them, in workgroups of 1024
// threads that fill a compute unit alone, and 128 rows or more took one workgroup per row.
// Measured (both kernels back to back, V = 151936, before -> now): 16 rows K = 256 16.4 -> 14.0 us, K = 1024
// 20.0 -> 16.2; 32 rows K = 128 23.8 -> 17.6; 112 rows 53.9 -> 29.6; 256 rows 66 -> 54; 8 rows of 1024 12.0 -> 7.3.
// Rows whose maxima say little about their top K (masked tokens, an outlier, ties), by the ranking chunks, with one
// range of buckets and a select over the row in six passes, and now: 16 rows K = 256 half masked with -1e9 203 / 181 / 17
// us, equal logits 111 / 721 / 128; K = 1024 one token 1000 above the others 73 / 117 / 16, half masked with -inf 135 / 206 / 130;
// 256 rows K = 128 half masked with -1e9 56 / 296 / 58.  Their code costs the other rows 0.1 to 0.4 us a call.
#include <algorithm>
#include <cmath>

#include "common.hpp"

namespace ddt {

constexpr int kChunkThreads = 512;
constexpr int kChunkWaves = kChunkThreads / 64;
constexpr int kVecPerThread = kTopkChunkMax / 4 / kChunkThreads;
constexpr int kSlots = 4 * kVecPerThread + 2;  // float4 body + one head and one tail element
static_assert(kVecPerThread * 4 * kChunkThreads == kTopkChunkMax, "chunk must tile the workgroup");
constexpr int kRankCap = 4096;   // candidates of a row held on chip
constexpr int kBuckets = 1024;
constexpr int kCrowded = 384;    // members of a bucket beyond which ranking by pairs is slower than a sort

struct ChunkStat {
    double sum;        // sum of exp(x - max) over everything but one instance of the maximum
    float max, low;    // largest element, smallest (finite) group maximum
    float hot;         // hot bound: the elements that reach it are in the hot list (+inf: there is no list, or they did not fit)
    int32_t pad;
};

TopkPlan topk_plan(int batch, int B, int V, int K)
{
    TopkPlan p{};
    if (batch < 1 || B < 1 || V < 1 || K < 1 || K > V) return p;
    const long long rows = (long long)batch * B;
    // two workgroups per compute unit, chunks of at least 1024 elements, at most one chunk per lane of a wave
    const int c_min = (V + kTopkChunkMax - 1) / kTopkChunkMax;
    const int want = (int)std::min<long long>({(512 + rows - 1) / rows, std::max(1, V / 1024), 64});
    // A row that one workgroup holds is finished by it: one launch (8 rows of 3000, K = 200: 8.4 us, with two
    // chunks 11.8) -- unless its 512 maxima are too few to bound K (16 rows of 4000, K = 1024: 16.0 us, with
    // three chunks 12.4).
    const bool one = c_min == 1 && 3LL * K / 2 <= kChunkThreads;
    const int want_c = one ? 1 : std::max(c_min, want);
    int len = (V + want_c - 1) / want_c;
    len = (len + 3) / 4 * 4;
    p.chunk_len = len;
    p.chunks = (V + len - 1) / len;
    // threads per group: as many as leave half as many maxima again as ranks are wanted
    p.group = 8;
    while (p.group > 1 && (long long)p.chunks * std::min(kChunkThreads, len / 4) / p.group < 3LL * K / 2) p.group >>= 1;
    p.maxima = kChunkThreads / p.group;
    // Hot bound: the hot_rank-th largest of the chunk's 64 (fewer in a short chunk) maxima of 8 threads.
    // With c elements wanted, evenly spread over g groups, a share 1 - exp(-c / g) of the groups has one.
    const double share = (double)K / p.chunks, c = 2.2 * share + 12.0;
    const int g = std::max(1, std::min(64, len / 32));
    p.hot_rank = (int)(g * (1.0 - std::exp(-c / g)));
    if (p.hot_rank < 1) p.hot_rank = 1;
    // (A tenth of a chunk is what the maxima of 32 elements can tell apart: beyond it the lists would lack some.)
    p.hot_cap = c > 0.1 * len ? 0 : c <= 40.0 ? 64 : c <= 90.0 ? 128 : c <= 200.0 ? 256 : c <= 420.0 ? 512 : 0;  // (0: most elements would be hot)
    p.max_off = 0;
    p.stat_off = align_up((size_t)rows * p.chunks * p.maxima * sizeof(float), 256);
    p.hot_off = align_up(p.stat_off + (size_t)rows * p.chunks * sizeof(ChunkStat), 256);
    p.bytes = align_up(p.hot_off + (size_t)rows * p.chunks * p.hot_cap * sizeof(uint64_t), 256);
    p.ok = true;
    return p;
}

// A bound on topk_plan(...).bytes over every call of at most this many rows, elements and ranks: a workspace made
// for the largest call serves the smaller ones, whose chunks may be more and whose hot lists may be longer (there
// are none where K is large).  A chunk leaves 64 maxima, statistics and 64 hot places; beyond these, groups of
// fewer than eight threads leave less than 6 K maxima a row (512 in a row of one chunk), and a hot list of c
// elements wanted has at most 64 + 3.2 (c - 12) places, c - 12 being 2.2 K / chunks; neither exceeds 512 a chunk.
size_t topk_scratch_upper(int batch, int B, int V, int K)
{
    const long long rows = (long long)batch * B, c_min = (V + kTopkChunkMax - 1) / kTopkChunkMax;
    const long long chunks = std::max(rows * c_min, std::min({rows + 511, 64 * rows, rows * std::max(1, V / 1024)}));
    const long long maxima = std::min(64 * chunks + rows * (6 * K + kChunkThreads), (long long)kChunkThreads * chunks);
    const long long places = std::min(64 * chunks + rows * (7 * K + K / 16), 512 * chunks);
    return 3 * 256 + (size_t)maxima * sizeof(float) + (size_t)chunks * sizeof(ChunkStat) + (size_t)places * sizeof(uint64_t);
}

// exp(y) for y <= 0 in fp64 to a relative error below 4e-11: y = (64 n + j) ln2/64 + r with
// |r| <= ln2/128, so exp(y) = 2^n * 2^(j/64) * exp(r); 2^(j/64) comes from a 64-entry table and
// exp(r) from its Taylor polynomial of degree 3 (remainder r^4/24 < 3.6e-11; the reduction by one
// fp64 multiple of ln2/64 is off by less than 6e-14).  The row's log-sum-exp needs its sum to some
// 1e-8 for a log-probability that is right to the last fp32 bit; every fp64 instruction here is
// paid 9.7 million times a step.  64 n + j is read off the low bits of y * 64/ln2 + 1.5 * 2^52.
// 0 far below the fp64 range.
__device__ const double kExp2Table[64] = {
    0x1.0000000000000p+0, 0x1.02c9a3e778061p+0, 0x1.059b0d3158574p+0, 0x1.0874518759bc8p+0,
    0x1.0b5586cf9890fp+0, 0x1.0e3ec32d3d1a2p+0, 0x1.11301d0125b51p+0, 0x1.1429aaea92de0p+0,
    0x1.172b83c7d517bp+0, 0x1.1a35beb6fcb75p+0, 0x1.1d4873168b9aap+0, 0x1.2063b88628cd6p+0,
    0x1.2387a6e756238p+0, 0x1.26b4565e27cddp+0, 0x1.29e9df51fdee1p+0, 0x1.2d285a6e4030bp+0,
    0x1.306fe0a31b715p+0, 0x1.33c08b26416ffp+0, 0x1.371a7373aa9cbp+0, 0x1.3a7db34e59ff7p+0,
    0x1.3dea64c123422p+0, 0x1.4160a21f72e2ap+0, 0x1.44e086061892dp+0, 0x1.486a2b5c13cd0p+0,
    0x1.4bfdad5362a27p+0, 0x1.4f9b2769d2ca7p+0, 0x1.5342b569d4f82p+0, 0x1.56f4736b527dap+0,
    0x1.5ab07dd485429p+0, 0x1.5e76f15ad2148p+0, 0x1.6247eb03a5585p+0, 0x1.6623882552225p+0,
    0x1.6a09e667f3bcdp+0, 0x1.6dfb23c651a2fp+0, 0x1.71f75e8ec5f74p+0, 0x1.75feb564267c9p+0,
    0x1.7a11473eb0187p+0, 0x1.7e2f336cf4e62p+0, 0x1.82589994cce13p+0, 0x1.868d99b4492edp+0,
    0x1.8ace5422aa0dbp+0, 0x1.8f1ae99157736p+0, 0x1.93737b0cdc5e5p+0, 0x1.97d829fde4e50p+0,
    0x1.9c49182a3f090p+0, 0x1.a0c667b5de565p+0, 0x1.a5503b23e255dp+0, 0x1.a9e6b5579fdbfp+0,
    0x1.ae89f995ad3adp+0, 0x1.b33a2b84f15fbp+0, 0x1.b7f76f2fb5e47p+0, 0x1.bcc1e904bc1d2p+0,
    0x1.c199bdd85529cp+0, 0x1.c67f12e57d14bp+0, 0x1.cb720dcef9069p+0, 0x1.d072d4a07897cp+0,
    0x1.d5818dcfba487p+0, 0x1.da9e603db3285p+0, 0x1.dfc97337b9b5fp+0, 0x1.e502ee78b3ff6p+0,
    0x1.ea4afa2a490dap+0, 0x1.efa1bee615a27p+0, 0x1.f50765b6e4540p+0, 0x1.fa7c1819e90d8p+0};
__device__ __forceinline__ double exp_nonpositive(double y, const double *s_tab)
{
    y = fmax(y, -800.0);
    const double t = fma(y, 92.33248261689366, 0x1.8p52);      // 64 / ln 2
    const double r = fma(t - 0x1.8p52, -0x1.62e42fefa39efp-7, y);  // ln2/64
    const int ki = __double2loint(t);
    double p = fma(r, 1.0 / 6.0, 0.5);
    p = fma(r, p, 1.0);
    p = fma(r, p, 1.0);
    return ldexp(s_tab[ki & 63] * p, ki >> 6);
}

// ------------------------------------------------------------------------------------------
// A row's top K from what its chunks left.  NT threads.
// ------------------------------------------------------------------------------------------
struct FinishLds {
    uint64_t list[kRankCap];    // the candidates
    uint64_t sorted[kRankCap];  // bucket by bucket
    uint32_t cnt[kBuckets];
    int start[kBuckets + 1];
    int wave[17];
    int found[3];               // the bucket that holds the rank looked for, what the buckets above it hold, what it holds
    uint32_t low, high;         // range of the maxima in a crowded bucket
    double exc;                 // log1p(sum over everything but the first maximum), i.e. lse - max
    int n_list, crowded;
};
struct FinishArgs {
    int V, K, chunks, chunk_len, maxima, hot_cap;
};

template <int NT>
__device__ void finish_row(const float *p, const FinishArgs a, const float *maxima, const ChunkStat *stat, const uint64_t *hot,
                           FinishLds &L, int32_t *tok, float *lp)
{
    constexpr int NW = NT / 64, PRE = 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n_max = a.chunks * a.maxima, n_hot = a.chunks * a.hot_cap, K = a.K;
    const int cap_shift = a.hot_cap ? 31 - __builtin_clz(a.hot_cap) : 0;
    // Everything the common case reads, requested together.  Every wave holds the statistics of all chunks,
    // one per lane (of the first 64; beyond, they are read as needed), so that what follows from them
    // needs no barrier.
    ChunkStat st;
    st.max = st.low = -INFINITY;
    st.hot = -INFINITY;
    st.sum = 0.0;
    if (lane < a.chunks) st = stat[lane];
    float g[PRE];
    uint64_t h[PRE];
#pragma unroll
    for (int u = 0; u < PRE; ++u) g[u] = tid + u * NT < n_max ? maxima[tid + u * NT] : -INFINITY;
#pragma unroll
    for (int u = 0; u < PRE; ++u) h[u] = tid + u * NT < n_hot ? hot[tid + u * NT] : 0ull;
    for (int i = tid; i < kBuckets; i += NT) L.cnt[i] = 0u;
    if (tid == 0) {
        L.n_list = L.crowded = 0;
        L.found[0] = kBuckets;
        L.low = ~0u;
        L.high = 0u;
    }
    __syncthreads();
    // ---- the K-th largest group maximum, to the resolution of kBuckets equal buckets over the range of
    //      the maxima, bucket 0 the highest.  (Float subtraction, scaling and truncation are monotone: an
    //      element above another never lands in a later bucket.) ----
    float vmax = st.max;
    uint32_t vlow = st.low > -INFINITY ? float_key(st.low) : ~0u;
    for (int c = lane + 64; c < a.chunks; c += 64) {
        vmax = fmaxf(vmax, stat[c].max);
        if (stat[c].low > -INFINITY) vlow = min(vlow, float_key(stat[c].low));
    }
    const float hi = wave_max_f32(vmax);
    vlow = wave_min_u32(vlow);
    // The range of the buckets ends at the second largest chunk maximum: one token far above the others (a confident
    // row) does not stretch it.  What lies above is in bucket 0.
    const uint64_t tops = __builtin_amdgcn_ballot_w64(vmax == hi);
    float top = wave_max_f32(lane == __builtin_ctzll(tops) ? -INFINITY : vmax), low = vlow == ~0u ? hi : key_float(vlow);
    if (!(top > low)) top = hi;
    float ceiling = INFINITY;  // (of the maxima still counted: at first, bucket 0 holds those above the range too)
    float inv = (float)kBuckets / fmaxf(top - low, 1e-30f);
    auto bucket_of = [&](float v) { return (int)fminf(fmaxf((top - v) * inv, 0.0f), (float)(kBuckets - 1)); };
    auto each_maximum = [&](auto &&f) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < PRE; ++u)
            if (g[u] > -INFINITY) f(g[u]);
        for (int i = tid + PRE * NT; i < n_max; i += NT) {
            const float v = maxima[i];
            if (v > -INFINITY) f(v);
        }
    };
    each_maximum([&](float v) { atomicAdd(&L.cnt[bucket_of(v)], 1u); });
    __syncthreads();
    const double mx = (double)hi;
    // log-sum-exp from the chunk statistics (fp64, fixed order), by one whole wave.  The chunk sums leave one
    // instance of their own maximum out; the first chunk that holds the row's maximum stays that way,
    // every other gets its instance back.
    auto log_sum_exp = [&]() {
        bool owned = false;
        double part = 0.0;
        for (int c0 = 0; c0 < a.chunks; c0 += 64) {
            const ChunkStat t = c0 == 0 ? st : (c0 + lane < a.chunks ? stat[c0 + lane] : ChunkStat{0.0, -INFINITY, -INFINITY, 0.0f, 0});
            const uint64_t top = __builtin_amdgcn_ballot_w64(c0 + lane < a.chunks && t.max == hi);
            const bool owner = !owned && top != 0ull && lane == __builtin_ctzll(top);
            owned = owned || top != 0ull;
            if (c0 + lane < a.chunks) part += (t.sum + (owner ? 0.0 : 1.0)) * exp((double)t.max - mx);
        }
        part = wave_sum_f64_lane63(part);
        if (lane == 63) L.exc = log1p(part);
    };
    // cumulative populations, highest bucket first; the counters are left empty
    constexpr int PB = kBuckets / NT;
    auto scan = [&](int want, bool starts) {  // (all threads)
        int mine = 0, c[PB];
#pragma unroll
        for (int j = 0; j < PB; ++j) {
            c[j] = (int)L.cnt[tid * PB + j];
            mine += c[j];
        }
        const int incl = wave_scan_inclusive_i32(mine);
        if (lane == 63) L.wave[wave] = incl;
        __syncthreads();
        int before = incl - mine;
#pragma unroll
        for (int w = 0; w < NW; ++w) before += w < wave ? L.wave[w] : 0;
#pragma unroll
        for (int j = 0; j < PB; ++j) {
            if (starts) L.start[tid * PB + j] = before;
            else L.cnt[tid * PB + j] = 0u;
            if (before < want && before + c[j] >= want) L.found[0] = tid * PB + j, L.found[1] = before, L.found[2] = c[j];
            before += c[j];
        }
        __syncthreads();
    };
    scan(K, false);
    // (Fewer maxima than ranks: no bound.  All elements of a short row are candidates then.)
    const bool all = L.found[0] == kBuckets && a.V <= kRankCap;
    const bool bounded = L.found[0] != kBuckets || all;
    int want = K;
    // A bucket that holds many maxima at once (an outlier or masked tokens stretch the range, most of it empty):
    // the same again over the maxima of that bucket alone.
    for (int round = 0; bounded && !all && __builtin_expect(L.found[2] > 64 + 3 * K / 8, 0) && round < 8; ++round) {  // (uniform)
        const int crowded = L.found[0];
        want -= L.found[1];
        uint32_t kl = ~0u, kh = 0u;
        each_maximum([&](float v) {
            if (v <= ceiling && v >= low && bucket_of(v) == crowded) kl = min(kl, float_key(v)), kh = max(kh, float_key(v));
        });
        kl = wave_min_u32(kl);
        kh = ~wave_min_u32(~kh);
        if (lane == 63 && kl <= kh) {
            atomicMin(&L.low, kl);
            atomicMax(&L.high, kh);
        }
        __syncthreads();
        kl = L.low;
        kh = L.high;
        top = ceiling = key_float(kh);
        low = key_float(kl);
        inv = kl == kh ? 1e38f : (float)kBuckets / fmaxf(top - low, 1e-30f);  // (one value: what lies below it is far away)
        if (kl != kh) each_maximum([&](float v) { if (v <= top && v >= low) atomicAdd(&L.cnt[bucket_of(v)], 1u); });
        __syncthreads();
        if (tid == 0) {
            L.low = ~0u;
            L.high = 0u;
            if (kl == kh) L.found[0] = L.found[1] = L.found[2] = 0;
        }
        if (kl != kh) scan(want, false);
        else __syncthreads();
    }
    const int last = all ? kBuckets - 1 : bounded ? L.found[0] : -1;  // elements of buckets 0 .. last are candidates, at least K of them
    const bool whole = a.hot_cap == 0;           // the row is read again, all of it
    auto composite = [&](float x, int i) -> uint64_t {
        return ((uint64_t)float_key(x) << 32) | (uint64_t)(uint32_t)(~(uint32_t)i);
    };
    auto emit = [&](int rank, uint64_t cc) {
        tok[rank] = (int32_t)(~(uint32_t)cc);
        lp[rank] = (float)(((double)key_float((uint32_t)(cc >> 32)) - mx) - L.exc);
    };
    // a chunk whose hot list may lack candidates: it has some, and its bound falls among their buckets
    auto lacks = [&](float max, float bound) { return (bound == INFINITY || bucket_of(bound) <= last) && bucket_of(max) <= last; };
    uint64_t lacking = __builtin_amdgcn_ballot_w64(lane < a.chunks && (st.hot == INFINITY || bucket_of(st.hot) <= last));  // of the first 64
    if (lacking != 0ull) lacking &= __builtin_amdgcn_ballot_w64(bucket_of(st.max) <= last);
    auto reserve = [&](int n) -> int {  // n list places for this thread (one atomic per wave)
        const int incl = wave_scan_inclusive_i32(n);
        const int total = __builtin_amdgcn_readlane(incl, 63);
        if (total == 0) return 0;
        int base = 0;
        if (lane == 63) base = atomicAdd(&L.n_list, total);
        return __builtin_amdgcn_readlane(base, 63) + incl - n;
    };
    if (!whole && bounded)
        for (int b0 = 0; b0 < n_hot; b0 += PRE * NT) {  // (uniform)
            if (b0 > 0) {
#pragma unroll
                for (int u = 0; u < PRE; ++u) h[u] = b0 + tid + u * NT < n_hot ? hot[b0 + tid + u * NT] : 0ull;
            }
            bool take[PRE];
            int n = 0;
#pragma unroll
            for (int u = 0; u < PRE; ++u) {
                const int i = b0 + tid + u * NT, c = i >> cap_shift;
                take[u] = h[u] != 0ull && bucket_of(key_float((uint32_t)(h[u] >> 32))) <= last &&
                          !(c < 64 ? (bool)((lacking >> c) & 1ull) : lacks(stat[c].max, stat[c].hot));
                n += take[u] ? 1 : 0;
            }
            int at = reserve(n);
#pragma unroll
            for (int u = 0; u < PRE; ++u)
                if (take[u]) {
                    if (at < kRankCap) L.list[at] = h[u];
                    ++at;
                }
        }
    auto put = [&](float x, int id, bool take, int &at) {
        if (take) {
            if (at < kRankCap) L.list[at] = composite(x, id);
            ++at;
        }
    };
    auto rescan = [&](int begin, int end) {  // (uniform over the workgroup)
        for (int i0 = begin; i0 < end; i0 += PRE * NT) {
            float x[PRE];
            bool take[PRE];
            int n = 0;
#pragma unroll
            for (int u = 0; u < PRE; ++u) x[u] = i0 + u * NT + tid < end ? p[i0 + u * NT + tid] : 0.0f;
#pragma unroll
            for (int u = 0; u < PRE; ++u) {
                take[u] = i0 + u * NT + tid < end && bucket_of(x[u]) <= last;
                n += take[u] ? 1 : 0;
            }
            int at = reserve(n);
#pragma unroll
            for (int u = 0; u < PRE; ++u) put(x[u], i0 + u * NT + tid, take[u], at);
        }
    };
    if (whole && bounded) rescan(0, a.V);
    for (int c0 = 0; c0 < a.chunks && !whole && bounded; c0 += 64) {
        uint64_t todo = lacking;
        if (c0 > 0) {
            const ChunkStat t = stat[min(c0 + lane, a.chunks - 1)];
            todo = __builtin_amdgcn_ballot_w64(c0 + lane < a.chunks && lacks(t.max, t.hot));
        }
        for (; todo != 0ull; todo &= todo - 1ull) {
            const int begin = (c0 + __builtin_ctzll(todo)) * a.chunk_len;
            rescan(begin, min(begin + a.chunk_len, a.V));
        }
    }
    __syncthreads();
    int m = L.n_list;
    if (wave == NW - 1) log_sum_exp();  // (this wave has the fewest candidates)
    if (__builtin_expect(bounded && m <= kRankCap, 1)) {
        if (m <= NT / 8) {
            // all pairs: the threads of a wave share the element they compare with (a broadcast read), and
            // each element's comparisons are dealt to NT / E threads
            int E = 64;
            while (E < m) E <<= 1;
            const int parts = NT / E, e = tid & (E - 1), part_no = tid / E;
            const uint64_t mine = e < m ? L.list[e] : 0ull;
            const int j1 = min(m, (part_no + 1) * ((m + parts - 1) / parts));
            int above = 0;
            for (int j = part_no * ((m + parts - 1) / parts); j < j1; ++j) above += L.list[j] > mine ? 1 : 0;
            if (e < m && above) atomicAdd(&L.cnt[e], (uint32_t)above);
            __syncthreads();
            if (tid < m && (int)L.cnt[tid] < K) emit((int)L.cnt[tid], mine);
            return;
        }
        // by buckets over the candidates' own range: a candidate's rank is the population of the buckets above
        // its own plus the larger members of its bucket
        const float least = top - (float)(last + 1) / inv;  // (about the smallest candidate)
        const float inv2 = (float)kBuckets / fmaxf(top - least, 1e-30f);
        auto bucket2 = [&](uint64_t cc) { return (int)fminf(fmaxf((top - key_float((uint32_t)(cc >> 32))) * inv2, 0.0f), (float)(kBuckets - 1)); };
        constexpr int PER = kRankCap / NT;
        uint64_t mine[PER];
        int bkt[PER], pos[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int i = tid + u * NT;
            bkt[u] = pos[u] = 0;
            mine[u] = 0ull;
            if (i < m) {
                mine[u] = L.list[i];
                bkt[u] = bucket2(mine[u]);
                pos[u] = (int)atomicAdd(&L.cnt[bkt[u]], 1u);
                if (pos[u] == kCrowded && !(all && bkt[u] == kBuckets - 1)) L.crowded = 1;
            }
        }
        __syncthreads();
        if (__builtin_expect(!L.crowded, 1)) {
            scan(0, true);
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (tid + u * NT < m) L.sorted[L.start[bkt[u]] + pos[u]] = mine[u];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                if (tid + u * NT >= m) break;
                const int bs = L.start[bkt[u]], nb = (int)L.cnt[bkt[u]];
                if (bs >= K) continue;
                int above = bs;
#pragma unroll 4
                for (int j = 0; j < nb; ++j) above += L.sorted[bs + j] > mine[u] ? 1 : 0;
                if (above < K) emit(above, mine[u]);
            }
            return;
        }
    } else {
        // Too few maxima, or too many elements that reach the bound (ties among them): the K-th largest element of
        // the row itself, ten bits of its distance d from the maximum (as order-preserving integers) at a time, until
        // what lies at or above its bucket fits on chip.  Where one value has too many elements for that, those
        // above it are ranked and the first of its own follow in the order of their ids.
        const uint32_t key_hi = float_key(hi), range = key_hi - (bounded ? float_key(low) : 0x007FFFFFu);  // (-inf)
        auto distance = [&](float v) { return key_hi - float_key(v); };
        int shift = max(0, 22 - __builtin_clz(range | 1u)), chosen;
        uint32_t base = 0u, buckets = (range >> shift) + 1u;
        want = K;
        for (;;) {
            for (int i0 = 0; i0 < a.V; i0 += 8 * NT) {
                float x[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) x[u] = i0 + u * NT + tid < a.V ? p[i0 + u * NT + tid] : 0.0f;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    // the first lane's bucket takes all its lanes at once (a masked row has most of them in one)
                    const uint32_t d = distance(x[u]), bk = (d - base) >> shift;
                    const bool on = i0 + u * NT + tid < a.V && d >= base && bk < buckets;
                    const uint64_t any = __builtin_amdgcn_ballot_w64(on);
                    if (any == 0ull) continue;
                    const int first = __builtin_ctzll(any);
                    const uint32_t b0 = (uint32_t)__builtin_amdgcn_readlane((int)bk, first);
                    const uint64_t same = __builtin_amdgcn_ballot_w64(on && bk == b0);
                    if (lane == first) atomicAdd(&L.cnt[b0], (uint32_t)__builtin_popcountll(same));
                    else if (on && bk != b0) atomicAdd(&L.cnt[bk], 1u);
                }
            }
            __syncthreads();
            scan(want, false);
            const uint32_t bk = (uint32_t)L.found[0];
            want -= L.found[1];
            chosen = K - want + L.found[2];
            base += bk << shift;
            if (chosen <= kRankCap || shift == 0) break;
            const int finer = max(0, shift - 10);
            buckets = 1u << (shift - finer);
            shift = finer;
        }
        const bool tied = chosen > kRankCap;
        const uint32_t limit = base + ((1u << shift) - 1u);  // the largest distance chosen
        if (tid == 0) L.n_list = 0;
        __syncthreads();
        for (int i0 = 0; i0 < a.V; i0 += 8 * NT) {
            float x[8];
            uint32_t take = 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = i0 + u * NT + tid < a.V ? p[i0 + u * NT + tid] : 0.0f;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t d = distance(x[u]);
                take |= i0 + u * NT + tid < a.V && (tied ? d < base : d <= limit) ? 1u << u : 0u;
            }
            int at = reserve(__builtin_popcount(take));
#pragma unroll
            for (int u = 0; u < 8; ++u) put(x[u], i0 + u * NT + tid, (take >> u) & 1u, at);
        }
        for (int i0 = 0, have = 0; tied && i0 < a.V && have < want; i0 += 8 * NT) {  // (uniform)
            const int i = i0 + tid * 8;
            uint32_t bits = 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i + u < a.V && distance(p[i + u]) == base) bits |= 1u << u;
            const int n = __builtin_popcount(bits), incl = wave_scan_inclusive_i32(n);
            if (lane == 63) L.wave[wave] = incl;
            __syncthreads();
            int at = have + incl - n, total = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                at += w < wave ? L.wave[w] : 0;
                total += L.wave[w];
            }
            for (; bits != 0u && at < want; bits &= bits - 1u, ++at) {
                const int id = i + __builtin_ctz(bits);
                emit(K - want + at, composite(p[id], id));
            }
            have += total;
            __syncthreads();
        }
        __syncthreads();
        m = L.n_list;
        if (m == 0) return;
    }
    // a bucket of many (equal values, clusters far apart): a bitonic sort of all candidates, descending.  A wave has
    // 128 consecutive places of its own, so only steps of 128 places and more wait for the others.
    int n = 128;
    while (n < m) n <<= 1;
    for (int i = m + tid; i < n; i += NT) L.list[i] = 0ull;
    __syncthreads();
    for (int k = 2; k <= n; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int e = tid; e < n / 2; e += NT) {
                const int at = ((e & ~(j - 1)) << 1) | (e & (j - 1));
                const uint64_t x = L.list[at], y = L.list[at + j];
                const bool descending = (at & k) == 0;
                if ((x < y) == descending) L.list[at] = y, L.list[at + j] = x;
            }
            const int next = j > 1 ? j >> 1 : k;  // the next step's distance
            if (j >= 128 || next >= 128) __syncthreads();
            else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    __syncthreads();
    for (int i = tid; i < min(m, K); i += NT) emit(i, L.list[i]);
}

// ------------------------------------------------------------------------------------------
// Chunk kernel
// ------------------------------------------------------------------------------------------
template <bool FINISH>
__global__ __launch_bounds__(kChunkThreads, 4) void topk_chunk_kernel(
    const float *__restrict__ logits, int V, int chunk_len, int chunks, int group, int hot_rank, int hot_cap, float *maxima,
    ChunkStat *stat, uint64_t *hot, int K, int maxima_per_chunk, int32_t *__restrict__ topk_tok, float *__restrict__ topk_lp)
{
    const FinishArgs a{V, K, chunks, chunk_len, maxima_per_chunk, hot_cap};
    __shared__ float s_fmax[kChunkWaves], s_group[64];
    __shared__ uint32_t s_low[kChunkWaves];
    __shared__ double s_dsum[kChunkWaves];
    __shared__ int s_neq[kChunkWaves], s_count;
    __shared__ double s_exp2[64];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int c = blockIdx.x;
    const size_t row = (size_t)blockIdx.z * gridDim.y + blockIdx.y;
    const int start = c * a.chunk_len;
    const int n = min(a.chunk_len, a.V - start);
    const float *p = logits + row * (size_t)a.V + start;

    // ---- load: scalar head up to 16-byte alignment, float4 body, scalar tail; all of a
    //      thread's loads are in flight together.  Empty slots hold -inf: no effect on a maximum, an
    //      exp term of 0 ----
    int head = (int)((4 - ((reinterpret_cast<uintptr_t>(p) >> 2) & 3)) & 3);
    if (head > n) head = n;
    const int nvec = (n - head) >> 2;
    const int tail0 = head + 4 * nvec;
    const float4 *pv = reinterpret_cast<const float4 *>(p + head);
    float x[kSlots];
#pragma unroll
    for (int u = 0; u < kVecPerThread; ++u) {
        const int j = tid + u * kChunkThreads;
        const float4 v = j < nvec ? pv[j] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        x[4 * u + 0] = v.x;
        x[4 * u + 1] = v.y;
        x[4 * u + 2] = v.z;
        x[4 * u + 3] = v.w;
    }
    x[kSlots - 2] = tid < head ? p[tid] : -INFINITY;
    x[kSlots - 1] = tid < n - tail0 ? p[tail0 + tid] : -INFINITY;
    if (tid < 64) s_exp2[tid] = kExp2Table[tid];
    if (tid == 0) s_count = 0;
    // element index of slot s within the chunk, -1 if the slot is empty
    auto slot_index = [&](int s) -> int {
        if (s < 4 * kVecPerThread) {
            const int j = tid + (s >> 2) * kChunkThreads;
            return j < nvec ? head + 4 * j + (s & 3) : -1;
        }
        if (s == kSlots - 2) return tid < head ? tid : -1;
        return tid < n - tail0 ? tail0 + tid : -1;
    };
    // loads that hold an element in at least one lane of this wave (uniform)
    const int wave_base = __builtin_amdgcn_readfirstlane(tid & ~63);
    int loads = 0;
#pragma unroll
    for (int u = 0; u < kVecPerThread; ++u) loads += wave_base + u * kChunkThreads < nvec ? 1 : 0;
    const bool edges = wave_base == 0 && (head > 0 || n > tail0);

    // ---- maxima of the threads, of groups of `group` of them, and of groups of eight ----
    float tmax = fmaxf(x[kSlots - 2], x[kSlots - 1]);
#pragma unroll
    for (int s = 0; s < 4 * kVecPerThread; ++s) tmax = fmaxf(tmax, x[s]);
    float g = tmax;
    const float g1 = g;
    g = fmaxf(g, dpp_f<0xB1>(g, g));
    const float g2 = g;
    g = fmaxf(g, dpp_f<0x4E>(g, g));
    const float g4 = g;
    g = fmaxf(g, dpp_f<0x141>(g, g));
    const float mine = group == 8 ? g : group == 4 ? g4 : group == 2 ? g2 : g1;
    if ((lane & (group - 1)) == 0) maxima[((row * a.chunks + c) * kChunkThreads + tid) / group] = mine;
    if ((lane & 7) == 0) s_group[tid >> 3] = g;
    const float wmax = wave_max_f32(g);
    const uint32_t low = wave_min_u32(mine > -INFINITY ? float_key(mine) : ~0u);
    if (lane == 63) {
        s_fmax[wave] = wmax;
        s_low[wave] = low;
    }
    __syncthreads();
    float cmax = s_fmax[0];
#pragma unroll
    for (int w = 1; w < kChunkWaves; ++w) cmax = fmaxf(cmax, s_fmax[w]);

    // ---- the hot bound: a value that hot_rank of the 64 maxima of eight threads reach and few more, found
    //      by bisection (each wave for itself: no barrier); then the hot elements, in no order ----
    uint64_t *const out = hot + (row * a.chunks + c) * (size_t)a.hot_cap;
    float bound = -INFINITY;
    if (a.hot_cap > 0) {
        const float v = s_group[lane];
        float up = cmax;
        bound = -wave_max_f32(v > -INFINITY ? -v : -INFINITY);
        if (__builtin_popcountll(__builtin_amdgcn_ballot_w64(v > -INFINITY)) < hot_rank) bound = -INFINITY;
        for (int i = 0; i < 9; ++i) {
            const float mid = 0.5f * (bound + up);
            const bool enough = __builtin_popcountll(__builtin_amdgcn_ballot_w64(v >= mid)) >= hot_rank;
            bound = enough ? mid : bound;
            up = enough ? up : mid;
        }
    }
    if (bound > -INFINITY) {
        int cnt = 0;
#pragma unroll
        for (int s = 0; s < kSlots; ++s) cnt += x[s] >= bound ? 1 : 0;
        const int incl = wave_scan_inclusive_i32(cnt), total = __builtin_amdgcn_readlane(incl, 63);
        if (total > 0) {
            int base = 0;
            if (lane == 63) base = atomicAdd(&s_count, total);
            int at = __builtin_amdgcn_readlane(base, 63) + incl - cnt;
            if (cnt > 0) {
#pragma unroll
                for (int s = 0; s < kSlots; ++s)
                    if (x[s] >= bound) {
                        if (at < a.hot_cap)
                            out[at] = ((uint64_t)float_key(x[s]) << 32) | (uint64_t)(uint32_t)(~(uint32_t)(start + slot_index(s)));
                        ++at;
                    }
            }
        }
    }

    // ---- sum of exp(x - cmax) in fp64, fixed reduction order, one instance of the maximum left
    //      out: the row's log-sum-exp is formed as max + log1p(sum over everything else), which
    //      stays accurate when one token holds nearly all the probability (its log-probability
    //      is -log1p(tiny), and a sum that starts at 1 would have rounded the tiny part away).
    //      Elements equal to the maximum are counted, not added; most waves hold none.
    //      (The elements of a load go through the exponential side by side, in one basic block:
    //      one at a time each is a chain of dependent fp64 instructions and an LDS read.) ----
    double acc = 0.0;
    int neq = 0;
    const bool has_max = __builtin_amdgcn_ballot_w64(tmax == cmax) != 0ull;
    auto exp_load = [&](int s0, int cnt) __attribute__((always_inline)) {
        double e[8];
#pragma unroll
        for (int j = 0; j < cnt; ++j) e[j] = exp_nonpositive((double)x[s0 + j] - (double)cmax, s_exp2);
        if (has_max) {
#pragma unroll
            for (int j = 0; j < cnt; ++j) {
                const bool eq = x[s0 + j] == cmax;
                neq += eq ? 1 : 0;
                e[j] = eq ? 0.0 : e[j];
            }
        }
#pragma unroll
        for (int j = 0; j < cnt; ++j) acc += e[j];
    };
    static_assert(kVecPerThread == 3, "the grouping below is written for three loads per thread");
    if (loads >= 2) exp_load(0, 8);
    else if (loads == 1) exp_load(0, 4);
    if (loads == 3) exp_load(8, 4);
    if (edges) exp_load(4 * kVecPerThread, 2);
    acc = wave_sum_f64_lane63(acc);
    neq = wave_scan_inclusive_i32(neq);
    if (lane == 63) {
        s_dsum[wave] = acc;
        s_neq[wave] = neq;
    }
    __syncthreads();
    const int hot_count = s_count;
    if (tid >= hot_count && tid < a.hot_cap) out[tid] = 0ull;  // (no candidate)
    if (tid == 0) {
        double S = s_dsum[0];
        int n_max = s_neq[0];
        uint32_t lowest = s_low[0];
        for (int w = 1; w < kChunkWaves; ++w) {
            S += s_dsum[w];
            n_max += s_neq[w];
            lowest = min(lowest, s_low[w]);
        }
        ChunkStat r;
        r.sum = S + (double)(n_max - 1);  // everything but one instance of the chunk maximum
        r.max = cmax;
        r.low = lowest == ~0u ? -INFINITY : key_float(lowest);
        r.hot = bound > -INFINITY && hot_count <= a.hot_cap ? bound : INFINITY;
        r.pad = 0;
        stat[row * a.chunks + c] = r;
    }
    if constexpr (FINISH) {
        __shared__ __align__(16) FinishLds L;
        __syncthreads();  // (what this workgroup wrote, it reads back)
        finish_row<kChunkThreads>(p, a, maxima + row * a.maxima, stat + row, hot + row * (size_t)a.hot_cap, L,
                                  topk_tok + row * (size_t)a.K, topk_lp + row * (size_t)a.K);
    }
}

constexpr int kFinishThreads = 1024;
__global__ __launch_bounds__(kFinishThreads) void topk_finish_kernel(
    const float *__restrict__ logits, const float *__restrict__ maxima, const ChunkStat *__restrict__ stat,
    const uint64_t *__restrict__ hot, int V, int K, int chunks, int chunk_len, int maxima_per_chunk, int hot_cap,
    int32_t *__restrict__ topk_tok, float *__restrict__ topk_lp)
{
    const FinishArgs a{V, K, chunks, chunk_len, maxima_per_chunk, hot_cap};
    __shared__ __align__(16) FinishLds L;
    const size_t row = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
    finish_row<kFinishThreads>(logits + row * (size_t)a.V, a, maxima + row * (size_t)a.chunks * a.maxima,
                               stat + row * (size_t)a.chunks, hot + row * (size_t)a.chunks * a.hot_cap, L,
                               topk_tok + row * (size_t)a.K, topk_lp + row * (size_t)a.K);
}
}  // namespace ddt

extern "C" int ddtree_topk(const float *logits, int batch, int B, int V, int K, int32_t *topk_tok,
                           float *topk_lp, void *workspace, size_t workspace_bytes, void *stream)
{
    using namespace ddt;
    if (!logits || !topk_tok || !topk_lp) return DDTREE_ERR_ARG;
    if (batch < 1 || batch > DDTREE_MAX_BATCH || B < 1 || B > DDTREE_MAX_B || V < 1 || K < 1 ||
        K > V || K > DDTREE_MAX_N)
        return DDTREE_ERR_ARG;
    const TopkPlan p = topk_plan(batch, B, V, K);
    if (!p.ok) return DDTREE_ERR_ARG;
    if (!ws_ok(workspace, workspace_bytes, p.bytes)) return DDTREE_ERR_WORKSPACE;
    char *ws = static_cast<char *>(workspace);
    float *maxima = reinterpret_cast<float *>(ws + p.max_off);
    ChunkStat *stat = reinterpret_cast<ChunkStat *>(ws + p.stat_off);
    uint64_t *hot = reinterpret_cast<uint64_t *>(ws + p.hot_off);
    // (Scalars one by one, what is wanted first in front: the first 14 words of the arguments are in registers when a
    // kernel starts, a structure by value is not among them.)
    hipStream_t st = as_stream(stream);
    if (p.chunks == 1) {
        DDT_LAUNCH(DDTREE_KERNEL_TOPK_CHUNK, st, topk_chunk_kernel<true>, dim3(1, B, batch), dim3(kChunkThreads), 0, st, logits, V,
                   p.chunk_len, p.chunks, p.group, p.hot_rank, p.hot_cap, maxima, stat, hot, K, p.maxima, topk_tok, topk_lp);
        return launch_status();
    }
    DDT_LAUNCH(DDTREE_KERNEL_TOPK_CHUNK, st, topk_chunk_kernel<false>, dim3(p.chunks, B, batch), dim3(kChunkThreads), 0, st, logits,
               V, p.chunk_len, p.chunks, p.group, p.hot_rank, p.hot_cap, maxima, stat, hot, K, p.maxima, topk_tok, topk_lp);
    DDT_LAUNCH(DDTREE_KERNEL_TOPK_MERGE, st, topk_finish_kernel, dim3(B, batch), dim3(kFinishThreads), 0, st, logits, maxima,
               stat, hot, V, K, p.chunks, p.chunk_len, p.maxima, p.hot_cap, topk_tok, topk_lp);
    return launch_status();
}
