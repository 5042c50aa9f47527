// Greedy verifier walk (paper Section 4.4, second paragraph, and Figure 1b) and cache compaction
// (Section 4.4, last sentence).
//
//   argmax kernel  HBM-bound scan of the target logits: one workgroup per (row, segment),
//                  coalesced 16-byte loads, first-maximum semantics (lowest id among equal
//                  maxima), one (value, index) partial per segment.
//   walk kernel    one workgroup per sequence: folds the partials into the posterior token of
//                  every node, then decides acceptance for all nodes at once: node i is accepted
//                  iff every node on its root path carries the token its parent's posterior
//                  chose.  The accepted nodes form the single path the sequential walk of the
//                  paper visits, and the deepest one yields the bonus token.
//   compact kernel copies the accepted tree rows of K and V behind the cache.
#include <algorithm>

#include "common.hpp"

namespace ddt {

constexpr int kArgmaxThreads = 256;

AcceptPlan accept_plan(int batch, int T, int V)
{
    AcceptPlan p{};
    long long rows = (long long)batch * T;
    // About 3000 workgroups stream closest to the HBM rate; a segment of 4096 elements is four 16-byte loads
    // a thread (65 rows of 151936: 8.5 us, with at least 8192 elements 9.1; 404 rows of 50021: 13.8 and 14.7).
    int S = (int)((3072 + rows - 1) / rows);
    int s_cap = V / 4096 > 0 ? V / 4096 : 1;
    if (S > s_cap) S = s_cap;
    if (S < 1) S = 1;
    int len = (V + S - 1) / S;
    len = (len + 3) / 4 * 4;
    p.seg_len = len;
    p.splits = (V + len - 1) / len;
    p.part_off = 0;
    p.bytes = align_up((size_t)rows * p.splits * 8, 256);
    return p;
}

// A bound on accept_plan(...).bytes over every call of at most this many rows and elements.
size_t accept_scratch_upper(int batch, int T, int V)
{
    const long long rows = (long long)batch * T;
    return align_up((size_t)std::min(rows + 3071, rows * std::max(1, V / 4096)) * 8, 256);
}

// A segment's best: the value's order-preserving key, and below it the complement of the token id, so that the larger
// of two is the larger value or, of equal ones, the lower id.
typedef unsigned long long ArgPart;
constexpr ArgPart kNoPart = 0ull;  // (below everything)
__device__ __forceinline__ ArgPart arg_part(float v, int i) { return (ArgPart)float_key(v) << 32 | (uint32_t)~i; }
__device__ __forceinline__ int arg_token(ArgPart p) { return (int)~(uint32_t)p; }
// Against the lane that CTRL names.  (On two registers through DPP a step costs some 50 cycles, value and id exchanged
// through LDS 190: scan and walk, launch to launch, of 17 rows of 151936 8.1 -> 6.8 us, 65 of 32003 7.7 -> 6.5, 257 of 151936 28.2 -> 27.6.)
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ ArgPart arg_max_dpp(ArgPart p)
{
    const ArgPart o = (ArgPart)dpp_u<CTRL, ROW_MASK>((uint32_t)(p >> 32)) << 32 | dpp_u<CTRL, ROW_MASK>((uint32_t)p);
    return o > p ? o : p;
}

__device__ __forceinline__ void arg_update(float &bv, int &bi, float v, int i)
{
    if (v > bv || (v == bv && i < bi)) {
        bv = v;
        bi = i;
    }
}

// Temperature sampling (Section 4.4: verification follows the target's decoding rule, greedy or
// temperature-based sampling).  The token selected at a node is argmax_v (logit[v] / tau + g[v])
// with Gumbel noise g = -log(-log(u)), which is a sample from softmax(logit / tau); u in (0,1)
// comes from a counter-based generator keyed by (seed, row, v), so the draw does not depend on
// how the scan is split over threads:
//     mix(x):  x ^= x >> 16; x *= 0x7feb352d; x ^= x >> 15; x *= 0x846ca68b; x ^= x >> 16
//     h = mix(mix(v ^ seed_lo) + 0x9E3779B9 * row + seed_hi),   u = ((h >> 8) + 0.5) / 2^24
struct SampleArgs {
    float inv_tau;       // 0 selects the greedy rule
    uint32_t seed_lo, seed_hi;
};
__device__ __forceinline__ uint32_t sample_mix(uint32_t x)
{
    x ^= x >> 16;
    x *= 0x7feb352du;
    x ^= x >> 15;
    x *= 0x846ca68bu;
    x ^= x >> 16;
    return x;
}
// the key of one element from its hash
__device__ __forceinline__ float sample_key(float logit, uint32_t h, const SampleArgs &sa)
{
    // -ln u in fp32 without losing the draws that matter most (u close to 1 gives the largest
    // noise): for k < 2^23, u = (k + 0.5) / 2^24 is exact in fp32; otherwise w = 1 - u =
    // (2^24 - 1 - k + 0.5) / 2^24 is, and -ln(1 - w) is taken from its series when w is small
    const uint32_t k = h >> 8;
    const bool low = k < (1u << 23);
    const float frac = ((float)(low ? k : 16777215u - k) + 0.5f) * (1.0f / 16777216.0f);  // u or w
    const float la = -0.69314718056f * __builtin_amdgcn_logf(low ? frac : 1.0f - frac);
    const float series = frac * (1.0f + frac * (0.5f + frac * (0.333333343f + frac * 0.25f)));
    const float nl = (!low && frac < 0.015625f) ? series : la;
    const float g = -0.69314718056f * __builtin_amdgcn_logf(nl);  // g = -ln(-ln u)
    return fmaf(logit, sa.inv_tau, g);
}

// The workgroup's best, valid in thread 0.
__device__ __forceinline__ ArgPart workgroup_best(float bv, int bi, ArgPart *s_best)
{
    ArgPart p = arg_part(bv, bi);
    p = arg_max_dpp<0xB1>(p);
    p = arg_max_dpp<0x4E>(p);
    p = arg_max_dpp<0x141>(p);
    p = arg_max_dpp<0x140>(p);
    p = arg_max_dpp<0x142, 0xA>(p);
    p = arg_max_dpp<0x143, 0xC>(p);
    if ((threadIdx.x & 63) == 63) s_best[threadIdx.x >> 6] = p;
    __syncthreads();
    p = s_best[0];
#pragma unroll
    for (int w = 1; w < kArgmaxThreads / 64; ++w) p = s_best[w] > p ? s_best[w] : p;
    return p;
}

__device__ __forceinline__ float4 load_streamed(const float4 *p)  // (read once: marked non-temporal)
{
    const float *q = reinterpret_cast<const float *>(p);
    return make_float4(__builtin_nontemporal_load(q), __builtin_nontemporal_load(q + 1), __builtin_nontemporal_load(q + 2),
                       __builtin_nontemporal_load(q + 3));
}

__global__ __launch_bounds__(kArgmaxThreads) void accept_argmax_kernel(
    const float *__restrict__ logits, int T, int V, int seg_len, int splits,
    const int32_t *__restrict__ n_nodes, ArgPart *__restrict__ part)
{
    __shared__ ArgPart s_parts[kArgmaxThreads / 64];
    const int tid = threadIdx.x;
    const int seg = blockIdx.x, i = blockIdx.y, seq = blockIdx.z;
    if (i > n_nodes[seq]) return;  // padding row: never read, the walk ignores its partial
    const size_t rowi = (size_t)seq * T + i;
    const int start = seg * seg_len;
    const int n = min(seg_len, V - start);
    const float *p = logits + rowi * (size_t)V + start;

    float bv = -INFINITY;
    int bi = 0x7FFFFFFF;
    int head = (int)((4 - ((reinterpret_cast<uintptr_t>(p) >> 2) & 3)) & 3);
    if (head > n) head = n;
    if (tid < head) {
        const float x = p[tid];
        if (x >= bv) { bv = x; bi = start + tid; }
    }
    const int nvec = (n - head) >> 2;
    const float4 *pv = reinterpret_cast<const float4 *>(p + head);
    // eight independent 16-byte loads in flight per thread and iteration: about 128 KB per compute
    // unit, what it takes to cover the HBM latency at full bandwidth
    constexpr int kInFlight = 8;
    for (int j0 = tid; j0 < nvec; j0 += kInFlight * kArgmaxThreads) {
        float4 x[kInFlight];
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int j = j0 + u * kArgmaxThreads;
            x[u] = j < nvec ? load_streamed(pv + j) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
        }
#pragma unroll
        for (int u = 0; u < kInFlight; ++u) {
            const int ia = start + head + 4 * (j0 + u * kArgmaxThreads);
            if (x[u].x > bv) { bv = x[u].x; bi = ia; }
            if (x[u].y > bv) { bv = x[u].y; bi = ia + 1; }
            if (x[u].z > bv) { bv = x[u].z; bi = ia + 2; }
            if (x[u].w > bv) { bv = x[u].w; bi = ia + 3; }
        }
    }
    const int tail0 = head + 4 * nvec;
    if (tid < n - tail0) {
        const float x = p[tail0 + tid];
        if (x > bv) { bv = x; bi = start + tail0 + tid; }
    }
    const ArgPart best_part = workgroup_best(bv, bi, s_parts);
    if (tid == 0) part[rowi * splits + seg] = best_part;
}

// The sampled scan, bound by the vector ALUs: the hash of an element is four 32-bit multiplies, a
// quarter-rate instruction each, and its key two logarithms more.  Most elements are settled by their hash:
// the noise is bounded by g = -ln(-ln u) <= -ln(1 - u), so an element can reach a key wb already found in the
// row only if 1 - u <= exp(logit / tau - wb), a comparison of the hash with a threshold that is formed
// once for the four elements of a load, from the largest of them, and then for the few that pass.  wb is
// the best key of the whole workgroup (in LDS) and starts at a lower bound from the first load's hashes.
// Measured (scan alone, tau = 0.8): 257 rows of 151936 47.3 -> 37.0 us, 258 rows (two trees) 48.9 -> 39.4, 17 rows 10.9 -> 7.6, 65 rows of 32003 9.0 -> 7.6; before,
// every wave pruned against its own best with a bound a factor of two wide, and took its whole first round
// of 32 elements a lane in full.  Four rows to a workgroup, sharing the half of the hash that does not
// depend on the row, was slower than one (38 us against 36): fewer, longer-lived workgroups.  A greedy scan of
// the same bytes takes 25 us.
__global__ __launch_bounds__(kArgmaxThreads) void accept_sample_kernel(
    const float *__restrict__ logits, int T, int V, int seg_len, int splits,
    const int32_t *__restrict__ n_nodes, ArgPart *__restrict__ part, SampleArgs sa)
{
    __shared__ ArgPart s_parts[kArgmaxThreads / 64];
    __shared__ uint32_t s_best;  // a lower bound on the row's best key, order-preserving
    const int tid = threadIdx.x;
    const int seg = blockIdx.x, i = blockIdx.y, seq = blockIdx.z;
    if (i > n_nodes[seq]) return;  // padding row: never read, the walk ignores its partial
    const size_t rowi = (size_t)seq * T + i;
    const uint32_t row_term = 0x9E3779B9u * (uint32_t)rowi + sa.seed_hi;
    const int start = seg * seg_len;
    const int n = min(seg_len, V - start);
    const float *p = logits + rowi * (size_t)V + start;
    int head = (int)((4 - ((reinterpret_cast<uintptr_t>(p) >> 2) & 3)) & 3);
    if (head > n) head = n;
    const int nvec = (n - head) >> 2, tail0 = head + 4 * nvec;
    const float4 *pv = reinterpret_cast<const float4 *>(p + head);
    auto hash = [&](int id) { return sample_mix(sample_mix((uint32_t)id ^ sa.seed_lo) + row_term); };

    auto load = [&](int j) { return j < nvec ? load_streamed(pv + j) : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY); };
    float4 x = load(tid);
    if (tid == 0) s_best = 0u;
    float bv = -INFINITY;
    int bi = 0x7FFFFFFF;
    // the scalar elements in front of the 16-byte loads, and those behind them, which are looked at last: elements are
    // taken in the order of their ids, so that of equal keys the lowest stays
    if (tid < head) arg_update(bv, bi, sample_key(p[tid], hash(start + tid), sa), start + tid);
    const float behind = tid < n - tail0 ? p[tail0 + tid] : 0.0f;
    __syncthreads();
    {
        // for u >= 1/2, -ln u <= 2 ln 2 (1 - u), so g >= -ln(1.387 (1 - u))
        const float xe[4] = {x.x, x.y, x.z, x.w};
        float low = -INFINITY;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t h = hash(start + head + 4 * tid + e);
            const float g = -0.693147f * (__builtin_amdgcn_logf((float)(~h) + 256.0f) - 32.0f) - 0.33f;
            low = fmaxf(low, (h >> 31) ? fmaf(xe[e], sa.inv_tau, g) : -INFINITY);
        }
        low = wave_max_f32(low);
        low -= fabsf(low) * 1e-6f;
        if ((tid & 63) == 0 && low > -INFINITY) atomicMax(&s_best, float_key(low));
    }
    __syncthreads();
    const float scale = sa.inv_tau * 1.44269504f;
    // (the loop is uniform over a wave: the wave maximum below wants all its lanes in every round)
    for (int jb = tid & ~63; jb < nvec; jb += kArgmaxThreads) {
        const int j = jb + (tid & 63);
        const float4 c = x;
        x = load(j + kArgmaxThreads);
        // (another wave's key may or may not be there yet: any of them will do)
        const uint32_t best = __hip_atomic_load(&s_best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        // With k = h >> 8, 2^32 (1 - u) = 2^32 - 256 k - 128 >= ~h - 127: only an element with
        // ~h <= 2^32 exp(x / tau - wb) + 127 can matter.  (The margin covers the rounding of keys and threshold.)
        const float wb = key_float(best) * 1.44269504f, bias = best ? 32.003f + (4e-7f * fabsf(wb) - wb) : INFINITY;
        auto limit = [&](float v) {
            const float t = __builtin_amdgcn_exp2f(fminf(fmaf(v, scale, bias), 32.0f));
            return t < 4294960000.0f ? ~(uint32_t)(t + 129.0f) : 0u;
        };
        const int ia = start + head + 4 * j;
        uint32_t h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = hash(ia + e);
        const float top = fmaxf(fmaxf(c.x, c.y), fmaxf(c.z, c.w));
        bool need = j < nvec && max(max(h[0], h[1]), max(h[2], h[3])) >= limit(top);
        if (__builtin_amdgcn_ballot_w64(need) == 0ull) continue;
        // Masked tokens (-1e9): their noise vanishes in the rounding and all keys are equal.  No key exceeds
        // logit / tau + 25 ln 2, and one that only equals this thread's best has the higher id.  (16 x 129 rows of
        // 50021, two thirds masked: 160 -> 85 us.)
        need = need && fmaf(top, sa.inv_tau, 17.4f) > bv;
        if (__builtin_amdgcn_ballot_w64(need) == 0ull) continue;
        const float xe[4] = {c.x, c.y, c.z, c.w};
        const float before = bv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool this_one = need && h[e] >= limit(xe[e]);
            if (__builtin_amdgcn_ballot_w64(this_one) == 0ull) continue;
            const float k = sample_key(xe[e], h[e], sa);
            if (this_one && k > bv) {
                bv = k;
                bi = ia + e;
            }
        }
        if (__builtin_amdgcn_ballot_w64(bv > before) != 0ull) {
            const float wmax = wave_max_f32(bv);
            if ((tid & 63) == 0) atomicMax(&s_best, float_key(wmax));
        }
    }
    if (tid < n - tail0) arg_update(bv, bi, sample_key(behind, hash(start + tail0 + tid), sa), start + tail0 + tid);
    const ArgPart best_part = workgroup_best(bv, bi, s_parts);
    if (tid == 0) part[rowi * splits + seg] = best_part;
}

// One workgroup per sequence, `lanes` (a power of two) per row.
constexpr int kWalkMaxThreads = 1024;
__global__ __launch_bounds__(kWalkMaxThreads) void accept_walk_kernel(
    const ArgPart *__restrict__ part, int T, int splits, int lanes, int B, const int32_t *__restrict__ tokens,
    const int32_t *__restrict__ parent, const int32_t *__restrict__ depth,
    const int32_t *__restrict__ n_nodes, int32_t *__restrict__ path,
    int32_t *__restrict__ n_accepted, int32_t *__restrict__ bonus_token,
    int32_t *__restrict__ posterior)
{
    __shared__ int s_post[DDTREE_MAX_N + 1];
    __shared__ int s_tok[DDTREE_MAX_N + 1];
    __shared__ int s_par[DDTREE_MAX_N + 1];
    __shared__ int s_dep[DDTREE_MAX_N + 1];
    __shared__ int s_path[DDTREE_MAX_B + 1];
    __shared__ int s_len;
    const int tid = threadIdx.x, threads = blockDim.x;
    const int seq = blockIdx.x;
    const int n = n_nodes[seq];
    const size_t base = (size_t)seq * T;
    const int sub = tid & (lanes - 1), rows = threads / lanes;
    constexpr int kPer = 8;  // partial results of a lane requested together
    for (int i = tid / lanes; i - tid / lanes < T; i += rows) {  // (uniform: the lanes of a row stay together)
        // Everything a row needs is requested before the node count is looked at, so that its
        // arrival and theirs overlap: its partial results (padding rows have none written: what is
        // read there is never used), its token, parent and depth.
        const bool on = i < T;
        const ArgPart *pp = part + (base + (on ? i : 0)) * splits;
        ArgPart a[kPer], best = kNoPart;
#pragma unroll
        for (int u = 0; u < kPer; ++u) {  // (past the end: the last one once more, which changes nothing)
            a[u] = kNoPart;
            if (u * lanes < splits) a[u] = pp[min(sub + u * lanes, splits - 1)];
        }
        int tk = -1, pr = -1, dp = 0;
        if (on && sub == 0) tk = tokens[base + i], pr = parent[base + i], dp = depth[base + i];
#pragma unroll
        for (int u = 0; u < kPer; ++u) best = a[u] > best ? a[u] : best;
        for (int q = sub + kPer * lanes; q < splits; q += lanes) best = pp[q] > best ? pp[q] : best;
        // (the lanes of a row are neighbours; each step leaves the larger in both of a pair, so that mirrored lanes will do)
        if (lanes >= 2) best = arg_max_dpp<0xB1>(best);
        if (lanes >= 4) best = arg_max_dpp<0x4E>(best);
        if (lanes >= 8) best = arg_max_dpp<0x141>(best);
        if (lanes >= 16) best = arg_max_dpp<0x140>(best);
        for (int d = 16; d < lanes; d *= 2) {
            const ArgPart o = __shfl_xor(best, d, 64);
            best = o > best ? o : best;
        }
        const int bi = arg_token(best);
        if (on && sub == 0) {
            const bool in_tree = i <= n;
            const int post = in_tree ? bi : -1;
            s_post[i] = post;
            s_tok[i] = in_tree ? tk : -1;
            s_par[i] = in_tree ? pr : -1;
            s_dep[i] = dp;
            if (posterior) posterior[base + i] = post;
        }
    }
    if (tid <= B) s_path[tid] = tid == 0 ? 0 : -1;
    if (tid == 0) s_len = 0;
    __syncthreads();
    for (int i = 1 + tid; i <= n; i += threads) {
        bool ok = true;
        int j = i;
        while (j > 0 && ok) {
            const int pj = s_par[j];
            ok = s_tok[j] == s_post[pj];
            j = pj;
        }
        if (ok) {
            const int d = s_dep[i];
            if (d >= 1 && d <= B) {
                s_path[d] = i;
                atomicMax(&s_len, d);
            }
        }
    }
    __syncthreads();
    if (tid <= B) path[(size_t)seq * (B + 1) + tid] = s_path[tid];
    if (tid == 0) {
        const int len = s_len;
        n_accepted[seq] = len;
        bonus_token[seq] = s_post[s_path[len]];
    }
}

struct CompactArgs {
    int32_t dst_row[DDTREE_MAX_BATCH];
};

constexpr int kCompactThreads = 256;
__global__ __launch_bounds__(kCompactThreads) void compact_kernel(
    const int32_t *__restrict__ path, const int32_t *__restrict__ n_accepted, int T, int B, int row_words, int dst0,
    const uint32_t *__restrict__ k_tree, const uint32_t *__restrict__ v_tree,
    uint32_t *__restrict__ k_cache, uint32_t *__restrict__ v_cache, CompactArgs args)
{
    const int j = blockIdx.x, seq = blockIdx.y;
    // Bound by latencies: a launch, the path, the row.  The path and its length are requested together (entries behind
    // the path are allocated and hold -1), K and V likewise; the first sequence's row is a scalar argument.  (A round of
    // eight layers, each with attention, merge and append: 206 -> 189 us with this and the like in attn_common.hpp.)
    const int len = n_accepted[seq], node = path[(size_t)seq * (B + 1) + j];
    const int dst_row = seq == 0 ? dst0 : args.dst_row[seq];
    if (j > len || node < 0 || node >= T) return;
    const size_t src = ((size_t)seq * T + node) * row_words;
    const size_t dst = ((size_t)dst_row + j) * row_words;
    for (int w = threadIdx.x; w < row_words; w += kCompactThreads) {
        const uint32_t k = k_tree[src + w], v = v_tree[src + w];
        k_cache[dst + w] = k;
        v_cache[dst + w] = v;
    }
}

}  // namespace ddt

// Scratch of ddtree_accept_noalloc: the partial argmaxes live in this array instead of a caller's
// workspace.  Every GPU the library runs on holds its own copy until the process ends.  In host
// code the array's name is only a handle for hipGetSymbolAddress; the device address it returns
// (one per device) is what the kernels are given.
namespace ddt {
constexpr size_t kNoAllocScratchBytes = DDTREE_NOALLOC_SCRATCH_BYTES;  // 32768 (value, index) partials
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];
constexpr int kNoAllocMaxDevices = 64;
}  // namespace ddt

// Device address of the scratch array on the current device, looked up once per device.
static int noalloc_scratch(void **out)
{
    static std::atomic<void *> ptrs[ddt::kNoAllocMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= ddt::kNoAllocMaxDevices) return DDTREE_ERR_HIP;
    void *p = ptrs[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(ddt::scratch)) != hipSuccess || !p) return DDTREE_ERR_HIP;
        ptrs[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return DDTREE_OK;
}

static int accept_impl(const float *target_logits, int batch, int T, int V, const int32_t *tokens,
                       const int32_t *parent, const int32_t *depth, const int32_t *n_nodes,
                       int32_t *path, int32_t *n_accepted, int32_t *bonus_token, int32_t *posterior,
                       int B, void *workspace, size_t workspace_bytes, void *stream, bool sample,
                       ddt::SampleArgs sa)
{
    using namespace ddt;
    if (!target_logits || !tokens || !parent || !depth || !n_nodes || !path || !n_accepted ||
        !bonus_token)
        return DDTREE_ERR_ARG;
    if (batch < 1 || batch > DDTREE_MAX_BATCH || T < 2 || T > DDTREE_MAX_N + 1 || V < 1 || B < 1 ||
        B > DDTREE_MAX_B)
        return DDTREE_ERR_ARG;
    AcceptPlan p = accept_plan(batch, T, V);
    if (!ws_ok(workspace, workspace_bytes, p.bytes)) return DDTREE_ERR_WORKSPACE;
    ArgPart *part = reinterpret_cast<ArgPart *>(static_cast<char *>(workspace) + p.part_off);
    hipStream_t st = as_stream(stream);
    if (sample)
        DDT_LAUNCH(DDTREE_KERNEL_ACCEPT_ARGMAX, st, accept_sample_kernel, dim3(p.splits, T, batch), dim3(kArgmaxThreads), 0, st,
                   target_logits, T, V, p.seg_len, p.splits, n_nodes, part, sa);
    else
        DDT_LAUNCH(DDTREE_KERNEL_ACCEPT_ARGMAX, st, accept_argmax_kernel, dim3(p.splits, T, batch), dim3(kArgmaxThreads), 0, st,
                   target_logits, T, V, p.seg_len, p.splits, n_nodes, part);
    // as many lanes per row as there are partial results, within one workgroup; every row at once (T = 1025: but one)
    int lanes = 1;
    while (lanes < 64 && lanes < p.splits && 2 * lanes * T <= kWalkMaxThreads) lanes *= 2;
    const int threads = std::min(kWalkMaxThreads, std::max(64, (lanes * T + 63) / 64 * 64));
    DDT_LAUNCH(DDTREE_KERNEL_ACCEPT_WALK, st, accept_walk_kernel, dim3(batch), dim3(threads), 0, st, part, T, p.splits, lanes,
                       B, tokens, parent, depth, n_nodes, path, n_accepted, bonus_token, posterior);
    return launch_status();
}

extern "C" int ddtree_accept(const float *target_logits, int batch, int T, int V,
                             const int32_t *tokens, const int32_t *parent, const int32_t *depth,
                             const int32_t *n_nodes, int32_t *path, int32_t *n_accepted,
                             int32_t *bonus_token, int32_t *posterior, int B, void *workspace,
                             size_t workspace_bytes, void *stream)
{
    return accept_impl(target_logits, batch, T, V, tokens, parent, depth, n_nodes, path, n_accepted,
                       bonus_token, posterior, B, workspace, workspace_bytes, stream, false,
                       ddt::SampleArgs{0.0f, 0u, 0u});
}

extern "C" int ddtree_accept_noalloc(const float *target_logits, int batch, int T, int V,
                                     const int32_t *tokens, const int32_t *parent, const int32_t *depth,
                                     const int32_t *n_nodes, int32_t *path, int32_t *n_accepted,
                                     int32_t *bonus_token, int32_t *posterior, int B, void *stream)
{
    using namespace ddt;
    if (!target_logits || !tokens || !parent || !depth || !n_nodes || !path || !n_accepted || !bonus_token)
        return DDTREE_ERR_ARG;
    if (batch < 1 || batch > DDTREE_MAX_BATCH || T < 2 || T > DDTREE_MAX_N + 1 || V < 1 || B < 1 ||
        B > DDTREE_MAX_B)
        return DDTREE_ERR_ARG;
    // the partials of this shape must fit the static array (nothing here can grow it)
    if (accept_plan(batch, T, V).bytes > kNoAllocScratchBytes) return DDTREE_ERR_WORKSPACE;
    void *ws = nullptr;
    const int rc = noalloc_scratch(&ws);
    if (rc != DDTREE_OK) return rc;
    // Every partial the walk reads is written by the scan of the same call (rows up to n_nodes,
    // all segments), so nothing in the array has to start at zero.
    return accept_impl(target_logits, batch, T, V, tokens, parent, depth, n_nodes, path, n_accepted,
                       bonus_token, posterior, B, ws, kNoAllocScratchBytes, stream, false,
                       ddt::SampleArgs{0.0f, 0u, 0u});
}

extern "C" int ddtree_accept_sampled(const float *target_logits, int batch, int T, int V,
                                     const int32_t *tokens, const int32_t *parent,
                                     const int32_t *depth, const int32_t *n_nodes, float temperature,
                                     uint64_t seed, int32_t *path, int32_t *n_accepted,
                                     int32_t *bonus_token, int32_t *posterior, int B,
                                     void *workspace, size_t workspace_bytes, void *stream)
{
    if (!(temperature > 0.0f) || !(temperature < 1e30f)) return DDTREE_ERR_ARG;
    return accept_impl(target_logits, batch, T, V, tokens, parent, depth, n_nodes, path, n_accepted,
                       bonus_token, posterior, B, workspace, workspace_bytes, stream, true,
                       ddt::SampleArgs{1.0f / temperature, (uint32_t)seed, (uint32_t)(seed >> 32)});
}

extern "C" int ddtree_compact(const void *k_tree, const void *v_tree, const int32_t *path,
                              const int32_t *n_accepted, const int32_t *dst_row, int batch, int T,
                              int B, int Hkv, int D, int elem_bytes, void *k_cache, void *v_cache,
                              void *stream)
{
    using namespace ddt;
    if (!k_tree || !v_tree || !path || !n_accepted || !dst_row || !k_cache || !v_cache)
        return DDTREE_ERR_ARG;
    if (batch < 1 || batch > DDTREE_MAX_BATCH || T < 2 || B < 1 || B > DDTREE_MAX_B || Hkv < 1 ||
        D < 1 || (elem_bytes != 2 && elem_bytes != 4))
        return DDTREE_ERR_ARG;
    const long long row_bytes = (long long)Hkv * D * elem_bytes;
    if (row_bytes % 4 != 0) return DDTREE_ERR_ARG;
    for (const void *t : {k_tree, v_tree, static_cast<const void *>(k_cache), static_cast<const void *>(v_cache)})
        if (reinterpret_cast<uintptr_t>(t) & 3u) return DDTREE_ERR_ARG;  // rows are copied in 4-byte words
    CompactArgs args;
    for (int s = 0; s < batch; ++s) {
        if (dst_row[s] < 0) return DDTREE_ERR_ARG;
        args.dst_row[s] = dst_row[s];
    }
    hipLaunchKernelGGL(compact_kernel, dim3(B + 1, batch), dim3(kCompactThreads), 0, as_stream(stream),
                       path, n_accepted, T, B, (int)(row_bytes / 4), dst_row[0],
                       static_cast<const uint32_t *>(k_tree), static_cast<const uint32_t *>(v_tree),
                       static_cast<uint32_t *>(k_cache), static_cast<uint32_t *>(v_cache), args);
    return launch_status();
}
