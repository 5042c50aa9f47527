// Library-level entry points of the C ABI that belong to no single stage: version, error text,
// scratch sizing, and the event-timing hook used by the benchmark.
#include <algorithm>

#include "common.hpp"

namespace ddt {
Profiler &profiler()
{
    static Profiler p;
    return p;
}

static void profiler_destroy(Profiler &p)
{
    for (int k = 0; k < DDTREE_KERNEL_COUNT; ++k) {
        if (p.start[k]) {
            for (int i = 0; i < p.capacity; ++i) {
                (void)hipEventDestroy(p.start[k][i]);
                (void)hipEventDestroy(p.stop[k][i]);
            }
            delete[] p.start[k];
            delete[] p.stop[k];
            p.start[k] = p.stop[k] = nullptr;
        }
        p.count[k] = p.seen[k] = 0;
    }
    p.mask = 0;
    p.capacity = 0;
    p.every = 1;
}
}  // namespace ddt

extern "C" int ddtree_version(void) { return 100; }

extern "C" const char *ddtree_error_string(int code)
{
    switch (code) {
    case DDTREE_OK: return "ok";
    case DDTREE_ERR_ARG: return "bad argument (null pointer, shape, size or dtype)";
    case DDTREE_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case DDTREE_ERR_HIP: return "HIP runtime error at launch";
    default: return "unknown error code";
    }
}

extern "C" size_t ddtree_workspace_bytes(int batch, int B, int V, int N, int Hq, int Hkv, int D,
                                         int max_sum_L)
{
    using namespace ddt;
    (void)max_sum_L;
    if (batch < 1 || batch > DDTREE_MAX_BATCH || B < 1 || B > DDTREE_MAX_B || V < 1 || N < 1 ||
        N > DDTREE_MAX_N || Hq < 1 || Hkv < 1 || Hq % Hkv != 0 || D < 8 || D > 256 || D % 8 != 0)
        return 0;
    const int K = N < V ? N : V;
    const int T = N + 1;
    size_t need = topk_scratch_upper(batch, B, V, K);
    const size_t a = attn_scratch_upper(batch, T, Hq, Hkv, D);
    if (a > need) need = a;
    const size_t c = accept_scratch_upper(batch, T, V);
    if (c > need) need = c;
    return need < 256 ? 256 : need;
}

extern "C" size_t ddtree_verify_attn_workspace_bytes(int batch, int T, int Hq, int Hkv, int D, int dtype,
                                                    long long sum_L)
{
    using namespace ddt;
    if (batch < 1 || batch > DDTREE_MAX_BATCH || T < 1 || T > DDTREE_MAX_N + 1 || Hq < 1 || Hkv < 1 ||
        Hq % Hkv != 0 || D < 8 || D > 256 || D % 8 != 0 || sum_L < 0)
        return 0;
    return attn_scratch_bytes(batch, T, Hq, Hkv, D, dtype, sum_L);
}

extern "C" int ddtree_profile_enable(unsigned kernel_mask, int capacity)
{
    return ddtree_profile_enable_every(kernel_mask, capacity, 1);
}

extern "C" int ddtree_profile_enable_every(unsigned kernel_mask, int capacity, int every)
{
    using namespace ddt;
    Profiler &p = profiler();
    profiler_destroy(p);
    if (kernel_mask == 0) return DDTREE_OK;
    if (capacity < 1 || capacity > (1 << 20) || (kernel_mask >> DDTREE_KERNEL_COUNT) != 0 || every < 1)
        return DDTREE_ERR_ARG;
    p.capacity = capacity;
    p.every = every;
    for (int k = 0; k < DDTREE_KERNEL_COUNT; ++k) {
        if (!(kernel_mask & (1u << k))) continue;
        p.start[k] = new hipEvent_t[capacity];
        p.stop[k] = new hipEvent_t[capacity];
        for (int i = 0; i < capacity; ++i)
            if (hipEventCreate(&p.start[k][i]) != hipSuccess || hipEventCreate(&p.stop[k][i]) != hipSuccess)
                return DDTREE_ERR_HIP;
    }
    p.mask = kernel_mask;
    return DDTREE_OK;
}

extern "C" int ddtree_profile_reset(void)
{
    ddt::Profiler &p = ddt::profiler();
    for (int k = 0; k < DDTREE_KERNEL_COUNT; ++k) p.count[k] = p.seen[k] = 0;
    return DDTREE_OK;
}

extern "C" int ddtree_profile_read(int kernel_id, float *ms_out, int max_records)
{
    ddt::Profiler &p = ddt::profiler();
    if (kernel_id < 0 || kernel_id >= DDTREE_KERNEL_COUNT || !ms_out || max_records < 0)
        return DDTREE_ERR_ARG;
    if (!(p.mask & (1u << kernel_id))) return 0;
    const int n = p.count[kernel_id] < max_records ? p.count[kernel_id] : max_records;
    for (int i = 0; i < n; ++i)
        if (hipEventElapsedTime(&ms_out[i], p.start[kernel_id][i], p.stop[kernel_id][i]) != hipSuccess)
            return DDTREE_ERR_HIP;
    return n;
}

// Host-side self-check (no GPU): the attention kernel's launch arithmetic (attn.hip) and the
// invariants of the top-K and accept plans that their kernels index by.
namespace ddt {
int attn_selftest_host();
}
extern "C" int ddtree_selftest_host(void)
{
    using namespace ddt;
    if (const int rc = attn_selftest_host()) return rc;
    // top-K: chunks tile the row and stay within what a chunk workgroup holds; the scratch holds what
    // the kernels index
    const int Vs[] = {1, 2, 7, 64, 1000, 1024, 4096, 12288, 12289, 20000, 50001, 100000, 151936, 172032, 200003, 344064, 688128, 1000000};
    const int Ks[] = {1, 2, 16, 64, 255, 256, 257, 512, 1024};
    const int rows_[] = {1, 2, 3, 8, 16, 17, 64, 127, 128, 1024};
    for (int V : Vs)
        for (int K : Ks)
            for (int rows : rows_) {
                if (K > V) continue;
                const TopkPlan p = topk_plan(1, rows, V, K);
                if (!p.ok) return 10001;
                if (p.chunk_len % 4 != 0 || p.chunk_len < 1 || p.chunk_len > kTopkChunkMax) return 10004;
                if ((long long)(p.chunks - 1) * p.chunk_len >= V || (long long)p.chunks * p.chunk_len < V) return 10005;
                if (p.group < 1 || p.group > 8 || (p.group & (p.group - 1)) || p.maxima * p.group != 512) return 10006;
                if (p.hot_rank < 1 || p.hot_rank > 64 || p.hot_cap < 0 || (p.hot_cap & (p.hot_cap - 1))) return 10007;
                const size_t per = (size_t)rows * p.chunks;
                if (p.stat_off < per * p.maxima * 4 || p.hot_off < p.stat_off + per * 24 || p.bytes < p.hot_off + per * p.hot_cap * 8)
                    return 10010;
                if ((p.stat_off & 255u) || (p.hot_off & 255u) || (p.bytes & 255u)) return 10011;
                // a workspace for these sizes serves every smaller call: all K of this shape, fewer rows, shorter rows
                if (rows <= DDTREE_MAX_B) {
                    const size_t have = ddtree_workspace_bytes(1, rows, V, K, 1, 1, 96, 0);
                    for (int k = 1; k <= K; ++k)
                        if (topk_plan(1, rows, V, k).bytes > have) return 10012;
                    for (int r = 1; r < rows; ++r)
                        for (int k : {1, K / 2 + 1, K})
                            if (topk_plan(1, r, V, k).bytes > have) return 10013;
                    for (int v : Vs)
                        if (v < V && topk_plan(1, rows, v, std::min(v, K)).bytes > have) return 10014;
                }
            }
    for (int batch : {1, 3, 16, 64})  // many rows, and odd ones
        for (int B : {1, 5, 16, 17, 32})
            for (int V : Vs)
                for (int K : Ks)
                    for (int b = 1; b <= batch && K <= V; b += 1 + b / 5)
                        for (int k = K; k >= 1; k -= 1 + k / 7)
                            if (topk_plan(b, B, V, k).bytes > topk_scratch_upper(batch, B, V, K)) return 10015;
    // accept: segments tile the row in multiples of four, scratch holds one partial per segment
    for (int V : Vs)
        for (int T : {2, 17, 65, 257, 513, 1025})
            for (int batch : {1, 16, 64}) {
                const AcceptPlan p = accept_plan(batch, T, V);
                if (p.seg_len % 4 != 0 || p.seg_len < 1 || p.splits < 1) return 10021;
                if ((long long)(p.splits - 1) * p.seg_len >= V || (long long)p.splits * p.seg_len < V) return 10022;
                if (p.bytes < (size_t)batch * T * p.splits * 8 || (p.bytes & 255u)) return 10023;
                for (int b = 1; b <= batch; b += 1 + b / 3)
                    for (int t = T; t >= 2; t -= 1 + t / 5)
                        if (accept_plan(b, t, V).bytes > accept_scratch_upper(batch, T, V)) return 10024;
            }
    return 0;
}
