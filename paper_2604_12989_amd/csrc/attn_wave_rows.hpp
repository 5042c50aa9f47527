// Attention of a block of query rows (or two) over a key range, every wave with key sub-tiles of its own: the
// body of attn_wave_kernel, and of attn_mfma_kernel for the few rows that are left beside its whole tiles.
#pragma once

#include "attn_common.hpp"

namespace ddt {

// Sizes that follow from the head dim D and the row blocks per wave RB.
template <int D, int RB>
struct WaveShape {
    static_assert(D == 64 || RB == 1, "64 rows of 128 dims would take 192 registers a lane for results and queries alone");
    static constexpr int waves = 8;
    static constexpr int threads = 64 * waves;
    static constexpr int stages = D == 128 ? 1 : 2;  // sub-tiles of a wave in LDS
    static constexpr int row_bytes = D * 2;                  // one key or value row in LDS
    static constexpr int tile_bytes = kSK * row_bytes;       // K or V sub-tile
    static constexpr int mask_bytes = 256;                   // a mask word per row of the sub-tile's row blocks
    static constexpr int stage_bytes = 2 * tile_bytes + mask_bytes;
    static constexpr int ring_bytes = stages * stage_bytes;  // per wave
    static constexpr int dma = tile_bytes / 1024;            // load instructions per K or V sub-tile
    static constexpr int rows_per_dma = kSK / dma;
    static constexpr int chunks = row_bytes / 16;            // 16-byte chunks per row
    static constexpr int epi_row = D * 4 + 16;               // fp32 results: rows 4 banks apart
    static constexpr int epi_bytes = RB * 32 * epi_row;      // per wave
    static constexpr int main_bytes = waves * (ring_bytes > epi_bytes ? ring_bytes : epi_bytes);
    static constexpr int lds_bytes = 256 + main_bytes + waves * RB * 32 * 8;
    static_assert(lds_bytes <= 160 * 1024, "fits the LDS of a compute unit");
};

// What a workgroup does with its row group and key range.  Args: AttnWaveArgs, or what attn_mfma_kernel has; WIDE:
// partial results are fp32 rows.
template <int D, int RB, bool WIDE, class Args>
__device__ __forceinline__ void attn_wave_rows(const Args &args, const AttnWaveItem &item)
{
    using S = WaveShape<D, RB>;
    constexpr int KS = D / 16, DB = D / 32, NI = S::dma, NW = S::waves, NS = S::stages;
    // Heads of 64: a weight is the sum of two bf16 numbers (2^-17 off), each with a product of its own, and the
    // reference of a row its true maximum so far, so that weights stay within 1: what fp32 weights give on the
    // vector ALUs, where these heads ran before.  The second product is hidden behind the waits for the keys.
    constexpr bool TWO = D == 64;
    constexpr float kSlack = TWO ? 0.0f : 16.0f;
    const int T = args.T, Hq = args.Hq, Hkv = args.Hkv;
    const float scale_log2e = args.scale_log2e;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    unsigned char *const smem =
        smem_raw + ((0u - (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem_raw) & 255u);
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;

    const int seq = item.seq, hk = item.hk, L = item.kv_len, G = args.group_size;
    const int r0 = item.r0, r1 = item.r1, n_cache = item.n_cache;
    const int n = max(0, (item.t_end - item.t_begin - wave + NW - 1) / NW);  // sub-tiles of this wave: every NW-th
    const int t_first = item.t_begin + wave;

    const int W2 = ((T + 63) >> 6) * 2;  // 32-bit words per mask row
    const uint32_t *const mask32 = reinterpret_cast<const uint32_t *>(args.mask) + (size_t)seq * T * W2;

    // ---- requests: each row's own mask bit (a padding row produces zeros) for the combining threads,
    //      the queries, the first two sub-tiles ----
    constexpr int CH = D / 8;                  // threads per row when rows are combined, 8 dims each
    constexpr int RPP = S::threads / CH;       // rows per pass
    constexpr int PASSES = (RB * 32 + RPP - 1) / RPP;
    uint32_t own[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int r = r0 + p * RPP + tid / CH;
        const int nd = div_by(min(r, r1 - 1), G, args.g_magic);
        own[p] = mask32[(size_t)nd * W2 + (nd >> 5)] >> (nd & 31);
    }
    bf16x8 qreg[RB][KS];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = min(r0 + rb * 32 + l32, r1 - 1);  // (rows past the end repeat the last one and are never stored)
        const int nd = div_by(r, G, args.g_magic);
        const uint16_t *qp = args.q + ((size_t)(seq * T + nd) * Hq + hk * G + (r - nd * G)) * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qreg[rb][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(qp + ks * 16));
    }
    // the mask row that this lane fetches words of (lane 32 * rb + r: row r of block rb)
    const uint32_t *const mrow = mask32 + (size_t)div_by(min(r0 + (RB == 2 ? lane : l32), r1 - 1), G, args.g_magic) * W2;

    const uint32_t pitch = (uint32_t)Hkv * S::row_bytes;  // bytes between consecutive keys in global memory
    const unsigned char *const kc0 = reinterpret_cast<const unsigned char *>(args.k_cache) + ((size_t)item.kv_start * Hkv + hk) * S::row_bytes;
    const unsigned char *const vc0 = reinterpret_cast<const unsigned char *>(args.v_cache) + ((size_t)item.kv_start * Hkv + hk) * S::row_bytes;
    const unsigned char *const kt0 = reinterpret_cast<const unsigned char *>(args.k_tree) + ((size_t)seq * T * Hkv + hk) * S::row_bytes;
    const unsigned char *const vt0 = reinterpret_cast<const unsigned char *>(args.v_tree) + ((size_t)seq * T * Hkv + hk) * S::row_bytes;
    unsigned char *const ring = smem + wave * S::ring_bytes;

    // LDS layout of a sub-tile: rows of D elements, 16-byte chunks moved about inside a row (or a pair
    // of rows for D = 64) so that neither the 16-byte K reads (a lane a row) nor the transposing V
    // reads (a half-wave four rows) meet on a bank.  K: chunk c of row r sits at c ^ (r & 15)
    // (D = 64: c ^ (r / 2 & 7)); V: 64-byte block b at b ^ (r & 3) (D = 64: b ^ (r / 2 & 1)).
    const int d_row = lane / S::chunks, d_pos = lane % S::chunks;
    auto k_chunk = [&](int i) __attribute__((always_inline)) {  // source chunk of this lane's slot in load i
        return D == 128 ? d_pos ^ d_row ^ ((i & 3) * 4) : d_pos ^ (d_row >> 1) ^ ((i & 1) * 4);
    };
    const int v_chunk = D == 128 ? d_pos ^ (d_row << 2) : d_pos ^ (((d_row >> 1) & 1) << 2);
    constexpr int KV = D == 128 ? 4 : 2;  // distinct K source chunks of a lane
    uint32_t k_off[KV];
#pragma unroll
    for (int i = 0; i < KV; ++i) k_off[i] = __umul24((uint32_t)d_row, pitch) + k_chunk(i) * 16;
    const uint32_t v_off = __umul24((uint32_t)d_row, pitch) + v_chunk * 16;
    auto dma = [&](const unsigned char *base, uint32_t off, unsigned char *dst) __attribute__((always_inline)) {
        asm volatile("" : "+v"(off));
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(base + off),
                                         (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
    };
    auto issue = [&](int i, bool is_k) __attribute__((always_inline)) {
        const int t = t_first + i * NW;
        const bool cache = t < n_cache;
        const int tl = cache ? t : t - n_cache;
        const unsigned char *base = (is_k ? (cache ? kc0 : kt0) : (cache ? vc0 : vt0)) + (uint64_t)(uint32_t)tl * (kSK * pitch);
        const int vmax = min(kSK, (cache ? L : T) - tl * kSK) - 1;
        unsigned char *dst = ring + (i % NS) * S::stage_bytes + (is_k ? 0 : S::tile_bytes);
        if (vmax == kSK - 1) {
#pragma unroll
            for (int u = 0; u < NI; ++u)
                dma(base + (uint32_t)(u * S::rows_per_dma) * pitch, is_k ? k_off[u % KV] : v_off, dst + u * 1024);
        } else {
            // rows past the end repeat the last valid one: the sub-tile holds finite data everywhere
#pragma unroll
            for (int u = 0; u < NI; ++u)
                dma(base, __umul24((uint32_t)min(u * S::rows_per_dma + d_row, vmax), pitch) + (is_k ? k_chunk(u) : v_chunk) * 16,
                    dst + u * 1024);
        }
    };
    // mask words of a tree sub-tile, one per row of the row blocks, fetched into its stage ahead of its
    // keys (a lane past the row blocks repeats a row)
    auto issue_mask = [&](int i) __attribute__((always_inline)) {
        const int t = t_first + i * NW;
        if (t >= n_cache)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(mrow + (t - n_cache)),
                                             (__attribute__((address_space(3))) void *)(ring + (i % NS) * S::stage_bytes + 2 * S::tile_bytes),
                                             4, 0, 0);
    };
    if (n > 0) {
        issue_mask(0);
        issue(0, true);
        issue(0, false);
    }
    if (NS > 1 && n > 1) {
        issue_mask(1);
        issue(1, true);
        issue(1, false);
    }
#pragma unroll
    for (int p = 0; p < PASSES; ++p) asm volatile("" : "+v"(own[p]));
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+v"(qreg[rb][ks]));

    // per-lane LDS read addresses inside a stage
    const uint32_t k_base = lds_base + wave * S::ring_bytes +
                            (D == 128 ? l32 * 256 + ((half ^ (l32 & 15)) << 4) : l32 * 128 + ((half ^ ((l32 >> 1) & 7)) << 4));
    const int lm = lane & 15, dim16 = (lane >> 4) & 1, vrow = 4 * half + (lm >> 2);
    const uint32_t v_base = lds_base + wave * S::ring_bytes + S::tile_bytes + vrow * S::row_bytes +
                            ((D == 128 ? vrow & 3 : (vrow >> 1) & 1) << 6) + 32 * dim16 + 8 * (lm & 3);

    const uint32_t m_base = lds_base + wave * S::ring_bytes + 2 * S::tile_bytes + l32 * 4;

    u32x4 kf[KS];
    u32x2 vf[2][DB][2];
#pragma unroll
    for (int i = 0; i < KS; ++i) kf[i] = (u32x4){0u, 0u, 0u, 0u};
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < DB; ++b) vf[a][b][0] = vf[a][b][1] = (u32x2){0u, 0u};
    floatx16 o[RB][DB];
    floatx4 l_acc[RB];
    float m_ref[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        m_ref[rb] = -INFINITY;
        l_acc[rb] = (floatx4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int v = 0; v < 16; ++v) o[rb][db][v] = 0.0f;
    }
    // selector of the row sums: see attn.hip
    const uint32_t sel_bits = (lane == 0 || lane == 32 || lane == 17 || lane == 49) ? 0x3f803f80u : 0u;
    const bf16x8 sel = __builtin_bit_cast(bf16x8, (u32x4){sel_bits, sel_bits, sel_bits, sel_bits});

    floatx16 s[RB];
    uint32_t p[RB][8], p_low[RB][TWO ? 8 : 1];
    float m_use[RB];
    auto mfma_s = [&](int rb, auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        const bf16x8 a = __builtin_bit_cast(bf16x8, kf[i]);
        if constexpr (i == 0) {
            floatx16 z;
#pragma unroll
            for (int v = 0; v < 16; ++v) z[v] = 0.0f;
            s[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[rb][i], z, 0, 0, 0);
        } else {
            s[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[rb][i], s[rb], 0, 0, 0);
        }
    };
    auto mfma_o = [&](int rb, auto I) __attribute__((always_inline)) {
        constexpr int t2 = decltype(I)::value / DB, db = decltype(I)::value % DB;
        const bf16x8 a = __builtin_bit_cast(
            bf16x8, (u32x4){vf[t2][db][0].x, vf[t2][db][0].y, vf[t2][db][1].x, vf[t2][db][1].y});
        const bf16x8 b = __builtin_bit_cast(bf16x8, (u32x4){p[rb][4 * t2], p[rb][4 * t2 + 1], p[rb][4 * t2 + 2], p[rb][4 * t2 + 3]});
        o[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, o[rb][db], 0, 0, 0);
        if constexpr (db == DB - 1) l_acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sel, b, l_acc[rb], 0, 0, 0);
        if constexpr (TWO) {
            const bf16x8 low = __builtin_bit_cast(
                bf16x8, (u32x4){p_low[rb][4 * t2], p_low[rb][4 * t2 + 1], p_low[rb][4 * t2 + 2], p_low[rb][4 * t2 + 3]});
            o[rb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, low, o[rb][db], 0, 0, 0);
            if constexpr (db == DB - 1) l_acc[rb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(sel, low, l_acc[rb], 0, 0, 0);
        }
    };
    // mask of the block's scores, then its reference: heads of 128 rescale their accumulators only where a score
    // outgrows the reference by more than 2^16 (bf16 weights and fp32 sums carry that as well as 1)
    auto prepare = [&](int rb, bool masked, uint32_t w32) __attribute__((always_inline)) {
        if (masked) {
            const uint32_t w = (w32 >> (4 * half)) & 0x0F0F0F0Fu;  // this lane's keys: 8 * (v / 4) + 4 * half + v % 4
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const uint32_t keep = (uint32_t)__builtin_amdgcn_sbfe((int)w, (v >> 2) * 8 + (v & 3), 1);
                s[rb][v] = __uint_as_float((__float_as_uint(s[rb][v]) & keep) | (0xFF800000u & ~keep));
            }
        }
        float tmax = s[rb][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, s[rb][v]);
        tmax *= scale_log2e;
        if (__builtin_amdgcn_ballot_w64(tmax > m_ref[rb] + kSlack) != 0ull) {
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
            tmax = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
            const float m_new = fmaxf(m_ref[rb], tmax);
            const float alpha = m_ref[rb] > -INFINITY ? __builtin_amdgcn_exp2f(m_ref[rb] - m_new) : 0.0f;
            m_ref[rb] = m_new;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) o[rb][db][v] *= alpha;
            l_acc[rb][0] *= __shfl(alpha, lane & 15, 64);
            l_acc[rb][1] *= __shfl(alpha, 16 + (lane & 15), 64);
        }
        m_use[rb] = m_ref[rb] > -INFINITY ? m_ref[rb] : 0.0f;
    };
    auto weights = [&](int rb, auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        const float e0 = __builtin_amdgcn_exp2f(fmaf(s[rb][2 * i], scale_log2e, -m_use[rb]));
        const float e1 = __builtin_amdgcn_exp2f(fmaf(s[rb][2 * i + 1], scale_log2e, -m_use[rb]));
        p[rb][i] = f2bf_pair(e0, e1);
        if constexpr (TWO) {
            p_low[rb][i] = f2bf_pair(e0 - __uint_as_float(p[rb][i] << 16), e1 - __uint_as_float(p[rb][i] & 0xFFFF0000u));
            asm volatile("" : "+v"(p_low[rb][i]));
        }
        asm volatile("" : "+v"(p[rb][i]));
    };

    auto step = [&](int i) __attribute__((always_inline)) {
        const int t = t_first + i * NW;
        const uint32_t st = (uint32_t)(i % NS) * S::stage_bytes;
        // K(i) has landed: behind it only V(i) and, where there is one, sub-tile i + 1 were requested
        if (NS > 1 && i + 1 < n) vm_wait<3 * NI>(); else vm_wait<NI>();
        static_for<0, KS>([&](auto I) { lds_rd128<0>(kf[decltype(I)::value], (k_base + st) ^ (uint32_t)(decltype(I)::value * 32)); });
        uint32_t w[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)  // (read for cache sub-tiles too, where nobody looks at it)
            asm volatile("ds_read_b32 %0, %1" : "=v"(w[rb]) : "v"(m_base + st + rb * 128) : "memory");
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int u = 0; u < KS; ++u) asm volatile("" : "+v"(kf[u]));
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) asm volatile("" : "+v"(w[rb]));
        // its stage takes the next K
        if (i + NS < n) {
            issue_mask(i + NS);
            issue(i + NS, true);
        }
        const bool tree = t >= n_cache;
        const int valid = min(kSK, (tree ? T : L) - (tree ? t - n_cache : t) * kSK);
        const bool masked = tree || valid < kSK;
        const uint32_t vbits = valid < kSK ? (1u << valid) - 1u : ~0u;
        static_for<0, KS>([&](auto I) { mfma_s(0, I); });
        // V(i) has landed
        if (i + NS < n) vm_wait<(2 * NS - 1) * NI>(); else if (NS > 1 && i + 1 < n) vm_wait<2 * NI>(); else vm_wait<0>();
        static_for<0, 2 * DB>([&](auto I) {
            constexpr int t2 = decltype(I)::value / DB, db = decltype(I)::value % DB;
            lds_rdtr<t2 * 16 * S::row_bytes>(vf[t2][db][0], (v_base + st) ^ (uint32_t)(db * 64));
            lds_rdtr<(t2 * 16 + 8) * S::row_bytes>(vf[t2][db][1], (v_base + st) ^ (uint32_t)(db * 64));
        });
        prepare(0, masked, (tree ? w[0] : ~0u) & vbits);
        if constexpr (RB == 2) {
            static_for<0, 8>([&](auto I) {
                if constexpr (decltype(I)::value % 2 == 0) mfma_s(1, IC<decltype(I)::value / 2>{});
                weights(0, I);
                __builtin_amdgcn_sched_barrier(0);
            });
        } else {
            static_for<0, 8>([&](auto I) { weights(0, I); });
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < DB; ++b) asm volatile("" : "+v"(vf[a][b][0]), "+v"(vf[a][b][1]));
        if (i + NS < n) issue(i + NS, false);  // its stage takes the next V
        if constexpr (RB == 2) {
            prepare(1, masked, (tree ? w[1] : ~0u) & vbits);
            static_for<0, 8>([&](auto I) {
                if constexpr (decltype(I)::value % 2 == 0) mfma_o(0, IC<decltype(I)::value / 2>{});
                weights(1, I);
                __builtin_amdgcn_sched_barrier(0);
            });
        } else {
            static_for<0, 2 * DB>([&](auto I) { mfma_o(0, I); });
        }
        if constexpr (RB == 2) static_for<0, 2 * DB>([&](auto I) { mfma_o(1, I); });
    };
    for (int i = 0; i < n; ++i) step(i);

    // ---- the eight waves' results are combined in LDS (the rings are idle: every request of a wave
    //      has landed before its last sub-tile was worked on) ----
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    float2 *const stat = reinterpret_cast<float2 *>(smem + S::main_bytes);  // (reference, sum) per wave and row
    unsigned char *const stg = smem + wave * S::epi_bytes;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const float lo = __shfl(l_acc[rb][0], l32 & 15, 64), hi = __shfl(l_acc[rb][1], l32 & 15, 64);
        if (half == 0) stat[(wave * RB + rb) * 32 + l32] = make_float2(m_ref[rb], l32 < 16 ? lo : hi);
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                *reinterpret_cast<float4 *>(stg + (rb * 32 + l32) * S::epi_row + (db * 32 + g4 * 8 + half * 4) * 4) =
                    make_float4(o[rb][db][4 * g4], o[rb][db][4 * g4 + 1], o[rb][db][4 * g4 + 2], o[rb][db][4 * g4 + 3]);
    }
    __syncthreads();
    const size_t rows_seq = (size_t)T * Hq;
    const int c8 = (tid % CH) * 8;
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        const int rl = ps * RPP + tid / CH, r = r0 + rl;
        if (rl >= RB * 32) break;  // (more threads than rows)
        float2 ms[NW];
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            ms[w] = stat[w * RB * 32 + rl];
            m = fmaxf(m, ms[w].x);
        }
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        float l = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = ms[w].x > -INFINITY ? __builtin_amdgcn_exp2f(ms[w].x - m) : 0.0f;
            l += f * ms[w].y;
            const float4 *src = reinterpret_cast<const float4 *>(smem + w * S::epi_bytes + rl * S::epi_row + c8 * 4);
            const float4 a = src[0], b = src[1];
            acc[0] = fmaf(f, a.x, acc[0]), acc[1] = fmaf(f, a.y, acc[1]), acc[2] = fmaf(f, a.z, acc[2]), acc[3] = fmaf(f, a.w, acc[3]);
            acc[4] = fmaf(f, b.x, acc[4]), acc[5] = fmaf(f, b.y, acc[5]), acc[6] = fmaf(f, b.z, acc[6]), acc[7] = fmaf(f, b.w, acc[7]);
        }
        const float inv = ((own[ps] & 1u) && l > 0.0f) ? 1.0f / l : 0.0f;
        const int nd = div_by(min(r, r1 - 1), G, args.g_magic);
        const size_t rs = (size_t)nd * Hq + hk * G + (r - nd * G);  // row within the sequence
        if (item.ranges == 1) {
            if (r < r1) {
                uint4 val;
                val.x = f2bf_pair(acc[0] * inv, acc[1] * inv), val.y = f2bf_pair(acc[2] * inv, acc[3] * inv);
                val.z = f2bf_pair(acc[4] * inv, acc[5] * inv), val.w = f2bf_pair(acc[6] * inv, acc[7] * inv);
                *reinterpret_cast<uint4 *>(args.out + (seq * rows_seq + rs) * D + c8) = val;
            }
            continue;
        }
        const size_t slot_row = (size_t)(item.first_slot + item.split) * rows_seq + rs;
        float2 *const lse = args.lse + (size_t)item.first_slot * rows_seq + rs;
        const float lse2 = inv > 0.0f ? m + __builtin_amdgcn_logf(l) : -INFINITY;
        // key ranges that this row does not have (rows of attn_mfma_kernel's whole tiles have more): empty
        if (r < r1 && c8 == 0 && item.split == 0)
            for (int sx = item.splits; sx < item.ranges; ++sx) lse[(size_t)sx * rows_seq] = make_float2(-INFINITY, 1.0f);
        if constexpr (WIDE) {
            if (r < r1) {
                float4 *const dst = reinterpret_cast<float4 *>(static_cast<float *>(args.part) + slot_row * D + c8);
                dst[0] = make_float4(acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
                dst[1] = make_float4(acc[4] * inv, acc[5] * inv, acc[6] * inv, acc[7] * inv);
                if (c8 == 0) lse[(size_t)item.split * rows_seq] = make_float2(lse2, 1.0f);
            }
        } else {
            // an fp16 partial is relative to its row's largest magnitude (see attn.hip)
            float amax = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(acc[e]));
#pragma unroll
            for (int d = CH / 2; d >= 1; d >>= 1) amax = fmaxf(amax, __shfl_xor(amax, d, 64));
            amax *= inv;
            const float scale = (amax > 0.0f && amax < INFINITY) ? amax : 1.0f;
            const float mul = inv / scale;
            if (r < r1) {
                uint4 val;
                val.x = f2h_pair(acc[0] * mul, acc[1] * mul), val.y = f2h_pair(acc[2] * mul, acc[3] * mul);
                val.z = f2h_pair(acc[4] * mul, acc[5] * mul), val.w = f2h_pair(acc[6] * mul, acc[7] * mul);
                *reinterpret_cast<uint4 *>(static_cast<uint16_t *>(args.part) + slot_row * D + c8) = val;
                if (c8 == 0) lse[(size_t)item.split * rows_seq] = make_float2(lse2, scale);
            }
        }
    }
}

}  // namespace ddt
