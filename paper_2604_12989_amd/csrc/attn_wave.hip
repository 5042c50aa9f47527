// Tree attention for little work: few query rows, short caches, heads of 64.
//
// attn_mfma_kernel (attn.hip) shares each key tile between eight waves of 32 query rows, and a call of
// few rows and keys is over before that pays: at 65 nodes of four heads per KV head and 2048 keys it ran
// 4-5 key tiles per workgroup, 1.5 us each, between 4 us of prologue and 2.5 us of epilogue, and left half
// of the compute units idle.  Here every wave walks key sub-tiles of its own: a workgroup owns one block
// of 32 query rows (or two), its eight waves take the 32-key sub-tiles of its key range in turn, each
// into LDS that no other wave touches, so the key loop has no barrier; the eight results are combined in
// LDS at the end.  A key range is cut eight times finer than the partial results that leave the
// workgroup, and there are more, smaller workgroups.
//
// What bounds it: latencies (launch and arguments 1.5 us, first keys 2 us, combining and storing 2 us);
// then a step of eight sub-tiles, 1.2 us at D = 128, mostly waiting for the L2 (every 32 rows read
// all keys: 16 KB per wave and step), which is why attn_mfma_kernel takes over where there are many
// rows per key (attn_plan.hip weighs the two).
// Measured, attention and merge together: D = 128, 17 nodes x 300 keys 14.7 -> 8.6 us, 65 x 2048 20.1 -> 15.2,
// 61 x 3001 21.9 -> 15.7, and launch to launch 14.9 -> 14.2 since a single sequence's entry is requested with the other
// arguments (32 query and 8 KV heads); D = 64, 65 x 2047, 16 and 4 heads 147 (one workgroup
// per node and head on the vector ALUs) -> 11 us.
#include "attn_wave_rows.hpp"

namespace ddt {

template <int D, int RB, bool WIDE>
__global__ __launch_bounds__((WaveShape<D, RB>::threads))
__attribute__((amdgpu_waves_per_eu(WaveShape<D, RB>::waves / 4, WaveShape<D, RB>::waves / 4)))
void attn_wave_kernel(const AttnWaveArgs args)
{
    AttnWaveItem item;
    if (!attn_wave_item(args, (int)blockIdx.x, item)) return;
    attn_wave_rows<D, RB, WIDE>(args, item);
}

template <int D, int RB, bool WIDE>
static bool launch_one(const AttnWaveArgs &args, hipStream_t st)
{
    using S = WaveShape<D, RB>;
    static std::atomic<bool> allowed{false};
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(attn_wave_kernel<D, RB, WIDE>), S::lds_bytes, allowed)) return false;
    DDT_LAUNCH(DDTREE_KERNEL_ATTN, st, (attn_wave_kernel<D, RB, WIDE>), dim3((unsigned)args.grid), dim3(S::threads),
               S::lds_bytes, st, args);
    return true;
}

// (heads of 64 leave fp32 partials only)
bool attn_wave_launch(const AttnWaveArgs &args, int D, int row_blocks, bool wide, hipStream_t st)
{
    if (D == 128) return wide ? launch_one<128, 1, true>(args, st) : launch_one<128, 1, false>(args, st);
    return row_blocks == 2 ? launch_one<64, 2, true>(args, st) : launch_one<64, 1, true>(args, st);
}

}  // namespace ddt
