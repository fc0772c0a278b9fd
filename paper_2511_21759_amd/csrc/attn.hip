// Stand-alone launches of the attention core (see attn_core.h).
#include "attn_rows.h"
#include "choose.h"
#include "launch.h"

namespace odb {

// gx work items (QT row tiles of a unit) of H heads, VS workgroups each (choose.h: attention_place)
template <int DH, int QT, int NW, bool SHARED, int VS>
__global__ __launch_bounds__(64 * NW) void attn_kernel(AttnArgs a, float sc, int gx, int one_xcd) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const AttentionPlace p = attention_place(blockIdx.x, gx, VS, one_xcd != 0);
    if (p.head >= a.H) return;              // (the last eight units need not all exist)
    attn_wg<DH, QT, NW, SHARED, VS>(a, sc, p.item, p.head, p.part, smem);
}

// Many rows per (sequence, head): K/V tiles shared through LDS by all rows of a workgroup (attn_rows.h)
template <int DH, int NW, int QTW, int NS>
static void launch_rows(AttnArgs a, float sc, hipStream_t s) {
    allow_lds<attn_rows_kernel<DH, NW, QTW, NS>>(attn_rows_smem_bytes<DH, NS>());      // (the ring may need more than the default LDS limit)
    const int tiles_per_seq = a.units_per_seq * a.tiles_per_unit;
    const int chunks = (tiles_per_seq + NW * QTW - 1) / (NW * QTW);
    dim3 grid((a.units / a.units_per_seq) * chunks, a.H);
    // (flattened: the kernel then maps all row chunks of a head to one XCD - 38.9 -> 38.2 us at 1024 rows)
    if (a.H % 8 == 0 && grid.x > 1) grid = dim3(grid.x * grid.y, 1);
    attn_rows_kernel<DH, NW, QTW, NS><<<grid, 64 * NW, attn_rows_smem_bytes<DH, NS>(), s>>>(a, sc);
}

// QT row tiles of one unit per workgroup, its NW waves split the keys.
template <int DH, int QT, int NW, bool SHARED, int VS>
static void launch_split_as(AttnArgs a, float sc, int items, bool one_xcd, hipStream_t s) {
    constexpr int lds = attn_smem_bytes<DH, QT, NW, VS>();
    allow_lds<attn_kernel<DH, QT, NW, SHARED, VS>>(lds);
    attn_kernel<DH, QT, NW, SHARED, VS><<<attention_grid(items, a.H, VS), 64 * NW, lds, s>>>(a, sc, items, one_xcd);
}
template <int QT, int NW, bool SHARED, int VS>
static void launch_split(AttnArgs a, float sc, int items, bool one_xcd, hipStream_t s) {
    if (a.dh == 128) launch_split_as<128, QT, NW, SHARED, VS>(a, sc, items, one_xcd, s);
    else launch_split_as<64, QT, NW, SHARED, VS>(a, sc, items, one_xcd, s);
}
// One row tile per workgroup.  Where items and heads leave compute units idle the channels of an item go to two or four
// workgroups: a compute unit takes in 16 KiB per 32 keys of 128 channels (8 of K, 8 of V), 278 KB at 512 keys, at not much more than
// 90 GB/s; with a quarter of V it is 10 KiB.  With the merge behind one barrier (attn_core.h): 8.0 -> 6.2 us at 32 heads, 512 keys and
// 32 rows, 8.4 -> 7.6 at 64 rows (two workgroups an item), 7.3 -> 6.1 at 8 heads and 128 rows.
template <bool SHARED>
static void launch_one_tile(AttnArgs a, float sc, int items, bool one_xcd, hipStream_t s) {
    if (items * a.H * 4 <= kComputeUnits) launch_split<1, 8, SHARED, 4>(a, sc, items, one_xcd, s);
    else if (items * a.H * 2 <= kComputeUnits) launch_split<1, 8, SHARED, 2>(a, sc, items, one_xcd, s);
    else launch_split<1, 8, SHARED, 1>(a, sc, items, one_xcd, s);
}

void launch_attention(AttnArgs a, hipStream_t s) {
    const float sc = 1.4426950408889634f / sqrtf((float)a.dh);
    if (a.split_tile > 0) {
        // decoded-share step: one row tile per workgroup, block_0 tiles first, then the speculative units'
        launch_one_tile<true>(a, sc, a.mt_total, a.dh == 128 && a.H % 8 == 0 && a.mt_total > 1, s);
        return;
    }
    const AttentionChoice c = attention_choice(a.dh, a.H, a.L, a.fresh > 0, a.units, a.units_per_seq, a.tiles_per_unit);
    if (c.way == 3) {
        if (a.dh == 128) {
            if (c.rows8) launch_rows<128, 8, 2, 8>(a, sc, s);
            else launch_rows<128, 4, 2, 6>(a, sc, s);
        } else {
            if (c.rows8) launch_rows<64, 8, 2, 8>(a, sc, s);
            else launch_rows<64, 4, 2, 6>(a, sc, s);
        }
    } else if (c.way == 1) {
        launch_one_tile<false>(a, sc, a.units * a.tiles_per_unit, c.one_xcd, s);
    } else {
        launch_split<2, 4, false, 1>(a, sc, a.units * ((a.tiles_per_unit + 1) / 2), c.one_xcd, s);
    }
}

}  // namespace odb
