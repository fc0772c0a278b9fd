// Stand-alone launches of the attention core (see attn_core.h).
#include <mutex>

#include "attn_rows.h"
#include "choose.h"

namespace odb {

template <int DH, int QT, int NW, bool SHARED = false>
__global__ __launch_bounds__(64 * NW) void attn_kernel(AttnArgs a, float sc) {
    __shared__ __attribute__((aligned(16))) char smem[attn_smem_bytes<QT, NW>()];
    attn_wg<DH, QT, NW, SHARED>(a, sc, blockIdx.x, blockIdx.y, smem);
}

// The same with a one-dimensional grid whose ids are mapped so that the gx work items of a head (the row tiles of
// a draft, the drafts of a block: they read the same cached K/V) run on one XCD (id % 8) and share its L2:
// id = xcd + 8 * (item + gx * (head / 8)), head = xcd + 8 * (head / 8).  H must be a multiple of 8.
template <int DH, int QT, int NW, bool SHARED = false>
__global__ __launch_bounds__(64 * NW) void attn_xcd_kernel(AttnArgs a, float sc, int gx) {
    __shared__ __attribute__((aligned(16))) char smem[attn_smem_bytes<QT, NW>()];
    const int xcd = blockIdx.x & 7, j = blockIdx.x >> 3;
    attn_wg<DH, QT, NW, SHARED>(a, sc, j % gx, xcd + 8 * (j / gx), smem);
}

// Many rows per (sequence, head): K/V tiles shared through LDS by all rows of a workgroup (attn_rows.h)
template <int DH, int NW, int QTW, int NS>
static void launch_rows(AttnArgs a, float sc, hipStream_t s) {
    static std::once_flag attr_once;        // once per instantiation: the ring may need more than the default LDS limit
    std::call_once(attr_once, [] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_rows_kernel<DH, NW, QTW, NS>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, attn_rows_smem_bytes<DH, NS>());
    });
    const int tiles_per_seq = a.units_per_seq * a.tiles_per_unit;
    const int chunks = (tiles_per_seq + NW * QTW - 1) / (NW * QTW);
    dim3 grid((a.units / a.units_per_seq) * chunks, a.H);
    // (flattened: the kernel then maps all row chunks of a head to one XCD - 38.9 -> 38.2 us at 1024 rows)
    if (a.H % 8 == 0 && grid.x > 1) grid = dim3(grid.x * grid.y, 1);
    attn_rows_kernel<DH, NW, QTW, NS><<<grid, 64 * NW, attn_rows_smem_bytes<DH, NS>(), s>>>(a, sc);
}

// QT row tiles of one unit per workgroup, its NW waves split the keys.
template <int QT, int NW, bool SHARED = false>
static void launch_split(AttnArgs a, float sc, int items, bool one_xcd, hipStream_t s) {
    if (one_xcd) attn_xcd_kernel<128, QT, NW, SHARED><<<dim3(items * a.H), 64 * NW, 0, s>>>(a, sc, items);
    else if (a.dh == 128) attn_kernel<128, QT, NW, SHARED><<<dim3(items, a.H), 64 * NW, 0, s>>>(a, sc);
    else attn_kernel<64, QT, NW, SHARED><<<dim3(items, a.H), 64 * NW, 0, s>>>(a, sc);
}

void launch_attention(AttnArgs a, hipStream_t s) {
    const float sc = 1.4426950408889634f / sqrtf((float)a.dh);
    if (a.split_tile > 0) {
        // decoded-share step: one row tile per workgroup, block_0 tiles first, then the speculative units'
        launch_split<1, 8, true>(a, sc, a.mt_total, a.dh == 128 && a.H % 8 == 0 && a.mt_total > 1, s);
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
        launch_split<1, 8>(a, sc, a.units * a.tiles_per_unit, c.one_xcd, s);
    } else {
        launch_split<2, 4>(a, sc, a.units * ((a.tiles_per_unit + 1) / 2), c.one_xcd, s);
    }
}

}  // namespace odb
