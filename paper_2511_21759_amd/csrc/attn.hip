// Stand-alone launches of the attention core (see attn_core.h).
#include <mutex>

#include "attn_rows.h"

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

// QT row tiles of one unit per workgroup, its NW waves split the keys.  The work items of a head are kept on one XCD where the heads
// allow it (8.7 -> 8.4 us at 32 rows; 11.8 -> 11.3 us at four drafts, a quarter of the K/V fetches).
template <int QT, int NW, bool SHARED = false>
static void launch_split(AttnArgs a, float sc, int items, hipStream_t s) {
    if (a.dh == 128 && a.H % 8 == 0 && items > 1) attn_xcd_kernel<128, QT, NW, SHARED><<<dim3(items * a.H), 64 * NW, 0, s>>>(a, sc, items);
    else if (a.dh == 128) attn_kernel<128, QT, NW, SHARED><<<dim3(items, a.H), 64 * NW, 0, s>>>(a, sc);
    else attn_kernel<64, QT, NW, SHARED><<<dim3(items, a.H), 64 * NW, 0, s>>>(a, sc);
}

void launch_attention(AttnArgs a, hipStream_t s) {
    const float sc = 1.4426950408889634f / sqrtf((float)a.dh);
    if (a.split_tile > 0) {
        // decoded-share step: one row tile per workgroup, block_0 tiles first, then the speculative units'
        launch_split<1, 8, true>(a, sc, a.mt_total, s);
        return;
    }
    // Three ways to share the work out: one row tile per workgroup of eight waves, two row tiles of a unit per workgroup of four
    // (a K/V tile fetched from L2 then serves 32 rows), or the many-row kernel (it serves 128 or 256 rows, but a wave walks
    // over all keys).  The fewest microseconds by what they measured at heads of 128 channels, n = 32-key tiles and
    // r = workgroups per compute unit:
    //   one tile   8 heads, 8 x 32 rows, n = 19: 8.4 us (many-row: 20.4); 32 heads, 4 x 32 rows, n = 16: 8.6 (two tiles: 10.5),
    //              8 x 32 rows: 17.4, n = 94: 49.6 (steps only: a refresh gains nothing, r = 2.4, n = 10: 17.3, r = 8, n = 32: 72)
    //   two tiles  32 heads, 8 x 32 rows, n = 16: 12.2, n = 94: 40.5; refreshes r = 1.25, n = 10: 15.5, r = 1.7, n = 54: 40,
    //              r = 2.5, n = 20: 31.4, r = 4, n = 32: 55
    //   many rows  8 x 32 rows, n = 16: 19.1, n = 94: 79.5; refreshes n = 10: 13.2, n = 20: 22.6, n = 32: 35, n = 54: 47
    const int tiles_per_seq = a.units_per_seq * a.tiles_per_unit, seqs = a.units / a.units_per_seq;
    const double n = (a.L + 31) / 32;
    const int items1 = a.units * a.tiles_per_unit, items2 = a.units * ((a.tiles_per_unit + 1) / 2);
    const double r1 = items1 * a.H / 256.0, r2 = items2 * a.H / 256.0;
    const double t1 = a.fresh == 0 ? 1e30 : 5.0 + (r1 <= 1.0 ? 0.22 * n : r1 * (2.0 + 0.22 * n));
    const double t2 = (a.fresh > 0 ? 5.0 : 8.0) + (r2 < 1.0 ? 1.0 : r2) * (2.5 + 0.36 * n);
    const int wgs4 = seqs * ((tiles_per_seq + 7) / 8) * a.H, wgs8 = seqs * ((tiles_per_seq + 15) / 16) * a.H;
    // (256 rows per workgroup when that still gives every compute unit a workgroup, else 128)
    const double t3 = wgs8 >= 256 ? 3.0 + (wgs8 + 255) / 256 * 1.3 * n : 3.0 + (wgs4 + 255) / 256 * 0.95 * n;
    if (tiles_per_seq >= 16 && (a.fresh == 0 || a.tiles_per_unit % 2 == 0) && t3 <= t1 && t3 <= t2) {
        if (a.dh == 128) {
            if (wgs8 >= 256) launch_rows<128, 8, 2, 8>(a, sc, s);
            else launch_rows<128, 4, 2, 6>(a, sc, s);
        } else {
            if (wgs8 >= 256) launch_rows<64, 8, 2, 8>(a, sc, s);
            else launch_rows<64, 4, 2, 6>(a, sc, s);
        }
    } else if (t1 <= t2) {
        launch_split<1, 8>(a, sc, items1, s);
    } else {
        launch_split<2, 4>(a, sc, items2, s);
    }
}

}  // namespace odb
