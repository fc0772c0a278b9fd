// Which kernel variant a launch takes, as plain functions of its sizes (no HIP: they can be tried on the CPU).
#pragma once
#include <math.h>
#include <stddef.h>

namespace odb {

constexpr int kComputeUnits = 256;

// Attention of a step (`step`) or a refresh over L cached positions: `units` drafts or sequences of tiles_per_unit 16-row tiles,
// units_per_seq of them per sequence.  Three ways to share the work out: one row tile per workgroup of eight waves (1; steps only:
// a refresh gains nothing), two row tiles of a unit per workgroup of four (2: a K/V tile fetched from L2 then serves 32 rows), or
// the many-row kernel (3: it serves 128 or, with rows8, 256 rows, but a wave walks over all keys).
//
// A first choice by rows stands - many rows from 16 row tiles per sequence, else two tiles from 128 such workgroups on - unless
// the model below puts another way 10 % under it (20 % for a refresh, where its error is larger).  The model was fitted to 2760 measured calls (4 to 64 heads of 64 and 128
// channels, 160 to 3040 keys, steps of 16 to 2048 rows, refreshes of 48 to 3000 positions): rounds of 256 workgroups, each a fixed
// time and a time per 32-key tile (n of them), beside the K/V bytes that the XCDs fetch at 6.6 TB/s - every XCD that runs
// a part of a head fetches that head - as the root of both squares.  What it picks is 0.6 % off the fastest on average (the
// first choice alone: 17 %; a model without rounds and fetches: 4.3 %, and up to twice the first choice's time).  Microseconds
// measured, one tile / two tiles / many rows:
//   32 heads of 128, L 544: 4 x 32 rows 7.6 / 10.3 / -, 6 x 32 13.0 / 10.6 / -, 8 x 32 13.5 / 10.8 / 18.1
//   12 heads of 128, L 1056, 4 x (4 x 32) rows 33.8 / 19.7 / -; 8 heads of 128, L 544, 8 x 32 rows 7.1 / 10.6 / 17.8
//   28 heads of 128, L 3040, 2 x (5 x 64) rows 128 / 123 / 78; 16 heads of 64, L 1056, 2 x (8 x 64) rows 19.8 / 15.9 / 26.2
//
// one_xcd: the workgroups of a head go to one XCD, which then fetches that head's K/V alone (8.7 -> 8.4 us at 32 rows of 32
// heads; 11.8 -> 11.3 at four drafts).  Not in a refresh: the O projection behind it, whose K slices lie on other XCDs than
// the heads that wrote them, loses more (200 rows of 16 heads: attention 8.0 -> 7.1 us, O 10.0 -> 12.7).
struct AttentionChoice { int way; bool rows8, one_xcd; };
inline AttentionChoice attention_choice(int dh, int H, int L, bool step, int units, int units_per_seq, int tiles_per_unit) {
    const int per_seq = units_per_seq * tiles_per_unit, seqs = units / units_per_seq;
    const int items1 = units * tiles_per_unit, items2 = units * ((tiles_per_unit + 1) / 2);
    const int wgs4 = seqs * ((per_seq + 7) / 8) * H, wgs8 = seqs * ((per_seq + 15) / 16) * H;
    const bool wide = dh == 128, heads8 = H % 8 == 0, may_rows = per_seq >= 16 && (!step || tiles_per_unit % 2 == 0);
    const bool rows8 = wgs8 >= kComputeUnits;       // 256 rows per workgroup when that still gives every compute unit one, else 128
    const double n = (L + 31) / 32, kv_us = n * 32 * dh * 4 * seqs * H / 6.6e6;
    auto us = [&](int wgs, int wgs_per_head, bool one_xcd, double base, double round, double tile) {
        const double walk = base + (wgs + kComputeUnits - 1) / kComputeUnits * (round + tile * n);
        const double fetch = kv_us * (one_xcd ? 1 : wgs_per_head < 8 ? wgs_per_head : 8);
        return sqrt(walk * walk + fetch * fetch);
    };
    double t[4] = {0, 1e30, 1e30, 1e30};
    if (step) t[1] = wide ? us(items1 * H, per_seq, heads8 && items1 > 1, 0.9, 3.7, 0.173) : us(items1 * H, per_seq, false, 3.6, 1.0, 0.076);
    t[2] = wide ? us(items2 * H, items2 / seqs, step && heads8 && items2 > 1, step ? 0.5 : 1.7, step ? 5.2 : 3.9, step ? 0.28 : 0.27)
                : us(items2 * H, items2 / seqs, false, step ? 4.5 : 4.4, step ? 0.8 : 0.7, step ? 0.166 : 0.14);
    if (may_rows)
        t[3] = rows8 ? us(wgs8, (per_seq + 15) / 16, heads8, wide ? 5.8 : 4.1, wide ? 6.9 : 3.0, wide ? 1.12 : 0.81)
                     : us(wgs4, (per_seq + 7) / 8, heads8, wide ? 0.0 : 4.8, wide ? 6.0 : 0.0, wide ? 0.73 : 0.6);
    int way = may_rows ? 3 : !step || (tiles_per_unit >= 2 && items2 * H >= 128) ? 2 : 1;
    t[way] *= step ? 0.9 : 0.8;
    for (int w = 1; w <= 3; w++)
        if (t[w] < t[way]) way = w;
    return AttentionChoice{way, rows8, step && wide && heads8 && (way == 1 ? items1 : items2) > 1};
}

// Item, head and channel part of workgroup `id` of an attention launch of gx items per head and `parts` workgroups per item.  Ids are
// dealt over the XCDs (id % 8), and workgroups that read the same cached K/V should share an L2.  one_xcd (a multiple of eight heads): all
// of a head, id = xcd + 8 * (part + parts * (item + gx * (head / 8))), head = xcd + 8 * (head / 8).  Else those of an item, whose keys all
// of them read: id = u % 8 + 8 * (part + parts * (u / 8)), u = item + gx * head; heads beyond the last have nothing to do.
// With the parts of an item side by side, on XCDs of their own, they fetched K from memory as often: 28 heads, 3000 keys, 64 rows in two
// parts 38.8 us, now 27.6 (one part 31.3); 32 rows in four 33.0, 16.7 (20.5); 32 heads, 2000 keys, 16 rows in four 15.1, 11.8 (15.1).
struct AttentionPlace { int item, head, part; };
constexpr AttentionPlace attention_place(int id, int gx, int parts, bool one_xcd) {
    const int xcd = id & 7, j = id >> 3, x = j / parts, u = one_xcd ? x : xcd + 8 * x, q = u / gx;
    return AttentionPlace{u - q * gx, one_xcd ? xcd + 8 * q : q, j - x * parts};
}
constexpr int attention_grid(int gx, int H, int parts) { return 8 * parts * ((gx * H + 7) / 8); }

// K slices of the tile kernel (gemm_tile.h), which need not divide K; `room` bounds the bytes of partial sums.
//
// The count with the smallest time by the model below; up to 128 rows it has to lie 2 % under the largest power of two that divides
// K and fits one round of workgroups.  The model was fitted to 6400 launches measured inside refreshes (m_tiles 3 to 188, d from 512 to 8192; 7 % off
// at the root mean square): a launch lasts as long as its fullest compute unit has blocks and k-tiles of the LONGEST slice, up
// to 128 rows at least as long as the weight stream; then there is the epilogue on the few compute units that own a block, or
// the merge pass.  It matters too on which of the eight XCDs, which take the workgroups in turn, blocks meet: slices that share
// no factor with eight make every XCD read all of A, blocks per row of blocks that share none make every XCD that works
// on a column of blocks read its weights, and where there are few of them, counts that bring the workgroups of one slice
// together on one XCD cost about a microsecond.
// Over 858 sizes that take the tile kernel it is 2.8 % faster than the power of two on average and slower by more than 3 % at 12;
// a model with mean slices and without the XCDs was 1.7 % faster and slower by more than 3 % at 108, up to 28 %.
// Microseconds with the merge pass, by slices: 1232 rows, N 1280, K 5120: 4 29.3, 5 37.6; 144 rows, N 3584, K 18944: 8 44.8,
// 9 50.8; 640 rows, N 4096, K 12288: 2 96.7, 3 76.3; 128 rows, N 4096, K 4096: 5 20.1, 6 19.1, 8 20.4.
enum class TileEpilogue { qkv, swiglu, resid };
inline int tile_slices(TileEpilogue epi, int m_tiles, int n_tiles, int k_tiles, size_t room, double *time = nullptr) {
    const bool wide = m_tiles > 8;                          // two n-tiles per wave
    const int m_blocks = (m_tiles + 7) / 8, n_blocks = (n_tiles + (wide ? 15 : 7)) / (wide ? 16 : 8), blocks = m_blocks * n_blocks;
    const double a_mb = m_tiles * (double)k_tiles / 1024, w_mb = n_tiles * (double)k_tiles / 1024, out_mb = m_tiles * (double)n_tiles / 1024;
    auto fits = [&](int ks) { return ks == 1 || (k_tiles / ks >= 8 && (size_t)ks * m_tiles * n_tiles * 1024 <= room); };
    auto gcd8 = [](int x) { return x % 8 == 0 ? 8 : x % 4 == 0 ? 4 : x % 2 == 0 ? 2 : 1; };
    auto least = [](int a, int b) { return a < b ? a : b; };
    auto us = [&](int ks) {
        const int rounds = (blocks * ks + kComputeUnits - 1) / kComputeUnits, longest = (k_tiles + ks - 1) / ks;
        const int gk = gcd8(ks), gx = gcd8(n_blocks * ks);
        if (!wide) {
            const double loop = rounds * (0.22 * longest + 0.93) + 0.05 * a_mb * least(n_blocks, 8 / gk) + 0.03 * w_mb;
            return (loop > 0.18 * w_mb ? loop : 0.18 * w_mb) + (ks == 1 ? 7.1 * rounds : 7.15 + 0.5 * ks * out_mb);
        }
        const double loop = rounds * (0.36 * longest + 0.42) + 0.05 * w_mb * least(m_blocks, 8 / gx);
        if (ks == 1) return loop + rounds * (epi == TileEpilogue::qkv ? 17.5 : epi == TileEpilogue::swiglu ? 10.5 : 10.4);
        const double merge = epi == TileEpilogue::qkv ? 15.1 : epi == TileEpilogue::swiglu ? 14.1 : 7.2, sums = ks * out_mb;
        const double crowd = (gx == 8 ? 1.66 / n_blocks : 0) + (blocks * ks > 230 ? 0.44 : 0);
        return loop + merge + 0.302 * sums + (sums > 26 ? 0.1 * (sums - 26) : 0) + crowd;      // (beyond 26 MB they leave the L2s)
    };
    int best = 1;
    while (blocks * best * 2 <= kComputeUnits && k_tiles % (best * 2) == 0 && fits(best * 2)) best *= 2;
    double best_us = (wide ? 1.0 : 0.98) * us(best);
    for (int ks = 1; ks <= 16; ks++)
        if (fits(ks) && us(ks) < best_us) { best = ks; best_us = us(ks); }
    if (time) *time = us(best);
    return best;
}

// Gate/up of 129 to 256 rows: n-tiles per group of the streaming kernel in blocks of 64 rows, or 0 where the LDS-ring or tile kernel
// runs.  Up to 512 n-tiles (d_ff 4096) the streaming kernel wins as long as its groups and row blocks make one round of
// workgroups, or K is short; a second round costs it a whole pass over K.  us at 144 / 256 rows, streaming against tile kernel:
// d 1024, d_ff 3072 (one round) 10.8 / 11.1 and 22.5 / 23.9; d 3072, d_ff 3072 (one) 21.9 / 21.9 and 27.1 / 29.6; d 1280,
// d_ff 4096 (two) 20.2 / 26.6 and 24.1 / 26.7; d 2048, d_ff 4096 (two) 28.5 / 35.6 and 28.6 / 31.4; d 4096, d_ff 4096 (two)
// 48.9 / 63.4 and 35.4 / 42.8; with groups of three d 2048, d_ff 2048 (two) 17.1 / 22.7 and 23.9 / 26.3, d 3072 23.1 / 31.4
// and 25.1 / 27.8.
inline int swiglu_row_block_group(int m_tiles, int n_tiles, int k_tiles) {
    if (m_tiles <= 8 || m_tiles > 16 || n_tiles > 2 * kComputeUnits) return 0;
    const int group = n_tiles <= kComputeUnits ? 3 : 6, wgs = (n_tiles + group - 1) / group * ((m_tiles + 3) / 4);
    return wgs <= kComputeUnits || k_tiles <= (group == 3 ? 80 : 40) ? group : 0;
}

// QKV and gate/up from 33 rows on in small blocks of rows on the streaming kernel: row tiles (2 or 4) and n-tiles of a workgroup, or
// mt = 0 where another kernel runs.  `else_tile`: the tile kernel and its merge pass would take the call, not a streaming kernel of
// wider row blocks.
//
// 32 rows and the fewest n-tiles that make one round of workgroups.  Beyond four of them: at 65 to 128 rows 64 rows and three or four
// n-tiles while that is one round, else 32 rows and four, two workgroups to a compute unit, as long as those of a
// compute unit together take in little enough (KiB: (2 row + 4 n-tiles) x K each; it takes in about 80 GB/s): a wider row block
// needs fewer reads, but the small ones hide each other's prologue and epilogue.  A streaming kernel of one round of wide row blocks wins
// as soon as the small ones do not fit the chip together.  Fitted over eleven widths, 48 to 1024 rows, models of up to 600 MB so that the weights come
// from HBM.  Microseconds a layer:
//   QKV, d 256, 512 rows: 4.8, tile kernel 21.2; d 1024, 320 rows 9.2, tile 24.6; d 1536, 144 rows 10.7, tile 25.7; d 2048, 320 rows
//   23.3, tile 31.2; d 1024, 96 rows 6.0, 96-row blocks 9.0; d 2560, 128 rows 16.4, slab kernel 20.8
//   gate/up, d 1024, d_ff 3072, 112 rows 7.5, the same in 32-row blocks 8.3; d 1536, d_ff 4096, 128 rows 10.7, two rounds of three
//   n-tiles 20.0; d 2560, d_ff 6912, 192 rows 52.4 (2430 KiB), tile 41.2
struct RowBlock { int mt, ng; };
inline RowBlock row_block(int m_tiles, int n_tiles, int k_tiles, bool else_tile) {
    const int blocks = (m_tiles + 1) / 2;
    for (int ng = 1; ng <= 3; ng++)
        if ((n_tiles + ng - 1) / ng * blocks <= kComputeUnits) return RowBlock{2, ng};
    if (m_tiles > 4 && (n_tiles + 3) / 4 * blocks <= kComputeUnits) return RowBlock{2, 4};
    if (m_tiles > 4 && m_tiles <= 8)
        for (int ng = 3; ng <= 4; ng++)
            if ((n_tiles + ng - 1) / ng * 2 <= kComputeUnits) return RowBlock{4, ng};
    const int wgs = (n_tiles + 3) / 4 * blocks;
    const double kib = wgs * 6.0 * k_tiles / kComputeUnits;
    const bool small = m_tiles <= 4 ? kib <= 460 : m_tiles <= 8 ? kib <= 600 : else_tile ? kib <= 1800 : wgs <= 2 * kComputeUnits;
    return small ? RowBlock{2, 4} : RowBlock{0, 0};
}

// Gate/up beyond 128 rows in blocks of 96 rows and six n-tiles on the streaming kernel: one round of workgroups instead of the tile
// kernel, where the small blocks above would take in more than 1200 KiB (us: d 2048, d_ff 5632, 192 rows 20.5, small blocks 31.0, tile
// 34.0; d 3072, d_ff 3072, 384 rows 23.1, 38.1, 36.0; d 1536, d_ff 4096, 144 rows 15.4, 15.0, 25.3), and instead of the LDS-ring
// kernel over a short K (d 1024, d_ff 3072, 320 to 384 rows 11.9, 13.7).
inline bool swiglu_wide_block(int m_tiles, int n_tiles, int k_tiles, bool else_tile) {
    if (m_tiles <= 8 || (n_tiles + 5) / 6 * ((m_tiles + 5) / 6) > kComputeUnits) return false;
    return else_tile ? (n_tiles + 3) / 4 * ((m_tiles + 1) / 2) * 6.0 * k_tiles / kComputeUnits > 1200 : m_tiles > 16 && m_tiles <= 24 && k_tiles <= 32;
}

// O and down from 33 rows on in blocks with all of K in a workgroup: row tiles (2 or 4) and n-tiles, or mt = 0 where K is split.
//
// Up to 128 rows the smallest of 32 x 16, 32 x 32 and 64 x 32 that makes one round, beyond 64 columns (the sums of squares cover as
// many) and 32 rows, else 64, counted per XCD, which takes whole columns of blocks.  A second and third round still pay over a
// short K.  Splitting K costs an exchange or a merge pass, about 5 us; blocks of all of K take in (mt + ng) x K KiB each, which
// is what they lose by beyond the limits.  Measured as above, us a layer:
//   d 1024: O of 128 rows 4.4, K split 6.5; of 333 rows 5.5, 11.3; of 1008 rows 8.2, 14.5; down (d_ff 3072) of 128 rows 7.9, 8.1; of 64
//   rows 8.2, 7.3 with K split in the kernel; of 192 rows 12.0, 11.5; of 333 rows 9.5, 14.3;
//   d 4096: O of 128 rows 17.1, 18.9, of 256 rows 22.5, 26.3, of 48 rows 12.2, 11.8 with K split in the kernel;
//   down, d 1024, d_ff 8192, 144 rows 17.4, 14.1; d 1280, d_ff 5120, 192 rows 17.4, 15.7; d 2560, d_ff 6912, 192 rows 23.4, 22.3
inline RowBlock resid_block(int m_tiles, int n_tiles, int k_tiles) {
    if (m_tiles <= 2 || (m_tiles <= 16 && n_tiles <= 64 && k_tiles > (m_tiles <= 8 ? 96 : 64))) return RowBlock{0, 0};      // (the K-split kernel takes these)
    if (m_tiles <= 8) {
        const RowBlock shapes[3] = {{2, 1}, {2, 2}, {4, 2}};
        for (const RowBlock &b : shapes)
            if ((n_tiles + b.ng - 1) / b.ng * ((m_tiles + b.mt - 1) / b.mt) <= kComputeUnits)
                return (b.mt + b.ng) * k_tiles <= (m_tiles > 4 ? 800 : b.ng == 1 ? 240 : 400) ? b : RowBlock{0, 0};
        return RowBlock{0, 0};
    }
    const int columns = (n_tiles / 4 + 7) / 8, two = (m_tiles + 1) / 2 * columns, four = (m_tiles + 3) / 4 * columns, round = kComputeUnits / 8;
    if (two <= round && k_tiles <= 128) return RowBlock{2, 4};
    if (four <= round && k_tiles <= 128) return RowBlock{4, 4};
    if (k_tiles <= 64 && two <= 3 * round) return RowBlock{2, 4};
    // (two rounds over a longer K only where every XCD has as many columns: twelve of them at d 768, down of 2048 rows 26.8 us, tile kernel 22.3)
    if (k_tiles <= (n_tiles % 32 == 0 ? 64 : 48) && four <= 2 * round) return RowBlock{4, 4};
    return RowBlock{0, 0};
}

// O of a step of 65 to 128 rows in two blocks of rows, both of which read the weights, through ordinary loads unless that costs the
// attention more: where the K/V that a step reads fit the memory-side cache but not with O's weights beside them, the weights
// are read past it.  Steps at d 4096 of 128 and 96 rows, weights past the cache against through it: 12 layers, 1024 keys (201 MB of
// K/V, 403 of O) 0.986 and 0.992; 8 layers, 1024 keys 0.991, 0.997; 24 layers, 512 keys 0.991, 1.003; 4 layers, 2048 keys 0.983, 0.987; where K/V do not
// fit, 32 layers, 512 keys (268 MB) 1.003, 1.012, 16 layers, 2048 keys 1.008, 1.008; where both fit, 4 layers, 512 keys 1.03.
// At 8 layers and 1024 keys the attention takes 9.8 us a layer so, 12.4 with the weights in its way; O itself 17.1 instead of 16.7.
inline bool weights_past_cache(double kv_bytes, double weight_bytes) {
    const double cache = 250e6;            // (256 MiB; activations and partial sums pass through it too)
    return kv_bytes <= cache && kv_bytes + weight_bytes > cache;
}

// O and down of up to 32 rows whose K is split over four workgroups: n-tiles of a block, or 0 where a workgroup has all of K (3 KiB a
// k-tile for each of its rows and columns; the same line as for more rows above) or K cannot be split.  As many blocks as make one round:
// down at d 1024, d_ff 3072 on 64 workgroups with all of K 10.4 us, on 256 with a quarter 7.1.
inline int few_rows_split(int m_tiles, int n_tiles, int k_tiles) {
    if (m_tiles > 2 || 3 * k_tiles <= 240 || k_tiles % 32 != 0 || n_tiles > kComputeUnits) return 0;
    return n_tiles <= kComputeUnits / 4 ? 1 : n_tiles <= kComputeUnits / 2 ? 2 : 4;
}

// Up to 32 rows whose K cannot be split so: where the n-tiles make a second round of workgroups, which is not full or over a longer K, the
// tile kernel and its merge pass.  Packed drafts come here from three and more row tiles, which ran there before.  us, all of K in a workgroup
// and tile kernel: down at d 5120, d_ff 13824 49.9, 31.2; d 4352, d_ff 11776 41.8, 26.1; d 8192, d_ff 22016 85.9, 71.2; O at d 4352 21.8,
// 15.7; d 5120 21.2, 18.8; d 6144 25.2, 22.3; d 8192, two full rounds, 32.8, 35.4; one round: down at d 3584, d_ff 9728 20.4, 21.2.
inline bool few_rows_tile(int n_tiles, int k_tiles) {
    return n_tiles > kComputeUnits && (k_tiles > n_tiles || n_tiles < 2 * kComputeUnits);
}

// Whether a step packs its drafts' rows densely (api.hip): row tiles packed, and with every draft in tiles of its own.  Two tiles fewer at
// least, as the kernels of few rows take two at a time, and enough of them to pay for the places looked up row by row and for
// V written key by key.
// Microseconds a step, padded and packed: 8B shape, 8 layers, 4 -> 2 tiles 1015 and 882, 8 -> 6 1250 and 1164, 10 -> 8 1642 and 1277,
// 16 -> 13 1718 and 1677, 32 -> 14 2735 and 1850; 1k-wide model 8 -> 6 299 and 298, 12 -> 10 355 and 328; before this line 10 -> 9
// 1578 and 1562 (1k 322 and 323), 128 -> 120 7738 and 7723.
inline bool dense_rows_pay(int dense, int padded) {
    if ((dense + 1) / 2 >= (padded + 1) / 2) return false;
    return padded > 8 ? dense <= 8 || 20 * dense <= 17 * padded : 4 * dense <= 3 * padded;
}

// QKV on the slab kernel (gemm_slab.h): n-tiles per workgroup, or 0 where another kernel runs.  One row block (97 to 128 rows): three
// while that is one round of workgroups, beyond it six, which is one round up to twice as far and half as many reads of A
// (us at 128 rows with three and with six: d 4096 31.1 and 40.2, d 5120 68.7 and 51.1, d 8192 112.5 and 83.7, where the
// streaming kernel took 105.3); 20.7 at d 2560 against 22.6 in groups of two there.  Up to 384 n-tiles the streaming kernel in blocks of
// 64 rows and three n-tiles makes one round (d 2048: 13.4 us against 17.1).  Two row blocks: 44 us at 160 to 256 rows of the 8B shape on 2 x 128 workgroups, against 54 to 58 us
// on the tile kernel and its merge pass and 50 us in 192 blocks of 128 x 128.
inline int qkv_slab_group(int m_tiles, int n_tiles) {
    if (m_tiles > 6 && m_tiles <= 8 && n_tiles > 384) return n_tiles <= 3 * kComputeUnits ? 3 : 6;
    return m_tiles > 8 && m_tiles <= 16 && n_tiles > 384 && n_tiles <= 768 ? 6 : 0;
}

// Block shape for the LDS-ring kernel - mbt 16-row tiles by 64 * wn columns - or wn = 0 when the tile kernel
// should run instead.  With T blocks on 256 compute units a launch takes ceil(T / 256) block-times, and a
// block-time shrinks more slowly than the block (the k-step is bound by its barrier and operand delivery as
// much as by its MFMAs).  In units of the 256 x 256 block at K = 4096: 256-row blocks of 192 / 128 columns 0.87 / 0.68;
// 128-row blocks of 256 / 192 / 128 columns 0.66 / 0.60 / 0.46 (measured with one group of waves; with two, in us at 96 to
// 190 blocks: 88 for the 256 x 256 block, 0.86 / 0.72 and 0.69 / 0.64 / 0.48).  The
// shape with the smallest rounds x block-time wins among those whose block slots are at least `least` useful (a
// ragged last block counts by its real rows); below that for every shape the 128-row tile kernel wins
// (measured at 640 rows).  The 128-row blocks serve shapes that would leave compute units idle: QKV at 512 rows
// (256 blocks of 128 x 192 instead of 192 of 256 x 128: 83 -> 69 us), every wide projection at 640 rows (five row
// blocks that fit exactly: refresh 14.7 -> 13.0 ms), the 256-row step (7.6 -> 7.2 ms).  144 to 176 rows count as 192: both
// kernels run two row blocks for them, gate/up at 160 rows takes 73.9 us on the tile kernel and 65 us in 128 x 192 blocks.
//
// per_xcd: the launch gives a column of blocks to one XCD, so a round is 32 blocks of the fullest XCD: 11 x 22 blocks of
// 128 x 192 at 1300 rows of N = 4096 are 33 on six of the XCDs, two rounds and 97 us (the tile kernel: 61), while 10 x 22
// at 1232 rows take 56 us (67 and 62 on the tile kernel).  Up to K = 1024 a shape needs to be 45 % useful only: the block-times are
// short and the tile kernel pays its merge pass all the same (K 768, N 2304: 15.1 us in 128 x 128 blocks at 1008 rows and 20.6
// in 128 x 192 at 1536, 28.8 and 29.1 on the tile kernel; K 768, N 4096, 512 rows: 11.2 and 21.7).
struct BigChoice { int mbt, wn; };
inline BigChoice big_choice_by(int m, int n_tiles, bool per_xcd, double least) {
    BigChoice best{16, 0};
    if (m <= 8 || n_tiles < 32) return best;
    const double m_tiles = m < 12 ? 12 : m;     // (see above)
    const double rel16[5] = {0, 0, 0.68, 0.87, 1.0}, rel8[5] = {0, 0, 0.46, 0.60, 0.66};
    double best_cost = 0;
    for (int mbt = 16; mbt >= 8; mbt -= 8)
        for (int wn = 4; wn >= 2; wn--) {
            const int mb = (m + mbt - 1) / mbt, nb = (n_tiles + 4 * wn - 1) / (4 * wn);
            const int rounds = per_xcd ? (mb * ((nb + 7) / 8) + kComputeUnits / 8 - 1) / (kComputeUnits / 8) : (mb * nb + kComputeUnits - 1) / kComputeUnits;
            const double useful = (m_tiles / (double)mbt) * (n_tiles / (4.0 * wn)) / ((double)rounds * kComputeUnits);
            const double cost = rounds * (mbt == 16 ? rel16[wn] : rel8[wn]);
            // (a 128-row shape has to promise 5 % over the best 256-row one: the unit times are measurements)
            if (useful >= least && (best.wn == 0 || cost < best_cost * (mbt == 8 && best.mbt == 16 ? 0.95 : 1.0) - 1e-9)) {
                best = BigChoice{mbt, wn};
                best_cost = cost;
            }
        }
    return best;
}
inline BigChoice big_choice(int m, int n_tiles, int k_tiles) { return big_choice_by(m, n_tiles, true, k_tiles <= 32 ? 0.45 : 0.65); }
// The LM head by its own numbers: as many statistics per row as before, which decide with the rest whether a step fits the fixed area.
inline BigChoice lm_block_choice(int m, int n_tiles) { return big_choice_by(m, n_tiles, false, 0.7); }

// QKV in small blocks of rows (row_block): from 33 rows on, up to 128 rows where the slab kernel does not run or 64 rows and four n-tiles
// make one round (up to 512 n-tiles), beyond where no block of the LDS-ring kernel is chosen.
inline RowBlock qkv_row_block(int m_tiles, int n_tiles, int k_tiles) {
    const int slab = qkv_slab_group(m_tiles, n_tiles);
    if (m_tiles <= 2) return RowBlock{0, 0};
    if (m_tiles <= 8) return slab == 0 || n_tiles <= 512 ? row_block(m_tiles, n_tiles, k_tiles, false) : RowBlock{0, 0};
    const bool narrow = n_tiles <= kComputeUnits && m_tiles <= 16;
    return slab == 0 && (narrow || !big_choice(m_tiles, n_tiles, k_tiles).wn) ? row_block(m_tiles, n_tiles, k_tiles, !narrow) : RowBlock{0, 0};
}

// What runs where big_choice decided until the blocks below were measured: a block shape of the LDS-ring kernel - mbt x 16 rows by
// 64 * wn columns, its last round split over `ks` workgroups a block - or the tile kernel (wn = 0).
//
// `now` stands - the shape big_choice picks, or the tile kernel - unless another block promises 4 % by the model of big_us, or more with
// its last round split.  Blocks of 192 and 320 rows serve counts of rows that 128 and 256 divide badly (8B shape: gate/up of 608 rows in
// 256 blocks of 320 x 192 135 -> 111 us, of 320 rows in 192 x 192 124 -> 69, QKV of 1408 rows in 320 x 256 194 -> 151, down of 3008
// rows in 192 x 256 311 -> 281).  Splitting K in the blocks of the last, half empty round fills it (256 x 256 blocks: down of 2048 rows
// 128 blocks on 256 compute units 240 -> 202 us; QKV of 2048 rows one and a half rounds 220 -> 207).  The gain is less than the
// idle units suggest, as the others run at a lower clock the more of them multiply; the exchange costs 7 us a block of 256 x 256.
// Launches timed one by one, the chip idle between them, flatter the split: inside a call, behind other kernels, it takes 5 to 20 % more
// than the model against other blocks, most for gate/up.  What it has to promise there: split_margin.
// Over 222 measured sizes (d 1024 to 4096, 176 to 3008 rows) the launches take 0.956 of the time on average, 0.951 with the best of
// these blocks everywhere.  Splits of other shapes would add 0.4 %.
struct BigPlan { int mbt, wn, ks; };
constexpr int kSplitMbt = 16, kSplitWn = 4;                     // the shape whose last round may be split
// blocks of the fullest XCD, which takes whole columns of blocks and runs kXcdUnits of them at a time
constexpr int kXcdUnits = kComputeUnits / 8;
inline int big_per_xcd(int mbt, int wn, int m, int n) { return (m + mbt - 1) / mbt * (((n + 4 * wn - 1) / (4 * wn) + 7) / 8); }
// Microseconds of a launch, fitted to 4180 measured (6 % off at the root mean square): a block's time by shape and K when all
// compute units work; the last round between 0.57 and 1 of that by its fill; 3.4 a round, the epilogue (under the next round by half), the
// exchange of a split block.  A single row block of 192 rows takes 8 % more: half as many workgroups as two of 128 stream the weights
// (gate/up of 144 to 192 rows in calls, 192 x 192 and 128 x 192: d 4096, d_ff 12288 63.9 and 61.6 us, d 3584, d_ff 9728 53.0 and 49.2).
inline double big_us(TileEpilogue epi, int mbt, int wn, int ks, int m, int n, int k) {
    const double at4096[4][3] = {{43.9, 59.6, 70.9}, {76.0, 71.5, 93.8}, {74.6, 98.9, 112.1}, {98.5, 114.1, 143.3}};    // mbt 8 .. 20, wn 2 .. 4
    const int per = big_per_xcd(mbt, wn, m, n), all = (m + mbt - 1) / mbt * ((n + 4 * wn - 1) / (4 * wn));
    const double area = mbt * wn / 64.0, full = at4096[mbt / 4 - 2][wn - 2] * k / 128 * (mbt == 12 && m <= 12 ? 1.08 : 1);
    const double out = (epi == TileEpilogue::swiglu ? 0 : epi == TileEpilogue::qkv ? 13.2 : 14.3) * area;
    const int whole = ks > 1 ? per / kXcdUnits : (per + kXcdUnits - 1) / kXcdUnits - 1;
    const int rounds = ((per - whole * kXcdUnits) * ks + kXcdUnits - 1) / kXcdUnits;
    double fill = (all - whole * (double)kComputeUnits) * ks / kComputeUnits - (rounds - 1);
    fill = fill < 0.02 ? 0.02 : fill > 1 ? 1 : fill;
    return out * (1 + 0.5 * whole) + 3.4 * (whole + rounds) + full * whole + full / ks * (rounds - 1 + 0.57 + 0.43 * fill) +
           (ks > 1 ? 0.9 + 6.8 * area * (ks - 1) : 0);
}
// Two workgroups add up a split block's sums (gemm_big.h: big_exchange).  Each first takes a number from the block's arrival counter.  Even:
// it leaves its sums, then adds two to the ready counter.  Odd: it waits until the ready counter has passed its number, that is, until
// as many have left their sums as took even numbers before it.  Neither counter is ever reset, so a wait ends whatever else runs:
// every even number below an odd one belongs to a workgroup that runs and waits for nobody.  (With counters set back to zero by
// whoever waited, launches that overlap - two streams on one model, which the interface forbids - lost counts: a workgroup then waited
// for ever, or every later launch of the block was out of step.)  Both counters wrap round at 2^32, in step.
constexpr bool exchange_waits(unsigned number) { return number % 2 == 1; }
constexpr bool exchange_ready(unsigned number, unsigned ready) { return (int)(ready - (number + 1)) >= 0; }

// Share of `now`'s time by the model that unsplit blocks may take at most.  Gate/up in 128-row blocks over a long K gives less than the
// model says (in calls, 128 x 256 against 256 x 128 blocks, which it puts 5 % behind: 256 rows at d 5120, d_ff 13824 85.8 and 84.5 us;
// 512 rows at d 3072, d_ff 8192 49.3 and 51.0).
inline double block_margin(TileEpilogue epi, int mbt, int k) { return mbt == 8 && k > 96 && epi == TileEpilogue::swiglu ? 0.95 : 0.96; }
// Share of `now`'s time by the model that a split last round may take at most.  From kernel traces of whole calls, split against
// `now`, us (d, d_ff, rows; promised):
//   the same blocks unsplit: gate/up 3072, 8192, 1536 136 / 144 (0.90), 5120, 13824, 2048 434 / 466 (0.94)
//   O and down: down 2048, 5632, 3000 86 / 93 (0.92), 4096, 12288, 2048 183 / 203 (0.83); O 5120, 1168 rows 92 / 86 (0.935)
//   256 x 192: QKV 4096, 2048 rows 190 / 197 (0.92), 3584, 2048 rows 165 / 163 (0.94); gate/up 4096, 12288, 896 169 / 172 (0.89),
//     2560, 6912, 1408 106 / 104, 2304, 6144, 2048 111 / 104, 2048, 5632, 2048 96 / 90 (0.92 to 0.93)
//   256 x 128: gate/up 3072, 8192, 512 56.7 / 53.7 (0.90), 5120, 13824, 256 87.4 / 86.7 (0.85); QKV 5120, 512 rows 93.9 / 92.6 (0.92)
// And split_lead: how much more it has to promise than unsplit blocks.  Split against those: gate/up 3072, 8192, 1536 132 / 124 (192 x 256; 0.95
// of their time promised), 4096, 12288, 960 167 / 161 (0.96), 5120, 13824, 1856 418 / 423 (320 x 256; 0.99); QKV 4096, 1856 rows 190 / 181
// (0.98), 5120, 1536 rows 215 / 211 (0.96); down 2048, 5632, 2720 79 / 89 (192 x 192; 0.97).
inline double split_margin(TileEpilogue epi, BigChoice now) {
    if (epi == TileEpilogue::resid) return 0.93;
    if (now.wn == 2) return 0;
    if (now.wn == 4 && now.mbt == kSplitMbt) return 0.94;
    return epi == TileEpilogue::qkv ? 0.93 : 0.905;
}
inline double split_lead(TileEpilogue epi) { return epi == TileEpilogue::resid ? 1 : 1.06; }
// room: bytes for partial sums; may_exchange: workgroups of a launch may exchange them
inline BigPlan big_plan(TileEpilogue epi, BigChoice now, int m, int n, int k, size_t room, bool may_exchange) {
    BigPlan best{now.mbt, now.wn, 1};
    double now_us = 0;
    if (now.wn) now_us = big_us(epi, now.mbt, now.wn, 1, m, n, k);
    else (void)tile_slices(epi, m, n, k, room, &now_us);
    double best_us = 1e30;
    auto consider = [&](int mbt, int wn, int ks) {
        const double us = big_us(epi, mbt, wn, ks, m, n, k);
        if (us * (ks > 1 ? split_lead(epi) : 1) < best_us && us < (ks > 1 ? split_margin(epi, now) : block_margin(epi, mbt, k)) * now_us) { best = BigPlan{mbt, wn, ks}; best_us = us; }
    };
    for (int mbt = 8; mbt <= 20; mbt += 4)
        for (int wn = mbt % 8 == 4 ? 3 : 2; wn <= 4; wn++) consider(mbt, wn, 1);         // (no narrow blocks of 192 and 320 rows)
    const int left = big_per_xcd(kSplitMbt, kSplitWn, m, n) % kXcdUnits;
    if (may_exchange && m >= kSplitMbt && left > 0 && (size_t)left * 8 * kSplitMbt * kSplitWn * 4096 <= room) consider(kSplitMbt, kSplitWn, 2);
    return best;
}

}  // namespace odb
