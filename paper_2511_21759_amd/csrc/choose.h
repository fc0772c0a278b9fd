// Which kernel variant a launch takes, as plain functions of its sizes (no HIP: they can be tried on the CPU).
#pragma once
#include <math.h>

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
struct AttentionChoice { int way; bool rows8; };
inline AttentionChoice attention_choice(int dh, int H, int L, bool step, int units, int units_per_seq, int tiles_per_unit) {
    const int per_seq = units_per_seq * tiles_per_unit, seqs = units / units_per_seq;
    const int items1 = units * tiles_per_unit, items2 = units * ((tiles_per_unit + 1) / 2);
    const int wgs4 = seqs * ((per_seq + 7) / 8) * H, wgs8 = seqs * ((per_seq + 15) / 16) * H;
    const bool wide = dh == 128, heads8 = H % 8 == 0, may_rows = per_seq >= 16 && (!step || tiles_per_unit % 2 == 0);
    const bool rows8 = wgs8 >= kComputeUnits;       // 256 rows per workgroup when that still gives every compute unit one, else 128
    const double n = (L + 31) / 32, kv_us = n * 32 * dh * 4 * seqs * H / 6.6e6;
    // (one_xcd: the launch keeps the workgroups of a head on one XCD)
    auto us = [&](int wgs, int wgs_per_head, bool one_xcd, double base, double round, double tile) {
        const double walk = base + (wgs + kComputeUnits - 1) / kComputeUnits * (round + tile * n);
        const double fetch = kv_us * (one_xcd ? 1 : wgs_per_head < 8 ? wgs_per_head : 8);
        return sqrt(walk * walk + fetch * fetch);
    };
    double t[4] = {0, 1e30, 1e30, 1e30};
    if (step) t[1] = wide ? us(items1 * H, per_seq, heads8 && items1 > 1, 0.9, 3.7, 0.173) : us(items1 * H, per_seq, false, 3.6, 1.0, 0.076);
    t[2] = wide ? us(items2 * H, items2 / seqs, heads8 && items2 > 1, step ? 0.5 : 1.7, step ? 5.2 : 3.9, step ? 0.28 : 0.27)
                : us(items2 * H, items2 / seqs, false, step ? 4.5 : 4.4, step ? 0.8 : 0.7, step ? 0.166 : 0.14);
    if (may_rows)
        t[3] = rows8 ? us(wgs8, (per_seq + 15) / 16, heads8, wide ? 5.8 : 4.1, wide ? 6.9 : 3.0, wide ? 1.12 : 0.81)
                     : us(wgs4, (per_seq + 7) / 8, heads8, wide ? 0.0 : 4.8, wide ? 6.0 : 0.0, wide ? 0.73 : 0.6);
    int way = may_rows ? 3 : !step || (tiles_per_unit >= 2 && items2 * H >= 128) ? 2 : 1;
    t[way] *= step ? 0.9 : 0.8;
    for (int w = 1; w <= 3; w++)
        if (t[w] < t[way]) way = w;
    return AttentionChoice{way, rows8};
}

}  // namespace odb
