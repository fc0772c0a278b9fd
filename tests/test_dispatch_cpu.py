"""The rules that pick a kernel variant by sizes (csrc/choose.h, plain host functions), against measured times: what a rule picks is
at most a stated share slower than the fastest variant that was measured at that size on an MI355X."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_21759_amd", "csrc")

SHIM = r"""
#include "choose.h"
using namespace odb;
extern "C" {
int attention_way(int dh, int H, int L, int step, int units, int ups, int tpu) { return attention_choice(dh, H, L, step != 0, units, ups, tpu).way; }
int attention_one_xcd(int dh, int H, int L, int step, int units, int ups, int tpu) { return attention_choice(dh, H, L, step != 0, units, ups, tpu).one_xcd; }
void attention_at(int id, int gx, int parts, int one_xcd, int *out) {
    const AttentionPlace p = attention_place(id, gx, parts, one_xcd != 0);
    out[0] = p.item; out[1] = p.head; out[2] = p.part;
}
int attention_wgs(int gx, int H, int parts) { return attention_grid(gx, H, parts); }
int swiglu_group(int m, int n, int k) { return swiglu_row_block_group(m, n, k); }
int qkv_slab(int m, int n) { return qkv_slab_group(m, n); }
int big_block(int m, int n, int k) { const BigChoice c = big_choice(m, n, k); return c.wn ? c.mbt * 10 + c.wn : 0; }
int plan(int epi, int now_mbt, int now_wn, int m, int n, int k, size_t room, int may) {
    const BigPlan p = big_plan((TileEpilogue)epi, BigChoice{now_mbt, now_wn}, m, n, k, room, may != 0);
    return p.wn ? p.mbt * 100 + p.wn * 10 + p.ks : 0;
}
int waits(unsigned number) { return exchange_waits(number); }
int ready(unsigned number, unsigned count) { return exchange_ready(number, count); }
int qkv_rows(int m, int n, int k) { const RowBlock b = qkv_row_block(m, n, k); return b.mt * 10 + b.ng; }
int resid_rows(int m, int n, int k) { const RowBlock b = resid_block(m, n, k); return b.mt * 10 + b.ng; }
int packed(int dense, int padded) { return dense_rows_pay(dense, padded); }
int few_split(int m, int n, int k) { return few_rows_split(m, n, k); }
int few_tile(int n, int k) { return few_rows_tile(n, k); }
int past_cache(double kv, double weights) { return weights_past_cache(kv, weights); }
int slices(int epi, int m_tiles, int n_tiles, int k_tiles, size_t room) { return tile_slices((TileEpilogue)epi, m_tiles, n_tiles, k_tiles, room); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs a host C++ compiler")
    d = tmp_path_factory.mktemp("rules")
    src, so = str(d / "shim.cpp"), str(d / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", "-I", CSRC, src, "-o", so], check=True)
    return ctypes.CDLL(so)


# head_dim, heads, cached positions, step, units, units per sequence, row tiles per unit -> us a layer of each way that can run
ATTENTION = [
    (128, 20, 3040, 1, 8, 4, 2, {1: 78.7, 2: 38.6}),
    (128, 12, 1056, 1, 16, 4, 2, {1: 33.8, 2: 19.7}),
    (128, 28, 544, 1, 5, 5, 2, {1: 17.8, 2: 11.5}),
    (128, 22, 3040, 1, 24, 8, 2, {1: 137.3, 2: 139.9, 3: 77.9}),
    (128, 40, 544, 1, 2, 2, 4, {1: 13.2, 2: 10.3}),
    (128, 32, 544, 1, 6, 6, 2, {1: 13.0, 2: 10.6}),
    (128, 32, 544, 1, 4, 4, 2, {1: 7.6, 2: 10.3}),
    (128, 32, 544, 1, 8, 8, 2, {1: 13.5, 2: 10.8, 3: 18.1}),
    (128, 8, 544, 1, 8, 8, 2, {1: 7.1, 2: 10.6, 3: 17.8}),
    (128, 32, 3040, 1, 32, 8, 4, {1: 362.5, 2: 302.3, 3: 124.9}),
    (128, 64, 1056, 1, 16, 8, 4, {1: 170.1, 2: 127.8, 3: 52.9}),
    (64, 48, 3040, 1, 4, 4, 2, {1: 45.4, 2: 26.6}),
    (64, 24, 1056, 1, 8, 4, 2, {1: 18.4, 2: 13.1}),
    (64, 48, 3040, 1, 24, 8, 2, {1: 122.0, 2: 137.2, 3: 86.6}),
    (64, 16, 1056, 1, 16, 8, 4, {1: 19.8, 2: 15.9, 3: 26.2}),
    (64, 4, 3040, 1, 6, 6, 4, {1: 14.1, 2: 25.6, 3: 67.5}),
    (64, 64, 1056, 1, 3, 3, 2, {1: 18.0, 2: 12.9}),
    (128, 8, 160, 1, 1, 1, 1, {1: 5.8, 2: 6.9}),
    (128, 64, 3040, 1, 1, 1, 2, {1: 33.1, 2: 40.1}),
    (128, 12, 544, 1, 9, 9, 1, {1: 9.0, 2: 10.8}),
    (64, 32, 1056, 1, 3, 3, 3, {1: 16.0, 2: 13.2}),
    (128, 32, 1024, 0, 1, 1, 64, {2: 52.7, 3: 32.7}),
    (128, 32, 611, 0, 1, 1, 39, {2: 30.5, 3: 21.7}),
    (128, 8, 333, 0, 3, 1, 21, {2: 14.9, 3: 13.1}),
    (64, 12, 384, 0, 1, 1, 24, {2: 6.8, 3: 12.8}),
    (64, 16, 1024, 0, 1, 1, 64, {2: 14.1, 3: 25.4}),
    (128, 64, 512, 0, 4, 1, 32, {2: 144.4, 3: 62.8}),
    (128, 12, 1700, 0, 1, 1, 107, {2: 59.2, 3: 46.6}),
    (128, 32, 3000, 0, 1, 1, 188, {2: 343.2, 3: 219.9}),
    (128, 20, 100, 0, 1, 1, 7, {2: 6.2}),
]


@pytest.mark.parametrize("case", ATTENTION)
def test_attention_way_is_near_the_fastest_measured(rules, case):
    *sizes, us = case
    way = rules.attention_way(*sizes)
    assert way in us, "a way that cannot run at this size"
    # (the rule stays with its first choice up to 10 %; the model is off by a few percent beside that)
    assert us[way] <= 1.15 * min(us.values())


def test_heads_stay_on_one_xcd_in_steps_only(rules):
    """A refresh leaves the heads spread (the O projection behind it is faster), and only heads of 128 channels in eights can be
    mapped."""
    for H in (8, 12, 16, 32):
        for dh in (64, 128):
            for units, tpu in ((1, 1), (1, 2), (4, 2), (8, 4)):
                got = rules.attention_one_xcd(dh, H, 544, 1, units, units, tpu)
                way = rules.attention_way(dh, H, 544, 1, units, units, tpu)
                items = units * (tpu if way == 1 else (tpu + 1) // 2)
                assert got == (dh == 128 and H % 8 == 0 and items > 1)
                assert not rules.attention_one_xcd(dh, H, 16 * tpu * units, 0, 1, 1, tpu * units)


@pytest.mark.parametrize("H,gx,parts,one_xcd", [
    (28, 4, 2, 0), (28, 2, 4, 0), (28, 8, 1, 0), (20, 6, 2, 0), (6, 8, 4, 0), (1, 1, 4, 0), (5, 3, 1, 0),
    (32, 1, 4, 0), (32, 2, 4, 1), (32, 4, 2, 1), (8, 5, 4, 1), (16, 3, 1, 1),
])
def test_workgroups_that_read_the_same_keys_share_an_xcd(rules, H, gx, parts, one_xcd):
    at, wgs, out = {}, rules.attention_wgs(gx, H, parts), (ctypes.c_int * 3)()
    for i in range(wgs):
        rules.attention_at(i, gx, parts, one_xcd, out)
        if out[1] < H:
            assert tuple(out) not in at
            at[tuple(out)] = i % 8
    assert set(at) == {(x, h, p) for x in range(gx) for h in range(H) for p in range(parts)}
    for h in range(H):
        for x in range(gx):
            assert len({at[x, h, p] for p in range(parts)}) == 1
        assert not one_xcd or len({at[x, h, 0] for x in range(gx)}) == 1
    units = [sum(v == x for (_, _, p), v in at.items() if p == 0) for x in range(8)]
    assert max(units) - min(units) <= 1 or one_xcd


# projection, row tiles, n-tiles, k-tiles -> us of the tile kernel and its merge pass by K slices
SLICES = [
    ("down", 16, 96, 192, {1: 75.4, 2: 41.5, 3: 31.5, 4: 26.2, 5: 23.6, 6: 21.9, 7: 21.2, 8: 19.9, 9: 20.0, 10: 19.5, 11: 20.1, 12: 19.2, 14: 20.1, 16: 17.7}),
    ("down", 77, 80, 160, {1: 65.2, 2: 39.3, 3: 35.4, 4: 29.8, 5: 37.8}),
    ("down", 40, 160, 216, {1: 96.3, 2: 54.3, 3: 44.6, 4: 38.3, 5: 44.6}),
    ("down", 28, 176, 200, {1: 86.8, 2: 50.6, 3: 40.6, 4: 34.1, 5: 39.0, 6: 48.1}),
    ("down", 28, 192, 256, {1: 108.2, 2: 59.8, 3: 47.4, 4: 40.7, 5: 39.0, 6: 49.4}),
    ("qkv", 64, 96, 16, {1: 24.6, 2: 21.5, 3: 22.5, 4: 23.7}),
    ("o", 28, 192, 96, {1: 48.2, 2: 30.5, 3: 26.5, 4: 24.7, 5: 25.9, 6: 31.3}),
    ("down", 4, 176, 200, {1: 50.4, 2: 31.5, 3: 24.9, 4: 21.6, 5: 20.2, 6: 19.9, 7: 18.7, 8: 18.3, 9: 18.5, 10: 19.3, 11: 20.4, 12: 25.7, 14: 25.4, 16: 23.6}),
    ("down", 7, 512, 896, {1: 244.5, 2: 139.8, 3: 106.1, 4: 91.3, 5: 128.7, 6: 111.2, 7: 104.8, 8: 109.2, 9: 120.3}),
    ("o", 8, 256, 128, {1: 42.2, 2: 27.4, 3: 22.4, 4: 21.6, 5: 20.1, 6: 19.1, 7: 19.0, 8: 20.4, 9: 25.2, 10: 24.9, 11: 24.6, 12: 25.1, 14: 25.8, 16: 26.6}),
    ("down", 8, 256, 384, {1: 110.9, 2: 62.8, 3: 47.7, 4: 41.7, 5: 37.0, 6: 34.3, 7: 32.4, 8: 33.0, 9: 43.4, 10: 41.2, 11: 41.4, 12: 40.4, 14: 38.2, 16: 40.0}),
    ("down", 64, 256, 384, {1: 171.5, 2: 110.0, 3: 137.6, 4: 119.5}),
    ("down", 40, 256, 384, {1: 163.1, 2: 96.7, 3: 76.3, 4: 101.9}),
    ("o", 40, 256, 128, {1: 62.8, 2: 42.6, 3: 38.1, 4: 50.2}),
    ("o", 16, 256, 128, {1: 62.5, 2: 36.5, 3: 29.2, 4: 26.8, 5: 25.4, 6: 25.1, 7: 25.2, 8: 26.3}),
    ("down", 16, 256, 384, {1: 164.5, 2: 88.6, 3: 65.2, 4: 53.3, 5: 47.6, 6: 46.9, 7: 45.3, 8: 44.1}),
    ("o", 13, 128, 64, {1: 35.2, 2: 22.0, 3: 18.5, 4: 17.5, 5: 15.4, 6: 15.1, 7: 15.0, 8: 15.9, 9: 16.1, 10: 17.3, 11: 16.6, 12: 18.3, 14: 18.5, 16: 20.0}),
    ("down", 9, 224, 592, {1: 223.4, 2: 118.4, 3: 86.6, 4: 68.5, 5: 60.7, 6: 54.7, 7: 53.2, 8: 48.2, 9: 54.6, 10: 68.1, 11: 67.3, 12: 60.2, 14: 60.5, 16: 58.7}),
    ("down", 9, 128, 176, {1: 74.6, 2: 41.0, 3: 31.1, 4: 26.0, 5: 23.3, 6: 21.6, 7: 19.9, 8: 19.3, 9: 18.9, 10: 18.2, 11: 18.0, 12: 18.1, 13: 17.9, 14: 17.9, 15: 18.2, 16: 17.7}),
    ("o", 3, 160, 80, {1: 23.3, 2: 17.9, 3: 15.1, 4: 12.7, 5: 12.3, 6: 12.0, 7: 11.8, 8: 12.1, 9: 13.4, 10: 13.4, 11: 14.6, 12: 14.3, 14: 18.9, 16: 16.8}),
    ("down", 63, 64, 96, {1: 43.5, 2: 26.6, 3: 22.4, 4: 21.3, 5: 19.9, 6: 19.7, 7: 24.7, 8: 20.8}),
    ("gu", 9, 704, 64, {1: 35.5, 2: 31.8, 3: 45.2, 4: 42.2, 5: 44.4}),
    ("qkv", 13, 384, 64, {1: 43.0, 2: 30.5, 3: 27.8, 4: 27.6, 5: 28.8, 6: 38.3}),
]


@pytest.mark.parametrize("case", SLICES)
def test_tile_slices_are_near_the_fastest_measured(rules, case):
    name, m, n, k, us = case
    epi = {"qkv": 0, "gu": 1}.get(name, 2)
    ks = rules.slices(epi, m, n, k, ctypes.c_size_t(64 << 20))
    assert ks in us, "a count that does not fit"
    assert us[ks] <= 1.1 * min(us.values())


def test_tile_slices_keep_to_the_room_and_to_the_matrix(rules):
    """A slice has eight k-tiles, the partial sums fit, and an unsplit launch needs no room."""
    for m in (1, 3, 8, 9, 39, 188):
        for n in (16, 48, 256, 1024):
            for k in (8, 24, 64, 896):
                for room in (0, 1 << 20, 32 << 20):
                    for epi in (0, 1, 2):
                        ks = rules.slices(epi, m, n, k, ctypes.c_size_t(room))
                        assert ks == 1 or (k // ks >= 8 and ks * m * n * 1024 <= room)


# row tiles, n-tiles, k-tiles -> us of gate/up on the streaming kernel in row blocks and on the tile kernel
SWIGLU = [
    (9, 192, 16, 6.3, 18.2), (16, 256, 24, 11.9, 21.5), (9, 384, 32, 10.8, 22.5), (16, 384, 32, 11.1, 23.9), (16, 512, 32, 22.1, 26.5),
    (9, 512, 40, 20.2, 24.1), (16, 512, 40, 26.6, 26.7), (9, 384, 64, 16.0, 24.9), (16, 384, 96, 21.9, 29.6), (16, 512, 64, 35.6, 31.4),
    (9, 256, 64, 17.1, 23.9), (16, 256, 64, 22.7, 26.3), (13, 256, 80, 25.0, 24.4), (13, 256, 96, 30.2, 25.2), (16, 512, 96, 49.5, 37.4), (16, 256, 128, 40.2, 31.2), (9, 512, 128, 48.9, 35.4), (16, 512, 128, 63.4, 42.8),
]


@pytest.mark.parametrize("m,n,k,stream,tile", SWIGLU)
def test_swiglu_takes_row_blocks_where_they_are_faster(rules, m, n, k, stream, tile):
    us = stream if rules.swiglu_group(m, n, k) else tile
    assert us <= 1.05 * min(stream, tile)
    assert rules.swiglu_group(8, n, k) == 0 and rules.swiglu_group(17, n, k) == 0 and rules.swiglu_group(m, 513, k) == 0


# n-tiles -> us of QKV at 128 rows in blocks of 3 and 6 n-tiles and on the streaming kernel (0)
QKV_SLAB = [
    (480, {3: 20.7, 6: 28.0, 0: 22.6}),
    (528, {3: 22.7, 6: 30.3, 0: 24.5}), (672, {3: 28.3, 6: 36.8, 0: 30.9}), (768, {3: 31.1, 6: 40.2, 0: 31.8}), (864, {3: 61.4, 6: 45.6, 0: 66.2}),
    (960, {3: 68.7, 6: 51.1, 0: 73.4}), (1152, {3: 81.7, 6: 60.1, 0: 84.5}), (1344, {3: 96.0, 6: 72.7, 0: 102.7}), (1536, {3: 112.5, 6: 83.7, 0: 105.3}),
]


@pytest.mark.parametrize("n,us", QKV_SLAB)
def test_qkv_of_97_to_128_rows_takes_the_fastest_width(rules, n, us):
    for m in (7, 8):
        assert us[rules.qkv_slab(m, n)] <= 1.02 * min(us.values())
    assert rules.qkv_slab(6, n) == 0 and rules.qkv_slab(17, n) == 0
    assert rules.qkv_slab(7, 384) == 0
    assert rules.qkv_slab(9, n) == (6 if n <= 768 else 0)


# n-tiles, rows -> us of the O projection (first table), QKV and gate/up (second) by block (16-row tiles * 10 + units of 64 columns;
# 0: tile kernel and merge pass)
BLOCKS = [
    (96, 3008, {0: 33.4, 162: 33.3, 163: 40.0, 164: 46.8, 82: 40.2, 83: 28.5, 84: 33.1}),
    (160, 2048, {0: 47.4, 162: 45.3, 163: 55.6, 164: 63.7, 82: 60.9, 83: 40.3, 84: 48.1}),
    (176, 2048, {0: 53.0, 162: 48.4, 163: 57.9, 164: 67.4, 82: 65.7, 83: 43.7, 84: 52.0}),
    (192, 1536, {0: 51.8, 162: 51.0, 163: 61.6, 164: 72.1, 82: 62.2, 83: 42.7, 84: 50.8}),
    (192, 2048, {0: 54.1, 162: 52.3, 163: 62.1, 164: 73.0, 82: 70.6, 83: 46.5, 84: 56.6}),
    (192, 3008, {0: 97.4, 162: 101.1, 163: 67.3, 164: 79.2, 82: 98.2, 83: 83.7, 84: 99.9}),
    (224, 1232, {0: 62.6, 162: 56.8, 163: 68.7, 164: 79.8, 82: 70.7, 83: 49.9, 84: 55.4}),
    (256, 1008, {0: 49.5, 162: 63.0, 163: 74.7, 164: 87.0, 82: 46.4, 83: 56.1, 84: 60.8}),
    (256, 1232, {0: 67.4, 162: 63.9, 163: 75.1, 164: 87.1, 82: 80.2, 83: 56.8, 84: 62.4}),
    (256, 1536, {0: 66.5, 162: 64.3, 163: 75.6, 164: 87.8, 82: 88.7, 83: 100.2, 84: 64.0}),
    (256, 2048, {0: 79.0, 162: 78.3, 163: 87.0, 164: 95.5, 82: 96.9, 83: 108.7, 84: 73.6}),
    (320, 1008, {0: 85.2, 162: 75.3, 163: 90.7, 164: 105.4, 82: 103.5, 83: 69.4, 84: 73.8}),
    (320, 2048, {0: 157.5, 162: 165.1, 163: 122.0, 164: 129.4, 82: 168.4, 83: 142.6, 84: 159.0}),
    (384, 768, {0: 102.7, 162: 94.1, 163: 109.0, 164: 127.9, 82: 117.2, 83: 75.4, 84: 90.4}),
    (384, 1536, {0: 162.8, 162: 185.8, 163: 119.9, 164: 140.8, 82: 189.5, 83: 152.5, 84: 177.0}),
    (512, 608, {0: 114.6, 162: 122.6, 163: 139.3, 164: 163.4, 82: 159.0, 83: 104.4, 84: 118.4}),
    (512, 1232, {0: 217.5, 162: 250.8, 163: 174.1, 164: 185.0, 82: 246.7, 83: 206.5, 84: 232.6}),
    (256, 1312, {0: 61.5, 83: 97.0}),           # 11 x 22 blocks: 33 on six of the XCDs
    (1024, 512, {0: 41.6, 162: 37.8, 163: 41.4, 164: 45.4, 82: 46.3, 83: 54.6, 84: 35.4}),
    (864, 512, {0: 52.4, 162: 43.6, 163: 48.5, 164: 54.4, 82: 54.5, 83: 65.8, 84: 40.8}),
    (480, 1008, {0: 54.9, 162: 51.1, 163: 56.7, 164: 62.7, 82: 60.5, 83: 72.3, 84: 46.5}),
    (576, 768, {0: 60.1, 162: 54.6, 163: 63.6, 164: 71.2, 82: 67.0, 83: 79.7, 84: 52.2}),
    (672, 608, {0: 71.0, 162: 108.4, 163: 73.3, 164: 79.9, 82: 78.4, 83: 89.7, 84: 58.9}),
    (512, 768, {0: 63.7, 162: 58.1, 163: 68.1, 164: 77.0, 82: 76.4, 83: 94.3, 84: 55.3}),
    (768, 512, {0: 74.0, 162: 67.5, 163: 80.8, 164: 89.2, 82: 86.5, 83: 58.2, 84: 62.6}),
    (1536, 512, {0: 128.2, 162: 119.3, 163: 86.0, 164: 87.8, 82: 118.7, 83: 101.5, 84: 114.0}),
    (768, 640, {0: 75.4, 162: 124.5, 163: 81.2, 164: 88.0, 82: 87.6, 83: 104.7, 84: 66.0}),
    (1536, 640, {0: 134.9, 162: 175.1, 163: 147.2, 164: 172.2, 82: 154.2, 83: 146.1, 84: 117.0}),
    (768, 1024, {0: 136.1, 162: 131.8, 163: 93.2, 164: 96.1, 82: 134.8, 83: 115.6, 84: 122.9}),
    (1536, 1024, {0: 200.2, 162: 188.0, 163: 165.3, 164: 176.7, 82: 240.3, 83: 204.0, 84: 179.4}),
    (960, 512, {0: 90.8, 162: 85.9, 163: 97.5, 164: 108.9, 82: 107.7, 83: 125.8, 84: 81.5}),
    (1536, 608, {0: 292.6, 162: 356.9, 163: 304.1, 164: 342.9, 82: 311.3, 83: 297.5, 84: 233.0}),
]


@pytest.mark.parametrize("n,rows,us", BLOCKS)
def test_blocks_are_near_the_fastest_measured(rules, n, rows, us):
    block = rules.big_block(rows // 16, n, 128)
    assert block in us and us[block] <= 1.15 * min(us.values())


# k-tiles up to 32: n-tiles, rows, k-tiles -> us by block
SHORT_K = [
    (192, 640, 16, {0: 18.9, 162: 12.6, 163: 14.7, 164: 16.4, 82: 9.0, 83: 10.6, 84: 11.7}),
    (256, 512, 24, {0: 21.7, 162: 15.5, 163: 18.4, 164: 20.8, 82: 11.2, 83: 13.3, 84: 14.7}),
    (144, 1008, 24, {0: 28.8, 162: 22.8, 163: 27.9, 164: 31.6, 82: 15.1, 83: 19.6, 84: 20.5}),
    (144, 1536, 24, {0: 29.1, 162: 23.5, 163: 28.9, 164: 32.2, 82: 24.7, 83: 20.6, 84: 21.3}),
    (144, 3008, 24, {0: 31.1, 162: 39.5, 163: 30.3, 164: 33.4, 82: 37.4, 83: 34.6, 84: 37.1}),
    (384, 384, 32, {0: 24.3, 162: 19.3, 163: 22.4, 164: 25.4, 82: 13.7, 83: 16.2, 84: 17.7}),
    (1024, 640, 32, {0: 46.6, 162: 37.3, 163: 44.8, 164: 28.6, 82: 35.6, 83: 31.2, 84: 34.6}),
    (64, 2048, 32, {0: 20.0, 162: 24.4, 163: 30.9, 164: 36.8, 82: 16.3, 83: 21.5, 84: 25.1}),
    (192, 768, 32, {0: 29.3, 162: 25.7, 163: 31.3, 164: 35.8, 82: 17.3, 83: 21.6, 84: 23.5}),
]


@pytest.mark.parametrize("n,rows,k,us", SHORT_K)
def test_blocks_over_a_short_k(rules, n, rows, k, us):
    block = rules.big_block(rows // 16, n, k)
    assert block in us and us[block] <= 1.15 * min(us.values())


# projection (0 QKV, 1 gate/up, 2 O and down), rows, n-tiles, k-tiles, block before the rule (0: tile kernel) -> us by block (16-row
# tiles * 100 + units of 64 columns * 10 + workgroups that share a block of the last round)
PLANS = [
    (1, 320, 1536, 128, 0, {0: 123.7, 1231: 69.3, 1241: 83.1, 1631: 87.6, 2031: 90.8, 2041: 107.4}),
    (1, 608, 1536, 128, 841, {841: 135.4, 2031: 112.9, 2041: 125.5, 1231: 139.2, 1241: 166.6, 1642: 157.3}),
    (1, 704, 1536, 128, 1641, {1641: 171.9, 1231: 141.1, 1642: 159.6, 1241: 167.1, 2031: 199.4}),
    (0, 768, 768, 128, 841, {841: 95.9, 1231: 78.4, 1241: 92.7, 2031: 114.4, 1642: 120.5}),
    (1, 1024, 1536, 128, 1631, {1631: 197.2, 1642: 188.9, 1231: 219.3, 2031: 226.9, 1241: 264.1}),
    (0, 1408, 768, 128, 1641, {1641: 194.0, 2041: 151.3, 1231: 162.8, 1642: 173.6, 1241: 183.1}),
    (2, 1536, 256, 384, 1621, {1621: 211.2, 1642: 177.9, 1231: 190.9, 1241: 241.5, 2031: 277.1}),
    (0, 2048, 768, 128, 1631, {1631: 220.1, 1642: 207.1, 1231: 243.0, 2031: 248.6, 1241: 279.5}),
    (2, 2048, 256, 384, 1621, {1621: 240.4, 1642: 202.3, 1241: 268.0, 2031: 302.8, 1231: 355.0}),
    (2, 3008, 256, 384, 1631, {1631: 311.4, 1241: 280.9, 2031: 323.9, 1642: 348.1, 2041: 372.3}),
    (2, 3008, 256, 128, 1631, {1631: 128.8, 1241: 114.7, 2031: 132.9, 2041: 154.8, 1231: 155.1}),
]


@pytest.mark.parametrize("epi,rows,n,k,now,us", PLANS)
def test_plans_are_near_the_fastest_measured(rules, epi, rows, n, k, now, us):
    rules.plan.argtypes = [ctypes.c_int] * 6 + [ctypes.c_size_t, ctypes.c_int]
    picked = rules.plan(epi, now // 100 if now else 16, now // 10 % 10, rows // 16, n, k, 96 << 20, 1)
    assert picked in us and us[picked] <= 1.05 * min(us.values()) and us[picked] <= us[now]


# the same from kernel traces of whole calls, where the launches follow each other: a split last round is not worth there what it is by itself
PLANS_IN_CALLS = [
    (1, 144, 1536, 128, 831, {831: 57.7, 1231: 61.7}),          # one row block of 192 rows
    (1, 192, 1536, 128, 831, {831: 57.4, 1231: 62.7}),
    (1, 192, 1216, 112, 0, {831: 46.9, 1231: 53.5, 0: 61.1}),
    (1, 192, 1728, 160, 0, {1231: 82.7, 0: 92.9}),
    (1, 704, 1728, 160, 1631, {1631: 200.1, 1241: 195.4, 1642: 189.5}),
    (1, 512, 864, 80, 1621, {1621: 42.9, 841: 40.7, 1642: 46.5}),
    (1, 512, 1024, 96, 1621, {1621: 51.0, 841: 49.3, 1642: 56.0}),
    (1, 960, 1536, 128, 1631, {1631: 174.0, 1241: 161.0, 1642: 166.9}),
    (1, 1536, 864, 80, 1631, {1631: 102.4, 1241: 98.9, 1642: 104.8}),
    (1, 1536, 1024, 96, 1641, {1641: 139.2, 1241: 124.0, 1642: 132.2}),
    (1, 1856, 768, 72, 1631, {1631: 100.9, 1241: 93.2, 1642: 106.9}),
    (1, 1856, 1728, 160, 1641, {1641: 454.3, 2041: 423.5, 1642: 418.0}),
    (1, 2048, 704, 64, 1631, {1631: 87.4, 1642: 95.4}),
    (1, 2048, 768, 72, 1631, {1631: 99.9, 1642: 104.8}),
    (1, 2048, 1216, 112, 1641, {1641: 245.6, 1642: 229.2}),
    (0, 512, 960, 160, 1621, {1621: 91.7, 841: 88.9, 1642: 94.3}),
    (0, 1536, 960, 160, 1631, {1631: 223.4, 1241: 210.6, 1642: 214.8}),
    (0, 1856, 768, 128, 1631, {1631: 193.1, 1241: 180.9, 1642: 189.8}),
    (0, 2048, 672, 112, 1631, {1631: 161.9, 1642: 163.1}),
    (0, 2048, 768, 128, 1631, {1631: 197.1, 1642: 190.1}),
    (2, 1792, 224, 112, 1621, {1621: 62.7, 841: 59.5}),
    (1, 256, 1728, 160, 1621, {1621: 84.5, 841: 85.8}),
    (1, 1024, 512, 48, 1621, {1621: 28.9, 841: 27.9}),
    (0, 1024, 480, 80, 1621, {1621: 51.8, 841: 47.6}),
    (2, 1200, 320, 160, 1621, {1621: 86.0, 1231: 80.7, 1642: 92.2}),
    (2, 1856, 256, 384, 1621, {1621: 197.7, 1642: 178.1}),
    (2, 2720, 128, 176, 1621, {1621: 89.4, 1231: 88.6, 1642: 79.0}),
]


@pytest.mark.parametrize("epi,rows,n,k,now,us", PLANS_IN_CALLS)
def test_plans_are_no_slower_inside_calls(rules, epi, rows, n, k, now, us):
    rules.plan.argtypes = [ctypes.c_int] * 6 + [ctypes.c_size_t, ctypes.c_int]
    picked = rules.plan(epi, now // 100 if now else 16, now // 10 % 10, rows // 16, n, k, 96 << 20, 1)
    assert picked in us and us[picked] <= 1.015 * min(us.values()) and us[picked] <= us[now]


def test_sizes_of_the_gpu_test_of_the_split_take_it(rules):
    from test_gpu_many_rows import SPLIT
    rules.plan.argtypes = [ctypes.c_int] * 6 + [ctypes.c_size_t, ctypes.c_int]
    for d, f, rows, which in SPLIT:
        m, room = (rows + 15) // 16, max(32 << 20, (rows + 15) // 16 * 16 * d * 16)
        epi, n, k = {"qkv": (0, 3 * d // 16, d // 32), "gate/up": (1, 2 * f // 16, d // 32), "down": (2, d // 16, f // 32)}[which]
        block = rules.big_block(m, n, k)
        assert block and rules.plan(epi, block // 10, block % 10, m, n, k, room, 1) == 1642


def _resid_plan(rules, m, n, k, room):
    """O or down beyond 128 rows: the plan where no block with all of K is taken (128-row blocks only over a K up to the columns)."""
    if rules.resid_rows(m, n, k):
        return None
    block = rules.big_block(m, n, k)
    if block < 160 and k > n:
        block = 0
    return rules.plan(2, block // 10 if block else 16, block % 10, m, n, k, room, 1)


def _qkv_kernel(rules, m, n, k, room):
    rows, slab, block = rules.qkv_rows(m, n, k), rules.qkv_slab(m, n), rules.big_block(m, n, k)
    if rows:
        return "rows %d" % rows
    if m <= 6:
        return "few" if m <= 2 else "stream"
    if slab:
        return "slab %d" % slab
    plan = rules.plan(0, block // 10 if block else 16, block % 10, m, n, k, room, 1)
    return "big %d" % plan if plan else "tile"


def test_sizes_of_the_gpu_test_of_tall_blocks_take_them(rules):
    from test_gpu_many_rows import TALL, TALL_BATCH
    rules.plan.argtypes = [ctypes.c_int] * 6 + [ctypes.c_size_t, ctypes.c_int]
    seen = set()
    for d, f, rows, plans in TALL + [(d, f, 16 * n * tiles, plans) for d, f, n, tiles, plans in TALL_BATCH]:
        m, room = (rows + 15) // 16, min(96 << 20, max(32 << 20, (rows + 15) // 16 * 16 * d * 16))
        for which, plan in plans.items():
            if which == "qkv":
                assert _qkv_kernel(rules, m, 3 * d // 16, d // 32, room) == "big %d" % plan
            elif which == "gate/up":
                block = rules.big_block(m, f // 8, d // 32)
                assert rules.plan(1, block // 10 if block else 16, block % 10, m, f // 8, d // 32, room, 1) == plan
            else:
                assert _resid_plan(rules, m, d // 16, (d if which == "O" else f) // 32, room) == plan
            seen.add(("resid" if which in ("O", "down") else which, plan))
    assert seen == {(w, p) for w in ("qkv", "gate/up", "resid") for p in (1231, 1241, 2031, 2041)}


def test_sizes_of_the_gpu_test_of_packed_drafts_are_packed(rules):
    from test_gpu_many_rows import DENSE
    rules.plan.argtypes = [ctypes.c_int] * 6 + [ctypes.c_size_t, ctypes.c_int]
    for d, dh, f, batch, b, S, kernel, way in DENSE:
        m, tpu = (batch * S * b + 15) // 16, (b + 15) // 16
        assert rules.packed(m, batch * S * tpu), (b, S, batch)
        for room in (32 << 20, min(96 << 20, max(32 << 20, m * 16 * d * 16))):          # of the fixed area, of the model's own scratch
            assert _qkv_kernel(rules, m, 3 * d // 16, d // 32, room) == kernel, (d, b, S)
        assert rules.attention_way(dh, d // dh, 110, 1, batch * S, S, tpu) == way, (d, b, S)
    blocks = ["rows 21", "rows 22", "rows 23", "rows 24", "rows 43", "rows 44", "slab 3", "slab 6"]
    rings = ["big %d" % p for p in (821, 831, 841, 1231, 1241, 1621, 1631, 1641, 1642, 2031, 2041)]
    assert {case[6] for case in DENSE} == {"few", "stream", "tile", *blocks, *rings}
    assert not rules.packed(5, 6)


def test_plans_exchange_only_where_there_is_room_for_it(rules):
    rules.plan.argtypes = [ctypes.c_int] * 6 + [ctypes.c_size_t, ctypes.c_int]
    split = lambda room, may: rules.plan(2, 16, 2, 128, 256, 384, room, may) == 1642
    assert split(32 << 20, 1) and not split((32 << 20) - 1, 1) and not split(96 << 20, 0)      # 128 blocks of 256 KiB
    for m in range(9, 190):
        for n in (64, 96, 160, 256, 480, 768, 1536):
            p = rules.plan(2, 16, 3, m, n, 128, 96 << 20, 1)
            if p % 10 == 2:                    # two counters a split block; the whole rounds' blocks are not split
                left = (m + 15) // 16 * ((n // 16 + (n % 16 > 0) + 7) // 8) % 32
                assert p == 1642 and 0 < left and 2 * 8 * left <= 1024


# ---- the counters of a block that two workgroups share ---------------------------------------------------------------------------

def _exchange(steps, launches, start):
    """Every order in which the workgroups of `launches` overlapping launches (two each) can take their steps on one block's two
    counters, from (start, start): the states in which somebody waits and nobody can go on, and whether a workgroup ever went on from its
    wait before as many had counted themselves ready as that takes.  A workgroup is (place in its program, its number)."""
    first = (start, start, ((0, 0),) * (2 * launches))
    seen, todo, stuck, early = {first}, [first], [], False
    while todo:
        arrive, ready, groups = state = todo.pop()
        moved = False
        for i, (place, number) in enumerate(groups):
            after = steps(arrive, ready, place, number)
            if after is None:
                continue
            moved = True
            if place == 1 and steps is not RESET and after[2] == DONE and number % 2 == 1:
                done = sum(1 for g in groups if g[0] == DONE and g[1] % 2 == 0)
                early = early or done < ((number - start) % 2 ** 32 + 1) // 2
            nxt = (after[0], after[1], tuple(sorted(groups[:i] + ((after[2], after[3]),) + groups[i + 1:])))
            if nxt not in seen:
                seen.add(nxt)
                todo.append(nxt)
        if not moved and any(place != DONE for place, _ in groups):
            stuck.append(state)
    return stuck, early


DONE = 9


def RESET(arrive, ready, place, number):
    """Counters that start at zero and that the second workgroup sets back: the form that overlapping launches break."""
    if place == 0:
        return arrive + 1, ready, 1, arrive
    if place == 1 and number != 1:
        return arrive, ready + 1, DONE, number
    if place == 1:
        return (arrive, ready, 2, number) if ready == 1 else None
    if place == 2:
        return 0, ready, 3, number
    return (arrive, 0, DONE, number) if place == 3 else None


@pytest.mark.parametrize("start", [0, 2, 2 ** 31 - 2, 2 ** 31, 2 ** 32 - 4, 2 ** 32 - 2])
def test_a_shared_blocks_workgroups_never_wait_for_ever(rules, start):
    rules.waits.argtypes = [ctypes.c_uint]
    rules.ready.argtypes = [ctypes.c_uint] * 2
    M = 2 ** 32

    def steps(arrive, ready, place, number):
        if place == 0:
            return (arrive + 1) % M, ready, 1, arrive
        if place == 1 and not rules.waits(number):
            return arrive, (ready + 2) % M, DONE, number
        if place == 1 and rules.ready(number, ready):
            return arrive, ready, DONE, number
        return None

    for launches in (1, 2, 3):
        stuck, early = _exchange(steps, launches, start)
        assert not stuck and not early
    # alone on the counters, launch after launch
    assert _exchange(RESET, 1, 0)[0] == [] and _exchange(RESET, 2, 0)[0]


# O and down beyond 128 rows, rows, n-tiles, k-tiles -> us inside calls in blocks of 64 x 64 with all of K (44), on the tile kernel (0)
@pytest.mark.parametrize("rows,n,k,us", [
    (2048, 48, 64, {44: 26.8, 0: 22.3}), (1952, 48, 64, {44: 25.6, 0: 22.2}), (1792, 48, 64, {44: 22.8, 0: 21.8}),
    (2048, 48, 24, {44: 14.9, 0: 17.7}), (1024, 48, 64, {44: 11.8, 0: 19.1}), (1024, 128, 64, {44: 23.7, 0: 25.3}),
    (1296, 96, 48, {44: 19.7, 0: 24.2}), (1296, 80, 40, {44: 17.9, 0: 20.5}),
])
def test_resid_blocks_where_they_are_faster(rules, rows, n, k, us):
    assert us[rules.resid_rows(rows // 16, n, k)] == min(us.values())


@pytest.mark.parametrize("m,n,k,blocks_of", [
    (2, 64, 96, 1), (1, 64, 96, 1), (2, 128, 256, 2), (2, 256, 128, 4), (2, 256, 384, 4),      # O and down, a round of 256 workgroups at most
    (2, 64, 32, 0), (2, 64, 80, 0),        # a short K stays whole
    (2, 128, 176, 0), (2, 64, 88, 0),      # four slices of eight waves do not divide it
    (2, 272, 384, 0), (3, 64, 96, 0),      # too many blocks; more than 32 rows have rules of their own
])
def test_few_rows_split_k_where_it_fits(rules, m, n, k, blocks_of):
    assert rules.few_split(m, n, k) == blocks_of


# 32 rows (three drafts of 10 packed take the same), n-tiles, k-tiles -> us with all of K in a workgroup, on the tile kernel with its merge pass
@pytest.mark.parametrize("n,k,whole,tile", [
    (320, 432, 49.9, 31.2), (272, 368, 41.8, 26.1), (512, 688, 85.9, 71.2), (272, 136, 21.8, 15.7), (320, 160, 21.2, 18.8), (384, 192, 25.2, 22.3),
    (512, 256, 32.8, 35.4), (224, 304, 20.4, 21.2), (160, 216, 15.0, 16.1), (224, 112, 9.4, 13.5), (160, 80, 7.8, 11.3),
])
def test_few_rows_over_more_than_a_round_of_columns(rules, n, k, whole, tile):
    assert rules.few_split(2, n, k) == 0 and rules.few_tile(n, k) == (tile < whole)


# steps of 128 and 96 rows at d 4096: layers, keys -> time with O's weights past the memory-side cache over time with them in it
@pytest.mark.parametrize("layers,keys,ratios", [
    (4, 512, [1.031]), (4, 1024, [1.019]), (4, 2048, [0.983, 0.987]), (4, 3072, [0.964, 0.954]), (8, 512, [0.994, 1.001]), (8, 1024, [0.991, 0.997]),
    (8, 2048, [1.000, 1.008]), (12, 512, [0.990, 1.000]), (12, 1024, [0.986, 0.992]), (12, 2048, [1.001, 1.007]), (16, 512, [0.992, 1.005]),
    (16, 1024, [0.997, 1.016]), (16, 2048, [1.008, 1.008]), (24, 512, [0.991, 1.003]), (24, 1024, [1.000, 1.009]), (24, 2048, [1.003, 1.013]),
    (32, 512, [1.003, 1.012]), (32, 1024, [1.004, 1.014]), (32, 2048, [1.002, 1.013]),
])
def test_wide_weights_do_not_displace_the_cache(rules, layers, keys, ratios):
    rules.past_cache.argtypes = [ctypes.c_double] * 2
    past = rules.past_cache(layers * keys * 4096 * 4, layers * 4096 * 4096 * 2)
    for ratio in ratios:
        assert (ratio if past else 1.0) <= 1.006 * min(1.0, ratio)


def test_sizes_of_the_gpu_test_of_weights_past_the_cache_take_that_path(rules):
    from test_gpu_many_rows import PAST_CACHE
    rules.past_cache.argtypes = [ctypes.c_double] * 2
    for d, layers, keys in PAST_CACHE:
        assert rules.resid_rows(8, d // 16, d // 32) == 42
        kv, weights = 2 * layers * keys * d * 4, layers * d * d * 2
        assert rules.past_cache(2 * kv, weights) and not rules.past_cache(kv, weights)
    assert not rules.packed(8, 8)


@pytest.mark.parametrize("dense,padded,pays", [
    (2, 4, 1), (1, 4, 1), (5, 8, 1), (6, 8, 1), (8, 10, 1), (10, 12, 1), (13, 16, 1), (14, 32, 1), (80, 96, 1),
    (2, 2, 0), (1, 2, 0), (3, 4, 0), (7, 8, 0), (9, 10, 0), (120, 128, 0),
])
def test_drafts_are_packed_where_it_pays(rules, dense, padded, pays):
    assert rules.packed(dense, padded) == pays
