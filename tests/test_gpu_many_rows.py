"""GPU parity of the GEMM kernels beyond 128 rows at shapes where their row blocks end raggedly: 128- and 256-row blocks
of the LDS-ring kernel, the tile kernel with and without its K split, and the partial sums of squares of 64 columns that
all of them leave for the next RMSNorm.  Element by element against the oracle, with the bars of test_gpu_parity."""
import numpy as np
import pytest

from oracle import odb_oracle as o
from paper_2511_21759_amd import binding as B
from paper_2511_21759_amd import workloads as W
from test_gpu_parity import KV_TOL, LOGIT_TOL, Pair, check_decisions, rel_err, run_prefill_case, run_step_case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPE = dict(n_layers=2, d_model=1024, n_heads=8, head_dim=128, d_ff=3072, vocab=4096, rope_base=10000.0,
             rms_eps=1e-5, mask_id=4095)


@pytest.fixture(scope="module")
def mid():
    p = Pair(SHAPE)
    yield p
    p.close()


@pytest.mark.parametrize("Bn,P,R", [
    (1, 100, 33),      # 9 row tiles: the first count with 64-column partial sums
    (2, 90, 50),       # 18 row tiles: two row blocks of 128, the second almost empty
    (1, 420, 227),     # 647 rows: 41 row tiles, one beyond five blocks of 128
    (3, 140, 193),     # three sequences of an odd length, 63 row tiles
    (1, 700, 303),     # 1003 rows
])
def test_refresh_with_ragged_row_blocks(mid, Bn, P, R):
    wl = W.decode_workload(mid.shape, P, R, 16, 1, 500 + P, batch=Bn)
    run_prefill_case(mid, wl.tokens, wl.resp_off, "%d x %d" % (Bn, P + R))


@pytest.mark.parametrize("Bn,b,S", [
    (1, 16, 9),        # 144 step rows
    (1, 23, 17),       # 34 row tiles, padded rows inside every draft
    (2, 64, 8),        # 1024 step rows
])
def test_step_with_ragged_row_blocks(mid, Bn, b, S):
    wl = W.decode_workload(mid.shape, 70, 90, b, S, 600 + b, batch=Bn)
    cache, oc = run_prefill_case(mid, wl.tokens, wl.resp_off, "step set-up")
    run_step_case(mid, cache, oc, wl.drafts, wl.block_off, 0.9, "%d x %d x %d" % (Bn, S, b))


# ---- dispatch by width: 33 to 256 rows of models between the tiny and the 8B width -------------------------------------

def _width(d, f, layers=1):
    return dict(n_layers=layers, d_model=d, n_heads=d // 128, head_dim=128, d_ff=f, vocab=2048, rope_base=10000.0,
                rms_eps=1e-5, mask_id=2047)


@pytest.mark.parametrize("d,f,rows", [
    (1024, 3072, [(3, 16), (4, 16), (5, 16), (7, 16), (4, 32)]),   # K split over 64-row blocks, one and two n-tiles per group
    (1024, 5120, [(1, 16), (5, 16), (8, 16)]),                     # gate/up in groups of three
    (2048, 2048, [(3, 16), (7, 16)]),                              # K split with two and four n-tiles per block
    (1024, 3072, [(1, 9), (2, 16)]),                               # up to 32 rows: down split over K, one n-tile and a ring of three
    (512, 5120, [(1, 16), (1, 32)]),                               # a ring of one
    (2048, 4096, [(2, 16)]),                                       # two n-tiles, a ring of four
    (2304, 2816, [(2, 16)]),                                       # K that four slices do not divide: all of it, a ring of one (O: of three)
    (2304, 4096, [(2, 16)]),                                       # four n-tiles
    (1024, 10240, [(2, 9)]),                                       # and the other rings: one n-tile, two stages
    (1280, 10240, [(2, 16)]),                                      # two n-tiles, two
    (2304, 10240, [(1, 16)]),                                      # four n-tiles, two
    (1280, 3072, [(2, 16)]),                                       # two n-tiles, three
    (1280, 5120, [(1, 16)]),                                       # and one
    (2304, 3072, [(1, 32)]),                                       # four n-tiles, three
    (2304, 5120, [(2, 16)]),                                       # and one
    (1536, 512, [(7, 16), (4, 32)]),                               # QKV from 97 rows on: blocks of 64 rows and three n-tiles
    (2560, 512, [(7, 16), (4, 32)]),                               # and through LDS
    (2816, 6400, [(7, 16), (4, 32), (9, 16), (16, 16)]),           # all rows through LDS; from 9 row tiles two row blocks for QKV
    (4352, 512, [(7, 16), (4, 32), (1, 16), (2, 16), (4, 7)]),     # QKV of 816 n-tiles: six per workgroup from 97 rows on; O of up to 32 rows,
                                                                   # packed ones too, on the tile kernel
])
def test_step_by_width(d, f, rows):
    p = Pair(_width(d, f))
    try:
        for S, b in rows:
            wl = W.decode_workload(p.shape, 40, 40, b, S, 700 + S)
            cache, oc = run_prefill_case(p, wl.tokens, wl.resp_off, "set-up at d = %d" % d)
            run_step_case(p, cache, oc, wl.drafts, wl.block_off, 0.9, "d = %d, %d x %d" % (d, S, b))
    finally:
        p.close()


@pytest.mark.parametrize("heads,b,S", [
    (8, 32, 8),        # 16 row tiles of one sequence: one row tile per workgroup, not the many-row kernel
    (32, 32, 5),       # 320 one-tile items: two row tiles per workgroup
    (32, 64, 8),       # 128 rows per workgroup pay again
    (2, 16, 20),       # single-tile units, few heads that no XCD mapping takes
])
def test_step_attention_by_size(heads, b, S):
    """The three ways to share the attention of a step out, at the sizes between them."""
    p = Pair(dict(_width(heads * 128, 512), vocab=512, mask_id=511))
    try:
        wl = W.decode_workload(p.shape, 150, 100, b, S, 900 + S)
        cache, oc = run_prefill_case(p, wl.tokens, wl.resp_off, "set-up with %d heads" % heads)
        run_step_case(p, cache, oc, wl.drafts, wl.block_off, 0.9, "%d heads, %d x %d" % (heads, S, b))
    finally:
        p.close()


@pytest.mark.parametrize("heads,dh,b,S", [
    (32, 128, 32, 1),      # 64 workgroups: the channels of an item go to four
    (32, 128, 16, 3),      # 96, and two drafts with padded rows below: two workgroups each
    (32, 128, 23, 2),
    (32, 128, 16, 5),      # 160: one
    (8, 64, 16, 8),        # heads of 64 channels, four workgroups
    (8, 64, 16, 9),        # and two
    (16, 64, 32, 32),      # many rows of heads of 64: 128 of them a workgroup
    (16, 64, 32, 128),     # and 256
])
def test_step_attention_channels_dealt_out(heads, dh, b, S):
    """One-tile attention with the output channels of an item on one, two and four workgroups; many rows of heads of 64."""
    p = Pair(dict(_width(heads * dh, 512), n_heads=heads, head_dim=dh, vocab=512, mask_id=511))
    try:
        wl = W.decode_workload(p.shape, 150, 107, b, S, 920 + S)
        cache, oc = run_prefill_case(p, wl.tokens, wl.resp_off, "set-up with %d heads" % heads)
        run_step_case(p, cache, oc, wl.drafts, wl.block_off, 0.9, "%d heads, %d x %d" % (heads, S, b))
    finally:
        p.close()


@pytest.mark.parametrize("d,f,steps,refresh", [
    (256, 768, [(3, 16), (9, 23)], [(1, 630), (3, 333)]),     # one to four n-tiles per workgroup, O / down in blocks of 32 rows
    (768, 2048, [(5, 16), (3, 43)], [(1, 333)]),              # K of three k-tiles a wave: rings of one stage
    (1024, 3072, [(3, 16), (4, 29)], [(1, 333), (1, 650)]),   # O / down in blocks of 32 x 16, 32 x 64 and 64 x 64
    (1280, 512, [], [(3, 333)]),                              # O in three rounds of blocks
    (1536, 512, [(5, 16), (9, 16)], [(1, 333)]),              # O in blocks of 32 x 32
    (2048, 512, [(3, 16)], [(1, 333), (1, 500)]),             # two rounds of blocks of 64 x 64
    (4096, 512, [(5, 16), (9, 16)], []),                      # O in blocks of 64 x 32 and 64 x 64
    (4096, 4096, [(1, 32), (7, 16)], []),                     # O of 32 rows with K split; gate/up in groups of four
    (2560, 4096, [(3, 16)], []),                              # gate/up of 33 to 128 rows beyond the small blocks: groups of two,
    (2816, 4096, [(4, 16)], []),                              # of two with a ring of one,
    (1792, 6144, [(4, 16)], []),                              # of three,
    (1280, 6144, [(7, 16)], []),                              # of three and eight row tiles,
    (1536, 8192, [(4, 16), (5, 16)], []),                     # of four; down with K split, four n-tiles and a ring of two
    (1280, 8192, [(3, 16)], []),                              # of four with a ring of one
    (1536, 7168, [(5, 16)], []),                              # down with K split, four n-tiles: a ring of one
    (1536, 9216, [(5, 16)], []),                              # and of three
    (1280, 3072, [(3, 16)], []),                              # two n-tiles and a ring of three
    (256, 5120, [(3, 16), (9, 16)], []),                      # one n-tile and a ring of one; sums over 64 columns and a ring of one
    (256, 4096, [(9, 16)], []),                               # and of two
    (256, 8448, [], [(1, 268)]),                              # gate/up in 128 x 256 blocks
    (2560, 256, [], [(1, 268)]),                              # gate/up on the tile kernel with a merge pass
    (3584, 512, [(17, 16)], []),                              # QKV so
])
def test_row_blocks_by_width(d, f, steps, refresh):
    """QKV, gate/up, O and down in small blocks of rows (33 rows and more), the last block and the drafts ragged."""
    p = Pair(dict(_width(d, f), vocab=512, mask_id=511))
    try:
        for S, b in steps:
            wl = W.decode_workload(p.shape, 40, 60, b, S, 760 + S)
            cache, oc = run_prefill_case(p, wl.tokens, wl.resp_off, "set-up at d = %d" % d)
            run_step_case(p, cache, oc, wl.drafts, wl.block_off, 0.9, "d = %d, %d x %d" % (d, S, b))
        for Bn, L in refresh:
            wl = W.decode_workload(p.shape, L - 60, 60, 16, 1, 770 + L, batch=Bn)
            run_prefill_case(p, wl.tokens, wl.resp_off, "d = %d, %d x %d" % (d, Bn, L))
    finally:
        p.close()


# d, layers, cached positions of steps of four sequences in eight row tiles whose O reads its weights past the memory-side cache
# (test_dispatch_cpu.py); rings of one and of four stages
PAST_CACHE = [(2304, 3, 2090), (3072, 3, 1500)]


@pytest.mark.parametrize("b,d,layers,L", [(32, *PAST_CACHE[0]), (29, *PAST_CACHE[1])])
def test_step_whose_weights_are_read_past_the_cache(b, d, layers, L):
    """O in blocks of 64 rows with non-temporal weight loads, where the K/V of four sequences fill the memory-side cache, against the same
    drafts as two sequences of two each, whose weights go through it: both are within the bar of the oracle, so twice that apart."""
    shape = dict(_width(d, 256, layers), vocab=512, mask_id=511)
    wl = W.decode_workload(shape, L - 60, 60, b, 2, 780 + b, batch=2)
    model = B.odb_model_create(shape)
    B.odb_model_init_random(model, W.WEIGHT_SEED, W.WEIGHT_STD)
    out = []
    try:
        for tokens, drafts in ((np.repeat(wl.tokens, 2, axis=0), wl.drafts.reshape(4, 1, b)), (wl.tokens, wl.drafts)):
            cache = B.odb_cache_create(model, len(tokens), L)
            B.odb_prefill(model, cache, torch.from_numpy(np.ascontiguousarray(tokens)).cuda(), wl.resp_off)
            dg = torch.from_numpy(np.ascontiguousarray(drafts)).cuda()
            z, again = (B.odb_block_step_logits(model, cache, dg, wl.block_off, 512).cpu().numpy() for _ in range(2))
            assert np.array_equal(z, again)
            out.append(z.reshape(4, b, 512))
            B.odb_cache_destroy(cache)
        B.odb_model_status(model)
        for i in range(4):
            assert rel_err(out[0][i], out[1][i]) <= 2 * LOGIT_TOL
    finally:
        B.odb_model_destroy(model)


@pytest.mark.parametrize("rows", [(9, 16), (3, 64), (13, 16), (8, 32)])
def test_narrow_step_beyond_128_rows(mid, rows):
    """129 to 256 rows at d = 1024: row blocks of 64 in the streaming kernels, 64-column sums from the K-split kernel."""
    S, b = rows
    wl = W.decode_workload(mid.shape, 60, 90, b, S, 950 + S)
    cache, oc = run_prefill_case(mid, wl.tokens, wl.resp_off, "set-up")
    run_step_case(mid, cache, oc, wl.drafts, wl.block_off, 0.9, "%d x %d" % (S, b))


@pytest.mark.parametrize("L", [300, 600])
def test_refresh_with_slices_that_do_not_divide_k(L):
    """Five and three K slices of the tile kernel at row-block counts that leave a power of two with idle compute units."""
    p = Pair(dict(_width(4096, 512), vocab=512, mask_id=511))
    try:
        wl = W.decode_workload(p.shape, L - 40, 40, 16, 1, 990, batch=1)
        run_prefill_case(p, wl.tokens, wl.resp_off, "%d positions" % L)
    finally:
        p.close()


@pytest.mark.parametrize("d,batch", [
    (4096, 4),         # 2048 rows: O and down in blocks of 256 x 128, two k-tiles per stage
    (3072, 4),         # O in blocks of 128 x 192: sums of squares of 64 columns from waves of 48
    (5120, 4),         # blocks of 256 x 192, the last one two thirds full
    (5120, 2),         # 1024 rows: O in blocks of 128 x 192
])
def test_batched_refresh_equals_its_sequences_one_by_one(d, batch):
    """Wide residual projections in the blocks that many rows take, against the same sequences alone (512 rows, other blocks and
    kernels): logits within the parity bar.  500 positions: the last row tile of every sequence is ragged."""
    import torch
    from paper_2511_21759_amd import binding as B
    shape = dict(_width(d, 512), vocab=512, mask_id=511)
    model = B.odb_model_create(shape)
    try:
        B.odb_model_init_random(model, W.WEIGHT_SEED, W.WEIGHT_STD)
        tok = torch.randint(0, 511, (batch, 500), generator=torch.Generator().manual_seed(d), dtype=torch.int32).cuda()
        many = B.odb_cache_create(model, batch, 500)
        one = B.odb_cache_create(model, 1, 500)
        got = B.odb_prefill_logits(model, many, tok, 300, shape["vocab"])
        for i in range(batch):
            ref = B.odb_prefill_logits(model, one, tok[i:i + 1].contiguous(), 300, shape["vocab"])
            assert (got[i] - ref[0]).abs().max().item() <= 2e-2 * ref.abs().max().item()
            assert not torch.equal(got[i], ref[0])          # another order of sums: the other kernels ran
        B.odb_model_status(model)
        B.odb_cache_destroy(many)
        B.odb_cache_destroy(one)
    finally:
        B.odb_model_destroy(model)


# ---- the fixed scratch area: the same bits as the growing one, up to its limit ------------------------------------------

@pytest.mark.parametrize("d,f,vocab,b,S", [
    (1024, 117248, 32768, 16, 8),      # exactly at the limit with LM statistics per 32 n-tiles; they are written per 8
    (1536, 6144, 4096, 32, 11),        # 352 rows: more K slices than the rest of the area would hold
    (1024, 79104, 160000, 16, 11),     # 176 rows at the limit with LM statistics per 16 n-tiles, none narrower
])
def test_static_scratch_step_adds_in_the_same_order(d, f, vocab, b, S):
    import numpy as np
    from paper_2511_21759_amd import binding as B
    from test_zz_no_alloc import compare, cuda_i32
    shape = dict(_width(d, f), vocab=vocab, mask_id=vocab - 1)
    model = B.odb_model_create(shape)
    try:
        B.odb_model_init_random(model, W.WEIGHT_SEED, W.WEIGHT_STD)
        wl = W.decode_workload(shape, 40, 90, b, S, 700 + S)
        cache = B.odb_cache_create(model, 1, wl.tokens.shape[1])
        B.odb_prefill(model, cache, cuda_i32(wl.tokens), wl.resp_off)
        compare(model, cache, np.ascontiguousarray(wl.drafts), wl.block_off, 0.9, "d %d, d_ff %d, %d rows" % (d, f, b * S))
        B.odb_cache_destroy(cache)
    finally:
        B.odb_model_destroy(model)


def test_scratch_that_cannot_grow_past_the_least_room():
    """A refresh of 1300 positions would take 86 MB for partial sums; with memory for 32 MiB of them it runs all the same, and so
    do the calls behind it."""
    import numpy as np
    import torch
    from paper_2511_21759_amd import binding as B
    shape = dict(_width(4096, 512), vocab=512, mask_id=511)
    wl = W.decode_workload(shape, 1200, 100, 16, 3, 77)
    tok, dr = (torch.from_numpy(np.ascontiguousarray(x, np.int32)).cuda() for x in (wl.tokens, wl.drafts))
    out = []
    for limit in (None, 120 << 20):
        model = B.odb_model_create(shape)
        B.odb_model_init_random(model, W.WEIGHT_SEED, W.WEIGHT_STD)
        cache = B.odb_cache_create(model, 1, 1300)
        whole, refused = torch.empty, []
        if limit:
            def empty(n, **kw):
                if isinstance(n, int) and n > limit:
                    refused.append(n)
                    raise RuntimeError("out of memory")
                return whole(n, **kw)
            torch.empty = empty
        try:
            a = [t.clone() for t in B.odb_prefill(model, cache, tok, wl.resp_off)]
            n_refused = len(refused)
            a += [t.clone() for t in B.odb_block_step(model, cache, dr, wl.block_off, 0.9)]
            B.odb_prefill(model, cache, tok, wl.resp_off)
            B.odb_model_status(model)
            assert len(refused) == n_refused == (1 if limit else 0), "asked once, not on every call"
        finally:
            torch.empty = whole
            B.odb_cache_destroy(cache)
            B.odb_model_destroy(model)
        out.append(a)
    for i in (0, 2):
        assert torch.allclose(torch.log(out[0][i]), torch.log(out[1][i]), atol=2e-2)


@pytest.mark.parametrize("vocab", [50000, 70000])
def test_lm_head_of_one_row_block_with_a_ragged_last_block(vocab):
    """33 to 128 rows against vocabularies that take blocks of 256 (up to 65536 columns) and 512 columns and fill the last one in part;
    most winning tokens are in that block."""
    assert vocab % (512 if vocab > 65536 else 256) != 0
    p = Pair(dict(n_layers=1, d_model=256, n_heads=2, head_dim=128, d_ff=256, vocab=vocab, rope_base=10000.0, rms_eps=1e-5, mask_id=5))
    try:
        lm = np.random.default_rng(vocab).normal(0, 0.02, (vocab, 256)).astype(np.float32)
        lm[-24:] *= 6
        p.set(o.T_LM, 0, lm)
        for S, b in ((3, 16), (8, 16)):
            wl = W.decode_workload(p.shape, 20, 30, b, S, 40 + S)
            cache, oc = run_prefill_case(p, wl.tokens, wl.resp_off, "set-up")
            _, am, _, _ = run_step_case(p, cache, oc, wl.drafts, wl.block_off, 0.9, "vocab %d, %d x %d" % (vocab, S, b))
            assert (am >= vocab - 24).mean() > 0.5
    finally:
        p.close()


# ---- blocks of 192 and 320 rows, and a last round split over two workgroups a block, each at the smallest sizes that take it -------

# d, d_ff, rows, which projections run in which blocks (test_dispatch_cpu.py: the plans of these sizes)
TALL = [
    (256, 8192, 267, {"gate/up": 1231}),       # 192 x 192: a row block of 75 rows behind a whole one
    (256, 5120, 779, {"gate/up": 1241}),
    (256, 12288, 523, {"gate/up": 2031}),
    (256, 6144, 1291, {"gate/up": 2041}),
    (1024, 256, 2059, {"qkv": 1231}),          # the heads' boundaries inside a wave's columns
]


@pytest.mark.parametrize("d,f,rows,plans", TALL)
def test_refresh_in_blocks_of_192_and_320_rows(d, f, rows, plans):
    p = Pair(_width(d, f))
    try:
        wl = W.decode_workload(p.shape, rows - 40, 40, 8, 1, 900 + d)
        run_prefill_case(p, wl.tokens, wl.resp_off, "d %d, d_ff %d, %d rows" % (d, f, rows))
    finally:
        p.close()


# The same where it takes more rows: sequences of 16 * tiles - 5 positions, the last by the oracle, the others as they come out alone (in the
# blocks of fewer rows): each is within the bar of the oracle, so twice that apart.
# d, d_ff, sequences, row tiles of each, which projections run in which blocks
TALL_BATCH = [
    (1280, 256, 5, 29, {"qkv": 1241}),
    (1536, 256, 7, 23, {"qkv": 2031}),
    (1792, 256, 13, 13, {"qkv": 2041}),
    (2304, 256, 7, 23, {"O": 1231, "down": 1231}),      # sums of squares over 64 columns from waves of 48
    (3328, 256, 7, 23, {"O": 1241, "down": 1241}),
    (4352, 1536, 7, 23, {"O": 2031, "down": 2031}),
    (4864, 256, 7, 23, {"O": 2041}),
]


@pytest.mark.parametrize("d,f,batch,tiles,plans", TALL_BATCH)
def test_refresh_of_a_batch_in_blocks_of_192_and_320_rows(d, f, batch, tiles, plans):
    p, L, off, H = Pair(_width(d, f)), 16 * tiles - 5, 16, d // 128
    try:
        wl = W.decode_workload(p.shape, off, L - off, 8, 1, 900 + d, batch=batch)
        tokens, cache = torch.from_numpy(wl.tokens).cuda(), p.cache(batch, L)
        logits = B.odb_prefill_logits(p.model, cache, tokens, off, p.cfg.vocab).cpu().numpy()
        conf, am = B.odb_prefill(p.model, cache, tokens, off)
        c, conf_o, am_o, z = o.prefill(p.cfg, p.w, wl.tokens[-1], off, return_logits=True)
        assert rel_err(logits[-1], z) <= LOGIT_TOL
        check_decisions(conf[-1].cpu().numpy(), am[-1].cpu().numpy(), conf_o, am_o, z, np.abs(logits[-1] - z).max(), "last sequence")
        for kv, ref in ((0, c.k[0]), (1, c.v[0])):
            assert rel_err(B.odb_cache_read(cache, 0, kv, batch - 1, 0, L, H, 128), ref) <= KV_TOL
        one = p.cache(1, L)
        for i in range(batch):
            alone = B.odb_prefill_logits(p.model, one, tokens[i:i + 1].contiguous(), off, p.cfg.vocab).cpu().numpy()
            assert rel_err(logits[i], alone[0]) <= 2 * LOGIT_TOL, "sequence %d" % i
            for kv in (0, 1):
                got, ref = (B.odb_cache_read(x, 0, kv, j, 0, L, H, 128) for x, j in ((cache, i), (one, 0)))
                assert rel_err(got, ref) <= 2 * KV_TOL, "sequence %d" % i
        B.odb_model_status(p.model)
    finally:
        p.close()


# d, d_ff, rows, which projection's blocks (test_dispatch_cpu.py: the plans of these sizes)
SPLIT = [
    (3328, 10240, 971, "gate/up"),     # 32 whole blocks of an XCD and eight split ones, the last row block ragged
    (3328, 6144, 1643, "down"),        # 14 split blocks, no whole ones
    (3840, 256, 1931, "qkv"),          # 32 whole ones and 16 split, with V's transposition
]


@pytest.mark.parametrize("d,f,rows,which", SPLIT)
def test_split_last_round_repeats_and_agrees_with_whole_blocks(d, f, rows, which):
    """Blocks of 256 x 256, of which those of the last round are split over two workgroups.  The same bits whichever of the two arrives
    last, launch after launch on the same counters, and the whole blocks' values up to the order of two fp32 sums, which may turn every
    rounding to binary16 behind them: a head input that is rounded differently moves a logit by 2^-11 / sqrt(3) of its deviation
    0.02 sqrt(d), and a confidence by as much; four times that for the roundings in front of it and both sides."""
    p = Pair(_width(d, f, layers=2))
    H = d // 128
    try:
        wl = W.decode_workload(p.shape, rows - 95, 95, 8, 1, 77)
        tokens, cache = torch.from_numpy(wl.tokens).cuda(), p.cache(1, wl.tokens.shape[1])
        first = [x.clone() for x in B.odb_prefill(p.model, cache, tokens, wl.resp_off)]
        kv = B.odb_cache_read(cache, 1, 0, 0, 0, rows, H, 128)
        for _ in range(8):
            again = B.odb_prefill(p.model, cache, tokens, wl.resp_off)
            assert torch.equal(first[0], again[0]) and torch.equal(first[1], again[1])
        assert np.array_equal(kv, B.odb_cache_read(cache, 1, 0, 0, 0, rows, H, 128))
        B.odb_set_option(p.model, B.OPT_KSPLIT_REDUCE, 0)
        whole = B.odb_prefill(p.model, cache, tokens, wl.resp_off)
        assert float((whole[0].double() - first[0].double()).norm() / whole[0].double().norm()) <= 4 * 2.0 ** -11 / 3 ** 0.5 * 0.02 * d ** 0.5
        kv_whole = B.odb_cache_read(cache, 1, 0, 0, 0, rows, H, 128)
        # (a key is rounded to binary16: half a unit in the last place of the largest, twice as one of each side)
        assert np.abs(kv - kv_whole).max() <= 2 * 2.0 ** -11 * np.abs(kv_whole).max()
        B.odb_model_status(p.model)
        if which == "qkv":
            B.odb_set_option(p.model, B.OPT_KSPLIT_REDUCE, 1)
            assert (rows + 15) // 16 == 11 * 11            # as many row tiles in eleven sequences
            wl = W.decode_workload(p.shape, 100, 11 * 16 - 5 - 100, 8, 1, 78, batch=11)
            run_prefill_case(p, wl.tokens, wl.resp_off, "QKV in split blocks")
    finally:
        p.close()


# ---- drafts packed densely -------------------------------------------------------------------------------------------------------

# d, head_dim, d_ff, batch, b, S, QKV's kernel and the attention's way behind 110 cached positions (test_dispatch_cpu.py: that these sizes take them)
DENSE = [
    (1024, 128, 512, 1, 7, 4, "few", 1),           # two row tiles; units that begin inside a tile, keys of two drafts in a lane's four rows
    (1536, 128, 512, 1, 7, 4, "few", 1),           # two n-tiles a workgroup
    (2816, 128, 512, 1, 7, 4, "few", 1),           # three
    (1792, 128, 512, 1, 7, 4, "few", 1),           # two, a ring of one
    (256, 64, 512, 3, 5, 4, "rows 21", 1),         # heads of 64, four row tiles
    (1024, 128, 512, 1, 1, 40, "rows 22", 1),      # drafts of one row
    (1024, 128, 512, 1, 33, 4, "rows 24", 1),      # three tiles and two key tiles a draft: nine row tiles
    (1024, 128, 512, 1, 11, 9, "rows 23", 1),      # nine padded tiles, seven packed
    (1280, 128, 512, 1, 12, 8, "rows 23", 1),      # a ring of one
    (2304, 128, 512, 1, 5, 13, "rows 44", 1),
    (2560, 128, 512, 1, 20, 6, "rows 44", 1),
    (1792, 128, 512, 1, 20, 6, "rows 43", 1),
    (1536, 128, 512, 1, 20, 6, "rows 43", 1),
    (2816, 128, 512, 1, 9, 6, "stream", 1),        # four row tiles in the streaming kernel of 64 rows
    (2816, 128, 512, 1, 5, 13, "stream", 1),       # five row tiles in the streaming kernel of 96 rows
    (2816, 128, 512, 1, 24, 5, "slab 3", 1),       # eight row tiles through LDS
    (2816, 128, 512, 1, 20, 8, "slab 6", 2),       # ten, two row blocks
    (2304, 128, 512, 1, 36, 5, "slab 6", 2),       # twelve, weights of both row blocks past the cache
    (1024, 128, 512, 1, 20, 16, "rows 24", 1),     # 20 row tiles
    (1024, 128, 512, 2, 9, 32, "rows 24", 1),      # 36
    (3584, 128, 512, 1, 52, 5, "tile", 3),         # the tile kernel and its merge pass; the many-row attention, four tiles a draft
    (2048, 128, 512, 1, 51, 8, "big 821", 2),      # 128-row blocks: 26 row tiles of 32
    (512, 128, 512, 1, 50, 41, "big 831", 3),
    (1280, 128, 512, 1, 7, 183, "big 841", 1),
    (768, 128, 512, 1, 50, 41, "big 1621", 3),     # 256-row blocks
    (768, 128, 512, 1, 53, 58, "big 1631", 3),
    (1792, 128, 512, 1, 50, 41, "big 1641", 3),
    (512, 128, 512, 1, 25, 164, "big 1231", 3),    # 192-row blocks, 257 row tiles
    (2048, 128, 512, 1, 20, 80, "big 1241", 3),
    (1536, 128, 512, 2, 39, 33, "big 2031", 2),    # 320-row blocks
    (1280, 128, 512, 2, 25, 82, "big 2041", 3),
    (3840, 128, 512, 1, 17, 113, "big 1642", 3),   # the last round split
]


@pytest.mark.parametrize("d,dh,f,batch,b,S", [case[:6] for case in DENSE] + [
    (1024, 128, 512, 1, 33, 2),      # six padded tiles, five packed: they stay padded
])
def test_step_with_dense_rows(d, dh, f, batch, b, S):
    p = Pair(dict(_width(d, f), n_heads=d // dh, head_dim=dh))
    try:
        wl = W.decode_workload(p.shape, 50, 60, b, S, 800 + b, batch=batch)
        cache, oc = run_prefill_case(p, wl.tokens, wl.resp_off, "set-up at d = %d" % d)
        run_step_case(p, cache, oc, wl.drafts, wl.block_off, 0.9, "d = %d, %d x %d x %d" % (d, batch, S, b))
        # the same bits whatever the scratch held before: another step and another refresh between two of the same
        dg, tokens = torch.from_numpy(wl.drafts).cuda(), torch.from_numpy(wl.tokens).cuda()
        first = [x.clone() for x in B.odb_block_step(p.model, cache, dg, wl.block_off, 0.9)]
        B.odb_block_step(p.model, cache, (dg + 1) % p.shape["vocab"], wl.block_off, 0.9)
        B.odb_prefill(p.model, cache, tokens, wl.resp_off)
        for x, y in zip(first, B.odb_block_step(p.model, cache, dg, wl.block_off, 0.9)):
            assert torch.equal(x, y)
        B.odb_model_status(p.model)
    finally:
        p.close()


def test_dense_rows_in_the_fixed_area():
    p = Pair(_width(1024, 512))
    try:
        wl = W.decode_workload(p.shape, 50, 60, 7, 4, 31)
        cache = p.cache(1, wl.tokens.shape[1])
        B.odb_prefill(p.model, cache, torch.from_numpy(wl.tokens).cuda(), wl.resp_off)
        dg = torch.from_numpy(wl.drafts).cuda()
        want = B.odb_block_step(p.model, cache, dg, wl.block_off, 0.9)
        got = B.odb_block_step_static(p.model, cache, dg, wl.block_off, 0.9, *[torch.empty_like(x) for x in want])
        for x, y in zip(want, got):
            assert torch.equal(x, y)
    finally:
        p.close()
