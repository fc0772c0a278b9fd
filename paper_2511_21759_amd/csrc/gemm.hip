// Stand-alone launches of the weight-streaming GEMM (see gemm_core.h).
#include "choose.h"
#include "gemm_slab.h"
#include "launch.h"

namespace odb {

template <int MT, int NG, int PF, class Epi, bool IL = false, bool NTW = true>
__global__ __launch_bounds__(64 * WK) void gemm_stream_kernel(GemmArgs g, Epi epi) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    gemm_wg<MT, NG, PF, Epi, IL, NTW>(g, epi, blockIdx.x, blockIdx.y * MT, smem);
}

constexpr int kStreamWGs = kComputeUnits;      // one workgroup per compute unit
// Every workgroup of the streaming kernels reads the same activation tiles; started at the same k-tile they ask the
// same L2 channels for them at the same time.  Workgroup wg starts kKRot * wg k-tiles further on and wraps round
// (7 is coprime to the 12 and 16 k-tiles per wave of the 8B shape; of 1, 3, 5 and 7 the multipliers 3 and 7 leave the
// 32-row gate/up kernel at its 33.0 us, 1 and 5 cost it 0.6 us): the down projection 22.5 -> 20.7 us at 32 rows,
// gate/up 49.0 -> 47.4 us at 128 rows; the order of a workgroup's fp32 sums depends on its index, not on the run.
constexpr int kKRot = 7;

// The streaming kernel with K split over KS workgroups per block of n-tiles, for projections whose activations
// are long (the down projection: every workgroup of the plain kernel reads all 32 x 12288 of them through L2,
// which costs as much as a third of its weight stream).  Workgroup (n-block, ks) adds k-slice ks for NG n-tiles
// and leaves its sums in partial[ks]; each workgroup then bumps the block's arrival counter, and the one that
// arrives last adds the KS partial sums in slice order (so the result does not depend on who was last) and runs
// the epilogue.  Nobody waits: the other workgroups simply exit.  Partial sums and counter travel as
// device-coherent accesses, ordered by a wait for the stores' completion before the counter is touched; cache-wide
// fences (a release / acquire pair) were measured to stall the weight streams of every workgroup on the chip
// (108 us instead of 20 us in a traffic model of this kernel).  The counter is back at zero when the kernel ends.
// What follows the k-loop is a chain of latencies - sums through LDS, stores out, counter, sums back in: 16-byte accesses, one
// pass through LDS and all of a wave's tiles requested at once took O and down of 64 rows at d 4096 from 20.4 to 19.9 us on average,
// down of 32 rows from 20.6 to 20.2, and at d 1024, 128 rows O from 7.2 to 6.6 and down from 8.5 to 7.9.
// (RB: blockIdx.y numbers blocks of MT row tiles.  SPAN64: sums of squares over 64 columns, NormOut::span; with NG = 4 and N a
// multiple of 64 a block is one such sum.)
template <int MT, int NG, int PF, int KS, bool RB = false, bool SPAN64 = false>
__global__ __launch_bounds__(64 * WK) void gemm_stream_ksplit_kernel(GemmArgs g, EpiResid epi, float *partial, unsigned *arrive) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    static_assert(!SPAN64 || NG == 4, "one sum per block");
    float *s_q = reinterpret_cast<float *>(smem);            // (SPAN64) [MT * NG][16], in the finishing workgroup
    __shared__ unsigned s_old;
    const int ks = blockIdx.x % KS, nb = blockIdx.x / KS, nblocks = g.nwg;
    GemmArgs gs = g;
    gs.A += (size_t)ks * g.k_len * g.MT_total * kTileElems;
    gs.W += (size_t)ks * g.k_len * kTileElems;
    const size_t slice = (size_t)g.MT_total * g.NT * 256;
    const int mt0 = RB ? blockIdx.y * MT : 0, mt1 = RB && mt0 + MT < g.MT_total ? mt0 + MT : g.MT_total;
    gemm_wg<MT, NG, PF, EpiPartial, false>(gs, EpiPartial{partial + ks * slice, g.NT, g.MT_total}, nb, mt0, smem);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wave's partial sums have been written
    __syncthreads();
    arrive += RB ? blockIdx.y * nblocks + nb : nb;
    if (threadIdx.x == 0) s_old = __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s_old != KS - 1) return;
    // The slices of all tiles of a wave are requested together with what the epilogue reads.
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    constexpr int TW = (MT * NG + WK - 1) / WK;             // tiles of a wave
    u32x4 v[TW][KS];
    ResidPre pre[TW];
    auto tile_of = [&](int u, int &mt, int &nt) __attribute__((always_inline)) {      // (every block has NG n-tiles: set at the launch)
        const int t = wv + u * WK;
        mt = mt0 + t / NG;
        nt = nb * NG + t % NG;
        return t < MT * NG && mt < mt1;
    };
#pragma unroll
    for (int u = 0; u < TW; u++) {
        int mt, nt;
        if (!tile_of(u, mt, nt)) continue;
        const unsigned at = ((unsigned)mt * g.NT + nt) * 1024 + lane * 16;
#pragma unroll
        for (int s = 0; s < KS; s++)
            v[u][s] = __builtin_amdgcn_raw_buffer_load_b128(sums_rsrc(partial + s * slice, slice * 4), at, 0, kDeviceScope);
        pre[u] = epi_preload(epi, mt, nt, lane);
    }
#pragma unroll
    for (int u = 0; u < TW; u++) {
        int mt, nt;
        if (!tile_of(u, mt, nt)) continue;
        f32x4 c = __builtin_bit_cast(f32x4, v[u][0]);
#pragma unroll
        for (int s = 1; s < KS; s++) c += __builtin_bit_cast(f32x4, v[u][s]);
        if constexpr (SPAN64) {                     // the block's four n-tiles make one partial sum of squares
            const float sq = EpiResid::over_row(epi.put(mt, nt, c, lane, pre[u]));
            if (lane < 16) s_q[(wv + u * WK) * 16 + lane] = sq;
        } else {
            epi_apply(epi, mt, nt, c, lane, 0, pre[u]);
        }
    }
    if constexpr (SPAN64) {
        __syncthreads();
        for (int i = threadIdx.x; i < (mt1 - mt0) * 16; i += 64 * WK) {
            const float *p = s_q + (i >> 4) * 64 + (i & 15);
            epi.no.ssq[(size_t)(mt0 * 16 + i) * epi.no.n_ssq + nb] = (p[0] + p[16]) + (p[32] + p[48]);
        }
    }
    if (threadIdx.x == 0) __hip_atomic_store(arrive, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kSplitKS = 4, kSplitNG = 4, kSplitPF = 4;      // (2 x 2 n-tiles, rings of 2, 6 and 8 measured slower)
static bool ksplit_fits(GemmShape sh, int nblocks, Workspace ws) {       // nblocks: blocks of rows and n-tiles
    return ws.arrive && nblocks * kSplitKS <= kStreamWGs && nblocks <= 1024 &&
           (size_t)kSplitKS * sh.M_tiles * sh.N_tiles * 1024 <= ws.partial_bytes;
}
// shapes the K-split kernel takes: 33 to 96 rows without a fused norm, n-blocks x KS workgroups within the chip,
// k-slices that the waves and the ring divide, room for the partial sums
static bool ksplit_ok(GemmShape sh, Workspace ws) {
    return sh.M_tiles > 2 && sh.M_tiles <= 6 && sh.K_tiles % (kSplitKS * WK * kSplitPF) == 0 &&
           ksplit_fits(sh, (sh.N_tiles + kSplitNG - 1) / kSplitNG, ws);
}
static GemmArgs stream_args(const u16 *a, const u16 *w, GemmShape sh, NormIn ni, int k_len, int nwg) {
    GemmArgs g;
    g.A = a; g.W = w; g.KT = sh.K_tiles; g.MT_total = sh.M_tiles; g.NT = sh.N_tiles;
    g.ssq = ni.ssq; g.n_ssq = ni.n_ssq; g.eps = ni.eps; g.inv_d = 1.0f / (float)(sh.K_tiles * 32);
    g.k_len = k_len; g.k_rot = kKRot;
    set_shares(g, nwg);
    return g;
}
template <int MT, int NG, int PF, int KS, bool RB = false, bool SPAN64 = false>
static void launch_ksplit_as(const u16 *a, const u16 *w, GemmShape sh, EpiResid e, Workspace ws, hipStream_t s) {
    // (N is a multiple of 256, so the blocks have NG n-tiles each)
    const GemmArgs g = stream_args(a, w, sh, NormIn{nullptr, 0, 0.f}, sh.K_tiles / KS, sh.N_tiles / NG);
    const dim3 grid(g.nwg * KS, RB ? (sh.M_tiles + MT - 1) / MT : 1);
    constexpr int lds = gemm_smem_bytes(MT, NG);
    allow_lds<gemm_stream_ksplit_kernel<MT, NG, PF, KS, RB, SPAN64>>(lds);
    gemm_stream_ksplit_kernel<MT, NG, PF, KS, RB, SPAN64><<<grid, 64 * WK, lds, s>>>(g, e, ws.partial, ws.arrive);
}
template <int NG>
static void launch_ksplit_few(const u16 *a, const u16 *w, GemmShape sh, EpiResid e, Workspace ws, hipStream_t s) {
    const int kw = sh.K_tiles / (kSplitKS * WK);
    if (kw % 4 == 0) launch_ksplit_as<2, NG, 4, kSplitKS>(a, w, sh, e, ws, s);
    else if (kw % 3 == 0) launch_ksplit_as<2, NG, 3, kSplitKS>(a, w, sh, e, ws, s);
    else if (kw % 2 == 0) launch_ksplit_as<2, NG, 2, kSplitKS>(a, w, sh, e, ws, s);
    else launch_ksplit_as<2, NG, 1, kSplitKS>(a, w, sh, e, ws, s);
}
static void launch_stream_ksplit(const u16 *a, const u16 *w, GemmShape sh, EpiResid e, Workspace ws, hipStream_t s) {
    if (sh.M_tiles <= 4) launch_ksplit_as<4, kSplitNG, 4, kSplitKS>(a, w, sh, e, ws, s);
    else launch_ksplit_as<6, kSplitNG, 2, kSplitKS>(a, w, sh, e, ws, s);
}

// The same kernel for narrow models (N up to 2048 from 33 to 128 rows, up to 1024 from 129 to 256): blocks of 64 rows and one, two or four n-tiles, so
// that four k-slices of every block make up to 256 workgroups, and as many ring stages as a wave has k-tiles where that is two
// or three.  At d = 1024, d_ff = 3072 and 128 rows it replaces the tile kernel on 32 and 64 workgroups and its merge pass:
// O 6.7 + 3.7, down 9.0 + 3.7 us before, 6.6 and 7.9 now (blocks of all 128 rows and one n-tile: 7.4 and 9.7 us); at 192 rows
// 7.6 + 4.4 and 11.6 + 4.4 before, 9.3 and 11.7 now.
static int ksplit_narrow_ng(GemmShape sh, Workspace ws) {
    if (sh.M_tiles <= 2 || sh.M_tiles > 16 || sh.K_tiles % (kSplitKS * WK) != 0) return 0;
    const int rb = (sh.M_tiles + 3) / 4, ng = sh.N_tiles <= 64 ? (rb <= 2 ? rb : 4) : sh.N_tiles <= 128 && rb <= 2 ? 2 * rb : 0;
    return ng && ksplit_fits(sh, (sh.N_tiles + ng - 1) / ng * rb, ws) ? ng : 0;
}
template <int NG, bool SPAN64 = false>
static void launch_ksplit_narrow(const u16 *a, const u16 *w, GemmShape sh, EpiResid e, Workspace ws, hipStream_t s) {
    const int kw = sh.K_tiles / (kSplitKS * WK);
    if (kw % 3 == 0) launch_ksplit_as<4, NG, 3, kSplitKS, true, SPAN64>(a, w, sh, e, ws, s);
    else if (kw % 2 == 0) launch_ksplit_as<4, NG, 2, kSplitKS, true, SPAN64>(a, w, sh, e, ws, s);
    else launch_ksplit_as<4, NG, 1, kSplitKS, true, SPAN64>(a, w, sh, e, ws, s);
}

// The persistent streaming kernel for up to 128 rows: MT row tiles per wave (2, 4, 6 or 8: 32-row steps),
// NG n-tiles per group, a PF-deep ring.
// The per-projection choices below are the fastest measured on MI355X; K_tiles that the ring depth does not
// divide fall back to a ring of one.
template <int MT, int NG, int PF, bool IL, bool NTW = true, class Epi>
static void launch_stream(const u16 *a, const u16 *w, GemmShape sh, NormIn ni, Epi e, hipStream_t s) {
    const int kw = sh.K_tiles / WK;                // K_tiles is a multiple of 8 (checked at model creation)
    const int groups = (sh.N_tiles + NG - 1) / NG;
    dim3 grid(groups < kStreamWGs ? groups : kStreamWGs, (sh.M_tiles + MT - 1) / MT);
    const GemmArgs g = stream_args(a, w, sh, ni, sh.K_tiles, grid.x);
    constexpr int lds = gemm_smem_bytes(MT, NG);
    if (kw % PF == 0) {
        allow_lds<gemm_stream_kernel<MT, NG, PF, Epi, IL, NTW>>(lds);
        gemm_stream_kernel<MT, NG, PF, Epi, IL, NTW><<<grid, 64 * WK, lds, s>>>(g, e);
    } else {
        allow_lds<gemm_stream_kernel<MT, NG, 1, Epi, IL, NTW>>(lds);
        gemm_stream_kernel<MT, NG, 1, Epi, IL, NTW><<<grid, 64 * WK, lds, s>>>(g, e);
    }
}

// O and down beyond 128 rows, whose sums of squares cover 64 columns: blocks of 32 or 64 rows (MT) and 64 columns with all of K in a
// workgroup, so that nothing is exchanged and no merge pass follows.  Where they are taken: choose.h.
constexpr int kBlockNG = 4;
template <int MT>
__global__ __launch_bounds__(64 * WK) void gemm_block_kernel(GemmArgs g, EpiResid epi) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int NG = kBlockNG;
    float *s_q = reinterpret_cast<float *>(smem + gemm_smem_bytes(MT, NG));
    // ids go round-robin over the XCDs: the row blocks of a column of blocks meet on one, which then fetches its weights once
    const int rb = (g.MT_total + MT - 1) / MT, j = blockIdx.x >> 3, nb = (j / rb) * 8 + (blockIdx.x & 7), mt0 = (j % rb) * MT;
    if (nb >= g.nwg) return;
    gemm_wg<MT, NG, 1, EpiResidSums<NG>, true, false>(g, EpiResidSums<NG>{epi, s_q, mt0, nb * NG}, nb, mt0, smem);
    __syncthreads();
    if (epi.no.hb && threadIdx.x < MT * 16 && mt0 * 16 + threadIdx.x < g.MT_total * 16) {
        const float *p = s_q + (threadIdx.x >> 4) * (NG * 16) + (threadIdx.x & 15);
        epi.no.ssq[(size_t)(mt0 * 16 + threadIdx.x) * epi.no.n_ssq + nb] = (p[0] + p[16]) + (p[32] + p[48]);
    }
}
template <int MT>
static void launch_block(const u16 *a, const u16 *w, GemmShape sh, EpiResid e, hipStream_t s) {
    // (N is a multiple of 256: every block has four n-tiles)
    const GemmArgs g = stream_args(a, w, sh, NormIn{nullptr, 0, 0.f}, sh.K_tiles, sh.N_tiles / kBlockNG);
    const int rb = (sh.M_tiles + MT - 1) / MT, grid = 8 * rb * ((g.nwg + 7) / 8);
    constexpr int lds = gemm_smem_bytes(MT, kBlockNG) + MT * kBlockNG * 16 * 4;
    allow_lds<gemm_block_kernel<MT>>(lds);
    gemm_block_kernel<MT><<<grid, 64 * WK, lds, s>>>(g, e);
}

// Narrow models: a projection whose n-tiles give fewer than 256 groups of the usual width takes smaller groups, the
// smallest that still fit one per compute unit (the groups below were picked for N = 12288 and 24576; at d = 1024 they
// leave three quarters of the chip idle: QKV of 128 rows 14.9 us and gate/up 17.9 us on 64 workgroups).  `widest` is
// the usual group, `has3` whether a group of three exists beside one and two.
static int stream_ng(int n_tiles, int widest, bool has3) {
    if (n_tiles <= kStreamWGs) return 1;
    if (n_tiles <= 2 * kStreamWGs) return 2;
    if (has3 && n_tiles <= 3 * kStreamWGs) return 3;
    return widest;
}
// QKV and gate/up in small blocks of rows (choose.h: row_block).  Several row blocks read a weight tile: ordinary loads, through L2.
// With 32 rows and four n-tiles the ring has one stage, so that two workgroups share a compute unit.
template <class Epi>
static void launch_row_blocks(RowBlock b, const u16 *a, const u16 *w, GemmShape sh, NormIn ni, Epi e, hipStream_t s) {
    if (b.mt == 4 && b.ng == 3) launch_stream<4, 3, 2, true, false>(a, w, sh, ni, e, s);
    else if (b.mt == 4) launch_stream<4, 4, 2, true, false>(a, w, sh, ni, e, s);
    else if (b.ng == 1) launch_stream<2, 1, 1, true, false>(a, w, sh, ni, e, s);
    else if (b.ng == 2) launch_stream<2, 2, 2, true, false>(a, w, sh, ni, e, s);
    else if (b.ng == 3) launch_stream<2, 3, 4, true, false>(a, w, sh, ni, e, s);
    else launch_stream<2, 4, 1, true, false>(a, w, sh, ni, e, s);
}

// n-tiles of a workgroup of the tile kernel
static int tile_columns(int m_tiles) { return m_tiles > 8 ? 16 : 8; }

template <class Epi> constexpr TileEpilogue tile_epilogue_of = TileEpilogue::resid;
template <> constexpr TileEpilogue tile_epilogue_of<EpiQKV> = TileEpilogue::qkv;
template <> constexpr TileEpilogue tile_epilogue_of<EpiQKVDense> = TileEpilogue::qkv;
template <> constexpr TileEpilogue tile_epilogue_of<EpiSwiGLU> = TileEpilogue::swiglu;

template <class Epi>
static void launch_tile(const u16 *a, const u16 *w, GemmShape sh, NormIn ni, Epi e, Workspace ws, bool may_split,
                        hipStream_t s) {
    TileArgs g;
    g.A = a; g.W = w; g.KT = sh.K_tiles; g.MT_total = sh.M_tiles; g.NT = sh.N_tiles;
    g.ssq = ni.ssq; g.n_ssq = ni.n_ssq; g.eps = ni.eps; g.inv_d = 1.0f / (float)(sh.K_tiles * 32);
    g.partial = ws.partial;
    const int m_blocks = (sh.M_tiles + 7) / 8;
    const int per_wg = tile_columns(sh.M_tiles);
    g.n_blocks = (sh.N_tiles + per_wg - 1) / per_wg;
    const int ks = may_split ? tile_slices(tile_epilogue_of<Epi>, sh.M_tiles, sh.N_tiles, sh.K_tiles, ws.partial_bytes) : 1;
    g.KS = ks;
    dim3 grid(g.n_blocks * ks, m_blocks);
    // (8 waves x 1 n-tile, ring of 8) for the multi-draft step, (8 x 2, ring of 4) for compute-bound shapes:
    // the best of the shapes tried on MI355X (4-wave workgroups of 1, 2 or 4 n-tiles per wave, 8 x 2 with a ring of 8
    // and 2 or 4 k-tiles per barrier were all slower or equal - occupancy beats wider tiles here; 8 x 4 spills)
    // (a single block of rows, which O and down alone bring here: every weight tile is read once, non-temporally)
    if (is_resid<Epi>::value && m_blocks == 1) {
        if constexpr (is_resid<Epi>::value) gemm_tile_kernel<1, 8, Epi, true><<<grid, 512, 0, s>>>(g, e);
    } else {
        gemm_tile_kernel<2, 4, Epi><<<grid, 512, 0, s>>>(g, e);
    }
    if (ks > 1) {
        if constexpr (!is_row_stats<Epi>::value)
            tile_epilogue_kernel<Epi><<<dim3((sh.N_tiles + 7) / 8, sh.M_tiles), 512, 0, s>>>(g, e);
    }
}

// blocks of MBT x 16 rows through LDS (gemm_big.h), 64 * WN columns wide
template <int WN, class Epi, int MBT = 16, int KS = 1>
static void launch_big_wn(const u16 *a, const u16 *w, GemmShape sh, NormIn ni, Epi e, hipStream_t s, Workspace ws = Workspace{}) {
    BigArgs g;
    g.A = a; g.W = w; g.KT = sh.K_tiles; g.MT_total = sh.M_tiles; g.NT = sh.N_tiles;
    g.ssq = ni.ssq; g.n_ssq = ni.n_ssq; g.eps = ni.eps; g.inv_d = 1.0f / (float)(sh.K_tiles * 32);
    g.m_blocks = (sh.M_tiles + MBT - 1) / MBT;
    g.n_blocks = (sh.N_tiles + 4 * WN - 1) / (4 * WN);
    g.partial = ws.partial; g.exchange = ws.exchange;
    const int per_xcd = big_per_xcd(MBT, WN, sh.M_tiles, sh.N_tiles);
    g.whole = KS > 1 ? per_xcd / kXcdUnits * kXcdUnits : per_xcd;
    allow_lds<gemm_big_kernel<WN, Epi, MBT, KS>>(big_smem_bytes(WN, MBT));
    dim3 grid(8 * (g.whole + (per_xcd - g.whole) * KS));
    gemm_big_kernel<WN, Epi, MBT, KS><<<grid, 512, big_smem_bytes(WN, MBT), s>>>(g, e);
}

static BigChoice big_choice(GemmShape sh) { return big_choice(sh.M_tiles, sh.N_tiles, sh.K_tiles); }

template <class Epi>
static void launch_big_as(BigChoice c, const u16 *a, const u16 *w, GemmShape sh, NormIn ni, Epi e, hipStream_t s) {
    switch (c.wn) {
        case 2:
            if (c.mbt == 8) launch_big_wn<2, Epi, 8>(a, w, sh, ni, e, s);
            else launch_big_wn<2, Epi, 16>(a, w, sh, ni, e, s);
            break;
        case 3:
            if (c.mbt == 8) launch_big_wn<3, Epi, 8>(a, w, sh, ni, e, s);
            else launch_big_wn<3, Epi, 16>(a, w, sh, ni, e, s);
            break;
        default:
            if (c.mbt == 8) launch_big_wn<4, Epi, 8>(a, w, sh, ni, e, s);
            else launch_big_wn<4, Epi, 16>(a, w, sh, ni, e, s);
    }
}
// QKV, gate/up, O and down beyond 128 rows in the blocks that big_plan picks, `now` being the choice it starts from
template <class Epi>
static void launch_big_or_tile(BigChoice now, const u16 *a, const u16 *w, GemmShape sh, NormIn ni, Epi e, Workspace ws, hipStream_t s) {
    static_assert(2 * 8 * (kXcdUnits - 1) <= 1024, "two counters for every split block (Workspace::exchange)");
    const BigPlan p = big_plan(tile_epilogue_of<Epi>, now, sh.M_tiles, sh.N_tiles, sh.K_tiles, ws.partial_bytes, ws.exchange != nullptr);
    if (p.wn == 0) launch_tile(a, w, sh, ni, e, ws, true, s);
    else if (p.ks == 2) launch_big_wn<kSplitWn, Epi, kSplitMbt, 2>(a, w, sh, ni, e, s, ws);
    else if (p.mbt == 12 && p.wn == 3) launch_big_wn<3, Epi, 12>(a, w, sh, ni, e, s);
    else if (p.mbt == 12) launch_big_wn<4, Epi, 12>(a, w, sh, ni, e, s);
    else if (p.mbt == 20 && p.wn == 3) launch_big_wn<3, Epi, 20>(a, w, sh, ni, e, s);
    else if (p.mbt == 20) launch_big_wn<4, Epi, 20>(a, w, sh, ni, e, s);
    else launch_big_as(BigChoice{p.mbt, p.wn}, a, w, sh, ni, e, s);
}

// The slab kernel (gemm_slab.h): blocks of 128 rows against NTB n-tiles.
template <int NTB, bool NTW, class Epi>
static void launch_slab(const u16 *a, const u16 *w, GemmShape sh, NormIn ni, Epi e, hipStream_t s) {
    SlabArgs g;
    g.A = a; g.W = w; g.KT = sh.K_tiles; g.MT_total = sh.M_tiles; g.NT = sh.N_tiles;
    g.ssq = ni.ssq; g.n_ssq = ni.n_ssq; g.eps = ni.eps; g.inv_d = 1.0f / (float)(sh.K_tiles * 32);
    allow_lds<gemm_slab_kernel<NTB, Epi, NTW>>(slab_smem_bytes(NTB));
    gemm_slab_kernel<NTB, Epi, NTW><<<dim3((g.NT + NTB - 1) / NTB, (g.MT_total + 7) / 8), 512, slab_smem_bytes(NTB), s>>>(g, e);
}

template <class Epi>
static void launch_qkv_as(const u16 *xa, const u16 *w, GemmShape sh, NormIn ni, Epi e, Workspace ws, hipStream_t s) {
    // (Up to 96 rows a ring of ONE stage is the fastest since the weight tiles are loaded non-temporally - 2048 waves
    // with one group of tiles each in flight keep the HBM stream full, and fewer outstanding weight loads per
    // compute unit leave the activation loads less to queue behind: 1.9 % per step at 32 rows for this and the
    // gate/up projection together, 1.5 % at 64 rows, 0.5 % at 96.)
    const int ng = stream_ng(sh.N_tiles, 3, false), slab = qkv_slab_group(sh.M_tiles, sh.N_tiles);
    const RowBlock rows = qkv_row_block(sh.M_tiles, sh.N_tiles, sh.K_tiles);
    if (rows.mt) launch_row_blocks(rows, xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 2 && ng == 1) launch_stream<2, 1, 4, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 2 && ng == 2) launch_stream<2, 2, 2, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 2) launch_stream<2, 3, 1, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 4) launch_stream<4, 3, 1, true>(xa, w, sh, ni, e, s);          // 33..64 rows: still eight waves
    else if (sh.M_tiles <= 6) launch_stream<6, 3, 1, true>(xa, w, sh, ni, e, s);          // 65..96 rows
    else if (slab == 3) launch_slab<3, true>(xa, w, sh, ni, e, s);
    else if (slab == 6 && (sh.M_tiles <= 8 || sh.M_tiles >= 12)) launch_slab<6, true>(xa, w, sh, ni, e, s);
    else if (slab == 6) launch_slab<6, false>(xa, w, sh, ni, e, s);
    else launch_big_or_tile(big_choice(sh), xa, w, sh, ni, e, ws, s);
}
void launch_gemm_qkv(const u16 *xa, const u16 *w, GemmShape sh, NormIn ni, QkvOut out, Workspace ws, hipStream_t s) {
    if (out.dense_rows > 0) launch_qkv_as(xa, w, sh, ni, EpiQKVDense{out}, ws, s);
    else launch_qkv_as(xa, w, sh, ni, EpiQKV{out}, ws, s);
}
void launch_gemm_resid(const u16 *a, const u16 *w, GemmShape sh, float *h, int ldh, NormOut no, Workspace ws,
                       hipStream_t s) {
    EpiResid e{h, ldh, no, sh.M_tiles};
    // Up to 96 rows K is split over four workgroups that add up their sums in the kernel (gemm_stream_ksplit_kernel) unless it is
    // short; a step of the 8B shape with down so took 3.55 -> 3.47 ms at 32 rows, with both 4.25 -> 4.03 at 64 and 4.77 -> 4.71 at 96.
    // At 97 to 128 rows, where its ring is down to two stages, it loses to the tile kernel, whose K split over workgroups also splits
    // the activation reads, with a separate pass that adds the partial sums.  Beyond, the blocks of the LDS-ring kernel where they fill
    // the chip (choose.h: big_choice, big_plan).
    // Blocks with all of K in a workgroup, where they are short enough (choose.h): d 1024 at 128 rows, O 6.5 -> 4.4 us.
    const RowBlock rows = resid_block(sh.M_tiles, sh.N_tiles, sh.K_tiles);
    const NormIn none{nullptr, 0, 0.f};
    if (rows.mt && no.span == 64) {
        if (rows.mt == 2) launch_block<2>(a, w, sh, e, s);
        else launch_block<4>(a, w, sh, e, s);
    }
    else if (rows.mt) {
        if (rows.mt == 4 && sh.past_cache) launch_stream<4, 2, 4, true, true>(a, w, sh, none, e, s);
        else if (rows.mt == 4) launch_stream<4, 2, 4, true, false>(a, w, sh, none, e, s);
        else if (rows.ng == 2) launch_stream<2, 2, 4, true, false>(a, w, sh, none, e, s);
        else launch_stream<2, 1, 4, true, false>(a, w, sh, none, e, s);
    }
    else if (const int ng = ksplit_narrow_ng(sh, ws)) {
        if (ng == 1) launch_ksplit_narrow<1>(a, w, sh, e, ws, s);
        else if (ng == 2) launch_ksplit_narrow<2>(a, w, sh, e, ws, s);
        else if (no.span == 64) launch_ksplit_narrow<4, true>(a, w, sh, e, ws, s);
        else launch_ksplit_narrow<4>(a, w, sh, e, ws, s);
    }
    else if (const int few = few_rows_split(sh.M_tiles, sh.N_tiles, sh.K_tiles); few && ksplit_fits(sh, sh.N_tiles / few, ws)) {
        if (few == 1) launch_ksplit_few<1>(a, w, sh, e, ws, s);
        else if (few == 2) launch_ksplit_few<2>(a, w, sh, e, ws, s);
        else launch_ksplit_few<4>(a, w, sh, e, ws, s);
    }
    else if (ksplit_ok(sh, ws)) launch_stream_ksplit(a, w, sh, e, ws, s);
    else if (sh.M_tiles <= 8 && (sh.M_tiles > 2 || few_rows_tile(sh.N_tiles, sh.K_tiles))) launch_tile(a, w, sh, none, e, ws, true, s);
    else if (sh.M_tiles <= 2) {
        // (as many ring stages as divide a wave's k-tiles: with one O of 32 rows at d 1024 took 5.0 us)
        const int kw = sh.K_tiles / WK;
        if (kw % 8 == 0) launch_stream<2, 1, 8, false>(a, w, sh, none, e, s);
        else if (kw % 4 == 0) launch_stream<2, 1, 4, false>(a, w, sh, none, e, s);
        else if (kw % 3 == 0) launch_stream<2, 1, 3, false>(a, w, sh, none, e, s);
        else launch_stream<2, 1, 2, false>(a, w, sh, none, e, s);
    }
    else {
        // (128-row blocks only for the O projection: at 1024 rows of the 8B shape 256 blocks of 128 x 128 take 47.7 us against 50.4 for
        // the tile kernel and its merge pass; the down projection, three times as long in K, takes 126 us against 105)
        const BigChoice now = big_choice(sh);
        launch_big_or_tile(now.mbt == 16 || sh.K_tiles <= sh.N_tiles ? now : BigChoice{16, 0}, a, w, sh, none, e, ws, s);
    }
}
void launch_gemm_swiglu(const u16 *xa, const u16 *w, GemmShape sh, NormIn ni, u16 *act, unsigned *status, Workspace ws,
                        hipStream_t s) {
    EpiSwiGLU e{act, sh.M_tiles, status};
    const int ng = stream_ng(sh.N_tiles, 6, true), rb = swiglu_row_block_group(sh.M_tiles, sh.N_tiles, sh.K_tiles);
    const bool slab = sh.M_tiles > 6 && sh.M_tiles <= 8 && ng == 6, big = sh.M_tiles > 8 && !rb && big_choice(sh).wn;
    RowBlock rows{0, 0};
    if (sh.M_tiles > 2 && !slab && !big) rows = row_block(sh.M_tiles, sh.N_tiles, sh.K_tiles, sh.M_tiles > 8 && !rb);
    if (!rb && swiglu_wide_block(sh.M_tiles, sh.N_tiles, sh.K_tiles, !big)) launch_stream<6, 6, 1, true, false>(xa, w, sh, ni, e, s);
    else if (rows.mt) launch_row_blocks(rows, xa, w, sh, ni, e, s);
    else if (rb == 6) launch_stream<4, 6, 2, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 2 && ng == 1) launch_stream<2, 1, 4, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 2 && ng == 2) launch_stream<2, 2, 2, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 4 && ng == 2) launch_stream<4, 2, 2, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 2 && ng == 3) launch_stream<2, 3, 1, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 4 && ng == 3) launch_stream<4, 3, 1, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 6 && ng == 3) launch_stream<6, 3, 1, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 8 && ng == 3) launch_stream<8, 3, 1, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 2) launch_stream<2, 6, 1, true>(xa, w, sh, ni, e, s);
    // (33 to 64 rows, up to 1024 n-tiles: groups of four leave fewer compute units idle - d 2560, d_ff 6912 20.0 -> 15.9 us)
    else if (sh.M_tiles <= 4 && sh.N_tiles <= 4 * kStreamWGs) launch_stream<4, 4, 2, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 4) launch_stream<4, 6, 1, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 6) launch_stream<6, 6, 1, true>(xa, w, sh, ni, e, s);
    else if (slab) launch_slab<6, true>(xa, w, sh, ni, e, s);
    else launch_big_or_tile(big_choice(sh), xa, w, sh, ni, e, ws, s);
}

constexpr int kLmNG = 6;      // n-tiles per group of the LM head at up to 32 rows

// partials per row that launch_gemm_lmstats writes
// Up to 32 rows the group is four n-tiles wide where that leaves fewer padded slots in a workgroup's last group
// (126464 columns: 31 n-tiles per workgroup = eight groups of four with one slot idle, against six groups of six
// with five; measured 166 -> 159 us).
static int lm_ng(int n_tiles) {
    const int per = (n_tiles + kStreamWGs - 1) / kStreamWGs;
    return (per + 3) / 4 * 4 < (per + kLmNG - 1) / kLmNG * kLmNG ? 4 : kLmNG;
}
// Beyond 128 rows the LM head of a long vocabulary always runs on the LDS-ring kernel, 256 columns wide where no other width is chosen
// (129..191 rows leave part of a 256-row block empty, and still measure 283 us against 427 us on the tile kernel:
// the vocabulary is long enough to be bound by the weight stream either way)
// At 144 to 176 rows blocks narrower than that serve vocabularies whose 256-column blocks leave compute units idle, up to 65536;
// beyond, their statistics (twice as many, over 1 MiB) would not fit the room that lm_stats_excess counts on.
static BigChoice lm_big(GemmShape sh) {
    const BigChoice c = lm_block_choice(sh.M_tiles, sh.N_tiles);
    if (sh.N_tiles < 32 || (c.wn && (sh.M_tiles >= 12 || sh.N_tiles <= 16 * kStreamWGs))) return c;
    return BigChoice{16, 4};
}
// From 33 to 128 rows the LM head runs on the LDS-ring kernel as one row block, 64 * lm_one_wn columns wide: the widest block
// that makes no more than a round of workgroups shorter (see launch_gemm_lmstats).
static bool lm_one_block(int m_tiles) { return m_tiles > 2 && m_tiles <= 8; }
static int lm_one_wn(int n_tiles) { return n_tiles <= 8 * kStreamWGs ? 2 : n_tiles <= 16 * kStreamWGs ? 4 : 8; }
int lm_stats_parts(int n_tiles, int m_tiles) {
    if (lm_one_block(m_tiles)) return (n_tiles + 4 * lm_one_wn(n_tiles) - 1) / (4 * lm_one_wn(n_tiles));
    if (m_tiles <= 2) {
        const int ng = lm_ng(n_tiles);
        const int groups = (n_tiles + ng - 1) / ng;
        return (groups < kStreamWGs ? groups : kStreamWGs) * ng;
    }
    if (const int wn = lm_big(GemmShape{m_tiles, n_tiles, 0}).wn) return (n_tiles + 4 * wn - 1) / (4 * wn);
    return (n_tiles + tile_columns(m_tiles) - 1) / tile_columns(m_tiles);
}

void launch_gemm_lmstats(const u16 *xa, const u16 *w, GemmShape sh, NormIn ni, float *stats, Workspace ws,
                         hipStream_t s) {
    const int parts = lm_stats_parts(sh.N_tiles, sh.M_tiles);
    if (sh.M_tiles <= 2 && lm_ng(sh.N_tiles) == 4) launch_stream<2, 4, 4, true>(xa, w, sh, ni, EpiLMStats<gemm_slots(2, 4)>(stats, parts), s);
    else if (sh.M_tiles <= 2) launch_stream<2, kLmNG, 4, true>(xa, w, sh, ni, EpiLMStats<gemm_slots(2, kLmNG)>(stats, parts), s);
    else if (lm_one_block(sh.M_tiles)) {
        // 33..128 rows.  A streaming workgroup reads all activation rows once per group of six n-tiles, and with 31
        // n-tiles per workgroup that is five to six times [rows x d] through each compute unit's vector-memory path,
        // more than its weights: at 128 rows the kernel was bound by that path (244 us, 4.2 TB/s).  A block of 512
        // columns reads the activations once for 32 n-tiles; a vocabulary of 126464 gives 247 such workgroups, one round
        // on the chip.  With the weights copied through the LDS ring it takes 170 us at 96 rows and 168 at 128, against 191
        // and 174 us on the tile kernel, which loads them into registers four k-tiles ahead.  A vocabulary of 32000 is 63 such
        // blocks (42.7 us at d = 1024 and 128 rows) and 250 of 128 columns.
        const TileLMStats e{stats, parts};
        switch (lm_one_wn(sh.N_tiles)) {
            case 2: launch_big_wn<2, TileLMStats, 8>(xa, w, sh, ni, e, s); break;
            case 4: launch_big_wn<4, TileLMStats, 8>(xa, w, sh, ni, e, s); break;
            default: launch_big_wn<8, TileLMStats, 8>(xa, w, sh, ni, e, s);
        }
    }
    else if (lm_big(sh).wn) launch_big_as(lm_big(sh), xa, w, sh, ni, TileLMStats{stats, parts}, s);
    else launch_tile(xa, w, sh, ni, TileLMStats{stats, parts}, ws, false, s);
}
void launch_gemm_store(const u16 *xa, const u16 *w, GemmShape sh, NormIn ni, float *out, int units, int rpu_pad,
                       int valid, int ld, Workspace ws, hipStream_t s) {
    EpiStore e{out, units, rpu_pad, valid, ld};
    if (sh.M_tiles <= 2) launch_stream<2, 3, 8, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 4) launch_stream<4, 3, 4, true>(xa, w, sh, ni, e, s);
    else if (sh.M_tiles <= 8) launch_stream<8, 3, 2, false>(xa, w, sh, ni, e, s);
    else if (big_choice(sh).wn) launch_big_as(big_choice(sh), xa, w, sh, ni, e, s);
    else launch_tile(xa, w, sh, ni, e, ws, false, s);
}

}  // namespace odb
