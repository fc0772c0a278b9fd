// binary16 MFMA GEMM  C[M,N] = A[M,K] * W[N,K]^T  for the compute-bound shapes (the cache-refresh
// prefill, the batched long-context step: from 129 rows on where its blocks fill the chip) and the LM head from 33 rows on.
// Same operand layouts and epilogues as gemm_core.h / gemm_tile.h.
//
// A workgroup of eight waves computes a 256 x (64 WN) block of C over all of K, WN = 4, 3 or 2 (256, 192 or
// 128 columns: the narrower blocks exist for shapes whose count of 256-wide blocks fills the compute units
// badly), or with MBT = 8, 12 or 20 a block of 128, 192 or 320 rows.  Per k-tile it needs MBT 1 KiB
// tiles of A and 4 WN of W; they are copied from global memory straight into LDS (global_load ... lds, no registers in
// between) into a ring of stages.  The waves form a 2 x 4 grid, each owning MBT/2 x WN output tiles.
// Operand bytes per flop are half those of the 128-row tile kernel, which is what matters here:
// a re-read that misses the 4 MiB L2 of an XCD is served at HBM-like bandwidth (about 7 TB/s measured
// on MI355X, against 22 TB/s for L2 hits), so the ids of the workgroups are also mapped to blocks
// such that the workgroups resident on one XCD share their weight panels and rows of A.
#pragma once
#include <type_traits>
#include "choose.h"
#include "gemm_tile.h"

namespace odb {

// k-tiles per stage and stages in the ring: one barrier interval covers a stage.  A 256-row block of 192 or 256 columns has 24 or
// 32 MFMAs per wave and k-tile, enough to hide the operand reads of the other group of waves; 256 x 128 and the 128-row blocks
// have 8 to 16, so their stages are two k-tiles deep (measured on the loop alone at K = 4096: 128 x 128 blocks 43.3 -> 37.1 us
// at 1024 x 4096, 128 x 192 blocks 56.1 -> 52.4 us at 256 x 24576; 256 x 256 blocks equal.  256 x 128 blocks, two layers of a
// refresh of 4 x 512 positions, one k-tile with four stages -> two with three: O 167.9 -> 153.2 us, down 420.8 -> 387.8).
// (Blocks of 192 rows: two k-tiles up to 192 columns, 12 to 18 MFMAs a wave and k-tile; of 320 rows one, as 256 rows of these widths.)
constexpr int big_kp(int wn, int mbt) { return (mbt == 8 && wn <= 4) || (mbt == 12 && wn <= 3) || (mbt == 16 && wn == 2) ? 2 : 1; }
constexpr int big_stages(int wn, int mbt) { return mbt == 8 || big_kp(wn, mbt) == 2 ? 3 : 4; }
constexpr int big_stage_tiles(int wn, int mbt) { return big_kp(wn, mbt) * (mbt + 4 * wn); }
constexpr int big_smem_bytes(int wn, int mbt) { return big_stages(wn, mbt) * big_stage_tiles(wn, mbt) * 1024 + 320 * 4; }   // ring, row scales
// per-wave scratch of the epilogues, in the ring's place once the k-loop is over
constexpr int kBigScratch = 4096;

struct BigArgs {
    const u16 *A, *W;
    int KT, MT_total, NT;
    int m_blocks, n_blocks;
    const float *ssq;          // fused RMSNorm of the input rows (see GemmArgs)
    int n_ssq;
    float eps, inv_d;
    // an XCD's blocks from number `whole` on are split over KS workgroups each, which add their sums up (big_exchange)
    int whole;
    float *partial;
    unsigned *exchange;        // two counters a split block
};

// ---- epilogues of a wave's MW x WT output tiles ------------------------------------------------------------------
// A wave's tiles are finished row of tiles by row of tiles; what a row reads from global memory (the residual, the RoPE
// table) is requested while the row before it is worked on, index arithmetic is done once per row and column of tiles,
// and values beyond the binary16 range are collected and reported once.  (One tile at a time, each waiting for its own
// loads, this tail was 15 of the 103 us of the QKV projection at 1024 rows.)
// mtw, ntw: the wave's first row tile and n-tile; rstd: row scales of the wave's rows; scr: kBigScratch bytes of LDS.
template <int MW, int WT>
__device__ __forceinline__ void big_epilogue(const EpiQKV &e, f32x4 (&acc)[MW][WT], int mtw, int ntw, const BigArgs &g,
                                             const float *rstd, char *scr, int lane) {
    const QkvOut &o = e.o;
    const int mi = lane & 15, gq = lane >> 4;
    int sec[WT], hd[WT], p0[WT];
#pragma unroll
    for (int j = 0; j < WT; j++) {
        const int nt = ntw + j < g.NT ? ntw + j : g.NT - 1;
        sec[j] = o.fd_d.quot(nt);
        const int rt = nt - sec[j] * (o.d >> 4);
        hd[j] = o.fd_dh.quot(rt);
        p0[j] = (rt - hd[j] * (o.dh >> 4)) * 16;
    }
    struct Row { int unit, tu; bool spec; f32x4 cs[WT]; };         // cs: (cos, sin) of the lane's two channel pairs
    auto fetch = [&](int m) __attribute__((always_inline)) {
        Row r;
        const int mt = mtw + m < g.MT_total ? mtw + m : g.MT_total - 1;
        r.spec = o.split_tile > 0 && mt >= o.split_tile;
        const int tpu = pick(r.spec, o.tiles_per_unit_b, o.tiles_per_unit), mtu = pick(r.spec, mt - o.split_tile, mt);
        r.unit = pick(r.spec, o.fd_tpu_b, o.fd_tpu).quot(mtu);
        r.tu = mtu - r.unit * tpu;
        const int pos = o.rowpos ? o.rowpos[mt * 16 + mi] : o.pos_off + r.tu * 16 + mi;
        const float *tab = o.rope + (size_t)pos * o.dh + 4 * gq;
#pragma unroll
        for (int j = 0; j < WT; j++) r.cs[j] = sec[j] < 2 ? *reinterpret_cast<const f32x4 *>(tab + p0[j]) : f32x4{0.f, 0.f, 0.f, 0.f};
        return r;
    };
    bool bad = false;
    Row next = fetch(0);
#pragma unroll
    for (int m = 0; m < MW; m++) {
        const Row r = next;
        if (m + 1 < MW) next = fetch(m + 1);
        const int mt = mtw + m;
        if (mt >= g.MT_total) break;
        const float rs = rstd[m * 16 + mi];
        const f32x4 rs4 = *reinterpret_cast<const f32x4 *>(rstd + m * 16 + 4 * gq);
        u16 *kdst = pick(r.spec, o.k_b, o.k) + r.unit * pick(r.spec, o.k_b_unit_stride, o.k_unit_stride) + (size_t)r.tu * (o.dh / 32) * kTileElems;
        u16 *vdst = pick(r.spec, o.v_b, o.v) + r.unit * pick(r.spec, o.v_b_unit_stride, o.v_unit_stride) +
                    (size_t)(r.tu >> 1) * (o.dh / 16) * kTileElems + lane * 8 + 4 * (r.tu & 1);
        const size_t khs = pick(r.spec, o.k_b_head_stride, o.k_head_stride), vhs = pick(r.spec, o.v_b_head_stride, o.v_head_stride);
        // V goes out transposed: lane (gq, ni) takes rows 4 gq .. 4 gq + 3 of column ni, through the wave's scratch
        f32x4 (*tr)[64] = reinterpret_cast<f32x4 (*)[64]>(scr);
#pragma unroll
        for (int j = 0; j < WT; j++)
            if (sec[j] == 2) tr[j][lane] = acc[m][j];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // stores before the transposed reads
#pragma unroll
        for (int j = 0; j < WT; j++) {
            if (ntw + j >= g.NT) break;
            if (sec[j] < 2) {
                const f32x4 c = acc[m][j] * rs, cs = r.cs[j];
                const float y0 = c[0] * cs[0] - c[1] * cs[1], y1 = c[1] * cs[0] + c[0] * cs[1];
                const float y2 = c[2] * cs[2] - c[3] * cs[3], y3 = c[3] * cs[2] + c[2] * cs[3];
                u16 *dst = (sec[j] == 0 ? o.q + ((size_t)hd[j] * o.q_mt + mt) * (o.dh / 32) * kTileElems : kdst + hd[j] * khs) +
                           (p0[j] >> 5) * kTileElems;
                const int kk = (p0[j] & 16) + 4 * gq;
                bad |= out_of_f16(y0, y1, y2, y3);
                st_f16x4(dst + ((kk >> 3) * 16 + mi) * 8 + (kk & 7), y0, y1, y2, y3);
            } else {
                const float *base = reinterpret_cast<const float *>(&tr[j][0]) + ((mi >> 2) * 16 + 4 * gq) * 4 + (mi & 3);
                const float y0 = base[0] * rs4[0], y1 = base[4] * rs4[1], y2 = base[8] * rs4[2], y3 = base[12] * rs4[3];
                bad |= out_of_f16(y0, y1, y2, y3);
                st_f16x4(vdst + hd[j] * vhs + (p0[j] >> 4) * kTileElems, y0, y1, y2, y3);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // reads before the next row's stores
    }
    if (bad && o.status) atomicOr(o.status, kStatusSaturated);
}

// The same for dense rows (QkvOut); what depends on the row alone is found once per row of tiles.
template <int MW, int WT>
__device__ __forceinline__ void big_epilogue(const EpiQKVDense &e, f32x4 (&acc)[MW][WT], int mtw, int ntw, const BigArgs &g,
                                             const float *rstd, char *scr, int lane) {
    const QkvOut &o = e.o;
    const int mi = lane & 15, gq = lane >> 4;
    int sec[WT], hd[WT], p0[WT];
#pragma unroll
    for (int j = 0; j < WT; j++) {
        const int nt = ntw + j < g.NT ? ntw + j : g.NT - 1;
        sec[j] = o.fd_d.quot(nt);
        const int rt = nt - sec[j] * (o.d >> 4);
        hd[j] = o.fd_dh.quot(rt);
        p0[j] = (rt - hd[j] * (o.dh >> 4)) * 16;
    }
    f32x4 (*tr)[64] = reinterpret_cast<f32x4 (*)[64]>(scr);
    bool bad = false;
#pragma unroll
    for (int m = 0; m < MW; m++) {
        const int mt = mtw + m < g.MT_total ? mtw + m : g.MT_total - 1;
        const bool live = mtw + m < g.MT_total;
        const int row = mt * 16 + mi, unit = o.fd_valid.quot(row), i = row - unit * o.valid;
        const bool in = live && row < o.dense_rows;
        f32x4 cs[WT];
#pragma unroll
        for (int j = 0; j < WT; j++) {
            cs[j] = sec[j] < 2 ? *reinterpret_cast<const f32x4 *>(o.rope + (size_t)(o.pos_off + i) * o.dh + p0[j] + 4 * gq) : f32x4{0.f, 0.f, 0.f, 0.f};
            if (sec[j] == 2) tr[j][lane] = acc[m][j];
        }
        u16 *qd = o.q + ((size_t)unit * o.tiles_per_unit + (i >> 4)) * (o.dh / 32) * kTileElems + (i & 15) * 8;
        u16 *kd = o.k + unit * o.k_unit_stride + (size_t)(i >> 4) * (o.dh / 32) * kTileElems + (i & 15) * 8;
        u16 *vd[4];
        bool vin[4];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int vrow = mt * 16 + 4 * gq + r, vu = o.fd_valid.quot(vrow), vi = vrow - vu * o.valid;
            vin[r] = live && vrow < o.dense_rows;
            vd[r] = o.v + vu * o.v_unit_stride + (size_t)(vi >> 5) * (o.dh / 16) * kTileElems + ((vi & 15) >> 2) * 128 + mi * 8 + 4 * ((vi >> 4) & 1) + (vi & 3);
        }
        const float rs = rstd[m * 16 + mi];
        const f32x4 rs4 = *reinterpret_cast<const f32x4 *>(rstd + m * 16 + 4 * gq);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // stores before the transposed reads
#pragma unroll
        for (int j = 0; j < WT; j++) {
            if (ntw + j >= g.NT) break;
            if (sec[j] < 2) {
                const f32x4 c = acc[m][j] * rs;
                const float y0 = c[0] * cs[j][0] - c[1] * cs[j][1], y1 = c[1] * cs[j][0] + c[0] * cs[j][1];
                const float y2 = c[2] * cs[j][2] - c[3] * cs[j][3], y3 = c[3] * cs[j][2] + c[2] * cs[j][3];
                const int kk = (p0[j] & 16) + 4 * gq;
                bad |= live && out_of_f16(y0, y1, y2, y3);
                u16 *dst = (sec[j] == 0 ? qd + (size_t)hd[j] * o.q_mt * (o.dh / 32) * kTileElems : kd + hd[j] * o.k_head_stride) +
                           (p0[j] >> 5) * kTileElems + (kk >> 3) * 128 + (kk & 7);
                if (in) st_f16x4(dst, y0, y1, y2, y3);
            } else {
                const float *base = reinterpret_cast<const float *>(&tr[j][0]) + ((mi >> 2) * 16 + 4 * gq) * 4 + (mi & 3);
                const f32x4 y = f32x4{base[0], base[4], base[8], base[12]} * rs4;
                bad |= live && out_of_f16(y[0], y[1], y[2], y[3]);
#pragma unroll
                for (int r = 0; r < 4; r++)
                    if (vin[r]) vd[r][hd[j] * o.v_head_stride + (p0[j] >> 4) * kTileElems] = f2h(y[r]);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // reads before the next row's stores
    }
    if (bad && o.status) atomicOr(o.status, kStatusSaturated);
}

template <int MW, int WT>
__device__ __forceinline__ void big_epilogue(const EpiSwiGLU &e, f32x4 (&acc)[MW][WT], int mtw, int ntw, const BigArgs &g,
                                             const float *rstd, char *, int lane) {
    const int mi = lane & 15, gq = lane >> 4;
    u16 *dst[WT];
#pragma unroll
    for (int j = 0; j < WT; j++) {
        const int ch = (ntw + j) * 8 + 2 * gq, kk = ch & 31;      // channel of the lane's first (gate, up) pair
        dst[j] = e.act + ((size_t)((ntw + j) >> 2) * e.mt_total + mtw) * kTileElems + ((kk >> 3) * 16 + mi) * 8 + (kk & 7);
    }
    bool bad = false;
#pragma unroll
    for (int m = 0; m < MW; m++) {
        if (mtw + m < g.MT_total) {
            const float rs = rstd[m * 16 + mi];
#pragma unroll
            for (int j = 0; j < WT; j++) {
                if (ntw + j >= g.NT) break;
                const f32x4 c = acc[m][j] * rs;
                const float y0 = EpiSwiGLU::act2(c[0], c[1]), y1 = EpiSwiGLU::act2(c[2], c[3]);
                bad |= out_of_f16(y0, y1, 0.f, 0.f);
                *reinterpret_cast<uint32_t *>(dst[j] + m * kTileElems) = pack4(y0, y1, 0.f, 0.f).x;
            }
        }
    }
    if (bad && e.status) atomicOr(e.status, kStatusSaturated);
}

// Sums of squares go out per 64 columns.  WT = 4: the wave's columns are one such sum.  WT = 2 or 3: the wave leaves what it has per row
// and 32 or 16 columns in its scratch, [parts][MW * 16 rows], and the workgroup adds them up.  (N is a multiple of 256, so only
// a block of 192 columns can reach beyond it, and then by whole sums.)
template <int WT> constexpr int resid_parts() { return WT == 3 ? 3 : 1; }
template <int MW, int WT>
__device__ __forceinline__ void big_epilogue(const EpiResid &e, f32x4 (&acc)[MW][WT], int mtw, int ntw, const BigArgs &g,
                                             const float *, char *scr, int lane) {
    const NormOut &no = e.no;
    const int mi = lane & 15, gq = lane >> 4;
    float *s_q = reinterpret_cast<float *>(scr);
    static_assert(resid_parts<WT>() * MW * 16 * 4 <= kBigScratch, "sums of a wave");
    f32x4 gn[WT], hv[WT];
    float *hp = e.h + (size_t)(mtw * 16 + mi) * e.ld + ntw * 16 + 4 * gq;
    u16 *xp[WT];
    bool in[WT];
    int col[WT];
#pragma unroll
    for (int j = 0; j < WT; j++) {
        in[j] = WT != 3 || ntw + j < g.NT;
        col[j] = (in[j] ? ntw + j : g.NT - 1) * 16 + 4 * gq;
        gn[j] = no.hb ? *reinterpret_cast<const f32x4 *>(no.gain + col[j]) : f32x4{0.f, 0.f, 0.f, 0.f};
        const int kk = ((ntw + j) & 1) * 16 + 4 * gq;
        xp[j] = no.hb + ((size_t)((ntw + j) >> 1) * e.mt_total + mtw) * kTileElems + ((kk >> 3) * 16 + mi) * 8 + (kk & 7);
    }
    auto fetch = [&](int m) __attribute__((always_inline)) {
        const int mt = mtw + m < g.MT_total ? mtw + m : g.MT_total - 1;
        const float *p = e.h + (size_t)(mt * 16 + mi) * e.ld;
#pragma unroll
        for (int j = 0; j < WT; j++) hv[j] = *reinterpret_cast<const f32x4 *>(p + col[j]);
    };
    bool bad = false;
    fetch(0);
#pragma unroll
    for (int m = 0; m < MW; m++) {
        f32x4 v[WT];
#pragma unroll
        for (int j = 0; j < WT; j++) v[j] = hv[j] + acc[m][j];
        if (mtw + m >= g.MT_total) break;
        if (m + 1 < MW) fetch(m + 1);
        float q[WT];
#pragma unroll
        for (int j = 0; j < WT; j++) {
            q[j] = 0.f;
            if (!in[j]) continue;
            *reinterpret_cast<f32x4 *>(hp + (size_t)m * 16 * e.ld + j * 16) = v[j];
            if (no.hb) {
                const f32x4 y = v[j] * gn[j];
                bad |= out_of_f16(y[0], y[1], y[2], y[3]);
                st_f16x4(xp[j] + m * kTileElems, y[0], y[1], y[2], y[3]);
                q[j] = v[j][0] * v[j][0] + v[j][1] * v[j][1] + v[j][2] * v[j][2] + v[j][3] * v[j][3];
            }
        }
        if (no.hb) {
            if constexpr (WT == 3) {
#pragma unroll
                for (int j = 0; j < WT; j++) {
                    const float t = EpiResid::over_row(q[j]);
                    if (lane < 16) s_q[j * MW * 16 + m * 16 + lane] = t;
                }
            } else {
                float t = q[0];
#pragma unroll
                for (int j = 1; j < WT; j++) t += q[j];
                t = EpiResid::over_row(t);
                if (lane < 16) {
                    if constexpr (WT == 4) no.ssq[(size_t)((mtw + m) * 16 + lane) * no.n_ssq + (ntw >> 2)] = t;
                    else s_q[m * 16 + lane] = t;
                }
            }
        }
    }
    if (bad && no.status) atomicOr(no.status, kStatusSaturated);
}

template <int MW, int WT>
__device__ __forceinline__ void big_epilogue(const EpiStore &e, f32x4 (&acc)[MW][WT], int mtw, int ntw, const BigArgs &g,
                                             const float *rstd, char *, int lane) {
#pragma unroll
    for (int m = 0; m < MW; m++)
#pragma unroll
        for (int j = 0; j < WT; j++)
            if (mtw + m < g.MT_total && ntw + j < g.NT) e(mtw + m, ntw + j, acc[m][j] * rstd[m * 16 + (lane & 15)], lane, 0);
}

// Adds the sums of the two workgroups of a split block (number `at` of the launch's split ones).  The first to arrive leaves its sums in
// the workspace, waits for the stores and counts itself ready; the second waits for that (choose.h: exchange_ready), adds them to its own
// and goes on to the epilogue (returns true): one addition per element, the same bits whoever is second.
// Stores, loads and counters are device-scope accesses without cache-wide fences, as in gemm_stream_ksplit_kernel.
template <int MW, int WT>
__device__ __forceinline__ bool big_exchange(f32x4 (&acc)[MW][WT], const BigArgs &g, int at, int w, int lane, unsigned *s_old) {
    constexpr unsigned bytes = 8 * MW * WT * 1024;
    unsigned *arrive = g.exchange + 2 * at;
    float *sums = g.partial + (size_t)at * (bytes / 4);
    if (threadIdx.x == 0) *s_old = __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const unsigned number = *s_old;
    const unsigned off = w * (MW * WT * 1024) + lane * 16;
    if (!exchange_waits(number)) {
#pragma unroll
        for (int m = 0; m < MW; m++)
#pragma unroll
            for (int j = 0; j < WT; j++)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[m][j]), sums_rsrc(sums, bytes), off + (m * WT + j) * 1024, 0, kDeviceScope);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (threadIdx.x == 0) (void)__hip_atomic_fetch_add(arrive + 1, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }
    if (threadIdx.x == 0)
        while (!exchange_ready(number, __hip_atomic_load(arrive + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) __builtin_amdgcn_s_sleep(1);
    __syncthreads();
    constexpr int B = 16;                       // tiles requested together
#pragma unroll
    for (int t0 = 0; t0 < MW * WT; t0 += B) {
        u32x4 v[B];
#pragma unroll
        for (int t = 0; t < B; t++)
            if (t0 + t < MW * WT) v[t] = __builtin_amdgcn_raw_buffer_load_b128(sums_rsrc(sums, bytes), off + (t0 + t) * 1024, 0, kDeviceScope);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < B; t++)
            if (t0 + t < MW * WT) acc[(t0 + t) / WT][(t0 + t) % WT] += __builtin_bit_cast(f32x4, v[t]);
        __builtin_amdgcn_sched_barrier(0);
    }
    return true;
}

// MBT: 16-row tiles per block, 16 (256 rows) or 8 (128 rows: twice the blocks for shapes that leave compute
// units idle otherwise; per flop it needs 1.4 x the operand bytes of the 256-row block), or 12 and 20 for counts of rows that those divide
// badly (choose.h: big_plan).  KS: workgroups for a block of the last round, 1, or 2 in blocks of 256 x 256.  WN = 8: a single block of 128 rows
// against 512 columns, for the LM head at 33 to 128 rows; W is then read once, non-temporally.
template <int WN, class Epi, int MBT = 16, int KS = 1>
__global__ __launch_bounds__(512) void gemm_big_kernel(BigArgs g, Epi epi) {
    static_assert((WN >= 2 && WN <= 4) || (WN == 8 && MBT == 8), "block width in units of 64 columns");
    static_assert(MBT % 4 == 0 && MBT >= 8 && MBT <= 20, "rows per block");
    static_assert(KS == 1 || KS == 2, "one workgroup stores, the other adds");
    constexpr int CW = 4;                       // waves side by side; two rows of them
    constexpr int WT = WN;                      // 16-column tiles per wave
    constexpr int MW = MBT / 2;                 // 16-row tiles per wave
    constexpr int NS = big_stages(WN, MBT), KP = big_kp(WN, MBT), TK = MBT + 4 * WN, ST = KP * TK;     // tiles per k-tile, per stage
    extern __shared__ __attribute__((aligned(16))) char smem[];
    typedef frag_t stage_t[ST][64];                                          // per k-tile: MBT tiles of A, then 4 WN of W
    stage_t *ring = reinterpret_cast<stage_t *>(smem);
    float *s_rstd = reinterpret_cast<float *>(smem + NS * ST * 1024);

    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave index, scalar
    const int wm = w / CW, wn = w % CW;                  // position of the wave in the 2 x CW grid
    // Workgroup ids go round-robin over the 8 XCDs.  The ids that land on one XCD walk down the row
    // blocks of a column of blocks before they move to that XCD's next column, so concurrently
    // resident workgroups of an XCD share weight panels (and all of them the rows of A) in its L2.
    const int xcd = blockIdx.x % 8, jx = blockIdx.x / 8;
    const bool split = KS > 1 && jx >= g.whole;
    const int blk = split ? g.whole + (jx - g.whole) / KS : jx, ks = split ? (jx - g.whole) % KS : 0;
    const int nb = (blk / g.m_blocks) * 8 + xcd, mb = blk % g.m_blocks;
    if (nb >= g.n_blocks) return;
    const int ns_all = g.KT / KP;               // stages (K is a multiple of 256: k-tiles come in eights)
    const int s_lo = split ? ks * ns_all / KS : 0, ns = (split ? (ks + 1) * ns_all / KS : ns_all) - s_lo;
    const int mt0 = mb * MBT, nt0 = nb * 4 * WN;

    // the first half of the waves copies the MBT tiles of A of every k-tile, the second half the 4 WN of W
    constexpr int PA = MBT / CW, PW = 4 * WN / CW, PMAX = PA > PW ? PA : PW;
    const u16 *src[PMAX];
    size_t kstride;
    const int per = w < CW ? PA : PW, slot0 = w < CW ? PA * w : MBT + (w - CW) * PW;
    if (w < CW) {
#pragma unroll
        for (int i = 0; i < PMAX; i++) {
            int mt = mt0 + PA * w + (i < PA ? i : PA - 1);
            mt = mt < g.MT_total ? mt : g.MT_total - 1;
            src[i] = g.A + ((size_t)s_lo * KP * g.MT_total + mt) * kTileElems;
        }
        kstride = (size_t)g.MT_total * kTileElems;
    } else {
#pragma unroll
        for (int i = 0; i < PMAX; i++) {
            int nt = nt0 + PW * (w - CW) + (i < PW ? i : PW - 1);
            nt = nt < g.NT ? nt : g.NT - 1;
            src[i] = g.W + ((size_t)nt * g.KT + s_lo * KP) * kTileElems;
        }
        kstride = kTileElems;
    }
    // (the tile addresses are wave-uniform, so they live in scalar registers; a lane adds its 16 bytes)
    const unsigned lane_off = lane * 16;
    auto issue = [&](int slot, int s) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < KP; q++)
#pragma unroll
            for (int i = 0; i < PMAX; i++)
                if (i < per) {
                    const void *from = reinterpret_cast<const char *>(src[i] + (size_t)(s * KP + q) * kstride) + lane_off;
                    auto *to = (__attribute__((address_space(3))) void *)(&ring[slot][q * TK + slot0 + i][0]);
                    if (WN == 8 && w >= CW) __builtin_amdgcn_global_load_lds(from, to, 16, 0, 2);
                    else __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
                }
    };

#pragma unroll
    for (int j = 0; j < NS - 1; j++)
        if (j < ns) issue(j, j);

    // row scales of the fused RMSNorm: one to four threads per row, behind the ring's first copies
    {
        constexpr int TR = 512 / (MBT * 16);
        const int r = threadIdx.x / TR, part = threadIdx.x % TR;
        float t = 1.f;
        if (g.ssq && r < MBT * 16) {
            int row = mt0 * 16 + r;
            row = row < g.MT_total * 16 ? row : g.MT_total * 16 - 1;
            const float *p = g.ssq + (size_t)row * g.n_ssq;
            t = 0.f;
            for (int i = part * 4; i < g.n_ssq; i += TR * 4) {          // n_ssq is a multiple of 4
                const f32x4 v = *reinterpret_cast<const f32x4 *>(p + i);
                t += (v[0] + v[1]) + (v[2] + v[3]);
            }
#pragma unroll
            for (int o = 1; o < TR; o <<= 1) t += __shfl_xor(t, o);
            t = 1.0f / sqrtf(t * g.inv_d + g.eps);
        }
        if (part == 0 && r < MBT * 16) s_rstd[r] = t;
    }

    f32x4 acc[MW][WT];
#pragma unroll
    for (int m = 0; m < MW; m++)
#pragma unroll
        for (int j = 0; j < WT; j++) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Two groups of four waves (the two rows of the wave grid; waves w and w + 4 share a SIMD) work in opposite phases:
    // while one issues the MFMAs of a stage, the other reads its operands of that stage (or the next) from LDS and
    // requests the copies of a later one, and the barrier between two phases swaps them.  LDS reads, copies and MFMAs
    // of different waves overlap; in one wave they do not: the same loop with reads of stage s + 1 spread between the
    // MFMAs of stage s in every wave, all eight in step, took 366 us where this one takes 318 (gate/up at 2048 rows;
    // the MFMAs alone take 220 us there, at the clock the chip holds under them).
    // Phases: group 0 reads stage s in phase 2s and multiplies it in 2s + 1, group 1 one phase later.  Stage s + NS - 1
    // goes into the slot of stage s - 1, whose last reads (group 1, phase 2s - 1) were complete before the barrier
    // in front of phase 2s; its copies have landed when both groups have waited for them, before phase 2(s + NS - 1).
    static_assert(NS >= 3, "slot arithmetic");
    frag_t a[KP][MW], b[KP][WT];
    auto wait_stage = [&](bool more) __attribute__((always_inline)) {       // all but the latest NS - 2 stages have landed
        if (!more) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if (PA == PW || w < CW) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KP * PA * (NS - 2)) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(KP * PW * (NS - 2)) : "memory");
    };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the first stages have landed (and the row sums, behind them)
    __syncthreads();
    if (wm == 1) __builtin_amdgcn_s_barrier();
    for (int s = 0, slot = 0; s < ns; s++) {
        const stage_t &st = ring[slot];
#pragma unroll
        for (int q = 0; q < KP; q++) {
#pragma unroll
            for (int j = 0; j < WT; j++) b[q][j] = st[q * TK + MBT + wn * WT + j][lane];
#pragma unroll
            for (int m = 0; m < MW; m++) a[q][m] = st[q * TK + wm * MW + m][lane];
        }
        const bool more = s + NS - 1 < ns;
        if (more) issue(slot == 0 ? NS - 1 : slot - 1, s + NS - 1);
        slot = slot == NS - 1 ? 0 : slot + 1;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (wm == 1) wait_stage(more);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < KP; q++)
#pragma unroll
            for (int m = 0; m < MW; m++)
#pragma unroll
                for (int i = 0; i < WT; i++) {
                    // to and fro: one operand changes from MFMA to MFMA, never both (MFMAs alone, normal values: 1.884 PFLOP/s; 1.845 when
                    // both change at the end of a row - the clock under them hangs on the power they take)
                    const int j = m & 1 ? WT - 1 - i : i;
                    acc[m][j] = mfma16(b[q][j], a[q][m], acc[m][j]);
                }
        if (wm == 0) wait_stage(more);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
    }
    if (wm == 0) __builtin_amdgcn_s_barrier();
    __syncthreads();            // the ring is reused below

    if constexpr (KS > 1)
        if (split && !big_exchange<MW, WT>(acc, g, (blk - g.whole) * 8 + xcd, w, lane, reinterpret_cast<unsigned *>(smem))) return;

    if constexpr (is_row_stats<Epi>::value) {
        // softmax statistics per row over this workgroup's columns: lane-local, across the four lane
        // groups, across the wave's four tiles, then across the four waves of a row half through LDS
        float *st_m = reinterpret_cast<float *>(smem);               // [CW column waves][256 rows]
        float *st_s = st_m + CW * 256;
        int *st_a = reinterpret_cast<int *>(st_s + CW * 256);
        const int mi = lane & 15, gq = lane >> 4;
#pragma unroll
        for (int m = 0; m < MW; m++) {
            const int r = wm * MW * 16 + m * 16 + mi;
            float rm = -INFINITY, rs = 0.f;
            int ra = 0x7fffffff;
#pragma unroll
            for (int j = 0; j < WT; j++) {
                const int nt = nt0 + wn * WT + j;
                if (nt < g.NT) {
                    f32x4 c = acc[m][j] * s_rstd[r];
                    float cm = c[0];
                    int ca = nt * 16 + 4 * gq;
#pragma unroll
                    for (int x = 1; x < 4; x++)
                        if (c[x] > cm) { cm = c[x]; ca = nt * 16 + 4 * gq + x; }
                    float cs = 0.f;
#pragma unroll
                    for (int x = 0; x < 4; x++) cs += __expf(c[x] - cm);
                    merge_stat(rm, rs, ra, cm, cs, ca);
                }
            }
#pragma unroll
            for (int o = 16; o <= 32; o <<= 1) {
                float om = __shfl_xor(rm, o), os = __shfl_xor(rs, o);
                int oa = __shfl_xor(ra, o);
                merge_stat(rm, rs, ra, om, os, oa);
            }
            if (gq == 0) {
                st_m[wn * 256 + r] = rm;
                st_s[wn * 256 + r] = rs;
                st_a[wn * 256 + r] = ra;
            }
        }
        __syncthreads();
        for (int r = threadIdx.x; r < MBT * 16; r += 512) {
            const int row = mt0 * 16 + r;
            float rm = st_m[r], rs = st_s[r];
            int ra = st_a[r];
#pragma unroll
            for (int x = 1; x < CW; x++) merge_stat(rm, rs, ra, st_m[x * 256 + r], st_s[x * 256 + r], st_a[x * 256 + r]);
            if (row < g.MT_total * 16) {
                float *p = epi.stats + ((size_t)row * epi.n_part + nb) * 3;
                p[0] = rm;
                p[1] = rs;
                p[2] = __int_as_float(ra);
            }
        }
    } else {
        big_epilogue<MW, WT>(epi, acc, mt0 + wm * MW, nt0 + wn * WT, g, s_rstd + wm * MW * 16, smem + w * kBigScratch, lane);
        if constexpr (is_resid<Epi>::value && (WT == 2 || WT == 3)) {
            if (epi.no.hb) {        // the waves side by side make WN partial sums of 64 columns
                __syncthreads();
                constexpr int P = 4 / (WT == 2 ? 2 : 1);         // parts of a sum
                for (int i = threadIdx.x; i < WN * MBT * 16; i += 512) {
                    const int r = i % (MBT * 16), c = i / (MBT * 16), row = mt0 * 16 + r, wr = r / (MW * 16), rr = r % (MW * 16);
                    float q[P];
#pragma unroll
                    for (int x = 0; x < P; x++) {
                        const int part = c * P + x, wv = part / resid_parts<WT>(), in = part % resid_parts<WT>();
                        q[x] = reinterpret_cast<const float *>(smem + (wr * CW + wv) * kBigScratch)[in * MW * 16 + rr];
                    }
                    float t;
                    if constexpr (P == 4) t = (q[0] + q[1]) + (q[2] + q[3]);
                    else t = q[0] + q[1];
                    if (row < g.MT_total * 16 && (nb * WN + c) * 4 < g.NT) epi.no.ssq[(size_t)row * epi.no.n_ssq + nb * WN + c] = t;
                }
            }
        }
    }
}

}  // namespace odb
