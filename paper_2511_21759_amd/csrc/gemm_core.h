// Device-side core of the weight-streaming binary16 MFMA GEMM  C[M,N] = A[M,K] * W[N,K]^T
// for few rows (launched from gemm.hip).
//
// A (activations) is tile-major [k_tile][m_tile][512], W is [n_tile][k_tile][512]
// (see common.h for the tile).  The work is persistent in spirit: nwg workgroups
// (one per compute unit) split the n-tiles into equal contiguous ranges, and the
// eight waves of a workgroup split K into eight slices.  Each wave therefore
// walks, NG n-tiles at a time, along contiguous runs of 1 KiB weight tiles,
// loading them straight into MFMA operand registers through a ring of PF stages
// that keeps running across the boundary between one group of n-tiles and the
// next, so the HBM stream never drains.  The eight K-slices of an output tile
// are added through LDS in a fixed order, so results do not depend on scheduling.
//
// Variant (template parameter of gemm_wg): IL hands the k-tiles to the waves round-robin instead of in contiguous
// slices, so that the workgroup as a whole reads eight KiB of contiguous weights per step
// (measured 5 % faster on the wide gate/up stream, slightly slower on the down projection).
//
// The epilogues fuse what follows each projection in the transformer block:
// RoPE + scatter of Q/K/V into the attention layouts, the residual add (plus the
// input of the next RMSNorm), SiLU(gate)*up, and the per-row softmax statistics
// of the LM head (logits are never stored).
#pragma once
#include "model.h"


namespace odb {

constexpr int WK = 8;    // waves per workgroup = K slices

struct GemmArgs {
    const u16 *A, *W;
    // fused RMSNorm of the input rows: A holds binary16(x * gain) and ssq[row][0..n_ssq) partial sums
    // of x^2; the result rows are scaled by 1/sqrt(sum/d + eps).  ssq == nullptr: A is used as is.
    const float *ssq;
    int KT, MT_total, NT, n_ssq;
    float eps, inv_d;
    // k-tiles this call covers (KT, or a slice of it).  A and W then point at the first k-tile of the slice; KT stays the
    // distance between the n-tiles of W.
    int k_len;
    // > 0: workgroup wg walks its k-tiles starting at (wg * k_rot) % (k-tiles per wave) and wraps round, so that the
    // workgroups, which all read the same activation tiles, do not ask the same L2 channels for them at the same time
    int k_rot;
    // workgroups that share the n-tiles, n-tiles of each where that divides them (else 0), divisor for k_rot: a workgroup
    // has nothing to request before it knows its tiles, and three divisions are 0.2 us
    int nwg, per;
    FastDiv fd_kw;
};
// (host) the fields that follow from the others
inline void set_shares(GemmArgs &g, int nwg) {
    g.nwg = nwg;
    g.per = g.NT % nwg == 0 ? g.NT / nwg : 0;
    g.fd_kw = FastDiv::make(g.k_len / WK);
}

// m-tiles per reduction pass: the sums of up to eighteen tiles per wave (144 KiB) go through LDS at a time.  A pass costs two
// barriers and a chain of LDS latencies whatever its size: with six tiles (48 KiB) the tail of a 64-row workgroup of 4 x 4
// tiles was four passes and 3.9 us.
constexpr int gemm_mc(int mt, int ng) {
    int mc = mt;
    while (mt % mc != 0 || mc * ng > 18) mc--;
    return mc;
}
// output tiles that a wave finishes: (m-chunk, tile) pairs, see gemm_wg
constexpr int gemm_slots(int mt, int ng) { return mt / gemm_mc(mt, ng) * ((gemm_mc(mt, ng) * ng + WK - 1) / WK); }
constexpr int gemm_red_bytes(int mt, int ng) { return WK * gemm_mc(mt, ng) * ng * 1024; }
constexpr int gemm_smem_bytes(int mt, int ng) { return gemm_red_bytes(mt, ng) + mt * 16 * 4; }    // red + row scales

// Hooks for epilogues that read global memory (the residual tile, the RoPE table): epi_preload issues those loads
// before the partial sums go through LDS, epi_apply hands their result to the epilogue, so that their latency runs
// under the reduction instead of in the tail of the kernel.  Default: nothing to preload.
struct NoPre {};
template <class Epi>
__device__ __forceinline__ NoPre epi_preload(const Epi &, int, int, int) { return NoPre{}; }
template <class Epi>
__device__ __forceinline__ void epi_apply(Epi &epi, int mt, int nt, f32x4 c, int lane, int slot, NoPre) { epi(mt, nt, c, lane, slot); }

// the sum of the eight waves' values: a chain of three additions, not of seven, and the smaller error
template <class F>
__device__ __forceinline__ auto pairwise(F f) {
    static_assert(WK == 8, "three levels");
    return ((f(0) + f(1)) + (f(2) + f(3))) + ((f(4) + f(5)) + (f(6) + f(7)));
}

// One workgroup's share of the GEMM: n-tiles [wg*NT/nwg, (wg+1)*NT/nwg), m-tiles mt0 .. mt0+MT-1.
// The epilogue is called as epi(mt, nt, c, lane, slot): slot numbers the (m-chunk, tile) pairs that
// this wave serves, the same in every group of n-tiles, so a stateful epilogue can keep one
// accumulator per slot; epi.finish(mt, part, lane, slot) follows once per slot at the end.
// smem: gemm_smem_bytes(MT, NG) bytes.  NTW: the weight tiles are read by this workgroup only, non-temporally.
template <int MT, int NG, int PF, class Epi, bool IL = false, bool NTW = true>
__device__ __forceinline__ void gemm_wg(const GemmArgs &g, Epi epi, int wg, int mt0, char *smem) {
    constexpr int MC = gemm_mc(MT, NG);                // m-tiles reduced per pass through LDS
    constexpr int SPW = (MC * NG + WK - 1) / WK;          // reduced tiles a wave serves per m-chunk
    static_assert(MT % MC == 0 && MT <= 8, "m chunking");
    f32x4 (*red)[MC * NG][64] = reinterpret_cast<f32x4 (*)[MC * NG][64]>(smem);
    float *s_rstd = reinterpret_cast<float *>(smem + gemm_red_bytes(MT, NG));

    // (all arguments in one go: read where they are first used they are a chain of scalar-cache misses)
    asm volatile("" ::"s"(g.A), "s"(g.W), "s"(g.ssq), "s"(g.KT), "s"(g.MT_total), "s"(g.NT), "s"(g.n_ssq), "s"(g.k_len), "s"(g.k_rot),
                 "s"(g.nwg), "s"(g.per), "s"(g.fd_kw.mul), "s"(g.fd_kw.div));
    const int lane = threadIdx.x & 63, wk = threadIdx.x >> 6;
    const int n_lo = g.per ? wg * g.per : (int)((unsigned)wg * (unsigned)g.NT / (unsigned)g.nwg);      // (32-bit: wg * NT stays far below 2^32)
    const int n_hi = g.per ? n_lo + g.per : (int)((unsigned)(wg + 1) * (unsigned)g.NT / (unsigned)g.nwg);
    if (n_lo >= n_hi) return;
    const int KW = g.k_len / WK;
    const int ngroups = (n_hi - n_lo + NG - 1) / NG;
    const int k0 = IL ? wk : wk * KW, kst = IL ? WK : 1;      // first k-tile of this wave and its stride

    // Row scales of the fused RMSNorm.  A row's partial sums (up to 256 of them) are one 16-byte
    // load per lane; the loads of all RPW rows of this wave are issued back to back and BEFORE the
    // first stage, so that waiting for them does not wait for the weight stream (loads return in
    // order), and they are only reduced after the ring has been filled.
    constexpr int RPW = MT * 16 / WK;                      // rows per wave
    float q[RPW];
    f32x4 sv[RPW];
    const int si = 4 * lane, sic = si < g.n_ssq - 4 ? si : g.n_ssq - 4;     // n_ssq is a multiple of 4
    if (g.ssq) {
#pragma unroll
        for (int j = 0; j < RPW; j++) {
            int row = mt0 * 16 + wk + j * WK;
            row = row < g.MT_total * 16 ? row : g.MT_total * 16 - 1;
            sv[j] = *reinterpret_cast<const f32x4 *>(g.ssq + (size_t)row * g.n_ssq + sic);
            q[j] = 0.f;
        }
        for (int i0 = 256; i0 < g.n_ssq; i0 += 256) {   // rows wider than 4096 only
            const int i = i0 + si, ic = i < g.n_ssq - 4 ? i : g.n_ssq - 4;
#pragma unroll
            for (int j = 0; j < RPW; j++) {
                int row = mt0 * 16 + wk + j * WK;
                row = row < g.MT_total * 16 ? row : g.MT_total * 16 - 1;
                const f32x4 v = *reinterpret_cast<const f32x4 *>(g.ssq + (size_t)row * g.n_ssq + ic);
                q[j] += i < g.n_ssq ? (v[0] + v[1]) + (v[2] + v[3]) : 0.f;
            }
        }
    }

    const u16 *wbase = g.W + (size_t)k0 * kTileElems + lane * 8;
    const u16 *ap[MT];
#pragma unroll
    for (int m = 0; m < MT; m++) {
        int mt = mt0 + m < g.MT_total ? mt0 + m : g.MT_total - 1;
        ap[m] = g.A + ((size_t)k0 * g.MT_total + mt) * kTileElems + lane * 8;
    }
    const size_t a_step = (size_t)g.MT_total * kTileElems * kst;

    frag_t wb[PF][NG], ab[PF][MT];
    int rot = 0;
    if (g.k_rot > 0) {
        const int x = wg * g.k_rot;                     // below 2^16
        rot = x - g.fd_kw.quot(x) * KW;
    }
    auto load_stage = [&](int slot, int grp, int k_seq) __attribute__((always_inline)) {
        int kk = k_seq + rot;
        kk = kk >= KW ? kk - KW : kk;
#pragma unroll
        for (int n = 0; n < NG; n++) {
            int nt = n_lo + grp * NG + n;
            nt = nt < n_hi ? nt : n_hi - 1;
            const u16 *p = wbase + ((size_t)nt * g.KT + kk * kst) * kTileElems;
            wb[slot][n] = NTW ? ld_frag_stream(p) : ld_frag(p);
        }
#pragma unroll
        for (int m = 0; m < MT; m++) ab[slot][m] = ld_frag(ap[m] + kk * a_step);
    };
#pragma unroll
    for (int s = 0; s < PF; s++) load_stage(s, 0, s);
    if (g.ssq) {
        // 64 lane-partials per row -> one sum per row: transposed through LDS (row stride 65 floats keeps
        // the gather conflict-free), then lane l adds RPW of the partials of row l % RPW and the 64 / RPW
        // lanes of a row finish with shuffles.  A wave only touches its own part of the reduction buffer: no barrier before
        // the one in front of the first sums, which publishes the scales too.
        // (RP: RPW rounded up to a power of two - six row tiles over eight waves give twelve rows per wave;
        // the lanes of the rows beyond RPW add stale scratch and are dropped)
        constexpr int RP = RPW <= 4 ? 4 : RPW <= 8 ? 8 : 16;
        static_assert(RPW <= 16 && RP * 65 * 4 <= MC * NG * 1024, "a wave's part of the buffer");
        float *tmp = reinterpret_cast<float *>(&red[wk][0][0]);
#pragma unroll
        for (int j = 0; j < RPW; j++)
            tmp[j * 65 + lane] = q[j] + (si < g.n_ssq ? (sv[j][0] + sv[j][1]) + (sv[j][2] + sv[j][3]) : 0.f);
        const int row = lane % RP, part = lane / RP;
        float t = 0.f;
#pragma unroll
        for (int i = 0; i < RP; i++) t += tmp[row * 65 + part * RP + i];
#pragma unroll
        for (int o = RP; o < 64; o <<= 1) t += __shfl_xor(t, o);
        if (lane < RPW) s_rstd[wk + lane * WK] = 1.0f / sqrtf(t * g.inv_d + g.eps);
    } else if (lane < RPW) {
        s_rstd[wk + lane * WK] = 1.0f;
    }

    for (int grp = 0; grp < ngroups; grp++) {
        f32x4 acc[MT][NG];
#pragma unroll
        for (int m = 0; m < MT; m++)
#pragma unroll
            for (int n = 0; n < NG; n++) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};

        for (int kb = 0; kb < KW; kb += PF) {
#pragma unroll
            for (int s = 0; s < PF; s++) {
#pragma unroll
                for (int m = 0; m < MT; m++)
#pragma unroll
                    for (int n = 0; n < NG; n++) acc[m][n] = mfma16(wb[s][n], ab[s][m], acc[m][n]);
                // refill this slot with the step PF ahead, which may belong to the next group
                int kn = kb + s + PF, gn = grp;
                if (kn >= KW) { kn -= KW; gn++; }
                if (gn < ngroups) load_stage(s, gn, kn);
            }
        }

        // add the eight K-slices through LDS, MC m-tiles at a time; the wave that owns a tile runs its epilogue
#pragma unroll
        for (int mc = 0; mc < MT; mc += MC) {
            decltype(epi_preload(epi, 0, 0, 0)) pre[SPW];
#pragma unroll
            for (int u = 0; u < SPW; u++) {
                const int t = wk + u * WK, m = t / NG, n = t % NG;
                const int mt = mt0 + mc + m, nt = n_lo + grp * NG + n;
                if (t < MC * NG && mt < g.MT_total && nt < n_hi) pre[u] = epi_preload(epi, mt, nt, lane);
            }
#pragma unroll
            for (int m = 0; m < MC; m++)
#pragma unroll
                for (int n = 0; n < NG; n++) red[wk][m * NG + n][lane] = acc[mc + m][n];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < SPW; u++) {
                const int t = wk + u * WK;
                if (t >= MC * NG) break;
                const int m = t / NG, n = t % NG;
                const int mt = mt0 + mc + m, nt = n_lo + grp * NG + n;
                if (mt < g.MT_total && nt < n_hi) {
                    f32x4 c;
                    if (!epi.transposed(nt)) {
                        c = pairwise([&](int w) { return red[w][t][lane]; });
                        c *= s_rstd[(mc + m) * 16 + (lane & 15)];
                    } else {
                        // hand lane (g, ni) the four rows 4g..4g+3 of column ni instead of four columns of one row
                        const int ni = lane & 15, gq = lane >> 4;
                        const float *base = reinterpret_cast<const float *>(&red[0][t][0]);
                        const int stride = MC * NG * 64 * 4;        // floats between the waves' copies
#pragma unroll
                        for (int r = 0; r < 4; r++) {
                            const int src = ((ni >> 2) * 16 + 4 * gq + r) * 4 + (ni & 3);
                            const float v = pairwise([&](int w) { return base[w * stride + src]; });
                            c[r] = v * s_rstd[(mc + m) * 16 + 4 * gq + r];
                        }
                    }
                    epi_apply(epi, mt, nt, c, lane, (mc / MC) * SPW + u, pre[u]);
                }
            }
            if (mc + MC < MT || grp + 1 < ngroups) __syncthreads();         // (the buffer is written again)
        }
    }
    // epilogues that accumulate over the n-tiles of the workgroup write their result now
#pragma unroll
    for (int mc = 0; mc < MT; mc += MC)
#pragma unroll
        for (int u = 0; u < SPW; u++) {
            const int t = wk + u * WK;         // a tile this wave served in every group
            if (t < MC * NG && mt0 + mc + t / NG < g.MT_total)
                epi.finish(mt0 + mc + t / NG, wg * NG + t % NG, lane, (mc / MC) * SPW + u);
        }
}

// ---- epilogues ------------------------------------------------------------------
// Default:    lane l holds C[row = 16*mt + (l&15)][col = 16*nt + 4*(l>>4) + r], r = 0..3.
// Transposed: lane l holds C[row = 16*mt + 4*(l>>4) + r][col = 16*nt + (l&15)].

__device__ inline void st_f16x4(u16 *p, float a, float b, float c, float d) { *reinterpret_cast<uint2 *>(p) = pack4(a, b, c, d); }

// (by-value pick: `c ? x : y` on two struct members is an lvalue conditional, which the compiler turns into a
// select of addresses and then parks the members on the stack)
template <class T>
__device__ __forceinline__ T pick(bool c, T a, T b) { return c ? a : b; }

struct QkvPre { f32x4 cs; u16 *dst; bool rotate; };
struct EpiQKV {
    QkvOut o;
    __device__ bool transposed(int nt) const { return nt * 16 >= 2 * o.d; }
    __device__ void finish(int, int, int, int) const {}
    // where a tile goes, and the (cos, sin) of the lane's two channel pairs: requested before the sums are there
    __device__ QkvPre preload(int mt, int nt, int lane) const {
        const int mi = lane & 15, g = lane >> 4;
        // unit and tile inside the unit; in the decoded-share step the speculative units have their own size and K/V area
        const bool spec = o.split_tile > 0 && mt >= o.split_tile;
        const int tpu = pick(spec, o.tiles_per_unit_b, o.tiles_per_unit), mtu = pick(spec, mt - o.split_tile, mt);
        const int unit = pick(spec, o.fd_tpu_b, o.fd_tpu).quot(mtu), tu = mtu - unit * tpu;
        u16 *kdst = pick(spec, o.k_b, o.k) + unit * pick(spec, o.k_b_unit_stride, o.k_unit_stride);
        u16 *vdst = pick(spec, o.v_b, o.v) + unit * pick(spec, o.v_b_unit_stride, o.v_unit_stride);
        const size_t khs = pick(spec, o.k_b_head_stride, o.k_head_stride), vhs = pick(spec, o.v_b_head_stride, o.v_head_stride);
        // (index arithmetic on tiles with precomputed multipliers)
        const int sec = o.fd_d.quot(nt), rt = nt - sec * (o.d >> 4);
        const int hd = o.fd_dh.quot(rt), p0 = (rt - hd * (o.dh >> 4)) * 16;            // p0 is a multiple of 16
        QkvPre p;
        p.rotate = sec < 2;
        if (sec < 2) {
            // physical channel 2j is logical j, 2j+1 is j + dh/2: each adjacent pair is a RoPE pair
            const int pos = o.rowpos ? o.rowpos[mt * 16 + mi] : o.pos_off + tu * 16 + mi;
            p.cs = *reinterpret_cast<const f32x4 *>(o.rope + (size_t)pos * o.dh + p0 + 4 * g);
            const int kk = (p0 & 16) + 4 * g;                 // k-element of the lane's first channel inside the 32-wide tile
            p.dst = (sec == 0 ? o.q + (((size_t)hd * o.q_mt + mt) * (o.dh / 32) + p0 / 32) * kTileElems
                              : kdst + hd * khs + ((size_t)tu * (o.dh / 32) + p0 / 32) * kTileElems) + ((kk >> 3) * 16 + mi) * 8 + (kk & 7);
        } else {
            // V^T tile: row = channel, the 32 keys of a tile sit in k-slot 8*g + 4*half + r
            p.cs = f32x4{1.f, 0.f, 1.f, 0.f};
            p.dst = vdst + hd * vhs + ((size_t)(tu >> 1) * (o.dh / 16) + p0 / 16) * kTileElems + lane * 8 + 4 * (tu & 1);
        }
        return p;
    }
    __device__ void apply(f32x4 c, const QkvPre &p) const {
        if (p.rotate)
            c = f32x4{c[0] * p.cs[0] - c[1] * p.cs[1], c[1] * p.cs[0] + c[0] * p.cs[1],
                      c[2] * p.cs[2] - c[3] * p.cs[3], c[3] * p.cs[2] + c[2] * p.cs[3]};
        note_saturation(o.status, c[0], c[1], c[2], c[3]);
        st_f16x4(p.dst, c[0], c[1], c[2], c[3]);
    }
    __device__ void operator()(int mt, int nt, f32x4 c, int lane, int) const { apply(c, preload(mt, nt, lane)); }
};
__device__ __forceinline__ QkvPre epi_preload(const EpiQKV &e, int mt, int nt, int lane) { return e.preload(mt, nt, lane); }
__device__ __forceinline__ void epi_apply(EpiQKV &e, int, int, f32x4 c, int, int, const QkvPre &pre) { e.apply(c, pre); }

// The same for dense rows (QkvOut), as kernels of their own: the index arithmetic would cost the others registers.  A lane's row of
// Q and K has a unit of its own, and the four rows of V that a lane holds may lie in two units, so they are stored one by one.
struct EpiQKVDense {
    QkvOut o;
    __device__ bool transposed(int nt) const { return nt * 16 >= 2 * o.d; }
    __device__ void finish(int, int, int, int) const {}
    struct Col { int sec, hd, p0; };           // Q, K or V, head, first physical channel of an n-tile
    __device__ Col column(int nt) const {
        const int sec = o.fd_d.quot(nt), rt = nt - sec * (o.d >> 4), hd = o.fd_dh.quot(rt);
        return Col{sec, hd, (rt - hd * (o.dh >> 4)) * 16};
    }
    // the (cos, sin) of the lane's two channel pairs: requested before the sums are there
    __device__ f32x4 preload(int mt, int nt, int lane) const {
        asm volatile("" : "+v"(lane));          // (the rows' places are found where they are used: kept over the k-loop they spill)
        const Col n = column(nt);
        if (n.sec == 2) return f32x4{1.f, 0.f, 1.f, 0.f};
        const int row = mt * 16 + (lane & 15), i = row - o.fd_valid.quot(row) * o.valid;
        return *reinterpret_cast<const f32x4 *>(o.rope + (size_t)(o.pos_off + i) * o.dh + n.p0 + 4 * (lane >> 4));
    }
    __device__ void apply(int mt, int nt, f32x4 c, int lane, f32x4 cs) const {
        asm volatile("" : "+v"(lane));
        const Col n = column(nt);
        const int mi = lane & 15, g = lane >> 4;
        if (n.sec < 2) {
            c = f32x4{c[0] * cs[0] - c[1] * cs[1], c[1] * cs[0] + c[0] * cs[1], c[2] * cs[2] - c[3] * cs[3], c[3] * cs[2] + c[2] * cs[3]};
            note_saturation(o.status, c[0], c[1], c[2], c[3]);
            const int row = mt * 16 + mi, unit = o.fd_valid.quot(row), i = row - unit * o.valid, kk = (n.p0 & 16) + 4 * g;
            u16 *base = n.sec == 0 ? o.q + ((size_t)n.hd * o.q_mt + unit * o.tiles_per_unit) * (o.dh / 32) * kTileElems
                                   : o.k + unit * o.k_unit_stride + n.hd * o.k_head_stride;
            if (row < o.dense_rows)
                st_f16x4(base + ((size_t)(i >> 4) * (o.dh / 32) + n.p0 / 32) * kTileElems + ((kk >> 3) * 16 + (i & 15)) * 8 + (kk & 7), c[0], c[1], c[2], c[3]);
        } else {
            note_saturation(o.status, c[0], c[1], c[2], c[3]);
            u16 *base = o.v + n.hd * o.v_head_stride + (n.p0 / 16) * kTileElems + mi * 8;
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int row = mt * 16 + 4 * g + r, unit = o.fd_valid.quot(row), i = row - unit * o.valid;
                if (row < o.dense_rows)
                    base[unit * o.v_unit_stride + (size_t)(i >> 5) * (o.dh / 16) * kTileElems + ((i & 15) >> 2) * 128 + 4 * ((i >> 4) & 1) + (i & 3)] = f2h(c[r]);
            }
        }
    }
    __device__ void operator()(int mt, int nt, f32x4 c, int lane, int) const { apply(mt, nt, c, lane, preload(mt, nt, lane)); }
};
__device__ __forceinline__ f32x4 epi_preload(const EpiQKVDense &e, int mt, int nt, int lane) { return e.preload(mt, nt, lane); }
__device__ __forceinline__ void epi_apply(EpiQKVDense &e, int mt, int nt, f32x4 c, int lane, int, f32x4 pre) { e.apply(mt, nt, c, lane, pre); }

// h += C.  With a NormOut it also prepares the next RMSNorm: hb = binary16(h * gain) in the
// operand layout and the sum of squares of this tile's 16 columns per row.
// What EpiResid reads from global memory for one output tile: the residual values and (when the tile also feeds the
// next RMSNorm) the norm's gain - both requested before the sums are there, not in a chain behind them.
struct ResidPre { f32x4 hv, gn; };
struct EpiResid {
    float *h;
    int ld;
    NormOut no;
    int mt_total;
    __device__ bool transposed(int) const { return false; }
    __device__ void finish(int, int, int, int) const {}
    __device__ ResidPre preload(int mt, int nt, int lane) const {
        const int mi = lane & 15, g = lane >> 4, row = mt * 16 + mi, col = nt * 16 + 4 * g;
        ResidPre p;
        p.hv = *reinterpret_cast<const f32x4 *>(h + (size_t)row * ld + col);
        p.gn = no.hb ? *reinterpret_cast<const f32x4 *>(no.gain + col) : f32x4{0.f, 0.f, 0.f, 0.f};
        return p;
    }
    __device__ void operator()(int mt, int nt, f32x4 c, int lane, int) const { apply(mt, nt, c, lane, preload(mt, nt, lane)); }
    // h += c and the next norm's input for one output tile; returns the lane's sum of squares over its four columns
    __device__ float put(int mt, int nt, f32x4 c, int lane, const ResidPre &pre) const {
        const int mi = lane & 15, g = lane >> 4, row = mt * 16 + mi, col = nt * 16 + 4 * g;
        float *p = h + (size_t)row * ld + col;
        f32x4 v = pre.hv + c;
        *reinterpret_cast<f32x4 *>(p) = v;
        if (!no.hb) return 0.f;
        const int kk = (nt & 1) * 16 + 4 * g;
        const f32x4 y = v * pre.gn;
        note_saturation(no.status, y[0], y[1], y[2], y[3]);
        *reinterpret_cast<uint2 *>(no.hb + ((size_t)(nt >> 1) * mt_total + mt) * kTileElems + ((kk >> 3) * 16 + mi) * 8 + (kk & 7)) =
            pack4(y[0], y[1], y[2], y[3]);
        return v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
    }
    __device__ static float over_row(float q) {         // sum over the four lanes of a row
        q += __shfl_xor(q, 16);
        return q + __shfl_xor(q, 32);
    }
    __device__ void apply(int mt, int nt, f32x4 c, int lane, const ResidPre &pre) const {
        const float q = over_row(put(mt, nt, c, lane, pre));
        if (no.hb && lane < 16) no.ssq[(size_t)(mt * 16 + lane) * no.n_ssq + nt] = q;
    }
};

__device__ __forceinline__ ResidPre epi_preload(const EpiResid &e, int mt, int nt, int lane) { return e.preload(mt, nt, lane); }
__device__ __forceinline__ void epi_apply(EpiResid &e, int mt, int nt, f32x4 c, int lane, int, const ResidPre &pre) { e.apply(mt, nt, c, lane, pre); }

// The same with the sums of squares left in LDS, s_q[row tile][n-tile][16 rows] of the workgroup's block, for sums over 64 columns.
template <int NG>
struct EpiResidSums {
    EpiResid r;
    float *s_q;
    int mt0, nt0;
    __device__ bool transposed(int) const { return false; }
    __device__ void finish(int, int, int, int) const {}
};
template <int NG>
__device__ __forceinline__ ResidPre epi_preload(const EpiResidSums<NG> &e, int mt, int nt, int lane) { return e.r.preload(mt, nt, lane); }
template <int NG>
__device__ __forceinline__ void epi_apply(EpiResidSums<NG> &e, int mt, int nt, f32x4 c, int lane, int, const ResidPre &pre) {
    const float q = EpiResid::over_row(e.r.put(mt, nt, c, lane, pre));
    if (lane < 16) e.s_q[((mt - e.mt0) * NG + nt - e.nt0) * 16 + lane] = q;
}

// W_gu interleaves the rows of W_gate and W_up (physical row 2j = gate j, 2j+1 = up j)
struct EpiSwiGLU {
    u16 *act;
    int mt_total;
    unsigned *status;
    __device__ bool transposed(int) const { return false; }
    __device__ void finish(int, int, int, int) const {}
    // silu(gate) * up with the hardware exponential and reciprocal (each good to 1 ulp; the result is rounded to
    // binary16 next): the exact division and exponential are some forty instructions per pair in the kernel's tail
    __device__ static float act2(float gate, float up) { return gate * __builtin_amdgcn_rcpf(1.0f + __expf(-gate)) * up; }
    __device__ void operator()(int mt, int nt, f32x4 c, int lane, int) const {
        const int mi = lane & 15, g = lane >> 4;
        const int j = nt * 8 + 2 * g;                         // channel of the first (gate, up) pair
        const float y0 = act2(c[0], c[1]), y1 = act2(c[2], c[3]);
        const int kk = j & 31;
        note_saturation(status, y0, y1, 0.f, 0.f);
        u16 *dst = act + ((size_t)(j >> 5) * mt_total + mt) * kTileElems + ((kk >> 3) * 16 + mi) * 8 + (kk & 7);
        *reinterpret_cast<uint32_t *>(dst) = pack2(y0, y1);
    }
};

// Softmax statistics of the LM head without ever storing logits.  A wave serves the same
// (m-tile, n-slot) pairs in every group of n-tiles of its workgroup, so it keeps a running
// (max, sum exp(z - max), argmax) per row and slot in registers and writes ONE partial per row and
// slot at the end: stats[row][part], part = workgroup * NG + n-slot.  Ties keep the lowest token id.
// PASSES = slots per wave (see gemm_wg).
// (Exponentials are the hardware instruction, relative error about 1e-6 at the arguments that matter: they sit between
// the groups of the weight stream, and the error of a confidence is dominated by that of the logits, about 1e-3.)
template <int PASSES>
struct EpiLMStats {
    float *stats;
    int n_part;
    float rm[PASSES], rs[PASSES];
    int ra[PASSES];
    __host__ __device__ EpiLMStats(float *st, int np) : stats(st), n_part(np) {
#pragma unroll
        for (int p = 0; p < PASSES; p++) { rm[p] = -INFINITY; rs[p] = 0.f; ra[p] = 0x7fffffff; }
    }
    __device__ bool transposed(int) const { return false; }
    __device__ void operator()(int mt, int nt, f32x4 c, int lane, int pass) {
        const int g = lane >> 4;
        float m = c[0];
        int a = nt * 16 + 4 * g;
#pragma unroll
        for (int r = 1; r < 4; r++)
            if (c[r] > m) { m = c[r]; a = nt * 16 + 4 * g + r; }
        float s = 0.f;
#pragma unroll
        for (int r = 0; r < 4; r++) s += __expf(c[r] - m);
#pragma unroll
        for (int p = 0; p < PASSES; p++)
            if (p == pass) {
                float nm = fmaxf(rm[p], m);
                rs[p] = rs[p] * (rm[p] == nm ? 1.f : __expf(rm[p] - nm)) + s * (m == nm ? 1.f : __expf(m - nm));
                ra[p] = rm[p] > m ? ra[p] : (m > rm[p] ? a : (ra[p] < a ? ra[p] : a));
                rm[p] = nm;
            }
    }
    __device__ void finish(int mt, int part, int lane, int pass) const {
        const int mi = lane & 15, g = lane >> 4;
        float m = -INFINITY, s = 0.f;
        int a = 0x7fffffff;
#pragma unroll
        for (int p = 0; p < PASSES; p++)
            if (p == pass) { m = rm[p]; s = rs[p]; a = ra[p]; }
#pragma unroll
        for (int o = 16; o <= 32; o <<= 1) {
            float om = __shfl_xor(m, o), os = __shfl_xor(s, o);
            int oa = __shfl_xor(a, o);
            float nm = fmaxf(m, om);
            s = s * (m == nm ? 1.f : __expf(m - nm)) + os * (om == nm ? 1.f : __expf(om - nm));
            a = m > om ? a : (om > m ? oa : (a < oa ? a : oa));
            m = nm;
        }
        if (g == 0) {
            float *p = stats + ((size_t)(mt * 16 + mi) * n_part + part) * 3;
            p[0] = m;
            p[1] = s;
            p[2] = __int_as_float(a);
        }
    }
};

// plain fp32 store of the valid rows (unit u, i < valid) to a compact row-major matrix
struct EpiStore {
    float *out;
    int units, rpu_pad, valid, ld;
    __device__ bool transposed(int) const { return false; }
    __device__ void finish(int, int, int, int) const {}
    __device__ void operator()(int mt, int nt, f32x4 c, int lane, int) const {
        int row = mt * 16 + (lane & 15);
        int u = row / rpu_pad, i = row % rpu_pad;
        if (u < units && i < valid)
            *reinterpret_cast<f32x4 *>(out + ((size_t)u * valid + i) * ld + nt * 16 + 4 * (lane >> 4)) = c;
    }
};

// One K slice's sums, left for the workgroup that finishes the tile (gemm.hip: gemm_stream_ksplit_kernel):
// p[m_tile][n_tile][lane] holds the lane's fragment.  Written with device-coherent stores (sc1) so that a workgroup on
// another XCD reads them without any cache-wide fence.
constexpr int kDeviceScope = 16;            // sc1 in the cache policy operand of a buffer load or store
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t sums_rsrc(const float *p, size_t bytes) {     // p: the same in all lanes
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p), 0, (int)(unsigned)bytes, 0x00027000);
}
struct EpiPartial {
    float *p;
    int nt_total, mt_total;
    __device__ bool transposed(int) const { return false; }
    __device__ void finish(int, int, int, int) const {}
    __device__ void operator()(int mt, int nt, f32x4 c, int lane, int) const {
        const unsigned at = ((unsigned)mt * nt_total + nt) * 1024 + lane * 16;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, c), sums_rsrc(p, (size_t)mt_total * nt_total * 1024), at, 0, kDeviceScope);
    }
};

}  // namespace odb
