// binary16 MFMA GEMM  C[M,N] = A[M,K] * W[N,K]^T  for the wide projections at 97 to 128 rows (and QKV at two such row
// blocks): a workgroup owns 128 rows and NTB n-tiles, and everything it reads goes through LDS.
//
// What bounds these shapes is the way of the operands into a compute unit: it needs all the activations (1 MB at 128 rows
// of K = 4096) beside its share of the weights, and the two add up (copies alone at 128 rows: QKV 15 us for the
// activations, 19 us for the weights, 28 us for both; gate/up 17, 37 and 46): requests are served in order, so what comes
// from L2 waits behind what comes from HBM, also when different waves ask for the two (separate rings for A and W, the
// latter twice as deep: no gain).  What can be saved is the rest.  Eight waves copy the tiles of a stage (two k-tiles)
// straight from global memory into a ring of LDS stages, 110 KiB of copies in flight per compute unit, and the LDS reads
// and MFMAs run entirely under the copies; the streaming kernel (gemm_core.h), whose loads wait in MFMA registers, took
// 46.5 us for gate/up and 32.5 for QKV at 128 rows, this one 42.4 and 31.0.  Below 97 rows the streaming kernel stays ahead
// (64 rows: 36.6 us for either, QKV 24.6 against 27.9).
#pragma once
#include "gemm_big.h"

namespace odb {

struct SlabArgs {
    const u16 *A, *W;
    int KT, MT_total, NT;
    const float *ssq;          // fused RMSNorm of the input rows (see GemmArgs)
    int n_ssq;
    float eps, inv_d;
};

constexpr int kSlabKP = 2;                                                    // k-tiles per stage
constexpr int slab_stages(int ntb) { return 150 / (kSlabKP * (8 + ntb)); }
constexpr int slab_smem_bytes(int ntb) { return slab_stages(ntb) * kSlabKP * (8 + ntb) * 1024 + 128 * 4; }

// NTW: the weight tiles are loaded non-temporally.
template <int NTB, class Epi, bool NTW>
__global__ __launch_bounds__(512) void gemm_slab_kernel(SlabArgs g, Epi epi) {
    constexpr int CS = NTB % 2 == 0 ? 2 : 1, RS = 4 / CS;       // the four waves of a group over columns and rows
    constexpr int WT = NTB / CS, MW = 8 / RS;                   // tiles per wave
    constexpr int TK = 8 + NTB, ST = kSlabKP * TK, NS = slab_stages(NTB);       // tiles per k-tile and stage, stages
    static_assert(NS >= 3, "ring");
    static_assert(NS * ST >= 64 + 8 * kBigScratch / 1024 && 4 * MW * WT <= 64, "scratch of the epilogues");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float *s_rstd = reinterpret_cast<float *>(smem + NS * ST * 1024);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = w >> 2, wr = (w & 3) / CS, wc = (w & 3) % CS;
    const int nt0 = blockIdx.x * NTB, mt0 = blockIdx.y * 8;
    const int ns = g.KT / kSlabKP;                              // stages (k-tiles come in eights)

    // Of a stage's kSlabKP x NTB tiles of W wave w copies those numbered w, w + 8, .., of its 16 tiles of A those numbered
    // 7 - w and 15 - w.  A single row block reads W once, non-temporally (gate/up 44.7 -> 42.5 us at 128 rows).  Of two row
    // blocks the second finds the tiles in L2 or not, but only a nearly empty one gains by their being kept there (QKV of d 3072 at 144
    // rows 30.4 -> 27.8 us, at 256 31.0 -> 31.6; over all widths 4 % faster at 144 rows, equal at 176, 1.5 % slower at 256).  The
    // workgroups walk K from different places, so that they do not ask the same L2 channels for the same tiles of A at once.
    constexpr int PW = (kSlabKP * NTB + 7) / 8, RW = (kSlabKP * NTB - 1) % 8 + 1, PA = kSlabKP;
    const bool fw = w < RW;                                     // whether this wave has PW tiles of W to copy or one less
    const char *srcw[PW], *srca[PA];
#pragma unroll
    for (int i = 0; i < PW; i++) {
        int t = i * 8 + w;
        t = t < kSlabKP * NTB ? t : 0;
        const int nt = nt0 + t % NTB < g.NT ? nt0 + t % NTB : g.NT - 1;
        srcw[i] = reinterpret_cast<const char *>(g.W + ((size_t)nt * g.KT + t / NTB) * kTileElems);
    }
#pragma unroll
    for (int i = 0; i < PA; i++) {
        const int mt = mt0 + 7 - w < g.MT_total ? mt0 + 7 - w : g.MT_total - 1;
        srca[i] = reinterpret_cast<const char *>(g.A + ((size_t)i * g.MT_total + mt) * kTileElems);
    }
    const size_t astep = (size_t)kSlabKP * g.MT_total * kTileElems * 2, wstep = (size_t)kSlabKP * kTileElems * 2;
    const unsigned lane_off = lane * 16;
    const int rot = (int)(blockIdx.x * 7u % (unsigned)ns);
    auto issue = [&](int slot, int s) __attribute__((always_inline)) {
        int sk = s + rot;
        sk = sk >= ns ? sk - ns : sk;
        const size_t ow = sk * wstep, oa = sk * astep;
#pragma unroll
        for (int i = 0; i < PW; i++) {
            const int t = i * 8 + w;
            if (i < PW - 1 || fw)
                __builtin_amdgcn_global_load_lds(reinterpret_cast<const void *>(srcw[i] + ow + lane_off),
                                                 (__attribute__((address_space(3))) void *)(smem + (slot * ST + t / NTB * TK + 8 + t % NTB) * 1024), 16, 0, NTW ? 2 : 0);
        }
#pragma unroll
        for (int i = 0; i < PA; i++)
            __builtin_amdgcn_global_load_lds(reinterpret_cast<const void *>(srca[i] + oa + lane_off),
                                             (__attribute__((address_space(3))) void *)(smem + (slot * ST + i * TK + 7 - w) * 1024), 16, 0, 0);
    };
#pragma unroll
    for (int j = 0; j < NS - 1; j++)
        if (j < ns) issue(j, j);

    // row scales of the fused RMSNorm: four threads per row, behind the ring's first copies
    {
        const int r = threadIdx.x >> 2, part = threadIdx.x & 3;
        float t = 1.f;
        if (g.ssq) {
            const int row = mt0 * 16 + r < g.MT_total * 16 ? mt0 * 16 + r : g.MT_total * 16 - 1;
            const float *p = g.ssq + (size_t)row * g.n_ssq;
            t = 0.f;
#pragma unroll 8
            for (int i = part * 4; i < g.n_ssq; i += 16) {              // n_ssq is a multiple of 4
                const f32x4 v = *reinterpret_cast<const f32x4 *>(p + i);
                t += (v[0] + v[1]) + (v[2] + v[3]);
            }
            t += __shfl_xor(t, 1);
            t += __shfl_xor(t, 2);
            t = 1.0f / sqrtf(t * g.inv_d + g.eps);
        }
        if (part == 0) s_rstd[r] = t;
    }

    f32x4 acc[MW][WT];
#pragma unroll
    for (int m = 0; m < MW; m++)
#pragma unroll
        for (int j = 0; j < WT; j++) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Two groups of four waves share K: group 0 takes the even stages, group 1 the odd ones.  In the interval behind the
    // barrier of stage s its group reads its operands from LDS while the other group multiplies those of stage s - 1
    // (all eight waves in step, reading and multiplying every stage, left the chain of the two on the critical path).
    // Stage s has landed when every wave has waited for its own copies of it, in front of that barrier; there the reads of
    // stage s - 1 are complete too, and its slot takes stage s + NS - 1.
    frag_t a[kSlabKP][MW], b[kSlabKP][WT];
#pragma unroll
    for (int q = 0; q < kSlabKP; q++) {
#pragma unroll
        for (int j = 0; j < WT; j++) b[q][j] = frag_t{{0, 0, 0, 0}};
#pragma unroll
        for (int m = 0; m < MW; m++) a[q][m] = frag_t{{0, 0, 0, 0}};
    }
    auto mfmas = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kSlabKP; q++)
#pragma unroll
            for (int m = 0; m < MW; m++)
#pragma unroll
                for (int j = 0; j < WT; j++) acc[m][j] = mfma16(b[q][j], a[q][m], acc[m][j]);
    };
    for (int s = 0, slot = 0; s < ns; s++) {
        if (s + NS - 2 >= ns) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else if (fw) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((PW + PA) * (NS - 2)) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((PW - 1 + PA) * (NS - 2)) : "memory");
        __builtin_amdgcn_s_barrier();
        if ((s & 1) == grp) {
            const frag_t (*st)[64] = reinterpret_cast<const frag_t (*)[64]>(smem + slot * ST * 1024);
#pragma unroll
            for (int q = 0; q < kSlabKP; q++) {
#pragma unroll
                for (int j = 0; j < WT; j++) b[q][j] = st[q * TK + 8 + wc * WT + j][lane];
#pragma unroll
                for (int m = 0; m < MW; m++) a[q][m] = st[q * TK + wr * MW + m][lane];
            }
        }
        if (s + NS - 1 < ns) issue(slot == 0 ? NS - 1 : slot - 1, s + NS - 1);
        slot = slot == NS - 1 ? 0 : slot + 1;
        if ((s & 1) != grp) mfmas();               // (nothing but zeros before a group's first stage)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
    if (((ns - 1) & 1) == grp) mfmas();
    __syncthreads();            // the ring is reused below; publishes s_rstd where nothing else did

    // Add the groups' sums: each wave hands the rows that its counterpart finishes over through LDS
    constexpr int MH = MW / 2;                     // row tiles finished by group 0; group 1 takes the others
    f32x4 (*xch)[64] = reinterpret_cast<f32x4 (*)[64]>(smem + (w & 3) * MW * WT * 1024);       // 4 x MW x WT KiB
#pragma unroll
    for (int m = 0; m < MW; m++)
#pragma unroll
        for (int j = 0; j < WT; j++)
            if ((m < MH) == (grp == 1)) xch[m * WT + j][lane] = acc[m][j];
    __syncthreads();
#pragma unroll
    for (int m = 0; m < MW; m++)
#pragma unroll
        for (int j = 0; j < WT; j++)
            if ((m < MH) == (grp == 0)) acc[m][j] += xch[m * WT + j][lane];
    auto finish = [&](auto M0) __attribute__((always_inline)) {
        constexpr int m0 = decltype(M0)::value;
        const int mtw = mt0 + wr * MW + m0;
        if (mtw >= g.MT_total) return;
        f32x4 c[MH][WT];
#pragma unroll
        for (int m = 0; m < MH; m++)
#pragma unroll
            for (int j = 0; j < WT; j++) c[m][j] = acc[m0 + m][j];
        BigArgs bg{};
        bg.MT_total = g.MT_total;
        bg.NT = g.NT;
        big_epilogue<MH, WT>(epi, c, mtw, nt0 + wc * WT, bg, s_rstd + (mtw - mt0) * 16, smem + 64 * 1024 + w * kBigScratch, lane);
    };
    if (grp == 0) finish(std::integral_constant<int, 0>{});
    else finish(std::integral_constant<int, MH>{});
}

}  // namespace odb
