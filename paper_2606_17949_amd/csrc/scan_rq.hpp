// The bank scan of the exact k-nearest-neighbour search (RouteBalance Sec. 4.2:
// the KNN lookup of Alg. 1) for a batch whose whole query tile fits in the
// registers of one workgroup: bf16 rows of NKS full k-steps, at most
// (RQ_WAVES / RS) * QW * 16 queries.
#pragma once

#include "knn_common.hpp"

namespace rb {

namespace {

// Global -> LDS load of 4 bytes per lane (lane l's bytes land at dst + 4*l).
__device__ __forceinline__ void dma4(__amdgpu_buffer_rsrc_t r, float *dst, uint32_t voffset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 4,
                                             (int)voffset, 0, 0, 0);
}

// Bank fragments travel from HBM to LDS in whole 128-byte lines: one
// global-to-LDS load brings 8 rows x 128 bytes (two k-steps of each row,
// eight 16-byte chunks of one line per group of 8 lanes), so every line is
// fetched by one instruction. In LDS, load f of a stage (row group
// rg = f % 4 of the block, k-step pair f / 4) holds row rg*8 + ri's chunk c
// (quarter c % 4 of k-step 2*(f/4) + c/4) at position
// 8*ri + (c ^ rq_perm(ri) ^ 2*(rg & 1)), rq_perm taking the row pairs of a
// group to 0, 1, 4, 5. The MFMA A-fragment read (lane (col, jg): row col,
// quarter jg of one k-step) then puts the sixteen lanes that LDS serves
// together (lanes 8p..8p+7 and 32+8p..32+8p+7: eight rows at quarters jg
// and jg + 2) on distinct bank groups, as it does the sixteen rows of one
// quarter: no bank conflicts (a plain XOR with the row, which spreads only
// the latter, costs four conflict cycles per read).
__device__ __forceinline__ int rq_perm(int ri)
{
    return ((ri >> 1) & 1) | ((ri >> 2) << 2);
}
__device__ __forceinline__ uint32_t rq_chunk(int ri, int rg, int c)
{
    return (uint32_t)(8 * ri + (c ^ rq_perm(ri) ^ (2 * (rg & 1))));
}

// One workgroup per bank chunk; RQ_WAVES waves, two per SIMD, in RS row
// halves of RQ_WAVES / RS query slots. Wave w owns the queries of slot
// w % (RQ_WAVES / RS), [16*QW*slot, 16*QW*(slot+1)), and holds their
// fragments for every k-step in registers for the whole kernel, so no query
// byte is loaded twice. The chunk goes by in blocks of RQ_ROWS rows (two
// 16-row MFMA tiles); with RS = 1 every wave takes both tiles of a block,
// with RS = 2 the waves of row half h take tile h (so a batch of up to 64
// requests still keeps all eight waves busy). Each block's k-steps are cut
// into SPB stages, which global-to-LDS loads bring in whole 128-byte lines
// into a ring of S slots, S - 1 stages ahead of the MFMAs, so
// that every bank byte crosses from L2 into the compute unit once and serves
// all the waves. A block leaves, per request and row tile, the largest
// <q, x> - |x|^2/2 of the tile's rows: a few maxima over registers and lane
// rows, which wait in LDS until a super tile (RQ_EPS row tiles) is complete
// and then go out, 64 bytes per request and all requests of a super tile side
// by side (request by request, as many DRAM pages took them and a batch of 64
// over 1,000,000 x 768 took 305 us for 286), with the super tile's maximum. No
// bound, list or candidate test holds a wave up between two blocks (one at a
// time, the candidates of the bounded scan took about a tenth of it).
template <int NKS, int QW, int RS, int SPB, int S, bool FOLDED>
__global__ __launch_bounds__(RQ_WAVES * WAVE, 1) void rq_scan_kernel(const ScanArgs A)
{
    constexpr int TT = RQ_ROWS / 16;
    constexpr int KSTG = NKS / SPB;             // k-steps of one stage
    constexpr int F = KSTG * TT;                // fragments of one stage
    constexpr int FPW = F / RQ_WAVES;           // of them, loaded by each wave
    constexpr int QPW = QW * 16;                // queries of one wave
    constexpr int NQS = RQ_WAVES / RS;          // query slots
    constexpr int TW = TT / RS;                 // tiles of a block each wave takes
    constexpr int BPS = RQ_EPS / TT;            // blocks of a super tile
    static_assert(NKS % SPB == 0 && F % RQ_WAVES == 0, "whole stages, equal shares");
    static_assert(KSTG % 2 == 0 && TT == 2, "stages of whole k-step pairs, 32-row blocks");
    // With four query groups a wave holds 192 registers of query fragments;
    // both tiles' accumulators would not fit beside them, so such a wave
    // takes the tiles of a block one after the other (one stage per block)
    constexpr bool TSEQ = QW >= 4 && TW == 2;
    constexpr int TA = TSEQ ? 1 : TW;           // tiles whose accumulators are live together
    static_assert(!TSEQ || SPB == 1, "tiles one after the other within one stage");
    static_assert(RS == 1 || RS == 2, "one or two row halves");
    constexpr int NM = TA * QW;                 // maxima of one block (TSEQ: of one tile)
    static_assert(NM == 1 || NM == 2 || NM == 4, "one register holds a block's results");
    static_assert(RQ_ROWS <= WAVE, "one norm per lane");

    extern __shared__ __align__(16) uint8_t smem[];
    const RqLayout L = rq_layout(QW, RS, KSTG, S);
    i32x4 *ring = (i32x4 *)(smem + L.ring);              // [S][F][64] fragments
    float *nslot = (float *)(smem + L.norms);            // [S][64] |x|^2 of a block's rows
    float *stg = (float *)(smem + L.stage);              // [RS][RQ_EPS][PITCH] maxima
    float *sst = (float *)(smem + L.sup);                // [NQS * QPW][rq_hold] super tiles' maxima

    const int c = blockIdx.x;
    if (c >= A.n_chunks)
        return;
    const int tid = threadIdx.x, lane = tid & 63;
    __builtin_assume(tid < RQ_WAVES * WAVE);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int slot_q = wave % NQS, half = wave / NQS;   // query slot, row half
    const int col = lane & 15, jg = lane >> 4;
    const uint32_t rowb = (uint32_t)A.d * 2;
    const long cbeg = (long)c * A.rows_per_chunk;        // of the launch's rows
    const long nleft = min(A.rows - cbeg, A.rows_per_chunk);
    const int nrows = nleft > 0 ? (int)nleft : 0;
    const long rbeg = A.row0 + cbeg;
    const int n_blk = (nrows + RQ_ROWS - 1) / RQ_ROWS;
    const int n_stg = n_blk * SPB;
    const int qw0 = slot_q * QPW;
    const bool active = qw0 < A.B;   // (a wave past the batch only loads its share)

    // ---- the wave's queries: fragments of every k-step (zero past the batch)
    const __amdgpu_buffer_rsrc_t rq = make_rsrc(A.queries, (uint32_t)A.B * rowb);
    i32x4 qf[QW][NKS];
#pragma unroll
    for (int g = 0; g < QW; ++g) {
        const int q = qw0 + g * 16 + col;
        const uint32_t base = q < A.B ? (uint32_t)q * rowb + jg * 16 : OFF_NONE;
#pragma unroll
        for (int s = 0; s < NKS; ++s)
            qf[g][s] = buffer_load16(rq, base + s * KSTEP_BYTES);
    }

    // ---- stage z (block z / SPB, its k-steps from (z % SPB) * KSTG) into
    // slot z % S: this wave's FPW fragments and, with a block's first stage,
    // the last wave loads the block's row norms. Every stage issues the same
    // fragment loads whether or not it fetches anything (past the last block
    // the resource is empty and the slot gets zeros).
    const __amdgpu_buffer_rsrc_t rbk =
        make_rsrc(A.bank + (size_t)rbeg * rowb, (uint32_t)nrows * rowb);
    const __amdgpu_buffer_rsrc_t rnm = make_rsrc(A.bank_norms + rbeg, (uint32_t)nrows * 4u);
    const __amdgpu_buffer_rsrc_t rnone = make_rsrc(A.bank, 0u);
    // this lane's place in a load: row ri of the row group, the chunk of the
    // 128-byte line that lands at its position (rq_chunk inverted)
    const int dri = lane >> 3;
    auto dma_chunk = [&](int rg) { return (lane & 7) ^ rq_perm(dri) ^ (2 * (rg & 1)); };
    auto issue = [&](int z) {
        const int slot = z % S, bz = z / SPB, st = z - bz * SPB;
        const bool real = z < n_stg;
        const __amdgpu_buffer_rsrc_t r = real ? rbk : rnone;
#pragma unroll
        for (int j = 0; j < FPW; ++j) {
            const int f = wave + RQ_WAVES * j;
            const int rg = f % 4, pair = st * (KSTG / 2) + f / 4;
            const uint32_t vo = (uint32_t)(bz * RQ_ROWS + rg * 8 + dri) * rowb +
                                pair * (2 * KSTEP_BYTES) + dma_chunk(rg) * 16;
            dma16(r, ring + (slot * F + f) * WAVE, vo);
        }
        if (st == 0 && wave == RQ_WAVES - 1)
            dma4(real ? rnm : rnone, nslot + slot * WAVE,
                 lane < RQ_ROWS ? (uint32_t)(bz * RQ_ROWS + lane) * 4u : OFF_NONE);
    };

    // ---- pipeline prologue: stages 0 .. S-2
#pragma unroll
    for (int z = 0; z < S - 1; ++z) {
        __builtin_amdgcn_sched_barrier(0);
        issue(z);
        __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();

    // the block tile of wave tile t
    auto tile_of = [&](int t) { return RS == 2 ? half : t; };
    // accumulators of wave tiles t0 .. t0+TA-1 from -|x|^2/2 of their rows
    // (past the chunk -inf, or no number in a tile with no row of it), the
    // norms of block b in norm slot `slot`
    auto init_acc = [&](f32x4(&ac)[TA][QW], int slot, int b, int t0) {
#pragma unroll
        for (int t = 0; t < TA; ++t) {
            const int tt = tile_of(t0 + t), r0 = b * RQ_ROWS + tt * 16;
            const f32x4 xn = *(const f32x4 *)(nslot + slot * WAVE + tt * 16 + jg * 4);
            f32x4 h;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                h[e] = -0.5f * xn[e];
            if (r0 + 16 > nrows) {   // (the chunk's last block only)
                const float past = r0 < nrows ? -INFINITY : __builtin_nanf("");
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    h[e] = r0 + jg * 4 + e < nrows ? h[e] : past;
            }
#pragma unroll
            for (int g = 0; g < QW; ++g)
                ac[t][g] = h;
        }
    };
    // the MFMAs of stage ST (in slot `slot`) for wave tiles t0 .. t0+TA-1
    auto mfma_tiles = [&](auto ST, f32x4(&ac)[TA][QW], int slot, int t0) {
        constexpr int st = decltype(ST)::value;
        // the lane's A fragment of tile tt, k-step j of the stage: row col of
        // the tile, quarter jg, at load (j/2)*4 + rg
        const i32x4 *fr = ring + slot * F * WAVE;
        uint32_t fbase[TA][2];
#pragma unroll
        for (int t = 0; t < TA; ++t) {
            const int tt = tile_of(t0 + t);
            const int ri = col & 7, rg = tt * 2 + (col >> 3);
#pragma unroll
            for (int h = 0; h < 2; ++h)
                fbase[t][h] = (uint32_t)rg * WAVE + rq_chunk(ri, rg, 4 * h + jg);
        }
        static_for<0, KSTG>([&](auto J) {
            constexpr int j = decltype(J)::value, s = st * KSTG + j;
            i32x4 a[TA];
#pragma unroll
            for (int t = 0; t < TA; ++t)
                a[t] = fr[(j / 2) * 4 * WAVE + fbase[t][j & 1]];
#pragma unroll
            for (int t = 0; t < TA; ++t)
#pragma unroll
                for (int g = 0; g < QW; ++g)
                    ac[t][g] = mfma_step<1>(a[t], qf[g][s], ac[t][g]);
        });
        // two k-steps of fragment reads in flight: the reads of k-steps 0 and
        // 1, then per k-step its MFMAs and the reads two ahead
        __builtin_amdgcn_sched_group_barrier(0x100, 2 * TA, 0);
        static_for<0, KSTG>([&](auto J) {
            __builtin_amdgcn_sched_group_barrier(0x008, TA * QW, 0);
            if constexpr (decltype(J)::value + 2 < KSTG)
                __builtin_amdgcn_sched_group_barrier(0x100, TA, 0);
        });
    };
    // ---- results. What emit and flush derive from the lane is computed each
    // time, from a lane index the compiler cannot hoist it from: held through
    // the MFMA loops beside 192 registers of requests, it takes the registers
    // that keep bank fragments in flight.
    auto fresh_lane = [&]() -> int {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    constexpr int PITCH = stage_pitch(NQS * QPW), STG_BUF = RQ_EPS * PITCH;   // of one buffer
    auto stg_of = [&](int sl) { return RS == 2 ? (sl & 1) * STG_BUF : 0; };
    auto emit = [&](f32x4(&ac)[TA][QW], int b, int t0) {
        float m[4];
        static_for<0, 4>([&](auto I) {
            constexpr int i = decltype(I)::value, j = NM == 4 ? i : NM == 2 ? i / 2 : 0;
            m[i] = max4(ac[j / QW][j % QW]);
        });
        const float r = rows_max4(m[0], m[1], m[2], m[3]);
        // lane row lr holds maximum (wave tile, group) = (i / QW, i % QW), i =
        // lr with its two bits swapped (NM = 4) or lr % NM
        const int l = fresh_lane(), lr = l >> 4;
        const int i = NM == 4 ? (lr >> 1) | ((lr & 1) << 1) : lr % NM;
        const int e = (b % BPS) * TT + tile_of(t0 + i / QW);
        if (lr < NM)
            stg[stg_of(b / BPS) + e * PITCH + slot_q * QPW + (i % QW) * 16 + (l & 15)] = r;
    };
    // entries of blocks past the chunk in its last super tile
    auto fill_past = [&]() {
        for (int b = n_blk; b % BPS != 0; ++b)
#pragma unroll
            for (int t = 0; t < TT; ++t)
                if (RS == 1 || t == half)
                    for (int q = lane; q < QPW; q += WAVE)
                        stg[stg_of(b / BPS) + ((b % BPS) * TT + t) * PITCH + slot_q * QPW + q] =
                            __builtin_nanf("");
    };
    // super tile sl of the chunk from LDS to the workspace: 16 requests per
    // instruction, four lanes of four entries each. The super tiles' maxima
    // wait in LDS for HOLD of them (most chunks have no more) and go out
    // request by request, because the selection reads all of a request's: a
    // 16-byte piece every fourth super tile cost 24 us of 434 at 256 requests,
    // the scattered stores holding up the loads behind them. RS = 1: each wave
    // its own requests; else the waves share them out (the first NQS * QW).
    constexpr int HOLD = rq_hold(QW, RS);
    constexpr int GPW = RS == 1 ? QW : (NQS * QW + RQ_WAVES - 1) / RQ_WAVES;   // groups per wave
    const bool flushes = RS == 1 ? active : wave * GPW < NQS * QW;
    const int fq0 = RS == 1 ? qw0 : wave * GPW * 16;
    const long sup0 = (long)c * A.sup_per_chunk;
    int settle = 0;   // stages until this wave's last flush no longer counts
    // maxima of super tiles s0 .. s1-1 (one HOLD) of this wave's requests;
    // past the last one taken, no numbers
    auto put_sup = [&](int s0, int s1) {
        for (int i = fresh_lane(); i < GPW * 16 * HOLD; i += WAVE) {
            const int q = fq0 + i / HOLD, j = i % HOLD;
            if (q < A.B && s0 + j < A.sup_per_chunk)
                A.m.sup[sup0 + s0 + j + q * A.m.sup_q] =
                    s0 + j < s1 ? sst[q * HOLD + j] : __builtin_nanf("");
        }
    };
    auto flush = [&](int sl) {
        static_assert(RQ_EPS == 16, "four lanes of four entries");
        const int l = fresh_lane(), part = l & 3, lq = l >> 2;
        const float *src = stg + stg_of(sl) + part * 4 * PITCH + fq0 + lq;
        float *const ent = A.m.ent + (sup0 + sl) * A.m.ent_s;
        // (out-of-range lanes fall outside the resource, so that every flush
        // is GPW stores at least)
#pragma unroll
        for (int i = 0; i < GPW; ++i) {
            const int q = fq0 + 16 * i + lq;
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = src[16 * i + e * PITCH];
            float m = max4(v);
            m = fmaxf(m, dpp<0xb1>(m));   // quad_perm [1,0,3,2]
            m = fmaxf(m, dpp<0x4e>(m));   // quad_perm [2,3,0,1]
            if (part == 0)
                sst[q * HOLD + sl % HOLD] = m;
            put_entries<FOLDED>(make_rsrc(ent + (long)(fq0 + 16 * i) * A.m.ent_q, 0x7fffffffu),
                                q < A.B, (uint32_t)(lq * A.m.ent_q), l, v);
        }
        settle = S - 1;
        if (sl % HOLD == HOLD - 1)
            put_sup(sl + 1 - HOLD, sl + 1);
    };
    // this wave's part of stage z has landed once at most FPW*(S-2) loads are
    // outstanding, the fragment loads of the S-2 stages issued after it, and
    // the stores of a flush where those came after it too (stores count like
    // loads, in order; waiting as if they did not would wait for later loads);
    // the barrier then tells that every wave's part has and that every wave is
    // done with stage z - 1, whose slot the next load reuses
    auto next_stage = [&](int z) {
        __builtin_amdgcn_sched_barrier(0);
        if (settle > 0) {
            wait_vmcnt<FPW * (S - 2) + GPW>();
            --settle;
        } else {
            wait_vmcnt<FPW * (S - 2)>();
        }
        stream_barrier();
        issue(z + S - 1);
        __builtin_amdgcn_sched_barrier(0);
    };

    int z = 0;   // the stage being consumed
    for (int b = 0; b < n_blk; ++b) {
        if constexpr (TSEQ) {
            // one stage per block; its tiles one after the other
            next_stage(z);
            const int slot = z % S;
            if (active) {
                static_for<0, TW>([&](auto T) {
                    f32x4 acc[TA][QW];
                    init_acc(acc, slot, b, T.value);
                    mfma_tiles(Int<0>{}, acc, slot, T.value);
                    emit(acc, b, T.value);
                });
            }
            ++z;
        } else {
            f32x4 acc[TA][QW];
            static_for<0, SPB>([&](auto ST) {
                next_stage(z);
                const int slot = z % S;
                if constexpr (decltype(ST)::value == 0) {
                    // two halves' entries of the super tile before are in LDS
                    if (RS == 2 && flushes && b > 0 && b % BPS == 0)
                        flush(b / BPS - 1);
                    init_acc(acc, slot, b, 0);
                }
                if (active)
                    mfma_tiles(ST, acc, slot, 0);
                ++z;
            });
            if (active)
                emit(acc, b, 0);
        }
        if (RS == 1 && flushes && b % BPS == BPS - 1)
            flush(b / BPS);
    }
    // the last super tile, and those of the chunk's share that it has no rows for
    fill_past();
    if (RS == 2) {
        stream_barrier();
        if (flushes && n_blk > 0)
            flush((n_blk - 1) / BPS);
    } else if (flushes && n_blk % BPS != 0) {
        flush(n_blk / BPS);
    }
    if (flushes) {
        // maxima that still wait, and no numbers in the rest of the share
        const int done = (n_blk + BPS - 1) / BPS;
        for (int s0 = done / HOLD * HOLD; s0 < A.sup_per_chunk; s0 += HOLD)
            put_sup(s0, done);
    }
    // (no global-to-LDS load may still be in flight when the workgroup ends)
    wait_vmcnt<0>();
}

template <int NKS, int QW, int RS, int SPB, int S>
hipError_t launch_rq_scan(const ScanArgs &a, size_t lds, int grid, hipStream_t s)
{
    auto kern = a.m.folded ? rq_scan_kernel<NKS, QW, RS, SPB, S, true>
                           : rq_scan_kernel<NKS, QW, RS, SPB, S, false>;
    hipError_t e = hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(RQ_WAVES * WAVE), lds, s, a);
    return hipGetLastError();
}

// The instantiations of one row length: the (QW, RS) the plan may choose for
// it (plan_knn's tables; QW * NKS * 4 registers of query fragments stay
// within 192).
template <int NKS>
hipError_t launch_rq_nks(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    constexpr int SPB = rq_spb(NKS), S = RQ_SLOTS;
#define RB_RQ(QW_, RS_)                                                                          \
    if (p.qw == QW_ && p.rs == RS_)                                                              \
        return launch_rq_scan<NKS, QW_, RS_, SPB, S>(a, p.lds_bytes, p.grid, s);
    if constexpr (NKS == 12) {
        RB_RQ(1, 2)
        RB_RQ(2, 2)
        RB_RQ(4, 2)
        RB_RQ(4, 1)
    } else if constexpr (NKS == 16 || NKS == 24) {
        RB_RQ(1, 2)
        RB_RQ(2, 2)
        RB_RQ(2, 1)
    } else if constexpr (NKS == 32) {
        RB_RQ(1, 2)
        RB_RQ(1, 1)
    }
#undef RB_RQ
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace rb
