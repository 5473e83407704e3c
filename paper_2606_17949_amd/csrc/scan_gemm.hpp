// The bank scan of the exact k-nearest-neighbour search (RouteBalance Sec. 4.2:
// the KNN lookup of Alg. 1) for large batches, where the distance pass is a
// dense contraction bound by the matrix cores: bf16 rows of any length, batches
// that the query-resident scan cannot hold (and small batches of rows too long
// for the LDS-resident one).
#pragma once

#include "knn_common.hpp"

namespace rb {

namespace {

// One v_mfma_f32_32x32x16_bf16: D = A*B + C over 16 elements of K, A 32 bank
// rows, B 32 requests. Lane l holds, of both operands, row (or request) l % 32
// at K positions 8*(l/32) .. 8*(l/32)+7; of D, request l % 32 of rows
// 8*(r/4) + 4*(l/32) + r%4 in register r.
__device__ __forceinline__ f32x16 mfma32(const i32x4 &a, const i32x4 &b, const f32x16 &c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// One workgroup of GM_WAVES waves (two per SIMD) per (bank chunk, tile of
// 64 * TPQ requests). The chunk goes by in macro tiles of GM_ROWS rows; wave w
// holds the inner products of rows 64*(w%4) .. +63 with requests
// 32*TPQ*(w/4) .. +32*TPQ-1 of the tile, 2 x TPQ tiles of 32 x 32 in up to 128
// accumulator registers, while K goes by in stages of GM_KST elements: each
// stage brings the macro tile's rows and the request tile, one 128-byte piece
// of each row, from L2 (the other request tiles of the chunk run on the same
// XCD, so a bank row comes from HBM once) into one of two LDS slots. A load
// brings 8 rows x 128 bytes; row ri of load group g keeps its 16-byte chunk c
// at position 8*ri + (c ^ ri ^ (g & 1)), which spreads the rows of a fragment
// read over distinct LDS bank groups. A stage is four k-steps of 16; every
// wave reads the fragments of the next k-step while the MFMAs of the
// current one run (for 256 requests 12 fragment reads, 32 MFMAs of 32x32x16
// per stage and wave). The one barrier of a stage sits before its last k-step,
// whose fragments are already in registers: past it, the slot just read takes
// the loads of the stage after next and the fragments of the next stage's
// first k-step are read, so that the matrix cores keep working across the
// barrier. After a macro tile's last stage each wave takes, per request, the
// maxima of its accumulators (a lane's 16 rows of a 32 x 32 tile are one
// entry, a macro tile's 16 entries one super tile) into LDS; they go out after
// the next barrier, 64 bytes per request. With OUT = GM_VALUES the accumulators
// themselves go out in place of the entries.
template <int TPQ, int OUT>
__global__ __launch_bounds__(GM_WAVES * WAVE, 1) void gemm_scan_kernel(const ScanArgs A)
{
    constexpr int QRY = 64 * TPQ;                 // requests of a tile
    constexpr int NROW = GM_ROWS / 8;             // loads of a stage's rows,
    constexpr int NLOAD = NROW + QRY / 8;         //   and of its requests
    constexpr int LPW = NLOAD / GM_WAVES;         // of them, issued by each wave
    constexpr int LPR = NROW / GM_WAVES;          // the first LPR take rows
    constexpr int TPR = 2;                        // 32-row tiles per wave
    static_assert(GM_ROWS == 256 && GM_KST == 64 && GM_WAVES == 8 && GM_SLOTS == 2,
                  "the wave, load and stage layout below");
    static_assert(GM_ROWS / 16 == GM_EPS, "a macro tile is a super tile");

    extern __shared__ __align__(16) uint8_t smem[];
    const GemmLayout L = gemm_layout(TPQ);
    float *nslot = (float *)(smem + L.norms);        // [2][GM_ROWS] |x|^2 of macro tiles rt & 1
    constexpr int PITCH = stage_pitch(QRY);
    float *stg = (float *)(smem + L.stage);          // [GM_EPS][PITCH] a macro tile's maxima

    int t, c;
    chunk_and_tile(A.n_chunks, A.n_qt, &c, &t);
    if (c >= A.n_chunks)
        return;
    const int tid = threadIdx.x, lane = tid & 63;
    __builtin_assume(tid < GM_WAVES * WAVE);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave & 3, wq = wave >> 2;   // row quarter, request half of the macro tile
    const int hl = lane >> 5;                  // K half of a fragment
    const uint32_t rowb = (uint32_t)A.d * 2;
    const long cbeg = (long)c * A.rows_per_chunk;   // of the launch's rows
    const long nleft = min(A.rows - cbeg, A.rows_per_chunk);
    const int nrows = nleft > 0 ? (int)nleft : 0;
    const long rbeg = A.row0 + cbeg;
    const int n_rt = (nrows + GM_ROWS - 1) / GM_ROWS;
    const int nks = A.nks;                     // stages of one macro tile (at least 2)
    const int n_stg = n_rt * nks;
    const int q0 = t * QRY;
    const int nq = min(QRY, A.B - q0);         // requests of this tile

    // ---- stage z (macro tile z / nks, K part z % nks) into slot z & 1: this
    // wave's LPW loads (rows first, then requests) and, with a macro tile's
    // first stage, the last wave loads its 256 row norms. Every stage issues
    // the same loads whether or not they fetch anything (past the last stage
    // the resource is empty and the slot gets zeros); rows past the chunk and
    // requests past the batch fall outside their resources and load zero.
    const __amdgpu_buffer_rsrc_t rbk =
        make_rsrc(A.bank + (size_t)rbeg * rowb, (uint32_t)nrows * rowb);
    const __amdgpu_buffer_rsrc_t rqr =
        make_rsrc(A.queries + (size_t)q0 * rowb, (uint32_t)max(nq, 0) * rowb);
    const __amdgpu_buffer_rsrc_t rnm = make_rsrc(A.bank_norms + rbeg, (uint32_t)nrows * 4u);
    const __amdgpu_buffer_rsrc_t rnone = make_rsrc(A.bank, 0u);
    // Lane l of every load brings row l/8 of its group, chunk
    // (l % 8) ^ (l/8) ^ (g % 2); a wave's groups g = wave + 8*j all have the
    // parity of the wave, so one byte offset serves all of its loads (and none
    // those of its last stage that lie past the row: they load zero).
    const int chunk = (lane & 7) ^ (lane >> 3) ^ (wave & 1);
    const uint32_t lo = (uint32_t)(lane >> 3) * rowb + (uint32_t)chunk * 16;
    const int kc_end = (A.d / 8 - chunk + 7) / 8;   // stages in which the chunk exists
    // load j of stage z
    auto issue_load = [&](int z, int j) {
        const int slot = z & 1, rt = z / nks, kc = z - rt * nks;
        const bool real = z < n_stg;
        const bool rows = j < LPR;
        const int f = wave + GM_WAVES * j;                // load index in the stage
        const int r0 = rows ? rt * GM_ROWS + 8 * f : 8 * (f - NROW);
        dma16(real ? (rows ? rbk : rqr) : rnone,
              (i32x4 *)(smem + L.ring) + (slot * GM_SLOT_LOADS + f) * WAVE,
              kc < kc_end ? lo + (uint32_t)r0 * rowb + (uint32_t)kc * (GM_KST * 2) : OFF_NONE);
    };
    // with a macro tile's first stage, the last wave loads the tile's norms
    // into slot rt & 1 (they are read when that stage's MFMAs begin, before
    // the loads of tile rt + 2 reuse the slot)
    auto issue_norms = [&](int z) {
        const int rt = z / nks;
        if (z - rt * nks == 0 && wave == GM_WAVES - 1)
            dma16(z < n_stg ? rnm : rnone, (i32x4 *)(nslot + (rt & 1) * GM_ROWS),
                  (uint32_t)(rt * GM_ROWS * 4 + lane * 16));
    };
    auto issue = [&](int z) {
#pragma unroll
        for (int j = 0; j < LPW; ++j)
            issue_load(z, j);
        issue_norms(z);
    };

    // Fragment places: tile i of the wave's rows (row ra = 64*wr + 32*i +
    // lane%32: load group ra/8, row ra%8 in it) has chunk cq = 2*s + hl of
    // its k-step s at position (ra/8)*64 + 8*(ra%8) + (cq ^ (ra%8) ^ (ra/8 % 2))
    // of the slot; the same for the requests (tile u: 128*wq + 32*u +
    // lane%32) in the second half of the slot. As a byte address:
    // p ^ (32*s) ^ (slot << 16), p the address of k-step 0 in slot 0 (the
    // ring starts the LDS allocation and a slot is 64 KiB).
    static_assert(GM_SLOT_LOADS * WAVE * 16 == 1 << 16 && NLOAD <= GM_SLOT_LOADS,
                  "slot offset as one address bit");
    uint32_t pa[TPR], pb[TPQ];
#pragma unroll
    for (int i = 0; i < TPR; ++i) {
        const int ra = 64 * wr + 32 * i + (lane & 31);
        pa[i] = (uint32_t)((ra >> 3) * WAVE + 8 * (ra & 7) + (hl ^ (ra & 7) ^ ((ra >> 3) & 1))) * 16;
    }
#pragma unroll
    for (int u = 0; u < TPQ; ++u) {
        const int rq = 32 * TPQ * wq + 32 * u + (lane & 31);
        pb[u] = (uint32_t)((NROW + (rq >> 3)) * WAVE + 8 * (rq & 7) +
                           (hl ^ (rq & 7) ^ ((rq >> 3) & 1))) * 16;
    }
    // fragments of k-step s from the slot whose address bit is sx
    auto frag_a = [&](uint32_t sx, auto S, int i) -> i32x4 {
        return *(const i32x4 *)(smem + L.ring + (pa[i] ^ (sx ^ (32u * decltype(S)::value))));
    };
    auto frag_b = [&](uint32_t sx, auto S, int u) -> i32x4 {
        return *(const i32x4 *)(smem + L.ring + (pb[u] ^ (sx ^ (32u * decltype(S)::value))));
    };
    f32x16 acc[TPR][TPQ];
    // the MFMAs of one k-step on (fa, fb), request tile by request tile;
    // with NEXT, the fragments of k-step S of the slot at sx come in
    // meanwhile: the row fragments first, each request fragment as soon as
    // the MFMAs that read its register have been issued; loads J0 .. J1-1 of
    // stage zl go out spread over the request tiles, so that the address unit
    // takes them while the matrix cores work
    auto mma_step = [&](i32x4(&fa)[TPR], i32x4(&fb)[TPQ], uint32_t sx, auto S, auto NEXT,
                        auto J0, auto J1, int zl) {
        constexpr bool next = decltype(NEXT)::value;
        constexpr int j0 = decltype(J0)::value, j1 = decltype(J1)::value;
        constexpr int per = (j1 - j0 + TPQ - 1) / TPQ;   // loads per request tile
        // (no instruction moves across a k-step's bounds, which keeps the
        // fragments of at most two k-steps live)
        __builtin_amdgcn_sched_barrier(0);
        i32x4 na[TPR];
        if constexpr (next) {
#pragma unroll
            for (int i = 0; i < TPR; ++i)
                na[i] = frag_a(sx, S, i);
        }
#pragma unroll
        for (int u = 0; u < TPQ; ++u) {
#pragma unroll
            for (int i = 0; i < TPR; ++i)
                acc[i][u] = mfma32(fa[i], fb[u], acc[i][u]);
            if constexpr (next)
                fb[u] = frag_b(sx, S, u);
#pragma unroll
            for (int i = 0; i < per; ++i)
                if (j0 + u * per + i < j1)
                    issue_load(zl, j0 + u * per + i);
        }
        if constexpr (next) {
#pragma unroll
            for (int i = 0; i < TPR; ++i)
                fa[i] = na[i];
        }
        // the order above, kept by the scheduler
        if constexpr (next)
            __builtin_amdgcn_sched_group_barrier(0x100, TPR, 0);
        static_for<0, TPQ>([&](auto) {
            __builtin_amdgcn_sched_group_barrier(0x008, TPR, 0);
            if constexpr (next)
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            if constexpr (per > 0)
                __builtin_amdgcn_sched_group_barrier(0x010, per, 0);
        });
        __builtin_amdgcn_sched_barrier(0);
    };
    constexpr int LH = LPW / 2;   // a stage's loads go out in two halves

    // a macro tile's maxima from LDS to the workspace, 16 requests per
    // instruction, four lanes of four entries each; the super tiles' maxima
    // wait in LDS for GM_HOLD of them and go out request by request, because
    // the selection reads all of a request's. Always GPW stores at least
    // (lanes with nothing to store fall outside the resource).
    constexpr int GPW = QRY / 16 / GM_WAVES;
    const long sup0 = (long)c * A.sup_per_chunk;
    const int fq0 = wave * GPW * 16;
    float *sst = (float *)(smem + L.sup);   // [QRY][GM_HOLD]
    // maxima of super tiles s0 .. s1-1 of this wave's requests; past the last
    // one taken, no numbers
    auto put_sup = [&](int s0, int s1) {
        for (int i = lane; i < GPW * 16 * GM_HOLD; i += WAVE) {
            const int q = fq0 + i / GM_HOLD, j = i % GM_HOLD;
            if (q < nq && s0 + j < A.sup_per_chunk)
                A.m.sup[sup0 + s0 + j + (q0 + q) * A.m.sup_q] =
                    s0 + j < s1 ? sst[q * GM_HOLD + j] : __builtin_nanf("");
        }
    };
    auto flush = [&](int rt) {
        const int part = lane & 3;
        const float *src = stg + part * 4 * PITCH + fq0 + (lane >> 2);
        float *const ent = A.m.ent + (sup0 + rt) * A.m.ent_s + (q0 + fq0) * A.m.ent_q;
#pragma unroll
        for (int i = 0; i < GPW; ++i) {
            const int q = fq0 + 16 * i + (lane >> 2);
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = src[16 * i + e * PITCH];
            float m = max4(v);
            m = fmaxf(m, dpp<0xb1>(m));   // quad_perm [1,0,3,2]
            m = fmaxf(m, dpp<0x4e>(m));   // quad_perm [2,3,0,1]
            if (part == 0)
                sst[q * GM_HOLD + rt % GM_HOLD] = m;
            if constexpr (OUT != GM_VALUES)
                put_entries<OUT == GM_FOLDED>(make_rsrc(ent + 16L * i * A.m.ent_q, 0x7fffffffu),
                                              q < nq, (uint32_t)((lane >> 2) * A.m.ent_q), lane,
                                              v);
        }
        if (rt % GM_HOLD == GM_HOLD - 1)
            put_sup(rt + 1 - GM_HOLD, rt + 1);
    };
    __builtin_amdgcn_sched_barrier(0);
    issue(0);
#pragma unroll
    for (int j = 0; j < LH; ++j)
        issue_load(1, j);
    // stage 0 has landed once at most the first half of the loads of stage 1
    // is outstanding; after the barrier, every wave's part has
    wait_vmcnt<LH>();
    stream_barrier();
    __builtin_amdgcn_sched_barrier(0);
    i32x4 fa[TPR], fb[TPQ];
#pragma unroll
    for (int i = 0; i < TPR; ++i)
        fa[i] = frag_a(0u, Int<0>{}, i);
#pragma unroll
    for (int u = 0; u < TPQ; ++u)
        fb[u] = frag_b(0u, Int<0>{}, u);
    for (int z = 0, rt = 0, kc = 0; z < n_stg; ++z) {
        const uint32_t rs = (uint32_t)(z & 1) << 16, rn = rs ^ (1u << 16);
        if (kc == 0) {
            // a macro tile's accumulators start from -|x|^2/2 of their rows
            // (-inf for rows past the chunk), so that they end as
            // <q, x> - |x|^2/2; the tile's norms landed two barriers ago
            const float *nm = nslot + (rt & 1) * GM_ROWS;
#pragma unroll
            for (int i = 0; i < TPR; ++i) {
                // (no number in an entry with no row of the chunk)
                const float past = rt * GM_ROWS + 64 * wr + 32 * i + 4 * hl < nrows
                                       ? -INFINITY
                                       : __builtin_nanf("");
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int r0 = 64 * wr + 32 * i + 8 * g + 4 * hl;
                    const f32x4 xn = *(const f32x4 *)(nm + r0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float h = rt * GM_ROWS + r0 + e < nrows ? -0.5f * xn[e] : past;
#pragma unroll
                        for (int u = 0; u < TPQ; ++u)
                            acc[i][u][4 * g + e] = h;
                    }
                }
            }
        }
        // k-steps 0-2 of the stage, each with the next one's fragment reads;
        // k-step 0 also sends the second half of the loads of stage z + 1
        mma_step(fa, fb, rs, Int<1>{}, Bool<true>{}, Int<LH>{}, Int<LPW>{}, z + 1);
        // the macro tile before is in LDS whole (its last stage's maxima went
        // there before the last barrier but one; its entries' place is taken
        // again at least one barrier later): it goes out behind the loads
        const bool flushed = kc == 1 && rt > 0;
        if (flushed)
            flush(rt - 1);
        mma_step(fa, fb, rs, Int<2>{}, Bool<true>{}, Int<0>{}, Int<0>{}, 0);
        mma_step(fa, fb, rs, Int<3>{}, Bool<true>{}, Int<0>{}, Int<0>{}, 0);
        // this wave's loads of stage z + 1 (sent with the previous stage's
        // last k-step and this stage's first) have landed and its reads of
        // slot z & 1 are done; after the barrier the same holds for every
        // wave, so the slot takes stage z + 2
        __builtin_amdgcn_sched_barrier(0);
        if (flushed && OUT != GM_VALUES)
            wait_vmcnt<GPW>();
        else
            wait_vmcnt<0>();
        stream_barrier();
        // k-step 3, with the reads of the next stage's first k-step and the
        // first half of the loads of stage z + 2 (after a macro tile's last
        // stage the fragments are read again once its values are out, which
        // keeps them from being held through that work)
        issue_norms(z + 2);
        mma_step(fa, fb, rn, Int<0>{}, Bool<true>{}, Int<0>{}, Int<LH>{}, z + 2);
        if (kc != nks - 1) {
            ++kc;
            continue;
        }
        kc = 0;
        // ---- end of macro tile rt: the lane's maximum over its 16 rows of
        // each 32 x 32 tile is entry 2 * (32-row tile) + K half of request
        // 32*TPQ*wq + 32*u + lane%32
        static_for<0, TPR>([&](auto I) {
            constexpr int i = decltype(I)::value;
            static_for<0, TPQ>([&](auto U) {
                constexpr int u = decltype(U)::value;
                __builtin_amdgcn_sched_barrier(0);
                const f32x16 &v = acc[i][u];
                float m = v[0];
#pragma unroll
                for (int r = 1; r < 16; ++r)
                    m = fmaxf(m, v[r]);
                stg[(2 * (2 * wr + i) + hl) * PITCH + 32 * TPQ * wq + 32 * u + (lane & 31)] = m;
                if constexpr (OUT == GM_VALUES) {
                    // every row's value: four rows of a request at a time, the
                    // row tiles' requests side by side (a row tile past the
                    // chunk is the next chunk's)
                    const int q = 32 * TPQ * wq + 32 * u + (lane & 31);
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int r0 = rt * GM_ROWS + 64 * wr + 32 * i + 8 * g;   // (of the chunk)
                        float *const at =
                            A.acc + (((cbeg + r0) >> 4) * A.B + q0) * 16 + (g & 1) * 8;
                        store16_nt(make_rsrc(at, 0x7fffffffu),
                                   q < nq && r0 < nrows ? (uint32_t)(q * 16 + hl * 4) * 4u
                                                        : OFF_NONE,
                                   f32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]});
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
#pragma unroll
        for (int i = 0; i < TPR; ++i)
            fa[i] = frag_a(rn, Int<0>{}, i);
#pragma unroll
        for (int u = 0; u < TPQ; ++u)
            fb[u] = frag_b(rn, Int<0>{}, u);
        ++rt;
    }

    // the last macro tile, and the super tiles of the chunk's share that it
    // has no rows for
    stream_barrier();
    if (n_rt > 0)
        flush(n_rt - 1);
    // (maxima that still wait, and no numbers in the rest of the share)
    for (int s0 = n_rt / GM_HOLD * GM_HOLD; s0 < A.sup_per_chunk; s0 += GM_HOLD)
        put_sup(s0, n_rt);
    // (no global-to-LDS load may still be in flight when the workgroup ends)
    wait_vmcnt<0>();
}

}  // namespace

}  // namespace rb
