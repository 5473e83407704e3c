// The bank scan of the exact k-nearest-neighbour search (RouteBalance Sec. 4.2:
// the KNN lookup of Alg. 1) for request tiles that stay in LDS: fp32 banks,
// bf16 batches of at most 64 requests over rows or banks the query-resident
// scan does not take, and large bf16 batches over small banks.
#pragma once

#include "knn_common.hpp"

namespace rb {

namespace {

// What bounds it: fp32 batches of some tens of requests the fp32 MFMA rate
// (64 flop per cycle and SIMD), small batches the bank stream, small banks
// the latency of one row tile's loads. So the request tile (NG groups of 16,
// every k-step) is loaded into LDS once per workgroup and then only read; a
// wave takes 16-row tiles of its own contiguous share of the bank, which come
// from HBM straight into MFMA operand registers, RES_RING k-steps ahead
// across tile ends, and no wave waits for another after the request tile has
// landed. A row tile leaves one value per request, the largest
// <q, x> - |x|^2/2 of its 16 rows; eps consecutive tiles (a super tile, all
// one wave's) one more; some scans keep every row's value too, which spares the
// selection from computing any again. There is no bound, no list and no
// candidate test: the selection takes the k best super tiles and recomputes
// the few row tiles that matter.
template <int DT, int NG>
__global__ __launch_bounds__(RES_WAVES * WAVE, 1) void res_scan_kernel(const ScanArgs A)
{
    constexpr int VEC = Elem<DT>::VEC, ESZ = Elem<DT>::ESZ;
    constexpr int KS = 4 * VEC;              // elements of one k-step
    constexpr int R = RES_RING;
    constexpr int NQ = (NG + 3) / 4;         // result registers: four groups each
    constexpr int NB = NG < 4 ? NG : 4;      // request fragments in flight
    extern __shared__ __align__(16) uint8_t smem[];
    i32x4 *qs = (i32x4 *)smem;               // [nks][NG][64] request fragments

    int t, c;
    chunk_and_tile(A.n_chunks, A.n_qt, &c, &t);
    if (c >= A.n_chunks)
        return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int n_waves = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, jg = lane >> 4;
    const int q0 = t * NG * 16;
    const int nks = A.nks;
    const uint32_t rowb = (uint32_t)A.d * ESZ;

    // this wave's super tiles [s0, s1), its row tiles [t0, t1)
    const long gw = (long)c * n_waves + wave, n_gw = (long)A.n_chunks * n_waves;
    const long s0 = gw * A.n_sup / n_gw, s1 = (gw + 1) * A.n_sup / n_gw;
    const long t0 = s0 * A.eps;
    const int n_tiles = (int)(min(s1 * A.eps, A.n_tiles) - t0);
    const int nrows = (int)(min(A.rows, (t0 + n_tiles) * 16) - t0 * 16);   // of the share

    // bank fragments: k-step ls of the share's tile lt into registers; rows
    // past the bank fall outside the resource and load zero, and so do the
    // lanes past the row in its last k-step
    const __amdgpu_buffer_rsrc_t rbk = make_rsrc(A.bank + (size_t)(A.row0 + t0 * 16) * rowb,
                                                 n_tiles > 0 ? (uint32_t)nrows * rowb : 0u);
    const __amdgpu_buffer_rsrc_t rnm =
        make_rsrc(A.bank_norms + A.row0 + t0 * 16, n_tiles > 0 ? (uint32_t)nrows * 4u : 0u);
    float *norms = (float *)(smem + (size_t)nks * NG * WAVE * 16) + wave * 2 * 256;
    const bool tail_ok = (nks - 1) * KS + jg * VEC < A.d;
    uint32_t lvo = (uint32_t)col * rowb + jg * 16;   // tile lt, k-step ls
    int ls = 0;
    auto issue = [&](i32x4 &a) {
        a = buffer_load16(rbk, ls == nks - 1 && !tail_ok ? OFF_NONE : lvo);
        lvo += KSTEP_BYTES;
        if (++ls == nks) {
            ls = 0;
            lvo += 16 * rowb - (uint32_t)nks * KSTEP_BYTES;
        }
    };
    // the request tile, straight into LDS (zero past the batch and past the
    // row), ahead of the bank's loads
    {
        const __amdgpu_buffer_rsrc_t rq = make_rsrc(A.queries, (uint32_t)A.B * rowb);
        for (int f = wave; f < nks * NG; f += n_waves) {
            const int sf = f / NG, q = q0 + (f - sf * NG) * 16 + col;
            dma16(rq, qs + f * WAVE,
                  q < A.B && (sf < nks - 1 || tail_ok)
                      ? (uint32_t)q * rowb + sf * KSTEP_BYTES + jg * 16
                      : OFF_NONE);
        }
    }
    // |x|^2 of the rows of 16 tiles at a time, into the wave's own LDS (two
    // slots): like the request tile not through registers, whose use would
    // make the wave wait for the bank loads in flight. The norms of tiles
    // 16b .. 16b + 15 are sent for at tile 16(b - 1), at least 16 k-steps and
    // so more than a ring of bank loads before their use.
    static_assert(R < 16, "norms land before the bank loads sent for after them are used");
    auto issue_norms = [&](int batch) {
        dma16(rnm, (i32x4 *)(norms + (batch & 1) * 256), (uint32_t)(batch * 256 + lane * 4) * 4u);
    };
    issue_norms(0);
    __builtin_amdgcn_sched_barrier(0);
    i32x4 ring[R];
#pragma unroll
    for (int u = 0; u < R; ++u)
        issue(ring[u]);
    // the request tile has landed once at most the loads after it are
    // outstanding, and after the barrier in every wave
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<R>();
    stream_barrier();
    __builtin_amdgcn_sched_barrier(0);

    // where this lane's results go: lane row r of result register v holds
    // group 4*v + (r with its two bits swapped), request col
    const int gsw = (jg >> 1) | ((jg & 1) << 1);
    float *sup[NQ], *ent[NQ];
    bool own[NQ];
#pragma unroll
    for (int v = 0; v < NQ; ++v) {
        const int g = 4 * v + gsw, q = q0 + g * 16 + col;
        own[v] = g < NG && q < A.B;
        sup[v] = A.m.sup + s0 + (own[v] ? q : 0) * A.m.sup_q;
        ent[v] = A.m.ent + s0 * A.m.ent_s + (own[v] ? q : 0) * A.m.ent_q;
    }
    // They wait in registers, entries until their super tile is complete,
    // super tiles until there are RES_HOLD, and go out as whole lines (one
    // value at a time, a line left the cache with a piece of it between two
    // stores: 64 requests over 4,000,000 x 128 bf16 took 386 us for 250, 16
    // over 2,000,000 x 384 fp32 678 for 578).
    static_assert(RES_HOLD == 16 && SEL_MAX_EPS <= 16, "what a lane holds");
    f32x16 ehold[NQ], shold[NQ];
    const float nan = __builtin_nanf("");
    auto clear = [&](f32x16(&h)[NQ]) {
#pragma unroll
        for (int v = 0; v < NQ; ++v)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                h[v][e] = nan;
    };
    // the super tile's entries (those past the bank hold no number)
    auto put_ent = [&]() {
#pragma unroll
        for (int v = 0; v < NQ; ++v) {
            if (own[v]) {
                if (A.eps == 2)
                    *(f32x2 *)ent[v] = f32x2{ehold[v][0], ehold[v][1]};
#pragma unroll
                for (int e = 0; e < 16; e += 4)
                    if (e + 4 <= A.eps)
                        *(f32x4 *)(ent[v] + e) = f32x4{ehold[v][e], ehold[v][e + 1],
                                                       ehold[v][e + 2], ehold[v][e + 3]};
            }
            ent[v] += A.m.ent_s;
        }
        clear(ehold);
    };
    auto put_sup = [&](int n) {   // the first n held
#pragma unroll
        for (int v = 0; v < NQ; ++v) {
            if (own[v]) {
#pragma unroll
                for (int e = 0; e < RES_HOLD; e += 4) {
                    if (e + 4 <= n)
                        *(f32x4_any *)(sup[v] + e) = f32x4{shold[v][e], shold[v][e + 1],
                                                           shold[v][e + 2], shold[v][e + 3]};
                    else
#pragma unroll
                        for (int i = e; i < e + 4; ++i)
                            if (i < n)
                                sup[v][i] = shold[v][i];
                }
            }
            sup[v] += n;
        }
    };
    clear(ehold);
    clear(shold);

    f32x4 acc[NG];
    float smax[NQ];
#pragma unroll
    for (int v = 0; v < NQ; ++v)
        smax[v] = nan;
    // tile of the share, its k-step, its place in the super tile, that one's among those held
    int tile = 0, s = 0, es = 0, ss = 0;
    auto start_tile = [&]() {
        // the accumulators start from -|x|^2/2 of their rows (-inf past the bank)
        const f32x4 xn = *(const f32x4 *)(norms + (tile & 31) * 16 + jg * 4);
        f32x4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            h[e] = tile * 16 + jg * 4 + e < nrows ? -0.5f * xn[e] : -INFINITY;
#pragma unroll
        for (int g = 0; g < NG; ++g)
            acc[g] = h;
        if ((tile & 15) == 0)
            issue_norms(tile / 16 + 1);
    };
    auto end_tile = [&]() {
        float m[4 * NQ];
#pragma unroll
        for (int g = 0; g < 4 * NQ; ++g)
            m[g] = g < NG ? max4(acc[g < NG ? g : 0]) : -INFINITY;
        if (A.acc) {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int q = q0 + g * 16 + col;
                if (q < A.B)
                    *(f32x4 *)(A.acc + ((size_t)(t0 + tile) * A.B + q) * 16 + jg * 4) = acc[g];
            }
        }
        const bool last = es == A.eps - 1 || tile == n_tiles - 1;
#pragma unroll
        for (int v = 0; v < NQ; ++v) {
            const float r = rows_max4(m[4 * v], m[4 * v + 1], m[4 * v + 2], m[4 * v + 3]);
            ehold[v][es] = r;
            smax[v] = fmaxf(smax[v], r);
            shold[v][ss] = smax[v];
            if (last)
                smax[v] = nan;
        }
        if (last) {
            if (A.eps > 1 && !A.acc)
                put_ent();
            if (++ss == RES_HOLD) {
                put_sup(RES_HOLD);
                ss = 0;
            }
        }
        es = last ? 0 : es + 1;
        ++tile;
    };
    if (n_tiles > 0)
        start_tile();
    // One position per (tile, k-step), in order; position x sits in ring slot
    // x % R and, once used, makes room for position x + R. Every position
    // sends its load whether or not there is anything left to fetch, so that
    // a slot's load always has R - 1 others behind it when it is waited for.
    const long n_pos = (long)n_tiles * nks;
    for (long x = 0; x < n_pos; x += R) {
        static_for<0, R>([&](auto U) {
            constexpr int u = decltype(U)::value;
            const i32x4 *fr = qs + s * NG * WAVE + lane;
            i32x4 bq[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j)
                bq[j] = fr[j * WAVE];
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                acc[g] = mfma_step<DT>(ring[u], bq[g % NB], acc[g]);
                if (g + NB < NG)
                    bq[g % NB] = fr[(g + NB) * WAVE];
            }
            issue(ring[u]);
            if (++s == nks) {
                s = 0;
                if (tile < n_tiles) {   // (past the share: nothing to write)
                    end_tile();
                    start_tile();
                }
            }
        });
    }
    put_sup(ss);
    // (no global-to-LDS load may still be in flight when the workgroup ends)
    wait_vmcnt<0>();
}

template <int DT, int NG>
hipError_t launch_res_scan(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    auto kern = res_scan_kernel<DT, NG>;
    hipError_t e = hipFuncSetAttribute((const void *)kern,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)p.lds_bytes);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(kern, dim3(p.grid), dim3(p.wg_waves * WAVE), p.lds_bytes, s, a);
    return hipGetLastError();
}

template <int DT>
hipError_t launch_res(const KnnPlan &p, const ScanArgs &a, hipStream_t s)
{
    switch (p.ng) {
    case 1: return launch_res_scan<DT, 1>(p, a, s);
    case 2: return launch_res_scan<DT, 2>(p, a, s);
    case 3: return launch_res_scan<DT, 3>(p, a, s);
    case 4: return launch_res_scan<DT, 4>(p, a, s);
    case 5: return launch_res_scan<DT, 5>(p, a, s);
    case 6: return launch_res_scan<DT, 6>(p, a, s);
    case 7: return launch_res_scan<DT, 7>(p, a, s);
    case 8: return launch_res_scan<DT, 8>(p, a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

}  // namespace rb
