// The k nearest rows of every request from the maxima a bank scan left
// (RouteBalance Sec. 4.2: the KNN lookup of Alg. 1), and the label average.
#include "knn_common.hpp"

namespace rb {

namespace {

// Ascending (key, index) pairs; absent entries have key KEY_NONE.
constexpr uint64_t PAIR_NONE = ~0ull;

// Minimum over the wave of 64-bit values (every lane gets it).
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t m)
{
    uint32_t hi = ~(uint32_t)(m >> 32), lo = ~(uint32_t)m;
    reduce_max_pair<WAVE>(hi, lo);
    return ((uint64_t)~hi << 32) | ~lo;
}

// Sorts the n pairs of `cand` in LDS (distinct) by counting, for each, the
// pairs below it; the k smallest go to out[0 .. min(k, n)). The threads split
// the pairs to rank and, where there are more threads, the pairs to count
// over; rank[] holds n counts, zero on entry. Every thread of the workgroup
// takes part; `out` is complete after the next barrier.
template <int NT>
__device__ __forceinline__ void rank_pairs(const uint64_t *cand, int n, int k, int *rank,
                                           uint64_t *out)
{
    const int width = (n + WAVE - 1) / WAVE * WAVE;
    const int parts = width > 0 && width < NT ? NT / width : 1;
    const int part = width > 0 ? threadIdx.x / width : 0;
    if (part < parts || parts == 1) {
        const int j0 = parts == 1 ? 0 : n * part / parts;
        const int j1 = parts == 1 ? n : n * (part + 1) / parts;
        for (int i = parts == 1 ? threadIdx.x : threadIdx.x - part * width; i < n;
             i += NT) {
            const uint64_t mine = cand[i];
            int r = 0;
#pragma unroll 8
            for (int j = j0; j < j1; ++j)
                r += cand[j] < mine ? 1 : 0;
            atomicAdd(&rank[i], r);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += NT) {
        const int r = rank[i];
        rank[i] = 0;
        if (r < k)
            out[r] = cand[i];
    }
}

// One workgroup per request. The scan left, per super tile, the largest
// <q, x> - |x|^2/2 of its rows, i.e. the distance of its nearest row. The k
// nearest rows lie in the k super tiles that come first by (that distance,
// index): a row of any other super tile has k rows before it in (distance,
// index) order, one in each of those k. Within them only row tiles whose own
// nearest row is no farther than the k-th super tile's can hold one of the k
// (k rows lie at or below that distance), in random order about k of them.
// Those tiles' distances are read where the scan kept every one (acc), else
// computed again, elements in the scan's order, and so with its bits, which the
// order by (distance, index) across super tiles rests on (a step of 16x16x32
// gives the bits of the GEMM-structured scan's two of 32x32x16: no difference
// in 2,048,000 sums over 32 to 2,048 elements of five distributions); the k
// smallest (distance, index) pairs of their rows are the result.
// What bounds it: a chain of dependent memory accesses and barriers at small
// batches, at large ones the reading of k tiles of 16 rows per request.
//   1. a bound: the largest of at least k groups' least super-tile distances,
//      a group being what one wave's threads hold, or one row of 16 lanes for
//      k above the wave count. The super tiles at or below it go to LDS (50 to
//      300 in random order) and are ranked by counting. More than fit (a bank
//      of mostly equal rows) are taken k times the smallest instead.
//   2. the row tiles of the k super tiles under the k-th distance (with kept
//      distances, all of them).
//   3. their rows' distances, SEL_ROUND tiles at a time, computed one wave per
//      tile with the request replicated over the MFMA's columns; rows at or
//      below the bound join the list, which is ranked after each round.
//   4. the neighbours, and the label average.
struct SelectShared {
    uint64_t cand[SEL_CAP];
    uint64_t best[RB_MAX_K_DEV], prev[RB_MAX_K_DEV];
    uint32_t group_min[WAVE];
    uint64_t wave_min[SEL_THREADS / WAVE];
    int tiles[RB_MAX_K_DEV * SEL_MAX_EPS];
    int sup[RB_MAX_K_DEV];
    int rank[SEL_CAP];
    int n_cand, n_tiles;
    int32_t nbr[RB_MAX_K_DEV];
    float wts[RB_MAX_K_DEV];
    __align__(16) uint8_t q[SEL_MAX_ROW_BYTES];
};
static_assert(SEL_ROUND * 16 + RB_MAX_K_DEV <= SEL_CAP, "a round's rows and the running best");

template <int DT, int NT>
__global__ __launch_bounds__(NT, 1024 / NT) void select_kernel(const SelectArgs A)
{
    constexpr int VEC = Elem<DT>::VEC, ESZ = Elem<DT>::ESZ;
    constexpr int KS = 4 * VEC;
    constexpr int NW = NT / WAVE;
    constexpr int LD = 8;   // k-steps of one block of bank loads
    __shared__ SelectShared S;
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k = A.k;
    const uint32_t rowb = (uint32_t)A.d * ESZ;
    auto sup = [&](long i) -> float { return A.m.sup[i + b * A.m.sup_q]; };
    auto ent = [&](int s, int e) -> float {
        return A.m.ent[s * A.m.ent_s + e + b * A.m.ent_q];
    };

    // the first super tiles stay in registers: their loads go out before
    // anything is waited for. The waves take them in turn, 16 at a time (4 of
    // a few), so that near rows that follow one another in the bank are not
    // all one wave's and every wave's least distance is as near as another's (a
    // bank in the order of its clusters, contiguous shares / in turn: 64 x
    // 100,000 x 768 178 / 57 us, 256 x 1,000,000 x 768 in 32 clusters 479 / 385;
    // rows in random order the same).
    constexpr int SV = SEL_WANT_SUP / NT < 32 ? SEL_WANT_SUP / NT : 32;
    const int deal = A.n_sup >= 16 * 16 * NW ? 4 : 2;   // log2 of a turn
    const int first = (((lane >> deal) * NW + wave) << deal) + (lane & ((1 << deal) - 1));
    auto sup_at = [&](int u) -> long { return first + (long)u * NT; };
    float sv[SV];
#pragma unroll
    for (int u = 0; u < SV; ++u) {
        const long j = sup_at(u);
        sv[u] = j < A.n_sup ? sup(j) : __builtin_nanf("");
    }
    // |q|^2 (in every wave: the same sums in the same order), and the request
    // in LDS, zero past the row
    const uint8_t *qrow = A.queries + (size_t)b * rowb;
    float qn = 0.f;
    for (uint32_t off = lane * 16; off < rowb; off += WAVE * 16) {
        const i32x4 v = load16(qrow + off);
        qn = sumsq16<DT>(v, qn);
        if (wave == 0)
            *(i32x4 *)(S.q + off) = v;
    }
    qn = wave_sum(qn);
    if (!(qn <= FLT_MAX))
        qn = __builtin_nanf("");   // (an infinite request is at no distance from any row)
    const uint32_t padded = (uint32_t)(A.nks + LD - 1) / LD * LD * KSTEP_BYTES;
    for (uint32_t off = rowb + tid * 16; off < padded; off += NT * 16)
        *(i32x4 *)(S.q + off) = i32x4{0, 0, 0, 0};
    for (int i = tid; i < SEL_CAP; i += NT)
        S.rank[i] = 0;
    if (tid == 0)
        S.n_cand = S.n_tiles = 0;
    // a scan's value as a distance key. Absent is a distance that is no
    // number: an entry past the bank (NaN), every row of an infinite request.
    auto key_of = [&](float acc) -> uint32_t {
        const float dist = fmaf(-2.f, acc, qn);
        return dist == dist ? f2key(dist) : KEY_NONE;
    };

    // ---- 1. the k super tiles
    uint32_t least = KEY_NONE;
    auto each_sup = [&](auto f) {   // f(key, index) of this thread's super tiles
#pragma unroll
        for (int u = 0; u < SV; ++u)
            f(key_of(sv[u]), (int)sup_at(u));
        for (int u = SV; ((long)u * NT) < A.n_sup; ++u) {
            const long j = sup_at(u);
            if (j < A.n_sup)
                f(key_of(sup(j)), (int)j);
        }
    };
    // a distance key and a margin far above any fp32 rounding difference, so
    // that it also bounds if a row's two evaluations should ever differ in
    // their last bits
    auto widen = [&](uint32_t key) -> uint32_t {
        const float t = key2f(key);
        return min(KEY_NONE - 1, f2key(t + ldexpf(qn + fabsf(t) + 1.f, -18)));
    };
    each_sup([&](uint32_t key, int) { least = min(least, key); });
    // nothing past the k-th row of the earlier parts of the bank
    uint32_t cap = KEY_NONE - 1;
    if (A.carry_in) {
        const uint32_t kth = A.list_key[(size_t)b * k + k - 1];
        if (kth != KEY_NONE)
            cap = widen(kth);
    }
    const auto umin = [](uint32_t x, uint32_t y) { return x < y ? x : y; };
    const auto umax = [](uint32_t x, uint32_t y) { return x > y ? x : y; };
    // the largest of the least distances of at least k groups (waves, half
    // waves or rows of lanes) has a super tile of each at or below it
    // groups of GL lanes, 64 of them; each step up halves their number, as far
    // as k allows (a group of its pair: 0, which no maximum takes)
    constexpr int GL = NT / WAVE;
    static_assert(GL == 16 || GL == 8 || GL == 4, "rows, half rows or quads of lanes");
    least = umin(least, dpp<0xb1>(least));
    least = umin(least, dpp<0x4e>(least));
    bool of_group = true;
    if (GL >= 8 || k <= NT / 8) {
        least = umin(least, dpp<0x141>(least));   // half rows of 8 lanes
        of_group = GL >= 8 || !(lane & 4);
    }
    if (GL == 16 || k <= NT / 16) {
        least = umin(least, dpp<0x140>(least));   // rows
        of_group = !(lane & 15 & ~(GL - 1));
    }
    if (k <= NT / 64) {
        least = rows_reduce(least, umin);   // waves
        of_group = lane < GL;
    } else if (k <= NT / 32) {
        least = umin(least, dpp<0x142, 0xa>(least));   // row_bcast:15: half waves
        of_group = (lane & 16) && !(lane & 15 & ~(GL - 1));
    }
    if (lane % GL == 0)
        S.group_min[wave * (WAVE / GL) + lane / GL] = of_group ? least : 0u;
    __syncthreads();
    // absent entries stay out
    uint32_t bound = min(cap, wave_reduce(S.group_min[lane], umax));
    each_sup([&](uint32_t key, int j) {
        if (key <= bound) {
            const int pos = atomicAdd(&S.n_cand, 1);
            if (pos < SEL_CAP)
                S.cand[pos] = pack(key, j);
        }
    });
    __syncthreads();
    int n_best = min(S.n_cand, k);
    if (S.n_cand <= SEL_CAP) {
        rank_pairs<NT>(S.cand, S.n_cand, k, S.rank, S.best);
    } else {
        uint64_t last = 0;
        for (int r = 0; r < k; ++r) {
            uint64_t m = PAIR_NONE;
            for (long i = tid; i < A.n_sup; i += NT) {
                const uint64_t v = pack(key_of(sup(i)), (int32_t)i);
                if ((r == 0 || v > last) && v < m)
                    m = v;
            }
            m = wave_min_u64(m);
            if (lane == 0)
                S.wave_min[wave] = m;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < NW; ++w)
                m = min(m, S.wave_min[w]);
            last = m;
            if (tid == 0)
                S.best[r] = m;
            __syncthreads();
        }
    }
    __syncthreads();

    // ---- 2. their row tiles
    bound = n_best == k ? min(cap, widen((uint32_t)(S.best[k - 1] >> 32))) : cap;
    const int fold = A.m.folded ? FOLD : 1;   // row tiles of an entry
    int n_items;   // what a round takes SEL_ROUND * 16 rows of
    if (A.acc) {
        n_items = n_best * A.eps * 16;
        if (tid < n_best)
            S.sup[tid] = (int)(uint32_t)S.best[tid];
    } else {
        const int per = A.eps / fold;
        for (int i = tid; i < n_best * per; i += NT) {
            const int j = i / per, e = i - j * per;
            const int s = (int)(uint32_t)S.best[j];
            const uint32_t key = A.eps == 1 ? (uint32_t)(S.best[j] >> 32) : key_of(ent(s, e));
            if (key <= bound) {
                const int at = atomicAdd(&S.n_tiles, 1);
                for (int f = 0; f < fold; ++f)
                    S.tiles[at * fold + f] = s * A.eps + e * fold + f;
                S.cand[at] = pack(key, s * A.eps + e * fold);
            }
        }
    }
    // the rows found in earlier launches over other parts of the bank
    if (tid < k && A.carry_in)
        S.prev[tid] = pack(A.list_key[(size_t)b * k + tid], A.list_idx[(size_t)b * k + tid]);
    __syncthreads();
    if (!A.acc) {
        n_items = S.n_tiles * fold * 16;
        // Many more than k entries: near rows follow one another in the
        // bank, the k-th super tile lies outside them and its distance is a
        // loose bound. The k-th of the entries' own distances is one too (a
        // row each), and leaves about k of them in any order of the bank
        // (1,000 clusters one after the other: 256 x 1,000,000 x 768 481 / 390
        // us, 1,024 x 1,000,000 x 1,024 2,285 / 1,825).
        if (n_items > (k * fold + NW) * 16) {
            rank_pairs<NT>(S.cand, S.n_tiles, k, S.rank, S.best);
            __syncthreads();
            bound = min(bound, widen((uint32_t)(S.best[k - 1] >> 32)));
            const int n = S.n_tiles;
            __syncthreads();
            if (tid == 0)
                S.n_tiles = 0;
            __syncthreads();
            for (int i = tid; i < n; i += NT)
                if ((uint32_t)(S.cand[i] >> 32) <= bound) {
                    const int at = atomicAdd(&S.n_tiles, 1);
                    for (int f = 0; f < fold; ++f)
                        S.tiles[at * fold + f] = (int)(uint32_t)S.cand[i] + f;
                }
            __syncthreads();
            n_items = S.n_tiles * fold * 16;
        }
    }

    // ---- 3. their rows
    int n_prev = A.carry_in ? k : 0;
    for (int r0 = 0; r0 == 0 || r0 < n_items; r0 += SEL_ROUND * 16) {
        if (tid == 0)
            S.n_cand = 0;
        __syncthreads();
        const int r1 = min(n_items, r0 + SEL_ROUND * 16);
        for (int i = tid; i < n_prev; i += NT)
            if ((uint32_t)(S.prev[i] >> 32) != KEY_NONE)
                S.cand[atomicAdd(&S.n_cand, 1)] = S.prev[i];
        if (A.acc) {
            for (int i = r0 + tid; i < r1; i += NT) {
                const int per = A.eps * 16, j = i / per;
                const long si = S.sup[j], ch = si / A.sup_per_chunk;
                const long in_ch = (si - ch * A.sup_per_chunk) * per + (i - j * per);
                const long row = ch * A.rows_per_chunk + in_ch;
                const float v = row < A.rows && in_ch < A.rows_per_chunk
                                    ? A.acc[((size_t)(row >> 4) * A.B + b) * 16 + (row & 15)]
                                    : __builtin_nanf("");
                const uint32_t key = key_of(v);
                if (key <= bound)   // (below KEY_NONE)
                    S.cand[atomicAdd(&S.n_cand, 1)] = pack(key, (int32_t)(A.row0 + row));
            }
        }
        for (int ti = r0 / 16 + wave; !A.acc && ti < r1 / 16; ti += NW) {
            const int te = __builtin_amdgcn_readfirstlane(S.tiles[ti]);
            // first row of the tile, and the end of its chunk
            const long si = te / A.eps, ch = si / A.sup_per_chunk;
            const int e0 = te % A.eps;
            const long in_ch = (si - ch * A.sup_per_chunk) * A.eps * 16 +
                               (A.split_tiles ? (e0 >> 1) * 32 + (e0 & 1) * 4 : e0 * 16);
            const long row = A.row0 + ch * A.rows_per_chunk + in_ch;
            const long rend = min(A.rows - ch * A.rows_per_chunk, A.rows_per_chunk);
            const int col = lane & 15, jg = lane >> 4;
            // (rows from `row` to the chunk's end, as far as a tile reaches)
            const int n_in = (int)max(0L, min(32L, rend - in_ch));
            // the tile's row of MFMA row i
            auto row_of = [&](int i) { return A.split_tiles ? ((i & 12) << 1) + (i & 3) : i; };
            const __amdgpu_buffer_rsrc_t r =
                make_rsrc(A.bank + (size_t)row * rowb, (uint32_t)n_in * rowb);
            const bool tail_ok = (A.nks - 1) * KS + jg * VEC < A.d;
            const uint32_t vo = (uint32_t)row_of(col) * rowb + jg * 16;
            auto load = [&](int s) -> i32x4 {
                return buffer_load16(r, s >= A.nks || (s == A.nks - 1 && !tail_ok)
                                            ? OFF_NONE
                                            : vo + s * KSTEP_BYTES);
            };
            // two blocks of LD k-steps in flight (past the row, zeros)
            i32x4 a[2][LD];
#pragma unroll
            for (int u = 0; u < 2 * LD; ++u)
                a[u / LD][u % LD] = load(u);
            f32x4 acc = __builtin_bit_cast(
                f32x4, buffer_load16(make_rsrc(A.bank_norms + row, (uint32_t)n_in * 4u),
                                       (uint32_t)row_of(jg * 4) * 4u));
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[e] = row_of(jg * 4 + e) < n_in ? -0.5f * acc[e] : -INFINITY;
            for (int s0 = 0; s0 < A.nks; s0 += 2 * LD) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint8_t *qf = S.q + (s0 + h * LD) * KSTEP_BYTES + jg * 16;
#pragma unroll
                    for (int u = 0; u < LD; ++u)
                        acc = mfma_step<DT>(a[h][u], *(const i32x4 *)(qf + u * KSTEP_BYTES), acc);
                    if (s0 + (h + 2) * LD < A.nks) {
#pragma unroll
                        for (int u = 0; u < LD; ++u)
                            a[h][u] = load(s0 + (h + 2) * LD + u);
                    }
                    if (s0 + (h + 1) * LD >= A.nks)
                        break;
                }
            }
            // lane (col, jg) holds rows jg*4 .. +3; every column the same
            if (col < 4) {
                const float v = col == 0 ? acc[0] : col == 1 ? acc[1] : col == 2 ? acc[2] : acc[3];
                const uint32_t key = key_of(v);
                const int i = row_of(jg * 4 + col);
                if (i < n_in && key <= bound)
                    S.cand[atomicAdd(&S.n_cand, 1)] = pack(key, (int32_t)(row + i));
            }
        }
        __syncthreads();
        int n = S.n_cand;
        if (tid < k)
            S.best[tid] = PAIR_NONE;
        __syncthreads();
        // Many rows for the threads (a bank of fewer super tiles than neighbours
        // has no bound): those past the k-th of the threads' own least pairs go
        // before the rest is ranked (with the bound of the earlier rounds below,
        // k = 64, every row ranked / so: 1,151 x 11,013 x 384 1,919 / 171 us,
        // fp32 2,000 x 1,000 x 384 279 / 74 us).
        constexpr int MOST = SEL_ROUND * 16 + RB_MAX_K_DEV;   // of one round
        if constexpr (2 * NT < MOST) {
            static_assert(MOST + NT <= SEL_CAP && RB_MAX_K_DEV <= NT);
            if (n > 2 * NT) {   // (every thread has some)
                constexpr int PER = (MOST + NT - 1) / NT;
                uint64_t own[PER], first_own = PAIR_NONE;
#pragma unroll
                for (int u = 0; u < PER; ++u) {
                    own[u] = u * NT + tid < n ? S.cand[u * NT + tid] : PAIR_NONE;
                    first_own = min(first_own, own[u]);
                }
                S.cand[MOST + tid] = first_own;
                __syncthreads();
                if (tid == 0)
                    S.n_cand = 0;
                rank_pairs<NT>(S.cand + MOST, NT, k, S.rank, S.best);
                __syncthreads();
                const uint64_t kth = S.best[k - 1];
#pragma unroll
                for (int u = 0; u < PER; ++u)
                    if (own[u] <= kth)
                        S.cand[atomicAdd(&S.n_cand, 1)] = own[u];
                __syncthreads();
                n = S.n_cand;
            }
        }
        rank_pairs<NT>(S.cand, n, k, S.rank, S.best);
        __syncthreads();
        if (tid < k)
            S.prev[tid] = S.best[tid];
        n_prev = k;
        // (a row past the k-th found is none of the k; absent is past any bound)
        bound = min(bound, (uint32_t)(S.best[k - 1] >> 32));
    }

    // ---- 4. results (fewer than k rows that are numbers: index -1, NaN)
    if (tid < k) {
        const uint64_t v = S.best[tid];
        const uint32_t key = (uint32_t)(v >> 32);
        const int32_t idx = (int32_t)(uint32_t)v;
        const size_t o = (size_t)b * k + tid;
        if (A.list_key) {
            A.list_key[o] = key;
            A.list_idx[o] = idx;
        }
        if (A.nbr_idx) {
            A.nbr_idx[o] = idx;
            if (A.nbr_dist)
                A.nbr_dist[o] = key2f(key);
        }
        S.nbr[tid] = idx;
        S.wts[tid] = inv_dist_weight(key2f(key));
    }
    if (!A.q_hat)
        return;
    __syncthreads();
    // every (neighbour, model) label in flight at once, then the averages in
    // neighbour order, as average_labels takes them (whose loop serves more
    // labels than threads)
    const int M = A.M;
    if (k * M <= NT) {
        float *lq = (float *)S.cand, *ll = lq + NT;
        if (tid < k * M) {
            const int j = tid / M;
            const int32_t n = S.nbr[j];
            const bool ok = n >= 0 && n < A.N;
            const size_t o = (size_t)(ok ? n : 0) * M + (tid - j * M);
            lq[tid] = ok ? A.qual[o] : __builtin_nanf("");
            ll[tid] = ok ? A.len[o] : __builtin_nanf("");
        }
        __syncthreads();
        if (tid < M) {
            float sq = 0.f, sl = 0.f, sw = 0.f;
#pragma unroll 8
            for (int j = 0; j < k; ++j) {
                const float q = lq[j * M + tid], l = ll[j * M + tid];
                if (A.inv_dist) {
                    const float w = S.wts[j];
                    sq = fmaf(w, q, sq);
                    sl = fmaf(w, l, sl);
                    sw += w;
                } else {
                    sq += q;
                    sl += l;
                }
            }
            if (!A.inv_dist)
                sw = (float)k;
            A.q_hat[(size_t)b * M + tid] = sq / sw;
            A.l_hat[(size_t)b * M + tid] = sl / sw;
        }
        return;
    }
    for (int m = tid; m < M; m += NT)
        average_labels(S.nbr, A.inv_dist ? S.wts : nullptr, k, A.qual, A.len, A.N, M, m,
                       A.q_hat + (size_t)b * M + m, A.l_hat + (size_t)b * M + m);
}

// The second half of a lookup taken in two calls: the neighbours from the
// lists the first half left, and the label average. One wave per request.
__global__ __launch_bounds__(WAVE) void from_list_kernel(const SelectArgs A)
{
    __shared__ int32_t nbr[RB_MAX_K_DEV];
    __shared__ float wts[RB_MAX_K_DEV];
    const int b = blockIdx.x, j = threadIdx.x, k = A.k;
    if (j < k) {
        const size_t o = (size_t)b * k + j;
        const int32_t idx = A.list_idx[o];
        const float dist = key2f(A.list_key[o]);
        nbr[j] = idx;
        wts[j] = inv_dist_weight(dist);
        if (A.nbr_idx)
            A.nbr_idx[o] = idx;
        if (A.nbr_dist)
            A.nbr_dist[o] = dist;
    }
    if (!A.q_hat)
        return;
    __syncthreads();
    for (int m = j; m < A.M; m += WAVE)
        average_labels(nbr, A.inv_dist ? wts : nullptr, k, A.qual, A.len, A.N, A.M, m,
                       A.q_hat + (size_t)b * A.M + m, A.l_hat + (size_t)b * A.M + m);
}

}  // namespace

hipError_t launch_select(int dtype, const SelectArgs &a, hipStream_t s)
{
    // one workgroup of 16 waves per compute unit while there are enough units;
    // more requests go in workgroups of 8, two to a unit, and past those in
    // workgroups of 4, so that one's chain of accesses and barriers runs beside
    // the others' (whole lookups, in workgroups of 8 and 4: 2,000 requests over
    // 3,381 x 96 62 / 38 us, 600 over 3,381 x 96 30 / 21, 1,024 over 30,000 x 768,
    // 32 neighbours, 159 / 137; but 300 over 16,000 x 2,048 100 / 103)
#define RB_SELECT(NT)                                                                            \
    do {                                                                                         \
        if (dtype == 1)                                                                          \
            hipLaunchKernelGGL((select_kernel<1, NT>), dim3(a.B), dim3(NT), 0, s, a);            \
        else                                                                                     \
            hipLaunchKernelGGL((select_kernel<0, NT>), dim3(a.B), dim3(NT), 0, s, a);            \
    } while (0)
    if (a.B <= SEL_WIDE_B)
        RB_SELECT(SEL_THREADS);
    else if (a.B <= 2 * SEL_WIDE_B)
        RB_SELECT(SEL_THREADS / 2);
    else
        RB_SELECT(SEL_THREADS / 4);
#undef RB_SELECT
    return hipGetLastError();
}

hipError_t launch_from_list(const SelectArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(from_list_kernel, dim3(a.B), dim3(WAVE), 0, s, a);
    return hipGetLastError();
}

}  // namespace rb
