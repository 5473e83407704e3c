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

// Sorts the n pairs of `cand` in LDS (distinct but for PAIR_NONE) by counting,
// for each, the pairs below it; the k smallest go to out[0 .. min(k, n)).
// Every thread of the workgroup takes part; no barrier inside.
__device__ __forceinline__ void rank_pairs(const uint64_t *cand, int n, int k, uint64_t *out)
{
    for (int i = threadIdx.x; i < n; i += SEL_THREADS) {
        const uint64_t mine = cand[i];
        int r = 0;
        for (int j = 0; j < n; ++j)
            r += cand[j] < mine ? 1 : 0;
        if (r < k)
            out[r] = mine;
    }
}

// One workgroup per request. The scan left, per super tile, the largest
// <q, x> - |x|^2/2 of its rows, i.e. the distance of its nearest row. The k
// nearest rows lie in the k super tiles that come first by (that distance,
// index): a row of any other super tile has k rows before it in (distance,
// index) order, one in each of those k. Within them only row tiles whose own
// nearest row is no farther than the k-th super tile's can hold one of the k
// (k rows lie at or below that distance), in random order about k of them.
// Those tiles' distances are computed again, with the scan's own sequence of
// MFMA steps (so with its bits), and the k smallest (distance, index) pairs
// of their rows are the result. What bounds it: a chain of about five
// dependent memory accesses at small batches, at large ones the reading of
// k tiles (16 rows) per request.
//   1. a bound: every wave takes the k-th smallest of its lanes' two smallest
//      super-tile distances; the workgroup the least of those. The super
//      tiles at or below the bound go to LDS (about k times the wave count
//      in random order) and are ranked by counting. More than fit (a bank of
//      mostly equal rows) are taken k times the smallest instead.
//   2. the row tiles of the k super tiles under the k-th distance.
//   3. their rows' distances, SEL_ROUND tiles at a time: one wave per tile,
//      the request replicated over the MFMA's columns; rows at or below the
//      bound join the list, which is ranked after each round.
//   4. the neighbours, and the label average.
struct SelectShared {
    uint64_t cand[SEL_CAP];
    uint64_t best[RB_MAX_K_DEV], prev[RB_MAX_K_DEV];
    uint32_t wave_t[SEL_THREADS / WAVE];
    uint64_t wave_min[SEL_THREADS / WAVE];
    int tiles[RB_MAX_K_DEV * SEL_MAX_EPS];
    int n_cand, n_tiles;
    int32_t nbr[RB_MAX_K_DEV];
    float wts[RB_MAX_K_DEV];
    __align__(16) uint8_t q[SEL_MAX_ROW_BYTES];
};
static_assert(SEL_ROUND * 16 + RB_MAX_K_DEV <= SEL_CAP, "a round's rows and the running best");

template <int DT>
__global__ __launch_bounds__(SEL_THREADS) void select_kernel(const SelectArgs A)
{
    constexpr int VEC = Elem<DT>::VEC, ESZ = Elem<DT>::ESZ;
    constexpr int KS = 4 * VEC;
    constexpr int NW = SEL_THREADS / WAVE;
    constexpr int LD = 12;   // k-steps of bank loads in flight
    __shared__ SelectShared S;
    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int k = A.k;
    const uint32_t rowb = (uint32_t)A.d * ESZ;
    const float *sup = A.sup + (size_t)b * A.n_sup;
    const float *ent = A.ent + (size_t)b * A.n_sup * A.eps;

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
    for (uint32_t off = rowb + tid * 16; off < (uint32_t)A.nks * KSTEP_BYTES; off += SEL_THREADS * 16)
        *(i32x4 *)(S.q + off) = i32x4{0, 0, 0, 0};
    if (tid == 0)
        S.n_cand = S.n_tiles = 0;
    // a maximum as a distance key; an entry past the bank (NaN) is absent
    auto key_of = [&](float acc) -> uint32_t {
        return acc == acc ? f2key(fmaf(-2.f, acc, qn)) : KEY_NONE;
    };

    // ---- 1. the k super tiles
    uint32_t m1 = KEY_NONE, m2 = KEY_NONE;
    for (long i = tid; i < A.n_sup; i += 8 * SEL_THREADS) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const long j = i + (long)u * SEL_THREADS;
            v[u] = j < A.n_sup ? sup[j] : __builtin_nanf("");
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t key = key_of(v[u]);
            m2 = min(m2, max(m1, key));
            m1 = min(m1, key);
        }
    }
    {
        // the k-th smallest of the wave's lane values: the largest prefix
        // with fewer than k of them below it
        uint32_t prefix = 0;
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t trial = prefix | (1u << bit);
            if (popc(ballot(m1 < trial)) + popc(ballot(m2 < trial)) < k)
                prefix = trial;
        }
        if (lane == 0)
            S.wave_t[wave] = prefix;
    }
    __syncthreads();
    uint32_t bound = KEY_NONE - 1;   // absent entries stay out
#pragma unroll
    for (int w = 0; w < NW; ++w)
        bound = min(bound, S.wave_t[w]);
    for (long i = tid; i < A.n_sup; i += 8 * SEL_THREADS) {
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const long j = i + (long)u * SEL_THREADS;
            v[u] = j < A.n_sup ? sup[j] : __builtin_nanf("");
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t key = key_of(v[u]);
            if (key <= bound) {
                const int pos = atomicAdd(&S.n_cand, 1);
                if (pos < SEL_CAP)
                    S.cand[pos] = pack(key, (int32_t)(i + (long)u * SEL_THREADS));
            }
        }
    }
    __syncthreads();
    int n_best = min(S.n_cand, k);
    if (S.n_cand <= SEL_CAP) {
        rank_pairs(S.cand, S.n_cand, k, S.best);
    } else {
        uint64_t last = 0;
        for (int r = 0; r < k; ++r) {
            uint64_t m = PAIR_NONE;
            for (long i = tid; i < A.n_sup; i += SEL_THREADS) {
                const uint64_t v = pack(key_of(sup[i]), (int32_t)i);
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

    // ---- 2. their row tiles (the bound widened by a margin far above any
    // fp32 rounding difference, so that it also holds if a row's two
    // evaluations should ever differ in their last bits)
    if (n_best == k) {
        const float t = key2f((uint32_t)(S.best[k - 1] >> 32));
        bound = min(KEY_NONE - 1, f2key(t + ldexpf(qn + fabsf(t) + 1.f, -18)));
    }
    for (int i = tid; i < n_best * A.eps; i += SEL_THREADS) {
        const int j = i / A.eps, e = i - j * A.eps;
        const int s = (int)(uint32_t)S.best[j];
        bool in = true;
        if (A.eps > 1)
            in = key_of(ent[(size_t)s * A.eps + e]) <= bound;
        if (in)
            S.tiles[atomicAdd(&S.n_tiles, 1)] = s * A.eps + e;
    }
    // the rows found in earlier launches over other parts of the bank
    if (tid < k && A.carry_in)
        S.prev[tid] = pack(A.list_key[(size_t)b * k + tid], A.list_idx[(size_t)b * k + tid]);
    __syncthreads();
    const int n_tiles = S.n_tiles;

    // ---- 3. their rows
    int n_prev = A.carry_in ? k : 0;
    for (int r0 = 0; r0 == 0 || r0 < n_tiles; r0 += SEL_ROUND) {
        if (tid == 0)
            S.n_cand = 0;
        __syncthreads();
        for (int i = tid; i < n_prev; i += SEL_THREADS)
            if ((uint32_t)(S.prev[i] >> 32) != KEY_NONE)
                S.cand[atomicAdd(&S.n_cand, 1)] = S.prev[i];
        for (int ti = r0 + wave; ti < min(n_tiles, r0 + SEL_ROUND); ti += NW) {
            const int te = __builtin_amdgcn_readfirstlane(S.tiles[ti]);
            const long row = A.row0 + (long)te * 16;      // first row of the tile
            const long rend = A.row0 + A.rows;
            const int col = lane & 15, jg = lane >> 4;
            const long n_in = min(16L, rend - row);
            const __amdgpu_buffer_rsrc_t r =
                make_rsrc(A.bank + (size_t)row * rowb, (uint32_t)n_in * rowb);
            const bool tail_ok = (A.nks - 1) * KS + jg * VEC < A.d;
            const uint32_t vo = (uint32_t)col * rowb + jg * 16;
            auto load = [&](int s) -> i32x4 {
                return buffer_load16(r, s >= A.nks || (s == A.nks - 1 && !tail_ok)
                                            ? OFF_NONE
                                            : vo + s * KSTEP_BYTES);
            };
            f32x4 acc;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[e] = jg * 4 + e < n_in ? -0.5f * A.bank_norms[row + jg * 4 + e] : -INFINITY;
            for (int s0 = 0; s0 < A.nks; s0 += LD) {
                i32x4 a[LD];
#pragma unroll
                for (int u = 0; u < LD; ++u)
                    a[u] = load(s0 + u);
#pragma unroll
                for (int u = 0; u < LD; ++u)
                    if (s0 + u < A.nks)
                        acc = mfma_step<DT>(
                            a[u], *(const i32x4 *)(S.q + (s0 + u) * KSTEP_BYTES + jg * 16), acc);
            }
            // lane (col, jg) holds rows jg*4 .. +3; every column the same
            if (col < 4) {
                const float v = col == 0 ? acc[0] : col == 1 ? acc[1] : col == 2 ? acc[2] : acc[3];
                const uint32_t key = f2key(fmaf(-2.f, v, qn));
                // (a distance that is not a number is no neighbour)
                if (v == v && jg * 4 + col < n_in && key <= bound)
                    S.cand[atomicAdd(&S.n_cand, 1)] = pack(key, (int32_t)(row + jg * 4 + col));
            }
        }
        __syncthreads();
        const int n = S.n_cand;
        if (tid < k)
            S.best[tid] = PAIR_NONE;
        __syncthreads();
        rank_pairs(S.cand, n, k, S.best);
        __syncthreads();
        if (tid < k)
            S.prev[tid] = S.best[tid];
        n_prev = k;
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
    for (int m = tid; m < A.M; m += SEL_THREADS)
        average_labels(S.nbr, A.inv_dist ? S.wts : nullptr, k, A.qual, A.len, A.N, A.M, m,
                       A.q_hat + (size_t)b * A.M + m, A.l_hat + (size_t)b * A.M + m);
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
    if (dtype == 1)
        hipLaunchKernelGGL(select_kernel<1>, dim3(a.B), dim3(SEL_THREADS), 0, s, a);
    else
        hipLaunchKernelGGL(select_kernel<0>, dim3(a.B), dim3(SEL_THREADS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_from_list(const SelectArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(from_list_kernel, dim3(a.B), dim3(WAVE), 0, s, a);
    return hipGetLastError();
}

}  // namespace rb
