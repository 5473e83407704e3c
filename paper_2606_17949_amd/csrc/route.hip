// Request-instance scoring and the greedy online assignment (RouteBalance
// Eq. 1 score, Eq. 2 cost, the dead-reckoned latency of Sec. 4.2, and the
// greedy per-batch loop of Alg. 1), for gfx950.
//
// Both kernels evaluate the score with the same arithmetic (explicit fused
// multiply-adds, reciprocal rates, and the two Eq. 1 ratios as IEEE divisions
// so that the instance at a maximum gets exactly 1), so the dense score matrix
// and the scores the greedy loop sees at the batch-start state agree bit for
// bit.
#include "common.hpp"
#include "kernels.hpp"

namespace rb {

namespace {

// Latency of a request with prompt l and predicted output lv on an instance
// with queued prefill p, active decode a and reciprocal rates rP = 1/P,
// rD = 1/D: the queued prefill plus this prompt drains at P, then the active
// decode plus this output at D.
__device__ __forceinline__ float latency(float p, float a, float rP, float rD, float l, float lv)
{
    return fmaf(p + l, rP, (a + lv) * rD);
}

// Eq. 2 expected cost: input tokens at the input price plus predicted output
// tokens at the output price.
__device__ __forceinline__ float cost(float l, float lv, float cin, float cout)
{
    return fmaf(l, cin, lv * cout);
}

// x / max, or 0 for a zero maximum.
__device__ __forceinline__ float ratio(float x, float m) { return m > 0.f ? x / m : 0.f; }

// The state-independent part of Eq. 1: w_qual*Q + w_cost*(1 - C/Cmax).
__device__ __forceinline__ float base_score(float qv, float C, float cmax, float wq, float wc)
{
    return fmaf(wq, qv, wc * (1.f - ratio(C, cmax)));
}

// Eq. 1: base + w_lat*(1 - T/Tmax).
__device__ __forceinline__ float full_score(float base, float T, float tmax, float wl)
{
    return fmaf(wl, 1.f - ratio(T, tmax), base);
}

// Alg. 1 budget filter on the Eq. 2 cost C of a request with budget b, and
// the availability mask: whether instance i is a candidate.
__device__ __forceinline__ bool admitted(float C, float b, const uint8_t *mask, int i)
{
    return (!mask || mask[i] != 0) && C <= b;
}

// One wave per request row of the dense score matrix. With a budget or a
// mask (opt.budget, opt.mask; opt.order is not read) the maxima run over the
// request's candidates and the other instances score NaN, as in the greedy
// loop's first step.
__global__ __launch_bounds__(256) void score_kernel(const float *__restrict__ q_hat,
                                                    const float *__restrict__ l_hat,
                                                    const int32_t *__restrict__ plen, int B, int M,
                                                    const InstArgs in, int I, float wq, float wl,
                                                    float wc, const AssignOpts opt,
                                                    float *__restrict__ S0)
{
    const int lane = lane_id();
    const int r = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (r >= B)
        return;
    const float l = (float)plen[r];
    const float *qr = q_hat + (size_t)r * M;
    const float *lr = l_hat + (size_t)r * M;
    const float nan = __builtin_nanf("");
    const float budget = opt.budget ? opt.budget[r] : INFINITY;
    float cmax = -INFINITY, tmax = -INFINITY;
    for (int i = lane; i < I; i += WAVE) {
        const int m = in.model[i];
        const float lv = (unsigned)m < (unsigned)M ? lr[m] : nan;
        const float C = cost(l, lv, in.cin[i], in.cout[i]);
        if (!admitted(C, budget, opt.mask, i))
            continue;
        cmax = fmaxf(cmax, C);
        tmax = fmaxf(tmax, latency(in.p[i], in.a[i], 1.f / in.P[i], 1.f / in.D[i], l, lv));
    }
    cmax = wave_max(cmax);
    tmax = wave_max(tmax);
    for (int i = lane; i < I; i += WAVE) {
        const int m = in.model[i];
        const bool mv = (unsigned)m < (unsigned)M;
        const float lv = mv ? lr[m] : nan;
        const float qv = mv ? qr[m] : nan;
        const float C = cost(l, lv, in.cin[i], in.cout[i]);
        const float T = latency(in.p[i], in.a[i], 1.f / in.P[i], 1.f / in.D[i], l, lv);
        S0[(size_t)r * I + i] = admitted(C, budget, opt.mask, i)
                                    ? full_score(base_score(qv, C, cmax, wq, wc), T, tmax, wl)
                                    : nan;
    }
}

// Longest-predicted-first order (Alg. 1; Sec. 4.1 keys a request by the
// maximum over models of its predicted length). Each request's position is
// the number of requests before it under (key descending, index ascending),
// a total order, so the positions form a permutation: order[pos] = r. Every
// workgroup ranks LPT_RANK requests against all B keys, LPT_TILE at a time in
// LDS, its four waves a quarter of them each. What bounds it is latency: a
// tile's keys are all loaded together, and few requests per workgroup keep the
// count short (1,024 requests of 16 models: 25 us in workgroups of 256 with
// 256 keys at a time).
constexpr int LPT_THREADS = 256;
constexpr int LPT_RANK = WAVE;
constexpr int LPT_TILE = 2048;

__global__ __launch_bounds__(LPT_THREADS) void lpt_order_kernel(const float *__restrict__ l_hat,
                                                                 int B, int M,
                                                                 int32_t *__restrict__ order)
{
    __shared__ uint64_t keys[LPT_TILE];
    __shared__ uint64_t own[LPT_RANK];
    __shared__ int pos[LPT_RANK];
    // ascending in this 64-bit key is descending in the length, then
    // ascending in the index
    auto key_of = [&](int r) {
        const float *row = l_hat + (size_t)r * M;
        float mx = row[0];
#pragma unroll 8
        for (int m = 1; m < M; ++m)
            mx = fmaxf(mx, row[m]);
        return ((uint64_t)~f2key(mx) << 32) | (uint32_t)r;
    };
    const int tid = threadIdx.x, lane = lane_id(), part = tid / WAVE;
    const int r = blockIdx.x * LPT_RANK + lane;
    if (tid < LPT_RANK) {
        pos[tid] = 0;
        own[tid] = r < B ? key_of(r) : ~0ull;
    }
    for (int base = 0; base < B; base += LPT_TILE) {
        const int n = min(LPT_TILE, B - base);
        if (base > 0)
            __syncthreads();
#pragma unroll 4
        for (int i = tid; i < n; i += LPT_THREADS)
            keys[i] = key_of(base + i);
        __syncthreads();
        const uint64_t mine = own[lane];
        const int j0 = n * part / (LPT_THREADS / WAVE), j1 = n * (part + 1) / (LPT_THREADS / WAVE);
        int c = 0;
#pragma unroll 8
        for (int j = j0; j < j1; ++j)
            c += keys[j] < mine ? 1 : 0;
        atomicAdd(&pos[lane], c);
    }
    __syncthreads();
    if (tid < LPT_RANK && r < B)
        order[pos[tid]] = r;
}

// Greedy assignment. Wave 0 runs the sequential loop over requests; waves
// 1..15 fill, one chunk of steps ahead, an LDS double buffer with what does
// not depend on the state: per (request, instance) the base score and the
// predicted output length on the instance's model. Step t decides request
// order[t] (arrival order when order is null). An instance outside the
// request's candidate set (unavailable in mask, or over the request's budget
// in the Eq. 2 cost) gets a NaN base score: it is left out of both maxima and
// its key is NO_KEY whatever its queues and predictions hold, so that it is
// never picked. WIDTH = 16 (I <= 16):
// instance i = lane % 16, replicated in the four rows of 16 lanes, so every
// reduction stays inside a row and leaves its result in every lane. WIDTH = 64:
// instance i = lane + 64*u in register slot u. Per request: the latency
// maximum, then the pick. Latencies are positive (queues and lengths are
// non-negative, prompts at least one token, rates positive), so the Eq. 1
// score orders the candidates as S*Tmax = base*Tmax + w_lat*(Tmax - T) does,
// which needs no division; both T and S*Tmax are non-negative (scores lie in
// [0, 1]), so their float bits order as integers. One integer
// maximum, a ballot of the lanes that hold it and a find-first-set give the
// largest score and, among equal scores, the lowest instance index;
// the lanes holding that instance update its state.
//
// The loop is bound by its chain of dependent instructions, so everything but
// the pick itself is taken off it: while step t's maximum is reduced, every
// lane works out step t+1's latency both as the state stands and as it would
// be had it been picked, and the former's maximum. A pick only adds to its
// instance's queues (lengths are not negative), so the maximum of step t+1 is
// the larger of that maximum and the picked lane's second latency: one lane
// read instead of a second reduction. (ns a step with both reductions in the
// chain, and now: 231 / 138 on 13 instances, 268 / 165 on 64, 330 / 260 on 128,
// 495 / 398 on 256; the loop is bound by instruction issue, about 2 ns each.)
// The pick's latency and Tmax are captured, one step per lane, and every 64 steps the wave writes the picks and computes their Eq. 1 scores
// (with the division, exactly as the dense score kernel does) in one vector
// pass. A request without candidates gets -1 and changes no state.
constexpr int ASSIGN_THREADS = 1024;
constexpr int ASSIGN_LDS_FLOATS = 8192;   // per buffer: chunk rows x instances x 2

// A request's base scores and predicted lengths over the instance set, as the
// loop reads them: what does not depend on the state.
struct Pair {
    float base, lv;   // base NaN: not a candidate
};

// Keys of the pick as signed integers: S*Tmax bits, those of a non-candidate,
// and what the maximum starts from (no candidate holds it).
constexpr int NO_KEY = (int)0x80000000, LEAST_KEY = (int)0x80000001;

template <int IPL, int WIDTH, bool DECIDED>
__global__ __launch_bounds__(ASSIGN_THREADS) void assign_kernel(
    const float *__restrict__ q_hat, const float *__restrict__ l_hat,
    const int32_t *__restrict__ plen, int B, int M, const InstArgs in, int I, float wq, float wl,
    float wc, const AssignOpts opt, int32_t *__restrict__ assign, float *__restrict__ chosen,
    float *__restrict__ decided)
{
    static_assert(WIDTH == 64 || IPL == 1, "a 16-lane row holds one slot");
    constexpr int IP = IPL * WIDTH;                       // instances per LDS row
    constexpr int CH = ASSIGN_LDS_FLOATS / (2 * IP);      // requests per chunk
    __shared__ Pair pair_s[2][CH + 2][IP];   // (two rows of slack: the loop reads ahead)
    __shared__ float l_s[2][CH + 2];
    __shared__ int32_t r_s[2][CH];
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_ch = (B + CH - 1) / CH;
    auto inst = [&](int u) { return WIDTH == 16 ? (lane & 15) : lane + WAVE * u; };
    // maximum over the instance set, as an unsigned maximum of order-preserving
    // keys (a DPP step folds into one v_max_u32; no NaN canonicalisation)
    auto fmax_all = [&](float v) {
        const auto umax = [](uint32_t x, uint32_t y) { return x > y ? x : y; };
        if constexpr (WIDTH == 16)
            return key2f(row16_reduce(f2key(v), umax));
        else
            return key2f(wave_reduce(f2key(v), umax));
    };

    // producers: step t = c*CH + j into slot j of buffer c & 1, one wave per step
    auto produce = [&](int c) {
        const int buf = c & 1;
        for (int j = wave - 1; j < CH; j += ASSIGN_THREADS / WAVE - 1) {
            const int t = c * CH + j;
            if (t >= B)
                break;
            const int r = opt.order ? opt.order[t] : t;
            const float l = (float)plen[r];
            const float *qr = q_hat + (size_t)r * M;
            const float *lr = l_hat + (size_t)r * M;
            const float budget = opt.budget ? opt.budget[r] : INFINITY;
            float qv[IPL], lv[IPL], C[IPL];
            bool cand[IPL];
            float cmax = -INFINITY;
#pragma unroll
            for (int u = 0; u < IPL; ++u) {
                const int i = inst(u);
                const int m = i < I ? in.model[i] : -1;
                const bool ok = (unsigned)m < (unsigned)M;
                qv[u] = ok ? qr[m] : 0.f;
                lv[u] = ok ? lr[m] : 0.f;
                C[u] = cost(l, lv[u], ok ? in.cin[i] : 0.f, ok ? in.cout[i] : 0.f);
                // Alg. 1 budget filter on the Eq. 2 cost, and availability
                cand[u] = ok && admitted(C[u], budget, opt.mask, i);
                if (cand[u])
                    cmax = fmaxf(cmax, C[u]);
            }
            cmax = fmax_all(cmax);
            if (lane < (WIDTH == 16 ? 16 : WAVE)) {
#pragma unroll
                for (int u = 0; u < IPL; ++u) {
                    Pair v;
                    v.base = base_score(qv[u], C[u], cmax, wq, wc);
                    if (!cand[u])
                        v.base = __builtin_nanf("");
                    v.lv = lv[u];
                    pair_s[buf][j][lane + WAVE * u] = v;
                }
            }
            if (lane == 0) {
                l_s[buf][j] = l;
                r_s[buf][j] = r;
            }
        }
    };

    if (wave > 0) {
        produce(0);
        __syncthreads();
        for (int c = 0; c < n_ch; ++c) {
            if (c + 1 < n_ch)
                produce(c + 1);
            __syncthreads();
        }
        return;
    }

    // consumer: instance state in registers
    const int col = WIDTH == 16 ? (lane & 15) : lane;   // this lane's column of an LDS row
    float p[IPL], a[IPL], rP[IPL], rD[IPL];
    bool valid[IPL];
#pragma unroll
    for (int u = 0; u < IPL; ++u) {
        const int i = inst(u);
        // an instance whose model id is outside [0, M) is never chosen
        const int m = i < I ? in.model[i] : -1;
        valid[u] = (unsigned)m < (unsigned)M;
        p[u] = valid[u] ? in.p[i] : 0.f;
        a[u] = valid[u] ? in.a[i] : 0.f;
        rP[u] = valid[u] ? 1.f / in.P[i] : 0.f;
        rD[u] = valid[u] ? 1.f / in.D[i] : 0.f;
    }
    const auto imax = [](int x, int y) { return x > y ? x : y; };
    // maximum over the instance set, in every lane
    auto imax_all = [&](int v) {
        v = row16_reduce(v, imax);
        if constexpr (WIDTH == 64)
            v = rows_reduce(v, imax);
        return v;
    };
    auto lane_of = [](float v, int src) {
        return __builtin_bit_cast(float,
                                  __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
    };
    // As signed integers, the bits of non-negative floats order as the floats,
    // above those of any negative one (a negative quality may give some
    // instances scores below zero; qualities lie in [0, 1], so the best one's
    // is not).
    // Tmax is at least TINY (no latency is that small).
    constexpr int TINY = 0x00800000;
    // Lane NONE stands for "no instance" (WIDTH = 16: the rows past the first
    // are copies, so one of the last may).
    constexpr int NONE = 48;
    // Steps go in blocks of 64: lane s captures the pick of step (block + s).
    int cap_i = -1;
    float cap_t = 0.f, cap_m = 0.f;
    __syncthreads();   // chunk 0 is ready
    for (int c = 0; c < n_ch; ++c) {
        const int buf = c & 1;
        const int rows = min(CH, B - c * CH);
        float bs[IPL], lv[IPL], T[IPL], l;      // this step
        float bs1[IPL], lv1[IPL], l1;           // the next one
        // (past the chunk: whatever lies there, for no step)
        auto fetch = [&](int j, float(&bsx)[IPL], float(&lvx)[IPL], float &lx) {
#pragma unroll
            for (int u = 0; u < IPL; ++u) {
                const Pair v = pair_s[buf][j][col + WAVE * u];
                bsx[u] = v.base;
                lvx[u] = v.lv;
            }
            lx = l_s[buf][j];
        };
        fetch(0, bs, lv, l);
        fetch(1, bs1, lv1, l1);
        int tb = TINY;
        bool cand[IPL];
#pragma unroll
        for (int u = 0; u < IPL; ++u) {
            T[u] = latency(p[u], a[u], rP[u], rD[u], l, lv[u]);
            cand[u] = bs[u] == bs[u];
            tb = imax(tb, cand[u] ? __float_as_int(T[u]) : 0);
        }
        float tmax = __int_as_float(imax_all(tb));
        for (int jb = 0; jb < rows; jb += WAVE) {
            const int nb = __builtin_amdgcn_readfirstlane(min(WAVE, rows - jb));
            for (int slot = 0; slot < nb; ++slot) {
                float bs2[IPL], lv2[IPL], l2;   // the step after, in flight
                fetch(jb + slot + 2, bs2, lv2, l2);
                // S * Tmax; the candidates by a test kept from the step before
                // or, one slot, made again (256 instances: 397 ns a step for
                // 421; 13 instances: 138 for 154)
                int key[IPL], kb = LEAST_KEY;
#pragma unroll
                for (int u = 0; u < IPL; ++u) {
                    const float v = fmaf(bs[u], tmax, wl * (tmax - T[u]));
                    const bool c = WIDTH == 64 ? cand[u] : bs[u] == bs[u];
                    key[u] = c ? __float_as_int(v) : NO_KEY;
                    kb = imax(kb, key[u]);
                }
                // the state after a pick of the lane's instance, and the next
                // step's latencies without and with it (0 for its non-candidates)
                float p1[IPL], a1[IPL], T0[IPL], T1[IPL], tn[IPL];
                int t0 = TINY;
                bool cand1[IPL];
#pragma unroll
                for (int u = 0; u < IPL; ++u) {
                    p1[u] = p[u] + l;
                    a1[u] = a[u] + lv[u];
                    T0[u] = latency(p[u], a[u], rP[u], rD[u], l1, lv1[u]);
                    T1[u] = latency(p1[u], a1[u], rP[u], rD[u], l1, lv1[u]);
                    cand1[u] = bs1[u] == bs1[u];
                    t0 = imax(t0, cand1[u] ? __float_as_int(T0[u]) : 0);
                    tn[u] = cand1[u] && (WIDTH == 64 || lane < NONE) ? T1[u] : 0.f;
                }
                t0 = imax_all(t0);
                const int kmax = imax_all(kb);   // (LEAST_KEY, which no lane holds, without candidates)
                // lowest instance holding the maximum (slots ascend in index)
                int istar, src;
                float tp = T[0], tx = tn[0];
                if constexpr (WIDTH == 16) {
                    // (the four rows hold the same instances)
                    istar = src = (int)__builtin_ctzll((ballot(key[0] == kmax) & 0xffffull) |
                                                       (1ull << NONE));
                } else {
                    istar = -1;
                    int ustar = 0;
#pragma unroll
                    for (int u = 0; u < IPL; ++u) {
                        const uint64_t mk = ballot(key[u] == kmax);
                        if (istar < 0 && mk != 0) {
                            istar = WAVE * u + (int)__builtin_ctzll(mk);
                            ustar = u;
                        }
                    }
#pragma unroll
                    for (int u = 1; u < IPL; ++u) {
                        tp = ustar == u ? T[u] : tp;
                        tx = ustar == u ? tn[u] : tx;
                    }
                    src = istar & (WAVE - 1);
                }
                const float tpick = lane_of(tp, src);
                float tnext = lane_of(tx, src);
                if (WIDTH == 64)
                    tnext = istar >= 0 ? tnext : 0.f;
                // capture the pick in lane `slot`: the instance, its latency, Tmax
                const bool mine = lane == slot;
                cap_i = mine ? istar : cap_i;
                cap_t = mine ? tpick : cap_t;
                cap_m = mine ? tmax : cap_m;
                if (DECIDED) {
                    // the row of Eq. 1 scores this step saw, at the state
                    // before its update (NaN outside the candidate set), with
                    // the division of the dense score kernel
                    const int rq = r_s[buf][jb + slot];
                    float *drow = decided + (size_t)rq * I;
#pragma unroll
                    for (int u = 0; u < IPL; ++u) {
                        const int i = inst(u);
                        if (lane < (WIDTH == 16 ? 16 : WAVE) && i < I)
                            drow[i] = bs[u] == bs[u] ? full_score(bs[u], T[u], tmax, wl)
                                                     : __builtin_nanf("");
                    }
                }
                tmax = __int_as_float(imax(t0, __float_as_int(tnext)));
#pragma unroll
                for (int u = 0; u < IPL; ++u) {
                    const bool hit = inst(u) == istar;
                    p[u] = hit ? p1[u] : p[u];
                    a[u] = hit ? a1[u] : a[u];
                    T[u] = hit ? T1[u] : T0[u];
                    bs[u] = bs1[u];
                    lv[u] = lv1[u];
                    cand[u] = cand1[u];
                    bs1[u] = bs2[u];
                    lv1[u] = lv2[u];
                }
                l = l1;
                l1 = l2;
            }
            // write the block's picks and their Eq. 1 scores in one pass
            if (lane < nb) {
                const int rblk = r_s[buf][jb + lane];
                const int pick = WIDTH == 16 && cap_i == NONE ? -1 : cap_i;
                assign[rblk] = pick;
                if (chosen)
                    chosen[rblk] = pick >= 0 ? full_score(pair_s[buf][jb + lane][pick].base, cap_t,
                                                          cap_m, wl)
                                             : __builtin_nanf("");
            }
        }
        __syncthreads();   // buffer c & 1 may now be refilled; chunk c + 1 is ready
    }
#pragma unroll
    for (int u = 0; u < IPL; ++u) {
        const int i = inst(u);
        if (lane < (WIDTH == 16 ? 16 : WAVE) && i < I && valid[u]) {
            in.p[i] = p[u];
            in.a[i] = a[u];
        }
    }
}

// The same loop for more than 256 instances, which one wave would walk slot
// by slot (512 instances: 0.77 us a step, bound by instruction issue). The
// first CW waves hold SL slots of 64 instances each (instance wave*64*SL + 64*u
// + lane) and every step take the pick of their own, with what the others need
// to go on if it wins: its index, the next step's latency after the pick, and
// the maximum of the wave's other latencies then. After one barrier every wave
// reads all of them and finds the winner, so a step costs one exchange through
// LDS. The other eight waves are the producers: a group of GR steps is decided while
// the group after the next is made, a row of it (one request) per wave, cut
// into GR pieces so that the producers meet every step's barrier too. Their
// global loads run a group ahead (and the request's index two), so no barrier
// waits for one. (512 instances: 767 ns a step on one wave, 500 so; 1,000: 1,392
// and 938. Four waves of two slots: 607. The longest piece of a row sets the
// step: with all loads in the first piece 526, with a row's reciprocal taken
// once and an exact-remainder step per ratio 579.)
constexpr int WIDE_PRODUCERS = 8;

struct WidePick {
    int key, inst;      // key of the wave's pick (LEAST_KEY: none), its instance
    int t0;             // the next step's largest latency bits with the state as it stands
    float tn;           // the pick's, after the pick (0: not its candidate)
};
struct WideCap {
    float T, base;      // of the pick, for its score
};

template <int CW, int SL>
struct WideShared {
    static constexpr int IP = CW * WAVE * SL;   // instances
    static constexpr int GR = 4096 / IP;        // steps of a group
    static_assert(GR >= 4 && GR <= WIDE_PRODUCERS && GR % 2 == 0, "a row per producer");
    Pair pair[3][GR][IP];
    float l[3][GR];
    int r[3][GR];
    WidePick pick[2][CW];
    WideCap cap[2][CW];
};

template <int CW, int SL, bool DECIDED>
__global__ __launch_bounds__((CW + WIDE_PRODUCERS) * WAVE) void assign_wide_kernel(
    const float *__restrict__ q_hat, const float *__restrict__ l_hat,
    const int32_t *__restrict__ plen, int B, int M, const InstArgs in, int I, float wq, float wl,
    float wc, const AssignOpts opt, int32_t *__restrict__ assign, float *__restrict__ chosen,
    float *__restrict__ decided)
{
    using Sh = WideShared<CW, SL>;
    constexpr int GR = Sh::GR, NS = CW * SL;   // slots of 64 instances
    constexpr int PS = NS / (GR / 2);                  // slots per piece of a row
    extern __shared__ __align__(16) uint8_t wide_smem[];
    Sh &S = *(Sh *)wide_smem;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const auto imax = [](int x, int y) { return x > y ? x : y; };
    const auto fmx = [](float x, float y) { return fmaxf(x, y); };
    const int n_gr = (B + GR - 1) / GR;

    if (wave >= CW) {
        // ---- producers
        const int w = wave - CW;
        if (w >= GR) {
            for (int t = -2; t < B; ++t)
                stream_barrier();
            return;
        }
        int model[NS];
        float cin[NS], cout[NS];
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int i = u * WAVE + lane;
            const int m = i < I ? in.model[i] : -1;
            // -1: no candidate ever
            model[u] = (unsigned)m < (unsigned)M && (!opt.mask || opt.mask[i] != 0) ? m : -1;
            cin[u] = i < I ? in.cin[i] : 0.f;
            cout[u] = i < I ? in.cout[i] : 0.f;
        }
        struct Req {
            int r;
            float l, budget;
        };
        auto request = [&](int g) {   // this wave's request of group g
            const int t = g * GR + w;
            Req q{-1, 0.f, 0.f};
            if (t < B) {
                q.r = opt.order ? opt.order[t] : t;
                q.l = (float)plen[q.r];
                q.budget = opt.budget ? opt.budget[q.r] : INFINITY;
            }
            return q;
        };
        float qv[NS], lv[NS];
        auto labels = [&](const Req &q, float(&qx)[NS], float(&lx)[NS], int u0, int u1) {
            const size_t o = (size_t)(q.r < 0 ? 0 : q.r) * M;
#pragma unroll
            for (int u = u0; u < u1; ++u) {
                const int m = model[u] < 0 ? 0 : model[u];
                qx[u] = q_hat[o + m];
                lx[u] = l_hat[o + m];
            }
        };
        float cmax = 0.f;
        // piece k of the row of request q into group buffer g % 3: its costs
        // and their maximum first, then the base scores
        float C[NS];
        auto piece = [&](auto K, const Req &q, int g) {
            constexpr int k = decltype(K)::value;
            if constexpr (k == 0)
                cmax = -INFINITY;
            if constexpr (k < GR / 2) {
#pragma unroll
                for (int u = k * PS; u < (k + 1) * PS; ++u) {
                    C[u] = cost(q.l, lv[u], cin[u], cout[u]);
                    // Alg. 1 budget filter on the Eq. 2 cost, and availability
                    const bool cand = model[u] >= 0 && C[u] <= q.budget;
                    cmax = fmaxf(cmax, cand ? C[u] : -INFINITY);
                    C[u] = cand ? C[u] : __builtin_nanf("");
                }
            } else {
                if constexpr (k == GR / 2)
                    cmax = rows_reduce(row16_reduce(cmax, fmx), fmx);
                Pair *row = S.pair[g % 3][w];
#pragma unroll
                for (int u = (k - GR / 2) * PS; u < (k - GR / 2 + 1) * PS; ++u) {
                    Pair v;
                    v.base = base_score(qv[u], C[u], cmax, wq, wc);
                    if (C[u] != C[u])
                        v.base = __builtin_nanf("");
                    v.lv = model[u] >= 0 ? lv[u] : 0.f;
                    row[u * WAVE + lane] = v;
                }
                if constexpr (k == GR - 1) {
                    if (lane == 0) {
                        S.l[g % 3][w] = q.l;
                        S.r[g % 3][w] = q.r;
                    }
                }
            }
        };
        // groups 0 and 1 before the first step (sixteen slots both, always,
        // and each group after them: as a condition it costs them registers,
        // and 1,000 instances 1,160 ns a step for 935)
        for (int g = 0; g < (SL > 1 ? 2 : min(2, n_gr)); ++g) {
            const Req q = request(g);
            labels(q, qv, lv, 0, NS);
            static_for<0, GR>([&](auto K) { piece(K, q, g); });
        }
        Req q = request(2), qn = request(3);
        labels(q, qv, lv, 0, NS);
        stream_barrier();
        stream_barrier();   // (the deciding waves' first latencies)
        for (int g = 0; g < n_gr; ++g) {
            // (with every piece a share of the loads of the next group's row; all
            // with the first where sixteen slots leave no registers to spread them)
            float qx[NS], lx[NS];
            const Req qnn = request(g + 4);
            static_for<0, GR>([&](auto K) {
                constexpr int k = decltype(K)::value;
                if (g * GR + k < B) {
                    if (SL > 1 || g + 2 < n_gr) {
                        labels(qn, qx, lx, SL == 1 ? k * (NS / GR) : k == 0 ? 0 : NS,
                               SL == 1 ? (k + 1) * (NS / GR) : NS);
                        piece(K, q, g + 2);
                    }
                    stream_barrier();
                }
            });
            q = qn;
            qn = qnn;
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                qv[u] = qx[u];
                lv[u] = lx[u];
            }
        }
        return;
    }

    // ---- consumers: instance state in registers
    const int i0 = wave * WAVE * SL + lane;   // instance of slot u: i0 + 64*u
    float p[SL], a[SL], rP[SL], rD[SL];
    bool valid[SL];
#pragma unroll
    for (int u = 0; u < SL; ++u) {
        const int i = i0 + u * WAVE;
        const int m = i < I ? in.model[i] : -1;
        valid[u] = (unsigned)m < (unsigned)M;
        p[u] = valid[u] ? in.p[i] : 0.f;
        a[u] = valid[u] ? in.a[i] : 0.f;
        rP[u] = valid[u] ? 1.f / in.P[i] : 0.f;
        rD[u] = valid[u] ? 1.f / in.D[i] : 0.f;
    }
    auto wave_imax = [&](int v) { return rows_reduce(row16_reduce(v, imax), imax); };
    // over the waves' packets, one per lane of every CW
    static_assert(CW == 4 || CW == 8, "quads or half rows of lanes");
    auto imax_waves = [&](int v) {
        v = imax(v, dpp<0xb1>(v));
        v = imax(v, dpp<0x4e>(v));
        if constexpr (CW == 8)
            v = imax(v, dpp<0x141>(v));
        return v;
    };
    auto lane_of = [](float v, int src) {
        return __builtin_bit_cast(float,
                                  __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
    };
    constexpr int TINY = 0x00800000;   // as in the narrow loop
    // (the instance state is written at the very end only)
    int cap_i = -1, cap_r = 0;
    float cap_t = 0.f, cap_m = 0.f, cap_b = 0.f;
    float bs[SL], lv[SL], T[SL], l, bs1[SL], lv1[SL], l1;
    auto fetch = [&](int t, float(&bsx)[SL], float(&lvx)[SL], float &lx) {
        const int g = (unsigned)t / GR, k = t - g * GR, buf = g % 3;
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            const Pair v = S.pair[buf][k][i0 + u * WAVE];
            bsx[u] = v.base;
            lvx[u] = v.lv;
        }
        lx = S.l[buf][k];
    };
    stream_barrier();   // groups 0 and 1 are ready
    fetch(0, bs, lv, l);
    fetch(1, bs1, lv1, l1);
#pragma unroll
    for (int u = 0; u < SL; ++u)
        T[u] = latency(p[u], a[u], rP[u], rD[u], l, lv[u]);
    // the first step's largest latency, through the packets of step -1
    int tt = TINY;
#pragma unroll
    for (int u = 0; u < SL; ++u)
        tt = imax(tt, bs[u] == bs[u] ? __float_as_int(T[u]) : 0);
    tt = wave_imax(tt);
    if (lane == 0)
        S.pick[1][wave].t0 = tt;
    stream_barrier();
    float tmax = __int_as_float(imax_waves(S.pick[1][lane & (CW - 1)].t0));
    for (int t = 0; t < B; ++t) {
        float bs2[SL], lv2[SL], l2;   // the step after the next, in flight
        fetch(t + 2, bs2, lv2, l2);
        int key[SL], kb = LEAST_KEY;
        float p1[SL], a1[SL], T0[SL], T1[SL], tn[SL];
        int tz = 0;
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            const float v = fmaf(bs[u], tmax, wl * (tmax - T[u]));
            key[u] = bs[u] == bs[u] ? __float_as_int(v) : NO_KEY;
            kb = imax(kb, key[u]);
        }
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            p1[u] = p[u] + l;
            a1[u] = a[u] + lv[u];
            T0[u] = latency(p[u], a[u], rP[u], rD[u], l1, lv1[u]);
            T1[u] = latency(p1[u], a1[u], rP[u], rD[u], l1, lv1[u]);
            const bool c1 = bs1[u] == bs1[u];
            tz = imax(tz, c1 ? __float_as_int(T0[u]) : 0);
            tn[u] = c1 ? T1[u] : 0.f;
        }
        kb = wave_imax(kb);
        tz = wave_imax(tz);
        // the wave's lowest instance holding its maximum
        float tp = T[0], tx = tn[0], bp = bs[0];
        uint64_t mk = ballot(key[0] == kb);
        int us = 0;
#pragma unroll
        for (int u = 1; u < SL; ++u) {
            const uint64_t m2 = ballot(key[u] == kb);
            if (mk == 0) {
                mk = m2;
                us = u;
                tp = T[u];
                tx = tn[u];
                bp = bs[u];
            }
        }
        const bool none = kb == LEAST_KEY;
        const int src = none ? 0 : (int)__builtin_ctzll(mk);
        if (lane == src) {
            S.pick[t & 1][wave] =
                WidePick{kb, none ? -1 : i0 + us * WAVE, tz, none ? 0.f : tx};
            S.cap[t & 1][wave] = WideCap{tp, bp};
        }
        stream_barrier();
        const WidePick pk = S.pick[t & 1][lane & (CW - 1)];
        const int kmax = imax_waves(pk.key);
        const int tm = imax_waves(pk.t0);
        const int ws = (int)__builtin_ctzll(ballot(pk.key == kmax));   // (below CW)
        const int istar = __builtin_amdgcn_readlane(pk.inst, ws);
        const float tnext = lane_of(pk.tn, ws);
        if (wave == 0) {
            // capture the pick in lane t % 64
            const WideCap cp = S.cap[t & 1][ws];
            const int rt = S.r[(unsigned)t / GR % 3][t % GR];
            const bool mine = lane == (t & 63);
            cap_i = mine ? istar : cap_i;
            cap_r = mine ? rt : cap_r;
            cap_t = mine ? cp.T : cap_t;
            cap_b = mine ? cp.base : cap_b;
            cap_m = mine ? tmax : cap_m;
            if ((t & 63) == 63 || t == B - 1) {
                if (lane <= (t & 63)) {
                    assign[cap_r] = cap_i;
                    if (chosen)
                        chosen[cap_r] = cap_i >= 0 ? full_score(cap_b, cap_t, cap_m, wl)
                                                   : __builtin_nanf("");
                }
            }
        }
        if (DECIDED) {
            const int rq = S.r[(unsigned)t / GR % 3][t % GR];
            float *drow = decided + (size_t)rq * I;
#pragma unroll
            for (int u = 0; u < SL; ++u)
                if (i0 + u * WAVE < I)
                    drow[i0 + u * WAVE] = bs[u] == bs[u] ? full_score(bs[u], T[u], tmax, wl)
                                                         : __builtin_nanf("");
        }
        tmax = __int_as_float(imax(imax(tm, __float_as_int(tnext)), TINY));
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            const bool hit = i0 + u * WAVE == istar;
            p[u] = hit ? p1[u] : p[u];
            a[u] = hit ? a1[u] : a[u];
            T[u] = hit ? T1[u] : T0[u];
            bs[u] = bs1[u];
            lv[u] = lv1[u];
            bs1[u] = bs2[u];
            lv1[u] = lv2[u];
        }
        l = l1;
        l1 = l2;
    }
#pragma unroll
    for (int u = 0; u < SL; ++u) {
        const int i = i0 + u * WAVE;
        if (i < I && valid[u]) {
            in.p[i] = p[u];
            in.a[i] = a[u];
        }
    }
}

__global__ __launch_bounds__(256) void iota_kernel(int32_t *__restrict__ out, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        out[i] = i;
}

__global__ __launch_bounds__(256) void advance_kernel(const InstArgs in, int I, float dt)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= I)
        return;
    in.p[i] = fmaxf(0.f, in.p[i] - in.P[i] * dt);
    in.a[i] = fmaxf(0.f, in.a[i] - in.D[i] * dt);
}

}  // namespace

hipError_t launch_score(const float *q_hat, const float *l_hat, const int32_t *plen, int B, int M,
                        const InstArgs &in, int I, float wq, float wl, float wc,
                        const AssignOpts &opt, float *S0, hipStream_t s)
{
    hipLaunchKernelGGL(score_kernel, dim3((B + 3) / 4), dim3(256), 0, s, q_hat, l_hat, plen, B, M,
                       in, I, wq, wl, wc, opt, S0);
    return hipGetLastError();
}

hipError_t launch_lpt_order(const float *l_hat, int B, int M, int32_t *order, hipStream_t s)
{
    hipLaunchKernelGGL(lpt_order_kernel, dim3((B + LPT_RANK - 1) / LPT_RANK),
                       dim3(LPT_THREADS), 0, s, l_hat, B, M, order);
    return hipGetLastError();
}

hipError_t launch_assign(const float *q_hat, const float *l_hat, const int32_t *plen, int B,
                         int M, const InstArgs &in, int I, float wq, float wl, float wc,
                         const AssignOpts &opt, int32_t *assign, float *chosen, float *decided,
                         hipStream_t s)
{
#define RB_ASSIGN(KERN, THREADS, LDS)                                                            \
    hipLaunchKernelGGL((KERN), dim3(1), dim3(THREADS), LDS, s, q_hat, l_hat, plen, B, M, in, I,  \
                       wq, wl, wc, opt, assign, chosen, decided)
#define RB_NARROW(N, W)                                                                          \
    do {                                                                                         \
        if (decided)                                                                             \
            RB_ASSIGN((assign_kernel<N, W, true>), ASSIGN_THREADS, 0);                           \
        else                                                                                     \
            RB_ASSIGN((assign_kernel<N, W, false>), ASSIGN_THREADS, 0);                          \
    } while (0)
#define RB_WIDE(CW, SL)                                                                              \
    do {                                                                                         \
        const size_t lds = sizeof(WideShared<CW, SL>);                                           \
        const void *f = decided ? (const void *)assign_wide_kernel<CW, SL, true>                 \
                                : (const void *)assign_wide_kernel<CW, SL, false>;               \
        const hipError_t e = hipFuncSetAttribute(                                                \
            f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);                            \
        if (e != hipSuccess)                                                                     \
            return e;                                                                            \
        if (decided)                                                                             \
            RB_ASSIGN((assign_wide_kernel<CW, SL, true>), (CW + WIDE_PRODUCERS) * WAVE, lds);    \
        else                                                                                     \
            RB_ASSIGN((assign_wide_kernel<CW, SL, false>), (CW + WIDE_PRODUCERS) * WAVE, lds);   \
    } while (0)
    // one wave walks up to four slots of 64 instances faster than several
    // exchange theirs (256 instances: 398 against 523 ns a step; 512: 800
    // against 526)
    if (I <= 16)
        RB_NARROW(1, 16);
    else if (I <= WAVE)
        RB_NARROW(1, 64);
    else if (I <= 2 * WAVE)
        RB_NARROW(2, 64);
    else if (I <= 4 * WAVE)
        RB_NARROW(4, 64);
    else if (I <= 8 * WAVE)
        RB_WIDE(8, 1);
    else if (I <= 16 * WAVE)
        RB_WIDE(8, 2);
    else
        return hipErrorInvalidValue;
#undef RB_WIDE
#undef RB_NARROW
#undef RB_ASSIGN
    return hipGetLastError();
}

hipError_t launch_iota(int32_t *out, int n, hipStream_t s)
{
    hipLaunchKernelGGL(iota_kernel, dim3((n + 255) / 256), dim3(256), 0, s, out, n);
    return hipGetLastError();
}

hipError_t launch_advance(const InstArgs &in, int I, float dt, hipStream_t s)
{
    hipLaunchKernelGGL(advance_kernel, dim3((I + 255) / 256), dim3(256), 0, s, in, I, dt);
    return hipGetLastError();
}

}  // namespace rb
