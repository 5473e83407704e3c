// Exact k-nearest-neighbour search over the labelled reference bank
// (RouteBalance Sec. 4.2: the KNN lookup of Alg. 1), for gfx950: bank norms,
// label averages, the plan of a search and its launches.
//
// Kernels of one search:
//   a scan         the bank once through MFMA; per request and row tile it
//                  leaves the largest <q, x> - |x|^2/2 (scan_rq.hpp,
//                  scan_gemm.hpp, scan_res.hpp)
//   select_kernel  per request: the k nearest rows from those maxima, sorted,
//                  then optionally the label gather and average (Sec. 4.2: one
//                  lookup predicts quality and length for every model)
// Order everywhere: distance ascending, equal distances by the lower bank
// index. Distances are |q|^2 + |x|^2 - 2<q,x> with fp32 products and
// accumulation; the scan accumulates -|x|^2/2 + <q,x>, and a distance is
// |q|^2 - 2*acc.
#include "knn_common.hpp"

namespace rb {

namespace {

// ------------------------------------------------------------------ norms

// Squared norms of rows, one wave per row, 16-byte lanes, fixed reduction tree.
template <int DT>
__global__ __launch_bounds__(256) void bank_norms_kernel(const uint8_t *__restrict__ bank, int N,
                                                         int d, float *__restrict__ norms)
{
    const int lane = lane_id();
    const long wave_g = ((long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const long n_waves = ((long)gridDim.x * blockDim.x) >> 6;
    const int row_bytes = d * Elem<DT>::ESZ;
    for (long n = wave_g; n < N; n += n_waves) {
        const uint8_t *row = bank + n * row_bytes;
        float s = 0.f;
        for (int off = lane * 16; off < row_bytes; off += WAVE * 16)
            s = sumsq16<DT>(load16(row + off), s);
        s = wave_sum(s);
        if (lane == 0)
            norms[n] = s;
    }
}

// One workgroup per request; nbr_dist is read only for the weighted average.
__global__ __launch_bounds__(64) void predict_kernel(const int32_t *__restrict__ nbr_idx,
                                                     const float *__restrict__ nbr_dist, int k,
                                                     const float *__restrict__ qual,
                                                     const float *__restrict__ len, int N, int M,
                                                     float *__restrict__ q_hat,
                                                     float *__restrict__ l_hat)
{
    __shared__ int32_t nbr[RB_MAX_K_DEV];
    __shared__ float wts[RB_MAX_K_DEV];
    const int b = blockIdx.x;
    for (int j = threadIdx.x; j < k; j += blockDim.x) {
        nbr[j] = nbr_idx[(size_t)b * k + j];
        if (nbr_dist)
            wts[j] = inv_dist_weight(nbr_dist[(size_t)b * k + j]);
    }
    __syncthreads();
    for (int m = threadIdx.x; m < M; m += blockDim.x)
        average_labels(nbr, nbr_dist ? wts : nullptr, k, qual, len, N, M, m,
                       q_hat + (size_t)b * M + m, l_hat + (size_t)b * M + m);
}

// ------------------------------------------------------------------ host side

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

thread_local hipEvent_t t_scan_begin = nullptr, t_scan_end = nullptr;

// The least workspace a call of these sizes asks for. rb_workspace_size is
// what decides which sizes rb_route_batch_noalloc takes (those whose
// workspace fits its static array), so the figure stays where callers found
// it when the scans kept candidate lists: a request's bounds and lists over
// the chunks of the scan that took it, and the overflow of its candidates. 0:
// refused (more lists than the merge took: banks of over 2 TB).
size_t contract_bytes(int B, int N, int d, int dtype, int k, int num_cu, int reserve)
{
    const int vec = dtype == 1 ? 8 : 4;
    const int nks = (d + 4 * vec - 1) / (4 * vec);
    const bool ragged = d % (4 * vec) != 0;
    // query-resident: {query groups per wave, row halves, fewest ring bytes}
    int rs = 0;
    if (dtype == 1 && !ragged && B >= 1 &&
        (B > 64 || (long)N >= (long)RQ_SMALL_B_MIN_ROWS * num_cu)) {
        static const int tab[][4] = {{12, 1, 2, 0}, {12, 2, 2, 0}, {12, 4, 2, 0}, {12, 4, 1, 0},
                                     {16, 1, 2, 0}, {16, 2, 2, 0}, {16, 2, 1, 0}, {24, 1, 2, 0},
                                     {24, 2, 2, 0}, {24, 2, 1, 0}, {32, 1, 2, 0}, {32, 1, 1, 0}};
        for (const auto &t : tab) {
            if (t[0] != nks || 8 / t[2] * t[1] * 16 < B)
                continue;
            // (two slots of half blocks, of whole ones for 12 k-steps)
            const long kstg = nks == 12 ? 12 : nks / 2;
            const long lds = 2 * kstg * 2048 + 2 * 256 + 8L * t[1] * 16 * (k + 1) * 8;
            if (lds <= (long)LDS_LIMIT) {
                rs = t[2];
                break;
            }
        }
    }
    const bool gemm = dtype == 1 && B > 256 && rs == 0 && d % 64 == 0 && d >= 128 &&
                      131072L + 2048 + 256L * k * 8 + 4096 + 6144 <= (long)LDS_LIMIT;
    int ng = 1;
    while (ng < 16 && ng * 16 < B)
        ng *= 2;
    for (; ng > 1; ng /= 2) {
        const int slots = ng < 16 || (dtype == 1 && !ragged) ? 4 : 2;
        if ((slots * ng + 1) * 1024L + 16L * ng * (k * 8 + 16) + 2048 + 12288 <= (long)LDS_LIMIT)
            break;
    }
    const int n_qt = rs ? 1 : gemm ? (B + 255) / 256 : B > 0 ? (B + 16 * ng - 1) / (16 * ng) : 1;
    long chunks = num_cu / n_qt;
    if (reserve > 0) {
        const long per_xcd = (num_cu / 8 - reserve) / n_qt;
        if (per_xcd >= 1)
            chunks = per_xcd * 8;
        if (gemm)
            chunks = (num_cu - 8L * reserve) / n_qt;
    }
    if (chunks < 1)
        chunks = 1;
    if (chunks > ((long)N + 15) / 16)
        chunks = ((long)N + 15) / 16;
    const long rowb = (long)d * (dtype == 1 ? 2 : 4);
    long rpc = ((long)N + chunks - 1) / chunks;
    rpc = (rpc + 15) / 16 * 16;
    while (rpc * rowb >= (1L << 31) - (1L << 20)) {
        chunks *= 2;
        rpc = ((long)N + chunks - 1) / chunks;
        rpc = (rpc + 15) / 16 * 16;
    }
    const long n_chunks = ((long)N + rpc - 1) / rpc;
    long S = N / 32 < 2048 ? 2048 : N / 32 > 32768 ? 32768 : N / 32;
    S = (S > N ? N : S) / 64 * 64;
    const long G = S / 16 < k ? 0 : S / 16;
    const bool two = rs && B > 128 && (long)N / 32 > 32768 && rpc >= 1024;
    const size_t W = (size_t)n_chunks * (rs ? rs : 1) * (two ? 2 : 1), b = (size_t)B;
    if (W > 4096)
        return 0;
    const long pairs = 512L * ng;
    const size_t cap = rs ? 1 : gemm ? 64 * 128 - 64 : pairs > 128 ? pairs - 128 : 1;
    const size_t wgs = rs ? n_chunks : (n_chunks + 7) / 8 * 8 * n_qt;
    return 2 * align256(b * 4) + align256(b * (G > 0 ? G : 1) * 4) + align256(b * W * 4) +
           2 * align256(b * W * k * 4) + align256(wgs * 8 * 3 * cap * 4);
}

// The (query groups per wave, row halves) of the query-resident scan for B
// requests of nks k-steps: the first, in order of capacity, that holds them (a
// wave holds qw * nks * 4 registers of query fragments, at most 192).
bool rq_shape(int nks, int B, int *qw, int *rs)
{
    static const int tab[][3] = {{12, 1, 2}, {12, 2, 2}, {12, 4, 2}, {12, 4, 1},
                                 {16, 1, 2}, {16, 2, 2}, {16, 2, 1}, {24, 1, 2},
                                 {24, 2, 2}, {24, 2, 1}, {32, 1, 2}, {32, 1, 1}};
    for (const auto &t : tab) {
        if (t[0] == nks && RQ_WAVES / t[2] * t[1] * 16 >= B) {
            *qw = t[1];
            *rs = t[2];
            return true;
        }
    }
    return false;
}

// Entries of a super tile.
int entries_of(const KnnPlan &p) { return p.folded ? p.eps / FOLD : p.eps; }

// The bank in equal parts of whole super tiles whose maxima stay within
// `limit` bytes (fixed: those of the workspace's other sections): one, of
// whole or else of folded entries, if that can be, else as few as folded
// entries allow (512 x 4,000,000 x 384 within 64 MB: 1,538 us in ten parts,
// 1,404 in three of folded entries, 1,265 in one within 553 MB).
void plan_parts(KnnPlan *p, size_t limit)
{
    const size_t b = p->B > 0 ? p->B : 1;
    const size_t fixed = 2 * align256(b * p->k * 4) + 4 * 256;
    const size_t per_sup = b * 4 * (p->eps > 1 ? 1 + entries_of(*p) : 1);
    const long rows = (long)p->eps * 16;
    const long all = ((long)p->N + rows - 1) / rows;
    // (every chunk of the other scans may end in a partial super tile)
    const long spare = p->kind == 0 ? 0 : p->n_chunks;
    long fit = limit > fixed ? (long)((limit - fixed) / per_sup) - spare : 0;
    if (fit < 1)
        fit = 1;
    if (all > fit && p->kind != 0 && !p->folded) {
        p->folded = true;
        plan_parts(p, limit);
        return;
    }
    p->n_seg = (int)((all + fit - 1) / fit);
    p->seg_rows = (all + p->n_seg - 1) / p->n_seg * rows;
}

// Super tiles up to SEL_WANT_SUP per request: row tiles of one of the
// LDS-resident scan's.
int res_eps(int N)
{
    const long all_tiles = ((long)N + 15) / 16;
    int eps = 1;
    while (eps < SEL_MAX_EPS && all_tiles > SEL_WANT_SUP * eps)
        eps *= 2;
    return eps;
}

// Bytes of single values the LDS-resident scan keeps at most. Else the
// selection computes k row tiles again for every request by itself, a
// sixteenth of each MFMA's columns used: fp32 batches keep them, as far as the
// workspace may, where that is more work than a sixteenth of the scan's
// (2,022 x 2,312 x 512, 64 neighbours: 529 us computed again, 102 kept; 1,000 x
// 48,000 x 384, 10 neighbours: 354 and 332). bf16 scans, sixteen times as fast,
// lose more to the stores over all but small banks.
size_t keep_limit(int dtype, int N, int d, int k)
{
    const bool keep = dtype == 0 ? (long)N <= 16L * k * d : N <= KEEP_ROWS;
    return keep ? MAXIMA_LIMIT : KEEP_LIMIT;
}

// Whether the GEMM-structured scan keeps every row's value, as far as the
// workspace may: 4 bytes stored a row and request where the selection would
// read 32 k d of the bank again for each (computed again / kept: 1,024 x 12,000
// x 2,048 160 / 96 us, with 32 neighbours 329 / 121, 1,024 x 12,000 x 1,000 85 /
// 74, 1,024 x 16,000 x 1,024 88 / 87; past the line 1,024 x 16,000 x 640 61 / 77).
bool gemm_keeps(int N, int d, int k) { return 2L * N <= 3L * k * d; }

// bf16 batches of more than SEL_WIDE_B requests over a small bank, whose
// selections take longer than the scan if they compute row tiles again.
bool keeps_small_bank(int B, int N, int d, int k)
{
    return B > SEL_WIDE_B && N <= KEEP_ROWS && (long)N <= 1024L * k &&
           (long)N * d <= KEEP_ROWS * 1024L;
}

// Bytes of the LDS-resident scan's layout over a bank of single row tiles, every
// row's value kept.
size_t res_bytes(int B, int N, int k)
{
    const size_t b = B, tiles = ((size_t)N + 15) / 16;
    return 2 * align256(b * k * 4) + align256(b * tiles * 4) + align256(b * tiles * 64);
}

// Chunks for n_qt request tiles: one workgroup per compute unit (the LDS use
// allows no more). With `reserve`, that many units of each XCD stay free. The
// tiles of a chunk share an XCD but for those of the last n_chunks % 8 chunks,
// which are spread over neighbouring XCDs (chunk_and_tile), so that no XCD gets
// more workgroups than it has units (measured at B = 1,024, d = 1,024: 248
// workgroups 1,821 us per launch against 1,942 us for 224, the most whole
// chunks).
long plan_chunks(const KnnPlan *p, int num_cu, int reserve)
{
    const long chunks = (num_cu - 8L * reserve) / p->n_qt;
    return chunks < 1 ? 1 : chunks;
}

// Groups of 16 requests that fit LDS for every k-step of the LDS-resident
// scan, beside the norms of every wave's tiles; at most RES_MAX_NG.
constexpr size_t RES_NORM_BYTES = RES_WAVES * 2 * 256 * sizeof(float);
int res_groups(int nks)
{
    const int ng = (int)((LDS_LIMIT - RES_NORM_BYTES) / ((size_t)nks * WAVE * 16));
    return ng < RES_MAX_NG ? ng : RES_MAX_NG;
}

// The LDS-resident scan. Request tiles: as many groups of 16 requests as fit
// (res_groups), evenly over the tiles. Waves:
// eight per workgroup, fewer when there are not enough super tiles to go
// round (a bank of 2,048 rows is 128 row tiles: one wave on each of 128
// compute units).
void plan_res(KnnPlan *p, int num_cu, int reserve, size_t limit)
{
    const int B = p->B;
    const long rowb = (long)p->d * (p->dtype == 1 ? 2 : 4);
    const int groups = B > 0 ? (B + 15) / 16 : 1;
    const int ng = res_groups(p->nks);
    p->n_qt = (groups + ng - 1) / ng;
    p->ng = (groups + p->n_qt - 1) / p->n_qt;
    p->lds_bytes = (size_t)p->nks * p->ng * WAVE * 16 + RES_NORM_BYTES;
    p->eps = res_eps(p->N);
    plan_parts(p, limit);
    p->n_sup = p->seg_rows / (p->eps * 16);
    long chunks = plan_chunks(p, num_cu, reserve);
    long waves = (p->n_sup + chunks - 1) / chunks;
    if (waves > RES_WAVES)
        waves = RES_WAVES;
    p->wg_waves = (int)waves;
    if (chunks > (p->n_sup + waves - 1) / waves)
        chunks = (p->n_sup + waves - 1) / waves;
    // a wave's share is addressed with 32-bit offsets
    while ((p->n_sup / (chunks * waves) + 1) * p->eps * 16 * rowb >= (1L << 31) - (1L << 20))
        chunks *= 2;
    p->n_chunks = (int)chunks;
    p->grid = ((p->n_chunks + 7) / 8) * 8 * p->n_qt;
    p->rows_per_chunk = p->seg_rows;   // (its super tiles follow one another over all rows)
    p->sup_per_chunk = p->n_sup;
}

// The query-resident and the GEMM-structured scan: chunks of contiguous rows,
// whole 16-row tiles, each with super tiles of its own.
void plan_chunked(KnnPlan *p, int num_cu, int reserve, size_t limit)
{
    const long rowb = (long)p->d * 2;
    p->eps = p->kind == 1 ? RQ_EPS : GM_EPS;
    long chunks = plan_chunks(p, num_cu, reserve), most = chunks;
    while ((p->N / most + 32) * rowb >= (1L << 31) - (1L << 20))   // (as below)
        most *= 2;
    p->n_chunks = (int)most;
    plan_parts(p, limit);
    const long rows = p->seg_rows < p->N ? p->seg_rows : p->N;
    if (chunks > (rows + 15) / 16)
        chunks = (rows + 15) / 16;
    long rpc = ((rows + chunks - 1) / chunks + 15) / 16 * 16;
    while (rpc * rowb >= (1L << 31) - (1L << 20)) {   // 32-bit offsets
        chunks *= 2;
        rpc = ((rows + chunks - 1) / chunks + 15) / 16 * 16;
    }
    p->rows_per_chunk = rpc;
    p->n_chunks = (int)((rows + rpc - 1) / rpc);
    p->sup_per_chunk = (rpc + p->eps * 16 - 1) / (p->eps * 16);
    p->n_sup = p->n_chunks * p->sup_per_chunk;
    p->grid = p->kind == 1 ? p->n_chunks : ((p->n_chunks + 7) / 8) * 8 * p->n_qt;
}

// What the layout of any batch of up to B requests takes at most, whatever scan
// and how many parts it goes by. It is asked for, so that a workspace sized
// for a program's largest batch holds the smaller ones too (folded entries and
// parts make the layouts themselves go up and down with B: 1,006 requests over
// 4,000,000 x 384 take 1,073 MB, 1,024 of them 321).
size_t ordered_bytes(int B, int N, int d, int dtype, int k, int num_cu)
{
    const size_t b = B > 0 ? B : 1;
    const long rowb = (long)d * (dtype == 1 ? 2 : 4);
    // LDS-resident scan: bf16 batches of at most 64, or over a small bank
    const size_t b0 = dtype == 1 && b > 64 && !keeps_small_bank(B, N, d, k) ? 64 : b;
    const size_t eps = res_eps(N), n0 = ((size_t)N + 16 * eps - 1) / (16 * eps);
    const size_t all = b0 * n0 * eps * 64, kl = keep_limit(dtype, N, d, k);
    const size_t keep = all < kl ? all : kl;
    size_t ent = eps > 1 ? b0 * n0 * eps * 4 : 0;
    ent = ent > keep ? ent : keep;
    const size_t res = b0 * n0 * 4 + ent;
    // the others: every chunk may end in a partial super tile, and its rows
    // are rounded up to a whole tile
    size_t chunked = 0;
    if (dtype == 1 && (b > 32 || (long)N >= (long)GM_ROWS * num_cu)) {
        size_t chunks = (size_t)num_cu, split = 2 * (size_t)((long)N * rowb >> 30) + 2;
        chunks = chunks > split ? chunks : split;
        const size_t n12 = (size_t)N / (RQ_EPS * 16) + chunks + chunks / 16 + 2;
        chunked = b * n12 * 4 * (1 + RQ_EPS);
        const size_t values = b * n12 * 4 + b * (((size_t)N + 15) / 16) * 64;
        if (gemm_keeps(N, d, k) && values > chunked)
            chunked = values;
    }
    static_assert(RQ_EPS == GM_EPS, "one size of super tile");
    size_t maxima = res > chunked ? res : chunked;
    // (a part takes at least one super tile)
    const size_t most = MAXIMA_LIMIT > b * 4 * (1 + RQ_EPS) ? MAXIMA_LIMIT : b * 4 * (1 + RQ_EPS);
    maxima = maxima < most ? maxima : most;
    return 2 * align256(b * k * 4) + maxima + 3 * 256;
}

}  // namespace

void set_scan_events(hipEvent_t begin, hipEvent_t end)
{
    t_scan_begin = begin;
    t_scan_end = end;
}

int plan_knn(int B, int N, int d, int dtype, int k, int num_cu, KnnPlan *p, int reserve,
             size_t limit)
{
    const int vec = dtype == 1 ? 8 : 4;
    const long rowb = (long)d * (dtype == 1 ? 2 : 4);
    if ((long)B * rowb >= (1L << 31))
        return -1;   // the query resource is addressed with 32-bit offsets
    *p = KnnPlan{};
    p->dtype = dtype;
    p->B = B;
    p->N = N;
    p->d = d;
    p->k = k;
    p->nks = (d + 4 * vec - 1) / (4 * vec);
    p->contract = contract_bytes(B, N, d, dtype, k, num_cu, reserve);
    // (a lower limit is one workspace's, not a size that is asked for)
    p->ordered = limit == MAXIMA_LIMIT ? ordered_bytes(B, N, d, dtype, k, num_cu) : 0;
    if (p->contract == 0)
        return -1;
    // bf16 rows of 384, 512, 768 or 1,024 elements go to the query-resident
    // scan when the batch fits one workgroup's registers; a batch of at most
    // 64 requests only over a bank of at least RQ_SMALL_B_MIN_ROWS rows per
    // compute unit (below, its start, every wave loading its queries, costs
    // more than that of the LDS-resident scan). Other bf16 batches of more
    // than 64 requests go to the GEMM-structured scan, in tiles of 128
    // requests if one tile holds them, else of 256; so do smaller ones that do
    // not fit LDS as one tile (33 to 64 requests of 1,536 or 2,048 elements:
    // the LDS-resident scan reads the bank for two), over at least a macro
    // tile of rows per compute unit (64 requests, 1,536 elements: 490 us for
    // 577 over 700,000 rows, 61 for 64 over 48,001, but 57 for 40 over 32,001).
    // Everything else, all fp32 batches among it, goes to the LDS-resident scan,
    // and so does a large bf16 batch over a small bank, if the workspace can
    // keep its values (10 neighbours: 2,000 x 3,000 x 768 73 us by the
    // GEMM-structured scan, 54 so, 600 x 8,000 x 1,024 54 and 42; but 1,024 x
    // 8,000 x 2,048 86 and 135, and one neighbour, 1,024 x 8,000 x 768, 38 and 41).
    const bool rq_rows = B > 64 || (long)N >= (long)RQ_SMALL_B_MIN_ROWS * num_cu;
    if (dtype == 1 && d % (4 * vec) == 0 && rq_rows && rq_shape(p->nks, B, &p->qw, &p->rs)) {
        p->kind = 1;
        p->n_qt = 1;
        p->lds_bytes =
            rq_layout(p->qw, p->rs, p->nks / rq_spb(p->nks), RQ_SLOTS).bytes;
        plan_chunked(p, num_cu, reserve, limit);
    } else if (dtype == 1 && !(keeps_small_bank(B, N, d, k) && res_bytes(B, N, k) <= limit) &&
               (B > 64 || ((B + 15) / 16 > res_groups(p->nks) &&
                           (long)N >= (long)GM_ROWS * num_cu))) {
        p->kind = 2;
        p->qw = B > 128 ? 4 : 2;
        p->n_qt = (B + 64 * p->qw - 1) / (64 * p->qw);
        p->lds_bytes = gemm_layout(p->qw).bytes;
        plan_chunked(p, num_cu, reserve, limit);
    } else {
        p->kind = 0;
        plan_res(p, num_cu, reserve, limit);
    }
    const size_t b = (size_t)B;
    size_t off = 0;
    p->off_lkey = off;
    off += align256(b * k * 4);
    p->off_lidx = off;
    off += align256(b * k * 4);
    p->off_sup = off;
    off += align256(b * p->n_sup * 4);
    p->off_ent = off;
    const size_t keep = align256(b * (((size_t)N + 15) / 16) * 64);
    p->keep_acc = p->kind != 1 && p->n_seg == 1 && off + keep <= limit &&
                  keep <= (p->kind == 0 ? keep_limit(dtype, N, d, k)
                           : gemm_keeps(N, d, k) ? MAXIMA_LIMIT
                                                 : 0);
    off += p->keep_acc ? keep : p->eps > 1 ? align256(b * p->n_sup * entries_of(*p) * 4) : 0;
    p->bytes = off;
    return 0;
}

hipError_t launch_bank_norms(const void *bank, int dtype, int N, int d, float *norms,
                             hipStream_t s)
{
    long waves = N;
    int grid = (int)((waves + 3) / 4);
    if (grid > 65536)
        grid = 65536;
    if (dtype == 1)
        hipLaunchKernelGGL(bank_norms_kernel<1>, dim3(grid), dim3(256), 0, s,
                           (const uint8_t *)bank, N, d, norms);
    else
        hipLaunchKernelGGL(bank_norms_kernel<0>, dim3(grid), dim3(256), 0, s,
                           (const uint8_t *)bank, N, d, norms);
    return hipGetLastError();
}

hipError_t launch_knn(const KnnPlan &p, const void *queries, const void *bank,
                      const float *bank_norms, void *ws, int32_t *nbr_idx, float *nbr_dist,
                      const float *bank_qual, const float *bank_len, int M, float *q_hat,
                      float *l_hat, bool inv_dist, hipStream_t s, int phases)
{
    uint8_t *w = (uint8_t *)ws;
    hipError_t e;
    SelectArgs sa{};
    sa.queries = (const uint8_t *)queries;
    sa.bank = (const uint8_t *)bank;
    sa.bank_norms = bank_norms;
    sa.B = p.B;
    sa.d = p.d;
    sa.nks = p.nks;
    sa.k = p.k;
    sa.eps = p.eps;
    sa.n_sup = p.n_sup;
    sa.rows_per_chunk = p.rows_per_chunk;
    sa.sup_per_chunk = p.sup_per_chunk;
    sa.split_tiles = p.kind == 2;
    sa.m.sup = (float *)(w + p.off_sup);
    sa.m.ent = (float *)(w + p.off_ent);
    // super tiles request by request; the entries super tile by super tile, as
    // the scans write them
    sa.m.sup_q = p.n_sup;
    sa.m.ent_q = entries_of(p);
    sa.m.ent_s = p.B * sa.m.ent_q;
    sa.m.folded = p.folded;
    sa.acc = p.keep_acc ? sa.m.ent : nullptr;
    sa.list_key = (uint32_t *)(w + p.off_lkey);
    sa.list_idx = (int32_t *)(w + p.off_lidx);
    sa.qual = bank_qual;
    sa.len = bank_len;
    sa.N = p.N;
    sa.M = M;
    sa.inv_dist = inv_dist;
    if (!(phases & KNN_LISTS)) {
        sa.nbr_idx = nbr_idx;
        sa.nbr_dist = nbr_dist;
        sa.q_hat = q_hat;
        sa.l_hat = l_hat;
        return launch_from_list(sa, s);
    }
    ScanArgs a{};
    a.queries = sa.queries;
    a.bank = sa.bank;
    a.bank_norms = bank_norms;
    a.B = p.B;
    a.d = p.d;
    a.nks = p.kind != 2 ? p.nks : p.d > GM_KST ? (p.d + GM_KST - 1) / GM_KST : 2;
    a.n_chunks = p.n_chunks;
    a.n_qt = p.n_qt;
    a.eps = p.eps;
    a.n_sup = p.n_sup;
    a.rows_per_chunk = p.rows_per_chunk;
    a.sup_per_chunk = p.sup_per_chunk;
    a.m = sa.m;
    a.acc = p.keep_acc ? a.m.ent : nullptr;
    const bool timed = t_scan_begin && t_scan_end;
    for (int seg = 0; seg < p.n_seg; ++seg) {
        const bool last = seg == p.n_seg - 1;
        a.row0 = seg * p.seg_rows;
        a.rows = last ? p.N - a.row0 : p.seg_rows;
        if (p.kind == 0) {
            a.n_tiles = (a.rows + 15) / 16;
            a.n_sup = (a.n_tiles + p.eps - 1) / p.eps;
            a.m.sup_q = sa.m.sup_q = a.n_sup;
        }
        if (timed && seg == 0 && (e = hipEventRecord(t_scan_begin, s)) != hipSuccess)
            return e;
        e = p.kind == 2   ? launch_scan_gemm(p, a, s)
            : p.kind == 1 ? launch_scan_rq(p, a, s)
            : p.dtype == 1 ? launch_scan_res_bf16(p, a, s)
                           : launch_scan_res_f32(p, a, s);
        if (e != hipSuccess)
            return e;
        if (timed && last && (e = hipEventRecord(t_scan_end, s)) != hipSuccess)
            return e;
        sa.row0 = a.row0;
        sa.rows = a.rows;
        sa.n_sup = a.n_sup;
        sa.carry_in = seg > 0;
        const bool out = last && (phases & KNN_MERGE) != 0;
        sa.nbr_idx = out ? nbr_idx : nullptr;
        sa.nbr_dist = out ? nbr_dist : nullptr;
        sa.q_hat = out ? q_hat : nullptr;
        sa.l_hat = out ? l_hat : nullptr;
        if ((e = launch_select(p.dtype, sa, s)) != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t launch_predict(const int32_t *nbr_idx, const float *nbr_dist, int B, int k,
                          bool inv_dist, const float *bank_qual, const float *bank_len, int N,
                          int M, float *q_hat, float *l_hat, hipStream_t s)
{
    hipLaunchKernelGGL(predict_kernel, dim3(B), dim3(64), 0, s, nbr_idx,
                       inv_dist ? nbr_dist : nullptr, k, bank_qual, bank_len, N, M, q_hat, l_hat);
    return hipGetLastError();
}

}  // namespace rb
