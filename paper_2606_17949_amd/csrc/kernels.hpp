// Internal launch interface between the C ABI layer and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace rb {

constexpr size_t LDS_LIMIT = 160 * 1024;
constexpr int RB_MAX_K_DEV = 64;    // largest k (the ABI limit)
// The query-resident scan (bf16 rows of 384, 512, 768 or 1024 elements, a
// batch that fits its waves' registers): RQ_WAVES waves, blocks of RQ_ROWS
// bank rows, a ring of stages of a block's k-steps in LDS.
constexpr int RQ_WAVES = 8;
constexpr int RQ_ROWS = 32;
constexpr int RQ_EPS = 16;     // row tiles of a super tile
constexpr int RQ_SLOTS = 4;    // ring slots
// super tiles whose maxima wait in LDS, as many as fit beside the ring
__host__ __device__ constexpr int rq_hold(int qw, int rs) { return qw == 4 && rs == 1 ? 8 : 16; }
// stages of a block: whole blocks of 12 k-steps, else half blocks
constexpr int rq_spb(int nks) { return nks == 12 ? 1 : 2; }
constexpr int RQ_SMALL_B_MIN_ROWS = 2048;   // bank rows per compute unit, batches of <= 64
// The GEMM-structured scan (bf16 rows): GM_WAVES waves per workgroup, macro
// tiles of GM_ROWS bank rows by a tile of 128 or 256 requests, K in stages of
// GM_KST elements in GM_SLOTS LDS slots of up to GM_SLOT_LOADS loads.
constexpr int GM_WAVES = 8;
constexpr int GM_ROWS = 256;
constexpr int GM_KST = 64;
constexpr int GM_SLOTS = 2;
constexpr int GM_SLOT_LOADS = 64;
constexpr int GM_EPS = 16;     // entries of a macro tile
constexpr int GM_HOLD = 8;     // macro tiles whose maxima wait in LDS
enum GmOut { GM_ENTRIES, GM_FOLDED, GM_VALUES };   // what goes out beside the super tiles' maxima
// The LDS-resident scan: up to RES_WAVES waves per workgroup, each with
// RES_RING k-steps of bank loads in flight; request tiles of up to RES_MAX_NG
// groups of 16.
constexpr int RES_WAVES = 8;
constexpr int RES_RING = 8;
constexpr int RES_MAX_NG = 8;
constexpr int RES_HOLD = 16;   // super tiles whose maxima a wave holds
// The selection: one workgroup of SEL_THREADS threads per request (half of
// them for more than SEL_WIDE_B requests, a quarter for more than twice as
// many); up to SEL_CAP super tiles or rows held in LDS at once; SEL_ROUND row
// tiles recomputed per round.
constexpr int SEL_THREADS = 1024;
constexpr int SEL_WIDE_B = 256;
constexpr int SEL_CAP = 2048;
constexpr int SEL_ROUND = 64;
constexpr int SEL_MAX_EPS = 16;            // row tiles per super tile, at most
constexpr int SEL_MAX_ROW_BYTES = 8192;    // of one embedding (RB_MAX_D fp32)
constexpr long SEL_WANT_SUP = 16384;       // super tiles per request worth reading one by one
// bf16 batches of more than SEL_WIDE_B requests over at most this many rows
// (and 1,024 k, and 1,024 elements times it) go to the LDS-resident scan, which
// keeps their values.
constexpr int KEEP_ROWS = 8192;
// Bytes of maxima a call's workspace takes at most: a bank that would leave
// more goes by with folded entries, then in parts, each with its own scan and
// selection.
constexpr size_t MAXIMA_LIMIT = (size_t)1 << 30;
// Row tiles of one entry where the bank would otherwise go by in parts: the
// selection then computes up to FOLD times the row tiles again, and the maxima
// take 20 bytes for 68.
constexpr int FOLD = 4;

// Bytes of single values a scan keeps at most where storing them is not known
// to cost less than computing some again: then the selection takes 10 us
// for 19 (it computes no row tile again), while 26 MB of them made a scan of
// 64 x 100,000 take 55 us for 44.
constexpr size_t KEEP_LIMIT = (size_t)8 << 20;

// How one rb_knn_topk call is split.
//  * the bank in n_seg parts of seg_rows rows (one, unless the maxima would
//    pass the limit), each scanned and selected from by itself, the selection
//    under the k-th distance of the parts before;
//  * scan: the part in n_chunks row ranges, the requests in n_qt tiles, one
//    workgroup per (chunk, tile), `grid` of them; per request it leaves n_sup
//    super tiles of eps row tiles;
//  * selection: one workgroup per request.
struct KnnPlan {
    int kind;           // 0 LDS-resident scan, 1 query-resident scan, 2 GEMM-structured scan
    int dtype;          // 0 fp32, 1 bf16
    int B, N, d, k;
    int nks;            // 64-byte k-steps per row
    int ng;             // LDS-resident scan: groups of 16 requests per tile,
    int wg_waves;       //   waves per workgroup,
    bool keep_acc;      //   (and GEMM-structured scan) every row's value kept (at off_ent)
    int qw, rs;         // query-resident scan: query groups per wave, row halves; GEMM-structured
                        //   scan: 32-request tiles per wave (qw)
    int n_seg, n_qt, n_chunks, eps, grid;
    bool folded;        // an entry is of FOLD row tiles (not by the LDS-resident scan)
    long seg_rows, n_sup, rows_per_chunk, sup_per_chunk;
    size_t lds_bytes;
    size_t off_sup, off_ent, off_lkey, off_lidx, bytes;
    size_t contract, ordered;   // bytes of workspace a call asks for at least
};

// limit: bytes the maxima may take (they are cut to it by taking the bank in
// parts).
int plan_knn(int B, int N, int d, int dtype, int k, int num_cu, KnnPlan *p, int reserve = 0,
             size_t limit = MAXIMA_LIMIT);

// Events recorded around the bank-scan kernel when set (per host thread).
void set_scan_events(hipEvent_t begin, hipEvent_t end);

hipError_t launch_bank_norms(const void *bank, int dtype, int N, int d, float *norms,
                             hipStream_t s);
// The halves of launch_knn: the bank scan and the selection (which leave the
// neighbours in the workspace), and the outputs from those lists.
enum KnnPhases { KNN_LISTS = 1, KNN_MERGE = 2, KNN_ALL = 3 };
// With q_hat non-null, the second half also averages the labels (inv_dist: with
// inverse-distance weights instead of the plain mean).
hipError_t launch_knn(const KnnPlan &p, const void *queries, const void *bank,
                      const float *bank_norms, void *ws, int32_t *nbr_idx, float *nbr_dist,
                      const float *bank_qual, const float *bank_len, int M, float *q_hat,
                      float *l_hat, bool inv_dist, hipStream_t s, int phases = KNN_ALL);
hipError_t launch_predict(const int32_t *nbr_idx, const float *nbr_dist, int B, int k,
                          bool inv_dist, const float *bank_qual, const float *bank_len, int N,
                          int M, float *q_hat, float *l_hat, hipStream_t s);

struct InstArgs {
    const int32_t *model;
    float *p, *a;
    const float *P, *D, *cin, *cout;
};

// Options of the greedy loop; null pointers are the defaults (arrival order,
// no budgets, every instance available).
struct AssignOpts {
    const int32_t *order;    // [B] request decided at each step
    const float *budget;     // [B] per-request cost budget
    const uint8_t *mask;     // [I] nonzero = available
};

// The dense score matrix; opt's budget and mask restrict each row's
// candidates (its order is not read).
hipError_t launch_score(const float *q_hat, const float *l_hat, const int32_t *plen, int B, int M,
                        const InstArgs &in, int I, float wq, float wl, float wc,
                        const AssignOpts &opt, float *S0, hipStream_t s);

hipError_t launch_lpt_order(const float *l_hat, int B, int M, int32_t *order, hipStream_t s);
// out[i] = i for i < n (the arrival order, when the caller asks for it).
hipError_t launch_iota(int32_t *out, int n, hipStream_t s);
hipError_t launch_assign(const float *q_hat, const float *l_hat, const int32_t *plen, int B,
                         int M, const InstArgs &in, int I, float wq, float wl, float wc,
                         const AssignOpts &opt, int32_t *assign, float *chosen, float *decided,
                         hipStream_t s);
hipError_t launch_advance(const InstArgs &in, int I, float dt, hipStream_t s);

}  // namespace rb
