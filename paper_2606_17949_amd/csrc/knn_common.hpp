// Helpers and argument blocks shared by the k-NN kernels (gfx950, wave64).
#pragma once

#include <float.h>

#include "common.hpp"
#include "kernels.hpp"

namespace rb {

// Every scan writes, per request and 16-row tile of the bank, the largest
// <q, x> - |x|^2/2 of the tile's rows (the nearest row's distance is |q|^2 - 2
// times that), and the maximum over every eps such entries (a super tile, of
// eps * 16 consecutive rows). The rows go by in chunks, each with super tiles
// of its own; entries and super tiles without a row hold NaN. The entries of
// FOLD consecutive row tiles go out as one where the plan says so.
struct Maxima {
    float *sup;          // of request q: super tile s at s + q*sup_q
    float *ent;          // its entry e at s*ent_s + e + q*ent_q (unused when eps is 1 or when
    long sup_q;          //   every row's value is kept)
    long ent_s, ent_q;
    bool folded;         // an entry is of FOLD row tiles
};

struct ScanArgs {
    const uint8_t *queries, *bank;
    const float *bank_norms;
    int B, d, nks, n_chunks, n_qt;   // nks: k-steps of a row (GEMM scan: stages)
    long row0, rows;      // bank rows [row0, row0 + rows) of this launch
    long n_tiles, n_sup;  // their 16-row tiles (LDS-resident scan); super tiles per request
    int eps;
    long rows_per_chunk, sup_per_chunk;   // (LDS-resident scan: one chunk of all rows)
    Maxima m;
    float *acc;           // [row tiles][B][16] every row's <q, x> - |x|^2/2, or null
};

// The selection from those maxima.
struct SelectArgs {
    const uint8_t *queries, *bank;
    const float *bank_norms;
    int B, d, nks, k, eps;
    long row0, rows, n_sup, rows_per_chunk, sup_per_chunk;
    Maxima m;
    const float *acc;     // as ScanArgs has it
    uint32_t *list_key;   // [B][k] neighbours as distance keys and indices, in and out
    int32_t *list_idx;    //   (null: not kept)
    bool split_tiles;     // entries 2t and 2t + 1 of a super tile are rows 0-3, 8-11, 16-19,
                          // 24-27 and the others of its 32-row tile t
    bool carry_in;        // the lists hold the neighbours of earlier parts of the bank
    int32_t *nbr_idx;     // results, null in all but the last part
    float *nbr_dist;
    const float *qual, *len;
    int N, M;
    float *q_hat, *l_hat;
    bool inv_dist;
};

hipError_t launch_select(int dtype, const SelectArgs &a, hipStream_t s);
hipError_t launch_from_list(const SelectArgs &a, hipStream_t s);

// Floats between two entries of the maxima staged in LDS (entry by entry,
// n_req requests each, a multiple of 32): a wave writes one entry of
// consecutive requests and reads back four entries of 16 requests in four lane
// groups, 4 * pitch = 16 (mod 64) apart, both over distinct banks. (Request by
// request, 16 entries each, a write took sixteen lanes to one bank: 61 M
// conflict cycles a launch of 512 x 4,000,000 x 384, 31 M of 1,024 x 1,000,000
// x 1,024, 3.9 M of 256 x 1,000,000 x 768; so 9.1 M, 2.5 M and 1.4 M.)
__host__ __device__ constexpr int stage_pitch(int n_req) { return (n_req + 63) / 64 * 64 + 4; }

// Byte offsets of the query-resident scan's LDS regions.
struct RqLayout {
    uint32_t ring, norms, stage, sup, bytes;
};

__host__ __device__ inline RqLayout rq_layout(int qw, int rs, int kstg, int stages)
{
    RqLayout L;
    uint32_t o = 0;
    L.ring = o;    // [stages][kstg * RQ_ROWS / 16][64] bank fragments
    o += (uint32_t)stages * kstg * (RQ_ROWS / 16) * WAVE * 16;
    L.norms = o;   // [stages][64] |x|^2 of the rows of a block (with its first stage)
    o += (uint32_t)stages * WAVE * 4;
    L.stage = o;   // [rs][RQ_EPS][stage_pitch(RQ_WAVES / rs * 16 * qw)] maxima of a super
    // tile (two buffers where two waves share a request)
    o += (uint32_t)rs * RQ_EPS * stage_pitch(RQ_WAVES / rs * 16 * qw) * 4;
    L.sup = o;     // [RQ_WAVES / rs * 16 * qw][rq_hold] maxima of the last super tiles
    o += (uint32_t)RQ_WAVES / rs * qw * 16 * rq_hold(qw, rs) * 4;
    L.bytes = o;
    return L;
}

// Workgroup -> (chunk c, request tile t) of a scan with request tiles (c =
// n_chunks: nothing to do): workgroups go to the eight XCDs round robin, so
// every request tile of one of the first 8 * (n_chunks / 8) chunks lands on one
// XCD, where a bank line fetched for one is an L2 hit for the others. The last
// n_chunks % 8 chunks take the remaining workgroups in order of XCD (x) and
// then of dispatch (s): rank L among them, chunk base + L / n_qt, tile L % n_qt,
// so that a chunk's tiles sit on as few XCDs as the counts allow, and no XCD
// gets more workgroups than its share of them (three tiles of 85 chunks, whole
// chunks to an XCD, left five XCDs of 32 units with 33: one more round of the
// whole scan).
__device__ __forceinline__ void chunk_and_tile(int n_chunks, int n_qt, int *c, int *t)
{
    const int per8 = 8 * n_qt;
    const int full = (n_chunks / 8) * per8;
    if ((int)blockIdx.x < full) {
        const int rem = blockIdx.x % per8;
        *t = rem / 8;
        *c = (blockIdx.x / per8) * 8 + rem % 8;
    } else {
        const int j = blockIdx.x - full, x = j % 8, s = j / 8;
        const int tail = (n_chunks % 8) * n_qt, q = tail / 8, r = tail % 8;
        const int L = x * q + min(x, r) + s;
        *t = L % n_qt;
        *c = s < q + (x < r) ? (n_chunks / 8) * 8 + L / n_qt : n_chunks;
    }
}

// Byte offsets of the GEMM-structured scan's LDS regions.
struct GemmLayout {
    uint32_t ring, norms, stage, sup, bytes;
};

__host__ __device__ inline GemmLayout gemm_layout(int tpq)
{
    GemmLayout L;
    uint32_t o = 0;
    L.ring = o;    // [GM_SLOTS][GM_SLOT_LOADS][64] row and request fragments of a stage
    o += (uint32_t)GM_SLOTS * GM_SLOT_LOADS * WAVE * 16;
    L.norms = o;   // [2][GM_ROWS] |x|^2 of a macro tile's rows
    o += 2u * GM_ROWS * 4;
    L.stage = o;   // [GM_EPS][stage_pitch(64 * tpq)] a macro tile's maxima
    o += (uint32_t)GM_EPS * stage_pitch(64 * tpq) * 4;
    L.sup = o;     // [64 * tpq][GM_HOLD] maxima of the last macro tiles
    o += 64u * tpq * GM_HOLD * 4;
    L.bytes = o;
    return L;
}

// The bank-scan launchers (LDS-resident: one translation unit per element
// type; query-resident: one per row length).
hipError_t launch_scan_res_bf16(const KnnPlan &p, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_res_f32(const KnnPlan &p, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_gemm(const KnnPlan &p, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_rq(const KnnPlan &p, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_rq12(const KnnPlan &p, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_rq16(const KnnPlan &p, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_rq24(const KnnPlan &p, const ScanArgs &a, hipStream_t s);
hipError_t launch_scan_rq32(const KnnPlan &p, const ScanArgs &a, hipStream_t s);

namespace {

template <int DT> struct Elem;
template <> struct Elem<0> { static constexpr int VEC = 4, ESZ = 4; };   // fp32
template <> struct Elem<1> { static constexpr int VEC = 8, ESZ = 2; };   // bf16

constexpr int KSTEP_BYTES = 64;   // bytes of one row in one k-step (4 lanes x 16 bytes)

// Sum of squares of the 16-byte group held in v, added to s in element order.
template <int DT>
__device__ __forceinline__ float sumsq16(const i32x4 &v, float s)
{
    if constexpr (DT == 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t w = (uint32_t)v[e];
            const float x0 = bf16lo(w), x1 = bf16hi(w);
            s = fmaf(x0, x0, s);
            s = fmaf(x1, x1, s);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = __int_as_float(v[e]);
            s = fmaf(x, x, s);
        }
    }
    return s;
}

// One 16x16 MFMA tile step over 16 bytes of K per lane, D = A*B + C:
//   bf16: one v_mfma_f32_16x16x32_bf16 (8 elements per lane)
//   fp32: four v_mfma_f32_16x16x4_f32 (element e of every lane in step e)
// A and B hold the same K positions in the same lanes, so the dot products
// come out right whatever order the hardware assigns K within a step.
template <int DT>
__device__ __forceinline__ f32x4 mfma_step(const i32x4 &a, const i32x4 &b, const f32x4 &c)
{
    if constexpr (DT == 1) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    } else {
        f32x4 d = c;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            d = __builtin_amdgcn_mfma_f32_16x16x4f32(__int_as_float(a[e]), __int_as_float(b[e]), d,
                                                     0, 0, 0);
        return d;
    }
}

__device__ __forceinline__ float max4(const f32x4 &v)
{
    return fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3]));
}

// Maxima of four registers over the wave's four rows of 16 lanes, column by
// column: lane row r of the result holds the maximum of argument
// (r with its two bits swapped) in that column.
__device__ __forceinline__ float rows_max4(float m0, float m1, float m2, float m3)
{
    auto swap32 = [](float a, float b) {
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b),
                                                        false, false);
        return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
    };
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(swap32(m0, m1)),
                                                    __float_as_uint(swap32(m2, m3)), false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}

__device__ __forceinline__ i32x4 load16(const uint8_t *p) { return *(const i32x4 *)p; }

// Raw buffer resource over [base, base + bytes): loads at or past the end
// return zero, which masks rows past a chunk and queries past the batch.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes,
                                             0x00020000);
}

__device__ __forceinline__ i32x4 buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t voffset)
{
    return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voffset, 0, 0));
}

constexpr uint32_t OFF_NONE = 0x80000000u;   // a buffer offset past any resource

// 16 bytes per lane, not kept in the caches for their own sake (256 requests
// over 1,000,000 x 768: 425 us a batch for 434 with plain stores).
__device__ __forceinline__ void store16_nt(__amdgpu_buffer_rsrc_t r, uint32_t voffset,
                                           const f32x4 &v)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, v), r, (int)voffset, 0, 2);
}

// Lane l's four entries of a request (entries 4*(l % 4) .. +3 of its super
// tile) to its place `at` (in floats, of the first entry, in resource r), as
// they are or folded into one: one store either way. `in`: whether the lane
// has anything to store. (The choice at run time, in the flush, cost the scan
// of 512 x 4,000,000 x 384 0.6 %.)
static_assert(FOLD == 4, "a lane's four entries are one folded entry");
template <bool FOLDED>
__device__ __forceinline__ void put_entries(__amdgpu_buffer_rsrc_t r, bool in, uint32_t at, int l,
                                            const f32x4 &v)
{
    if (FOLDED)
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(max4(v)), r,
                                              (int)(in ? (at + (l & 3)) * 4u : OFF_NONE), 0, 2);
    else
        store16_nt(r, in ? (at + (l & 3) * 4) * 4u : OFF_NONE, v);
}

// Global -> LDS load of 16 bytes per lane through the buffer resource: lane l's
// bytes land at dst + 16*l (dst is the same for the whole wave); a lane whose
// offset falls outside the resource writes zeros. Completion is counted by
// the wave's vector memory counter, like a load into registers.
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, i32x4 *dst, uint32_t voffset)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16,
                                             (int)voffset, 0, 0, 0);
}

// Wait until at most N vector memory operations of this wave are outstanding
// (they complete in issue order).
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "the counter has six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

__device__ __forceinline__ uint64_t pack(uint32_t key, int32_t idx)
{
    return ((uint64_t)key << 32) | (uint32_t)idx;
}

// Weight of a neighbour at squared distance d2 in the distance-weighted
// average: the inverse of its Euclidean distance, finite at distance 0 (a
// negative d2 from fp32 cancellation counts as 0).
__device__ __forceinline__ float inv_dist_weight(float d2)
{
    return 1.f / (sqrtf(fmaxf(d2, 0.f)) + 1e-6f);
}

// The label gather and average: sum over neighbours j = 0..k-1 in order,
// divided by k, or (wts non-null) weighted by wts[j] and divided by the sum
// of the weights. A neighbour index outside [0, N) makes both averages NaN
// instead of reading out of bounds (the check does not end the loop, so the
// k loads can all be in flight together).
__device__ __forceinline__ void average_labels(const int32_t *nbr, const float *wts, int k,
                                               const float *qual, const float *len, int N, int M,
                                               int m, float *q_out, float *l_out)
{
    float sq = 0.f, sl = 0.f, sw = 0.f;
    bool bad = false;
    if (wts) {
#pragma unroll 8
        for (int j = 0; j < k; ++j) {
            const int32_t n = nbr[j];
            const bool ok = n >= 0 && n < N;
            bad |= !ok;
            const size_t o = (size_t)(ok ? n : 0) * M + m;
            const float w = wts[j];
            sq = fmaf(w, qual[o], sq);
            sl = fmaf(w, len[o], sl);
            sw += w;
        }
    } else {
#pragma unroll 8
        for (int j = 0; j < k; ++j) {
            const int32_t n = nbr[j];
            const bool ok = n >= 0 && n < N;
            bad |= !ok;
            const size_t o = (size_t)(ok ? n : 0) * M + m;
            sq += qual[o];
            sl += len[o];
        }
        sw = (float)k;
    }
    *q_out = bad ? __builtin_nanf("") : sq / sw;
    *l_out = bad ? __builtin_nanf("") : sl / sw;
}

}  // namespace

}  // namespace rb
