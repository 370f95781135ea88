// Gathered contraction  Logit[r, c] = sum_k H[r, k] * E[cand_s[c], k]   (Eq. 2 on the columns of
// the candidate list; the paper's separate "construct E_LSH" copy is fused away: candidate rows
// of E are gathered straight into the matrix-core operands).
//
// Besides the logits every tile leaves, per hidden row, the pair (max, sum exp(logit - max)) over
// its 16 candidates: the selection combines these into the row's log-sum-exp without touching the
// exponential of every logit again.  The fused kernels (fused.h) leave a richer record per row and
// tile (TileRecord): also the word id of the maximum, the second largest logit of the tile and
// its word id -- enough for the selection to finish, in the common case, without reading a
// single logit or candidate id back.
//
// Work unit ("tile"): one sentence s, one group of 16 hidden rows (M-tile) and 16 candidates.
// A workgroup of WAVES waves splits the hidden dimension between its waves; every wave issues
// v_mfma_f32_16x16x4_f32 over its share of k and the partial 16x16 tiles are summed through LDS
// in a fixed wave order (deterministic).
//
// Operand layout of v_mfma_f32_16x16x4_f32 (A is 16x4, B is 4x16, D is 16x16, 64 lanes):
//   lane l supplies A[i = l % 16][k = l / 16] and B[k = l / 16][j = l % 16];
//   lane l receives D[i = 4 * (l / 16) + r][j = l % 16] in accumulator register r = 0..3.
// The k slots of one instruction may hold any four k indices as long as A and B agree, so lane l
// loads ONE 16-byte chunk of its candidate's row (fp32: 4 consecutive k, bf16: 8) and feeds one
// element per instruction: per load instruction a wave touches 16 rows x 64 contiguous bytes.
//
// Drivers of the tile code:
//   k_logits_stream  many tiles, rows of at most 2048 values: candidate rows through LDS in contiguous
//                    pieces, hidden rows in registers (up to 32 beams at a time);
//   k_logits_estage  33..64 beams, fp32 rows of 513 to 1024 values: the same change of places, all
//                    beams at once;
//   k_logits_pass, k_logits_few, k_logits_rows   the full vocabulary: all hidden rows of the call against all words (up to 48
//                    rows that fit in LDS and suit its split; up to 48; more);
//   k_logits_hlds    one wave per tile, the sentence's hidden rows staged in LDS: rows of more than 2048
//                    values, and where an option names it;
//   k_logits<WAVES>  a workgroup of 16 or 4 waves per (tile, row group), k split over the waves: rows
//                    shorter than a 16-byte chunk, hidden rows that do not fit in LDS, options;
//   k_logits_wave    one wave per tile, up to four row groups in the wave, hidden rows read from
//                    global memory (the same cases with many tiles; logits_hlds = 0);
//   fused.h          the same tiles inside the kernels that also produce the candidate list.
#pragma once
#include <cfloat>

#include "candidates.h"
#include "device_utils.h"

namespace lshbeam {

typedef float floatx4 __attribute__((ext_vector_type(4)));

template <typename ET> struct ElemTraits;
template <> struct ElemTraits<float> {
    static constexpr int VEC = 4;  // elements per 16-byte load
    __device__ static __forceinline__ void widen(const uint4& v, float (&out)[4]) {
        out[0] = __uint_as_float(v.x); out[1] = __uint_as_float(v.y); out[2] = __uint_as_float(v.z); out[3] = __uint_as_float(v.w);
    }
    __device__ static __forceinline__ void load16(const float* p, float (&out)[4]) {   // (any alignment)
        const Float4U v = *reinterpret_cast<const Float4U*>(p);
        out[0] = v.x; out[1] = v.y; out[2] = v.z; out[3] = v.w;
    }
};
template <> struct ElemTraits<uint16_t> {
    static constexpr int VEC = 8;
    __device__ static __forceinline__ void widen(const uint4& v, float (&out)[8]) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = __uint_as_float(w[i] << 16);
            out[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        }
    }
    __device__ static __forceinline__ void load16(const uint16_t* p, float (&out)[8]) {
        const Chunk16U<uint16_t> v = *reinterpret_cast<const Chunk16U<uint16_t>*>(p);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            out[2 * i] = __uint_as_float(v.w[i] << 16);
            out[2 * i + 1] = __uint_as_float(v.w[i] & 0xFFFF0000u);
        }
    }
};

// One logit by its definition: products in the order of k, summed in fp32 by one lane (any d, any alignment).  A NaN
// ends it: a row that holds one must not hold up the others (one of 320 hidden rows, V = 40000: 1.33 -> 0.27 ms a step).
template <typename ET>
__device__ __forceinline__ float plain_dot(const ET* e, const float* h, int d) {
    constexpr int VEC = ElemTraits<ET>::VEC;
    float sum = 0.f;
    int k = 0;
    for (; k + VEC <= d && sum == sum; k += VEC) {
        float x[VEC];
        ElemTraits<ET>::load16(e + k, x);
#pragma unroll
        for (int q = 0; q < VEC; ++q) sum = fmaf(x[q], h[k + q], sum);
    }
    for (; k < d && sum == sum; ++k) sum = fmaf(elem_f32(e + k), h[k], sum);
    return sum;
}

// Logits made of bf16 planes, or of rows whose last elements met zeros, are right wherever they are finite.  An
// infinite element meets zero planes and makes NaN, one within 2^119 of the end of the fp32 range rounds to an
// infinite plane: any such value, of either side, leaves an infinity or a NaN in every sum it enters.  Those are
// made again here, by redo(i) = plain_dot of logit i (per lane; addresses must be valid on lanes without a logit
// too).  Costs a fused multiply-add per logit and one test; a logit that is redone costs its wave about 20 us.
template <int N, typename Redo>
__device__ __forceinline__ void settle_non_finite(float (&x)[N], Redo&& redo) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) t = fmaf(x[i], 0.f, t);   // (0 or NaN)
    if (__builtin_expect(__ballot(t != t) == 0ull, 1)) return;
#pragma unroll 1
    for (int i = 0; i < N; ++i) {
        float v = x[0];
#pragma unroll
        for (int j = 1; j < N; ++j) v = i == j ? x[j] : v;   // (a variable index would put x in memory)
        if (__ballot(!(fabsf(v) < INFINITY)) == 0ull) continue;
        if (!(fabsf(v) < INFINITY)) v = redo(i);
#pragma unroll
        for (int j = 0; j < N; ++j) x[j] = i == j ? v : x[j];
    }
}

// exp(x - mx) for a logit and the largest of its record.  A record whose logits are all -inf has (-inf, 0): the
// difference to the lowest finite value is -inf too, that to -inf would be NaN, and the row's log-sum-exp with it.
__device__ __forceinline__ float exp_below(float x, float mx) { return expf(x - fmaxf(mx, -FLT_MAX)); }

// Per (hidden row, tile) record of the fused kernels (the other kernels store the first two fields
// only, as a float2 array in the same place): x = largest logit of the tile's candidates,
// y = sum exp(logit - x), z = second largest logit (-inf if the tile has one candidate), w = word id
// of the largest (the lowest column among equals; as bits).  The id of the second largest goes to
// a parallel int32 array (-1 if none).  The plain kernels store only (x, y) as a float2.
typedef float4 TileRecord;
struct TileRecords {
    TileRecord* rec;   // [rows, pitch]
    int32_t* id2;      // [rows, pitch] word id of each record's second largest logit, -1 if none
    int64_t pitch;     // records per hidden row
};

// Records that stand for groups of tiles.  A kernel whose workgroup j of G walks the tiles j,
// j + G, j + 2G, ... of a sentence leaves one record for every kGroupTiles of them: record
// j + m G covers the tiles j + (kGroupTiles m + i) G, i < kGroupTiles.  (Fifty rows of per-tile
// records were 140 KB per sentence, all of which has to enter the one CU that selects.)
constexpr int kGroupTiles = 8;
__host__ __device__ inline int group_records(int ntiles, int G) {   // record slots per hidden row
    const int per_wg = (ntiles + G - 1) / G;
    return ntiles < G ? ntiles : G * ((per_wg + kGroupTiles - 1) / kGroupTiles);
}

constexpr int kTileN = 16;  // candidates per tile
// Columns per record of the kernels that serve the full vocabulary.  (Their selection is bound by what
// the one CU per sentence pulls in: a record per 16 words was 240 KB for 12 rows and V = 40000,
// 15.5 us; a record per 64 words: 8 us.  Opening a wide tile reads 48 more logits.)
constexpr int kWideN = 64;
constexpr int kTileM = 16;  // hidden rows per tile
constexpr int kMaxSentencesLogits = 4096;

// One (hidden row, tile) record from the 16 lanes that hold the row's logits of the tile's columns
// (a DPP row: 16 consecutive lanes, lane jc = column jc; `valid` lanes hold a logit x of a real
// candidate `id`).  Eq. 1 denominator, first stage: (max, sum of exp(logit - max)).  RICH (the
// fused kernels): plus the second largest logit and the two word ids, as a TileRecord; otherwise
// the pair alone, as a float2 in the same array (the contraction kernels of the many-tile plans
// are bound by bandwidth and instruction issue, and the longer epilogue cost them 4-8 %).
// Called by whole DPP rows; rows with row_ok false store nothing.  SHARE: see store_shared_result.
template <bool SHARE, bool RICH>
__device__ __forceinline__ void tile_record_store(const TileRecords& recs, size_t at, bool row_ok, bool valid,
                                                  float x, int jc, int32_t id) {
    const float mx = row16_max(valid ? x : -INFINITY);
    const float se = row16_sum(valid ? exp_below(x, mx) : 0.f);
    if constexpr (!RICH) {
        if (jc == 0 && row_ok) reinterpret_cast<float2*>(recs.rec)[at] = make_float2(mx, se);
    } else {
        // the lowest column that holds the maximum; the largest of the others and its lowest column
        const int c1 = row16_min_i32((valid && x == mx) ? jc : 16);
        const float mx2 = row16_max((valid && jc != c1) ? x : -INFINITY);
        const int c2 = row16_min_i32((valid && jc != c1 && x == mx2) ? jc : 16);
        if (row_ok) {
            if (jc == (c1 < 16 ? c1 : 0)) {   // (no column equals the maximum: NaN logits)
                unsigned long long* rec = reinterpret_cast<unsigned long long*>(recs.rec + at);
                const uint32_t idb = (uint32_t)(c1 < 16 ? id : -1);
                store_shared_result<SHARE>(rec, ((unsigned long long)__float_as_uint(se) << 32) | __float_as_uint(mx));
                store_shared_result<SHARE>(rec + 1, ((unsigned long long)idb << 32) | __float_as_uint(mx2));
            }
            if (jc == (c2 < 16 ? c2 : 0)) store_shared_result<SHARE>(&recs.id2[at], c2 < 16 ? id : (int32_t)-1);
        }
    }
}

// MTB tiles: logits of hidden rows [16 mt, 16 (mt + MTB)) of sentence s against 16 candidates,
// this lane's candidate being row j of E (lanes beyond the list hold any valid row; their results
// are dropped; row groups beyond B are computed on clamped rows and dropped too).  The candidate
// rows are loaded once for all MTB row groups.  Called by all WAVES*64 threads of the workgroup;
// contains 2 MTB workgroup barriers.  h_lds, if given, is an LDS copy of the sentence's B hidden
// rows (16-byte aligned, pitch h_pitch floats; 0 = d).  [row_lo, row_hi) restricts the call to
// a range of the sentence's rows (mt counts groups of 16 from row_lo; h_lds then holds that range).
//
// CHUNKS: a row holds at least one 16-byte chunk of E.  Rows are then read with 16-byte loads from whatever
// address they start at (d = 1001 fp32, rows 4 bytes off a multiple of 16: element by element was three times
// slower); the chunk that would reach past the row's end is read from the row's last VEC elements instead, of
// which those that were counted already are zeroed on both sides.  Otherwise elements are read one by one.
// QUADS (with CHUNKS): lanes load candidates' chunks for each other (quads_to_operand); the same sums.
template <typename ET, int WAVES, int UNROLL, bool CHUNKS, int MTB = 1, bool RICH = false, bool SHARE = false, bool QUADS = false>
__device__ __forceinline__ void logits_tile(const ET* __restrict__ E, int64_t ld, int d,
                                            const float* __restrict__ H, int B, int s, int mt,
                                            int nt, int C, int64_t j, float* __restrict__ logits,
                                            int64_t cpitch, TileRecords recs, float (*red)[4][kWave],
                                            const float* h_lds = nullptr, int h_pitch = 0,
                                            int row_lo = 0, int row_hi = -1, int tn = kTileN) {
    // tn <= 16: candidates of this tile (columns tn .. 15 of the matrix instruction stay unused;
    // narrower tiles are an option of the fused plans, see select_tile_width)
    constexpr int VEC = ElemTraits<ET>::VEC;
    constexpr int KSTEP = 4 * VEC;  // k covered by one 64-lane load
    if (h_pitch == 0) h_pitch = d;
    if (row_hi < 0) row_hi = B;
    const int tid = threadIdx.x, ln = lane_id(), wv = wave_id();
    const int col = ln & 15, kq = ln >> 4;
    const int nks = (d + KSTEP - 1) / KSTEP;
    const int n0 = nt * tn;
    const bool col_used = (QUADS ? quad_row() : col) < tn;   // lanes of unused columns load no candidate row
    const ET* erow = E + (QUADS ? (int64_t)operand_to_quads((int32_t)j) : j) * ld;
    // the sentence's hidden rows, from LDS when the caller has them staged there ([B][d]);
    // rows beyond B are clamped like the candidate: never stored
    const float* hrow[MTB];
#pragma unroll
    for (int m = 0; m < MTB; ++m) {
        const int hr = min(row_lo + (mt + m) * kTileM + col, row_hi - 1);
        hrow[m] = h_lds ? h_lds + (size_t)(hr - row_lo) * h_pitch : H + ((size_t)s * B + hr) * d;
    }

    floatx4 acc[MTB];
#pragma unroll
    for (int m = 0; m < MTB; ++m) acc[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int ks0 = wv; ks0 < nks; ks0 += WAVES * UNROLL) {
        float ev[UNROLL][VEC], hv[MTB][UNROLL][VEC];
        uint4 raw[UNROLL];
#pragma unroll
        for (int uu = 0; uu < UNROLL; ++uu) {
            const int k = (ks0 + uu * WAVES) * KSTEP + kq * VEC;
            if constexpr (QUADS) {
                const int kl = (ks0 + uu * WAVES) * KSTEP + quad_piece() * VEC;
                raw[uu] = make_uint4(0u, 0u, 0u, 0u);
                if (kl < d && col_used) {
                    const Chunk16U<ET> c = *reinterpret_cast<const Chunk16U<ET>*>(erow + min(kl, d - VEC));
                    raw[uu] = make_uint4(c.w[0], c.w[1], c.w[2], c.w[3]);
                }
#pragma unroll
                for (int m = 0; m < MTB; ++m)
#pragma unroll
                    for (int q = 0; q < VEC; q += 4) {
                        Float4U h4 = {0.f, 0.f, 0.f, 0.f};
                        if (k < d) h4 = *reinterpret_cast<const Float4U*>(hrow[m] + min(k, d - VEC) + q);
                        hv[m][uu][q] = h4.x; hv[m][uu][q + 1] = h4.y;
                        hv[m][uu][q + 2] = h4.z; hv[m][uu][q + 3] = h4.w;
                    }
            } else if (CHUNKS) {
                if (k < d) {
                    const int at = min(k, d - VEC);
                    if (col_used) {
                        ElemTraits<ET>::load16(erow + at, ev[uu]);
                    } else {
#pragma unroll
                        for (int q = 0; q < VEC; ++q) ev[uu][q] = 0.f;
                    }
#pragma unroll
                    for (int m = 0; m < MTB; ++m)
#pragma unroll
                        for (int q = 0; q < VEC; q += 4) {
                            const Float4U h4 = *reinterpret_cast<const Float4U*>(hrow[m] + at + q);
                            hv[m][uu][q] = h4.x; hv[m][uu][q + 1] = h4.y;
                            hv[m][uu][q + 2] = h4.z; hv[m][uu][q + 3] = h4.w;
                        }
                } else {
#pragma unroll
                    for (int q = 0; q < VEC; ++q) {
                        ev[uu][q] = 0.f;
#pragma unroll
                        for (int m = 0; m < MTB; ++m) hv[m][uu][q] = 0.f;
                    }
                }
            } else {
#pragma unroll
                for (int q = 0; q < VEC; ++q) {
                    const bool in = (k + q) < d;
                    ev[uu][q] = (in && col_used) ? elem_f32(erow + k + q) : 0.f;
#pragma unroll
                    for (int m = 0; m < MTB; ++m) hv[m][uu][q] = in ? hrow[m][k + q] : 0.f;
                }
            }
        }
        if constexpr (QUADS) {
#pragma unroll
            for (int uu = 0; uu < UNROLL; ++uu)
                ElemTraits<ET>::widen(make_uint4(quads_to_operand(raw[uu].x), quads_to_operand(raw[uu].y), quads_to_operand(raw[uu].z), quads_to_operand(raw[uu].w)), ev[uu]);
        }
        if (CHUNKS && d % VEC != 0) {   // (uniform) leading elements of a row's last chunk that were counted before
#pragma unroll
            for (int uu = 0; uu < UNROLL; ++uu) {
                const int drop = (ks0 + uu * WAVES) * KSTEP + kq * VEC - (d - VEC);
#pragma unroll
                for (int m = 0; m < MTB; ++m)
#pragma unroll
                    for (int q = 0; q < VEC; ++q) hv[m][uu][q] = q >= drop ? hv[m][uu][q] : 0.f;
                // (both sides: either may hold an infinity.  A loop of its own: with the two in one, the fused kernels'
                // first scalar loads come to wait for each other, 16.1 -> 16.25 us a step)
#pragma unroll
                for (int q = 0; q < VEC; ++q) ev[uu][q] = q >= drop ? ev[uu][q] : 0.f;
            }
        }
#pragma unroll
        for (int uu = 0; uu < UNROLL; ++uu)
#pragma unroll
            for (int q = 0; q < VEC; ++q)
#pragma unroll
                for (int m = 0; m < MTB; ++m)
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(hv[m][uu][q], ev[uu][q], acc[m],
                                                                  0, 0, 0);
    }

    LSH_TRACE(1, 3);
    LSH_TRACE_WG(5);
#pragma unroll
    for (int m = 0; m < MTB; ++m) {
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wv][r][ln] = acc[m][r];
        __syncthreads();
        LSH_TRACE_WG(7);
        if (tid < kTileM * kTileN) {
            const int i = tid >> 4, jc = tid & 15;
            const int src = (i >> 2) * 16 + jc, r = i & 3;
            float sum = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) sum += red[w][r][src];
            const int row = row_lo + (mt + m) * kTileM + i, c = n0 + jc;
            const bool valid = row < row_hi && jc < tn && c < C;
            // (SHARE: other workgroups of this kernel read the results; see store_shared_result)
            if (valid) store_shared_result<SHARE>(&logits[((size_t)s * B + row) * cpitch + c], sum);
            tile_record_store<SHARE, RICH>(recs, ((size_t)s * B + row) * recs.pitch + nt, row < row_hi, valid, sum,
                                           jc, (int32_t)j);
        }
        __syncthreads();
    }
    LSH_TRACE(1, 4);
}

// All row groups of one tile of candidates, the candidate rows being read once for up to four
// groups (64 beams) at a time.
template <typename ET, int WAVES, int UNROLL, bool CHUNKS, int FIXED_MT = 0, bool RICH = false, bool SHARE = false, bool QUADS = false>
__device__ __forceinline__ void logits_tile_all_rows(const ET* __restrict__ E, int64_t ld, int d,
                                                     const float* __restrict__ H, int B, int s,
                                                     int nt, int C, int64_t j,
                                                     float* __restrict__ logits, int64_t cpitch,
                                                     TileRecords recs, float (*red)[4][kWave],
                                                     const float* h_lds = nullptr, int h_pitch = 0,
                                                     int row_lo = 0, int row_hi = -1, int tn = kTileN) {
    // loads in flight per row group shrink as the groups grow: the operands of all groups have
    // to fit the register budget of a 1024-thread workgroup
    // (measured: keeping the full unroll in 256-thread workgroups, where registers would allow
    // it, is slower -- the hidden-row loads of four groups then crowd out the candidate rows)
    constexpr int U4 = UNROLL >= 4 ? UNROLL / 4 : 1;
    constexpr int U2 = ElemTraits<ET>::VEC > 4 ? U4 : (UNROLL >= 2 ? UNROLL / 2 : 1);
    // FIXED_MT: the caller knows the number of row groups at compile time (only that case is
    // instantiated, so its registers do not count against the others)
    const int MT = FIXED_MT ? FIXED_MT : ((row_hi < 0 ? B : row_hi - row_lo) + kTileM - 1) / kTileM;
    if (MT == 1) {
        logits_tile<ET, WAVES, UNROLL, CHUNKS, 1, RICH, SHARE, QUADS>(E, ld, d, H, B, s, 0, nt, C, j, logits, cpitch,
            recs, red, h_lds, h_pitch, row_lo, row_hi, tn);
    } else if (MT == 2) {
        logits_tile<ET, WAVES, U2, CHUNKS, 2, RICH, SHARE, QUADS>(E, ld, d, H, B, s, 0, nt, C, j, logits, cpitch,
            recs, red, h_lds, h_pitch, row_lo, row_hi, tn);
    } else if (ElemTraits<ET>::VEC > 4) {  // bf16: twice the registers per load, two groups at most
        for (int mt = 0; mt < MT; mt += 2)
            logits_tile<ET, WAVES, U2, CHUNKS, 2, RICH, SHARE, QUADS>(E, ld, d, H, B, s, mt, nt, C, j, logits, cpitch,
            recs, red, h_lds, h_pitch, row_lo, row_hi, tn);
    } else {
        for (int mt = 0; mt < MT; mt += 4)
            logits_tile<ET, WAVES, U4, CHUNKS, 4, RICH, SHARE, QUADS>(E, ld, d, H, B, s, mt, nt, C, j, logits, cpitch,
            recs, red, h_lds, h_pitch, row_lo, row_hi, tn);
    }
}

template <typename ET, int WAVES, int UNROLL, bool CHUNKS>
__global__ void __launch_bounds__(WAVES * kWave)
k_logits(const ET* __restrict__ E, int64_t ld, int d, const float* __restrict__ H, int S, int B,
         const int32_t* __restrict__ cand, const int32_t* __restrict__ count, int V,
         float* __restrict__ logits, int64_t cpitch, TileRecords recs) {
    __shared__ uint32_t tile_pref[kMaxSentencesLogits + 1];
    __shared__ float red[WAVES][4][kWave];

    const int tid = threadIdx.x, ln = lane_id(), wv = wave_id();
    (void)tid;
    const int MT = (B + kTileM - 1) / kTileM;

    LSH_TRACE(1, 0);
    // Workgroups are dealt to the 8 XCDs round-robin by the dispatcher; renumber them so that
    // consecutive logical ids (which take neighbouring tiles) share an XCD and its L2.
    // (Only worth it when several M-tiles re-read the same candidate rows; with one M-tile the
    // plain order lets the first workgroups dispatched be the ones that have work.)
    const uint32_t G = gridDim.x;
    const uint32_t per_xcd = G >> 3;
    const uint32_t logical = ((G & 7u) || MT == 1) ? blockIdx.x
                                                   : (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    const int col = ln & 15;

    // With a single sentence the first tile's candidate ids do not depend on the count: request
    // them together with it instead of after it (one dependent memory round trip less).
    const bool spec = (S == 1) && (cand != nullptr);
    int32_t jspec = 0;
    if (spec) {
        const uint32_t c0 = (logical / (uint32_t)MT) * kTileN + col;
        if (c0 < (uint32_t)V) jspec = cand[c0];
    }

    // exclusive prefix of tiles per sentence (wave 0, 64 sentences at a time)
    if (wv == 0) {
        uint32_t carry = 0;
        for (int base = 0; base < S; base += kWave) {
            const int s = base + ln;
            uint32_t n = 0;
            if (s < S) {
                const int C = count ? count[s] : V;
                n = (uint32_t)MT * (uint32_t)((C + kTileN - 1) / kTileN);
            }
            const uint32_t incl = wave_incl_scan(n);
            if (s < S) tile_pref[s] = carry + incl - n;
            carry += wave_read_lane(incl, kWave - 1);
        }
        if (ln == 0) tile_pref[S] = carry;
    }
    __syncthreads();
    LSH_TRACE(1, 1);
    const uint32_t total_tiles = tile_pref[S];

    for (uint32_t t = logical; t < total_tiles; t += G) {
        int lo = 0, hi = S;  // sentence: last s with tile_pref[s] <= t
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (tile_pref[mid] <= t) lo = mid; else hi = mid;
        }
        const int s = lo;
        const uint32_t tl = t - tile_pref[s];
        const int nt = tl / MT, mt = tl - nt * MT;
        const int C = count ? count[s] : V;
        const int n0 = nt * kTileN;

        // out-of-range lanes are clamped onto a valid row; their results are never stored
        const int cidx = min(n0 + col, C - 1);
        int64_t j;
        if (spec && t == logical)  // column 0 of a tile is always a real candidate
            j = (n0 + col < C) ? jspec : __shfl(jspec, ln & ~15, kWave);
        else
            j = cand ? cand[(size_t)s * V + cidx] : cidx;
        LSH_TRACE(1, 2);
        logits_tile<ET, WAVES, UNROLL, CHUNKS>(E, ld, d, H, B, s, mt, nt, C, j, logits, cpitch, recs, red);
    }
}

// Throughput variant for steps with many tiles (many sentences): ONE WAVE per tile of 16
// candidates, all k and all MT groups of 16 hidden rows in that wave.  No LDS, no barrier: the
// accumulators go straight from the matrix core to the stores, and a candidate row is read once
// however many beams there are.  Waves of a workgroup take consecutive tiles; the grid is
// persistent.
//
// Whole rounds (every wave of the grid one tile) run this way.  A last (or only) round that would
// occupy fewer than half of the waves is different: while all waves stream, the kernel runs at the
// memory system's rate, but a few hundred waves left alone with a 64 KB tile each run at one
// wave's latency-bound rate, and that tail was a sixth of the kernel.  Such a remainder is
// therefore dealt to whole workgroups, whose four waves split k and sum their partial tiles
// through LDS in wave order (logits_tile): four times as many waves share the same bytes.
template <typename ET, int MT, int UNROLL, bool CHUNKS>
__global__ void __launch_bounds__(256)
k_logits_wave(const ET* __restrict__ E, int64_t ld, int d, const float* __restrict__ H, int S, int B,
              const int32_t* __restrict__ cand, const int32_t* __restrict__ count, int V,
              float* __restrict__ logits, int64_t cpitch, TileRecords recs) {
    constexpr int VEC = ElemTraits<ET>::VEC;
    constexpr int KSTEP = 4 * VEC;
    __shared__ uint32_t tile_pref[kMaxSentencesLogits + 1];
    __shared__ float red[4][4][kWave];
    const int ln = lane_id(), wv = wave_id();
    LSH_TRACE(1, 0);
    if (wv == 0) {
        uint32_t carry = 0;
        for (int base = 0; base < S; base += kWave) {
            const int s = base + ln;
            uint32_t n = 0;
            if (s < S) n = (uint32_t)(((count ? count[s] : V) + kTileN - 1) / kTileN);
            const uint32_t incl = wave_incl_scan(n);
            if (s < S) tile_pref[s] = carry + incl - n;
            carry += wave_read_lane(incl, kWave - 1);
        }
        if (ln == 0) tile_pref[S] = carry;
    }
    __syncthreads();
    LSH_TRACE(1, 1);
    const uint32_t total_tiles = tile_pref[S];
    const uint32_t nwaves = gridDim.x * 4u;
    const int col = ln & 15, kq = ln >> 4;
    const int nks = (d + KSTEP - 1) / KSTEP;
    // tiles [0, wave_tiles) one wave each; the rest one workgroup each
    const uint32_t whole = total_tiles / nwaves * nwaves;
    const uint32_t wave_tiles = ((total_tiles - whole) * 2u > nwaves) ? total_tiles : whole;
    auto sentence_of = [&](uint32_t t) {
        int lo = 0, hi = S;  // last s with tile_pref[s] <= t
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (tile_pref[mid] <= t) lo = mid; else hi = mid;
        }
        return lo;
    };

    // workgroup b takes the consecutive tiles [b * per_wg, (b + 1) * per_wg), dealt round-robin to
    // its waves: neighbouring tiles (same sentence, same hidden rows in L1) stay together, and
    // with fewer tiles than waves every workgroup (hence every CU) still gets its share
    const uint32_t per_wg = (wave_tiles + gridDim.x - 1) / gridDim.x;
    const uint32_t wg_end = min(wave_tiles, (blockIdx.x + 1u) * per_wg);
    for (uint32_t t = blockIdx.x * per_wg + wv; t < wg_end; t += 4u) {
        const int s = sentence_of(t);
        const int nt = (int)(t - tile_pref[s]);
        const int C = count ? count[s] : V;
        const int n0 = nt * kTileN;
        const int cidx = min(n0 + col, C - 1);  // clamped lanes are never stored
        const int64_t j = cand ? cand[(size_t)s * V + cidx] : cidx;
        const ET* erow = E + j * ld;
        const float* hrow[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            hrow[mt] = H + ((size_t)s * B + min(mt * kTileM + col, B - 1)) * d;

        floatx4 acc[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int ks0 = 0; ks0 < nks; ks0 += UNROLL) {
            float ev[UNROLL][VEC], hv[MT][UNROLL][VEC];
#pragma unroll
            for (int uu = 0; uu < UNROLL; ++uu) {
                const int k = (ks0 + uu) * KSTEP + kq * VEC;
                if (CHUNKS) {
                    if (k < d) {
                        const int at = min(k, d - VEC), drop = k - at;
                        ElemTraits<ET>::load16(erow + at, ev[uu]);
#pragma unroll
                        for (int q = 0; q < VEC; ++q) ev[uu][q] = q >= drop ? ev[uu][q] : 0.f;   // (on both sides: either may hold an infinity)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                            for (int q = 0; q < VEC; q += 4) {
                                const Float4U h4 = *reinterpret_cast<const Float4U*>(hrow[mt] + at + q);
                                const float x[4] = {h4.x, h4.y, h4.z, h4.w};
#pragma unroll
                                for (int i = 0; i < 4; ++i) hv[mt][uu][q + i] = q + i >= drop ? x[i] : 0.f;
                            }
                    } else {
#pragma unroll
                        for (int q = 0; q < VEC; ++q) {
                            ev[uu][q] = 0.f;
#pragma unroll
                            for (int mt = 0; mt < MT; ++mt) hv[mt][uu][q] = 0.f;
                        }
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < VEC; ++q) {
                        const bool in = (k + q) < d;
                        ev[uu][q] = in ? elem_f32(erow + k + q) : 0.f;
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) hv[mt][uu][q] = in ? hrow[mt][k + q] : 0.f;
                    }
                }
            }
#pragma unroll
            for (int uu = 0; uu < UNROLL; ++uu)
#pragma unroll
                for (int q = 0; q < VEC; ++q)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(hv[mt][uu][q], ev[uu][q],
                                                                       acc[mt], 0, 0, 0);
        }
        // lane (col, kq) holds rows 16 mt + 4 kq + r of column n0 + col: 16 lanes per row
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = mt * kTileM + 4 * kq + r, c = n0 + col;
                const bool valid = row < B && c < C;
                const float x = acc[mt][r];
                if (valid) logits[((size_t)s * B + row) * cpitch + c] = x;
                tile_record_store<false, false>(recs, ((size_t)s * B + row) * recs.pitch + nt, row < B, valid, x, col,
                                         (int32_t)j);
            }
    }

    // the remainder: one workgroup per tile, k split over its four waves (uniform per workgroup)
    for (uint32_t t = wave_tiles + blockIdx.x; t < total_tiles; t += gridDim.x) {
        const int s = sentence_of(t);
        const int nt = (int)(t - tile_pref[s]);
        const int C = count ? count[s] : V;
        const int cidx = min(nt * kTileN + col, C - 1);
        const int64_t j = cand ? cand[(size_t)s * V + cidx] : cidx;
        logits_tile_all_rows<ET, 4, (UNROLL < 4 ? UNROLL : 4), CHUNKS, MT>(E, ld, d, H, B, s, nt, C, j,
                                                                        logits, cpitch, recs, red);
    }
}

// The wave-per-tile kernel with the hidden rows in LDS.  Measured on this machine: a stream of
// 16-byte loads that hits in cache still costs as much load-path throughput as one that goes to
// memory -- gathering candidate rows alone runs at 6.7 TB/s, with an equal stream of hidden-row
// loads beside it at 3.4 TB/s.  The A operands therefore must not come through the vector memory
// path at all: a workgroup (WAVES waves, consecutive tiles, so mostly one sentence) stages the
// sentence's hidden rows in LDS once and every tile reads them with ds_read_b128.  More rows
// than LDS holds are taken in groups, a workgroup each: every group reads the candidate rows
// again (the groups of a block of tiles run on one XCD, so from its L2 mostly), which is still far less load traffic than
// hidden rows coming through the vector memory path.  The row
// pitch is the next value >= d that is 4 modulo 32: consecutive rows then start 4 banks apart
// and eight lanes x 16 bytes (eight rows, same k) cover all 32 banks exactly once.
__host__ __device__ inline int hlds_pitch(int d) {
    int p = (d + 7) & ~7;
    while (p % 32 != 4) p += 4;
    return p;
}
// The last chunk of a row whose length is no multiple of the chunk is read from the row's last VEC elements
// (addresses of any alignment are fine for 16-byte loads); in LDS the hidden row continues with the matching
// chunk -- its last VEC values, those counted already replaced by zero -- so the loop knows nothing of it.
//
// bf16 candidate rows: the hidden rows are staged as three bf16
// planes hi + mid + lo = h exactly (8 + 8 + 8 significand bits: each plane is the remainder so
// far truncated to bf16), and the contraction runs on v_mfma_f32_16x16x32_bf16 -- a lane's
// 16-byte chunk of its candidate row IS that instruction's B operand (8 consecutive k), no
// widening; three instructions per chunk against eight fp32 ones at a quarter of the cycles each.
// Products of two bf16 values are exact in fp32, so the result differs from the widened fp32
// contraction by summation order only.  Plane rows are pitched 8 modulo 64 elements (16 modulo
// 128 bytes: eight rows x 16 bytes cover all banks once).
__host__ __device__ inline int hlds_pitch_planes(int d) {
    int p = (d + 7) & ~7;
    while (p % 64 != 8) p += 8;
    return p;
}
// dynamic LDS: tile prefix (S + 1 words, rounded to 4), split-k reduction buffer, hidden rows
// (fp32, or three bf16 planes)
__host__ __device__ inline size_t hlds_lds_bytes(int S, int rows, int d, int waves, bool planes = false) {
    const size_t hidden = planes ? (size_t)rows * hlds_pitch_planes(d) * 6 : (size_t)rows * hlds_pitch(d) * 4;
    return ((size_t)((S + 1 + 3) & ~3) + (size_t)waves * 4 * kWave) * 4 + hidden;
}
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ uint4 load_chunk(const uint16_t* p) {   // 16 bytes, any alignment
    const Chunk16U<uint16_t> c = *reinterpret_cast<const Chunk16U<uint16_t>*>(p);
    return make_uint4(c.w[0], c.w[1], c.w[2], c.w[3]);
}
// Four hidden values as the three bf16 planes of k_logits_hlds (exactly x = hi + mid + lo), to LDS.
__device__ __forceinline__ void store_planes4(char* dst, size_t plane_bytes, const float (&x)[4]) {
    uint32_t hi[4], mid[4], lo[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        hi[q] = __float_as_uint(x[q]) & 0xFFFF0000u;
        const float r1 = x[q] - __uint_as_float(hi[q]);          // exact
        mid[q] = __float_as_uint(r1) & 0xFFFF0000u;
        lo[q] = __float_as_uint(r1 - __uint_as_float(mid[q]));   // exact, <= 8 bits
    }
    *reinterpret_cast<uint2*>(dst) = make_uint2((hi[0] >> 16) | (hi[1] & 0xFFFF0000u), (hi[2] >> 16) | (hi[3] & 0xFFFF0000u));
    *reinterpret_cast<uint2*>(dst + plane_bytes) =
        make_uint2((mid[0] >> 16) | (mid[1] & 0xFFFF0000u), (mid[2] >> 16) | (mid[3] & 0xFFFF0000u));
    *reinterpret_cast<uint2*>(dst + 2 * plane_bytes) =
        make_uint2((lo[0] >> 16) | (lo[1] & 0xFFFF0000u), (lo[2] >> 16) | (lo[3] & 0xFFFF0000u));
}

// Tiles are dealt to the XCDs by their number inside the sentence: tile t of every sentence below `shared`
// (the tiles that surely lie among the top-frequent words all sentences have in common, where those are the
// lowest ids) goes to XCD t mod 8, so that its 16 rows enter one L2 and serve the other sentences from there;
// of the tiles beyond, in the order of the words, every XCD has an eighth in one piece, so that words that
// several sentences want are mostly on the same XCD for all of them; and as its workgroups take them interleaved,
// at about the same time (64 x 10 beams, V = 200000, d = 1024 bf16: 48 % of the requests hit the L2; 17 % where tiles
// beyond went to XCD (t + s) mod 8, every workgroup with a stretch of its own).
struct XcdTiles {   // the tiles of one sentence that belong to XCD x
    uint32_t n0;        // how many of them lie below `shared`
    uint32_t first1;    // the first one beyond
    uint32_t n;         // all
};
__host__ __device__ __forceinline__ uint32_t tiles_mod8(uint32_t begin, uint32_t end, uint32_t r) {   // t in [begin, end), t mod 8 == r
    return end > begin ? ((end + 7u - r) >> 3) - ((begin + 7u - r) >> 3) : 0u;
}
__host__ __device__ __forceinline__ XcdTiles xcd_tiles(uint32_t ntiles, uint32_t shared, uint32_t s, uint32_t x) {
    XcdTiles t;
    const uint32_t cut = shared < ntiles ? shared : ntiles, m = ntiles - cut;
    t.n0 = tiles_mod8(0u, cut, x);
    t.first1 = cut + m * x / 8u;
    t.n = t.n0 + (cut + m * (x + 1u) / 8u - t.first1);
    return t;
}
__host__ __device__ __forceinline__ uint32_t xcd_tile(const XcdTiles& t, uint32_t x, uint32_t i) {   // its i-th
    return i < t.n0 ? x + 8u * i : t.first1 + (i - t.n0);
}
// The tiles of one sentence that a workgroup takes, in two arithmetic progressions.
struct TileRun {
    uint32_t n, head, a0, a1, b0, b1;   // tile u < n: a0 + u a1 below `head`, else b0 + u b1
    __host__ __device__ __forceinline__ uint32_t tile(uint32_t u) const { return u < head ? a0 + u * a1 : b0 + u * b1; }
};
// of an XCD's tiles those from `first` on, every `every`-th, n in all
__host__ __device__ __forceinline__ TileRun xcd_run(const XcdTiles& t, uint32_t x, uint32_t first, uint32_t every, uint32_t n) {
    const uint32_t head = t.n0 > first ? (t.n0 - first + every - 1u) / every : 0u;
    return {n, head, x + 8u * first, 8u * every, t.first1 + first - t.n0, every};
}
// G workgroups on each of 8 XCDs dealt to sentences by weight (equal ones: 1 each, S <= 8 G of them).  With the weights of
// the sentences in front summed to w, of all to W, those of a sentence on XCD x begin at dealt_from(w) and end where the
// next one's begin: a few more or less per XCD, and 8 G / W per unit of weight, give or take one, in all.
__host__ __device__ __forceinline__ uint32_t dealt_from(uint32_t w, uint32_t x, uint32_t W, uint32_t G) { return (w * G + (x * W >> 3)) / W; }
__host__ __device__ __forceinline__ uint32_t dealt_sentence(uint32_t b, uint32_t x, uint32_t S, uint32_t G) {   // (equal weights)
    return ((b + 1u) * S - (x * S >> 3) - 1u) / G;
}
// Whether shares as large as the lists are worth working out: with equal ones the longest list takes twice as long as all of them
// together would with even ones, and three tiles more; with short rows, 1.3 times.  us a step, equal shares and so: d = 1000 fp32,
// V = 40000, one list of 32 x 10 beams four times the others 108, 69; of 64 x 10 176, 97; eight sentences, one list three times their
// mean 56, 49; d = 300, lists from 4000 to 14000, 64 x 10 155, 148; 40 x 6 84, 73; d = 88, V = 170000, 64 x 10 379, 324; 15 x 26 461, 421.  Long
// rows lose more by leaving the XCD that has them for other sentences (64 x 10, V = 200000, d = 1024 bf16, a longest list of 1.5 times the
// mean: 475, 694; V = 40000, d = 1000 fp32: 226, 279; of 1.8 times: 461, 499; 239, 201).
__host__ __device__ __forceinline__ bool dealt_by_count(uint32_t most, uint32_t sum, uint32_t S, uint32_t G, int row_bytes) {   // (in tiles)
    return S <= 4u * G && G <= 192u && sum < (1u << 23) &&
           (float)most * (float)S > (row_bytes <= 1600 ? 1.3f : 2.f) * (float)sum + 24.f * (float)G;
}
// A list's weight: its tiles, or as much as a workgroup takes (8 G (least) >= sum + S (least) >= W; W < 2^24 + 4 G).
__host__ __device__ __forceinline__ uint32_t least_weight(uint32_t sum, uint32_t S, uint32_t G) { return (sum + 8u * G - S - 1u) / (8u * G - S); }
// What number `first` of the `mine` workgroups a sentence has on an XCD takes, with `before` of its `all` < 4096 on the XCDs in
// front (ntiles <= 2^20): of the tiles that all sentences share they take turns, of the others every XCD has its share.
__host__ __device__ __forceinline__ TileRun dealt_run(uint32_t ntiles, uint32_t shared, uint32_t first, uint32_t mine, uint32_t before, uint32_t all) {
    const uint32_t cut = shared < ntiles ? shared : ntiles, at = before + first;
    const uint32_t begin = cut + (ntiles - cut) * before / all + first, end = cut + (ntiles - cut) * (before + mine) / all;
    const uint32_t head = cut > at ? (cut - at + all - 1u) / all : 0u;
    return {head + (end > begin ? (end - begin + mine - 1u) / mine : 0u), head, at, all, begin - head * mine, mine};
}

// Eight hidden values as the A operands of three v_mfma_f32_16x16x32_bf16: their planes.
__device__ __forceinline__ void split_planes8(const float (&x)[8], uint4 (&out)[3]) {
    uint32_t w[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t a[2][3];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const float v = x[2 * i + j];
            a[j][0] = __float_as_uint(v) & 0xFFFF0000u;
            const float r1 = v - __uint_as_float(a[j][0]);        // exact
            a[j][1] = __float_as_uint(r1) & 0xFFFF0000u;
            a[j][2] = __float_as_uint(r1 - __uint_as_float(a[j][1]));   // exact, <= 8 bits
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) w[p][i] = (a[0][p] >> 16) | (a[1][p] & 0xFFFF0000u);
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) out[p] = make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]);
}

template <typename ET, int MT, int WAVES, int UNROLL, bool PLANES = false>
__global__ void __launch_bounds__(WAVES * kWave) __attribute__((amdgpu_waves_per_eu(4)))
k_logits_hlds(const ET* __restrict__ E, int64_t ld, int d, const float* __restrict__ H, int S, int B,
              int group_rows /*row group g takes rows [g, g + 1) * group_rows of every sentence;
                               group_rows <= 16 MT*/,
              int gx /*workgroups per row group, a multiple of 8*/, int ngroups, int rem_div, int shared /*see above*/,
              const int32_t* __restrict__ cand, const int32_t* __restrict__ count, int V,
              float* __restrict__ logits, int64_t cpitch, TileRecords recs) {
    constexpr int VEC = ElemTraits<ET>::VEC;
    constexpr int KSTEP = 4 * VEC;
    extern __shared__ uint32_t hsm[];
    // grid = gx * ngroups workgroups.  Workgroup ids go round the 8 XCDs, and the row groups that read
    // the same candidate rows should share an L2: ids that are congruent modulo 8 and consecutive
    // otherwise form the row groups of one block of tiles.
    const uint32_t wg_slot = blockIdx.x >> 3, xcd = blockIdx.x & 7u;
    const uint32_t bx = wg_slot / (uint32_t)ngroups, wgs = (uint32_t)gx >> 3;   // this workgroup of its XCD's
    const int by = (int)(wg_slot % (uint32_t)ngroups);
    const int row0 = by * group_rows, Bg = min(group_rows, B - row0);
    uint32_t* tile_pref = hsm;
    float (*red)[4][kWave] = reinterpret_cast<float (*)[4][kWave]>(hsm + ((S + 1 + 3) & ~3));
    float* hl = reinterpret_cast<float*>(hsm + ((S + 1 + 3) & ~3) + WAVES * 4 * kWave);
    const int pitch = hlds_pitch(d);
    // PLANES (bf16 rows): hidden rows as three bf16 planes, bf16 matrix instructions
    static_assert(!PLANES || VEC == 8, "bf16 planes need bf16 rows");
    const int ppitch_h = hlds_pitch_planes(d);
    uint16_t* hplane = reinterpret_cast<uint16_t*>(hl);
    const size_t plane_stride = (size_t)group_rows * ppitch_h;
    const int tid = threadIdx.x, ln = lane_id(), wv = wave_id();
    auto ntiles_of = [&](int s) { return (uint32_t)(((count ? count[s] : V) + kTileN - 1) / kTileN); };
    LSH_TRACE(1, 0);
    if (wv == 0) {   // exclusive prefix of the XCD's tiles over the sentences
        uint32_t carry = 0;
        for (int base = 0; base < S; base += kWave) {
            const int s = base + ln;
            const uint32_t n = s < S ? xcd_tiles(ntiles_of(s), (uint32_t)shared, (uint32_t)s, xcd).n : 0u;
            const uint32_t incl = wave_incl_scan(n);
            if (s < S) tile_pref[s] = carry + incl - n;
            carry += wave_read_lane(incl, kWave - 1);
        }
        if (ln == 0) tile_pref[S] = carry;
    }
    __syncthreads();
    LSH_TRACE(1, 1);
    const uint32_t total_tiles = tile_pref[S];
    const uint32_t nwaves = wgs * (uint32_t)WAVES;
    const int col = ln & 15, kq = ln >> 4;
    const int nks = (d + KSTEP - 1) / KSTEP;
    const uint32_t whole = total_tiles / nwaves * nwaves;
    // a last round that fills at most 1 / rem_div of the waves is dealt to whole workgroups that
    // split k (below); a fuller one runs as one more wave-per-tile round (measured with rem_div = 4
    // against 2: S = 32, B = 20: 117 -> 83 us; the 64-sentence bf16 shape: 229 -> 221 us)
    const uint32_t wave_tiles = ((total_tiles - whole) * (uint32_t)rem_div > nwaves) ? total_tiles : whole;
    auto sentence_of = [&](uint32_t t) {
        int lo = 0, hi = S;  // last s with tile_pref[s] <= t
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (tile_pref[mid] <= t) lo = mid; else hi = mid;
        }
        return lo;
    };
    int staged = -1;
    auto stage = [&](int s) {  // workgroup-uniform; barriers inside
        if (s == staged) return;
        __syncthreads();  // everyone is done with the previous sentence's rows
        const float* Hs = H + ((size_t)s * B + row0) * d;
        const int whole_k = d - d % VEC;
        auto put = [&](int r, int k, const float (&x)[4]) {
            if constexpr (PLANES)
                store_planes4(reinterpret_cast<char*>(hplane + (size_t)r * ppitch_h + k), plane_stride * 2, x);
            else
                *reinterpret_cast<float4*>(hl + (size_t)r * pitch + k) = make_float4(x[0], x[1], x[2], x[3]);
        };
        constexpr int AHEAD = 4, T = WAVES * kWave;
        const int w4 = whole_k >> 2, n = Bg * w4;   // (e / w4 below: e < 2^16, exact as small_div is)
        const float inv = __builtin_amdgcn_rcpf((float)w4);
        for (int e0 = tid; e0 < n; e0 += AHEAD * T) {
            Float4U v[AHEAD];
            int r[AHEAD], k[AHEAD];
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) {
                const int e = min(e0 + j * T, n - 1);
                r[j] = (int)(((float)e + 0.5f) * inv);
                k[j] = 4 * (e - r[j] * w4);
                v[j] = *reinterpret_cast<const Float4U*>(Hs + (size_t)r[j] * d + k[j]);
            }
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) {
                const float x[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
                if (e0 + j * T < n) put(r[j], k[j], x);
            }
        }
        if (whole_k < d && tid < Bg * (VEC / 4)) {   // the partial chunk that ends each row
            const int r = tid / (VEC / 4), k0 = 4 * (tid % (VEC / 4));
            float x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = d - VEC + k0 + q;
                x[q] = k >= whole_k ? Hs[(size_t)r * d + k] : 0.f;
            }
            put(r, whole_k + k0, x);
        }
        __syncthreads();
        staged = s;
    };

    // whole rounds: one wave per tile; the workgroup walks its consecutive tiles sentence by
    // sentence (all of its waves in the same sentence, so one staging serves them)
    const uint32_t per_wg = (wave_tiles + wgs - 1) / wgs;
    const uint32_t wg_begin = min(wave_tiles, bx * per_wg);
    const uint32_t wg_end = min(wave_tiles, wg_begin + per_wg);
    for (uint32_t seg = wg_begin; seg < wg_end;) {
        const int s = sentence_of(seg);
        const uint32_t seg_end = min(wg_end, tile_pref[s + 1]);
        stage(s);
        LSH_TRACE(1, 2);
        const XcdTiles xt = xcd_tiles(ntiles_of(s), (uint32_t)shared, (uint32_t)s, xcd);
        const int C = count ? count[s] : V;
        for (uint32_t t = seg + wv; t < seg_end; t += WAVES) {
            const int nt = (int)xcd_tile(xt, xcd, t - tile_pref[s]);
            const int n0 = nt * kTileN;
            const int cidx = min(n0 + col, C - 1);  // clamped lanes are never stored
            const int64_t j = cand ? cand[(size_t)s * V + cidx] : cidx;
            const ET* erow = E + j * ld;
            const float* hrow[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) hrow[mt] = hl + (size_t)min(mt * kTileM + col, Bg - 1) * pitch;
            floatx4 acc[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
            if constexpr (PLANES) {
                // the rolling prefetch of the branch below, on raw 16-byte chunks (half the
                // registers of the widened form, so twice the loads in flight)
                constexpr int UP = 2 * UNROLL;
                const uint16_t* hp[MT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) hp[mt] = hplane + (size_t)min(mt * kTileM + col, Bg - 1) * ppitch_h;
                const uint16_t* er = reinterpret_cast<const uint16_t*>(erow);
                uint4 eb[UP];
                const int klast = d - VEC;
#pragma unroll
                for (int uu = 0; uu < UP; ++uu) {
                    eb[uu] = load_chunk(er + min(uu * KSTEP + kq * VEC, klast));
                    __builtin_amdgcn_sched_barrier(0);
                }
                uint4 hn[MT][3];
                auto read_planes = [&](int k, uint4 (&dst)[MT][3]) {
                    const bool in = k < d;
                    const int kc = in ? k : 0;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int pnum = 0; pnum < 3; ++pnum) {
                            const uint4 h = *reinterpret_cast<const uint4*>(hp[mt] + pnum * plane_stride + kc);
                            dst[mt][pnum] = in ? h : make_uint4(0u, 0u, 0u, 0u);
                        }
                };
                read_planes(kq * VEC, hn);
                for (int ks0 = 0; ks0 < nks; ks0 += UP) {
#pragma unroll
                    for (int uu = 0; uu < UP; ++uu) {
                        const int k = (ks0 + uu) * KSTEP + kq * VEC;
                        uint4 hv[MT][3];
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                            for (int pnum = 0; pnum < 3; ++pnum) hv[mt][pnum] = hn[mt][pnum];
                        read_planes(k + KSTEP, hn);
                        const bf16x8 b = __builtin_bit_cast(bf16x8, eb[uu]);
#pragma unroll
                        for (int pnum = 0; pnum < 3; ++pnum)
#pragma unroll
                            for (int mt = 0; mt < MT; ++mt)
                                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                    __builtin_bit_cast(bf16x8, hv[mt][pnum]), b, acc[mt], 0, 0, 0);
                        eb[uu] = load_chunk(er + min(k + UP * KSTEP, klast));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            } else {
                // Rolling prefetch: UNROLL candidate-row loads stay in flight all the time.  Slot
                // uu is consumed (LDS read of the hidden rows, VEC matrix instructions) and at
                // once refilled with the chunk UNROLL k-steps ahead, so memory latency and
                // arithmetic overlap inside the wave instead of alternating.  Addresses past
                // the row are clamped into it (no branch around a load); such chunks meet
                // hidden values forced to zero.
                float ev[UNROLL][VEC];
                const int klast = d - VEC;
#pragma unroll
                for (int uu = 0; uu < UNROLL; ++uu) {
                    ElemTraits<ET>::load16(erow + min(uu * KSTEP + kq * VEC, klast), ev[uu]);
                    __builtin_amdgcn_sched_barrier(0);  // issue order = consumption order
                }
                // the hidden chunk of a slot is read from LDS one slot ahead, so that its latency
                // hides behind the previous slot's matrix instructions
                float hn[MT][VEC];
                auto read_hidden = [&](int k, float (&dst)[MT][VEC]) {
                    const bool in = k < d;
                    const int kc = in ? k : 0;
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int q = 0; q < VEC; q += 4) {
                            const float4 h4 = *reinterpret_cast<const float4*>(hrow[mt] + kc + q);
                            dst[mt][q] = in ? h4.x : 0.f; dst[mt][q + 1] = in ? h4.y : 0.f;
                            dst[mt][q + 2] = in ? h4.z : 0.f; dst[mt][q + 3] = in ? h4.w : 0.f;
                        }
                };
                read_hidden(kq * VEC, hn);
                for (int ks0 = 0; ks0 < nks; ks0 += UNROLL) {
#pragma unroll
                    for (int uu = 0; uu < UNROLL; ++uu) {
                        const int k = (ks0 + uu) * KSTEP + kq * VEC;
                        float hv[MT][VEC];
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                            for (int q = 0; q < VEC; ++q) hv[mt][q] = hn[mt][q];
                        read_hidden(k + KSTEP, hn);  // next slot (past the row: zeros)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                            for (int q = 0; q < VEC; ++q)
                                acc[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(hv[mt][q], ev[uu][q], acc[mt], 0, 0, 0);
                        // (unconditional: a branch around the load would make the compiler wait
                        // for every outstanding load at the top of the round; past the end of the
                        // row the clamped address re-reads its last chunk, a cache hit)
                        ElemTraits<ET>::load16(erow + min(k + UNROLL * KSTEP, klast), ev[uu]);
                        // keep the refill here: the scheduler would otherwise sink it towards
                        // its use a round later and leave one or two loads in flight
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            LSH_TRACE(1, 3);
            float out[MT * 4];
#pragma unroll
            for (int i = 0; i < MT * 4; ++i) out[i] = acc[i / 4][i % 4];
            settle_non_finite(out, [&](int i) {
                int quad = 4 * kq;
                asm volatile("" : "+v"(quad));   // (no address of this is worked out in advance)
                return plain_dot(erow, H + ((size_t)s * B + row0 + min(i / 4 * kTileM + quad + i % 4, Bg - 1)) * d, d);
            });
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int row = row0 + mt * kTileM + 4 * kq + r, c = n0 + col;
                    const bool valid = row < row0 + Bg && c < C;
                    const float x = out[4 * mt + r];
                    if (valid) logits[((size_t)s * B + row) * cpitch + c] = x;
                    tile_record_store<false, false>(recs, ((size_t)s * B + row) * recs.pitch + nt, row < row0 + Bg, valid,
                                             x, col, (int32_t)j);
                }
        }
        seg = seg_end;
    }
    LSH_TRACE(1, 4);

    // the remainder: one workgroup per tile, k split over its waves, hidden rows from LDS
    for (uint32_t t = wave_tiles + bx; t < total_tiles; t += wgs) {
        const int s = sentence_of(t);
        stage(s);
        const int nt = (int)xcd_tile(xcd_tiles(ntiles_of(s), (uint32_t)shared, (uint32_t)s, xcd), xcd, t - tile_pref[s]);
        const int C = count ? count[s] : V;
        const int cidx = min(nt * kTileN + col, C - 1);
        const int64_t j = cand ? cand[(size_t)s * V + cidx] : cidx;
        // (the split-k tile code reads fp32 rows as they are in memory: from there when LDS holds bf16 planes, or rows
        // that end in a partial chunk, which `stage` has moved)
        const bool as_is = !PLANES && d % VEC == 0;
        logits_tile_all_rows<ET, WAVES, (UNROLL < 4 ? UNROLL : 4), true, MT>(
            E, ld, d, H, B, s, nt, C, j, logits, cpitch, recs, red,
            as_is ? hl : nullptr, as_is ? pitch : 0, row0, row0 + Bg);
    }
}

// Many tiles.  What bounded k_logits_hlds was neither the fabric nor the matrix pipe but the load path of
// the CU: a lane that fetches the matrix operand it needs itself makes every 16 lanes touch 16 rows -- 16
// cache lines for 256 bytes.  Here candidate rows travel in contiguous pieces, straight from memory
// to LDS (global_load_lds, 16 bytes per lane, any row alignment), and the lanes pick their operands out of
// LDS.  What bounds it then is the instructions a wave issues (with every row in L2 it took as long), and how
// much of what several sentences want one L2 serves.  32 sentences x 10 beams, V = 40000, d = 1000 fp32 (261 MB of
// rows): 38 -> 33 us since the kernel works addresses out once per tile, has its loads between the matrix
// instructions and four units of them in flight; 64 x 10, V = 200000, d = 1024 bf16 (1.38 GB): 183 -> 136 us, 10 TB/s
// of rows; 8 x 5, d = 1024 bf16: 11.4 -> 10.4 us.
//
// The four waves of a workgroup share a tile, each with a quarter of k, and keep the A operands of all MT * 16
// hidden rows for their quarter in REGISTERS for as long as the workgroup stays with the sentence.  A step is 64
// bytes of every candidate row (16 fp32 values for four v_mfma_f32_16x16x4, or 32 bf16 for three
// v_mfma_f32_16x16x32_bf16, one per plane of the hidden values).  What a wave asks for at a time is a unit: KSN
// steps of TS tiles -- TS > 1 where rows are short, or one of PARTS parts of its quarter where they are
// long.  RING units' places in LDS per wave (four for long rows, two for short ones, whose units are larger): the
// others arrive while one is contracted.  GT tiles are summed and stored together.  The 16-byte piece p of row
// c lies at piece p ^ (c >> shift) of the row's place, so that 16 lanes reading the same piece of 16 rows meet
// different banks.  The quarters' partial tiles are summed through LDS in order; the results are stored behind the
// next unit's wait, so that the stores never stand between a wait and the loads it is for.
//
// The tiles of a sentence are dealt to the XCDs by their number (XcdTiles above).
constexpr int kStreamTiles = 32;   // tiles of a block, whose candidates come to LDS together
constexpr int stream_ts(int KSN, int MT) { return KSN == 4 ? (MT == 1 ? 2 : 1) : KSN == 1 ? (MT == 1 ? 4 : 2) : MT == 1 ? 2 : 1; }
// Workgroups per CU: the registers of the A operands, and LDS -- of one row group of long rows, 76 KB, two.
constexpr int stream_wgs(bool bf16, int MT, int KSN, int PARTS) { return KSN == 4 && MT == 1 ? 2 : (bf16 ? 3 : 1) * MT * KSN * PARTS * 4 <= (bf16 ? 96 : 80) ? 3 : 2; }
// Its LDS: the waves' partial tiles, the waves' rings, two blocks of candidates, and what the workgroup takes (for an even cut,
// the tiles in front of every 64 sentences).  (The same for any number of sentences.  With tables of all of them only one workgroup of long rows
// ran on a CU from 510 sentences on: fp32, V = 5000, d = 1000: 600 x 2 beams 188 us a step, 83 so; 2048 x 1 542, 199.)
template <int MT, int KSN> struct StreamLds {
    static constexpr int TS = KSN == 4 ? 1 : stream_ts(KSN, MT);                   // tiles of a unit
    static constexpr int RING = KSN == 4 ? 2 * stream_ts(KSN, MT) : 2;             // units' places per wave
    static constexpr int GT = stream_ts(KSN, MT);                                  // tiles whose quarters are summed together
    static constexpr int NI = TS * KSN;                                            // load instructions of a unit, KiB of its place
    static constexpr size_t kRed = (size_t)4 * GT * MT * 4 * kWave * 4, kRings = (size_t)4 * RING * NI * 1024;
    static constexpr size_t kIds = kRed + kRings, kPref = kIds + (size_t)2 * kStreamTiles * kTileN * 4;
    static constexpr size_t kBytes = kPref + kWave * 4;
};
// Whether steps of a row's last part that are past its end are left out: of two or three parts of rows that have such steps, and
// where a step is dear.  (The branches cost more than they save where there are none.  fp32, us a step without and with them:
// 100 x 24 beams, d = 264, V = 30000, five steps of eight: 148, 120; d = 520, nine of twelve: 196, 178; d = 400, seven of eight:
// 140, 132; d = 512, all eight: 137.6, 138.9; 32 x 10, d = 264: 37.6, 35.1; d = 512: 37.2, 37.5; d = 800, 13 of 16: 48.3, 48.2.)
constexpr bool stream_may_trim(int PARTS) { return PARTS == 2 || PARTS == 3; }
constexpr bool stream_must_trim(bool bf16, int PARTS) { return bf16 && PARTS > 3; }
// Of the workgroups on a CU the one that came first takes the issue slots that both want: of two with as many tiles the other was a
// fifth slower and then had the CU to itself, half used.  (The first 256 workgroups of a launch go to a CU each.)  So the waves of the
// others have the higher priority in a part of their groups of tiles: in five of eight, and as good as always in the first eight,
// for workgroups that have no more.  64 x 10 beams, V = 200000, d = 1024 bf16: workgroups took 74 to 109 us for equal shares, 101 to
// 120 so; a step over one input 154.4 -> 144.0 us (half of the groups 145.8, six of eight 146.4, all of them 154.2), over changing ones 157.2 ->
// 150.2, as sentences that go through the vocabulary side by side find more in L2 (0.53 GB instead of 0.72 from memory); 32 x 10, V = 40000, d = 1000 fp32, four groups: 45.5 -> 44.4 (half 45.4).  Where three share a CU the second and the third have it: 20 x 20 to
// 60 x 24 beams, d = 100 to 512 bf16, V = 60000 0.98 to 1.00 of the time, 24 x 32, d = 100 45.7 -> 44.5; fp32 20 x 20, d = 200 42.7 -> 42.3, 60 x 30,
// d = 300 120.6 -> 118.7, d = 64 98.2 -> 98.8; up to 6 hidden rows 1.00 to 1.004.
constexpr uint32_t kCus = 256;
__device__ __forceinline__ bool young_first(int g) { return (g < 8 ? 0xFE : 0xB6) >> (g & 7) & 1; }
// Whether the hidden rows (bf16 words; that many in a workgroup's group) come through LDS (STAGE).  A lane that loads its operand itself, two
// pieces of 16 bytes, has every 16 lanes touch as many rows twice as there are hidden rows, 16 at most; through LDS each takes a trip more, and
// rows that only fill a group of 16 cost as much as others.  us a step without and with (V = 40000 .. 60000): d = 1536, 32 x 16 beams 44.3, 39.8, 24 x 6
// 28.9, 27.3, 24 x 3 26.1, 25.3, 40 x 1 26.9, 26.7; d = 1064 (two of three parts in the ring) 40.0, 38.6, 28.2, 27.6, 26.0, 26.1, 24 x 2 24.0, 24.3; d = 1024
// 36.0, 34.1, 24.9, 24.6, 23.0, 22.8, 40 x 1 23.7, 23.9; d = 640 35.5, 34.5, 25.1, 25.1, 23.5, 23.6, 24 x 2 22.2, 22.5; d = 512 29.5, 27.7, 24 x 8 21.9, 21.8, 24 x 4
// 19.9, 20.1, 24 x 2 18.9, 19.3; d = 256 27.4, 26.7, 20.4, 20.3, 18.0, 18.2; d = 96 29.6, 29.5, 20.0, 20.3, 24 x 12 22.1, 22.4; two row groups: 24 x 32, d = 512 45.9,
// 43.9, d = 256 40.1, 39.1, d = 100 45.0, 44.5.  64 x 10, V = 200000, d = 1024 99.6, 98.3 (lists of 6000).  With fp32 words, one piece: 32 x 10, d = 1000, 44.7, 45.1.
// Units that the ring does not hold are loaded behind it; their lines brought to L2 in front cost more (32 x 10, d = 1536 34.5 -> 34.9; 8 x 32, d = 512 32.0 -> 32.4).
// Hidden rows of an odd number of values start at odd multiples of 4 bytes, which costs a lane that loads its own 16 bytes more than it costs LDS: 12 x 2, d = 683
// 21.6, 21.1, d = 1001 21.8, 21.2, d = 511 18.4, 18.1; 40 x 1, d = 901 26.4, 25.8, d = 399 22.0, 21.6; 32 x 4, d = 301 22.9, 22.1; d = 201, 16 x 1 16.1, 16.3, 32 x 2 18.9, 18.7; but
// d = 602, 32 x 2 23.6, 23.7.
constexpr bool stream_stages(bool bf16, int KSN, int rows, bool odd) {
    return bf16 && rows >= (KSN == 1 ? 17 : odd ? 1 : KSN == 2 ? 8 : 3);
}
// f(integral_constant 0), ..., f(integral_constant N - 1)
template <int N, int I = 0, typename F> __device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

__device__ __forceinline__ TileRun uniform(const TileRun& r) {
    return {wave_read_lane(r.n, 0), wave_read_lane(r.head, 0), wave_read_lane(r.a0, 0), wave_read_lane(r.a1, 0), wave_read_lane(r.b0, 0), wave_read_lane(r.b1, 0)};
}
// The sentence of workgroup bx of XCD x, its candidates and its tiles.
struct StreamDeal { uint32_t s, C; TileRun run; };
// w0: weights of the sentences in front of s, w1: with its own, W: of all.
__device__ __forceinline__ StreamDeal deal_by_weight(uint32_t s, uint32_t C, uint32_t w0, uint32_t w1, uint32_t W, uint32_t G,
                                                     uint32_t shared, uint32_t x, uint32_t bx) {
    const uint32_t ln = lane_id();                                            // (lane i: XCD i)
    const uint32_t b0 = dealt_from(w0, ln & 7u, W, G), n = dealt_from(w1, ln & 7u, W, G) - b0, incl = wave_incl_scan(ln < 8u ? n : 0u);
    const uint32_t mine = wave_read_lane(n, (int)x), before = wave_read_lane(incl, (int)x) - mine;
    return {s, C, dealt_run((C + kTileN - 1u) / kTileN, shared, bx - wave_read_lane(b0, (int)x), mine, before, wave_read_lane(incl, 7))};
}
// The same number for every sentence (per > 0), or dealt as equally as they come.
__device__ __forceinline__ StreamDeal deal_equally(const int32_t* __restrict__ count, int V, uint32_t S, uint32_t G, uint32_t per,
                                                   uint32_t shared, uint32_t x, uint32_t bx, uint32_t s) {
    const uint32_t C = (uint32_t)__builtin_amdgcn_readfirstlane(count ? count[s] : V);
    if (per == 0) return deal_by_weight(s, C, s, s + 1u, S, G, shared, x, bx);
    const XcdTiles xt = xcd_tiles((C + kTileN - 1u) / kTileN, shared, s, x);
    const uint32_t first = bx - s * per;
    return {s, C, xcd_run(xt, x, first, per, xt.n > first ? (xt.n - first + per - 1u) / per : 0u)};
}
__device__ __forceinline__ uint32_t tiles_in(const int32_t* __restrict__ count, uint32_t s, uint32_t S) {   // (no branch around the load)
    return ((uint32_t)count[min(s, S - 1u)] + kTileN - 1u) / kTileN;
}
// Whether the lists' lengths ask for shares by weight (dealt_by_count); the tiles of all lists.
__device__ __forceinline__ bool lists_differ(const int32_t* __restrict__ count, uint32_t S, uint32_t G, int row_bytes, uint32_t* all) {
    constexpr uint32_t AT_ONCE = 6;
    const uint32_t ln = lane_id();
    uint32_t most = 0, sum = 0;
    for (uint32_t c = 0; c < S; c += AT_ONCE * kWave) {
        uint32_t n[AT_ONCE];
#pragma unroll
        for (uint32_t j = 0; j < AT_ONCE; ++j) n[j] = tiles_in(count, c + j * kWave + ln, S);
#pragma unroll
        for (uint32_t j = 0; j < AT_ONCE; ++j) { most = max(most, n[j]); sum += c + j * kWave + ln < S ? n[j] : 0u; }
    }
    *all = wave_sum(sum);
    return dealt_by_count((uint32_t)wave_max_f32((float)most), *all, S, G, row_bytes);
}
__device__ __forceinline__ StreamDeal deal_by_count(const int32_t* __restrict__ count, uint32_t S, uint32_t G, uint32_t sum,
                                                    uint32_t shared, uint32_t x, uint32_t bx) {
    const uint32_t ln = lane_id(), least = least_weight(sum, S, G);
    uint32_t W = 0, w0 = 0, w1 = 1, s = 0, front = 0;
    for (uint32_t c = 0; c < S; c += kWave) W += wave_sum(c + ln < S ? max(tiles_in(count, c + ln, S), least) : 0u);
    for (uint32_t c = 0; c < S; c += kWave) {
        const uint32_t w = c + ln < S ? max(tiles_in(count, c + ln, S), least) : 0u, incl = front + wave_incl_scan(w);
        const uint64_t begun = __ballot(c + ln < S && dealt_from(incl - w, x, W, G) <= bx);   // (the last of them has bx)
        if (begun == 0ull) break;
        const int i = kWave - 1 - __clzll(begun);
        s = c + i;
        w1 = wave_read_lane(incl, i);
        w0 = w1 - wave_read_lane(w, i);
        front = wave_read_lane(incl, kWave - 1);
    }
    return deal_by_weight(s, (uint32_t)__builtin_amdgcn_readfirstlane(count[s]), w0, w1, W, G, shared, x, bx);
}

// STAGE: see stream_stages.
template <typename ET, int MT, int KSN, int PARTS, bool EVEN, bool TRIM, bool STAGE = false>
__global__ void __launch_bounds__(256, (stream_wgs(sizeof(ET) == 2, MT, KSN, PARTS)))
k_logits_stream(const ET* __restrict__ E, int64_t ld, int d, const float* __restrict__ H, int S, int B,
                int group_rows /*row group g takes rows [g, g + 1) * group_rows of every sentence; <= 16 MT*/,
                int wgs /*workgroups per XCD and row group*/, int ngroups,
                int per /*workgroups per XCD and sentence; 0: dealt*/,
                int shared, const int32_t* __restrict__ cand, const int32_t* __restrict__ count, int V,
                float* __restrict__ logits, int64_t cpitch, TileRecords recs) {
    constexpr bool BF = sizeof(ET) == 2;
    constexpr int VEC = ElemTraits<ET>::VEC, KSTEP = 4 * VEC;
    constexpr int PP = 4 * KSN;                                               // 16-byte pieces of a row in a unit
    static_assert(KSN == 1 || KSN == 2 || KSN == 4, "");
    constexpr int SH = PP == 4 ? 2 : PP == 8 ? 1 : 0;
    using Lds = StreamLds<MT, KSN>;
    constexpr int TS = Lds::TS, RING = Lds::RING, GT = Lds::GT, GU = GT / TS; // GU: units of a part of GT tiles
    // 16-byte registers of A operands per step and row group: fp32 values; their three bf16 planes; for four parts
    // those registers run out, and the values are split when they are used
    constexpr bool LATE = BF && PARTS > 3;
    constexpr int NH = LATE ? 2 : BF ? 3 : 1;
    constexpr int NI = Lds::NI;
    // Chains of sums per quarter: a part's products go to chain part % CHAINS.  More than one for fp32 rows of more than 1024
    // values, so that the full vocabulary's logits are as near as those of k_logits_rows, which took some of
    // these calls before this kernel was faster: root mean square over the products' sizes, V = 2000, 8 x 16 rows, dense: d = 1100
    // 0.91e-8 there, 1.42e-8 with one chain, 0.77e-8 with four (8 x 16, 32.1, 23.8, 22.3 us); d = 1536 0.93, 1.41, 0.78 (45.7,
    // 27.3, 25.6); hidden rows near words: 2.58e-8, 2.24, 1.05.
    constexpr int CHAINS = !BF && !EVEN && PARTS > 4 ? 4 : 1;
    constexpr int RPI = kWave / PP;                                           // rows per load instruction
    extern __shared__ uint4 ssm[];
    // (the ring behind other things: the address in M0 is its place less the load's offset, and must not be negative)
    char* sm = reinterpret_cast<char*>(ssm);
    float (*red)[GT][MT][4][kWave] = reinterpret_cast<float (*)[GT][MT][4][kWave]>(sm);   // [wave]
    static_assert(Lds::kRed >= (PARTS - 1) * KSN * 64, "");
    int32_t* ids = reinterpret_cast<int32_t*>(sm + Lds::kIds);                         // [two blocks of tiles][16]
    uint32_t* shares = reinterpret_cast<uint32_t*>(sm + Lds::kPref);                       // [64]: a StreamDeal; EVEN: tiles in front of every 64 sentences
    // grid = 8 * wgs * ngroups; ids go round the XCDs, the row groups of one block of tiles follow each other on one
    const uint32_t xcd = blockIdx.x & 7u, slot_x = blockIdx.x >> 3;
    const uint32_t bx = slot_x / (uint32_t)ngroups;
    const bool young = blockIdx.x >= kCus;
    const int row0 = (int)(slot_x % (uint32_t)ngroups) * group_rows, Bg = min(group_rows, B - row0);
    const int tid = threadIdx.x, ln = lane_id(), q = __builtin_amdgcn_readfirstlane(wave_id());   // q: the wave's quarter of k
    const int col = ln & 15, kq = ln >> 4;
    char* ring = sm + Lds::kRed + q * (RING * NI * 1024);
    const uint32_t ring_at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring);
    auto ntiles_of = [&](int C) { return (uint32_t)((C + kTileN - 1) / kTileN); };
    const int nks = (d + KSTEP - 1) / KSTEP, nst = (nks + 3) >> 2, k0 = q * nst * KSTEP;   // steps of a wave's quarter
    // STAGE: as many units of the hidden rows of the sentence known in front (part p of row group m is number m PARTS + p) as the ring
    // holds come there, where nothing is yet, while the count and the candidates are on their way.  Pieces of a row lie as those of
    // the words do, in blocks of PPH.
    constexpr int SB = VEC / 4, PPH = 4 * KSN * SB < 16 ? 4 * KSN * SB : 16, SUBS = 4 * KSN * SB / PPH, SHH = PPH == 4 ? 2 : PPH == 8 ? 1 : 0;
    constexpr int UNITS = MT * PARTS, HELD = RING * NI / (KSN * SB), STAGED = !STAGE ? 0 : HELD < UNITS ? HELD : UNITS;
    static_assert(!STAGE || !EVEN, "an even cut knows no sentence in front");
    auto stage_hidden = [&](int at_s) __attribute__((always_inline)) {
        const float* hb = H + ((size_t)at_s * B + row0) * d;
        const int lrow = ln / PPH, lp = ln % PPH;
#pragma unroll
        for (int i = 0; i < STAGED * SUBS; ++i)
#pragma unroll
            for (int j = 0; j < PPH / 4; ++j) {
                const int part = i / SUBS % PARTS, row = j * (kWave / PPH) + lrow, p = i % SUBS * PPH + (lp ^ (row >> SHH));
                const int k = p / SB < 4 * (nst - part * KSN) ? k0 + part * (KSN * KSTEP) + p / SB * VEC : d;
                load_to_lds16(hb + (size_t)min(i / SUBS / PARTS * kTileM + row, Bg - 1) * d + min(k, d - VEC) + 4 * (p % SB), ring + i * (PPH * 256) + j * 1024);
            }
    };
    LSH_TRACE_WG(8);
    // Who takes what.  A workgroup has one sentence, and all or some of the sentence's workgroups take turns:
    //   per > 0: workgroup i of a sentence's `per` on this XCD has the tiles i, i + per, ... of those of the XCD (XcdTiles);
    //   per = 0, where that would leave many without work, and where lists are of very different lengths: as dealt_from and
    //   dealt_run say.  (40 sentences x 6, d = 1096 fp32: 48 us cut evenly, 40 dealt; 33 x 15: 44, 39.5.)
    //   EVEN (more sentences than such shares suit: launch_logits_stream): the tiles of all
    //   sentences in a row, cut evenly.
    int s = 0, C = 0;
    TileRun run{};
    uint32_t seg = 0, seg_end = 0, wg_end = 0;
    uint32_t s0 = 0;                                                          // the sentence known in front
    bool moved = false;                                                       // (uniform) it is another now
    auto count_of = [&](int at) { const int n = count ? count[min(at, S - 1)] : V; return at < S ? n : 0; };
    if constexpr (!EVEN) {
        s0 = __builtin_amdgcn_readfirstlane(per > 0 ? bx / (uint32_t)per : dealt_sentence(bx, xcd, (uint32_t)S, (uint32_t)wgs));
        if constexpr (STAGED > 0) stage_hidden((int)s0);
        else {   // the hidden rows' lines into this XCD's L2 (and the ring, where nothing is yet) while the count is on its way
            const char* hb = reinterpret_cast<const char*>(H + ((size_t)s0 * B + row0) * d);
            if (q > 0)
                for (uint32_t at = (tid - kWave) * 128u; at < (uint32_t)(Bg * d) * 4u; at += 192u * 128u) load_to_lds4(hb + at, ring);
        }
        const StreamDeal dl = deal_equally(count, V, (uint32_t)S, (uint32_t)wgs, (uint32_t)per, (uint32_t)shared, xcd, bx, s0);
        s = (int)dl.s; C = (int)dl.C; run = uniform(dl.run);
    } else {   // (every wave for itself, to the same result)
        static_assert(kMaxSentencesLogits <= kWave * kWave, "a lane per 64 sentences");
        constexpr int AHEAD = 8;
        uint32_t total = 0, in_front = ~0u;                                   // (lane c: tiles in front of sentence 64 c)
        for (int c0 = 0; c0 * kWave < S; c0 += AHEAD) {
            int n[AHEAD];
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) n[j] = count_of((c0 + j) * kWave + ln);
#pragma unroll
            for (int j = 0; j < AHEAD; ++j) {
                if (ln == c0 + j && (c0 + j) * kWave < S) in_front = total;
                total += wave_sum(ntiles_of(n[j]));
            }
        }
        shares[ln] = in_front;
        const uint32_t per_wg = (total + 8u * (uint32_t)wgs - 1u) / (8u * (uint32_t)wgs);
        seg = min(total, (xcd * (uint32_t)wgs + bx) * per_wg);
        wg_end = min(total, seg + per_wg);
        if (seg == wg_end) return;
    }
    // parts of which the wave's quarter has every piece, inside the row
    const int last_steps = nst - (PARTS - 1) * KSN;                           // steps of the last part
    uint32_t whole_parts = 0;
#pragma unroll
    for (int p = 0; p < PARTS; ++p)
        if (nst - p * KSN >= KSN && k0 + (p + 1) * KSN * KSTEP <= d) whole_parts |= 1u << p;
    // piece (4 st + kq) of row col: the low two bits of st change lanes' places, the others move on
    const char* place[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) place[j] = ring + (col * PP + (((4 * j + kq) & (PP - 1)) ^ (col >> SH))) * 16;
    // instruction i of a tile brings its pieces 64 i .. 64 i + 63: row i RPI + lr, piece swz ^ (i RPI >> SH)
    const int lr = ln / PP, swz = (ln % PP) ^ (lr >> SH);
    uint32_t loff[KSN];                                                       // byte of its row a lane brings in part 0
#pragma unroll
    for (int i = 0; i < KSN; ++i) loff[i] = (uint32_t)(16 * (swz ^ (i * RPI >> SH))) + (uint32_t)(k0 * (int)sizeof(ET));
    const uint32_t ld_bytes = (uint32_t)(ld * (int64_t)sizeof(ET));           // (the host: below 2^31)
    for (;;) {
        if constexpr (EVEN) {   // the last sentence with at most `seg` tiles in front of it
            const uint32_t in_front = shares[ln];
            const int c = kWave - 1 - __clzll(__ballot(in_front <= seg)), at = c * kWave + ln, mine = count_of(at);
            const uint32_t incl = wave_read_lane(in_front, c) + wave_incl_scan(ntiles_of(mine)), pref = incl - ntiles_of(mine);
            const int i = kWave - 1 - __clzll(__ballot(at < S && pref <= seg));
            s = c * kWave + i;
            C = wave_read_lane((uint32_t)mine, i);
            seg_end = min(wg_end, wave_read_lane(incl, i));
            run = {seg_end - seg, 0u, 0u, 0u, seg - wave_read_lane(pref, i), 1u};
        }
        int n = (int)run.n;
        auto tile_of = [&](int t) __attribute__((always_inline)) { return (int)run.tile((uint32_t)t); };
        // candidates of block b (kStreamTiles tiles): two loads per wave
        auto load_ids1 = [&](int b, int e) __attribute__((always_inline)) {       // 64 of them, from the e-th on
            const int c = min(tile_of(min(b * kStreamTiles + (e + ln) / kTileN, n - 1)) * kTileN + col, C - 1);   // clamped columns are never stored
            int32_t* to = ids + (b & 1) * kStreamTiles * kTileN + e;
            if (cand) load_to_lds4(cand + (size_t)s * V + c, to); else to[ln] = c;
        };
        auto load_ids = [&](int b) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < kStreamTiles * kTileN / 256; ++j) load_ids1(b, q * (kStreamTiles * kTileN / 4) + j * kWave);
        };
        if (EVEN || (q > 0 && n > 0)) load_ids(0);
        if constexpr (!EVEN) {
            // (The first wave reads all counts while the others' candidates come, its own share of those among them: 0.6 us less than
            // before them.)
            if (q == 1 || q == 2) { if (n > 0) load_ids1(0, (q - 1) * kWave); }
            if (q == 0) {
                uint32_t all = 0;
                const bool differ = count && lists_differ(count, (uint32_t)S, (uint32_t)wgs, d * (int)sizeof(ET), &all);
                if (differ) {
                    const StreamDeal dl = deal_by_count(count, (uint32_t)S, (uint32_t)wgs, all, (uint32_t)shared, xcd, bx);
                    if (ln == 0) {
                        shares[0] = dl.s; shares[1] = dl.C; shares[2] = dl.run.n; shares[3] = dl.run.head;
                        shares[4] = dl.run.a0; shares[5] = dl.run.a1; shares[6] = dl.run.b0; shares[7] = dl.run.b1;
                    }
                }
                if (ln == 0) shares[8] = differ;
            }
        }
        wait_vmem<0>();
        lds_barrier();
        if constexpr (!EVEN) {
            if (wave_read_lane(shares[8], 0)) {
                const uint4 x = reinterpret_cast<const uint4*>(shares)[0], y = reinterpret_cast<const uint4*>(shares)[1];
                s = wave_read_lane(x.x, 0); C = wave_read_lane(x.y, 0);
                run = uniform(TileRun{x.z, x.w, y.x, y.y, y.z, y.w});
                n = (int)run.n;
                moved = s != (int)s0;
                if (n > 0) {
                    load_ids(0);
                    wait_vmem<0>();
                    lds_barrier();
                }
            }
            if (n == 0) return;
        }
        LSH_TRACE_WG(9);
        const int groups = (n + GT - 1) / GT, sets = (n + TS - 1) / TS, units = sets * PARTS;
        // unit u = part u % PARTS of the TS tiles of set u / PARTS; ptr: the addresses of its tiles' part 0
        const char* ptr[TS][KSN];
        auto address = [&](int g) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                const int32_t* at = ids + (min(g * TS + t, n - 1) & (2 * kStreamTiles - 1)) * kTileN + lr;
#pragma unroll
                for (int i = 0; i < KSN; ++i) ptr[t][i] = reinterpret_cast<const char*>(E) + ((uint64_t)(uint32_t)at[i * RPI] * ld_bytes + loff[i]);
            }
        };
        // where a lane's pieces of a unit's part are: ptr, but for pieces past the quarter (not needed) and past the row,
        // which are the row's last chunk
        const char* from[TS][KSN];
        auto locate = [&](auto part_c) __attribute__((always_inline)) {
            constexpr int part = decltype(part_c)::value;
            const bool is_whole = whole_parts >> part & 1u;                   // (uniform)
#pragma unroll
            for (int i = 0; i < KSN; ++i) {
                int64_t move = 0;
                if (!is_whole) {
                    int p = swz ^ (i * RPI >> SH);
                    asm volatile("" : "+v"(p));   // (every part's offsets worked out in advance would take too many registers)
                    const int left = 4 * (nst - part * KSN);
                    const int k = p < left ? min(k0 + part * (KSN * KSTEP) + p * VEC, d - VEC) : d - VEC;
                    move = k * (int)sizeof(ET) - (int)loff[i] - part * KSN * 64;
                }
#pragma unroll
                for (int t = 0; t < TS; ++t) from[t][i] = is_whole ? ptr[t][i] : ptr[t][i] + move;
            }
        };
        // the loads of a unit of that part, step i of its tiles; at: LDS address of its place
        auto fill1 = [&](auto part_c, uint32_t at, auto i_c) __attribute__((always_inline)) {
            constexpr int off = decltype(part_c)::value * KSN * 64, i = decltype(i_c)::value;
            static_for<TS>([&](auto t) __attribute__((always_inline)) {
                load_to_lds16_at<(decltype(t)::value * KSN + i) * 1024, off>(from[decltype(t)::value][i], at);
            });
        };
        auto fill_ring = [&]() __attribute__((always_inline)) {
            static_for<RING>([&](auto u_c) __attribute__((always_inline)) {
                constexpr int u = decltype(u_c)::value;
                using Part = std::integral_constant<int, u % PARTS>;
                if (u < units) {
                    if constexpr (u % PARTS == 0) address(u / PARTS);
                    locate(Part{});
                    static_for<KSN>([&](auto i) __attribute__((always_inline)) { fill1(Part{}, ring_at + u * (NI * 1024), i); });
                }
            });
        };
        // A operands: hidden row col of every row group (clamped: results dropped), zeros past d; a partial chunk
        // holds the row's last VEC values, those counted already replaced by zero, as `fill1` reads it
        uint4 h[MT][PARTS * KSN][NH];
        const float* hb = H + ((size_t)s * B + row0) * d;
        auto keep = [&](int m, int st, float (&x)[VEC]) __attribute__((always_inline)) {
            const int k = st < nst ? k0 + st * KSTEP + kq * VEC : d, drop = k - min(k, d - VEC);
#pragma unroll
            for (int e = 0; e < VEC; ++e) x[e] = e >= drop ? x[e] : 0.f;
            if constexpr (LATE) {
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    h[m][st][e] = make_uint4(__float_as_uint(x[4 * e]), __float_as_uint(x[4 * e + 1]), __float_as_uint(x[4 * e + 2]), __float_as_uint(x[4 * e + 3]));
            } else if constexpr (BF) split_planes8(x, h[m][st]);
            else h[m][st][0] = make_uint4(__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3]));
        };
        auto load_hidden = [&](auto from_c) __attribute__((always_inline)) {       // units from the from-th on
#pragma unroll
            for (int i = decltype(from_c)::value * KSN; i < MT * PARTS * KSN; ++i) {
                const int m = i / (PARTS * KSN), st = i % (PARTS * KSN);
                const float* hrow = hb + (size_t)min(m * kTileM + col, Bg - 1) * d;
                const int k = st < nst ? k0 + st * KSTEP + kq * VEC : d, at = min(k, d - VEC);
                float x[VEC];
#pragma unroll
                for (int e = 0; e < VEC; e += 4) {
                    const Float4U v = *reinterpret_cast<const Float4U*>(hrow + at + e);
                    x[e] = v.x; x[e + 1] = v.y; x[e + 2] = v.z; x[e + 3] = v.w;
                }
                if ((st & (BF ? 1 : 3)) == (BF ? 1 : 3)) __builtin_amdgcn_sched_barrier(0);   // (a few addresses at a time)
                keep(m, st, x);
            }
        };
        if (STAGED == 0 || moved) {   // (uniform)
            fill_ring();
            load_hidden(std::integral_constant<int, 0>{});
        } else {   // (the candidates are asked for before the values are split: 12 x 12 beams, d = 640, V = 100000 31.8 -> 31.1 us a step)
            float x[STAGED * KSN + 1][VEC];
#pragma unroll
            for (int i = 0; i < STAGED * KSN; ++i)
#pragma unroll
                for (int e = 0; e < SB; ++e) {
                    const int p = (i % KSN * 4 + kq) * SB + e;                // (p / PPH does not depend on the lane)
                    const uint4 v = *reinterpret_cast<const uint4*>(ring + (i / KSN * SUBS + (i % KSN * 4 * SB) / PPH) * (PPH * 256) + (col * PPH + ((p % PPH) ^ (col >> SHH))) * 16);
                    x[i][4 * e] = __uint_as_float(v.x); x[i][4 * e + 1] = __uint_as_float(v.y); x[i][4 * e + 2] = __uint_as_float(v.z); x[i][4 * e + 3] = __uint_as_float(v.w);
                }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                // (they have left the ring)
            __builtin_amdgcn_sched_barrier(0);
            fill_ring();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < STAGED * KSN; ++i) keep(i / (PARTS * KSN), i % (PARTS * KSN), x[i]);
            load_hidden(std::integral_constant<int, STAGED>{});
        }
        if (STAGED < UNITS || moved) __builtin_amdgcn_s_waitcnt(0x0F70);       // vmcnt(0): the compiler must not wait for them in the loop
        __builtin_amdgcn_sched_barrier(0);
        LSH_TRACE_WG(10);
        float out[GT][MT];
        // thread (i, col) has row 16 m + i, column col of every tile: 16 lanes per row (waves without rows: nothing)
        float* lrow = logits + ((size_t)s * B + row0 + (tid >> 4)) * cpitch + col;
        float2* rrow = reinterpret_cast<float2*>(recs.rec) + ((size_t)s * B + row0 + (tid >> 4)) * recs.pitch;
        uint32_t again = 0;                                                   // a bit for every tile of the block with logits to settle
        // As settle_non_finite, with the logits each thread has stored, for the tiles of a block.
        auto settle = [&](int t0) __attribute__((always_inline)) {
            for (uint32_t left = again; left; left &= left - 1u) {
                int me = tid;
                asm volatile("" : "+v"(me));   // (nothing of this is kept in registers during the loop)
                const int t = t0 + __ffs(left) - 1, nt = tile_of(t);
                const bool in = nt * kTileN + (me & 15) < C;
                const ET* row = E + (int64_t)ids[(t & (2 * kStreamTiles - 1)) * kTileN + (me & 15)] * ld;
#pragma unroll 1
                for (int m = 0; m < MT && 4 * q + m * kTileM < Bg; ++m) {     // (uniform: four rows per wave)
                    const int r = (me >> 4) + m * kTileM;
                    float* at = lrow + (size_t)(m * kTileM) * cpitch + nt * kTileN;
                    float x = in && r < Bg ? *at : -INFINITY;
                    if (in && r < Bg && !(fabsf(x) < INFINITY)) *at = x = plain_dot(row, hb + (size_t)r * d, d);
                    const float mx = row16_max(x);
                    const float se = row16_sum(in && r < Bg ? exp_below(x, mx) : 0.f);
                    if ((me & 15) == 0 && r < Bg) rrow[(size_t)(m * kTileM) * recs.pitch + nt] = make_float2(mx, se);
                }
            }
            again = 0;
        };
        // (without branches up to the stores: the tiles' chains of dependent instructions run side by side)
        auto store_out = [&](int g) __attribute__((always_inline)) {
            if (4 * q >= Bg) return;                                          // (uniform)
            float mx[GT][MT], se[GT][MT];
            int nt[GT];
            bool valid[GT][MT];
#pragma unroll
            for (int t = 0; t < GT; ++t) {
                nt[t] = tile_of(g * GT + t);
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    valid[t][m] = (tid >> 4) + m * kTileM < Bg && g * GT + t < n && nt[t] * kTileN + col < C;
            }
#pragma unroll
            for (int t = 0; t < GT; ++t)
#pragma unroll
                for (int m = 0; m < MT; ++m) mx[t][m] = row16_max(valid[t][m] ? out[t][m] : -INFINITY);
#pragma unroll
            for (int t = 0; t < GT; ++t)
#pragma unroll
                for (int m = 0; m < MT; ++m) se[t][m] = row16_sum(valid[t][m] ? exp_below(out[t][m], mx[t][m]) : 0.f);
#pragma unroll
            for (int t = 0; t < GT; ++t)
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    if (valid[t][m]) lrow[(size_t)(m * kTileM) * cpitch + nt[t] * kTileN] = out[t][m];
                    // (column 0 of a tile is always a candidate)
                    if (valid[t][m] && col == 0) rrow[(size_t)(m * kTileM) * recs.pitch + nt[t]] = make_float2(mx[t][m], se[t][m]);
                    // (a NaN or +inf among the logits.  -inf is right: a value's planes, each cut off, agree in sign)
                    if (__builtin_expect(__ballot(se[t][m] != se[t][m]) != 0ull, 0)) again |= 1u << ((g * GT + t) & (kStreamTiles - 1));
                }
            // (a block's candidates are replaced a barrier after its last tile at the earliest)
            const int last = min(g * GT + GT, n) - 1;
            if (__builtin_expect(again != 0u, 0) && ((last & (kStreamTiles - 1)) == kStreamTiles - 1 || last == n - 1)) settle(last & ~(kStreamTiles - 1));
        };
        floatx4 acc[CHAINS][GT][MT];
        uint32_t slot = 0;                                                    // byte of the ring where the next unit is
        // The units of a group.  STEADY: every one of them is there and is followed by another RING units on.
        auto contract = [&](auto steady_c, int g) __attribute__((always_inline)) {
            constexpr bool STEADY = decltype(steady_c)::value;
            static_for<GU * PARTS>([&](auto i_c) __attribute__((always_inline)) {
                constexpr int part = decltype(i_c)::value % PARTS, gu = decltype(i_c)::value / PARTS, next = (part + RING) % PARTS;
                using Next = std::integral_constant<int, next>;
                if (!STEADY && gu > 0 && g * GU + gu >= sets) return;         // (uniform: the last group's)
                const int u = (g * GU + gu) * PARTS + part;
                // (the unit's own loads are older than those of the units behind it, NI each)
                if (STEADY || u + RING - 1 < units) wait_vmem<(RING - 1) * NI>(); else wait_vmem<0>();
                uint4 ev[TS][KSN];
#pragma unroll
                for (int t = 0; t < TS; ++t)
#pragma unroll
                    for (int st = 0; st < KSN; ++st)
                        ev[t][st] = *reinterpret_cast<const uint4*>(place[st & 3] + slot + t * (KSN * 1024) + (st >> 2) * 256);
                const bool more = STEADY || u + RING < units;
                if constexpr (next == 0) address(min(g * GU + gu + (part + RING) / PARTS, sets - 1));
                locate(Next{});
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // (every operand has left the unit's place)
                __builtin_amdgcn_sched_barrier(0);
                static_for<KSN>([&](auto st_c) __attribute__((always_inline)) {
                    constexpr int st = decltype(st_c)::value;
                    // (steps past the quarter meet zeros, or, TRIM, are left out)
                    const bool is_step = !TRIM || part < PARTS - 1 || st == 0 || st < last_steps;   // (uniform)
#pragma unroll
                    for (int t = 0; t < TS && is_step; ++t) {
                        const uint4 e = ev[t][st];
                        const uint32_t ew[4] = {e.x, e.y, e.z, e.w};
                        if constexpr (BF) {
#pragma unroll
                            for (int m = 0; m < MT; ++m) {
                                uint4 hp[3];
                                if constexpr (LATE) {
                                    const uint4 a = h[m][part * KSN + st][0], b = h[m][part * KSN + st][1];
                                    float x[8] = {__uint_as_float(a.x), __uint_as_float(a.y), __uint_as_float(a.z), __uint_as_float(a.w),
                                                  __uint_as_float(b.x), __uint_as_float(b.y), __uint_as_float(b.z), __uint_as_float(b.w)};
                                    split_planes8(x, hp);
                                } else {
#pragma unroll
                                    for (int p = 0; p < 3; ++p) hp[p] = h[m][part * KSN + st][p];
                                }
#pragma unroll
                                for (int p = 0; p < 3; ++p)
                                    acc[0][gu * TS + t][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, hp[p]),
                                                                                           __builtin_bit_cast(bf16x8, e), acc[0][gu * TS + t][m], 0, 0, 0);
                            }
                        } else {
#pragma unroll
                            for (int x = 0; x < 4; ++x)
#pragma unroll
                                for (int m = 0; m < MT; ++m) {
                                    const uint4 hv = h[m][part * KSN + st][0];
                                    const uint32_t hx = x == 0 ? hv.x : x == 1 ? hv.y : x == 2 ? hv.z : hv.w;
                                    floatx4& sum = acc[part % CHAINS][gu * TS + t][m];
                                    sum = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(hx), __uint_as_float(ew[x]), sum, 0, 0, 0);
                                }
                        }
                    }
                    // the next unit for this place, its loads between the matrix instructions
                    if (more) fill1(Next{}, ring_at + slot, st_c);
                    __builtin_amdgcn_sched_barrier(0);
                });
                slot = slot + NI * 1024 == RING * NI * 1024 ? 0u : slot + NI * 1024;
            });
        };
        for (int g = 0;; ++g) {
            if (g > 0) store_out(g - 1);
            if (g == groups) break;
            if (young) { if (young_first(g)) __builtin_amdgcn_s_setprio(1); else __builtin_amdgcn_s_setprio(0); }
#pragma unroll
            for (int t = 0; t < GT; ++t)
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int c = 0; c < CHAINS; ++c) acc[c][t][m] = floatx4{0.f, 0.f, 0.f, 0.f};
            if ((g + 1) * (GU * PARTS) + RING <= units) contract(std::true_type{}, g); else contract(std::false_type{}, g);
#pragma unroll
            for (int t = 0; t < GT; ++t)
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        red[q][t][m][r][ln] = CHAINS == 1 ? acc[0][t][m][r]
                                                          : (acc[0][t][m][r] + acc[1 % CHAINS][t][m][r]) + (acc[2 % CHAINS][t][m][r] + acc[3 % CHAINS][t][m][r]);
            lds_barrier();
            // thread (i, col) sums row i, column col of every tile: 16 lanes per row
            const int i = tid >> 4;
#pragma unroll
            for (int t = 0; t < GT; ++t)
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    if (4 * q + m * kTileM >= Bg) { out[t][m] = 0.f; continue; }
                    float sum = 0.f;
#pragma unroll
                    for (int w = 0; w < 4; ++w) sum += red[w][t][m][i & 3][(i >> 2) * 16 + col];
                    out[t][m] = sum;
                }
            // the candidates of the next block, once this one is under way (every wave is through with the one before)
            if ((g * GT & (kStreamTiles - 1)) == GT && g * GT / kStreamTiles * kStreamTiles + kStreamTiles < n) load_ids(g * GT / kStreamTiles + 1);
            lds_barrier();
        }
        LSH_TRACE_WG(11);
        if (!EVEN) return;
        seg = seg_end;
        if (seg == wg_end) return;
        __syncthreads();                                                      // (the candidates are read no more)
    }
}

// 33..64 beams, fp32 rows, d <= 1024: the operands change places.  The hidden rows do not fit in
// LDS (64 x 4 KB) and taking them in groups makes every group pull the candidate rows through
// the vector memory path again, which is what bounds that kernel.  Here the HIDDEN rows live in
// registers and the CANDIDATE rows pass through LDS: a workgroup of 16 waves = 4 row groups x 4
// slices of 256 k; wave (g, q) keeps the A operands of rows 16 g .. 16 g + 15, k in [256 q,
// 256 q + 256) in 64 registers for the whole kernel (16 k-steps x 4), and the workgroup walks the
// tiles of its sentence: every wave copies ONE candidate row of the next tile (4 KB, contiguous:
// whole cache lines) into the other half of a double-buffered LDS tile while all waves contract
// the current tile out of LDS (ds_read_b128 = the B operand of four matrix instructions).  A
// candidate row is loaded once per tile, whatever the number of beams.  The partial tiles of
// the four slices are summed through LDS in slice order, the wave of slice q finishing
// accumulator register q of its row group (a quarter of the tile's logits and softmax partials
// each: one wave finishing all of it was the critical path).  One barrier per tile.
// ONE record (max, sum exp) per hidden row for every kGroupTiles tiles the workgroup walks (the
// tiles j0 + (kGroupTiles m + i) G, i < kGroupTiles, at index j0 + m G; select.h): the
// selection's pass over the records is bound by what one CU can pull, and fifty rows of per-tile
// records were 140 KB per sentence.
//   LDS: 2 x 16 rows x 1028 floats (pitch 4 modulo 32: conflict-free 16-byte reads) + 2 x 12 KB of
//   partial tiles = 155.6 KB: one workgroup per CU.  Columns d .. 1023 of the tile are zeroed
//   once (they meet A operands that are zero, and 0 x garbage may be NaN).
//
// UNION: the sentence's candidate list is made here too, from the bitmaps an earlier kernel left
// for the parts of the sentence (k_part_bitmaps) and the top-frequent words: every workgroup ORs
// them in the LDS the tiles will use later, scans the popcounts, and the thread that owns a bit
// whose tile is one of this workgroup's writes its id to the list in memory and, for the
// workgroup's first kEsIdTiles tiles, to a small LDS table (later tiles read their ids back from
// the list).  All this runs while the A operands are on their way; the union kernel, its launch
// and the trip of the list through memory go away.
constexpr int kEsPitch = 1028, kEsSlice = 256, kEsSlices = 4;
constexpr int kEsIdTiles = 16;
constexpr int kEsUnionParts = 6;   // part bitmaps the kernel can OR (64 rows hashed 12 at a time)
// LDS: the two tiles, the partial tiles, the running record of each of the 64 rows (registers are
// all taken), and for UNION the id table.
__host__ __device__ inline size_t estage_lds_bytes(bool with_union = false) {
    return ((size_t)2 * kTileN * kEsPitch + (size_t)2 * 12 * 4 * kWave + 2 * 64 +
            (with_union ? kEsIdTiles * kTileN : 0)) * 4;
}
// LDS words the union needs inside the tile buffers (bitmap + scan scratch)
__host__ __device__ inline size_t estage_union_words(int V) { return (size_t)bitmap_words_padded(V) + 64; }
constexpr int kEsCoopBits = 8;   // list positions of one tile in one thread from which its wave shares the work
struct EstageUnion {
    const uint32_t* parts;    // [S, nparts, ceil(V/32)] bitmaps
    int nparts;
    const int32_t* topfreq;   // [T]
    int T;
    int32_t* cand;            // out: [S, V] ascending candidate ids
    int32_t* count;           // out: [S]
};

template <int MT, bool UNION>
__global__ void __launch_bounds__(1024)
k_logits_estage(const float* __restrict__ E, int64_t ld, int d, const float* __restrict__ H, int S,
                int B, const int32_t* __restrict__ cand, const int32_t* __restrict__ count, int V,
                float* __restrict__ logits, int64_t cpitch, TileRecords recs, EstageUnion un) {
    constexpr int KSTEP = 16, NSTEP = kEsSlice / KSTEP;
    extern __shared__ uint32_t esm[];
    float* etile = reinterpret_cast<float*>(esm);                         // [2][16][kEsPitch]
    float* red = etile + 2 * kTileN * kEsPitch;                           // [2][16 waves][3][64]
    float2* run = reinterpret_cast<float2*>(red + 2 * 12 * 4 * kWave);            // [64 rows] record so far
    uint32_t* ids_lds = reinterpret_cast<uint32_t*>(run + 64);                    // UNION: [kEsIdTiles][16]
    const int tid = threadIdx.x, ln = lane_id(), wv = wave_id();
    const int col = ln & 15, kk = ln >> 4;
    const int g = wv >> 2, q = wv & 3;                                     // row group, k slice
    const int s = blockIdx.x % S, j0 = blockIdx.x / S, G = gridDim.x / S;  // tiles j0, j0 + G, ...

    // A operands: rows 16 g + col (clamped), k = 256 q + 16 step + 4 kk + (0..3); zero past d
    float a[NSTEP][4];
    auto load_a = [&]() {
        const int row = min(g * kTileM + col, B - 1);
        const float* hrow = H + ((size_t)s * B + row) * d;
#pragma unroll
        for (int st = 0; st < NSTEP; ++st) {
            const int k = q * kEsSlice + st * KSTEP + 4 * kk;
            const float4 h = *reinterpret_cast<const float4*>(hrow + min(k, d - 4));
            const bool in = k < d && g < MT;
            a[st][0] = in ? h.x : 0.f; a[st][1] = in ? h.y : 0.f;
            a[st][2] = in ? h.z : 0.f; a[st][3] = in ? h.w : 0.f;
        }
    };
    int C;
    if constexpr (UNION) {
        // Loads return in order: everything the union reads is asked for first (the first 4096
        // bitmap words of up to kEsUnionParts parts, the first 3072 top-frequent ids), the A operands
        // after it -- they arrive while the union is being made: the barriers in here are
        // lds_barrier, which does not wait for them.
        uint32_t* bm = esm;
        uint32_t* wsum = bm + bitmap_words_padded(V);
        const int nwords = (V + 31) >> 5;
        const uint32_t* pb = un.parts + (size_t)s * un.nparts * nwords;
        constexpr int SLOTS = 4, PARTS = kEsUnionParts;
        uint32_t pw[SLOTS][PARTS];
#pragma unroll
        for (int u = 0; u < SLOTS; ++u)
#pragma unroll
            for (int b = 0; b < PARTS; ++b) pw[u][b] = 0u;
        // (words past the end repeat the last; parts and slots that do not exist are skipped by
        // uniform branches: a load that hits in cache costs the load path as much as one that misses)
#pragma unroll
        for (int u = 0; u < SLOTS; ++u) {
            if (u * 1024 >= nwords) break;
#pragma unroll
            for (int b = 0; b < PARTS; ++b) {
                if (b >= un.nparts) break;
                pw[u][b] = pb[(size_t)b * nwords + min(tid + u * 1024, nwords - 1)];
            }
        }
        const int32_t tf0 = (tid < un.T) ? un.topfreq[tid] : -1;
        const int32_t tf1 = (tid + 1024 < un.T) ? un.topfreq[tid + 1024] : -1;
        const int32_t tf2 = (tid + 2048 < un.T) ? un.topfreq[tid + 2048] : -1;
        __builtin_amdgcn_sched_barrier(0);   // (issue order = the order written here)
        load_a();
#pragma unroll
        for (int u = 0; u < SLOTS; ++u) {
            uint32_t x = 0;
#pragma unroll
            for (int b = 0; b < PARTS; ++b) x |= pw[u][b];
            if (tid + u * 1024 < nwords) bm[tid + u * 1024] = x;
        }
        for (int i = tid + SLOTS * 1024; i < nwords; i += 1024) {
            uint32_t x = 0;
            for (int b = 0; b < un.nparts; ++b) x |= pb[(size_t)b * nwords + i];   // (nparts <= kEsUnionParts)
            bm[i] = x;
        }
        lds_barrier();
        LSH_TRACE(1, 13);
        if (un.T > 0) mark_ids_of_wave(bm, V, tf0);
        if (un.T > 1024) mark_ids_of_wave(bm, V, tf1);
        if (un.T > 2048) mark_ids_of_wave(bm, V, tf2);
        for (int i = 3072 + tid; i - tid < un.T; i += 1024) mark_ids_of_wave(bm, V, (i < un.T) ? un.topfreq[i] : -1);
        lds_barrier();
        const int per_thread = (nwords + 1023) / 1024;
        const int wbeg = min(tid * per_thread, nwords), wend = min(wbeg + per_thread, nwords);
        uint32_t mine = 0;
        for (int i = wbeg; i < wend; ++i) mine += __popc(bm[i]);
        uint32_t total;
        uint32_t pos = block_incl_scan<true>(mine, wsum, &total) - mine;   // list position of my first bit
        C = (int)total;
        LSH_TRACE(1, 14);
        // my bits are list positions [pos, pos + mine); of the tiles they fall into, this
        // workgroup's are those congruent to j0 modulo G.  A thread with a few positions of such a
        // tile skips to its first bit (whole words by popcount) and writes the ids out itself; one
        // with kEsCoopBits or more (the dense words of the top-frequent ids put a whole tile into
        // one thread) hands them to the lanes of its wave, each finding one id by rank -- sixteen
        // dependent steps of a single lane, in every workgroup, used to be most of this phase.
        {
            const uint32_t end = pos + mine;
            const int t0 = (int)(pos >> 4);
            int nt = t0 + (j0 - t0 % G + G) % G;
            int k = nt / G;
            auto pending = [&]() { return mine != 0u && (uint32_t)nt * kTileN < end; };
            while (__ballot(pending()) != 0ull) {   // (uniform)
                const bool has = pending();
                const uint32_t lo = has ? max(pos, (uint32_t)nt * kTileN) : 0u;
                const uint32_t hi = has ? min(end, (uint32_t)nt * kTileN + kTileN) : 0u;
                const uint32_t n = hi - lo;
                if (has && n < (uint32_t)kEsCoopBits) {
                    uint32_t skip = lo - pos;
                    int i = wbeg;
                    uint32_t bits = bm[i];
                    for (uint32_t c = __popc(bits); skip >= c; c = __popc(bits)) { skip -= c; bits = bm[++i]; }
                    for (; skip; --skip) bits &= bits - 1u;
                    for (uint32_t at = lo; at < hi; ++at) {
                        while (!bits) bits = bm[++i];
                        const int32_t id = (i << 5) + (__ffs(bits) - 1);
                        bits &= bits - 1u;
                        un.cand[(size_t)s * V + at] = id;
                        if (k < kEsIdTiles) ids_lds[k * kTileN + (int)(at & 15u)] = (uint32_t)id;
                    }
                }
                for (uint64_t heavy = __ballot(has && n >= (uint32_t)kEsCoopBits); heavy; heavy &= heavy - 1) {   // (uniform)
                    const int o = __ffsll((unsigned long long)heavy) - 1;
                    const uint32_t o_lo = wave_read_lane(lo, o), o_n = wave_read_lane(n, o), o_pos = wave_read_lane(pos, o);
                    const int o_k = (int)wave_read_lane((uint32_t)k, o);
                    int i = (int)wave_read_lane((uint32_t)wbeg, o);
                    if ((uint32_t)ln < o_n) {
                        uint32_t r = o_lo - o_pos + (uint32_t)ln;      // my bit's rank in the owner's words
                        uint32_t bits = bm[i];
                        for (uint32_t c = __popc(bits); r >= c; c = __popc(bits)) { r -= c; bits = bm[++i]; }
                        const int32_t id = (i << 5) + (int32_t)nth_set_bit(bits, r);
                        const uint32_t at = o_lo + (uint32_t)ln;
                        un.cand[(size_t)s * V + at] = id;
                        if (o_k < kEsIdTiles) ids_lds[o_k * kTileN + (int)(at & 15u)] = (uint32_t)id;
                    }
                }
                if (has) { nt += G; ++k; }
            }
        }
        LSH_TRACE(1, 15);
        if (j0 == 0 && tid == 0) un.count[s] = C;
        lds_barrier();   // the table is written and the bitmap done with (the ids of later tiles are read
                         // back from the list only after many full barriers)
    } else {
        C = count ? count[s] : V;
    }
    const int ntiles = (C + kTileN - 1) / kTileN;
    if (j0 >= ntiles) return;                                             // (whole workgroup)
    LSH_TRACE(1, 0);

    // this wave's candidate row of a tile, 4 KB as up to four 16-byte loads per lane
    const int d4 = d >> 2;
    auto id_of = [&](int nt) -> int64_t {                                  // (any nt >= 0)
        if constexpr (UNION) {
            // (waves past the end of the list, and tiles past the last, take a candidate that
            // exists: their rows are never stored)
            if (nt >= ntiles) nt = j0;
            const int cidx = nt * kTileN + (nt * kTileN + wv < C ? wv : 0);
            const int k = (nt - j0) / G;
            return k < kEsIdTiles ? (int64_t)ids_lds[k * kTileN + (cidx & 15)] : (int64_t)un.cand[(size_t)s * V + cidx];
        }
        const int cidx = min(nt * kTileN + wv, C - 1);                     // clamped rows are never stored
        return cand ? (int64_t)cand[(size_t)s * V + cidx] : (int64_t)cidx;
    };
    auto row_of = [&](int64_t j) { return reinterpret_cast<const float4*>(E + j * ld); };
    float4 st0, st1, st2, st3;   // (named registers: an array captured by the lambdas goes to scratch)
    const int c0 = min(ln, d4 - 1), c1 = min(ln + kWave, d4 - 1), c2 = min(ln + 2 * kWave, d4 - 1),
              c3 = min(ln + 3 * kWave, d4 - 1);
    auto load_row = [&](const float4* r) { st0 = r[c0]; st1 = r[c1]; st2 = r[c2]; st3 = r[c3]; };
    auto store_row = [&](int buf) {
        float4* dst = reinterpret_cast<float4*>(etile + ((size_t)buf * kTileN + wv) * kEsPitch);
        if (ln < d4) dst[ln] = st0;
        if (ln + kWave < d4) dst[ln + kWave] = st1;
        if (ln + 2 * kWave < d4) dst[ln + 2 * kWave] = st2;
        if (ln + 3 * kWave < d4) dst[ln + 3 * kWave] = st3;
    };
    load_row(row_of(id_of(j0)));
    int64_t id_next = id_of(j0 + G);   // candidate ids are fetched a tile ahead of their rows
    if constexpr (!UNION) load_a();
    // zero the columns d .. 1023 of both buffers (never written by the row copies)
    {
        const int padw = kEsSlices * kEsSlice - d;                         // a multiple of 4, < 1024
        for (int e = tid; e < 2 * kTileN * padw; e += 1024) {
            const int r = e / padw, c = e - r * padw;
            etile[(size_t)r * kEsPitch + d + c] = 0.f;
        }
    }
    LSH_TRACE(1, 1);
    store_row(0);
    __syncthreads();
    LSH_TRACE(1, 2);

    int buf = 0;
    // (max, sum exp) of a row over the tiles of the current group: kept in LDS by the lane that
    // writes the row's records (column 0), which alone reads and writes its slot
    if (g < MT && col == 0) run[g * kTileM + 4 * kk + q] = make_float2(-INFINITY, 0.f);
    int kt = 0;                                 // tiles done
    for (int nt = j0; nt < ntiles; nt += G, buf ^= 1, ++kt) {
        const bool more = nt + G < ntiles;
        if (more) {                                                        // in flight during the contraction
            load_row(row_of(id_next));
            id_next = id_of(nt + 2 * G);
        }
        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
        if (g < MT) {
            const float* bt = etile + ((size_t)buf * kTileN + col) * kEsPitch + q * kEsSlice + 4 * kk;
#pragma unroll
            for (int st = 0; st < NSTEP; ++st) {
                const float4 b = *reinterpret_cast<const float4*>(bt + st * KSTEP);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[st][0], b.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[st][1], b.y, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[st][2], b.z, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[st][3], b.w, acc, 0, 0, 0);
            }
            // the wave of slice q finishes accumulator register q of its row group (rows 16 g +
            // 4 kk + q): it keeps that register and leaves the other three for its siblings
            float* rp = red + (((size_t)buf * 16 + wv) * 3) * kWave;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (r != q) rp[(r < q ? r : r - 1) * kWave + ln] = acc[r];
        }
#ifdef LSHBEAM_TRACE
        LSH_TRACE_UPTO(1, 3 + 2 * ((nt - j0) / G), 11);
#endif
        if (more) store_row(buf ^ 1);   // the other half was last read before the previous barrier
        __syncthreads();
#ifdef LSHBEAM_TRACE
        LSH_TRACE_UPTO(1, 4 + 2 * ((nt - j0) / G), 12);
#endif
        if (g < MT) {
            // x = sum over the four slices in slice order (this wave's own share in its place)
            const float own = (q == 0) ? acc[0] : (q == 1) ? acc[1] : (q == 2) ? acc[2] : acc[3];
            float x = 0.f;
#pragma unroll
            for (int qq = 0; qq < kEsSlices; ++qq) {
                float part = own;
                if (qq != q)   // wave-uniform
                    part = red[(((size_t)buf * 16 + (g * 4 + qq)) * 3 + (q < qq ? q : q - 1)) * kWave + ln];
                x = (qq == 0) ? part : x + part;
            }
            const int n0 = nt * kTileN;
            const int row = g * kTileM + 4 * kk + q, c = n0 + col;
            const bool valid = row < B && c < C;
            if (valid) logits[((size_t)s * B + row) * cpitch + c] = x;
            const float mx = row16_max(valid ? x : -INFINITY);
            const float se = row16_sum(valid ? exp_below(x, mx) : 0.f);
            if (col == 0) {
                // (one fast exponential, no branch: 16 waves share the CU's issue slots, and every
                // instruction here is paid once per tile by each of them)
                float2 acc2 = run[g * kTileM + 4 * kk + q];
                const float hi = fmaxf(acc2.x, mx);
                const float e = __expf(fminf(acc2.x, mx) - fmaxf(hi, -FLT_MAX));   // exp(-|difference|); 0 for the first tile
                acc2.y = (mx > acc2.x) ? fmaf(acc2.y, e, se) : fmaf(se, e, acc2.y);
                acc2.x = hi;
                const bool group_end = kt % kGroupTiles == kGroupTiles - 1 || !more;
                if (group_end && row < B)
                    reinterpret_cast<float2*>(recs.rec)[((size_t)s * B + row) * recs.pitch + j0 +
                                                        (size_t)(kt / kGroupTiles) * G] = acc2;
                run[g * kTileM + 4 * kk + q] = group_end ? make_float2(-INFINITY, 0.f) : acc2;
            }
        }
    }
}

// Full vocabulary: every hidden row meets every word, so sentences do not matter and the contraction
// is one matrix product, R rows x V words.  (Taken sentence by sentence each of them gathered all of
// E again: 32 sentences x 160 MB.)  Few rows: bound by the one pass over E (k_logits_few, k_logits_pass
// below); many: by the matrix pipe.
//
// A workgroup of four waves makes MT * 16 rows x 64 WF words, in blocks of 32 k, on bf16 matrix instructions.  The
// hidden rows pass through LDS (double-buffered, as three bf16 planes, split on the way in).  bf16 words meet
// all three planes: exact products.  fp32 words are split into three planes as well, in registers, each plane
// the nearest bf16 to what is left, and eight of the nine plane products are made; the ninth is at most 2^-34 of the
// whole.  The products of two first planes have an accumulator of their own: these instructions cut off what an addend
// has below the accumulator's last place, and all the smaller products lost their ends there, every 32 k.
// rms of the error over the sum of the products' sizes, n of d = 1000 products not zero, against fp64 sums:
//                                        n = 1      8        32      1000
//   fp32 instructions                  2.53e-8  2.73e-8  2.78e-8  2.81e-8
//   fp32 words, 8 products             2.53e-8  1.44e-8  1.16e-8  0.91e-8
//     in one accumulator               3.40e-8  5.39e-8  5.52e-8  2.38e-8
//     6 products (those from 2^-23 on) 2.60e-8  1.47e-8  1.17e-8  0.91e-8
//   bf16 words                         2.52e-8  1.44e-8  1.16e-8  0.91e-8
//     in one accumulator               3.35e-8  3.77e-8  3.75e-8  1.65e-8
// Six products are 10 % faster (below) and leave out up to 2^-24 of a product, as much as rounding it once: a sum of
// one product was off by up to 1.0e-7 instead of 6.0e-8.
//
// A wave owns 16 WF words and all the rows; nobody else needs those words, so their chunks go from memory straight into the A operand registers, kRowsAhead blocks ahead.  With WF = 2
// (fp32, 8 MT WF instructions of 16 cycles per 3 MT 16-byte LDS reads) and WF = 4 (bf16, 3 MT WF per 3 MT
// reads) the LDS rate is no bound.  Words are the A operand, so that a lane ends up with
// four consecutive words of one hidden row (a 16-byte store).  The operands of a block are read from
// LDS in two halves, each while the other half's instructions run; without that, and with the loads
// placed by the compiler, the same tiles took a quarter longer.  MT is the host's choice.
// Any d >= one chunk and any pitch: chunks are loaded from any element's address.
// 320 rows, V = 40000, d = 1000: fp32 175 us (146 TFLOP/s of the product, 1170 of plane products: a large bf16 product
// of matrices reaches 1230 on this card, a large fp32 one 154), 157 us with six products in one accumulator;
// k_logits_hlds with fp32 instructions 370 us.  bf16 (d = 1024) 87 us, in one accumulator 86; widened 334.
constexpr int kRowsK = 32;
constexpr int kRowsPitch = 40 * 2;   // LDS bytes per hidden row and plane: 16-byte reads without conflicts
__host__ __device__ constexpr size_t rows_lds_bytes(int MT) {
    return (size_t)2 * 3 * ((MT + 1) / 2 * 32) * kRowsPitch + 4 * kTileM * sizeof(float2);
}
template <typename ET> __host__ __device__ constexpr int few_planes() { return sizeof(ET) == 2 ? 3 : 1; }

// The 16 bytes of a row of d >= 16 / sizeof(ET) elements that begin at element k, zeros past the row's
// end: what lies past it is never read (one clamped load, then shifted into place in registers).
template <typename ET>
__device__ __forceinline__ Chunk16U<ET> load_chunk_end(const ET* row, int k, int d) {
    constexpr int CK = 16 / (int)sizeof(ET);
    const int at = min(k, d - CK);
    Chunk16U<ET> c = *reinterpret_cast<const Chunk16U<ET>*>(row + at);
    const int s = min(k - at, CK);                  // elements to drop in front
    if constexpr (sizeof(ET) == 2) {
        if (s & 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) c.w[i] = (c.w[i] >> 16) | (i < 3 ? c.w[i < 3 ? i + 1 : 3] << 16 : 0u);
        }
    }
    constexpr int ONE = 4 / (int)sizeof(ET);        // elements per word
    if (s & ONE) { c.w[0] = c.w[1]; c.w[1] = c.w[2]; c.w[2] = c.w[3]; c.w[3] = 0u; }
    if (s & (2 * ONE)) { c.w[0] = c.w[2]; c.w[1] = c.w[3]; c.w[2] = 0u; c.w[3] = 0u; }
    if (s & (4 * ONE)) { c.w[0] = 0u; c.w[1] = 0u; c.w[2] = 0u; c.w[3] = 0u; }
    return c;
}
// The same shifts of a chunk that is here already: without its first s elements, zeros behind.  (Called from load_chunk_end it cost
// k_logits_few 14 registers and, 27 rows, V = 51168, d = 1312, 32 us of 88.)
template <typename ET>
__device__ __forceinline__ void drop_front(Chunk16U<ET>& c, int s) {
    if constexpr (sizeof(ET) == 2) {
        if (s & 1) {
#pragma unroll
            for (int i = 0; i < 4; ++i) c.w[i] = (c.w[i] >> 16) | (i < 3 ? c.w[i < 3 ? i + 1 : 3] << 16 : 0u);
        }
    }
    constexpr int ONE = 4 / (int)sizeof(ET);        // elements per word
    if (s & ONE) { c.w[0] = c.w[1]; c.w[1] = c.w[2]; c.w[2] = c.w[3]; c.w[3] = 0u; }
    if (s & (2 * ONE)) { c.w[0] = c.w[2]; c.w[1] = c.w[3]; c.w[2] = 0u; c.w[3] = 0u; }
    if (s & (4 * ONE)) { c.w[0] = 0u; c.w[1] = 0u; c.w[2] = 0u; c.w[3] = 0u; }
}
template <typename ET> __device__ __forceinline__ bf16x8 as_bf16x8(const Chunk16U<ET>& c) {
    return __builtin_bit_cast(bf16x8, make_uint4(c.w[0], c.w[1], c.w[2], c.w[3]));
}

// Two values as three pairs of bf16, each the nearest to what is left (v_cvt_pk_bf16_f32): a = hi + mid + lo exactly,
// |mid| at most 2^-8 and |lo| 2^-17 of |a|'s power of two.  (Not where the nearest bf16 is infinite, which
// settle_non_finite mends; and a plane ends at 2^-133, so that values below 2^-110 lose bits: that shows in a logit
// only where the other side holds values beyond 2^100.)
__device__ __forceinline__ void split_near(float a, float b, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    auto pack = [](float x, float y) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2{x, y}), bf16x2)); };
    hi = pack(a, b);
    a -= __uint_as_float(hi << 16);
    b -= __uint_as_float(hi & 0xFFFF0000u);
    mid = pack(a, b);
    a -= __uint_as_float(mid << 16);
    b -= __uint_as_float(mid & 0xFFFF0000u);
    lo = pack(a, b);
}

// The end of both kernels: lane (col, kk) holds, in x[m][f], the logits of hidden row row0 + 16 m + col
// and the words word0 + 16 f + 4 kk + (0..3).  Stores them and a record (max, sum exp) per row and 64
// words, which are one, two or four waves' (WF = 4, 2, 1); part: LDS for 4 x 16 pairs.  PLANES: the logits come
// from bf16 planes (settle_non_finite).  Called by all four waves.
template <bool PLANES, typename ET, int MT, int WF>
__device__ __forceinline__ void finish_wide(floatx4 (&x)[MT][WF], const ET* __restrict__ E, int64_t ld, int d,
                                            const float* __restrict__ H, int row0, int word0, int R, int V,
                                            float* __restrict__ logits, int64_t cpitch, TileRecords recs, float2* part) {
    static_assert(WF == 4 || WF == 2 || WF == 1, "64 words are one, two or four waves'");
    const int ln = lane_id(), wv = wave_id(), col = ln & 15, kk = ln >> 4;
    const int w0 = word0 + 4 * kk;
    if constexpr (PLANES) {
        float v[MT * WF * 4];
#pragma unroll
        for (int i = 0; i < MT * WF * 4; ++i) v[i] = x[i / (4 * WF)][i / 4 % WF][i % 4];
        settle_non_finite(v, [&](int i) {
            const int row = min(row0 + i / (4 * WF) * kTileM + col, R - 1), w = min(w0 + 16 * (i / 4 % WF) + i % 4, V - 1);
            return plain_dot(E + (int64_t)w * ld, H + (size_t)row * d, d);
        });
#pragma unroll
        for (int i = 0; i < MT * WF * 4; ++i) x[i / (4 * WF)][i / 4 % WF][i % 4] = v[i];
    }
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int row = row0 + m * kTileM + col;
        float mx = -INFINITY;
#pragma unroll
        for (int f = 0; f < WF; ++f) {
            const int w = w0 + 16 * f;
            if (row < R && w < V)   // (columns past V inside the row's pitch are never read)
                *reinterpret_cast<float4*>(&logits[(size_t)row * cpitch + w]) = make_float4(x[m][f][0], x[m][f][1], x[m][f][2], x[m][f][3]);
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, w + r < V ? x[m][f][r] : -INFINITY);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        float se = 0.f;
#pragma unroll
        for (int f = 0; f < WF; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) se += w0 + 16 * f + r < V ? exp_below(x[m][f][r], mx) : 0.f;
        se += __shfl_xor(se, 16);
        se += __shfl_xor(se, 32);
        float2 a = make_float2(mx, se);
        if constexpr (WF < 4) {
            if (kk == 0) part[wv * kTileM + col] = a;
            lds_barrier();
#pragma unroll
            for (int o = 1; o < 4 / WF; ++o) {
                const float2 q = part[((wv + o) & 3) * kTileM + col];   // (a wave past V: -inf, 0)
                const float hi = fmaxf(a.x, q.x);
                a = make_float2(hi, a.y * exp_below(a.x, hi) + q.y * exp_below(q.x, hi));
            }
            lds_barrier();
        }
        if ((wv & (4 / WF - 1)) == 0 && kk == 0 && row < R && word0 < V)
            reinterpret_cast<float2*>(recs.rec)[(size_t)row * recs.pitch + word0 / kWideN] = a;
    }
}

template <typename ET, int MT, int WF>
__global__ void __launch_bounds__(256, 2)
k_logits_rows(const ET* __restrict__ E, int64_t ld, int d, const float* __restrict__ H, int R, int V,
              int gx /*tiles of 64 WF words*/, int ngroups, float* __restrict__ logits, int64_t cpitch, TileRecords recs) {
    constexpr bool BF = sizeof(ET) == 2;
    constexpr int PITCH = kRowsPitch, NP = 3;
    constexpr int HP = (MT + 1) / 2, LROWS = HP * 32;         // hidden rows are staged 32 at a time
    constexpr int PE = BF ? 1 : 3;                            // planes of the words
    constexpr int PER_WF = BF ? 1 : 2, NC = PER_WF * WF;      // 16-byte chunks of E per lane and block
    constexpr int kRowsAhead = 2;                             // blocks of E in registers: 8 loads in flight
    constexpr int CK = 16 / (int)sizeof(ET);                  // elements per chunk
    constexpr int M0 = (MT + 1) / 2;                          // row tiles in the first half of a block
    constexpr int kBuf = NP * LROWS * PITCH;                  // bytes per buffer
    extern __shared__ uint32_t rsm[];
    char* sm = reinterpret_cast<char*>(rsm);
    // (the row groups of one tile of words run on one XCD, one after the other: they share its L2)
    const uint32_t slot = blockIdx.x >> 3;
    const int bx = (int)((slot / (uint32_t)ngroups) * 8u + (blockIdx.x & 7u));
    if (bx >= gx) return;
    const int row0 = (int)(slot % (uint32_t)ngroups) * MT * kTileM;
    const int tid = threadIdx.x, ln = lane_id(), wv = wave_id();
    const int col = ln & 15, kk = ln >> 4;
    const int word0 = bx * (64 * WF) + wv * (16 * WF);
    const int lr = tid >> 3, lc = 4 * (tid & 7);              // this thread's hidden row (of 32) and k inside a block
    const float* hsrc[HP];
#pragma unroll
    for (int p = 0; p < HP; ++p) hsrc[p] = H + (size_t)min(row0 + 32 * p + lr, R - 1) * d;
    const ET* esrc[WF];
#pragma unroll
    for (int f = 0; f < WF; ++f) esrc[f] = E + (int64_t)min(word0 + 16 * f + col, V - 1) * ld;

    Float4U st[HP];
    Chunk16U<ET> ev[kRowsAhead][NC];
    auto load_hidden = [&](int i) {
#pragma unroll
        for (int p = 0; p < HP; ++p) st[p] = *reinterpret_cast<const Float4U*>(hsrc[p] + i * kRowsK + lc);
    };
    auto load_words = [&](int i, Chunk16U<ET> (&e)[NC]) {     // word tile f: 8 consecutive k, one chunk or two
#pragma unroll
        for (int c = 0; c < NC; ++c)
            e[c] = *reinterpret_cast<const Chunk16U<ET>*>(esrc[c / PER_WF] + i * kRowsK + kk * 8 + (c % PER_WF) * CK);
    };
    auto store_hidden = [&](int buf) {
#pragma unroll
        for (int p = 0; p < HP; ++p) {
            char* dst = sm + buf * kBuf + (32 * p + lr) * PITCH + lc * 2;
            const float x[4] = {st[p].x, st[p].y, st[p].z, st[p].w};
            if constexpr (BF) {
                store_planes4(dst, (size_t)LROWS * PITCH, x);
            } else {
                uint2 w[3];
                split_near(x[0], x[1], w[0].x, w[1].x, w[2].x);
                split_near(x[2], x[3], w[0].y, w[1].y, w[2].y);
#pragma unroll
                for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(dst + q * (LROWS * PITCH)) = w[q];
            }
        }
    };
    floatx4 acc[MT][WF], low[MT][WF];                         // products of two first planes; all others
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int f = 0; f < WF; ++f) acc[m][f] = low[m][f] = floatx4{0.f, 0.f, 0.f, 0.f};
    // half h of a block: row tiles [0, M0) or [M0, MT)
    struct Operands { uint4 b[M0][NP]; };
    struct Words { uint4 p[WF][PE]; };                        // the words' operands: their chunk, or its three planes
    auto read_half = [&](int buf, int h, Operands& o) {
        const char* hb = sm + buf * kBuf + col * PITCH + 16 * kk + h * M0 * kTileM * PITCH;
#pragma unroll
        for (int m = 0; m < M0; ++m)
#pragma unroll
            for (int p = 0; p < NP; ++p)
                if (h == 0 || M0 + m < MT)
                    o.b[m][p] = *reinterpret_cast<const uint4*>(hb + (p * LROWS + m * kTileM) * PITCH);
    };
    auto make_words = [&](const Chunk16U<ET> (&e)[NC], Words& w) {
#pragma unroll
        for (int f = 0; f < WF; ++f) {
            if constexpr (BF) {
                w.p[f][0] = make_uint4(e[f].w[0], e[f].w[1], e[f].w[2], e[f].w[3]);
            } else {
                uint32_t q[3][4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const Chunk16U<ET>& c = e[f * PER_WF + (PER_WF > 1 ? i / 2 : 0)];
                    split_near(__uint_as_float(c.w[2 * (i % 2)]), __uint_as_float(c.w[2 * (i % 2) + 1]), q[0][i], q[1][i], q[2][i]);
                }
#pragma unroll
                for (int p = 0; p < PE; ++p) w.p[f][p] = make_uint4(q[p][0], q[p][1], q[p][2], q[p][3]);
            }
        }
    };
    auto contract = [&](const Operands& o, int h, const Words& w) {
        // (smallest products first; the third planes' own, at most 2^-34 of the whole, is left out)
#pragma unroll
        for (int sum = PE == 1 ? 2 : 3; sum >= 0; --sum)
#pragma unroll
            for (int pe = 0; pe < PE; ++pe) {
                const int p = sum - pe;
                if (p < 0 || p >= NP) continue;
#pragma unroll
                for (int m = 0; m < M0; ++m)
#pragma unroll
                    for (int f = 0; f < WF; ++f)
                        if (h * M0 + m < MT) {
                            const int mm = h * M0 + m < MT ? h * M0 + m : 0;
                            floatx4& to = sum ? low[mm][f] : acc[mm][f];
                            to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf16x8, w.p[f][pe]), __builtin_bit_cast(bf16x8, o.b[m][p]), to, 0, 0, 0);
                        }
            }
    };
    const int nfull = d / kRowsK, rem = d - nfull * kRowsK;
    auto load_rest = [&](Chunk16U<ET> (&e)[NC]) {             // (zeros past d on both sides)
        const int k0 = nfull * kRowsK;
#pragma unroll
        for (int p = 0; p < HP; ++p) {
            const Chunk16U<float> c = load_chunk_end<float>(hsrc[p], k0 + lc, d);
            st[p] = __builtin_bit_cast(Float4U, c);
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) e[c] = load_chunk_end<ET>(esrc[c / PER_WF], k0 + kk * 8 + (c % PER_WF) * CK, d);
    };
    Operands o0, o1;
    Words w0, w1;
    int buf = 0;
    if (nfull) {
        // (the order in which the loop issues its loads, so that its waits count the same on both ways in)
        load_hidden(0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j + 1 < kRowsAhead; ++j) {
            load_words(min(j, nfull - 1), ev[j]);
            __builtin_amdgcn_sched_barrier(0);
        }
        store_hidden(0);
        load_hidden(min(1, nfull - 1));
        __builtin_amdgcn_sched_barrier(0);
        load_words(min(kRowsAhead - 1, nfull - 1), ev[kRowsAhead - 1]);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        read_half(0, 0, o0);
        make_words(ev[0], w0);
        for (int i0 = 0; i0 < nfull; i0 += kRowsAhead) {
#pragma unroll
            for (int j = 0; j < kRowsAhead; ++j) {
                const int i = i0 + j;
                if (i >= nfull) break;              // (uniform)
                read_half(buf, 1, o1);
                contract(o0, 0, w0);
                __builtin_amdgcn_sched_barrier(0);  // (the wait for the hidden rows stays behind the instructions)
                store_hidden(buf ^ 1);              // (last read before the previous barrier; past the last block: unused)
                load_hidden(min(i + 2, nfull - 1));
                lds_barrier();
                read_half(buf ^ 1, 0, o0);
                if (kRowsAhead > 1) make_words(ev[(j + 1) % kRowsAhead], w1);   // (the next block's, among this one's instructions)
                contract(o1, 1, w0);
                load_words(min(i + kRowsAhead, nfull - 1), ev[j]);
                __builtin_amdgcn_sched_barrier(0);
                w0 = w1;
                buf ^= 1;
            }
        }
        buf ^= 1;                                   // (the other buffer may still be being read)
    }
    if (rem) {
        load_rest(ev[0]);
        store_hidden(buf);
        lds_barrier();
        make_words(ev[0], w0);
        read_half(buf, 0, o0);
        contract(o0, 0, w0);
        read_half(buf, 1, o1);
        contract(o1, 1, w0);
    }
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int f = 0; f < WF; ++f) acc[m][f] += low[m][f];
    finish_wide<true>(acc, E, ld, d, H, row0, word0, R, V, logits, cpitch, recs, reinterpret_cast<float2*>(sm + 2 * kBuf));
}

// The same for a few hidden rows (MT * 16, at most 48): bound by the pass over E.  A wave owns 16 words; what
// counts is that every wave keeps long pieces of its rows in flight: blocks of 128 k (512 or 256 bytes
// of a row, asked for together), the next block under way while the current one meets the hidden rows in LDS
// (double-buffered, as above).
// 12 rows, V = 40000, d = 1000 fp32: 30.8 us (5.2 TB/s), as k_logits_hlds, but records of 64 words: the selection takes
// 9.4 us after them, 16.1 after records of 16; V = 200000: 161 and 174 us; bf16, d = 1024: 17.0 us, widened 24.3.
constexpr int kFewK = 128;
template <typename ET> __host__ __device__ constexpr int few_pitch() {   // LDS bytes per hidden row and plane
    return sizeof(ET) == 2 ? (kFewK + 8) * 2 : (kFewK + 4) * 4;
}
template <typename ET> __host__ __device__ constexpr size_t few_lds_bytes(int MT) {
    return (size_t)2 * few_planes<ET>() * MT * kTileM * few_pitch<ET>() + 4 * kTileM * sizeof(float2);
}
template <typename ET, int MT>
__global__ void __launch_bounds__(256, 3)
k_logits_few(const ET* __restrict__ E, int64_t ld, int d, const float* __restrict__ H, int R, int V,
             float* __restrict__ logits, int64_t cpitch, TileRecords recs) {
    constexpr bool BF = sizeof(ET) == 2;
    constexpr int PITCH = few_pitch<ET>(), NP = few_planes<ET>(), CK = 16 / (int)sizeof(ET);
    constexpr int NC = kFewK / (4 * CK);                      // chunks (steps) per lane and block
    constexpr int HP = MT * 2;                                // 16-byte chunks of hidden rows per thread and block
    constexpr int kPlane = MT * kTileM * PITCH, kBuf = NP * kPlane;
    extern __shared__ uint32_t rsm[];
    char* sm = reinterpret_cast<char*>(rsm);
    const int tid = threadIdx.x, ln = lane_id(), wv = wave_id();
    const int col = ln & 15, kk = ln >> 4;
    const int word0 = blockIdx.x * kWideN + wv * kTileN;
    const int lr = tid >> 5, lc = 4 * (tid & 31);             // this thread's hidden row (of 8) and k inside a block
    const float* hsrc[HP];
#pragma unroll
    for (int p = 0; p < HP; ++p) hsrc[p] = H + (size_t)min(8 * p + lr, R - 1) * d;
    const ET* esrc = E + (int64_t)min(word0 + col, V - 1) * ld;
    const int nfull = d / kFewK, rem = d - nfull * kFewK, nblk = nfull + (rem ? 1 : 0);

    Float4U st[HP];
    Chunk16U<ET> e0[NC], e1[NC];
    auto load_words = [&](int i, Chunk16U<ET> (&e)[NC]) {
        if (i < nfull) {   // (uniform)
#pragma unroll
            for (int c = 0; c < NC; ++c) e[c] = *reinterpret_cast<const Chunk16U<ET>*>(esrc + i * kFewK + c * 4 * CK + kk * CK);
        } else {
#pragma unroll
            for (int c = 0; c < NC; ++c) e[c] = load_chunk_end<ET>(esrc, i * kFewK + c * 4 * CK + kk * CK, d);
        }
    };
    auto load_hidden = [&](int i) {
#pragma unroll
        for (int p = 0; p < HP; ++p) st[p] = __builtin_bit_cast(Float4U, load_chunk_end<float>(hsrc[p], i * kFewK + lc, d));
    };
    auto store_hidden = [&](int buf) {
#pragma unroll
        for (int p = 0; p < HP; ++p) {
            char* dst = sm + buf * kBuf + (8 * p + lr) * PITCH + lc * (BF ? 2 : 4);
            const float x[4] = {st[p].x, st[p].y, st[p].z, st[p].w};
            if constexpr (BF) store_planes4(dst, kPlane, x);
            else *reinterpret_cast<float4*>(dst) = make_float4(x[0], x[1], x[2], x[3]);
        }
    };
    floatx4 acc[MT][1], low[MT];                              // low: bf16, as in k_logits_rows
#pragma unroll
    for (int m = 0; m < MT; ++m) acc[m][0] = low[m] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto contract = [&](int buf, const Chunk16U<ET> (&e)[NC]) {
        const char* hb = sm + buf * kBuf + col * PITCH + 16 * kk;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                if constexpr (BF) {
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        floatx4& to = p ? low[m] : acc[m][0];
                        to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            as_bf16x8(e[c]), *reinterpret_cast<const bf16x8*>(hb + p * kPlane + m * kTileM * PITCH + 64 * c), to, 0, 0, 0);
                    }
                } else {
                    const float4 b = *reinterpret_cast<const float4*>(hb + m * kTileM * PITCH + 64 * c);
                    acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(e[c].w[0]), b.x, acc[m][0], 0, 0, 0);
                    acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(e[c].w[1]), b.y, acc[m][0], 0, 0, 0);
                    acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(e[c].w[2]), b.z, acc[m][0], 0, 0, 0);
                    acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(e[c].w[3]), b.w, acc[m][0], 0, 0, 0);
                }
            }
    };
    // block i is contracted from `cur` while block i + 1 is on its way to `nxt`
    auto turn = [&](int i, Chunk16U<ET> (&cur)[NC], Chunk16U<ET> (&nxt)[NC]) {
        const int buf = i & 1;
        if (i + 1 < nblk) {   // (uniform)
            load_hidden(i + 1);
            load_words(i + 1, nxt);
        }
        __builtin_amdgcn_sched_barrier(0);
        contract(buf, cur);
        __builtin_amdgcn_sched_barrier(0);
        if (i + 1 < nblk) store_hidden(buf ^ 1);              // (last read before the previous barrier)
        lds_barrier();
    };
    load_hidden(0);
    load_words(0, e0);
    store_hidden(0);
    lds_barrier();
    for (int i = 0; i < nblk; i += 2) {
        turn(i, e0, e1);
        if (i + 1 < nblk) turn(i + 1, e1, e0);
    }
    if constexpr (BF) {
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m][0] += low[m];
    }
    finish_wide<BF>(acc, E, ld, d, H, 0, word0, R, V, logits, cpitch, recs, reinterpret_cast<float2*>(sm + 2 * kBuf));
}

// The same where the hidden rows fit in LDS whole, which is what most calls of few rows have: one workgroup per CU loads them once
// and shares out the words, so that nothing but E passes through the CU's load path afterwards (k_logits_few's workgroups, of
// 64 words each, read all hidden rows for every 256 KB of E), no barrier stands in the loop and every CU has the same to
// do: 625 workgroups of V = 40000 were two on some CUs and three on others.  A wave has `rounds` times 16 words in a row, eight to
// sixteen chunks of every lane on their way (all sixteen always, no branch for rows of up to eight steps: 1 % faster for d = 1000, 2 to 9 %
// slower for d = 99 to 176), the next tile's while one is finished; every workgroup leaves ONE record per hidden row, for its
// 16 W rounds words, as the selection is bound by what one CU pulls in.  The sums are k_logits_few's, bit for bit.
// us a step, k_logits_few and so: 12 rows, V = 40000, d = 1000 46.7, 41.9 (the pass over cold E 37.6, 36.4, selection 8.4, 5.5); 45
// rows, V = 94357, d = 216 56, 45; 22 rows, V = 97522, d = 80 35, 26; 22 rows, V = 140258, d = 1016 155, 151; bf16: 4 rows, V = 129085,
// d = 336 32, 29.
constexpr int kPassRing = 16;    // chunks of a lane on their way
constexpr int kPassWaves = 12;   // at most: registers for the ring and the operands on their way from LDS
template <typename ET> __host__ __device__ inline int pass_pitch(int d) {   // elements per hidden row and plane, zeros past d
    constexpr int KSTEP = 64 / (int)sizeof(ET);
    int p = (d + KSTEP - 1) / KSTEP * KSTEP;
    while (sizeof(ET) == 2 ? p % 64 != 8 : p % 32 != 4) p += sizeof(ET) == 2 ? 8 : 4;
    return p;
}
template <typename ET> __host__ __device__ inline size_t pass_lds_bytes(int MT, int d) {
    return (size_t)few_planes<ET>() * MT * kTileM * pass_pitch<ET>(d) * sizeof(ET) + (size_t)kPassWaves * MT * kTileM * sizeof(float2);
}
template <typename ET> constexpr int pass_most_tiles() { return sizeof(ET) == 2 ? 1 : 3; }   // (row groups; two of bf16 words, V = 191422, d = 912: 134 us, k_logits_few 119)
// Waves of a workgroup and how many times 16 words for each: the least that 256 workgroups have in all, and of those the most waves;
// eight at least where there is work for them (d = 1200, V = 59224, 15 rows: three times with five waves 72 us a step, k_logits_few 68).
// waves = 0: k_logits_few has the call (B: beams of a sentence; ld: elements).  The lines are drawn through 1489 (fp32) and 1530
// (bf16) shapes of d = 16 to 1536, V = 8200 to 250000, both kernels measured on each; numbers are means of a step so over one of k_logits_few.
//   fp32, more than 16 words for a wave: 0.52 to 0.94, but 1.03 where nine waves at most have more than 2 MB.  16 words for nine waves or
//   more 0.95.  With fewer waves (V <= 32768) k_logits_few's several small workgroups on a CU are as fast: 1.02 on average up to d = 128 and 1.06
//   with four waves; but 0.95 where its blocks of 128 values are nearly a third padding, 0.94 for rows of one or two whole lines of 128 bytes
//   and five waves, 0.97 for one row group of long rows (d >= 600; d > 128 with five waves) and 0.95 for three.  Rows of two to four whole blocks 1.08.
//   bf16, whose three planes of hidden rows stand in front of half the bytes: 1.1 to 1.4 for V < 70000, but 0.93 for long rows of
//   few words, where k_logits_few is a chain of blocks in two workgroups per CU.  From 33 times 16 words for a workgroup on 0.89; from 19 on 0.95 for d >= 144 and
//   0.92 with more than eight beams (the selection reads 64 words' records), else 1.1; 17 and 18 for d >= 600 0.94, else 1.1.
struct PassPlan { int waves, rounds; };
template <typename ET>
inline PassPlan pass_plan(int R, int B, int V, int d, int64_t ld) {
    constexpr PassPlan no{0, 0};
    const int groups = (R + kTileM - 1) / kTileM;
    if (groups > pass_most_tiles<ET>() || pass_lds_bytes<ET>(groups, d) > kMaxDynLds || ld * (int64_t)sizeof(ET) >= (int64_t)1 << 27) return no;
    const int64_t tiles = (V + kTileN - 1) / kTileN;
    PassPlan p = no;
    for (int W = tiles >= 8 * 256 ? 8 : 4; W <= kPassWaves; ++W) {
        const int rounds = (int)((tiles + 256 * W - 1) / (256 * W));
        if (!p.waves || W * rounds <= p.waves * p.rounds) p = {W, rounds};
    }
    const int each = p.waves * p.rounds;                                        // times 16 words, a workgroup
    const int64_t bytes = (int64_t)each * kTileN * d * (int64_t)sizeof(ET);     // of its words
    bool pays;
    if (sizeof(ET) == 2) {
        pays = each >= 33 || (each >= 19 && (d >= 144 || B > 8)) || (each >= 17 && d >= 600) ||
               (each == 5 && d >= 900);
    } else if (p.rounds <= 2 && d % kFewK == 0 && d > kFewK && d <= 4 * kFewK) {
        pays = false;
    } else if (p.rounds >= 2 || p.waves >= 9) {
        pays = p.waves > 9 || bytes <= (int64_t)2 << 20;
    } else {
        const int padded = (d + kFewK - 1) / kFewK * kFewK;
        const bool lines = d <= 64 && ld % 32 == 0, more_waves = p.waves >= 5;
        pays = (d > kFewK && 5 * padded >= 7 * d) || (more_waves && lines) || (groups == 1 && (d >= 600 || (more_waves && d > kFewK))) ||
               (groups == 3 && more_waves && (d <= 64 || d > kFewK));
    }
    return pays ? p : no;
}
template <typename ET, int MT>
__global__ void __launch_bounds__(kPassWaves * kWave)
k_logits_pass(const ET* __restrict__ E, int64_t ld, int d, const float* __restrict__ H, int R, int V, int rounds,
              float* __restrict__ logits, int64_t cpitch, TileRecords recs) {
    constexpr bool BF = sizeof(ET) == 2;
    constexpr int NP = few_planes<ET>(), CK = 16 / (int)sizeof(ET), KSTEP = 4 * CK, RING = kPassRing;
    extern __shared__ uint4 psm[];
    char* sm = reinterpret_cast<char*>(psm);
    const int pitch = pass_pitch<ET>(d), row_bytes = pitch * (int)sizeof(ET), plane = MT * kTileM * row_bytes;
    float2* part = reinterpret_cast<float2*>(sm + NP * plane);               // [waves][16 MT]
    const int tid = threadIdx.x, ln = lane_id(), wv = __builtin_amdgcn_readfirstlane(wave_id()), W = blockDim.x >> 6;
    const int col = ln & 15, kk = ln >> 4;
    const int nst = (d + KSTEP - 1) / KSTEP, groups = (nst + RING - 1) / RING;
    const int64_t tile0 = ((int64_t)blockIdx.x * W + wv) * rounds;
    Chunk16U<ET> e[RING];
    const char* base = nullptr;                               // the tile's first row (uniform)
    uint32_t mine = 0;                                        // this lane's row from there, in bytes (the host: 16 rows below 2^31)
    const int last = d - CK;
    // (steps past the row: one address for all lanes, which costs the load path next to nothing, and no branch around the load)
    auto load = [&](int st) {
        const uint32_t at = mine + (uint32_t)min(st * KSTEP + kk * CK, last) * (uint32_t)sizeof(ET);
        const uint32_t in_row = __builtin_amdgcn_readfirstlane(st < nst ? ~0u : 0u);
        return *reinterpret_cast<const Chunk16U<ET>*>(base + (at & in_row));
    };
    auto begin = [&](int64_t tile) {
        base = reinterpret_cast<const char*>(E + tile * kTileN * ld);
        mine = (uint32_t)min(col, (int)(V - 1 - tile * kTileN)) * (uint32_t)(ld * (int64_t)sizeof(ET));
#pragma unroll
        for (int j = 0; j < RING / 2; ++j) e[j] = load(j);
        if (nst > RING / 2)   // (uniform)
#pragma unroll
            for (int j = RING / 2; j < RING; ++j) e[j] = load(j);
    };
    const bool works = tile0 * kTileN < V;   // (uniform)
    // Hidden rows, zeros past d and for rows past R; asked for ahead of the first words, all at once.
    const int quads = pitch >> 2, rows = min(R, MT * kTileM);  // (four elements)
    auto zero_rows = [&](char* of) {
        float4* to = reinterpret_cast<float4*>(of + rows * row_bytes);
        for (int i = tid; i < (MT * kTileM - rows) * row_bytes / 16; i += W * kWave) to[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    };
    if constexpr (!BF) {
        const int whole = d >> 2, pieces = (whole + kWave - 1) / kWave, pad = quads - whole;
        for (int u = wv, r = 0; u < rows * pieces; u += W) {  // (uniform)
            while ((r + 1) * pieces <= u) ++r;
            const int q = (u - r * pieces) * kWave + ln;
            if (q < whole) load_to_lds16(H + (size_t)r * d + 4 * q, sm + r * row_bytes + (q - ln) * 16);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (works) begin(tile0);
        __builtin_amdgcn_sched_barrier(0);
        for (int i = tid; i < rows * pad; i += W * kWave) {
            const int r = small_div(i, pad), q = whole + i - r * pad;
            float x[4] = {0.f, 0.f, 0.f, 0.f};
            if (q == whole)
#pragma unroll
                for (int k = 0; k < 3; ++k) if (4 * q + k < d) x[k] = H[(size_t)r * d + 4 * q + k];
            *reinterpret_cast<float4*>(sm + r * row_bytes + 16 * q) = make_float4(x[0], x[1], x[2], x[3]);
        }
        zero_rows(sm);
        if (works) wait_vmem<RING / 2>(); else wait_vmem<0>();   // (as many loads of words at least are younger; waves that fill the padding have waited there for all of theirs)
    } else {
        constexpr int AT_ONCE = 8;   // (loads behind the words' would wait for those)
        bool begun = false;
        for (int i0 = tid; i0 - tid < rows * quads; i0 += AT_ONCE * W * kWave) {   // (uniform)
            Float4U v[AT_ONCE];
            int r[AT_ONCE], q[AT_ONCE];
#pragma unroll
            for (int a = 0; a < AT_ONCE; ++a) {
                const int i = min(i0 + a * W * kWave, rows * quads - 1);       // (the last one again)
                r[a] = small_div(i, quads);
                q[a] = i - r[a] * quads;
                v[a] = *reinterpret_cast<const Float4U*>(H + (size_t)r[a] * d + min(4 * q[a], d - 4));
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!begun && works) begin(tile0);
            __builtin_amdgcn_sched_barrier(0);
            begun = true;
#pragma unroll
            for (int a = 0; a < AT_ONCE; ++a) {
                const int drop = max(4 * q[a] - (d - 4), 0);
                const float y[4] = {v[a].x, v[a].y, v[a].z, v[a].w};
                float x[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int from = k + drop;
                    x[k] = from == 0 ? y[0] : from == 1 ? y[1] : from == 2 ? y[2] : from == 3 ? y[3] : 0.f;
                }
                store_planes4(sm + r[a] * row_bytes + 8 * q[a], plane, x);
            }
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) zero_rows(sm + p * plane);
    }
    lds_barrier();
    float run_max[MT], run_sum[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) { run_max[m] = -INFINITY; run_sum[m] = 0.f; }
    const char* hb = sm + col * row_bytes + 16 * kk;
    for (int r = 0; r < rounds && (tile0 + r) * kTileN < V; ++r) {           // (uniform)
        const int word0 = (int)(tile0 + r) * kTileN;
        floatx4 acc[MT], low[MT];                             // low: bf16, as in k_logits_rows
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = low[m] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto use = [&](int st, const Chunk16U<ET>& c) {
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const char* at = hb + st * 64 + m * kTileM * row_bytes;
                if constexpr (BF) {
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        floatx4& to = p ? low[m] : acc[m];
                        to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(c), *reinterpret_cast<const bf16x8*>(at + p * plane), to, 0, 0, 0);
                    }
                } else {
                    const float4 b = *reinterpret_cast<const float4*>(at);
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(c.w[0]), b.x, acc[m], 0, 0, 0);
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(c.w[1]), b.y, acc[m], 0, 0, 0);
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(c.w[2]), b.z, acc[m], 0, 0, 0);
                    acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(c.w[3]), b.w, acc[m], 0, 0, 0);
                }
            }
        };
        for (int g = 0; g + 1 < groups; ++g) {
#pragma unroll
            for (int j = 0; j < RING; ++j) {
                use(g * RING + j, e[j]);
                e[j] = load((g + 1) * RING + j);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        const int st0 = (groups - 1) * RING, end = nst - 1 - st0;              // the row's last step, which may reach past its end
        Chunk16U<ET> tail = e[0];
#pragma unroll
        for (int j = 0; j < RING; ++j) {
            if (j < end) use(st0 + j, e[j]);   // (uniform)
            if (j == end) tail = e[j];
            if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (all operands at once would take too many registers)
        }
        drop_front(tail, max(0, min((nst - 1) * KSTEP + kk * CK - last, CK)));
        use(nst - 1, tail);
        if (r + 1 < rounds && word0 + kTileN < V) begin(tile0 + r + 1);         // (on its way while this one is finished)
        __builtin_amdgcn_sched_barrier(0);
        // lane (col, kk): hidden row 16 m + col, words word0 + 4 kk + (0..3)
        const int w = word0 + 4 * kk;
        float x[MT * 4];
#pragma unroll
        for (int i = 0; i < MT * 4; ++i) x[i] = BF ? acc[i / 4][i % 4] + low[i / 4][i % 4] : acc[i / 4][i % 4];
        if constexpr (BF)
            settle_non_finite(x, [&](int i) {
                int me = col, at = w;
                asm volatile("" : "+v"(me), "+v"(at));   // (nothing of this is worked out in advance)
                return plain_dot(E + (int64_t)min(at + i % 4, V - 1) * ld, H + (size_t)min(i / 4 * kTileM + me, R - 1) * d, d);
            });
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int row = m * kTileM + col;
            if (row < R && w < V)   // (columns past V inside the row's pitch are never read)
                *reinterpret_cast<float4*>(&logits[(size_t)row * cpitch + w]) = make_float4(x[4 * m], x[4 * m + 1], x[4 * m + 2], x[4 * m + 3]);
            float mx = -INFINITY, se = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) mx = fmaxf(mx, w + i < V ? x[4 * m + i] : -INFINITY);
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
#pragma unroll
            for (int i = 0; i < 4; ++i) se += w + i < V ? exp_below(x[4 * m + i], mx) : 0.f;
            se += __shfl_xor(se, 16);
            se += __shfl_xor(se, 32);
            const float hi = fmaxf(run_max[m], mx);
            run_sum[m] = run_sum[m] * exp_below(run_max[m], hi) + se * exp_below(mx, hi);
            run_max[m] = hi;
        }
    }
    if (kk == 0)
#pragma unroll
        for (int m = 0; m < MT; ++m) part[wv * (MT * kTileM) + m * kTileM + col] = make_float2(run_max[m], run_sum[m]);
    lds_barrier();
    if (tid < MT * kTileM && tid < R) {
        float2 a = part[tid];
        for (int o = 1; o < W; ++o) {
            const float2 q = part[o * (MT * kTileM) + tid];   // (a wave past V: -inf, 0)
            const float hi = fmaxf(a.x, q.x);
            a = make_float2(hi, a.y * exp_below(a.x, hi) + q.y * exp_below(q.x, hi));
        }
        reinterpret_cast<float2*>(recs.rec)[(size_t)tid * recs.pitch + blockIdx.x] = a;
    }
}

}  // namespace lshbeam
