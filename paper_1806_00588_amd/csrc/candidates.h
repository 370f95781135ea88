// Winner-take-all hashing, cuckoo probe, bucket walk and candidate-list compaction.
//
//   k_row_codes   : band codes (Eq. 4-8) of n rows; used on E at build time and for inspection.
//   k_candidates  : one workgroup per sentence.  Hashes the sentence's B hidden rows, probes the
//                   per-band cuckoo tables (Algorithm 1, lines 1-2), walks the hit spans
//                   (lines 3-6) marking a V-bit presence bitmap held in LDS, ORs in the
//                   top-frequent words (Eq. 3) and compacts the bitmap into an ascending id list
//                   (Eq. 10 with t = 1).
//   k_part_bitmaps: the same hashing for a range of a sentence's rows, the bitmap left in global
//                   memory (sentences with many beams are hashed by several workgroups).
//   k_hit_rows    : hit threshold t > 1 (Eq. 9-10 in full): one workgroup per hidden row counts
//                   the row's collisions per word in LDS and leaves the thresholded bitmap.
//   k_union_compact: OR of a sentence's part / row bitmaps + top-frequent words + compaction.
//
// The paper keeps an integer hit matrix L[B,V] in global memory and compacts it with a shared-
// memory scan by lane 0 of each warp.  With t = 1 only "hit at least once" matters, so L
// collapses to one bit per word per sentence; V bits fit in LDS (25 KB at V = 200k), the marks
// are idempotent LDS atomic ORs, and compaction is a popcount + wave prefix sum.  Unequal span
// lengths (the paper's warp-divergence problem) are handled by flattening: the spans' numbers of
// aligned groups of four ids are prefix-summed across all (row, band) pairs and the flat range of
// groups is dealt to threads evenly, each finding its span by binary search.
#pragma once
#include <type_traits>
#include "device_utils.h"

namespace lshbeam {

// One slot of a cuckoo table: 16 bytes so a probe is a single 128-bit load.
struct __attribute__((aligned(16))) Slot {
    int32_t key;     // band code, or -1 when empty (codes are >= 0)
    uint32_t start;  // first position of the span in the band's flat word array
    uint32_t len;    // span length
    uint32_t pad;
};

// Per-band description of its cuckoo table: two multiplicative hashes over one slot array.
struct __attribute__((aligned(32))) BandMeta {
    uint32_t slot_off;  // first slot of this band in the concatenated slot array
    uint32_t shift;     // 32 - log2(capacity)
    uint32_t a0, b0, a1, b1;
    uint32_t pad0, pad1;
};

__host__ __device__ __forceinline__ uint32_t cuckoo_hash(uint32_t a, uint32_t b, uint32_t key,
                                                         uint32_t shift) {
    return (a * key + b) >> shift;
}

// Both slots are loaded unconditionally: no dependent second probe, no divergence.  In two
// halves for callers that have other work to do while the loads are in flight.
__device__ __forceinline__ void cuckoo_load(const Slot* __restrict__ slots, const BandMeta& m,
                                            int32_t code, int4* s0, int4* s1) {
    const uint32_t h0 = cuckoo_hash(m.a0, m.b0, (uint32_t)code, m.shift);
    const uint32_t h1 = cuckoo_hash(m.a1, m.b1, (uint32_t)code, m.shift);
    *s0 = *reinterpret_cast<const int4*>(slots + m.slot_off + h0);
    *s1 = *reinterpret_cast<const int4*>(slots + m.slot_off + h1);
}
__device__ __forceinline__ void cuckoo_resolve(const int4& s0, const int4& s1, int32_t code,
                                               uint32_t* start, uint32_t* len) {
    const bool hit0 = s0.x == code, hit1 = s1.x == code;
    *start = hit0 ? (uint32_t)s0.y : (uint32_t)s1.y;
    *len = hit0 ? (uint32_t)s0.z : (hit1 ? (uint32_t)s1.z : 0u);
}
// The hit-count kernel (threshold t > 1) cuts the vocabulary into kHitSlices ranges of
// hit_slice_words(V) ids and gives every (hidden row, slice) its own workgroup.  Spans are sorted
// by id, so the part of a span that falls into slice q is contiguous; where slices 1, 2, 3 begin
// inside every span is computed once at build time and stored beside the slot (x, y, z of a
// uint4; positions relative to the span's start).
constexpr int kHitSlices = 4;
__host__ __device__ inline int hit_slice_words(int V) {  // ids per slice: a multiple of 128
    return (((V + kHitSlices - 1) / kHitSlices) + 127) & ~127;
}

// The probe restricted to vocabulary slice q: (start, len) of the span's part inside it.  The
// cut positions of both candidate slots are loaded along with the slots (no dependent load).
__device__ __forceinline__ void cuckoo_find_slice(const Slot* __restrict__ slots,
                                                  const uint4* __restrict__ cuts, const BandMeta& m,
                                                  int32_t code, int q, uint32_t* start, uint32_t* len) {
    const uint32_t h0 = cuckoo_hash(m.a0, m.b0, (uint32_t)code, m.shift);
    const uint32_t h1 = cuckoo_hash(m.a1, m.b1, (uint32_t)code, m.shift);
    const int4 s0 = *reinterpret_cast<const int4*>(slots + m.slot_off + h0);
    const int4 s1 = *reinterpret_cast<const int4*>(slots + m.slot_off + h1);
    const uint4 c0 = cuts[m.slot_off + h0], c1 = cuts[m.slot_off + h1];
    const bool hit0 = s0.x == code, hit1 = s1.x == code;
    const uint32_t st = hit0 ? (uint32_t)s0.y : (uint32_t)s1.y;
    const uint32_t ln = hit0 ? (uint32_t)s0.z : (hit1 ? (uint32_t)s1.z : 0u);
    const uint4 c = hit0 ? c0 : c1;
    const uint32_t lo = (q == 0) ? 0u : (q == 1) ? c.x : (q == 2) ? c.y : c.z;
    const uint32_t hi = (q == 0) ? c.x : (q == 1) ? c.y : (q == 2) ? c.z : ln;
    *start = st + min(lo, ln);
    *len = (ln && hi > lo) ? min(hi, ln) - min(lo, ln) : 0u;
}

// Band codes (Eq. 4-8) of n rows, any pitch and alignment.  A workgroup copies `rows` = 2^lg_rows of
// them to LDS in 16-byte pieces, a wave per row; one thread per (row, permutation) takes the windowed
// argmax there (strict '>', so the lowest k wins a tie; a permutation's window positions stay in
// registers from row to row), one per (row, band) packs the codes, first code in the most significant
// bits.  The floor is one pass over the rows.  AHEAD (one permutation per thread, so that nothing else is read from
// memory): a workgroup stays for many groups of rows, and the next one is on its way, straight to the other half of
// its LDS, while this one is hashed.  V = 40000, d = 1000, P = 32, K = 8 (160 MB): 36 -> 30 us, 5.4 TB/s
// (a thread per (row, band) gathering from memory took 151).
// LDS: rows x pitch bytes (a multiple of 16; AHEAD: twice), then rows x P 16-bit codes.
constexpr int kRowCodeThreads = 256, kRowCodeWindow = 16;   // (longer windows are read again for every row)
inline size_t row_codes_pitch(int d, size_t elem) { return ((size_t)d * elem + 15) & ~(size_t)15; }
inline size_t row_codes_lds(int rows, int d, size_t elem, int P, bool ahead) {
    return rows * ((ahead ? 2 : 1) * row_codes_pitch(d, elem) + 2 * (size_t)P);
}
// Window positions in registers, room for two rows; and few permutations: with more the windows' LDS reads bound the
// kernel, and fewer, larger groups of rows do better (bf16, V = 200000, d = 1024: 64 permutations 109 us, 132 AHEAD;
// V = 150000, d = 300, 60: 59, 63; fp32, V = 100000, d = 1000, 48 of 16 positions: 122, 97; d = 512 bf16, 24: 33, 28;
// d = 64, 16: 32, 23).
constexpr int kRowCodeAheadP = 48;
inline bool row_codes_ahead(int d, size_t elem, int P, int K) {
    return P <= kRowCodeAheadP && K <= kRowCodeWindow && row_codes_lds(1, d, elem, P, true) <= 78 * 1024;
}
// Rows per workgroup, at most 16.  AHEAD: as few as have a window for every thread.  Otherwise as many as leave room for
// four workgroups on a CU and for two on every CU.
inline int row_codes_lg_rows(int64_t n, int d, size_t elem, int P, bool ahead) {
    int lg = 4;
    if (ahead)
        while (lg > 0 && (P << (lg - 1)) >= kRowCodeThreads) --lg;
    const size_t lds = ahead || P > kRowCodeThreads ? 78 * 1024 : 39 * 1024;   // (many permutations: their loads are shared by more rows)
    while (lg > 0 && (row_codes_lds(1 << lg, d, elem, P, ahead) > lds || (n >> lg) < 512)) --lg;
    return lg;
}
// FIRST is what the first workgroups of a build's launch do while their first rows are on their way (build_tables.h); NotFirst: nothing.
// kRaw: the permutations are the caller's as they came, and positions outside a row count as 0.  (AHEAD only.  Without it each of many
// workgroups reads its windows, and a look at every position made each wait for its load: V = 200000, d = 1024 bf16, 64
// permutations, the build 192 -> 216 us.)
struct NotFirst {
    static constexpr bool kRaw = false;
    __device__ void run() const {}
};
template <typename ET, bool AHEAD, class FIRST>
__global__ void __launch_bounds__(kRowCodeThreads)
k_row_codes(const ET* __restrict__ X, int64_t ld, int64_t n, int d, const int32_t* __restrict__ perms, int P, int K,
            int W, int bits, int lg_rows, int32_t* __restrict__ out, int64_t row_stride, int64_t band_stride, FIRST first) {
    static_assert(AHEAD || !FIRST::kRaw, "windows longer than kRowCodeWindow are read as they are");
    constexpr int CK = 16 / (int)sizeof(ET), NW = kRowCodeThreads / kWave;
    extern __shared__ uint4 row_sm[];
    const int rows = 1 << lg_rows, pitch = (int)((d * sizeof(ET) + 15) & ~(size_t)15);
    char* half[2] = {reinterpret_cast<char*>(row_sm), reinterpret_cast<char*>(row_sm) + (AHEAD ? (size_t)rows * pitch : 0)};
    uint16_t* codes = reinterpret_cast<uint16_t*>(half[1] + (size_t)rows * pitch);   // [rows][P]
    const int tid = threadIdx.x, ln = lane_id(), rw = __builtin_amdgcn_readfirstlane(wave_id());
    const int nch = d / CK, rest = d - nch * CK, u = P / W;
    const int64_t groups = (n + rows - 1) >> lg_rows;
    constexpr int MOST = 16 / NW;   // rows of a wave
    ET tail[MOST];                  // the elements behind a row's whole chunks, a lane each
    auto load = [&](int64_t g, char* to) {
#pragma unroll
        for (int j = 0; j < MOST; ++j) {
            const int r = rw + j * NW;
            if (r >= rows) break;   // (uniform)
            const ET* row = X + min((g << lg_rows) + r, n - 1) * ld;
            if (ln < rest) tail[j] = row[nch * CK + ln];
            for (int p = 0; p < nch; p += kWave)
                if (p + ln < nch) load_to_lds16(row + (size_t)CK * (p + ln), to + (size_t)r * pitch + 16 * p);
        }
    };
    auto argmax = [&](const ET* row, const int (&idx)[kRowCodeWindow], const int32_t* pm) {
        float v[kRowCodeWindow];
#pragma unroll
        for (int k = 0; k < kRowCodeWindow; ++k)
            if (k < K) v[k] = elem_f32(row + idx[k]);   // (uniform)
        int best = 0;
        float bv = v[0];
#pragma unroll
        for (int k = 1; k < kRowCodeWindow; ++k)
            if (k < K && v[k] > bv) { bv = v[k]; best = k; }
        for (int k = kRowCodeWindow; k < K; ++k) {
            const float x = elem_f32(row + pm[k]);
            if (x > bv) { bv = x; best = k; }
        }
        return best;
    };
    int idx[kRowCodeWindow];
    auto window = [&](int p) {
        const int32_t* pm = perms + (size_t)p * K;
#pragma unroll
        for (int k = 0; k < kRowCodeWindow; ++k)
            if (k < K) idx[k] = pm[k];
        if constexpr (FIRST::kRaw) {
#pragma unroll
            for (int k = 0; k < kRowCodeWindow; ++k)
                if (k < K) idx[k] = (uint32_t)idx[k] < (uint32_t)d ? idx[k] : 0;
        }
    };
    const int np0 = min(P, kRowCodeThreads), at_once = kRowCodeThreads / np0;  // (AHEAD) rows hashed side by side
    const int my_r = small_div(tid, np0), my_p = tid - my_r * np0;
    if (AHEAD) window(my_p);
    load(blockIdx.x, half[0]);
    first.run();
    int b = 0;
    for (int64_t g = blockIdx.x; g < groups; g += gridDim.x) {                // (without AHEAD: once)
        char* stage = half[b];
        wait_vmem<0>();
#pragma unroll
        for (int j = 0; j < MOST; ++j)
            if (rw + j * NW < rows && ln < rest) reinterpret_cast<ET*>(stage + (size_t)(rw + j * NW) * pitch)[nch * CK + ln] = tail[j];
        lds_barrier();
        if (AHEAD && g + gridDim.x < groups) load(g + gridDim.x, half[b ^ 1]);
        if (AHEAD) {
            if (my_r < at_once)
                for (int r = my_r; r < rows; r += at_once)
                    codes[r * P + my_p] = (uint16_t)argmax(reinterpret_cast<const ET*>(stage + (size_t)r * pitch), idx, nullptr);
        } else {
            for (int p0 = 0; p0 < P; p0 += kRowCodeThreads) {
                const int np = min(P - p0, kRowCodeThreads), side = kRowCodeThreads / np;   // (uniform)
                const int r0 = small_div(tid, np), p = p0 + tid - r0 * np;
                if (r0 >= side) continue;
                window(p);
                for (int r = r0; r < rows; r += side)
                    codes[r * P + p] = (uint16_t)argmax(reinterpret_cast<const ET*>(stage + (size_t)r * pitch), idx, perms + (size_t)p * K);
            }
        }
        lds_barrier();
        const int64_t row0 = g << lg_rows;
        for (int i = tid; i < (W << lg_rows); i += kRowCodeThreads) {
            const int r = i & (rows - 1), w = i >> lg_rows;
            int32_t code = 0;
            for (int q = 0; q < u; ++q) code = (code << bits) | codes[r * P + w * u + q];
            if (row0 + r < n) out[(row0 + r) * row_stride + w * band_stride] = code;
        }
        b ^= 1;
    }
}

constexpr int kCandThreads = 1024;
constexpr int kCandWaves = kCandThreads / kWave;
// Hidden values staged in LDS per chunk of rows (floats): at least this much (or one row, if a row
// is longer), more when a step's sentences have more beams and LDS has room (the host decides per
// step and passes the size along: CandArgs::stage_words, a multiple of 4).
constexpr int kDirectFlag = 32;      // word of the scan scratch that holds the direct walk's verdict
constexpr int kCandStage = 12288;
constexpr int kCandStageRows = 32;   // a larger stage is sized for at most this many rows
__host__ __device__ inline int candidates_min_stage(int d) {
    return ((d > kCandStage ? d : kCandStage) + 3) & ~3;
}

// Rows of a sentence are processed in chunks small enough that the chunk's hidden rows fit the
// LDS stage and its (row, band) pairs fit one workgroup-wide scan.
__host__ __device__ inline int candidates_rows_per_chunk(int B, int d, int W, int stage_words) {
    int rows = stage_words / d;
    if (rows > kCandThreads / W) rows = kCandThreads / W;
    if (rows > B) rows = B;
    return rows < 1 ? 1 : rows;
}

// LDS words k_candidates needs.  The stage always holds at least one hidden row.
// Words reserved for the V-bit bitmap: rounded to 4 so that what follows is 16-byte aligned.
__host__ __device__ inline int bitmap_words_padded(int V) { return (((V + 31) >> 5) + 3) & ~3; }

__host__ __device__ inline size_t candidates_lds_words(int V, int P, int K, int stage_words) {
    return (size_t)bitmap_words_padded(V) + (size_t)stage_words + (size_t)P * K +
           3 * (size_t)kCandThreads + 64;
}

// Branch-free search in an ascending LDS array of kCandThreads entries whose first entry is 0:
// the last index whose value is <= e.  Always ten steps, so two searches interleave well.
__device__ __forceinline__ int last_not_above(const uint32_t* pref, uint32_t e) {
    int lo = 0;
#pragma unroll
    for (int step = kCandThreads / 2; step >= 1; step >>= 1)
        if (pref[lo + step] <= e) lo += step;
    return lo;
}

// Marks the ids of a list in an LDS bitmap.  Ids that fall into the same bitmap word are OR-ed
// inside the wave first and one lane issues the atomic: same-address LDS atomics serialise, and
// frequent-word ids tend to be consecutive.  `first` is this thread's already loaded list[tid]
// (or -1).  Called by all kCandThreads threads.
__device__ __forceinline__ void mark_ids_of_wave(uint32_t* bm, int V, int32_t id) {
    const int ln = lane_id();
    const bool ok = id >= 0 && id < V;
    const uint32_t word = ok ? (uint32_t)(id >> 5) : 0xFFFFFFFFu;
    const uint32_t bit = ok ? (1u << (id & 31)) : 0u;
    uint64_t todo = __ballot(ok);
    bool grouped = true;
    while (todo && grouped) {
        const int leader = __ffsll((unsigned long long)todo) - 1;
        const uint32_t w0 = wave_read_lane(word, leader);
        const bool mine = ok && word == w0;
        const uint64_t grp = __ballot(mine);
        const uint32_t ored = wave_or(mine ? bit : 0u);
        if (ln == leader) atomicOr(&bm[w0], ored);
        todo &= ~grp;
        grouped = __popcll(grp) > 1;  // scattered ids: stop grouping, plain atomics below
    }
    if (ok && ((todo >> ln) & 1ull)) atomicOr(&bm[word], bit);
}
// `second`: list[tid + kCandThreads] likewise (or -1; id_list_second() asks for it).
__device__ __forceinline__ int32_t id_list_second(const int32_t* __restrict__ list, int T) {
    const int i = (int)threadIdx.x + kCandThreads;
    return (T > kCandThreads && i < T) ? list[i] : -1;   // (a uniform branch for short lists)
}
template <bool SECOND = false>
__device__ __forceinline__ void mark_id_list(uint32_t* bm, int V, const int32_t* __restrict__ list,
                                             int T, int32_t first, int32_t second = -1) {
    // the first round (with SECOND, the first two) has its ids in registers: kept apart from the
    // loop so that it contains no load (and no wait that would also cover loads the caller has
    // in flight)
    if (T > 0) mark_ids_of_wave(bm, V, first);
    if (SECOND && T > kCandThreads) mark_ids_of_wave(bm, V, second);
    for (int i = (SECOND ? 2 : 1) * kCandThreads + (int)threadIdx.x; i - (int)threadIdx.x < T; i += kCandThreads)
        mark_ids_of_wave(bm, V, (i < T) ? list[i] : -1);
}

// Arguments of candidate generation (everything k_candidates takes except its outputs).
struct CandArgs {
    const float* H;          // [S*B, d] hidden rows
    int B, d;
    const int32_t* perms;    // [P, K]
    int P, K, W, bits;
    const Slot* slots;
    const BandMeta* bands;   // [W]
    const int32_t* words;    // [W, V]
    int V;
    const int32_t* topfreq;  // [T]
    int T;
    const uint4* cuts;       // per slot: where the vocabulary slices 1, 2, 3 begin inside its span
    int stage_words;         // LDS words for the staged hidden rows (>= d, a multiple of 4)
    // derived on the host (set_derived), so that no division stands before the kernel's first loads
    int rows_chunk;          // candidates_rows_per_chunk(B, d, W, stage_words)
    int u;                   // P / W codes per band
};

inline void set_derived(CandArgs& a) {
    a.rows_chunk = candidates_rows_per_chunk(a.B, a.d, a.W, a.stage_words);
    a.u = a.P / a.W;
}

// Builds sentence s's presence bitmap (V bits, at smem[0 .. ceil(V/32))) in LDS: hashing, cuckoo
// probes, bucket walk and the top-frequent words.  Only the sentence's rows [row_begin, row_end)
// are hashed (row_end < 0: all B).  Called by all kCandThreads threads of a workgroup with
// candidates_lds_words() words of LDS; ends with a workgroup barrier.
// DEEP (for the kernels that have the registers): walks of more than two groups of ids per thread
// keep four or eight span reads in flight, and the second thousand of top-frequent ids is asked for up
// front too.
template <bool DEEP = false>
__device__ __forceinline__ void build_presence_bitmap(const CandArgs& a, int s, uint32_t* smem,
                                                      int row_begin = 0, int row_end = -1) {
    const float* __restrict__ H = a.H;
    const int B = a.B, d = a.d, P = a.P, K = a.K, W = a.W, bits = a.bits, V = a.V, T = a.T;
    const int32_t* __restrict__ perms = a.perms;
    const Slot* __restrict__ slots = a.slots;
    const BandMeta* __restrict__ bands = a.bands;
    const int32_t* __restrict__ words = a.words;
    const int32_t* __restrict__ topfreq = a.topfreq;
    const int nwords = (V + 31) >> 5;
    const int stage_words = a.stage_words;
    uint32_t* bm = smem;                                   // presence bitmap, V bits
    const int bmw = bitmap_words_padded(V);
    float* stage = reinterpret_cast<float*>(bm + bmw);     // the chunk's hidden rows [rows][d]
    int32_t* lperms = reinterpret_cast<int32_t*>(bm + bmw + stage_words);  // perms [P][K]
    uint32_t* p_group = bm + bmw + stage_words + P * K;    // first group of four ids of each pair's span in the chunk
    uint32_t* p_len = p_group + kCandThreads;              // its length | misalignment << 30
    uint32_t* p_pref = p_len + kCandThreads;               // exclusive prefix of the spans' numbers of groups
    uint32_t* wsum = p_pref + kCandThreads;                // scan scratch (>= kCandWaves + 1)

    const int tid = threadIdx.x;
    const int u = a.u;
    const int rows_per_chunk = a.rows_chunk;
    if (row_end < 0) row_end = B;
    LSH_TRACE(0, 0);
    LSH_TRACE_WG(0);

    // Everything whose address is known up front is requested before anything is waited for:
    // this thread's band descriptor (its (row-in-chunk, band) pair is fixed), its first
    // top-frequent id, and its share of the first chunk of hidden rows.
    const uint32_t my_w = (uint32_t)(tid - small_div(tid, W) * W);   // (tid < 1024, W <= P <= 1024)
    const BandMeta my_meta = bands[my_w];
    const int32_t tf_first = (tid < T) ? topfreq[tid] : -1;
    const int32_t tf_second = DEEP ? id_list_second(topfreq, T) : -1;
    const float* H0 = H + (size_t)s * B * d;
    Float4U r0 = {}, r1 = {}, r2 = {}, r3 = {};   // (rows start at any float)
    {
        const int n4 = (min(rows_per_chunk, row_end - row_begin) * d) >> 2;
        if (n4 > 0) {
            const Float4U* H4 = reinterpret_cast<const Float4U*>(H0 + (size_t)row_begin * d);
            r0 = H4[min(tid, n4 - 1)];
            r1 = H4[min(tid + kCandThreads, n4 - 1)];
            r2 = H4[min(tid + 2 * kCandThreads, n4 - 1)];
            r3 = H4[min(tid + 3 * kCandThreads, n4 - 1)];
        }
    }
    const int32_t perm_first = (tid < P * K) ? perms[tid] : 0;
    __builtin_amdgcn_sched_barrier(0);  // keep the loads above where they are: issued first
    for (int i = tid; i < nwords; i += kCandThreads) bm[i] = 0u;
    if (tid < P * K) lperms[tid] = perm_first;
    for (int i = tid + kCandThreads; i < P * K; i += kCandThreads) lperms[i] = perms[i];
    LSH_TRACE(0, 1);
    // (no barrier here: the first chunk's staging barrier below also covers the cleared bitmap
    // and the staged permutations)
    bool topfreq_marked = false;

    for (int row0 = row_begin; row0 < row_end; row0 += rows_per_chunk) {
        const int rows = min(rows_per_chunk, row_end - row0);
        // The chunk's hidden rows are contiguous: copy them to LDS with coalesced loads (a row's
        // P*K permuted coordinates touch nearly every cache line of the row anyway), so that the
        // permuted gathers of Eq. 5 are LDS reads and no global load depends on another.
        const float* Hc = H0 + (size_t)row0 * d;
        const int nval = rows * d;
        {
            const Float4U* H4 = reinterpret_cast<const Float4U*>(Hc);
            float4* S4 = reinterpret_cast<float4*>(stage);
            auto put = [&](int e, const Float4U& r) { S4[e] = make_float4(r.x, r.y, r.z, r.w); };
            const int n4 = nval >> 2;
            for (int e0 = tid; e0 < n4; e0 += 4 * kCandThreads) {  // 4 independent loads in flight
                if (row0 != row_begin || e0 != tid) {  // the very first batch is already in registers
                    r0 = H4[min(e0, n4 - 1)];
                    r1 = H4[min(e0 + kCandThreads, n4 - 1)];
                    r2 = H4[min(e0 + 2 * kCandThreads, n4 - 1)];
                    r3 = H4[min(e0 + 3 * kCandThreads, n4 - 1)];
                }
                put(e0, r0);
                if (e0 + kCandThreads < n4) put(e0 + kCandThreads, r1);
                if (e0 + 2 * kCandThreads < n4) put(e0 + 2 * kCandThreads, r2);
                if (e0 + 3 * kCandThreads < n4) put(e0 + 3 * kCandThreads, r3);
            }
            if (tid < (nval & 3)) stage[(nval & ~3) + tid] = Hc[(nval & ~3) + tid];
        }
        LSH_TRACE(0, 12);
        if (tid == 0) wsum[kDirectFlag] = 0u;   // "a span of this chunk is too long for the direct walk"
        __syncthreads();
        LSH_TRACE(0, 2);
        LSH_TRACE_WG(1);

        // Eq. 4-5: one thread per (row, permutation) takes the windowed argmax from the staged
        // row (strict '>' in window order, so the lowest k wins a tie); codes go to LDS.  When
        // the chunk has more codes than threads, each pair's thread computes its own u codes.
        const int npairs = rows * W;
        const bool par_codes = rows * P <= kCandThreads;
        uint32_t* codes = p_pref;  // free until the scan below
        auto wta = [&](const float* sv, const int32_t* pm) {
            int best = 0;
            float bv = -INFINITY;
            bool first = true;
            for (int k0 = 0; k0 < K; k0 += 8) {  // 8 window entries per round of LDS reads
                int idx[8];
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) idx[j] = pm[min(k0 + j, K - 1)];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = sv[idx[j]];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    if (k0 + j < K && (first || v[j] > bv)) { bv = v[j]; best = k0 + j; }
                    first = false;
                }
            }
            return best;
        };
        if (par_codes) {
            if (tid < rows * P) {
                const int i = small_div(tid, P), p = tid - i * P;
                codes[tid] = (uint32_t)wta(stage + (size_t)i * d, lperms + (size_t)p * K);
            }
            __syncthreads();
        }
        // Eq. 6-8 (first code most significant), then Algorithm 1 lines 1-2 for this pair
        uint32_t start = 0, len = 0, w = 0;
        int32_t code = 0;
        int4 slot0, slot1;
        if (tid < npairs) {
            const int i = small_div(tid, W);
            w = my_w;
            for (int q = 0; q < u; ++q) {
                const int best = par_codes
                    ? (int)codes[i * P + (int)w * u + q]
                    : wta(stage + (size_t)i * d, lperms + ((size_t)w * u + q) * K);
                code = (code << bits) | best;
            }
        }
        // (threads without a pair probe code 0 of their band and drop the result: a load inside
        // the branch would have to be waited for where the branch ends)
        cuckoo_load(slots, my_meta, code, &slot0, &slot1);
        // Eq. 3: the top-frequent words are members of every candidate list.  Marked here, while
        // the first chunk's probes are on their way (the bitmap was cleared before the staging
        // barrier; every consumer of the bitmap comes after the barrier that ends the chunk).
        if (!topfreq_marked) {
            mark_id_list<DEEP>(bm, V, topfreq, T, tf_first, tf_second);
            topfreq_marked = true;
            LSH_TRACE(0, 11);
        }
        // (the compiler would otherwise compare the slots -- and wait for them -- right after
        // the loads, before the marking; this pins their first use here)
        asm volatile("" : "+v"(slot0.x), "+v"(slot0.y), "+v"(slot0.z), "+v"(slot1.x), "+v"(slot1.y),
                          "+v"(slot1.z) :: "memory");
        if (tid < npairs) cuckoo_resolve(slot0, slot1, code, &start, &len);
        // Short spans are walked without the scan and the search below: kCandThreads / npairs
        // threads share a span, each taking every subs-th aligned group of four ids of the flat
        // word array (the array is padded, so a group may reach past a span's end but never past
        // the allocation), at most kDirectGroups groups per thread.  One span too long for that:
        // the flat walk for the whole chunk.
        constexpr int kDirectGroups = 4;
        const int subs = kCandThreads / npairs;
        {
            const size_t flat = (size_t)w * V + start;
            const uint32_t mis = (uint32_t)flat & 3u;
            p_group[tid] = (uint32_t)(flat >> 2);               // first group (W * V < 2^34)
            p_len[tid] = len | (mis << 30);                     // (len <= V <= 2^24)
            if (((len + mis + 3) >> 2) > (uint32_t)(subs * kDirectGroups)) wsum[kDirectFlag] = 1u;
        }
        __syncthreads();  // codes[] aliases p_pref
        LSH_TRACE(0, 3);
        LSH_TRACE_WG(2);
        if (wsum[kDirectFlag] == 0u) {   // (uniform)
            const int sub = small_div(tid, npairs), pair = tid - sub * npairs;
            const uint32_t g0 = p_group[pair], lm = p_len[pair];
            const uint32_t slen = lm & 0x3FFFFFFFu, smis = lm >> 30;
            const uint32_t ngroups = (sub < subs && slen) ? (slen + smis + 3) >> 2 : 0u;
            const int4* __restrict__ words4 = reinterpret_cast<const int4*>(words);
            int4 grp[kDirectGroups];
#pragma unroll
            for (int j = 0; j < kDirectGroups; ++j) {
                const uint32_t g = (uint32_t)(sub + subs * j);
                if (j > 0 && __ballot(g < ngroups) == 0ull) { grp[j] = make_int4(0, 0, 0, 0); continue; }   // (uniform)
                grp[j] = words4[(size_t)g0 + (g < ngroups ? g : 0u)];
            }
#pragma unroll
            for (int j = 0; j < kDirectGroups; ++j) {
                const uint32_t g = (uint32_t)(sub + subs * j);
                if (__ballot(g < ngroups) == 0ull) continue;   // (uniform)
                const uint32_t p0 = 4u * g;                    // position of the group's first id in the span + smis
                const int32_t ids[4] = {grp[j].x, grp[j].y, grp[j].z, grp[j].w};
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (g < ngroups && p0 + c >= smis && p0 + c < smis + slen)
                        atomicOr(&bm[ids[c] >> 5], 1u << (ids[c] & 31));
            }
            __syncthreads();
            LSH_TRACE(0, 5);
            LSH_TRACE_WG(3);
            continue;
        }
        const uint32_t my_groups = len ? (len + (((uint32_t)((size_t)w * V + start)) & 3u) + 3u) >> 2 : 0u;
        uint32_t total;
        const uint32_t incl = block_incl_scan(my_groups, wsum, &total);
        LSH_TRACE(0, 4);
        p_pref[tid] = incl - my_groups;
        __syncthreads();
        // Algorithm 1 lines 3-6 as a flat walk over the aligned groups of four ids of all spans of the chunk: group e
        // belongs to the last pair whose exclusive prefix is <= e.  (By single ids, four times the searches, ten reads of LDS at
        // unlike banks each: of 12000 ids of 160 spans, 64 x 10 beams, V = 200000, 5.7 us, 3 so.)  An index past the end is clamped
        // for the load and skipped for the mark: hundreds of atomics on the last group's words would serialise.  Long walks
        // keep four reads in flight per thread (eight beyond eight groups per thread: a round is a trip to memory), short ones two.
        const int4* __restrict__ words4 = reinterpret_cast<const int4*>(words);
        auto walk = [&](auto width_tag) {
            constexpr int NW = decltype(width_tag)::value;
            for (uint32_t e0 = tid; e0 < total; e0 += NW * kCandThreads) {
                uint32_t e[NW];
                int l[NW];
                int4 grp[NW];
#pragma unroll
                for (int q = 0; q < NW; ++q) e[q] = min(e0 + (uint32_t)(q * kCandThreads), total - 1);
#pragma unroll
                for (int q = 0; q < NW; ++q) l[q] = last_not_above(p_pref, e[q]);
#pragma unroll
                for (int q = 0; q < NW; ++q) {
                    e[q] -= p_pref[l[q]];   // (the group's number in its span)
                    grp[q] = words4[(size_t)p_group[l[q]] + e[q]];
                }
#pragma unroll
                for (int q = 0; q < NW; ++q) {
                    const uint32_t lm = p_len[l[q]], smis = lm >> 30, send = smis + (lm & 0x3FFFFFFFu), p0 = 4u * e[q];
                    const int32_t ids[4] = {grp[q].x, grp[q].y, grp[q].z, grp[q].w};
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        if (e0 + (uint32_t)(q * kCandThreads) < total && p0 + c >= smis && p0 + c < send)
                            atomicOr(&bm[ids[c] >> 5], 1u << (ids[c] & 31));
                }
            }
        };
        if (DEEP && total > 8u * kCandThreads) walk(std::integral_constant<int, 8>{});
        else if (DEEP && total > 2u * kCandThreads) walk(std::integral_constant<int, 4>{});
        else walk(std::integral_constant<int, 2>{});
        __syncthreads();
        LSH_TRACE(0, 5);
        LSH_TRACE_WG(3);
    }
    if (!topfreq_marked) {  // no rows to hash
        __syncthreads();
        mark_id_list<DEEP>(bm, V, topfreq, T, tf_first, tf_second);
        __syncthreads();
    }
}

// Compaction of a V-bit LDS bitmap into the ascending id list out[0..count) (Eq. 10's selection
// made dense; the paper's Fig. 5 step).  Each wave owns a contiguous range of bitmap words (a
// multiple of 64 of them); popcount + wave prefix sum give every lane the output offset of its
// word's ids.  A sparse word is expanded by its own lane (neighbouring lanes write neighbouring
// addresses).  Dense words -- the top-frequent ids usually fill whole words, and they sit next
// to each other, in one wave's range -- would make each lane write a long private run, 128 bytes
// apart from its neighbour's, and that one wave would expand them all: they are put on a list
// in LDS instead (word, output offset) and, after a barrier, expanded by ALL waves, 32 lanes per
// word, one lane per bit, so that the stores are contiguous.  Dense words beyond the list's
// capacity are expanded by their own wave, two at a time.
// PARTS workgroups with the same bitmap share the work: wave w of workgroup `part` has range w PARTS + part of 16 PARTS, and every
// workgroup counts all of them.
// Called by all kCandThreads threads; wsum is LDS scratch of 16 PARTS words, ndense one word, dlist LDS
// room for dcap entries.
template <int PARTS>
__device__ __forceinline__ void compact_bitmap(const uint32_t* bm, int nwords, uint32_t* wsum, uint32_t* ndense,
                                               uint2* dlist, int dcap, int32_t* __restrict__ out,
                                               int32_t* __restrict__ count_out, int part) {
    static_assert(kCandWaves * PARTS <= kWave, "a lane per range");
    const int tid = threadIdx.x, wv = wave_id(), ln = lane_id();
    int per_range = (nwords + kCandWaves * PARTS - 1) / (kCandWaves * PARTS);
    per_range = (per_range + kWave - 1) / kWave * kWave;
#pragma unroll
    for (int p = 0; p < PARTS; ++p) {
        const int beg = (wv * PARTS + p) * per_range, end = min(nwords, beg + per_range);
        uint32_t cnt = 0;
        for (int i = beg + ln; i < end; i += kWave) cnt += __popc(bm[i]);
        cnt = wave_sum(cnt);
        if (ln == 0) wsum[wv * PARTS + p] = cnt;
    }
    if (tid == 0) *ndense = 0;  // entries on the dense list
    __syncthreads();
    const int range = __builtin_amdgcn_readfirstlane(wv * PARTS + part);
    const uint32_t in_range = ln < kCandWaves * PARTS ? wsum[ln] : 0u, upto = wave_incl_scan(in_range);
    uint32_t running = wave_read_lane(upto - in_range, range);
    const uint32_t total = wave_read_lane(upto, kWave - 1);
    const int wbeg = range * per_range, wend = min(nwords, wbeg + per_range);
    const int half = ln >> 5, hbit = ln & 31;
    for (int i0 = wbeg; i0 < wend; i0 += kWave) {
        const int i = i0 + ln;
        const uint32_t bitsw = (i < wend) ? bm[i] : 0u;
        const uint32_t c = __popc(bitsw);
        const uint32_t incl = wave_incl_scan(c);
        const uint32_t off = running + incl - c;
        const bool dense = c >= 12;
        uint64_t dmask = __ballot(dense);
        if (!dense) {
            uint32_t b = bitsw, o = off;
            while (b) {
                out[o++] = (i << 5) + (__ffs(b) - 1);
                b &= b - 1;
            }
        }
        if (dmask) {  // wave-uniform
            uint32_t base = 0;
            if (ln == 0) base = atomicAdd(ndense, (uint32_t)__popcll(dmask));
            base = wave_read_lane(base, 0);
            const uint32_t pos = base + lanes_below(dmask);
            const bool listed = dense && pos < (uint32_t)dcap;
            if (listed) dlist[pos] = make_uint2((uint32_t)i, off);
            dmask = __ballot(dense && !listed);
        }
        while (dmask) {  // wave-uniform: what the list had no room for
            const int la = __ffsll((unsigned long long)dmask) - 1;
            dmask &= dmask - 1;
            const int lb = dmask ? __ffsll((unsigned long long)dmask) - 1 : la;
            const bool have_b = dmask != 0;
            dmask &= dmask - 1;  // no-op on zero
            const uint32_t wa = wave_read_lane(bitsw, la), wb = wave_read_lane(bitsw, lb);
            const uint32_t oa = wave_read_lane(off, la), ob = wave_read_lane(off, lb);
            const uint32_t wbits = half ? wb : wa;
            const uint32_t woff = half ? ob : oa;
            const int wlane = half ? lb : la;
            const bool set = ((wbits >> hbit) & 1u) && (half == 0 || have_b);
            const uint32_t pos = __popc(wbits & ((1u << hbit) - 1u));
            if (set) out[woff + pos] = ((i0 + wlane) << 5) + hbit;
        }
        running += wave_read_lane(incl, kWave - 1);
    }
    if (part == 0 && tid == 0) *count_out = (int32_t)total;
    __syncthreads();
    // the listed dense words: half a wave per word, all waves
    const int nlisted = (int)min(*ndense, (uint32_t)dcap);
    for (int k = 2 * wv + half; k < nlisted; k += 2 * kCandWaves) {
        const uint2 ent = dlist[k];
        const uint32_t wbits = bm[ent.x];
        const uint32_t pos = __popc(wbits & ((1u << hbit) - 1u));
        if ((wbits >> hbit) & 1u) out[ent.y + pos] = (int32_t)((ent.x << 5) + (uint32_t)hbit);
    }
}

// LDS of k_union_compact: the bitmap (rounded to an even number of words), 64 words of scan
// scratch, the dense-word list of compact_bitmap.
constexpr int kUnionDenseCap = 2048;
__host__ __device__ inline size_t union_compact_lds_words(int V) {
    return (size_t)bitmap_words_padded(V) + 64 + 2 * (size_t)kUnionDenseCap;
}

// Requires W <= kCandThreads.  Where the chip has CUs for them and the bitmap is long, kCandParts workgroups per sentence: each makes
// the whole bitmap, which takes no longer beside the others, and writes a part of the list.  One workgroup alone is bound by
// instruction issue there: with V = 200000 a wave expands seven times 64 words (4.8 us).  The line is at three times 64 words for a wave.
// us a step with four less one with one (d = 256 bf16, 1000 to 2000 top-frequent words), V = 40000, 50000 / 65600, 80000, 100000, 200000:
// 8 x 5 beams +0.2, +0.1 / -0.1, -0.3, -0.4, -1.3; 5 x 17 -0.1, -0.2 / -0.5, -0.7, -0.8, -1.8; 32 x 10 +0.1, +0.1 / -0.5, -0.7, -0.7, -1.7;
// 13 x 6 0.0, -0.2 / -0.5, -0.7, -0.8, -1.6; 64 x 10 -0.6, -0.5 / -0.6, -0.9, -1.0, -2.4.  Workgroup p S + s is part p of sentence s, so that the
// parts of a sentence are on one XCD where S is a multiple of 8.
constexpr int kCandParts = 4;
inline bool candidates_split(int S, int V) { return S * kCandParts <= 256 && V > 2 * kCandWaves * kWave * 32; }
template <int PARTS>
__global__ void LSH_PAGE_ALIGNED __launch_bounds__(kCandThreads)
k_candidates(CandArgs a, int S, int32_t* __restrict__ cand, int32_t* __restrict__ count) {
    extern __shared__ uint32_t smem[];
    const int part = PARTS == 1 ? 0 : blockIdx.x / S, s = PARTS == 1 ? blockIdx.x : blockIdx.x - part * S;
    const int nwords = (a.V + 31) >> 5;
    uint32_t* wsum = smem + candidates_lds_words(a.V, a.P, a.K, a.stage_words) - 64;
    build_presence_bitmap<true>(a, s, smem);
    // (the staged hidden rows are no longer needed: their room takes the dense-word list; nor are the prefixes in front of wsum)
    uint2* dlist = reinterpret_cast<uint2*>(smem + bitmap_words_padded(a.V));
    compact_bitmap<PARTS>(smem, nwords, wsum, wsum - 1, dlist, a.stage_words / 2, cand + (size_t)s * a.V, count + s, part);
    LSH_TRACE(0, 6);
}

// What further workgroups of a launch that hashes do, those from Args::first on: nothing, there are none.
struct Alone {
    struct Args { int first; };
    static constexpr bool kAny = false;
    static __device__ void run(const Args&, uint32_t*) {}
};

// Sentences with many beams: the hidden rows of a sentence are hashed a chunk at a time, so one
// workgroup per sentence serialises ceil(B / rows per chunk) rounds of dependent memory round
// trips.  Here the sentence is cut into `nparts` parts of `part_rows` rows, one workgroup each;
// every part leaves its own V-bit bitmap (without the top-frequent words) in global memory at
// part_bitmaps[(s * nparts + part) * ceil(V/32)], and the consumer ORs the parts (Eq. 3's union).
template <class Beside>
__global__ void __launch_bounds__(kCandThreads)
k_part_bitmaps(CandArgs a, int part_rows, int nparts, uint32_t* __restrict__ part_bitmaps, typename Beside::Args beside) {
    extern __shared__ uint32_t smem[];
    if (Beside::kAny && (int)blockIdx.x >= beside.first) return Beside::run(beside, smem);
    const int s = blockIdx.x / nparts, part = blockIdx.x - s * nparts;
    const int nwords = (a.V + 31) >> 5;
    a.T = 0;
    build_presence_bitmap<true>(a, s, smem, part * part_rows, min(a.B, (part + 1) * part_rows));
    uint32_t* out = part_bitmaps + (size_t)blockIdx.x * nwords;
    for (int i = threadIdx.x; i < nwords; i += kCandThreads) out[i] = smem[i];
}

// ---------------------------------------------------------------------------------------------
// Threshold t > 1 (Eq. 9-10 in full): the hit matrix L[i, j] counts in how many bands row i and
// word j collide, and a word is a candidate iff some row reaches t.  One workgroup per (hidden
// row, vocabulary slice) keeps its part of that row of L in LDS as 16-bit counters (the paper
// keeps L in global memory), adds one for every id of the row's W hit spans that falls into the
// slice (Algorithm 1), and leaves the thresholded bits as its part of the row's V-bit bitmap in
// global memory.  The consumer ORs the sentence's row bitmaps with the top-frequent words
// (Eq. 3).
// ---------------------------------------------------------------------------------------------

// LDS words of k_hit_rows without its load list: counters (2 per word, in blocks of 64 ids), the
// hidden row, codes (2 per word), scan scratch, three per-span arrays.
__host__ __device__ inline size_t hit_rows_fixed_lds_words(int V, int d, int P) {
    return (size_t)hit_slice_words(V) / 2 + (size_t)((d + 3) & ~3) + ((size_t)P + 1) / 2 + 32 +
           3 * (size_t)kCandThreads + 64;
}
constexpr int kHitListMin = 2048, kHitListMax = 16384;  // load-list entries per pass

// grid = S*B*kHitSlices workgroups (hidden row r = block / kHitSlices, slice q = block %
// kHitSlices).  Requires W <= kCandThreads (one span per thread), W * V < 2^30 (a 16-byte group
// index and a 4-bit mask share a word) and list_cap >= kHitListMin.
template <class Beside>
__global__ void __launch_bounds__(kCandThreads)
k_hit_rows(CandArgs a, int t, int list_cap, uint32_t* __restrict__ row_bitmaps /*[S*B, nwords]*/, typename Beside::Args beside) {
    extern __shared__ uint32_t smem[];
    if (Beside::kAny && (int)blockIdx.x >= beside.first) return Beside::run(beside, smem);
    const int V = a.V, d = a.d, P = a.P, K = a.K, W = a.W, bits = a.bits;
    const int u = P / W;
    const int nwords = (V + 31) >> 5;
    const int Vq = hit_slice_words(V);                                 // ids of a slice
    uint32_t* cnt32 = smem;                                            // Vq 16-bit counters
    const int ncnt = Vq / 2;                                           // counter words
    float* rowv = reinterpret_cast<float*>(cnt32 + ncnt);              // the hidden row
    uint16_t* codes = reinterpret_cast<uint16_t*>(rowv + ((d + 3) & ~3));
    uint32_t* wsum = reinterpret_cast<uint32_t*>(codes) + (P + 1) / 2;  // scan scratch
    uint32_t* sp_pref = wsum + 32;                 // first list entry of each span (+ the total)
    uint32_t* sp_where = sp_pref + kCandThreads + 64;  // first 16-byte group << 2 | misalignment
    uint32_t* sp_len = sp_where + kCandThreads;
    uint32_t* list = sp_len + kCandThreads;        // load list [list_cap]
    const int r = blockIdx.x / kHitSlices, slice = blockIdx.x % kHitSlices;
    const int id0 = slice * Vq;                                        // first id of the slice
    const int tid = threadIdx.x, wv = wave_id(), ln = lane_id();
    const float* hrow = a.H + (size_t)r * d;

    LSH_TRACE(3, 0);
    // this thread's band descriptor is needed only after the codes: request it now
    const BandMeta my_meta = a.bands[min(tid, W - 1)];
    for (int i = tid; i < d; i += kCandThreads) rowv[i] = hrow[i];
    for (int i = tid; i < ncnt; i += kCandThreads) cnt32[i] = 0u;
    __syncthreads();
    LSH_TRACE(3, 1);

    // Eq. 4-5: one windowed argmax per permutation (strict '>' in window order, so the lowest k
    // wins a tie); window entries are fetched eight at a time, as 16-byte loads when K allows
    const bool pvec = (K & 3) == 0 && ((uintptr_t)a.perms & 15) == 0;
    for (int p = tid; p < P; p += kCandThreads) {
        const int32_t* pm = a.perms + (size_t)p * K;
        int best = 0;
        float bv = -INFINITY;
        bool first = true;
        for (int k0 = 0; k0 < K; k0 += 8) {
            int idx[8];
            float v[8];
            if (pvec) {
                const int4 q0 = *reinterpret_cast<const int4*>(pm + k0);
                const int4 q1 = *reinterpret_cast<const int4*>(pm + min(k0 + 4, K - 4));
                idx[0] = q0.x; idx[1] = q0.y; idx[2] = q0.z; idx[3] = q0.w;
                idx[4] = q1.x; idx[5] = q1.y; idx[6] = q1.z; idx[7] = q1.w;
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) idx[j] = pm[min(k0 + j, K - 1)];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = rowv[idx[j]];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (k0 + j < K && (first || v[j] > bv)) { bv = v[j]; best = k0 + j; }
                first = false;
            }
        }
        codes[p] = (uint16_t)best;
    }
    __syncthreads();
    LSH_TRACE(3, 2);

    // Eq. 6-8 and Algorithm 1 lines 1-2: thread w packs band w's code and probes its table.
    // Span ids are read in aligned groups of four (one 16-byte load): the span covers
    // `ngroups` of them starting at group `grp0` of the flat word array, its first id sitting
    // at position `mis` of the first group.
    uint32_t grp0 = 0, mis = 0, len = 0, ngroups = 0;
    if (tid < W) {
        int32_t code = 0;
        for (int q = 0; q < u; ++q) code = (code << bits) | codes[tid * u + q];
        uint32_t start;
        cuckoo_find_slice(a.slots, a.cuts, my_meta, code, slice, &start, &len);
        if (len) {
            const size_t g0 = (size_t)tid * V + start;
            grp0 = (uint32_t)(g0 >> 2);
            mis = (uint32_t)(g0 & 3);
            ngroups = (mis + len + 3) >> 2;
        }
    }
    uint32_t total;
    const uint32_t first_entry = block_incl_scan(ngroups, wsum, &total) - ngroups;
    sp_pref[tid] = (tid < W) ? first_entry : total;
    if (tid == 0) sp_pref[kCandThreads] = total;
    sp_where[tid] = (grp0 << 2) | mis;
    sp_len[tid] = len;
    __syncthreads();
    LSH_TRACE(3, 3);

    // Algorithm 1 lines 3-6: L[i, word] += 1 for every id of every hit span.  Spans have unequal
    // lengths (the source of the paper's divergence problem): they are flattened into a list of
    // 16-byte loads in LDS -- entry = group index << 4 | which of its four ids belong to the
    // span.  Every thread writes an equal, contiguous share of the list (it finds the span of
    // its first entry by search and walks on from there), and the workgroup then consumes the
    // list interleaved, kHitInFlight loads per thread in flight.  Lists longer than list_cap
    // are handled in passes.
    const int4* words4 = reinterpret_cast<const int4*>(a.words);
    constexpr int kHitInFlight = 8;
    // Counter of word id: 64 consecutive ids share 32 LDS words, id & 31 picks the word and bit 5
    // of the id its half, so that the thresholding pass below gets whole bitmap words from a
    // ballot over the low halves and one over the high halves.
    auto bump = [&](int32_t id, uint32_t ok) {
        id -= id0;  // position inside the slice (masked-out ids of neighbouring spans may be outside)
        if (ok) atomicAdd(&cnt32[((id >> 6) << 5) | (id & 31)], (id & 32) ? 0x10000u : 1u);
    };
    for (uint32_t pass0 = 0; pass0 < total; pass0 += (uint32_t)list_cap) {
        const uint32_t pass1 = min(total, pass0 + (uint32_t)list_cap);
        // an odd share keeps the threads' writes on different LDS banks
        const uint32_t share = ((pass1 - pass0 + kCandThreads - 1) / kCandThreads) | 1u;
        const uint32_t f_lo = pass0 + (uint32_t)tid * share;
        const uint32_t f_hi = min(pass1, f_lo + share);
        if (f_lo < f_hi) {
            int w = last_not_above(sp_pref, f_lo);  // the non-empty span that holds entry f_lo
            uint32_t base = sp_pref[w], ng = sp_pref[w + 1] - base;
            uint32_t where = sp_where[w], slen = sp_len[w];
            uint32_t k = f_lo - base;
            for (uint32_t f = f_lo; f < f_hi; ++f) {
                while (k >= ng) {  // next non-empty span (there is one: f < total)
                    ++w;
                    base = sp_pref[w];
                    ng = sp_pref[w + 1] - base;
                    where = sp_where[w];
                    slen = sp_len[w];
                    k = 0;
                }
                const int m = (int)(where & 3u);
                const int lo = max(m - (int)(4 * k), 0);
                const int hi = min(m + (int)slen - (int)(4 * k), 4);
                const uint32_t mask = ((1u << hi) - 1u) & ~((1u << lo) - 1u);
                list[f - pass0] = (((where >> 2) + k) << 4) | mask;
                ++k;
            }
        }
        __syncthreads();
        LSH_TRACE(3, 7);
        const int n = (int)(pass1 - pass0);
        for (int f0 = tid; f0 < n; f0 += kHitInFlight * kCandThreads) {
            uint32_t e[kHitInFlight];
            int4 x[kHitInFlight];
#pragma unroll
            for (int j = 0; j < kHitInFlight; ++j) {
                const int f = f0 + j * kCandThreads;
                e[j] = (f < n) ? list[f] : 0u;  // entry 0: group 0, nothing valid
            }
#pragma unroll
            for (int j = 0; j < kHitInFlight; ++j) x[j] = words4[e[j] >> 4];
#pragma unroll
            for (int j = 0; j < kHitInFlight; ++j) {
                bump(x[j].x, e[j] & 1u); bump(x[j].y, e[j] & 2u);
                bump(x[j].z, e[j] & 4u); bump(x[j].w, e[j] & 8u);
            }
        }
        LSH_TRACE(3, 4);
        __syncthreads();
    }
    LSH_TRACE(3, 5);
    // Eq. 10 for this row: bit j = (L[i, j] >= t).  Lane l of a wave reads counter word
    // 64 * c + l: its low half belongs to id 128 * c + 64 * (l / 32) + l % 32, its high half to
    // that id + 32, so the two ballots are four consecutive bitmap words (in the order
    // lo[31:0], hi[31:0], lo[63:32], hi[63:32]); lanes 0..3 store them.
    uint32_t* out = row_bitmaps + (size_t)r * nwords;
    const int w0 = id0 >> 5;                          // the slice's first bitmap word
    const int nchunks = (ncnt + kWave - 1) / kWave;   // counters of ids beyond V stay zero
    for (int c0 = wv; c0 < nchunks; c0 += 4 * kCandWaves) {  // four LDS reads in flight
        uint32_t x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = (c0 + q * kCandWaves) * kWave + ln;
            x[q] = (i < ncnt) ? cnt32[i] : 0u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int c = c0 + q * kCandWaves;
            const uint64_t lo = __ballot((int)(x[q] & 0xFFFFu) >= t);
            const uint64_t hi = __ballot((int)(x[q] >> 16) >= t);
            const uint32_t mine = (ln == 0) ? (uint32_t)lo : (ln == 1) ? (uint32_t)hi
                                : (ln == 2) ? (uint32_t)(lo >> 32) : (uint32_t)(hi >> 32);
            if (ln < 4 && 4 * c + ln < ncnt / 16 && w0 + 4 * c + ln < nwords) out[w0 + 4 * c + ln] = mine;
        }
    }
    LSH_TRACE(3, 6);
}

// OR of B bitmaps of nwords words each (nwords apart) into the LDS bitmap bm; called by all
// kCandThreads threads, no barrier inside.
__device__ __forceinline__ void union_row_bitmaps(const uint32_t* __restrict__ rb, int B, int nwords,
                                                  uint32_t* bm) {
    // Two, four, eight or twelve rows' words are asked for together (a row twice is as good as once), of the rows behind a last full twelve four or
    // eight, and of more than kCandThreads words two of each thread: one trip to memory for 12 rows of 1250 words, where four rows and a word at a
    // time took six.  us a step: 500 bands, 12 beams, V = 40000 29.0 -> 28.5; 4 x 22 beams, V = 90102 69.5 -> 66.1.  Twelve for the last rows too: 1 x 13,
    // V = 90000 27.0 instead of 26.1.  (Up to eight rows have a loop of their own: 1 x 5 in the other one 22.8 -> 23.3.)
    auto words = [&](auto rows_c, auto two_c, int i) __attribute__((always_inline)) {
        constexpr int MOST = decltype(rows_c)::value, N = decltype(two_c)::value;
        const int at[2] = {i, min(i + kCandThreads, nwords - 1)};
        uint32_t x[N] = {};
        auto rows = [&](auto n_c, int b0) __attribute__((always_inline)) {
            constexpr int ROWS = decltype(n_c)::value;
            uint32_t v[ROWS][N];
#pragma unroll
            for (int b = 0; b < ROWS; ++b)
#pragma unroll
                for (int e = 0; e < N; ++e) v[b][e] = rb[(size_t)min(b0 + b, B - 1) * nwords + at[e]];
#pragma unroll
            for (int b = 0; b < ROWS; ++b)
#pragma unroll
                for (int e = 0; e < N; ++e) x[e] |= v[b][e];
        };
        if constexpr (MOST < 12) rows(rows_c, 0);
        else {
            int b0 = 0;
            for (; B - b0 > 8; b0 += 12) rows(rows_c, b0);
            if (B - b0 > 4) rows(std::integral_constant<int, 8>{}, b0);
            else if (B - b0 > 0) rows(std::integral_constant<int, 4>{}, b0);
        }
#pragma unroll
        for (int e = 0; e < N; ++e) bm[at[e]] = x[e];
    };
    auto all = [&](auto rows_c) __attribute__((always_inline)) {
        const int tid = threadIdx.x;
        for (int i = tid; i < nwords; i += 2 * kCandThreads)
            if (nwords - (i - tid) > kCandThreads) words(rows_c, std::integral_constant<int, 2>{}, i);   // (uniform)
            else words(rows_c, std::integral_constant<int, 1>{}, i);
    };
    if (B <= 2) all(std::integral_constant<int, 2>{});
    else if (B <= 4) all(std::integral_constant<int, 4>{});
    else if (B <= 8) all(std::integral_constant<int, 8>{});
    else all(std::integral_constant<int, 12>{});
}

// grid = S workgroups: OR of the sentence's B row bitmaps and the top-frequent words, compacted.
__global__ void __launch_bounds__(kCandThreads)
k_union_compact(const uint32_t* __restrict__ row_bitmaps, int B, int V,
                const int32_t* __restrict__ topfreq, int T, int32_t* __restrict__ cand,
                int32_t* __restrict__ count) {
    extern __shared__ uint32_t smem[];  // union_compact_lds_words(V)
    const int s = blockIdx.x, tid = threadIdx.x;
    const int nwords = (V + 31) >> 5;
    uint32_t* bm = smem;
    uint32_t* wsum = smem + bitmap_words_padded(V);
    uint2* dlist = reinterpret_cast<uint2*>(wsum + 64);
    const int32_t tf_first = (tid < T) ? topfreq[tid] : -1;
    const int32_t tf_second = id_list_second(topfreq, T);
    union_row_bitmaps(row_bitmaps + (size_t)s * B * nwords, B, nwords, bm);
    __syncthreads();
    mark_id_list<true>(bm, V, topfreq, T, tf_first, tf_second);
    __syncthreads();
    compact_bitmap<1>(bm, nwords, wsum, wsum + kCandWaves, dlist, kUnionDenseCap, cand + (size_t)s * V, count + s, 0);
}

}  // namespace lshbeam
