// Device-side construction of the per-band bucket tables and cuckoo tables (section "Cuckoo
// lookup", first step: T_w = {band code: [word ids]} flattened, CuckooT_w = {band code:
// (start, length)}).
//
//   1. k_build_begin: permutations checked and copied, hash parameters drawn, tables cleared.  (Where the scan
//      writes the slots there is nothing to clear, and with few permutations the first workgroups of k_row_codes do the rest: BuildFirst.)
//   2. k_row_codes (candidates.h): band codes of every embedding row, [W, V].
//   3. Every band's words are grouped by code, ids ascending inside a code: a stable radix sort of
//      the code alone (words start in id order), up to kRadixBits bits of it per pass -- ONE pass for
//      codes of up to 12 bits.  k_radix_count, k_radix_scan, k_radix_scatter.
//   4. The table code -> span.  Direct tables, where all the codes there can be have room for little: both hash
//      functions are the code itself (direct_band_meta), so that every key has its own slot, no insertion can fail,
//      and with one pass the slots come straight out of the scan.  Otherwise k_key_count / k_key_emit find the span
//      starts in the sorted codes ("keys"), and
//   5. cuckoo insertion follows, one thread per key, all bands at once (Alcantara et al.'s scheme for
//      two hash functions): a thread swaps its item into its first slot with a 64-bit
//      atomicExch; if that evicts an item, the thread carries the evicted item to that item's
//      other slot, and so on.  A chain longer than the limit marks the band as failed; failed bands
//      alone are redone with new hash parameters.
//   6. The 8-byte (code, key index) words are expanded into the 16-byte slots the probe reads.
//
// What bounds it is the pass over the embedding rows (2); the rest is a chain of short kernels.  Nothing
// is copied to the host before the whole chain is under way where tables for the most keys a band can have
// are small or nearly full (lshbeam.hip); parameters are drawn on the device, and one wait ends the build (with a copy
// of the status words where something was inserted).  V = 40000, d = 1000 fp32, 8 bands of 12 bits, with the first step on the tables: 107 us, of which 30 us
// k_row_codes (160 MB at 5.4 TB/s), 23 us the sort and the slots (count 4.8, scan 6.5, scatter 10) and 16 us the step;
// with cuckoo insertion for these codes 156, or 206 where it failed once; with the scan in one workgroup per band and a
// sum over the chunks in front in every workgroup of the scatter 130.
#pragma once
#include "candidates.h"

namespace lshbeam {

constexpr uint64_t kCuckooEmpty = ~0ull;
constexpr int kRadixThreads = 512, kRadixWaves = kRadixThreads / kWave, kRadixBits = 12, kRadixMinChunk = 2048;
constexpr int kScanDigits = 256;   // digits per workgroup of the scan
constexpr int kBuildBeginBlocks = 64;   // x extent of k_build_begin; as many "bad permutation" words

// A band is cut into chunks, a workgroup of the sort each: every vocabulary slice of the hit-count kernel into
// `per_slice` of them, so that where the slices begin inside a span is a sum over whole chunks.  Elements per chunk:
// enough that the digit counters (2^12 of them to write, scan and read per workgroup) do not outweigh the
// elements, few enough to use the chip, and at most 65535, which the 16-bit counters hold.
struct RadixChunks {
    int slice, per_slice, size;
    __host__ __device__ int count() const { return kHitSlices * per_slice; }
    __device__ void range(int c, int64_t V, int64_t* begin, int64_t* end) const {
        const int q = c / per_slice;
        const int64_t first = (int64_t)q * slice, last = min(first + slice, V);
        *begin = min(first + (int64_t)(c - q * per_slice) * size, last);
        *end = min(*begin + size, last);
    }
};
inline RadixChunks radix_chunks(int64_t V, int W) {
    int64_t c = (V * W / 256 + 1023) / 1024 * 1024;
    if (c < kRadixMinChunk) c = kRadixMinChunk;
    if (c > 32768) c = 32768;
    RadixChunks r;
    r.slice = hit_slice_words((int)V);
    r.per_slice = (int)((r.slice + c - 1) / c);
    r.size = ((r.slice + r.per_slice - 1) / r.per_slice + kWave - 1) / kWave * kWave;
    return r;
}
inline size_t radix_scatter_lds(int digits) { return (size_t)digits * (kRadixWaves * 2 + 4); }

// Hash parameters of band w at the given attempt: a SplitMix64 sequence read at that place.
__host__ __device__ inline BandMeta draw_band_meta(uint64_t seed, int w, int W, int attempt, uint32_t cap, int lg) {
    uint32_t r[4];
    for (int i = 0; i < 4; ++i) {
        uint64_t z = seed + 0x9E3779B97F4A7C15ull * (4ull * ((uint64_t)attempt * (uint32_t)W + (uint32_t)w) + (uint64_t)i + 1ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        r[i] = (uint32_t)(z ^ (z >> 31));
    }
    BandMeta m{};
    m.slot_off = (uint32_t)w * cap;
    m.shift = 32u - (uint32_t)lg;
    m.a0 = r[0] | 1u; m.b0 = r[1]; m.a1 = r[2] | 1u; m.b1 = r[3];
    return m;
}

// Both hash functions the code itself and an even offset, modulo the slots: a direct table has 2^lg slots for codes of
// fewer than lg bits.  (Every thread without work of its own probes code 0 of its band: with offsets of their own the
// bands' slots for it are on different memory channels.  A step of V = 20000, d = 512, 2 x 4 beams, 16 bands of 12 bits, took
// 0.22 us more than with cuckoo tables where every band's was its first slot, and takes the same so.)
__host__ __device__ inline uint32_t direct_offset(int w, int lg) { return ((uint32_t)w * 0x9E3779B1u >> (32 - lg)) & ~1u; }
__host__ __device__ inline BandMeta direct_band_meta(int w, int lg) {
    BandMeta m{};
    m.slot_off = (uint32_t)w << lg;
    m.shift = 32u - (uint32_t)lg;
    m.a0 = m.a1 = 1u << m.shift;
    m.b0 = m.b1 = direct_offset(w, lg) << m.shift;
    return m;
}

// grid (kBuildBeginBlocks, W + 1).  Row w < W: band w's hash parameters and empty table (only the bands
// flagged in `redo`, if given), its `failed` flag cleared.  Row W (first attempt): the permutations are
// copied, entries outside [0, d) replaced by 0 and reported (bad_perms[block], zeroed before, in host memory), the tickets zeroed.
__global__ void __launch_bounds__(256)
k_build_begin(uint64_t* __restrict__ table, BandMeta* __restrict__ bands, int W, uint32_t cap, int lg, bool direct, uint64_t seed,
              int attempt, const uint32_t* __restrict__ redo, uint32_t* __restrict__ failed, uint32_t* __restrict__ n_keys,
              const int32_t* __restrict__ perms_in, int n_perms, int d, int32_t* __restrict__ perms,
              uint32_t* __restrict__ bad_perms, unsigned int* __restrict__ tickets, int n_tickets) {
    const int w = blockIdx.y, tid = threadIdx.x;
    const uint32_t first = blockIdx.x * blockDim.x + tid, step = gridDim.x * blockDim.x;
    if (w < W) {
        const bool again = !redo || redo[w];
        if (first == 0) {
            failed[w] = 0u;
            if (n_keys) n_keys[w] = 0u;
            if (again) bands[w] = direct ? direct_band_meta(w, lg) : draw_band_meta(seed, w, W, attempt, 1u << lg, lg);
        }
        if (again)
            for (uint32_t i = first; i < cap; i += step) table[(size_t)w * cap + i] = kCuckooEmpty;
        return;
    }
    if (!perms_in) return;
    __shared__ uint32_t bad;
    if (tid == 0) bad = 0u;
    __syncthreads();
    for (uint32_t i = first; i < (uint32_t)n_perms; i += step) {
        const int32_t x = perms_in[i];
        const bool ok = x >= 0 && x < d;
        perms[i] = ok ? x : 0;
        if (!ok) bad = 1u;
    }
    for (uint32_t i = first; i < (uint32_t)n_tickets; i += step) tickets[i] = 0u;
    __syncthreads();
    if (tid == 0 && bad) bad_perms[blockIdx.x] = 1u;
}

// The same for direct tables whose slots the scan writes, by the first workgroups of k_row_codes AHEAD: 2 us and a kernel boundary less.
struct BuildFirst {
    static constexpr bool kRaw = true;
    const int32_t* perms_in;
    int32_t* perms;
    uint32_t* bad_perms;
    BandMeta* bands;
    uint32_t* n_keys;
    unsigned int* tickets;
    int n_perms, d, W, lg, n_tickets;
    __device__ __forceinline__ void run() const {
        if (blockIdx.x >= (uint32_t)kBuildBeginBlocks) return;
        const int at = (int)(blockIdx.x * blockDim.x + threadIdx.x), step = min((int)gridDim.x, kBuildBeginBlocks) * (int)blockDim.x;
        for (int i = at; i < n_perms; i += step) {
            const int32_t x = perms_in[i];
            const bool ok = (uint32_t)x < (uint32_t)d;
            perms[i] = ok ? x : 0;
            if (!ok) bad_perms[blockIdx.x] = 1u;
        }
        for (int i = at; i < n_tickets; i += step) tickets[i] = 0u;
        for (int w = at; w < W; w += step) {
            n_keys[w] = 0u;
            bands[w] = direct_band_meta(w, lg);
        }
    }
};

// ---- the sort: a workgroup per chunk and band ------------------------------------------------------

// Whose chunk a workgroup takes.  Workgroup ids go round the eight XCDs: of eight bands each has its chunks on one XCD, so
// that a line which chunks of the scatter write 4 bytes at a time is put together in one L2 and leaves it once.  Bands of a last round
// of fewer than eight have theirs on all, as their XCDs alone would be busy.  V = 40000, 8 bands of 12 bits: scatter 11.6 -> 10.1 us.
struct BandChunk {
    int w, c;
    __device__ __forceinline__ BandChunk(int chunks, int W) {
        const int id = (int)blockIdx.x, rounds = W >> 3, slot = id >> 3;
        if (id < 8 * rounds * chunks) { w = slot / chunks; c = slot - w * chunks; w = 8 * w + (id & 7); }
        else { w = id / chunks; c = id - w * chunks; }
    }
};

// counts[w][chunk][digit] (16 bits, digits in pairs); groups[w][chunk][group]: their sums over kScanDigits digits
__global__ void __launch_bounds__(kRadixThreads)
k_radix_count(const int32_t* __restrict__ codes /*[W, V]*/, int64_t V, int W, RadixChunks ch, int shift, int digits,
              uint32_t* __restrict__ counts, uint32_t* __restrict__ groups) {
    extern __shared__ uint32_t hist[];
    const int tid = threadIdx.x, chunks = ch.count();
    const BandChunk bc(chunks, W);
    const int w = bc.w, c = bc.c;
    for (int i = tid; i < digits / 2; i += kRadixThreads) hist[i] = 0u;
    __syncthreads();
    int64_t begin, end;
    ch.range(c, V, &begin, &end);
    const int32_t* src = codes + (size_t)w * V;
#pragma unroll 4
    for (int64_t i = begin + tid; i < end; i += kRadixThreads) {
        const uint32_t dg = ((uint32_t)src[i] >> shift) & (uint32_t)(digits - 1);
        atomicAdd(&hist[dg >> 1], (dg & 1u) ? 65536u : 1u);
    }
    __syncthreads();
    uint32_t* out = counts + ((size_t)w * chunks + c) * (digits / 2);
    for (int i = tid; i < digits / 2; i += kRadixThreads) out[i] = hist[i];
    const int ng = (digits + kScanDigits - 1) / kScanDigits;
    for (int g = wave_id(); g < ng; g += kRadixWaves) {
        uint32_t n = 0;
        for (int i = lane_id(); i < kScanDigits / 2 && g * (kScanDigits / 2) + i < digits / 2; i += kWave) {
            const uint32_t x = hist[g * (kScanDigits / 2) + i];
            n += (x & 0xFFFFu) + (x >> 16);
        }
        n = wave_sum(n);
        if (lane_id() == 0) groups[((size_t)w * chunks + c) * ng + g] = n;
    }
}

// grid (groups of kScanDigits digits, W), a thread per pair of digits: where the words of each digit of each
// chunk go in the band (starts[w][chunk][digit]).  EMIT (the only pass, direct tables): a digit is a code, its slot is
// written here, with the places where the vocabulary slices begin in its span (sums over the chunks in front); slots
// past the codes are empty.
template <bool EMIT>
__global__ void __launch_bounds__(kScanDigits / 2)
k_radix_scan(const uint32_t* __restrict__ counts, const uint32_t* __restrict__ groups, RadixChunks ch, int digits,
             uint32_t* __restrict__ starts, Slot* __restrict__ slots, uint4* __restrict__ cuts, uint32_t* __restrict__ n_keys) {
    constexpr int AHEAD = 24;
    static_assert(kScanDigits / 2 == 2 * kWave && (1 << kRadixBits) / kScanDigits <= 16, "two waves; a lane of 16 per group");
    __shared__ uint32_t wsum[4];
    const int tid = threadIdx.x, w = blockIdx.y, g = blockIdx.x, ng = gridDim.x, chunks = ch.count();
    const int pair = g * (kScanDigits / 2) + tid, pitch = digits / 2;
    const bool in = pair < pitch;
    const uint32_t* mine = counts + (size_t)w * chunks * pitch + min(pair, pitch - 1);
    uint32_t* out = starts + (size_t)w * chunks * digits + 2 * pair;
    // (the counters and the sums are asked for together: one trip to memory for up to AHEAD chunks)
    uint32_t x[AHEAD];
    auto load = [&](int c0) {
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) x[j] = mine[(size_t)min(c0 + j, chunks - 1) * pitch];
    };
    load(0);
    uint32_t before = 0;                                        // words of lower groups: 16 lanes per chunk
    for (int c = tid >> 4; c < chunks; c += kScanDigits / 32)
        if ((tid & 15) < g) before += groups[((size_t)w * chunks + c) * ng + (tid & 15)];
    uint32_t lo = 0, hi = 0, cut_lo[3] = {}, cut_hi[3] = {};
    for (int c0 = 0;;) {
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            if constexpr (EMIT) {
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    if (c0 + j == (q + 1) * ch.per_slice) { cut_lo[q] = lo; cut_hi[q] = hi; }
            }
            const uint32_t n = c0 + j < chunks ? x[j] : 0u;
            lo += n & 0xFFFFu; hi += n >> 16;
        }
        c0 += AHEAD;
        if (c0 >= chunks) break;
        load(c0);
    }
    if (!in) lo = hi = 0;
    // words of lower digits: of the lower groups, and of the lanes and the wave in front
    const uint32_t incl = wave_incl_scan(lo + hi), keys = wave_sum((lo ? 1u : 0u) + (hi ? 1u : 0u));
    before = wave_sum(before);
    if (lane_id() == kWave - 1) { wsum[2 * wave_id()] = incl; wsum[2 * wave_id() + 1] = before; }
    __syncthreads();
    const uint32_t at = wsum[1] + wsum[3] + (tid >= kWave ? wsum[0] : 0u) + incl - (lo + hi);
    if constexpr (EMIT) {
        if (lane_id() == 0) atomicAdd(&n_keys[w], keys);
        if (in) {
            const uint32_t mask = 2u * digits - 1u, offset = direct_offset(w, 32 - __clz(mask));
            const size_t b0 = (size_t)w * 2 * digits, s0 = b0 + ((2 * pair + offset) & mask), e0 = b0 + ((2 * pair + digits + offset) & mask);
            slots[s0] = Slot{lo ? 2 * pair : -1, at, lo, 0u};
            slots[s0 + 1] = Slot{hi ? 2 * pair + 1 : -1, at + lo, hi, 0u};
            slots[e0] = slots[e0 + 1] = Slot{-1, 0u, 0u, 0u};
            cuts[s0] = make_uint4(cut_lo[0], cut_lo[1], cut_lo[2], lo);
            cuts[s0 + 1] = make_uint4(cut_hi[0], cut_hi[1], cut_hi[2], hi);
        }
    }
    if (!in) return;
    uint2 run = make_uint2(at, at + lo);
    for (int c0 = 0; c0 < chunks; c0 += AHEAD) {
        if (chunks > AHEAD) load(c0);                           // (once more, from the caches)
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            if (c0 + j < chunks) *reinterpret_cast<uint2*>(out + (size_t)(c0 + j) * digits) = run;
            run.x += x[j] & 0xFFFFu; run.y += x[j] >> 16;
        }
    }
}

// Stable scatter of one chunk.  A wave owns a contiguous piece of the chunk and has digit counters of
// its own in LDS (16 bits: a chunk has at most 65535 words), so order inside the chunk needs no
// exchange but one prefix over the waves; inside a wave, words of equal digit are ranked by ballots, one
// per digit bit.  (The vector instructions of the ballots bound it -- about 100 per 64 words -- which is why
// a band is cut into chunks.)  ids_in == null: ids are the positions.
__global__ void __launch_bounds__(kRadixThreads)
k_radix_scatter(const int32_t* __restrict__ codes_in, const int32_t* __restrict__ ids_in, int64_t V, int W, RadixChunks ch, int shift,
                int bits, const uint32_t* __restrict__ starts, int32_t* __restrict__ codes_out,
                int32_t* __restrict__ ids_out) {
    extern __shared__ uint32_t rsm[];
    const int digits = 1 << bits;
    uint32_t* base = rsm;                                                   // [digit]
    uint16_t* wpos = reinterpret_cast<uint16_t*>(rsm + digits);             // [wave][digit]
    const int tid = threadIdx.x, ln = lane_id(), wv = wave_id(), chunks = ch.count();
    const BandChunk bc(chunks, W);
    const int w = bc.w, c = bc.c;
    const int32_t* src = codes_in + (size_t)w * V;
    uint32_t* wpos32 = rsm + digits;
    for (int i = tid; i < digits * kRadixWaves / 2; i += kRadixThreads) wpos32[i] = 0u;   // (digits >= 2)
    const uint2* st = reinterpret_cast<const uint2*>(starts) + ((size_t)w * chunks + c) * (digits / 2);
    uint2* base2 = reinterpret_cast<uint2*>(base);
#pragma unroll 4
    for (int i = tid; i < digits / 2; i += kRadixThreads) base2[i] = st[i];
    __syncthreads();
    int64_t begin, end;
    ch.range(c, V, &begin, &end);
    const int piece = (((int)(end - begin) + kRadixWaves - 1) / kRadixWaves + kWave - 1) / kWave * kWave;
    const int64_t p0 = begin + (int64_t)wv * piece, p1 = min(p0 + piece, end);
    const uint32_t mask = (uint32_t)digits - 1u;
    constexpr int AHEAD = 8;                                // words per lane asked for at a time
    for (int64_t i0 = p0; i0 < p1; i0 += AHEAD * kWave) {
        uint32_t code[AHEAD];
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) code[j] = (uint32_t)src[min(i0 + j * kWave + ln, p1 - 1)];
#pragma unroll
        for (int j = 0; j < AHEAD; ++j)
            if (i0 + j * kWave + ln < p1) {
                const uint32_t dg = (code[j] >> shift) & mask;
                atomicAdd(&wpos32[((uint32_t)wv * digits + dg) >> 1], (dg & 1u) ? 65536u : 1u);
            }
    }
    __syncthreads();
    for (int i = tid; i < digits / 2; i += kRadixThreads) {  // exclusive prefix over the waves, two digits at a time
        uint32_t n[kRadixWaves], run = 0;                    // (no carry from the low half: a chunk fits 16 bits)
#pragma unroll
        for (int v = 0; v < kRadixWaves; ++v) n[v] = wpos32[v * (digits / 2) + i];
#pragma unroll
        for (int v = 0; v < kRadixWaves; ++v) {
            wpos32[v * (digits / 2) + i] = run;
            run += n[v];
        }
    }
    __syncthreads();
    uint16_t* pos = wpos + wv * digits;
    for (int64_t i0 = p0; i0 < p1; i0 += AHEAD * kWave) {   // (uniform in the wave)
        uint32_t code[AHEAD];
        int32_t id[AHEAD];
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            const int64_t i = min(i0 + j * kWave + ln, p1 - 1);
            code[j] = (uint32_t)src[i];
            id[j] = ids_in ? ids_in[(size_t)w * V + i] : (int32_t)i;
        }
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            const uint32_t dg = (code[j] >> shift) & mask;
            const bool in = i0 + j * kWave + ln < p1;
            uint64_t same = __ballot(in);
            for (int b = 0; b < bits; ++b) {
                const uint64_t set = __ballot((dg >> b) & 1u);
                same &= ((dg >> b) & 1u) ? set : ~set;
            }
            const uint32_t rank = lanes_below(same), n = (uint32_t)__popcll(same);
            if (in) {
                const uint32_t before = pos[dg];
                const size_t at = (size_t)w * V + base[dg] + before + rank;
                if (codes_out) codes_out[at] = (int32_t)code[j];
                ids_out[at] = id[j];
                if (rank == n - 1u) pos[dg] = (uint16_t)(before + n);   // (after every lane's read: one wave, LDS in order)
            }
        }
    }
}

// ---- keys of a band, from its sorted codes: grid (chunks, W) ---------------------------------------------

__device__ __forceinline__ bool starts_span(const int32_t* __restrict__ codes, int64_t i) {
    return i == 0 || codes[i] != codes[i - 1];
}
// spans[w][chunk]: span starts in the chunk
__global__ void __launch_bounds__(kRadixThreads)
k_key_count(const int32_t* __restrict__ codes /*[W, V] sorted*/, int64_t V, RadixChunks ch, uint32_t* __restrict__ spans) {
    __shared__ uint32_t wsum[kRadixWaves + 1];
    const int32_t* src = codes + (size_t)blockIdx.y * V;
    int64_t begin, end;
    ch.range(blockIdx.x, V, &begin, &end);
    uint32_t n = 0, all;
    for (int64_t i = begin + threadIdx.x; i < end; i += kRadixThreads) n += starts_span(src, i) ? 1u : 0u;
    block_incl_scan(n, wsum, &all);
    if (threadIdx.x == 0) spans[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = all;
}
__global__ void __launch_bounds__(kRadixThreads)
k_key_emit(const int32_t* __restrict__ codes, int64_t V, RadixChunks ch, const uint32_t* __restrict__ spans,
           int32_t* __restrict__ key_code, uint32_t* __restrict__ key_start, uint32_t key_pitch, uint32_t* __restrict__ n_keys) {
    __shared__ uint32_t wsum[kRadixWaves + 1];
    const int tid = threadIdx.x, ln = lane_id(), wv = wave_id(), w = blockIdx.y, c = blockIdx.x;
    const int32_t* src = codes + (size_t)w * V;
    uint32_t n = 0, before, mine = 0, all;
    for (int i = tid; i < c; i += kRadixThreads) n += spans[(size_t)w * gridDim.x + i];
    block_incl_scan(n, wsum, &before);                       // keys of the chunks in front
    int64_t begin, end;
    ch.range(c, V, &begin, &end);
    const int piece = (((int)(end - begin) + kRadixWaves - 1) / kRadixWaves + kWave - 1) / kWave * kWave;
    const int64_t p0 = begin + (int64_t)wv * piece, p1 = min(p0 + piece, end);
    for (int64_t i = p0 + ln; i < p1; i += kWave) mine += starts_span(src, i) ? 1u : 0u;
    // (lane totals scanned over the workgroup: the waves in front, then the wave's own from its ballots)
    const uint32_t incl = block_incl_scan(mine, wsum, &all);
    uint32_t k = before + wave_read_lane(incl - mine, 0);
    for (int64_t i0 = p0; i0 < p1; i0 += kWave) {
        const int64_t i = i0 + ln;
        const bool head = i < p1 && starts_span(src, i);
        const uint64_t heads = __ballot(head);
        if (head) {
            const size_t at = (size_t)w * key_pitch + k + lanes_below(heads);
            key_code[at] = src[i];
            key_start[at] = (uint32_t)i;
        }
        k += (uint32_t)__popcll(heads);
    }
    if (c == (int)gridDim.x - 1 && tid == 0) n_keys[w] = before + all;
}

// ---- cuckoo tables -------------------------------------------------------------------------------

// grid (key_pitch / 256, W), one thread per key.  Item = code << 32 | key index.  `failed[w]` is set when
// a chain in band w exceeds max_chain (the item in hand is dropped: the band is redone).
__global__ void __launch_bounds__(256)
k_cuckoo_insert(uint64_t* __restrict__ table, const BandMeta* __restrict__ bands, const int32_t* __restrict__ key_code,
                uint32_t key_pitch, const uint32_t* __restrict__ n_keys, int max_chain,
                const uint32_t* __restrict__ redo, uint32_t* __restrict__ failed) {
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    const int w = blockIdx.y;
    if (k >= n_keys[w] || (redo && !redo[w])) return;
    const BandMeta m = bands[w];
    const uint32_t my_code = (uint32_t)key_code[(size_t)w * key_pitch + k];
    uint64_t item = ((uint64_t)my_code << 32) | (uint64_t)k;
    uint32_t pos = cuckoo_hash(m.a0, m.b0, my_code, m.shift);
    for (int step = 0; step < max_chain; ++step) {
        const uint64_t old = atomicExch((unsigned long long*)&table[m.slot_off + pos], (unsigned long long)item);
        if (old == kCuckooEmpty) return;
        item = old;  // carry the evicted item to its other slot
        const uint32_t code = (uint32_t)(old >> 32);
        const uint32_t h0 = cuckoo_hash(m.a0, m.b0, code, m.shift);
        const uint32_t h1 = cuckoo_hash(m.a1, m.b1, code, m.shift);
        pos = (pos == h0) ? h1 : h0;
    }
    failed[w] = 1u;
}

// grid (cap / 256, W).  8-byte table words -> the 16-byte slots of the probe, and beside every used slot
// where the vocabulary slices 1, 2, 3 of the hit-count kernel begin inside its span (ids are ascending
// there): lower bounds of slice * slice_ids, relative to the span's start.  (Cuts of empty slots are never used.)
__global__ void __launch_bounds__(256)
k_cuckoo_finalize(const uint64_t* __restrict__ table, uint32_t cap, const uint32_t* __restrict__ key_start,
                  uint32_t key_pitch, const uint32_t* __restrict__ n_keys, const int32_t* __restrict__ words, uint32_t V,
                  int slice_ids, Slot* __restrict__ slots, uint4* __restrict__ cuts) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const int w = blockIdx.y;
    if (i >= cap) return;
    const size_t at = (size_t)w * cap + i;
    const uint64_t e = table[at];
    Slot s{-1, 0u, 0u, 0u};
    if (e != kCuckooEmpty) {
        const uint32_t k = (uint32_t)e;
        const uint32_t* starts = key_start + (size_t)w * key_pitch;
        s.key = (int32_t)(uint32_t)(e >> 32);
        s.start = starts[k];
        s.len = (k + 1 < n_keys[w] ? starts[k + 1] : V) - s.start;
        const int32_t* span = words + (size_t)w * V + s.start;
        // first position whose id is >= the bound: the three searches side by side, since each step waits
        // for its load
        uint32_t lo[3] = {0u, 0u, 0u};
        for (uint32_t n = s.len; n; n >>= 1) {   // (answers lie in [lo, lo + n])
            int32_t id[3];
            const uint32_t half = n >> 1;
#pragma unroll
            for (int q = 0; q < 3; ++q) id[q] = span[min(lo[q] + half, s.len - 1u)];
#pragma unroll
            for (int q = 0; q < 3; ++q)
                if (lo[q] + half < s.len && id[q] < (q + 1) * slice_ids) lo[q] += half + 1u;
        }
        cuts[at] = make_uint4(lo[0], lo[1], lo[2], s.len);
    }
    slots[at] = s;
}

}  // namespace lshbeam
