// C ABI of the lshbeam library (see include/lshbeam.h): table build, decode step, beam
// bookkeeping, inspection.  gfx950 only.  Host side: argument validation, the choice of the
// launch plan, kernel launches, the hash parameters of the cuckoo tables (and a host fallback of
// the table build).  Every per-step computation runs in the HIP kernels of candidates.h /
// fused.h / logits.h / select.h / beam.h, the table build in those of build_tables.h.
#include "../../include/lshbeam.h"

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <cctype>
#include <new>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

#include "beam.h"
#include "build_tables.h"
#include "candidates.h"
#include "fused.h"
#include "logits.h"
#include "report.h"
#include "select.h"
#include "workspace.h"

using namespace lshbeam;

// Working memory of lsh_decode_step_static, the variant of the decode step for callers that
// cannot allocate: one array per GPU, part of the loaded code object, held until the process
// ends.  In host code `scratch` only names the symbol; the memory of the current device's copy is
// found once per device by scratch_of_device() and kernels are handed that address.
constexpr size_t kScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_addr[kMaxDevices];   // device address of `scratch` on each GPU, or null

// Address of the current device's copy of `scratch` (the device must be current: each GPU holds
// its own copy at its own address).
hipError_t scratch_of_device(int dev, void** out) {
    *out = nullptr;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void* p = g_scratch_addr[dev].load(std::memory_order_acquire);
    if (!p) {
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_addr[dev].store(p, std::memory_order_release);
    }
    *out = p;
    return hipSuccess;
}

constexpr int kMaxV = 1 << 24;
constexpr int kMaxB = 256;
constexpr int kTicketSlots = 256;   // workspaces per handle that can take the one-launch plan
constexpr int kTicketBlock = 64;    // counters per workspace = sentences of a fused step at most


struct Band {
    int n_keys = 0;      // distinct codes (-1: in n_keys_dev)
    int capacity = 0;    // slots of its cuckoo table
    BandMeta meta{};
};
struct HostBand : Band {           // a band being built on the host
    std::vector<int32_t> keys;     // distinct band codes, ascending
    std::vector<int32_t> offsets;  // keys.size() + 1 span boundaries into the band's word array
};

struct KeptBlock { void* p = nullptr; size_t bytes = 0; };   // device memory that may be kept for the next build

// Launch-plan options of a handle (lsh_set_option); kAuto = the library's own rule.
enum Opt {
    kOptFused, kOptFusedGrid, kOptLogitsGrid, kOptLogitsWaves, kOptLogitsHlds, kOptLogitsEstage,
    kOptHldsRem, kOptLogitsPlanes, kOptHldsRows, kOptPartRows, kOptStageRows, kOptOneLaunch, kOptFusedTile,
    kOptEstageUnion, kOptFirstTiles, kNumOpts
};
constexpr int kAuto = -1;
const char* const kOptNames[kNumOpts] = {
    "fused", "fused_grid", "logits_grid", "logits_waves", "logits_hlds", "logits_estage",
    "hlds_rem", "logits_planes", "hlds_rows", "part_rows", "stage_rows", "one_launch", "fused_tile",
    "estage_union", "first_tiles"};

}  // namespace

// Device start/stop events of the kernels of the steps it is handed to (lsh_decode_step_timed).
struct lsh_profiler {
    int max_launches = 0;
    std::vector<hipEvent_t> ev[LSH_NUM_KERNELS];  // start/stop pairs
    int used[LSH_NUM_KERNELS] = {0, 0, 0, 0, 0};
};

struct lsh_tables {
    int device = 0;
    const void* E = nullptr;
    int V = 0, d = 0, dtype = 0, K = 0, P = 0, W = 0, u = 0, bits = 0;
    int64_t ld = 0;
    KeptBlock arena;                 // device memory of everything below
    KeptBlock slot_block;            // ... but the slots and cuts, where their number was not known before the rest
    int32_t* perms_dev = nullptr;    // [P, K]
    int32_t* codes_dev = nullptr;    // [W, V] band codes of the embedding rows
    int32_t* words_dev = nullptr;    // [W, V] word ids grouped by band code
    Slot* slots_dev = nullptr;       // all bands' cuckoo slots, concatenated
    uint4* cuts_dev = nullptr;       // per slot: where vocabulary slices 1..3 begin in its span
    BandMeta* bands_dev = nullptr;   // [W]
    uint32_t* n_keys_dev = nullptr;  // [W] distinct codes of each band, where `bands` does not know them
    std::vector<Band> bands;         // what the inspection calls know about each band
    int wg_candidates_lds = 0;
    int wg_fused_lds = 0;
    int wg_hit_rows_lds = 0;   // 0: the hit-count kernel cannot run on these tables (t > 1 unsupported)
    int hit_list_cap = 0;
    int wg_union_logits_lds = 0;
    int built_on_device = 0, build_attempts = 0;  // how the tables came about (inspection)
    void* scratch_dev = nullptr;                  // this device's copy of the static scratch array
    // Ticket counters of the one-launch plan: kTicketSlots blocks of kTicketBlock counters in
    // device memory, all zero between steps (the kernel that uses a block leaves it zero).  A
    // block belongs to one workspace address for the life of the handle, so steps that run at the
    // same time -- which must use different workspaces -- never share counters.  The table is a
    // cache behind the const handle: guarded by its own mutex, it changes no result.
    unsigned int* tickets_dev = nullptr;
    mutable std::mutex ticket_mu;
    mutable const void* ticket_owner[kTicketSlots] = {};
    mutable int ticket_used = 0;
    // The counters for the step that works in `workspace`, or null when all blocks are taken (the
    // step then ends with a selection kernel of its own).
    unsigned int* tickets_for(const void* workspace) const {
        std::lock_guard<std::mutex> lock(ticket_mu);
        for (int i = 0; i < ticket_used; ++i)
            if (ticket_owner[i] == workspace) return tickets_dev + (size_t)i * kTicketBlock;
        if (!tickets_dev || ticket_used == kTicketSlots) return nullptr;
        ticket_owner[ticket_used] = workspace;
        return tickets_dev + (size_t)(ticket_used++) * kTicketBlock;
    }
    int opt[kNumOpts];                            // launch-plan options, kAuto unless set
    int option(int which, int dflt) const { return opt[which] == kAuto ? dflt : opt[which]; }
};

namespace {

struct SplitMix64 {
    uint64_t s;
    uint64_t next() {
        uint64_t z = (s += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    }
};

inline int code_bits(int K) {
    int b = 0;
    while ((1 << b) < K) ++b;
    return b;
}

// Two-choice cuckoo insertion (Pagh & Rodler) of the band's keys into `cap` slots.  Returns false
// if some insertion exceeds the eviction limit with these hash parameters.
bool cuckoo_try(const HostBand& hb, const BandMeta& m, int cap, Slot* slots) {
    for (int i = 0; i < cap; ++i) slots[i] = Slot{-1, 0u, 0u, 0u};
    int lg = 0;
    while ((1 << lg) < cap) ++lg;
    const int max_kicks = 16 * (lg + 1);
    for (size_t q = 0; q < hb.keys.size(); ++q) {
        Slot cur{hb.keys[q], (uint32_t)hb.offsets[q], (uint32_t)(hb.offsets[q + 1] - hb.offsets[q]), 0u};
        const uint32_t h0 = cuckoo_hash(m.a0, m.b0, (uint32_t)cur.key, m.shift);
        const uint32_t h1 = cuckoo_hash(m.a1, m.b1, (uint32_t)cur.key, m.shift);
        bool placed = false;
        if (slots[h0].key < 0) { slots[h0] = cur; placed = true; }
        else if (slots[h1].key < 0) { slots[h1] = cur; placed = true; }
        uint32_t pos = h0;
        for (int kick = 0; !placed && kick < max_kicks; ++kick) {
            // take slot `pos`; its occupant moves to its own other slot, evicting in turn
            std::swap(cur, slots[pos]);
            const uint32_t e0 = cuckoo_hash(m.a0, m.b0, (uint32_t)cur.key, m.shift);
            const uint32_t e1 = cuckoo_hash(m.a1, m.b1, (uint32_t)cur.key, m.shift);
            pos = (pos == e0) ? e1 : e0;
            if (slots[pos].key < 0) { slots[pos] = cur; placed = true; }
        }
        if (!placed) return false;
    }
    return true;
}

lsh_status build_cuckoo(HostBand& hb, SplitMix64& rng, std::vector<Slot>& out, uint32_t slot_off) {
    int cap = 2;
    while ((size_t)cap < 2 * hb.keys.size()) cap <<= 1;
    std::vector<Slot> slots;
    for (int grow = 0; grow < 4; ++grow, cap <<= 1) {
        slots.resize(cap);
        int lg = 0;
        while ((1 << lg) < cap) ++lg;
        for (int attempt = 0; attempt < 16; ++attempt) {
            BandMeta m{};
            m.slot_off = slot_off;
            m.shift = 32u - (uint32_t)lg;
            m.a0 = (uint32_t)rng.next() | 1u;
            m.b0 = (uint32_t)rng.next();
            m.a1 = (uint32_t)rng.next() | 1u;
            m.b1 = (uint32_t)rng.next();
            if (cuckoo_try(hb, m, cap, slots.data())) {
                hb.capacity = cap;
                hb.meta = m;
                out.insert(out.end(), slots.begin(), slots.end());
                return LSH_OK;
            }
        }
    }
    return LSH_ERR_BUILD_FAILED;
}

// What a step's launches share: the (read-only) tables, the stream, and the caller's profiler.
struct StepCtx {
    const lsh_tables* t;
    hipStream_t st;
    lsh_profiler* prof;
};

template <typename... KArgs, typename... Args>
void launch(const StepCtx& cx, int which, void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t shmem,
            Args... args) {
    lsh_profiler* pf = cx.prof;
    hipStream_t stream = cx.st;
    if (pf && which >= 0 && pf->used[which] < pf->max_launches) {
        const int i = pf->used[which]++;
        hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)shmem, stream, pf->ev[which][2 * i],
                              pf->ev[which][2 * i + 1], 0, args...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, (uint32_t)shmem, stream, args...);
    }
}

Workspace carve(const lsh_tables* t, const lsh_step_params* sp, void* base) {
    return carve_workspace(sp->S, sp->B, t->V, sp->full_vocab != 0, base);
}

bool step_params_ok(const lsh_tables* t, const lsh_step_params* sp) {
    return t && sp && sp->S >= 1 && sp->B >= 1 && sp->B <= kMaxB && sp->T >= 0 &&
           sp->S <= kMaxSentencesLogits && (int64_t)sp->S * sp->B <= (int64_t)INT32_MAX / 2;
}

int env_int(const char* name, int dflt) {
    const char* v = std::getenv(name);
    return (v && *v) ? std::atoi(v) : dflt;
}

// Raises a kernel's dynamic-LDS limit to (nearly) a CU's whole LDS, once per kernel and device.
// The limit belongs to the kernel, not to a table: it is never set to what one table needs, and
// the decode step makes no driver call besides its launches once a kernel has been through here.
template <auto KFN>
hipError_t allow_whole_lds() {
    static std::atomic<uint64_t> done{0};  // one bit per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = (dev >= 0 && dev < 64) ? (1ull << dev) : 0ull;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    e = hipFuncSetAttribute((const void*)KFN, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxDynLds);
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}

// How many candidates a sentence's list will hold at least: its top-frequent words and what its hidden rows
// hit by chance (bands independent, codes evenly spread; rows near clustered words hit more).
inline double expected_candidates(const lsh_tables* t, const lsh_step_params* sp) {
    const double m = t->W * std::pow((double)t->K, -(double)t->u);   // expected bands in which a row and a word collide
    double below = 0.0, p = std::exp(-m);
    for (int i = 0; i < std::min<int>(sp->threshold, 64); ++i) { below += p; p *= m / (i + 1); }
    const double missed = (1.0 - std::min(1.0, (double)sp->T / t->V)) * std::pow(std::min(1.0, below), sp->B);
    return t->V * (1.0 - missed);
}

// Little work per step (few sentences x 16-row groups): every workgroup of the logits grid
// regenerates the candidates itself (k_cand_logits); otherwise one candidates workgroup per
// sentence, then the logits grid.  LSHBEAM_FUSED=0/1 overrides the size rule (for tests and
// measurements), never the hard limits.
bool step_is_fused(const lsh_tables* t, const lsh_step_params* sp) {
    const int MT = (sp->B + kTileM - 1) / kTileM;
    const bool possible = !sp->full_vocab && (size_t)t->wg_fused_lds <= kMaxDynLds && sp->S <= 64;
    // (with three or more groups of 16 beams the separate split-k kernel, one (tile, group) per
    // workgroup at a time, is faster than the fused kernel's all-groups-per-tile loop)
    if (t->opt[kOptFused] != kAuto) return possible && t->opt[kOptFused] != 0;
    // What the workgroups do one after the other, in tiles for each of the 256, outweighs the kernel saved beyond
    // (measured over S = 1 .. 16 and B = 4 .. 32 on six shapes, us a step fused / in three kernels):
    //   one row group, 2.4 with long fp32 rows (d = 1000: 4 x 12 beams, 1.9 tiles, 23.2 / 27.4; 6 x 8, 2.4, 26.1 / 26.7;
    //   8 x 4, 2.6, 27.3 / 24.7), 1.9 with shorter ones (d = 512: 8 x 12, 1.9, 20.7 / 22.9; 12 x 8, 2.4, 22.2 / 21.7), 1.8 with bf16
    //   (d = 1024: 3 x 16, 1.6, 22.0 / 25.0; 4 x 12, 1.9, 24.7 / 23.9; V = 100000: 2 x 12, 2.05, 26.8 / 26.1);
    //   two, 1.5 (d = 1000, V = 40000: 1 x 26, 0.7, 25.6 / 30.1; 1 x 32, 0.8, 36.0 / 33.4; 2 x 24, 1.4, 31.3 / 33.0; d = 1536, 1 x 17,
    //   24.1 / 29.5; d = 512 bf16, 2 x 24, 25.8 / 28.4.  The fused kernel's sums, of 16 waves' instead of 4, are also nearer: 1.0e-8 of
    //   the products' sizes against 1.7e-8.)  With a hit threshold, clustered words make the lists longer than expected, which does not
    //   decide it: 118 bands, t = 3, d = 216, 4 x 9 beams, 40.9 / 36.6; 173 bands, t = 4, d = 88, 4 x 1, 22.2 / 24.2.
    const double tiles = sp->S * expected_candidates(t, sp) / (256 * kTileN);
    if (!possible || sp->S * MT > 8 || MT > 2) return false;
    return tiles <= (MT == 2 ? 1.5 : t->dtype != LSH_F32 ? 1.8 : t->d > 512 ? 2.4 : 1.9);
}

// LDS words for the staged hidden rows of a step: room for all B rows of a sentence (up to
// kCandStageRows; LSHBEAM_STAGE_ROWS overrides, 0 = never more than the minimum) where LDS has
// it beside everything else the kernel keeps there, else the minimum stage.
int stage_words_for(const lsh_tables* t, int B, bool fused_kernel) {
    const int mn = candidates_min_stage(t->d);
    const int rows = std::min(B, std::max(0, t->option(kOptStageRows, kCandStageRows)));
    const int64_t want = ((int64_t)rows * t->d + 3) & ~(int64_t)3;
    const size_t other = fused_kernel ? fused_lds_words(t->V, t->P, t->K, 0)
                                      : candidates_lds_words(t->V, t->P, t->K, 0);
    const size_t room = kMaxDynLds / sizeof(uint32_t);
    const int64_t cap = room > other ? (int64_t)((room - other) & ~(size_t)3) : 0;
    return (int)std::max<int64_t>(mn, std::min(want, cap));
}

// Rows of a sentence hashed per workgroup when the sentence is cut into parts (t = 1, more beams
// than one chunk of hashing holds even with the step's stage); 0 = the sentence is hashed by one
// workgroup.  Parts take the minimum stage.  LSHBEAM_PART_ROWS forces a part size (for tests and
// measurements).
int part_rows_of(const lsh_tables* t, const lsh_step_params* sp, int stage_words) {
    if (sp->full_vocab || sp->threshold != 1) return 0;
    const int rpc = candidates_rows_per_chunk(sp->B, t->d, t->W, candidates_min_stage(t->d));
    const int forced = t->option(kOptPartRows, 0);
    if (forced > 0) return std::min(forced, rpc);
    return sp->B > candidates_rows_per_chunk(sp->B, t->d, t->W, stage_words) ? rpc : 0;
}

// Whether a row of E holds a 16-byte chunk: what every contraction but the elementwise forms needs.
inline bool has_chunks(const lsh_tables* t) { return t->d >= (t->dtype == LSH_F32 ? 4 : 8); }

// The first tiles made beside the hashing (first_tiles_count).
FirstTiles first_tiles_plan(const lsh_tables* t, const lsh_step_params* sp, const float* H, const int32_t* topfreq, const Workspace& w, int blocks) {
    FirstTiles f{t->E, t->ld, H, t->d, sp->S, sp->B, 0, blocks, topfreq, w.logits, w.cpitch, w.records()};
    if (!has_chunks(t) || t->option(kOptFusedTile, 0) > 0 || t->opt[kOptFusedGrid] != kAuto) return f;
    f.tiles = first_tiles_count(sp->S, sp->B, sp->T, t->V, blocks, expected_candidates(t, sp), t->opt[kOptFirstTiles]);
    return f;
}
inline int first_tiles_blocks(const FirstTiles& f) { return std::min(f.tiles * f.S, std::max(0, 256 - f.first)); }

template <typename ET, int WAVES>
void launch_logits_w(const StepCtx& cx, int grid, bool chunks, const float* H,
                     const lsh_step_params* sp, const int32_t* cand, const int32_t* count,
                     const Workspace& w) {
    const lsh_tables* t = cx.t;
    constexpr int UNROLL = (WAVES >= 16) ? 4 : 8;
    const ET* E = (const ET*)t->E;
    if (chunks)
        launch(cx, 1, k_logits<ET, WAVES, UNROLL, true>, dim3(grid), dim3(WAVES * kWave), 0, E,
               t->ld, t->d, H, sp->S, sp->B, cand, count, t->V, w.logits, w.cpitch, w.records());
    else
        launch(cx, 1, k_logits<ET, WAVES, UNROLL, false>, dim3(grid), dim3(WAVES * kWave), 0, E,
               t->ld, t->d, H, sp->S, sp->B, cand, count, t->V, w.logits, w.cpitch, w.records());
}

template <typename ET, int MT>
void launch_logits_wave(const StepCtx& cx, int grid, bool chunks, const float* H,
                        const lsh_step_params* sp, const int32_t* cand, const int32_t* count,
                        const Workspace& w) {
    const lsh_tables* t = cx.t;
    // loads in flight per lane: 32 (fp32) / 64 (bf16) bytes of E per step, plus MT times that of H
    constexpr int UNROLL = ((MT == 1) ? 8 : 4) / (ElemTraits<ET>::VEC / 4);
    const ET* E = (const ET*)t->E;
    if (chunks)
        launch(cx, 1, k_logits_wave<ET, MT, UNROLL, true>, dim3(grid), dim3(256), 0, E, t->ld, t->d,
               H, sp->S, sp->B, cand, count, t->V, w.logits, w.cpitch, w.records());
    else
        launch(cx, 1, k_logits_wave<ET, MT, UNROLL, false>, dim3(grid), dim3(256), 0, E, t->ld, t->d,
               H, sp->S, sp->B, cand, count, t->V, w.logits, w.cpitch, w.records());
}

// k_logits_hlds over the sentence's rows in groups: a group's rows must fit in LDS.  Up to 78 KB
// two 8-wave workgroups share a CU, beyond that one 16-wave workgroup has it alone.  Returns 0
// if even one 16-row group does not fit (very large d): the caller then keeps the hidden rows
// in global memory.
constexpr size_t kHldsHalf = 78 * 1024;
inline int hlds_group_rows(const lsh_tables* t, int S, int B, int d) {
    const int forced = t->option(kOptHldsRows, 0);  // 16 or 32 (measurements)
    if (forced == 16 || forced == 32)
        return hlds_lds_bytes(S, std::min(forced, B), d, 16) <= kMaxDynLds ? std::min(forced, B) : 0;
    // up to 32 beams: one group; more: groups of 16, a workgroup each (measured at S = 4: B = 50,
    // V = 100k: 51 us with groups of 16, 46 with 32, 55 with the rows in global memory; B = 48,
    // V = 40k: 48 / 54 / 51)
    if (B > 32) return hlds_lds_bytes(S, 16, d, 16) <= kMaxDynLds ? 16 : 0;
    for (int rows : {32, 16})
        if (hlds_lds_bytes(S, std::min(rows, B), d, 16) <= kMaxDynLds) return std::min(rows, B);
    return 0;
}

template <typename ET>
void launch_logits_hlds(const StepCtx& cx, int64_t tiles_n, const float* H,
                        const lsh_step_params* sp, const int32_t* cand, const int32_t* count,
                        const Workspace& w, int group_rows) {
    const lsh_tables* t = cx.t;
    constexpr int U1 = 8 / (ElemTraits<ET>::VEC / 4), U2 = 4 / (ElemTraits<ET>::VEC / 4);
    // (1024-thread workgroups have 128 registers per lane: one load less in flight)
    constexpr int U2W = (U2 > 2) ? U2 - 1 : U2;
    const ET* E = (const ET*)t->E;
    // one launch: a workgroup serves one group of `rows` hidden rows (the last group may be smaller)
    const int rows = std::min(group_rows, sp->B);
    const int ngroups = (sp->B + rows - 1) / rows;
    // tiles that surely lie among the top-frequent words (T distinct ones, where they are the lowest ids); a
    // few such tiles are not worth the uneven shares of the XCDs
    const int shared = cand && sp->T >= 32 * kTileN ? sp->T / kTileN : 0;
#define LSH_HLDS(MTV, WV, UV, PL)                                                                    \
    do {                                                                                             \
        auto kfn = k_logits_hlds<ET, MTV, WV, UV, PL>;                                               \
        const size_t lds = hlds_lds_bytes(sp->S, rows, t->d, WV, PL);                                \
        const int gx = (int)(std::min<int64_t>(                                                      \
            tiles_n, std::max(1, t->option(kOptLogitsGrid, 4096 / WV) / ngroups)) + 7) / 8 * 8;      \
        launch(cx, 1, kfn, dim3(gx * ngroups), dim3(WV * kWave), lds, E, t->ld, t->d, H, sp->S, sp->B,   \
               rows, gx, ngroups, t->option(kOptHldsRem, 4), shared, cand, count, t->V, w.logits,      \
               w.cpitch, w.records());                                                      \
    } while (0)
    // bf16 rows, up to 16 hidden rows per group, two workgroups per CU: the hidden rows go to LDS
    // as three bf16 planes and the contraction runs on bf16 matrix instructions
    // (LSHBEAM_LOGITS_PLANES=0: widened to fp32 as for every other shape)
    if constexpr (std::is_same<ET, uint16_t>::value) {
        if (rows <= kTileM && hlds_lds_bytes(sp->S, rows, t->d, 8, true) <= kHldsHalf &&
            t->option(kOptLogitsPlanes, 1)) {
            LSH_HLDS(1, 8, U1, true);
            return;
        }
    }
    const bool two = rows > kTileM;
    const bool small = hlds_lds_bytes(sp->S, rows, t->d, 8) <= kHldsHalf;
    if (small) { if (two) LSH_HLDS(2, 8, U2, false); else LSH_HLDS(1, 8, U1, false); }
    else { if (two) LSH_HLDS(2, 16, U2W, false); else LSH_HLDS(1, 16, U1, false); }
#undef LSH_HLDS
}

// Whether an option names k_logits_hlds (or its absence): it wins over k_logits_stream.
inline bool names_hlds(const lsh_tables* t) {
    return t->opt[kOptLogitsHlds] != kAuto || t->opt[kOptHldsRows] != kAuto || t->opt[kOptHldsRem] != kAuto ||
           t->opt[kOptLogitsPlanes] != kAuto;
}
// k_logits_stream: steps of 64 bytes per unit and parts of a wave's quarter of the row; whether the last has fewer steps.
struct StreamPlan { int ksn, parts; bool short_last; };
template <typename ET> StreamPlan stream_plan(int d) {
    constexpr int kstep = 4 * ElemTraits<ET>::VEC;
    const int nst = ((d + kstep - 1) / kstep + 3) / 4;
    return nst <= 1 ? StreamPlan{1, 1, false} : nst <= 4 ? StreamPlan{2, (nst + 1) / 2, nst % 2 != 0} : StreamPlan{4, (nst + 3) / 4, nst % 4 != 0};
}
// Hidden rows per workgroup (0: the kernel does not take the step): more than 16 beams in even groups of at most 16, every
// group with its own pass over the candidate rows (from the XCD's L2), or of at most 32 where the rows are so short that
// this pass is what counts.  fp32, d = 1000, V = 40000: 1 x 32 beams 40 us with 32 rows per workgroup, 33 with 16; 9 x 17: 50, 48;
// d = 256, V = 10000: 9 x 32 29, 28; 64 x 20 43, 48.  Rows of two parts: groups of 32 where these hold no more empty rows than groups
// of 16 would, up to six steps always, with seven from four expected tiles for each of the 256 CUs on, with eight from nine (us with
// 16 and 32 rows; d = 264: 20 x 20, V = 40000, 52.0, 45.8, 16 x 28, V = 10000, 38.6, 36.6, full vocabulary of 2000, 128 rows, 14.7, 14.0; d = 440:
// 54.1, 47.8, 39.9, 38.2, 15.9, 16.1; d = 448, 10 x 18, V = 14000, 2.8 tiles, 30.5, 31.7; d = 512: 32 x 31, V = 40000, 86, 80, 20 x 20 53.9, 52.2, 10 x 90,
// V = 20000, 113, 105, 8 x 32, V = 40000, 44.5, 47); three groups of 16 stay (24 x 40, V = 60000, 189, 200).  (The longest bf16
// rows, four parts, need 16 registers more than there are; the spills cost less than the other kernel does: 32 sentences x 10
// beams, V = 40000, 34 us against 67 of k_logits_hlds for d = 1664, 35 against 76 for 2048.)
template <typename ET> int stream_rows(const lsh_tables* t, const lsh_step_params* sp) {
    if (!has_chunks(t) || t->ld * (int64_t)sizeof(ET) >= (int64_t)1 << 31) return 0;
    const StreamPlan p = stream_plan<ET>(t->d);
    if (p.parts > (sizeof(ET) == 2 ? 4 : 8)) return 0;
    const bool whole = (sp->B + kTileM - 1) / kTileM % 2 == 0;   // groups of 32 have no more padding than groups of 16
    const bool two = sp->B > kTileM && (p.ksn < 4 || (sizeof(ET) == 4 && p.parts == 2 && whole &&
                                                      (t->d <= 384 || sp->S * expected_candidates(t, sp) >= (t->d <= 448 ? 1024 : 2304) * kTileN)));
    const int most = two ? 2 * kTileM : kTileM, groups = (sp->B + most - 1) / most;
    return (sp->B + groups - 1) / groups;
}
template <typename ET>
void launch_logits_stream(const StepCtx& cx, int64_t tiles_n, const float* H, const lsh_step_params* sp,
                          const int32_t* cand, const int32_t* count, const Workspace& w, int rows) {
    const lsh_tables* t = cx.t;
    const StreamPlan p = stream_plan<ET>(t->d);
    const int ngroups = (sp->B + rows - 1) / rows;
    // tiles that surely lie among the top-frequent words (T distinct ones, where they are the lowest ids); a
    // few such tiles are not worth the uneven shares of the XCDs
    const int shared = cand && sp->T >= 32 * kTileN ? sp->T / kTileN : 0;
    int wgs = (int)std::min<int64_t>((tiles_n + 7) / 8, std::max(1, t->option(kOptLogitsGrid, 256 * stream_wgs(sizeof(ET) == 2, rows > kTileM ? 2 : 1, p.ksn, p.parts)) / 8 / ngroups));
    int per = wgs / sp->S;
    // A workgroup stays with one sentence: where the same number for every sentence leaves at most an eighth of them without
    // work; or dealt to them, unless some sentence would get less than nine tenths of its share and that costs its workgroups more
    // tiles than an even cut costs (two, six with bf16 words), or less than two workgroups, so that shares could not follow the lists'
    // lengths.  us a step dealt, cut evenly: V = 20000, d = 1000 fp32, 300 x 2 beams 110, 75; 90 x 20 166, 122; V = 10000, d = 700, 200 x 3,
    // lists of 1140, 100, 85, of 450 54, 49 (bf16 54, 50 and 35, 36.5); V = 42000, d = 288, 37 x 43, 208, 178; V = 48000, d = 1072 bf16, 37 x 17, 67, 74;
    // V = 20000, d = 1000, 100 x 5, 68, 70; V = 200000, d = 1024 bf16, 33 x 15, 143, 154.
    const bool same = per * sp->S * 8 >= wgs * 7;
    bool even = !same && (sp->S > 4 * wgs || wgs >= 512);
    if (!same && !even) {
        const double each = sp->S * expected_candidates(t, sp) / (8.0 * kTileN * wgs);   // tiles for a workgroup
        const double most = 8.0 * wgs / (8 * wgs / sp->S * sp->S);                       // the largest share's part of that
        even = most > 1.0 / 0.9 && each * (most - 1.0) > (sizeof(ET) == 2 ? 6.0 : 2.0);
    }
    if (!same) per = 0;
    if (per > 0) wgs = per * sp->S;
    const bool stage = stream_stages(sizeof(ET) == 2, p.ksn, rows, t->d % 2 != 0);
#define LSH_STREAM(MTV, KSNV, PV)                                                                             \
    do {                                                                                                      \
        constexpr bool must = stream_must_trim(sizeof(ET) == 2, PV), may = stream_may_trim(PV) || must;       \
        constexpr bool SOME = stream_stages(sizeof(ET) == 2, KSNV, kTileM * MTV, true), ALL = stream_stages(sizeof(ET) == 2, KSNV, kTileM * (MTV - 1) + 1, false);  \
        const bool trim = may && p.short_last;                                                                \
        launch(cx, 1, even ? k_logits_stream<ET, MTV, KSNV, PV, true, may>                                    \
                      : trim ? (stage ? k_logits_stream<ET, MTV, KSNV, PV, false, may, SOME> : k_logits_stream<ET, MTV, KSNV, PV, false, may, ALL>) \
                      : stage ? k_logits_stream<ET, MTV, KSNV, PV, false, must, SOME> : k_logits_stream<ET, MTV, KSNV, PV, false, must, ALL>,     \
               dim3(8 * wgs * ngroups), dim3(256), StreamLds<MTV, KSNV>::kBytes, (const ET*)t->E, t->ld, t->d, H, sp->S, sp->B, rows, wgs, ngroups, per, shared, cand, count, \
               t->V, w.logits, w.cpitch, w.records());                                                        \
    } while (0)
#define LSH_STREAM2(KSNV, PV) do { if (rows > kTileM) LSH_STREAM(2, KSNV, PV); else LSH_STREAM(1, KSNV, PV); } while (0)
    if (p.ksn == 1) LSH_STREAM2(1, 1); else if (p.ksn == 2 && p.parts == 2) LSH_STREAM2(2, 2); else if (p.ksn == 2) LSH_STREAM2(2, 1);
    else if constexpr (sizeof(ET) == 2) switch (p.parts) { case 2: LSH_STREAM(1, 4, 2); break; case 3: LSH_STREAM(1, 4, 3); break; default: LSH_STREAM(1, 4, 4); }
    else switch (p.parts) {
        case 2: LSH_STREAM2(4, 2); break; case 3: LSH_STREAM(1, 4, 3); break; case 4: LSH_STREAM(1, 4, 4); break;
        case 5: LSH_STREAM(1, 4, 5); break; case 6: LSH_STREAM(1, 4, 6); break; case 7: LSH_STREAM(1, 4, 7); break;
        default: LSH_STREAM(1, 4, 8);
    }
#undef LSH_STREAM2
#undef LSH_STREAM
}

// k_logits_estage (takes_estage).  About one workgroup per CU, dealt evenly to the sentences.
// Returns its workgroups per sentence: each leaves one record per hidden row for all its tiles.
// un, if given: the kernel makes the candidate list itself, from the bitmaps of the sentence's parts.
constexpr int kEsMinD = 512;
int launch_logits_estage(const StepCtx& cx, const float* H, const lsh_step_params* sp,
                         const int32_t* cand, const int32_t* count, const Workspace& w,
                         const EstageUnion* un = nullptr) {
    const lsh_tables* t = cx.t;
    const float* E = (const float*)t->E;
    const int MT = (sp->B + kTileM - 1) / kTileM;
    const size_t lds = estage_lds_bytes(un != nullptr);
    const int per_sentence = std::max(1, t->option(kOptLogitsGrid, 256) / sp->S);
    const dim3 grid((unsigned)(per_sentence * sp->S)), block(1024);
#define LSH_ESTAGE(MTV, UN)                                                                          \
    do {                                                                                             \
        auto kfn = k_logits_estage<MTV, UN>;                                                         \
        launch(cx, 1, kfn, grid, block, lds, E, t->ld, t->d, H, sp->S, sp->B, cand, count, t->V,     \
               w.logits, w.cpitch, w.records(), un ? *un : EstageUnion{});                           \
    } while (0)
    if (un) { if (MT <= 3) LSH_ESTAGE(3, true); else LSH_ESTAGE(4, true); }
    else { if (MT <= 3) LSH_ESTAGE(3, false); else LSH_ESTAGE(4, false); }
#undef LSH_ESTAGE
    return per_sentence;
}

// Whether a step's contraction is k_logits_estage: 33..64 beams, fp32 rows of 513 to 1024 values (shorter ones
// leave half of its four slices of k or more without work: k_logits_stream is 1.2 to 1.9 times faster there,
// 1.1 to 1.3 times slower beyond), 16-byte aligned operands, at most 256 sentences (option logits_estage = 0: the other
// drivers).  Not one sentence of up to two tiles for each of the workgroups: all 256 make the sentence's union and load its
// hidden rows for those, which the stream's row groups share out.  A fourth row group draws the line closer on both
// sides (us a step, estage / stream; d = 1000, 8 bands of 12 bits: V = 40000, 33 beams 43.2 / 36.0, 40: 45.1 / 37.2, 64: 49.9 /
// 47.2; V = 60000, 50: 50.2 / 48.0, 64: 55.8 / 61.4; V = 100000, 33: 51.9 / 50.3, 50: 58.9 / 62.7; V = 4000, 33: 28.1 / 27.7, 64:
// 34.1 / 35.1; V = 1000, 33: 27.0 / 27.2; d = 600: 1.0 to 1.35 times faster on this side of the line).  With two sentences
// only the shorter rows gain (V = 40000, 33 beams: d = 600 42.6 / 39.0, d = 1000 40.8 / 42.6; 64: 54.2 / 53.7, 53.6 / 57.2).
bool takes_estage(const lsh_tables* t, const lsh_step_params* sp, const float* H) {
    const bool aligned = (t->d % 4 == 0) && (t->ld % 4 == 0) && ((uintptr_t)t->E % 16 == 0) && ((uintptr_t)H % 16 == 0);
    const bool able = t->dtype == LSH_F32 && aligned && !sp->full_vocab && sp->B > 2 * kTileM && sp->B <= 4 * kTileM &&
                      t->d > kEsMinD && t->d <= kEsSlices * kEsSlice && sp->S <= 256 && estage_lds_bytes(true) <= kMaxDynLds &&
                      t->option(kOptLogitsEstage, 1) && !t->option(kOptLogitsWaves, 0);
    const bool named = t->opt[kOptLogitsEstage] != kAuto || t->opt[kOptEstageUnion] != kAuto || t->opt[kOptLogitsGrid] != kAuto;
    if (!able || sp->S > 1 || named || names_hlds(t) || !stream_rows<float>(t, sp)) return able;
    const double tiles = expected_candidates(t, sp) / kTileN;
    return sp->B > 3 * kTileM ? tiles < 64 || tiles > 430 : tiles < 8 || tiles > 512;
}

// Returns 0 if the kernel it launched leaves one record per hidden row and tile, else the number
// of record groups per sentence (see select_sentence).
template <typename ET>
int launch_logits(const StepCtx& cx, const float* H, const lsh_step_params* sp,
                  const int32_t* cand, const int32_t* count, const Workspace& w,
                  const EstageUnion* un = nullptr) {
    const lsh_tables* t = cx.t;
    const bool chunks = has_chunks(t);
    const int MT = (sp->B + kTileM - 1) / kTileM;
    const int64_t tiles_n = (int64_t)sp->S * ((t->V + kTileN - 1) / kTileN);  // upper bound
    const int64_t max_tiles = tiles_n * MT;
    // k_logits_stream wherever it takes the rows.  Where it does not and there are few (sentence, M-tile) groups,
    // little work per step and it is latency that counts, so k is split across the 16 waves of a workgroup and
    // the partial tiles are summed through LDS; otherwise one wave per 16-candidate tile.
    // (the full-vocabulary mode has V / 16 tiles per sentence, known here: thousands of tiles
    // are "many" even for one sentence -- 29.9 against 37.1 us at V = 40000)
    const bool few = sp->S * MT <= 8 && !(count == nullptr && tiles_n >= 1024);
    // (fused = 0 asks for the fused plan's arithmetic in kernels of its own: k split over 16 waves as there)
    const bool as_fused = few && MT <= 2 && t->opt[kOptFused] == 0;
    const int rows = names_hlds(t) || as_fused ? 0 : stream_rows<ET>(t, sp);
    const int mode = t->option(kOptLogitsWaves, few && !rows ? 16 : 1);
    // one wave per tile with the sentence's hidden rows staged in LDS, more than 32 rows in
    // groups; LSHBEAM_LOGITS_HLDS=0 keeps the rows in global memory (k_logits_wave)
    const int group_rows = hlds_group_rows(t, sp->S, sp->B, t->d);
    // 33..64 beams: hidden rows in registers, candidate rows through LDS (LSHBEAM_LOGITS_ESTAGE=0:
    // the other drivers)
    if (takes_estage(t, sp, H)) {
        return launch_logits_estage(cx, H, sp, cand, count, w, un);
    } else if (mode == 1 && rows > 0) {
        launch_logits_stream<ET>(cx, tiles_n, H, sp, cand, count, w, rows);
    } else if (mode == 1 && chunks && group_rows > 0 && t->option(kOptLogitsHlds, 1)) {
        launch_logits_hlds<ET>(cx, tiles_n, H, sp, cand, count, w, group_rows);
    } else if (mode == 1 && MT <= 4) {
        const int grid = (int)std::min<int64_t>((tiles_n + 3) / 4, t->option(kOptLogitsGrid, 1024));
        switch (MT) {
            case 1: launch_logits_wave<ET, 1>(cx, grid, chunks, H, sp, cand, count, w); break;
            case 2: launch_logits_wave<ET, 2>(cx, grid, chunks, H, sp, cand, count, w); break;
            case 3: launch_logits_wave<ET, 3>(cx, grid, chunks, H, sp, cand, count, w); break;
            default: launch_logits_wave<ET, 4>(cx, grid, chunks, H, sp, cand, count, w); break;
        }
    } else if (mode >= 16) {
        const int grid = (int)std::min<int64_t>(max_tiles, t->option(kOptLogitsGrid, 256));
        launch_logits_w<ET, 16>(cx, grid, chunks, H, sp, cand, count, w);
    } else {
        const int grid = (int)std::min<int64_t>(max_tiles, t->option(kOptLogitsGrid, 2048));
        launch_logits_w<ET, 4>(cx, grid, chunks, H, sp, cand, count, w);
    }
    return 0;
}

// Full vocabulary: one matrix product over all hidden rows of the call.  Up to 48 rows (fp32; 32 with bf16
// words) the pass over E is what counts: k_logits_pass or k_logits_few.  Beyond that k_logits_rows; its row groups are as
// even as they come in units of 16 rows, and among the splits the accumulators leave room for, the one
// with the least work on the fullest CU is taken: two workgroups of m row tiles on a CU take 3 + m, one alone 1.5 + 0.6 m
// (in no unit; for d from 96 to 1536 and either type each is within 12 % of that, up to a factor of d's own).
// Over V = 10000 .. 100000, d = 128 .. 1536 and 48 .. 640 rows (181 shapes of each type, every m measured)
// the choice is 0.1 % slower than the best one on average and 6 % at most.
// Where even k_logits_stream, with a tile of 16 words and groups of hidden rows per workgroup and k split over its waves, has
// at most 512 workgroups' worth of tiles in groups of 32 rows (1024 in groups of 16), it is the faster one: the others then
// run few workgroups through a long chain of k blocks (31 rows, V = 2009, d = 1181: 22.8 -> 10.6 us; 128 rows, V = 2000, d = 1100:
// 32.1 -> 22.3, V = 1000, 256 rows: 34.4 -> 22.5).  Its logits are as near: k_logits_stream's CHAINS.
constexpr int kRowsMinD = 8;   // (a row holds at least one 16-byte chunk)
// Row tiles per workgroup at most: what the 256 registers of a lane leave room for.
template <typename ET> constexpr int rows_max_mt() { return sizeof(ET) == 2 ? 4 : 5; }
bool takes_rows(const lsh_tables* t, const lsh_step_params* sp) {   // (an option that names another driver wins)
    lsh_step_params all = *sp;
    all.S = 1;
    all.B = sp->S * sp->B;
    const int rows = t->dtype == LSH_F32 ? stream_rows<float>(t, &all) : stream_rows<uint16_t>(t, &all);
    const int wide = t->dtype == LSH_F32 ? 2 * kTileM : std::max(rows, kTileM);
    const int64_t tiles = (t->V + kTileN - 1) / kTileN;
    if (rows > 0 && tiles * ((all.B + wide - 1) / wide) <= 512) return false;
    return sp->full_vocab && t->d >= kRowsMinD && t->opt[kOptLogitsWaves] == kAuto && t->opt[kOptLogitsEstage] == kAuto &&
           t->opt[kOptLogitsHlds] == kAuto && t->opt[kOptHldsRows] == kAuto && t->opt[kOptLogitsGrid] == kAuto &&
           t->option(kOptLogitsPlanes, 1) != 0;
}
// Returns the words a record is for.
template <typename ET>
int launch_logits_rows(const StepCtx& cx, const float* H, int R, int B, const Workspace& w) {
    const lsh_tables* t = cx.t;
    const int tiles = (R + kTileM - 1) / kTileM;
    constexpr int WF = sizeof(ET) == 2 ? 4 : 2, FEW = sizeof(ET) == 2 ? 2 : 3;
    const PassPlan p = pass_plan<ET>(R, B, t->V, t->d, t->ld);
    if (p.waves) {
        constexpr int PASS = pass_most_tiles<ET>();
        const int words = p.waves * p.rounds * kTileN;
        const size_t lds = pass_lds_bytes<ET>(tiles, t->d);
        const dim3 grid((unsigned)((t->V + words - 1) / words)), block(p.waves * kWave);
#define LSH_PASS(MTV)                                                                                                \
    launch(cx, 1, k_logits_pass<ET, MTV>, grid, block, lds, (const ET*)t->E, t->ld, t->d, H, R, t->V, \
           p.rounds, w.logits, w.cpitch, w.records())
        if (tiles == 1) LSH_PASS(1);
        else if constexpr (PASS == 3) { if (tiles == 2) LSH_PASS(2); else LSH_PASS(3); }
#undef LSH_PASS
        return words;
    }
    if (tiles <= FEW) {
        const dim3 grid((unsigned)((t->V + kWideN - 1) / kWideN)), block(256);
#define LSH_FEW(MTV)                                                                                           \
    launch(cx, 1, k_logits_few<ET, MTV>, grid, block, few_lds_bytes<ET>(MTV), (const ET*)t->E, t->ld, t->d, H, R, t->V, \
           w.logits, w.cpitch, w.records())
        if (tiles == 1) LSH_FEW(1); else if (tiles == 2) LSH_FEW(2); else LSH_FEW(3);
#undef LSH_FEW
        return kWideN;
    }
    const int gx = (t->V + 64 * WF - 1) / (64 * WF);
    int mt = rows_max_mt<ET>();
    double best = 1e30;
    for (int m = 1; m <= rows_max_mt<ET>(); ++m) {
        const int n = (tiles + m - 1) / m * gx;
        const int left = n % 512;   // pairs of workgroups on every CU, then what is left
        const double two = 3 + m, one = 1.5 + 0.6 * m;
        const double cost = n / 512 * two + (left > 256 ? two : left ? one : 0);
        if (cost < best) { best = cost; mt = m; }
    }
    const int ng = (tiles + mt - 1) / mt;
    const dim3 grid((unsigned)((gx + 7) / 8 * 8 * ng)), block(256);
#define LSH_ROWS(MTV)                                                                                          \
    launch(cx, 1, k_logits_rows<ET, MTV, WF>, grid, block, rows_lds_bytes(MTV), (const ET*)t->E, t->ld, t->d, H, R, \
           t->V, gx, ng, w.logits, w.cpitch, w.records())
    switch (mt) {
        case 1: LSH_ROWS(1); break; case 2: LSH_ROWS(2); break; case 3: LSH_ROWS(3); break; case 4: LSH_ROWS(4); break;
        default: if constexpr (rows_max_mt<ET>() == 5) LSH_ROWS(5);
    }
#undef LSH_ROWS
    return kWideN;
}

template <typename ET>
hipError_t allow_logits_lds() {
    constexpr int U1 = 8 / (ElemTraits<ET>::VEC / 4), U2 = 4 / (ElemTraits<ET>::VEC / 4);
    constexpr int U2W = (U2 > 2) ? U2 - 1 : U2;
    hipError_t e = hipSuccess;
#define LSH_ALLOW(...)                                                   \
    do {                                                                 \
        if (e == hipSuccess) e = allow_whole_lds<k_logits_hlds<ET, __VA_ARGS__>>(); \
    } while (0)
    LSH_ALLOW(1, 8, U1, false); LSH_ALLOW(2, 8, U2, false);
    LSH_ALLOW(1, 16, U1, false); LSH_ALLOW(2, 16, U2W, false);
    if constexpr (std::is_same<ET, uint16_t>::value) LSH_ALLOW(1, 8, U1, true);
#undef LSH_ALLOW
#define LSH_ALLOW(MTV, KSNV, PV)                                                                        \
    do {                                                                                            \
        constexpr bool must = stream_must_trim(sizeof(ET) == 2, PV), may = stream_may_trim(PV) || must; \
        constexpr bool SOME = stream_stages(sizeof(ET) == 2, KSNV, kTileM * MTV, true), ALL = stream_stages(sizeof(ET) == 2, KSNV, kTileM * (MTV - 1) + 1, false);  \
        if (e == hipSuccess) e = allow_whole_lds<k_logits_stream<ET, MTV, KSNV, PV, false, must, SOME>>();  \
        if (e == hipSuccess) e = allow_whole_lds<k_logits_stream<ET, MTV, KSNV, PV, false, may, SOME>>();   \
        if (e == hipSuccess) e = allow_whole_lds<k_logits_stream<ET, MTV, KSNV, PV, false, must, ALL>>();   \
        if (e == hipSuccess) e = allow_whole_lds<k_logits_stream<ET, MTV, KSNV, PV, false, may, ALL>>();    \
        if (e == hipSuccess) e = allow_whole_lds<k_logits_stream<ET, MTV, KSNV, PV, true, may>>();      \
    } while (0)
    LSH_ALLOW(1, 1, 1); LSH_ALLOW(1, 2, 1); LSH_ALLOW(1, 4, 2); LSH_ALLOW(1, 4, 3); LSH_ALLOW(1, 4, 4);
    LSH_ALLOW(2, 1, 1); LSH_ALLOW(2, 2, 1); LSH_ALLOW(1, 2, 2); LSH_ALLOW(2, 2, 2);
    if constexpr (sizeof(ET) == 4) {
        LSH_ALLOW(2, 4, 2);
        LSH_ALLOW(1, 4, 5); LSH_ALLOW(1, 4, 6); LSH_ALLOW(1, 4, 7); LSH_ALLOW(1, 4, 8);
    }
#undef LSH_ALLOW
    return e;
}

// What allow_whole_lds does, for every kernel of a step (about a hundred: asked for one by one they took 1 to 2 us of every build).
hipError_t allow_step_lds(int dev) {
    static std::atomic<uint64_t> done{0};  // one bit per device
    const uint64_t bit = (dev >= 0 && dev < 64) ? (1ull << dev) : 0ull;
    if (bit && (done.load(std::memory_order_acquire) & bit)) return hipSuccess;
    hipError_t e = hipSuccess;
#define LSH_ALLOW(...) do { if (e == hipSuccess) e = (__VA_ARGS__); } while (0)
    LSH_ALLOW(allow_whole_lds<k_candidates<1>>());
    LSH_ALLOW(allow_whole_lds<k_candidates<kCandParts>>());
    LSH_ALLOW((allow_whole_lds<k_logits_pass<float, 1>>()));
    LSH_ALLOW((allow_whole_lds<k_logits_pass<float, 2>>()));
    LSH_ALLOW((allow_whole_lds<k_logits_pass<float, 3>>()));
    LSH_ALLOW((allow_whole_lds<k_logits_pass<uint16_t, 1>>()));
    LSH_ALLOW(allow_whole_lds<k_hit_rows<Alone>>());
    LSH_ALLOW(allow_whole_lds<k_hit_rows<FirstTilesBeside<float>>>());
    LSH_ALLOW(allow_whole_lds<k_hit_rows<FirstTilesBeside<uint16_t>>>());
    LSH_ALLOW(allow_whole_lds<k_union_compact>());
    LSH_ALLOW(allow_whole_lds<k_part_bitmaps<Alone>>());
    LSH_ALLOW(allow_whole_lds<k_part_bitmaps<FirstTilesBeside<float>>>());
    LSH_ALLOW(allow_whole_lds<k_part_bitmaps<FirstTilesBeside<uint16_t>>>());
#define LSH_ALLOW_FUSED(ET, AL)                                          \
    LSH_ALLOW((allow_whole_lds<k_union_logits<ET, AL, false>>()));         \
    LSH_ALLOW((allow_whole_lds<k_union_logits<ET, AL, true>>()));          \
    LSH_ALLOW((allow_whole_lds<k_cand_logits<ET, AL, false>>()));          \
    LSH_ALLOW((allow_whole_lds<k_cand_logits<ET, AL, false, AL>>()));     \
    LSH_ALLOW((allow_whole_lds<k_cand_logits<ET, AL, true>>()))
    LSH_ALLOW_FUSED(float, true);
    LSH_ALLOW_FUSED(float, false);
    LSH_ALLOW_FUSED(uint16_t, true);
    LSH_ALLOW_FUSED(uint16_t, false);
#undef LSH_ALLOW_FUSED
    LSH_ALLOW(allow_logits_lds<float>());
    LSH_ALLOW(allow_logits_lds<uint16_t>());
    LSH_ALLOW((allow_whole_lds<k_logits_estage<3, false>>()));
    LSH_ALLOW((allow_whole_lds<k_logits_estage<4, false>>()));
    LSH_ALLOW((allow_whole_lds<k_logits_estage<3, true>>()));
    LSH_ALLOW((allow_whole_lds<k_logits_estage<4, true>>()));
#undef LSH_ALLOW
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}

#define HIP_TRY(expr)                                   \
    do {                                                \
        hipError_t e_ = (expr);                         \
        if (e_ != hipSuccess) {                         \
            (void)hipGetLastError();                    \
            return e_ == hipErrorOutOfMemory ? LSH_ERR_OOM : LSH_ERR_HIP; \
        }                                               \
    } while (0)

// Device memory that stays with the library for the next build on the device: a block that held a handle, one that
// held the slots of one, and one that a build worked in, together at most kKeptBytes (a driver allocation or release of a few MiB takes 20 to
// 60 us, as long as the kernels of the build; an index is rebuilt where the embeddings change).  Given back by
// lsh_release_kept() and wherever an allocation of a build fails; guarded by its own mutex.  A block is kept only
// once the device has finished everything that was launched with it.
constexpr size_t kKeptBytes = (size_t)192 << 20;
enum KeptKind { kHandleBlock, kSlotBlock, kBuildBlock, kKeptKinds };
std::mutex g_kept_mu;
KeptBlock g_kept[kMaxDevices][kKeptKinds];

// Puts b in the block's place and returns what was there; b itself where there is no room for it.
KeptBlock swap_kept(int dev, KeptKind kind, KeptBlock b) {
    std::lock_guard<std::mutex> lock(g_kept_mu);
    size_t others = 0;
    for (int k = 0; k < kKeptKinds; ++k)
        if (k != kind) others += g_kept[dev][k].bytes;
    if (b.bytes + others <= kKeptBytes) std::swap(b, g_kept[dev][kind]);
    return b;
}
// Returns what that device's free memory grows by at least: blocks are in pages of 2 MiB (smaller ones share them).
size_t give_back_kept(int dev = -1) {
    constexpr size_t kPage = (size_t)2 << 20;
    size_t bytes = 0;
    for (int d = 0; d < kMaxDevices; ++d)
        for (int k = 0; k < kKeptKinds; ++k) {
            const KeptBlock b = swap_kept(d, (KeptKind)k, KeptBlock{});
            if (b.p && d == dev && b.bytes >= kPage) bytes += (b.bytes + kPage - 1) / kPage * kPage;
            if (b.p) (void)hipFree(b.p);
        }
    return bytes;
}
// An allocation of a build: where memory has run out, once more without the kept blocks.
hipError_t alloc_device(void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes ? bytes : 1);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        (void)give_back_kept();
        e = hipMalloc(p, bytes ? bytes : 1);
    }
    return e;
}
hipError_t take_block(int dev, KeptKind kind, size_t bytes, KeptBlock* out) {
    if (dev < kMaxDevices && bytes <= kKeptBytes) {
        const KeptBlock b = swap_kept(dev, kind, KeptBlock{});
        if (b.p && b.bytes >= bytes) { *out = b; return hipSuccess; }
        if (b.p) (void)hipFree(b.p);
    }
    out->bytes = bytes;
    return alloc_device(&out->p, bytes);
}
// idle: nothing that was launched uses the block any more (set where this waits for it).
void release_block(int dev, KeptKind kind, KeptBlock b, bool& idle) {
    if (!b.p) return;
    if (dev < kMaxDevices && b.bytes <= kKeptBytes) {
        if (!idle) {   // (as hipFree would)
            int cur = 0;
            idle = hipGetDevice(&cur) == hipSuccess && (cur == dev || hipSetDevice(dev) == hipSuccess) &&
                   hipDeviceSynchronize() == hipSuccess;
            if (cur != dev) (void)hipSetDevice(cur);
        }
        if (idle) b = swap_kept(dev, kind, b);
    }
    if (b.p) (void)hipFree(b.p);
}

// Regions of one device allocation, each 256-byte aligned: sized with base = null, then placed.
struct Carver {
    char* base;
    size_t bytes = 0;
    template <typename T> T* take(size_t n) {
        T* p = reinterpret_cast<T*>(base + bytes);
        bytes += align_up(n * sizeof(T));
        return base ? p : nullptr;
    }
};

lsh_status place_slots(lsh_tables* t, uint64_t n_slots) {
    if (t->slot_block.p) (void)hipFree(t->slot_block.p);
    t->slot_block = KeptBlock{};
    const size_t slot_bytes = align_up(n_slots * sizeof(Slot));
    HIP_TRY(take_block(t->device, kSlotBlock, slot_bytes + n_slots * sizeof(uint4), &t->slot_block));
    t->slots_dev = (Slot*)t->slot_block.p;
    t->cuts_dev = (uint4*)((char*)t->slot_block.p + slot_bytes);
    return LSH_OK;
}

// Host path of the table build: codes are copied back, every band's (code, id) pairs are sorted
// and inserted into its cuckoo table on the host, then uploaded.
lsh_status build_on_host(lsh_tables* t, hipStream_t st, SplitMix64& rng) {
    const size_t V = t->V, W = t->W;
    std::vector<Slot> slots_host;
    std::vector<int32_t> codes(V * W);
    HIP_TRY(hipMemcpyAsync(codes.data(), t->codes_dev, V * W * sizeof(int32_t), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));

    // per band: group word ids by code (ids ascending inside a span), then the cuckoo table
    std::vector<int32_t> words(V * W);
    std::vector<uint64_t> order(V);
    std::vector<HostBand> hbs(W);
    for (size_t w = 0; w < W; ++w) {
        for (size_t j = 0; j < V; ++j)
            order[j] = ((uint64_t)(uint32_t)codes[w * V + j] << 32) | (uint64_t)j;
        std::sort(order.begin(), order.end());
        HostBand& hb = hbs[w];
        for (size_t i = 0; i < V; ++i) {
            const int32_t code = (int32_t)(order[i] >> 32);
            if (i == 0 || code != hb.keys.back()) {
                hb.keys.push_back(code);
                hb.offsets.push_back((int32_t)i);
            }
            words[w * V + i] = (int32_t)(uint32_t)order[i];
        }
        hb.offsets.push_back((int32_t)V);
        hb.n_keys = (int)hb.keys.size();
        const lsh_status rc = build_cuckoo(hb, rng, slots_host, (uint32_t)slots_host.size());
        if (rc != LSH_OK) return rc;
    }
    std::vector<BandMeta> metas(W);
    for (size_t w = 0; w < W; ++w) metas[w] = hbs[w].meta;

    // where the vocabulary slices of the hit-count kernel begin inside every span
    std::vector<uint4> cuts_host(slots_host.size(), make_uint4(0u, 0u, 0u, 0u));
    const int slice_ids = hit_slice_words(t->V);
    for (size_t w = 0; w < W; ++w) {
        const BandMeta& m = hbs[w].meta;
        for (int i = 0; i < hbs[w].capacity; ++i) {
            const Slot& sl = slots_host[m.slot_off + i];
            if (sl.key < 0) continue;
            const int32_t* span = words.data() + w * V + sl.start;
            uint32_t c[3];
            for (int q = 1; q <= 3; ++q)
                c[q - 1] = (uint32_t)(std::lower_bound(span, span + sl.len, q * slice_ids) - span);
            cuts_host[m.slot_off + i] = make_uint4(c[0], c[1], c[2], sl.len);
        }
    }
    const lsh_status rc = place_slots(t, slots_host.size());
    if (rc != LSH_OK) return rc;
    HIP_TRY(hipMemcpyAsync(t->cuts_dev, cuts_host.data(), cuts_host.size() * sizeof(uint4),
                           hipMemcpyHostToDevice, st));
    HIP_TRY(hipMemcpyAsync(t->words_dev, words.data(), V * W * sizeof(int32_t), hipMemcpyHostToDevice, st));
    HIP_TRY(hipMemcpyAsync(t->slots_dev, slots_host.data(), slots_host.size() * sizeof(Slot),
                           hipMemcpyHostToDevice, st));
    HIP_TRY(hipMemcpyAsync(t->bands_dev, metas.data(), W * sizeof(BandMeta), hipMemcpyHostToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));
    t->bands.assign(hbs.begin(), hbs.end());   // (their Band parts)
    return LSH_OK;
}

struct DevBuf {  // temporary device memory of the build, released on every exit path
    void* p = nullptr;
    ~DevBuf() { if (p) (void)hipFree(p); }
    hipError_t alloc(size_t bytes) { return alloc_device(&p, bytes); }
};

struct BuildBlock {  // what a build works in, kept for the next one
    int dev = 0;
    KeptBlock block;
    bool idle = false;
    ~BuildBlock() { release_block(dev, kBuildBlock, block, idle); }
};

// (`first` with kRaw: where row_codes_ahead)
template <typename ET, class FIRST = NotFirst>
hipError_t launch_row_codes(hipStream_t st, const ET* X, int64_t ld, int64_t n, int d, const int32_t* perms, int P, int K,
                            int W, int bits, int32_t* out, int64_t row_stride, int64_t band_stride, FIRST first = {}) {
    const bool ahead = row_codes_ahead(d, sizeof(ET), P, K);
    const int lg = row_codes_lg_rows(n, d, sizeof(ET), P, ahead);
    const size_t lds = row_codes_lds(1 << lg, d, sizeof(ET), P, ahead);
    int64_t groups = (n + (1 << lg) - 1) >> lg;
    if (ahead) groups = std::min<int64_t>(groups, 256 * std::min<size_t>(8, 158 * 1024 / lds));   // (as many as run at a time)
    if (FIRST::kRaw && !ahead) return hipErrorInvalidValue;   // (what `first` does would be left out)
    auto go = [&](auto ahead_c, auto f) -> hipError_t {
        constexpr auto kernel = k_row_codes<ET, decltype(ahead_c)::value, decltype(f)>;
        const hipError_t e = allow_whole_lds<kernel>();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(kRowCodeThreads), lds, st, X, ld, n, d, perms, P, K, W, bits, lg, out,
                           row_stride, band_stride, f);
        return hipGetLastError();
    };
    return ahead ? go(std::true_type{}, first) : go(std::false_type{}, NotFirst{});
}

// The table build (build_tables.h).  The bucket and cuckoo tables are made on the device; `on_host`, a band
// that keeps failing its insertion or a table beyond 32-bit slot numbers takes the host path instead.
lsh_status build_all(lsh_tables* t, hipStream_t st, const int32_t* perms_in, uint64_t seed, bool on_host) {
    const int64_t V = t->V, W = t->W;
    const size_t n_perms = (size_t)t->P * t->K, n_tickets = (size_t)kTicketSlots * kTicketBlock;
    const int code_bits = t->u * t->bits;
    const int passes = (code_bits + kRadixBits - 1) / kRadixBits, pass_bits = (code_bits + passes - 1) / passes;
    const int digits = 1 << pass_bits, groups_n = (digits + kScanDigits - 1) / kScanDigits;
    const RadixChunks ch = radix_chunks(V, (int)W);
    const int chunks = ch.count();
    // a band has at most key_pitch keys; a cuckoo table has a power of two of at least three slots per key (load
    // <= 1/3: two-choice cuckoo insertion then succeeds at the first attempt almost always)
    const uint32_t key_pitch = (uint32_t)std::min<int64_t>(V, (int64_t)1 << code_bits);
    constexpr uint64_t kSlotBytes = sizeof(Slot) + sizeof(uint4) + sizeof(uint64_t);
    auto lg_for = [](uint32_t keys) { int lg = 1; while ((1ull << lg) < 3ull * keys) ++lg; return lg; };
    int lg = lg_for(key_pitch);
    // Direct tables, with a slot for every code there can be (and as many empty ones: twice the keys at least), where
    // they are no larger than cuckoo tables for the keys, or where they are small.  Nothing is inserted there, and
    // the tables a step probes are half as large or less.  What they save: an insertion that fails ends with its
    // longest chain, 100 us (12-bit codes that all occur failed the first attempt one build in two: 8 bands, V = 40000,
    // d = 1000, with the first step: 156 or 206 us, 130 so).  (LSHBEAM_CUCKOO_CHAIN, for the tests of the insertion, asks for cuckoo tables.)
    const int chain = env_int("LSHBEAM_CUCKOO_CHAIN", -1);
    auto takes_direct = [&](int cuckoo_lg) {
        return chain < 0 && (code_bits + 1 <= cuckoo_lg || (passes == 1 && ((uint64_t)W << (code_bits + 1)) * (sizeof(Slot) + sizeof(uint4)) <= (4ull << 20)));
    };
    bool direct = takes_direct(lg);
    if (direct) lg = code_bits + 1;
    // Tables for the most keys there can be, so that nothing has to be known before they are placed, where those are
    // at most 32 MiB (V = 14000, 10 bands of 16-bit codes, 26 MB: 118 us, 141 with the keys counted first: one wait),
    // or where so many words share the codes that hardly one will be missing.  Otherwise the keys are counted: 16-bit
    // codes have room for 65536 keys and 27000 to 42000 come up (V = 100000, 12 bands: 100 MB of slots, 50 for the
    // keys there are; 370 us, 340 so).
    const uint64_t most_bytes = ((uint64_t)W << lg) * kSlotBytes;
    const bool blind = most_bytes <= (32ull << 20) || (V >= 8ll << code_bits && most_bytes <= (1ull << 30));
    const bool emit = direct && passes == 1 && blind;   // the scan writes the slots
    auto table_bytes = [&]() { return ((uint64_t)W << lg) * sizeof(uint64_t); };
    // A counted table takes the place of what the sort is through with, where that is large enough or can be made so
    // within reason.
    const size_t sort_buf = align_up((size_t)V * W * sizeof(int32_t));
    const size_t sort_spare = passes > 1 ? sort_buf * std::min(passes, 3) : 0;
    const size_t spare_bytes = blind ? sort_spare : std::max<size_t>(sort_spare, std::min<uint64_t>(table_bytes(), 64ull << 20));

    struct Status { uint32_t *failed[2], *n_keys; } stat{};
    uint32_t *status_dev = nullptr, *counts = nullptr, *groups = nullptr, *starts = nullptr, *key_start = nullptr;
    uint64_t* table = nullptr;
    int32_t *key_code = nullptr, *code_buf[2] = {}, *id_buf[2] = {};
    const size_t status_words = 3 * (size_t)W;
    Report report;
    static_assert(Report::kWords >= kBuildBeginBlocks, "a word per workgroup of k_build_begin");
    HIP_TRY(report.take());
    BuildBlock work;   // (what only the build needs)
    work.dev = t->device;
    for (int pass = 0; pass < 2; ++pass) {
        Carver c{(char*)t->arena.p};
        t->perms_dev = c.take<int32_t>(n_perms);
        t->tickets_dev = c.take<unsigned int>(n_tickets);
        t->bands_dev = c.take<BandMeta>(W);
        t->n_keys_dev = c.take<uint32_t>(W);
        t->codes_dev = c.take<int32_t>((size_t)V * W);
        // 16 bytes of slack: k_hit_rows reads ids with 16-byte loads that may straddle the end
        t->words_dev = c.take<int32_t>((size_t)V * W + 4);
        if (blind) {
            t->slots_dev = c.take<Slot>((size_t)W << lg);
            t->cuts_dev = c.take<uint4>((size_t)W << lg);
        }
        Carver b{(char*)work.block.p};
        status_dev = b.take<uint32_t>(status_words);
        if (blind && !emit) table = b.take<uint64_t>((size_t)W << lg);
        counts = b.take<uint32_t>((size_t)W * chunks * (digits / 2));
        groups = b.take<uint32_t>((size_t)W * chunks * groups_n);
        starts = b.take<uint32_t>((size_t)W * chunks * digits);
        if (!emit) {
            key_code = b.take<int32_t>((size_t)W * key_pitch);
            key_start = b.take<uint32_t>((size_t)W * key_pitch);
        }
        char* spare = b.take<char>(spare_bytes);
        if (!emit) {        // (pass p writes code_buf[p % 2] and, but for the last, id_buf[p % 2])
            code_buf[(passes - 1) & 1] = b.take<int32_t>((size_t)V * W);
            code_buf[passes & 1] = passes > 1 ? (int32_t*)spare : nullptr;
            id_buf[0] = spare && passes > 1 ? (int32_t*)(spare + sort_buf) : nullptr;
            id_buf[1] = spare && passes > 2 ? (int32_t*)(spare + 2 * sort_buf) : nullptr;
        }
        if (!blind) table = (uint64_t*)spare;
        if (!pass) {
            HIP_TRY(take_block(t->device, kHandleBlock, c.bytes, &t->arena));
            HIP_TRY(take_block(t->device, kBuildBlock, b.bytes, &work.block));
        }
    }
    stat.n_keys = emit ? t->n_keys_dev : status_dev;
    stat.failed[0] = status_dev + W;
    stat.failed[1] = stat.failed[0] + W;
    DevBuf late;

    const dim3 begin_grid(kBuildBeginBlocks, (unsigned)W + 1), b256(256);
    auto begin = [&](int attempt, const uint32_t* redo, bool with_tables) {
        hipLaunchKernelGGL(k_build_begin, begin_grid, b256, 0, st, table, t->bands_dev, (int)W,
                           with_tables && !emit ? 1u << lg : 0u, lg, direct, seed, attempt, redo, stat.failed[attempt & 1],
                           emit ? stat.n_keys : nullptr,
                           attempt || (with_tables && !blind) ? nullptr : perms_in, (int)n_perms, t->d, t->perms_dev, report.words,
                           t->tickets_dev, (int)n_tickets);
    };
    report.idle = false;
    auto row_codes = [&](const int32_t* perms, auto first) {
        return t->dtype == LSH_F32
            ? launch_row_codes(st, (const float*)t->E, t->ld, V, t->d, perms, t->P, t->K, t->W, t->bits, t->codes_dev, 1, V, first)
            : launch_row_codes(st, (const uint16_t*)t->E, t->ld, V, t->d, perms, t->P, t->K, t->W, t->bits, t->codes_dev, 1, V, first);
    };
    if (emit && row_codes_ahead(t->d, t->dtype == LSH_F32 ? 4 : 2, t->P, t->K)) {
        HIP_TRY(row_codes(perms_in, BuildFirst{perms_in, t->perms_dev, report.words, t->bands_dev, stat.n_keys, t->tickets_dev, (int)n_perms,
                                               t->d, (int)W, lg, (int)n_tickets}));
    } else {
        begin(0, nullptr, blind);
        HIP_TRY(row_codes(t->perms_dev, NotFirst{}));
    }

    std::vector<uint32_t> status(status_words);
    auto wait = [&]() -> lsh_status {
        HIP_TRY(hipStreamSynchronize(st));
        work.idle = report.idle = true;   // (until the next launch)
        for (int i = 0; i < kBuildBeginBlocks; ++i)
            if (report.words[i]) return LSH_ERR_INVALID_ARG;
        return LSH_OK;
    };
    auto read_status = [&]() -> lsh_status {
        HIP_TRY(hipMemcpyAsync(status.data(), status_dev, status_words * sizeof(uint32_t), hipMemcpyDeviceToHost, st));
        return wait();
    };
    const uint32_t* keys_h = status.data();
    SplitMix64 host_rng{seed};
    if (on_host) {
        const lsh_status rc = read_status();
        return rc != LSH_OK ? rc : build_on_host(t, st, host_rng);
    }

    const dim3 sort_grid((unsigned)chunks * (unsigned)W), key_grid((unsigned)chunks, (unsigned)W), sort_block(kRadixThreads);
    HIP_TRY(allow_whole_lds<k_radix_scatter>());
    const int32_t *codes_in = t->codes_dev, *ids_in = nullptr;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * pass_bits;
        hipLaunchKernelGGL(k_radix_count, sort_grid, sort_block, (size_t)digits * 2, st, codes_in, V, (int)W, ch, shift, digits, counts, groups);
        const dim3 scan_grid((unsigned)groups_n, (unsigned)W), scan_block(kScanDigits / 2);
        if (emit)
            hipLaunchKernelGGL(k_radix_scan<true>, scan_grid, scan_block, 0, st, (const uint32_t*)counts, (const uint32_t*)groups, ch,
                               digits, starts, t->slots_dev, t->cuts_dev, stat.n_keys);
        else
            hipLaunchKernelGGL(k_radix_scan<false>, scan_grid, scan_block, 0, st, (const uint32_t*)counts, (const uint32_t*)groups, ch,
                               digits, starts, nullptr, nullptr, nullptr);
        int32_t* ids_out = p == passes - 1 ? t->words_dev : id_buf[p & 1];
        hipLaunchKernelGGL(k_radix_scatter, sort_grid, sort_block, radix_scatter_lds(digits), st, codes_in, ids_in, V, (int)W, ch,
                           shift, pass_bits, (const uint32_t*)starts, code_buf[p & 1], ids_out);
        codes_in = code_buf[p & 1];
        ids_in = ids_out;
    }
    t->bands.resize(W);
    auto finish = [&](auto&& n_keys, auto&& meta) {
        for (int64_t w = 0; w < W; ++w) {
            t->bands[w].n_keys = n_keys(w);
            t->bands[w].capacity = 1 << lg;
            t->bands[w].meta = meta(w);
        }
        t->built_on_device = 1;
        return LSH_OK;
    };
    if (emit) {
        HIP_TRY(hipGetLastError());
        const lsh_status rc = wait();
        t->build_attempts = 1;
        return rc != LSH_OK ? rc : finish([](int64_t) { return -1; }, [&](int64_t w) { return direct_band_meta((int)w, lg); });
    }
    // (the counters are free again: at least one per chunk and band)
    hipLaunchKernelGGL(k_key_count, key_grid, sort_block, 0, st, codes_in, V, ch, counts);
    hipLaunchKernelGGL(k_key_emit, key_grid, sort_block, 0, st, codes_in, V, ch, (const uint32_t*)counts, key_code,
                       key_start, key_pitch, stat.n_keys);
    if (!blind) {
        lsh_status rc = read_status();
        if (rc != LSH_OK) return rc;
        lg = lg_for(*std::max_element(keys_h, keys_h + W));
        direct = takes_direct(lg);
        if (direct) lg = code_bits + 1;
        if (((uint64_t)W << lg) >= (1ull << 32)) return build_on_host(t, st, host_rng);
        rc = place_slots(t, (uint64_t)W << lg);
        if (rc != LSH_OK) return rc;
        if (table_bytes() > spare_bytes) {
            HIP_TRY(late.alloc(table_bytes()));
            table = (uint64_t*)late.p;
        }
        work.idle = report.idle = false;
        begin(0, nullptr, true);
    }
    // LSHBEAM_CUCKOO_CHAIN shortens the eviction chains (tests of the retry and fallback paths)
    const int max_chain = chain >= 0 ? chain : 16 * (lg + 1);
    const dim3 insert_grid((key_pitch + 255) / 256, (unsigned)W), slot_grid(((1u << lg) + 255) / 256, (unsigned)W);
    std::vector<int> drawn(W, 0);   // the attempt whose parameters each band has
    for (int attempt = 0; attempt < 24; ++attempt) {
        t->build_attempts = attempt + 1;
        const uint32_t* redo = attempt ? stat.failed[(attempt - 1) & 1] : nullptr;
        work.idle = report.idle = false;
        if (attempt) begin(attempt, redo, true);
        hipLaunchKernelGGL(k_cuckoo_insert, insert_grid, b256, 0, st, table, (const BandMeta*)t->bands_dev,
                           (const int32_t*)key_code, key_pitch, (const uint32_t*)stat.n_keys, max_chain, redo,
                           stat.failed[attempt & 1]);
        hipLaunchKernelGGL(k_cuckoo_finalize, slot_grid, b256, 0, st, (const uint64_t*)table, 1u << lg,
                           (const uint32_t*)key_start, key_pitch, (const uint32_t*)stat.n_keys,
                           (const int32_t*)t->words_dev, (uint32_t)V, hit_slice_words(t->V), t->slots_dev, t->cuts_dev);
        HIP_TRY(hipGetLastError());
        const lsh_status rc = read_status();
        if (rc != LSH_OK) return rc;
        if (attempt) for (int64_t w = 0; w < W; ++w)
            if (status[(stat.failed[(attempt - 1) & 1] - status_dev) + w]) drawn[w] = attempt;
        const uint32_t* failed_h = status.data() + (stat.failed[attempt & 1] - status_dev);
        if (std::any_of(failed_h, failed_h + W, [](uint32_t f) { return f != 0; })) continue;
        return finish([&](int64_t w) { return (int)keys_h[w]; }, [&](int64_t w) {
            return direct ? direct_band_meta((int)w, lg) : draw_band_meta(seed, (int)w, (int)W, drawn[w], 1u << lg, lg);
        });
    }
    return build_on_host(t, st, host_rng);
}

// The decode step behind every public variant of it: validation, launch plan, launches.
lsh_status decode_step_impl(const lsh_tables* t, const float* H_dev, const float* beam_scores_dev,
                            const int32_t* topfreq_dev, const lsh_step_params* sp,
                            void* workspace_dev, size_t workspace_bytes, int32_t* out_beam_dev,
                            int32_t* out_word_dev, float* out_score_dev, void* hip_stream,
                            lsh_profiler* prof) {
    if (!t || !H_dev || !beam_scores_dev || !sp || !workspace_dev || !out_beam_dev ||
        !out_word_dev || !out_score_dev)
        return LSH_ERR_INVALID_ARG;
    if (!step_params_ok(t, sp)) return LSH_ERR_INVALID_ARG;
    if (!sp->full_vocab && sp->T > 0 && !topfreq_dev) return LSH_ERR_INVALID_ARG;
    if (!sp->full_vocab && sp->threshold < 1) return LSH_ERR_INVALID_ARG;
    if (!sp->full_vocab && sp->threshold > 1 && t->wg_hit_rows_lds == 0) return LSH_ERR_UNSUPPORTED;
    if ((uintptr_t)workspace_dev % kAlign) return LSH_ERR_INVALID_ARG;
    const Workspace w = carve(t, sp, workspace_dev);
    if (workspace_bytes < w.bytes) return LSH_ERR_WORKSPACE_TOO_SMALL;
    const StepCtx cx{t, (hipStream_t)hip_stream, prof};
    const int32_t* cand = nullptr;
    const int32_t* count = nullptr;
    const bool fused = step_is_fused(t, sp);
    const int stage = stage_words_for(t, sp->B, fused);
    CandArgs ca{H_dev, sp->B, t->d, t->perms_dev, t->P, t->K, t->W, t->bits, t->slots_dev,
                t->bands_dev, t->words_dev, t->V, topfreq_dev, sp->T, t->cuts_dev, stage};
    set_derived(ca);
    // Bitmaps made by an earlier kernel, to be OR-ed per sentence: one per hidden row when the
    // hit threshold is above 1 (Eq. 9-10), one per part of the sentence when it has many beams.
    const uint32_t* parts = nullptr;
    int nparts = 0;
    FirstTiles first{};
    if (!sp->full_vocab && sp->threshold > 1) {
        const int blocks = sp->S * sp->B * kHitSlices;
        if (fused) first = first_tiles_plan(t, sp, H_dev, topfreq_dev, w, blocks);
        const dim3 grid(blocks + first_tiles_blocks(first)), block(kCandThreads);
#define LSH_HIT_ROWS(BESIDE, ...) launch(cx, 3, k_hit_rows<BESIDE>, grid, block, (size_t)t->wg_hit_rows_lds, ca, (int)sp->threshold, t->hit_list_cap, w.row_bitmaps, __VA_ARGS__)
        if (!first.tiles) LSH_HIT_ROWS(Alone, Alone::Args{});
        else if (t->dtype == LSH_F32) LSH_HIT_ROWS(FirstTilesBeside<float>, first);
        else LSH_HIT_ROWS(FirstTilesBeside<uint16_t>, first);
#undef LSH_HIT_ROWS
        parts = w.row_bitmaps;
        nparts = sp->B;
    } else if (const int pr = part_rows_of(t, sp, stage)) {
        nparts = (sp->B + pr - 1) / pr;
        ca.stage_words = candidates_min_stage(t->d);
        set_derived(ca);
        if (fused) first = first_tiles_plan(t, sp, H_dev, topfreq_dev, w, sp->S * nparts);
        const dim3 grid(sp->S * nparts + first_tiles_blocks(first)), block(kCandThreads);
#define LSH_PARTS(BESIDE, ...) launch(cx, 4, k_part_bitmaps<BESIDE>, grid, block, (size_t)t->wg_candidates_lds, ca, pr, nparts, w.row_bitmaps, __VA_ARGS__)
        if (!first.tiles) LSH_PARTS(Alone, Alone::Args{});
        else if (t->dtype == LSH_F32) LSH_PARTS(FirstTilesBeside<float>, first);
        else LSH_PARTS(FirstTilesBeside<uint16_t>, first);
#undef LSH_PARTS
        parts = w.row_bitmaps;
    }
    bool selected = false;   // the step's tail already ran inside the fused kernel
    bool wide = false;       // tile records of rec_groups columns
    int rec_groups = 0;      // tile records per hidden row, if not one per tile (launch_logits)
    if (fused) {
        // One launch per step: the last workgroup of each sentence also runs the selection
        // (option one_launch = 0: a selection kernel follows instead; also when no ticket block
        // is left for this workspace or the step has more sentences than a block has counters).
        TailArgs tail{nullptr, beam_scores_dev, w.lse, out_beam_dev, out_word_dev, out_score_dev,
                      std::max(0, t->option(kOptFusedTile, 0))};
        if (t->option(kOptOneLaunch, 0) && sp->S <= kTicketBlock) tail.tickets = t->tickets_for(workspace_dev);
        selected = tail.tickets != nullptr;
        const int per_sentence = std::min(kMaxFusedGrid, std::max(1, t->option(kOptFusedGrid, 256) / sp->S));
        const dim3 grid((unsigned)(per_sentence * sp->S)), block(kCandThreads);
        const bool f32 = t->dtype == LSH_F32, al = has_chunks(t);
        if (parts) {
            const size_t lds = (size_t)t->wg_union_logits_lds;
#define LSH_UNION_LOGITS(ET, AL, OL)                                                              \
    launch(cx, 1, k_union_logits<ET, AL, OL>, grid, block, lds, parts, nparts, topfreq_dev, sp->T, \
           (const ET*)t->E, t->ld, t->d, H_dev, sp->S, sp->B, t->V, w.cand, w.count, w.logits,    \
           w.cpitch, w.records(), tail, first.tiles)
#define LSH_UNION_LOGITS2(ET, AL) \
    do { if (selected) LSH_UNION_LOGITS(ET, AL, true); else LSH_UNION_LOGITS(ET, AL, false); } while (0)
            if (f32) { if (al) LSH_UNION_LOGITS2(float, true); else LSH_UNION_LOGITS2(float, false); }
            else { if (al) LSH_UNION_LOGITS2(uint16_t, true); else LSH_UNION_LOGITS2(uint16_t, false); }
#undef LSH_UNION_LOGITS2
#undef LSH_UNION_LOGITS
        } else {
            const size_t lds = fused_lds_words(t->V, t->P, t->K, stage) * sizeof(uint32_t);
#define LSH_CAND_LOGITS(...)                                                                      \
    launch(cx, 1, k_cand_logits<__VA_ARGS__>, grid, block, lds, ca, (decltype(e))t->E, t->ld, sp->S,  \
           w.cand, w.count, w.logits, w.cpitch, w.records(), tail)
#define LSH_CAND_LOGITS2(ET, AL)                                                                  \
    do {                                                                                         \
        const ET* e = nullptr;                                                                   \
        if (selected) LSH_CAND_LOGITS(ET, AL, true);                                             \
        else if (AL && takes_quads(sizeof(ET) == 2, t->d, t->ld, sp->S)) LSH_CAND_LOGITS(ET, AL, false, AL); \
        else LSH_CAND_LOGITS(ET, AL, false);                                                     \
    } while (0)
            if (f32) { if (al) LSH_CAND_LOGITS2(float, true); else LSH_CAND_LOGITS2(float, false); }
            else { if (al) LSH_CAND_LOGITS2(uint16_t, true); else LSH_CAND_LOGITS2(uint16_t, false); }
#undef LSH_CAND_LOGITS2
#undef LSH_CAND_LOGITS
        }
        cand = w.cand;
        count = w.count;
    } else {
        // a few part bitmaps ahead of k_logits_estage: that kernel ORs them itself (option
        // estage_union = 0: a union kernel of its own, as for the other drivers)
        EstageUnion un{parts, nparts, topfreq_dev, sp->T, w.cand, w.count};
        const bool fold = parts && nparts <= kEsUnionParts && takes_estage(t, sp, H_dev) && t->option(kOptEstageUnion, 1) &&
                          estage_union_words(t->V) <= (size_t)2 * kTileN * kEsPitch;
        if (fold) {
            cand = w.cand;
            count = w.count;
        } else if (parts) {
            // union of the sentence's bitmaps + top-frequent words + compaction
            launch(cx, 0, k_union_compact, dim3(sp->S), dim3(kCandThreads),
                   union_compact_lds_words(t->V) * sizeof(uint32_t), parts, nparts, t->V,
                   topfreq_dev, sp->T, w.cand, w.count);
            cand = w.cand;
            count = w.count;
        } else if (!sp->full_vocab) {
            const size_t lds = candidates_lds_words(t->V, t->P, t->K, stage) * sizeof(uint32_t);
            if (candidates_split(sp->S, t->V))
                launch(cx, 0, k_candidates<kCandParts>, dim3(sp->S * kCandParts), dim3(kCandThreads), lds, ca, sp->S, w.cand, w.count);
            else launch(cx, 0, k_candidates<1>, dim3(sp->S), dim3(kCandThreads), lds, ca, sp->S, w.cand, w.count);
            cand = w.cand;
            count = w.count;
        }
        // (on the full vocabulary all hidden rows of the call meet the same words: the contraction
        // takes them as the rows of one sentence, so that E is not read again for every sentence)
        lsh_step_params rows = *sp;
        if (sp->full_vocab) { rows.S = 1; rows.B = sp->S * sp->B; }
        wide = takes_rows(t, sp);
        if (wide && t->dtype == LSH_F32) rec_groups = launch_logits_rows<float>(cx, H_dev, rows.B, sp->B, w);
        else if (wide) rec_groups = launch_logits_rows<uint16_t>(cx, H_dev, rows.B, sp->B, w);
        else if (t->dtype == LSH_F32) rec_groups = launch_logits<float>(cx, H_dev, &rows, cand, count, w, fold ? &un : nullptr);
        else launch_logits<uint16_t>(cx, H_dev, &rows, cand, count, w);
    }
    if (!selected) {
#define LSH_SELECT(...)                                                                               \
    launch(cx, 2, k_select<__VA_ARGS__>, dim3(sp->S), dim3(kSelThreads), 0, (const float*)w.logits,  \
           w.cpitch, (const TileRecord*)w.partials, (const int32_t*)w.ids2, w.ppitch, cand, count, t->V, \
           sp->B, beam_scores_dev, w.lse, out_beam_dev, out_word_dev, out_score_dev,                   \
           fused ? std::max(0, t->option(kOptFusedTile, 0)) : 0, rec_groups)
        // (the fused kernels leave rich records, k_logits_estage one record for a group of tiles)
        if (wide && sp->B <= kSelWaves && t->V <= 1024 * rec_groups) LSH_SELECT(false, false, true, 16);   // (as many records as lists take)
        else if (wide && sp->B > kSelWaves && sp->B <= 2 * kSelWaves && t->V <= 512 * rec_groups) LSH_SELECT(false, false, true, 32);
        else if (wide && sp->B > 2 * kSelWaves && sp->B <= 4 * kSelWaves && t->V <= 512 * rec_groups) LSH_SELECT(false, false, true, 64);
        else if (wide) LSH_SELECT(false, false, true, 0);
        else if (rec_groups > 0) LSH_SELECT(false, true);
        else if (fused && sp->B <= kSelWaves) LSH_SELECT(true, false, false, 16);
        else if (fused && sp->B <= 2 * kSelWaves) LSH_SELECT(true, false, false, 32);
        else if (fused) LSH_SELECT(true, false, false, 64);   // (by option, any number)
        else if (sp->B <= kSelWaves) LSH_SELECT(false, false, false, 16);
        else if (sp->B <= 2 * kSelWaves) LSH_SELECT(false, false, false, 32);
        else if (sp->B <= 4 * kSelWaves) LSH_SELECT(false, false, false, 64);
        else LSH_SELECT(false, false, false, 0);
#undef LSH_SELECT
    }
    HIP_TRY(hipGetLastError());
    return LSH_OK;
}

}  // namespace

extern "C" {

const char* lsh_status_string(lsh_status s) {
    switch (s) {
        case LSH_OK: return "ok";
        case LSH_ERR_INVALID_ARG: return "invalid argument";
        case LSH_ERR_UNSUPPORTED: return "unsupported parameter";
        case LSH_ERR_BUILD_FAILED: return "cuckoo table build failed";
        case LSH_ERR_OOM: return "out of device memory";
        case LSH_ERR_HIP: return "HIP runtime error";
        case LSH_ERR_WORKSPACE_TOO_SMALL: return "workspace too small";
        case LSH_ERR_SCRATCH_TOO_SMALL: return "step too large for the built-in scratch buffer";
    }
    return "unknown status";
}

int32_t lsh_step_is_fused(const lsh_tables* t, const lsh_step_params* sp) {
    return (step_params_ok(t, sp) && step_is_fused(t, sp)) ? 1 : 0;
}

const char* lsh_kernel_name(int32_t which) {
    switch (which) {
        case 0: return "k_candidates";
        case 1: return "k_logits";
        case 2: return "k_select";
        case 3: return "k_hit_rows";
        case 4: return "k_part_bitmaps";
    }
    return "";
}

void lsh_free_tables(lsh_tables* t) {
    if (!t) return;
    bool idle = false;
    release_block(t->device, kHandleBlock, t->arena, idle);
    release_block(t->device, kSlotBlock, t->slot_block, idle);
    delete t;
}

void lsh_release_kept(void) {
    // (One release in eight shows in hipMemGetInfo up to 0.15 ms after hipFree has returned, and who asks for the memory may look
    // there first.  At most 2 ms: somebody else may have taken it meanwhile.)
    size_t before = 0, now = 0, total = 0;
    int dev = -1;
    const bool look = hipGetDevice(&dev) == hipSuccess && hipMemGetInfo(&before, &total) == hipSuccess;
    const size_t bytes = give_back_kept(look ? dev : -1);
    const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(2);
    while (bytes && hipMemGetInfo(&now, &total) == hipSuccess && now < before + bytes && std::chrono::steady_clock::now() < until)
        std::this_thread::sleep_for(std::chrono::microseconds(20));
}

lsh_status lsh_build_tables(const void* E_dev, const int32_t* perms_dev, const lsh_build_params* p,
                            void* hip_stream, lsh_tables** out) {
    if (!E_dev || !perms_dev || !p || !out) return LSH_ERR_INVALID_ARG;
    *out = nullptr;
    if (p->V < 1 || p->V > kMaxV || p->d < 1 || p->ld_e < p->d) return LSH_ERR_INVALID_ARG;
    if (p->e_dtype != LSH_F32 && p->e_dtype != LSH_BF16) return LSH_ERR_INVALID_ARG;
    if (p->K < 2 || p->K > p->d || p->K > 32768) return LSH_ERR_INVALID_ARG;
    if (p->P < 1 || p->bands < 1 || p->P % p->bands != 0) return LSH_ERR_INVALID_ARG;
    const int bits = code_bits(p->K), u = p->P / p->bands;
    if ((int64_t)u * bits > 30) return LSH_ERR_INVALID_ARG;
    if (candidates_lds_words(p->V, p->P, p->K, candidates_min_stage(p->d)) * 4 > kMaxDynLds ||
        p->bands > kCandThreads)
        return LSH_ERR_UNSUPPORTED;
    hipStream_t st = (hipStream_t)hip_stream;

    lsh_tables* t = new (std::nothrow) lsh_tables();
    if (!t) return LSH_ERR_OOM;
    struct Guard { lsh_tables* t; ~Guard() { if (t) lsh_free_tables(t); } } guard{t};
    HIP_TRY(hipGetDevice(&t->device));
    HIP_TRY(scratch_of_device(t->device, &t->scratch_dev));
    // launch-plan options: the library's own rules unless LSHBEAM_<NAME> is set in the environment
    // at this point (read once, here) or lsh_set_option changes them later
    for (int i = 0; i < kNumOpts; ++i) {
        std::string name = "LSHBEAM_";
        for (const char* c = kOptNames[i]; *c; ++c) name += (char)std::toupper((unsigned char)*c);
        t->opt[i] = env_int(name.c_str(), kAuto);
    }
    t->E = E_dev; t->V = p->V; t->d = p->d; t->ld = p->ld_e; t->dtype = p->e_dtype;
    t->K = p->K; t->P = p->P; t->W = p->bands; t->u = u; t->bits = bits;
    const lsh_status brc = build_all(t, st, perms_dev, p->seed ^ 0xC0FFEE1234ABCDEFull, env_int("LSHBEAM_HOST_BUILD", 0) != 0);
    if (brc != LSH_OK) return brc;

    // (with the minimum stage; a step may ask for more)
    t->wg_candidates_lds = (int)(candidates_lds_words(t->V, t->P, t->K, candidates_min_stage(t->d)) * sizeof(uint32_t));
    {   // LDS plan of k_hit_rows: whatever the counters leave goes to the load list
        const size_t fixed = hit_rows_fixed_lds_words(t->V, t->d, t->P);
        const size_t room = kMaxDynLds / sizeof(uint32_t);
        size_t cap = room > fixed ? (room - fixed) / 1024 * 1024 : 0;
        if (cap > (size_t)kHitListMax) cap = kHitListMax;
        if (cap >= (size_t)kHitListMin && (uint64_t)t->W * (uint64_t)t->V < (1ull << 30)) {
            t->hit_list_cap = (int)cap;
            t->wg_hit_rows_lds = (int)((fixed + cap) * sizeof(uint32_t));
        }
    }
    t->wg_union_logits_lds = (int)(union_logits_lds_words(t->V) * sizeof(uint32_t));
    t->wg_fused_lds = (int)(fused_lds_words(t->V, t->P, t->K, candidates_min_stage(t->d)) * sizeof(uint32_t));
    HIP_TRY(allow_step_lds(t->device));
    guard.t = nullptr;
    *out = t;
    return LSH_OK;
}

size_t lsh_step_workspace_bytes(const lsh_tables* t, const lsh_step_params* sp) {
    if (!step_params_ok(t, sp)) return 0;
    return carve(t, sp, nullptr).bytes;
}

lsh_status lsh_decode_step(const lsh_tables* t, const float* H_dev, const float* beam_scores_dev,
                           const int32_t* topfreq_dev, const lsh_step_params* sp,
                           void* workspace_dev, size_t workspace_bytes, int32_t* out_beam_dev,
                           int32_t* out_word_dev, float* out_score_dev, void* hip_stream) {
    return decode_step_impl(t, H_dev, beam_scores_dev, topfreq_dev, sp, workspace_dev, workspace_bytes,
                            out_beam_dev, out_word_dev, out_score_dev, hip_stream, nullptr);
}

lsh_status lsh_decode_step_timed(const lsh_tables* t, const float* H_dev, const float* beam_scores_dev,
                                 const int32_t* topfreq_dev, const lsh_step_params* sp,
                                 void* workspace_dev, size_t workspace_bytes, int32_t* out_beam_dev,
                                 int32_t* out_word_dev, float* out_score_dev, void* hip_stream,
                                 lsh_profiler* prof) {
    return decode_step_impl(t, H_dev, beam_scores_dev, topfreq_dev, sp, workspace_dev, workspace_bytes,
                            out_beam_dev, out_word_dev, out_score_dev, hip_stream, prof);
}

size_t lsh_static_scratch_bytes(void) { return kScratchBytes; }

lsh_status lsh_decode_step_static(const lsh_tables* t, const float* H_dev, const float* beam_scores_dev,
                                  const int32_t* topfreq_dev, const lsh_step_params* sp,
                                  int32_t* out_beam_dev, int32_t* out_word_dev, float* out_score_dev,
                                  void* hip_stream) {
    if (!step_params_ok(t, sp)) return LSH_ERR_INVALID_ARG;
    if (!t->scratch_dev) return LSH_ERR_HIP;
    if (carve(t, sp, nullptr).bytes > kScratchBytes) return LSH_ERR_SCRATCH_TOO_SMALL;
    // (nothing in the workspace has to start from zero: every kernel writes what a later one reads)
    return decode_step_impl(t, H_dev, beam_scores_dev, topfreq_dev, sp, t->scratch_dev, kScratchBytes,
                            out_beam_dev, out_word_dev, out_score_dev, hip_stream, nullptr);
}

lsh_status lsh_set_option(lsh_tables* t, const char* name, int32_t value) {
    if (!t || !name || value < kAuto) return LSH_ERR_INVALID_ARG;
    for (int i = 0; i < kNumOpts; ++i)
        if (std::strcmp(name, kOptNames[i]) == 0) { t->opt[i] = value; return LSH_OK; }
    return LSH_ERR_INVALID_ARG;
}

lsh_status lsh_get_option(const lsh_tables* t, const char* name, int32_t* value_out) {
    if (!t || !name || !value_out) return LSH_ERR_INVALID_ARG;
    for (int i = 0; i < kNumOpts; ++i)
        if (std::strcmp(name, kOptNames[i]) == 0) { *value_out = t->opt[i]; return LSH_OK; }
    return LSH_ERR_INVALID_ARG;
}

/* ---- inspection ----------------------------------------------------------------------------- */

lsh_status lsh_debug_codes(const lsh_tables* t, const float* H_dev, int32_t R, int32_t* codes_host) {
    if (!t || !H_dev || !codes_host || R < 1) return LSH_ERR_INVALID_ARG;
    int32_t* tmp = nullptr;
    const int64_t n = (int64_t)R * t->W;
    HIP_TRY(hipMalloc((void**)&tmp, n * sizeof(int32_t)));
    hipError_t e = launch_row_codes<float>(nullptr, H_dev, t->d, R, t->d, t->perms_dev, t->P, t->K, t->W, t->bits, tmp, t->W, 1);
    if (e == hipSuccess) e = hipMemcpy(codes_host, tmp, n * sizeof(int32_t), hipMemcpyDeviceToHost);
    (void)hipFree(tmp);
    HIP_TRY(e);
    return LSH_OK;
}

lsh_status lsh_debug_embedding_codes(const lsh_tables* t, int32_t row0, int32_t n, int32_t* codes_host) {
    if (!t || !codes_host || row0 < 0 || n < 0 || (int64_t)row0 + n > t->V) return LSH_ERR_INVALID_ARG;
    // (band by band, turned into rows on the host)
    std::vector<int32_t> band(n);
    for (int w = 0; w < t->W && n > 0; ++w) {
        HIP_TRY(hipMemcpy(band.data(), t->codes_dev + (size_t)w * t->V + row0, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost));
        for (int i = 0; i < n; ++i) codes_host[(size_t)i * t->W + w] = band[i];
    }
    return LSH_OK;
}

lsh_status lsh_debug_bucket(const lsh_tables* t, int32_t band, int32_t code, int32_t* words_host,
                            int32_t cap, int32_t* n_out) {
    if (!t || !n_out || band < 0 || band >= t->W || cap < 0 || (cap > 0 && !words_host))
        return LSH_ERR_INVALID_ARG;
    // read the two slots the device would read, from device memory
    const BandMeta& m = t->bands[band].meta;
    *n_out = -1;
    if (code < 0) return LSH_OK;
    const uint32_t h[2] = {cuckoo_hash(m.a0, m.b0, (uint32_t)code, m.shift),
                           cuckoo_hash(m.a1, m.b1, (uint32_t)code, m.shift)};
    for (int q = 0; q < 2; ++q) {
        Slot sl;
        HIP_TRY(hipMemcpy(&sl, t->slots_dev + m.slot_off + h[q], sizeof(Slot), hipMemcpyDeviceToHost));
        if (sl.key == code) {
            *n_out = (int32_t)sl.len;
            const size_t ncopy = std::min<size_t>(sl.len, (size_t)cap);
            if (ncopy)
                HIP_TRY(hipMemcpy(words_host, t->words_dev + (size_t)band * t->V + sl.start,
                                  ncopy * sizeof(int32_t), hipMemcpyDeviceToHost));
            return LSH_OK;
        }
    }
    return LSH_OK;
}

// Distinct codes of a band.
static lsh_status keys_of_band(const lsh_tables* t, int32_t band, int32_t* n) {
    *n = t->bands[band].n_keys;
    if (*n < 0) HIP_TRY(hipMemcpy(n, t->n_keys_dev + band, sizeof(int32_t), hipMemcpyDeviceToHost));
    return LSH_OK;
}

lsh_status lsh_debug_csr(const lsh_tables* t, int32_t band, int32_t* n_keys_out, int32_t* keys_host,
                         int32_t* offsets_host, int32_t cap_keys, int32_t* words_host) {
    if (!t || band < 0 || band >= t->W || !n_keys_out) return LSH_ERR_INVALID_ARG;
    const Band& b = t->bands[band];
    int32_t n_keys = 0;
    const lsh_status rc = keys_of_band(t, band, &n_keys);
    if (rc != LSH_OK) return rc;
    *n_keys_out = n_keys;
    if (keys_host && offsets_host && cap_keys >= n_keys) {
        // the used slots of the band's cuckoo table, in key order
        std::vector<Slot> slots(b.capacity);
        HIP_TRY(hipMemcpy(slots.data(), t->slots_dev + b.meta.slot_off, slots.size() * sizeof(Slot), hipMemcpyDeviceToHost));
        slots.erase(std::remove_if(slots.begin(), slots.end(), [](const Slot& x) { return x.key < 0; }), slots.end());
        std::sort(slots.begin(), slots.end(), [](const Slot& x, const Slot& y) { return x.key < y.key; });
        if ((int)slots.size() != n_keys) return LSH_ERR_BUILD_FAILED;
        for (int i = 0; i < n_keys; ++i) { keys_host[i] = slots[i].key; offsets_host[i] = (int32_t)slots[i].start; }
        offsets_host[n_keys] = n_keys ? (int32_t)(slots[n_keys - 1].start + slots[n_keys - 1].len) : 0;
    }
    if (words_host)
        HIP_TRY(hipMemcpy(words_host, t->words_dev + (size_t)band * t->V, (size_t)t->V * sizeof(int32_t),
                          hipMemcpyDeviceToHost));
    return LSH_OK;
}

lsh_status lsh_debug_build_info(const lsh_tables* t, int32_t* on_device_out, int32_t* attempts_out) {
    if (!t || !on_device_out || !attempts_out) return LSH_ERR_INVALID_ARG;
    *on_device_out = t->built_on_device;
    *attempts_out = t->build_attempts;
    return LSH_OK;
}

lsh_status lsh_debug_cuckoo_shape(const lsh_tables* t, int32_t band, int32_t* capacity_out,
                                  int32_t* n_keys_out) {
    if (!t || band < 0 || band >= t->W || !capacity_out || !n_keys_out) return LSH_ERR_INVALID_ARG;
    *capacity_out = t->bands[band].capacity;
    return keys_of_band(t, band, n_keys_out);
}

lsh_status lsh_debug_candidates(const lsh_tables* t, const void* workspace_dev,
                                const lsh_step_params* sp, int32_t s, int32_t* cand_host,
                                int32_t cap, int32_t* n_out) {
    if (!t || !workspace_dev || !n_out || !step_params_ok(t, sp) || sp->full_vocab || s < 0 ||
        s >= sp->S || cap < 0 || (cap > 0 && !cand_host))
        return LSH_ERR_INVALID_ARG;
    const Workspace w = carve(t, sp, const_cast<void*>(workspace_dev));
    HIP_TRY(hipDeviceSynchronize());
    int32_t n = 0;
    HIP_TRY(hipMemcpy(&n, w.count + s, sizeof(int32_t), hipMemcpyDeviceToHost));
    *n_out = n;
    const size_t ncopy = (size_t)std::min(n, cap);
    if (ncopy)
        HIP_TRY(hipMemcpy(cand_host, w.cand + (size_t)s * t->V, ncopy * sizeof(int32_t),
                          hipMemcpyDeviceToHost));
    return LSH_OK;
}

lsh_status lsh_debug_counts(const lsh_tables* t, const void* workspace_dev, const lsh_step_params* sp,
                            int32_t* counts_host) {
    if (!t || !workspace_dev || !counts_host || !step_params_ok(t, sp)) return LSH_ERR_INVALID_ARG;
    if (sp->full_vocab) {
        for (int s = 0; s < sp->S; ++s) counts_host[s] = t->V;
        return LSH_OK;
    }
    const Workspace w = carve(t, sp, const_cast<void*>(workspace_dev));
    HIP_TRY(hipDeviceSynchronize());
    HIP_TRY(hipMemcpy(counts_host, w.count, (size_t)sp->S * sizeof(int32_t), hipMemcpyDeviceToHost));
    return LSH_OK;
}

lsh_status lsh_debug_logprobs(const lsh_tables* t, const void* workspace_dev,
                              const lsh_step_params* sp, int32_t s, float* lp_host, int32_t cap,
                              int32_t* n_out) {
    if (!t || !workspace_dev || !n_out || !lp_host || !step_params_ok(t, sp) || s < 0 ||
        s >= sp->S || cap < 1)
        return LSH_ERR_INVALID_ARG;
    const Workspace w = carve(t, sp, const_cast<void*>(workspace_dev));
    HIP_TRY(hipDeviceSynchronize());
    int32_t C = t->V;
    if (!sp->full_vocab) HIP_TRY(hipMemcpy(&C, w.count + s, sizeof(int32_t), hipMemcpyDeviceToHost));
    *n_out = C;
    const int n = std::min(C, cap);
    if (n == 0) return LSH_OK;
    float* tmp = nullptr;
    HIP_TRY(hipMalloc((void**)&tmp, (size_t)sp->B * cap * sizeof(float)));
    hipLaunchKernelGGL(k_logprobs_dump, dim3((unsigned)((n + 255) / 256), (unsigned)sp->B), dim3(256), 0,
                       0, (const float*)w.logits, w.cpitch, (const float*)w.lse, s * sp->B, sp->B, n,
                       tmp, (int64_t)cap);
    hipError_t e = hipMemcpy(lp_host, tmp, (size_t)sp->B * cap * sizeof(float), hipMemcpyDeviceToHost);
    (void)hipFree(tmp);
    HIP_TRY(e);
    return LSH_OK;
}

/* ---- per-kernel timing ---------------------------------------------------------------------- */

void lsh_profiler_destroy(lsh_profiler* pf) {
    if (!pf) return;
    for (int k = 0; k < LSH_NUM_KERNELS; ++k)
        for (hipEvent_t e : pf->ev[k]) (void)hipEventDestroy(e);
    delete pf;
}

lsh_status lsh_profiler_create(int32_t max_launches, lsh_profiler** out) {
    if (!out || max_launches < 1 || max_launches > (1 << 16)) return LSH_ERR_INVALID_ARG;
    *out = nullptr;
    lsh_profiler* pf = new (std::nothrow) lsh_profiler();
    if (!pf) return LSH_ERR_OOM;
    pf->max_launches = max_launches;
    for (int k = 0; k < LSH_NUM_KERNELS; ++k)
        for (int i = 0; i < 2 * max_launches; ++i) {
            hipEvent_t e;
            if (hipEventCreate(&e) != hipSuccess) {
                (void)hipGetLastError();
                lsh_profiler_destroy(pf);
                return LSH_ERR_HIP;
            }
            pf->ev[k].push_back(e);
        }
    *out = pf;
    return LSH_OK;
}

lsh_status lsh_profiler_read(lsh_profiler* pf, double mean_ms_out[LSH_NUM_KERNELS],
                             int32_t launches_out[LSH_NUM_KERNELS]) {
    if (!pf || !mean_ms_out || !launches_out) return LSH_ERR_INVALID_ARG;
    HIP_TRY(hipDeviceSynchronize());
    for (int k = 0; k < LSH_NUM_KERNELS; ++k) {
        double total = 0.0;
        for (int i = 0; i < pf->used[k]; ++i) {
            float ms = 0.f;
            HIP_TRY(hipEventElapsedTime(&ms, pf->ev[k][2 * i], pf->ev[k][2 * i + 1]));
            total += ms;
        }
        launches_out[k] = pf->used[k];
        mean_ms_out[k] = pf->used[k] ? total / pf->used[k] : 0.0;
        pf->used[k] = 0;
    }
    return LSH_OK;
}

lsh_status lsh_beam_advance(const lsh_beam_params* bp, int32_t step, const int32_t* out_beam_dev,
                            const int32_t* out_word_dev, const float* out_score_dev,
                            const float* const* states_in, float* const* states_out,
                            int32_t* backptr_dev, int32_t* words_dev, float* scores_dev,
                            float* next_scores_dev, void* hip_stream) {
    if (!bp || !out_beam_dev || !out_word_dev || !out_score_dev || !backptr_dev || !words_dev ||
        !scores_dev || !next_scores_dev)
        return LSH_ERR_INVALID_ARG;
    if (bp->S < 1 || bp->B < 1 || bp->B > kMaxB || (int64_t)bp->S * bp->B > INT32_MAX / 2 ||
        bp->n_states < 0 || bp->n_states > kMaxBeamStates || bp->max_len < 1 || step < 0 ||
        step >= bp->max_len || (bp->n_states > 0 && (bp->state_dim < 1 || !states_in || !states_out)))
        return LSH_ERR_INVALID_ARG;
    BeamStatePtrs ptrs{};
    for (int k = 0; k < bp->n_states; ++k) {
        if (!states_in[k] || !states_out[k] || states_in[k] == states_out[k]) return LSH_ERR_INVALID_ARG;
        ptrs.in[k] = states_in[k];
        ptrs.out[k] = states_out[k];
    }
    const size_t R = (size_t)bp->S * bp->B, off = (size_t)step * R;
    hipLaunchKernelGGL(k_beam_advance, dim3((unsigned)R, (unsigned)std::max(bp->n_states, 1)), dim3(256), 0,
                       (hipStream_t)hip_stream, ptrs, (int)bp->n_states, (int)bp->state_dim, (int)bp->B,
                       (int)bp->eos, out_beam_dev, out_word_dev, out_score_dev, backptr_dev + off,
                       words_dev + off, scores_dev + off, next_scores_dev);
    HIP_TRY(hipGetLastError());
    return LSH_OK;
}

lsh_status lsh_beam_backtrace(const lsh_beam_params* bp, int32_t n_steps, const int32_t* backptr_dev,
                              const int32_t* words_dev, const float* scores_dev, int32_t* tokens_dev,
                              int32_t* length_dev, float* best_score_dev, void* hip_stream) {
    if (!bp || !backptr_dev || !words_dev || !scores_dev || !tokens_dev || !length_dev || !best_score_dev)
        return LSH_ERR_INVALID_ARG;
    if (bp->S < 1 || bp->B < 1 || bp->B > kMaxB || bp->max_len < 1 || n_steps < 0 ||
        n_steps > bp->max_len || (int64_t)n_steps * bp->B > INT32_MAX / 2)
        return LSH_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_beam_backtrace, dim3((unsigned)bp->S), dim3(kWave), 0, (hipStream_t)hip_stream,
                       (int)bp->S, (int)bp->B, (int)bp->eos, (int)n_steps, backptr_dev, words_dev,
                       scores_dev, (int)bp->max_len, tokens_dev, length_dev, best_score_dev);
    HIP_TRY(hipGetLastError());
    return LSH_OK;
}

}  // extern "C"
